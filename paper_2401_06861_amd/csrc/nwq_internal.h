// Internal declarations shared by the engine's HIP translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <complex>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/nwq.h"

namespace nwq {

using cd = std::complex<double>;

constexpr int kBlock = 256;          // threads per workgroup for streaming kernels
constexpr int kWave = 64;            // CDNA wavefront width

// Gate / superoperator matrices passed by value as kernel arguments.
struct Mat2 { double2 m[4]; };       // 2x2, row-major
struct Mat4 { double2 m[16]; };      // 4x4, row-major
struct Diag4 { double2 d[4]; };      // diagonal entries indexed by u = b0 + 2 b1

// Qubit set of a k-qubit dense kernel (k <= 4).
struct QSet {
  int sorted[4];                     // ascending positions (zero-insertion order)
  unsigned long long off[4];         // 2^{q_j} in the operator's own order
};

// Streaming launch shape chosen by the autotuner (per kernel class and
// target bucket).
struct LaunchCfg {
  int ppt = 4;                       // pairs / groups / elements per thread (1, 2, 4, 8; 16 where allowed;
                                     // 32, 64, 128: split-workgroup kernels of 256, 512, 1024 threads)
  int nt = 0;                        // flags: bit 0 non-temporal loads and stores; bit 1 (shapes 32, 64,
                                     // 128 only) XCD-contiguous workgroup order
};

// Launch shapes are kept in three buckets per class, by the lowest target
// bit of the launch: below 3 the partner amplitudes of a group share one
// 128-byte line (a non-temporal hint then costs a second fetch of the line);
// from 3 to 10 the streams of a group are within 16 KiB of each other; from
// 11 up they are 32 KiB or more apart.  The best shape differs between them
// (on MI355X at 30 qubits: 1 group per thread, 16 with the hint, 4 with the
// hint for the 2x2 kernel).
constexpr int kBuckets = 3;
constexpr int kMaxTargetBits = 64;   // lowest target bits with their own tuned launch shape
inline int bucket_of(int lowest_bit) { return lowest_bit < 3 ? 0 : (lowest_bit < 11 ? 1 : 2); }

// Kernel classes (also the timing classes of nwq_timing_read).
enum KClass {
  KC_RESET = 0, KC_SV1Q = 1, KC_DIAG = 2, KC_PERM = 3, KC_SV2Q = 4,
  KC_FUSED = 5, KC_DM1 = 6, KC_DM2 = 7, KC_REDUCE = 8, KC_COUNT = 9
};

// ---- launchers (kernels_sv.hip) -------------------------------------------
void launch_fill_basis0(hipStream_t s, double2* a, unsigned long long len);
void launch_sv_1q(hipStream_t s, double2* a, int nbits, int q, const Mat2& m, const LaunchCfg& cfg);
void launch_sv_diag(hipStream_t s, double2* a, int nbits, int q0, int q1, const Diag4& d, const LaunchCfg& cfg);
void launch_sv_swap1(hipStream_t s, double2* a, int nbits, int q, const LaunchCfg& cfg);
void launch_sv_swap2(hipStream_t s, double2* a, int nbits, int qa, int qb,
                     unsigned long long offA, unsigned long long offB, const LaunchCfg& cfg);
void launch_sv_2q(hipStream_t s, double2* a, int nbits, int q0, int q1, const Mat4& m, const LaunchCfg& cfg);
// k-qubit operator on the given qubits (operator index bit j = qubits[j]);
// dev_matrix is the dense 2^k x 2^k, or with pauli (k = 4 only) the 32-entry
// compact form of a Pauli-pattern 16 x 16: the 16 diagonal entries, then the
// 4 x 4 among operator indices 0, 5, 10, 15.
void launch_sv_kq(hipStream_t s, double2* a, int nbits, int k, const int* qubits, const double2* dev_matrix,
                  const LaunchCfg& cfg, bool pauli = false);

// ---- reductions (kernels_reduce.hip) --------------------------------------
struct TileShape {
  int c;                    // low contiguous bits in the tile
  int m;                    // number of high bits
  int hi[8];                // the high bit positions, ascending
};
// Blocks of a reduction over 2^nbits entries: one row of partials has as many.
int pauli_grid(int nbits);
// One pass of the tiled Pauli-term kernel: a device table of `count` terms;
// partial sums go to partials[row * grid + block].
constexpr int kTileTerms = 16;
struct TermDev {
  unsigned long long xl;    // x mask in tile-local bit positions
  unsigned long long zl;    // z bits inside the tile, tile-local positions
  unsigned long long zo;    // z bits outside the tile, global positions
  int y;                    // popcount(x & z) mod 4
  int row;
  // one amplitude of each pair: half > 0, those with register bit half - 1
  // clear; waves != 0, those on waves with even parity under it; else all
  int half;
  unsigned waves;
  double scale;             // sign of Re(i^y w), 2 where each pair counts once
};
TermDev pauli_term(const TileShape& t, unsigned long long x, unsigned long long z, int row);
void launch_pauli_tile(hipStream_t s, const double2* a, int nbits, const TileShape& t,
                       const TermDev* terms, int count, double* partials, int grid);
// Terms with no flipped bits (x = 0): z masks (global bit positions) and
// rows by value; partials as above, with the same grid.
constexpr int kDiagTerms = 32;
struct ZMasks {
  unsigned long long z[kDiagTerms];
  int row[kDiagTerms];
};
void launch_pauli_diag(hipStream_t s, const double2* a, int nbits, const ZMasks& zs, int count, double* partials,
                       int grid);
// One term with wide x support, pairs read from global memory; partials[block].
void launch_pauli_pairs(hipStream_t s, const double2* a, int nbits, unsigned long long x, unsigned long long z,
                        int y, double* partials, int grid);
// DM: Tr(rho P_t) for each term, complex partials partials[(2*row + {0,1}) * grid + block].
int dm_pauli_grid(int n);
void launch_dm_pauli(hipStream_t s, const double2* rho, int n, const TermDev* terms, int count,
                     double* partials, int grid);
// sum |a_j|^2 over len entries into partials[block]
int sumsq_grid(unsigned long long len);
void launch_sumsq(hipStream_t s, const double2* a, unsigned long long len, double* partials, int grid);
// out[r] = sum_b partials[r * grid + b] (fixed order); if coeffs: out[rows] = sum_r coeffs[r] out[r]
void launch_reduce_rows(hipStream_t s, const double* partials, int rows, int grid,
                        const double* coeffs, double* out);

// ---- fused LDS blocks (kernels_fuse.hip) ----------------------------------
struct FusedOp {            // one gate inside a fused block of the per-gate LDS kernel, tile-local bits
  int kind;                 // 0: 1q dense, 1: 1q diag, 2: 2q dense, 3: 2q member swap, 4: 2q diag
  int lo, hi;               // sorted tile-local bit positions (hi unused for 1q)
  int o0, o1;               // kind 2: local offsets of q0, q1; kind 3: offsets swapped; kind 4: local bits of q0, q1
  int mat;                  // start of its matrix in the block program's matrix table (double2 units)
};
// One op of the register-blocked kernels: a code (kind and register bits) and
// the start of its entries in the matrix table (double2 units).
struct RbOp {
  int code, mat;
};
// Pairs of register bits B0 < B1 are numbered B1 (B1 - 1) / 2 + B0.
inline int rb_pair(int b0, int b1) { return b1 * (b1 - 1) / 2 + b0; }
enum RbCode {
  kRbGen1 = 0,              // + B: dense 2x2
  kRbR001 = 4,              // + B: 2x2 with a real M[0][0]
  kRbReal1 = 8,             // + B: real 2x2
  kRbXt1 = 12,              // + B: real diagonal, imaginary off-diagonal entries
  kRbDense2 = 16,           // + pair: dense 4x4, index u = bit B0 + 2 bit B1
  kRbReal2 = 22,            // + pair: real 4x4
  kRbPar2 = 28,             // + pair: entry (r, c) real where r ^ c has even parity, else imaginary
  kRbCx = 34,               // + 2 pair (+ 1 when the control is B1): CX
  kRbSwap = 46,             // + pair
  kRbDiagAll = 52,          // diagonal over all register bits (one entry per register)
  kRbDiag1 = 53,            // + B: 1q diagonal, entries M[0] and M[3]
  kRbDiag2 = 57,            // + pair: 2q diagonal, entries M[u]
  kRbDense16 = 63,          // 16x16 in register order (4 register bits)
  kRbPauli16 = 64,          // its Pauli-channel pattern: the 16 diagonal entries, then the 4x4 among
                            // registers 0, 5, 10, 15 (4 register bits)
  kRbCopy = 65              // pads an odd op count (4 register bits)
};
inline int rb_cx_code(int control, int target) {
  return control < target ? kRbCx + 2 * rb_pair(control, target) : kRbCx + 2 * rb_pair(target, control) + 1;
}
// Op sets, each with kernels of its own: state-vector circuits (1q, 4x4, one
// diagonal form, permutations), density-matrix superoperators (4x4 and 16x16
// kinds), VQE programs (1q kinds, 1q and 2q diagonals, permutations; matrices
// read from per-vector tables).
constexpr int kRbSetSV = 0, kRbSetDM = 1, kRbSetVQE = 2;
struct FusedBlockDev {
  int c, m;                 // tile = low c bits + m high bits
  int hi[8];
  int op_begin, op_count;   // range in the op table
};
void launch_fused_block(hipStream_t s, double2* a, int nbits, const FusedBlockDev& blk,
                        const FusedOp* ops, const double2* mats);
// Register-blocked blocks (kernels_fuse.hip).  A tile of 2^k entries belongs
// to 2^(k - R) threads of 2^R registers each (R = 3 or 4, 8 <= k <= 13).  In
// each phase R tile bits are register bits and the others thread bits; every
// index map (global address, LDS address) is linear over GF(2) in the thread
// and register bits, so a map is given by the images of the single bits, which
// are XORed together.
constexpr int kRbThreadBits = 10;   // most thread bits (k = 13, R = 3)
constexpr int kRbBarrierBefore = 1, kRbBarrierInside = 2, kRbFlagBits = 2;
struct RbPhase {
  int op_begin;             // RbOps (an even number at 4 register bits; the op table ends with two spare entries)
  int count_flags;          // op count << kRbFlagBits | flags
  // The LDS exchange that leads into this phase (not for the first): entries
  // where the previous phase's registers are written and where this phase's
  // are read.  kRbBarrierBefore: other waves may still read the entries that
  // are written; kRbBarrierInside: a wave reads entries of others (else all it
  // reads are its own, and LDS serves a wave in order).
  unsigned short wr_t[kRbThreadBits], wr_r[4], rd_t[kRbThreadBits], rd_r[4];
};
// The bits of v deposited, lowest first, at the set bits of mask.
__host__ __device__ inline unsigned long long deposit_bits(unsigned long long v, unsigned long long mask) {
  unsigned long long r = 0;
  for (; mask; mask &= mask - 1, v >>= 1)
    if (v & 1ull) r |= mask & (~mask + 1ull);
  return r;
}
// Between the LDS writes and reads of an exchange (and back): a barrier where
// waves exchange entries.  Inside a wave LDS serves accesses in order, and the
// fence, which takes no instruction, keeps the compiler to that order.
__device__ __forceinline__ void exchange_barrier(bool across_waves) {
  if (across_waves) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  }
}
struct RbBlock {
  int k;
  int ph_begin, ph_count;   // range in the phase table
  // ops and matrix entries of the block's program, contiguous from its first
  // op's (0 entries: the matrices lie elsewhere)
  int prog_ops, prog_mats;
  unsigned long long tile;  // the tile's bits of the global index
  // global index of the first phase's entries (loaded) and the last's (stored)
  unsigned long long ld_t[kRbThreadBits], ld_r[4], st_t[kRbThreadBits], st_r[4];
};
// batch > 1: blockIdx.y = batch element b works on a + b * 2^nbits with the
// matrix table mats + b * mat_stride; max_grid caps the tiles' grid (0: 16384).
// non_temporal: global loads and stores of the tiles.  mask: bits of the global
// index outside the tile that the block's tiles run over (the block leaves
// tiles with other bits set alone: used when they are known to hold zeros,
// which a block maps to zeros).
void launch_fused_rb(hipStream_t s, double2* a, int nbits, const RbBlock& blk, const RbPhase* phases, const RbOp* ops,
                     const double2* mats, int rbits, int set, bool non_temporal, unsigned long long mask,
                     int batch = 1, int mat_stride = 0, int max_grid = 0);
// nwq_set_fusion_flags / nwq_vqe_set_flags bits
constexpr int kFusedNonTemporal = 1;
constexpr int kFusedDirect = 2;      // first / last phase straight between HBM and registers where its lanes
                                     // cover contiguous runs
constexpr int kFusedGateFusion = 4;  // SV circuits (host side): gate products before the blocks are planned,
                                     // where they save FP64 work, and merged diagonals (circuit.hip)

// ---- error handling (engine.hip) ------------------------------------------
int set_error(int code, const std::string& msg);
int check_hip(hipError_t e, const char* what);

// Dynamic LDS above 64 KiB: up to the CU's whole 160 KiB less the kernel's
// static LDS (the resident VQE kernels take up to that).  enable_dynamic_lds
// raises a kernel's limit to it once per kernel and device, under a lock: the
// limit is process-wide state of the kernel, so setting it per launch from
// several host threads raced with launches of the same kernel elsewhere, and a
// smaller value set for one launch could undercut another's.
constexpr int kMaxDynamicLds = 160 * 1024;
int enable_dynamic_lds(const void* kernel);

}  // namespace nwq
