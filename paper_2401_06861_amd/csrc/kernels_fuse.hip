// Fused k-qubit blocks: a run of gates whose qubits all lie in one tile set
// T = {0..c-1} u {hi_0..hi_{m-1}} is applied to each tile of 2^(c+m)
// amplitudes staged in LDS, so the block costs one read and one write of the
// vector instead of one per gate.  The low c bits give 2^m contiguous chunks
// of 2^c amplitudes (c >= 3: whole 128-byte lines); the high bits pick which
// chunks form a tile.  Inside LDS each gate is a pass
// over the tile with a barrier between gates.
#include <type_traits>

#include "nwq_internal.h"

namespace nwq {
namespace {

constexpr int kFuseBlock = 256;

__device__ __forceinline__ unsigned ins0(unsigned p, int q) { return ((p >> q) << (q + 1)) | (p & ((1u << q) - 1u)); }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}

// Global index of tile entry l: low c bits in place, bit c + i of l on
// qubit hi[i].
template <class Blk>
__device__ __forceinline__ unsigned long long tile_index(unsigned long long base, unsigned l, unsigned cmask, int c,
                                                         int m, const Blk& blk) {
  unsigned long long g = base | (l & cmask);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (i < m && ((l >> (c + i)) & 1u)) g |= 1ull << blk.hi[i];
  return g;
}

// Clang vector of two doubles: stays in registers where copies of HIP's
// double2 struct can go through scratch.
typedef double vd2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ vd2 ldv(const double2* p) { return *reinterpret_cast<const vd2*>(p); }
__device__ __forceinline__ void stv(double2* p, vd2 v) { *reinterpret_cast<vd2*>(p) = v; }

// Tile staging in chunks of kStage entries per thread: all loads of a chunk
// are issued before the first LDS write (and all LDS reads before the first
// global store), so each thread keeps kStage requests in flight instead of
// one.  Tiles of at least kStage * kFuseBlock entries take whole chunks.
constexpr int kStage = 8;

__global__ __launch_bounds__(kFuseBlock) void k_fused(double2* __restrict__ a, int nbits, FusedBlockDev blk,
                                                      const FusedOp* __restrict__ ops,
                                                      const double2* __restrict__ mats) {
  extern __shared__ double2 t[];
  const int c = blk.c, m = blk.m, k = c + m;
  const unsigned len = 1u << k, nt = blockDim.x;
  const unsigned long long ntiles = 1ull << (nbits - k);
  const unsigned cmask = (1u << c) - 1u;
  // the block's program into this XCD's L2: its ops are read one after the other
  for (int i = threadIdx.x; i < blk.op_count; i += nt) {
    const int x = *reinterpret_cast<const int*>(mats + ops[blk.op_begin + i].mat);
    asm volatile("" ::"v"(x));
  }
  for (unsigned long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    unsigned long long base = tile << c;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i < m) {
        const int q = blk.hi[i];
        base = ((base >> q) << (q + 1)) | (base & ((1ull << q) - 1ull));
      }
    }
    __syncthreads();
    if (len >= kStage * nt) {
      for (unsigned l0 = threadIdx.x; l0 < len; l0 += kStage * nt) {
        vd2 r[kStage];
#pragma unroll
        for (int j = 0; j < kStage; ++j) r[j] = ldv(a + tile_index(base, l0 + j * nt, cmask, c, m, blk));
#pragma unroll
        for (int j = 0; j < kStage; ++j) stv(t + l0 + j * nt, r[j]);
      }
    } else {
      for (unsigned l = threadIdx.x; l < len; l += nt) t[l] = a[tile_index(base, l, cmask, c, m, blk)];
    }
    FusedOp next = ops[blk.op_begin];
    for (int oi = 0; oi < blk.op_count; ++oi) {
      const FusedOp op = next;
      next = ops[blk.op_begin + min(oi + 1, blk.op_count - 1)];
      const double2* M = mats + op.mat;
      __syncthreads();
      switch (op.kind) {
        case 0: {   // 1q dense on local bit lo
          const double2 m0 = M[0], m1 = M[1], m2 = M[2], m3 = M[3];
          const unsigned off = 1u << op.lo;
          for (unsigned p = threadIdx.x; p < (len >> 1); p += nt) {
            const unsigned i0 = ins0(p, op.lo);
            const double2 v0 = t[i0], v1 = t[i0 + off];
            t[i0] = cfma(m0, v0, cmul(m1, v1));
            t[i0 + off] = cfma(m2, v0, cmul(m3, v1));
          }
          break;
        }
        case 1: {   // 1q diagonal
          const double2 d0 = M[0], d1 = M[1];
          for (unsigned l = threadIdx.x; l < len; l += nt) t[l] = cmul(((l >> op.lo) & 1u) ? d1 : d0, t[l]);
          break;
        }
        case 2: {   // 2q dense, operator order offsets o0, o1
          const unsigned o0 = (unsigned)op.o0, o1 = (unsigned)op.o1;
          for (unsigned p = threadIdx.x; p < (len >> 2); p += nt) {
            const unsigned b = ins0(ins0(p, op.lo), op.hi);
            const unsigned idx[4] = {b, b + o0, b + o1, b + o0 + o1};
            double2 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = t[idx[u]];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              double2 acc = cmul(M[4 * r], v[0]);
#pragma unroll
              for (int cc = 1; cc < 4; ++cc) acc = cfma(M[4 * r + cc], v[cc], acc);
              t[idx[r]] = acc;
            }
          }
          break;
        }
        case 3: {   // exchange two members of each quad (CX, SWAP)
          const unsigned oa = (unsigned)op.o0, ob = (unsigned)op.o1;
          for (unsigned p = threadIdx.x; p < (len >> 2); p += nt) {
            const unsigned b = ins0(ins0(p, op.lo), op.hi);
            const double2 x = t[b + oa], y = t[b + ob];
            t[b + oa] = y;
            t[b + ob] = x;
          }
          break;
        }
        default: {  // 2q diagonal, bits o0 (u bit 0) and o1 (u bit 1)
          const double2 d0 = M[0], d1 = M[1], d2 = M[2], d3 = M[3];
          for (unsigned l = threadIdx.x; l < len; l += nt) {
            const unsigned u = ((l >> op.o0) & 1u) | (((l >> op.o1) & 1u) << 1);
            const double2 d = (u & 2u) ? ((u & 1u) ? d3 : d2) : ((u & 1u) ? d1 : d0);
            t[l] = cmul(d, t[l]);
          }
          break;
        }
      }
    }
    __syncthreads();
    if (len >= kStage * nt) {
      for (unsigned l0 = threadIdx.x; l0 < len; l0 += kStage * nt) {
        vd2 r[kStage];
#pragma unroll
        for (int j = 0; j < kStage; ++j) r[j] = ldv(t + l0 + j * nt);
#pragma unroll
        for (int j = 0; j < kStage; ++j) stv(a + tile_index(base, l0 + j * nt, cmask, c, m, blk), r[j]);
      }
    } else {
      for (unsigned l = threadIdx.x; l < len; l += nt) a[tile_index(base, l, cmask, c, m, blk)] = t[l];
    }
  }
}

}  // namespace

void launch_fused_block(hipStream_t s, double2* a, int nbits, const FusedBlockDev& blk, const FusedOp* ops,
                        const double2* mats) {
  const int k = blk.c + blk.m;
  const unsigned long long ntiles = 1ull << (nbits - k);
  const unsigned long long cap = 1ull << 20;
  const unsigned grid = (unsigned)(ntiles < cap ? ntiles : cap);
  const size_t lds = sizeof(double2) << k;
  if (lds > 65536) (void)enable_dynamic_lds((const void*)k_fused);
  // A tile of up to 2^8 takes one wave, so no gate waits for others at its
  // barrier; with that, the program in L2 and each op read one gate ahead, 400
  // gates on a 7-qubit register go from 346 to 194 us (240 gates on 12 bits:
  // 466 -> 378 us).
  const unsigned threads = k > 8 ? (unsigned)kFuseBlock : 64u;
  hipLaunchKernelGGL(k_fused, dim3(grid), dim3(threads), lds, s, a, nbits, blk, ops, mats);
}

}  // namespace nwq

// ===========================================================================
// Register-blocked variant.  Each of the 2^(k-R) threads of a tile holds 2^R
// amplitudes that differ on R tile bits (the phase's register bits, R = 3 or
// 4); every gate of the phase acts on those bits only and runs in registers.
// Between phases the tile is exchanged through LDS, its real parts first and
// then its imaginary parts, so that a tile of 2^12 takes 32 KB.
//
// R trades registers for phases: R = 4 applies more gates per exchange but
// needs 117 to 128 VGPRs (two register sets; the density-matrix set would take
// 132, and spills nine to keep four waves on a SIMD: 14 qubits 52.4 -> 50.5 ms,
// 11 qubits 1.80 -> 1.69); R = 3 fits 70, updates in place and takes twice the
// phases.
//
// What bounds it: the vector units and the power they draw.  On the 30-qubit
// depth-40 brickwork the HBM traffic of the 32 blocks of width 12 takes 0.18 s
// and their FP64 instructions 0.13 s; the VALU is busy 82 % of the cycles at a
// clock that sinks to 1.9 GHz (density matrices 59 % at 2.15), and with three
// workgroups per CU and every tile read from cache 274 of 284 ms remained.
// Four workgroups of four waves share a CU (no tile is loaded ahead: the other
// workgroups' arithmetic hides a tile's loads, and the exchanges of one wave
// the scalar loads of another).
// Exchanges whose two phases keep the same tile bits on the wave index stay
// inside a wave and need no barrier.  Against one workgroup of 2^13 tiles with
// the next tile loaded ahead (221 VGPRs, 128 KB), three per CU (135 VGPRs, op
// switch structurised) and four: 284, 278 and 277 ms; a 24-qubit circuit of
// random pairs 1.72, 1.48 and 1.35 ms, the noisy TFIM on 14 qubits 58.3, 54.8
// and 50.5 ms.
// ===========================================================================
namespace nwq {
namespace {

__device__ __forceinline__ vd2 mkv(double a, double b) { vd2 r; r.x = a; r.y = b; return r; }
__device__ __forceinline__ vd2 vmul(vd2 a, vd2 b) { return mkv(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x)); }
__device__ __forceinline__ vd2 vfma(vd2 a, vd2 b, vd2 c) {
  return mkv(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
// Every gate helper reads the register set x and writes all of y; x and y may be
// the same array.  With 4 register bits the op loop alternates two register
// sets, so each gate's results land directly in the registers the next gate
// reads (an in-place update ends every op with a copy of all 16 amplitudes
// back into the loop-carried registers).  With 3 register bits the second set
// would push the kernel past 128 VGPRs, so it updates in place.
//
// The parts of a matrix known to be zero are skipped.  2x2: KIND 0 general (8
// FP64 instructions per amplitude), 1 a real M[0][0] (U3; 7), 2 real (RY, H;
// 4), 3 real diagonal and imaginary off-diagonal entries (RX; 4).
template <int NV, int B, int KIND>
__device__ __forceinline__ void rb_dense1(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
  const vd2 m0 = ldv(M), m1 = ldv(M + 1), m2 = ldv(M + 2), m3 = ldv(M + 3);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (j & (1 << B)) continue;
    const vd2 a = x[j], b = x[j | (1 << B)];
    if constexpr (KIND == 2) {
      y[j] = mkv(fma(m0.x, a.x, m1.x * b.x), fma(m0.x, a.y, m1.x * b.y));
      y[j | (1 << B)] = mkv(fma(m2.x, a.x, m3.x * b.x), fma(m2.x, a.y, m3.x * b.y));
      continue;
    }
    if constexpr (KIND == 3) {
      y[j] = mkv(fma(m0.x, a.x, -(m1.y * b.y)), fma(m0.x, a.y, m1.y * b.x));
      y[j | (1 << B)] = mkv(fma(m3.x, b.x, -(m2.y * a.y)), fma(m3.x, b.y, m2.y * a.x));
      continue;
    }
    if constexpr (KIND == 1) {
      const vd2 c = vmul(m1, b);
      y[j] = mkv(fma(m0.x, a.x, c.x), fma(m0.x, a.y, c.y));
    } else {
      y[j] = vfma(m0, a, vmul(m1, b));
    }
    y[j | (1 << B)] = vfma(m2, a, vmul(m3, b));
  }
}

// 4x4 with operator index u = bit B0 + 2 bit B1 (B0 < B1: the host orders the
// operator).  KIND 0 dense (16 FP64 instructions per amplitude); 1 all real
// (8); 2 entry (r, c) real where r ^ c has even parity, else imaginary (the
// superoperator of RX with its noise; 8).
template <int NV, int B0, int B1, int KIND>
__device__ __forceinline__ void rb_dense2(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (j & ((1 << B0) | (1 << B1))) continue;
    const int idx[4] = {j, j | (1 << B0), j | (1 << B1), j | (1 << B0) | (1 << B1)};
    vd2 in[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) in[u] = x[idx[u]];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (KIND == 0) {
        vd2 acc = vmul(ldv(M + 4 * r), in[0]);
#pragma unroll
        for (int c = 1; c < 4; ++c) acc = vfma(ldv(M + 4 * r + c), in[c], acc);
        y[idx[r]] = acc;
      } else {
        // the diagonal entry is real in both kinds
        const double d = M[5 * r].x;
        double re = d * in[r].x, im = d * in[r].y;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (c == r) continue;
          if (KIND == 1 || __builtin_popcount(r ^ c) % 2 == 0) {
            const double m = M[4 * r + c].x;
            re = fma(m, in[c].x, re);
            im = fma(m, in[c].y, im);
          } else {
            const double m = M[4 * r + c].y;
            re = fma(-m, in[c].y, re);
            im = fma(m, in[c].x, im);
          }
        }
        y[idx[r]] = mkv(re, im);
      }
    }
  }
}

// Dense 16x16 over all four register bits, the matrix in register order:
// y[r] = sum_c M[16 r + c] x[c] (4-register-bit kernel only).
template <int NV>
__device__ __forceinline__ void rb_dense16(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
  if constexpr (NV == 16) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      vd2 acc = vmul(ldv(M + 16 * r), x[0]);
#pragma unroll
      for (int c = 1; c < 16; ++c) acc = vfma(ldv(M + 16 * r + c), x[c], acc);
      y[r] = acc;
    }
  }
}

// A 16x16 with the pattern of a Pauli channel after a diagonal gate, in
// register order: M[u] is the diagonal entry of register u, M[16 + 4 i + j]
// the 4x4 among registers 5i and 5j (4-register-bit kernel only).
template <int NV>
__device__ __forceinline__ void rb_pauli16(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
  if constexpr (NV == 16) {
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (u % 5 != 0) y[u] = vmul(ldv(M + u), x[u]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      vd2 acc = vmul(ldv(M + 16 + 4 * i), x[0]);
#pragma unroll
      for (int j = 1; j < 4; ++j) acc = vfma(ldv(M + 16 + 4 * i + j), x[5 * j], acc);
      y[5 * i] = acc;
    }
  }
}

// Exchange of members (base | OA) and (base | OB) of each quad over bits B0, B1.
template <int NV, int B0, int B1, int OA, int OB>
__device__ __forceinline__ void rb_swap2(const vd2 (&x)[NV], vd2 (&y)[NV]) {
  constexpr int Q = (1 << B0) | (1 << B1);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (j & Q) continue;
    const vd2 a = x[j | OA], b = x[j | OB];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int m = ((u & 1) ? (1 << B0) : 0) | ((u & 2) ? (1 << B1) : 0);
      if (m != OA && m != OB) y[j | m] = x[j | m];
    }
    y[j | OA] = b;
    y[j | OB] = a;
  }
}

// Diagonal over all register bits: entry j for register j.
template <int NV>
__device__ __forceinline__ void rb_diag_all(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
#pragma unroll
  for (int j = 0; j < NV; ++j) y[j] = vmul(ldv(M + j), x[j]);
}

// 1q diagonal of a 2x2 table entry on register bit B (M[0], M[3]).
template <int NV, int B>
__device__ __forceinline__ void rb_diag1(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
  const vd2 d0 = ldv(M), d1 = ldv(M + 3);
#pragma unroll
  for (int j = 0; j < NV; ++j) y[j] = vmul(((j >> B) & 1) ? d1 : d0, x[j]);
}

// 2q diagonal on register bits B0 (u bit 0), B1 (u bit 1): entries M[u].
template <int NV, int B0, int B1>
__device__ __forceinline__ void rb_diag2(const vd2 (&x)[NV], vd2 (&y)[NV], const double2* __restrict__ M) {
  const vd2 d[4] = {ldv(M), ldv(M + 1), ldv(M + 2), ldv(M + 3)};
#pragma unroll
  for (int j = 0; j < NV; ++j) y[j] = vmul(d[((j >> B0) & 1) + 2 * ((j >> B1) & 1)], x[j]);
}

// The case bodies of rb_apply; bit positions at or above R never occur for
// that R (the guard keeps their templates from being instantiated).
template <int R, int B, int SEL>   // SEL: rb_dense1's KIND, or 4 = rb_diag1
__device__ __forceinline__ void rb_c1(const vd2 (&x)[1 << R], vd2 (&y)[1 << R], const double2* M) {
  if constexpr (B < R) {
    if constexpr (SEL == 4) rb_diag1<(1 << R), B>(x, y, M);
    else rb_dense1<(1 << R), B, SEL>(x, y, M);
  }
}
template <int R, int B0, int B1, int SEL>   // SEL: rb_dense2's KIND, 3 SWAP, 4 diagonal
__device__ __forceinline__ void rb_c2(const vd2 (&x)[1 << R], vd2 (&y)[1 << R], const double2* M) {
  constexpr int NV = 1 << R;
  if constexpr (B1 < R) {
    if constexpr (SEL == 3) rb_swap2<NV, B0, B1, (1 << B0), (1 << B1)>(x, y);
    else if constexpr (SEL == 4) rb_diag2<NV, B0, B1>(x, y, M);
    else rb_dense2<NV, B0, B1, SEL>(x, y, M);
  }
}
template <int R, int C, int T>   // CX: control C, target T
__device__ __forceinline__ void rb_cx(const vd2 (&x)[1 << R], vd2 (&y)[1 << R]) {
  if constexpr (C < R && T < R) rb_swap2<(1 << R), (C < T ? C : T), (C < T ? T : C), (1 << C), (1 << C) | (1 << T)>(x, y);
}

// One gate: a switch over the op's code; every case is specialised on its
// register bits.  The compiler turns the switch into a tree of compares and
// the cases are straight-line FP64 code, so the set of cases is kept to what
// a kind of program can hold (SET): with every kind in one kernel the two
// register sets took 99 KB of code, more than the 64 KB instruction cache two
// compute units share.
template <int R, int SET>
__device__ __forceinline__ void rb_apply(int code, const double2* __restrict__ M, const vd2 (&x)[1 << R],
                                         vd2 (&y)[1 << R]) {
  constexpr int NV = 1 << R;
#define NWQ_RB1(BASE, SEL) \
  case BASE + 0: rb_c1<R, 0, SEL>(x, y, M); return; \
  case BASE + 1: rb_c1<R, 1, SEL>(x, y, M); return; \
  case BASE + 2: rb_c1<R, 2, SEL>(x, y, M); return; \
  case BASE + 3: rb_c1<R, 3, SEL>(x, y, M); return;
#define NWQ_RB2(BASE, SEL) \
  case BASE + 0: rb_c2<R, 0, 1, SEL>(x, y, M); return; \
  case BASE + 1: rb_c2<R, 0, 2, SEL>(x, y, M); return; \
  case BASE + 2: rb_c2<R, 1, 2, SEL>(x, y, M); return; \
  case BASE + 3: rb_c2<R, 0, 3, SEL>(x, y, M); return; \
  case BASE + 4: rb_c2<R, 1, 3, SEL>(x, y, M); return; \
  case BASE + 5: rb_c2<R, 2, 3, SEL>(x, y, M); return;
#define NWQ_RBX(P, LO, HI) \
  case kRbCx + 2 * P: rb_cx<R, LO, HI>(x, y); return; \
  case kRbCx + 2 * P + 1: rb_cx<R, HI, LO>(x, y); return;
  if constexpr (SET == kRbSetDM) {
    switch (code) {
      NWQ_RB2(kRbDense2, 0)
      NWQ_RB2(kRbReal2, 1)
      NWQ_RB2(kRbPar2, 2)
      case kRbDense16: rb_dense16<NV>(x, y, M); return;
      case kRbPauli16: rb_pauli16<NV>(x, y, M); return;
      default: break;
    }
  } else {
    switch (code) {
      NWQ_RB1(kRbGen1, 0)
      NWQ_RB1(kRbReal1, 2)
      NWQ_RB1(kRbXt1, 3)
      NWQ_RBX(0, 0, 1)
      NWQ_RBX(1, 0, 2)
      NWQ_RBX(2, 1, 2)
      NWQ_RBX(3, 0, 3)
      NWQ_RBX(4, 1, 3)
      NWQ_RBX(5, 2, 3)
      NWQ_RB2(kRbSwap, 3)
      default: break;
    }
    if constexpr (SET == kRbSetSV) {
      switch (code) {
        NWQ_RB1(kRbR001, 1)
        NWQ_RB2(kRbDense2, 0)
        case kRbDiagAll: rb_diag_all<NV>(x, y, M); return;
        default: break;
      }
    } else {
      switch (code) {
        NWQ_RB1(kRbDiag1, 4)
        NWQ_RB2(kRbDiag2, 4)
        default: break;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NV; ++j) y[j] = x[j];   // kRbCopy
#undef NWQ_RB1
#undef NWQ_RB2
#undef NWQ_RBX
}

// Global loads and stores of tile entries; NT: non-temporal (each entry is
// read and written once per block, so nothing is worth keeping in cache).
template <bool NT>
__device__ __forceinline__ vd2 gld(const double2* p) {
  if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const vd2*>(p));
  else return ldv(p);
}
template <bool NT>
__device__ __forceinline__ void gst(double2* p, vd2 v) {
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<vd2*>(p));
  else stv(p, v);
}

// XOR of the images of the set bits of v; images of register j: a constant
// combination of the register bits' images.
__device__ __forceinline__ unsigned thread_image(unsigned v, const unsigned short (&img)[kRbThreadBits]) {
  unsigned x = 0;
#pragma unroll
  for (int i = 0; i < kRbThreadBits; ++i) x ^= (unsigned)((int)(v << (31 - i)) >> 31) & img[i];
  return x;
}
__device__ __forceinline__ unsigned long long thread_image(unsigned v, const unsigned long long (&img)[kRbThreadBits]) {
  unsigned long long x = 0;
#pragma unroll
  for (int i = 0; i < kRbThreadBits; ++i) x ^= (unsigned long long)(long long)((int)(v << (31 - i)) >> 31) & img[i];
  return x;
}
template <class T>
__device__ __forceinline__ T register_image(int j, const T (&img)[4]) {
  T x = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if ((j >> i) & 1) x ^= img[i];
  return x;
}

// One component of the tile in LDS, from LDS address 0 (the kernel has no
// other LDS; going through the dynamic array's symbol would add its base to
// every address).
typedef __attribute__((address_space(3))) double* lds_double;
__device__ __forceinline__ lds_double lds_at(unsigned byte) { return (lds_double)byte; }

template <int R, int SET, bool NT>
__global__ __launch_bounds__(R == 4 ? 512 : 1024) __attribute__((amdgpu_waves_per_eu(4))) void k_fused_rb(double2* __restrict__ a0, RbBlock blk,
                                                                  const RbPhase* __restrict__ phases,
                                                                  const RbOp* __restrict__ ops,
                                                                  const double2* __restrict__ mats0,
                                                                  unsigned long long state_stride, int mat_stride,
                                                                  unsigned long long ntiles, unsigned long long mask,
                                                                  unsigned long long step) {
  constexpr int NV = 1 << R;
  // batch element blockIdx.y: its own state and its own matrix table
  double2* __restrict__ a = a0 + (size_t)blockIdx.y * state_stride;
  const double2* __restrict__ mats = mats0 + (size_t)blockIdx.y * mat_stride;
  const unsigned tid = threadIdx.x, nt = blockDim.x;
  const int P = blk.ph_count;
  if (blockIdx.x >= ntiles) return;
  const RbPhase* __restrict__ pp = phases + blk.ph_begin;
  const unsigned long long gl_ld = thread_image(tid, blk.ld_t), gl_st = thread_image(tid, blk.st_t);
  vd2 v[NV];
  // the tile's index bits plus gridDim.x, carried over the mask's gaps
  auto advance = [&](unsigned long long base) { return ((base | ~mask) + step) & mask; };
  unsigned long long tile = blockIdx.x, base = deposit_bits(tile, mask);
  // One load per 64-byte line brings the block's program into this XCD's L2,
  // ahead of the first tile's loads: each phase and op is read through the
  // scalar cache when its turn comes, one after the other, and a workgroup
  // with few tiles would wait out a miss to memory for every one of them
  // (380 gates of a 10-qubit circuit in one block: 250 -> 150 us).
  auto warm = [&](const char* p, unsigned bytes) {
    for (unsigned i = tid * 64u; i < bytes; i += nt * 64u) {
      const int x = *reinterpret_cast<const int*>(p + i);
      asm volatile("" ::"v"(x));
    }
  };
  warm(reinterpret_cast<const char*>(pp), P * sizeof(RbPhase));
  {
    const RbOp* po = ops + pp[0].op_begin;
    warm(reinterpret_cast<const char*>(po), blk.prog_ops * sizeof(RbOp));
    if (blk.prog_mats > 0) {
      warm(reinterpret_cast<const char*>(mats + po[0].mat), blk.prog_mats * sizeof(double2));
    } else {   // 2x2 entries spread over a larger table
      for (unsigned i = tid; i < (unsigned)blk.prog_ops; i += nt) {
        const int x = *reinterpret_cast<const int*>(mats + po[i].mat);
        asm volatile("" ::"v"(x));
      }
    }
  }
  for (;;) {
    {
      const double2* __restrict__ p = a + (base | gl_ld);
#pragma unroll
      for (int j = 0; j < NV; ++j) v[j] = gld<NT>(p + register_image(j, blk.ld_r));
    }
    for (int pi = 0; pi < P; ++pi) {
      const RbPhase ph = pp[pi];
      if (pi > 0) {
        const unsigned wa = thread_image(tid, ph.wr_t) << 3, ra = thread_image(tid, ph.rd_t) << 3;
        const bool across = (ph.count_flags & kRbBarrierInside) != 0;
        exchange_barrier((ph.count_flags & kRbBarrierBefore) != 0);
#pragma unroll
        for (int j = 0; j < NV; ++j) *lds_at(wa ^ (register_image(j, ph.wr_r) << 3)) = v[j].x;
        exchange_barrier(across);
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j].x = *lds_at(ra ^ (register_image(j, ph.rd_r) << 3));
        exchange_barrier(across);
#pragma unroll
        for (int j = 0; j < NV; ++j) *lds_at(wa ^ (register_image(j, ph.wr_r) << 3)) = v[j].y;
        exchange_barrier(across);
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j].y = *lds_at(ra ^ (register_image(j, ph.rd_r) << 3));
      }
      const RbOp* __restrict__ po = ops + ph.op_begin;
      const int nops = ph.count_flags >> kRbFlagBits;
      // the next ops' codes are loaded while this one runs (the table ends
      // with two spare entries)
      if constexpr (R == 4) {
        // two gates per trip, v -> w -> v (the host pads an odd count with a copy)
        vd2 w[NV];
        RbOp o0 = po[0], o1 = po[1];
        for (int oi = 0; oi < nops; oi += 2) {
          const RbOp n0 = po[oi + 2], n1 = po[oi + 3];
          rb_apply<R, SET>(o0.code, mats + o0.mat, v, w);
          rb_apply<R, SET>(o1.code, mats + o1.mat, w, v);
          o0 = n0;
          o1 = n1;
        }
      } else {
        RbOp o = po[0];
        for (int oi = 0; oi < nops; ++oi) {
          const RbOp nx = po[oi + 1];
          rb_apply<R, SET>(o.code, mats + o.mat, v, v);
          o = nx;
        }
      }
    }
    double2* __restrict__ out = a + (base | gl_st);
#pragma unroll
    for (int j = 0; j < NV; ++j) gst<NT>(out + register_image(j, blk.st_r), v[j]);
    tile += gridDim.x;
    if (tile >= ntiles) break;
    base = advance(base);
  }
}

}  // namespace

void launch_fused_rb(hipStream_t s, double2* a, int nbits, const RbBlock& blk, const RbPhase* phases, const RbOp* ops,
                     const double2* mats, int rbits, int set, bool non_temporal, unsigned long long mask, int batch,
                     int mat_stride, int max_grid) {
  const unsigned long long ntiles = 1ull << __builtin_popcountll(mask);
  // 1024 workgroups of width 12 run at a time; many more of them than that keep
  // the last round short (n=30: 286 ms with 4096, 278 with 16384)
  const unsigned long long cap = max_grid > 0 ? (unsigned long long)max_grid : 16384;
  const unsigned grid = (unsigned)(ntiles < cap ? ntiles : cap);
  const size_t lds = sizeof(double) << blk.k;   // at most 64 KiB
  const unsigned long long stride = batch > 1 ? (1ull << nbits) : 0ull;
  const unsigned long long step = deposit_bits(grid, mask);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid, batch), dim3(1u << (blk.k - rbits)), lds, s, a, blk, phases, ops, mats, stride,
                       mat_stride, ntiles, mask, step);
  };
  auto pick = [&](auto R, auto SET) {
    if (non_temporal) go(k_fused_rb<decltype(R)::value, decltype(SET)::value, true>);
    else go(k_fused_rb<decltype(R)::value, decltype(SET)::value, false>);
  };
  using R3 = std::integral_constant<int, 3>;
  using R4 = std::integral_constant<int, 4>;
  if (set == kRbSetVQE) {   // 4 register bits only
    pick(R4{}, std::integral_constant<int, kRbSetVQE>{});
  } else if (set == kRbSetDM) {
    if (rbits == 3) pick(R3{}, std::integral_constant<int, kRbSetDM>{});
    else pick(R4{}, std::integral_constant<int, kRbSetDM>{});
  } else {
    if (rbits == 3) pick(R3{}, std::integral_constant<int, kRbSetSV>{});
    else pick(R4{}, std::integral_constant<int, kRbSetSV>{});
  }
}

}  // namespace nwq
