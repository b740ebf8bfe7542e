// Deterministic reductions: Pauli-term expectation values of a state vector,
// Tr(rho P) of a density matrix, and sums of squared moduli.
//
// Every reduction has a fixed order: per-lane partials, a wave64 xor-shuffle
// tree, per-wave slots in LDS combined in wave order, per-block partials in
// global memory, and a second stage that sums each row of block partials in
// a fixed order.  No atomics, so results are bitwise reproducible for a given
// input size and launch shape, whatever else runs on the device.
//
// Pauli term P = i^{|x&z|} X^x Z^z acts as P|j> = i^y (-1)^{|j&z|} |j^x>, so
//   <P> = sum_j i^y (-1)^{|j&z|} conj(a_{j^x}) a_j .
// For x != 0 the contributions of j and j^x are complex conjugates, so the
// sum over j with bit h(x) clear of 2 Re(...) gives <P> with no imaginary
// residue; for x = 0 the summand (-1)^{|j&z|} |a_j|^2 is real.
//
// Tiling: a workgroup stages a tile of 2^(c+m) amplitudes in LDS -- 2^m
// contiguous chunks of 2^c amplitudes (c >= 4: 256-byte runs) whose high bits sit at m chosen positions -- so every term whose
// flipped bits x lie inside the tile finds its partner in LDS.  The host
// groups terms into passes of tiles that cover their x bits.
#include <algorithm>

#include "nwq_internal.h"

namespace nwq {
namespace {

constexpr int kRedBlock = 256;
constexpr int kRedWaves = kRedBlock / kWave;
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Tile-local index l -> global index (without the tile base): low c bits
// pass through; bit c+i of l goes to position hi[i].
__device__ __forceinline__ unsigned long long scatter_local(unsigned l, int c, int m, const TileShape& t) {
  unsigned long long g = l & ((1u << c) - 1u);
#pragma unroll 8
  for (int i = 0; i < 8; ++i)
    if (i < m && ((l >> (c + i)) & 1u)) g |= 1ull << t.hi[i];
  return g;
}

// Per-term sums over tiles: each thread holds 8 amplitudes of the tile, reads
// their partners from LDS and keeps one accumulator per term across all tiles
// it visits, so the wave and workgroup reductions happen once per launch.
//
// A term's sum runs over one amplitude of each pair (j, j ^ x), split so that
// no lane idles (pauli_term): by the highest flipped bit when that is a
// register bit (4 of the 8 amplitudes), by waves when it is on the wave index,
// and over all amplitudes (each pair twice) when all flipped bits are lane
// bits.  The sign parity(j & z) splits over register, thread and tile bits.
// Two workgroups share a CU: one loads while the other sums.
//
// Bound by HBM and LDS reads: 16 bytes per amplitude and pass, and the same
// again from LDS per term, half of it where pairs are split.  The Ising
// chain's 27 X terms on 27 qubits: 5.2 ms in 5 passes of 2^11 tiles with a
// pair test per lane -> 1.41 ms in 3 passes of 2^12 (512
// threads; the first, 12 terms, 0.54, the others, 8 and 7, 0.43: 5 TB/s).
typedef double vd2r __attribute__((ext_vector_type(2)));
constexpr int kTileRegs = 8;
__device__ __forceinline__ double flip(double v, unsigned sign) {
  return __hiloint2double((int)((unsigned)__double2hiint(v) ^ sign), __double2loint(v));
}
// Re (IM = 0) or the -Im part's partner (IM = 1) of sum_j (-1)^{|j & zr|} conj(p_j) v_j over
// the registers with bit H - 1 clear (H = 0: all).
template <int IM, int H, bool Z>
__device__ __forceinline__ double tile_sum(const vd2r (&v)[kTileRegs], const vd2r* __restrict__ t, unsigned at,
                                           unsigned xr, unsigned zr, unsigned shift, unsigned mask) {
  vd2r p[kTileRegs];
#pragma unroll
  for (int j = 0; j < kTileRegs; ++j)
    if (H == 0 || !((j >> (H - 1)) & 1)) p[j] = t[(at ^ (((unsigned)j ^ xr) << shift)) & mask];
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int j = 0; j < kTileRegs; ++j)
    if (H == 0 || !((j >> (H - 1)) & 1)) {
      const unsigned sg = Z ? (unsigned)(__builtin_popcount(j & zr) & 1) << 31 : 0u;
      s0 = fma(flip(p[j].x, sg), IM ? v[j].y : v[j].x, s0);
      s1 = fma(flip(p[j].y, sg), IM ? v[j].x : v[j].y, s1);
    }
  return IM ? s0 - s1 : s0 + s1;
}
template <int IM, int H>
__device__ __forceinline__ double tile_term(const vd2r (&v)[kTileRegs], const vd2r* __restrict__ t, unsigned at,
                                            unsigned xr, unsigned zr, unsigned shift, unsigned mask) {
  return zr == 0u ? tile_sum<IM, H, false>(v, t, at, xr, zr, shift, mask)
                  : tile_sum<IM, H, true>(v, t, at, xr, zr, shift, mask);
}
template <int TPL, bool NT>   // 16 accumulators
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_pauli_tile(
    const double2* __restrict__ a, int nbits, TileShape t, int shift, const TermDev* __restrict__ terms, int count,
    double* __restrict__ partials) {
  extern __shared__ double2 lds_tile[];
  vd2r* __restrict__ lt = reinterpret_cast<vd2r*>(lds_tile);
  const int k = t.c + t.m;
  const unsigned tile_len = 1u << k, mask = tile_len - 1u, tid = threadIdx.x;
  const unsigned long long ntiles = 1ull << (nbits - k);
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const unsigned long long own = scatter_local(tid, t.c, t.m, t);
  unsigned long long off[kTileRegs];
#pragma unroll
  for (int j = 0; j < kTileRegs; ++j) off[j] = scatter_local((unsigned)j << shift, t.c, t.m, t);
  auto base_of = [&](unsigned long long tile) {   // tile index over the bits outside the tile
    unsigned long long base = tile << t.c;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < t.m) {
        const int q = t.hi[i];
        base = ((base >> q) << (q + 1)) | (base & ((1ull << q) - 1ull));
      }
    return base;
  };
  double acc[TPL];
#pragma unroll
  for (int i = 0; i < TPL; ++i) acc[i] = 0.0;
  for (unsigned long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const unsigned long long base = base_of(tile);
    vd2r v[kTileRegs];
#pragma unroll
    for (int j = 0; j < kTileRegs; ++j)
      {
        const vd2r* from = reinterpret_cast<const vd2r*>(a + ((base | off[j]) | own));
        v[j] = vd2r{0.0, 0.0};
        if ((tid | ((unsigned)j << shift)) < tile_len) v[j] = NT ? __builtin_nontemporal_load(from) : *from;
      }
    // the terms' lines into the scalar cache at once, not one miss per term (9
    // to 11 qubits: 16 -> 10 us)
    if (tile == blockIdx.x) {
      int x[TPL];
#pragma unroll
      for (int i = 0; i < TPL; ++i) x[i] = terms[min(i, count - 1)].row;
#pragma unroll
      for (int i = 0; i < TPL; ++i) asm volatile("" ::"s"(x[i]));
    }
    __syncthreads();   // previous tile's readers are done
#pragma unroll
    for (int j = 0; j < kTileRegs; ++j) {
      const unsigned l = tid | ((unsigned)j << shift);
      if (l < tile_len) lt[l] = v[j];
    }
    __syncthreads();
    for (int ti = 0; ti < count; ++ti) {
      const unsigned xl = (unsigned)terms[ti].xl, zl = (unsigned)terms[ti].zl, wm = terms[ti].waves;
      if (__builtin_popcount(((unsigned)wave * kWave) & wm) & 1) continue;
      const unsigned at = tid ^ (xl & ((1u << shift) - 1u)), xr = xl >> shift, zr = zl >> shift;
      double s;
      switch (terms[ti].half + ((terms[ti].y & 1) << 2)) {
        case 0: s = tile_term<0, 0>(v, lt, at, xr, zr, shift, mask); break;
        case 1: s = tile_term<0, 1>(v, lt, at, xr, zr, shift, mask); break;
        case 2: s = tile_term<0, 2>(v, lt, at, xr, zr, shift, mask); break;
        case 3: s = tile_term<0, 3>(v, lt, at, xr, zr, shift, mask); break;
        case 4: s = tile_term<1, 0>(v, lt, at, xr, zr, shift, mask); break;
        case 5: s = tile_term<1, 1>(v, lt, at, xr, zr, shift, mask); break;
        case 6: s = tile_term<1, 2>(v, lt, at, xr, zr, shift, mask); break;
        default: s = tile_term<1, 3>(v, lt, at, xr, zr, shift, mask); break;
      }
      const unsigned outer = (unsigned)__builtin_popcountll(base & terms[ti].zo);
      s = flip(s, (((unsigned)__popc(tid & zl & ((1u << shift) - 1u)) + outer) & 1u) << 31);
      // a branch to the term's accumulator, not 16 selects
#define NWQ_ACC(I) \
  case I: acc[I] += s; asm volatile("" : "+v"(acc[I])); break;
      switch (ti) {
        NWQ_ACC(0) NWQ_ACC(1) NWQ_ACC(2) NWQ_ACC(3) NWQ_ACC(4) NWQ_ACC(5) NWQ_ACC(6) NWQ_ACC(7)
        NWQ_ACC(8) NWQ_ACC(9) NWQ_ACC(10) NWQ_ACC(11) NWQ_ACC(12) NWQ_ACC(13) NWQ_ACC(14) NWQ_ACC(15)
      }
#undef NWQ_ACC
    }
  }
  __syncthreads();
  double* red = reinterpret_cast<double*>(lds_tile);   // [wave][term]; the host sizes it
#pragma unroll
  for (int i = 0; i < TPL; ++i) {
    if (i < count) {
      const double w = wave_sum(acc[i]);
      if (lane == 0) red[wave * TPL + i] = w;
    }
  }
  __syncthreads();
  if ((int)tid < count) {
    double s = 0.0;
    for (unsigned w = 0; w < blockDim.x / kWave; ++w) s += red[w * TPL + tid];
    partials[(unsigned long long)terms[tid].row * gridDim.x + blockIdx.x] = s * terms[tid].scale;
  }
}

// Terms with no flipped bits: <Z^z> = sum_j (-1)^{|j & z|} |a_j|^2.  A
// workgroup visits chunks of 2048 consecutive entries (grid-stride); thread
// tid reads entries B + 256 e + tid (e < 8), one coalesced load each.  The
// sign of entry j splits as the parities of (j & z) over three disjoint bit
// fields: tid (fixed per thread), e (bits 8 to 10) and the chunk base B
// (uniform, scalar work).  The sums over e with the signs of all 8 possible
// fields of z are one Walsh-Hadamard transform of the thread's 8 values, so a
// term costs a pick and an add per thread and chunk instead of a sign and an
// add per entry, and up to 32 terms run at the rate of the loads (26 terms of
// the Ising chain on 27 qubits: 0.68 ms in two passes of 13 -> 0.37 ms).
// Loads are non-temporal, and with xcd_order (grid a multiple of 8)
// workgroup i starts at chunk (i mod 8) G/8 + floor(i / 8), so each of the 8
// XCDs (dealt workgroups in turn) reads contiguous chunks on every sweep.  The
// chunks each block visits, and so the rounding of the sums, are fixed by the
// grid size alone.
template <int TPL>
__global__ __launch_bounds__(kRedBlock) void k_pauli_diag(const double2* __restrict__ a, unsigned long long len,
                                                          ZMasks zs, int count, double* __restrict__ partials,
                                                          int xcd_order) {
  constexpr int EPT = 8;
  static_assert(kRedBlock == 256 && TPL <= 32, "entry e sits at bit 8 + log2 e; a thread's signs fill one word");
  __shared__ double s_acc[TPL][kRedWaves];
  constexpr unsigned long long kChunk = (unsigned long long)kRedBlock * EPT;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const unsigned tid = threadIdx.x;
  unsigned own = 0;   // bit t: parity(tid & z_t)
#pragma unroll
  for (int t = 0; t < TPL; ++t)
    if (t < count) own |= ((unsigned)__popc(tid & (unsigned)(zs.z[t] & 0xFFull)) & 1u) << t;
  double acc[TPL];
#pragma unroll
  for (int t = 0; t < TPL; ++t) acc[t] = 0.0;
  const unsigned long long first =
      xcd_order ? (unsigned long long)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)) : blockIdx.x;
  for (unsigned long long B = first * kChunk; B < len; B += (unsigned long long)gridDim.x * kChunk) {
    double p[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const unsigned long long i = B + (unsigned long long)e * kRedBlock + tid;
      const vd2r v = i < len ? __builtin_nontemporal_load(reinterpret_cast<const vd2r*>(a + i)) : vd2r{0.0, 0.0};
      p[e] = fma(v.x, v.x, v.y * v.y);
    }
#pragma unroll
    for (int h = 1; h < EPT; h <<= 1)
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (!(e & h)) {
          const double u = p[e], w = p[e | h];
          p[e] = u + w;
          p[e | h] = u - w;
        }
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
      if (t < count) {
        const unsigned long long z = zs.z[t];
        const unsigned cb = (unsigned)__builtin_popcountll(B & z) & 1u;   // B has no bits below 11
        double w;
        switch ((unsigned)(z >> 8) & 7u) {
          case 0: w = p[0]; break;
          case 1: w = p[1]; break;
          case 2: w = p[2]; break;
          case 3: w = p[3]; break;
          case 4: w = p[4]; break;
          case 5: w = p[5]; break;
          case 6: w = p[6]; break;
          default: w = p[7]; break;
        }
        acc[t] += flip(w, (((own >> t) ^ cb) & 1u) << 31);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    if (t < count) {
      const double w = wave_sum(acc[t]);
      if (lane == 0) s_acc[t][wave] = w;
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < count) {
    double s = 0.0;
    for (int w = 0; w < kRedWaves; ++w) s += s_acc[threadIdx.x][w];
    partials[(unsigned long long)zs.row[threadIdx.x] * gridDim.x + blockIdx.x] = s;
  }
}

// One term whose flipped bits do not fit a tile: pairs (j, j^x) over the
// j with bit h (the lowest bit of x) clear, read straight from global memory.
__global__ __launch_bounds__(kRedBlock) void k_pauli_pairs(const double2* __restrict__ a, int nbits,
                                                           unsigned long long x, unsigned long long z, int y,
                                                           double* __restrict__ partials) {
  __shared__ double accw[kRedWaves];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int h = __ffsll((long long)x) - 1;
  const unsigned long long npairs = 1ull << (nbits - 1);
  double s = 0.0;
  for (unsigned long long p = (unsigned long long)blockIdx.x * kRedBlock + threadIdx.x; p < npairs;
       p += (unsigned long long)gridDim.x * kRedBlock) {
    const unsigned long long j = ((p >> h) << (h + 1)) | (p & ((1ull << h) - 1ull));
    const double2 v = a[j];
    const double2 q = a[j ^ x];
    const double wr = fma(q.x, v.x, q.y * v.y);
    const double wi = fma(q.x, v.y, -q.y * v.x);
    double r;
    switch (y & 3) {
      case 0: r = wr; break;
      case 1: r = -wi; break;
      case 2: r = -wr; break;
      default: r = wi; break;
    }
    r *= 2.0;
    s += (__popcll(j & z) & 1) ? -r : r;
  }
  s = wave_sum(s);
  if (lane == 0) accw[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < kRedWaves; ++w) r += accw[w];
    partials[blockIdx.x] = r;
  }
}

// Tr(rho P) = sum_r rho[r, r^x] i^y (-1)^{|r&z|} over the 2^n rows.
__global__ __launch_bounds__(kRedBlock) void k_dm_pauli(const double2* __restrict__ rho, int n,
                                                        const TermDev* __restrict__ terms, int count,
                                                        double* __restrict__ partials) {
  __shared__ double accr[kRedWaves], acci[kRedWaves];
  const unsigned long long dim = 1ull << n;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (int ti = 0; ti < count; ++ti) {
    const TermDev T = terms[ti];    // for DM the masks are global: xl = x, zl = z
    double sr = 0.0, si = 0.0;
    for (unsigned long long r = (unsigned long long)blockIdx.x * kRedBlock + threadIdx.x; r < dim;
         r += (unsigned long long)gridDim.x * kRedBlock) {
      const double2 v = rho[r * dim + (r ^ T.xl)];
      double vr = v.x, vi = v.y;
      switch (T.y & 3) {   // multiply by i^y
        case 1: { const double t0 = vr; vr = -vi; vi = t0; break; }
        case 2: vr = -vr; vi = -vi; break;
        case 3: { const double t0 = vr; vr = vi; vi = -t0; break; }
        default: break;
      }
      if (__popcll(r & T.zl) & 1) { vr = -vr; vi = -vi; }
      sr += vr;
      si += vi;
    }
    sr = wave_sum(sr);
    si = wave_sum(si);
    if (lane == 0) { accr[wave] = sr; acci[wave] = si; }
    __syncthreads();
    if (threadIdx.x == 0) {
      double a0 = 0.0, a1 = 0.0;
      for (int w = 0; w < kRedWaves; ++w) { a0 += accr[w]; a1 += acci[w]; }
      partials[(unsigned long long)(2 * ti) * gridDim.x + blockIdx.x] = a0;
      partials[(unsigned long long)(2 * ti + 1) * gridDim.x + blockIdx.x] = a1;
    }
    __syncthreads();
  }
}

template <int EPT>
__global__ __launch_bounds__(kRedBlock) void k_sumsq(const double2* __restrict__ a, unsigned long long len,
                                                     double* __restrict__ partials) {
  __shared__ double accw[kRedWaves];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  double s = 0.0;
  const unsigned long long stride = (unsigned long long)gridDim.x * kRedBlock * EPT;
  for (unsigned long long i0 = (unsigned long long)blockIdx.x * kRedBlock * EPT + threadIdx.x; i0 < len; i0 += stride) {
    double2 v[EPT];
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const unsigned long long i = i0 + (unsigned long long)j * kRedBlock;
      v[j] = i < len ? a[i] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int j = 0; j < EPT; ++j) s += fma(v[j].x, v[j].x, v[j].y * v[j].y);
  }
  s = wave_sum(s);
  if (lane == 0) accw[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < kRedWaves; ++w) r += accw[w];
    partials[blockIdx.x] = r;
  }
}

// Second stage: one wave per row, lane-strided partial sums (four chains, so
// that a row's loads are in flight together) then the xor tree; optional
// coefficient-weighted total in row order by one lane.  53 rows of 2048
// partials: 190 us with 4 waves and one chain -> 26 us with 16.
constexpr int kRowWaves = 16;
__global__ __launch_bounds__(kRowWaves * kWave) void k_reduce_rows(const double* __restrict__ partials, int rows,
                                                                   int grid, const double* __restrict__ coeffs,
                                                                   double* __restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (int r = wave; r < rows; r += kRowWaves) {
    const double* __restrict__ row = partials + (unsigned long long)r * grid;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int b = lane;
    for (; b + 7 * kWave < grid; b += 8 * kWave) {
      double v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = row[b + i * kWave];
#pragma unroll
      for (int i = 0; i < 8; ++i) s[i & 3] += v[i];
    }
    for (; b < grid; b += kWave) s[0] += row[b];
    const double w = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
    if (lane == 0) out[r] = w;
  }
  if (coeffs != nullptr) {
    __syncthreads();
    __threadfence_block();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int r = 0; r < rows; ++r) t = fma(coeffs[r], out[r], t);
      out[rows] = t;
    }
  }
}

}  // namespace

int pauli_grid(int nbits) {
  return nbits >= 22 ? 2048 : nbits <= 11 ? 1 : 1 << (nbits - 11);
}

// Threads of a tile of 2^k: 8 amplitudes each, at least one wave.
static int tile_shift(int k) { return std::max(6, k - 3); }

TermDev pauli_term(const TileShape& t, unsigned long long x, unsigned long long z, int row) {
  auto local = [&](unsigned long long mask) {
    unsigned long long l = mask & ((1ull << t.c) - 1ull);
    for (int i = 0; i < t.m; ++i)
      if ((mask >> t.hi[i]) & 1ull) l |= 1ull << (t.c + i);
    return l;
  };
  unsigned long long inside = (1ull << t.c) - 1ull;
  for (int i = 0; i < t.m; ++i) inside |= 1ull << t.hi[i];
  TermDev d{};
  d.xl = local(x);
  d.zl = local(z & inside);
  d.zo = z & ~inside;
  d.y = __builtin_popcountll(x & z) & 3;
  d.row = row;
  // Re(i^y w): wr, -wi, -wr, wi
  d.scale = d.y == 1 || d.y == 2 ? -1.0 : 1.0;
  const int shift = tile_shift(t.c + t.m), top = 63 - __builtin_clzll(d.xl);
  if (top >= shift) {
    d.half = top - shift + 1;
  } else if (top >= 6) {
    d.waves = 1u << top;
    // with a wave bit that the term leaves alone, so that terms split differently
    for (int b = top + 1 < shift ? top + 1 : 6; b != top; b = b + 1 < shift ? b + 1 : 6)
      if (!((d.xl >> b) & 1ull)) {
        d.waves |= 1u << b;
        break;
      }
  }
  if (top >= 6) d.scale *= 2.0;   // one amplitude of each pair
  return d;
}

void launch_pauli_tile(hipStream_t s, const double2* a, int nbits, const TileShape& t, const TermDev* terms,
                       int count, double* partials, int grid) {
  const int shift = tile_shift(t.c + t.m);
  const size_t lds = std::max<size_t>(sizeof(double2) << (t.c + t.m), (sizeof(double) * kTileTerms << shift) / kWave);
  // States beyond the 256 MB cache are read past it (27 X terms on 27 qubits: 1.47
  // -> 1.41 ms); smaller ones stay in it from pass to pass (24 qubits 0.28 ms
  // against 0.30).
  auto kern = nbits >= 25 ? k_pauli_tile<kTileTerms, true> : k_pauli_tile<kTileTerms, false>;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(1u << shift), lds, s, a, nbits, t, shift, terms, count, partials);
}

void launch_pauli_diag(hipStream_t s, const double2* a, int nbits, const ZMasks& zs, int count, double* partials,
                       int grid) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kRedBlock), 0, s, a, 1ull << nbits, zs, count, partials,
                       grid % 8 == 0 ? 1 : 0);
  };
  if (count <= 16) go(k_pauli_diag<16>);
  else go(k_pauli_diag<kDiagTerms>);
}

void launch_pauli_pairs(hipStream_t s, const double2* a, int nbits, unsigned long long x, unsigned long long z,
                        int y, double* partials, int grid) {
  hipLaunchKernelGGL(k_pauli_pairs, dim3(grid), dim3(kRedBlock), 0, s, a, nbits, x, z, y, partials);
}

int dm_pauli_grid(int n) {
  const unsigned long long dim = 1ull << n;
  const unsigned long long g = (dim + kRedBlock - 1) / kRedBlock;
  return (int)(g < 256 ? g : 256);
}

void launch_dm_pauli(hipStream_t s, const double2* rho, int n, const TermDev* terms, int count, double* partials,
                     int grid) {
  hipLaunchKernelGGL(k_dm_pauli, dim3(grid), dim3(kRedBlock), 0, s, rho, n, terms, count, partials);
}

int sumsq_grid(unsigned long long len) {
  const unsigned long long g = (len + kRedBlock * 4 - 1) / (kRedBlock * 4);
  return (int)(g < 2048 ? g : 2048);
}

void launch_sumsq(hipStream_t s, const double2* a, unsigned long long len, double* partials, int grid) {
  hipLaunchKernelGGL(k_sumsq<4>, dim3(grid), dim3(kRedBlock), 0, s, a, len, partials);
}

void launch_reduce_rows(hipStream_t s, const double* partials, int rows, int grid, const double* coeffs,
                        double* out) {
  hipLaunchKernelGGL(k_reduce_rows, dim3(1), dim3(kRowWaves * kWave), 0, s, partials, rows, grid, coeffs, out);
}

}  // namespace nwq
