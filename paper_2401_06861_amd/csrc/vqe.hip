// VQE energies and adjoint gradients for batches of parameter vectors.
//
// The VQE experiment of the paper (Sec. III, Fig. 4) evaluates
// E(theta) = <psi(theta)|H|psi(theta)> for a parametrised circuit.  Here the
// gradient is computed by adjoint differentiation (Jones & Gacon,
// arXiv:2009.02823): with phi = U_G...U_1|0>, lambda = H phi, E = Re<phi|lambda>,
// then for k = G..1:  g_k = Im<lambda|P_k|phi>  (for U_k = exp(-i theta P_k/2)),
// phi <- U_k^dag phi,  lambda <- U_k^dag lambda.
//
// Two execution paths share the op encoding:
//  * Resident (n <= 12): one workgroup owns one theta vector and keeps phi and
//    lambda in registers (k_vqe_reg; programs too long for its tables: in LDS,
//    k_vqe_lds) for the whole forward pass, H application and backward sweep;
//    a persistent grid walks the batch.  One launch per batch.
//  * Global (any n): one launch per gate over all B states (blockIdx.y = batch
//    element), phi and lambda in HBM, gradient partials per (state, gate, block)
//    reduced in a fixed order; the whole schedule is captured once per batch
//    size in a hipGraph and replayed.  With B = 1 and no graph this is the
//    plain per-circuit path.
// Every reduction has a fixed order that does not depend on B, so a theta
// vector gives bit-identical results alone or inside any batch.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>

#include "engine.h"

namespace nwq {

enum VqeKind { OP_ROT = 0, OP_RZZ = 1, OP_FIX1 = 2, OP_CX = 3, OP_CZ = 4, OP_SWAP = 5 };

struct VqeOp {
  int kind;
  int q0, q1;
  int param;   // theta index (OP_ROT, OP_RZZ), else -1
  int axis;    // OP_ROT: 0 X, 1 Y, 2 Z
  int slot;    // gradient slot (ordinal among parametrised ops), else -1
  int mat;     // OP_FIX1: index into the fixed-matrix table (8 double2: U then U^dag)
  int pad;
};

struct VqeTerm {
  unsigned long long x, z;
  double c;
  int y;       // popcount(x & z) mod 4
  int pad;
};

namespace {

typedef double vd2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned ins0(unsigned p, int q) { return ((p >> q) << (q + 1)) | (p & ((1u << q) - 1u)); }
__device__ __forceinline__ unsigned long long ins0l(unsigned long long p, int q) {
  return ((p >> q) << (q + 1)) | (p & ((1ull << q) - 1ull));
}
__device__ __forceinline__ vd2 mk(double a, double b) { vd2 r; r.x = a; r.y = b; return r; }
__device__ __forceinline__ vd2 cmul(vd2 a, vd2 b) { return mk(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x)); }
__device__ __forceinline__ vd2 cfma(vd2 a, vd2 b, vd2 c) {
  return mk(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ vd2 ld(const double2* p) { return *reinterpret_cast<const vd2*>(p); }
__device__ __forceinline__ void st(double2* p, vd2 v) { *reinterpret_cast<vd2*>(p) = v; }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Sum over a full wave (all 64 lanes active) with DPP lane moves only, no LDS
// traffic: pairs within quads, quads (half mirror), half rows (mirror), then
// rows 0 -> 1 and 2 -> 3 (broadcast of lane 15) and rows 0..1 -> 3
// (broadcast of lane 31); lane 63 ends with the total, which every lane
// reads.  Lanes a move does not write add 0.  The order is fixed.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_full(double v) {
  v += dpp_move<0xB1>(v);         // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);         // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);        // row_half_mirror
  v += dpp_move<0x140>(v);        // row_mirror
  v += dpp_move<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

// 2x2 matrices.  Rotations exp(-i t P/2) are built branch-free (the axis
// picks entries with selects) and fixed gates are loaded from the table in
// separate code paths: with this toolchain a branchy construction of the
// rotation matrix whose results merged with the table load was compiled to
// code that dropped the imaginary part of the RZ diagonal, so the two cases
// are never merged into one value.  The adjoint of a rotation is the
// rotation by -t.
struct M2 { vd2 m0, m1, m2, m3; };

__device__ __forceinline__ M2 rot_matrix(int axis, double theta, bool dag) {
  double s, c;
  sincos(0.5 * theta, &s, &c);
  s = dag ? -s : s;
  const double z = 0.0;
  M2 r;
  r.m0 = mk(c, axis == 2 ? -s : z);
  r.m1 = mk(axis == 1 ? -s : z, axis == 0 ? -s : z);
  r.m2 = mk(axis == 1 ? s : z, axis == 0 ? -s : z);
  r.m3 = mk(c, axis == 2 ? s : z);
  return r;
}

__device__ __forceinline__ M2 fixed_matrix(int mat, const double2* fixed, bool dag) {
  const double2* f = fixed + 8 * mat + (dag ? 4 : 0);
  M2 r;
  r.m0 = ld(f); r.m1 = ld(f + 1); r.m2 = ld(f + 2); r.m3 = ld(f + 3);
  return r;
}

// RZZ: diagonal e^{-i t/2} (even parity), e^{+i t/2} (odd parity)
__device__ __forceinline__ void rzz_phases(double theta, bool dag, vd2& even, vd2& odd) {
  double s, c;
  sincos(0.5 * theta, &s, &c);
  s = dag ? -s : s;
  even = mk(c, -s);
  odd = mk(c, s);
}

template <typename Idx>
__device__ __forceinline__ void pairs_apply(double2* v, Idx N, int q, const M2& m, Idx tid, Idx nt) {
  const Idx off = Idx(1) << q;
  for (Idx p = tid; p < (N >> 1); p += nt) {
    const Idx i0 = ((p >> q) << (q + 1)) | (p & (off - 1));
    const vd2 a = ld(v + i0), b = ld(v + i0 + off);
    st(v + i0, cfma(m.m0, a, cmul(m.m1, b)));
    st(v + i0 + off, cfma(m.m2, a, cmul(m.m3, b)));
  }
}

// Contribution Im( conj(l0) (P phi)_0 + conj(l1) (P phi)_1 ) of one pair for a
// single-qubit Pauli generator on the pair's qubit, written with scalar
// selects only (no per-axis branches building vectors; see rot_matrix):
//   X: Im(conj(l0) p1) + Im(conj(l1) p0)
//   Y: Re(conj(l1) p0) - Re(conj(l0) p1)        ((Y phi)_0 = -i p1, (Y phi)_1 = i p0)
//   Z: Im(conj(l0) p0) - Im(conj(l1) p1)
__device__ __forceinline__ double pair_grad(int axis, vd2 p0, vd2 p1, vd2 l0, vd2 l1) {
  const double im01 = l0.x * p1.y - l0.y * p1.x;
  const double im10 = l1.x * p0.y - l1.y * p0.x;
  const double re01 = l0.x * p1.x + l0.y * p1.y;
  const double re10 = l1.x * p0.x + l1.y * p0.y;
  const double im00 = l0.x * p0.y - l0.y * p0.x;
  const double im11 = l1.x * p1.y - l1.y * p1.x;
  const double gx = im01 + im10, gy = re10 - re01, gz = im00 - im11;
  return axis == 0 ? gx : (axis == 1 ? gy : gz);
}

// ---------------------------------------------------------------------------
// Gate application on one state held in LDS (or in global memory for the
// per-gate path: same code, different pointer).  Threads tid..nt stride.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void apply_op_state(double2* v, int n, const VqeOp& op, const double* th, const double2* fixed, bool dag,
                               unsigned tid, unsigned nt) {
  const unsigned N = 1u << n;
  switch (op.kind) {
    case OP_ROT:
      pairs_apply<unsigned>(v, N, op.q0, rot_matrix(op.axis, th[op.param], dag), tid, nt);
      break;
    case OP_FIX1:
      pairs_apply<unsigned>(v, N, op.q0, fixed_matrix(op.mat, fixed, dag), tid, nt);
      break;
    case OP_RZZ: {
      vd2 e, o;
      rzz_phases(th[op.param], dag, e, o);
      for (unsigned j = tid; j < N; j += nt) {
        const unsigned par = ((j >> op.q0) ^ (j >> op.q1)) & 1u;
        st(v + j, cmul(par ? o : e, ld(v + j)));
      }
      break;
    }
    case OP_CZ: {
      for (unsigned j = tid; j < N; j += nt)
        if (((j >> op.q0) & (j >> op.q1)) & 1u) { const vd2 x = ld(v + j); st(v + j, mk(-x.x, -x.y)); }
      break;
    }
    default: {   // OP_CX (control q0, target q1) or OP_SWAP: exchange two members of each quad
      const int lo = min(op.q0, op.q1), hi = max(op.q0, op.q1);
      const unsigned oa = op.kind == OP_CX ? (1u << op.q0) : (1u << op.q0);
      const unsigned ob = op.kind == OP_CX ? (1u << op.q0) + (1u << op.q1) : (1u << op.q1);
      for (unsigned p = tid; p < (N >> 2); p += nt) {
        const unsigned b = ins0(ins0(p, lo), hi);
        const vd2 x = ld(v + b + oa), y = ld(v + b + ob);
        st(v + b + oa, y);
        st(v + b + ob, x);
      }
      break;
    }
  }
}

// One backward step on (phi, lam): returns this thread's gradient partial
// (0 for unparametrised ops) and applies U^dag to both states.
__device__ __forceinline__ double adjoint_step(double2* phi, double2* lam, int n, const VqeOp& op, const double* th,
                               const double2* fixed, unsigned tid, unsigned nt) {
  const unsigned N = 1u << n;
  double g = 0.0;
  if (op.kind == OP_ROT) {
    const M2 m = rot_matrix(op.axis, th[op.param], true);
    const unsigned off = 1u << op.q0;
    for (unsigned p = tid; p < (N >> 1); p += nt) {
      const unsigned i0 = ins0(p, op.q0);
      const vd2 p0 = ld(phi + i0), p1 = ld(phi + i0 + off);
      const vd2 l0 = ld(lam + i0), l1 = ld(lam + i0 + off);
      g += pair_grad(op.axis, p0, p1, l0, l1);
      st(phi + i0, cfma(m.m0, p0, cmul(m.m1, p1)));
      st(phi + i0 + off, cfma(m.m2, p0, cmul(m.m3, p1)));
      st(lam + i0, cfma(m.m0, l0, cmul(m.m1, l1)));
      st(lam + i0 + off, cfma(m.m2, l0, cmul(m.m3, l1)));
    }
  } else if (op.kind == OP_RZZ) {
    vd2 e, o;
    rzz_phases(th[op.param], true, e, o);
    for (unsigned j = tid; j < N; j += nt) {
      const unsigned par = ((j >> op.q0) ^ (j >> op.q1)) & 1u;
      const vd2 p = ld(phi + j), l = ld(lam + j);
      const double t = l.x * p.y - l.y * p.x;   // Im(conj(l) p), generator Z Z = +-1
      g += par ? -t : t;
      st(phi + j, cmul(par ? o : e, p));
      st(lam + j, cmul(par ? o : e, l));
    }
  } else {
    apply_op_state(phi, n, op, th, fixed, true, tid, nt);
    apply_op_state(lam, n, op, th, fixed, true, tid, nt);
  }
  return g;
}

// (H phi)_j = sum_t c_t i^y (-1)^{|(j^x)&z|} phi_{j^x}
__device__ __forceinline__ vd2 h_apply_at(const double2* phi, unsigned long long j, const VqeTerm* terms, int nterms,
                                          const double* cb) {
  vd2 acc = mk(0.0, 0.0);
  for (int t = 0; t < nterms; ++t) {
    const VqeTerm T = terms[t];
    const double tc = cb ? cb[t] : T.c;
    const unsigned long long k = j ^ T.x;
    vd2 v = ld(phi + k);
    switch (T.y & 3) {
      case 1: v = mk(-v.y, v.x); break;
      case 2: v = mk(-v.x, -v.y); break;
      case 3: v = mk(v.y, -v.x); break;
      default: break;
    }
    const double c = (__popcll(k & T.z) & 1) ? -tc : tc;
    acc.x = fma(c, v.x, acc.x);
    acc.y = fma(c, v.y, acc.y);
  }
  return acc;
}

// ---------------------------------------------------------------------------
// LDS-resident persistent kernel (n <= 12), for programs whose tables and
// gradient partials do not fit the register-resident kernel's LDS
// ---------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT) void k_vqe_lds(int n, const VqeOp* __restrict__ ops, int nops,
                                                const double2* __restrict__ fixed, const VqeTerm* __restrict__ terms,
                                                int nterms, int nslots, const int* __restrict__ slot_param,
                                                const double* __restrict__ theta, int P, int B,
                                                const double* __restrict__ coeffs,
                                                double* __restrict__ E, double* __restrict__ grad) {
  extern __shared__ double2 lds[];
  constexpr int NW = NT / kWave;
  const unsigned N = 1u << n;
  double2* phi = lds;
  double2* lam = lds + N;
  double* red = reinterpret_cast<double*>(grad ? lds + 2 * N : lds + N);   // [NW] scratch
  double* gpart = red + NW;                                              // [nslots][NW]
  const unsigned tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    const double* th = theta + (size_t)b * P;
    __syncthreads();
    for (unsigned j = tid; j < N; j += NT) phi[j] = make_double2(j == 0 ? 1.0 : 0.0, 0.0);
    __syncthreads();
    for (int i = 0; i < nops; ++i) {
      apply_op_state(phi, n, ops[i], th, fixed, false, tid, NT);
      __syncthreads();
    }
    // lambda = H phi and E = Re <phi|lambda>
    double e = 0.0;
    for (unsigned j = tid; j < N; j += NT) {
      const vd2 l = h_apply_at(phi, j, terms, nterms, coeffs ? coeffs + (size_t)b * nterms : nullptr);
      const vd2 p = ld(phi + j);
      e += p.x * l.x + p.y * l.y;
      if (grad) st(lam + j, l);
    }
    e = wave_sum(e);
    if (lane == 0) red[wave] = e;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < NW; ++w) s += red[w];
      E[b] = s;
    }
    if (!grad) continue;
    for (int i = nops - 1; i >= 0; --i) {
      const VqeOp op = ops[i];
      const double g = adjoint_step(phi, lam, n, op, th, fixed, tid, NT);
      if (op.slot >= 0) {
        const double w = wave_sum(g);
        if (lane == 0) gpart[op.slot * NW + wave] = w;
      }
      __syncthreads();
    }
    // grad[b][p] = sum over the slots of p (slot order) of the wave partials (wave order)
    if (tid == 0) {
      for (int p = 0; p < P; ++p) grad[(size_t)b * P + p] = 0.0;
      for (int s = 0; s < nslots; ++s) {
        double v = 0.0;
        for (int w = 0; w < NW; ++w) v += gpart[s * NW + w];
        grad[(size_t)b * P + slot_param[s]] += v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Register-resident kernel (n <= 12).  One workgroup per theta vector holds
// phi (and lambda on the way back) in registers, 8 amplitudes per thread over
// 3 register bits; the program runs as register phases (as the fused blocks
// do) with an LDS exchange between them, forward and then backward through
// the same phases.  k_vqe_lds passes the whole state through LDS, with a
// barrier, for every gate, and one thread adds up the gradient.  Here LDS is
// crossed once per phase (40 phases for the 280 gates of n=12, L=8, 29 of them
// inside a wave), the angles' sines are computed once per vector, the program
// and the Hamiltonian's terms are read from LDS, RZ and RZZ turn only the half
// of the amplitudes whose phase differs (a global phase changes neither the
// energy nor the gradient), RY and RX are three shears in place, and each
// parameter's slots are added by a thread of its own.  256 vectors with
// gradients: n=8, L=4 149 -> 76 us, n=12, L=8 1020 -> 244 us a call.
// What bounds it: the chain of ops of one vector on one CU.  At n=12 an op
// takes about 0.4 us forward, half of it FP64 issue of the two waves per SIMD,
// the rest the dispatch; at n=8 one wave has the CU to itself.
// ---------------------------------------------------------------------------
struct RegOpV {
  int code;          // RegVCode + 32 (gradient slot + 1)
  int mat;           // fixed 2x2: index into the fixed-matrix table; RV_YZ: gradient slot of RZ
  int param, param2; // theta indices (RV_YZ: of RY and RZ) or -1
};
// register-bit pairs B0 < B1 numbered as rb_pair
enum RegVCode { RV_ROT = 0 /* + 3 axis + B */, RV_FIX = 9 /* + B */, RV_RZZ = 12 /* + pair */, RV_CZ = 15,
                RV_CX = 18 /* + 2 pair + (control is B1) */, RV_SWAP = 24,
                RV_YZ = 27 /* + B: RY, then RZ with the next entry's numbers and slot */ };

// A turn by an angle f as three shears, x0 -= t x1; x1 += s x0; x0 -= t x1 with
// t = tan(f / 2) and s = sin f: three FMAs per pair and component instead of
// two products and two FMAs, each in place (products into new registers end
// every case of the op switch with copies back into the loop's registers, as
// long as the arithmetic itself).  RX and RY take the sine and cosine of
// theta / 2 themselves, exact to rounding for every finite theta, and flip both
// signs where the cosine is negative (a global sign), so that |f| <= pi/2 and
// |t| <= 1.  (Multiples of pi held in two doubles, subtracted first, are off by
// |theta| 1e-33 and leave |f| beyond pi / 2 from |theta| = 2^53 on: gradients of
// 4 qubits at angles of 1e12 to 1e24 were 5e-10 off, energies 4e-9.)
// Against 80-bit arithmetic (n=8, L=4, 32 vectors) the gradients are 7.4e-16
// off with shears, 8.2e-16 with the products, 9.8e-16 with k_vqe_lds.
__device__ __forceinline__ vd2 shear_of(double theta) {
  double sf, cf;
  sincos(0.5 * theta, &sf, &cf);
  if (cf < 0.0) sf = -sf;
  return mk(sf / (1.0 + fabs(cf)), sf);   // tan(f / 2), sin f
}

// Eight amplitudes as separate doubles (as 16-byte vectors in the op loop, every
// case of the switch builds new register tuples and copies them back).
struct Amp8 {
  double x[8], y[8];
};

// Gate `code` on the registers with (c, s) its angle's shear_of (RX, RY) or the
// cosine and sine of the whole angle (RZ, RZZ), or F its fixed matrix; DAG: the
// adjoint, with the sum of Im<l|P|p> over the registers first (g) and both
// vectors turned.
template <int B, int AX>
__device__ __forceinline__ void rv_turn(Amp8& v, double c, double s) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j & (1 << B)) continue;
    const int k = j | (1 << B);
    if constexpr (AX == 0) {          // [[cos, -i sin], [-i sin, cos]]
      v.x[j] = fma(c, v.y[k], v.x[j]);
      v.y[j] = fma(-c, v.x[k], v.y[j]);
      v.x[k] = fma(s, v.y[j], v.x[k]);
      v.y[k] = fma(-s, v.x[j], v.y[k]);
      v.x[j] = fma(c, v.y[k], v.x[j]);
      v.y[j] = fma(-c, v.x[k], v.y[j]);
    } else if constexpr (AX == 1) {   // [[cos, -sin], [sin, cos]]
      v.x[j] = fma(-c, v.x[k], v.x[j]);
      v.y[j] = fma(-c, v.y[k], v.y[j]);
      v.x[k] = fma(s, v.x[j], v.x[k]);
      v.y[k] = fma(s, v.y[j], v.y[k]);
      v.x[j] = fma(-c, v.x[k], v.x[j]);
      v.y[j] = fma(-c, v.y[k], v.y[j]);
    } else {                          // diag(1, e^{i theta})
      const double t = s * v.y[k];
      v.y[k] = fma(c, v.y[k], s * v.x[k]);
      v.x[k] = fma(c, v.x[k], -t);
    }
  }
}
// Im<l|P|p> of the generator on register bit B, in four chains (one would be as
// many dependent FMAs).
template <int B, int AX>
__device__ __forceinline__ double rv_grad(const Amp8& p, const Amp8& l) {
  double g[4] = {0.0, 0.0, 0.0, 0.0};
  int n = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j & (1 << B)) continue;
    const int k = j | (1 << B);
    double& h = g[n++ & 3];
    if constexpr (AX == 0) {
      h = fma(l.x[j], p.y[k], h);
      h = fma(-l.y[j], p.x[k], h);
      h = fma(l.x[k], p.y[j], h);
      h = fma(-l.y[k], p.x[j], h);
    } else if constexpr (AX == 1) {
      h = fma(l.x[k], p.x[j], h);
      h = fma(l.y[k], p.y[j], h);
      h = fma(-l.x[j], p.x[k], h);
      h = fma(-l.y[j], p.y[k], h);
    } else {
      h = fma(l.x[j], p.y[j], h);
      h = fma(-l.y[j], p.x[j], h);
      h = fma(-l.x[k], p.y[k], h);
      h = fma(l.y[k], p.x[k], h);
    }
  }
  return (g[0] + g[1]) + (g[2] + g[3]);
}
template <int B, int AX, bool DAG>
__device__ __forceinline__ void rv_rot(Amp8& p, Amp8& l, double c, double s, double& g) {
  if constexpr (DAG) {
    g = rv_grad<B, AX>(p, l);
    s = -s;
    if constexpr (AX != 2) c = -c;
  }
  rv_turn<B, AX>(p, c, s);
  if constexpr (DAG) rv_turn<B, AX>(l, c, s);
}
template <int B, bool DAG>
__device__ __forceinline__ void rv_yz(Amp8& p, Amp8& l, vd2 ay, vd2 az, double& gy, double& gz) {
  if constexpr (DAG) {
    rv_rot<B, 2, true>(p, l, az.x, az.y, gz);
    rv_rot<B, 1, true>(p, l, ay.x, ay.y, gy);
  } else {
    rv_turn<B, 1>(p, ay.x, ay.y);
    rv_turn<B, 2>(p, az.x, az.y);
  }
}
template <int B>
__device__ __forceinline__ void rv_mat(Amp8& v, const double2* __restrict__ M) {
  const vd2 m0 = ld(M), m1 = ld(M + 1), m2 = ld(M + 2), m3 = ld(M + 3);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j & (1 << B)) continue;
    const int k = j | (1 << B);
    const vd2 a = mk(v.x[j], v.y[j]), b = mk(v.x[k], v.y[k]);
    const vd2 u = cfma(m0, a, cmul(m1, b)), w = cfma(m2, a, cmul(m3, b));
    v.x[j] = u.x;
    v.y[j] = u.y;
    v.x[k] = w.x;
    v.y[k] = w.y;
  }
}
template <int B, bool DAG>
__device__ __forceinline__ void rv_fix(Amp8& p, Amp8& l, const double2* __restrict__ F) {
  rv_mat<B>(p, F + (DAG ? 4 : 0));
  if constexpr (DAG) rv_mat<B>(l, F + 4);
}
template <int B0, int B1, bool DAG>
__device__ __forceinline__ void rv_rzz(Amp8& p, Amp8& l, double c, double s, double& g) {
  if constexpr (DAG) s = -s;
  double g2[2] = {0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool odd = ((j >> B0) ^ (j >> B1)) & 1;
    if constexpr (DAG) {
      g2[j & 1] = fma(odd ? -l.x[j] : l.x[j], p.y[j], g2[j & 1]);
      g2[j & 1] = fma(odd ? l.y[j] : -l.y[j], p.x[j], g2[j & 1]);
      if (j == 7) g = g2[0] + g2[1];
    }
    if (!odd) continue;
    auto turn = [&](Amp8& v) {
      const double t = s * v.y[j];
      v.y[j] = fma(c, v.y[j], s * v.x[j]);
      v.x[j] = fma(c, v.x[j], -t);
    };
    turn(p);
    if constexpr (DAG) turn(l);
  }
}
template <int B0, int B1, bool DAG>
__device__ __forceinline__ void rv_cz(Amp8& p, Amp8& l) {
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (((j >> B0) & (j >> B1)) & 1) {
      p.x[j] = -p.x[j];
      p.y[j] = -p.y[j];
      if constexpr (DAG) {
        l.x[j] = -l.x[j];
        l.y[j] = -l.y[j];
      }
    }
}
template <int MASK, int OA, int OB, bool DAG>
__device__ __forceinline__ void rv_swap(Amp8& p, Amp8& l) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j & MASK) continue;
    auto swap = [](double& a, double& b) {
      const double t = a;
      a = b;
      b = t;
    };
    swap(p.x[j | OA], p.x[j | OB]);
    swap(p.y[j | OA], p.y[j | OB]);
    if constexpr (DAG) {
      swap(l.x[j | OA], l.x[j | OB]);
      swap(l.y[j | OA], l.y[j | OB]);
    }
  }
}

template <bool DAG>
__device__ __forceinline__ void rv_apply(int code, Amp8& p, Amp8& l, vd2 a, vd2 az, const double2* __restrict__ F,
                                         double& g, double& gz) {
  const double c = a.x, s = a.y;
#define NWQ_RV_ROT(AX) \
  case RV_ROT + 3 * AX + 0: rv_rot<0, AX, DAG>(p, l, c, s, g); break; \
  case RV_ROT + 3 * AX + 1: rv_rot<1, AX, DAG>(p, l, c, s, g); break; \
  case RV_ROT + 3 * AX + 2: rv_rot<2, AX, DAG>(p, l, c, s, g); break;
#define NWQ_RV_PAIR(P, LO, HI) \
  case RV_RZZ + P: rv_rzz<LO, HI, DAG>(p, l, c, s, g); break; \
  case RV_CZ + P: rv_cz<LO, HI, DAG>(p, l); break; \
  case RV_CX + 2 * P: rv_swap<(1 << LO) | (1 << HI), (1 << LO), (1 << LO) | (1 << HI), DAG>(p, l); break; \
  case RV_CX + 2 * P + 1: rv_swap<(1 << LO) | (1 << HI), (1 << HI), (1 << LO) | (1 << HI), DAG>(p, l); break; \
  case RV_SWAP + P: rv_swap<(1 << LO) | (1 << HI), (1 << LO), (1 << HI), DAG>(p, l); break;
  switch (code) {
    NWQ_RV_ROT(0)
    NWQ_RV_ROT(1)
    NWQ_RV_ROT(2)
    case RV_FIX + 0: rv_fix<0, DAG>(p, l, F); break;
    case RV_FIX + 1: rv_fix<1, DAG>(p, l, F); break;
    case RV_FIX + 2: rv_fix<2, DAG>(p, l, F); break;
    NWQ_RV_PAIR(0, 0, 1)
    NWQ_RV_PAIR(1, 0, 2)
    NWQ_RV_PAIR(2, 1, 2)
    case RV_YZ + 0: rv_yz<0, DAG>(p, l, a, az, g, gz); break;
    case RV_YZ + 1: rv_yz<1, DAG>(p, l, a, az, g, gz); break;
    case RV_YZ + 2: rv_yz<2, DAG>(p, l, a, az, g, gz); break;
    default: break;
  }
#undef NWQ_RV_ROT
#undef NWQ_RV_PAIR
}

constexpr int kRegMaxThreads = 512;   // n = 12
constexpr int kRegTerms = 64;         // Hamiltonian terms staged at a time

// Sum over each row of 16 lanes, in every lane.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return v;
}

// A phase's exchange read from the LDS copy of the program: images of thread
// and register bits as packed 16-bit pairs, wave-uniform.
struct RegMap {
  unsigned t[5], r[2];
};
__device__ __forceinline__ unsigned uni(unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ RegMap reg_map(const unsigned* w) {
  RegMap m;
#pragma unroll
  for (int i = 0; i < 5; ++i) m.t[i] = uni(w[i]);
  m.r[0] = uni(w[5]);
  m.r[1] = uni(w[6]);
  return m;
}
__device__ __forceinline__ unsigned thread_slot(unsigned v, const RegMap& m) {
  unsigned x = 0;
#pragma unroll
  for (int i = 0; i < 9; ++i) x ^= (unsigned)((int)(v << (31 - i)) >> 31) & ((m.t[i >> 1] >> (16 * (i & 1))) & 0xFFFFu);
  return x;
}
__device__ __forceinline__ unsigned register_slot(int j, const RegMap& m) {
  return ((j & 1) ? m.r[0] & 0xFFFFu : 0u) ^ ((j & 2) ? m.r[0] >> 16 : 0u) ^ ((j & 4) ? m.r[1] & 0xFFFFu : 0u);
}
// layout_phases' slot of an entry of 8 bytes
__device__ __forceinline__ unsigned slot8(unsigned e) {
  const unsigned f = e ^ (e >> 4) ^ (e >> 8);   // n <= 12
  return (e & ~15u) | (f & 15u);
}

// The two numbers of an op's angle (i even: its own, odd: of RZ in RV_YZ).
__device__ __forceinline__ void stage_angle(double2* cs, int i, const RegOpV& op, const double* __restrict__ th) {
  const int code = op.code & 31, param = (i & 1) ? op.param2 : op.param;
  if (param < 0) return;
  const bool whole = (i & 1) || (code >= RV_ROT + 6 && code < RV_YZ);   // RZ, RZZ
  vd2 a;
  if (whole) {
    double s, c;
    sincos(th[param], &s, &c);
    a = mk(c, s);
  } else {
    a = shear_of(th[param]);
  }
  st(cs + i, a);
}

// phases[0 .. P): the program's; phases[P]: where the last phase's registers go
// in LDS (wr_*) and which entries they are (rd_*).  pslots[poff[p] .. poff[p+1])
// are the slots of parameter p.
__global__ __launch_bounds__(kRegMaxThreads) void k_vqe_reg(
    int n, const RbPhase* __restrict__ phases, int P, const RegOpV* __restrict__ ops, int nops,
    const double2* __restrict__ fixed, const VqeTerm* __restrict__ terms, int nterms, int nslots,
    const int* __restrict__ poff, const int* __restrict__ pslots, const double* __restrict__ theta, int nparams, int B,
    const double* __restrict__ coeffs, double* __restrict__ E, double* __restrict__ grad) {
  extern __shared__ double2 lds[];
  const unsigned tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave, NW = (int)(nt + kWave - 1) / kWave;
  const int nb = n < 3 ? 3 : n;
  // entries of threads beyond the state (fewer than 8 * 64 amplitudes) stay zero and off LDS
  const bool live = (tid >> (nb - 3)) == 0;
  double* bufx = reinterpret_cast<double*>(lds);                 // real parts of 2^nb entries
  double* bufy = bufx + (1u << nb);                              // imaginary parts
  double2* cs = lds + (1u << nb);                                // [nops][2] the angles' two numbers
  unsigned* lph = reinterpret_cast<unsigned*>(cs + 2 * nops);        // [P + 1] phases (16 words each)
  int2* lop = reinterpret_cast<int2*>(lph + 16 * (P + 1));       // [nops] (code, mat)
  double* red = reinterpret_cast<double*>(lop + nops);           // [8]
  int4* lterm = reinterpret_cast<int4*>(red + 8);                // [kRegTerms] Hamiltonian terms
  double* gpart = reinterpret_cast<double*>(lterm + kRegTerms);  // [nslots][NW][4]
  // The program is copied to LDS once: read op by op through the scalar cache
  // it would be a chain of misses (0.7 us per op).
  static_assert(sizeof(RbPhase) == 64, "16 words");
  for (int i = tid; i < 16 * (P + 1); i += nt) lph[i] = reinterpret_cast<const unsigned*>(phases)[i];
  for (int i = tid; i < nops; i += nt) lop[i] = *reinterpret_cast<const int2*>(ops + i);
  Amp8 p, l;
  auto write = [&](const Amp8& v, const RegMap& m) {
    const unsigned t = thread_slot(tid, m);
    if (!live) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bufx[t ^ register_slot(j, m)] = v.x[j];
      bufy[t ^ register_slot(j, m)] = v.y[j];
    }
  };
  auto read = [&](Amp8& v, const RegMap& m) {
    const unsigned t = thread_slot(tid, m);
    if (!live) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v.x[j] = bufx[t ^ register_slot(j, m)];
      v.y[j] = bufy[t ^ register_slot(j, m)];
    }
  };
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    const double* th = theta + (size_t)b * nparams;
    __syncthreads();   // the previous vector's readers of cs, buf and gpart are done
    for (int i = tid; i < 2 * nops; i += nt) stage_angle(cs, i, ops[i >> 1], th);
#pragma unroll
    for (int j = 0; j < 8; ++j) p.x[j] = p.y[j] = 0.0;
    if (tid == 0) p.x[0] = 1.0;
    __syncthreads();
    // phase words: op_begin, op_count and flags, wr_t (5), wr_r (2), rd_t (5), rd_r (2)
    double none = 0.0;
    int2 od = lop[0];
    vd2 a = ld(cs), az = ld(cs + 1);
    for (int pi = 0; pi < P; ++pi) {
      const unsigned* ph = lph + 16 * pi;
      const int begin = (int)uni(ph[0]), cf = (int)uni(ph[1]);
      const int count = cf >> kRbFlagBits;
      if (pi > 0) {
        const RegMap wr = reg_map(ph + 2), rd = reg_map(ph + 9);
        write(p, wr);
        exchange_barrier((cf & kRbBarrierInside) != 0);
        read(p, rd);
      }
      for (int i = begin; i < begin + count; ++i) {   // the next op is read while this one runs
        const int in = i + 1 < nops ? i + 1 : 0;
        const int2 odn = lop[in];
        const vd2 an = ld(cs + 2 * in), azn = ld(cs + 2 * in + 1);
        const int code = (int)uni((unsigned)od.x) & 31;
        rv_apply<false>(code, p, l, a, az, fixed + 8 * (int)uni((unsigned)od.y), none, none);
        od = odn;
        a = an;
        az = azn;
      }
    }
    // lambda = H phi and E = Re <phi|lambda>: every register's partners are in buf
#pragma unroll
    for (int j = 0; j < 8; ++j) l.x[j] = l.y[j] = 0.0;
    {
      const RegMap wr = reg_map(lph + 16 * P + 2), en = reg_map(lph + 16 * P + 9);
      write(p, wr);
      __syncthreads();
      const unsigned et = thread_slot(tid, en);
      double e = 0.0;
      for (int t0 = 0; t0 < nterms; t0 += kRegTerms) {   // terms through LDS, kRegTerms at a time
        const int cnt = min(kRegTerms, nterms - t0);
        if (t0 > 0) __syncthreads();
        for (int i = tid; i < cnt; i += nt) {
          const VqeTerm T = terms[t0 + i];
          const double tc = coeffs ? coeffs[(size_t)b * nterms + t0 + i] : T.c;
          lterm[i] = make_int4(__double2loint(tc), __double2hiint(tc), (int)((unsigned)T.x | ((unsigned)T.z << 16)), T.y);
        }
        __syncthreads();
        if (!live) continue;
        int4 w = lterm[0];
        for (int t = 0; t < cnt; ++t) {
          const int4 wn = lterm[t + 1 < cnt ? t + 1 : t];
          const unsigned x = uni((unsigned)w.z) & 0xFFFFu, z = uni((unsigned)w.z) >> 16;
          const int y = (int)uni((unsigned)w.w) & 3;
          const double tc = __hiloint2double(w.y, w.x);
          w = wn;
          // signs (-1)^{|k & z|} of the entries k = e ^ x, e this register's: the
          // thread's part once, the registers' parts uniform (parities are linear)
          const double tp = (((unsigned)__popc((et ^ x) & z) ^ ((unsigned)y >> 1)) & 1u) ? -tc : tc;
          auto sign = [&](int j) { return (__popc(register_slot(j, en) & z) & 1) ? -tp : tp; };
          if (x == 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              l.x[j] = fma(sign(j), p.x[j], l.x[j]);
              l.y[j] = fma(sign(j), p.y[j], l.y[j]);
            }
            continue;
          }
          const unsigned lx = slot8(et ^ x);
          double vx[8], vy[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const unsigned sl = lx ^ slot8(register_slot(j, en));
            vx[j] = bufx[sl];
            vy[j] = bufy[sl];
          }
          if (y & 1) {   // i^y: 1, i, -1, -i
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              l.x[j] = fma(-sign(j), vy[j], l.x[j]);
              l.y[j] = fma(sign(j), vx[j], l.y[j]);
            }
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              l.x[j] = fma(sign(j), vx[j], l.x[j]);
              l.y[j] = fma(sign(j), vy[j], l.y[j]);
            }
          }
        }
      }
      if (live) {
#pragma unroll
        for (int j = 0; j < 8; ++j) e += p.x[j] * l.x[j] + p.y[j] * l.y[j];
      }
      e = wave_sum_full(e);
      if (lane == 0) red[wave] = e;
      __syncthreads();
      if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < NW; ++w) s += red[w];
        E[b] = s;
      }
    }
    if (!grad) continue;
    if (nops > 0) {
      od = lop[nops - 1];
      a = ld(cs + 2 * nops - 2);
      az = ld(cs + 2 * nops - 1);
    }
    for (int pi = P - 1; pi >= 0; --pi) {
      const unsigned* ph = lph + 16 * pi;
      const int begin = (int)uni(ph[0]), cf = (int)uni(ph[1]);
      const int count = cf >> kRbFlagBits;
      for (int i = begin + count - 1; i >= begin; --i) {
        const int in = i > 0 ? i - 1 : 0;
        const int2 odn = lop[in];
        const vd2 an = ld(cs + 2 * in), azn = ld(cs + 2 * in + 1);
        const int word = (int)uni((unsigned)od.x), mat = (int)uni((unsigned)od.y);
        double g = 0.0, gz = 0.0;
        rv_apply<true>(word & 31, p, l, a, az, fixed + 8 * mat, g, gz);
        // sums over the 16 lanes of each row; the rows and waves are added at the end
        if (word >= 32) {
          g = row_sum(g);
          if ((lane & 15) == 0) gpart[(((word >> 5) - 1) * NW + wave) * 4 + (lane >> 4)] = g;
        }
        if ((word & 31) >= RV_YZ) {
          gz = row_sum(gz);
          if ((lane & 15) == 0) gpart[(mat * NW + wave) * 4 + (lane >> 4)] = gz;
        }
        od = odn;
        a = an;
        az = azn;
      }
      if (pi > 0) {   // back through the exchange that led into this phase
        const RegMap wr = reg_map(ph + 9), rd = reg_map(ph + 2);
        const bool across = (cf & kRbBarrierInside) != 0;
        write(p, wr);
        exchange_barrier(across);
        read(p, rd);
        exchange_barrier(across);
        write(l, wr);
        exchange_barrier(across);
        read(l, rd);
      }
    }
    __syncthreads();
    for (int q = tid; q < nparams; q += nt) {
      double v = 0.0;
      for (int i = poff[q]; i < poff[q + 1]; ++i)
        for (int w = 0; w < 4 * NW; ++w) v += gpart[pslots[i] * 4 * NW + w];
      grad[(size_t)b * nparams + q] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// Global per-gate kernels: grid (blocks per state, B)
// ---------------------------------------------------------------------------
constexpr int kVqeBlock = 256;

__global__ __launch_bounds__(kVqeBlock) void k_vqe_init(double2* __restrict__ phi, int n) {
  const unsigned long long N = 1ull << n;
  double2* v = phi + (size_t)blockIdx.y * N;
  for (unsigned long long j = (unsigned long long)blockIdx.x * kVqeBlock + threadIdx.x; j < N;
       j += (unsigned long long)gridDim.x * kVqeBlock)
    v[j] = make_double2(j == 0 ? 1.0 : 0.0, 0.0);
}

// Grid-stride loops of the per-gate kernels take kU groups per thread per
// step, all loads issued before the arithmetic; the tail takes one.
constexpr int kU = 4;

__device__ __forceinline__ void pairs_apply_g(double2* v, unsigned long long N, int q, const M2& m,
                                              unsigned long long tid, unsigned long long nt) {
  const unsigned long long off = 1ull << q, np = N >> 1;
  unsigned long long p = tid;
  for (; p + (kU - 1) * nt < np; p += kU * nt) {
    unsigned long long i0[kU];
    vd2 a[kU], b[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      i0[u] = ins0l(p + u * nt, q);
      a[u] = ld(v + i0[u]);
      b[u] = ld(v + i0[u] + off);
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      st(v + i0[u], cfma(m.m0, a[u], cmul(m.m1, b[u])));
      st(v + i0[u] + off, cfma(m.m2, a[u], cmul(m.m3, b[u])));
    }
  }
  for (; p < np; p += nt) {
    const unsigned long long i0 = ins0l(p, q);
    const vd2 a = ld(v + i0), b = ld(v + i0 + off);
    st(v + i0, cfma(m.m0, a, cmul(m.m1, b)));
    st(v + i0 + off, cfma(m.m2, a, cmul(m.m3, b)));
  }
}

__global__ __launch_bounds__(kVqeBlock) void k_vqe_gate(double2* __restrict__ states, int n, VqeOp op,
                                                        const double2* __restrict__ fixed,
                                                        const double* __restrict__ theta, int P, int dag) {
  const unsigned long long N = 1ull << n;
  double2* v = states + (size_t)blockIdx.y * N;
  const double* th = theta + (size_t)blockIdx.y * P;
  const unsigned long long tid = (unsigned long long)blockIdx.x * kVqeBlock + threadIdx.x;
  const unsigned long long nt = (unsigned long long)gridDim.x * kVqeBlock;
  switch (op.kind) {
    case OP_ROT:
      pairs_apply_g(v, N, op.q0, rot_matrix(op.axis, th[op.param], dag != 0), tid, nt);
      break;
    case OP_FIX1:
      pairs_apply_g(v, N, op.q0, fixed_matrix(op.mat, fixed, dag != 0), tid, nt);
      break;
    case OP_RZZ: {
      vd2 e, o;
      rzz_phases(th[op.param], dag != 0, e, o);
      unsigned long long j = tid;
      for (; j + (kU - 1) * nt < N; j += kU * nt) {
        vd2 x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) x[u] = ld(v + j + u * nt);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const unsigned long long i = j + u * nt;
          const unsigned par = (unsigned)(((i >> op.q0) ^ (i >> op.q1)) & 1ull);
          st(v + i, cmul(par ? o : e, x[u]));
        }
      }
      for (; j < N; j += nt) {
        const unsigned par = (unsigned)(((j >> op.q0) ^ (j >> op.q1)) & 1ull);
        st(v + j, cmul(par ? o : e, ld(v + j)));
      }
      break;
    }
    case OP_CZ: {   // negate the quarter with both bits set
      const int lo = min(op.q0, op.q1), hi = max(op.q0, op.q1);
      const unsigned long long o11 = (1ull << op.q0) + (1ull << op.q1);
      for (unsigned long long p = tid; p < (N >> 2); p += nt) {
        const unsigned long long i = ins0l(ins0l(p, lo), hi) + o11;
        const vd2 x = ld(v + i);
        st(v + i, mk(-x.x, -x.y));
      }
      break;
    }
    default: {
      const int lo = min(op.q0, op.q1), hi = max(op.q0, op.q1);
      const unsigned long long oa = 1ull << op.q0;
      const unsigned long long ob = op.kind == OP_CX ? (1ull << op.q0) + (1ull << op.q1) : (1ull << op.q1);
      const unsigned long long nq = N >> 2;
      unsigned long long p = tid;
      for (; p + (kU - 1) * nt < nq; p += kU * nt) {
        unsigned long long b[kU];
        vd2 x[kU], y[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          b[u] = ins0l(ins0l(p + u * nt, lo), hi);
          x[u] = ld(v + b[u] + oa);
          y[u] = ld(v + b[u] + ob);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          st(v + b[u] + oa, y[u]);
          st(v + b[u] + ob, x[u]);
        }
      }
      for (; p < nq; p += nt) {
        const unsigned long long b = ins0l(ins0l(p, lo), hi);
        const vd2 x = ld(v + b + oa), y = ld(v + b + ob);
        st(v + b + oa, y);
        st(v + b + ob, x);
      }
      break;
    }
  }
}

// lambda = H phi, energy partials epart[b * G + block]
__global__ __launch_bounds__(kVqeBlock) void k_vqe_hphi(const double2* __restrict__ phi, double2* __restrict__ lam,
                                                        int n, const VqeTerm* __restrict__ terms, int nterms,
                                                        const double* __restrict__ coeffs,
                                                        double* __restrict__ epart, int store_lam) {
  __shared__ double red[kVqeBlock / kWave];
  const unsigned long long N = 1ull << n;
  const double2* p = phi + (size_t)blockIdx.y * N;
  double2* l = lam + (size_t)blockIdx.y * N;
  double e = 0.0;
  for (unsigned long long j = (unsigned long long)blockIdx.x * kVqeBlock + threadIdx.x; j < N;
       j += (unsigned long long)gridDim.x * kVqeBlock) {
    const vd2 h = h_apply_at(p, j, terms, nterms, coeffs ? coeffs + (size_t)blockIdx.y * nterms : nullptr);
    const vd2 v = ld(p + j);
    e += v.x * h.x + v.y * h.y;
    if (store_lam) st(l + j, h);
  }
  e = wave_sum(e);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = e;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kVqeBlock / kWave; ++w) s += red[w];
    epart[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
  }
}

// ---------------------------------------------------------------------------
// lambda = H phi over tiles staged in LDS (fused schedule).  A pass takes a
// tile shape (low c bits plus m high bits) and the terms whose flipped bits
// x lie inside it; the first pass also takes every diagonal term (x = 0) and
// writes lambda, later passes add to it.  For entry j of a tile (local index
// l) a term contributes c_t i^y (-1)^{|(j ^ x) & z|} phi[j ^ x], with the
// partner read from the tile; the sign splits into the tile-local bits
// (|(l ^ xl) & zl|) and a per-tile constant (|base & zo| + |x & z|, on the
// bits outside the tile).  The last pass also sums Re<phi|lambda> into the
// energy partial of its workgroup.  Terms whose flipped bits fit no tile
// take a gather pass of their own (k_vqe_hphi_wide).
// ---------------------------------------------------------------------------
constexpr int kHBlock = 512;      // threads per tile workgroup
constexpr int kHTileBits = 12;    // tiles of at most 2^12 entries: two workgroups per CU, one loads while one sums
constexpr int kHLow = 4;          // low bits of the later passes' tiles (8 high bits each)
constexpr int kHPer = (1 << kHTileBits) / kHBlock;
constexpr int kHMaxTerms = 128;   // terms per launch

struct HTerm {
  unsigned xl, zl;            // x and the z bits inside the tile, tile-local
  unsigned long long zo;      // z bits outside the tile (global)
  int y;                      // popcount(x & z) mod 4 (the i^y factor)
  int sx;                     // popcount(x & z) mod 2 (the sign of (j ^ x) vs j)
  int t;                      // index of the term (its coefficient)
  int pad;
};
struct HPass {
  int c, m;
  int hi[8];
  int first, last;
  int t_begin, n_diag, n_flip;   // diagonal terms first, then flipped ones
  int pad;
};

// Bound by the streams: 256 vectors of 20 qubits, Ising chain, 2.08 ms for the
// first pass (12 bits, 19 + 12 terms; 4.1 TB/s) and 2.36 for the second (8
// bits; 5.5 TB/s).  Tiles of 2^13, one workgroup per CU that loads or sums, with
// a select per term and entry, took 3.69 and 4.40.
template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kHBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_vqe_hphi_tile(
                                                           const double2* __restrict__ phi0, double2* __restrict__ lam0,
                                                           int n, HPass ps, const HTerm* __restrict__ hterms,
                                                           const VqeTerm* __restrict__ terms, int nterms,
                                                           const double* __restrict__ coeffs,
                                                           double* __restrict__ epart) {
  extern __shared__ double2 tl[];
  __shared__ double s_c[kHMaxTerms];
  __shared__ double red[kHBlock / kWave];
  const unsigned long long N = 1ull << n;
  const double2* __restrict__ phi = phi0 + (size_t)blockIdx.y * N;
  double2* __restrict__ lam = lam0 + (size_t)blockIdx.y * N;
  const int k = ps.c + ps.m;
  const unsigned len = 1u << k;
  const unsigned long long ntiles = 1ull << (n - k);
  const unsigned tid = threadIdx.x;
  const int nt = ps.n_diag + ps.n_flip;
  for (int i = tid; i < nt; i += kHBlock) {
    const int t = hterms[ps.t_begin + i].t;
    s_c[i] = coeffs ? coeffs[(size_t)blockIdx.y * nterms + t] : terms[t].c;
  }
  // Entry r of this thread is tile entry l = tid + r kHBlock; its global
  // index is the tile base plus the thread's part and a uniform part.
  auto scatter = [&](unsigned l) {
    unsigned long long gi = l & ((1u << ps.c) - 1u);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < ps.m && ((l >> (ps.c + i)) & 1u)) gi |= 1ull << ps.hi[i];
    return gi;
  };
  const unsigned long long own = scatter(tid);
  static_assert(kHPer == 8, "three register bits");
  constexpr int kHShift = 9;
  static_assert(1 << kHShift == kHBlock, "register bits above the thread's");
  double e = 0.0;
  for (unsigned long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    unsigned long long base = tile << ps.c;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i < ps.m) {
        const int q = ps.hi[i];
        base = ((base >> q) << (q + 1)) | (base & ((1ull << q) - 1ull));
      }
    }
    vd2 v[kHPer];
    double ax[kHPer], ay[kHPer];
#pragma unroll
    for (int r = 0; r < kHPer; ++r) {
      v[r] = mk(0.0, 0.0);
      vd2 a = mk(0.0, 0.0);
      if (tid + r * kHBlock < len) {
        const unsigned long long at = (base | scatter(r * kHBlock)) | own;
        v[r] = __builtin_nontemporal_load(reinterpret_cast<const vd2*>(phi + at));
        if (!FIRST) a = __builtin_nontemporal_load(reinterpret_cast<const vd2*>(lam + at));
      }
      ax[r] = a.x;
      ay[r] = a.y;
    }
    __syncthreads();   // the previous tile's readers are done (and s_c is written)
#pragma unroll
    for (int r = 0; r < kHPer; ++r)
      if (tid + r * kHBlock < len) st(tl + tid + r * kHBlock, v[r]);
    __syncthreads();
    // The sign of a term at entry l: the parity of (l & zl) splits into the
    // thread's bits (tid & zl) and the entry slot's (r kHBlock & zl); the bits
    // outside the tile (base & zo) and x & z are per tile and term.
    if (ps.n_diag > 0) {
      // the coefficients by their sign pattern over r, then one Walsh-Hadamard
      // transform: an add per term and thread, not one per entry
      double d[kHPer];
#pragma unroll
      for (int r = 0; r < kHPer; ++r) d[r] = 0.0;
      for (int i = 0; i < ps.n_diag; ++i) {
        const HTerm T = hterms[ps.t_begin + i];
        const unsigned pb = (unsigned)(__builtin_popcountll(base & T.zo) + __popc(tid & T.zl)) & 1u;
        const double c = pb ? -s_c[i] : s_c[i];
#define NWQ_HD(I) \
  case I: d[I] += c; asm volatile("" : "+v"(d[I])); break;
        switch ((T.zl >> kHShift) & 7u) {
          NWQ_HD(0) NWQ_HD(1) NWQ_HD(2) NWQ_HD(3) NWQ_HD(4) NWQ_HD(5) NWQ_HD(6) NWQ_HD(7)
        }
#undef NWQ_HD
      }
#pragma unroll
      for (int h = 1; h < kHPer; h <<= 1)
#pragma unroll
        for (int r = 0; r < kHPer; ++r)
          if (!(r & h)) {
            const double a = d[r], b = d[r | h];
            d[r] = a + b;
            d[r | h] = a - b;
          }
#pragma unroll
      for (int r = 0; r < kHPer; ++r) {
        ax[r] = fma(d[r], v[r].x, ax[r]);
        ay[r] = fma(d[r], v[r].y, ay[r]);
      }
    }
    for (int i = ps.n_diag; i < nt; ++i) {
      const HTerm T = hterms[ps.t_begin + i];
      // i^y: 1, i, -1, -i; the sign of 2 and 3 with the others
      const unsigned pb = (unsigned)(__builtin_popcountll(base & T.zo) + __popc(tid & T.zl) + T.sx + (T.y >> 1)) & 1u;
      const double c = pb ? -s_c[i] : s_c[i];
      const unsigned at = tid ^ (T.xl & (kHBlock - 1)), xr = T.xl >> kHShift, zr = (T.zl >> kHShift) & 7u;
      vd2 p[kHPer];
#pragma unroll
      for (int r = 0; r < kHPer; ++r) p[r] = ld(tl + ((at + (((unsigned)r ^ xr) << kHShift)) & (len - 1u)));
      auto cf = [&](int r) {   // the slot's sign is uniform
        const unsigned sg = (unsigned)(__builtin_popcount(r & zr) & 1) << 31;
        return __hiloint2double((int)((unsigned)__double2hiint(c) ^ sg), __double2loint(c));
      };
      if (T.y & 1) {
#pragma unroll
        for (int r = 0; r < kHPer; ++r) {
          ax[r] = fma(-cf(r), p[r].y, ax[r]);
          ay[r] = fma(cf(r), p[r].x, ay[r]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < kHPer; ++r) {
          ax[r] = fma(cf(r), p[r].x, ax[r]);
          ay[r] = fma(cf(r), p[r].y, ay[r]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kHPer; ++r) {
      if (tid + r * kHBlock >= len) continue;
      __builtin_nontemporal_store(mk(ax[r], ay[r]),
                                  reinterpret_cast<vd2*>(lam + ((base | scatter(r * kHBlock)) | own)));
      if (LAST) {   // from LDS again: held in registers it spills
        const vd2 a = ld(tl + tid + r * kHBlock);
        e += a.x * ax[r] + a.y * ay[r];
      }
    }
  }
  if (LAST) {
    e = wave_sum_full(e);
    if ((tid & (kWave - 1)) == 0) red[tid / kWave] = e;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < kHBlock / kWave; ++w) s += red[w];
      epart[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
  }
}

// Terms whose flipped bits span more high bits than a tile holds: partners
// gathered from global memory (as k_vqe_hphi), added to lambda (written on
// the first pass); the last pass also sums the energy partials.
template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kVqeBlock) void k_vqe_hphi_wide(const double2* __restrict__ phi0, double2* __restrict__ lam0,
                                                             int n, const VqeTerm* __restrict__ terms,
                                                             const int* __restrict__ tidx, int cnt, int nterms,
                                                             const double* __restrict__ coeffs,
                                                             double* __restrict__ epart) {
  __shared__ double red[kVqeBlock / kWave];
  const unsigned long long N = 1ull << n;
  const double2* __restrict__ p = phi0 + (size_t)blockIdx.y * N;
  double2* __restrict__ l = lam0 + (size_t)blockIdx.y * N;
  const double* cb = coeffs ? coeffs + (size_t)blockIdx.y * nterms : nullptr;
  double e = 0.0;
  for (unsigned long long j = (unsigned long long)blockIdx.x * kVqeBlock + threadIdx.x; j < N;
       j += (unsigned long long)gridDim.x * kVqeBlock) {
    vd2 acc = FIRST ? mk(0.0, 0.0) : ld(l + j);
    for (int i = 0; i < cnt; ++i) {
      const int t = tidx[i];
      const VqeTerm T = terms[t];
      const double tc = cb ? cb[t] : T.c;
      const unsigned long long k = j ^ T.x;
      vd2 v = ld(p + k);
      switch (T.y & 3) {
        case 1: v = mk(-v.y, v.x); break;
        case 2: v = mk(-v.x, -v.y); break;
        case 3: v = mk(v.y, -v.x); break;
        default: break;
      }
      const double c = (__popcll(k & T.z) & 1) ? -tc : tc;
      acc.x = fma(c, v.x, acc.x);
      acc.y = fma(c, v.y, acc.y);
    }
    st(l + j, acc);
    if (LAST) {
      const vd2 v = ld(p + j);
      e += v.x * acc.x + v.y * acc.y;
    }
  }
  if (LAST) {
    e = wave_sum(e);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int w = 0; w < kVqeBlock / kWave; ++w) s += red[w];
      epart[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
  }
}

// Backward step over all states; gradient partials gpart[(b * nslots + slot) * G + block]
__global__ __launch_bounds__(kVqeBlock) void k_vqe_adjoint(double2* __restrict__ phi, double2* __restrict__ lam,
                                                           int n, VqeOp op, const double2* __restrict__ fixed,
                                                           const double* __restrict__ theta, int P, int nslots,
                                                           double* __restrict__ gpart) {
  __shared__ double red[kVqeBlock / kWave];
  const unsigned long long N = 1ull << n;
  double2* pv = phi + (size_t)blockIdx.y * N;
  double2* lv = lam + (size_t)blockIdx.y * N;
  const double* th = theta + (size_t)blockIdx.y * P;
  const unsigned long long tid = (unsigned long long)blockIdx.x * kVqeBlock + threadIdx.x;
  const unsigned long long nt = (unsigned long long)gridDim.x * kVqeBlock;
  double g = 0.0;
  if (op.kind == OP_ROT) {
    const M2 m = rot_matrix(op.axis, th[op.param], true);
    const unsigned long long off = 1ull << op.q0, np = N >> 1;
    unsigned long long p = tid;
    // kU pairs per step; the gradient terms are added in pair order
    for (; p + (kU - 1) * nt < np; p += kU * nt) {
      unsigned long long i0[kU];
      vd2 p0[kU], p1[kU], l0[kU], l1[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        i0[u] = ins0l(p + u * nt, op.q0);
        p0[u] = ld(pv + i0[u]);
        p1[u] = ld(pv + i0[u] + off);
        l0[u] = ld(lv + i0[u]);
        l1[u] = ld(lv + i0[u] + off);
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        g += pair_grad(op.axis, p0[u], p1[u], l0[u], l1[u]);
        st(pv + i0[u], cfma(m.m0, p0[u], cmul(m.m1, p1[u])));
        st(pv + i0[u] + off, cfma(m.m2, p0[u], cmul(m.m3, p1[u])));
        st(lv + i0[u], cfma(m.m0, l0[u], cmul(m.m1, l1[u])));
        st(lv + i0[u] + off, cfma(m.m2, l0[u], cmul(m.m3, l1[u])));
      }
    }
    for (; p < np; p += nt) {
      const unsigned long long i0 = ins0l(p, op.q0);
      const vd2 p0 = ld(pv + i0), p1 = ld(pv + i0 + off);
      const vd2 l0 = ld(lv + i0), l1 = ld(lv + i0 + off);
      g += pair_grad(op.axis, p0, p1, l0, l1);
      st(pv + i0, cfma(m.m0, p0, cmul(m.m1, p1)));
      st(pv + i0 + off, cfma(m.m2, p0, cmul(m.m3, p1)));
      st(lv + i0, cfma(m.m0, l0, cmul(m.m1, l1)));
      st(lv + i0 + off, cfma(m.m2, l0, cmul(m.m3, l1)));
    }
  } else {   // OP_RZZ
    vd2 e, o;
    rzz_phases(th[op.param], true, e, o);
    unsigned long long j = tid;
    for (; j + (kU - 1) * nt < N; j += kU * nt) {
      vd2 x[kU], y[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        x[u] = ld(pv + j + u * nt);
        y[u] = ld(lv + j + u * nt);
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const unsigned long long i = j + u * nt;
        const unsigned par = (unsigned)(((i >> op.q0) ^ (i >> op.q1)) & 1ull);
        const double t = y[u].x * x[u].y - y[u].y * x[u].x;
        g += par ? -t : t;
        st(pv + i, cmul(par ? o : e, x[u]));
        st(lv + i, cmul(par ? o : e, y[u]));
      }
    }
    for (; j < N; j += nt) {
      const unsigned par = (unsigned)(((j >> op.q0) ^ (j >> op.q1)) & 1ull);
      const vd2 p = ld(pv + j), l = ld(lv + j);
      const double t = l.x * p.y - l.y * p.x;
      g += par ? -t : t;
      st(pv + j, cmul(par ? o : e, p));
      st(lv + j, cmul(par ? o : e, l));
    }
  }
  g = wave_sum(g);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = g;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kVqeBlock / kWave; ++w) s += red[w];
    gpart[((size_t)blockIdx.y * nslots + op.slot) * gridDim.x + blockIdx.x] = s;
  }
}

// Closing reductions in a fixed order that depends only on G: each slot's G
// gradient partials are summed by one wave (lanes stride over the partials,
// then a fixed shuffle tree) into ssum; then one workgroup per state sums
// the energy partials the same way and each parameter adds its slots in slot
// order.
constexpr int kFinBlock = 256;

// Slot sums: workgroup (chunk, b) gives one slot to each wave.
__global__ __launch_bounds__(kFinBlock) void k_vqe_slot_sums(const double* __restrict__ gpart, int G, int nslots,
                                                             double* __restrict__ ssum) {
  const int b = blockIdx.y;
  const int lane = threadIdx.x & (kWave - 1);
  const int s = blockIdx.x * (kFinBlock / kWave) + threadIdx.x / kWave;
  if (s >= nslots) return;
  const double* gp = gpart + ((size_t)b * nslots + s) * G;
  double v = 0.0;
  for (int k = lane; k < G; k += kWave) v += gp[k];
  v = wave_sum(v);
  if (lane == 0) ssum[(size_t)b * nslots + s] = v;
}

__global__ __launch_bounds__(kFinBlock) void k_vqe_finish(const double* __restrict__ epart, int G, int nslots,
                                                          const int* __restrict__ slot_param, int P,
                                                          const double* __restrict__ ssum, double* __restrict__ E,
                                                          double* __restrict__ grad) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (wave == 0) {
    double e = 0.0;
    for (int k = lane; k < G; k += kWave) e += epart[(size_t)b * G + k];
    e = wave_sum(e);
    if (lane == 0) E[b] = e;
  }
  if (!grad) return;
  for (int p = threadIdx.x; p < P; p += kFinBlock) {
    double g = 0.0;
    for (int s = 0; s < nslots; ++s)
      if (slot_param[s] == p) g += ssum[(size_t)b * nslots + s];
    grad[(size_t)b * P + p] = g;
  }
}

}  // namespace

namespace {
// ---------------------------------------------------------------------------
// Fused path (any n > tile): gates grouped into k-qubit blocks as for state
// vectors; the forward pass runs the register-blocked fused kernel over all
// B states with a per-vector matrix table, the backward pass holds tiles of
// phi and lambda in registers and sweeps each block's gates in reverse.
// ---------------------------------------------------------------------------
// Per-vector matrix table of the forward pass: entries [4i, 4i+4) hold op i's
// matrix (2x2 row-major, or the 4 diagonal entries of RZZ / CZ indexed by
// u = bit q0 + 2 bit q1).  Every case stores inside its own branch.
__global__ __launch_bounds__(256) void k_vqe_mats(const VqeOp* __restrict__ ops, int nops,
                                                  const double2* __restrict__ fixed,
                                                  const double* __restrict__ theta, int P,
                                                  double2* __restrict__ table) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= nops) return;
  const int b = blockIdx.y;
  const VqeOp op = ops[i];
  const double* th = theta + (size_t)b * P;
  double2* t = table + ((size_t)b * nops + i) * 4;
  if (op.kind == OP_ROT) {
    const M2 f = rot_matrix(op.axis, th[op.param], false);
    st(t + 0, f.m0); st(t + 1, f.m1); st(t + 2, f.m2); st(t + 3, f.m3);
  } else if (op.kind == OP_RZZ) {
    vd2 e, o;
    rzz_phases(th[op.param], false, e, o);
    st(t + 0, e); st(t + 1, o); st(t + 2, o); st(t + 3, e);
  } else if (op.kind == OP_FIX1) {
    for (int k = 0; k < 4; ++k) t[k] = fixed[8 * op.mat + k];
  } else if (op.kind == OP_CZ) {
    for (int k = 0; k < 4; ++k) st(t + k, mk(k == 3 ? -1.0 : 1.0, 0.0));
  } else {
    for (int k = 0; k < 4; ++k) st(t + k, mk(0.0, 0.0));
  }
}

// Backward block, register-blocked: a tile of phi and of lambda, 8 amplitudes of
// each per thread on three register bits, ops as in k_vqe_reg (RY and RX three
// shears, RZ after RY in one op, gradients in four chains).  Tiles come from HBM
// straight into registers and pass through LDS one component at a time; waves
// whose phases share the tile bits on their index do not wait for each other.
// The block's program and angles are staged in LDS, and each slot keeps a sum
// per wave and row of 16 lanes there (each written by one lane, so the order of
// additions is fixed).
//
// What bounds it: half HBM (two states read and written: 2.6 of 4.03 ms per
// block of 256 vectors of 20 qubits), half FP64 issue at four waves per SIMD;
// three waves per SIMD (no spill of 20 bytes) or tiles of 2^12 are slower
// (20 qubits, L = 8: 54.8, 56.8 and 58.0 ms per batch).  The kernel before took
// whole amplitudes through LDS with both states' next tile in registers (204
// VGPRs, two waves per SIMD): 6.28 ms per block, 73 ms per batch.
// Gradients against 80-bit arithmetic: 9.4e-16 off on 13 qubits, L = 4, and
// 8.4e-16 on 20, L = 1 (with that kernel 1.11e-15 and 1.22e-15).
constexpr int kBwdMaxTileBits = 11;   // 256 threads
constexpr int kBwdRegOps = 128;       // LDS: 4 KB of angles, 16 KB of gradient sums

// Global loads and stores of tile entries; NT: non-temporal (each entry of
// phi and lambda is read and written once per block).
template <bool NT>
__device__ __forceinline__ vd2 bgld(const double2* p) {
  if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const vd2*>(p));
  else return ld(p);
}
template <bool NT>
__device__ __forceinline__ void bgst(double2* p, vd2 v) {
  if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<vd2*>(p));
  else st(p, v);
}
// XOR of the images of the set bits of v.
__device__ __forceinline__ unsigned long long image_of(unsigned v, const unsigned long long* img, int bits) {
  unsigned long long x = 0;
#pragma unroll
  for (int i = 0; i < bits; ++i) x ^= (unsigned long long)(long long)((int)(v << (31 - i)) >> 31) & img[i];
  return x;
}

// LDS of a block: the exchange buffer, angles, phases, ops, sums.
inline size_t bwd_reg_lds(int k, int phases, int nops, int nlocal) {
  const int nw = std::max(1, (1 << (k - 3)) / kWave);
  return (sizeof(double) << k) + (size_t)nops * (2 * sizeof(double2) + sizeof(int2)) + (size_t)phases * sizeof(RbPhase) +
         (size_t)nlocal * nw * 4 * sizeof(double) + 64;
}

template <bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_vqe_bwd_reg(
    double2* __restrict__ phi0, double2* __restrict__ lam0, int n, RbBlock blk, const RbPhase* __restrict__ phases,
    const RegOpV* __restrict__ ops, int nops, const int* __restrict__ slots, int nlocal,
    const double2* __restrict__ fixed, const double* __restrict__ theta, int nparams, int nslots,
    double* __restrict__ gpart, unsigned long long ntiles, unsigned long long mask, unsigned long long step) {
  extern __shared__ double2 lds[];
  const unsigned tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave, NW = (int)(nt + kWave - 1) / kWave, P = blk.ph_count;
  double* buf = reinterpret_cast<double*>(lds);                      // one component of the tile
  double2* cs = lds + (1u << (blk.k - 1));                           // [nops][2] the angles' two numbers
  unsigned* lph = reinterpret_cast<unsigned*>(cs + 2 * nops);        // [P] phases (16 words each)
  int2* lop = reinterpret_cast<int2*>(lph + 16 * P);                 // [nops] (code, mat)
  double* gacc = reinterpret_cast<double*>(lop + nops);              // [nlocal][NW][4]
  double2* __restrict__ phi = phi0 + ((size_t)blockIdx.y << n);
  double2* __restrict__ lam = lam0 + ((size_t)blockIdx.y << n);
  const double* __restrict__ th = theta + (size_t)blockIdx.y * nparams;
  for (int i = tid; i < 16 * P; i += nt) lph[i] = reinterpret_cast<const unsigned*>(phases + blk.ph_begin)[i];
  for (int i = tid; i < nlocal * NW * 4; i += nt) gacc[i] = 0.0;
  for (int i = tid; i < nops; i += nt) lop[i] = *reinterpret_cast<const int2*>(ops + i);
  for (int i = tid; i < 2 * nops; i += nt) stage_angle(cs, i, ops[i >> 1], th);
  Amp8 p, l;
  auto exchange = [&](double (&v)[8], unsigned wt, const RegMap& wr, unsigned rt, const RegMap& rd, bool across) {
#pragma unroll
    for (int j = 0; j < 8; ++j) buf[wt ^ register_slot(j, wr)] = v[j];
    exchange_barrier(across);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = buf[rt ^ register_slot(j, rd)];
  };
  const unsigned long long gl_ld = image_of(tid, blk.ld_t, 8), gl_st = image_of(tid, blk.st_t, 8);
  auto reg_image = [](int j, const unsigned long long* r) {
    return ((j & 1) ? r[0] : 0ull) ^ ((j & 2) ? r[1] : 0ull) ^ ((j & 4) ? r[2] : 0ull);
  };
  __syncthreads();
  unsigned long long tile = blockIdx.x, base = deposit_bits(tile, mask);
  for (; tile < ntiles; tile += gridDim.x, base = ((base | ~mask) + step) & mask) {
    {
      const double2* __restrict__ a = phi + (base | gl_ld);
      const double2* __restrict__ b = lam + (base | gl_ld);
      vd2 v[8], w[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j] = bgld<NT>(a + reg_image(j, blk.ld_r));
        w[j] = bgld<NT>(b + reg_image(j, blk.ld_r));
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        p.x[j] = v[j].x;
        p.y[j] = v[j].y;
        l.x[j] = w[j].x;
        l.y[j] = w[j].y;
      }
    }
    int2 od = lop[0];
    vd2 a = ld(cs), az = ld(cs + 1);
    for (int pi = 0; pi < P; ++pi) {
      const unsigned* ph = lph + 16 * pi;
      const int begin = (int)uni(ph[0]), cf = (int)uni(ph[1]), count = cf >> kRbFlagBits;
      if (pi > 0) {
        const RegMap wr = reg_map(ph + 2), rd = reg_map(ph + 9);
        const unsigned wt = thread_slot(tid, wr), rt = thread_slot(tid, rd);
        const bool across = (cf & kRbBarrierInside) != 0;
        exchange_barrier((cf & kRbBarrierBefore) != 0);
        exchange(p.x, wt, wr, rt, rd, across);
        exchange_barrier(across);
        exchange(p.y, wt, wr, rt, rd, across);
        exchange_barrier(across);
        exchange(l.x, wt, wr, rt, rd, across);
        exchange_barrier(across);
        exchange(l.y, wt, wr, rt, rd, across);
      }
      for (int i = begin; i < begin + count; ++i) {   // the next op is read while this one runs
        const int in = i + 1 < nops ? i + 1 : 0;
        const int2 odn = lop[in];
        const vd2 an = ld(cs + 2 * in), azn = ld(cs + 2 * in + 1);
        const int word = (int)uni((unsigned)od.x), mat = (int)uni((unsigned)od.y);
        double g = 0.0, gz = 0.0;
        rv_apply<true>(word & 31, p, l, a, az, fixed + 8 * mat, g, gz);
        if (word >= 32) {
          g = row_sum(g);
          if ((lane & 15) == 0) gacc[(((word >> 5) - 1) * NW + wave) * 4 + (lane >> 4)] += g;
        }
        if ((word & 31) >= RV_YZ) {
          gz = row_sum(gz);
          if ((lane & 15) == 0) gacc[(mat * NW + wave) * 4 + (lane >> 4)] += gz;
        }
        od = odn;
        a = an;
        az = azn;
      }
    }
    double2* __restrict__ a1 = phi + (base | gl_st);
    double2* __restrict__ b1 = lam + (base | gl_st);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bgst<NT>(a1 + reg_image(j, blk.st_r), mk(p.x[j], p.y[j]));
      bgst<NT>(b1 + reg_image(j, blk.st_r), mk(l.x[j], l.y[j]));
    }
  }
  __syncthreads();
  for (int i = tid; i < nlocal; i += nt) {
    double v = 0.0;
    for (int w = 0; w < 4 * NW; ++w) v += gacc[i * 4 * NW + w];
    gpart[((size_t)blockIdx.y * nslots + slots[i]) * gridDim.x + blockIdx.x] = v;
  }
}

}  // namespace

// ===========================================================================
// Host: context
// ===========================================================================
struct VqeConfig {
  int mode = 0;        // 0 auto, 1 LDS-resident, 2 global per-gate (graph)
  int threads = 256;   // LDS kernel block size
  int blocks_per_state = 0;   // global path: 0 = derived from n
};

}  // namespace nwq

struct nwq_vqe {
  int n = 0, P = 0, nops = 0, nterms = 0, nslots = 0;
  hipStream_t user_stream = nullptr;
  hipStream_t stream = nullptr;       // own stream (graph capture needs a non-null stream)
  hipEvent_t ev_in = nullptr, ev_out = nullptr;
  std::vector<nwq::VqeOp> ops;
  std::vector<int> slot_param;
  nwq::VqeOp* d_ops = nullptr;
  double2* d_fixed = nullptr;
  nwq::VqeTerm* d_terms = nullptr;
  std::vector<nwq::VqeTerm> terms;   // host copy of the term table
  int* d_slot_param = nullptr;
  // register-resident path (n <= 12): phases, ops, parameter slots
  void* d_reg = nullptr;       // part of d_program
  void* d_program = nullptr;   // d_ops, d_fixed, d_terms, d_slot_param and d_reg
  int reg_phases = 0, reg_ops = 0;
  size_t reg_ops_off = 0, reg_poff_off = 0, reg_pslots_off = 0;
  // global path buffers
  int Bcap = 0;
  double2* d_phi = nullptr;
  double2* d_lam = nullptr;
  double* d_epart = nullptr;
  double* d_gpart = nullptr;
  double* d_theta = nullptr;   // staging copies for graph replays
  double* d_E = nullptr;
  double* d_grad = nullptr;
  double* d_coeffs = nullptr;  // staging copy of per-vector coefficients
  double2* d_table = nullptr;  // fused path: per-vector matrix table [B][nops][4]
  double* d_ssum = nullptr;    // per-slot gradient sums [B][nslots]
  // fused path program (built on first use)
  bool fused_built = false;
  int fused_k = 12;
  int low_bits = 0;            // low tile bits of the planned blocks: 0 = kVqeLowBits
  int fused_rbits = 4;         // register bits per phase of the forward kernel
  size_t fused_rop_off = 0, fused_slot_off = 0;   // backward ops and the slots of their gradient sums in d_fused
  // Before a block's gates phi is zero wherever a qubit that no earlier block
  // touched is set, so tiles set on such a qubit (outside the block's own) add
  // nothing to any Im<lambda|P|phi>; the dispatches that follow in the sweep
  // (earlier blocks, smaller supports) read none of them, and neither vector
  // is read after the sweep.  The first planned block runs tile 0 only.
  struct BwdRegBlock {
    nwq::RbBlock d;
    int op0, nops, slot0, nlocal;
    unsigned long long mask;   // index bits outside the tile that its tiles run over
  };
  std::vector<BwdRegBlock> bwd_reg;
  std::vector<nwq::RbBlock> fwd_blocks;
  // lambda = H phi of the fused schedule: tiled passes (and a gather pass for
  // terms that fit no tile), in launch order
  struct HLaunch {
    int wide;            // 1: k_vqe_hphi_wide over the term indices at widx[w_begin .. w_begin + w_count)
    nwq::HPass p;        // tiled pass (p.t_begin indexes the HTerm table)
    int w_begin, w_count;
  };
  std::vector<HLaunch> hlaunch;
  size_t fused_hterm_off = 0, fused_widx_off = 0;
  void* d_fused = nullptr;     // [backward phases][forward phases][forward ops][backward ops][H terms]
  size_t fused_fph_off = 0, fused_ops_off = 0;
  nwq::VqeConfig cfg;
  std::map<std::pair<int, int>, hipGraphExec_t> graphs;   // (B, want_grad) -> exec
  int fused_flags = 3;         // fused schedule: bit 0 non-temporal tile loads and stores, bit 1 direct
                               // HBM loads / stores of a forward block's first / last phase
  size_t program_bytes = 0;    // device bytes of d_program
  size_t fused_bytes = 0;      // device bytes of d_fused once built
};

namespace nwq {

static int vqe_fail(int code, const std::string& m) { return set_error(code, m); }

// Workgroups per state of the per-gate and fused schedules.  The partial
// sums (and so the rounding) depend on it, so it is fixed per context and
// never derived from B; the default fills the chip with one state (up to
// 1024 workgroups of 4 pairs per thread), the batch adds the rest.
static int blocks_per_state(const nwq_vqe* h) {
  if (h->cfg.blocks_per_state > 0) return h->cfg.blocks_per_state;
  const unsigned long long pairs = 1ull << (h->n - 1);
  const unsigned long long b = (pairs + kVqeBlock * 4 - 1) / (kVqeBlock * 4);
  return (int)std::max<unsigned long long>(1, std::min<unsigned long long>(b, 1024));
}

static size_t lds_bytes(const nwq_vqe* h, int threads, bool want_grad) {
  const size_t N = 1ull << h->n;
  const int NW = threads / kWave;
  return (want_grad ? 2 : 1) * N * sizeof(double2) + (size_t)NW * sizeof(double) +
         (want_grad ? (size_t)h->nslots * NW * sizeof(double) : 0);
}

static bool reg_fits(const nwq_vqe* h);
static bool lds_fits(const nwq_vqe* h, int threads, bool want_grad) {
  return h->n <= 12 && (reg_fits(h) || lds_bytes(h, threads, want_grad) <= 160 * 1024);
}

// The register-resident kernel: threads and LDS; its program is built with the
// context for n <= 12.
static int reg_threads(const nwq_vqe* h) { return std::max(kWave, h->n > 3 ? 1 << (h->n - 3) : 1); }
static size_t reg_lds_bytes(const nwq_vqe* h) {
  return (sizeof(double2) << std::max(3, h->n)) + (size_t)h->reg_ops * (2 * sizeof(double2) + sizeof(int2)) +
         (size_t)(h->reg_phases + 1) * sizeof(RbPhase) + kRegTerms * sizeof(int4) +
         (8 + (size_t)h->nslots * 4 * (reg_threads(h) / kWave)) * sizeof(double);
}
static bool reg_fits(const nwq_vqe* h) { return h->d_reg != nullptr && reg_lds_bytes(h) <= 160 * 1024; }

static int launch_reg(nwq_vqe* h, int B, const double* theta, const double* coeffs, double* E, double* grad,
                      hipStream_t s) {
  const size_t lds = reg_lds_bytes(h);
  if (lds > 65536) (void)enable_dynamic_lds((const void*)k_vqe_reg);
  const char* d = static_cast<const char*>(h->d_reg);
  hipLaunchKernelGGL(k_vqe_reg, dim3(std::min(B, 4096)), dim3(reg_threads(h)), lds, s, h->n,
                     reinterpret_cast<const RbPhase*>(d), h->reg_phases,
                     reinterpret_cast<const RegOpV*>(d + h->reg_ops_off), h->reg_ops, h->d_fixed, h->d_terms,
                     h->nterms, h->nslots, reinterpret_cast<const int*>(d + h->reg_poff_off),
                     reinterpret_cast<const int*>(d + h->reg_pslots_off), theta, h->P, B, coeffs, E, grad);
  return check_hip(hipGetLastError(), "k_vqe_reg");
}

static int launch_lds(nwq_vqe* h, int B, const double* theta, const double* coeffs, double* E, double* grad,
                      hipStream_t s) {
  if (reg_fits(h)) return launch_reg(h, B, theta, coeffs, E, grad, s);
  const int T = h->cfg.threads;
  const size_t lds = lds_bytes(h, T, grad != nullptr);
  const int grid = std::min(B, 4096);
#define NWQ_VQE_LDS(NTV)                                                                                     \
  do {                                                                                                       \
    if (lds > 65536) (void)enable_dynamic_lds((const void*)k_vqe_lds<NTV>);                                  \
    hipLaunchKernelGGL(k_vqe_lds<NTV>, dim3(grid), dim3(NTV), lds, s, h->n, h->d_ops, h->nops, h->d_fixed,   \
                       h->d_terms, h->nterms, h->nslots, h->d_slot_param, theta, h->P, B, coeffs, E, grad);  \
  } while (0)
  switch (T) {
    case 64: NWQ_VQE_LDS(64); break;
    case 128: NWQ_VQE_LDS(128); break;
    case 512: NWQ_VQE_LDS(512); break;
    case 1024: NWQ_VQE_LDS(1024); break;
    default: NWQ_VQE_LDS(256); break;
  }
#undef NWQ_VQE_LDS
  return check_hip(hipGetLastError(), "k_vqe_lds");
}

// Device bytes of the global-path buffers per parameter vector (what
// ensure_global allocates for each unit of its capacity).
static size_t global_bytes_per_vector(const nwq_vqe* h) {
  const size_t N = 1ull << h->n;
  const size_t G = (size_t)blocks_per_state(h);
  const size_t P = std::max(1, h->P), S = std::max(1, h->nslots), T = std::max(1, h->nterms), O = std::max(1, h->nops);
  return 2 * N * sizeof(double2) + G * sizeof(double) + S * G * sizeof(double) + 2 * P * sizeof(double) +
         sizeof(double) + T * sizeof(double) + O * 4 * sizeof(double2) + S * sizeof(double);
}

static int ensure_global(nwq_vqe* h, int B) {
  if (B <= h->Bcap) return NWQ_OK;
  int rc = check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
  if (rc) return rc;
  for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
  h->graphs.clear();
  for (void* p : {(void*)h->d_phi, (void*)h->d_lam, (void*)h->d_epart, (void*)h->d_gpart, (void*)h->d_theta,
                  (void*)h->d_E, (void*)h->d_grad, (void*)h->d_coeffs, (void*)h->d_table, (void*)h->d_ssum})
    if (p) (void)hipFree(p);
  h->d_phi = h->d_lam = h->d_table = nullptr;
  h->d_epart = h->d_gpart = h->d_theta = h->d_E = h->d_grad = h->d_coeffs = h->d_ssum = nullptr;
  h->Bcap = 0;
  const size_t N = 1ull << h->n;
  const int G = blocks_per_state(h);
  rc = check_hip(hipMalloc(&h->d_phi, (size_t)B * N * sizeof(double2)), "hipMalloc(vqe phi)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_lam, (size_t)B * N * sizeof(double2)), "hipMalloc(vqe lambda)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_epart, (size_t)B * G * sizeof(double)), "hipMalloc(vqe epart)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_gpart, (size_t)B * std::max(1, h->nslots) * G * sizeof(double)), "hipMalloc(vqe gpart)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_theta, (size_t)B * std::max(1, h->P) * sizeof(double)), "hipMalloc(vqe theta)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_E, (size_t)B * sizeof(double)), "hipMalloc(vqe E)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_grad, (size_t)B * std::max(1, h->P) * sizeof(double)), "hipMalloc(vqe grad)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_coeffs, (size_t)B * std::max(1, h->nterms) * sizeof(double)), "hipMalloc(vqe coeffs)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_table, (size_t)B * std::max(1, h->nops) * 4 * sizeof(double2)), "hipMalloc(vqe table)");
  if (!rc) rc = check_hip(hipMalloc(&h->d_ssum, (size_t)B * std::max(1, h->nslots) * sizeof(double)), "hipMalloc(vqe slot sums)");
  if (rc) return rc;
  h->Bcap = B;
  return NWQ_OK;
}

// The per-gate schedule for B states on stream s (captured into a graph by
// the batched path, launched directly by the per-circuit path).
static int launch_global(nwq_vqe* h, int B, const double* theta, const double* coeffs, double* E, double* grad,
                         hipStream_t s) {
  const int G = blocks_per_state(h);
  const dim3 grid(G, B);
  hipLaunchKernelGGL(k_vqe_init, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->n);
  for (int i = 0; i < h->nops; ++i)
    hipLaunchKernelGGL(k_vqe_gate, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->n, h->ops[i], h->d_fixed, theta, h->P, 0);
  hipLaunchKernelGGL(k_vqe_hphi, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->d_lam, h->n, h->d_terms, h->nterms,
                     coeffs, h->d_epart, grad != nullptr ? 1 : 0);
  if (grad != nullptr) {
    for (int i = h->nops - 1; i >= 0; --i) {
      const VqeOp& op = h->ops[i];
      if (op.slot >= 0) {
        hipLaunchKernelGGL(k_vqe_adjoint, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->d_lam, h->n, op, h->d_fixed,
                           theta, h->P, h->nslots, h->d_gpart);
      } else {
        hipLaunchKernelGGL(k_vqe_gate, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->n, op, h->d_fixed, theta, h->P, 1);
        hipLaunchKernelGGL(k_vqe_gate, grid, dim3(kVqeBlock), 0, s, h->d_lam, h->n, op, h->d_fixed, theta, h->P, 1);
      }
    }
  }
  if (grad != nullptr && h->nslots > 0)
    hipLaunchKernelGGL(k_vqe_slot_sums, dim3((h->nslots + kFinBlock / kWave - 1) / (kFinBlock / kWave), B),
                       dim3(kFinBlock), 0, s, h->d_gpart, G, h->nslots, h->d_ssum);
  hipLaunchKernelGGL(k_vqe_finish, dim3(B), dim3(kFinBlock), 0, s, h->d_epart, G, h->nslots,
                     h->d_slot_param, h->P, h->d_ssum, E, grad);
  return check_hip(hipGetLastError(), "vqe per-gate schedule");
}

// Fused program: blocks over the ops at tile width fused_k, forward phases for
// the register-blocked kernel, backward ops in reverse per block (at most
// kBwdRegOps per dispatch).
// Low tile bits of the fused schedule's blocks (clamped to [k - 8, k - 2] at
// width k).  Fewer low bits give shorter runs and fewer blocks (n=20, L=8, 256
// vectors: 6 forward and 8 backward blocks with 3, 51 ms per batch; 11 and 16
// with 6, 59 ms; 4 take 6 and 12 blocks of twice the run and 46 ms there).
constexpr int kVqeLowBits = 3;
constexpr int kVqeSeeds = 2;   // as many as it takes: 8 seeds plan no fewer blocks for the HEA ansatz

// A gate on register bits (3 register bits) before its permutations are folded.
struct RegGate {
  RegOpV o;
  int perm, b0, b1, slot;   // perm: 1 CX, 2 SWAP
  unsigned bits;
};
static RegGate reg_gate(const VqeOp& op, int r0, int r1, bool two) {
  const int pair = two ? rb_pair(std::min(r0, r1), std::max(r0, r1)) : 0;
  RegGate o{{0, std::max(0, op.mat), op.param, -1}, 0, r0, r1, op.slot, two ? (1u << r0) | (1u << r1) : 1u << r0};
  if (op.kind == OP_ROT) o.o.code = RV_ROT + 3 * op.axis + r0;
  else if (op.kind == OP_FIX1) o.o.code = RV_FIX + r0;
  else if (op.kind == OP_RZZ) o.o.code = RV_RZZ + pair;
  else if (op.kind == OP_CZ) o.o.code = RV_CZ + pair;
  else if (op.kind == OP_CX) o.o.code = RV_CX + 2 * pair + (r0 > r1 ? 1 : 0), o.perm = 1;
  else o.o.code = RV_SWAP + pair, o.perm = 2;
  return o;
}
static void fold_reg_gates(std::vector<RegGate>& pops, RbStage& stg) {
  fold_permutations(
      pops, 3, [](const RegGate& o) { return o.perm != 0; }, [](const RegGate& o) { return o.bits; },
      [](const RegGate& o, int j) { return o.perm == 1 ? reg_cx(o.b0, o.b1, j) : reg_swap(o.b0, o.b1, j); },
      stg.ld_perm, stg.st_perm);
}
static unsigned long long tile_bits(const Block& b) {
  unsigned long long t = (1ull << b.c) - 1ull;
  for (int i = 0; i < b.m; ++i) t |= 1ull << b.hi[i];
  return t;
}
static int build_fused(nwq_vqe* h) {
  if (h->fused_built) return NWQ_OK;
  const int low = h->low_bits > 0 ? h->low_bits : kVqeLowBits;
  const int n = h->n;
  std::vector<PGate> g(h->nops);
  for (int i = 0; i < h->nops; ++i) {
    const VqeOp& op = h->ops[i];
    const bool two = op.kind == OP_RZZ || op.kind == OP_CX || op.kind == OP_CZ || op.kind == OP_SWAP;
    g[i] = PGate{0, {op.q0, two ? op.q1 : -1}, two ? 2 : 1, {0, 0, 0}};
  }
  const int k = std::min(h->fused_k, n);
  const std::vector<Block> blocks = plan_blocks(g, n, std::max(k, 6), low, kVqeSeeds, true);
  if (blocks.empty() && h->nops > 0) return set_error(NWQ_EINVAL, "fusion planner made no progress");
  std::vector<RbPhase> fphases;     // forward
  std::vector<RbPhase> phases;      // backward
  std::vector<RbOp> fops;
  h->fwd_blocks.clear();
  h->bwd_reg.clear();
  std::vector<Block> padded(blocks);
  for (Block& b : padded) pad_block(b, n, std::max(k, 8));
  size_t max_bwd_lds = 0;
  for (const Block& b : padded) {
    const int kb = b.c + b.m;
    if (kb < 8) return set_error(NWQ_EINVAL, "fused VQE path needs tiles of at least 2^8 amplitudes");
    std::vector<std::array<int, 4>> lb(g.size());
    std::vector<int> nq(g.size(), 1);
    for (int gi : b.gates) {
      lb[gi] = {local_bit(b, g[gi].q[0]), g[gi].nq == 2 ? local_bit(b, g[gi].q[1]) : 0};
      nq[gi] = g[gi].nq;
    }
    const int fops0 = (int)fops.size();
    std::vector<RbStage> stages;
    for (const Phase& ph : plan_phases(b.gates, lb, nq, kb, b.c, h->fused_rbits)) {
      RbStage fp{};
      for (int i = 0; i < 4; ++i) fp.reg[i] = ph.reg[i] < 0 ? 0 : ph.reg[i];
      fp.op_begin = (int)fops.size();
      auto ridx = [&](int bit) {
        for (int i = 0; i < h->fused_rbits; ++i)
          if (ph.reg[i] == bit) return i;
        return -1;
      };
      // ops before their permutations are folded into the LDS offsets
      struct FwdOp {
        RbOp o;
        int perm, b0, b1;   // perm: 1 CX, 2 SWAP
        unsigned bits;
      };
      std::vector<FwdOp> pops;
      for (int gi : ph.gates) {
        const VqeOp& op = h->ops[gi];
        const int r0 = ridx(lb[gi][0]), r1 = nq[gi] == 2 ? ridx(lb[gi][1]) : 0;
        const int pair = nq[gi] == 2 ? rb_pair(std::min(r0, r1), std::max(r0, r1)) : 0;
        FwdOp f{{0, 4 * gi}, 0, r0, r1, nq[gi] == 2 ? (1u << r0) | (1u << r1) : 1u << r0};
        // the parts of a rotation that are zero for every theta are skipped
        if (op.kind == OP_ROT) f.o.code = (op.axis == 2 ? kRbDiag1 : op.axis == 1 ? kRbReal1 : kRbXt1) + r0;
        else if (op.kind == OP_FIX1) f.o.code = kRbGen1 + r0;
        else if (op.kind == OP_RZZ || op.kind == OP_CZ) f.o.code = kRbDiag2 + pair;   // symmetric in its qubits
        else if (op.kind == OP_CX) f.o.code = rb_cx_code(r0, r1), f.perm = 1;
        else f.o.code = kRbSwap + pair, f.perm = 2;
        pops.push_back(f);
      }
      fold_permutations(
          pops, h->fused_rbits, [](const FwdOp& o) { return o.perm != 0; }, [](const FwdOp& o) { return o.bits; },
          [](const FwdOp& o, int j) { return o.perm == 1 ? reg_cx(o.b0, o.b1, j) : reg_swap(o.b0, o.b1, j); },
          fp.ld_perm, fp.st_perm);
      for (const FwdOp& f : pops) fops.push_back(f.o);
      if (pops.size() % 2) fops.push_back(RbOp{kRbCopy, fops.back().mat});
      fp.op_count = (int)fops.size() - fp.op_begin;
      stages.push_back(fp);
    }
    if (stages.empty()) continue;
    RbBlock d;
    layout_rb_block(b, std::move(stages), h->fused_rbits, (h->fused_flags & kFusedDirect) != 0, d, fphases);
    d.prog_ops = (int)fops.size() - fops0;   // matrices: per-vector table
    h->fwd_blocks.push_back(d);
  }
  for (int i = 0; i < 2; ++i) fops.push_back(RbOp{kRbCopy, 0});   // read ahead, not run
  constexpr int kBwdBits = 3;
  // The backward sweep plans its own blocks when the forward width exceeds
  // what its kernels take (tiles of at most 2^11: 256 threads x 8 amplitudes):
  // any partition of the reversed gate list gives the same sweep.
  std::vector<Block> bpadded;
  const int kbw = std::min(k, kBwdMaxTileBits);
  if (kbw == k) {
    bpadded = padded;
  } else {
    bpadded = plan_blocks(g, n, std::max(kbw, 6), low, kVqeSeeds, true);
    if (bpadded.empty() && h->nops > 0) return set_error(NWQ_EINVAL, "fusion planner made no progress");
    for (Block& b : bpadded) pad_block(b, n, std::max(kbw, 8));
  }
  std::vector<RegOpV> rops;
  std::vector<int> slots;
  unsigned long long touched = 0;   // union of the tiles of the blocks before
  std::vector<unsigned long long> before;
  for (const Block& b : bpadded) {
    before.push_back(touched);
    touched |= tile_bits(b);
  }
  for (auto bit = bpadded.rbegin(); bit != bpadded.rend(); ++bit) {
    const Block& b = *bit;
    const int kb = b.c + b.m;
    std::vector<std::array<int, 4>> lb(g.size());
    std::vector<int> nq(g.size(), 1);
    std::vector<int> rev(b.gates.rbegin(), b.gates.rend());
    for (int gi : rev) {
      lb[gi] = {local_bit(b, g[gi].q[0]), g[gi].nq == 2 ? local_bit(b, g[gi].q[1]) : 0};
      nq[gi] = g[gi].nq;
    }
    for (size_t s0 = 0; s0 < rev.size(); s0 += kBwdRegOps) {
      const std::vector<int> chunk(rev.begin() + s0, rev.begin() + std::min(rev.size(), s0 + kBwdRegOps));
      nwq_vqe::BwdRegBlock blk{};
      blk.op0 = (int)rops.size();
      blk.slot0 = (int)slots.size();
      std::vector<unsigned> obits;   // register bits of each op of the chunk
      std::vector<RbStage> stages;
      for (const Phase& ph : plan_phases(chunk, lb, nq, kb, b.c, kBwdBits)) {
        RbStage stg{};
        for (int i = 0; i < kBwdBits; ++i) stg.reg[i] = ph.reg[i];
        stg.op_begin = (int)rops.size() - blk.op0;
        auto ridx = [&](int bit) {
          for (int i = 0; i < kBwdBits; ++i)
            if (ph.reg[i] == bit) return i;
          return -1;
        };
        std::vector<RegGate> pops;
        for (int gi : ph.gates)
          pops.push_back(reg_gate(h->ops[gi], ridx(lb[gi][0]), nq[gi] == 2 ? ridx(lb[gi][1]) : 0, nq[gi] == 2));
        fold_reg_gates(pops, stg);
        for (RegGate& o : pops) {
          int local = -1;
          if (o.slot >= 0) {
            local = (int)slots.size() - blk.slot0;
            slots.push_back(o.slot);
          }
          const int code = o.o.code;
          // an RY joins the RZ un-applied before it on its bit when nothing between them touches the bit
          if (code >= RV_ROT + 3 && code < RV_ROT + 6) {
            int j = (int)rops.size() - 1;
            while (j >= blk.op0 + stg.op_begin && !(obits[j - blk.op0] & o.bits)) --j;
            if (j >= blk.op0 + stg.op_begin && (rops[j].code & 31) == RV_ROT + 6 + o.b0) {
              rops[j] = RegOpV{RV_YZ + o.b0 + 32 * (local + 1), (rops[j].code >> 5) - 1, o.o.param, rops[j].param};
              continue;
            }
          }
          o.o.code += 32 * (local + 1);
          rops.push_back(o.o);
          obits.push_back(o.bits);
        }
        stg.op_count = (int)rops.size() - blk.op0 - stg.op_begin;
        stages.push_back(stg);
      }
      blk.nops = (int)rops.size() - blk.op0;
      blk.nlocal = (int)slots.size() - blk.slot0;
      layout_rb_block(b, std::move(stages), kBwdBits, true, blk.d, phases);
      blk.mask = before[bpadded.rend() - bit - 1] & ~blk.d.tile;
      max_bwd_lds = std::max(max_bwd_lds, bwd_reg_lds(kb, blk.d.ph_count, blk.nops, blk.nlocal));
      h->bwd_reg.push_back(blk);
    }
  }
  // lambda = H phi: the first pass takes tiles of the low kt bits with every
  // diagonal term and the terms whose flipped bits lie there; further passes
  // take tiles of kHLow low bits plus up to kt - kHLow high bits, greedily, for
  // the remaining terms; terms needing more high bits than that go to a
  // gather pass.  Tiles are widened to 2^kt entries with unused high bits.
  std::vector<HTerm> hterms;
  std::vector<int> widx;
  h->hlaunch.clear();
  {
    const int kt = std::min(n, kHTileBits);
    std::vector<int> diag, rest, wide;
    for (int t = 0; t < h->nterms; ++t) {
      const unsigned long long x = h->terms[t].x;
      if (x == 0) diag.push_back(t);
      else if ((x >> kt) == 0) rest.push_back(t);   // in the first pass
      else if (__builtin_popcountll(x >> kHLow) > kt - kHLow) wide.push_back(t);
      else rest.push_back(t);
    }
    auto add_pass = [&](int c, std::vector<int> hi, const std::vector<int>& dg, const std::vector<int>& fl) {
      for (int q = c; q < n && (int)hi.size() < kt - c; ++q)
        if (std::find(hi.begin(), hi.end(), q) == hi.end()) hi.push_back(q);
      std::sort(hi.begin(), hi.end());
      auto local = [&](unsigned long long mask) {
        unsigned l = (unsigned)(mask & ((1ull << c) - 1ull));
        for (size_t i = 0; i < hi.size(); ++i)
          if ((mask >> hi[i]) & 1ull) l |= 1u << (c + i);
        return l;
      };
      unsigned long long inside = (1ull << c) - 1ull;
      for (int q : hi) inside |= 1ull << q;
      std::vector<int> all(dg);
      all.insert(all.end(), fl.begin(), fl.end());
      for (size_t s0 = 0; s0 < all.size(); s0 += kHMaxTerms) {
        nwq_vqe::HLaunch L{};
        L.p.c = c;
        L.p.m = (int)hi.size();
        for (size_t i = 0; i < hi.size(); ++i) L.p.hi[i] = hi[i];
        L.p.t_begin = (int)hterms.size();
        for (size_t i = s0; i < std::min(all.size(), s0 + kHMaxTerms); ++i) {
          const VqeTerm& T = h->terms[all[i]];
          const int pc = __builtin_popcountll(T.x & T.z);
          hterms.push_back(HTerm{local(T.x), local(T.z & inside), T.z & ~inside, pc & 3, pc & 1, all[i], 0});
          if (T.x == 0) ++L.p.n_diag;
          else ++L.p.n_flip;
        }
        h->hlaunch.push_back(L);
      }
    };
    std::vector<int> first_flips, later;
    for (int t : rest) ((h->terms[t].x >> kt) == 0 ? first_flips : later).push_back(t);
    add_pass(kt, {}, diag, first_flips);
    const int c = std::min(kHLow, kt);
    while (!later.empty()) {
      std::vector<int> hi, take, keep;
      for (int t : later) {
        std::vector<int> need;
        for (int q = c; q < n; ++q)
          if (((h->terms[t].x >> q) & 1ull) && std::find(hi.begin(), hi.end(), q) == hi.end()) need.push_back(q);
        if ((int)(hi.size() + need.size()) <= kt - c) {
          hi.insert(hi.end(), need.begin(), need.end());
          take.push_back(t);
        } else {
          keep.push_back(t);
        }
      }
      add_pass(c, hi, {}, take);
      later.swap(keep);
    }
    if (!wide.empty()) {
      nwq_vqe::HLaunch L{};
      L.wide = 1;
      L.w_begin = 0;
      L.w_count = (int)wide.size();
      widx = wide;
      h->hlaunch.push_back(L);
    }
    for (size_t i = 0; i < h->hlaunch.size(); ++i) {
      h->hlaunch[i].p.first = i == 0;
      h->hlaunch[i].p.last = i + 1 == h->hlaunch.size();
    }
  }
  const size_t ph_bytes = phases.size() * sizeof(RbPhase);
  h->fused_fph_off = (ph_bytes + 255) & ~size_t(255);
  h->fused_ops_off = (h->fused_fph_off + fphases.size() * sizeof(RbPhase) + 255) & ~size_t(255);
  h->fused_rop_off = (h->fused_ops_off + fops.size() * sizeof(RbOp) + 255) & ~size_t(255);
  h->fused_slot_off = (h->fused_rop_off + rops.size() * sizeof(RegOpV) + 255) & ~size_t(255);
  h->fused_hterm_off = (h->fused_slot_off + slots.size() * sizeof(int) + 255) & ~size_t(255);
  h->fused_widx_off = (h->fused_hterm_off + hterms.size() * sizeof(HTerm) + 255) & ~size_t(255);
  const size_t total = h->fused_widx_off + widx.size() * sizeof(int) + 16;
  std::vector<char> prog(total, 0);
  if (!phases.empty()) std::memcpy(prog.data(), phases.data(), ph_bytes);
  if (!fphases.empty()) std::memcpy(prog.data() + h->fused_fph_off, fphases.data(), fphases.size() * sizeof(RbPhase));
  if (!fops.empty()) std::memcpy(prog.data() + h->fused_ops_off, fops.data(), fops.size() * sizeof(RbOp));
  if (!rops.empty()) std::memcpy(prog.data() + h->fused_rop_off, rops.data(), rops.size() * sizeof(RegOpV));
  if (!slots.empty()) std::memcpy(prog.data() + h->fused_slot_off, slots.data(), slots.size() * sizeof(int));
  if (!hterms.empty()) std::memcpy(prog.data() + h->fused_hterm_off, hterms.data(), hterms.size() * sizeof(HTerm));
  if (!widx.empty()) std::memcpy(prog.data() + h->fused_widx_off, widx.data(), widx.size() * sizeof(int));
  // dynamic LDS above 64 KiB is enabled here, outside any graph capture
  if (max_bwd_lds > (size_t)kMaxDynamicLds ||
      (sizeof(double2) << kHTileBits) > (size_t)kMaxDynamicLds)
    return set_error(NWQ_EINVAL, "VQE tile larger than the dynamic LDS limit");
  int rc = NWQ_OK;
  for (const void* f : {(const void*)k_vqe_hphi_tile<false, false>, (const void*)k_vqe_hphi_tile<true, false>,
                        (const void*)k_vqe_hphi_tile<false, true>, (const void*)k_vqe_hphi_tile<true, true>,
                        (const void*)k_vqe_bwd_reg<false>, (const void*)k_vqe_bwd_reg<true>})
    if (!rc) rc = enable_dynamic_lds(f);
  if (!rc) rc = check_hip(hipMalloc(&h->d_fused, total), "hipMalloc(vqe fused program)");
  if (!rc) rc = check_hip(hipMemcpy(h->d_fused, prog.data(), total, hipMemcpyHostToDevice), "hipMemcpy(vqe fused program)");
  if (rc) return rc;
  h->fused_built = true;
  h->fused_bytes = total;
  return NWQ_OK;
}

// Program of the register-resident path: the ops in phases of 3 register bits
// over the whole register (CX and SWAP folded into the exchanges where they
// can be), and the slots of each parameter in slot order.
static std::vector<char> build_reg(nwq_vqe* h) {
  const int nb = std::max(3, h->n);
  std::vector<std::array<int, 4>> lb(h->nops);
  std::vector<int> nq(h->nops), order(h->nops);
  for (int i = 0; i < h->nops; ++i) {
    const VqeOp& op = h->ops[i];
    const bool two = op.kind == OP_RZZ || op.kind == OP_CX || op.kind == OP_CZ || op.kind == OP_SWAP;
    lb[i] = {op.q0, two ? op.q1 : 0, 0, 0};
    nq[i] = two ? 2 : 1;
    order[i] = i;
  }
  std::vector<RbStage> stages;
  std::vector<RegOpV> rops;
  std::vector<unsigned> rbits;   // register bits of each op
  std::vector<Phase> plan = plan_phases(order, lb, nq, nb, 0, 3);
  if (plan.empty()) plan.push_back(Phase{{0, 1, 2, -1}, {}});   // no ops
  for (const Phase& ph : plan) {
    RbStage stg{};
    for (int i = 0; i < 3; ++i) stg.reg[i] = ph.reg[i];
    stg.op_begin = (int)rops.size();
    auto ridx = [&](int bit) {
      for (int i = 0; i < 3; ++i)
        if (ph.reg[i] == bit) return i;
      return -1;
    };
    std::vector<RegGate> pops;
    for (int gi : ph.gates) {
      const VqeOp& op = h->ops[gi];
      pops.push_back(reg_gate(op, ridx(op.q0), nq[gi] == 2 ? ridx(op.q1) : 0, nq[gi] == 2));
      pops.back().o.code += 32 * (op.slot + 1);
    }
    fold_reg_gates(pops, stg);
    for (size_t i = 0; i < pops.size(); ++i) {
      const RegGate& o = pops[i];
      // an RZ joins the RY before it on its bit when nothing between them touches the bit
      if ((o.o.code & 31) >= RV_ROT + 6 && (o.o.code & 31) < RV_FIX) {
        int j = (int)rops.size() - 1;
        while (j >= stg.op_begin && !(rbits[j] & o.bits)) --j;
        if (j >= stg.op_begin && (rops[j].code & 31) == RV_ROT + 3 + o.b0) {
          rops[j].code += RV_YZ - (RV_ROT + 3);
          rops[j].mat = (o.o.code >> 5) - 1;
          rops[j].param2 = o.o.param;
          continue;
        }
      }
      rops.push_back(o.o);
      rbits.push_back(o.bits);
    }
    stg.op_count = (int)rops.size() - stg.op_begin;
    stages.push_back(stg);
  }
  std::vector<RbPhase> phases;
  RbTileIo io;
  layout_phases(stages, 3, nb, 0, 4, phases, io);
  RbPhase end{};
  for (int j = 0; j < kRbThreadBits; ++j) {
    end.rd_t[j] = io.st_t[j];
    end.wr_t[j] = entry_slot(io.st_t[j], 4);
  }
  for (int j = 0; j < 4; ++j) {
    end.rd_r[j] = io.st_r[j];
    end.wr_r[j] = entry_slot(io.st_r[j], 4);
  }
  h->reg_phases = (int)phases.size();
  h->reg_ops = (int)rops.size();
  phases.push_back(end);
  std::vector<int> poff(h->P + 1, 0), pslots(h->nslots);
  for (int p : h->slot_param) ++poff[p + 1];
  for (int p = 0; p < h->P; ++p) poff[p + 1] += poff[p];
  std::vector<int> at(poff.begin(), poff.end() - 1);
  for (int sl = 0; sl < h->nslots; ++sl) pslots[at[h->slot_param[sl]]++] = sl;
  auto up = [](size_t x) { return (x + 63) & ~size_t(63); };
  h->reg_ops_off = up(phases.size() * sizeof(RbPhase));
  h->reg_poff_off = up(h->reg_ops_off + rops.size() * sizeof(RegOpV));
  h->reg_pslots_off = up(h->reg_poff_off + poff.size() * sizeof(int));
  std::vector<char> prog(h->reg_pslots_off + pslots.size() * sizeof(int) + 16, 0);
  std::memcpy(prog.data(), phases.data(), phases.size() * sizeof(RbPhase));
  if (!rops.empty()) std::memcpy(prog.data() + h->reg_ops_off, rops.data(), rops.size() * sizeof(RegOpV));
  std::memcpy(prog.data() + h->reg_poff_off, poff.data(), poff.size() * sizeof(int));
  if (!pslots.empty()) std::memcpy(prog.data() + h->reg_pslots_off, pslots.data(), pslots.size() * sizeof(int));
  return prog;
}

static int fused_grid(const nwq_vqe* h) {
  // workgroups per state, shared by the forward and backward launches (the
  // gradient partials have one slot per workgroup): sized on the backward tiles
  const int k = std::min(std::max(std::min(h->fused_k, kBwdMaxTileBits), 8), h->n);
  const unsigned long long ntiles = 1ull << (h->n - k);
  return (int)std::max<unsigned long long>(1, std::min<unsigned long long>(ntiles, blocks_per_state(h)));
}

static int launch_fused(nwq_vqe* h, int B, const double* theta, const double* coeffs, double* E, double* grad,
                        hipStream_t s) {
  int rc = build_fused(h);
  if (rc) return rc;
  const int G = fused_grid(h);
  const dim3 grid(G, B);
  const RbPhase* dfp = reinterpret_cast<const RbPhase*>(static_cast<char*>(h->d_fused) + h->fused_fph_off);
  const RbOp* dfo = reinterpret_cast<const RbOp*>(static_cast<char*>(h->d_fused) + h->fused_ops_off);
  const int stride = 4 * h->nops;
  hipLaunchKernelGGL(k_vqe_init, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->n);
  hipLaunchKernelGGL(k_vqe_mats, dim3((h->nops + 255) / 256, B), dim3(256), 0, s, h->d_ops, h->nops, h->d_fixed,
                     theta, h->P, h->d_table);
  // phi starts at |0...0>: amplitudes can be nonzero only where every qubit no
  // earlier block touched is zero, and a block maps each tile to itself and
  // zero tiles to zero, so each block runs only the tiles whose index is zero
  // on its non-tile qubits outside that support (the first block: tile 0)
  unsigned long long support = 0;
  for (size_t bi = 0; bi < h->fwd_blocks.size(); ++bi) {
    const RbBlock& d = h->fwd_blocks[bi];
    launch_fused_rb(s, h->d_phi, h->n, d, dfp, dfo, h->d_table, h->fused_rbits, kRbSetVQE,
                    (h->fused_flags & kFusedNonTemporal) != 0, support & ~d.tile, B, stride, G);
    support |= d.tile;
  }
  const HTerm* dht = reinterpret_cast<const HTerm*>(static_cast<char*>(h->d_fused) + h->fused_hterm_off);
  const int* dwi = reinterpret_cast<const int*>(static_cast<char*>(h->d_fused) + h->fused_widx_off);
  for (const auto& L : h->hlaunch) {
    const int sel = (L.p.first ? 1 : 0) | (L.p.last ? 2 : 0);
    if (L.wide) {
      auto kw = sel == 0 ? k_vqe_hphi_wide<false, false> : sel == 1 ? k_vqe_hphi_wide<true, false>
              : sel == 2 ? k_vqe_hphi_wide<false, true> : k_vqe_hphi_wide<true, true>;
      hipLaunchKernelGGL(kw, grid, dim3(kVqeBlock), 0, s, h->d_phi, h->d_lam, h->n, h->d_terms, dwi + L.w_begin,
                         L.w_count, h->nterms, coeffs, h->d_epart);
    } else {
      auto kt = sel == 0 ? k_vqe_hphi_tile<false, false> : sel == 1 ? k_vqe_hphi_tile<true, false>
              : sel == 2 ? k_vqe_hphi_tile<false, true> : k_vqe_hphi_tile<true, true>;
      const size_t lds = sizeof(double2) << (L.p.c + L.p.m);
      hipLaunchKernelGGL(kt, grid, dim3(kHBlock), lds, s, h->d_phi, h->d_lam, h->n, L.p, dht, h->d_terms, h->nterms,
                         coeffs, h->d_epart);
    }
  }
  if (grad != nullptr) {
    const RbPhase* dph = static_cast<const RbPhase*>(h->d_fused);
    const RegOpV* dro = reinterpret_cast<const RegOpV*>(static_cast<char*>(h->d_fused) + h->fused_rop_off);
    const int* dsl = reinterpret_cast<const int*>(static_cast<char*>(h->d_fused) + h->fused_slot_off);
    for (const auto& b : h->bwd_reg) {
      const unsigned long long nt = 1ull << __builtin_popcountll(b.mask);
      auto kern = (h->fused_flags & kFusedNonTemporal) ? k_vqe_bwd_reg<true> : k_vqe_bwd_reg<false>;
      hipLaunchKernelGGL(kern, grid, dim3(1u << (b.d.k - 3)),
                         bwd_reg_lds(b.d.k, b.d.ph_count, b.nops, b.nlocal), s, h->d_phi, h->d_lam, h->n, b.d, dph,
                         dro + b.op0, b.nops, dsl + b.slot0, b.nlocal, h->d_fixed, theta, h->P, h->nslots, h->d_gpart,
                         nt, b.mask, deposit_bits(G, b.mask));
    }
  }
  if (grad != nullptr && h->nslots > 0)
    hipLaunchKernelGGL(k_vqe_slot_sums, dim3((h->nslots + kFinBlock / kWave - 1) / (kFinBlock / kWave), B),
                       dim3(kFinBlock), 0, s, h->d_gpart, G, h->nslots, h->d_ssum);
  hipLaunchKernelGGL(k_vqe_finish, dim3(B), dim3(kFinBlock), 0, s, h->d_epart, G, h->nslots,
                     h->d_slot_param, h->P, h->d_ssum, E, grad);
  return check_hip(hipGetLastError(), "vqe fused schedule");
}

static int run_graph(nwq_vqe* h, int B, bool want_grad, bool with_coeffs) {
  const bool fused = h->cfg.mode == 3 || (h->cfg.mode == 0 && h->n > 12);
  const auto key = std::make_pair(B, (want_grad ? 1 : 0) | (with_coeffs ? 2 : 0) | (fused ? 4 : 0));
  auto it = h->graphs.find(key);
  if (it == h->graphs.end()) {
    if (fused) {
      const int rcb = build_fused(h);   // host planning and program upload stay outside the capture
      if (rcb) return rcb;
    }
    int rc = check_hip(hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
    if (rc) return rc;
    if (fused)
      rc = launch_fused(h, B, h->d_theta, with_coeffs ? h->d_coeffs : nullptr, h->d_E, want_grad ? h->d_grad : nullptr,
                        h->stream);
    else
      rc = launch_global(h, B, h->d_theta, with_coeffs ? h->d_coeffs : nullptr, h->d_E, want_grad ? h->d_grad : nullptr,
                         h->stream);
    hipGraph_t g = nullptr;
    const int rc2 = check_hip(hipStreamEndCapture(h->stream, &g), "hipStreamEndCapture");
    if (rc) return rc;
    if (rc2) return rc2;
    hipGraphExec_t ex = nullptr;
    rc = check_hip(hipGraphInstantiate(&ex, g, nullptr, nullptr, 0), "hipGraphInstantiate");
    (void)hipGraphDestroy(g);
    if (rc) return rc;
    it = h->graphs.emplace(key, ex).first;
  }
  return check_hip(hipGraphLaunch(it->second, h->stream), "hipGraphLaunch");
}

}  // namespace nwq

using namespace nwq;

extern "C" {

int nwq_vqe_create(int n, int n_ops, const int* types, const int* qubits, const int* params, int n_params,
                   int n_terms, const uint64_t* xmask, const uint64_t* zmask, const double* coeffs, void* stream,
                   nwq_vqe_handle* out) {
  if (!out) return vqe_fail(NWQ_EINVAL, "out handle pointer is NULL");
  *out = nullptr;
  if (n < 1 || n > 30) return vqe_fail(NWQ_ERANGE, "VQE register must have 1..30 qubits");
  if (n_ops < 0 || (n_ops > 0 && (!types || !qubits || !params))) return vqe_fail(NWQ_EINVAL, "bad op arrays");
  if (n_terms < 0 || (n_terms > 0 && (!xmask || !zmask || !coeffs))) return vqe_fail(NWQ_EINVAL, "bad term arrays");
  if (n_params < 0) return vqe_fail(NWQ_EINVAL, "negative parameter count");
  std::unique_ptr<nwq_vqe> h(new nwq_vqe());
  h->n = n;
  h->P = n_params;
  h->user_stream = static_cast<hipStream_t>(stream);
  std::vector<double2> fixed;
  for (int i = 0; i < n_ops; ++i) {
    const int t = types[i], a = qubits[2 * i], b = qubits[2 * i + 1], p = params[i];
    VqeOp op{};
    op.q0 = a;
    op.q1 = b;
    op.param = -1;
    op.slot = -1;
    op.mat = -1;
    const bool two = t == NWQ_GATE_CX || t == NWQ_GATE_CZ || t == NWQ_GATE_SWAP || t == NWQ_GATE_RZZ;
    if (a < 0 || a >= n || (two && (b < 0 || b >= n))) return vqe_fail(NWQ_ERANGE, "op " + std::to_string(i) + ": qubit out of range");
    if (two && a == b) return vqe_fail(NWQ_EDUP, "op " + std::to_string(i) + ": repeated qubit");
    const bool param = t == NWQ_GATE_RX || t == NWQ_GATE_RY || t == NWQ_GATE_RZ || t == NWQ_GATE_RZZ;
    if (param) {
      if (p < 0 || p >= n_params) return vqe_fail(NWQ_EINVAL, "op " + std::to_string(i) + ": parameter index out of range");
      op.param = p;
      op.slot = h->nslots++;
      h->slot_param.push_back(p);
      if (t == NWQ_GATE_RZZ) {
        op.kind = OP_RZZ;
      } else {
        op.kind = OP_ROT;
        op.axis = t == NWQ_GATE_RX ? 0 : (t == NWQ_GATE_RY ? 1 : 2);
      }
    } else if (t == NWQ_GATE_CX) {
      op.kind = OP_CX;
    } else if (t == NWQ_GATE_CZ) {
      op.kind = OP_CZ;
    } else if (t == NWQ_GATE_SWAP) {
      op.kind = OP_SWAP;
    } else if (t >= NWQ_GATE_I && t <= NWQ_GATE_TDG) {
      if (t == NWQ_GATE_I) continue;
      cd m[16];
      gate_matrix(t, nullptr, m);
      op.kind = OP_FIX1;
      op.mat = (int)(fixed.size() / 8);
      for (int k = 0; k < 4; ++k) fixed.push_back(make_double2(m[k].real(), m[k].imag()));
      const int tr[4] = {0, 2, 1, 3};   // U^dag = conj(U^T)
      for (int k = 0; k < 4; ++k) fixed.push_back(make_double2(m[tr[k]].real(), -m[tr[k]].imag()));
    } else {
      return vqe_fail(NWQ_EINVAL, "op " + std::to_string(i) + ": gate type not supported in a VQE program");
    }
    h->ops.push_back(op);
  }
  h->nops = (int)h->ops.size();
  std::vector<VqeTerm> terms(n_terms);
  const unsigned long long all = (1ull << n) - 1ull;
  for (int t = 0; t < n_terms; ++t) {
    if ((xmask[t] & ~all) || (zmask[t] & ~all)) return vqe_fail(NWQ_ERANGE, "Pauli mask has bits beyond n");
    if (!std::isfinite(coeffs[t])) return vqe_fail(NWQ_EINVAL, "non-finite coefficient");
    terms[t] = VqeTerm{xmask[t], zmask[t], coeffs[t], __builtin_popcountll(xmask[t] & zmask[t]) & 3, 0};
  }
  h->nterms = n_terms;
  h->terms = terms;
  int rc = check_hip(hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking), "hipStreamCreate");
  if (!rc) rc = check_hip(hipEventCreateWithFlags(&h->ev_in, hipEventDisableTiming), "hipEventCreate");
  if (!rc) rc = check_hip(hipEventCreateWithFlags(&h->ev_out, hipEventDisableTiming), "hipEventCreate");
  // the program's tables in one allocation and one copy
  std::vector<char> prog;
  std::vector<std::pair<void**, size_t>> parts;
  auto add = [&](void** dst, const void* src, size_t bytes) {
    parts.emplace_back(dst, prog.size());
    prog.resize((prog.size() + std::max<size_t>(bytes, 16) + 255) & ~size_t(255), 0);
    if (bytes) std::memcpy(prog.data() + parts.back().second, src, bytes);
  };
  add((void**)&h->d_ops, h->ops.data(), h->ops.size() * sizeof(VqeOp));
  add((void**)&h->d_fixed, fixed.data(), fixed.size() * sizeof(double2));
  add((void**)&h->d_terms, terms.data(), terms.size() * sizeof(VqeTerm));
  add((void**)&h->d_slot_param, h->slot_param.data(), h->slot_param.size() * sizeof(int));
  if (n <= 12 && h->nops <= 4096) {   // more does not fit the LDS
    const std::vector<char> reg = build_reg(h.get());
    add(&h->d_reg, reg.data(), reg.size());
  }
  if (!rc) rc = check_hip(hipMalloc(&h->d_program, prog.size()), "hipMalloc(vqe program)");
  if (!rc) rc = check_hip(hipMemcpy(h->d_program, prog.data(), prog.size(), hipMemcpyHostToDevice), "hipMemcpy(vqe program)");
  if (!rc) {
    h->program_bytes = prog.size();
    for (const auto& p : parts) *p.first = static_cast<char*>(h->d_program) + p.second;
  }
  if (rc) {
    nwq_vqe_destroy(h.release());
    return rc;
  }
  h->cfg.threads = n <= 8 ? 128 : 256;
  *out = h.release();
  return NWQ_OK;
}

int nwq_vqe_destroy(nwq_vqe_handle h) {
  if (!h) return NWQ_OK;
  if (h->stream) (void)hipStreamSynchronize(h->stream);
  for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
  for (void* p : {h->d_program, (void*)h->d_phi, (void*)h->d_lam,
                  (void*)h->d_epart, (void*)h->d_gpart, (void*)h->d_theta, (void*)h->d_E,
                  (void*)h->d_grad, (void*)h->d_coeffs, (void*)h->d_table, (void*)h->d_ssum, h->d_fused})
    if (p) (void)hipFree(p);
  if (h->ev_in) (void)hipEventDestroy(h->ev_in);
  if (h->ev_out) (void)hipEventDestroy(h->ev_out);
  if (h->stream) (void)hipStreamDestroy(h->stream);
  delete h;
  return NWQ_OK;
}

int nwq_vqe_memory(nwq_vqe_handle h, int B, size_t* held, size_t* at_B) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (B < 0 || B > 65535) return vqe_fail(NWQ_EINVAL, "batch size must be in [0, 65535]");
  const size_t per = global_bytes_per_vector(h);
  const size_t base = h->program_bytes + h->fused_bytes;
  if (held) *held = base + (size_t)h->Bcap * per;
  if (at_B) {
    // the LDS-resident path keeps no per-vector buffers; every other path
    // grows the capacity to B (never shrinks it)
    const bool lds = h->cfg.mode == 1 || (h->cfg.mode == 0 && lds_fits(h, h->cfg.threads, true));
    const size_t cap = lds ? (size_t)h->Bcap : std::max<size_t>(h->Bcap, (size_t)B);
    *at_B = base + cap * per;
  }
  return NWQ_OK;
}

int nwq_vqe_info(nwq_vqe_handle h, int* n_params, int* n_ops, int* n_slots) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (n_params) *n_params = h->P;
  if (n_ops) *n_ops = h->nops;
  if (n_slots) *n_slots = h->nslots;
  return NWQ_OK;
}

int nwq_vqe_set_config(nwq_vqe_handle h, int mode, int threads, int blocks_per_state_) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (mode < 0 || mode > 3) return vqe_fail(NWQ_EINVAL, "mode must be 0 (auto), 1 (LDS), 2 (per-gate) or 3 (fused)");
  if (mode == 3 && h->n < 8) return vqe_fail(NWQ_EINVAL, "the fused path needs n >= 8");
  if (threads != 64 && threads != 128 && threads != 256 && threads != 512 && threads != 1024)
    return vqe_fail(NWQ_EINVAL, "threads must be 64, 128, 256, 512 or 1024");
  if (blocks_per_state_ < 0 || blocks_per_state_ > 4096) return vqe_fail(NWQ_EINVAL, "blocks per state in [0, 4096]");
  if (mode == 1 && h->n > 12) return vqe_fail(NWQ_EINVAL, "the LDS-resident path holds n <= 12");
  if (blocks_per_state_ != h->cfg.blocks_per_state) {   // partial buffers and graphs depend on it
    (void)hipStreamSynchronize(h->stream);
    for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
    h->graphs.clear();
    h->cfg.blocks_per_state = blocks_per_state_;
    const int B = h->Bcap;
    h->Bcap = 0;
    if (B > 0) {
      const int rc = ensure_global(h, B);
      if (rc) return rc;
    }
  }
  h->cfg.mode = mode;
  h->cfg.threads = threads;
  return NWQ_OK;
}

static void drop_fused(nwq_vqe* h) {   // the stream is idle and no graph holds the program
  if (h->d_fused) (void)hipFree(h->d_fused);
  h->d_fused = nullptr;
  h->fused_built = false;
  h->fused_bytes = 0;
}

int nwq_vqe_set_flags(nwq_vqe_handle h, int flags) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (flags < 0 || flags > 3) return vqe_fail(NWQ_EINVAL, "flags must be in [0, 3]");
  if (flags != h->fused_flags) {   // the captured schedules hold the kernels
    (void)hipStreamSynchronize(h->stream);
    for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
    h->graphs.clear();
    if ((flags ^ h->fused_flags) & kFusedDirect) drop_fused(h);   // the phases' layouts are planned again on next use
    h->fused_flags = flags;
  }
  return NWQ_OK;
}

int nwq_vqe_set_lowbits(nwq_vqe_handle h, int c) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (c != 0 && (c < 3 || c > 8)) return vqe_fail(NWQ_EINVAL, "low tile bits must be 0 or in [3, 8]");
  if (c != h->low_bits) {   // the fused program is planned again on next use
    (void)hipStreamSynchronize(h->stream);
    for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
    h->graphs.clear();
    drop_fused(h);
    h->low_bits = c;
  }
  return NWQ_OK;
}

int nwq_vqe_get_config(nwq_vqe_handle h, int* mode, int* threads, int* blocks_per_state_) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (mode) *mode = h->cfg.mode;
  if (threads) *threads = h->cfg.threads;
  if (blocks_per_state_) *blocks_per_state_ = blocks_per_state(h);
  return NWQ_OK;
}

static int eval_common(nwq_vqe_handle h, int B, const double* theta, const double* coeffs, double* E, double* grad,
                       bool single) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (B < 1 || B > 65535) return vqe_fail(NWQ_EINVAL, "batch size must be in [1, 65535]");
  if ((!theta && h->P > 0) || !E) return vqe_fail(NWQ_EINVAL, "NULL theta or energy pointer");
  int rc = check_hip(hipEventRecord(h->ev_in, h->user_stream), "hipEventRecord");
  if (!rc) rc = check_hip(hipStreamWaitEvent(h->stream, h->ev_in, 0), "hipStreamWaitEvent");
  if (rc) return rc;
  const bool want_grad = grad != nullptr;
  const int mode = single ? 2 : h->cfg.mode;
  const bool use_lds = !single && (mode == 1 || (mode == 0 && h->n <= 12 && lds_fits(h, h->cfg.threads, want_grad)));
  if (use_lds) {
    if (!lds_fits(h, h->cfg.threads, want_grad)) return vqe_fail(NWQ_EINVAL, "program does not fit the LDS-resident path");
    rc = launch_lds(h, B, theta, coeffs, E, grad, h->stream);
  } else if (single) {
    rc = ensure_global(h, B);
    if (!rc) rc = launch_global(h, B, theta, coeffs, E, grad, h->stream);
  } else {
    rc = ensure_global(h, B);
    if (!rc && h->P > 0)
      rc = check_hip(hipMemcpyAsync(h->d_theta, theta, (size_t)B * h->P * sizeof(double), hipMemcpyDeviceToDevice, h->stream),
                     "hipMemcpyAsync(theta)");
    if (!rc && coeffs && h->nterms > 0)
      rc = check_hip(hipMemcpyAsync(h->d_coeffs, coeffs, (size_t)B * h->nterms * sizeof(double), hipMemcpyDeviceToDevice,
                                    h->stream), "hipMemcpyAsync(coeffs)");
    if (!rc) rc = run_graph(h, B, want_grad, coeffs != nullptr);
    if (!rc) rc = check_hip(hipMemcpyAsync(E, h->d_E, (size_t)B * sizeof(double), hipMemcpyDeviceToDevice, h->stream),
                            "hipMemcpyAsync(E)");
    if (!rc && want_grad && h->P > 0)
      rc = check_hip(hipMemcpyAsync(grad, h->d_grad, (size_t)B * h->P * sizeof(double), hipMemcpyDeviceToDevice, h->stream),
                     "hipMemcpyAsync(grad)");
  }
  if (rc) return rc;
  rc = check_hip(hipEventRecord(h->ev_out, h->stream), "hipEventRecord");
  if (!rc) rc = check_hip(hipStreamWaitEvent(h->user_stream, h->ev_out, 0), "hipStreamWaitEvent");
  return rc;
}

int nwq_vqe_eval(nwq_vqe_handle h, int B, const double* theta_dev, double* energy_dev, double* grad_dev) {
  return eval_common(h, B, theta_dev, nullptr, energy_dev, grad_dev, false);
}

int nwq_vqe_eval_coeffs(nwq_vqe_handle h, int B, const double* theta_dev, const double* coeffs_dev,
                        double* energy_dev, double* grad_dev) {
  return eval_common(h, B, theta_dev, coeffs_dev, energy_dev, grad_dev, false);
}

int nwq_vqe_eval_single(nwq_vqe_handle h, const double* theta_dev, double* energy_dev, double* grad_dev) {
  return eval_common(h, 1, theta_dev, nullptr, energy_dev, grad_dev, true);
}

}  // extern "C"

extern "C" {

int nwq_vqe_autotune(nwq_vqe_handle h, int B, int with_grad, double* best_ms) {
  if (!h) return vqe_fail(NWQ_EINVAL, "NULL handle");
  if (B < 1 || B > 65535) return vqe_fail(NWQ_EINVAL, "batch size must be in [1, 65535]");
  double *theta = nullptr, *E = nullptr, *grad = nullptr;
  hipEvent_t t0 = nullptr, t1 = nullptr;
  const size_t P = std::max(1, h->P);
  int rc = check_hip(hipMalloc(&theta, (size_t)B * P * sizeof(double)), "hipMalloc(autotune theta)");
  if (!rc) rc = check_hip(hipMalloc(&E, (size_t)B * sizeof(double)), "hipMalloc(autotune E)");
  if (!rc) rc = check_hip(hipMalloc(&grad, (size_t)B * P * sizeof(double)), "hipMalloc(autotune grad)");
  if (!rc) rc = check_hip(hipMemsetAsync(theta, 0, (size_t)B * P * sizeof(double), h->stream), "hipMemsetAsync");
  if (!rc) rc = check_hip(hipEventCreate(&t0), "hipEventCreate");
  if (!rc) rc = check_hip(hipEventCreate(&t1), "hipEventCreate");
  struct Cand { int mode, threads, bps; };
  std::vector<Cand> cands;
  if (reg_fits(h)) {   // whatever the workgroup size
    cands.push_back({1, h->cfg.threads, 0});
  } else if (h->n <= 12) {
    for (int t : {64, 128, 256, 512, 1024})
      if (lds_fits(h, t, with_grad != 0)) cands.push_back({1, t, 0});
  }
  const unsigned long long pairs = 1ull << (h->n - 1);
  for (int bps : {0, 8, 16, 32, 64, 128, 256, 512, 1024})
    if (bps == 0 || (unsigned long long)bps * 256 <= pairs) cands.push_back({2, h->cfg.threads, bps});
  if (h->n >= 13)
    for (int bps : {0, 16, 32, 64, 128, 256, 512, 1024})
      if (bps == 0 || (unsigned long long)bps * 256 <= pairs) cands.push_back({3, h->cfg.threads, bps});
  const VqeConfig saved = h->cfg;
  double best = 1e300;
  VqeConfig best_cfg = saved;
  hipStream_t user = h->user_stream;
  h->user_stream = h->stream;
  for (const Cand& c : cands) {
    if (rc) break;
    rc = nwq_vqe_set_config(h, c.mode, c.threads, c.bps);
    if (rc) break;
    rc = eval_common(h, B, theta, nullptr, E, with_grad ? grad : nullptr, false);   // warm-up (and graph capture)
    if (rc) break;
    rc = check_hip(hipEventRecord(t0, h->stream), "hipEventRecord");
    for (int r = 0; r < 3 && !rc; ++r) rc = eval_common(h, B, theta, nullptr, E, with_grad ? grad : nullptr, false);
    if (!rc) rc = check_hip(hipEventRecord(t1, h->stream), "hipEventRecord");
    if (!rc) rc = check_hip(hipEventSynchronize(t1), "hipEventSynchronize");
    float ms = 0.f;
    if (!rc) rc = check_hip(hipEventElapsedTime(&ms, t0, t1), "hipEventElapsedTime");
    if (!rc && ms / 3.0 < best) {
      best = ms / 3.0;
      best_cfg = h->cfg;
    }
  }
  h->user_stream = user;
  if (!rc) rc = nwq_vqe_set_config(h, best_cfg.mode, best_cfg.threads, best_cfg.blocks_per_state);
  else (void)nwq_vqe_set_config(h, saved.mode, saved.threads, saved.blocks_per_state);
  (void)hipStreamSynchronize(h->stream);
  if (t0) (void)hipEventDestroy(t0);
  if (t1) (void)hipEventDestroy(t1);
  for (void* p : {(void*)theta, (void*)E, (void*)grad})
    if (p) (void)hipFree(p);
  if (!rc && best_ms) *best_ms = best;
  return rc;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// One-call batched VQE for the Ising model (Sec. III, Fig. 4): the
// hardware-efficient ansatz and the open-chain transverse-field Ising
// Hamiltonian are built here, and the evaluation runs through a context kept
// per (device, n, L).  When (J, h) change, the context's term table is
// rewritten in place on the context's stream (the captured graphs read it at
// run time), so a new field costs no re-capture.
namespace {

struct BatchEntry {
  int device = -1, n = 0, L = 0;
  double J = 0.0, hx = 0.0;
  nwq_vqe_handle ctx = nullptr;
  std::vector<nwq::VqeTerm> terms;   // host copy of the table last uploaded (source of the async copy)
  unsigned long long used = 0;
};
constexpr size_t kBatchCacheMax = 8;
std::mutex g_batch_mu;
std::vector<BatchEntry> g_batch;
unsigned long long g_batch_clock = 0;

void tfim_terms(int n, double J, double hx, std::vector<nwq::VqeTerm>& out) {
  out.clear();
  for (int i = 0; i + 1 < n; ++i)
    out.push_back(nwq::VqeTerm{0ull, (1ull << i) | (1ull << (i + 1)), -J, 0, 0});
  for (int i = 0; i < n; ++i) out.push_back(nwq::VqeTerm{1ull << i, 0ull, -hx, 0, 0});
}

int batch_context(int device, int n, int L, double J, double hx, void* stream, BatchEntry** out) {
  for (auto& e : g_batch)
    if (e.device == device && e.n == n && e.L == L) {
      *out = &e;
      return NWQ_OK;
    }
  // ansatz: per layer RY on 0..n-1, RZ on 0..n-1, CX(0,1) .. CX(n-2,n-1)
  std::vector<int> types, qubits, params;
  for (int l = 0; l < L; ++l) {
    for (int axis = 0; axis < 2; ++axis)
      for (int q = 0; q < n; ++q) {
        types.push_back(axis == 0 ? NWQ_GATE_RY : NWQ_GATE_RZ);
        qubits.push_back(q);
        qubits.push_back(-1);
        params.push_back(l * 2 * n + axis * n + q);
      }
    for (int q = 0; q + 1 < n; ++q) {
      types.push_back(NWQ_GATE_CX);
      qubits.push_back(q);
      qubits.push_back(q + 1);
      params.push_back(-1);
    }
  }
  std::vector<nwq::VqeTerm> t;
  tfim_terms(n, J, hx, t);
  std::vector<uint64_t> xm, zm;
  std::vector<double> co;
  for (const auto& v : t) {
    xm.push_back(v.x);
    zm.push_back(v.z);
    co.push_back(v.c);
  }
  if (g_batch.size() >= kBatchCacheMax) {   // evict the least recently used context
    auto lru = std::min_element(g_batch.begin(), g_batch.end(),
                                [](const BatchEntry& a, const BatchEntry& b) { return a.used < b.used; });
    (void)nwq_vqe_destroy(lru->ctx);
    g_batch.erase(lru);
  }
  BatchEntry e;
  e.device = device;
  e.n = n;
  e.L = L;
  e.J = J;
  e.hx = hx;
  e.terms = t;
  int rc = nwq_vqe_create(n, (int)types.size(), types.data(), qubits.data(), params.data(), 2 * n * L, (int)t.size(),
                          xm.data(), zm.data(), co.data(), stream, &e.ctx);
  if (rc) return rc;
  g_batch.push_back(std::move(e));
  *out = &g_batch.back();
  return NWQ_OK;
}

}  // namespace

extern "C" {

int nwq_vqe_batch(int n, int L, const double* J_h, int B, const double* theta_dev, double* E_dev, double* grad_dev,
                  void* stream) {
  if (n < 1 || n > 30) return vqe_fail(NWQ_ERANGE, "nwq_vqe_batch needs 1..30 qubits");
  if (L < 1 || 2LL * n * L > (1LL << 24)) return vqe_fail(NWQ_EINVAL, "layer count out of range");
  if (!J_h || !std::isfinite(J_h[0]) || !std::isfinite(J_h[1])) return vqe_fail(NWQ_EINVAL, "J_h must hold finite J and h");
  if (B < 1 || B > 65535) return vqe_fail(NWQ_EINVAL, "batch size must be in [1, 65535]");
  if (!theta_dev || !E_dev) return vqe_fail(NWQ_EINVAL, "NULL theta or energy pointer");
  int device = 0;
  int rc = check_hip(hipGetDevice(&device), "hipGetDevice");
  if (rc) return rc;
  std::lock_guard<std::mutex> lock(g_batch_mu);
  BatchEntry* e = nullptr;
  rc = batch_context(device, n, L, J_h[0], J_h[1], stream, &e);
  if (rc) return rc;
  e->used = ++g_batch_clock;
  nwq_vqe_handle h = e->ctx;
  h->user_stream = static_cast<hipStream_t>(stream);
  if (e->J != J_h[0] || e->hx != J_h[1]) {
    // rewrite the term table on the context's stream, after its earlier
    // evaluations; the host copy is reused, so the previous upload from it
    // must have finished
    rc = check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize(vqe batch)");
    e->J = J_h[0];
    e->hx = J_h[1];
    tfim_terms(n, e->J, e->hx, e->terms);
    h->terms = e->terms;
    if (!rc)
      rc = check_hip(hipMemcpyAsync(h->d_terms, e->terms.data(), e->terms.size() * sizeof(nwq::VqeTerm),
                                    hipMemcpyHostToDevice, h->stream), "hipMemcpyAsync(vqe terms)");
    if (rc) return rc;
  }
  return eval_common(h, B, theta_dev, nullptr, E_dev, grad_dev, false);
}

int nwq_vqe_batch_release(void) {
  std::lock_guard<std::mutex> lock(g_batch_mu);
  int rc = NWQ_OK;
  for (auto& e : g_batch) {
    const int r = nwq_vqe_destroy(e.ctx);
    if (r && !rc) rc = r;
  }
  g_batch.clear();
  return rc;
}

}  // extern "C"
