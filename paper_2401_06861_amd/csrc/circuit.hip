// Whole-circuit application and the fusion planner.
//
// The planner walks the gate list and builds blocks: a block owns a tile set
// T = {0..c-1} u H with |H| <= k - c high qubits.  A gate joins the current
// block when its qubits lie in T and none of them is held by an earlier gate
// that was left out (so moving it forward never crosses a gate it does not
// commute with by disjointness).  Left-out gates start the next block.  Each
// block is one read and one write of the state through LDS, so the planner
// picks H for the most gates per block (grow_sets).
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>

#include "engine.h"

namespace nwq {

// The register-blocked kernels run a width of 13 in tiles of 2^12 (unless one
// tile holds the whole register): four workgroups of 2^12 tiles share a CU
// against two of 2^13, which costs more than the fewer blocks of width 13 save
// (with three against one: 30-qubit brickwork 278 ms in 32 blocks against 300 in
// 29; random pairs on 24 qubits 1.48 against 1.96).
int fusion_width(const nwq_state* h, int nbits) {
  return h->fuse_rb != 0 && nbits > h->fuse_k ? std::min(h->fuse_k, 12) : h->fuse_k;
}

// Fewer low bits leave room for more of the circuit's bits per block and give
// shorter HBM runs.  State vectors take as few as the block's 8 high slots
// allow (at least 3: whole 128-byte lines): at width 12 the depth-40 brickwork
// on 30 qubits runs in 260 ms with 4 low bits (32 blocks), 301 with 5 (40), 344
// with 6 (51) and 462 with 7 (74); 384 gates on random pairs of 24 qubits in
// 2.90 ms (25), 3.11 (27), 3.48 (30) and 3.63 (35).  On vec(rho) a qubit above
// the low bits takes two high slots (its column bit q and row bit q + n);
// density matrices keep at least 4 (n=14, width 12, noisy TFIM: 50 ms and 25
// blocks with 4, 76 ms and 41 with 5).
int fusion_low_bits(const nwq_state* h, int nbits) {
  const int k = fusion_width(h, nbits);
  if (nbits <= k) return nbits;
  const int c = h->fuse_c > 0 ? h->fuse_c : (h->kind == NWQ_KIND_DM ? 4 : 3);
  return std::min(std::max(c, k - 8), k - 2);
}

// ---------------------------------------------------------------------------
// Splitting a gate list into sets of bits (a block's high qubits, a phase's
// register bits).  Each round grows one set H (at most `room` bits beside the
// always-present `low` bits) from a first gate's bits, by the bits of a gate
// waiting at the front that lets the most gates in per added bit, and takes
// every gate the set then reaches.  Growing by gain follows the light cone of
// the bits it holds instead of the order of the list: the depth-40 brickwork
// on 30 qubits needs 32 sets of 12 bits (4 low) where taking gates in list
// order until the set is full needed 73 of 13, and the 20-qubit, 8-layer VQE
// ansatz 6 of 12 bits instead of 17.  `seeds` bounds the first gates tried per round
// (the set that takes the most gates is kept).
//
// The gates on one bit are taken in order, so what has been taken is a place
// in each bit's list of gates, and trying a bit visits only the gates that it
// lets in.  (Walking the list itself, a search stops early only when every bit
// is held by a gate left out: 43000 gates of a brickwork on 29 of 30 qubits
// took 1280 ms to plan, now 10.)
// Returns false when a gate needs more than `room` bits outside `low`.
// ---------------------------------------------------------------------------
namespace {

typedef unsigned long long u64;
inline int bits_of(u64 m) { return __builtin_popcountll(m); }

struct BitSet {
  u64 H = 0;                 // bits of the set outside low
  std::vector<int> gates;    // positions in the mask list, in order
};

// The gates on each bit, in list order, ended by -1.
struct BitLists {
  const std::vector<u64>& masks;
  u64 used = 0;
  std::array<int, 65> first{};   // bit b's gates: items from first[b] on
  std::vector<int> items;

  explicit BitLists(const std::vector<u64>& m) : masks(m) {
    for (u64 v : m) {
      used |= v;
      for (; v; v &= v - 1) ++first[__builtin_ctzll(v) + 1];
    }
    const int nb = 64 - __builtin_clzll(used | 1ull);
    for (int b = 0; b < nb; ++b) first[b + 1] += first[b] + 1;
    items.assign(first[nb], -1);
    std::array<int, 65> at(first);
    for (size_t i = 0; i < m.size(); ++i)
      for (u64 v = m[i]; v; v &= v - 1) items[at[__builtin_ctzll(v)]++] = (int)i;
  }
};

// How far each bit's gates have been taken, and the gates that wait next on all
// their bits.
struct Front {
  std::array<int, 64> at;
  std::array<int, 64> wait;   // gates on different bits
  int nwait = 0;

  // Whether g, next on bit b, is next on all its bits.
  bool ready(const BitLists& l, int g, int b) const {
    for (u64 v = l.masks[g] & ~(1ull << b); v; v &= v - 1)
      if (l.items[at[__builtin_ctzll(v)]] != g) return false;
    return true;
  }
  bool waits(const BitLists& l, int g) const { return l.items[at[__builtin_ctzll(l.masks[g])]] == g; }

  // Takes every gate inside T that can be taken, given that only gates on
  // `from` can start; returns their weight (a gate of several bits weighs more:
  // one-bit gates join whichever set holds their bit).
  int take(const BitLists& l, u64 T, u64 from, std::vector<int>* taken = nullptr) {
    int weight = 0;
    for (u64 work = from & T; work;) {
      const int b = __builtin_ctzll(work);
      work &= work - 1;
      for (int g; (g = l.items[at[b]]) >= 0 && ready(l, g, b);) {
        const u64 m = l.masks[g];
        if (m & ~T) {
          if (std::find(wait.begin(), wait.begin() + nwait, g) == wait.begin() + nwait) wait[nwait++] = g;
          break;
        }
        for (u64 v = m; v; v &= v - 1) ++at[__builtin_ctzll(v)];
        work |= m & ~(1ull << b);
        weight += (m & (m - 1)) ? 4 : 1;
        if (taken) taken->push_back(g);
      }
    }
    int n = 0;
    for (int i = 0; i < nwait; ++i)
      if (waits(l, wait[i])) wait[n++] = wait[i];
    nwait = n;
    return weight;
  }
  // The weight that take() would return.
  int weigh(const BitLists& l, u64 T, u64 from, std::vector<int>& taken) {
    taken.clear();
    int weight = 0;
    for (u64 work = from & T; work;) {
      const int b = __builtin_ctzll(work);
      work &= work - 1;
      for (int g; (g = l.items[at[b]]) >= 0;) {
        const u64 m = l.masks[g];
        if ((m & ~T) || !ready(l, g, b)) break;
        for (u64 v = m; v; v &= v - 1) ++at[__builtin_ctzll(v)];
        work |= m & ~(1ull << b);
        weight += (m & (m - 1)) ? 4 : 1;
        taken.push_back(g);
      }
    }
    for (int g : taken)
      for (u64 v = l.masks[g]; v; v &= v - 1) --at[__builtin_ctzll(v)];
    return weight;
  }
};

bool grow_sets(const std::vector<u64>& masks, u64 low, int room, int seeds, std::vector<BitSet>& out) {
  u64 high = 0;
  for (u64 m : masks) high |= m & ~low;
  if (high == 0) {   // one set holds every gate
    out.resize(masks.empty() ? 0 : 1);
    for (size_t i = 0; i < masks.size(); ++i) out[0].gates.push_back((int)i);
    return true;
  }
  const BitLists lists(masks);
  Front done;
  std::copy(lists.first.begin(), lists.first.end() - 1, done.at.begin());
  for (u64 v = lists.used; v; v &= v - 1) {
    const int b = __builtin_ctzll(v), g = lists.items[done.at[b]];
    if (b == __builtin_ctzll(masks[g]) && done.ready(lists, g, b)) done.wait[done.nwait++] = g;
  }
  std::vector<int> tried, taken, best_taken;
  tried.reserve(64);
  std::array<u64, 64> front, seen;   // first gates' bits; bits tried
  std::array<double, 64> gains;      // and what they gained
  // Grows H on f, from f's gates inside low and H on; returns the weight taken.
  auto grow = [&](Front& f, u64& H) {
    int score = f.take(lists, low | H, lists.used, &taken);
    for (;;) {
      const int free = room - bits_of(H);
      const u64 T = low | H;
      double gain_best = -1.0;
      int gate_best = 0, nseen = 0;   // ties: the first in the list
      u64 add = 0;
      for (int i = 0; i < f.nwait; ++i) {
        const int g = f.wait[i];
        const u64 need = masks[g] & ~T;
        if (bits_of(need) > free) continue;
        const int at = (int)(std::find(seen.begin(), seen.begin() + nseen, need) - seen.begin());
        if (at == nseen) {
          seen[nseen] = need;
          gains[nseen++] = (double)f.weigh(lists, T | need, need, tried) / bits_of(need);
        }
        if (gains[at] > gain_best || (gains[at] == gain_best && g < gate_best)) {
          gain_best = gains[at];
          gate_best = g;
          add = need;
        }
      }
      if (add == 0) return score;
      H |= add;
      score += f.take(lists, low | H, add, &taken);
    }
  };
  while (done.nwait > 0) {
    // in list order: the first gate's bits, then evenly spaced ones
    std::sort(done.wait.begin(), done.wait.begin() + done.nwait);
    if (bits_of(masks[done.wait[0]] & ~low) > room) return false;
    int nfront = 0;
    for (int i = 0; i < done.nwait && (seeds > 1 || nfront == 0); ++i) {
      const u64 m = masks[done.wait[i]] & ~low;
      if (bits_of(m) <= room && std::find(front.begin(), front.begin() + nfront, m) == front.begin() + nfront)
        front[nfront++] = m;
    }
    const int tries = std::min(seeds, nfront);
    u64 best_H = front[0];
    if (tries == 1) {
      taken.clear();
      grow(done, best_H);
    } else {
      const Front from = done;
      int best_score = -1;
      for (int t = 0; t < tries; ++t) {
        u64 H = front[t * nfront / tries];
        Front f = from;
        taken.clear();
        const int score = grow(f, H);
        if (score > best_score) {
          best_score = score;
          best_H = H;
          done = f;
          best_taken.swap(taken);
        }
      }
      taken.swap(best_taken);
    }
    std::sort(taken.begin(), taken.end());
    BitSet b;
    b.H = best_H;
    b.gates = taken;
    out.push_back(std::move(b));
  }
  return true;
}

// The sets of a list planned from its end: a plan of the reversed list, read
// backwards, is a plan of the list.
bool grow_sets_from_end(const std::vector<u64>& masks, u64 low, int room, int seeds, std::vector<BitSet>& out) {
  const std::vector<u64> rev(masks.rbegin(), masks.rend());
  if (!grow_sets(rev, low, room, seeds, out)) return false;
  const int last = (int)masks.size() - 1;
  std::reverse(out.begin(), out.end());
  for (BitSet& b : out) {
    std::reverse(b.gates.begin(), b.gates.end());
    for (int& i : b.gates) i = last - i;
  }
  return true;
}

// Passes over the state that a plan costs from |0...0>: per block the share of
// the tiles that can be nonzero (see apply_fused).
double passes_from_zero(const std::vector<BitSet>& sets, u64 all, u64 low) {
  double cost = 0.0;
  u64 support = 0;
  for (const BitSet& b : sets) {
    const u64 T = low | b.H;
    cost += std::ldexp(1.0, bits_of(support & ~T) - bits_of(all & ~T));
    support |= T;
  }
  return cost;
}

}  // namespace

// First gates tried per block of a circuit.  The search is widened as the
// passes it saves get dearer: a pass over 2^22 entries takes about 25 us, and
// each seed adds about 0.05 ms to planning a deep circuit.  Where it is one, a
// state vector's register phases too are searched once, from the front (fused
// circuits of 250 to 300 gates on 14 to 20 qubits 250-390 -> 235-365 us; at 22
// qubits no gain; a density matrix's phases are dearer than their search).
static int plan_seeds(int nbits) { return nbits < 22 ? 1 : (nbits < 26 ? 2 : 8); }

// Every block has at least two high slots (c <= k - 2), so the first
// remaining one- or two-qubit gate always fits and each round absorbs at
// least one gate (a four-bit DM superoperator is queued only when the width
// leaves four).  Planned from both ends of the list; the plan with fewer
// blocks is kept, or with `from_zero` (the plan only ever runs from |0...0>)
// the one with fewer passes.  Circuits plan the same way from any state, so
// that nwq_run_circuit gives the bits of nwq_reset + nwq_apply_circuit.
std::vector<Block> plan_blocks(const std::vector<PGate>& g, int n, int k, int c_req, int seeds, bool from_zero) {
  const int c = n <= k ? n : std::min(std::max(c_req, k - 8), k - 2);
  const int room = n <= k ? 0 : k - c;
  std::vector<u64> masks(g.size());
  for (size_t i = 0; i < g.size(); ++i)
    for (int j = 0; j < g[i].nq; ++j) masks[i] |= 1ull << g[i].q[j];
  const u64 all = (1ull << n) - 1ull, low = (1ull << c) - 1ull;
  std::vector<BitSet> sets, other;
  if (!grow_sets(masks, low, room, seeds, sets)) return {};   // cannot happen with two high slots; caller reports it
  if (sets.size() > 1 && grow_sets_from_end(masks, low, room, seeds, other)) {
    const double a = passes_from_zero(sets, all, low), b = passes_from_zero(other, all, low);
    if (from_zero ? b < a : (other.size() < sets.size() || (other.size() == sets.size() && b < a))) sets.swap(other);
  }
  std::vector<Block> out(sets.size());
  for (size_t i = 0; i < sets.size(); ++i) {
    out[i].c = c;
    for (int q = c; q < n; ++q)
      if ((sets[i].H >> q) & 1ull) out[i].hi[out[i].m++] = q;
    out[i].gates = std::move(sets[i].gates);
  }
  return out;
}

// Widen a block's tile with unused high qubits (ascending) up to width
// k_target (or n): more amplitudes per tile, same gates, same result.
void pad_block(Block& b, int n, int k_target) {
  const int want = std::min(k_target, n);
  for (int q = b.c; q < n && b.c + b.m < want && b.m < 8; ++q) {
    bool used = false;
    for (int i = 0; i < b.m; ++i) used |= b.hi[i] == q;
    if (!used) b.hi[b.m++] = q;
  }
  std::sort(b.hi, b.hi + b.m);
}

int local_bit(const Block& b, int q) {
  if (q < b.c) return q;
  for (int i = 0; i < b.m; ++i)
    if (b.hi[i] == q) return b.c + i;
  return -1;
}

// Encode one gate as a FusedOp of the per-gate LDS kernel (tile-local bits)
// and append its matrix entries.  Returns false for the identity (nothing to do).
static bool encode_op(const PGate& g, int b0, int b1, std::vector<double2>& mats, FusedOp& op,
                      const std::vector<cd>* side) {
  cd own[16];
  const cd* m = own;
  if (g.type == kGateDiag4 || g.type == kGateMat2 || g.type == kGateMat4) m = side->data() + (size_t)g.p[0];
  else gate_matrix(g.type, g.p, own);
  op = FusedOp{};
  op.mat = (int)mats.size();
  op.lo = g.nq == 2 ? std::min(b0, b1) : b0;
  op.hi = g.nq == 2 ? std::max(b0, b1) : 0;
  auto put = [&](const cd& v) { mats.push_back(make_double2(v.real(), v.imag())); };
  switch (g.type) {
    case NWQ_GATE_I:
      return false;
    case NWQ_GATE_CX:
      op.kind = 3;
      op.o0 = 1 << b0;
      op.o1 = (1 << b0) + (1 << b1);
      return true;
    case NWQ_GATE_SWAP:
      op.kind = 3;
      op.o0 = 1 << b0;
      op.o1 = 1 << b1;
      return true;
    case NWQ_GATE_CZ: case NWQ_GATE_RZZ: case kGateDiag4:   // operator order (q[0], q[1])
      op.kind = 4;
      op.o0 = b0;
      op.o1 = b1;
      for (int u = 0; u < 4; ++u) put(m[5 * u]);
      return true;
    case kGateMat4:   // operator order (q[0], q[1])
      op.kind = 2;
      op.o0 = 1 << b0;
      op.o1 = 1 << b1;
      for (int i = 0; i < 16; ++i) put(m[i]);
      return true;
    default:
      if (m[1] == 0.0 && m[2] == 0.0) {
        op.kind = 1;
        put(m[0]);
        put(m[3]);
      } else {
        op.kind = 0;
        for (int i = 0; i < 4; ++i) put(m[i]);
      }
      return true;
  }
}

// ---------------------------------------------------------------------------
// Ops of a register phase (register-blocked kernels)
// ---------------------------------------------------------------------------
namespace {

struct RegOp {
  enum Kind { DENSE1, DENSE2, CX, SWAP, DIAG, DENSE16 } kind;
  int b0 = 0, b1 = 0;        // register bits, operator order (CX: control, target)
  unsigned bits = 0;         // register bits it acts on (DIAG: bits its entries depend on)
  std::vector<cd> m;         // DENSE1: 2x2; DENSE2: 4x4 in the order (b0, b1); DIAG: an entry per
                             // register; DENSE16: the 16x16 in register order
  bool perm() const { return kind == CX || kind == SWAP; }
  int map(int j) const { return kind == CX ? reg_cx(b0, b1, j) : reg_swap(b0, b1, j); }
};

// Gate g on register bits rb[0 .. nq).  Returns false for the identity.
bool make_reg_op(const PGate& g, const int* rb, int rbits, const std::vector<cd>* side, RegOp& op) {
  const int nv = 1 << rbits;
  cd own[16];
  const cd* m = own;
  if (g.type >= kGateMat4) m = side->data() + (size_t)g.p[0];
  else gate_matrix(g.type, g.p, own);
  op = RegOp{};
  op.b0 = rb[0];
  op.b1 = g.nq >= 2 ? rb[1] : 0;
  for (int t = 0; t < g.nq; ++t) op.bits |= 1u << rb[t];
  switch (g.type) {
    case NWQ_GATE_I:
      return false;
    case NWQ_GATE_CX:
      op.kind = RegOp::CX;
      return true;
    case NWQ_GATE_SWAP:
      op.kind = RegOp::SWAP;
      return true;
    case NWQ_GATE_CZ: case NWQ_GATE_RZZ: case kGateDiag4:
      op.kind = RegOp::DIAG;
      for (int j = 0; j < nv; ++j) op.m.push_back(m[5 * (((j >> rb[0]) & 1) + 2 * ((j >> rb[1]) & 1))]);
      return true;
    case kGateMat4:
      op.kind = RegOp::DENSE2;
      op.m.assign(m, m + 16);
      return true;
    case kGateMat16: {   // operator index bit t on register bit rb[t]
      op.kind = RegOp::DENSE16;
      int inv[16];
      for (int u = 0; u < 16; ++u) {
        int j = 0;
        for (int t = 0; t < 4; ++t) j |= ((u >> t) & 1) << rb[t];
        inv[j] = u;
      }
      op.m.resize(256);
      for (int r = 0; r < 16; ++r)
        for (int c = 0; c < 16; ++c) op.m[r * 16 + c] = m[inv[r] * 16 + inv[c]];
      return true;
    }
    default:
      if (m[1] == 0.0 && m[2] == 0.0) {
        op.kind = RegOp::DIAG;
        for (int j = 0; j < nv; ++j) op.m.push_back(m[((j >> rb[0]) & 1) ? 3 : 0]);
      } else {
        op.kind = RegOp::DENSE1;
        op.m.assign(m, m + 4);
      }
      return true;
  }
}

// Diagonal ops of a phase move to the front, past ops on other bits and past
// permutations (D P = P D' with D'[j] = D[P(j)]), and merge with a diagonal
// they meet: the kernel applies any diagonal over the register bits with one
// complex product per amplitude, so the RZZ chain of a Trotter step costs one
// op per phase instead of one per gate.
void merge_diagonals(std::vector<RegOp>& ops, int rbits) {
  const int nv = 1 << rbits;
  std::vector<RegOp> out;
  for (RegOp& op : ops) {
    if (op.kind != RegOp::DIAG) {
      out.push_back(std::move(op));
      continue;
    }
    std::vector<cd> d = op.m, keep = op.m;   // keep: its form behind the op it stops at
    unsigned bits = op.bits;
    bool merged = false;
    for (size_t i = out.size(); i-- > 0;) {
      RegOp& o = out[i];
      if (o.kind == RegOp::DIAG) {
        for (int j = 0; j < nv; ++j) o.m[j] *= d[j];
        o.bits |= bits;
        merged = true;
        break;
      }
      if (!(o.bits & bits)) continue;
      if (!o.perm()) break;
      std::vector<cd> e(nv);
      for (int j = 0; j < nv; ++j) e[j] = d[o.map(j)];
      d.swap(e);
      bits |= o.bits;
    }
    if (!merged) {
      op.m = keep;
      out.push_back(std::move(op));
    }
  }
  ops.swap(out);
}

// The op's code, its entries appended to mats.
RbOp emit_reg_op(const RegOp& op, int set, std::vector<double2>& mats) {
  RbOp o{0, (int)mats.size()};
  auto put = [&](const cd& v) { mats.push_back(make_double2(v.real(), v.imag())); };
  auto real = [](const cd& v) { return v.imag() == 0.0; };
  auto imag = [](const cd& v) { return v.real() == 0.0; };
  const std::vector<cd>& m = op.m;
  switch (op.kind) {
    case RegOp::CX:
      o.code = rb_cx_code(op.b0, op.b1);
      break;
    case RegOp::SWAP:
      o.code = kRbSwap + rb_pair(std::min(op.b0, op.b1), std::max(op.b0, op.b1));
      break;
    case RegOp::DIAG:
      o.code = kRbDiagAll;
      for (const cd& v : m) put(v);
      break;
    case RegOp::DENSE1:
      if (real(m[0]) && real(m[1]) && real(m[2]) && real(m[3])) o.code = kRbReal1 + op.b0;
      else if (real(m[0]) && imag(m[1]) && imag(m[2]) && real(m[3])) o.code = kRbXt1 + op.b0;
      else if (real(m[0])) o.code = kRbR001 + op.b0;
      else o.code = kRbGen1 + op.b0;
      for (const cd& v : m) put(v);
      break;
    case RegOp::DENSE2: {
      const bool sw = op.b0 > op.b1;   // to index order (lower bit, higher bit)
      auto at = [&](int u) { return sw ? ((u & 1) << 1) | (u >> 1) : u; };
      bool all_real = set == kRbSetDM, parity = set == kRbSetDM;
      for (int r = 0; r < 4; ++r)
        for (int c = 0; c < 4; ++c) {
          const cd v = m[at(r) * 4 + at(c)];
          put(v);
          all_real = all_real && real(v);
          parity = parity && (__builtin_popcount(r ^ c) % 2 == 0 ? real(v) : imag(v));
        }
      o.code = (all_real ? kRbReal2 : (parity ? kRbPar2 : kRbDense2)) + rb_pair(std::min(op.b0, op.b1), std::max(op.b0, op.b1));
      break;
    }
    case RegOp::DENSE16: {
      // a Pauli channel after a diagonal gate (RZZ, CZ, ...) leaves the
      // entries of rho off the 4x4 diagonal scaled and mixes only the
      // diagonal ones (registers 0, 5, 10, 15 in either qubit order)
      bool pauli = true;
      for (int r = 0; r < 16 && pauli; ++r)
        for (int c = 0; c < 16 && pauli; ++c)
          if (r != c && !(r % 5 == 0 && c % 5 == 0) && m[r * 16 + c] != 0.0) pauli = false;
      o.code = pauli ? kRbPauli16 : kRbDense16;
      if (pauli) {
        for (int u = 0; u < 16; ++u) put(m[u * 17]);
        for (int i = 0; i < 4; ++i)
          for (int j = 0; j < 4; ++j) put(m[5 * i * 16 + 5 * j]);
      } else {
        for (const cd& v : m) put(v);
      }
      break;
    }
  }
  return o;
}

}  // namespace

// ---------------------------------------------------------------------------
// Gate products.  A two-qubit gate takes the one-qubit gates next to it on
// its two qubits (back to the previous and on to the next two-qubit gate on
// each: each of them commutes with everything it is moved past) and the
// product becomes one gate, when that costs less FP64 work than the gates one
// by one.  Runs of one-qubit gates on one qubit that are left become one 2x2
// the same way.  Costs are FP64 instructions per amplitude in the
// register-blocked kernel plus one per op for its dispatch.  Products act on
// at most two qubits, so blocks and register phases are planned over them as
// over gates.
// ---------------------------------------------------------------------------
namespace {

struct FuseItem {
  int gate = -1;              // an original gate (index into the gate list), or -1: a product
  int nb = 0, r[2] = {0, 0};  // product: its qubits; r[0] is bit 0 of the operator index
  cd m[16];                   // product: 2x2 (nb = 1) or 4x4 (nb = 2), row-major
};

bool is_diag(const cd* m, int dim) {
  for (int u = 0; u < dim; ++u)
    for (int v = 0; v < dim; ++v)
      if (u != v && m[u * dim + v] != 0.0) return false;
  return true;
}

int matrix_cost(const cd* m, int nb) {
  if (nb == 2) return is_diag(m, 4) ? 4 : 16;
  if (is_diag(m, 2)) return 4;
  auto real = [](const cd& v) { return v.imag() == 0.0; };
  auto imag = [](const cd& v) { return v.real() == 0.0; };
  if (real(m[0]) && real(m[3]) && ((real(m[1]) && real(m[2])) || (imag(m[1]) && imag(m[2])))) return 4;
  return real(m[0]) ? 7 : 8;
}

int gate_cost(const PGate& g) {
  switch (g.type) {
    case NWQ_GATE_I: return 0;
    case NWQ_GATE_CX: case NWQ_GATE_SWAP: return 0;   // register permutations
    case NWQ_GATE_CZ: case NWQ_GATE_RZZ: return 4;
    case kGateMat4: return 16;
    case kGateDiag4: return 4;
    default: {
      cd m[16];
      gate_matrix(g.type, g.p, m);
      return matrix_cost(m, 1);
    }
  }
}

// M <- G M, G acting on bit `pos` (0 or 1) of the 4x4 operator index
void lmul_1q(cd* M, const cd* G, int pos) {
  cd R[16];
  for (int u = 0; u < 4; ++u)
    for (int v = 0; v < 4; ++v) {
      cd acc = 0.0;
      for (int w = 0; w < 4; ++w)
        if ((u & ~(1 << pos)) == (w & ~(1 << pos))) acc += G[((u >> pos) & 1) * 2 + ((w >> pos) & 1)] * M[w * 4 + v];
      R[u * 4 + v] = acc;
    }
  std::memcpy(M, R, sizeof R);
}

// M <- G M, G a 4x4 in its own (q0, q1) index order; swapped: q0 is bit 1 here
void lmul_2q(cd* M, const cd* G, bool swapped) {
  auto sw = [&](int u) { return swapped ? ((u & 1) << 1) | (u >> 1) : u; };
  cd R[16];
  for (int u = 0; u < 4; ++u)
    for (int v = 0; v < 4; ++v) {
      cd acc = 0.0;
      for (int w = 0; w < 4; ++w) acc += G[sw(u) * 4 + sw(w)] * M[w * 4 + v];
      R[u * 4 + v] = acc;
    }
  std::memcpy(M, R, sizeof R);
}

// seq: the gates in order (indices into gates); r0 / r1: their qubits (r1 <
// 0 for one-qubit gates).  Returns the ops in application order.
std::vector<FuseItem> gate_products(const std::vector<int>& seq, const std::vector<PGate>& gates,
                                  const std::vector<int>& r0, const std::vector<int>& r1) {
  const int n = (int)seq.size();
  auto two = [&](int i) { return r1[i] >= 0; };
  // positions touching each bit, and each position's place in its bits' lists
  int nbit = 0;
  for (int i = 0; i < n; ++i) nbit = std::max(nbit, std::max(r0[i], r1[i]) + 1);
  std::vector<std::vector<int>> on(nbit);
  std::vector<int> at0(n), at1(n, -1);
  for (int i = 0; i < n; ++i) {
    at0[i] = (int)on[r0[i]].size();
    on[r0[i]].push_back(i);
    if (two(i)) {
      at1[i] = (int)on[r1[i]].size();
      on[r1[i]].push_back(i);
    }
  }
  std::vector<int> owner(n, -1), unit_at(n, -1);
  std::vector<FuseItem> units;
  for (int p = 0; p < n; ++p) {
    if (!two(p)) continue;
    std::vector<int> take;
    for (int side = 0; side < 2; ++side) {
      const std::vector<int>& lst = on[side == 0 ? r0[p] : r1[p]];
      const int here = side == 0 ? at0[p] : at1[p];
      for (int j = here - 1; j >= 0; --j) {
        const int t = lst[j];
        if (two(t) || owner[t] != -1) break;
        take.push_back(t);
      }
      for (int j = here + 1; j < (int)lst.size(); ++j) {
        const int t = lst[j];
        if (two(t)) break;
        take.push_back(t);
      }
    }
    if (take.empty()) continue;
    take.push_back(p);
    std::sort(take.begin(), take.end());
    FuseItem u;
    u.nb = 2;
    u.r[0] = r0[p];
    u.r[1] = r1[p];
    for (int i = 0; i < 16; ++i) u.m[i] = (i % 5 == 0) ? 1.0 : 0.0;
    int unfused = 0;
    for (int i : take) {
      const PGate& g = gates[seq[i]];
      unfused += gate_cost(g) + 1;
      cd G[16];
      gate_matrix(g.type, g.p, G);
      if (two(i)) lmul_2q(u.m, G, r0[i] != u.r[0]);
      else lmul_1q(u.m, G, r0[i] == u.r[0] ? 0 : 1);
    }
    if (matrix_cost(u.m, 2) + 1 >= unfused) continue;
    for (int i : take) owner[i] = (int)units.size();
    unit_at[p] = (int)units.size();
    units.push_back(u);
  }
  std::vector<FuseItem> out;
  for (int i = 0; i < n; ++i) {
    if (unit_at[i] >= 0) {
      out.push_back(units[unit_at[i]]);
      continue;
    }
    if (owner[i] != -1) continue;
    if (two(i)) {
      out.push_back(FuseItem{});
      out.back().gate = seq[i];
      continue;
    }
    std::vector<int> run{i};
    const std::vector<int>& lst = on[r0[i]];
    for (int j = at0[i] + 1; j < (int)lst.size(); ++j) {
      const int t = lst[j];
      if (two(t) || owner[t] != -1) break;
      run.push_back(t);
    }
    FuseItem u;
    u.nb = 1;
    u.r[0] = r0[i];
    u.m[0] = u.m[3] = 1.0;
    int unfused = 0;
    for (int t : run) {
      const PGate& g = gates[seq[t]];
      unfused += gate_cost(g) + 1;
      cd G[16];
      gate_matrix(g.type, g.p, G);
      const cd a = G[0] * u.m[0] + G[1] * u.m[2], b = G[0] * u.m[1] + G[1] * u.m[3];
      const cd c = G[2] * u.m[0] + G[3] * u.m[2], d = G[2] * u.m[1] + G[3] * u.m[3];
      u.m[0] = a; u.m[1] = b; u.m[2] = c; u.m[3] = d;
    }
    if (run.size() > 1 && matrix_cost(u.m, 1) + 1 < unfused) {
      for (int t : run) owner[t] = -2;
      out.push_back(u);
    } else {
      out.push_back(FuseItem{});
      out.back().gate = seq[i];
    }
  }
  return out;
}

}  // namespace

// Split a block's gates (tile-local bits) into register phases of at most
// rbits bits (grow_sets); pad each set to rbits, from tile bit c up first (a
// set above the low c bits keeps each wave's lanes on contiguous amplitudes,
// so the phase can move between registers and HBM directly when it is the
// block's first or last).  Empty when a gate has more than rbits bits.
std::vector<Phase> plan_phases(const std::vector<int>& order, const std::vector<std::array<int, 4>>& lb,
                               const std::vector<int>& nq, int k, int c, int rbits, bool quick) {
  std::vector<u64> masks(order.size());
  for (size_t i = 0; i < order.size(); ++i)
    for (int t = 0; t < nq[order[i]]; ++t) masks[i] |= 1ull << lb[order[i]][t];
  std::vector<BitSet> sets, other;
  if (!grow_sets(masks, 0, rbits, quick ? 1 : 2, sets)) return {};
  if (!quick && sets.size() > 1 && grow_sets_from_end(masks, 0, rbits, 2, other) && other.size() < sets.size())
    sets.swap(other);
  std::vector<Phase> out(sets.size());
  for (size_t i = 0; i < sets.size(); ++i) {
    unsigned S = (unsigned)sets[i].H;
    for (int b = c; b < k && __builtin_popcount(S) < rbits; ++b) S |= 1u << b;
    for (int b = 0; b < k && __builtin_popcount(S) < rbits; ++b) S |= 1u << b;
    Phase& ph = out[i];
    int r = 0;
    for (int b = 0; b < k; ++b)
      if ((S >> b) & 1u) ph.reg[r++] = b;
    for (; r < 4; ++r) ph.reg[r] = -1;
    for (int p : sets[i].gates) ph.gates.push_back(order[p]);
  }
  return out;
}

// Global offset of tile entry l: the low c bits stay in place, tile bit c + i
// lands on qubit hi[i].
static unsigned long long tile_entry_offset(int c, int m, const int* hi, unsigned l) {
  unsigned long long g = l & ((1u << c) - 1u);
  for (int i = 0; i < m; ++i)
    if ((l >> (c + i)) & 1u) g |= 1ull << hi[i];
  return g;
}

namespace {

// Images of the thread bits and register bits of a phase in tile entries
// (perm: the register-bit index a register's entry is read from or stored to;
// compositions of CX and SWAP are linear over GF(2)).  wave: the tile bits on
// the thread index above the lane (threads of one wave agree on them).
struct TileMap {
  int tbits = 0;
  unsigned t[kRbThreadBits] = {0}, r[4] = {0};
};
TileMap tile_map(const int* reg, const int* perm, unsigned wave, int rbits, int k, int banks) {
  TileMap m;
  unsigned S = wave;
  for (int i = 0; i < rbits; ++i) S |= 1u << reg[i];
  // 2^banks consecutive lanes (one LDS access of 128 bytes) have to cover
  // different banks: the low lane bits take tile bits of different residue
  // mod `banks` (entry_slot), the lowest ones.
  unsigned lanes = ~S & ((1u << k) - 1u), res = 0;
  for (int b = 0; b < k && res + 1 != 1u << banks; ++b)
    if (((lanes >> b) & 1u) && !((res >> (b % banks)) & 1u)) {
      res |= 1u << (b % banks);
      m.t[m.tbits++] = 1u << b;
      lanes &= ~(1u << b);
    }
  for (unsigned rest : {lanes, wave})
    for (int b = 0; b < k; ++b)
      if ((rest >> b) & 1u) m.t[m.tbits++] = 1u << b;
  for (int i = 0; i < rbits; ++i)
    for (int e = 0; e < rbits; ++e)
      if ((perm[1 << i] >> e) & 1) m.r[i] |= 1u << reg[e];
  return m;
}

}  // namespace

// LDS slot of a tile entry: bit i < banks is the parity of the entry's bits
// that are i mod banks, so that a step along any tile bit changes the bank.
unsigned short entry_slot(unsigned entry, int banks) {
  unsigned low = 0;
  for (int b = 0; b < 16; b += banks) low ^= entry >> b;
  const unsigned m = (1u << banks) - 1u;
  return (unsigned short)((entry & ~m) | (low & m));
}

// Lays register phases out over the k bits of a tile (appends them to `out`):
// lanes of the first and last keep the `low` low bits, entries of the LDS
// exchanges are 128 >> banks bytes.
void layout_phases(const std::vector<RbStage>& st, int rbits, int k, int low, int banks, std::vector<RbPhase>& out,
                   RbTileIo& io) {
  // Bits of the wave index: phases in a row share them as long as enough bits
  // above the low ones stay off all their register bits (the exchanges between
  // such phases stay inside a wave).
  const int wbits = std::max(0, k - rbits - 6);
  std::vector<unsigned> wave(st.size(), 0);
  std::vector<char> local(st.size(), 0);   // exchange into phase i stays inside a wave
  for (size_t i = 0; i < st.size();) {
    unsigned busy = (1u << std::min(low, std::max(0, k - rbits - wbits))) - 1u;
    size_t e = i;
    for (; e < st.size(); ++e) {
      unsigned S = busy;
      for (int r = 0; r < rbits; ++r) S |= 1u << st[e].reg[r];
      if (e > i && k - __builtin_popcount(S) < wbits) break;
      busy = S;
      if (k - __builtin_popcount(S) < wbits) {   // one phase: its lanes give up low bits
        busy = 0;
        for (int r = 0; r < rbits; ++r) busy |= 1u << st[e].reg[r];
        ++e;
        break;
      }
    }
    unsigned W = 0;
    for (int q = k - 1, n = 0; q >= 0 && n < wbits; --q)
      if (!((busy >> q) & 1u)) {
        W |= 1u << q;
        ++n;
      }
    for (size_t j = i; j < e; ++j) {
      wave[j] = W;
      local[j] = j > i || (j > 0 && wave[j - 1] == W);
    }
    i = e;
  }
  bool all_local = true;
  for (size_t i = 1; i < st.size(); ++i) all_local = all_local && local[i];
  for (size_t i = 0; i < st.size(); ++i) {
    RbPhase ph{};
    ph.op_begin = st[i].op_begin;
    ph.count_flags = st[i].op_count << kRbFlagBits;
    if (i > 0) {
      const TileMap wr = tile_map(st[i - 1].reg, st[i - 1].st_perm, wave[i - 1], rbits, k, banks);
      const TileMap rd = tile_map(st[i].reg, st[i].ld_perm, wave[i], rbits, k, banks);
      for (int j = 0; j < kRbThreadBits; ++j) {
        ph.wr_t[j] = entry_slot(wr.t[j], banks);
        ph.rd_t[j] = entry_slot(rd.t[j], banks);
      }
      for (int j = 0; j < 4; ++j) {
        ph.wr_r[j] = entry_slot(wr.r[j], banks);
        ph.rd_r[j] = entry_slot(rd.r[j], banks);
      }
      // A phase's registers go back to the entries they came from (its
      // permutations stay among one thread's), so only the first exchange of a
      // tile can overwrite entries that another wave still reads: the last
      // phase's of the tile before.
      ph.count_flags |= (local[i] ? 0 : kRbBarrierInside) | (i == 1 && !all_local ? kRbBarrierBefore : 0);
    }
    out.push_back(ph);
  }
  const TileMap ld = tile_map(st.front().reg, st.front().ld_perm, wave.front(), rbits, k, banks);
  const TileMap sv = tile_map(st.back().reg, st.back().st_perm, wave.back(), rbits, k, banks);
  for (int j = 0; j < kRbThreadBits; ++j) {
    io.ld_t[j] = (unsigned short)ld.t[j];
    io.st_t[j] = (unsigned short)sv.t[j];
  }
  for (int j = 0; j < 4; ++j) {
    io.ld_r[j] = (unsigned short)ld.r[j];
    io.st_r[j] = (unsigned short)sv.r[j];
  }
}

// Lays a block's register phases out.  The first and the last phase move
// between HBM and registers themselves, so their lanes have to cover
// contiguous runs (no register bit below the low bits) -- else, or without
// `direct`, a phase without ops on the top bits goes before (after).
void layout_rb_block(const Block& b, std::vector<RbStage> st, int rbits, bool direct, RbBlock& d,
                     std::vector<RbPhase>& out) {
  const int k = b.c + b.m;
  d = RbBlock{};
  d.k = k;
  d.tile = tile_entry_offset(b.c, b.m, b.hi, (1u << k) - 1u);
  auto contiguous = [&](const RbStage& s) {
    for (int r = 0; r < rbits; ++r)
      if (s.reg[r] < std::min(b.c, k - rbits)) return false;
    return true;
  };
  RbStage top{};
  for (int r = 0; r < rbits; ++r) top.reg[r] = k - rbits + r;
  for (int j = 0; j < 16; ++j) top.ld_perm[j] = top.st_perm[j] = j;
  if (!direct || !contiguous(st.front())) {
    top.op_begin = st.front().op_begin;
    st.insert(st.begin(), top);
  }
  if (!direct || !contiguous(st.back())) {
    top.op_begin = st.back().op_begin;
    st.push_back(top);
  }
  d.ph_begin = (int)out.size();
  d.ph_count = (int)st.size();
  RbTileIo io;
  layout_phases(st, rbits, k, std::min(b.c, 4), 4, out, io);   // 256-byte runs at least; doubles
  for (int j = 0; j < kRbThreadBits; ++j) {
    d.ld_t[j] = tile_entry_offset(b.c, b.m, b.hi, io.ld_t[j]);
    d.st_t[j] = tile_entry_offset(b.c, b.m, b.hi, io.st_t[j]);
  }
  for (int j = 0; j < 4; ++j) {
    d.ld_r[j] = tile_entry_offset(b.c, b.m, b.hi, io.ld_r[j]);
    d.st_r[j] = tile_entry_offset(b.c, b.m, b.hi, io.st_r[j]);
  }
}

// Runs a gate list through fused blocks over `nbits` bits of the vector (the
// qubit count for a state vector; 2n for the vectorised density matrix, whose
// queued 1q superoperators arrive as kGateMat4 gates with matrices in `side`).
int apply_fused(nwq_state* h, const std::vector<PGate>& gates_in, int nbits, const std::vector<cd>* side_in,
                bool from_zero, bool one_tile) {
  // One tile: the kernel that is fastest where one workgroup runs everything.
  // Up to 8 bits the LDS kernel (300 gates of a TFIM on 8 qubits 201 us against
  // 216 with R = 3; on 10 qubits 272 against 250), up to 12 bits R = 3 (380
  // gates on 10 qubits 293 us against 313 with R = 4), then R = 4 (500 gates
  // on 13 qubits 494 us against 530).
  const int kernel = one_tile ? (nbits < 9 ? 0 : nbits < 13 ? 2 : 1) : h->fuse_rb;
  const int flags = one_tile ? kFusedDirect : h->fuse_flags;
  // Gate products over the whole circuit (state vectors, register-blocked
  // kernels): they act on at most two qubits, so the blocks and their register
  // phases are planned over them as over gates, and no boundary cuts one.
  std::vector<PGate> prod_gates;
  std::vector<cd> prod_side;
  const bool products = (flags & kFusedGateFusion) && side_in == nullptr && kernel != 0;
  if (products) {
    std::vector<int> seq, r0, r1;
    for (size_t i = 0; i < gates_in.size(); ++i) {
      if (gates_in[i].type == NWQ_GATE_I) continue;
      seq.push_back((int)i);
      r0.push_back(gates_in[i].q[0]);
      r1.push_back(gates_in[i].nq == 2 ? gates_in[i].q[1] : -1);
    }
    for (const FuseItem& it : gate_products(seq, gates_in, r0, r1)) {
      if (it.gate >= 0) {
        prod_gates.push_back(gates_in[it.gate]);
        continue;
      }
      PGate g{};
      g.nq = it.nb;
      g.q[0] = it.r[0];
      g.q[1] = it.nb == 2 ? it.r[1] : 0;
      g.type = it.nb == 1 ? kGateMat2 : (is_diag(it.m, 4) ? kGateDiag4 : kGateMat4);
      g.p[0] = (double)prod_side.size();
      for (int i = 0; i < 16; ++i) prod_side.push_back(it.m[i]);
      prod_gates.push_back(g);
    }
  }
  const std::vector<PGate>& gates = products ? prod_gates : gates_in;
  const std::vector<cd>* side = products ? &prod_side : side_in;
  if (gates.empty()) {   // identities only
    h->last_blocks = h->last_fused_gates = h->last_phases = 0;
    return NWQ_OK;
  }
  const std::vector<Block> blocks = plan_blocks(gates, nbits, one_tile ? nbits : fusion_width(h, nbits),
                                                one_tile ? nbits : fusion_low_bits(h, nbits), plan_seeds(nbits), false);
  if (blocks.empty()) return set_error(NWQ_EINVAL, "fusion planner made no progress");
  // Program: [phase table][op table][matrix table] in one upload.
  std::vector<RbPhase> phases;
  std::vector<FusedOp> ops;    // per-gate LDS kernel
  std::vector<RbOp> rops;      // register-blocked kernels
  std::vector<double2> mats;
  const int set = h->kind == NWQ_KIND_DM ? kRbSetDM : kRbSetSV;
  const bool quick = one_tile || (set == kRbSetSV && plan_seeds(nbits) == 1);
  struct Launch { FusedBlockDev d; RbBlock r; bool rb; };
  const int rbits = kernel == 2 ? 3 : 4;
  std::vector<Launch> launches;
  for (Block b : blocks) {
    if (kernel != 0 && b.c + b.m < 8 && nbits >= 8) pad_block(b, nbits, 8);
    FusedBlockDev d{};
    d.c = b.c;
    d.m = b.m;
    for (int i = 0; i < b.m; ++i) d.hi[i] = b.hi[i];
    const int k = b.c + b.m;
    const bool rb = kernel != 0 && k >= 8;
    if (!rb) {
      d.op_begin = (int)ops.size();
      for (int gi : b.gates) {
        const PGate& g = gates[gi];
        if (g.nq > 2) return set_error(NWQ_EINVAL, "a four-bit operator needs the register-blocked kernel");
        FusedOp op;
        if (encode_op(g, local_bit(b, g.q[0]), g.nq == 2 ? local_bit(b, g.q[1]) : 0, mats, op, side))
          ops.push_back(op);
      }
      d.op_count = (int)ops.size() - d.op_begin;
      if (d.op_count > 0) launches.push_back({d, RbBlock{}, false});
      continue;
    }
    // the block's gates by block-local index (gid: the gate each one is), so
    // that planning costs time in the block's size, not the circuit's
    std::vector<int> gid, nq, order;
    std::vector<std::array<int, 4>> lb;
    for (int gi : b.gates) {
      if (gates[gi].type == NWQ_GATE_I) continue;
      if (gates[gi].nq > rbits) return set_error(NWQ_EINVAL, "an operator wider than the phase's register bits");
      std::array<int, 4> bits{};
      for (int t = 0; t < gates[gi].nq; ++t) bits[t] = local_bit(b, gates[gi].q[t]);
      order.push_back((int)gid.size());
      gid.push_back(gi);
      lb.push_back(bits);
      nq.push_back(gates[gi].nq);
    }
    if (order.empty()) continue;
    const size_t rops0 = rops.size(), mats0 = mats.size();
    std::vector<RbStage> stages;
    for (const Phase& ph : plan_phases(order, lb, nq, k, b.c, rbits, quick)) {
      RbStage stg{};
      for (int i = 0; i < 4; ++i) stg.reg[i] = ph.reg[i] < 0 ? 0 : ph.reg[i];
      stg.op_begin = (int)rops.size();
      auto ridx = [&](int bit) {
        for (int i = 0; i < rbits; ++i)
          if (ph.reg[i] == bit) return i;
        return -1;
      };
      std::vector<RegOp> pops;
      for (int li : ph.gates) {
        int rb_bits[4] = {0, 0, 0, 0};
        for (int t = 0; t < nq[li]; ++t) rb_bits[t] = ridx(lb[li][t]);
        RegOp op;
        if (make_reg_op(gates[gid[li]], rb_bits, rbits, side, op)) pops.push_back(std::move(op));
      }
      if (flags & kFusedGateFusion) merge_diagonals(pops, rbits);
      fold_permutations(
          pops, rbits, [](const RegOp& o) { return o.perm(); }, [](const RegOp& o) { return o.bits; },
          [](const RegOp& o, int j) { return o.map(j); }, stg.ld_perm, stg.st_perm);
      for (const RegOp& o : pops) rops.push_back(emit_reg_op(o, set, mats));
      if (rbits == 4 && pops.size() % 2) rops.push_back(RbOp{kRbCopy, rops.back().mat});
      stg.op_count = (int)rops.size() - stg.op_begin;
      stages.push_back(stg);
    }
    RbBlock r;
    layout_rb_block(b, std::move(stages), rbits, (flags & kFusedDirect) != 0, r, phases);
    r.prog_ops = (int)(rops.size() - rops0);
    r.prog_mats = (int)(mats.size() - mats0);
    launches.push_back({d, r, true});
  }
  const size_t ph_bytes = phases.size() * sizeof(RbPhase);
  const size_t ops_off = (ph_bytes + 255) & ~size_t(255);
  const size_t ops_bytes = ops.size() * sizeof(FusedOp);
  for (int i = 0; i < 2; ++i) rops.push_back(RbOp{kRbCopy, 0});   // read ahead, not run
  const size_t rops_off = (ops_off + ops_bytes + 255) & ~size_t(255);
  const size_t rops_bytes = rops.size() * sizeof(RbOp);
  const size_t mats_off = (rops_off + rops_bytes + 255) & ~size_t(255);
  const size_t total = mats_off + mats.size() * sizeof(double2) + 16;
  std::vector<char> prog(total, 0);
  if (!phases.empty()) std::memcpy(prog.data(), phases.data(), ph_bytes);
  if (!ops.empty()) std::memcpy(prog.data() + ops_off, ops.data(), ops_bytes);
  std::memcpy(prog.data() + rops_off, rops.data(), rops_bytes);
  if (!mats.empty()) std::memcpy(prog.data() + mats_off, mats.data(), mats.size() * sizeof(double2));
  void* dev = nullptr;
  if (total <= (2u << 20)) {
    const int rc = arena_put(h, prog.data(), total, &dev);
    if (rc) return rc;
  } else {
    if (total > h->fuse_cap) {
      if (h->fuse_dev) {
        int rc = check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        if (rc) return rc;
        (void)hipFree(h->fuse_dev);
        h->fuse_dev = nullptr;
      }
      int rc = check_hip(hipMalloc(&h->fuse_dev, total), "hipMalloc(fusion program)");
      if (rc) return rc;
      h->fuse_cap = total;
    }
    int rc = check_hip(hipMemcpyAsync(h->fuse_dev, prog.data(), total, hipMemcpyHostToDevice, h->stream),
                       "hipMemcpyAsync(fusion program)");
    if (rc) return rc;
    rc = check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize(fusion program)");
    if (rc) return rc;
    dev = h->fuse_dev;
  }
  const RbPhase* dph = static_cast<const RbPhase*>(dev);
  const FusedOp* dops = reinterpret_cast<const FusedOp*>(static_cast<char*>(dev) + ops_off);
  const RbOp* drops = reinterpret_cast<const RbOp*>(static_cast<char*>(dev) + rops_off);
  const double2* dmats = reinterpret_cast<const double2*>(static_cast<char*>(dev) + mats_off);
  // From |0...0>, amplitudes can be nonzero only where every bit outside the
  // qubits touched so far (`support`) is zero; a block maps each tile to
  // itself and zero tiles to zero, so it runs only the tiles whose index is
  // zero on its non-tile qubits outside the support (the first block: tile 0).
  unsigned long long support = 0;
  for (size_t li = 0; li < launches.size(); ++li) {
    const Launch& L = launches[li];
    timing_begin(h, KC_FUSED);
    if (L.rb) {
      const unsigned long long outside = ((1ull << nbits) - 1ull) & ~L.r.tile;
      launch_fused_rb(h->stream, h->data, nbits, L.r, dph, drops, dmats, rbits, set,
                      (flags & kFusedNonTemporal) != 0, from_zero ? outside & support : outside);
      support |= L.r.tile;
    } else {
      launch_fused_block(h->stream, h->data, nbits, L.d, dops, dmats);
      support = ~0ull;   // runs every tile (and may have touched any qubit)
    }
    timing_end(h);
    const int rc = check_hip(hipGetLastError(), "fused_block");
    if (rc) return rc;
  }
  if (one_tile) return NWQ_OK;
  h->last_blocks = (int)launches.size();
  h->last_fused_gates = 0;
  for (const PGate& g : gates_in) h->last_fused_gates += g.type != NWQ_GATE_I;
  h->last_phases = (int)phases.size();
  return NWQ_OK;
}

}  // namespace nwq

using namespace nwq;

extern "C" {

static int parse_circuit(int n, int n_gates, const int* types, const int* qubits, const double* params,
                         bool need_params, std::vector<PGate>& gates) {
  if (n_gates < 0 || (n_gates > 0 && (!types || !qubits))) return set_error(NWQ_EINVAL, "bad circuit arrays");
  gates.assign(n_gates, PGate{});
  for (int i = 0; i < n_gates; ++i) {
    PGate& g = gates[i];
    g.type = types[i];
    int nq = 0, np = 0;
    switch (g.type) {
      case NWQ_GATE_RX: case NWQ_GATE_RY: case NWQ_GATE_RZ: nq = 1; np = 1; break;
      case NWQ_GATE_U3: nq = 1; np = 3; break;
      case NWQ_GATE_CX: case NWQ_GATE_CZ: case NWQ_GATE_SWAP: nq = 2; break;
      case NWQ_GATE_RZZ: nq = 2; np = 1; break;
      default:
        if (g.type < 0 || g.type >= NWQ_GATE_COUNT) return set_error(NWQ_EINVAL, "gate " + std::to_string(i) + ": unknown type");
        nq = 1;
    }
    g.nq = nq;
    g.q[0] = qubits[2 * i];
    g.q[1] = nq == 2 ? qubits[2 * i + 1] : -1;
    for (int j = 0; j < 3; ++j) g.p[j] = params ? params[3 * i + j] : 0.0;
    if (np > 0 && need_params && params == nullptr) return set_error(NWQ_EINVAL, "params pointer is NULL");
    for (int j = 0; j < np; ++j)
      if (!std::isfinite(g.p[j])) return set_error(NWQ_EINVAL, "gate " + std::to_string(i) + ": non-finite parameter");
    for (int j = 0; j < nq; ++j)
      if (g.q[j] < 0 || g.q[j] >= n) return set_error(NWQ_ERANGE, "gate " + std::to_string(i) + ": qubit out of range");
    if (nq == 2 && g.q[0] == g.q[1]) return set_error(NWQ_EDUP, "gate " + std::to_string(i) + ": repeated qubit");
  }
  return NWQ_OK;
}

// A register of up to 13 qubits is one workgroup's tile: with fusion off its
// gates run one by one in a single launch (per 2048 gates, a program of at
// most 1.5 MB) instead of a launch each.  Launches are all that such a circuit
// costs, 3 us per gate: 380 gates of a TFIM on 10 qubits 1168 -> 250 us, 500
// on 13 1545 -> 415 us, of which planning takes 60 and 77.  Per-gate launches
// stay for a handful of gates (4 take 30 us, 8 take 62 against 26 to 36), for
// timed handles (times are kept per kernel class), for a stream under capture
// (a replay would read the upload ring again) and where there is no memory for
// the upload.
constexpr int kOneTileBits = 13, kOneTileMinGates = 8, kOneTileChunk = 2048;
static bool one_tile_circuit(nwq_state* h, int n_gates) {
  if (h->n > kOneTileBits || n_gates < kOneTileMinGates || h->timing) return false;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(h->stream, &st) != hipSuccess || st != hipStreamCaptureStatusNone ||
      arena_ready(h) != NWQ_OK) {
    (void)hipGetLastError();
    return false;
  }
  return true;
}

static int apply_circuit_common(nwq_handle h, int n_gates, const int* types, const int* qubits, const double* params,
                                bool from_zero) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  std::vector<PGate> gates;
  // validate everything before launching anything
  int rc0 = parse_circuit(h->n, n_gates, types, qubits, params, true, gates);
  if (rc0) return rc0;
  if (from_zero) {
    rc0 = nwq_reset(h);
    if (rc0) return rc0;
  }
  h->last_blocks = 0;
  h->last_fused_gates = 0;
  h->last_phases = 0;
  if (h->kind == NWQ_KIND_SV && h->fuse_k > 0 && n_gates > 0) return apply_fused(h, gates, h->n, nullptr, from_zero);
  size_t done = 0;   // gates that ran in one launch per chunk
  if (h->kind == NWQ_KIND_SV && one_tile_circuit(h, n_gates)) {
    while (done < gates.size()) {
      const size_t e = std::min(gates.size(), done + kOneTileChunk);
      const int rc = apply_fused(h, {gates.begin() + done, gates.begin() + e}, h->n, nullptr, false, true);
      if (rc == NWQ_ENOMEM) break;   // no room for the upload: nothing of the chunk has run
      if (rc) return rc;
      done = e;
    }
  }
  for (; done < gates.size(); ++done) {
    const PGate& g = gates[done];
    int rc;
    if (h->kind == NWQ_KIND_SV) {
      rc = sv_apply_gate_validated(h, g.type, g.q, g.p);
    } else {
      cd m[16];
      gate_matrix(g.type, g.p, m);
      rc = dm_apply_unitary(h, g.q, g.nq, m);
    }
    if (rc) return rc;
  }
  return NWQ_OK;
}

int nwq_apply_circuit(nwq_handle h, int n_gates, const int* types, const int* qubits, const double* params) {
  return apply_circuit_common(h, n_gates, types, qubits, params, false);
}

int nwq_run_circuit(nwq_handle h, int n_gates, const int* types, const int* qubits, const double* params) {
  return apply_circuit_common(h, n_gates, types, qubits, params, true);
}

int nwq_set_fusion_kernel(nwq_handle h, int kernel) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (kernel < 0 || kernel > 2) return set_error(NWQ_EINVAL, "fusion kernel must be 0, 1 or 2");
  if (h->kind == NWQ_KIND_DM && kernel != h->fuse_rb) {   // queued work runs on the kernel it was queued for
    const int rc = flush_all(h);
    if (rc) return rc;
  }
  h->fuse_rb = kernel;
  return NWQ_OK;
}

int nwq_set_fusion_flags(nwq_handle h, int flags) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (flags < 0 || flags > 7) return set_error(NWQ_EINVAL, "fusion flags must be in [0, 7]");
  h->fuse_flags = flags;
  return NWQ_OK;
}

int nwq_set_fusion_lowbits(nwq_handle h, int c) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (c != 0 && (c < 3 || c > 8)) return set_error(NWQ_EINVAL, "low tile bits must be 0 or in [3, 8]");
  if (h->kind == NWQ_KIND_DM && c != h->fuse_c) {   // queued superoperators run under the old tiles first
    const int rc = flush_all(h);
    if (rc) return rc;
  }
  h->fuse_c = c;
  return NWQ_OK;
}

int nwq_set_fusion(nwq_handle h, int k, int* k_out) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (k != 0 && (k < 6 || k > 13)) return set_error(NWQ_EINVAL, "fusion width must be 0 or in [6, 13]");
  if (h->kind == NWQ_KIND_DM) {   // queued superoperators are flushed under the old width first
    const int rc = flush_all(h);
    if (rc) return rc;
  }
  h->fuse_k = k;
  if (k_out) *k_out = k;
  return NWQ_OK;
}

int nwq_autotune_fusion(nwq_handle h, int n_gates, const int* types, const int* qubits, const double* params,
                        int reps, int* best_k, int* best_rb, double* ms_out) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (h->kind != NWQ_KIND_SV) return set_error(NWQ_EKIND, "fusion applies to state-vector handles");
  if (reps < 1 || reps > 100) return set_error(NWQ_EINVAL, "reps must be in [1, 100]");
  if (!best_k || !best_rb) return set_error(NWQ_EINVAL, "NULL output pointer");
  std::vector<PGate> gates;
  int rc = parse_circuit(h->n, n_gates, types, qubits, params, true, gates);
  if (rc) return rc;
  if (ms_out)
    for (int i = 0; i < NWQ_FUSION_CANDIDATES; ++i) ms_out[i] = -1.0;
  struct Cand { int k, rb; };
  std::vector<Cand> cands = {{0, 0}};
  for (int k = 6; k <= std::min(13, h->n); ++k) {
    cands.push_back({k, 0});
    if (h->n >= 8) {
      cands.push_back({k, 1});
      cands.push_back({k, 2});
    }
  }
  const int saved_k = h->fuse_k;
  const int saved_rb = h->fuse_rb;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  rc = check_hip(hipEventCreate(&e0), "hipEventCreate");
  if (!rc) rc = check_hip(hipEventCreate(&e1), "hipEventCreate");
  double best = 1e300;
  Cand pick{saved_k, saved_rb};
  std::array<double, NWQ_FUSION_CANDIDATES> timed;   // index: as ms_out
  auto slot = [](int k, int rb) { return k == 0 ? 0 : 1 + 3 * (k - 6) + rb; };
  for (const Cand& c : cands) {
    if (rc) break;
    h->fuse_k = c.k;
    h->fuse_rb = c.rb;
    const int runs = c.k == 0 ? 0 : fusion_width(h, h->nbits);
    if (runs < c.k) {   // the blocks of a narrower width: its time
      if (ms_out) ms_out[slot(c.k, c.rb)] = timed[slot(runs, c.rb)];
      continue;
    }
    double total = 0.0;
    for (int r = 0; r <= reps && !rc; ++r) {   // r == 0 is the untimed run
      rc = check_hip(hipEventRecord(e0, h->stream), "hipEventRecord");
      if (!rc) rc = apply_circuit_common(h, n_gates, types, qubits, params, true);   // from |0...0>
      if (!rc) rc = flush_all(h);
      if (!rc) rc = check_hip(hipEventRecord(e1, h->stream), "hipEventRecord");
      if (!rc) rc = check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
      float ms = 0.f;
      if (!rc) rc = check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
      if (r > 0) total += ms;
    }
    if (rc) break;
    const double per = timed[slot(c.k, c.rb)] = total / reps;
    if (ms_out) ms_out[slot(c.k, c.rb)] = per;
    if (per < best) {
      best = per;
      pick = c;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (rc) {
    h->fuse_k = saved_k;
    h->fuse_rb = saved_rb;
    return rc;
  }
  h->fuse_k = pick.k;
  h->fuse_rb = pick.rb;
  *best_k = pick.k;
  *best_rb = pick.rb;
  return nwq_reset(h);
}

int nwq_fusion_plan(int n, int k, int n_gates, const int* types, const int* qubits, int* n_blocks,
                    int* block_of_gate, int* block_qubits) {
  if (n < 1 || n > 34) return set_error(NWQ_ERANGE, "n outside [1, 34]");
  if (k < 6 || k > 13) return set_error(NWQ_EINVAL, "fusion width must be in [6, 13]");
  if (!n_blocks || (n_gates > 0 && !block_of_gate)) return set_error(NWQ_EINVAL, "NULL output pointer");
  std::vector<PGate> gates;
  int rc = parse_circuit(n, n_gates, types, qubits, nullptr, false, gates);
  if (rc) return rc;
  nwq_state defaults;   // a state vector's settings (no device memory)
  defaults.fuse_k = k;
  const std::vector<Block> blocks =
      plan_blocks(gates, n, fusion_width(&defaults, n), fusion_low_bits(&defaults, n), plan_seeds(n), false);
  if (n_gates > 0 && blocks.empty()) return set_error(NWQ_EINVAL, "fusion planner made no progress");
  *n_blocks = (int)blocks.size();
  for (size_t b = 0; b < blocks.size(); ++b) {
    for (int gi : blocks[b].gates) block_of_gate[gi] = (int)b;
    if (block_qubits) {
      unsigned long long mask = (1ull << blocks[b].c) - 1ull;
      for (int i = 0; i < blocks[b].m; ++i) mask |= 1ull << blocks[b].hi[i];
      block_qubits[2 * b] = (int)(mask & 0xffffffffull);
      block_qubits[2 * b + 1] = (int)(mask >> 32);
    }
  }
  return NWQ_OK;
}

int nwq_fusion_stats(nwq_handle h, int* blocks, int* gates) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (blocks) *blocks = h->last_blocks;
  if (gates) *gates = h->last_fused_gates;
  return NWQ_OK;
}

int nwq_fusion_phases(nwq_handle h, int* phases) {
  if (h == nullptr) return set_error(NWQ_EINVAL, "NULL handle");
  if (phases) *phases = h->last_phases;
  return NWQ_OK;
}

}  // extern "C"
