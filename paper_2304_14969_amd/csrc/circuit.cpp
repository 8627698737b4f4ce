// Circuit object and gate-fusion planner (host C++, float64).
//
// A random-circuit layer (Sec. III-C) is U(theta, phi, lambda) on every qubit
// followed by two-qubit couplers; applying each gate as its own HBM sweep costs
// one read and write of the whole ket per gate. The planner groups consecutive
// gates that act on at most kmax distinct qubits into one dense block whose
// matrix (the product of its gates, float64) is applied in a single sweep.
// SWAP gates never move data: they rename the positions later gates act on,
// and the circuit ends with that renaming applied to the state's labels
// (Table I: SWAP by qubit label swap).
#include <algorithm>
#include <cstring>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <mutex>
#include <string>

#include "circuit.h"
#include "qs_internal.h"

namespace qs {

namespace {

std::vector<cd> eye(int k) {
  const int d = 1 << k;
  std::vector<cd> m(size_t(d) * d, cd(0, 0));
  for (int i = 0; i < d; ++i) m[size_t(i) * d + i] = 1.0;
  return m;
}

// U(theta, phi, lambda) of Sec. III-C.
std::vector<cd> u3(double t, double p, double l) {
  const double c = std::cos(t / 2), s = std::sin(t / 2);
  return {cd(c, 0), -std::polar(1.0, l) * s, std::polar(1.0, p) * s, std::polar(1.0, p + l) * c};
}

// Two-qubit controlled 2x2: local bit 0 = control, bit 1 = target; acts when
// the control equals `cv`.
std::vector<cd> controlled(const std::vector<cd>& u, int cv) {
  std::vector<cd> m = eye(2);
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) m[size_t(cv + 2 * i) * 4 + (cv + 2 * j)] = u[size_t(i) * 2 + j];
  return m;
}

}  // namespace

bool gate_matrix(int kind, int nq, const double* p, std::vector<cd>* m, int* k_out) {
  const double r2 = 1.0 / std::sqrt(2.0);
  const std::vector<cd> X = {0.0, 1.0, 1.0, 0.0};
  const std::vector<cd> Y = {0.0, cd(0, -1), cd(0, 1), 0.0};
  const std::vector<cd> Z = {1.0, 0.0, 0.0, -1.0};
  int k = 0;
  switch (kind) {
    case QS_GATE_H: k = 1; *m = {r2, r2, r2, -r2}; break;
    case QS_GATE_X: k = 1; *m = X; break;
    case QS_GATE_Y: k = 1; *m = Y; break;
    case QS_GATE_Z: k = 1; *m = Z; break;
    case QS_GATE_U3: k = 1; *m = u3(p[0], p[1], p[2]); break;
    case QS_GATE_CZ: k = 2; *m = eye(2); (*m)[15] = -1.0; break;
    case QS_GATE_CP: k = 2; *m = eye(2); (*m)[15] = std::polar(1.0, p[0]); break;
    case QS_GATE_ISWAP:
      k = 2;
      *m = eye(2);
      (*m)[1 * 4 + 1] = 0.0; (*m)[2 * 4 + 2] = 0.0;
      (*m)[1 * 4 + 2] = cd(0, 1); (*m)[2 * 4 + 1] = cd(0, 1);
      break;
    case QS_GATE_SWAP:
      k = 2;
      *m = eye(2);
      (*m)[1 * 4 + 1] = 0.0; (*m)[2 * 4 + 2] = 0.0;
      (*m)[1 * 4 + 2] = 1.0; (*m)[2 * 4 + 1] = 1.0;
      break;
    case QS_GATE_CX: k = 2; *m = controlled(X, 1); break;
    case QS_GATE_CY: k = 2; *m = controlled(Y, 1); break;
    case QS_GATE_AX: k = 2; *m = controlled(X, 0); break;
    case QS_GATE_AY: k = 2; *m = controlled(Y, 0); break;
    case QS_GATE_AZ: k = 2; *m = controlled(Z, 0); break;
    case QS_GATE_CU3:
      if (p[3] != 0.0 && p[3] != 1.0) return false;
      k = 2;
      *m = controlled(u3(p[0], p[1], p[2]), int(p[3]));
      break;
    default: return false;
  }
  if (nq != k) return false;
  *k_out = k;
  return true;
}

namespace {

// m <- g m, where g acts on the block-local bits lp[0..gk) of a k-bit block.
// (Rows as planes of real and imaginary parts, so that the columns' sums run in
// vectors; std::complex's products would look for infinities and NaN each time.)
void left_apply(std::vector<cd>& m, int k, const std::vector<cd>& g, int gk, const int* lp) {
  constexpr int D = 1 << QS_MAX_FUSED;
  const int d = 1 << k, gd = 1 << gk;
  int mask = 0, off[D];
  for (int j = 0; j < gk; ++j) mask |= 1 << lp[j];
  for (int s = 0; s < gd; ++s) {
    off[s] = 0;
    for (int j = 0; j < gk; ++j) off[s] |= ((s >> j) & 1) << lp[j];
  }
  double xr[D * D], xi[D * D], yr[D], yi[D];
  for (int base = 0; base < d; ++base) {
    if (base & mask) continue;
    for (int s = 0; s < gd; ++s)
      for (int col = 0; col < d; ++col) {
        const cd v = m[size_t(base | off[s]) * d + col];
        xr[s * d + col] = v.real();
        xi[s * d + col] = v.imag();
      }
    for (int r = 0; r < gd; ++r) {
      for (int col = 0; col < d; ++col) yr[col] = yi[col] = 0;
      for (int s = 0; s < gd; ++s) {
        const double gr = g[size_t(r) * gd + s].real(), gi = g[size_t(r) * gd + s].imag();
        const double *pr = xr + s * d, *pi = xi + s * d;
        for (int col = 0; col < d; ++col) {
          yr[col] += gr * pr[col] - gi * pi[col];
          yi[col] += gr * pi[col] + gi * pr[col];
        }
      }
      for (int col = 0; col < d; ++col) m[size_t(base | off[r]) * d + col] = cd(yr[col], yi[col]);
    }
  }
}

struct Open {
  bool live = true;
  std::vector<int> qubits;
  std::vector<int> gates;
};

Block build_block(const Open& o, const std::vector<Gate>& gates) {
  Block b;
  std::vector<int> q = o.qubits;
  std::sort(q.begin(), q.end());
  b.k = int(q.size());
  for (int j = 0; j < b.k; ++j) b.q[j] = q[j];
  b.m = eye(b.k);
  b.ngates = int(o.gates.size());
  for (int gi : o.gates) {
    const Gate& g = gates[gi];
    int lp[QS_MAX_FUSED];
    for (int j = 0; j < g.k; ++j)
      lp[j] = int(std::lower_bound(q.begin(), q.end(), g.q[j]) - q.begin());
    left_apply(b.m, b.k, g.m, g.k, lp);
  }
  return b;
}

}  // namespace

std::vector<Block> fuse(const std::vector<Gate>& gates, int n, int kmax) {
  std::vector<Open> open;
  std::vector<int> owner(n, -1);
  std::vector<Block> out;
  auto emit = [&](int b) {
    out.push_back(build_block(open[b], gates));
    for (int q : open[b].qubits) owner[q] = -1;
    open[b].live = false;
  };
  for (int gi = 0; gi < int(gates.size()); ++gi) {
    const Gate& g = gates[gi];
    std::vector<int> touched;
    std::vector<int> uni(g.q, g.q + g.k);
    for (int j = 0; j < g.k; ++j) {
      const int b = owner[g.q[j]];
      if (b >= 0 && std::find(touched.begin(), touched.end(), b) == touched.end()) {
        touched.push_back(b);
        for (int q : open[b].qubits)
          if (std::find(uni.begin(), uni.end(), q) == uni.end()) uni.push_back(q);
      }
    }
    Open nb;
    if (int(uni.size()) <= kmax) {
      // merge: the touched blocks act on disjoint qubits, so their gate lists
      // may be concatenated in any order before this gate
      std::sort(touched.begin(), touched.end());
      for (int b : touched) {
        nb.gates.insert(nb.gates.end(), open[b].gates.begin(), open[b].gates.end());
        open[b].live = false;
      }
      nb.qubits = uni;
    } else {
      std::sort(touched.begin(), touched.end());
      for (int b : touched) emit(b);
      nb.qubits.assign(g.q, g.q + g.k);
    }
    nb.gates.push_back(gi);
    open.push_back(nb);
    for (int q : open.back().qubits) owner[q] = int(open.size()) - 1;
  }
  for (int b = 0; b < int(open.size()); ++b)
    if (open[b].live) emit(b);
  return out;
}

namespace {

// The gate list with its one-qubit gates multiplied into wider neighbours
// (float64): collected into the next gate of two or more qubits on their
// qubit, or, where none follows, into the last one; a gate on the same qubits
// as the gate before it on each of them is multiplied into that one. What
// stays are gates of two or more qubits and one product per qubit that only
// has one-qubit gates. The order keeps every qubit's gates in order.
std::vector<Gate> merge_gates(const std::vector<Gate>& gates, int n) {
  std::vector<Gate> out;
  std::vector<int> last(n, -1);  // per qubit: its last gate in out
  std::vector<std::vector<cd>> pend(n);
  auto at = [](const Gate& g, int q) { return int(std::find(g.q, g.q + g.k, q) - g.q); };
  for (const Gate& g : gates) {
    if (g.k == 1) {
      const int zero = 0;
      auto& u = pend[g.q[0]];
      if (u.empty()) u = eye(1);
      left_apply(u, 1, g.m, 1, &zero);
      continue;
    }
    int prev = last[g.q[0]];
    for (int j = 1; j < g.k; ++j)
      if (last[g.q[j]] != prev) prev = -1;
    const bool onto = prev >= 0 && out[prev].k == g.k;
    bool alone = !onto;
    for (int j = 0; j < g.k; ++j) alone = alone && pend[g.q[j]].empty();
    Gate w;
    if (!onto) {
      w = g;
      if (!alone) w.m = eye(g.k);
    }
    Gate& t = onto ? out[prev] : w;
    int lp[QS_MAX_FUSED];
    for (int j = 0; j < g.k; ++j) lp[j] = at(t, g.q[j]);
    for (int j = 0; j < g.k; ++j) {
      auto& u = pend[g.q[j]];
      if (!u.empty()) left_apply(t.m, t.k, u, 1, &lp[j]);
      u.clear();
    }
    if (!alone) left_apply(t.m, t.k, g.m, g.k, lp);
    if (onto) continue;
    for (int j = 0; j < g.k; ++j) last[g.q[j]] = int(out.size());
    out.push_back(std::move(w));
  }
  for (int q = 0; q < n; ++q) {
    if (pend[q].empty()) continue;
    if (last[q] >= 0) {
      const int b = at(out[last[q]], q);
      left_apply(out[last[q]].m, out[last[q]].k, pend[q], 1, &b);
      continue;
    }
    Gate w;
    w.k = 1;
    w.q[0] = q;
    w.m = std::move(pend[q]);
    out.push_back(std::move(w));
  }
  return out;
}

// Which gates a pass takes. A pass on a set of qubits runs every gate that
// the dependence order lets it run inside the set; the set is the low bits
// plus at most H qubits, grown by the ready gate that lets the most gates run
// per qubit it adds. (Taking front gates in circuit order while they fit,
// the rule before, needed 24.3 passes for 10 layers at 28 qubits where this
// one needs 16.8, and 11.3 against 7.9 for 8 layers at 20.)
struct PassPicker {
  const std::vector<Gate>& g;
  int n, max_k;
  std::vector<uint64_t> mask;             // qubits of each gate
  std::vector<std::vector<int>> per;      // gates of each qubit, in order
  std::vector<uint32_t> next;             // per qubit: its first gate not taken yet
  size_t left;

  PassPicker(const std::vector<Gate>& gates, int nq, int mk)
      : g(gates), n(nq), max_k(mk), mask(gates.size(), 0), per(nq), next(nq, 0), left(gates.size()) {
    for (size_t i = 0; i < gates.size(); ++i)
      for (int j = 0; j < gates[i].k; ++j) {
        mask[i] |= uint64_t(1) << gates[i].q[j];
        per[gates[i].q[j]].push_back(int(i));
      }
  }
  int front(const std::vector<uint32_t>& nx, int q) const {
    return nx[q] < per[q].size() ? per[q][nx[q]] : -1;
  }
  bool ready(const std::vector<uint32_t>& nx, int i) const {
    for (int j = 0; j < g[i].k; ++j)
      if (front(nx, g[i].q[j]) != i) return false;
    return true;
  }
  // runs all it can inside `set`, starting with the gates on `from`
  int run(uint64_t set, uint64_t from, std::vector<uint32_t>* nx, std::vector<int>* out) const {
    int count = 0;
    uint64_t look = from;
    while (look) {
      const int q = __builtin_ctzll(look);
      look &= look - 1;
      for (;;) {
        const int i = front(*nx, q);
        if (i < 0 || g[i].k > max_k || (mask[i] & ~set) || !ready(*nx, i)) break;
        for (int j = 0; j < g[i].k; ++j) ++(*nx)[g[i].q[j]];
        ++count;
        if (out) out->push_back(i);
        look |= mask[i];
      }
    }
    return count;
  }
  // The next pass: its gates (ascending) and the qubits chosen beyond `low`.
  std::vector<int> take(uint64_t low, int H, std::vector<int>* chosen) {
    uint64_t set = low;
    std::vector<uint32_t> base = next, trial;
    std::vector<int> out;
    run(set, set, &base, &out);
    for (int room = H; room > 0;) {
      double best = 0;
      uint64_t pick = 0;
      int first = -1;  // ties go to the earliest gate
      for (int q = 0; q < n; ++q) {
        const int i = front(base, q);
        if (i < 0 || g[i].k > max_k || (mask[i] & ((uint64_t(1) << q) - 1))) continue;
        const uint64_t add = mask[i] & ~set;
        const int cost = __builtin_popcountll(add);
        if (cost < 1 || cost > room || !ready(base, i)) continue;
        trial = base;
        const double gain = double(run(set | add, mask[i], &trial, nullptr)) / cost;
        if (gain > best || (gain == best && i < first)) best = gain, pick = add, first = i;
      }
      if (!pick) break;
      set |= pick;
      room -= __builtin_popcountll(pick);
      run(set, set, &base, &out);
    }
    std::sort(out.begin(), out.end());
    next = base;
    left -= out.size();
    for (int q = 0; q < n; ++q)
      if (((set & ~low) >> q) & 1) chosen->push_back(q);
    return out;
  }
  // The first ready gate (in order), taken: a gate too wide for a pass.
  int take_wide() {
    int i = -1;
    for (int q = 0; q < n; ++q) {
      const int f = front(next, q);
      if (f >= 0 && (i < 0 || f < i) && ready(next, f)) i = f;
    }
    for (int j = 0; j < g[i].k; ++j) ++next[g[i].q[j]];
    --left;
    return i;
  }
};

}  // namespace

bool narrow_gates(const std::vector<Gate>& gates) {
  for (const auto& g : gates)
    if (g.k > 2) return false;
  return true;
}

namespace {

// The rounds of a pass of gates of one or two qubits on tile bits tq[i], as
// pairs: each round takes two of the ready gates, those with the longest
// chains of later gates on their qubits. One-qubit gates (their qubits have no
// other gate in the pass) are joined two by two first.
void pair_rounds(TilePlan* plan, const std::vector<Gate>& gates, const std::vector<int>& pass,
                 const std::vector<std::vector<int>>& tq, int tile_bits) {
  struct Op { int a, b; std::vector<cd> m; };
  std::vector<Op> ops;
  int single = -1;  // a one-qubit gate waiting for another
  for (size_t i = 0; i < pass.size(); ++i) {
    const Gate& g = gates[pass[i]];
    if (g.k == 2) {
      ops.push_back({tq[i][0], tq[i][1], g.m});
    } else if (single < 0) {
      single = int(i);
    } else {
      Op o{tq[single][0], tq[i][0], eye(2)};
      const int bit0 = 0, bit1 = 1;
      left_apply(o.m, 2, gates[pass[single]].m, 1, &bit0);
      left_apply(o.m, 2, g.m, 1, &bit1);
      ops.push_back(std::move(o));
      single = -1;
    }
  }
  std::vector<int> last(tile_bits, -1);
  std::vector<int> need(ops.size(), 0), height(ops.size(), 1);
  std::vector<std::vector<int>> after(ops.size());
  for (size_t i = 0; i < ops.size(); ++i)
    for (int q : {ops[i].a, ops[i].b}) {
      if (last[q] >= 0) after[last[q]].push_back(int(i)), ++need[i];
      last[q] = int(i);
    }
  for (size_t i = ops.size(); i-- > 0;)
    for (int j : after[i]) height[i] = std::max(height[i], height[j] + 1);
  std::vector<int> ready;
  for (size_t i = 0; i < ops.size(); ++i)
    if (!need[i]) ready.push_back(int(i));
  auto emit = [&](const Op* o1, const Op* o2) {
    TileRound r;
    r.mode = TileMode::kPairs;
    r.mat = plan->reals.size();
    r.ng = o2 ? 2 : 1;
    int nb = 0;
    for (const Op* o : {o1, o2}) {
      if (!o) continue;
      r.bits[nb++] = o->a;
      r.bits[nb++] = o->b;
      for (const cd& v : o->m) {
        plan->reals.push_back(v.real());
        plan->reals.push_back(v.imag());
      }
    }
    for (int b = 0; nb < 4; ++b)
      if (std::find(r.bits, r.bits + nb, b) == r.bits + nb) r.bits[nb++] = b;
    plan->rounds.push_back(r);
  };
  // the last one-qubit gate joins a round that has room, or takes one of its own
  Op alone;
  bool waiting = single >= 0;
  if (waiting) {
    const int q = tq[single][0], bit0 = 0;
    alone = {q, -1, eye(2)};
    left_apply(alone.m, 2, gates[pass[single]].m, 1, &bit0);
  }
  auto give_partner = [&](const Op* o) {
    for (int b = 0; alone.b < 0; ++b)
      if (b != alone.a && !(o && (b == o->a || b == o->b))) alone.b = b;
  };
  while (!ready.empty()) {
    std::stable_sort(ready.begin(), ready.end(),
                     [&](int x, int y) { return height[x] > height[y]; });
    const int i = ready[0], j = ready.size() > 1 ? ready[1] : -1;
    if (j < 0 && waiting && ops[i].a != alone.a && ops[i].b != alone.a) {
      give_partner(&ops[i]);
      emit(&ops[i], &alone);
      waiting = false;
    } else {
      emit(&ops[i], j >= 0 ? &ops[j] : nullptr);
    }
    ready.erase(ready.begin(), ready.begin() + (j >= 0 ? 2 : 1));
    for (int x : {i, j}) {
      if (x < 0) continue;
      for (int y : after[x])
        if (!--need[y]) ready.push_back(y);
    }
  }
  if (waiting) {
    give_partner(nullptr);
    emit(&alone, nullptr);
  }
}

}  // namespace

double merged_gates(const std::vector<Gate>& gates, int n) {
  std::vector<int> last(n, -1);
  std::vector<char> one(n, 0);
  int count = 0;
  double singles = 0;
  for (const Gate& g : gates) {
    if (g.k == 1) {
      one[g.q[0]] = 1;
      continue;
    }
    if (last[g.q[0]] >= 0 && last[g.q[0]] == last[g.q[1]]) continue;
    last[g.q[0]] = last[g.q[1]] = count++;
  }
  for (int q = 0; q < n; ++q) singles += one[q] && last[q] < 0;
  return count + singles / 2;
}

std::vector<int> block_widths(const std::vector<Gate>& gates, int n, int kmax) {
  std::vector<int> out;
  std::vector<uint64_t> owner(n, 0);  // per qubit: the qubits of its open block
  auto close = [&](uint64_t b) {
    out.push_back(__builtin_popcountll(b));
    for (; b; b &= b - 1) owner[__builtin_ctzll(b)] = 0;
  };
  for (const Gate& g : gates) {
    uint64_t mine = 0, all = 0;
    for (int j = 0; j < g.k; ++j) {
      mine |= uint64_t(1) << g.q[j];
      all |= owner[g.q[j]];
    }
    all |= mine;
    if (__builtin_popcountll(all) > kmax) {
      for (int j = 0; j < g.k; ++j)
        if (owner[g.q[j]]) close(owner[g.q[j]]);
      all = mine;
    }
    for (uint64_t b = all; b; b &= b - 1) owner[__builtin_ctzll(b)] = all;
  }
  for (int q = 0; q < n; ++q)
    if (owner[q]) close(owner[q]);
  return out;
}

Block whole_block(const std::vector<Gate>& gates, int n) {
  const std::vector<Gate> merged = merge_gates(gates, n);
  Open o;
  for (int q = 0; q < n; ++q) o.qubits.push_back(q);
  for (size_t i = 0; i < merged.size(); ++i) o.gates.push_back(int(i));
  return build_block(o, merged);
}

namespace {

// What the rounds of a pass cost, in us per round (and gate of a sparse one):
// fits to whole runs of fourteen kinds of circuits (layers of random pairs, of
// neighbours, chains, rings, stars, gates on a few qubits only) in each form.
// A pair round holds two gates and a dense or sparse one all that four bits
// allow, so circuits that stay on few qubits, or go along a chain or a ring,
// need up to hundreds of times the rounds in pairs: 10 layers of a ring on 27
// qubits complex64 17.2 ms in dense rounds and 21.5 in pairs, of random pairs
// 12.0 and 8.0; 250 gates on four of 20 qubits 5.8 and 140 us. The ratios hardly
// depend on the size in complex64 (24 qubits; 12 qubits 0.80, 1.05, 1.73).
// Complex128 rounds wait for LDS and barriers while a CU has one tile (12
// qubits), where pairs do better, and are bound by the FMAs and the LDS
// bandwidth when it has four or more (24 qubits): 8 layers of neighbours on 12
// qubits 59 us in pairs and 65 in sparse rounds, 10 layers of a ring on 27 50.8
// and 36 ms.
struct RoundCost {
  double pair[2];          // a pair round of one gate, of two
  double group;            // a dense or a sparse round
  double gate[2];          // a sparse round's gates on one qubit, on two
  double pass;             // a pass of these over one of pair rounds, without the rounds
};
constexpr RoundCost kCost64{{6.7, 10.2}, 16.2, {0, 0}, -5};
constexpr RoundCost kCost128One{{1.23, 1.77}, 0.79, {0.47, 0.81}, 0.5};  // up to 19 qubits
constexpr RoundCost kCost128Two{{1.84, 2.67}, 0.75, {0.65, 1.12}, 0.5};  // 20 qubits
constexpr RoundCost kCost128{{22.6, 28.4}, 8.3, {5.7, 9.6}, 14};

// The rounds of a pass as groups of its gates: of the gates whose earlier ones
// are taken, those that fit W tile bits, in circuit order, until none does;
// `bits` are ascending, filled up with the lowest unused ones. Returns their
// number; out may be NULL.
struct Group {
  std::vector<int> bits, gates;
};
int greedy_groups(const std::vector<std::vector<int>>& tq, int tile_bits, int W,
                  std::vector<Group>* out) {
  int at[33] = {};  // gates of each bit, in order: list[at[x] .. at[x + 1])
  std::vector<uint32_t> mask(tq.size(), 0);
  for (size_t i = 0; i < tq.size(); ++i)
    for (int x : tq[i]) {
      mask[i] |= uint32_t(1) << x;
      ++at[x + 1];
    }
  for (int x = 0; x < tile_bits; ++x) at[x + 1] += at[x];
  std::vector<int> list(mask.size() ? at[tile_bits] : 0);
  int next[32];
  std::copy(at, at + tile_bits, next);
  for (size_t i = 0; i < tq.size(); ++i)
    for (int x : tq[i]) list[next[x]++] = int(i);
  std::copy(at, at + tile_bits, next);
  auto front = [&](int x) { return next[x] < at[x + 1] ? list[next[x]] : -1; };
  int count = 0;
  for (size_t left = tq.size(); left; ++count) {
    if (out) out->emplace_back();
    uint32_t set = 0;
    for (bool progress = true; progress;) {
      progress = false;
      int ready[32], nready = 0;
      for (int x = 0; x < tile_bits; ++x) {
        const int i = front(x);
        if (i < 0 || (mask[i] & ((uint32_t(1) << x) - 1))) continue;  // seen at its lowest bit
        bool first = true;
        for (int y : tq[i]) first = first && front(y) == i;
        if (first) ready[nready++] = i;
      }
      std::sort(ready, ready + nready);
      for (int r = 0; r < nready; ++r) {
        const int i = ready[r];
        if (__builtin_popcount(set | mask[i]) > W) continue;
        set |= mask[i];
        for (int y : tq[i]) ++next[y];
        if (out) out->back().gates.push_back(i);
        --left;
        progress = true;
      }
    }
    if (!out) continue;
    for (int b = 0; __builtin_popcount(set) < W; ++b) set |= uint32_t(1) << b;
    for (int b = 0; b < tile_bits; ++b)
      if ((set >> b) & 1) out->back().bits.push_back(b);
  }
  return count;
}

// Emits a group's round: the product of its gates (dense) or the gates one by
// one (sparse).
void group_round(TilePlan* plan, const std::vector<Gate>& gates, const std::vector<int>& pass,
                 const std::vector<std::vector<int>>& tq, const Group& group, int W, bool dense) {
  const std::vector<int>& rb = group.bits;
  TileRound r;
  r.mode = dense ? TileMode::kDense : TileMode::kSparse;
  for (int j = 0; j < W; ++j) r.bits[j] = rb[j];
  r.g0 = int(plan->gates.size());
  r.ng = int(group.gates.size());
  if (dense) {
    // the product of the round's gates on its W bits (local bit j = rb[j])
    std::vector<cd> u = eye(W);
    for (int gi : group.gates) {
      const Gate& g = gates[pass[gi]];
      int lp[QS_MAX_FUSED];
      for (int j = 0; j < g.k; ++j)
        lp[j] = int(std::find(rb.begin(), rb.end(), tq[gi][j]) - rb.begin());
      left_apply(u, W, g.m, g.k, lp);
    }
    r.mat = plan->mats.size();
    plan->mats.insert(plan->mats.end(), u.begin(), u.end());
  } else {
    // one-qubit gates folded into the round's two-qubit gates: into the
    // last two-qubit gate on their bit (from the left) when there is one,
    // else into the next (from the right); one-qubit products on bits no
    // two-qubit gate of the round touches stay one-qubit gates (they
    // commute with the rest of the round)
    struct Out { int kind, j1, j2; std::vector<cd> m; };
    std::vector<Out> outg;
    std::vector<int> last(W, -1);            // per round bit: its last two-qubit gate
    std::vector<std::vector<cd>> pend(W);    // per round bit: pending one-qubit product
    for (int gi : group.gates) {
      const Gate& g = gates[pass[gi]];
      const int j1 = int(std::find(rb.begin(), rb.end(), tq[gi][0]) - rb.begin());
      if (g.k == 1) {
        if (last[j1] >= 0) {
          Out& o = outg[size_t(last[j1])];
          const int at = o.j1 == j1 ? 0 : 1;
          left_apply(o.m, 2, g.m, 1, &at);
        } else {
          if (pend[j1].empty()) pend[j1] = eye(1);
          const int at = 0;
          left_apply(pend[j1], 1, g.m, 1, &at);
        }
        continue;
      }
      const int j2 = int(std::find(rb.begin(), rb.end(), tq[gi][1]) - rb.begin());
      std::vector<cd> m = eye(2);
      const int bit0 = 0, bit1 = 1, both[2] = {0, 1};
      if (!pend[j1].empty()) left_apply(m, 2, pend[j1], 1, &bit0);
      if (!pend[j2].empty()) left_apply(m, 2, pend[j2], 1, &bit1);
      left_apply(m, 2, g.m, 2, both);
      pend[j1].clear();
      pend[j2].clear();
      last[j1] = last[j2] = int(outg.size());
      outg.push_back({2, j1, j2, std::move(m)});
    }
    for (int j = 0; j < W; ++j)
      if (!pend[j].empty()) outg.push_back({1, j, 0, std::move(pend[j])});
    r.ng = int(outg.size());
    for (Out& o : outg) {
      TileGate tg;
      tg.kind = o.kind;
      tg.j1 = o.j1;
      tg.j2 = o.j2;
      tg.mat = plan->mats.size();
      plan->mats.insert(plan->mats.end(), o.m.begin(), o.m.end());
      plan->gates.push_back(tg);
    }
  }
  plan->rounds.push_back(r);
}

}  // namespace

TilePlan plan_tiles(const std::vector<Gate>& circuit, int n, int C, int H, int W,
                    TileForms forms, bool dense_price) {
  const std::vector<Gate> gates = merge_gates(circuit, n);
  TilePlan plan;
  plan.C = C;
  plan.H = H;
  plan.W = W;
  plan.forms = forms;
  const bool dense = forms == TileForms::kPairsDense || forms == TileForms::kDense;
  const RoundCost& cost = dense || dense_price ? kCost64
                          : n <= 19 ? kCost128One
                          : n == 20 ? kCost128Two
                                    : kCost128;
  std::vector<std::vector<int>> qb(gates.size());
  for (size_t i = 0; i < gates.size(); ++i) qb[i].assign(gates[i].q, gates[i].q + gates[i].k);
  PassPicker picker(gates, n, dense ? W : 2);
  const uint64_t low = (uint64_t(1) << (C < n ? C : n)) - 1;
  while (picker.left) {
    std::vector<int> hi;
    const std::vector<int> pass = picker.take(low, H, &hi);
    if (pass.empty()) {
      // only gates too wide for a round are ready: the first one as a block
      const int i = picker.take_wide();
      TileStep st;
      st.block = true;
      st.ngates = 1;
      std::vector<int> q(gates[i].q, gates[i].q + gates[i].k);
      std::vector<int> order(q.size());
      for (size_t j = 0; j < q.size(); ++j) order[j] = int(j);
      std::sort(q.begin(), q.end());
      st.blk.k = gates[i].k;
      for (int j = 0; j < st.blk.k; ++j) st.blk.q[j] = q[j];
      st.blk.ngates = 1;
      st.blk.m = eye(st.blk.k);
      int lp[QS_MAX_FUSED];
      for (int j = 0; j < gates[i].k; ++j)
        lp[j] = int(std::lower_bound(q.begin(), q.end(), gates[i].q[j]) - q.begin());
      left_apply(st.blk.m, st.blk.k, gates[i].m, gates[i].k, lp);
      st.mat = plan.mats.size();
      plan.mats.insert(plan.mats.end(), st.blk.m.begin(), st.blk.m.end());
      plan.steps.push_back(std::move(st));
      continue;
    }
    // row bits: the chosen ones, completed with the lowest unused high bits
    for (int q = C; q < n && int(hi.size()) < H; ++q)
      if (std::find(hi.begin(), hi.end(), q) == hi.end()) hi.push_back(q);
    std::sort(hi.begin(), hi.end());
    std::vector<int> tbit(n, -1);  // physical bit -> tile bit
    for (int q = 0; q < C; ++q) tbit[q] = q;
    for (int j = 0; j < H; ++j) tbit[hi[j]] = C + j;
    TileStep st;
    for (int j = 0; j < H; ++j) st.hb[j] = hi[j];
    st.r0 = int(plan.rounds.size());
    st.ngates = int(pass.size());
    std::vector<std::vector<int>> tq(pass.size());
    for (size_t i = 0; i < pass.size(); ++i)
      for (int x : qb[pass[i]]) tq[i].push_back(tbit[x]);
    // the rounds, in the cheaper of the two forms the plan may use
    bool narrow = true;
    for (int i : pass) narrow = narrow && gates[i].k <= 2;
    const bool pairs = narrow && forms != TileForms::kSparse && forms != TileForms::kDense;
    const bool groups = !pairs || forms != TileForms::kPairs;
    const size_t reals0 = plan.reals.size();
    double pair_cost = 0, group_cost = 0;
    if (pairs) {
      pair_rounds(&plan, gates, pass, tq, C + H);
      st.mode = TileMode::kPairs;
      for (size_t r = size_t(st.r0); r < plan.rounds.size(); ++r)
        pair_cost += cost.pair[plan.rounds[r].ng - 1];
    }
    if (pairs && (groups || dense_price)) {
      group_cost = cost.pass + cost.group * greedy_groups(tq, C + H, W, nullptr);
      for (int i : pass) group_cost += cost.gate[gates[i].k - 1];  // (none in dense rounds)
      plan.pair_cost += pair_cost;
      plan.group_cost += group_cost;
    }
    if (groups && (!pairs || group_cost < pair_cost)) {
      plan.rounds.resize(size_t(st.r0));
      plan.reals.resize(reals0);
      st.mode = dense ? TileMode::kDense : TileMode::kSparse;
      std::vector<Group> grp;
      greedy_groups(tq, C + H, W, &grp);
      for (const Group& g : grp) group_round(&plan, gates, pass, tq, g, W, dense);
    }
    st.nr = int(plan.rounds.size()) - st.r0;
    plan.steps.push_back(st);
  }
  return plan;
}

std::vector<float> float_pairs(const TilePlan& pl) {
  constexpr int kReals = 32;  // of a gate
  std::vector<float> out(pl.reals.size());
  double scale = 1.0;
  for (const TileRound& r : pl.rounds) {
    if (r.mode != TileMode::kPairs) continue;
    for (int g = 0; g < r.ng; ++g) {
      const double* m = pl.reals.data() + r.mat + g * kReals;
      float* f = out.data() + r.mat + g * kReals;
      double b[8] = {}, c[8] = {};  // squares before and after the cast, in 8 sums
      for (int i = 0; i < kReals; i += 8)
        for (int j = 0; j < 8; ++j) {
          f[i + j] = float(m[i + j] * scale);
          b[j] += m[i + j] * m[i + j];
          c[j] += double(f[i + j]) * double(f[i + j]);
        }
      double before = 0, after = 0;
      for (int j = 0; j < 8; ++j) before += b[j], after += c[j];
      scale *= std::sqrt(before / after);
      if (!(std::abs(scale - 1.0) < 1e-6)) scale = 1.0;  // a zero matrix, numbers out of range
    }
  }
  return out;
}

void pair_round_entry(const TileRound& r, size_t base, int32_t row[4]) {
  int asc[4];
  std::copy(r.bits, r.bits + 4, asc);
  std::sort(asc, asc + 4);
  row[0] = r.bits[0] | (r.bits[1] << 8) | (r.bits[2] << 16) | (r.bits[3] << 24);
  row[1] = asc[0] | (asc[1] << 8) | (asc[2] << 16) | (asc[3] << 24);
  row[2] = int32_t(base + r.mat);
  row[3] = r.ng > 1 ? 1 : 0;
}

void tile_tables(const TilePlan& pl, bool c64, std::vector<unsigned char>* out, TileOffsets* at) {
  std::vector<int32_t> tab;
  std::vector<float> ops;  // dense rounds
  for (const TileRound& r : pl.rounds) {
    int32_t row[4] = {r.bits[0] | (r.bits[1] << 8) | (r.bits[2] << 16) | (r.bits[3] << 24), r.g0,
                      r.ng, 0};
    if (r.mode == TileMode::kPairs) {
      pair_round_entry(r, 0, row);
    } else if (r.mode == TileMode::kDense) {
      row[1] = int32_t(ops.size());
      ops.resize(ops.size() + kRoundOperands);
      embed_round(pl.mats.data() + r.mat, ops.data() + row[1]);
    }
    tab.insert(tab.end(), row, row + 4);
  }
  auto up256 = [](size_t x) { return (x + 255) / 256 * 256; };
  at->gates = tab.size() * sizeof(int32_t);
  for (const auto& g : pl.gates) {
    tab.push_back(g.kind | (g.j1 << 4) | (g.j2 << 8));
    tab.push_back(int32_t(2 * g.mat));
  }
  const size_t esz = c64 ? sizeof(float) : sizeof(double);
  at->ops = up256(tab.size() * sizeof(int32_t));
  at->mats = up256(at->ops + ops.size() * sizeof(float));
  at->reals = up256(at->mats + 2 * pl.mats.size() * esz);
  out->assign(at->reals + pl.reals.size() * esz, 0);
  unsigned char* host = out->data();
  std::memcpy(host, tab.data(), tab.size() * sizeof(int32_t));
  if (!ops.empty()) std::memcpy(host + at->ops, ops.data(), ops.size() * sizeof(float));
  auto put = [&](unsigned char* to, double v) {
    const float f = float(v);
    if (c64)
      std::memcpy(to, &f, sizeof f);
    else
      std::memcpy(to, &v, sizeof v);
  };
  for (size_t i = 0; i < pl.mats.size(); ++i) {
    put(host + at->mats + 2 * i * esz, pl.mats[i].real());
    put(host + at->mats + (2 * i + 1) * esz, pl.mats[i].imag());
  }
  if (c64) {
    const std::vector<float> f = float_pairs(pl);
    if (!f.empty()) std::memcpy(host + at->reals, f.data(), f.size() * sizeof(float));
  } else if (!pl.reals.empty()) {
    std::memcpy(host + at->reals, pl.reals.data(), pl.reals.size() * sizeof(double));
  }
}

void embed_round(const cd* u, float* out) {
  for (int s4 = 0; s4 < 4; ++s4)
    for (int lane = 0; lane < 64; ++lane) {
      const cd x = u[(lane % 16) * 16 + 4 * s4 + lane / 16];
      out[(3 * s4 + 0) * 64 + lane] = float(x.real());
      out[(3 * s4 + 1) * 64 + lane] = float(x.imag());
      out[(3 * s4 + 2) * 64 + lane] = float(x.real() + x.imag());
    }
}

}  // namespace qs

// ------------------------------------------------------------------ C ABI

namespace qs {
void set_last_error(const char* msg);    // capi.cpp
void circuit_invalidate(qs_circuit* c);  // frees device copies (capi.cpp)
uint64_t next_generation();              // capi.cpp
}  // namespace qs

namespace {
int cfail(int code, const char* fmt, ...) {
  char buf[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  qs::set_last_error(buf);
  return code;
}
}  // namespace

namespace qs {
// The block plan alone: what a dense run without tiles or a batch needs,
// without the caller's choice of run mode that qs_circuit_plan records.
int circuit_plan_blocks(qs_circuit* c, int kmax) {
  if (!c) return cfail(QS_E_INVAL, "circuit is NULL");
  if (kmax == 0) kmax = 5;
  if (kmax < 1 || kmax > QS_MAX_FUSED) return cfail(QS_E_INVAL, "kmax = %d outside [1, %d]", kmax, QS_MAX_FUSED);
  circuit_invalidate(c);
  c->kmax = kmax;
  c->blocks = fuse(c->gates, c->n, kmax);
  c->planned = true;
  return QS_OK;
}

void circuit_plan_blocks_later(qs_circuit* c, int kmax) {
  if ((c->planned || c->due) && c->kmax == kmax) return;
  if (c->planned) circuit_invalidate(c);
  c->kmax = kmax;
  c->due = true;
}

void circuit_blocks_due(const qs_circuit* circuit) {
  static std::mutex mu;  // two threads may ask about one circuit
  std::lock_guard<std::mutex> lock(mu);
  qs_circuit* c = const_cast<qs_circuit*>(circuit);
  if (!c->due || c->planned) return;
  c->blocks = fuse(c->gates, c->n, c->kmax);
  c->planned = true;
  c->due = false;
}
}  // namespace qs

extern "C" {

int qs_circuit_create(int n, qs_circuit** out) {
  if (!out) return cfail(QS_E_INVAL, "out is NULL");
  if (n < 1 || n > 64) return cfail(QS_E_INVAL, "n = %d outside [1, 64]", n);
  qs_circuit* c = new qs_circuit();
  c->n = n;
  c->generation = qs::next_generation();
  c->pos.resize(n);
  for (int q = 0; q < n; ++q) c->pos[q] = q;
  *out = c;
  return QS_OK;
}

static int add_checked(qs_circuit* c, const int* qubits, int k, std::vector<qs::cd> m) {
  if (!c) return cfail(QS_E_INVAL, "circuit is NULL");
  if (!qubits) return cfail(QS_E_INVAL, "qubits is NULL");
  if (k < 1 || k > QS_MAX_FUSED) return cfail(QS_E_INVAL, "gate on %d qubits", k);
  for (int j = 0; j < k; ++j) {
    if (qubits[j] < 0 || qubits[j] >= c->n)
      return cfail(QS_E_INVAL, "qubit %d out of range [0, %d)", qubits[j], c->n);
    for (int i = 0; i < j; ++i)
      if (qubits[i] == qubits[j]) return cfail(QS_E_INVAL, "qubit %d used twice", qubits[j]);
  }
  for (const auto& v : m)
    if (!std::isfinite(v.real()) || !std::isfinite(v.imag()))
      return cfail(QS_E_INVAL, "non-finite matrix entry");
  qs::circuit_invalidate(c);
  qs::Gate g;
  g.k = k;
  for (int j = 0; j < k; ++j) g.q[j] = c->pos[qubits[j]];
  g.m = std::move(m);
  c->gates.push_back(std::move(g));
  return QS_OK;
}

int qs_circuit_add_gate(qs_circuit* c, int kind, const int* qubits, const double* params) {
  if (!c) return cfail(QS_E_INVAL, "circuit is NULL");
  if (!qubits) return cfail(QS_E_INVAL, "qubits is NULL");
  const int nq = (kind >= QS_GATE_CZ) ? 2 : 1;
  if ((kind == QS_GATE_U3 || kind == QS_GATE_CP || kind == QS_GATE_CU3) && !params)
    return cfail(QS_E_INVAL, "gate kind %d needs parameters", kind);
  if (kind == QS_GATE_U3 || kind == QS_GATE_CU3)
    for (int i = 0; i < 3; ++i)
      if (!std::isfinite(params[i])) return cfail(QS_E_INVAL, "non-finite parameter");
  if (kind == QS_GATE_CU3 && params[3] != 0.0 && params[3] != 1.0)
    return cfail(QS_E_INVAL, "control value %g is not 0 or 1", params[3]);
  if (kind == QS_GATE_CP && !std::isfinite(params[0])) return cfail(QS_E_INVAL, "non-finite parameter");
  std::vector<qs::cd> m;
  int k = 0;
  if (!qs::gate_matrix(kind, nq, params, &m, &k)) return cfail(QS_E_INVAL, "unknown gate kind %d", kind);
  if (kind == QS_GATE_SWAP) {
    for (int j = 0; j < 2; ++j)
      if (qubits[j] < 0 || qubits[j] >= c->n)
        return cfail(QS_E_INVAL, "qubit %d out of range [0, %d)", qubits[j], c->n);
    if (qubits[0] == qubits[1]) return cfail(QS_E_INVAL, "qubit %d used twice", qubits[0]);
    qs::circuit_invalidate(c);
    std::swap(c->pos[qubits[0]], c->pos[qubits[1]]);
    return QS_OK;
  }
  return add_checked(c, qubits, k, std::move(m));
}

int qs_circuit_add_matrix(qs_circuit* c, const int* qubits, int k, const double* m) {
  if (!m) return cfail(QS_E_INVAL, "matrix is NULL");
  if (k < 1 || k > QS_MAX_FUSED) return cfail(QS_E_INVAL, "gate on %d qubits", k);
  const size_t d = size_t(1) << k;
  std::vector<qs::cd> mm(d * d);
  for (size_t i = 0; i < d * d; ++i) mm[i] = qs::cd(m[2 * i], m[2 * i + 1]);
  return add_checked(c, qubits, k, std::move(mm));
}


int qs_circuit_plan(qs_circuit* c, int kmax) {
  if (int rc = qs::circuit_plan_blocks(c, kmax)) return rc;
  if (c->tiles < 0) c->tiles = 0;  // planning blocks asks for blocks
  return QS_OK;
}

int qs_circuit_use_tiles(qs_circuit* c, int on) {
  if (!c) return cfail(QS_E_INVAL, "circuit is NULL");
  c->tiles = on != 0 ? 1 : 0;
  return QS_OK;
}

int qs_circuit_tile_info(const qs_circuit* c, int dtype, int* passes, int* blocks, int* rounds) {
  if (!c) return cfail(QS_E_INVAL, "circuit is NULL");
  if (dtype != QS_C64 && dtype != QS_C128) return cfail(QS_E_INVAL, "unknown dtype %d", dtype);
  const int C = qs::tile_low_bits(dtype);
  if (c->n < C + 7) return cfail(QS_E_UNSUPPORTED, "%d qubits: fewer than one tile (%d)", c->n, C + 7);
  const qs::TilePlan pl = qs::plan_tiles(
      c->gates, c->n, C, 7, 4,
      dtype == QS_C64 ? qs::TileForms::kPairsDense : qs::TileForms::kPairsSparse);
  if (passes) *passes = pl.passes();
  if (blocks) *blocks = int(pl.steps.size()) - pl.passes();
  if (rounds) *rounds = int(pl.rounds.size());
  return QS_OK;
}

int qs_circuit_info(const qs_circuit* c, int* ngates, int* nblocks, int* max_k) {
  if (!c) return cfail(QS_E_INVAL, "circuit is NULL");
  qs::circuit_blocks_due(c);
  if (ngates) *ngates = int(c->gates.size());
  if (nblocks) *nblocks = c->planned ? int(c->blocks.size()) : -1;
  if (max_k) {
    int mk = 0;
    for (const auto& b : c->blocks) mk = std::max(mk, b.k);
    *max_k = mk;
  }
  return QS_OK;
}

int qs_circuit_block(const qs_circuit* c, int i, int* k, int* qubits, double* m) {
  if (!c || !k) return cfail(QS_E_INVAL, "NULL argument");
  qs::circuit_blocks_due(c);
  if (!c->planned) return cfail(QS_E_INVAL, "circuit is not planned");
  if (i < 0 || i >= int(c->blocks.size())) return cfail(QS_E_INVAL, "block %d out of range", i);
  const qs::Block& b = c->blocks[i];
  *k = b.k;
  if (qubits)
    for (int j = 0; j < b.k; ++j) qubits[j] = b.q[j];
  if (m)
    for (size_t e = 0; e < b.m.size(); ++e) {
      m[2 * e] = b.m[e].real();
      m[2 * e + 1] = b.m[e].imag();
    }
  return QS_OK;
}

}  // extern "C"
