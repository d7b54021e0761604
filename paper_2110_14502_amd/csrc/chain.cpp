// Choice and layout of the fused small subtrees (k_chain.hip).
#include <algorithm>

#include "executor.h"

namespace rqc {

namespace {

// A step of the row kernel on complex64 tensors is evaluated inside a fused
// subtree when its operands hold at most 2^11 elements (16 KB of LDS each),
// its output at most 2^12 and its product at most 2^16 multiply-adds: up to
// there one workgroup's time for the step (0.5-4 us) is below that of a launch
// (7-20 us for these sizes); beyond it the step's own launch spreads over
// more workgroups and wins.  A subtree is evaluated once per copy of its root, so a
// step that depends on the slice only is repeated for every bitstring of the group
// (and the reverse).  That does not undo the gain at any group: calls of 4 x 5 and 5 x 5
// circuits, slices x bitstrings, launches of their own / fused: 8 x 512 1845 / 837 us,
// 16 x 300 2370 / 1276, 8 x 1024 3970 / 2661, 15 x 4096 (the most copies a group has) 24847 /
// 18155.  Leaving such steps out of the subtrees above them gains 7 to 18 % more with
// hundreds of bitstrings and costs 10 % with one (16 FP16 slices of a 5x5 circuit 238 /
// 262 us).
constexpr int kOperandBits = 11, kOutputBits = 12, kWorkBits = 16;

// First-fit allocation of LDS elements.
struct Pool {
  std::vector<std::pair<int, int>> used;  // (offset, size), sorted
  int alloc(int n) {
    n = (n + 1) & ~1;  // 16-byte aligned tensors
    int at = 0;
    size_t i = 0;
    for (; i < used.size(); ++i) {
      if (used[i].first - at >= n) break;
      at = used[i].first + used[i].second;
    }
    used.insert(used.begin() + (long)i, {at, n});
    return at;
  }
  void release(int at) {
    for (size_t i = 0; i < used.size(); ++i)
      if (used[i].first == at) {
        used.erase(used.begin() + (long)i);
        return;
      }
  }
};

// Whether the step has the layouts the planner gives every step: the summed
// labels lowest in A and B in the same order, the free ones in C's order.
// rpos / cpos of c: C's address bits of the free labels of A / B.
bool chain_layout(const Step& st, ChainStep& c) {
  if ((int)st.la.size() != st.m + st.k || (int)st.lb.size() != st.n + st.k ||
      (int)st.lc.size() != st.m + st.n)
    return false;
  if (!std::equal(st.la.begin() + st.m, st.la.end(), st.lb.begin() + st.n)) return false;
  int ia = 0, ib = 0;
  for (int b = 0; b < st.m + st.n; ++b) {
    const int x = st.lc[(size_t)(st.m + st.n - 1 - b)];
    if (ia < st.m && st.la[(size_t)(st.m - 1 - ia)] == x) c.rpos[ia++] = (int8_t)b;
    else if (ib < st.n && st.lb[(size_t)(st.n - 1 - ib)] == x) c.cpos[ib++] = (int8_t)b;
    else return false;
  }
  return true;
}

}  // namespace

ChainPlan plan_chains(const rqc_plan* p, int prec) {
  const PlanData& pd = p->pd;
  const int nl = pd.tree.n_leaves;
  const size_t ns = pd.steps.size();
  ChainPlan out;
  out.tree_of_step.assign(ns, -1);
  std::vector<ChainStep> base(ns, ChainStep{});
  std::vector<char> small(ns, 0), cut(ns, 0);
  // Parent step of every step.
  std::vector<int> parent(ns, -1);
  for (size_t i = 0; i < ns; ++i)
    for (int x : {pd.steps[i].a, pd.steps[i].b})
      if (x >= nl) parent[(size_t)pd.step_of_node[x]] = (int)i;
  for (size_t i = 0; i < ns; ++i) {
    const Step& st = pd.steps[i];
    bool ok = !st.invariant && p->sel_kern[prec][i] == KERN_ROWS && st.m + st.k <= kOperandBits && st.n + st.k <= kOperandBits &&
              st.m + st.n <= kOutputBits && st.m + st.n + st.k <= kWorkBits && chain_layout(st, base[i]);
    // Operands and output in complex64.
    ok = ok && !step_lp_store(p, prec, i);
    for (int x : {st.a, st.b}) {
      if (x >= nl) ok = ok && !step_lp_store(p, prec, (size_t)pd.step_of_node[x]);
      else ok = ok && (int)pd.net.leaves[x].labels.size() <= kChainLeafBits;
    }
    small[i] = ok;
  }
  // One subtree: the steps below `root` up to leaves, resident tensors, steps
  // that are not small and cut ones.  -1: laid out; else a step to cut.
  auto gather = [&](size_t root, ChainTree& t) -> int {
    t = ChainTree();
    t.first = true;
    std::vector<int> stack{(int)root}, steps;
    while (!stack.empty()) {
      const int i = stack.back();
      stack.pop_back();
      steps.push_back(i);
      for (int x : {pd.steps[(size_t)i].a, pd.steps[(size_t)i].b}) {
        const int j = x >= nl ? pd.step_of_node[x] : -1;
        if (j >= 0 && small[(size_t)j] && !cut[(size_t)j]) {
          stack.push_back(j);
        } else {
          t.inputs.push_back(x);
          if (j >= 0 && !pd.steps[(size_t)j].invariant) t.first = false;
        }
      }
    }
    // Inputs of at most 16 elements first (the kernel loads them together).
    std::stable_partition(t.inputs.begin(), t.inputs.end(),
                          [&](int x) { return pd.layout[(size_t)x].size() <= 4; });
    // By level: a step comes one level after the later of its operands, so
    // steps of one level are independent; execution order within.
    std::sort(steps.begin(), steps.end());
    std::vector<int> level(ns, 0);
    for (int i : steps)
      for (int x : {pd.steps[(size_t)i].a, pd.steps[(size_t)i].b}) {
        const int j = x >= nl ? pd.step_of_node[x] : -1;
        if (j >= 0 && std::binary_search(steps.begin(), steps.end(), j))
          level[(size_t)i] = std::max(level[(size_t)i], level[(size_t)j] + 1);
      }
    std::stable_sort(steps.begin(), steps.end(),
                     [&](int x, int y) { return level[(size_t)x] < level[(size_t)y]; });
    t.steps = steps;
    // Lay the tensors out in that order; every input is loaded first, and a
    // level's operands go when the whole level is done.
    Pool pool;
    std::vector<int> at(pd.tree.left.size(), -1), slot(pd.tree.left.size(), -1);
    auto elems = [&](int x) { return ((1 << pd.layout[(size_t)x].size()) + 1) & ~1; };
    int peak = 0, n_slot = 0;
    for (int x : t.inputs) {
      at[(size_t)x] = pool.alloc(elems(x));
      peak = std::max(peak, at[(size_t)x] + elems(x));
      slot[(size_t)x] = n_slot++;
      t.input_lds.push_back(at[(size_t)x]);
    }
    std::vector<int> done;
    for (size_t q = 0; q < t.steps.size(); ++q) {
      const int i = t.steps[q];
      const Step& st = pd.steps[(size_t)i];
      ChainStep c = base[(size_t)i];
      c.m = (uint8_t)st.m, c.n = (uint8_t)st.n, c.k = (uint8_t)st.k;
      c.tiles = (uint16_t)(1 << (std::max(0, st.m - 4) + std::max(0, st.n - 3)));
      slot[(size_t)st.node] = n_slot++;
      if (i != (int)root) {
        at[(size_t)st.node] = pool.alloc(elems(st.node));
        peak = std::max(peak, at[(size_t)st.node] + elems(st.node));
        c.lds_c = (uint16_t)at[(size_t)st.node];
      }
      c.lds_a = (uint16_t)at[(size_t)st.a], c.lds_b = (uint16_t)at[(size_t)st.b];
      c.slot_a = (uint16_t)slot[(size_t)st.a], c.slot_b = (uint16_t)slot[(size_t)st.b];
      done.push_back(st.a);
      done.push_back(st.b);
      c.level_end = q + 1 == t.steps.size() || level[(size_t)t.steps[q + 1]] != level[(size_t)i];
      if (c.level_end) {
        for (int x : done) pool.release(at[(size_t)x]);
        done.clear();
      }
      t.prog.push_back(c);
    }
    if (peak <= kChainMaxElems && (int)t.steps.size() <= kChainMaxSteps && n_slot <= kChainMaxSlots) {
      out.lds_elems = std::max(out.lds_elems, peak);
      return -1;
    }
    // Too large: the biggest step below the root becomes a root of its own
    // (ties: the latest).  A single step always fits.
    int big = -1;
    for (int i : t.steps)
      if (i != (int)root && (big < 0 || pd.layout[(size_t)pd.steps[(size_t)i].node].size() >=
                                            pd.layout[(size_t)pd.steps[(size_t)big].node].size()))
        big = i;
    return big;
  };
  std::vector<ChainTree> later;
  for (size_t r = ns; r-- > 0;) {
    if (!small[r]) continue;
    const int up = parent[r];
    if (up >= 0 && small[(size_t)up] && !cut[r]) continue;  // inside its parent's subtree
    ChainTree t;
    for (int c = gather(r, t); c >= 0; c = gather(r, t)) cut[(size_t)c] = 1;
    (t.first ? out.trees : later).push_back(std::move(t));
  }
  std::reverse(out.trees.begin(), out.trees.end());
  std::reverse(later.begin(), later.end());
  out.trees.insert(out.trees.end(), later.begin(), later.end());
  for (size_t c = 0; c < out.trees.size(); ++c)
    for (int i : out.trees[c].steps) out.tree_of_step[(size_t)i] = (int)c;
  return out;
}

}  // namespace rqc
