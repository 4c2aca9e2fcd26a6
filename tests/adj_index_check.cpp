// Host checks of the gravity adjoint's indices (adj_index.hip is host code): random task sets, and for each the
// properties that the kernels rely on.  Prints "ok" and returns 0, or names the first property that fails.
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <random>
#include <vector>

#include "gc_internal.h"

using namespace gc;

// Allocations on any thread until one is refused (negative: none is).
static std::atomic<long> g_left{-1};
void* operator new(std::size_t n) {
  if (g_left.load() >= 0 && g_left.fetch_sub(1) == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

namespace {

struct Input {
  std::vector<gc_task> tasks;
  std::vector<int32_t> ranges, nodes;
  int32_t n_nodes = 0, n_ids = 0;
  AdjIndexInput in(int n_cu) const {
    return AdjIndexInput{tasks.data(), (int32_t)tasks.size(), ranges.data(), nodes.data(), n_nodes, n_ids, n_cu};
  }
  void add(int targets, const std::vector<int32_t>& node, const std::vector<std::pair<int32_t, int32_t>>& direct) {
    gc_task t{};
    t.i_begin = tasks.empty() ? 0 : tasks.back().i_begin + tasks.back().i_count;
    t.i_count = targets;
    t.n_first = (int32_t)nodes.size();
    t.n_count = (int32_t)node.size();
    t.j_first = (int32_t)ranges.size() / 2;
    t.j_nranges = (int32_t)direct.size();
    nodes.insert(nodes.end(), node.begin(), node.end());
    for (auto& r : direct) {
      ranges.push_back(r.first);
      ranges.push_back(r.second);
    }
    tasks.push_back(t);
  }
};

// form 0: short lists, some empty, repeated or out of order; 1: one stretch of tasks with neither nodes nor direct
// ranges after some with both; 2: lists longer than a table
Input make(int form, int seed, int n_tasks) {
  std::mt19937 rng((unsigned)(1000 * form + seed));
  auto upto = [&](int n) { return (int)(rng() % (unsigned)n); };
  Input x;
  x.n_nodes = 400 + upto(4000);
  x.n_ids = 8 * n_tasks + 3000;
  for (int t = 0; t < n_tasks; ++t) {
    const bool none = form == 1 ? t >= n_tasks / 8 && t < 7 * n_tasks / 8 : upto(4) == 0;
    std::vector<int32_t> node;
    std::vector<std::pair<int32_t, int32_t>> direct;
    if (!none) {
      const int n = form == 2 && upto(8) == 0 ? 3000 + upto(3000) : upto(60);
      for (int k = 0, at = upto(x.n_nodes); k < n; ++k, at = (at + 1 + upto(3)) % x.n_nodes) node.push_back(at);
      if (n && upto(3) == 0) node.push_back(node[(size_t)upto(n)]);
      for (int r = 0, at = upto(50); r < 4; ++r) {
        const int c = form == 2 && upto(16) == 0 ? 1200 : upto(30);
        direct.push_back({at, c});
        at += c + upto(20);
      }
    }
    x.add(upto(9), node, direct);
  }
  return x;
}

#define CHECK(cond)                                                      \
  do {                                                                   \
    if (!(cond)) {                                                       \
      std::printf("form %d seed %d: %s\n", form, seed, #cond);           \
      return 1;                                                          \
    }                                                                    \
  } while (0)

template <class T = int32_t>
const T* arr(const AdjIndex& a, int which) {
  return reinterpret_cast<const T*>(a.blob.get() + a.at[which]);
}

// One kind of source: every visit of every task lies in one item, its place names its source, no two visits of a task
// share a place, and no item has more tasks or more sources than the kernel has room for.
int check(const Input& x, const AdjIndex& a, bool direct, int form, int seed) {
  const int T = (int)x.tasks.size(), cap = direct ? kAdjMaxDirect : kAdjMaxNodes;
  const int waves = direct ? kAdjDirectWaves : kAdjNodeWaves, n_items = direct ? a.direct_items : a.node_items;
  const AdjItem* item = arr<AdjItem>(a, direct ? AdjIndex::kDirectItems : AdjIndex::kNodeItems);
  std::vector<std::vector<int32_t>> source((size_t)T);
  std::vector<int64_t> first((size_t)T + 1, 0);
  for (int t = 0; t < T; ++t) {
    const gc_task& k = x.tasks[(size_t)t];
    auto& s = source[(size_t)t];
    if (direct)
      for (int r = 0; r < k.j_nranges; ++r)
        for (int q = 0; q < x.ranges[2 * (k.j_first + r) + 1]; ++q) s.push_back(x.ranges[2 * (k.j_first + r)] + q);
    else
      s.assign(x.nodes.begin() + k.n_first, x.nodes.begin() + k.n_first + k.n_count);
    first[(size_t)t + 1] = first[(size_t)t] + (int64_t)s.size();
  }
  // with an item a task, the device writes places, cuts and keys: a record is a visit, and the cuts are even
  std::vector<uint16_t> place_;
  std::vector<int32_t> cuts_, key_;
  const uint16_t* place = arr<uint16_t>(a, direct ? AdjIndex::kDirectPlace : AdjIndex::kNodePlace);
  const int32_t* cuts = arr(a, direct ? AdjIndex::kDirectCuts : AdjIndex::kNodeCuts);
  const int32_t* key = arr(a, direct ? AdjIndex::kDirectKey : AdjIndex::kNodeKey);
  if (a.one_task) {
    place_.resize((size_t)first[(size_t)T]);
    cuts_.resize((size_t)n_items * (size_t)(waves + 1));
    for (auto& s : source) key_.insert(key_.end(), s.begin(), s.end());
    for (int i = 0; i < n_items; ++i) {
      const AdjItem& it = item[i];
      const int64_t e0 = it.base - first[(size_t)it.t0];
      CHECK(it.nt == 1 && e0 >= 0 && it.base + it.count <= first[(size_t)it.t0 + 1]);
      CHECK((size_t)it.cuts + (size_t)waves < cuts_.size());
      for (int w = 0; w <= waves; ++w) cuts_[(size_t)(it.cuts + w)] = (int32_t)(e0 + (int64_t)it.count * w / waves);
      for (int u = 0; u < it.count; ++u) place_[(size_t)(it.base + u)] = (uint16_t)u;
    }
    place = place_.data();
    cuts = cuts_.data();
    key = key_.data();
  }
  std::vector<uint8_t> seen((size_t)first[(size_t)T], 0);
  std::vector<std::vector<int32_t>> found((size_t)T);
  int64_t recs = 0;
  for (int i = 0; i < n_items; ++i) {
    const AdjItem& it = item[i];
    CHECK(it.nt >= 1 && it.nt <= kAdjMaxTasks && it.t0 >= 0 && it.t0 + it.nt <= T);
    CHECK(it.count >= 1 && it.count <= cap);
    recs += it.count;
    for (int k = 0; k < it.nt; ++k) {
      const int t = it.t0 + k;
      const int32_t* c = cuts + it.cuts + k * (waves + 1);
      std::vector<uint8_t> used((size_t)it.count, 0);
      for (int w = 0; w < waves; ++w) {
        CHECK(c[w] <= c[w + 1] && c[w] >= 0 && c[w + 1] <= (int64_t)source[(size_t)t].size());
        for (int e = c[w]; e < c[w + 1]; ++e) {
          const int64_t v = first[(size_t)t] + e;
          CHECK(!seen[(size_t)v]);
          seen[(size_t)v] = 1;
          CHECK(place[v] < it.count && !used[place[v]]);
          used[place[v]] = 1;
          found[(size_t)t].push_back(key[it.base + place[v]]);
        }
      }
    }
  }
  CHECK(recs == (direct ? a.direct_recs : a.node_recs));
  for (int t = 0; t < T; ++t) {
    std::sort(found[(size_t)t].begin(), found[(size_t)t].end());
    std::sort(source[(size_t)t].begin(), source[(size_t)t].end());
    CHECK(found[(size_t)t] == source[(size_t)t]);
  }
  const int32_t* sorted = arr(a, direct ? AdjIndex::kDirectSorted : AdjIndex::kNodeSorted);
  for (int64_t r = 1; r < recs; ++r) {  // by key, in record order within one
    const int32_t p = sorted[r - 1], q = sorted[r];
    CHECK(key[p] < key[q] || (key[p] == key[q] && p < q));
  }
  return 0;
}

}  // namespace

// A build in which the k-th allocation fails, for every k up to the last: std::bad_alloc or kAdjIndexNoMemory, and
// nothing else (an exception that leaves with threads running would end the process).
int without_memory() {
  const Input x = make(2, 7, 900);  // (enough visits for several threads)
  for (int n_cu : {1, 100000})
    for (long k = 0;; ++k) {
      AdjIndex a;
      int r = kAdjIndexNoMemory;
      g_left = k;
      try {
        r = adj_index_build(x.in(n_cu), &a);
      } catch (const std::bad_alloc&) {
      }
      const bool refused = g_left.exchange(-1) < 0;
      if (!refused) break;  // fewer than k + 1 allocations
      if (r != kAdjIndexNoMemory && r != kAdjIndexOk) {  // (threads that could not be made are done without)
        std::printf("allocation %ld: %d\n", k, r);
        return 1;
      }
    }
  std::puts("ok");
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && !std::strcmp(argv[1], "memory")) return without_memory();
  for (int form = 0; form < 3; ++form)
    for (int seed = 0; seed < 6; ++seed) {
      const Input x = make(form, seed, form == 2 ? 200 : 2000);
      // one CU: items of several tasks; 100,000 of them: an item a task
      for (int n_cu : {1, 100000}) {
        AdjIndex a;
        const int r = adj_index_build(x.in(n_cu), &a);
        CHECK(r == kAdjIndexOk);
        if (check(x, a, false, form, seed) || check(x, a, true, form, seed)) return 1;
      }
    }
  std::puts("ok");
  return 0;
}
