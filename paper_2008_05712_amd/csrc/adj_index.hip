// Indices of the gravity adjoint, built on the host at the first backward call of a batch (host code).
//
// Consecutive tasks are gathered into items whose distinct nodes (and, apart from them, direct sources)
// fit the task kernel's LDS table; every distinct source of an item has one gradient record, ascending
// within the item.  Records are then grouped by node (each node's run cut into chunks of at most
// kVisitChunk) and by source id, by counting sorts that keep the record order.
//
// The tasks are cut into segments that threads index side by side (an item never spans two), and
// what the device cannot write itself goes up in one block: one allocation and one copy.  For Plummer 262,144
// (18.4 M node and 9.3 M direct visits) that and the two passes over the visits are what a first call
// waits for.  Batches of few tasks have an item a task: the sorts alone are made here (4,096 uniform particles
// 0.41 ms the first call, 0.55 with records, places and cuts written here; 8,000: 1.2 and 1.6).
#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>
#include <numeric>
#include <thread>

#include "gc_internal.h"

namespace gc {
namespace {

// The items of one segment of tasks, over one kind of source.
struct Groups {
  std::vector<AdjItem> items;
  std::vector<int64_t> work;    // per item: (targets + 1) x visits
  std::vector<int32_t> key;     // per record: its node or source id
  std::vector<uint16_t> place;  // per visit: its record's place in its item
  std::vector<int32_t> cuts;    // per item and task: waves + 1 visits of the task
  int64_t first_visit = 0;      // of the segment
};

struct Mark {  // what a thread knows of one source
  int32_t owner = -1;  // the open item that has it
  int32_t seen = -1;   // the last task pass that met it
  int32_t times = 0;   // its visits by that task so far
  int32_t copies = 0;  // records it needs in the open item: its most visits by one task
  int32_t spot = 0;    // the first of them
};

struct Scratch {
  std::vector<Mark> mark;
  std::vector<uint64_t> bits;
  int32_t stamp = 0, pass = 0;
  void size_for(int32_t n_keys) {
    if (mark.size() < (size_t)n_keys) mark.resize((size_t)n_keys);
    if (bits.size() < (size_t)n_keys / 64 + 1) bits.resize((size_t)n_keys / 64 + 1, 0);
  }
};

// Items of tasks [ta, tb).  sources(t, buf) gives where task t's visits lie: the base of the array (read again
// after every call: `buf` may have moved) and the offset of its first; count(t) their number.  A source listed twice by one
// task has two records: no two visits of a task share one.
template <class Count, class Sources, class Base>
void group_tasks(const gc_task* tasks, int32_t ta, int32_t tb, int cap, int waves, int max_tasks, Count&& count,
                 Sources&& sources, Base&& base, Scratch& s, Groups* out) {
  struct Part {
    int32_t task, e0, n;  // the task's visits [e0, e0 + n)
    int64_t at;           // where they are
    bool sorted;
  };
  std::vector<Part> parts;
  std::vector<int32_t> buf, mine, tmp, cost, bound((size_t)waves + 1);
  std::vector<std::pair<int32_t, int32_t>> undo;  // sources of earlier parts that got more copies, and how many they had
  int32_t held = 0;                               // records of the open item
  Mark* M = s.mark.data();
  ++s.stamp;
  {
    int64_t visits = 0;
    for (int32_t t = ta; t < tb; ++t) visits += count(t);
    out->place.reserve((size_t)visits);
    out->key.reserve((size_t)visits / 2);
    out->cuts.reserve((size_t)(tb - ta) * (size_t)(waves + 1));
  }
  auto meet = [&](Part& p) {
    // (plain pointers and locals: nothing is reloaded for fear of aliasing)
    const int32_t* v = base(buf) + p.at;
    const size_t before = mine.size();
    mine.resize(before + (size_t)p.n);
    int32_t* add = mine.data() + before;
    const int32_t stamp = s.stamp, pass = ++s.pass, n = p.n;
    Mark* const marks = M;
    int32_t last = -1, out_of_order = 0, more = 0;
    for (int32_t e = 0; e < n; ++e) {
      const int32_t k = v[e];
      out_of_order |= last > k;
      last = k;
      Mark& m = marks[k];
      if (m.owner != stamp) {
        m = Mark{stamp, pass, 1, 1, 0};
        *add++ = k;
      } else if (m.seen != pass) {
        m.seen = pass;
        m.times = 1;
      } else if (++m.times > m.copies) {
        undo.push_back({k, m.copies});
        ++m.copies;
        ++more;
      }
    }
    p.sorted = !out_of_order;
    const size_t fresh = (size_t)(add - (mine.data() + before));
    mine.resize(before + fresh);
    held += (int32_t)fresh + more;
    return before;
  };
  auto close = [&]() {
    if (!mine.empty()) {
      // distinct sources ascending, through a bitmap where they lie close enough
      int32_t low = mine[0] >> 6, high = low;
      for (int32_t k : mine) {
        low = std::min(low, k >> 6);
        high = std::max(high, k >> 6);
      }
      if ((size_t)(high - low) < 8 * mine.size()) {
        for (int32_t k : mine) s.bits[(size_t)(k >> 6)] |= 1ull << (k & 63);
        size_t q = 0;
        for (int32_t w = low; w <= high; ++w) {
          for (uint64_t x = s.bits[(size_t)w]; x; x &= x - 1) mine[q++] = 64 * w + __builtin_ctzll(x);
          s.bits[(size_t)w] = 0;
        }
      } else {
        std::sort(mine.begin(), mine.end());
      }
      AdjItem it{parts[0].task, (int32_t)parts.size(), (int32_t)out->key.size(), 0, (int32_t)out->cuts.size()};
      for (int32_t k : mine) {
        M[k].spot = it.count;
        it.count += M[k].copies;
        for (int32_t q = 0; q < M[k].copies; ++q) out->key.push_back(k);
      }
      cost.assign((size_t)it.count, 0);
      size_t at = out->place.size();
      const size_t first = at;
      int64_t total = 0;
      for (const Part& p : parts) {
        const int32_t w = tasks[p.task].i_count + 1;
        const int32_t* v = base(buf) + p.at;
        if (!p.sorted) {
          tmp.assign(v, v + p.n);
          std::sort(tmp.begin(), tmp.end());
          v = tmp.data();
        }
        out->place.resize(at + (size_t)p.n);
        uint16_t* to = out->place.data() + at;
        int32_t* spent = cost.data();
        const Mark* const marks = M;
        int32_t last = -1, again = 0;
        const int32_t n = p.n;
        for (int32_t e = 0; e < n; ++e) {
          again = v[e] == last ? again + 1 : 0;
          last = v[e];
          const int32_t spot = marks[last].spot + again;
          to[e] = (uint16_t)spot;
          spent[spot] += w;
        }
        at += (size_t)n;
        total += (int64_t)w * p.n;
      }
      // the wavefronts' stretches of records: equal shares of the cost
      int64_t run = 0;
      int w = 1;
      bound[0] = 0;
      for (int32_t p = 0; p < it.count; ++p) {
        while (w < waves && run * waves >= total * w) bound[(size_t)w++] = p;
        run += cost[(size_t)p];
      }
      while (w <= waves) bound[(size_t)w++] = it.count;
      at = first;
      for (const Part& p : parts) {
        const uint16_t* q = out->place.data() + at;
        for (int x = 0; x <= waves; ++x)
          out->cuts.push_back(p.e0 + (int32_t)(std::lower_bound(q, q + p.n, bound[(size_t)x]) - q));
        at += (size_t)p.n;
      }
      out->items.push_back(it);
      out->work.push_back(total);
    }
    parts.clear();
    mine.clear();
    undo.clear();
    held = 0;
    ++s.stamp;
  };
  for (int32_t t = ta; t < tb; ++t) {
    const int64_t n = count(t);
    if (n == 0) {  // no visits, but a place among an item's consecutive tasks (a closed item needs none)
      if ((int)parts.size() >= max_tasks) close();
      if (!parts.empty()) parts.push_back(Part{t, 0, 0, 0, true});
      continue;
    }
    if (n > cap) {  // a long task: stretches of at most `cap` visits
      close();
      buf.clear();
      const int64_t at = sources(t, buf);
      for (int64_t e = 0; e < n; e += cap) {
        parts.push_back(Part{t, (int32_t)e, (int32_t)std::min<int64_t>(cap, n - e), at + e, true});
        (void)meet(parts[0]);
        close();
      }
      buf.clear();
      continue;
    }
    if ((int)parts.size() >= max_tasks) close();
    if (parts.empty()) buf.clear();
    Part p{t, 0, (int32_t)n, sources(t, buf), true};
    undo.clear();
    const size_t before = meet(p);
    if (held > cap) {  // it does not fit: take its marks back and open another item with it
      for (size_t q = before; q < mine.size(); ++q) M[mine[q]].owner = -1;
      mine.resize(before);
      for (size_t q = undo.size(); q-- > 0;) M[undo[q].first].copies = undo[q].second;
      close();
      buf.clear();
      p.at = sources(t, buf);
      (void)meet(p);
    }
    parts.push_back(p);
  }
  close();
}

// f(0) ... f(n - 1) on up to `threads` threads; false if one of them ran out of memory.  (Nothing may be thrown from here
// while threads run: std::bad_alloc comes from making one, too, beside std::system_error.)
template <class F>
bool run_jobs(int threads, int n, F&& f) {
  std::atomic<int> next{0};
  std::atomic<bool> ok{true};
  auto work = [&](int thread) {
    try {
      for (int j = next++; j < n; j = next++) f(thread, j);
    } catch (...) {
      ok = false;
    }
  };
  std::vector<std::thread> pool;
  pool.reserve((size_t)std::max(threads - 1, 0));
  try {
    for (int t = 1; t < std::min(threads, n); ++t) pool.emplace_back(work, t);
  } catch (...) {  // fewer threads than asked for
  }
  work(0);
  for (std::thread& t : pool) t.join();
  return ok;
}

// Records grouped by key: start (n_keys + 1 entries) and, in record order within a key, rec.  each(p, f) calls f(record,
// key) for slice p of the records, in order.  A thread counts and places a slice; the slices' places of a key follow
// one another.
template <class Each>
bool sort_by_key(int threads, int P, size_t n, int32_t n_keys, Each&& each, std::vector<int32_t>* start, int32_t* rec) {
  const size_t K = (size_t)n_keys;
  std::vector<int32_t> fill((size_t)P * K, 0), base((size_t)P, 0);
  start->resize(K + 1);
  auto keys = [&](int p) { return K * (size_t)p / (size_t)P; };
  bool ok = run_jobs(threads, P, [&](int, int p) {
    int32_t* const f = fill.data() + (size_t)p * K;
    each(p, [f](int32_t, int32_t k) { ++f[(size_t)k]; });
  });
  // the first place of each slice of each key: within a run of keys, then past the runs before
  ok = ok && run_jobs(threads, P, [&](int, int q) {
    int32_t at = 0;
    for (size_t k = keys(q); k < keys(q + 1); ++k)
      for (int p = 0; p < P; ++p) {
        int32_t& f = fill[(size_t)p * K + k];
        const int32_t c = f;
        f = at;
        at += c;
      }
    base[(size_t)q] = at;
  });
  int32_t sum = 0;
  for (int32_t& b : base) {
    const int32_t c = b;
    b = sum;
    sum += c;
  }
  ok = ok && run_jobs(threads, P, [&](int, int q) {
    for (size_t k = keys(q); k < keys(q + 1); ++k) {
      for (int p = 0; p < P; ++p) fill[(size_t)p * K + k] += base[(size_t)q];
      (*start)[k] = fill[k];
    }
  });
  (*start)[K] = (int32_t)n;
  return ok && run_jobs(threads, P, [&](int, int p) {
    int32_t* const f = fill.data() + (size_t)p * K;
    each(p, [f, rec](int32_t r, int32_t k) { rec[(size_t)f[(size_t)k]++] = r; });
  });
}

int slices(int threads, size_t n) { return (int)std::max<size_t>(1, std::min<size_t>((size_t)threads, n / 50000)); }

// One kind of source, ready to be laid out.
struct Side {
  std::vector<AdjItem> items;  // longest first
  size_t recs = 0, cuts = 0;
  int64_t visits = 0;
};

// Items longest first, to a part in 1,024 of the longest: a long one that starts last would leave most of the chip idle
// (814 -> 613 us for the node items of Plummer 262,144).
void longest_first(std::vector<AdjItem>* items, const std::vector<int64_t>& work) {
  constexpr int kSteps = 1024;
  const int64_t most = work.empty() ? 1 : std::max<int64_t>(1, *std::max_element(work.begin(), work.end()));
  auto step = [&](size_t k) { return kSteps - 1 - (int)((double)work[k] / (double)most * (kSteps - 1)); };
  std::vector<int32_t> at(kSteps + 1, 0);
  for (size_t k = 0; k < work.size(); ++k) ++at[(size_t)step(k) + 1];
  std::partial_sum(at.begin(), at.end(), at.begin());
  std::vector<AdjItem> sorted(items->size());
  for (size_t k = 0; k < work.size(); ++k) sorted[(size_t)at[(size_t)step(k)]++] = (*items)[k];
  items->swap(sorted);
}

// The places of the arrays, and room for those that are built here.
bool lay_out(const AdjIndexInput& in, const Side& node, const Side& direct, bool one_task, AdjIndex* out) {
  size_t bytes = 0;
  auto place = [&](int which, size_t b) {
    out->at[which] = bytes;
    bytes += (b + 255) / 256 * 256 + 256;
  };
  auto places = [&]() {
    place(AdjIndex::kNodePlace, 2 * (size_t)node.visits);
    place(AdjIndex::kDirectPlace, 2 * (size_t)direct.visits);
    place(AdjIndex::kNodeCuts, 4 * node.cuts);
    place(AdjIndex::kDirectCuts, 4 * direct.cuts);
    place(AdjIndex::kNodeKey, 4 * node.recs);
    place(AdjIndex::kDirectKey, 4 * direct.recs);
  };
  place(AdjIndex::kNodeItems, sizeof(AdjItem) * node.items.size());
  place(AdjIndex::kDirectItems, sizeof(AdjItem) * direct.items.size());
  place(AdjIndex::kNodeFirst, 4 * ((size_t)in.n_tasks + 1));
  place(AdjIndex::kNodeSorted, 4 * node.recs);
  place(AdjIndex::kDirectSorted, 4 * direct.recs);
  if (!one_task) places();
  place(AdjIndex::kChunkFirst, 4 * ((size_t)in.n_nodes + 1));
  // at most one partial chunk per node beside the full ones
  place(AdjIndex::kChunks, 8 * (node.recs / kVisitChunk + (size_t)in.n_nodes + 1));
  const size_t here = bytes;
  if (one_task) places();
  place(AdjIndex::kDirectPacked, 4 * direct.recs);
  place(AdjIndex::kDirectSortedKey, 4 * direct.recs);
  out->room = bytes;
  out->one_task = one_task;
  // (huge pages where the system gives them: the first touch of small ones takes as long as filling them)
  const size_t huge = (size_t)2 << 20;
  out->blob.reset(static_cast<char*>(std::aligned_alloc(huge, (here + huge - 1) / huge * huge)));
  if (!out->blob) return false;
  if (here >= huge) (void)madvise(out->blob.get(), here, MADV_HUGEPAGE);
  auto put = [&](int which, const std::vector<AdjItem>& v) {
    if (!v.empty()) std::memcpy(out->blob.get() + out->at[which], v.data(), sizeof(AdjItem) * v.size());
  };
  put(AdjIndex::kNodeItems, node.items);
  put(AdjIndex::kDirectItems, direct.items);
  out->node_items = (int32_t)node.items.size();
  out->direct_items = (int32_t)direct.items.size();
  for (const AdjItem& it : node.items) out->max_nodes = std::max(out->max_nodes, it.count);
  for (const AdjItem& it : direct.items) out->max_direct = std::max(out->max_direct, it.count);
  out->node_recs = (int64_t)node.recs;
  out->direct_recs = (int64_t)direct.recs;
  return true;
}

template <class T = int32_t>
T* array_of(AdjIndex* x, int which) {
  return reinterpret_cast<T*>(x->blob.get() + x->at[which]);
}

// The records of each node in chunks; each: as in sort_by_key.
template <class Each>
bool sort_nodes(const AdjIndexInput& in, int threads, int P, Each&& each, AdjIndex* out) {
  std::vector<int32_t> start;
  if (!sort_by_key(threads, P, (size_t)out->node_recs, in.n_nodes, each, &start, array_of(out, AdjIndex::kNodeSorted)))
    return false;
  int32_t* first = array_of(out, AdjIndex::kChunkFirst);
  int32_t* chunk = array_of(out, AdjIndex::kChunks);
  int32_t n_chunks = 0;
  for (int32_t n = 0; n < in.n_nodes; ++n) {
    first[n] = n_chunks;
    const int32_t end = start[(size_t)n + 1];
    for (int32_t c = start[(size_t)n]; c < end; c += kVisitChunk) {
      chunk[2 * n_chunks] = c;
      chunk[2 * n_chunks + 1] = std::min(c + kVisitChunk, end);
      ++n_chunks;
    }
  }
  first[in.n_nodes] = n_chunks;
  out->chunks = n_chunks;
  out->bytes = out->at[AdjIndex::kChunks] + 8 * (size_t)std::max(n_chunks, 1);
  return true;
}

// The direct records by source id.
template <class Each>
bool sort_direct(const AdjIndexInput& in, int threads, int P, Each&& each, AdjIndex* out) {
  std::vector<int32_t> start;
  return sort_by_key(threads, P, (size_t)out->direct_recs, in.n_ids, each, &start, array_of(out, AdjIndex::kDirectSorted));
}

// f(0, threads) and f(1, threads), side by side where there is more than one thread (60,000 Plummer particles in buckets
// of 32: 7.5 instead of 8.6 ms the first call).
template <class F>
bool both_sides(int threads, F&& f) {
  const int at_once = std::min(threads, 2), half = threads / at_once;
  std::atomic<bool> ok{true};
  const bool room = run_jobs(at_once, 2, [&](int, int j) {
    if (!f(j, half)) ok = false;
  });
  return room && ok;
}

// A node index at or past n_nodes among the entries of tasks [ta, tb), or -1.
int64_t bad_node(const AdjIndexInput& in, int32_t ta, int32_t tb) {
  for (int32_t t = ta; t < tb; ++t)
    for (int32_t e = 0; e < in.tasks[t].n_count; ++e)
      if (in.nodes[in.tasks[t].n_first + e] >= in.n_nodes) return (int64_t)in.tasks[t].n_first + e;
  return -1;
}

// Segments of consecutive tasks with about equal visits.
std::vector<int32_t> cut_tasks(int segs, const std::vector<int32_t>& noff, const std::vector<int32_t>& joff) {
  const int32_t T = (int32_t)noff.size() - 1;
  const int64_t visits = (int64_t)noff[(size_t)T] + joff[(size_t)T];
  std::vector<int32_t> cut((size_t)segs + 1, T);
  cut[0] = 0;
  for (int g = 1; g < segs; ++g) {
    int32_t lo = cut[(size_t)g - 1], hi = T;
    while (lo < hi) {
      const int32_t mid = lo + (hi - lo) / 2;
      if ((int64_t)noff[(size_t)mid] + joff[(size_t)mid] < visits * g / segs) lo = mid + 1;
      else hi = mid;
    }
    cut[(size_t)g] = lo;
  }
  return cut;
}

// An item per task (or stretch of a long one) and a record per visit, in order: records, places and cuts follow from the
// items alone and are written on the device; only the sorts are made here, from the lists themselves.
int index_tasks(const AdjIndexInput& in, int threads, const std::vector<int32_t>& noff, const std::vector<int32_t>& joff,
                AdjIndex* out) {
  Side side[2];
  const std::vector<int32_t>* off[2] = {&noff, &joff};
  const int cap[2] = {kAdjMaxNodes, kAdjMaxDirect}, waves[2] = {kAdjNodeWaves, kAdjDirectWaves};
  for (int k = 0; k < 2; ++k) {
    std::vector<int64_t> work;
    const std::vector<int32_t>& o = *off[k];
    for (int32_t t = 0; t < in.n_tasks; ++t)
      for (int32_t e = o[(size_t)t]; e < o[(size_t)t + 1]; e += cap[k]) {
        const int32_t n = std::min(cap[k], o[(size_t)t + 1] - e);
        side[k].items.push_back(AdjItem{t, 1, e, n, (int32_t)side[k].cuts});
        side[k].cuts += (size_t)waves[k] + 1;
        work.push_back((int64_t)(in.tasks[t].i_count + 1) * n);
      }
    side[k].recs = (size_t)o[(size_t)in.n_tasks];
    side[k].visits = o[(size_t)in.n_tasks];
    longest_first(&side[k].items, work);
  }
  if (!lay_out(in, side[0], side[1], true, out)) return kAdjIndexNoMemory;
  std::memcpy(array_of(out, AdjIndex::kNodeFirst), noff.data(), 4 * noff.size());
  const int segs = threads == 1 ? 1 : 4 * threads;
  const std::vector<int32_t> cut = cut_tasks(segs, noff, joff);
  std::atomic<int64_t> bad{-1};
  bool ok = run_jobs(threads, segs, [&](int, int g) {
    const int64_t wrong = bad_node(in, cut[(size_t)g], cut[(size_t)g + 1]);
    if (wrong >= 0) bad = wrong;
  });
  if (bad >= 0) {
    out->bad_entry = bad;
    return kAdjIndexBadNode;
  }
  ok = ok && both_sides(threads, [&](int k, int n) {
    const std::vector<int32_t>& o = *off[k];
    const int P = slices(n, side[k].recs);
    // the tasks of slice p
    auto first = [&](int p) {
      if (p == P) return in.n_tasks;
      return (int32_t)(std::lower_bound(o.begin(), o.end() - 1, (int32_t)(side[k].recs * (size_t)p / (size_t)P)) - o.begin());
    };
    if (k)
      return sort_direct(in, n, P, [&](int p, auto&& f) {
        int32_t r = o[(size_t)first(p)];
        for (int32_t t = first(p), e = first(p + 1); t < e; ++t)
          for (int32_t j = in.tasks[t].j_first, je = j + in.tasks[t].j_nranges; j < je; ++j)
            for (int32_t g = in.ranges[2 * j], ge = g + in.ranges[2 * j + 1]; g < ge; ++g) f(r++, g);
      }, out);
    return sort_nodes(in, n, P, [&](int p, auto&& f) {
      for (int32_t t = first(p), e = first(p + 1); t < e; ++t) {
        const int32_t* nodes = in.nodes + in.tasks[t].n_first;
        const int32_t r = o[(size_t)t];
        for (int32_t v = 0, c = in.tasks[t].n_count; v < c; ++v) f(r + v, nodes[v]);
      }
    }, out);
  });
  return ok ? kAdjIndexOk : kAdjIndexNoMemory;
}

}  // namespace

int adj_index_build(const AdjIndexInput& in, AdjIndex* out) {
  const int32_t T = in.n_tasks;
  std::vector<int32_t> noff((size_t)T + 1, 0), joff((size_t)T + 1, 0);
  int64_t nv = 0, nd = 0;
  for (int32_t t = 0; t < T; ++t) {
    noff[(size_t)t] = (int32_t)nv;
    joff[(size_t)t] = (int32_t)nd;
    nv += in.tasks[t].n_count;
    for (int32_t r = 0; r < in.tasks[t].j_nranges; ++r) nd += in.ranges[2 * (in.tasks[t].j_first + r) + 1];
    if (nv > INT32_MAX || nd > INT32_MAX) return kAdjIndexTooLarge;
  }
  noff[(size_t)T] = (int32_t)nv;
  joff[(size_t)T] = (int32_t)nd;
  // Enough items to fill the chip (four per CU), then as many tasks in each as share well.  Below five tasks an item the
  // shared records save less than finding them costs: uniform 57,555 in buckets of 32 (4,096 tasks) 2.6 ms the first
  // call and 145 us the others with an item a task, 4.2 and 162 with items of four; 30,000 in buckets of 16 1.9 and
  // 93 against 3.4 and 91.  Plummer 60,000 in buckets of 32 (6,455 tasks, items of six): 5.0 and 317 against 7.7 and 278,
  // 40,000 in buckets of 16 (seven) 5.9 and 282 against 6.2 and 203.
  const int per_item = T / (4 * std::max(in.n_cu, 1));
  const int64_t visits = nv + nd;
  const int32_t most_keys = std::max(in.n_nodes, in.n_ids);
  // one thread up to 600,000 visits (starting the others would cost more: with every visit's record written here 1.5
  // against 1.8 ms for 8,000 uniform particles in buckets of 16), then one per 200,000, at most 16, and at most 512 MB of
  // marks among them
  const int threads =
      visits < 600000 ? 1
                      : (int)std::min<int64_t>({16, std::max(1u, std::thread::hardware_concurrency()), 1 + visits / 200000,
                                                std::max<int64_t>(1, (512ll << 20) / (int64_t)(sizeof(Mark) * (size_t)most_keys + 1))});
  if (per_item < 5) return index_tasks(in, threads, noff, joff, out);
  const int max_tasks = std::min(kAdjMaxTasks, per_item);
  const int segs = threads == 1 ? 1 : 4 * threads;
  const std::vector<int32_t> cut = cut_tasks(segs, noff, joff);
  std::vector<Groups> found[2] = {std::vector<Groups>((size_t)segs), std::vector<Groups>((size_t)segs)};  // nodes, direct
  std::vector<Scratch> scratch((size_t)threads);
  std::atomic<int64_t> bad{-1};
  bool ok = run_jobs(threads, 2 * segs, [&](int thread, int job) {
    const int g = job >> 1;
    const int32_t ta = cut[(size_t)g], tb = cut[(size_t)g + 1];
    if (ta >= tb) return;
    Scratch& s = scratch[(size_t)thread];
    s.size_for(most_keys);
    Groups& to = found[job & 1][(size_t)g];
    if (job & 1) {
      to.first_visit = joff[(size_t)ta];
      group_tasks(
          in.tasks, ta, tb, kAdjMaxDirect, kAdjDirectWaves, max_tasks,
          [&](int32_t t) { return (int64_t)joff[(size_t)t + 1] - joff[(size_t)t]; },
          [&](int32_t t, std::vector<int32_t>& buf) {
            const int64_t at = (int64_t)buf.size();
            for (int32_t r = 0; r < in.tasks[t].j_nranges; ++r) {
              const int32_t g0 = in.ranges[2 * (in.tasks[t].j_first + r)], gn = in.ranges[2 * (in.tasks[t].j_first + r) + 1];
              const size_t q = buf.size();
              buf.resize(q + (size_t)gn);
              std::iota(buf.begin() + (int64_t)q, buf.end(), g0);
            }
            return at;
          },
          [](std::vector<int32_t>& buf) { return (const int32_t*)buf.data(); }, s, &to);
    } else {
      to.first_visit = noff[(size_t)ta];
      const int64_t e = bad_node(in, ta, tb);
      if (e >= 0) {
        bad = e;
        return;
      }
      group_tasks(
          in.tasks, ta, tb, kAdjMaxNodes, kAdjNodeWaves, max_tasks,
          [&](int32_t t) { return (int64_t)in.tasks[t].n_count; },
          [&](int32_t t, std::vector<int32_t>&) { return (int64_t)in.tasks[t].n_first; },
          [&](std::vector<int32_t>&) { return in.nodes; }, s, &to);
    }
  });
  if (bad >= 0) {
    out->bad_entry = bad;
    return kAdjIndexBadNode;
  }
  if (!ok) return kAdjIndexNoMemory;

  // the segments' records and cuts one after another
  Side side[2];
  std::vector<size_t> rec0[2], cut0[2];
  for (int k = 0; k < 2; ++k) {
    std::vector<int64_t> work;
    for (const Groups& g : found[k]) {
      rec0[k].push_back(side[k].recs);
      cut0[k].push_back(side[k].cuts);
      for (AdjItem it : g.items) {
        it.base += (int32_t)side[k].recs;
        it.cuts += (int32_t)side[k].cuts;
        side[k].items.push_back(it);
      }
      work.insert(work.end(), g.work.begin(), g.work.end());
      side[k].recs += g.key.size();
      side[k].cuts += g.cuts.size();
    }
    side[k].visits = k ? nd : nv;
    longest_first(&side[k].items, work);
  }
  if (!lay_out(in, side[0], side[1], false, out)) return kAdjIndexNoMemory;
  std::memcpy(array_of(out, AdjIndex::kNodeFirst), noff.data(), 4 * noff.size());
  ok = run_jobs(threads, 2 * segs, [&](int, int job) {
    const int k = job & 1;
    const size_t g = (size_t)(job >> 1);
    const Groups& q = found[k][g];
    auto put = [&](int which, const auto& v, size_t at) {
      if (!v.empty()) std::memcpy(out->blob.get() + out->at[which] + sizeof(v[0]) * at, v.data(), sizeof(v[0]) * v.size());
    };
    put(k ? AdjIndex::kDirectPlace : AdjIndex::kNodePlace, q.place, (size_t)q.first_visit);
    put(k ? AdjIndex::kDirectCuts : AdjIndex::kNodeCuts, q.cuts, cut0[k][g]);
    put(k ? AdjIndex::kDirectKey : AdjIndex::kNodeKey, q.key, rec0[k][g]);
  });
  ok = ok && both_sides(threads, [&](int k, int n) {
    const int32_t* key = array_of(out, k ? AdjIndex::kDirectKey : AdjIndex::kNodeKey);
    const size_t recs = side[k].recs;
    const int P = slices(n, recs);
    auto each = [&](int p, auto&& f) {
      for (size_t r = recs * (size_t)p / (size_t)P, e = recs * (size_t)(p + 1) / (size_t)P; r < e; ++r) f((int32_t)r, key[r]);
    };
    return k ? sort_direct(in, n, P, each, out) : sort_nodes(in, n, P, each, out);
  });
  return ok ? kAdjIndexOk : kAdjIndexNoMemory;
}

}  // namespace gc
