// Tile-task graph of one diagonal-block factorisation: the blocked
// right-looking Cholesky A = L L^T of an n x n block (nbk tiles of 64 x 64)
// with its inverse G = L^{-1} formed alongside, left-looking, as the tiles of
// L become final.  No HIP types: the engine builds the task lists of its
// persistent launches from it, the launch's kernel decodes tasks and their
// waits with it, and a CPU emulator in the tests runs the same lists on plain
// arrays.
//
// Tasks (tiles indexed (row, column), lower triangle):
//   F(k)        factor diagonal tile (k, k) (all its updates applied):
//               G_kk = L_kk^{-1} in place, log L_ii, first bad pivot
//   S(i, k)     solve L(i, k) = A(i, k) G_kk^T  (into the L buffer)
//   U(i, k, j)  A(i, k) -= L(i, j) L(k, j)^T   (j < k <= i)
//   A(r, c, m)  accumulate S(r, c) += L(r, m) G(m, c)   (c <= m <= r - 2)
//   R(j, c)     G(j, c) = -G_jj (S(j, c) + L(j, j-1) G(j-1, c))   (c < j)
//   C(k)        the chain from tile k to tile k+1 in one task: S(k+1, k),
//               then U(k+1, k+1, k) and F(k+1) on the tiles it holds
// G(j, c) goes into A(j, c) (read by nobody once S(j, c) has run), so on
// completion the block holds G in its lower triangle.  In the chained form
// (the one launches use) C(k) stands for S(k+1, k), U(k+1, k+1, k) and
// F(k+1): the factorisation's critical path -- each tile factor, the solve of
// the tile below it and that tile's last update -- then runs as one task per
// tile without handing tiles between workgroups, and C(k) publishes L(k+1, k)
// as soon as it is stored, before its update and factor.
//
// Readiness is tracked by one counter per tile and one per accumulator:
//   v(r, c): number of updates applied (0 .. c); c + 1 once L(r, c) (or G_cc
//            for r = c) is final; c + 2 once G(r, c) is final (r > c);
//   a(r, c): number of accumulated terms.
// Every task waits for counters to reach given values and then sets one
// counter (after its stores are complete).  A launch's task list is sorted
// by each task's latest start level (the longest chain of tasks after it,
// counted back from the end of the graph), ties by earliest start level, so
// every value a task waits for is set by a task earlier in the list (a
// dependency's latest start is strictly smaller), and the chain that bounds
// the factorisation -- each tile factor, the solve of the tile below it and
// that tile's last update -- comes before updates that are needed later.  A
// worker that takes tasks from the list in order only ever waits on tasks
// that running workers hold, so the launch cannot deadlock.
#pragma once

#include <stdint.h>

// Functions the device also calls (task decoding, waits) carry DL_DAG_FN,
// which a HIP translation unit defines as __host__ __device__ inline before
// including this header.
#ifndef DL_DAG_FN
#define DL_DAG_FN inline
#endif

#include <algorithm>
#include <map>
#include <tuple>
#include <vector>

namespace dl {
namespace dag {

enum : int { T_F = 0, T_S = 1, T_U = 2, T_A = 3, T_R = 4, T_C = 5 };

struct Task {
  int type;
  int i, k, j;  // F: (k, k, k); S: (i, k, k); U: (i, k, j); A: (r, c, m); R: (j, c, c);
                // C: (k + 1, k, k)
  int n = 1;    // U, A: the tasks of j, j + 1, .., j + n - 1 in one (see join)
};

// Counter indices within a block: tiles first, then accumulators.
DL_DAG_FN int64_t tile_ctr(int r, int c) { return (int64_t)r * (r + 1) / 2 + c; }
DL_DAG_FN int64_t acc_ctr(int nbk, int r, int c) {
  return (int64_t)nbk * (nbk + 1) / 2 + (int64_t)r * (r - 1) / 2 + c;
}
DL_DAG_FN int64_t counters_per_block(int nbk) { return (int64_t)nbk * nbk; }

// One wait: counter index and the value it must reach.
struct Wait {
  int64_t ctr;
  int value;
};

// The waits of task t (at most 4) and the counter it sets (and the value)
// when it completes.
DL_DAG_FN int waits_of(int nbk, const Task& t, Wait* w, Wait* sets) {
  int n = 0;
  const int last = t.j + t.n - 1;
  auto gfinal = [&](int m, int c) {  // G(m, c) final
    if (m == c) w[n++] = {tile_ctr(c, c), c + 1};
    else w[n++] = {tile_ctr(m, c), c + 2};
  };
  switch (t.type) {
    case T_F:
      w[n++] = {tile_ctr(t.k, t.k), t.k};
      *sets = {tile_ctr(t.k, t.k), t.k + 1};
      break;
    case T_S:
      w[n++] = {tile_ctr(t.i, t.k), t.k};
      w[n++] = {tile_ctr(t.k, t.k), t.k + 1};
      *sets = {tile_ctr(t.i, t.k), t.k + 1};
      break;
    case T_U:
      w[n++] = {tile_ctr(t.i, t.k), t.j};
      // L(i, last) final: so are the row's tiles before it, its updates
      w[n++] = {tile_ctr(t.i, last), last + 1};
      if (t.k != t.i) w[n++] = {tile_ctr(t.k, last), last + 1};
      *sets = {tile_ctr(t.i, t.k), last + 1};
      break;
    case T_A:  // (r, c, m) = (i, k, j); G(last, c) needed every G(m, c) before it
      if (t.j > t.k) w[n++] = {acc_ctr(nbk, t.i, t.k), t.j - t.k};
      w[n++] = {tile_ctr(t.i, last), last + 1};
      gfinal(last, t.k);
      *sets = {acc_ctr(nbk, t.i, t.k), last - t.k + 1};
      break;
    case T_R:  // (j, c) = (i, k)
      w[n++] = {tile_ctr(t.i, t.i), t.i + 1};
      if (t.i - 1 > t.k) w[n++] = {acc_ctr(nbk, t.i, t.k), t.i - 1 - t.k};
      w[n++] = {tile_ctr(t.i, t.i - 1), t.i};
      gfinal(t.i - 1, t.k);
      *sets = {tile_ctr(t.i, t.k), t.k + 2};
      break;
    case T_C:  // k = t.k: the waits of S(k+1, k), and the earlier updates of tile k+1
      w[n++] = {tile_ctr(t.k + 1, t.k), t.k};
      w[n++] = {tile_ctr(t.k, t.k), t.k + 1};
      w[n++] = {tile_ctr(t.k + 1, t.k + 1), t.k};
      *sets = {tile_ctr(t.k + 1, t.k + 1), t.k + 2};  // G(k+1, k+1) final
      break;
  }
  return n;
}

// The counter a task sets before it completes, if any: C(k) sets
// v(k+1, k) = k + 1 once L(k+1, k) is stored.  (Its final counter skips
// v(k+1, k+1) = k + 1, which only its own update would have set.)
DL_DAG_FN bool mid_set(const Task& t, Wait* s) {
  if (t.type != T_C) return false;
  *s = {tile_ctr(t.k + 1, t.k), t.k + 1};
  return true;
}

// The patience of a worker that polls for a counter, in clock ticks.  Only time spent
// polling counts, at most `step` for each poll: a process that is held off the
// card between two polls (time slices of other processes, a suspended queue) has
// not waited, for the workers it waits on were held off with it.
struct Patience {
  long long last;       // the clock at the poll before
  long long spent = 0;
  // After a poll that found nothing: true once `limit` is spent.
  DL_DAG_FN bool out(long long now, long long limit, long long step) {
    const long long d = now - last;
    spent += d < step ? d : step;
    last = now;
    return spent > limit;
  }
};

// All tasks of one block in phase order (step j: F(j), S(., j), R(j, .),
// U(., ., j), A(., ., j)), which is a valid order.  Chained: F(0), and in
// step j, C(j) in place of S(j+1, j) (it also stands for U(j+1, j+1, j) and
// F(j+1)).
inline std::vector<Task> phase_order(int nbk, bool inverse, bool chain = true) {
  std::vector<Task> q;
  q.reserve((size_t)nbk * (nbk + 1) * (nbk + 2) / (inverse ? 3 : 6) + (size_t)nbk * nbk);
  for (int j = 0; j < nbk; ++j) {
    if (!chain || j == 0) q.push_back({T_F, j, j, j});
    for (int i = j + 1; i < nbk; ++i)
      q.push_back(chain && i == j + 1 ? Task{T_C, j + 1, j, j} : Task{T_S, i, j, j});
    if (inverse)
      for (int c = 0; c < j; ++c) q.push_back({T_R, j, c, c});
    for (int k = j + 1; k < nbk; ++k)
      for (int i = k; i < nbk; ++i)
        if (!(chain && i == j + 1 && k == j + 1)) q.push_back({T_U, i, k, j});
    if (inverse)
      for (int c = 0; c <= j; ++c)
        for (int r = j + 2; r < nbk; ++r) q.push_back({T_A, r, c, j});
  }
  return q;
}

// The indices 0 .. n - 1 in increasing order of (a[i], b[i]), ties by index; both
// are levels from 0 to depth.
inline std::vector<int> by_levels(const std::vector<int>& a, const std::vector<int>& b,
                                  int depth) {
  const size_t n = a.size();
  std::vector<int> from(n), to(n);
  for (size_t i = 0; i < n; ++i) from[i] = (int)i;
  for (const std::vector<int>* key : {&b, &a}) {
    std::vector<size_t> at((size_t)depth + 2, 0);
    for (size_t i = 0; i < n; ++i) ++at[(*key)[i] + 1];
    for (int l = 0; l <= depth; ++l) at[l + 1] += at[l];
    for (size_t i = 0; i < n; ++i) to[at[(*key)[from[i]]]++] = from[i];
    from.swap(to);
  }
  return from;
}

// The block's tasks in phase order, with each one's earliest start level (longest
// chain of predecessors) and latest one (counted back from the end of the graph).
// Returns the last level.
inline int levels(int nbk, bool inverse, bool chain, std::vector<Task>& q,
                  std::vector<int>& asap, std::vector<int>& alap) {
  q = phase_order(nbk, inverse, chain);
  const size_t n = q.size();
  // the task that brings a counter to a value, by the counter's first place in
  // `prod` and the value (v(r, c): 0 .. c + 2, a(r, c): 0 .. r - 1 - c)
  std::vector<int> first((size_t)counters_per_block(nbk));
  int places = 0;
  for (int r = 0; r < nbk; ++r)
    for (int c = 0; c <= r; ++c) {
      first[tile_ctr(r, c)] = places;
      places += c + 3;
    }
  for (int r = 1; r < nbk; ++r)
    for (int c = 0; c < r; ++c) {
      first[acc_ctr(nbk, r, c)] = places;
      places += r - c;
    }
  std::vector<int> prod((size_t)places, -1), pred(4 * n, -1);
  asap.assign(n, 0);
  int depth = 0;
  // (phase order: a task's predecessors come before it)
  for (size_t t = 0; t < n; ++t) {
    Wait w[4], s;
    const int nw = waits_of(nbk, q[t], w, &s);
    for (int e = 0; e < nw; ++e) {
      if (w[e].value == 0) continue;
      // the task that brings the counter to the value (or past it: C(k)
      // steps v(k+1, k+1) by two)
      const int* p = &prod[first[w[e].ctr] + w[e].value];
      while (*p < 0) ++p;
      asap[t] = std::max(asap[t], asap[*p] + 1);
      pred[4 * t + e] = *p;
    }
    depth = std::max(depth, asap[t]);
    prod[first[s.ctr] + s.value] = (int)t;
    if (mid_set(q[t], &s)) prod[first[s.ctr] + s.value] = (int)t;
  }
  alap.assign(n, depth);
  for (size_t t = n; t-- > 0;)
    for (int e = 0; e < 4; ++e)
      if (const int p = pred[4 * t + e]; p >= 0) alap[p] = std::min(alap[p], alap[t] - 1);
  return depth;
}

// The block's tasks sorted by earliest start level, ties by latest start level, then
// by phase order.  Returns the tasks and, in `level` and `slack`, each one's
// earliest start level and the difference between its latest and earliest start
// levels.
inline std::vector<Task> schedule(int nbk, bool inverse, std::vector<int>* level = nullptr,
                                  std::vector<int>* slack = nullptr, bool chain = true) {
  std::vector<Task> q;
  std::vector<int> asap, alap;
  const int depth = levels(nbk, inverse, chain, q, asap, alap);
  const std::vector<int> idx = by_levels(asap, alap, depth);
  const size_t n = q.size();
  std::vector<Task> out(n);
  if (level) level->resize(n);
  if (slack) slack->resize(n);
  for (size_t t = 0; t < n; ++t) {
    out[t] = q[idx[t]];
    if (level) (*level)[t] = asap[idx[t]];
    if (slack) (*slack)[t] = alap[idx[t]] - asap[idx[t]];
  }
  return out;
}

// A task word: type and n - 1 (4 bits each), the three tile indices (12 bits
// each) and the block within the launch (20).
DL_DAG_FN uint64_t pack(const Task& t, int block) {
  return (uint64_t)t.type | ((uint64_t)(t.n - 1) << 4) | ((uint64_t)t.i << 8) |
         ((uint64_t)t.k << 20) | ((uint64_t)t.j << 32) | ((uint64_t)block << 44);
}
DL_DAG_FN Task unpack(uint64_t w, int* block) {
  *block = (int)(w >> 44);
  return Task{(int)(w & 0xf), (int)((w >> 8) & 0xfff), (int)((w >> 20) & 0xfff),
              (int)((w >> 32) & 0xfff), (int)((w >> 4) & 0xf) + 1};
}

// The tasks of single blocks, one list per block size (and inverse), as words of
// block 0 sorted by latest start level, ties by earliest start level, then by phase
// order.  The launches of a workspace repeat the same sizes: its lists share
// one of these.
struct Schedules {
  struct One {
    std::vector<uint64_t> words;
    std::vector<int> alap, asap;
  };
  std::map<std::tuple<int, bool, bool>, One> all;
  const One& at(int nbk, bool inverse, bool chain) {
    auto [it, fresh] = all.try_emplace({nbk, inverse, chain});
    One& one = it->second;
    if (!fresh) return one;
    std::vector<Task> q;
    std::vector<int> asap, alap;
    const int depth = levels(nbk, inverse, chain, q, asap, alap);
    one.words.reserve(q.size());
    one.alap.reserve(q.size());
    one.asap.reserve(q.size());
    for (int p : by_levels(alap, asap, depth)) {
      one.words.push_back(pack(q[p], 0));
      one.alap.push_back(alap[p]);
      one.asap.push_back(asap[p]);
    }
    return one;
  }
};

// The task list of one launch over several blocks (inverse[b]: block b's
// inverse is formed too): all blocks' tasks sorted by latest start level, then
// earliest start level, then block, then the block's own order.  The blocks' sorted
// lists are merged: with a schedule and a sort of everything for each of its lists, a
// workspace with blocks of 7 to 95 tiles was created in 42.5 ms, now in 21.2, one
// with blocks of 43 tiles in 4.2, now 2.0.
inline std::vector<uint64_t> launch_list(const std::vector<int>& nbks,
                                         const std::vector<char>& inverse, bool chain = true,
                                         Schedules* schedules = nullptr) {
  Schedules own;
  if (!schedules) schedules = &own;
  struct Part {
    const Schedules::One* one;
    uint64_t block;
    size_t at;
  };
  std::vector<Part> parts;
  size_t n = 0;
  for (size_t b = 0; b < nbks.size(); ++b) {
    parts.push_back({&schedules->at(nbks[b], inverse[b] != 0, chain), (uint64_t)b << 44, 0});
    n += parts[b].one->words.size();
  }
  std::vector<uint64_t> out;
  out.reserve(n);
  while (out.size() < n) {
    // the next pair of levels, and every block's tasks of that pair
    int64_t next = INT64_MAX;
    for (const Part& p : parts)
      if (p.at < p.one->words.size())
        next = std::min(next, ((int64_t)p.one->alap[p.at] << 32) | p.one->asap[p.at]);
    for (Part& p : parts)
      for (; p.at < p.one->words.size() &&
             (((int64_t)p.one->alap[p.at] << 32) | p.one->asap[p.at]) == next;
           ++p.at)
        out.push_back(p.one->words[p.at] | p.block);
  }
  return out;
}

// The list with the updates of a tile, and the terms of an accumulator, joined
// `most` (up to 16) at a time (j from one multiple of it to the next) into the
// word of the last of them: the tile is then read and written once for all of
// them, and their operands are loaded while the product before is formed.  Only
// the next task of the same tile waits on what a joined task would have set, so
// the list still only waits on earlier tasks.  The last update of a tile near
// the diagonal (i - k <= 4) stays alone: the chain waits for it.
inline std::vector<uint64_t> join(const std::vector<uint64_t>& list, int most) {
  std::vector<uint64_t> out;
  out.reserve(list.size());
  for (uint64_t w : list) {
    int b = 0;
    Task t = unpack(w, &b);
    if (t.type == T_U || t.type == T_A) {
      // one past the last index of the task's tile or accumulator that may join
      const int own = t.i == t.k ? t.k - 1 : t.k;  // C has the diagonal's last
      const int end = t.type == T_A ? t.i - 1 : (t.i - t.k <= 4 ? own - 1 : own);
      const int lo0 = t.j / most * most, lo = t.type == T_A && lo0 < t.k ? t.k : lo0;
      const int hi = lo0 + most < end ? lo0 + most : end;
      if (t.j < hi) {
        if (t.j + 1 < hi) continue;
        t.n = hi - lo;
        t.j = lo;
      }
    }
    out.push_back(pack(t, b));
  }
  return out;
}

// How many tasks to join in a launch of `words` tasks whose longest block has
// `nbk` tiles (the results are the same bits for any number).  By the tasks
// per step of the chain, with what 1 / 2 / 4 / 8 took in us:
//   * below 400 the workers mostly wait, and fewer of them take part in a tile's
//     updates: 2 x 15 tiles 274 / 250 / 243 / 264, 2 x 19 409 / 360 / 337 / 369,
//     1 x 32 701 / 667 / 614 / 684;
//   * then the chain competes with the updates, and the shortest tasks let it
//     through first: 15 x 10 216 / 227 / 246 / 273, 4 x 19 408 / 432 / 440 / 496,
//     2 x 32 690 / 724 / 742 / 802;
//   * from 850 on the updates' memory traffic counts: 9 x 19 620 / 541 / 520 / 607,
//     17 x 15 566 / 488 / 456 / 504, 2 x 43 1300 / 1193 / 1142 / 1229;
//   * from 2000 on it is all that does: 9 x 32 2826 / 2237 / 1932 / 1816, 31 x 19
//     2138 / 1743 / 1533 / 1435, 1 x 95 7806 / 6026 / 5153 / 4895.
inline int join_count(size_t words, int nbk) {
  const size_t per = words / (size_t)nbk;
  return per < 400 ? 4 : (per < 850 ? 1 : (per < 2000 ? 4 : 8));
}

inline std::vector<uint64_t> launch_list(const std::vector<int>& nbks, bool inverse,
                                         bool chain = true) {
  return launch_list(nbks, std::vector<char>(nbks.size(), inverse ? 1 : 0), chain);
}

}  // namespace dag
}  // namespace dl
