// k-clique search on a (kernelized) legally k-coloured graph (gfx950): the
// search the kernel is handed to.  A k-clique holds one vertex of every
// class; the search returns the lexicographically smallest one (class 0's
// vertex first, then class 1's, ...) among the live vertices, or none.
//
// Roots are the pairs (v0, v1) of live neighbours of class 0 x class 1 in
// lexicographic order: each wave starts with the one of its own number, the
// next ones come from an atomic counter.  (A counter over all pairs, dead and
// unconnected ones too, had every wave wait for it: 97 ns a pair on its one
// cache line, 3600 pairs 350 us.)
//
// Below a root a wave searches depth first, but by lists: the nodes of a level
// (partial cliques, in order, each with its common neighbourhood, the AND of
// the picked rows and the live mask over the classes left) give up to 64 picks
// of the next class at a time.  Lanes go over the picks' row words, as many
// picks at once as fit 64 lanes, the loads of four such steps in flight; a
// pick stays when every class after it still holds a candidate, and the picks
// that stay are the next level's list, as many as fit its room: the search
// goes below them before it comes back for the rest.  What one pick after the
// other made a chain of dependent loads (1.2 us each) is a few loads a list.
// Everything in a list comes before what is left for later, so the first list
// that reaches the last class holds, first, the smallest clique of what the
// wave searches.  12 classes of 90 at p = 0.4 and one planted clique, about
// 600 000 picks: 646 us one pick after the other with the counter, 100 now; it
// is bounded by the latency of the lists' loads and by the last roots to end.
//
// A root's level-2 node holds its class-2 vertices j, its children.  The wave
// that took it searches the first of them itself; once that has cost
// kClqShareAfter picks (or at once, where there are fewer roots than helpers) it
// opens the rest on its share word, and from then on any wave -- its own, or a
// helper (a wave of the first kClqHelperBlocks blocks that has run out of
// roots) -- takes the next kClqTake children with one atomic add.  The key of
// a child is (root, j) in lexicographic order; the smallest key with a clique
// holds the smallest clique overall: an atomic minimum over keys keeps it, and
// waves holding larger keys stop as soon as it is known.  Helpers only poll, a
// bounded number of times in a row, for work opened by waves that are already
// running; nothing else waits, so the launch cannot deadlock.
#include "kz_internal.h"

namespace kzi {

namespace {

constexpr int kClqWaves = 4;        // waves per workgroup
constexpr int kClqMaxWaves = 2048;  // waves of one launch (stack slots)
constexpr long long kClqNone = 0x7fffffffffffffffLL;
constexpr int kClqLdsWords = 1792;  // per-wave LDS lists when they fit
constexpr int kClqRoom = 16;        // nodes of a level's list at most
// share word of a slot: root << kClqSubBits | next child, or negative (no
// open children).  Vertices stay below kClqMaxN so that roots (< 2^40),
// children (< 2^21, plus at most one overshooting add of kClqTake per wave)
// and keys (root * s2 + j < 2^63) all fit.
constexpr int kClqSubBits = 22;
constexpr long long kClqSubMask = (1ll << kClqSubBits) - 1;
constexpr long long kClqClosed = -(1ll << 62);
constexpr int kClqMaxN = 1 << 21;
// a helper with no open child looks again at most this many times in a row
// (about 3.4 us apart) before it leaves: long enough for the long roots
// taken just before it to open, short enough not to hold the compute units
// from other work (other searches) while the last subtrees finish
constexpr int kClqIdlePolls = 32;
// a root opens its remaining children once its own wave has extended this
// many picks below it: short subtrees stay with their wave, long ones are
// shared (12 classes of 90 at p = 0.4, 608 000 picks: 227 us a call after 64,
// 170 after 512).  With fewer roots than helpers they open at once: 100 us
// against 225 on four roots of 2 000 picks; with more that costs (1 080 roots,
// 15 000 picks: 101 us against 73).
constexpr int kClqShareAfter = 512;
// only the waves of the first blocks help once the roots are gone; the rest
// leave, as their slots may serve other work
constexpr int kClqHelperBlocks = 64;
constexpr int kClqMaskWords = kClqMaxWaves / 64;  // bit t: slot t has an open root
constexpr int kClqTake = 8;  // children handed out per take (one atomic)

struct ClqHdr {
  alignas(128) long long best;    // smallest key with a clique
  alignas(128) long long next;    // roots handed out beyond the waves' first ones
  alignas(128) int active;        // waves started and still taking roots
  alignas(128) long long nodes;   // picks extended
  long long last;                 // 1 + the largest pair that was a root
  unsigned ticket, done;          // blocks that have ended (k_clique_alive, k_clique_search)
  long long pairs;                // live, connected (class 0, class 1) pairs
  long long live0;                // live vertices of class 0
  int bad_colour, bad_layout;
  int coff[kBatchK + 1], soff[kBatchK + 1];
};

// What the host gets.
struct ClqOut {
  long long best, nodes, last, live0;
  int s0, s1;  // vertices of classes 0 and 1 (1 when k = 1)
  int bad_colour, bad_layout;
};

// Layout from the sorted colours (one workgroup): class starts by binary
// search, segment offsets, and the checks (colours in range, sorted, row
// words = sum of the class segments).
__global__ void __launch_bounds__(256) k_clique_setup(const int32_t *__restrict__ colour, int n, int k, int R,
                                                      ClqHdr *h, long long *__restrict__ share,
                                                      long long *__restrict__ found_root,
                                                      unsigned long long *__restrict__ omask) {
  const int tid = threadIdx.x;
  for (int t = tid; t < kClqMaxWaves; t += blockDim.x) {
    share[t] = kClqClosed;
    found_root[t] = kClqNone;
  }
  if (tid < kClqMaskWords) omask[tid] = 0ull;
  if (tid == 0) {
    h->best = kClqNone;
    h->next = 0;
    h->nodes = 0;
    h->active = 0;
    h->last = 0;
    h->ticket = 0;
    h->done = 0;
    h->pairs = 0;
    h->live0 = 0;
    h->bad_colour = 0;
    h->bad_layout = 0;
  }
  __syncthreads();
  for (int v = tid; v < n; v += blockDim.x) {
    const int c = colour[v];
    if (c < 0 || c >= k) h->bad_colour = 1;
    else if (v > 0 && colour[v - 1] > c) h->bad_layout = 1;
  }
  __syncthreads();
  if (h->bad_colour || h->bad_layout) return;
  for (int c = tid; c <= k; c += blockDim.x) {
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (colour[mid] < c) lo = mid + 1;
      else hi = mid;
    }
    h->coff[c] = lo;
  }
  __syncthreads();
  if (tid == 0) {
    int w = 0;
    for (int c = 0; c < k; ++c) {
      h->soff[c] = w;
      w += (h->coff[c + 1] - h->coff[c] + 63) / 64;
    }
    h->soff[k] = w;
    if (w != R) h->bad_layout = 1;
  }
}

// The live mask in the rows' layout (bit j of word w of class c is vertex
// coff[c] + 64 (w - soff[c]) + j), a wave per word, and the live neighbours in
// class 1 of each live vertex of class 0, a wave per vertex (k = 1: 1 for a
// live vertex).  The last block to end sums these up: pre[i] = roots of the
// vertices of class 0 before the i-th.
__global__ void __launch_bounds__(256) k_clique_alive(const uint64_t *__restrict__ rows,
                                                      const uint8_t *__restrict__ vmask, int k, int R, ClqHdr *h,
                                                      uint64_t *__restrict__ am, long long *__restrict__ pre) {
  __shared__ unsigned mine;
  __shared__ long long part[4];
  __shared__ int live[4];
  if (h->bad_colour || h->bad_layout) return;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int c1 = h->coff[1], s0 = c1, s1 = k > 1 ? h->coff[2] - c1 : 0, w1 = (s1 + 63) / 64;
  for (int i = blockIdx.x * 4 + wid; i < R + s0; i += gridDim.x * 4) {
    if (i < R) {
      int c = 0;
      while (c + 1 < k && h->soff[c + 1] <= i) ++c;
      const int v = h->coff[c] + 64 * (i - h->soff[c]) + lane;
      const unsigned long long x = __ballot(v < h->coff[c + 1] && (!vmask || vmask[v]));
      if (lane == 0) am[i] = x;
    } else {
      const int v = i - R;
      long long cnt = vmask && !vmask[v] ? -1 : k > 1 ? 0 : 1;
      if (cnt == 0) {
        const uint64_t *r1 = rows + (long long)v * R + h->soff[1];
        for (int w = 0; w < w1; ++w) {
          const int u = 64 * w + lane;
          cnt += __popcll(r1[w] & __ballot(u < s1 && (!vmask || vmask[c1 + u])));
        }
      }
      if (lane == 0) pre[v] = cnt;
    }
  }
  // every wave's stores have landed before the one release below: the barrier
  // does not wait for them, and the release waits for its own wave's only
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();  // by one thread: a release writes the whole L2 back
    mine = atomicAdd(&h->ticket, 1u);
  }
  __syncthreads();
  if (mine != gridDim.x - 1) return;
  __threadfence();
  // counts of the waves' quarters, then their prefix sums
  const int q = (s0 + 3) / 4, lo = min(s0, wid * q), hi = min(s0, lo + q);
  // kAt loads in flight (100 000 vertices of class 0, one load after the other:
  // 0.47 ms a call, 0.33 with these)
  constexpr int kAt = 16;
  long long x[kAt];
  auto load = [&](int i0) {
#pragma unroll
    for (int j = 0; j < kAt; ++j) {
      const int i = i0 + j * kWave + lane;
      x[j] = i < hi ? pre[i] : -1ll;
    }
  };
  long long sum = 0;
  int n0 = 0;
  for (int i0 = lo; i0 < hi; i0 += kAt * kWave) {
    load(i0);
#pragma unroll
    for (int j = 0; j < kAt; ++j) {
      sum += max(x[j], 0ll);
      n0 += x[j] >= 0;
    }
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
  n0 = wave_sum(n0);
  if (lane == 0) {
    part[wid] = sum;
    live[wid] = n0;
  }
  __syncthreads();
  long long run = 0;
  for (int i = 0; i < wid; ++i) run += part[i];
  for (int i0 = lo; i0 < hi; i0 += kAt * kWave) {
    load(i0);
#pragma unroll
    for (int j = 0; j < kAt; ++j) {
      const int i = i0 + j * kWave + lane, y = (int)max(x[j], 0ll);  // below 2^21: 64 of them fit an int
      const int s = wave_scan(y);
      if (i < hi) pre[i] = run + s - y;
      run += __builtin_amdgcn_readlane(s, kWave - 1);
    }
  }
  if (threadIdx.x == 0) {
    bool empty = false;  // a class with no vertex: no clique, no root
    for (int c = 0; c < k; ++c) empty |= h->coff[c + 1] == h->coff[c];
    h->pairs = empty ? 0 : part[0] + part[1] + part[2] + part[3];
    h->live0 = live[0] + live[1] + live[2] + live[3];
  }
}

// The smallest key with a clique so far, the same in every lane (lane 0's
// read, broadcast): the wave's control flow must not split on it.
__device__ __forceinline__ long long best_now(const ClqHdr *h) {
  const long long b = __hip_atomic_load(&h->best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __shfl(b, 0, kWave);
}

// Takes the next kClqTake children of the root on a share word: (root, j),
// the first of them, or false when the word is closed or its children are
// all taken.  The add's old value decides, never an earlier read: an add
// that lands after the owner moved on to a new root takes that root's
// children; one past the last child only raises j further (at most one add
// per wave, far below the root bits).
__device__ __forceinline__ bool take_child(long long *share, long long S2, long long &r, int &j) {
  long long old = 0;
  if ((threadIdx.x & 63) == 0)
    old = __hip_atomic_fetch_add(share, (long long)kClqTake, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  old = __shfl(old, 0, kWave);
  if (old < 0 || (old & kClqSubMask) >= S2) return false;
  r = old >> kClqSubBits;
  j = (int)(old & kClqSubMask);
  return true;
}

// Writes a node's common neighbourhood over the words [lo, hi) of the classes
// from c0 on to out[0 .. hi - lo) (x(w) gives word w) and tells whether every one
// of those classes keeps a candidate.  The words load together, lanes over
// words; lane l then watches class c0 + l: whether the ballot of non-zero
// words has a bit in its word range.
template <typename F>
__device__ __forceinline__ bool extend_all(const int *soff, int c0, int k, int lane, uint64_t *out, F x) {
  const int lo = soff[c0], hi = soff[k];
  const int c = c0 + lane;
  const bool mine = c < k;
  const int cl = mine ? soff[c] : 0, ch = mine ? soff[c + 1] : 0;
  bool seen = false;
  for (int w0 = lo; w0 < hi; w0 += kWave) {
    const int w = w0 + lane;
    uint64_t v = 0;
    if (w < hi) {
      v = x(w);
      out[w - lo] = v;
    }
    const unsigned long long nz = __ballot(v != 0ull);
    if (mine && !seen && cl < w0 + kWave && ch > w0) {
      const int a = max(cl, w0) - w0, b = min(ch, w0 + kWave) - w0;
      const unsigned long long m = (b - a == 64 ? ~0ull : ((1ull << (b - a)) - 1)) << a;
      seen = (nz & m) != 0ull;
    }
  }
  return __ballot(mine && !seen) == 0ull;
}

// The search.  stack: kClqMaxWaves slots of k * R words; share: a word per
// slot; omask: the open-slot bit mask; found: per slot the key (int64) and
// the k picks.
// LDS: the lists live in LDS when they fit kClqLdsWords per wave with room for
// a node a level (then as many as fit, up to kClqRoom), else in the workspace
// with one.
template <bool LDS>
__global__ void __launch_bounds__(kClqWaves * 64) k_clique_search(const uint64_t *__restrict__ rows, int k, int R,
                                                                  const uint64_t *__restrict__ am,
                                                                  const long long *__restrict__ pre, ClqHdr *h,
                                                                  uint64_t *__restrict__ stack,
                                                                  long long *__restrict__ share,
                                                                  unsigned long long *__restrict__ omask,
                                                                  long long *__restrict__ found_root,
                                                                  int *__restrict__ found_pick,
                                                                  int32_t *__restrict__ clique, ClqOut *host) {
  __shared__ uint64_t lstack[LDS ? kClqWaves * kClqLdsWords : 1];
  __shared__ int pick_s[kClqWaves][kWave];  // the picks of the list at hand: node << kClqSubBits | class's vertex
  __shared__ int path_s[LDS ? 1 : kClqWaves][LDS ? 1 : kBatchK];
  __shared__ int coff_s[kBatchK + 1], soff_s[kBatchK + 1], loff_s[kBatchK + 1];
  __shared__ unsigned long long wg_nodes;
  __shared__ long long wg_last;
  __shared__ int wg_roots, wg_found, room_s;
  __shared__ unsigned ticket;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int slot = blockIdx.x * kClqWaves + wid;
  if (h->bad_colour || h->bad_layout) {
    if (blockIdx.x == 0) {
      if (threadIdx.x < k) clique[threadIdx.x] = -1;
      if (threadIdx.x == 0) *host = ClqOut{kClqNone, 0, 0, 0, 0, 0, h->bad_colour, h->bad_layout};
    }
    return;
  }
  for (int c = threadIdx.x; c <= k; c += blockDim.x) {
    coff_s[c] = h->coff[c];
    soff_s[c] = h->soff[c];
  }
  if (threadIdx.x == 0) {
    wg_nodes = 0;
    wg_last = 0;
    wg_roots = kClqWaves;
    wg_found = 0;
    atomicAdd(&h->active, kClqWaves);
  }
  __syncthreads();
  const int *coff = coff_s, *soff = soff_s;
  // a level's list: its nodes' words, and in LDS their paths (parent and pick)
  if (threadIdx.x == 0) {
    int o = k > 2 ? R - soff[2] : 0, per = 0;
    for (int d = 3; d < k; ++d) per += R - soff[d] + 1;
    const int room = LDS && per ? max(1, min(kClqRoom, (kClqLdsWords - o) / per)) : 1;
    for (int d = 2; d < k; ++d) {
      loff_s[d] = d == 2 ? 0 : LDS ? o : d * R;
      if (d > 2) o += room * (R - soff[d]) + (room + 1) / 2;
    }
    room_s = room;
  }
  __syncthreads();
  const int room = room_s;
  const int *loff = loff_s;
  uint64_t *cn = LDS ? lstack + wid * kClqLdsWords : stack + (long long)slot * k * R;
  int *pick = pick_s[wid];
  const int s0 = coff[1] - coff[0];
  const int s1 = k > 1 ? coff[2] - coff[1] : 1;
  const long long pairs = h->pairs;
  // children per root: the class-2 vertices (one pseudo-child below k = 3)
  const long long S2 = k > 2 ? max(coff[3] - coff[2], 1) : 1;
  // the ends of the classes over the last 64 words (bit 63: the last word)
  const unsigned long long ends = [&]() {
    bool e = false;
    const int w = R - kWave + lane;
    for (int c = 1; c <= k; ++c) e |= soff[c] == w + 1;
    return __ballot(e);
  }();
  long long nodes = 0;
  int v0 = -1, v1 = -1;  // the root at hand

  // the lists' words are written by one lane and read by others: in global
  // memory the wave waits for its writes before it reads them back
  auto written = [&]() {
    if constexpr (LDS) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  };
  auto paths = [&](int d) -> int * {
    if constexpr (LDS) return (int *)(cn + loff[d] + room * (R - soff[d]));
    else return path_s[wid] + d;
  };

  // The list at level d (lane d's `num` nodes): from position lane d's `at`
  // (64 * word of the list's class-d words + bit) up to 64 of its picks are
  // tried and the ones that stay put on level d + 1's list, up to `cap`;
  // class-2 vertices stop at `jend`.  False: none were left to try.
  int num = 0, at = 0;
  auto expand = [&](int d, int cap, int jend) -> bool {
    const int m = __builtin_amdgcn_readlane(num, d), p0 = __builtin_amdgcn_readlane(at, d);
    const int cw = soff[d + 1] - soff[d], rw = R - soff[d], nw = R - soff[d + 1];
    const uint64_t *from = cn + loff[d];
    uint64_t *to = cn + loff[d + 1];
    int *path = paths(d + 1);
    int f0 = p0 >> 6, cut = p0 & 63, have;
    for (;;) {  // 64 words of the list
      const int f = f0 + lane, node = f / cw, w = f - node * cw;
      uint64_t x = node < m ? from[node * rw + w] : 0ull;
      if (lane == 0) x &= ~0ull << cut;
      if (d == 2) {
        const int left = jend - 64 * w;
        x &= left >= 64 ? ~0ull : left <= 0 ? 0ull : (1ull << left) - 1;
      }
      const int c = __popcll(x);
      int p = wave_scan(c);
      have = min(__builtin_amdgcn_readlane(p, kWave - 1), kWave);
      if (have) {
        for (p -= c; x && p < kWave; ++p) {
          pick[p] = node << kClqSubBits | (64 * w + __builtin_ctzll(x));
          x &= x - 1;
        }
        break;
      }
      f0 += kWave;
      cut = 0;
      if (f0 >= m * cw) return false;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int got = 0, tried = have;
    if (nw <= kWave) {
      // lanes over (pick, word), `per` picks a step
      const int per = kWave / nw, g = lane / nw, w = lane - g * nw;
      const bool in = g < per;
      const bool end = in && ((ends >> (kWave - nw + w)) & 1ull);
      const unsigned long long E = __ballot(end), M = __ballot(in && !end);
      const unsigned long long below = (1ull << (in ? g * nw : 0)) - 1;
      const unsigned long long own = E & ~below & (nw * (g + 1) >= 64 ? ~0ull : (1ull << (nw * (g + 1))) - 1);
      const int base = coff[d], skip = soff[d + 1], off = skip - soff[d] + w;
      for (int t0 = 0; t0 < have && got < cap; t0 += 4 * per) {
        uint64_t x[4];
        int e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * per + g;
          x[u] = 0ull;
          e[u] = 0;
          if (in && t < have) {
            e[u] = pick[t];
            x[u] = rows[(long long)(base + (e[u] & (int)kClqSubMask)) * R + skip + w];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * per;
          if (t < have && got < cap) {
            if (in && t + g < have) x[u] &= from[(e[u] >> kClqSubBits) * rw + off];
            else x[u] = 0ull;
            // a class keeps a candidate: a non-zero word at its end, or a
            // carry into its end from the words before it
            const unsigned long long nz = __ballot(x[u] != 0ull);
            const unsigned long long full = nz | ((nz & M) + M);
            const bool ok = in && (own & ~full) == 0ull;
            const unsigned long long lead = __ballot(ok && w == 0);
            const int rank = __popcll(lead & below), room_left = cap - got, n = __popcll(lead);
            if (ok && rank < room_left) {
              to[(got + rank) * nw + w] = x[u];
              if (w == 0) path[got + rank] = e[u];
            }
            if (n > room_left) {  // the first without room is tried again
              const unsigned long long first = __ballot(ok && w == 0 && rank == room_left);
              tried = t + __builtin_amdgcn_readlane(g, __builtin_ctzll(first));
            } else if (n == room_left) {
              tried = min(have, t + per);
            }
            got += min(n, room_left);
          }
        }
      }
    } else {
      // rows wider than a wave: a pick at a time
      for (int t = 0; t < have; ++t) {
        const int e = __builtin_amdgcn_readfirstlane(pick[t]);
        const uint64_t *rv = rows + (long long)(coff[d] + (e & (int)kClqSubMask)) * R;
        const uint64_t *cd = from + (e >> kClqSubBits) * rw - soff[d];
        const bool ok = extend_all(soff, d + 1, k, lane, to + got * nw,
                                   [&](int w) { return cd[w] & rv[w]; });
        if (ok) {
          if (lane == 0) path[got] = e;
          if (++got == cap) {
            tried = t + 1;
            break;
          }
        }
      }
    }
    written();
    nodes += tried;
    const int e = __builtin_amdgcn_readfirstlane(pick[tried - 1]);
    const int next = (e >> kClqSubBits) * cw * 64 + (e & (int)kClqSubMask) + 1;
    if (lane == d) at = next;
    if (lane == d + 1) {
      at = 0;
      num = got;
    }
    return true;
  };

  // The first candidate at or after local index `j` of a class whose words in
  // a node's list entry are w[0 .. cw), or -1.
  auto first_at = [&](const uint64_t *wd, int cw, int j) -> int {
    for (int w0 = j >> 6; w0 < cw; w0 += kWave) {
      const int w = w0 + lane;
      uint64_t x = w < cw ? wd[w] : 0ull;
      if (w == (j >> 6)) x &= ~0ull << (j & 63);
      const unsigned long long b = __ballot(x != 0ull);
      if (b) {
        const int f = __builtin_ctzll(b);
        const unsigned lo = __builtin_amdgcn_readlane((unsigned)x, f), hi = __builtin_amdgcn_readlane((unsigned)(x >> 32), f);
        return 64 * (w0 + f) + (lo ? __builtin_ctz(lo) : 32 + __builtin_ctz(hi));
      }
    }
    return -1;
  };

  // Writes the clique: the picks of classes 0 and 1, those on the path to the
  // first node of the last level's list, and its candidate of the last class.
  auto record = [&](long long r, int last) {
    if (lane == 0) {
      int *out = found_pick + (long long)slot * k;
      int j = 0;
      out[0] = v0;
      if (k > 1) out[1] = v1;
      if (k > 2) {
        out[k - 1] = coff[k - 1] + last;
        j = last;
        for (int d = k - 1, node = 0; d > 2; --d) {
          const int e = paths(d)[node];
          j = e & (int)kClqSubMask;
          out[d - 1] = coff[d - 1] + j;
          node = e >> kClqSubBits;
        }
      }
      const long long key = r * S2 + j;
      found_root[slot] = key;
      __threadfence();
      atomicMin((long long *)&h->best, key);
      __threadfence();
      wg_found = 1;
    }
  };

  // The children j0 .. jend - 1 of root r (its node is the list at level 2):
  // true at the first clique, then recorded; false when there is none or a
  // smaller key already has one.  own: the root is this wave's and not shared
  // yet; then it may return false with j0 set to the first child left to share
  // (below jend), once it has cost enough.
  auto search = [&](long long r, int &j0, int jend, bool own, bool at_once) -> bool {
    int d = 2, steps = 0, left = at_once ? 0 : kClqShareAfter;
    long long low = r * S2 + j0;  // no clique to come has a smaller key
    if (lane == 2) {
      num = 1;
      at = j0;
    }
    for (;;) {
      if (d == k - 1) {
        const int cw = soff[k] - soff[d];
        const int j = first_at(cn + loff[d], cw, d == 2 ? j0 : 0);
        if (d == 2 && (j < 0 || j >= jend)) {
          j0 = jend;
          return false;
        }
        ++nodes;
        record(r, j);
        return true;
      }
      if ((++steps & 3) == 0 && best_now(h) < low) {
        j0 = jend;
        return false;
      }
      if (d == 2) {
        j0 = __builtin_amdgcn_readlane(at, 2);
        low = r * S2 + j0;
        if (own && left <= 0 && j0 < jend) return false;
      }
      const long long before = nodes;
      if (!expand(d, room, jend)) {
        if (d == 2) {
          j0 = jend;
          return false;
        }
        --d;
        continue;
      }
      left -= (int)(nodes - before);
      if (__builtin_amdgcn_readlane(num, d + 1)) ++d;
    }
  };

  // The common neighbourhood of the pair (v0, v1) over classes 2..k-1, the one
  // node of level 2: false when a class is left without a candidate (k >= 3).
  auto open_root = [&]() -> bool {
    const uint64_t *r0 = rows + (long long)v0 * R, *r1 = rows + (long long)v1 * R;
    const bool ok = extend_all(soff, 2, k, lane, cn, [&](int w) { return r0[w] & r1[w] & am[w]; });
    written();
    return ok;
  };

  bool done = false;
  // own roots: this wave's number, then in the order of the counter
  long long last = 0;
  for (long long u = slot; u < pairs;) {
    // the class-0 vertex: the last one with pre <= u, 64 at a time
    int i0 = 0;
    for (int len = s0; len > 1;) {
      const int step = (len + kWave - 1) / kWave, i = lane * step;
      const unsigned long long b = __ballot(i < len && pre[i0 + i] <= u);
      const int f = 63 - __builtin_clzll(b);
      i0 += f * step;
      len = min(step, len - f * step);
    }
    v0 = coff[0] + i0;
    v1 = -1;
    long long r = i0;
    if (k > 1) {
      // and its live neighbour in class 1 of that rank
      const uint64_t *r0 = rows + (long long)v0 * R;
      int rank = (int)(u - pre[i0]);
      for (int w0 = soff[1]; w0 < soff[2]; w0 += kWave) {
        const int w = w0 + lane;
        uint64_t x = w < soff[2] ? r0[w] & am[w] : 0ull;
        const int c = __popcll(x), p = wave_scan(c), all = __builtin_amdgcn_readlane(p, kWave - 1);
        if (rank < all) {
          const unsigned long long b = __ballot(p - c <= rank && rank < p);
          for (int t = rank - (p - c); t > 0 && x; --t) x &= x - 1;
          const int l1 = 64 * (w - soff[1]) + (x ? __builtin_ctzll(x) : 0);
          v1 = coff[1] + __builtin_amdgcn_readlane(l1, __builtin_ctzll(b));
          break;
        }
        rank -= all;
      }
      r = (long long)i0 * s1 + (v1 - coff[1]);
    }
    last = r + 1;
    if (r * S2 > best_now(h)) break;
    ++nodes;
    if (k <= 2) {
      record(r, 0);
      done = true;
      break;
    }
    if (open_root()) {
      int j = 0;
      done = search(r, j, (int)S2, true, pairs < kClqHelperBlocks * kClqWaves);
      if (!done && j < S2) {
        // the rest opened to every wave and taken as any helper takes it
        if (lane == 0) {
          __hip_atomic_store(&share[slot], (r << kClqSubBits) | j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicOr(&omask[slot >> 6], 1ull << (slot & 63));
        }
        long long rr;
        int j0;
        while (!done && take_child(&share[slot], S2, rr, j0) && rr * S2 + j0 <= best_now(h))
          done = search(rr, j0, (int)min((long long)j0 + kClqTake, S2), false, false);
        if (lane == 0) {
          atomicAnd(&omask[slot >> 6], ~(1ull << (slot & 63)));
          __hip_atomic_store(&share[slot], kClqClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      if (done) break;
    }
    if (lane == 0) u = kClqMaxWaves + (long long)atomicAdd((unsigned long long *)&h->next, 1ull);
    u = __shfl(u, 0, kWave);
  }
  if (lane == 0) {
    atomicMax(&wg_last, last);
    if (atomicAdd(&wg_roots, -1) == 1) atomicAdd(&h->active, -kClqWaves);
  }

  // out of roots: the waves of the first kClqHelperBlocks blocks help with
  // the open children, the smallest key first.  With none open, sleep and
  // look again, until no started wave is taking roots any more or
  // kClqIdlePolls looks in a row found nothing (waves not yet started are
  // not waited for: they find the roots gone and help, or leave, in turn).
  long long have = -1;  // the root whose pair neighbourhood is on the stack
  int polls = 0;
  while (!done && k > 2 && blockIdx.x < kClqHelperBlocks) {
    long long bestkey = kClqNone;
    int bslot = -1;
    {
      // lane l reads word l of the open-slot mask, then the share words of
      // its set bits
      unsigned long long bits =
          lane < kClqMaskWords ? __hip_atomic_load(&omask[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
      while (bits) {
        const int t = 64 * lane + __builtin_ctzll(bits);
        bits &= bits - 1;
        const long long v = __hip_atomic_load(&share[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const long long key =
            v >= 0 && (v & kClqSubMask) < S2 ? (v >> kClqSubBits) * S2 + (v & kClqSubMask) : kClqNone;
        if (key < bestkey) {
          bestkey = key;
          bslot = t;
        }
      }
      for (int off = 32; off > 0; off >>= 1) {
        const long long ok = __shfl_xor(bestkey, off, kWave);
        const int os = __shfl_xor(bslot, off, kWave);
        if (ok < bestkey || (ok == bestkey && os < bslot)) {
          bestkey = ok;
          bslot = os;
        }
      }
    }
    if (bestkey != kClqNone && bestkey <= best_now(h)) {
      polls = 0;  // look again at once after this child
      long long r;
      int j0;
      if (!take_child(&share[bslot], S2, r, j0)) continue;  // taken meanwhile
      if (r * S2 + j0 > best_now(h)) continue;
      if (r != have) {
        v0 = coff[0] + (int)(r / s1);
        v1 = coff[1] + (int)(r % s1);
        open_root();  // true: the owner opened it
        have = r;
      }
      done = search(r, j0, (int)min((long long)j0 + kClqTake, S2), false, false);
      continue;
    }
    if (polls >= kClqIdlePolls ||
        __shfl(__hip_atomic_load(&h->active, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), 0, kWave) == 0)
      break;
    __builtin_amdgcn_s_sleep(127);
    ++polls;
  }
  if (lane == 0) atomicAdd(&wg_nodes, (unsigned long long)nodes);
  // the last block to end copies the picks of the smallest key's slot to the
  // output (all -1 when there is no clique)
  __syncthreads();
  if (threadIdx.x == 0) {
    if (wg_nodes) atomicAdd((unsigned long long *)&h->nodes, wg_nodes);
    if (wg_last) atomicMax(&h->last, wg_last);
    if (wg_found) __threadfence();
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the sums above come before the ticket
    ticket = atomicAdd(&h->done, 1u);
  }
  __syncthreads();
  if (ticket != gridDim.x - 1) return;
  __threadfence();
  const long long best = __hip_atomic_load(&h->best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x == 0)
    *host = ClqOut{best, __hip_atomic_load(&h->nodes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                   __hip_atomic_load(&h->last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), h->live0, s0, s1, 0, 0};
  if (best == kClqNone) {
    for (int c = threadIdx.x; c < k; c += blockDim.x) clique[c] = -1;
    return;
  }
  for (int t = threadIdx.x; t < kClqMaxWaves; t += blockDim.x)
    if (found_root[t] == best)
      for (int c = 0; c < k; ++c) clique[c] = found_pick[(long long)t * k + c];
}

struct ClqWs {
  size_t hdr, am, pre, stack, share, omask, root, pick, total;
};

ClqWs clique_ws(int n, int k, int R) {
  ClqWs z{};
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t at = o;
    o += (b + 255) / 256 * 256;
    return at;
  };
  z.hdr = take(sizeof(ClqHdr));
  z.am = take(sizeof(uint64_t) * (size_t)(R > 0 ? R : 1));
  z.pre = take(sizeof(long long) * (size_t)(n > 0 ? n : 1));
  z.stack = take(sizeof(uint64_t) * (size_t)kClqMaxWaves * (size_t)k * (size_t)R);
  z.share = take(sizeof(long long) * kClqMaxWaves);
  z.omask = take(sizeof(uint64_t) * kClqMaskWords);
  z.root = take(sizeof(long long) * kClqMaxWaves);
  z.pick = take(sizeof(int) * (size_t)kClqMaxWaves * (size_t)k);
  z.total = o;
  return z;
}

}  // namespace
}  // namespace kzi

extern "C" {

int kz_clique_workspace_bytes(const kz_graph *g, int32_t k, size_t *bytes) {
  if (!g || !bytes || g->format != KZ_BITSET_U64 || k < 1 || k > kzi::kBatchK || g->n < 0 || g->row_words < 0)
    return KZ_EINVAL;
  *bytes = kzi::clique_ws(g->n, k, g->row_words).total;
  return KZ_OK;
}

int kz_find_clique(kz_ctx *ctx, const kz_graph *g, const int32_t *colour, int32_t k, const uint8_t *vmask, void *ws,
                   size_t ws_bytes, int32_t *clique, void *stream, kz_clique_result *res) {
  using namespace kzi;
  kz_clique_result r{};
  auto done = [&](int st) {
    r.status = st;
    if (res) *res = r;
    return st;
  };
  if (!ctx || !g || g->format != KZ_BITSET_U64 || k < 1 || g->n < 0 || g->row_words < 0) return done(KZ_EINVAL);
  if (k > kBatchK || g->n >= kClqMaxN) return done(KZ_ETOOLARGE);
  const int n = g->n, R = g->row_words;
  if (n > 0 && (!g->rows || !colour || !clique || !ws || (uintptr_t)ws % 256)) return done(KZ_EINVAL);
  if (n == 0) {  // no vertex: no clique
    if (clique && hipMemsetAsync(clique, 0xff, sizeof(int32_t) * (size_t)k, (hipStream_t)stream) != hipSuccess)
      return done(KZ_EHIP);
    return done(KZ_OK);
  }
  const ClqWs z = clique_ws(n, k, R);
  if (ws_bytes < z.total) return done(KZ_EWORKSPACE);
  if (hipSetDevice(ctx->device) != hipSuccess) return done(KZ_EHIP);
  hipStream_t s = (hipStream_t)stream;
  char *base = (char *)ws;
  ClqHdr *h = (ClqHdr *)(base + z.hdr);
  uint64_t *am = (uint64_t *)(base + z.am);
  long long *pre = (long long *)(base + z.pre);
  uint64_t *stack = (uint64_t *)(base + z.stack);
  long long *share = (long long *)(base + z.share);
  unsigned long long *omask = (unsigned long long *)(base + z.omask);
  long long *froot = (long long *)(base + z.root);
  int *fpick = (int *)(base + z.pick);
  hipLaunchKernelGGL(k_clique_setup, dim3(1), dim3(256), 0, s, colour, n, k, R, h, share, froot, omask);
  // 512 workgroups at most: each ends with a release, which writes its XCD's L2 back
  hipLaunchKernelGGL(k_clique_alive, dim3((unsigned)std::min((R + 2 * (n / k)) / 4 + 1, 512)), dim3(256), 0, s,
                     g->rows, vmask, k, R, h, am, pre);
  // A node of every level fits LDS: level d has at most R - d words left, as
  // every class before it has one (an empty class ends the search).
  long long words = std::max(R - 2, 0);
  for (int d = 3; d < k; ++d) words += std::max(R - d, 0) + 1;
  const dim3 grid(kClqMaxWaves / kClqWaves), block(kClqWaves * 64);
  if (words <= kClqLdsWords)
    hipLaunchKernelGGL(k_clique_search<true>, grid, block, 0, s, g->rows, k, R, am, pre, h, stack, share,
                       omask, froot, fpick, clique, (ClqOut *)ctx->pinned_dev);
  else
    hipLaunchKernelGGL(k_clique_search<false>, grid, block, 0, s, g->rows, k, R, am, pre, h, stack, share, omask,
                       froot, fpick, clique, (ClqOut *)ctx->pinned_dev);
  const ClqOut *hh = (const ClqOut *)ctx->pinned;
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return done(KZ_EHIP);
  if (hh->bad_colour) return done(KZ_ECOLOUR);
  if (hh->bad_layout) return done(KZ_EINVAL);
  r.found = hh->best != kClqNone;
  r.nodes = hh->nodes;
  const long long nroots = (long long)hh->s0 * hh->s1;
  r.roots = r.found ? hh->last : nroots;
  // the first picks: a live class-0 vertex for every pair up to there
  if (k > 1) r.nodes += std::min<long long>(r.roots, hh->live0 * hh->s1);
  return done(KZ_OK);
}

}  // extern "C"
