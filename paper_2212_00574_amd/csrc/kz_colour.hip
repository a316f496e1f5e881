// Upstream legal colouring (gfx950): Jones and Plassmann's parallel greedy
// colouring (SIAM J. Sci. Comput. 14(3), 1993) of a graph given as plain bit
// rows, for inputs that arrive without the legal colouring the colour-index
// method of section 4.2 needs.
//
// Every vertex v has the key (priority[v], v), compared lexicographically.
// A round takes every uncoloured vertex whose key beats the key of each of
// its uncoloured neighbours; each vertex taken gets the smallest colour that
// no neighbour coloured in an earlier round holds.
//
// The neighbours coloured before v are exactly those with larger keys (one
// with a smaller key waits for v), so the colours are those of the greedy
// colouring in order of falling keys, and v's round is one more than the
// largest round of a neighbour with a larger key.  That is what runs here:
// the vertices are ranked by their keys, and one workgroup goes through them
// 64 at a time.  A round as two dependent launches took about 11 us, and a
// graph has over a thousand rounds.
//
// While wave 0 resolves a block (its 64 vertices one after the other, lane j
// holding vertex j's smallest free colour, each colour given reaching the
// lanes next to it), the other waves gather for the next block what its rows
// see of the blocks before: a bitmap of the colours in use and the largest
// round; the block resolved meanwhile is merged in between two barriers.
//
// The rounds themselves, two kernels each, are the other way: one wave per
// vertex tests row & U (U: the uncoloured vertices; only they can beat it),
// then one wave per taken vertex marks the colours of row & ~U in an LDS bitmap
// and takes its lowest zero bit.  They win where the rounds are few: a random
// graph of average degree d has about 2 d of them (at 20000 vertices of degree
// 200 both ways take 7.2 to 7.6 ms, at degree 1000 38 ms and 9.9 ms), but the
// priorities may order a graph by its classes or its hubs (a complete bipartite
// graph of 20000 vertices, one side's priorities above the other's: 2 rounds in
// 1.6 ms, 46 ms by blocks).  So graphs of average degree below n / 100 run the
// rounds, and others the first few of them, from which rounds_left tells how many
// are to come (1.7 ms for that bipartite graph; 3000 vertices at p = 0.3, by blocks:
// 0.84 ms with and without).
#include <stddef.h>
#include <string.h>

#include <algorithm>

#include "kz.h"
#include "kz_internal.h"

namespace {

constexpr int kColWaves = 4;                // waves (vertices) per workgroup of the check
constexpr int kColMaxWords = 1024;          // row words (65536 vertices)
constexpr size_t kColAlign = 256;
constexpr int kColSlots = 32;               // spread of the degrees' sums
constexpr int kColFirstChunk = 8;           // rounds enqueued before the first look at the count
constexpr int kColMaxChunk = 128;           // ... and at most between two looks
constexpr int kColProbeN = 512;             // vertices from which the first rounds tell how many are to come
constexpr double kColProbe = 1.0 / 48;      // ... for this share of the blocks' time
constexpr double kColProbeHubs = 1.0 / 3;   // ... and while hubs are taken, for this one
constexpr int kColThreads = 1024;           // the greedy workgroup
constexpr int kColLdsWords = 32;            // words of a bitmap of colours kept in LDS (the rest in memory)
constexpr int kColLdsColours = 64 * kColLdsWords;
constexpr int kColLdsN = 16384;             // vertices up to which colours and rounds are kept in LDS
constexpr int kRankThreads = 256, kRankSpan = 256;  // vertices ranked, and compared with, by a workgroup

constexpr size_t kColHead = 256;            // bytes of the counters before the sums

struct ColCtr {
  int left;     // rounds: vertices not yet coloured; every round kernel returns at once at 0
  int bad;      // validation: a KZ_* status, most severe first (see k_col_check)
  int top;      // largest colour given
  int rounds;   // rounds
  unsigned long long gone;  // edges with an end coloured (rounds, where counted)
  char pad[kColHead - 24];
  // sums of the degrees and of their squares, over slots (col_slots) of a line
  // each: a graph's thousands of workgroups would queue at one.  They lie where
  // the greedy pass writes its order later (ColWs), so the workspace holds no more.
  struct alignas(64) {
    unsigned long long ends, squares;
  } sum[kColSlots];
};
static_assert(sizeof(ColCtr) <= kzi::kPinnedBytes, "read back into the context's pinned memory");
static_assert(offsetof(ColCtr, sum) == kColHead && kColHead % kColAlign == 0, "the sums take the order's place");

size_t col_up(size_t x) { return (x + kColAlign - 1) / kColAlign * kColAlign; }

// slots of the sums: as many as the order of n vertices has room for
int col_slots(int n) { return (int)std::min<size_t>(kColSlots, col_up(sizeof(int) * (size_t)n) / 64); }

// words of a bitmap of colours beyond those in LDS (a vertex's smallest free
// colour is at most n - 1)
int col_more(int n) { return n > kColLdsColours ? (n + 63) / 64 + 1 - kColLdsWords : 0; }

struct ColWs {
  size_t ctr, U, sel, rank, order, val, used, total;
};

ColWs col_ws(int n) {
  ColWs w{};
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t at = o;
    o += col_up(b);
    return at;
  };
  w.ctr = take(kColHead);
  w.order = take(sizeof(int) * (size_t)n);  // behind the counters: see ColCtr
  w.U = take(sizeof(uint64_t) * (size_t)((n + 63) / 64));
  w.sel = take((size_t)n);
  w.rank = take(sizeof(int) * (size_t)n);
  w.val = take(n > kColLdsN ? sizeof(unsigned) * (size_t)n : 0);
  w.used = take(2 * 64 * sizeof(uint64_t) * (size_t)col_more(n));
  w.total = o;
  return w;
}

__device__ __forceinline__ bool key_beats(unsigned long long pu, int u, unsigned long long pv, int v) {
  return pu > pv || (pu == pv && u > v);
}

// Validation and set-up, one wave per row: no bit at or beyond n
// (KZ_EINVAL), no self-loop (KZ_ESELFLOOP), symmetric (KZ_EASYM); the
// most severe found wins (EINVAL, then ESELFLOOP, then EASYM).  rank = 0,
// colour = -1, U = every vertex.
__global__ void __launch_bounds__(kColWaves * 64) k_col_check(int n, const uint64_t *__restrict__ rows, int R,
                                                              int *rank, int *colour, uint64_t *U, ColCtr *ctr,
                                                              int slots) {
  __shared__ unsigned long long ends, squares;
  if (threadIdx.x == 0) ends = squares = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int v = blockIdx.x * kColWaves + (threadIdx.x >> 6);
  const uint64_t *row = rows + (long long)v * R;
  int bad = 0, deg = 0;  // bad: 3 EINVAL, 2 ESELFLOOP, 1 EASYM
  for (int w = lane; v < n && w < R; w += 64) {
    unsigned long long x = row[w];
    const int lo = 64 * w;
    if (lo + 64 > n) {
      const unsigned long long past = lo >= n ? ~0ull : ~0ull << (n - lo);
      if (x & past) bad = max(bad, 3);
      x &= ~past;
    }
    deg += __popcll(x);
    while (x) {
      const int b = __builtin_ctzll(x);
      x &= x - 1;
      const int u = lo + b;
      if (u == v) bad = max(bad, 2);
      else if (!((rows[(long long)u * R + (v >> 6)] >> (v & 63)) & 1ull)) bad = max(bad, 1);
    }
  }
  for (int off = 32; off > 0; off >>= 1) bad = max(bad, __shfl_xor(bad, off, 64));
  deg = kzi::wave_sum(deg);
  if (lane == 0 && v < n) {
    rank[v] = 0;
    colour[v] = -1;
    if (bad) atomicMax(&ctr->bad, bad);
    if (v == 0) ctr->left = n;
    if ((v & 63) == 0) U[v >> 6] = n - v >= 64 ? ~0ull : (1ull << (n - v)) - 1;
    atomicAdd(&ends, (unsigned long long)deg);
    atomicAdd(&squares, (unsigned long long)deg * (unsigned long long)deg);
  }
  __syncthreads();
  if (threadIdx.x == 0 && ends) {
    auto &sum = ctr->sum[blockIdx.x % (unsigned)slots];
    atomicAdd(&sum.ends, ends);
    atomicAdd(&sum.squares, squares);
  }
}

// ---- the rounds themselves

// One round's choice, one wave per vertex: sel[v] = v is uncoloured and its
// key beats every uncoloured neighbour's.
__global__ void __launch_bounds__(kColWaves * 64) k_col_select(int n, const uint64_t *__restrict__ rows, int R,
                                                               const uint64_t *__restrict__ pri,
                                                               const uint64_t *__restrict__ U, uint8_t *sel,
                                                               ColCtr *ctr) {
  const int lane = threadIdx.x & 63;
  const int v = blockIdx.x * kColWaves + (threadIdx.x >> 6);
  if (ctr->left == 0 || ctr->bad) return;  // coloured in an earlier round of this chunk, or refused
  if (v == 0 && lane == 0) atomicAdd(&ctr->rounds, 1);
  if (v >= n) return;
  const bool unc = (U[v >> 6] >> (v & 63)) & 1ull;
  if (!unc) {
    if (lane == 0) sel[v] = 0;
    return;
  }
  const uint64_t *row = rows + (long long)v * R;
  const unsigned long long pv = pri[v];
  const int W = (n + 63) >> 6;
  bool beaten = false;
  for (int w0 = 0; w0 < W; w0 += 64) {
    const int w = w0 + lane;
    if (w < W) {
      unsigned long long x = row[w] & U[w];
      while (x && !beaten) {
        const int b = __builtin_ctzll(x);
        x &= x - 1;
        const int u = 64 * w + b;
        beaten = key_beats(pri[u], u, pv, v);
      }
    }
    if (__ballot(beaten)) break;
  }
  const bool taken = __ballot(beaten) == 0ull;
  if (lane == 0) sel[v] = taken ? 1 : 0;
}

// One round's colours, one wave per vertex taken: the smallest colour that
// no neighbour coloured earlier holds; then v leaves U.  `count`: its edges to the
// uncoloured are added to ctr->gone (none of those neighbours is taken in this
// round, so an edge counts once).
__global__ void __launch_bounds__(kColWaves * 64) k_col_colour(int n, const uint64_t *__restrict__ rows, int R,
                                                               const uint8_t *__restrict__ sel, uint64_t *U,
                                                               int *colour, ColCtr *ctr, int count) {
  __shared__ unsigned long long used[kColWaves][kColMaxWords];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int v = blockIdx.x * kColWaves + wid;
  // left is 0 here only if it was 0 when this round's select kernel read it
  // (that kernel then returned at once and sel is a previous round's): a
  // vertex taken in this round keeps it positive until its own wave below
  // has coloured it
  if (v >= n || ctr->left == 0 || ctr->bad || !sel[v]) return;
  const int W = (n + 63) >> 6;
  int ends = 0;
  unsigned long long *mine = used[wid];
  for (int w = lane; w < W; w += 64) mine[w] = 0ull;
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  const uint64_t *row = rows + (long long)v * R;
  for (int w = lane; w < W; w += 64) {
    const unsigned long long y = row[w], u = U[w];
    ends += __popcll(y & u);
    unsigned long long x = y & ~u;  // neighbours coloured in earlier rounds
    while (x) {
      const int b = __builtin_ctzll(x);
      x &= x - 1;
      const int c = colour[64 * w + b];
      if (c >= 0 && c < 64 * W) atomicOr(&mine[c >> 6], 1ull << (c & 63));
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // the lowest zero bit: the first word with a zero, in lane order
  int c = -1;
  for (int w0 = 0; w0 < W && c < 0; w0 += 64) {
    const int w = w0 + lane;
    const unsigned long long free = w < W ? ~mine[w] : 0ull;
    const unsigned long long has = __ballot(free != 0ull);
    if (has) {
      const int first = __builtin_ctzll(has);
      const unsigned long long f = __shfl(free, first, 64);
      c = 64 * (w0 + first) + __builtin_ctzll(f);
    }
  }
  if (c < 0) c = 64 * W;  // every colour below 64*W held (cannot happen: v has fewer than n neighbours)
  if (count) {
    ends = kzi::wave_sum(ends);
    if (lane == 0 && ends) atomicAdd(&ctr->gone, (unsigned long long)ends);
  }
  if (lane == 0) {
    colour[v] = c;
    atomicMax(&ctr->top, c);
    atomicAnd(&U[v >> 6], ~(1ull << (v & 63)));
    atomicSub(&ctr->left, 1);
  }
}

// ---- the greedy colouring in key order

// rank[v] += the vertices of a span of kRankSpan whose keys beat v's.
__global__ void __launch_bounds__(kRankThreads) k_col_rank(int n, const uint64_t *__restrict__ pri, int *rank) {
  __shared__ uint64_t sp[kRankThreads];
  const int t = threadIdx.x, v = blockIdx.x * kRankThreads + t;
  const uint64_t pv = v < n ? pri[v] : 0;
  const int u1 = min(n, (int)(blockIdx.y + 1) * kRankSpan);
  int cnt = 0;
  for (int u0 = blockIdx.y * kRankSpan; u0 < u1; u0 += kRankThreads) {
    __syncthreads();
    sp[t] = u0 + t < u1 ? pri[u0 + t] : 0;
    __syncthreads();
    const int m = min(kRankThreads, u1 - u0);
    for (int i = 0; i < m; ++i) cnt += key_beats(sp[i], u0 + i, pv, v);
  }
  if (v < n && cnt) atomicAdd(&rank[v], cnt);
}

__global__ void __launch_bounds__(256) k_col_order(int n, const int *__restrict__ rank, int *__restrict__ order) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v < n) order[rank[v]] = v;
}

__device__ __forceinline__ int wave_max(int v) {
  unsigned x = (unsigned)v;
  x = max(x, kzi::dpp<kzi::kDppRor + 8>(x));
  x = max(x, kzi::dpp<kzi::kDppRor + 4>(x));
  x = max(x, kzi::dpp<kzi::kDppRor + 2>(x));
  x = max(x, kzi::dpp<kzi::kDppRor + 1>(x));
  return max(max(__builtin_amdgcn_readlane((int)x, 0), __builtin_amdgcn_readlane((int)x, 16)),
             max(__builtin_amdgcn_readlane((int)x, 32), __builtin_amdgcn_readlane((int)x, 48)));
}

// The greedy colouring in key order (one workgroup, see the top).  val[u]:
// vertex u's round less one (high half) and colour (low half), in LDS for
// VLDS, else in memory.  A gather marks the colours it meets in a byte each
// (its wave's flags) and packs them by ballots: as atomics on the bitmap 64
// lanes would meet in a few words.  Colours from kColLdsColours on go to
// bitmaps in memory (`more` words a row).  What bounds it is a block's
// chain: the gather of a wave's rows (an LDS read and a byte written per
// neighbour coloured) or the 64 steps of the resolve, then the merge.
template <bool VLDS>
__global__ void __launch_bounds__(kColThreads) k_col_greedy(int n, const uint64_t *__restrict__ rows, int R,
                                                            const int *__restrict__ order, unsigned *gval,
                                                            unsigned long long *gused, int more, int *colour,
                                                            ColCtr *ctr) {
  constexpr int kPitch = kColLdsWords + 1;  // odd: 64 lanes reading a column meet no bank conflict
  constexpr int kW = kColThreads / 64;
  __shared__ unsigned sval[VLDS ? kColLdsN : 1];
  __shared__ unsigned long long sused[2][64][kPitch];
  __shared__ unsigned sflag[kW][kColLdsColours / 4];    // a byte per colour
  __shared__ unsigned long long done[VLDS ? kColLdsN / 64 : kColMaxWords];  // vertices coloured
  __shared__ unsigned long long adj[2][64], cross[64];  // a block's edges inside, and to the block before
  __shared__ int most[2][64];                           // largest round seen, of a block's rows
  __shared__ int resC[64], resR[64], blk[2][64];        // colours and rounds given; a block's vertices
  __shared__ int ncol;                                  // colours given so far
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = (n + 63) >> 6, NB = (n + 63) >> 6;
  auto far = [&](int par, int i) __attribute__((always_inline)) { return gused + (long long)(par * 64 + i) * more; };
  // word w of row i's bitmap (those in memory are written by atomics: read
  // past this unit's cache)
  auto load = [&](int par, int i, int w) __attribute__((always_inline)) {
    return w < kColLdsWords ? sused[par][i][w]
                            : __hip_atomic_load(far(par, i) + w - kColLdsWords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto mark = [&](int par, int i, int c) __attribute__((always_inline)) {
    if (c < kColLdsColours) atomicOr(&sused[par][i][c >> 6], 1ull << (c & 63));
    else atomicOr(far(par, i) + (c >> 6) - kColLdsWords, 1ull << (c & 63));
  };
  for (int w = tid; w < W; w += kColThreads) done[w] = 0ull;
  if (tid == 0) ncol = 0;
  // what the rows i0, i0 + step, ... of block `b` (buffer par) see of the
  // vertices done, and their edges inside the block and to the block before
  // (in the other buffer).  All first loads go out before any is used: every
  // row is read once, from memory.
  constexpr int kMine = (64 + kW - 2) / (kW - 1);  // rows a wave gathers
  constexpr int kAhead = 4;                        // words a lane loads at a time
  auto gather = [&](int b, int par, int i0, int step) __attribute__((always_inline)) {
    unsigned *flag = sflag[wid];
    const int words = (ncol + 128) / 64 + 1;  // bitmap words that may come into use until the block is resolved
    const int near = min(words, kColLdsWords);
    const int uj = blk[par][lane], pj = blk[par ^ 1][lane];  // clamped where a block is short
    unsigned long long in[kMine], before[kMine], x[kMine][kAhead];
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
      const uint64_t *row = rows + (long long)blk[par][min(i0 + q * step, 63)] * R;
      in[q] = row[uj >> 6];
      before[q] = row[pj >> 6];
#pragma unroll
      for (int t = 0; t < kAhead; ++t) x[q][t] = 64 * t + lane < W ? row[64 * t + lane] : 0ull;
    }
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
      const int i = i0 + q * step;
      if (i >= 64 || 64 * b + i >= n) break;
      for (int w = lane; w < 16 * near; w += 64) flag[w] = 0u;
      for (int w = kColLdsWords + lane; w < words; w += 64)
        if (w < kColLdsWords + more)
          __hip_atomic_store(far(par, i) + w - kColLdsWords, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (words > kColLdsWords) __builtin_amdgcn_s_waitcnt(0);
      __builtin_amdgcn_wave_barrier();
      int mr = 0;
      auto meet = [&](unsigned a) __attribute__((always_inline)) {
        const int c = (int)(a & 0xffff);
        if (c < kColLdsColours) ((unsigned char *)flag)[c] = 1;
        else mark(par, i, c);
      };
      auto word = [&](int w, unsigned long long y) __attribute__((always_inline)) {
        y &= w < W ? done[w] : 0ull;
        while (y) {
          // four neighbours a turn (the last one again where there are fewer)
          unsigned a[4];
          int u = 0;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            if (y) u = 64 * w + __builtin_ctzll(y);
            y &= y - 1;
            a[t] = VLDS ? sval[u] : gval[u];
          }
#pragma unroll
          for (int t = 0; t < 4; ++t) meet(a[t]);
          mr = max(mr, (int)(max(max(a[0], a[1]), max(a[2], a[3])) >> 16) + 1);
        }
      };
#pragma unroll
      for (int t = 0; t < kAhead; ++t)
        if (64 * t < W) word(64 * t + lane, x[q][t]);
      if (W > 64 * kAhead) {
        const uint64_t *row = rows + (long long)blk[par][i] * R;
        for (int w0 = 64 * kAhead; w0 < W; w0 += 64 * kAhead) {
          unsigned long long z[kAhead];
#pragma unroll
          for (int t = 0; t < kAhead; ++t) z[t] = w0 + 64 * t + lane < W ? row[w0 + 64 * t + lane] : 0ull;
#pragma unroll
          for (int t = 0; t < kAhead; ++t) word(w0 + 64 * t + lane, z[t]);
        }
      }
      __builtin_amdgcn_wave_barrier();
      for (int w = 0; w < near; ++w) {
        const unsigned long long m = __ballot(((unsigned char *)flag)[64 * w + lane] != 0);
        if (lane == 0) sused[par][i][w] = m;
      }
      mr = wave_max(mr);
      const unsigned long long e = __ballot(64 * b + lane < n && ((in[q] >> (uj & 63)) & 1ull));
      const unsigned long long c = __ballot(b > 0 && ((before[q] >> (pj & 63)) & 1ull));
      if (lane == 0) {
        most[par][i] = mr;
        adj[par][i] = e;
        cross[i] = c;
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  // block 0 sees nothing done
  if (wid == 0) {
    blk[0][lane] = order[min(lane, n - 1)];
    blk[1][lane] = blk[0][lane];
  }
  __syncthreads();
  if (wid > 0) gather(0, 0, wid - 1, kW - 1);
  __syncthreads();
  int top = 0, rounds = 0;
  for (int b = 0; b < NB; ++b) {
    const int par = b & 1;
    // the next block's vertices, before its gather (nobody reads this buffer)
    if (wid == 0 && b + 1 < NB) blk[par ^ 1][lane] = order[min(64 * (b + 1) + lane, n - 1)];
    __syncthreads();
    if (wid == 0) {
      // resolve block b: lane j's vertex, its smallest free colour m in word
      // mw of its bitmap, its largest round r seen
      const bool mine = 64 * b + lane < n;
      const unsigned long long e = mine ? adj[par][lane] : 0ull;
      int r = mine ? most[par][lane] : 0, mw = 0;
      unsigned long long word = mine ? load(par, lane, 0) : 0ull;
      while (word == ~0ull) word = load(par, lane, ++mw);
      int m = 64 * mw + __builtin_ctzll(~word);
      const int nb = min(64, n - 64 * b);
      for (int i = 0; i < nb; ++i) {
        const int c = __builtin_amdgcn_readlane(m, i), ri = __builtin_amdgcn_readlane(r, i) + 1;
        const int cw = c >> 6;
        const bool next = lane > i && ((e >> i) & 1ull);
        r = next ? max(r, ri) : r;
        word |= next && cw == mw ? 1ull << (c & 63) : 0ull;
        // colours of later words go to the bitmap, a full word gives way to
        // the next: both are rare
        if (__ballot((next && cw > mw) || word == ~0ull) != 0ull) {
          if (next && cw > mw) mark(par, lane, c);
          while (word == ~0ull) word = load(par, lane, ++mw);
        }
        m = 64 * mw + __builtin_ctzll(~word);
      }
      resC[lane] = m;
      resR[lane] = r;  // the round less one
      if (mine) {
        top = max(top, m + 1);
        rounds = max(rounds, r + 1);
      }
    } else if (b + 1 < NB) {
      gather(b + 1, par ^ 1, wid - 1, kW - 1);
    }
    __syncthreads();
    // merge block b into the state and into the next block's rows
    if (wid == 0) {
      const int v = blk[par][lane];
      if (64 * b + lane < n) {
        const unsigned x = (unsigned)resR[lane] << 16 | (unsigned)resC[lane];
        if (VLDS) sval[v] = x;
        else gval[v] = x;
        colour[v] = resC[lane];
        atomicOr(&done[v >> 6], 1ull << (v & 63));
      }
      const int t = wave_max(64 * b + lane < n ? resC[lane] + 1 : 0);
      if (lane == 0) ncol = max(ncol, t);
    }
    if (b + 1 < NB) {
      for (int i = wid; i < 64; i += kW) {
        if (64 * (b + 1) + i >= n) break;
        const bool hit = (cross[i] >> lane) & 1ull;
        if (hit) mark(par ^ 1, i, resC[lane]);
        const int mr = wave_max(hit ? resR[lane] + 1 : 0);
        if (lane == 0) most[par ^ 1][i] = max(most[par ^ 1][i], mr);
      }
    }
  }
  if (wid == 0) {
    top = wave_max(top);
    rounds = wave_max(rounds);
    if (lane == 0) {
      ctr->top = top - 1;
      ctr->rounds = rounds;
    }
  }
}

// ---- which way

// A graph's degrees, from the check.
struct ColDegrees {
  int n;
  unsigned long long ends, squares;
  double edges() const { return 0.5 * (double)ends; }
  bool sparse() const { return 100 * ends < (unsigned long long)n * (unsigned long long)n; }
  // most edges are a few hubs': the squares' sum is above twice that of even degrees
  bool hubs() const { return squares > 2 * (ends / (unsigned)n) * ends; }
  // times in us of a round (its last term is a vertex looking through all its
  // neighbours: the degree at an edge's end) and of all blocks
  double round_us() const { return 10 + 4e-4 * n + 3.2e-3 * (double)squares / std::max(1.0, (double)ends); }
  double blocks_us() const { return (n + 63) / 64 * (n > kColLdsN ? 20.0 : 12.0) + 3e-4 * edges(); }
  int probe(double share) const { return (int)(share * blocks_us() / round_us()); }
};

// The rounds to come, from what the last `rounds` of them took: `was` before
// them, `now` behind them.  At their rate the edges left last edges / e rounds; up
// to twice that where the vertices go at the same rate (a vertex then takes ever
// fewer edges along), and twice again on even degrees, where ever fewer vertices
// beat all their neighbours (3000 vertices at p = 0.3 have 1272 rounds; the first
// takes 4 vertices), not on hubs'.  Below 0: no edge went, no telling.
double rounds_left(const ColDegrees &d, const ColCtr &was, const ColCtr &now, int rounds) {
  const double before = d.edges() - (double)was.gone, left = d.edges() - (double)now.gone;
  if (left <= 0) return 0;
  const double e = ((double)now.gone - (double)was.gone) / rounds, v = (double)(was.left - now.left) / rounds;
  if (e <= 0) return -1;
  return left / e * (1 + std::min(1.0, 2 * (v / was.left) / (e / before))) * (d.hubs() ? 1 : 2.1);
}

// Whether the vertices taken had a quarter more edges than the uncoloured on the
// average: hubs come first, and what they tell may end with them.
bool hubs_first(const ColDegrees &d, const ColCtr &was, const ColCtr &now) {
  const double taken = (double)(was.left - now.left), before = d.edges() - (double)was.gone;
  return ((double)now.gone - (double)was.gone) * was.left > 1.25 * 2 * before * taken;
}

// Whether that many rounds take less time than the blocks.
bool by_rounds(const ColDegrees &d, double left) { return left >= 0 && left * d.round_us() < d.blocks_us(); }

}  // namespace

extern "C" {

int kz_colour_workspace_bytes(int32_t n, size_t *bytes) {
  if (!bytes || n < 0) return KZ_EINVAL;
  *bytes = col_ws(n).total;
  return KZ_OK;
}

int kz_colour_jp(kz_ctx *ctx, int32_t n, const uint64_t *rows, int32_t row_words, const uint64_t *priority,
                 void *ws, size_t ws_bytes, int32_t *colour, void *stream, kz_colour_result *res) {
  kz_colour_result r{};
  r.status = KZ_EINVAL;
  auto done = [&]() {
    if (res) *res = r;
    return r.status;
  };
  if (!ctx || n < 0 || row_words < 0) return done();
  if (n == 0) {
    r.status = KZ_OK;
    return done();
  }
  if (!rows || !priority || !colour || !ws || (uintptr_t)ws % kColAlign) return done();
  if (row_words < (n + 63) / 64) return done();
  if (row_words > kColMaxWords) {
    r.status = KZ_ETOOLARGE;
    return done();
  }
  const ColWs z = col_ws(n);
  if (ws_bytes < z.total) {
    r.status = KZ_EWORKSPACE;
    return done();
  }
  r.status = KZ_EHIP;
  if (hipSetDevice(ctx->device) != hipSuccess) return done();
  hipStream_t s = (hipStream_t)stream;
  char *base = (char *)ws;
  ColCtr *ctr = (ColCtr *)(base + z.ctr);
  uint64_t *U = (uint64_t *)(base + z.U);
  uint8_t *sel = (uint8_t *)(base + z.sel);
  int *rank = (int *)(base + z.rank), *order = (int *)(base + z.order);
  unsigned *val = (unsigned *)(base + z.val);
  unsigned long long *used = (unsigned long long *)(base + z.used);
  ColCtr *h = (ColCtr *)ctx->pinned;  // the context's pinned readback buffer (4 KiB)
  const dim3 grid((unsigned)((n + kColWaves - 1) / kColWaves)), block(kColWaves * 64);
  const unsigned blocks = (unsigned)((n + kRankThreads - 1) / kRankThreads);
  const int slots = col_slots(n);
  const size_t sums = kColHead + slots * sizeof(ctr->sum[0]);
  auto read_back = [&](size_t bytes) {
    return hipGetLastError() == hipSuccess &&
           hipMemcpyAsync(h, ctr, bytes, hipMemcpyDeviceToHost, s) == hipSuccess &&
           hipStreamSynchronize(s) == hipSuccess;
  };
  int ran = 0;  // rounds enqueued
  auto enqueue = [&](int rounds, bool count) {
    for (int i = 0; i < rounds; ++i) {
      hipLaunchKernelGGL(k_col_select, grid, block, 0, s, n, rows, (int)row_words, priority, U, sel, ctr);
      hipLaunchKernelGGL(k_col_colour, grid, block, 0, s, n, rows, (int)row_words, sel, U, colour, ctr, (int)count);
    }
    ran += rounds;
  };
  if (hipMemsetAsync(ctr, 0, sums, s) != hipSuccess) return done();
  hipLaunchKernelGGL(k_col_check, grid, block, 0, s, n, rows, (int)row_words, rank, colour, U, ctr, slots);
  // the first rounds go out with the check, as many as a share of the blocks'
  // time allows whatever the edges
  ColDegrees d{n, 0, 0};
  if (n >= kColProbeN) enqueue(std::max(1, d.probe(kColProbe)), true);
  if (!read_back(sums)) return done();
  if (h->bad) {
    r.status = h->bad == 3 ? KZ_EINVAL : h->bad == 2 ? KZ_ESELFLOOP : KZ_EASYM;
    return done();
  }
  for (int i = 0; i < slots; ++i) {
    d.ends += h->sum[i].ends;
    d.squares += h->sum[i].squares;
  }
  const bool sparse = d.sparse();
  const int probe = d.probe(kColProbeHubs);
  ColCtr was{};
  was.left = n;
  int chunk = kColFirstChunk, last = ran;
  for (;;) {
    // rounds in chunks, ended on the device: one readback per chunk (rounds
    // past the last one return at once)
    if (h->left == 0) {
      r.status = KZ_OK;
      r.rounds = h->rounds;
      r.colours = h->top + 1;
      return done();
    }
    if (last > 0 && h->left >= was.left) return done();  // cannot happen: every round takes the largest uncoloured key
    int next = chunk;
    if (!sparse) {
      const double left = last > 0 ? rounds_left(d, was, *h, last) : -1;
      if (by_rounds(d, left)) next = (int)std::min((double)chunk, left + 1);
      else if (last > 0 && ran < probe && hubs_first(d, was, *h)) next = std::min(chunk, probe - ran);
      else break;
    }
    was = *h;
    last = next;
    enqueue(next, !sparse);
    chunk = std::min(2 * chunk, kColMaxChunk);
    if (!read_back(kColHead)) return done();
  }
  hipLaunchKernelGGL(k_col_rank, dim3(blocks, (unsigned)((n + kRankSpan - 1) / kRankSpan)), dim3(kRankThreads), 0, s, n,
                     priority, rank);
  hipLaunchKernelGGL(k_col_order, dim3(blocks), dim3(kRankThreads), 0, s, n, rank, order);
  if (n <= kColLdsN)
    hipLaunchKernelGGL(k_col_greedy<true>, dim3(1), dim3(kColThreads), 0, s, n, rows, (int)row_words, order, val, used,
                       col_more(n), colour, ctr);
  else
    hipLaunchKernelGGL(k_col_greedy<false>, dim3(1), dim3(kColThreads), 0, s, n, rows, (int)row_words, order, val, used,
                       col_more(n), colour, ctr);
  if (!read_back(kColHead)) return done();
  r.status = KZ_OK;
  r.rounds = h->rounds;
  r.colours = h->top + 1;
  return done();
}

}  // extern "C"
