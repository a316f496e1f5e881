// HIP kernels (gfx950) of the colour-index kernelizer for sparse graphs
// given as CSR (both directions, column ids strictly increasing per row).
//
// The state is kept in the caller's order, in the output buffers themselves:
// vmask[v] (vertex alive) and emask[e] (entry e of col_idx alive; both
// directions of an edge always agree).  Per vertex the pass keeps PM(v), the
// set of colour classes holding an alive neighbour of v (KW 64-bit words).
//
// Tests (thesis section 4.2, vertex and edge colour indices):
//   vertex v fails   <=> PM(v) misses a class other than class(v);
//   edge {u,v} fails <=> some class outside {class(u), class(v)} holds no
//                        common alive neighbour.  Quick reject: such a class
//                        is certainly empty when PM(u) & PM(v) misses it;
//                        otherwise the entries of row v are looked up in row
//                        u and the classes of common alive neighbours
//                        collected, until every third class has one.
// Both directions of an edge are quick-rejected independently (same answer);
// the search of row v meets the reverse entry, so no index of it is kept.
#include <climits>

#include "kz_internal.h"

namespace kzi {

namespace {

__device__ __forceinline__ bool csr_bad(const Hdr *h) { return (h->bad_colour | h->bad_layout) != 0; }

// Adds two per-wave counts into counter slots (par, slot, j0) and (par,
// slot, j1) with one atomic each per workgroup of 4 waves: the counter lines
// take one update per workgroup instead of one per wave.  Every thread of the
// workgroup calls it.
__device__ __forceinline__ void wg_add2(Hdr *h, int par, int j0, long long a, int j1, long long b) {
  __shared__ long long sRed[4][2];
  const int wv = threadIdx.x >> 6;
  a = (long long)wave_sum((int)a);
  b = (long long)wave_sum((int)b);
  if ((threadIdx.x & 63) == 0) {
    sRed[wv][0] = a;
    sRed[wv][1] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const long long ta = sRed[0][0] + sRed[1][0] + sRed[2][0] + sRed[3][0];
    const long long tb = sRed[0][1] + sRed[1][1] + sRed[2][1] + sRed[3][1];
    const int slot = blockIdx.x % kCtrSlots;
    if (ta) atomicAdd(&h->ctr(par, slot, j0), (unsigned long long)ta);
    if (tb) atomicAdd(&h->ctr(par, slot, j1), (unsigned long long)tb);
  }
}

constexpr int kCsrTable = 1024;  // slots of the edge test's table of a row ...
constexpr int kCsrRow = 512;     // ... and the longest row it takes
// Where a lane merges two rows by itself (k_csr_edge).  Rows of up to kCsrShort
// entries together, in graphs of up to kCsrMean entries a row on the average: a
// table for a row of a few entries costs more than they do (200 000 vertices of
// 4 entries, 3 classes: 0.36 ms a call, 0.33 with this; a triangulated grid of
// 490 000 vertices 0.63 and 0.42; from 18 entries a row on 0.58 and 0.65, as waves
// then do both).  And in pass 1 rows that begin alike, for kCsrTry steps.
constexpr int kCsrMean = 16;
constexpr int kCsrShort = 48;
constexpr int kCsrTry = 24;

// Four entries of a row (rows start on 4 bytes only).
struct __attribute__((packed, aligned(4))) Four {
  int v[4];
};

__device__ __forceinline__ int csr_slot(int x) { return (int)(((unsigned)x * 2654435761u) >> 22); }

// OR over the wave, the same in every lane.
__device__ __forceinline__ unsigned wave_or(unsigned x) {
  x |= dpp<kDppRor + 8>(x);
  x |= dpp<kDppRor + 4>(x);
  x |= dpp<kDppRor + 2>(x);
  x |= dpp<kDppRor + 1>(x);
  return (unsigned)(__builtin_amdgcn_readlane((int)x, 0) | __builtin_amdgcn_readlane((int)x, 16) |
                    __builtin_amdgcn_readlane((int)x, 32) | __builtin_amdgcn_readlane((int)x, 48));
}

// Lane l's value of x.
__device__ __forceinline__ long long lane_value(long long x, int l) {
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)x, l);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)((unsigned long long)x >> 32), l);
  return (long long)(((unsigned long long)hi << 32) | lo);
}

// Row bounds of u, or false when they do not lie inside [0, nnz].
__device__ __forceinline__ bool row_ok(const int64_t *rp, int u, long long nnz, long long &b, long long &e) {
  b = rp[u];
  e = rp[u + 1];
  return b >= 0 && b <= e && e <= nnz;
}

// Whether u is among entries [vb, ve) of col_idx (strictly increasing).
// With `vec` (col_idx 16-byte aligned) the search walks aligned pieces of
// four entries, one 16-byte load each: a piece whose valid entries bracket u
// decides, otherwise half of the remaining pieces are dropped.  Entries of
// neighbouring rows that share a boundary piece are ignored; a piece that
// would reach past nnz is read entry by entry.
__device__ __forceinline__ bool row_has(const int32_t *ci, long long nnz, long long vb, long long ve, int u,
                                        bool vec) {
  if (vb >= ve) return false;
  if (!vec) {
    long long lo = vb, hi = ve;
    while (lo < hi) {
      const long long mid = lo + (hi - lo) / 2;
      if (ci[mid] < u) lo = mid + 1;
      else hi = mid;
    }
    return lo < ve && ci[lo] == u;
  }
  long long lo = vb >> 2, hi = (ve - 1) >> 2;  // pieces, inclusive
  while (lo <= hi) {
    const long long mid = lo + (hi - lo) / 2;
    const long long e0 = mid << 2;
    int x0, x1, x2, x3;
    if (e0 + 3 < nnz) {
      const int4 q = *(const int4 *)(ci + e0);
      x0 = q.x;
      x1 = q.y;
      x2 = q.z;
      x3 = q.w;
    } else {
      x0 = ci[e0];
      x1 = e0 + 1 < nnz ? ci[e0 + 1] : 0;
      x2 = e0 + 2 < nnz ? ci[e0 + 2] : 0;
      x3 = 0;
    }
    // the piece's entries inside [vb, ve): positions jf..jl
    const int jf = (int)(vb > e0 ? vb - e0 : 0);
    const int jl = (int)(ve - 1 - e0 < 3 ? ve - 1 - e0 : 3);
    const int f = jf == 0 ? x0 : jf == 1 ? x1 : jf == 2 ? x2 : x3;
    const int l = jl == 0 ? x0 : jl == 1 ? x1 : jl == 2 ? x2 : x3;
    if (u < f) {
      hi = mid - 1;
    } else if (u > l) {
      lo = mid + 1;
    } else {
      return (jf <= 0 && x0 == u) || (jf <= 1 && jl >= 1 && x1 == u) || (jf <= 2 && jl >= 2 && x2 == u) ||
             (jl >= 3 && x3 == u);
    }
  }
  return false;
}

// The same by a guess first: where the entries lie evenly, u's place among the
// ve - vb is near (ve - vb) u / n, so the 16 entries around it, loaded side by
// side, mostly hold it or tell that it is missing; else the search goes on over
// the entries on the side that they leave.  100 000 vertices, 50 entries a row:
// k_csr_first 131 -> 119 us; 72 of them are this search, a random line of a
// col_idx five times an L2 for each of 2.5 million entries.
__device__ __forceinline__ bool row_has_near(const int32_t *ci, long long nnz, long long vb, long long ve, int u,
                                             float inv_n, bool vec) {
  if (!vec || vb >= ve) return row_has(ci, nnz, vb, ve, u, vec);
  const int len = (int)min(ve - vb, 1ll << 30);
  const long long at = vb + (int)((float)len * ((float)u * inv_n)) - 8;
  const long long e0 = min(max(at, vb), ve - 1) & ~3ll;
  if (e0 + 16 > nnz) return row_has(ci, nnz, vb, ve, u, vec);
  int4 q[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) q[j] = *(const int4 *)(ci + e0 + 4 * j);
  // entries of the neighbouring rows count as below and above every vertex
  const int before = (int)max(vb - e0, 0ll), after = (int)min(ve - e0, 16ll);
  bool hit = false, below = before > 0, above = after < 16;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int x = j % 4 == 0 ? q[j / 4].x : j % 4 == 1 ? q[j / 4].y : j % 4 == 2 ? q[j / 4].z : q[j / 4].w;
    const bool in = j >= before && j < after;
    hit |= in && x == u;
    below |= in && x < u;
    above |= in && x > u;
  }
  if (hit || (below && above)) return hit;
  return below ? row_has(ci, nnz, e0 + 16, ve, u, vec) : row_has(ci, nnz, vb, e0, u, vec);
}

// Pass 1's sweep over the rows, one wave per row u: the colour range (stage
// 1), the structure and stage-2 checks, the start of the state (every entry
// alive, every vertex touched, the row of every entry recorded) and pass 1's
// vertex test with u's presence mask, all from one read of the row.
template <int KW>
__global__ void __launch_bounds__(256) k_csr_first(Plan p, const int64_t *rp, const int32_t *ci,
                                                   long long nnz, const int *colour, uint8_t *vmask,
                                                   uint8_t *emask) {
  Hdr *h = p.hdr;
  __shared__ unsigned long long sPM[4][KW];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int u = blockIdx.x * 4 + wv;
  const int n = p.n, k = p.k;
  int balance = 0;  // entries above the diagonal minus entries below it
  bool uf = false;  // u fails pass 1's vertex test
  const bool vec = ((uintptr_t)ci & 15) == 0;
  const float inv_n = 1.f / (float)n;
  long long b, e;
  // stage 1: every colour in [0,k) (also on rows whose bounds are broken)
  const int cu = u < n ? colour[u] : 0;
  if (u < n && lane == 0 && (cu < 0 || cu >= k)) h->bad_colour = 1;
  if (u < n && !row_ok(rp, u, nnz, b, e)) {
    if (lane == 0) atomicMax(&h->prio, P_EINVAL);
  } else if (u < n) {
    int pr = P_NONE;
    if (u == 0 && lane == 0 && rp[0] != 0) pr = P_EINVAL;
    if (u == n - 1 && lane == 0 && rp[n] != nnz) pr = P_EINVAL;
    if (lane < KW) sPM[wv][lane] = 0;
    unsigned long long mine = 0;  // classes met (KW == 1: atomics on one word would queue)
    __builtin_amdgcn_wave_barrier();
    for (long long i = b + lane; i < e; i += kWave) {
      const int v = ci[i];
      p.src[i] = u;
      emask[i] = 1;
      p.efail[i] = 0;
      if (v < 0 || v >= n || (i > b && ci[i - 1] >= v)) {
        pr = max(pr, P_EINVAL);
        continue;
      }
      if (v == u) {
        pr = max(pr, P_ESELFLOOP);
        continue;
      }
      const int cv = colour[v];
      if (cv == cu) pr = max(pr, P_EILLEGAL);
      if (cv >= 0 && cv < k) {
        if (KW == 1) mine |= 1ull << cv;
        else atomicOr(&sPM[wv][cv >> 6], 1ull << (cv & 63));
      }
      // Symmetry: every entry (u,v) with v > u must have its reverse (v,u),
      // found by binary search in row v; with as many entries below the
      // diagonal as above it (summed on the device at the pass's end), reversal
      // then maps the upper entries onto the lower ones, so the lower ones need
      // no search.
      if (v < u) {
        --balance;
        continue;
      }
      ++balance;
      long long vb, ve;
      const bool found = row_ok(rp, v, nnz, vb, ve) && row_has_near(ci, nnz, vb, ve, u, inv_n, vec);
      if (!found) pr = max(pr, P_EASYM);
    }
    if (pr) atomicMax(&h->prio, pr);
    if (KW == 1) {
      const unsigned lo = wave_or((unsigned)mine), hi = wave_or((unsigned)(mine >> 32));
      if (lane == 0) sPM[wv][0] = (unsigned long long)hi << 32 | lo;
    }
    __builtin_amdgcn_wave_barrier();
    // pass 1's vertex test: u fails iff some class other than its own is
    // missing from PM(u)
    bool fail = false;
    if (lane == KW) p.pm[(long long)u * (KW + 1) + KW] = (unsigned long long)(unsigned)cu;  // record: colour
    if (lane < KW) {
      const unsigned long long pm = sPM[wv][lane];
      p.pm[(long long)u * (KW + 1) + lane] = pm;
      const int lo = lane * 64;
      unsigned long long want = 0;
      if (k > lo) want = (k - lo >= 64) ? ~0ull : ((1ull << (k - lo)) - 1);
      if ((cu >> 6) == lane) want &= ~(1ull << (cu & 63));
      fail = (want & ~pm) != 0;
    }
    uf = __ballot(fail) != 0;
    if (lane == 0) {
      vmask[u] = uf ? 0 : 1;
      p.touched[1][u] = 1;
      p.touched[0][u] = 0;
    }
  }
  // removed vertices and the balance, counted with pass 1's counters
  wg_add2(h, 1, 0, lane == 0 && uf ? 1 : 0, 3, balance);
}

// Vertex test and presence masks of passes after the first.  One wave per
// vertex, lanes over its entries; only the alive vertices touched by the
// previous round.  Also resets this pass's bookkeeping.
template <int KW>
__global__ void __launch_bounds__(256) k_csr_vertex(Plan p, const int64_t *rp, const int32_t *ci,
                                                    const int *colour, uint8_t *vmask,
                                                    const uint8_t *emask, int pass) {
  Hdr *h = p.hdr;
  if (csr_bad(h) || h->prio || h->done) return;
  const int n = p.n, k = p.k;
  const int cur = pass & 1, nxt = cur ^ 1;
  {
    const long long gt = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = gt; i < n; i += stride) p.touched[nxt][i] = 0;
    if (gt < kCtrSlots * 4) h->ctr(nxt, gt / 4, gt % 4) = 0;
  }
  __shared__ unsigned long long sPM[4][KW];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int v = blockIdx.x * 4 + wv;
  if (v >= n) return;
  if (!vmask[v] || !p.touched[cur][v]) return;
  if (lane < KW) sPM[wv][lane] = 0;
  __builtin_amdgcn_wave_barrier();
  const long long b = rp[v], e = rp[v + 1];
  for (long long i = b + lane; i < e; i += kWave) {
    if (!emask[i]) continue;
    const int c = colour[ci[i]];
    atomicOr(&sPM[wv][c >> 6], 1ull << (c & 63));
  }
  __builtin_amdgcn_wave_barrier();
  // v fails iff some class other than its own is missing from PM(v)
  const int cv = colour[v];
  bool fail = false;
  if (lane < KW) {
    const unsigned long long pm = sPM[wv][lane];
    p.pm[(long long)v * (KW + 1) + lane] = pm;
    const int lo = lane * 64;
    unsigned long long want = 0;
    if (k > lo) want = (k - lo >= 64) ? ~0ull : ((1ull << (k - lo)) - 1);
    if ((cv >> 6) == lane) want &= ~(1ull << (cv & 63));
    fail = (want & ~pm) != 0;
  }
  const bool vf = __ballot(fail) != 0;
  if (lane == 0) {
    if (vf) {
      vmask[v] = 0;
      atomicAdd(&h->ctr(cur, blockIdx.x % kCtrSlots, 0), 1ull);
    }
  }
}

// Edge test, one thread per directed entry.  The quick reject is taken by
// each of an edge's two entries for itself: both see the same two presence
// masks; a failing entry is flagged for the apply pass, counted once per
// undirected edge (u < v) and marks its row touched.  The edges it leaves (u
// < v) are searched by the whole wave, up to four of a row u at a time, in
// step, so that four chains of loads are in flight: lanes over row v's
// entries, each looked up in a hash table of u's live neighbours in LDS (rows
// over kCsrRow entries: by binary search), and a byte per class tells what has
// been found (plain stores: as atomics on a mask the lanes would meet in one
// word).  The lane that meets u in row v knows the reverse entry, so a failing
// edge flags both.  Two kinds of edges a lane settles alone before that, by
// merging the rows up to its third classes: those of short rows, and in pass 1
// those whose rows begin alike, as in cliques or next to hubs: they find what
// they need in a few steps (cliques of 200 vertices, 2.7 million edges, 3 classes:
// 0.57 ms a call, 0.21 with this), where random rows pay one load more (2 % of a
// call).  How much alike: by the common neighbours that k - 2 classes take on the
// average (1 for 3 classes, then 3, 5.5, 8.4 up to 14.7 for 8) against the steps
// for one of them.  Bounded by the rows read (256 to 384 bytes of 128-byte
// lines an edge at degree 50) and their latency.  Three passes at 100 000
// vertices and 2.5 million edges with planted cliques: 376 -> 141 us at 30
// classes, 2920 -> 355 us at 4, where nearly every edge is searched (a lane
// per entry merged the two rows before).
template <bool FIRST, int KW>
__global__ void __launch_bounds__(256) k_csr_edge(Plan p, const int64_t *rp, const int32_t *ci,
                                                  long long nnz, const int *colour, const uint8_t *emask,
                                                  int pass, int per_wave, int shorts, int alike) {
  Hdr *h = p.hdr;
  if (csr_bad(h) || h->prio || h->done) return;
  constexpr int kAtOnce = 4;
  __shared__ int4 sTab[4][kCsrTable / 4];          // u's live neighbours, -1 where free
  __shared__ unsigned sSeen[4][kAtOnce][16 * KW];  // a byte per class
  const int k = p.k, cur = pass & 1, nxt = cur ^ 1;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const long long i = ((long long)blockIdx.x * 4 + wv) * per_wave + lane;
  bool act = lane < per_wave && i < nnz && (FIRST || emask[i]);
  int u = -1, v = -1, cu = 0, cv = 0, tested = 0, removed = 0;
  bool fail = false, open = false;  // open: passes the quick reject, some class to find
  if (act) {
    u = p.src[i];
    v = ci[i];
    act = FIRST || p.touched[cur][u] || p.touched[cur][v];
  }
  if (act) {
    tested = u < v;
    // each endpoint's record: its presence mask, then its colour
    const uint64_t *ru = p.pm + (long long)u * (KW + 1), *rv = p.pm + (long long)v * (KW + 1);
    unsigned long long mu[KW + 1], mv[KW + 1];
    if constexpr (KW == 1) {
      const ulonglong2 a = *(const ulonglong2 *)ru, c = *(const ulonglong2 *)rv;
      mu[0] = a.x;
      mu[1] = a.y;
      mv[0] = c.x;
      mv[1] = c.y;
    } else {
#pragma unroll
      for (int j = 0; j <= KW; ++j) {
        mu[j] = ru[j];
        mv[j] = rv[j];
      }
    }
    cu = (int)mu[KW];
    cv = (int)mv[KW];
#pragma unroll
    for (int j = 0; j < KW; ++j) {
      const int lo = j * 64;
      unsigned long long need = k > lo ? ((k - lo >= 64) ? ~0ull : ((1ull << (k - lo)) - 1)) : 0ull;
      if ((cu >> 6) == j) need &= ~(1ull << (cu & 63));
      if ((cv >> 6) == j) need &= ~(1ull << (cv & 63));
      fail |= (need & ~(mu[j] & mv[j])) != 0;
      open |= need != 0;
    }
    open = open && !fail && u < v;
    if (fail) {
      p.efail[i] = 1;
      removed = u < v;
    }
  }
  // entries are in row order: of the lanes marking one row, only the first
  // of each run stores the flag
  const int marks = fail ? u : -1, prev = __shfl_up(marks, 1, kWave);
  if (marks >= 0 && (lane == 0 || prev != marks)) p.touched[nxt][marks] = 1;
  long long vb = 0, ve = 0;
  if (open) {
    vb = rp[v];
    ve = rp[v + 1];
    long long a = rp[u], c = vb, back = -1;
    const long long ae = rp[u + 1];
    int room = INT_MAX;  // steps
    if (ae - a + ve - vb > shorts) {
      room = 0;
      if (FIRST && alike <= 4) {
        // (entries past a row's end may count: they only choose the way)
        const Four x = *(const Four *)(ci + min(a, nnz - 4)), y = *(const Four *)(ci + min(c, nnz - 4));
        int same = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) same += x.v[j] == y.v[0] || x.v[j] == y.v[1] || x.v[j] == y.v[2] || x.v[j] == y.v[3];
        if (same >= (ae - a > kCsrRow ? 1 : alike)) room = kCsrTry;
      }
    }
    if (room) {
      // the lane merges the two rows itself
      unsigned long long need[KW];
#pragma unroll
      for (int j = 0; j < KW; ++j) {
        const int lo = j * 64;
        need[j] = k > lo ? ((k - lo >= 64) ? ~0ull : ((1ull << (k - lo)) - 1)) : 0ull;
        if ((cu >> 6) == j) need[j] &= ~(1ull << (cu & 63));
        if ((cv >> 6) == j) need[j] &= ~(1ull << (cv & 63));
      }
      bool found = false;
      int x = ci[a], y = ci[c];
      for (int left = room;;) {
        const bool both = x == y, up = x <= y, down = y <= x;
        if (both && (FIRST || (emask[a] && emask[c]))) {
          const int cw = colour[x];
          unsigned long long some = 0;
#pragma unroll
          for (int j = 0; j < KW; ++j) {
            if ((cw >> 6) == j) need[j] &= ~(1ull << (cw & 63));
            some |= need[j];
          }
          found = some == 0ull;
          if (found) break;
        }
        if (y == u) back = c;
        a += up;
        c += down;
        if (a >= ae || c >= ve || --left == 0) break;
        if (up) x = ci[a];
        if (down) y = ci[c];
      }
      if (found) {
        open = false;
      } else if (a >= ae || c >= ve) {
        // past v in row u or past the end of row v, so past u there
        open = false;
        p.efail[i] = 1;
        if (back >= 0) p.efail[back] = 1;
        p.touched[nxt][u] = 1;
        p.touched[nxt][v] = 1;
        ++removed;
      }
    }
  }
  unsigned long long todo = __ballot(open);
  while (todo) {
    // the edges of one row u of this wave's entries
    const int l0 = __builtin_ctzll(todo);
    const int qu = __builtin_amdgcn_readlane(u, l0), qcu = __builtin_amdgcn_readlane(cu, l0);
    unsigned long long same = todo & __ballot(u == qu);
    todo &= ~same;
    const long long b = rp[qu];
    const int len = (int)(rp[qu + 1] - b);
    const bool hashed = len <= kCsrRow;
    int *tab = (int *)sTab[wv];
    __builtin_amdgcn_wave_barrier();
    if (hashed) {
#pragma unroll
      for (int t = 0; t < kCsrTable / 4 / kWave; ++t) sTab[wv][t * kWave + lane] = make_int4(-1, -1, -1, -1);
      __builtin_amdgcn_wave_barrier();
      for (int t = lane; t < len; t += kWave) {
        const int x = ci[b + t];
        if (!FIRST && !emask[b + t]) continue;
        int at = csr_slot(x);
        while (atomicCAS(&tab[at], -1, x) != -1) at = (at + 1) & (kCsrTable - 1);
      }
      __builtin_amdgcn_wave_barrier();
    }
    while (same) {
      int l[kAtOnce], qcv[kAtOnce];
      long long qb[kAtOnce], back[kAtOnce];
      int ql[kAtOnce];
      bool found[kAtOnce];
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        l[q] = same ? __builtin_ctzll(same) : -1;
        same &= same - 1;
        const int lq = max(l[q], 0);
        qb[q] = lane_value(vb, lq);
        ql[q] = (int)(lane_value(ve, lq) - qb[q]);
        qcv[q] = __builtin_amdgcn_readlane(cv, lq);
        back[q] = -1;  // the reverse entry, in the lane that meets it
        found[q] = l[q] < 0;
      }
      for (int w = lane; w < kAtOnce * 16 * KW; w += kWave) sSeen[wv][0][w] = 0u;
      __builtin_amdgcn_wave_barrier();
      for (int t = 0;; t += kWave) {
        int y[kAtOnce];
        bool live[kAtOnce];
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) {
          const bool in = !found[q] && t + lane < ql[q];
          y[q] = in ? ci[qb[q] + t + lane] : -1;
          live[q] = in && (FIRST || emask[qb[q] + t + lane]);
        }
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q)
          if (y[q] == qu) back[q] = qb[q] + t + lane;
        if (hashed) {
          int at[kAtOnce], z[kAtOnce];
#pragma unroll
          for (int q = 0; q < kAtOnce; ++q) {
            at[q] = csr_slot(y[q]);
            z[q] = tab[at[q]];
          }
#pragma unroll
          for (int q = 0; q < kAtOnce; ++q) {
            while (live[q] && z[q] != y[q] && z[q] != -1) {
              at[q] = (at[q] + 1) & (kCsrTable - 1);
              z[q] = tab[at[q]];
            }
            live[q] = live[q] && z[q] == y[q];
          }
        } else {
#pragma unroll
          for (int q = 0; q < kAtOnce; ++q) {
            int lo = 0, hi = live[q] ? len : 0;
            while (lo < hi) {
              const int mid = (lo + hi) >> 1;
              if (ci[b + mid] < y[q]) lo = mid + 1;
              else hi = mid;
            }
            live[q] = live[q] && lo < len && ci[b + lo] == y[q] && (FIRST || emask[b + lo]);
          }
        }
        bool more = false;
        int c[kAtOnce];
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) c[q] = live[q] ? colour[y[q]] : 0;
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q)
          if (live[q]) ((unsigned char *)sSeen[wv][q])[c[q]] = 1;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) {
          if (!found[q] && __ballot(live[q])) {
            bool all = true;
            for (int x = lane; all && x - lane < k; x += kWave)
              all = __ballot(x < k && x != qcu && x != qcv[q] && !((unsigned char *)sSeen[wv][q])[x]) == 0ull;
            found[q] = all;
          }
          more |= !found[q] && t + kWave < ql[q];
        }
        if (!more) break;
      }
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        if (found[q]) continue;
        if (back[q] >= 0) p.efail[back[q]] = 1;
        if (lane == l[q]) {
          p.efail[i] = 1;
          p.touched[nxt][u] = 1;
          p.touched[nxt][v] = 1;
          ++removed;
        }
      }
    }
  }
  wg_add2(h, cur, 2, tested, 1, removed);
}

// Removes the entries that failed this pass (after every test of the pass
// has read the old masks).  Four entries per thread.
__global__ void __launch_bounds__(256) k_csr_apply(Plan p, long long nnz, uint8_t *emask, int pass, kz_out *out) {
  const Hdr *h = p.hdr;
  if (h->done) return;
  // the other blocks may see the run done only when nothing fails, or on an
  // input error
  if (blockIdx.x == 0 && threadIdx.x < kWave) pass_end(p, pass, true, out);
  if (csr_bad(h) || h->prio) return;
  const long long i0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const long long i = i0 + j;
    if (i < nnz && p.efail[i]) {
      p.efail[i] = 0;
      emask[i] = 0;
    }
  }
}

inline unsigned grid_of(long long work, int per_block) {
  long long g = (work + per_block - 1) / per_block;
  return (unsigned)(g < 1 ? 1 : g);
}

}  // namespace

int csr_words(int k) { return k <= 64 ? 1 : (k <= 256 ? 4 : 16); }

void launch_csr_first(const Plan &p, const int64_t *rp, const int32_t *ci, long long nnz, const int *colour,
                      uint8_t *vmask, uint8_t *emask, hipStream_t s) {
  const dim3 grid(grid_of(p.n, 4)), block(256);
  const int kw = csr_words(p.k);
  if (kw == 1) hipLaunchKernelGGL((k_csr_first<1>), grid, block, 0, s, p, rp, ci, nnz, colour, vmask, emask);
  else if (kw == 4) hipLaunchKernelGGL((k_csr_first<4>), grid, block, 0, s, p, rp, ci, nnz, colour, vmask, emask);
  else hipLaunchKernelGGL((k_csr_first<16>), grid, block, 0, s, p, rp, ci, nnz, colour, vmask, emask);
}

void launch_csr_vertex(const Plan &p, const int64_t *rp, const int32_t *ci, const int *colour, uint8_t *vmask,
                       const uint8_t *emask, int pass, hipStream_t s) {
  const dim3 grid(grid_of(p.n, 4)), block(256);
  const int kw = csr_words(p.k);
#define KZ_CSR_V(W) hipLaunchKernelGGL((k_csr_vertex<W>), grid, block, 0, s, p, rp, ci, colour, vmask, emask, pass)
  if (kw == 1) KZ_CSR_V(1);
  else if (kw == 4) KZ_CSR_V(4);
  else KZ_CSR_V(16);
#undef KZ_CSR_V
}

void launch_csr_edge(const Plan &p, const int64_t *rp, const int32_t *ci, long long nnz, const int *colour,
                     const uint8_t *emask, int pass, bool first, hipStream_t s) {
  if (nnz <= 0) return;
  // entries a wave takes: fewer where whole waves of them would not fill the
  // chip's 8192 wave slots, as a wave searches its edges one group after the
  // other (1000 vertices, 100 000 edges: 206 us with 64, 58 us with 16)
  const int per_wave = nnz >= 64LL * 8192 ? 64 : nnz >= 32LL * 8192 ? 32 : 16;
  const dim3 grid(grid_of(nnz, 4 * per_wave)), block(256);
  const int kw = csr_words(p.k);
  // shorts: entries of two rows up to which lanes merge them; alike: how many of
  // the first four have to agree (5: no number does).  Rows too long for the
  // table are merged at the first sign, as they would be bisected.
  const int shorts = nnz <= (long long)kCsrMean * p.n ? kCsrShort : 0;
  const int alike = nnz < 4 || p.k > 8 ? 5 : p.k > 5 ? 3 : p.k - 2;
#define KZ_CSR_E(F, W) hipLaunchKernelGGL((k_csr_edge<F, W>), grid, block, 0, s, p, rp, ci, nnz, colour, emask, pass, per_wave, shorts, alike)
  if (first) {
    if (kw == 1) KZ_CSR_E(true, 1);
    else if (kw == 4) KZ_CSR_E(true, 4);
    else KZ_CSR_E(true, 16);
  } else {
    if (kw == 1) KZ_CSR_E(false, 1);
    else if (kw == 4) KZ_CSR_E(false, 4);
    else KZ_CSR_E(false, 16);
  }
#undef KZ_CSR_E
}

void launch_csr_apply(const Plan &p, long long nnz, uint8_t *emask, int pass, kz_out *out, hipStream_t s) {
  hipLaunchKernelGGL(k_csr_apply, dim3(grid_of(nnz, 1024)), dim3(256), 0, s, p, nnz, emask, pass, out);
}

}  // namespace kzi
