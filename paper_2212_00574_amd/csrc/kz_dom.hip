// Dominance reductions (thesis section 4.3, Definitions 4.3.1 and 4.3.2,
// Algorithms 1 and 2) on plain bit rows (gfx950).
//
// The algorithms are sequential sweeps whose deletions are visible to every
// later test, repeated until a sweep deletes nothing.  One workgroup runs a
// graph's whole fixpoint on the device (one launch, no host round trip):
// the sweep stays sequential over its steps, and each step's tests run in
// parallel over the workgroup's threads.
//
// Vertex dominance, step b: b deletes every node it dominates.  The set is
// the one b dominates at the start of the step: deleting a dominated a
// cannot make another node dominated by the same b (a node adjacent to a is
// in N(a), so in N(b), so adjacent to b), and the nodes b dominates are
// pairwise non-adjacent, so the edges removed are the sum of their degrees.
//
// Edge dominance, step a: the pairs (a, u), u in N(a), in index order; the
// edge {a,u} goes when some b in N(u), b != a, b not in N(a), sees all of
// N(a) & N(u).  Within the step only N(a) changes (it loses the u's already
// deleted: D), and the test is monotone in D -- W = N(a) & N(u) shrinks, the
// candidates N(u) \ N(a) grow, N(b) stays (it can only lose a, which is not
// in W).  So u is deleted iff its test holds with D restricted to the u's
// before it, a recursion with one solution, reached by parallel passes that
// start from D = {} and add every u whose test holds, until none is added.
#include "kz_internal.h"

namespace kzi {

namespace {

constexpr int kDomMaxWords = 1024;  // rows of at most 1024 words (n <= 65536)

struct DomHdr {
  long long dirs;    // set bits of the input (twice the edges)
  long long dv, de;  // deleted vertices, edges
  long long sweeps;  // sweeps that deleted something
  long long events;  // steps (vertex) or edges (edge) that deleted something
  long long passes;  // edge: parallel passes over a step's neighbours
  int prio;          // worst input problem (P_*)
  int pad[3];
};

__global__ void k_dom_init(DomHdr *h) {
  if (threadIdx.x == 0) {
    h->dirs = 0;
    h->dv = 0;
    h->de = 0;
    h->sweeps = 0;
    h->events = 0;
    h->passes = 0;
    h->prio = P_NONE;
  }
}

// Copies the rows into the state, sets every node alive, counts the set
// bits and checks the input: no bit at or beyond n, no self-loop, every bit
// mirrored.  One thread per row word.
__global__ void __launch_bounds__(256) k_dom_setup(const uint64_t *__restrict__ rows, uint64_t *__restrict__ st,
                                                   uint8_t *__restrict__ alive, int n, int R, DomHdr *h) {
  const long long total = (long long)n * R;
  const long long stride = (long long)gridDim.x * blockDim.x;
  unsigned long long cnt = 0;
  int pr = P_NONE;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int v = (int)(i / R), w = (int)(i % R);
    unsigned long long x = rows[i];
    st[i] = x;
    if (w == 0) alive[v] = 1;
    cnt += __popcll(x);
    const long long base = 64LL * w;
    if (base >= n) {
      if (x) pr = max(pr, (int)P_EINVAL);
      continue;
    }
    if (base + 64 > n) {
      const int keep = (int)(n - base);
      if (x >> keep) pr = max(pr, (int)P_EINVAL);
      x &= (1ull << keep) - 1;
    }
    while (x) {
      const int t = (int)base + __builtin_ctzll(x);
      x &= x - 1;
      if (t == v) pr = max(pr, (int)P_ESELFLOOP);
      else if (!((rows[(long long)t * R + (v >> 6)] >> (v & 63)) & 1ull)) pr = max(pr, (int)P_EASYM);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    cnt += __shfl_xor(cnt, off, kWave);
    pr = max(pr, __shfl_xor(pr, off, kWave));
  }
  if ((threadIdx.x & 63) == 0) {
    if (cnt) atomicAdd((unsigned long long *)&h->dirs, cnt);
    if (pr != P_NONE) atomicMax(&h->prio, pr);
  }
}

// ---- the sweeps
//
// One workgroup runs a graph's fixpoint.  Rows are read by groups of GL
// lanes, lane l of a group holding words l, l + GL, ... (WPL of them), so a
// row is one coalesced load; small graphs keep all rows in LDS (LDS = true).
// Both tests come down to the same loop: a set `cur` of nodes still thought
// dominated loses the neighbours of every x of a set T (row x is taken out
// of it, four rows in flight), and most of the time it is empty after a
// few rows, as the graphs are dense.  What bounds it is the chain of LDS or
// L2 reads of a step.  Edge mode on the evaluation recipe at 1100 nodes (rows
// in LDS) 73.9 -> 11.0 ms, at 1900 (rows in L2) 271 -> 26.8 ms; vertex mode
// 2.6 -> 0.87 and 5.5 -> 1.9 ms; the earlier form tested node by node, a
// chain of dependent loads per test.
constexpr int kDomLdsWords = 19840;  // rows kept in LDS up to this many words ...
constexpr int kDomLdsR = 32;         // ... and this row width (then at most 1102 nodes)
constexpr int kDomLdsNodes = 1152;

template <int GL, int WPL>
struct DomSet {
  uint64_t w[WPL];
};

// The lanes of my group with a bit, from a ballot over the wave.
template <int GL>
__device__ __forceinline__ unsigned long long group_lanes(bool p, int lane) {
  const unsigned long long b = __ballot(p);
  if (GL == kWave) return b;
  return (b >> (lane & ~(GL - 1))) & ((1ull << (GL & 63)) - 1);
}

// cur loses the neighbours of the nodes of T, until it is empty or T is.
// D (may be null): nodes x of D count only for the nodes before x.
template <int GL, int WPL>
__device__ __forceinline__ void dom_strike(const uint64_t *rows, int R, int lane, DomSet<GL, WPL> &cur,
                                           DomSet<GL, WPL> &T, const uint64_t *D) {
  constexpr int kAhead = WPL < 8 ? 4 : WPL < 16 ? 2 : 1;  // rows in flight
  const int gl = lane & (GL - 1), base = lane & ~(GL - 1);
  if constexpr (GL == 1) {
    // a row is a word: a lane's own loop
    static_assert(WPL == 1, "rows of one word");
    while (cur.w[0] && T.w[0]) {
      uint64_t m[kAhead];
      int x = 0;
#pragma unroll
      for (int i = 0; i < kAhead; ++i) {
        if (T.w[0]) x = __builtin_ctzll(T.w[0]);
        T.w[0] &= T.w[0] - 1;
        m[i] = rows[x * R] & (D && ((D[0] >> x) & 1ull) ? (1ull << x) - 1 : ~0ull);
      }
#pragma unroll
      for (int i = 0; i < kAhead; ++i) cur.w[0] &= ~m[i];
    }
    return;
  }
  for (;;) {
    bool mine = false, left = false;
    int x = 0;  // this lane's first node of T
#pragma unroll
    for (int j = WPL - 1; j >= 0; --j) {
      mine |= cur.w[j] != 0ull;
      if (T.w[j]) {
        left = true;
        x = 64 * (gl + GL * j) + __builtin_ctzll(T.w[j]);
      }
    }
    unsigned long long lanes = group_lanes<GL>(left, lane);
    if (group_lanes<GL>(mine, lane) == 0ull || lanes == 0ull) return;
    int f[kAhead], xs[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      f[i] = lanes ? __builtin_ctzll(lanes) : f[0];
      lanes &= lanes - 1;
      xs[i] = __shfl(x, base + f[i], kWave);
    }
    uint64_t rx[kAhead][WPL];
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
#pragma unroll
      for (int j = 0; j < WPL; ++j) {
        const int w = gl + GL * j;
        rx[i][j] = w < R ? rows[(long long)xs[i] * R + w] : 0ull;
      }
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int xw = xs[i] >> 6;
      const uint64_t below = (1ull << (xs[i] & 63)) - 1;
      const bool later = D && ((D[xw] >> (xs[i] & 63)) & 1ull);
#pragma unroll
      for (int j = 0; j < WPL; ++j) {
        const int w = gl + GL * j;
        const uint64_t m = !later || w < xw ? ~0ull : w == xw ? below : 0ull;
        cur.w[j] &= ~(rx[i][j] & m);
        if (gl == f[i] && w == xw) T.w[j] &= ~(1ull << (xs[i] & 63));
      }
    }
  }
}

// Whether row a lies inside row b.
__device__ __forceinline__ bool dom_inside(const uint64_t *ra, const uint64_t *rb, int R) {
  for (int w = 0; w < R; ++w)
    if (ra[w] & ~rb[w]) return false;
  return true;
}

// For sparse graphs, where a struck row takes out few nodes: whether row b has
// one of cur's nodes inside, a lane per word, up to the group's first.
template <int GL, int WPL>
__device__ __forceinline__ bool dom_scan(const uint64_t *rows, int R, int b, int lane, const DomSet<GL, WPL> &cur) {
  const uint64_t *rb = rows + (long long)b * R;
#pragma unroll 1
  for (int j = 0; j < WPL; ++j) {
    uint64_t cand = 0ull;
#pragma unroll
    for (int q = 0; q < WPL; ++q) cand = q == j ? cur.w[q] : cand;
    const int base = 64 * ((lane & (GL - 1)) + GL * j);
    while (group_lanes<GL>(cand != 0ull, lane) != 0ull) {
      bool hit = false;
      if (cand) {
        hit = dom_inside(rows + (long long)(base + __builtin_ctzll(cand)) * R, rb, R);
        cand &= cand - 1;
      }
      if (group_lanes<GL>(hit, lane) != 0ull) return true;
    }
  }
  return false;
}

__device__ __forceinline__ uint64_t dom_valid(int w, int n) {
  const int lo = 64 * w;
  return lo + 64 <= n ? ~0ull : lo < n ? (1ull << (n - lo)) - 1 : 0ull;
}

// Whether dom_scan is the faster one for a graph of that average degree.  Rows in
// memory: a scan is bounded by the loads of 64 rows at once, one for every word
// looked at until one has a bit that b lacks (0.77 us each with 16 waves at it, for 16
// b); striking takes about n ln(n) / degree rows, 4 or fewer at a time, a
// round trip each (1.2 to 3 us by the words a lane holds).  Scanned and struck: 2100
// nodes of degree 42 8 and 17 ms, of degree 210 2.8 and 2.4; 5000 of degree 250 20
// and 32, of degree 2500 8.5 and 2.9.
template <int NT, int GL, int WPL, bool LDS>
__device__ __forceinline__ bool dom_scans(float degree, int n, int R) {
  if (degree * degree * degree < 8.f * n) return true;
  if (LDS || 4.f * degree > n) return false;
  const float d = fmaxf(degree, 1e-3f), off = 1.f - d / (float)n;
  const float words = fminf(1.f / (1.f - __expf(-d / (float)R * off)), (float)R);
  const float scan = 0.012f * min(R, kWave) * 64.f * (float)((R + kWave - 1) / kWave) * off * words / 16.f;
  const float rows = fminf((float)n, (float)n * __logf((float)n) / d);
  const float strike = rows * (WPL == 1 ? 0.3f : WPL < 8 ? 0.6f : WPL < 16 ? 1.5f : 4.f) / (float)(NT / GL);
  return scan < strike;
}

// ---- vertex dominance (Definition 4.3.1): the whole fixpoint, one workgroup
//
// b dominates a iff they are not adjacent and no neighbour of a is outside
// N(b).  With M = the live nodes not adjacent to b (b itself apart), that is
// M less the neighbours of M's nodes (taken row by row in dense graphs: about
// n ln(n) / degree rows; tested node by node in sparse ones).  Most steps delete nothing, so every
// group tests a step of its own (group g: node b0 + g) on the same graph;
// the first step in sweep order that dominates a node is applied, and the
// scan goes on right after it.  Steps before it saw the graph the sequential
// sweep would have shown them (nothing was deleted in between); the results
// of the steps after it are dropped.
template <int NT, int GL, int WPL, bool LDS>
__global__ void __launch_bounds__(NT) k_dom_vertex_run(uint64_t *__restrict__ st,
                                                                uint8_t *__restrict__ alive, int n, int R,
                                                                DomHdr *h) {
  constexpr int kGroups = NT / GL;
  constexpr int kWords = LDS ? kDomLdsR : kDomMaxWords;
  __shared__ uint64_t sRows[LDS ? kDomLdsWords : 1];
  __shared__ uint64_t AL[kWords], D[kWords];  // live nodes; the nodes a step deletes
  __shared__ int dw[kWords];                  // the words of D that hold a node
  __shared__ int first[2], ndw;
  __shared__ unsigned long long nv, ne;
  const int tid = threadIdx.x, lane = tid & 63, gl = lane & (GL - 1);
  const int group = tid / GL;
  if (h->prio != P_NONE) return;
  uint64_t *rows = LDS ? sRows : st;
  if (LDS)
    for (int i = tid; i < n * R; i += NT) sRows[i] = st[i];
  for (int w = tid; w < R; w += NT) AL[w] = dom_valid(w, n);
  if (tid == 0) {
    nv = 0;
    ne = 0;
    first[0] = first[1] = n;
  }
  __syncthreads();
  const bool sparse = dom_scans<NT, GL, WPL, LDS>((float)h->dirs / (float)n, n, R);
  long long sweeps = 0, steps = 0;
  int par = 0;
  for (;;) {
    bool any_sweep = false;
    int b0 = 0;
    while (b0 < n) {
      const int b = b0 + group;
      DomSet<GL, WPL> cur, T;
      bool hit = false;
      if (b < n && ((AL[b >> 6] >> (b & 63)) & 1ull)) {
#pragma unroll
        for (int j = 0; j < WPL; ++j) {
          const int w = gl + GL * j;
          cur.w[j] = w < R ? AL[w] & ~rows[(long long)b * R + w] : 0ull;
          if (w == (b >> 6)) cur.w[j] &= ~(1ull << (b & 63));
          T.w[j] = cur.w[j];
        }
        if (sparse) {
          hit = dom_scan<GL, WPL>(rows, R, b, lane, cur);
        } else {
          dom_strike<GL, WPL>(rows, R, lane, cur, T, nullptr);
          bool some = false;
#pragma unroll
          for (int j = 0; j < WPL; ++j) some |= cur.w[j] != 0ull;
          hit = group_lanes<GL>(some, lane) != 0ull;
        }
        if (hit && gl == 0) atomicMin(&first[par], b);
      }
      __syncthreads();
      const int bf = first[par];
      par ^= 1;  // the other one is at n
      if (bf == n) {
        b0 += kGroups;
        continue;
      }
      // the step that dominates someone: its group has the set, or a scan knew
      // of one and the workgroup tests every node
      const uint64_t *rb = rows + (long long)bf * R;
      if (sparse) {
        for (int x0 = tid & ~63; x0 < n; x0 += NT) {
          const int x = x0 + lane, w = x0 >> 6;
          const uint64_t may = AL[w] & ~rb[w] & ~(w == (bf >> 6) ? 1ull << (bf & 63) : 0ull);
          const unsigned long long in =
              __ballot(((may >> lane) & 1ull) && dom_inside(rows + (long long)x * R, rb, R));
          if (lane == 0) D[w] = in;
        }
        for (int w = (n + 63) / 64 + tid; w < R; w += NT) D[w] = 0ull;
      } else if (b == bf) {
#pragma unroll
        for (int j = 0; j < WPL; ++j) {
          const int w = gl + GL * j;
          if (w < R) D[w] = cur.w[j];
        }
      }
      if (tid == 0) ndw = 0;
      __syncthreads();
      if (tid == 0) first[par ^ 1] = n;  // every thread has read it
      for (int w = tid; w < R; w += NT)
        if (D[w]) {
          dw[atomicAdd(&ndw, 1)] = w;
          AL[w] &= ~D[w];
          atomicAdd(&nv, (unsigned long long)__popcll(D[w]));
        }
      __syncthreads();
      // the deleted nodes lose their rows, a lane at each in LDS, a wave in memory
      // (17000 nodes without an edge, all but one deleted by the first step: 12.5
      // and 6.6 ms); their neighbours (all in N(b)) lose them, in the words listed
      // in dw.  Row b itself does not change.
      const int nd = ndw;
      if constexpr (!LDS) {
        constexpr int kWaves = NT / kWave;
        const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
        uint64_t mine = 0ull;  // every kWaves-th node of a word
        for (int i = wid; i < 64; i += kWaves) mine |= 1ull << i;
        for (int i = 0; i < nd; ++i) {
          const int w0 = dw[i];
          for (uint64_t m = D[w0] & mine; m; m &= m - 1) {
            const int x = 64 * w0 + __builtin_ctzll(m);
            uint64_t *rx = rows + (long long)x * R;
            int deg = 0;
            for (int w = lane; w < R; w += kWave) {
              deg += __popcll(rx[w]);
              rx[w] = 0;
            }
            deg = wave_sum(deg);
            if (lane == 0) {
              alive[x] = 0;
              if (deg) atomicAdd(&ne, (unsigned long long)deg);
            }
          }
        }
      }
      for (int x = tid; x < n; x += NT) {
        uint64_t *rx = rows + (long long)x * R;
        if ((D[x >> 6] >> (x & 63)) & 1ull) {
          if constexpr (LDS) {
            alive[x] = 0;
            unsigned long long deg = 0;
            for (int w = 0; w < R; ++w) {
              deg += __popcll(rx[w]);
              rx[w] = 0;
            }
            if (deg) atomicAdd(&ne, deg);
          }
        } else if ((rb[x >> 6] >> (x & 63)) & 1ull) {
          for (int i = 0; i < nd; ++i) {
            const int w = dw[i];
            const uint64_t y = rx[w];
            if (y & D[w]) rx[w] = y & ~D[w];
          }
        }
      }
      any_sweep = true;
      ++steps;
      b0 = bf + 1;
      __syncthreads();
    }
    if (!any_sweep) break;
    ++sweeps;
  }
  if (LDS)
    for (int i = tid; i < n * R; i += NT) st[i] = sRows[i];
  if (tid == 0) {
    h->dv = (long long)nv;
    h->de = (long long)ne;
    h->sweeps = sweeps;
    h->events = steps;
  }
}

// ---- edge dominance (Definition 4.3.2): the whole fixpoint, one workgroup
//
// Step a deletes {a, u} for the nodes u of N(a) that some b makes dominated:
// b a neighbour of u, not of a, and N(a) & N(u) inside N(b).  For one b those
// are the nodes of N(a) & N(b) less the neighbours of N(a) \ N(b).  A group
// takes one b at a time from the list of the nodes not adjacent to a (where a
// has few neighbours, of those next to one of them); nodes
// already deleted in the step (D) join the list, for the nodes after them,
// and count as gone from N(a) for the nodes after them.  In thin graphs (average
// degree below the root of n) every wave counts a's neighbours first: a node
// without any is no step, with no barrier; one with few needs no list of the
// others; and a turn that sees every neighbour found is the last (a star's
// leaves: the first b is enough).
template <bool LDS>
struct EdgeLds {
  static constexpr int kWords = LDS ? kDomLdsR : kDomMaxWords;
  uint64_t rows[LDS ? kDomLdsWords : 1];
  uint64_t na[kWords], D[kWords], Dn[kWords];  // N(a); deleted so far; found in this pass
  unsigned short list[LDS ? kDomLdsNodes : 64 * kDomMaxWords];
  int cnt[2], near[2];
  long long found;  // the last pass that found a node
  unsigned long long nd;
};

template <int NT, int GL, int WPL, bool LDS, bool THIN>
__device__ __forceinline__ void dom_edge_sweeps(uint64_t *__restrict__ st, int n, int R, DomHdr *h, EdgeLds<LDS> &S) {
  constexpr int kGroups = NT / GL;
  uint64_t *na = S.na, *D = S.D, *Dn = S.Dn;
  unsigned short *list = S.list;
  int *cnt = S.cnt;
  const int tid = threadIdx.x, lane = tid & 63, gl = lane & (GL - 1), group = tid / GL;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint64_t *rows = LDS ? S.rows : st;
  long long sweeps = 0, passes = 0;
  unsigned long long deleted = 0;  // this thread's share
  int par = 0;
  for (;;) {
    bool any_sweep = false;
    for (int a = 0; a < n; ++a) {
      // word w's nodes to the list, a lane per bit (the whole wave calls it)
      auto append = [&](int *count, int w, uint64_t m) __attribute__((always_inline)) {
        if (!m) return;
        int at = 0;
        if (lane == 0) at = atomicAdd(count, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if ((m >> lane) & 1ull)
          list[at + __popcll(m & ((1ull << lane) - 1))] = (unsigned short)(64 * w + lane);
      };
      auto self = [&](int w) { return w == (a >> 6) ? 1ull << (a & 63) : 0ull; };
      // few neighbours, many turns: only their neighbours can be b
      auto is_few = [&](int deg, int others) { return (long long)deg * deg < others && others > 2 * kGroups; };
      // their neighbours, gathered in Dn, from the list to the list
      auto nodes_next = [&](int deg) __attribute__((always_inline)) {
        for (int i = group; i < deg; i += kGroups) {
          const uint64_t *ru = rows + (long long)list[i] * R;
          for (int w = gl; w < R; w += GL) {
            const uint64_t x = ru[w];
            if (x) atomicOr((unsigned long long *)&Dn[w], (unsigned long long)x);
          }
        }
      };
      auto list_next = [&]() __attribute__((always_inline)) {
        for (int w = wid; w < R; w += NT / kWave) {
          append(&cnt[par], w, Dn[w] & ~na[w] & ~self(w));
          if (lane == 0) Dn[w] = 0;
        }
      };
      int deg = 0;
      bool few = false;
      if constexpr (THIN) {
        for (int w = lane; w < R; w += kWave) deg += __popcll(rows[(long long)a * R + w]);
        deg = wave_sum(deg);
        if (deg == 0) {
          ++passes;
          continue;
        }
        few = is_few(deg, n - 1 - deg);
      }
      for (int w = wid; w < R; w += NT / kWave) {
        const uint64_t x = rows[(long long)a * R + w];
        if (lane == 0) {
          na[w] = x;
          D[w] = 0;
          Dn[w] = 0;
        }
        if (THIN && few) append(&S.near[par], w, x);
        else append(&cnt[par], w, ~x & dom_valid(w, n) & ~self(w));
      }
      __syncthreads();
      if (tid == 0) {  // the next step's: nobody uses them in this one
        cnt[par ^ 1] = 0;
        if (THIN) S.near[par ^ 1] = 0;
      }
      bool grew = false;
      if (THIN && few) {
        nodes_next(deg);
        __syncthreads();
        list_next();
        __syncthreads();
      }
      int have = cnt[par];
      if constexpr (!THIN) {
        deg = n - 1 - have;
        if (is_few(deg, have)) {
          __syncthreads();
          if (tid == 0) cnt[par] = 0;
          __syncthreads();
          for (int w = wid; w < R; w += NT / kWave) append(&cnt[par], w, na[w]);
          __syncthreads();
          nodes_next(deg);
          __syncthreads();
          if (tid == 0) cnt[par] = 0;
          __syncthreads();
          list_next();
          __syncthreads();
          have = cnt[par];
        }
      }
      int old = 0;  // list entries the last pass has tested
      for (;;) {
        const long long pass = passes++;
        for (int i = group; i < have; i += kGroups) {
          const int b = list[i];
          const bool later = grew && ((D[b >> 6] >> (b & 63)) & 1ull);  // b counts for the nodes after it
          DomSet<GL, WPL> cur, T;
          bool left = false;  // nodes not found yet
#pragma unroll
          for (int j = 0; j < WPL; ++j) {
            const int w = gl + GL * j;
            cur.w[j] = T.w[j] = 0ull;
            if (w < R) {
              const uint64_t rb = rows[(long long)b * R + w], x = na[w];
              const uint64_t after = !later || w > (b >> 6) ? ~0ull
                                     : w == (b >> 6)        ? ~((2ull << (b & 63)) - 1)
                                                            : 0ull;
              uint64_t open = x & ~D[w];
              if (THIN) open &= ~__hip_atomic_load(&Dn[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              left |= open != 0ull;
              cur.w[j] = open & rb & after;
              T.w[j] = x & ~rb;
            }
          }
          if (THIN && group_lanes<GL>(left, lane) == 0ull) break;
          if (i < old) {
            // tested before: something changes only where T meets a node
            // deleted in this step
            bool meets = false;
#pragma unroll
            for (int j = 0; j < WPL; ++j) {
              const int w = gl + GL * j;
              meets |= w < R && (T.w[j] & D[w]) != 0ull;
            }
            if (group_lanes<GL>(meets, lane) == 0ull) continue;
          }
          dom_strike<GL, WPL>(rows, R, lane, cur, T, grew ? D : nullptr);
#pragma unroll
          for (int j = 0; j < WPL; ++j)
            if (cur.w[j]) {
              atomicOr((unsigned long long *)&Dn[gl + GL * j], (unsigned long long)cur.w[j]);
              S.found = pass;
            }
        }
        __syncthreads();
        if (S.found != pass) break;
        grew = true;
        old = have;
        for (int w = wid; w < R; w += NT / kWave) {
          const uint64_t add = Dn[w] & ~D[w];
          if (lane == 0) D[w] |= add;
          append(&cnt[par], w, add);
        }
        __syncthreads();
        have = cnt[par];
      }
      par ^= 1;
      if (!grew) continue;
      // apply: {a, u} for every u in D
      any_sweep = true;
      for (int w = tid; w < R; w += NT)
        if (D[w]) {
          rows[(long long)a * R + w] = na[w] & ~D[w];
          deleted += __popcll(D[w]);
        }
      for (int u = tid; u < n; u += NT)
        if ((D[u >> 6] >> (u & 63)) & 1ull) rows[(long long)u * R + (a >> 6)] &= ~(1ull << (a & 63));
      __syncthreads();
    }
    if (!any_sweep) break;
    ++sweeps;
  }
  if (LDS)
    for (int i = tid; i < n * R; i += NT) st[i] = S.rows[i];
  if (deleted) atomicAdd(&S.nd, deleted);
  __syncthreads();
  if (tid == 0) {
    h->de = (long long)S.nd;
    h->sweeps = sweeps;
    h->events = h->de;
    h->passes = passes;
  }
}

template <int NT, int GL, int WPL, bool LDS>
__global__ void __launch_bounds__(NT) k_dom_edge_run(uint64_t *__restrict__ st, int n, int R, DomHdr *h) {
  __shared__ EdgeLds<LDS> S;
  const int tid = threadIdx.x;
  if (h->prio != P_NONE) return;
  if (LDS)
    for (int i = tid; i < n * R; i += NT) S.rows[i] = st[i];
  if (tid == 0) {
    S.cnt[0] = S.cnt[1] = S.near[0] = S.near[1] = 0;
    S.found = -1;
    S.nd = 0;
  }
  __syncthreads();
  // a thin graph's steps look at their node first (what that takes is 6 to 20 % of
  // the short steps of dense graphs)
  const double mean = (double)h->dirs / n;
  if (mean * mean < n) dom_edge_sweeps<NT, GL, WPL, LDS, true>(st, n, R, h, S);
  else dom_edge_sweeps<NT, GL, WPL, LDS, false>(st, n, R, h, S);
}

int dom_status(int prio) {
  switch (prio) {
    case P_NONE: return KZ_OK;
    case P_ESELFLOOP: return KZ_ESELFLOOP;
    case P_EASYM: return KZ_EASYM;
    default: return KZ_EINVAL;
  }
}

}  // namespace
}  // namespace kzi

extern "C" {

int kz_dom_workspace_bytes(int32_t n, size_t *bytes) {
  if (!bytes || n < 0) return KZ_EINVAL;
  *bytes = 256;
  return KZ_OK;
}

int kz_dominance(kz_ctx *ctx, int32_t mode, int32_t n, const uint64_t *rows, int32_t row_words, void *ws,
                 size_t ws_bytes, uint8_t *vmask, uint64_t *emask, void *stream, kz_dom_result *res) {
  using namespace kzi;
  kz_dom_result r{};
  auto done = [&](int st) {
    r.status = st;
    if (res) *res = r;
    return st;
  };
  if (!ctx || (mode != KZ_DOM_VERTEX && mode != KZ_DOM_EDGE) || n < 0 || row_words < (n + 63) / 64)
    return done(KZ_EINVAL);
  if (n == 0) return done(KZ_OK);
  if (!rows || !ws || !vmask || !emask || (uintptr_t)ws % 256) return done(KZ_EINVAL);
  if (ws_bytes < sizeof(DomHdr)) return done(KZ_EWORKSPACE);
  if (row_words > kDomMaxWords) return done(KZ_ETOOLARGE);
  if (hipSetDevice(ctx->device) != hipSuccess) return done(KZ_EHIP);
  hipStream_t s = (hipStream_t)stream;
  DomHdr *h = (DomHdr *)ws;
  const int R = row_words;
  hipLaunchKernelGGL(k_dom_init, dim3(1), dim3(64), 0, s, h);
  const long long words = (long long)n * R;
  const int grid = (int)std::min<long long>((words + 255) / 256, 4096);
  hipLaunchKernelGGL(k_dom_setup, dim3(grid), dim3(256), 0, s, rows, emask, vmask, n, R, h);
  // rows in LDS where they fit; a group of 1 to 64 lanes a row, several words
  // a lane beyond 64; fewer waves at the barriers where the rows are short (64
  // nodes at p = 0.5, edges: 0.92 ms with 64 groups of 4 lanes, 0.24 with a lane a
  // row and one wave; 100 nodes at p = 0.1: 1.4 and 0.94 with 2 lanes)
#define KZ_DOM_V(NT, GL, WPL, LDS) \
  hipLaunchKernelGGL((k_dom_vertex_run<NT, GL, WPL, LDS>), dim3(1), dim3(NT), 0, s, emask, vmask, n, R, h)
#define KZ_DOM_E(NT, GL, WPL, LDS) \
  hipLaunchKernelGGL((k_dom_edge_run<NT, GL, WPL, LDS>), dim3(1), dim3(NT), 0, s, emask, n, R, h)
#define KZ_DOM(NT, GL, WPL, LDS)                          \
  do {                                                    \
    if (mode == KZ_DOM_VERTEX) KZ_DOM_V(NT, GL, WPL, LDS); \
    else KZ_DOM_E(NT, GL, WPL, LDS);                      \
  } while (0)
  if (words <= kDomLdsWords && R <= kDomLdsR) {
    if (R == 1) KZ_DOM(64, 1, 1, true);
    else if (R == 2) KZ_DOM(256, 2, 1, true);
    else if (R <= 4) KZ_DOM(256, 4, 1, true);
    else if (R <= 8) KZ_DOM(512, 8, 1, true);
    else if (R <= 16) KZ_DOM(1024, 16, 1, true);
    else KZ_DOM(1024, 32, 1, true);
  } else if (R <= 32) KZ_DOM(1024, 32, 1, false);
  else if (R <= 64) {
    // twice the groups for the edges; a vertex step that deletes drops the others'
    // work (twins 15 ms, 20 with 32 groups)
    if (mode == KZ_DOM_VERTEX) KZ_DOM_V(1024, 64, 1, false);
    else KZ_DOM_E(1024, 32, 2, false);
  } else if (R <= 256) KZ_DOM(1024, 64, 4, false);
  else if (R <= 512) KZ_DOM(1024, 64, 8, false);
  else KZ_DOM(1024, 64, 16, false);
#undef KZ_DOM
#undef KZ_DOM_V
#undef KZ_DOM_E
  DomHdr *hh = (DomHdr *)ctx->pinned;
  if (hipGetLastError() != hipSuccess ||
      hipMemcpyAsync(hh, h, sizeof(DomHdr), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return done(KZ_EHIP);
  r.input_edges = hh->dirs / 2;
  const int st0 = dom_status(hh->prio);
  if (st0 != KZ_OK) return done(st0);
  r.sweeps = (int32_t)hh->sweeps;
  r.deleted_vertices = hh->dv;
  r.deleted_edges = hh->de;
  r.events = hh->events;
  r.scans = hh->passes;
  return done(KZ_OK);
}

}  // extern "C"
