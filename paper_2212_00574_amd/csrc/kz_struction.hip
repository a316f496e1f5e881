// Struction (thesis section 4.1, Definition 4.1.1) on plain bit rows
// (gfx950).  Around a pivot p: A = the neighbours of p and B = the other
// vertices except p; C holds a node c(x, y) for every edge {x, y} inside B
// with x < y.  G' has the nodes A (in vertex order) followed by C (ordered
// by x, then y):
//   A-A: as in G;  C-C: c(x,y) ~ c(x',y') iff x = x' and y ~ y';
//   A-C: a ~ c(x,y) iff a ~ x and a ~ y (the rule that makes Lemmas 1 and 2
//   hold; the thesis states none), so omega(G') = omega(G) - 1.
//
// Plan: A in vertex order and, for every x in B, the count of its C nodes
// (neighbours y > x in B), scanned into offsets.  Build: the node map and M[v]
// = row v compressed onto A's index space (bit t = v ~ A[t]), then G': a node's
// A part is M[a] (A node) or M[x] & M[y] (C node), an A node's C part is the
// transpose of that, and a C node's C part is non-zero only inside its own
// first vertex's block (y ~ y').  A call enqueues all of it and waits once:
// the kernels take the node counts from the header and write nothing when they
// do not fit.
#include "kz_internal.h"

namespace kzi {

namespace {

struct StHdr {
  long long na, nc;    // |A|, |C|
  long long edges2;    // set bits of the input
  int prio;            // input problems (P_*)
  int fits;            // the outputs hold G'
};

constexpr int kStWaves = 4;  // waves (rows) per workgroup
// Workgroups of G's rows at most (the waves go round): a launch of 2^32 threads is
// refused, which the caller's room for nodes alone may ask for, and a workgroup
// without a row takes its slot all the same.
constexpr int kStBlocks = 1 << 16;

__device__ __forceinline__ bool bit(const uint64_t *row, int v) { return (row[v >> 6] >> (v & 63)) & 1ull; }

// Word w of B's mask: the vertices that are neither the pivot nor next to it.
__device__ __forceinline__ uint64_t b_word(const uint64_t *prow, int pivot, int n, int w) {
  const long long lo = 64LL * w;
  uint64_t valid = lo + 64 <= n ? ~0ull : lo < n ? (1ull << (n - lo)) - 1 : 0ull;
  if (w == (pivot >> 6)) valid &= ~(1ull << (pivot & 63));
  return ~prow[w] & valid;
}

// Bits of word w above vertex v.
__device__ __forceinline__ uint64_t above(int v, int w) {
  const int vw = v >> 6, b = v & 63;
  return w > vw ? ~0ull : w < vw ? 0ull : b == 63 ? 0ull : ~0ull << (b + 1);
}

// What a row gives the scan: set bits, C nodes (below 2^28: 2^28 rows of 2^22
// words are past any memory) with the problems found above them.
struct StRow {
  unsigned bits, nodes;
};
constexpr int kStPrio = 28;

// One wave per row v: validation (padding bits, self-loops, symmetry), its set
// bits, its place in A or its count of C nodes.  A lane per word counts; the words
// that hold a bit are then gone through with a lane per bit, four of them at a
// time, so that 256 reverse entries are looked up side by side.  Bounded by that
// latency (8 us at 1000 vertices) or, in sparse rows, by reading them: 20000
// vertices of degree 1, the whole call 0.92 ms with a lane per bit of every word,
// 0.17 with this.
__global__ void __launch_bounds__(kStWaves * kWave) k_st_check(const uint64_t *__restrict__ rows, int n, int R,
                                                               int pivot, int *__restrict__ alist,
                                                               StRow *__restrict__ out) {
  constexpr int kAt = 4;
  const int lane = threadIdx.x & 63, v = blockIdx.x * kStWaves + (threadIdx.x >> 6);
  if (v >= n) return;
  const uint64_t *row = rows + (long long)v * R, *prow = rows + (long long)pivot * R;
  const int vw = v >> 6;
  int cnt = 0, before = 0, nodes = 0;
  bool past = false, asym = false;
  for (int w0 = 0; w0 < R; w0 += kWave) {
    const int w = w0 + lane;
    uint64_t x = 0;
    if (w < R) {
      x = row[w];
      cnt += __popcll(x);
      before += __popcll(prow[w] & (w < vw ? ~0ull : w > vw ? 0ull : (1ull << (v & 63)) - 1));
      nodes += __popcll(x & b_word(prow, pivot, n, w) & above(v, w));
      const long long lo = 64LL * w;
      const uint64_t valid = lo + 64 <= n ? ~0ull : lo < n ? (1ull << (n - lo)) - 1 : 0ull;
      past |= (x & ~valid) != 0ull;
      x &= valid;
    }
    for (unsigned long long some = __ballot(x != 0ull); some;) {
      uint64_t z[kAt];
      int b[kAt];
#pragma unroll
      for (int i = 0; i < kAt; ++i) {
        const int l = some ? __builtin_ctzll(some) : 0;
        const unsigned lo = __builtin_amdgcn_readlane((unsigned)x, l);
        const unsigned hi = __builtin_amdgcn_readlane((unsigned)(x >> 32), l);
        const bool have = some && (((lane < 32 ? lo >> lane : hi >> (lane - 32)) & 1u) != 0u);
        b[i] = have;
        z[i] = have ? rows[(64LL * (w0 + l) + lane) * R + vw] : 0ull;
        some &= some - 1;
      }
#pragma unroll
      for (int i = 0; i < kAt; ++i) asym |= b[i] && !((z[i] >> (v & 63)) & 1ull);
    }
  }
  cnt = wave_sum(cnt);
  before = wave_sum(before);
  nodes = wave_sum(nodes);
  const bool loop = bit(row, v);
  int pr = P_NONE;
  if (__ballot(past)) pr = max(pr, (int)P_EINVAL);
  if (loop) pr = max(pr, (int)P_ESELFLOOP);
  if (__ballot(asym)) pr = max(pr, (int)P_EASYM);
  if (lane == 0) {
    const bool in_a = bit(prow, v);
    if (in_a) alist[before] = v;
    out[v] = StRow{(unsigned)cnt, (in_a || v == pivot ? 0u : (unsigned)nodes) | (unsigned)pr << kStPrio};
  }
}

// Scan of the counts into C offsets, and the header, here and for the host
// (one workgroup).
__global__ void __launch_bounds__(1024) k_st_scan(const StRow *__restrict__ in, const uint64_t *__restrict__ prow, int n,
                                                 int R, long long out_nodes, int out_words,
                                                 long long *__restrict__ coff, StHdr *h, StHdr *host) {
  __shared__ long long nodes[16], bits[16];
  __shared__ int prio[16], deg[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n + 1023) / 1024;
  const int lo = tid * per, hi = min(n, lo + per);
  long long s = 0, b = 0;
  int pr = P_NONE, a = 0;
  for (int v = lo; v < hi; ++v) {
    const StRow x = in[v];
    s += x.nodes & ((1u << kStPrio) - 1);
    b += x.bits;
    pr = max(pr, (int)(x.nodes >> kStPrio));
  }
  for (int w = tid; w < R; w += 1024) a += __popcll(prow[w]);
  long long upto = s;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const long long y = __shfl_up(upto, off, kWave);
    if (lane >= off) upto += y;
    b += __shfl_xor(b, off, kWave);
    a += __shfl_xor(a, off, kWave);
    pr = max(pr, __shfl_xor(pr, off, kWave));
  }
  if (lane == kWave - 1) {
    nodes[wave] = upto;
    bits[wave] = b;
    deg[wave] = a;
    prio[wave] = pr;
  }
  __syncthreads();
  long long run = upto - s, all = 0, na = 0;
  b = 0;
  pr = P_NONE;
  for (int i = 0; i < 16; ++i) {
    if (i < wave) run += nodes[i];
    all += nodes[i];
    b += bits[i];
    na += deg[i];
    pr = max(pr, prio[i]);
  }
  for (int v = lo; v < hi; ++v) {
    coff[v] = run;
    run += in[v].nodes & ((1u << kStPrio) - 1);
  }
  if (tid == 0) {
    coff[n] = all;
    h->na = na;
    h->nc = all;
    h->edges2 = b;
    h->prio = pr;
    h->fits = pr == P_NONE && na + all <= out_nodes && (na + all + 63) / 64 <= out_words;
    *host = *h;
  }
}

// The node map -- (v, -1) for A nodes, (x, y) for C nodes -- and M[v], bit t
// of word j = v ~ A[64 j + t].  One wave per vertex.
__global__ void __launch_bounds__(kStWaves * kWave) k_st_map(const uint64_t *__restrict__ rows, int n, int R, int pivot,
                                                             const int *__restrict__ alist,
                                                             const long long *__restrict__ coff,
                                                             const StHdr *__restrict__ h, int *__restrict__ map,
                                                             uint64_t *__restrict__ M) {
  const int lane = threadIdx.x & 63, v = blockIdx.x * kStWaves + (threadIdx.x >> 6);
  if (v >= n || !h->fits) return;
  const int na = (int)h->na, RA = (na + 63) / 64;
  const uint64_t *row = rows + (long long)v * R, *prow = rows + (long long)pivot * R;
  if (v < na && lane == 0) {
    map[2LL * v] = alist[v];
    map[2LL * v + 1] = -1;
  }
  for (int j = 0; j < RA; ++j) {
    const int t = 64 * j + lane;
    const unsigned long long m = __ballot(t < na && bit(row, alist[t]));
    if (lane == 0) M[(long long)v * RA + j] = m;
  }
  if (v == pivot || bit(prow, v)) return;
  long long at = na + coff[v];
  for (int w0 = 0; w0 < R; w0 += kWave) {
    const int w = w0 + lane;
    uint64_t x = w < R ? row[w] & b_word(prow, pivot, n, w) & above(v, w) : 0ull;
    int upto = __popcll(x);
    const int cnt = upto;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int y = __shfl_up(upto, off, kWave);
      if (lane >= off) upto += y;
    }
    long long p = at + upto - cnt;
    while (x) {
      const int y = 64 * w + __builtin_ctzll(x);
      x &= x - 1;
      map[2 * p] = v;
      map[2 * p + 1] = y;
      ++p;
    }
    at += __shfl(upto, kWave - 1, kWave);
  }
}

// G'.  The first RP waves take the A nodes' rows, word j of all of them each:
// lane q holds what node 64 j + q has in A, 64 of A at a time, and the
// transpose is those 64 rows' word.  The others take a C node's row each: the
// words of its own block by a ballot, the others (A part and zeros) a lane a
// word.  Bounded by the writes: 1000 vertices at p = 0.1, 206 MB, 31 to 41 us
// (a copy's rate); a thread per word that divided its index by RP and looped
// over the word's nodes took 180.
__global__ void __launch_bounds__(kStWaves * kWave) k_st_rows(const uint64_t *__restrict__ rows, int R,
                                                              const uint64_t *__restrict__ M,
                                                              const int *__restrict__ map,
                                                              const long long *__restrict__ coff,
                                                              const StHdr *__restrict__ h, int RP,
                                                              uint64_t *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  if (!h->fits) return;
  const long long na = h->na, np = na + h->nc;
  const int RA = (int)((na + 63) / 64);
  const long long step = (long long)gridDim.x * kStWaves;
  long long i = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kStWaves + (threadIdx.x >> 6)));
  for (; i < RP; i += step) {
    const long long q = 64 * i + lane;
    const uint64_t *mx = M, *my = M;
    if (q < np) {
      const int x = map[2 * q], y = map[2 * q + 1];
      mx += (long long)x * RA;
      my += (long long)(y < 0 ? x : y) * RA;
    }
    for (int j = 0; j < RA; ++j) {
      const unsigned long long col = wave_transpose64(q < np ? mx[j] & my[j] : 0ull, lane);
      const long long a = 64LL * j + lane;
      if (a < na) out[a * RP + i] = col;
    }
  }
  for (i += na - RP; i < np; i += step) {
    const int x = __builtin_amdgcn_readfirstlane(map[2 * i]), y = __builtin_amdgcn_readfirstlane(map[2 * i + 1]);
    const long long b0 = na + coff[x], b1 = na + coff[x + 1];  // the C nodes of x; not empty, this is one
    const int s0 = (int)(b0 >> 6), s1 = (int)((b1 - 1) >> 6) + 1;
    const uint64_t *mx = M + (long long)x * RA, *my = M + (long long)y * RA, *ry = rows + (long long)y * R;
    uint64_t *row = out + i * RP;
    for (int j = lane; j < RP; j += kWave)
      if (j < s0 || j >= s1) row[j] = j < RA ? mx[j] & my[j] : 0ull;
    for (int j = s0; j < s1; ++j) {
      const long long q = 64LL * j + lane;
      const unsigned long long c = __ballot(q >= b0 && q < b1 && bit(ry, map[2 * q + 1]));  // y !~ y: no diagonal
      if (lane == 0) row[j] = c | (j < RA ? mx[j] & my[j] : 0ull);
    }
  }
}

struct StWs {
  size_t hdr, alist, row, coff, M, total;
};

StWs st_ws(int n, int R) {
  StWs z{};
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t at = o;
    o += (b + 255) / 256 * 256;
    return at;
  };
  z.hdr = take(sizeof(StHdr));
  z.alist = take(sizeof(int) * (size_t)(n > 0 ? n : 1));
  z.row = take(sizeof(StRow) * (size_t)(n > 0 ? n : 1));
  z.coff = take(sizeof(long long) * (size_t)(n + 1));
  z.M = take(sizeof(uint64_t) * (size_t)(n > 0 ? n : 1) * (size_t)(R > 0 ? R : 1));
  z.total = o;
  return z;
}

int st_status(int prio) {
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

int kz_struction_workspace_bytes(int32_t n, int32_t row_words, size_t *bytes) {
  if (!bytes || n < 0 || row_words < (n + 63) / 64) return KZ_EINVAL;
  *bytes = kzi::st_ws(n, row_words).total;
  return KZ_OK;
}

int kz_struction(kz_ctx *ctx, int32_t n, const uint64_t *rows, int32_t row_words, int32_t pivot, void *ws,
                 size_t ws_bytes, uint64_t *out, int32_t out_row_words, int64_t out_nodes, int32_t *map,
                 void *stream, kz_struction_result *res) {
  using namespace kzi;
  kz_struction_result r{};
  auto done = [&](int st) {
    r.status = st;
    if (res) *res = r;
    return st;
  };
  if (!ctx || n < 1 || pivot < 0 || pivot >= n || row_words < (n + 63) / 64 || !rows || !ws || (uintptr_t)ws % 256)
    return done(KZ_EINVAL);
  const StWs z = st_ws(n, row_words);
  if (ws_bytes < z.total) return done(KZ_EWORKSPACE);
  if (hipSetDevice(ctx->device) != hipSuccess) return done(KZ_EHIP);
  hipStream_t s = (hipStream_t)stream;
  char *base = (char *)ws;
  StHdr *h = (StHdr *)(base + z.hdr);
  int *alist = (int *)(base + z.alist);
  StRow *row = (StRow *)(base + z.row);
  long long *coff = (long long *)(base + z.coff);
  uint64_t *M = (uint64_t *)(base + z.M);
  const int R = row_words;
  const dim3 grid((unsigned)((n + kStWaves - 1) / kStWaves)), block(kStWaves * kWave);
  // outputs that cannot hold a node are not written: the plan alone then
  const bool build = out && map && out_nodes > 0 && out_row_words > 0;
  hipLaunchKernelGGL(k_st_check, grid, block, 0, s, rows, n, R, pivot, alist, row);
  hipLaunchKernelGGL(k_st_scan, dim3(1), dim3(1024), 0, s, row, rows + (long long)pivot * R, n, R,
                     build ? out_nodes : -1, out_row_words, coff, h, (StHdr *)ctx->pinned_dev);
  if (build) {
    // a wave per node the output can hold, and no more than G' can have nor
    // than kStBlocks give
    const long long most = std::min<long long>(out_nodes, (long long)n * n / 2 + n) + out_row_words;
    const unsigned blocks = (unsigned)std::min<long long>((most + kStWaves - 1) / kStWaves, kStBlocks);
    hipLaunchKernelGGL(k_st_map, grid, block, 0, s, rows, n, R, pivot, alist, coff, h, map, M);
    hipLaunchKernelGGL(k_st_rows, dim3(blocks), block, 0, s, rows, R, M,
                       map, coff, h, out_row_words, out);
  }
  const StHdr *hh = (const StHdr *)ctx->pinned;
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return done(KZ_EHIP);
  r.input_edges = hh->edges2 / 2;
  const int st0 = st_status(hh->prio);
  if (st0 != KZ_OK) return done(st0);
  const long long np = hh->na + hh->nc;
  r.a_nodes = hh->na;
  r.c_nodes = hh->nc;
  r.nodes = np;
  r.row_words = (int32_t)((np + 63) / 64);
  if (!out) return done(KZ_OK);  // plan only
  if (!map || out_nodes < np || out_row_words < (np + 63) / 64) return done(KZ_EWORKSPACE);
  return done(KZ_OK);
}

}  // extern "C"
