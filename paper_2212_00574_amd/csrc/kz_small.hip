// A whole blocking call on a small graph in one workgroup (gfx950): class
// layout, packing, validation, every pass and the output, with the graph in
// LDS.  The general path spends a dozen launches of 3 to 8 us on it, most of
// them a few loads deep, and two looks from the host.
//
// The state is the class-major bit matrix A; a pass lists the edges to test
// (those above the diagonal with an endpoint touched by the round before, 64
// row words at a time) and tests one per lane, word by word over the two
// rows; the bits it removes are collected in B and taken out of A behind a
// barrier, so that a pass sees one state.  Edges of a vertex with no neighbour
// in some class fail by themselves (that class is a third one to all of
// them), so the vertex test needs no write to A.  Bounded by the vector
// instructions of one compute unit (an edge's test is about 115 a wave) and by
// the barriers.  100 dense vertices in 4 classes, two passes: 82 us in twelve
// launches, 39 here; 8 classes, ten passes: 316 and 84 us.
#include "kz_internal.h"

namespace kzi {

namespace {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallList = 128;  // edges a wave lists at a time

// A value from LDS that is the same in every lane.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// The result, and a header that stops the general path's kernels: they find
// nothing else of theirs in the workspace.
__device__ __forceinline__ void end_call(Hdr *h, const kz_out &o, kz_out *host) {
  h->out = o;
  h->bad_layout = 1;
  h->done = 1;
  *host = o;
}

template <bool DENSE>
__global__ void __launch_bounds__(kSmallThreads) k_small(const uint8_t *__restrict__ adj,
                                                         const uint64_t *__restrict__ rows, int row_words,
                                                         const int *__restrict__ colour, int n, int k,
                                                         uint8_t *vmask, uint8_t *emask, uint64_t *erows, Hdr *h,
                                                         kz_out *host) {
  __shared__ unsigned long long A[kSmallWords], B[kSmallWords];
  __shared__ unsigned short list[kSmallWaves][kSmallList];  // u << 8 | v
  __shared__ unsigned long long tm[2][kSmallR];             // touched slots of each block, per pass parity
  __shared__ int coff[kSmallK + 1], soff[kSmallK + 1], cnt[kSmallN / kWave][kSmallK];
  __shared__ short bstart[kSmallR], blen[kSmallR];
  __shared__ unsigned char bcls[kSmallR], cls[kSmallN], inv[kSmallN], perm[kSmallN], alive[kSmallN];
  __shared__ int prio, bad_colour, bad_layout, empty, removed_v, removed_e, tests;
  __shared__ unsigned long long ends;  // last words of the classes
  const int t = threadIdx.x, lane = t & 63, wid = __builtin_amdgcn_readfirstlane(t >> 6);
  if (t == 0) prio = bad_colour = bad_layout = empty = removed_v = removed_e = tests = 0;
  if (t < kSmallN / kWave * kSmallK) cnt[t / kSmallK][t % kSmallK] = 0;
  __syncthreads();
  // class sizes and every vertex's rank in its class among its wave's
  int c = -1, rank = 0;
  if (t < n) {
    c = colour[t];
    if (c < 0 || c >= k) bad_colour = 1;
    else if (!DENSE && t > 0 && colour[t - 1] > c) bad_layout = 1;
  }
  if (wid < (n + kWave - 1) / kWave)
    for (int x = 0; x < k; ++x) {
      const unsigned long long b = __ballot(c == x);
      if (c == x) rank = __popcll(b & ((1ull << lane) - 1));
      if (lane == 0) cnt[wid][x] = __popcll(b);
    }
  __syncthreads();
  if (wid == 0) {  // offsets, lane = class
    static_assert(kSmallN == 2 * kWave, "two waves of vertices");
    const int s = lane < k ? cnt[0][lane] + cnt[1][lane] : 0;
    const int w = (s + 63) / 64;
    const int is = wave_scan(s), iw = wave_scan(w);
    if (lane < k) {
      coff[lane] = is - s;
      soff[lane] = iw - w;
      if (s == 0) empty = 1;
    }
    const int R = __builtin_amdgcn_readlane(iw, kWave - 1);
    if (lane == 0) {
      coff[k] = __builtin_amdgcn_readlane(is, kWave - 1);
      soff[k] = R;
      if (!DENSE && R != row_words) bad_layout = 1;
    }
    if (!bad_colour && (DENSE || R == row_words))
      for (int b = 0; b < w && lane < k; ++b) {
        bcls[iw - w + b] = (unsigned char)lane;
        bstart[iw - w + b] = (short)(is - s + 64 * b);
        blen[iw - w + b] = (short)min(64, s - 64 * b);
      }
    unsigned long long e = 0ull;
    for (int x = 0; x < k; ++x) {
      const int end = __builtin_amdgcn_readlane(iw, x);
      if (end > 0 && end <= 64) e |= 1ull << (end - 1);
    }
    if (lane == 0) ends = e;
  }
  __syncthreads();
  kz_out o{};
  if (bad_colour | bad_layout) {
    if (t == 0) {
      o.result.status = bad_colour ? KZ_ECOLOUR : KZ_EINVAL;
      o.converged = 1;
      end_call(h, o, host);
    }
    return;
  }
  const int R = uni(soff[k]), Rs = R | 1;  // an odd row stride spreads the rows over the banks
  if (t < n) {
    int slot = t;
    if (DENSE) {
      slot = coff[c] + rank;
      if (wid) slot += cnt[0][c];
      inv[t] = (unsigned char)slot;
      perm[slot] = (unsigned char)t;
    }
    cls[slot] = (unsigned char)c;
    alive[slot] = 1;
  }
  for (int i = t; i < n * Rs; i += kSmallThreads) A[i] = 0ull;
  if (t < R) tm[0][t] = 0ull;
  __syncthreads();
  // the graph into A
  int pr = P_NONE;
  if (DENSE) {
    // the caller's rows, four entries a byte (in B, n / 4 bytes a row), a wave
    // per row, kAt rows in flight; then every word of A from its slots' bits
    constexpr int kAt = 4;
    unsigned char *nib = (unsigned char *)B;
    const int W = (n + 3) / 4;
    const bool whole = n % 4 == 0 && (uintptr_t)adj % 4 == 0;  // four entries are a word
    for (int u0 = wid; u0 < n; u0 += kAt * kSmallWaves) {
      unsigned x[kAt];
#pragma unroll
      for (int j = 0; j < kAt; ++j) {
        const int u = min(u0 + j * kSmallWaves, n - 1), v = 4 * lane;
        const uint8_t *row = adj + u * n;
        if (whole) {
          x[j] = v < n ? *(const unsigned *)(row + v) : 0u;
        } else {
          x[j] = 0u;
#pragma unroll
          for (int b = 0; b < 4; ++b) x[j] |= (unsigned)(v + b < n ? row[v + b] : 0) << (8 * b);
        }
      }
#pragma unroll
      for (int j = 0; j < kAt; ++j) {
        const int u = u0 + j * kSmallWaves;
        if (x[j] & ~0x01010101u) pr = P_EINVAL;
        // the four low bits side by side: no two products meet
        if (u < n && lane < W) nib[u * W + lane] = (unsigned char)((x[j] & 0x01010101u) * 0x10204080u >> 28);
      }
    }
    __syncthreads();
    for (int i = t; i < n * R; i += kSmallThreads) {
      const int u = i / R, w = i - u * R, len = blen[w];
      const unsigned char *row = nib + perm[u] * W, *at = perm + bstart[w];
      unsigned lo = 0u, hi = 0u;
      for (int j = 0; j < min(len, 32); ++j) lo |= (((unsigned)row[at[j] >> 2] >> (at[j] & 3)) & 1u) << j;
      for (int j = 32; j < len; ++j) hi |= (((unsigned)row[at[j] >> 2] >> (at[j] & 3)) & 1u) << (j - 32);
      A[u * Rs + w] = (unsigned long long)hi << 32 | lo;
    }
  } else {
    for (int i = t; i < n * R; i += kSmallThreads) {
      const int u = i / R, w = i - u * R;
      const unsigned long long x = rows[i];
      A[u * Rs + w] = x;
      if (blen[w] < 64 && (x >> blen[w])) pr = P_EINVAL;  // padding
    }
  }
  __syncthreads();
  // bits inside a class, and tiles that are not each other's transpose
  for (int i = t; i < n * R; i += kSmallThreads) {
    const int u = i / R, w = i - u * R;
    if (bcls[w] != cls[u]) continue;
    unsigned long long x = A[u * Rs + w] & (blen[w] < 64 ? (1ull << blen[w]) - 1 : ~0ull);
    const int s = u - coff[cls[u]], wu = soff[cls[u]] + (s >> 6);
    for (; x; x &= x - 1) {
      const int v = bstart[w] + __builtin_ctzll(x);
      pr = max(pr, v == u                                       ? (int)P_ESELFLOOP
                   : ((A[v * Rs + wu] >> (s & 63)) & 1ull) != 0ull ? (int)P_EILLEGAL
                                                                   : (int)P_EASYM);
    }
  }
  for (int q = wid; q < R * R; q += kSmallWaves) {
    const int X = q / R, Y = q - X * R;
    if (uni(bcls[X]) >= uni(bcls[Y])) continue;
    const int xl = uni(blen[X]), yl = uni(blen[Y]);
    const unsigned long long xm = xl < 64 ? (1ull << xl) - 1 : ~0ull, ym = yl < 64 ? (1ull << yl) - 1 : ~0ull;
    const unsigned long long e = lane < xl ? A[(bstart[X] + lane) * Rs + Y] & ym : 0ull;
    const unsigned long long et = lane < yl ? A[(bstart[Y] + lane) * Rs + X] & xm : 0ull;
    if (wave_transpose64(e, lane) != et) pr = max(pr, (int)P_EASYM);
  }
  if (pr) atomicMax(&prio, pr);
  __syncthreads();
  if (prio) {
    if (t == 0) {
      o.result.status = prio == P_EINVAL      ? KZ_EINVAL
                        : prio == P_ESELFLOOP ? KZ_ESELFLOOP
                        : prio == P_EASYM     ? KZ_EASYM
                                              : KZ_EILLEGAL;
      o.converged = 1;
      end_call(h, o, host);
    }
    return;
  }
  const unsigned long long last = (unsigned long long)(unsigned)uni((int)(ends >> 32)) << 32 | (unsigned)uni((int)ends);
  const bool none = uni(empty) != 0;
  // bits of the widest block: that many lanes a word, `per` words a wave
  int width = 1;
  for (int w = 0; w < R; ++w) width = max(width, uni(blen[w]));
  const int per = kWave / width, g = lane / width, bit = lane - g * width;
  for (int pass = 1;; ++pass) {
    const int cur = pass & 1, nxt = cur ^ 1;
    for (int i = t; i < n * Rs; i += kSmallThreads) B[i] = 0ull;
    if (t < R) tm[nxt][t] = 0ull;
    if (pass == 1 && t < R) tm[cur][t] = ~0ull;
    __syncthreads();
    // vertices: a neighbour in every other class
    if (t < n && alive[t]) {
      const int cu = cls[t], s = t - coff[cu];
      if ((tm[cur][soff[cu] + (s >> 6)] >> (s & 63)) & 1ull) {
        bool fail = none;
        unsigned long long any = 0ull;
        for (int w = 0, x = 0; w < R; ++w) {
          any |= A[t * Rs + w];
          if ((last >> w) & 1ull) {
            fail |= any == 0ull && x != cu;
            any = 0ull;
            ++x;
          }
        }
        if (fail) {
          alive[t] = 0;
          atomicAdd(&removed_v, 1);
        }
      }
    }
    // edges: a common neighbour in every third class
    int mine = 0, gone = 0;
    // edge {u, v}: true when some third class has no common neighbour
    auto lost = [&](int u, int v, int cu, int cv) {
      const unsigned long long *a = A + u * Rs, *d = A + v * Rs;
      bool fail = none;
      unsigned long long any = 0ull;
      int cx = 0;  // no class is empty, else none
      for (int x = 0; x < R; x += 4) {
        unsigned long long y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int z = min(x + j, R - 1);
          y[j] = a[z] & d[z];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (x + j < R) {
            any |= y[j];
            if ((last >> (x + j)) & 1ull) {
              fail |= any == 0ull && cx != cu && cx != cv;
              any = 0ull;
              ++cx;
            }
          }
        }
      }
      return fail;
    };
    auto drop = [&](int u, int v, int cu, int cv) {
      const int su = u - coff[cu], sv = v - coff[cv], wu = soff[cu] + (su >> 6), wv = soff[cv] + (sv >> 6);
      atomicOr(&B[u * Rs + wv], 1ull << (sv & 63));
      atomicOr(&B[v * Rs + wu], 1ull << (su & 63));
      atomicOr(&tm[nxt][wu], 1ull << (su & 63));
      atomicOr(&tm[nxt][wv], 1ull << (sv & 63));
      ++gone;
    };
    // wave w takes the row words w, w + 16, ..., a lane each
    for (int base = wid; base < n * R; base += kSmallThreads) {
      const int i = base + lane * kSmallWaves;
      unsigned long long M = 0ull;
      int u = 0, w = 0;
      if (i < n * R) {
        u = i / R;
        w = i - u * R;
        const int cu = cls[u], s = u - coff[cu];
        if (bcls[w] > cu) {
          M = A[u * Rs + w];
          if (!((tm[cur][soff[cu] + (s >> 6)] >> (s & 63)) & 1ull)) M &= tm[cur][w];
        }
      }
      const int m = __popcll(M);
      mine += m;
      if (k <= 2) continue;  // no third class
      const unsigned long long has = __ballot(m != 0);
      const int nw = __popcll(has);
      // Lanes over the words' bits, `per` words a step, or the edges listed and
      // a lane each.  A step is about 115 instructions a wave; listing takes 12
      // more for every bit of the fullest of the words in a list.
      const float fill = (float)wave_sum(m) / (float)max(nw, 1);
      if (fill * (float)per * (6.f * fill + 100.f) > 64.f * 115.f) {
        // the words with edges move to the first lanes
        const int below = __popcll(has & ((1ull << lane) - 1));
        const int to = 4 * (m ? below : nw + lane - below);  // a permutation
        const int lo = __builtin_amdgcn_ds_permute(to, (int)(unsigned)M);
        const int hi = __builtin_amdgcn_ds_permute(to, (int)(unsigned)(M >> 32));
        const int uw = __builtin_amdgcn_ds_permute(to, u << 8 | w);
        for (int q = 0; q < nw; q += per) {
          const int from = 4 * (q + g);
          const unsigned x = (unsigned)__builtin_amdgcn_ds_bpermute(from, lo);
          const unsigned y = (unsigned)__builtin_amdgcn_ds_bpermute(from, hi);
          const int e = __builtin_amdgcn_ds_bpermute(from, uw);
          if (g >= per || q + g >= nw || !(((bit < 32 ? x >> bit : y >> (bit - 32)) & 1u))) continue;
          const int p = e >> 8, wp = e & 255, v = bstart[wp] + bit, cp = cls[p], cv = bcls[wp];
          if (lost(p, v, cp, cv)) drop(p, v, cp, cv);
        }
        continue;
      }
      for (;;) {
        const int left = __popcll(M);
        int at = wave_scan(left);
        const int total = min(__builtin_amdgcn_readlane(at, kWave - 1), kSmallList);
        if (total == 0) break;
        for (at -= left; M && at < kSmallList; ++at) {
          list[wid][at] = (unsigned short)(u << 8 | (bstart[w] + __builtin_ctzll(M)));
          M &= M - 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int b = lane; b < total; b += kWave) {
          const int e = list[wid][b], p = e >> 8, v = e & 255, cp = cls[p], cv = cls[v];
          if (lost(p, v, cp, cv)) drop(p, v, cp, cv);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    mine = wave_sum(mine);
    gone = wave_sum(gone);
    if (lane == 0) {
      if (mine) atomicAdd(&tests, mine);
      if (gone) atomicAdd(&removed_e, gone);
    }
    __syncthreads();
    fold_pass(o, pass, n, removed_v, removed_e, tests);
    if (removed_e)
      for (int i = t; i < n * Rs; i += kSmallThreads) A[i] &= ~B[i];
    __syncthreads();
    if (t == 0) removed_v = removed_e = tests = 0;
    if (o.converged) break;
  }
  // the masks
  if (DENSE) {
    for (int v0 = 0; v0 < n; v0 += kWave) {
      const int v = v0 + lane, sl = inv[min(v, n - 1)], cv = cls[sl], j = sl - coff[cv];
      const unsigned long long *a = A + soff[cv] + (j >> 6);
      if (v < n) {
#pragma unroll 4
        for (int u = wid; u < n; u += kSmallWaves) emask[u * n + v] = (uint8_t)((a[inv[u] * Rs] >> (j & 63)) & 1ull);
      }
    }
    if (t < n) vmask[t] = alive[inv[t]];
  } else {
    for (int i = t; i < n * R; i += kSmallThreads) {
      const int u = i / R, w = i - u * R;
      erows[i] = A[u * Rs + w];
    }
    if (t < n) vmask[t] = alive[t];
  }
  if (t == 0) end_call(h, o, host);
}

}  // namespace

void launch_small(const kz_graph &g, const int32_t *colour, int k, uint8_t *vmask, void *emask, Hdr *h, kz_out *host,
                  hipStream_t s) {
  if (g.format == KZ_DENSE_U8)
    hipLaunchKernelGGL((k_small<true>), dim3(1), dim3(kSmallThreads), 0, s, g.adj, nullptr, 0, colour, g.n, k, vmask,
                       (uint8_t *)emask, nullptr, h, host);
  else
    hipLaunchKernelGGL((k_small<false>), dim3(1), dim3(kSmallThreads), 0, s, nullptr, g.rows, g.row_words, colour, g.n,
                       k, vmask, nullptr, (uint64_t *)emask, h, host);
}

}  // namespace kzi
