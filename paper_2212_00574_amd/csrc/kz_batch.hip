// Batched kernelization (gfx950): many graphs in one persistent launch.
//
// Each graph is a job: a sequence of synchronous passes (Definition 4.2.1's
// vertex and edge colour-index tests, applied to a snapshot), and each pass
// is a list of items: 128-vertex chunks for the vertex test and 64x64 block
// tiles (X < Y) for the edge test.  A workgroup takes the next graph from an
// atomic queue, sets it up and lists its first pass; its waves split the
// items.  The workgroup that finishes the last item of a pass carries the
// job on: it applies the tiles that changed and either ends the job or lists
// the next pass.
//
// A pass normally belongs to the workgroup that listed it ("solo": no other
// workgroup touches the job, so no cross-workgroup fences are needed).  A
// pass with more items than the workgroup has waves is "shared" once the
// queue is empty, or earlier when it is very large: it is published on a
// board, and workgroups claim runs of its
// items with a compare-and-swap on the job's claim word (a workgroup looking
// for work prefers a well-stocked shared pass to a new graph), keep their
// counts and touched bits in LDS, and merge them into the job's state in HBM
// before they report the run finished.  The run that completes the pass makes its workgroup the
// carrier.  Nobody waits for anybody: a pass is continued by whoever
// finishes it, so the launch cannot deadlock, and a workgroup with nothing
// to do leaves once every graph is finished (or after a few milliseconds
// without finding work).
//
// Graph g's rows follow the bit-row layout of the single-graph path
// (class-major slots; class c's segment has ceil(s_c/64) words) and sit at
// word offset row_offset[g] of the rows arena; its colours and vertex mask at
// vertex_offset[g].  The state is kept in the emask arena (same layout); the
// changed words of a pass go to the next-state arena (same layout); the
// changed-tile list and the item list sit at int offset 2*row_offset[g] of
// two list arenas of their own.
//
// Cache lines.  The L2 of each XCD is a write-back cache, and an invalidate
// (the acquire half of a fence) keeps lines that hold dirty bytes.  A line
// that a workgroup reads while another workgroup on the same XCD writes
// other bytes of it can therefore survive a fence with stale bytes.  So no
// 128-byte line is shared between two graphs (the host requires every
// graph's ranges to start on a line, and the list arenas are laid out per
// row word), and within a pass every line that is read is written by at
// most the item that reads it: a vertex item owns 128 vertices (one line of
// the vertex mask), and the item list starts on a line of its own, away
// from the changed-tile list that tiles append to during the pass.  Lines
// that several items write in one pass (next-state words, the changed-tile
// list) are read only by the carrier, after every writer has released them.  Graphs too large for this path (k > kBatchK, row words >
// kBatchR, or n > kBatchN) get status KZ_ETOOLARGE in their result and are
// left to the single-graph path.
#include "kz_internal.h"
#include "kz_mx.h"

namespace kzi {

namespace {

// Waves of a workgroup: all that a compute unit's registers hold.  Two workgroups
// of 8 or four of 4 keep as many in flight, but a cascade then has fewer of them
// to itself and sharing a pass costs more: 4096 graphs 12.2 ms, 27.9 and 82.4; 64
// graphs 2.3, 5.8 and 17.8.
constexpr int NW = kBatchWaves;
constexpr int kVertexItem = 1 << 30;                 // item = kVertexItem | chunk, else X | Y << kYShift
constexpr int kVChunk = 128;                         // vertices of a vertex item: one line of the vertex mask
constexpr int kYShift = 9, kXMask = (1 << kYShift) - 1;
constexpr unsigned long long kIdleTicks = 2000000;   // 20 ms of the 100 MHz wall clock
constexpr unsigned long long kHostPoll = 200;        // 2 us: session mode's look at the host's count
// Claim word: pass (24 bits) | items (20 bits) | next unclaimed item (20 bits).
constexpr int kItemBits = 20;
constexpr unsigned kItemMask = (1u << kItemBits) - 1;
// Rows of blocks whose tiles a wave lists together: the tiles that the waves of
// a workgroup take at the same time then share their rows (4096 graphs, four
// batches: 16.3 ms a row at a time, 15.8 with 4, 16.0 with 2 or 8).
constexpr int kStrip = 4;
// A pass is shared once the queue is empty, or earlier when it is very large or
// its job has run long.
constexpr int kShareBig = 2048;   // items
// A job that has run so many passes times the items of this one is shared
// though graphs wait: run by one workgroup a long cascade (74 passes on 1122
// vertices, 27 ms) outlasts all the other graphs' work (about 11 ms), shared it
// takes a third.  Seven batches of 4096 graphs, mean of a batch: 17.9 ms never,
// 17.4 from 7000 on, 15.6 from 5500, 15.1 from 4096, 15.5 from 3072 (a shared
// pass costs the others' time), 17.4 from 1536.
constexpr int kShareWork = 4096;

__device__ __forceinline__ unsigned long long bcast64(unsigned long long x, int lane) {
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)x, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(x >> 32), lane);
  return ((unsigned long long)hi << 32) | lo;
}

// A value every lane holds identically, moved to a scalar register: the job
// and item words come from LDS or memory, which the compiler takes to differ
// from lane to lane.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename T>
__device__ __forceinline__ T *uni(T *p) {
  const unsigned long long x = (unsigned long long)p;
  const unsigned lo = (unsigned)uni((int)x), hi = (unsigned)uni((int)(x >> 32));
  return (T *)(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ bool tbit(const unsigned *b, int i) { return (b[i >> 5] >> (i & 31)) & 1u; }

__device__ __forceinline__ unsigned long long lanes_below(int lane) {
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Agent-scope relaxed accesses to the job's shared words.
template <typename T>
__device__ __forceinline__ T ald(T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void ast(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Release and acquire at agent scope, each with its wait.  A release writes
// this XCD's L2 back (buffer_wbl2) and must not let the atomic that
// publishes become visible before that write-back has landed; the sequence
// the compiler emits for a release atomic on gfx950 issues the atomic right
// after buffer_wbl2 with no wait in between, and a workgroup on another XCD
// can then see the published word while the words it guards (a counter
// reset, next-state words, list entries) are still on their way.  So the
// release is a fence followed by an explicit wait for every outstanding
// memory operation (the write-back included), and the publishing atomic is
// relaxed.  The acquire writes back first (the invalidate keeps dirty
// lines, stale bytes and all, so a line must be clean when it arrives),
// then invalidates, and waits for both before the workgroup's barrier lets
// other waves load.
__device__ __forceinline__ void release_agent() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __builtin_amdgcn_s_waitcnt(0);
}
// Release to the host (system scope), with its wait, for results that the
// host reads from pinned memory.
__device__ __forceinline__ void release_system() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  __builtin_amdgcn_s_waitcnt(0);
}
__device__ __forceinline__ void acquire_system() {
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
  __builtin_amdgcn_s_waitcnt(0);
}
__device__ __forceinline__ void acquire_agent() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __builtin_amdgcn_s_waitcnt(0);
}

// A job's sizes and buffers.
struct GView {
  int g, n, k, R;
  int slack;  // classes a test may find without a witness: k - clique size
  const uint64_t *rows;
  uint64_t *cur, *nxt;
  const int *colour;
  uint8_t *valive;
  int *changed, *items;  // each starts on a 128-byte line
  BatchJob *J;
};

// What a workgroup keeps in LDS about the job it works on.
struct BatchLds {
  int coff[kBatchK + 1], soff[kBatchK + 1];
  short bcls[kBatchR];
  unsigned short bstart[kBatchR];
  unsigned char blen[kBatchR];
  unsigned tc[kBatchN / 32], tn[kBatchN / 32];    // vertices touched in the previous / this pass
  unsigned btc[kBatchR / 32], btn[kBatchR / 32];  // blocks touched in the previous / this pass
  int job, pass;       // the job and pass the copies above belong to
  int pass0;           // the job's first pass
  int shared;          // the pass is shared
  int got, base, cnt, nitems, next_item, last, reload;
  int prio, nchanged;  // this run (solo: this pass)
  unsigned long long removed_v, removed_e, tests;
  int gi, queue_empty, bad_colour, bad_layout, pick, quit, end, status;
  unsigned long long ticket;  // session mode: the ticket of the job being started
  GView view;          // the job whose items are run
};

// A job's descriptor: the batch's, or in session mode the copy its starter
// made of the host slot.
__device__ __forceinline__ kz_batch_graph job_desc(const BatchArgs &a, int g) {
  return a.session ? a.jobs[g].sdesc : a.graphs[g];
}

__device__ __forceinline__ GView gview(const BatchArgs &a, int g) {
  const kz_batch_graph G = job_desc(a, g);
  GView v;
  v.g = uni(g);
  v.n = uni(G.n);
  v.k = uni(G.k);
  v.R = uni(G.row_words);
  v.slack = uni(G.clique > 0 && G.clique < G.k ? G.k - G.clique : 0);
  if (a.ptrs || a.session) {
    const BatchPtrs P = a.session ? a.jobs[g].sptrs : a.ptrs[g];
    v.rows = uni(P.rows);
    v.cur = uni(P.emask);
    v.nxt = uni(P.next);
    v.colour = uni(P.colour);
    v.valive = uni(P.vmask);
    v.changed = uni(P.lists);
    v.items = uni(P.items);
  } else {
    v.rows = uni(a.rows + G.row_offset);
    v.cur = uni(a.emask + G.row_offset);
    v.nxt = uni(a.next + G.row_offset);
    v.colour = uni(a.colour + G.vertex_offset);
    v.valive = uni(a.vmask + G.vertex_offset);
    v.changed = uni(a.lists + 2 * G.row_offset);
    v.items = uni(a.items + 2 * G.row_offset);
  }
  v.J = uni(a.jobs + g);
  return v;
}

// ---- vertex test on 64 vertices (one wave): vertex v fails when more than
// `slack` other classes hold none of its neighbours; pass 1 also validates
// the rows.  A lane reads its row kVertexWords at a time, all loads of a turn
// in flight together: walking the classes one load at a time cost a memory
// round trip per class, and a cascade's passes wait for their vertex items.
constexpr int kVertexWords = 8;

__device__ __forceinline__ void vertex_chunk(const GView &V, BatchLds &S, int v0, bool first, int lane) {
  const int n = V.n, k = V.k, R = V.R;
  const uint64_t *src = V.cur;
  const int v = v0 + lane;
  const bool act = v < n && (first || (V.valive[v] && tbit(S.tc, v)));
  if (!__ballot(act)) return;
  const uint64_t *row = src + (long long)(act ? v : v0) * R;
  const int cv = act ? V.colour[v] : -1;
  int miss = 0;  // other classes without a neighbour
  int pr = 0, seen = 0;
  bool own = false;  // a bit in the row's own class
  unsigned long long any = 0;
#pragma unroll 1
  for (int t = 0; t < R; t += kVertexWords) {
    unsigned long long x[kVertexWords];
#pragma unroll
    for (int i = 0; i < kVertexWords; ++i) x[i] = row[min(t + i, R - 1)];
#pragma unroll
    for (int i = 0; i < kVertexWords; ++i) {
      const int w = t + i;
      if (w >= R) break;
      const int c = uni(S.bcls[w]);
      any |= x[i];
      own |= c == cv && x[i] != 0ull;
      if (w + 1 < uni(S.soff[c + 1])) continue;
      // the class's last word
      ++seen;
      const int s = uni(S.coff[c + 1]) - uni(S.coff[c]);
      if (first && act && (s & 63) && (x[i] >> (s & 63))) pr = max(pr, P_EINVAL);
      miss += c != cv && any == 0ull;
      any = 0;
    }
  }
  miss += k - seen;  // classes without a vertex
  if (first && act && own) {
    // bits inside a row's own class (invalid input): classify them
    const int w0 = S.soff[cv], w1 = S.soff[cv + 1], s = S.coff[cv + 1] - S.coff[cv], jv = v - S.coff[cv];
    for (int w = w0; w < w1; ++w) {
      unsigned long long y = row[w];
      if (w == w1 - 1 && (s & 63)) y &= (1ull << (s & 63)) - 1;
      while (y) {
        const int b = __builtin_ctzll(y);
        y &= y - 1;
        const int t = S.coff[cv] + (w - w0) * 64 + b;
        if (t == v) pr = max(pr, P_ESELFLOOP);
        else
          pr = max(pr, ((src[(long long)t * R + w0 + (jv >> 6)] >> (jv & 63)) & 1ull) ? (int)P_EILLEGAL
                                                                                       : (int)P_EASYM);
      }
    }
  }
  if (pr) atomicMax(&S.prio, pr);
  const bool fail = act && miss > V.slack;
  if (act) {
    if (first) V.valive[v] = fail ? 0 : 1;
    else if (fail) V.valive[v] = 0;
  }
  const int nf = wave_sum(fail ? 1 : 0);
  if (lane == 0 && nf) atomicAdd(&S.removed_v, (unsigned long long)nf);
}

// ---- edge test on tile (X, Y) (one wave): edge (u, v) fails when more than
// `slack` third classes hold no common neighbour.  Only pairs with a touched
// endpoint are tested again after pass 1; the others keep their outcome.
//
// The rows' words are multiplied as FP4 codes (kz_mx.h), a class's words
// summed up, so a zero sum is a class without a witness: no search is left.
// The wave takes the 32 columns u of one half of block X after the other (32
// sums and 32 minima in half floats fit the 128 registers that 16 waves of a
// workgroup leave each), over windows of kTileWords words of both blocks'
// rows in LDS of its own: pieces of consecutive rows load whole cache lines,
// where 64 lanes reading a word of 64 rows touch 64 lines for 512 bytes.  A
// class of more than four words ends early once every pair to test has a
// witness.  With slack the zero sums of a class are packed and added up as
// bit planes.  Tiles with few pairs to test (later passes: a third of the
// tiles of 4096 graphs of 4..16 classes of 8..128 vertices have up to 128)
// take them one per lane.  On those graphs a launch took 28.1 ms with a
// ballot per row and class, and takes 17.7 ms (12.1 ms with the order below, long
// cascades shared, and the tile's words kept in LDS):
// 16 waves keep the vector ALUs busy, about 2000 instructions a tile, 64 of
// them per class for the minima.  With clique sizes two below the classes
// (512 graphs) 44.3 and 9.6 ms.
constexpr int kTileWords = 7;  // odd: 64 lanes reading a column of words meet no bank conflict
constexpr int kTilePairs = 128;  // edges to test up to which they are taken one per lane
constexpr int kPlanes = 6;     // bits of a miss count (at most 62 third classes)

struct TileRows {
  unsigned long long u[kBlk][kTileWords], v[kBlk][kTileWords];
};

// A tile's words and pairs to test while the product needs all registers: in
// scratch memory they were 2.4 GB of writes a launch of 4096 graphs (six
// batches: 15.0 ms, 14.5 with this).
struct Kept {
  unsigned long long eu[kBlk], et[kBlk], pt[kBlk];
};

// 16 sums, element e's "zero" to bit e.
__device__ __forceinline__ unsigned zeros16(const mx_v16f &acc) {
  unsigned z = 0;
#pragma unroll
  for (int e = 15; e >= 0; --e) z = (z << 1) | min(mx_bits(acc[e]), 1u);
  return ~z & 0xffffu;
}

// Column half j of the pairs `want` (lane u: bits v) in the sums' layout: the
// inverse of mx_columns, quarter 0 in the low and quarter 1 in the high half.
__device__ __forceinline__ unsigned want_bits(unsigned long long want, int j, int lane) {
  unsigned out = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const unsigned x = (unsigned)(want >> (32 * i));
    const mx_u2 both = mx_split(x, x);  // lanes 0..31's, lanes 32..63's in both halves
    unsigned y = ((j ? both.y : both.x) >> ((lane >> 5) * 4)) & 0x0f0f0f0fu;
    y = (y | (y >> 4)) & 0x00ff00ffu;
    y = (y | (y >> 8)) & 0xffffu;
    out |= y << (16 * i);
  }
  return out;
}

// Orders the wave's reads and writes of LDS before it with those after it.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Words t .. t + nw - 1 of the rows of the block that starts at slot s0, into
// LDS: eight lanes a row, eight rows a load.  Rows past the block's end (not
// past the graph's) are the next block's; no pair to test is in them.
__device__ __forceinline__ void stage_rows(const GView &V, unsigned long long (*dst)[kTileWords], int s0, int t,
                                           int nw, int lane) {
  const int R = V.R, pc = lane & 7, top = V.n - 1 - s0;
  int r = lane >> 3;
  const char *base = (const char *)(V.cur + (long long)s0 * R + t);
  const unsigned word = 8u * (unsigned)min(pc, nw - 1);
  unsigned long long x[8];
  if (top >= kBlk - 1) {
    const unsigned off = 8u * (unsigned)(r * R) + word;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = *(const unsigned long long *)(base + (long long)(64 * i) * R + off);
  } else {
    asm volatile("" : "+v"(r));  // not kept from one window to the next
#pragma unroll
    for (int i = 0; i < 8; ++i)
      x[i] = *(const unsigned long long *)(base + (8u * (unsigned)(min(r + 8 * i, top) * R) + word));
  }
  if (pc < nw)
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[8 * i + r][pc] = x[i];
}

// Stages a window of both blocks' rows from word w on and returns its start.
__device__ __forceinline__ int stage_tile(const GView &V, TileRows &W, int xs, int ys, int w, int lane) {
  const int nw = min(kTileWords, V.R - w);
  wave_order();  // the previous window is read
  stage_rows(V, W.u, xs, w, nw, lane);
  stage_rows(V, W.v, ys, w, nw, lane);
  wave_order();
  return w;
}

// Lane u: the pairs (bits v) with at most `slack` third classes without a
// witness, as matrix products; the pairs to test are in `kept`.  t: first word of
// the window staged.
template <bool SLACK>
__device__ __forceinline__ unsigned long long tile_product(const GView &V, const BatchLds &S, int X, int Y, int lane,
                                                           const Kept &kept, TileRows &W, int t) {
  const int cx = uni(S.bcls[X]), cy = uni(S.bcls[Y]);
  const int xs = uni(S.bstart[X]), ys = uni(S.bstart[Y]);
  const bool two_u = uni(S.blen[X]) > 32, two_v = uni(S.blen[Y]) > 32;
  const mx_u2 *pu = (const mx_u2 *)W.u[lane], *pv = (const mx_u2 *)W.v[lane];
  // per column half j: the minima so far, two per register as half floats
  // (the sums are positive or zero, so they compare as whole numbers; the
  // conversion keeps zeros and only zeros zero), or with slack the bit planes
  // of the miss counts
  mx_us2 m[2][2][8];
  unsigned plane[2][kPlanes];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) m[j][i][e] = mx_us2{1, 1};
#pragma unroll
    for (int b = 0; b < kPlanes; ++b) plane[j][b] = 0u;
  }
  auto fold = [&](int j, const mx_v16f &a0, const mx_v16f &a1) __attribute__((always_inline)) {
    if constexpr (SLACK) {
      unsigned carry = zeros16(a0) | (two_v ? zeros16(a1) << 16 : 0u);
#pragma unroll
      for (int b = 0; b < kPlanes; ++b) {
        const unsigned x = plane[j][b];
        plane[j][b] = x ^ carry;
        carry &= x;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        m[j][0][e] = __builtin_elementwise_min(m[j][0][e], mx_halves(a0[2 * e], a0[2 * e + 1]));
      if (two_v)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          m[j][1][e] = __builtin_elementwise_min(m[j][1][e], mx_halves(a1[2 * e], a1[2 * e + 1]));
    }
  };
  int seen = 0;  // third classes with a word
#pragma unroll 1
  for (int c = 0; c < V.k; ++c) {
    const int w0 = uni(S.soff[c]), w1 = uni(S.soff[c + 1]);
    if (c == cx || c == cy || w0 == w1) continue;
    ++seen;
    // the whole class in the window where it fits one
    if (w0 >= t + kTileWords || (w1 > t + kTileWords && w1 - w0 <= kTileWords))
      t = stage_tile(V, W, xs, ys, w0, lane);
    if (w1 - w0 <= 2) {
      const bool two_w = w1 - w0 == 2;
      const mx_u2 u0 = pu[w0 - t], v0 = pv[w0 - t], us0 = mx_split(u0.x, u0.y), vs0 = mx_split(v0.x, v0.y);
      const mx_v8i V00 = mx_codes(vs0.x), V01 = mx_codes(vs0.y);
      mx_u2 us1 = {};
      mx_v8i V10 = {}, V11 = {};
      if (two_w) {
        const mx_u2 u1 = pu[w0 + 1 - t], v1 = pv[w0 + 1 - t], vs1 = mx_split(v1.x, v1.y);
        us1 = mx_split(u1.x, u1.y);
        V10 = mx_codes(vs1.x);
        V11 = mx_codes(vs1.y);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 1 && !two_u) break;
        const mx_v8i U0 = mx_codes(j ? us0.y : us0.x);
        mx_v16f a0 = mx_mma(V00, U0, mx_v16f{}), a1 = mx_mma(V01, U0, mx_v16f{});
        if (two_w) {
          const mx_v8i U1 = mx_codes(j ? us1.y : us1.x);
          a0 = mx_mma(V10, U1, a0);
          a1 = mx_mma(V11, U1, a1);
        }
        fold(j, a0, a1);
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 1 && !two_u) break;
      const unsigned wb = want_bits(kept.pt[lane], j, lane);
      if (w0 < t || w0 >= t + kTileWords) t = stage_tile(V, W, xs, ys, w0, lane);
      mx_v16f a0, a1;
      {
        const mx_u2 uw = pu[w0 - t], vw = pv[w0 - t], us = mx_split(uw.x, uw.y), vs = mx_split(vw.x, vw.y);
        const mx_v8i U = mx_codes(j ? us.y : us.x);
        a0 = mx_mma(mx_codes(vs.x), U, mx_v16f{});
        a1 = mx_mma(mx_codes(vs.y), U, mx_v16f{});
      }
#pragma unroll 1
      for (int w = w0 + 1; w < w1; ++w) {
        // every few words: done once each pair to test has a witness
        const int done = w - w0;
        if (done >= 4 && (done & (done - 1)) == 0 &&
            __ballot(((zeros16(a0) | (zeros16(a1) << 16)) & wb) != 0u) == 0ull)
          break;
        if (w >= t + kTileWords) t = stage_tile(V, W, xs, ys, w, lane);
        const mx_u2 uw = pu[w - t], vw = pv[w - t], us = mx_split(uw.x, uw.y), vs = mx_split(vw.x, vw.y);
        const mx_v8i U = mx_codes(j ? us.y : us.x);
        a0 = mx_mma(mx_codes(vs.x), U, a0);
        a1 = mx_mma(mx_codes(vs.y), U, a1);
      }
      fold(j, a0, a1);
    }
  }
  const int empty = V.k - 2 - seen;  // third classes without a vertex
  unsigned okb[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if constexpr (SLACK) {
      // misses + empty <= slack, bit plane by bit plane from the top
      const int room = V.slack - empty;
      unsigned less = 0u, equal = ~0u;
#pragma unroll
      for (int b = kPlanes - 1; b >= 0; --b) {
        const unsigned x = plane[j][b], r = (room >> b) & 1 ? ~0u : 0u;
        less |= equal & r & ~x;
        equal &= ~(x ^ r);
      }
      const unsigned ok = room < 0 ? 0u : less | equal;
      okb[0][j] = ok & 0xffffu;
      okb[1][j] = ok >> 16;
    } else {
      okb[0][j] = empty > 0 ? 0u : mx_pack_halves(m[j][0]);
      okb[1][j] = empty > 0 ? 0u : mx_pack_halves(m[j][1]);
    }
  }
  return mx_columns(okb, lane);
}

// The same for up to 2 * 64 pairs, one per lane and turn: a word costs two
// LDS reads and a few instructions, where the product takes all 4096 pairs.
__device__ __forceinline__ unsigned long long tile_pairs(const GView &V, const BatchLds &S, int X, int Y, int lane,
                                                         unsigned long long want, TileRows &W) {
  const int cx = uni(S.bcls[X]), cy = uni(S.bcls[Y]);
  const int xs = uni(S.bstart[X]), ys = uni(S.bstart[Y]);
  // the pairs listed in the rows' place, then two in registers.  The list's type
  // may alias the words', and fences keep its reads and writes between theirs: a
  // wave barrier alone orders no memory.
  typedef unsigned short __attribute__((may_alias)) Pair;
  Pair *list = (Pair *)W.u;
  const int cnt = __popcll(want);
  int at = cnt;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int x = __shfl_up(at, off, kWave);
    if (lane >= off) at += x;
  }
  const int total = __builtin_amdgcn_readlane(at, kWave - 1);
  at -= cnt;
  wave_order();
  for (unsigned long long x = want; x; x &= x - 1) list[at++] = (Pair)(lane << 6 | __builtin_ctzll(x));
  wave_order();
  const bool have0 = lane < total, have1 = lane + kWave < total;
  const int p0 = have0 ? list[lane] : 0, p1 = have1 ? list[lane + kWave] : 0;
  wave_order();
  const bool more = total > kWave;
  const unsigned long long *u0 = W.u[p0 >> 6], *v0 = W.v[p0 & 63], *u1 = W.u[p1 >> 6], *v1 = W.v[p1 & 63];
  int t = -kTileWords, miss0 = 0, miss1 = 0, seen = 0;
#pragma unroll 1
  for (int c = 0; c < V.k; ++c) {
    const int w0 = uni(S.soff[c]), w1 = uni(S.soff[c + 1]);
    if (c == cx || c == cy || w0 == w1) continue;
    ++seen;
    unsigned long long wit0 = have0 ? 0ull : 1ull, wit1 = have1 ? 0ull : 1ull;
#pragma unroll 1
    for (int w = w0; w < w1; ++w) {
      if (w >= t + kTileWords) t = stage_tile(V, W, xs, ys, w, lane);
      wit0 |= u0[w - t] & v0[w - t];
      if (more) wit1 |= u1[w - t] & v1[w - t];
      if (__ballot(wit0 == 0ull || wit1 == 0ull) == 0ull) break;
    }
    miss0 += wit0 == 0ull;
    miss1 += wit1 == 0ull;
  }
  const int room = V.slack - (V.k - 2 - seen);  // less the third classes without a vertex
  unsigned long long *ok = W.u[0];
  wave_order();
  ok[lane] = ~0ull;
  wave_order();
  if (have0 && miss0 > room) atomicAnd(&ok[p0 >> 6], ~(1ull << (p0 & 63)));
  if (have1 && miss1 > room) atomicAnd(&ok[p1 >> 6], ~(1ull << (p1 & 63)));
  wave_order();
  return ok[lane];
}

__device__ __forceinline__ void tile(const GView &V, BatchLds &S, int X, int Y, bool first, int lane, TileRows &W,
                                     Kept &kept) {
  const int R = V.R;
  const uint64_t *src = V.cur;
  const int xs = uni(S.bstart[X]), xl = uni(S.blen[X]), ys = uni(S.bstart[Y]), yl = uni(S.blen[Y]);
  const unsigned long long ymask = yl == 64 ? ~0ull : ((1ull << yl) - 1);
  const unsigned long long xmask = xl == 64 ? ~0ull : ((1ull << xl) - 1);
  const unsigned long long eu = src[(long long)(xs + min(lane, xl - 1)) * R + Y];
  const unsigned long long ev = src[(long long)(ys + min(lane, yl - 1)) * R + X];
  // the first window, in flight with the loads above (the pairs path's list
  // takes its place and stages again)
  stage_tile(V, W, xs, ys, 0, lane);
  unsigned long long Eu = lane < xl ? eu & ymask : 0ull;  // the edges of row u = lane
  unsigned long long ET = lane < yl ? ev : 0ull;          // and of row v = lane
  const unsigned long long TU = first ? ~0ull : __ballot(lane < xl && tbit(S.tc, xs + lane));
  const unsigned long long TV = first ? ~0ull : __ballot(lane < yl && tbit(S.tc, ys + lane));
  const unsigned long long Pt = Eu & (((TU >> lane) & 1ull) ? ~0ull : TV);
  unsigned long long Pu = Eu;
  const int cnt = wave_sum(__popcll(Pt));
  if (V.k - 2 > V.slack && cnt > 0) {
    kept.eu[lane] = Eu;
    kept.et[lane] = ET;
    kept.pt[lane] = Pt;
    asm volatile("" ::: "memory");  // read back, not kept
    const unsigned long long ok = cnt <= kTilePairs ? tile_pairs(V, S, X, Y, lane, Pt, W)
                                  : V.slack > 0    ? tile_product<true>(V, S, X, Y, lane, kept, W, 0)
                                                   : tile_product<false>(V, S, X, Y, lane, kept, W, 0);
    asm volatile("" ::: "memory");
    Eu = kept.eu[lane];
    ET = kept.et[lane];
    Pu = Eu & ~(kept.pt[lane] & ~ok);
  }
  // transposes: lane v gets bit v of every P(u) (rows u >= xl hold zero) and,
  // in pass 1, of every E(u), to check that the rows are symmetric
  const unsigned long long newET = wave_transpose64(Pu, lane);
  if (first) {
    const unsigned long long trE = wave_transpose64(Eu, lane);
    if (lane < yl && ((trE ^ ET) & xmask)) atomicMax(&S.prio, P_EASYM);
  }
  const bool chU = lane < xl && Eu != Pu;
  const bool chV = lane < yl && (ET & xmask) != newET;
  const unsigned long long bu = __ballot(chU), bv = __ballot(chV);
  if (bu | bv) {
    if (lane < xl) V.nxt[(long long)(xs + lane) * R + Y] = Pu;
    if (lane < yl) V.nxt[(long long)(ys + lane) * R + X] = newET;
    if (chU) atomicOr(&S.tn[(xs + lane) >> 5], 1u << ((xs + lane) & 31));
    if (chV) atomicOr(&S.tn[(ys + lane) >> 5], 1u << ((ys + lane) & 31));
    const int rem = wave_sum(lane < xl ? __popcll(Eu & ~Pu) : 0);
    if (lane == 0) {
      if (bu) atomicOr(&S.btn[X >> 5], 1u << (X & 31));
      if (bv) atomicOr(&S.btn[Y >> 5], 1u << (Y & 31));
      const int at = S.shared ? atomicAdd(&V.J->nchanged, 1) : atomicAdd(&S.nchanged, 1);
      V.changed[at] = X | (Y << kYShift);
      atomicAdd(&S.removed_e, (unsigned long long)rem);
    }
  }
  if (lane == 0 && cnt) atomicAdd(&S.tests, (unsigned long long)cnt);
}

// The workgroup's LDS, reachable from run_items as well as from the kernel.  The
// job's part comes first: its offsets then fit the 16 bits of an LDS
// instruction, where behind the waves' rows each access needs an address
// register (41 registers spilled, 29 with this; batch of 512 graphs with slack
// 8.29 ms, 8.20).
struct BatchShared {
  BatchLds job;
  TileRows rows[NW];
  Kept kept[NW];
};
__device__ __forceinline__ BatchShared &lds() {
  __shared__ BatchShared S;
  return S;
}

// The waves of the workgroup take the items of the claimed run one by one.
// A function of its own: a tile's sums need most of the registers, and next
// to the rest of the kernel the compiler keeps them in scratch memory (27 GB
// of writes a launch of 4096 graphs).
__device__ __attribute__((noinline)) void run_items() {
  BatchLds &S = lds().job;
  const int lane0 = threadIdx.x & 63, wid = uni((int)(threadIdx.x >> 6));
  TileRows &W = lds().rows[wid];
  GView V;
  V.n = uni(S.view.n);
  V.k = uni(S.view.k);
  V.R = uni(S.view.R);
  V.slack = uni(S.view.slack);
  V.cur = uni(S.view.cur);
  V.nxt = uni(S.view.nxt);
  V.colour = uni(S.view.colour);
  V.valive = uni(S.view.valive);
  V.changed = uni(S.view.changed);
  V.items = uni(S.view.items);
  V.J = uni(S.view.J);
  const bool first = uni(S.pass) == uni(S.pass0);
  const int cnt = uni(S.cnt), base = uni(S.base);
  for (;;) {
    // what an item computes from the lane stays inside the loop: hoisted, it
    // goes to scratch memory and back around every tile
    int i = 0, lane = lane0;
    asm volatile("" : "+v"(lane));
    if (lane == 0) i = atomicAdd(&S.next_item, 1);
    i = uni(i);
    if (i >= cnt) break;
    const int it = uni(V.items[base + i]);
    if (it & kVertexItem) {
      // both halves of the item's line of the vertex mask, by this wave
      const int v0 = (it & 0xffff) * kVChunk;
#pragma unroll 1
      for (int h = 0; h < kVChunk; h += kWave) vertex_chunk(V, S, v0 + h, first, lane);
    } else {
      tile(V, S, it & kXMask, (it >> kYShift) & kXMask, first, lane, W, lds().kept[wid]);
    }
  }
  __syncthreads();
}

__device__ void write_result(const BatchArgs &a, int g, const kz_result &r) {
  if (a.session) {
    // the outputs and the result reach memory before the done flag
    a.hres[g] = r;
    release_system();
    __hip_atomic_store(&a.hdone[g], a.jobs[g].ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return;
  }
  a.results[g] = r;
  atomicAdd(a.finished, 1);
}

// Ends job g with an input error (thread 0).
__device__ void fail_job(const BatchArgs &a, int g, int status) {
  kz_result r{};
  r.status = status;
  write_result(a, g, r);
}

// Ends job g after `passes` passes (thread 0).
__device__ void end_job(const BatchArgs &a, const GView &V, int passes) {
  BatchJob *J = V.J;
  const int rounds = ald(&J->rounds);
  const long long m = ald(&J->m);
  kz_result r{};
  r.status = 0;
  r.rounds = rounds;
  r.equals_input = rounds == 0;
  r.passes = passes;
  r.surviving_vertices = V.n - ald(&J->tot_removed_v);
  r.surviving_edges = m - ald(&J->tot_removed_e);
  r.input_edges = m;
  r.edge_tests = ald(&J->tot_tests);
  write_result(a, V.g, r);
}

// Lists the items of pass S.pass (the touched sets are in S.tc / S.btc) and
// opens it: solo (the whole list is this workgroup's run) or shared
// (published, this workgroup's first run taken).  Returns false when the
// pass has nothing to test: the job is then finished.
__device__ bool open_pass(const BatchArgs &a, const GView &V, BatchLds &S) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int n = V.n, R = V.R, p = S.pass;
  const int nw = (n + 31) >> 5, nbw = (R + 31) >> 5;
  if (tid == 0) {
    S.nitems = 0;
    // every pass number this job uses, the final empty one included: the
    // workgroup that ends the job keeps it in S.pass, and the slot's next
    // job must number its passes above it
    ast(&V.J->lastpass, p);
  }
  __syncthreads();
  // vertex chunks (128 vertices, four touched words) holding a touched vertex
  const int nvc = (n + kVChunk - 1) / kVChunk;
  for (int c0 = wid * kWave; c0 < nvc; c0 += NW * kWave) {
    const int c = c0 + lane;
    bool want = false;
    if (c < nvc) {
      unsigned t = 0;
#pragma unroll
      for (int j = 0; j < kVChunk / 32; ++j) t |= 4 * c + j < nw ? S.tc[4 * c + j] : 0u;
      want = t != 0u;
    }
    const unsigned long long b = __ballot(want);
    int at = 0;
    if (lane == 0 && b) at = atomicAdd(&S.nitems, __popcll(b));
    at = __builtin_amdgcn_readfirstlane(at);
    if (want) V.items[at + __popcll(b & lanes_below(lane))] = kVertexItem | c;
  }
  // tiles of two classes with a touched block: a wave takes kStrip rows X,
  // lanes over them and 64 / kStrip columns Y
  for (int X0 = kStrip * wid; X0 < R; X0 += kStrip * NW) {
    const int X = X0 + (lane & (kStrip - 1));
    const int cx = X < R ? S.bcls[X] : -1;
    const bool tx = X < R && tbit(S.btc, X);
    for (int y0 = X0 + 1; y0 < R; y0 += kWave / kStrip) {
      const int Y = y0 + lane / kStrip;
      const bool want = X < Y && Y < R && S.bcls[min(Y, R - 1)] != cx && (tx || tbit(S.btc, min(Y, R - 1)));
      const unsigned long long b = __ballot(want);
      int at = 0;
      if (lane == 0 && b) at = atomicAdd(&S.nitems, __popcll(b));
      at = __builtin_amdgcn_readfirstlane(at);
      if (want) V.items[at + __popcll(b & lanes_below(lane))] = X | (Y << kYShift);
    }
  }
  __syncthreads();
  const int ni = S.nitems;
  if (ni == 0) {
    if (tid == 0) end_job(a, V, p - S.pass0 + 1);
    __syncthreads();
    return false;
  }
  if (tid == 0) {
    bool shared = a.share == 1;
    if (a.share == 0 && ni > NW)
      shared = ni >= kShareBig || (p - S.pass0) * ni >= kShareWork ||
               (a.session ? ald(a.squeue) >= ald(a.dhead) : ald(a.queue) >= a.G);
    S.shared = shared;
    S.base = 0;
    S.cnt = shared ? min(ni, NW) : ni;
    S.next_item = 0;
    S.nchanged = 0;
    S.got = 1;
    if (shared) {
      BatchJob *J = V.J;
      ast(&J->removed_v, 0ull);
      ast(&J->removed_e, 0ull);
      ast(&J->tests, 0ull);
      ast(&J->prio, 0);
      ast(&J->nchanged, 0);
      ast(&J->done, 0u);
    }
  }
  __syncthreads();
  if (S.shared) {
    BatchJob *J = V.J;
    for (int i = tid; i < nw; i += NW * kWave) {
      ast(&J->touched[p & 1][i], S.tc[i]);
      ast(&J->touched[(p + 1) & 1][i], 0u);
    }
    for (int i = tid; i < nbw; i += NW * kWave) {
      ast(&J->btouched[p & 1][i], S.btc[i]);
      ast(&J->btouched[(p + 1) & 1][i], 0u);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      const unsigned long long cw = ((unsigned long long)p << (2 * kItemBits)) |
                                    ((unsigned long long)ni << kItemBits) | (unsigned long long)S.cnt;
      release_agent();
      __hip_atomic_exchange(&J->claim, cw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.board[V.g & a.board_mask], V.g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  return true;
}

// Sets up graph g (validation, layout, state) and opens its first pass.
// Returns false when the graph needs no pass (error, empty graph).
__device__ bool start_job(const BatchArgs &a, BatchLds &S, int g) {
  const int tid = threadIdx.x;
  if (a.session) {
    if (tid == 0) {
      BatchJob *J = a.jobs + g;
      J->sdesc = a.hgraphs[g];
      J->sptrs = a.hptrs[g];
      J->ticket = S.ticket;
    }
    __syncthreads();
  }
  const kz_batch_graph G = job_desc(a, g);
  const int n = G.n, k = G.k, R = G.row_words;
  int st = 0;
  if (n < 0 || k < 1 || R < 0 || G.clique < 0 || G.clique > k ||
      (!a.ptrs && !a.session && (G.row_offset < 0 || G.vertex_offset < 0)))
    st = KZ_EINVAL;
  else if (k > kBatchK || R > kBatchR || n > kBatchN) st = kBatchTooLarge;
  if (st != 0 || n == 0) {
    if (tid == 0) {
      if (st) {
        fail_job(a, g, st);
      } else {
        kz_result r{};
        r.equals_input = 1;
        write_result(a, g, r);
      }
    }
    return false;
  }
  const GView V = gview(a, g);
  // layout: colours are sorted class by class; class c starts at the first
  // vertex whose colour is >= c (binary search)
  // the layout copies in LDS are about to be overwritten: they no longer
  // belong to the job named in S.job (a later claim must reload them)
  if (tid == 0) {
    S.bad_colour = 0;
    S.bad_layout = 0;
    S.job = -1;
  }
  __syncthreads();
  for (int v = tid; v < n; v += NW * kWave) {
    const int c = V.colour[v];
    if (c < 0 || c >= k) S.bad_colour = 1;
    else if (v > 0 && V.colour[v - 1] > c) S.bad_layout = 1;
  }
  __syncthreads();
  if (S.bad_colour | S.bad_layout) {
    if (tid == 0) fail_job(a, g, S.bad_colour ? KZ_ECOLOUR : KZ_EINVAL);
    __syncthreads();
    return false;
  }
  for (int c = tid; c <= k; c += NW * kWave) {
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (V.colour[mid] < c) lo = mid + 1;
      else hi = mid;
    }
    S.coff[c] = lo;
  }
  __syncthreads();
  if (tid == 0) {
    int w = 0;
    for (int c = 0; c < k; ++c) {
      S.soff[c] = w;
      const int s = S.coff[c + 1] - S.coff[c];
      for (int b = 0; 64 * b < s && w + b < kBatchR; ++b) {
        S.bcls[w + b] = (short)c;
        S.bstart[w + b] = (unsigned short)(S.coff[c] + 64 * b);
        S.blen[w + b] = (unsigned char)min(64, s - 64 * b);
      }
      w += (s + 63) / 64;
    }
    S.soff[k] = w;
    if (w != R) S.bad_layout = 1;
  }
  __syncthreads();
  if (S.bad_layout) {
    if (tid == 0) fail_job(a, g, KZ_EINVAL);
    __syncthreads();
    return false;
  }
  // the layout goes to the job too (helpers load it from there)
  BatchJob *J = V.J;
  for (int c = tid; c <= k; c += NW * kWave) {
    J->coff[c] = S.coff[c];
    J->soff[c] = S.soff[c];
  }
  for (int b = tid; b < R; b += NW * kWave) {
    J->bcls[b] = S.bcls[b];
    J->bstart[b] = S.bstart[b];
    J->blen[b] = S.blen[b];
  }
  // state: the rows, every vertex and block touched
  for (long long i = tid; i < (long long)n * R; i += NW * kWave) V.cur[i] = V.rows[i];
  for (int i = tid; i < kBatchN / 32; i += NW * kWave) {
    S.tc[i] = ~0u;
    S.tn[i] = 0;
  }
  for (int i = tid; i < kBatchR / 32; i += NW * kWave) {
    S.btc[i] = ~0u;
    S.btn[i] = 0;
  }
  if (tid == 0) {
    ast(&J->rounds, 0);
    ast(&J->tot_removed_v, 0ll);
    ast(&J->tot_removed_e, 0ll);
    ast(&J->tot_tests, 0ll);
    ast(&J->m, 0ll);
    int p0 = 1;
    if (a.session) {
      // above every pass number a workgroup may still hold for this slot
      // (after the wrap, numbers from over 2^23 passes ago: a launch ends
      // within its lease, and with it every copy in LDS, long before that)
      p0 = ald(&J->lastpass) + 1;
      if (p0 >= (1 << 23)) p0 = 1;
    }
    ast(&J->pass0, p0);
    ast(&J->lastpass, p0);
    S.job = g;
    S.pass = p0;
    S.pass0 = p0;
    S.prio = 0;
    S.removed_v = 0;
    S.removed_e = 0;
    S.tests = 0;
  }
  __syncthreads();
  return open_pass(a, V, S);
}

// Claims a run of unclaimed items of job g (thread 0; S.got = 0: none left).
// A workgroup joining a pass it did not list loads the job's layout and
// touched sets after an acquire fence.
__device__ void claim(const BatchArgs &a, BatchLds &S, int g) {
  const int tid = threadIdx.x;
  BatchJob *J = a.jobs + g;
  // Every wave enters on S.got == 0, read after the previous barrier; thread
  // 0 rewrites S.got below, so it waits until each wave has made that read
  // (a late wave would otherwise see the new value, skip this function and
  // its barriers, and stay one barrier out of step with the others).
  __syncthreads();
  if (tid == 0) {
    unsigned long long old = __hip_atomic_load(&J->claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int got = 0, cp = 0;
    for (int tries = 0; tries < 64; ++tries) {
      const unsigned ni = (unsigned)(old >> kItemBits) & kItemMask, nx = (unsigned)old & kItemMask;
      if (nx >= ni) break;
      // guided run length: a share of what is left, between 2*NW and 8*NW
      // items (joining and reporting a run cost about as much as its tiles:
      // runs of NW items took 2.5 ms for 64 graphs and 10.9 for 1024, of 2*NW
      // 2.2 and 9.9; with 3*NW or 4*NW the cascades of 4096 take longer again)
      const unsigned rem = ni - nx;
      const unsigned c = min(rem, max(2u * NW, min(8u * NW, rem / (2u * gridDim.x))));
      if (__hip_atomic_compare_exchange_strong(&J->claim, &old, old + c, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT)) {
        got = 1;
        cp = (int)(old >> (2 * kItemBits));
        S.base = (int)nx;
        S.cnt = (int)c;
        S.nitems = (int)ni;
        break;
      }
    }
    S.reload = 0;
    if (got) {
      if (!(S.job == g && S.pass == cp)) {
        acquire_agent();  // the pass was listed by another workgroup
        // a new job in the slot has another first pass: its layout differs
        const int p0 = ald(&J->pass0);
        S.reload = S.job != g || S.pass0 != p0 ? 2 : 1;
        S.pass0 = p0;
        S.job = g;
        S.pass = cp;
        S.shared = 1;
      }
      S.next_item = 0;
    }
    S.got = got;
  }
  __syncthreads();
  if (S.got && S.reload) {
    const kz_batch_graph G = job_desc(a, g);
    const int p = S.pass, nw = (G.n + 31) >> 5, nbw = (G.row_words + 31) >> 5;
    if (S.reload == 2) {
      for (int c = tid; c <= G.k; c += NW * kWave) {
        S.coff[c] = J->coff[c];
        S.soff[c] = J->soff[c];
      }
      for (int b = tid; b < G.row_words; b += NW * kWave) {
        S.bcls[b] = J->bcls[b];
        S.bstart[b] = J->bstart[b];
        S.blen[b] = J->blen[b];
      }
    }
    for (int i = tid; i < nw; i += NW * kWave) {
      S.tc[i] = ald(&J->touched[p & 1][i]);
      S.tn[i] = 0;
    }
    for (int i = tid; i < nbw; i += NW * kWave) {
      S.btc[i] = ald(&J->btouched[p & 1][i]);
      S.btn[i] = 0;
    }
    if (tid == 0) {
      S.prio = 0;
      S.removed_v = 0;
      S.removed_e = 0;
      S.tests = 0;
    }
    __syncthreads();
  }
}

// Reports a finished run.  Solo: the run was the pass.  Shared: merge the
// run's counts and touched bits into the job, then count the run's items
// done; the run that completes the pass returns true, after an acquire
// fence.
__device__ bool retire(const GView &V, BatchLds &S) {
  const int tid = threadIdx.x;
  if (!S.shared) {
    if (tid == 0) S.got = 0;
    __syncthreads();
    return true;
  }
  BatchJob *J = V.J;
  const int tnx = (S.pass + 1) & 1;
  const int nw = (V.n + 31) >> 5, nbw = (V.R + 31) >> 5;
  for (int i = tid; i < nw; i += blockDim.x) {
    const unsigned x = S.tn[i];
    if (x) {
      atomicOr(&J->touched[tnx][i], x);
      S.tn[i] = 0;
    }
  }
  for (int i = tid; i < nbw; i += blockDim.x) {
    const unsigned x = S.btn[i];
    if (x) {
      atomicOr(&J->btouched[tnx][i], x);
      S.btn[i] = 0;
    }
  }
  if (tid == 0) {
    if (S.removed_v) atomicAdd(&J->removed_v, S.removed_v);
    if (S.removed_e) atomicAdd(&J->removed_e, S.removed_e);
    if (S.tests) atomicAdd(&J->tests, S.tests);
    if (S.prio) atomicMax(&J->prio, S.prio);
    S.removed_v = 0;
    S.removed_e = 0;
    S.tests = 0;
    S.prio = 0;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
    const unsigned add = (unsigned)S.cnt;
    release_agent();
    const unsigned now = __hip_atomic_fetch_add(&J->done, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
    S.last = (int)now == S.nitems;
    // acquire what the other workgroups wrote (and drop this CU's cached
    // copies of the job's merged state)
    if (S.last) acquire_agent();
    S.got = 0;
  }
  __syncthreads();
  return S.last;
}

// The carrier: applies the changed tiles, closes the pass, and ends the job
// or opens the next pass.  Returns true when a next pass is open.
__device__ bool carry(const BatchArgs &a, const GView &V, BatchLds &S) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  BatchJob *J = V.J;
  const int p = S.pass, R = V.R;
  const int nw = (V.n + 31) >> 5, nbw = (R + 31) >> 5;
  if (S.shared) {
    const int tnx = (p + 1) & 1;
    for (int i = tid; i < nw; i += NW * kWave) S.tn[i] = ald(&J->touched[tnx][i]);
    for (int i = tid; i < nbw; i += NW * kWave) S.btn[i] = ald(&J->btouched[tnx][i]);
    if (tid == 0) {
      S.removed_v = ald(&J->removed_v);
      S.removed_e = ald(&J->removed_e);
      S.tests = ald(&J->tests);
      S.prio = ald(&J->prio);
      S.nchanged = ald(&J->nchanged);
    }
    __syncthreads();
  }
  // apply: copy the changed tiles into the state
  const int nch = S.nchanged;
  for (int i = wid; i < nch; i += NW) {
    const int it = V.changed[i];
    const int X = it & kXMask, Y = (it >> kYShift) & kXMask;
    const int xs = S.bstart[X], xl = S.blen[X], ys = S.bstart[Y], yl = S.blen[Y];
    if (lane < xl) V.cur[(long long)(xs + lane) * R + Y] = V.nxt[(long long)(xs + lane) * R + Y];
    if (lane < yl) V.cur[(long long)(ys + lane) * R + X] = V.nxt[(long long)(ys + lane) * R + X];
  }
  if (tid == 0) {
    const long long rv = (long long)S.removed_v, re = (long long)S.removed_e;
    S.status = 0;
    if (p == S.pass0 && S.prio)
      S.status = S.prio == P_EINVAL      ? KZ_EINVAL
                 : S.prio == P_ESELFLOOP ? KZ_ESELFLOOP
                 : S.prio == P_EASYM     ? KZ_EASYM
                                         : KZ_EILLEGAL;
    if (p == S.pass0) ast(&J->m, (long long)S.tests);
    ast(&J->tot_tests, ald(&J->tot_tests) + (long long)S.tests);
    ast(&J->tot_removed_v, ald(&J->tot_removed_v) + rv);
    ast(&J->tot_removed_e, ald(&J->tot_removed_e) + re);
    if (!S.status && rv + re > 0) ast(&J->rounds, ald(&J->rounds) + 1);
    S.end = S.status != 0 || rv + re == 0;
  }
  __syncthreads();
  if (S.end) {
    if (tid == 0) {
      if (S.status) fail_job(a, V.g, S.status);
      else end_job(a, V, p - S.pass0 + 1);
    }
    __syncthreads();
    return false;
  }
  // next pass: what this pass touched is what the next one tests
  for (int i = tid; i < kBatchN / 32; i += NW * kWave) {
    S.tc[i] = i < nw ? S.tn[i] : 0u;
    S.tn[i] = 0;
  }
  for (int i = tid; i < kBatchR / 32; i += NW * kWave) {
    S.btc[i] = i < nbw ? S.btn[i] : 0u;
    S.btn[i] = 0;
  }
  if (tid == 0) {
    S.pass = p + 1;
    S.prio = 0;
    S.removed_v = 0;
    S.removed_e = 0;
    S.tests = 0;
  }
  __syncthreads();
  return open_pass(a, V, S);
}

// Looks on the board for the shared pass with the most unclaimed items, if
// it has at least `least` of them; -1 otherwise.
__device__ int find_job(const BatchArgs &a, BatchLds &S, unsigned least) {
  const int tid = threadIdx.x;
  if (tid < kWave) {
    unsigned long long key = 0;
    // kBatchBoard entries per step: their loads, then their claim words', in flight together
    for (int base = 0; base <= a.board_mask; base += kBatchBoard) {
      int gs[kBatchBoard / kWave];
#pragma unroll
      for (int j = 0; j < kBatchBoard / kWave; ++j)
        gs[j] = __hip_atomic_load(&a.board[base + j * kWave + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int j = 0; j < kBatchBoard / kWave; ++j) {
        if (gs[j] < 0) continue;
        const unsigned long long cw =
            __hip_atomic_load(&a.jobs[gs[j]].claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned ni = (unsigned)(cw >> kItemBits) & kItemMask, nx = (unsigned)cw & kItemMask;
        if (nx < ni && ni - nx >= least)
          key = max(key, ((unsigned long long)(ni - nx) << 32) | (unsigned)(gs[j] + 1));
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long o = (unsigned long long)__shfl_xor((long long)key, off, kWave);
      key = max(key, o);
    }
    if (tid == 0) S.pick = key ? (int)(key & 0xffffffffu) - 1 : -1;
  }
  __syncthreads();
  return S.pick;
}

// Session mode (thread 0): refreshes the device's copies of the host's
// request count and of the launch it asked to end.  They live in pinned host memory; one workgroup at a
// time reads them, at most every kHostPoll ticks.
__device__ void poll_host(const BatchArgs &a) {
  const unsigned long long now = wall_clock64();
  unsigned long long last = ald(a.hpoll);
  if (now - last < kHostPoll || !__hip_atomic_compare_exchange_strong(a.hpoll, &last, now, __ATOMIC_RELAXED,
                                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    return;
  const unsigned long long hh = __hip_atomic_load(a.head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  const unsigned long long hy = __hip_atomic_load(a.head + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  // the copy is written after the count's load has returned (it is the
  // operand); a taker's own acquire orders its reads of the host tables
  if (hh > ald(a.dhead)) __hip_atomic_fetch_max(a.dhead, hh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (hy > ald(a.dhead + 1)) __hip_atomic_fetch_max(a.dhead + 1, hy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Session mode (thread 0): takes the next published request, if any, and
// returns its slot (S.ticket: its ticket), else -1.
__device__ int take_request(const BatchArgs &a, BatchLds &S) {
  poll_host(a);
  unsigned long long h = ald(a.dhead), q = ald(a.squeue);
  while (q < h) {
    if (__hip_atomic_compare_exchange_strong(a.squeue, &q, q + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT)) {
      acquire_system();
      unsigned *e = a.ring + q % (unsigned long long)a.cap;
      unsigned slot = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      // the host wrote the entry before the count; should the entry still
      // read as free, look again for a while rather than take a bad slot
      for (int i = 0; i < 4096 && slot >= (unsigned)a.G; ++i) {
        __builtin_amdgcn_s_sleep(8);
        acquire_system();
        slot = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
      if (slot >= (unsigned)a.G) return -1;  // never observed: the request stays untaken for good
      S.ticket = __hip_atomic_load(a.htickets + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      // the host may write the entry again once it sees it read
      __hip_atomic_store(e, kRingFree, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      return (int)slot;
    }
  }
  return -1;
}

__global__ void __launch_bounds__(NW * 64, 4) k_batch(BatchArgs a) {
  BatchLds &S = lds().job;
  const int tid = threadIdx.x;
  if (tid == 0) {
    S.job = -1;
    S.pass = 0;
    S.pass0 = 0;
    S.got = 0;
    S.queue_empty = 0;
  }
  __syncthreads();
  int job = -1;
  const unsigned long long born = wall_clock64();  // session mode: the lease runs from here
  unsigned long long idle0 = 0;  // thread 0: when this workgroup ran out of work
  int backoff = 1;                // idle polls sleep 1, 2, 4 or 8 times between looks
  for (;;) {
    if (job >= 0) {
      if (!S.got) claim(a, S, job);
      if (S.got) {
        const GView V = gview(a, job);
        if (tid == 0) S.view = V;
        __syncthreads();
        run_items();
        if (retire(V, S) && !carry(a, V, S)) job = -1;
        continue;
      }
      job = -1;
    }
    // a shared pass with plenty of unclaimed items comes before a new graph
    if (!S.queue_empty) {
      job = find_job(a, S, 2u * NW);
      if (job >= 0) continue;
      __syncthreads();
      if (tid == 0) {
        if (a.session) {
          // past its lease a workgroup takes no new request, so the launch
          // ends and kernels queued behind it on the same hardware queue run
          const bool leased = a.lease_ticks && wall_clock64() - born > a.lease_ticks;
          S.gi = leased ? -1 : take_request(a, S);
        } else {
          const int t = atomicAdd(a.queue, 1);
          S.gi = t < a.G ? a.order[t] : -1;
          if (t >= a.G) S.queue_empty = 1;
        }
      }
      __syncthreads();
      const int g = S.gi;
      if (g >= 0) {
        if (start_job(a, S, g)) job = g;
        idle0 = 0;
        backoff = 1;
        continue;
      }
    }
    job = find_job(a, S, 1u);
    if (job >= 0) {
      idle0 = 0;
      backoff = 1;
      continue;
    }
    if (tid == 0) {
      const unsigned long long now = wall_clock64();
      if (!idle0) idle0 = now;
      // a session's workgroups stay for new requests until idle for idle_ticks
      // or, once the host has asked this launch to end, until idle
      S.quit = a.session ? now - idle0 > a.idle_ticks || (a.lease_ticks && now - born > a.lease_ticks) ||
                               ald(a.dhead + 1) >= a.launch
                         : __hip_atomic_load(a.finished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= a.G ||
                               now - idle0 > kIdleTicks;
    }
    __syncthreads();
    if (S.quit) break;
    // back off while idle: every look at the board is a few KiB of loads
    // that bypass the caches, and hundreds of idle workgroups looking at
    // once slow down the ones still working
    for (int i = 0; i < backoff; ++i) __builtin_amdgcn_s_sleep(32);
    backoff = backoff < 8 ? 2 * backoff : 8;
  }
}

// Estimates the time every graph keeps a workgroup (one wave per graph) into
// order[g], for k_batch_order: the passes to expect times what a pass takes
// (its fixed part is worth about 30 tiles).  The passes follow from the
// edges' density d, taken from kCostRows rows, and the class sizes: lam = the
// sum over the third classes of (1 - d^2)^s is how many classes an edge is
// expected to find no witness in.  Of 4096 graphs of 4..16 classes of 8..128
// vertices, p = 0.2..0.8, those with lam in 0.03 .. 0.3 run 8 to 16 passes on
// average and up to 119, the others 2 to 7; a long cascade that starts late
// keeps the launch waiting: 18.0 ms in order of size, 15.0 ms in this order,
// 14.7 ms in order of the true number of passes.  lam knows nothing of a clique
// size below the number of classes, where an edge survives that many empty
// ones: 512 such graphs of two less take the same in this order and as given
// (9.40 and 9.36 ms, 9.65 and 9.63), few graphs for the chip's workgroups.
constexpr int kCostRows = 16;
__global__ void __launch_bounds__(64) k_batch_cost(BatchArgs a) {
  const int g = blockIdx.x, lane = threadIdx.x;
  const kz_batch_graph G = a.graphs[g];
  const int n = G.n, k = G.k, R = G.row_words;
  unsigned cost = 0;
  if (n > 0 && k > 0 && k <= kBatchK && R > 0 && R <= kBatchR && n <= kBatchN && G.row_offset >= 0 &&
      G.vertex_offset >= 0) {
    const uint64_t *rows = a.rows + G.row_offset;
    const int *colour = a.colour + G.vertex_offset;
    int ones = 0;
    for (int w = lane; w < R; w += kWave)
#pragma unroll
      for (int i = 0; i < kCostRows; ++i) ones += __popcll(rows[(long long)(i * n / kCostRows) * R + w]);
    ones = wave_sum(ones);
    // lane c: where class c starts (the colours are sorted)
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (colour[mid] < lane) lo = mid + 1;
      else hi = mid;
    }
    const int next = __shfl_down(lo, 1, kWave);
    const float s = (float)((lane == kWave - 1 ? n : next) - lo);
    const float d = fminf((float)ones / (kCostRows * fmaxf((float)n - (float)n / (float)k, 1.f)), 0.999f);
    float lam = lane < k ? exp2f(s * __log2f(1.f - d * d)) : 0.f;
    for (int off = 32; off > 0; off >>= 1) lam += __shfl_xor(lam, off, kWave);
    lam *= (float)max(k - 2, 0) / (float)k;
    const float passes = lam < 0.01f  ? 3.f
                         : lam < 0.03f ? 6.f
                         : lam < 0.1f  ? 30.f
                         : lam < 0.3f  ? 40.f
                         : lam < 0.4f  ? 20.f
                         : lam < 0.5f  ? 10.f
                                       : 6.f;
    cost = (unsigned)(passes * (30.f + 0.5f * (float)R * (float)(R - 1)));
  }
  if (lane == 0) a.order[g] = (int)cost;
}

// Orders the graphs by their estimated time (`lpt` 2: order[] holds it), or
// by their sizes (1), largest first, so the persistent workgroups finish
// together, or keeps the given order (0); resets the queue, the finished
// count and the board.  One workgroup, bitonic sort in LDS for up to
// kBatchSortMax graphs.
__global__ void __launch_bounds__(1024) k_batch_order(BatchArgs a, int lpt) {
  __shared__ unsigned long long key[kBatchSortMax];
  const int t = threadIdx.x, G = a.G;
  if (t == 0) {
    *a.queue = 0;
    *a.finished = 0;
  }
  for (int i = t; i <= a.board_mask; i += 1024) a.board[i] = -1;
  if (!lpt || G > kBatchSortMax) {
    for (int i = t; i < G; i += 1024) a.order[i] = i;
    return;
  }
  int P = 1;
  while (P < G) P <<= 1;
  for (int i = t; i < P; i += 1024) {
    unsigned long long cost = 0;
    if (i < G) {
      if (lpt == 2) {
        cost = (unsigned)a.order[i];
      } else {
        const kz_batch_graph gg = a.graphs[i];
        const long long R = gg.row_words > 0 ? gg.row_words : 0;
        cost = (unsigned long long)(R * R * 64LL * (gg.k > 2 ? gg.k : 1) + gg.n);
        if (cost > 0xffffffffull) cost = 0xffffffffull;
      }
      key[i] = (~cost << 32) | (unsigned)i;  // ascending key = descending cost
    } else {
      key[i] = ~0ull;
    }
  }
  __syncthreads();
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = t; i < P; i += 1024) {
        const int j = i ^ stride;
        if (j > i) {
          const bool up = (i & size) == 0;
          const unsigned long long x = key[i], y = key[j];
          if ((x > y) == up) {
            key[i] = y;
            key[j] = x;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int i = t; i < G; i += 1024) a.order[i] = (int)(key[i] & 0xffffffffu);
}

}  // namespace

void launch_batch(const BatchArgs &args, const BatchConfig &cfg, hipStream_t s) {
  BatchArgs a = args;
  if (a.board_mask <= 0) a.board_mask = kBatchBoard - 1;
  // a session's queue and board are set up once, when its server is made
  if (!a.session) {
    // the estimate pays where graphs wait for a workgroup
    const bool cost = cfg.lpt && a.G > cfg.workgroups && a.G <= kBatchSortMax;
    if (cost) hipLaunchKernelGGL(k_batch_cost, dim3(a.G), dim3(64), 0, s, a);
    hipLaunchKernelGGL(k_batch_order, dim3(1), dim3(1024), 0, s, a, cost ? 2 : cfg.lpt);
  }
  hipLaunchKernelGGL(k_batch, dim3(cfg.workgroups), dim3(NW * kWave), 0, s, a);
}

}  // namespace kzi
