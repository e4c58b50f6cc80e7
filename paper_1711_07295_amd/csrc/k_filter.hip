// The bitmap filter over the length band -- the hot loop of the join.
//
// For every pair (i, j) of the band it evaluates the overlap bound of
// Theorem 1 (Eq. 2), UB = floor((|r| + |s| - popcount(b_r xor b_s)) / 2),
// and keeps the pair when UB reaches the overlap that the threshold needs
// (Table 1; Alg. 7, as the paper's GPU algorithm, Alg. 8, runs it).  With
// L = |r| + |s| and omin the least overlap that reaches t,
// UB >= omin  <=>  popcount(b_r xor b_s) <= L - 2 omin = slack,
// so each pair costs b/32 xor, b/32 accumulating popcounts and a compare.
//
// Work decomposition (size-ordered rows and columns, Section 2.3.2):
//   - a wave owns 64*R consecutive rows of one task, R per lane, with their
//     bitmaps in VGPRs for the whole tile;
//   - the wave walks the tile's columns in order; every column's bitmap is
//     wave-uniform and is read with scalar loads, one step of U columns
//     ahead, into two alternating register buffers;
//   - columns are swept in runs of one size, or, where the sizes are sparse,
//     of a few (ColRun); at a run's start each lane derives its threshold
//     from the row and column sizes, folding the length filter in (threshold
//     -1 = never kept), and in a run of several sizes the pairs that reach
//     the bound are tested at their own;
//   - the compare is folded into the popcount: the chain starts at
//     -(slack + 1), so a kept pair has a negative sum; the sums of a step's
//     U*R pairs are ORed and one ballot of the sign bit decides whether the
//     wave leaves the fast path to stage the kept (row, column) pairs at
//     their ballot ranks in its LDS buffer, which goes to the queue with one
//     reservation when full and at the end of every tile;
//   - self-join diagonal tiles add the triangle condition j < i.
// A launch starts one wave per tile, or, where it has very many tiles or a lot
// of wide work, persistent waves that take tiles from cursors split per XCD
// (tile_loop).  When the survivor queue is full the wave marks its reserved slots
// as sentinels, records (tile, column, row slab) of its first staged pair to resume
// from, sets the overflow flag and stops; the host verifies the queue and
// relaunches with the resume list.
#include <algorithm>

#include "ssj_internal.h"

namespace ssj {
namespace {

__device__ __forceinline__ uint32_t rfl(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ float rfl(float v) { return __uint_as_float(rfl(__float_as_uint(v))); }

__device__ __forceinline__ unsigned long long rfl64(unsigned long long v) {
  uint32_t lo = rfl((uint32_t)v), hi = rfl((uint32_t)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

// The launch's arguments, read from the kernel argument segment where they
// are used: the pointer is made opaque, so that no argument is kept in
// scalar registers across the sweeps (kept ones filled all 106 and spilled
// into vector registers, which set the waves per SIMD).
typedef const __attribute__((address_space(4))) FilterArgs *ArgPtr;

__device__ __forceinline__ ArgPtr args() {
  ArgPtr a = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

// Uniform data that is not written while the kernel runs (column bitmaps,
// sizes, group starts, the plan) is read through the constant address space:
// uniform loads from it always become scalar loads (s_load), whatever the
// slow path stores.
typedef const __attribute__((address_space(4))) uint32_t *const_u32_ptr;

template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_const(const T *p) {
  return (const __attribute__((address_space(4))) T *)(p);
}

// Index of this wave in the launch: workgroups of four waves, or of one in a
// direct launch.
__device__ __forceinline__ uint32_t wave_index() {
  return rfl(blockIdx.x * args()->cfg.block_waves + (threadIdx.x >> 6));
}

// A run of columns [j, end) of sizes lo .. hi that one sweep takes: one size
// group, or, where a group has fewer than kRunCols columns (the sparse tail
// of the size distribution), the groups of sizes up to lo + lo / 32 with
// it.  Every run starts with a chain of dependent loads (size, group starts,
// thresholds, first columns) of a few microseconds that its few steps
// cannot hide: with a run per group, a tile of a few hundred columns of
// 200 .. 500 tokens took 200 us and its launch waited for it.
//
// A run of several sizes is tested against the loosest of its thresholds: the
// slack a + c - 2 omin(a, c) falls nowhere by more than 1 as c grows inside
// the length band (omin is the ceiling of something that grows by at most
// 1/2 per token there), so slack(a, hi) + 1 bounds them.  The pairs it
// lets through are then tested at their own sizes.
struct ColRun {
  uint32_t lo, hi, end;
};
constexpr uint32_t kRunCols = 64;

__device__ __forceinline__ ColRun col_run(const_u32_ptr sstart, uint32_t col_base,
                                          uint32_t max_size, uint32_t c, uint32_t j, uint32_t c1) {
  const uint32_t wide = min(c + (c >> kRunShift), max_size);
  const uint32_t e1 = col_base + sstart[c + 1], e2 = col_base + sstart[wide + 1];
  const bool several = e1 < j + kRunCols && wide > c;
  ColRun r;
  r.lo = c;
  r.hi = several ? wide : c;
  // no more of the wider sizes than fill the run: a group that is long enough
  // gets its own threshold
  r.end = min(max(several ? min(e2, j + kRunCols) : e1, j + 1), c1);  // advances
  return r;
}

template <int W, int R>
struct Rows {
  uint32_t bits[R][2 * W];
  uint32_t size[R];
  uint32_t cmn[R];
  uint32_t cmx[R];
  uint32_t idx[R];
};

// Kept pairs are staged per wave in LDS and written to the queue in runs.
// Queue slots come from a chunk the wave reserves for itself (cfg.chunk
// slots per reservation), so reservations are few: same-address atomics
// from every XCD serialise at the memory side, and one per run would cost
// more than the filter.  A run never spans tiles, so the first staged entry
// always names a point of the current tile.  The unused end of a chunk is
// filled with sentinels (verification skips them) when the wave takes a
// new chunk and when it exits.
constexpr uint32_t kStage = kFilterStage;

// Two columns per accumulator: a wave's rows, at most, and its LDS words for their
// sizes, bands and bitmaps and for a step's 64 column sizes and bitmaps.
constexpr int kTwoRows = 192;
constexpr int kTwoWords = 5 * kTwoRows + 3 * 64;
constexpr int kMaxRowTiles = 6;

struct Sink {
  uint2 *stage;                // this wave's kStage LDS entries
  uint32_t *kept;              // ... kept values of a step, 64 words per row tile (matrix cores)
  uint32_t *rows;              // ... and kTwoWords words (two columns per accumulator)
                               // or 1024 16-bit dot products (matrix cores otherwise)
  uint32_t fill;               // entries staged (wave-uniform)
  uint32_t first_col;          // (column, row slab) of the first staged entry
  uint32_t first_slab;
  uint32_t first_end;          // end of the run of columns of that entry's step (matrix cores)
  uint32_t fail_col;           // resume point, set when the queue fills
  uint32_t fail_slab;
  uint32_t fail_end;
  uint32_t stripe;             // the wave's stripe of the queue
  uint32_t pos, end;           // the wave's reserved slots [pos, end) of that stripe
};

// Sentinels into the rest of the wave's chunk.
__device__ __forceinline__ void sink_pad(Sink &s) {
  const ArgPtr a = args();
  const uint32_t lane = threadIdx.x & 63;
  uint2 *q = a->queue + (unsigned long long)s.stripe * a->cfg.cap;
  for (uint32_t x = s.pos + lane; x < s.end; x += 64) q[x] = make_uint2(kSentinel, kSentinel);
  s.pos = s.end;
}

// `want` slots of the wave's stripe, or of the first stripe after it that
// holds `need` of them; what a full stripe had left becomes sentinels.
// False when no stripe has room.
__device__ __forceinline__ bool reserve(Sink &s, uint32_t want, uint32_t need) {
  const ArgPtr a = args();
  const uint32_t lane = threadIdx.x & 63, stripes = a->cfg.stripes, cap = a->cfg.cap;
  JoinCounters *ctr = a->ctr;
  for (uint32_t k = 0; k < stripes; ++k) {
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&ctr->queue_next[s.stripe][0], (unsigned long long)want);
    base = rfl64(base);
    s.pos = base < cap ? (uint32_t)base : cap;
    s.end = base + want < cap ? (uint32_t)base + want : cap;
    if (s.pos + need <= s.end) return true;
    sink_pad(s);
    s.stripe = (s.stripe + 1) & (stripes - 1);
  }
  return false;
}

// Copy the staged entries into the wave's chunk, reserving a new chunk
// when they do not fit in the current one (in a direct launch the tile's
// last run, which ends the wave, reserves only the slots it takes).  When
// the queue has no room for them, the reserved slots become sentinels, the
// first staged entry's point is left as the resume point and false is
// returned: every pair before that point is in the queue, none after it.
__device__ __forceinline__ bool flush(Sink &s, bool last = false) {
  const uint32_t n = rfl(s.fill);
  if (n == 0) return true;
  const ArgPtr a = args();
  const uint32_t lane = threadIdx.x & 63;
  if (s.pos + n > s.end) {
    sink_pad(s);
    if (!reserve(s, last && a->cfg.direct ? n : a->cfg.chunk, n)) {
      s.fill = 0;
      s.fail_col = s.first_col;
      s.fail_slab = s.first_slab;
      s.fail_end = s.first_end;
      return false;
    }
  }
  uint2 *q = a->queue + (unsigned long long)s.stripe * a->cfg.cap;
  __builtin_amdgcn_wave_barrier();
  for (uint32_t x = lane; x < n; x += 64) q[s.pos + x] = s.stage[x];
  __builtin_amdgcn_wave_barrier();
  s.pos += n;
  s.fill = 0;
  return true;
}

// What a wave needs to run one tile.
struct TileJob {
  uint32_t row0, row_end, c0, c1;
  bool diag;
  uint32_t first;  // resumed inside the tile: first slab (vector ALU) or pairs to skip (MFMA)
  uint32_t end;    // ... and the end of the step's run (MFMA), else 0
  const int32_t *slack;
  const uint32_t *cmin, *cmax;
  const_u32_ptr sstart;
  uint32_t col_base, col_max;  // first column and largest size of the column space
  uint32_t task;
  bool cosine;
  uint32_t p, q;
  float t;         // p / q
};

// A task's exact test.  With Cosine among the call's functions it is read again where it
// is used at 2048 bits and more (AGAIN): kept across the vector-ALU sweeps, its fields
// take scalar registers from the columns' buffers there (231 instructions a column
// against 217).  A class of 640 bits takes 0.25 ms with them kept and 0.27 without.
struct PairTest {
  const int32_t *slack;
  bool cosine;
  uint32_t p, q;
};
template <bool AGAIN>
__device__ __forceinline__ PairTest pair_test(const TileJob &jb) {
  if constexpr (!AGAIN) return PairTest{jb.slack, jb.cosine, jb.p, jb.q};
  const ArgPtr a = args();
  const auto *td = as_const(a->tasks) + jb.task;
  return PairTest{reinterpret_cast<const int32_t *>(a->tables + td->slack_off),
                  td->sim == SSJ_SIM_COSINE, td->p, td->q};
}

// Largest slack a + c' - 2 omin(a, c') a row of size a can have with a column of
// size c' in [lo, hi], all inside the band: exact for lo == hi, else at most
// 1 above slack(a, hi) (see ColRun).  Cosine's least overlap, the ceiling of
// t sqrt(a c), is bounded below in single precision (relative error of the
// three roundings and the root below 1e-6), so its slack is always a bound;
// the slow path decides each pair.
template <bool COS>
__device__ __forceinline__ int32_t run_slack(const TileJob &jb, uint32_t a, uint32_t lo,
                                             uint32_t hi) {
  const int32_t more = hi > lo ? 1 : 0;
  if (COS && jb.cosine) {
    const float x = jb.t * sqrtf((float)a * (float)hi) * (1.0f - 1.0e-6f);
    return (int32_t)(a + hi) - 2 * (int32_t)ceilf(x) + more;
  }
  return jb.slack[a + hi] + more;
}

// Whether a pair of sizes a and c inside the band, h differing bits, is kept:
// h <= a + c - 2 omin(a, c).  For Cosine: half of a + c - h, the overlap
// bound, reaches the threshold.
template <bool COS, class Test>
__device__ __forceinline__ bool pair_kept(const Test &jb, uint32_t a, uint32_t c, int32_t h) {
  if (COS && jb.cosine) {
    const int32_t s = (int32_t)(a + c) - h;
    return s >= 0 && cosine_reaches((uint32_t)s >> 1, a, c, jb.p, jb.q);
  }
  return h <= jb.slack[a + c];
}

// What a step's slow path needs when the run's thresholds are only bounds.
template <int R>
struct Exact {
  bool bound;
  const uint32_t (&bias)[R];
  const TileJob *job;
};

// popcount(x) + acc as one v_bcnt_u32_b32.  Written out so that the sum over
// a bitmap's words stays one accumulating chain (the compiler would otherwise
// split it into parallel chains joined by an extra add).
__device__ __forceinline__ uint32_t bcnt_acc(uint32_t x, uint32_t acc) {
  uint32_t r;
  asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
  return r;
}

// bias + popcount(b_r xor b_c) with bias = -(slack + 1): negative exactly
// when the pair is kept.  The compare is folded into the popcount chain's
// starting value, so the sign bits of many pairs can be ORed together and
// tested once.
template <int W, int R>
__device__ __forceinline__ uint32_t biased_distance(const Rows<W, R> &rw, const uint32_t *cb,
                                                    int r, uint32_t bias) {
  uint32_t h = bcnt_acc(rw.bits[r][0] ^ cb[0], bias);
#pragma unroll
  for (int e = 1; e < 2 * W; ++e) h = bcnt_acc(rw.bits[r][e] ^ cb[e], h);
  return h;
}

// Slow path: stage the kept pairs of columns [j, j+U), one (column, row
// slab) mask at a time in (column, slab) order, from the biased distances
// the step computed.  False when the queue filled (resume point in the
// sink).
template <int W, int R, int U, bool COS>
__device__ __forceinline__ bool emit(const Rows<W, R> &rw, const uint32_t (&d)[U][R], uint32_t j,
                                     const Exact<R> &ex, Sink &sink) {
  static_assert(U * R <= 32, "one word holds the step's kept flags");
  const unsigned long long below = __lanemask_lt();
  // bit u*R + r: this lane's pair (column j + u, row slab r) is kept; one
  // loop then stages the masks, so the staging code exists once
  uint32_t kb = 0;
#pragma unroll
  for (int x = U * R - 1; x >= 0; --x)
    kb = (kb << 1) | ((int32_t)d[x / R][x % R] < 0 ? 1u : 0u);
  if (ex.bound) {
    // each kept pair at its own sizes.  The
    // biased distance is bias + h, so h = d - bias.
    const PairTest test = pair_test<COS && W >= 32>(*ex.job);
#pragma unroll
    for (int x = 0; x < U * R; ++x) {
      const uint32_t c = as_const(args()->size_cols)[j + x / R];
      const uint32_t h = d[x / R][x % R] - ex.bias[x % R];
      if (((kb >> x) & 1u) &&
          !(c >= rw.cmn[x % R] && c <= rw.cmx[x % R] &&
            pair_kept<COS>(test, rw.size[x % R], c, (int32_t)h)))
        kb &= ~(1u << x);
    }
  }
  const uint32_t row_slab0 = rw.idx[0];  // this lane's row in slab r: + 64 r
#pragma unroll 1
  for (uint32_t x = 0; x < (uint32_t)(U * R); ++x) {
    const bool kp = (kb >> x) & 1u;
    const unsigned long long m = __ballot(kp);
    if (!m) continue;
    const uint32_t u = x / R, r = x - u * R;
    const uint32_t cnt = (uint32_t)__popcll(m);
    if (sink.fill + cnt > kStage && !flush(sink)) return false;
    if (sink.fill == 0) {
      sink.first_col = j + u;
      sink.first_slab = r;
    }
    if (kp)
      sink.stage[sink.fill + (uint32_t)__popcll(m & below)] =
          make_uint2(row_slab0 + 64u * r, j + u);
    sink.fill += cnt;
  }
  return true;
}

// Bitmaps of columns [j, j + U) into SGPRs.
template <int W, int U>
__device__ __forceinline__ void load_cols(const uint64_t *__restrict__ bm_cols, uint32_t j,
                                          uint32_t (&cb)[U][2 * W]) {
  const_u32_ptr p = (const_u32_ptr)as_const(bm_cols + (size_t)j * W);
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int e = 0; e < 2 * W; ++e) cb[u][e] = p[u * 2 * W + e];
}

// j, once every scalar load issued so far (the current step's columns)
// has arrived: the next step's load is then issued after that wait, on
// every path.
__device__ __forceinline__ uint32_t after(uint32_t j) {
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0); vmcnt, expcnt untouched
  return j;
}

// One step: columns [j, j + U) against the wave's rows.  The biased
// distances of its U*R pairs are ORed and one ballot of the sign bit tells
// whether any is kept; only then does the slow path stage them.  On a
// diagonal tile a pair off the lower triangle (j >= i) is made positive.
// False when the queue filled.
template <int W, int R, int U, bool DIAG, bool COS>
__device__ __forceinline__ bool step(const Rows<W, R> &rw, const Exact<R> &ex,
                                     const uint32_t (&cb)[U][2 * W], uint32_t j, Sink &sink) {
  uint32_t d[U][R];
  uint32_t acc = 0;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      uint32_t h = biased_distance<W, R>(rw, cb[u], r, ex.bias[r]);
      if (DIAG) h = j + u < rw.idx[r] ? h : 0u;
      d[u][r] = h;
      acc |= h;
    }
  const bool any = __ballot((int32_t)acc < 0) != 0;
  // (the expectation and the sweep's loop of one exit keep what the slow path needs out of
  // the fast one: without them a 2048-bit class of 150,000 long sets took 34.5 ms,
  // with them 30.1, one of 300,000 short sets at 512 bits 6.35 and 6.00; a class of
  // 60,000 at 64 bits, where most steps keep a pair, 0.35 ms without the
  // expectation and 0.36 with it)
  if (W >= 8 ? __builtin_expect(any, 0) : any)
    return emit<W, R, U, COS>(rw, d, j, ex, sink);
  return true;
}

// Columns [j, g1) of one run.
template <int W, int R, int U, bool DIAG, bool COS>
__device__ __forceinline__ bool sweep(const uint64_t *__restrict__ bm_cols, const Rows<W, R> &rw,
                                      const int32_t (&thr)[R], uint32_t j, uint32_t g1,
                                      bool bound, const TileJob &jb, Sink &sink) {
  uint32_t bias[R];
#pragma unroll
  for (int r = 0; r < R; ++r) bias[r] = (uint32_t)(-thr[r] - 1);
  const Exact<R> ex{bound, bias, &jb};
  // Scalar loads may return out of order, so a wave can only wait for all
  // of them.  Two register buffers alternate: the wait for the current
  // step's columns comes before the next step's load is issued (the next
  // address is made to depend on the current columns), so the next load
  // is in flight while the current step computes, and no registers are
  // copied between steps.
  uint32_t ba[U][2 * W], bb[U][2 * W];
  if (j + U <= g1) load_cols<W, U>(bm_cols, j, ba);
  bool ok = true;
  while (j + U <= g1) {
    const uint32_t jb = after(j + U);
    if (jb + U <= g1) load_cols<W, U>(bm_cols, jb, bb);
    ok = step<W, R, U, DIAG, COS>(rw, ex, ba, j, sink);
    j += U;
    if (!ok || j + U > g1) break;
    const uint32_t ja = after(j + U);
    if (ja + U <= g1) load_cols<W, U>(bm_cols, ja, ba);
    ok = step<W, R, U, DIAG, COS>(rw, ex, bb, j, sink);
    if (!ok) break;
    j += U;
  }
  if (!ok) return false;
  for (; j < g1; ++j) {
    uint32_t cb[1][2 * W];
    load_cols<W, 1>(bm_cols, j, cb);
    if (!step<W, R, 1, DIAG, COS>(rw, ex, cb, j, sink)) return false;
  }
  return true;
}

// One tile: rows [row0, row_end) of a row block (at most 64*R of them, R per
// lane, interleaved by 64), columns [c0, c1).  Returns false when the queue
// filled (a resume point has been recorded).
template <int W, int R, int U, bool COS>
__device__ __forceinline__ bool run_tile(const TileJob &jb, Sink &sink) {
  const ArgPtr ka = args();
  const uint64_t *__restrict__ bm_rows = ka->bm_rows, *__restrict__ bm_cols = ka->bm_cols;
  const uint32_t *__restrict__ size_rows = ka->size_rows, *__restrict__ size_cols = ka->size_cols;
  const uint32_t *__restrict__ cmin = jb.cmin, *__restrict__ cmax = jb.cmax;
  const uint32_t col_base = jb.col_base, row0 = jb.row0, row_end = jb.row_end, c0 = jb.c0,
                 c1 = jb.c1;
  const bool diag = jb.diag;
  uint32_t first_slab = jb.first;
  const uint32_t lane = threadIdx.x & 63;
  Rows<W, R> rw;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = row0 + 64u * r + lane;
    rw.idx[r] = i;
    if (i < row_end) {
      const uint32_t a = size_rows[i];
      rw.size[r] = a;
      rw.cmn[r] = cmin[a];
      rw.cmx[r] = cmax[a];
      const uint32_t *src = reinterpret_cast<const uint32_t *>(bm_rows + (size_t)i * W);
#pragma unroll
      for (int e = 0; e < 2 * W; ++e) rw.bits[r][e] = src[e];
    } else {
      rw.size[r] = 0;
      rw.cmn[r] = 0xFFFFFFFFu;
      rw.cmx[r] = 0;
#pragma unroll
      for (int e = 0; e < 2 * W; ++e) rw.bits[r][e] = 0;
    }
  }
  uint32_t j = c0;
  uint32_t c = j < c1 ? as_const(size_cols)[j] : 0u;
  while (j < c1) {
    const ColRun run = col_run(jb.sstart, col_base, jb.col_max, c, j, c1);
    const bool bound = run.hi > run.lo || (COS && jb.cosine);  // thresholds are bounds only
    int32_t thr[R];
    bool any_ok = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool in_band = run.lo <= rw.cmx[r] && run.hi >= rw.cmn[r];
      if (!in_band) thr[r] = -1;
      else thr[r] = run_slack<COS>(jb, rw.size[r], run.lo, min(run.hi, rw.cmx[r]));
      any_ok |= in_band;
    }
    // the next run's first size, while this run is swept
    if (run.end < c1) c = as_const(size_cols)[run.end];
    // resumed inside column j: its slabs below first_slab are already queued,
    // so column j runs alone with those slabs masked off
    const uint32_t gend = first_slab ? j + 1 : run.end;
    if (first_slab && gend < c1) c = as_const(size_cols)[gend];
    // a masked slab keeps nothing, also not at a pair's own sizes: -1 is
    // below every distance
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((uint32_t)r < first_slab) thr[r] = -1;
    first_slab = 0;
    if (__ballot(any_ok)) {
      const bool ok = diag ? sweep<W, R, U, true, COS>(bm_cols, rw, thr, j, gend, bound, jb, sink)
                           : sweep<W, R, U, false, COS>(bm_cols, rw, thr, j, gend, bound, jb, sink);
      if (!ok) return false;
    }
    j = gend;
  }
  // the tile's staged pairs go out before the next tile
  return flush(sink, true);
}

// The tile loop both kernels share, over the tiles [cfg.tile_lo,
// cfg.tile_hi) of the plan.  Waves first take the resume entries of a
// previous launch that fall in that range (entries k, k + waves, ... go to
// wave k), then fresh tiles, until the range is exhausted or the queue has
// filled.  run(job) runs one tile and returns false when the queue filled,
// with the resume point in the sink.
//
// Fresh tiles come from the partitioned cursors (persistent waves), or, in a
// direct launch (cfg.direct), each wave takes one tile and ends: no cursor
// is read, and the workgroup dispatch balances the tiles of an XCD, which
// gets every eighth run of kDirectDeal tiles (regions as the cursors have
// them would leave XCDs idle: nobody takes their neighbours' tiles).  The
// cursors cost a launch about 45 us that does not grow with its work: a wave
// that finds its own cursor dry reads the other 63 one after the other, a
// memory round trip each.  In a direct launch every tile a full queue keeps a
// wave from starting goes to the resume list (a round that resumes has no
// fresh tiles there: the first round had them all), and a round that
// resumes starts the waves the GPU holds, each with its share of the list.
constexpr uint32_t kDirectDeal = 8;

template <class Run>
__device__ __forceinline__ void tile_loop(Sink &sink, Run &&run) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = wave_index();
  uint32_t t = 0, col = 0, slab = 0, end = 0;
  uint32_t entry = wave;
  bool fresh = true;     // direct: the wave's tile is still to take
  bool stopped = false;  // this wave found the queue full
  bool undone = false;   // ... and left tile t to be done from (col, slab) on
  // Each XCD owns one contiguous region of the tile range, so that its
  // waves sweep neighbouring row blocks whose columns stay in its L2.
  // Inside a region the tiles are dealt to kSub sub-cursors in blocks of
  // kDeal, so that the cursors' atomics spread over kSub addresses (atomics
  // on one address from every XCD serialise) while the region is still
  // swept as one front.  Workgroups are dispatched to the XCDs round-robin:
  // a workgroup starts on its own XCD's region, takes that region's other
  // sub-cursors when its own runs dry, and then the other regions.
  constexpr uint32_t kSub = kParts / kXcds, kDeal = 4;
  const uint32_t xcd0 = blockIdx.x % kXcds, sub0 = (blockIdx.x / kXcds) % kSub;
  uint32_t visit = 0;
  for (;;) {
    const ArgPtr a = args();
    JoinCounters *ctr = a->ctr;
    const uint32_t tile_lo = a->cfg.tile_lo, tile_hi = a->cfg.tile_hi;
    const uint32_t n_tiles = tile_hi - tile_lo;
    const uint32_t n_resume = min(a->cfg.n_resume_in, a->cfg.resume_cap);
    // the queue is full once a wave has left something to be done
    const bool full =
        stopped ||
        rfl(__hip_atomic_load(&ctr->n_resume, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
    if (full) {
      // The tile, and what the wave has left of the resume entries (entry, entry + waves,
      // ...), stay to be done: one reservation for 64 of them.  One each, on one
      // address, took most of a round of a small queue over many tiles: a 40,000-slot
      // queue over 25,000 tiles 0.62 ms a round, so 0.10.  The count of what was left
      // is also the sign that the queue is full: a flag of its own, stored by every
      // wave that finds it so, took 0.12 ms of such a round.
      do {
        const uint64_t e = entry + (uint64_t)lane * a->cfg.waves;
        uint32_t rt = t, rc = col, rs = slab, re = end;  // lane 63: the tile
        bool left = undone && lane == 63;
        if (lane < 63 && e < n_resume) {
          const Resume *in = a->resume_in + e;
          rt = in->tile, rc = in->col, rs = in->slab, re = in->end;
          left = rt >= tile_lo && rt < tile_hi;
        }
        const unsigned long long m = __ballot(left);
        if (m) {
          uint32_t at = 0;
          if (lane == 0) at = atomicAdd(&ctr->n_resume, (uint32_t)__popcll(m));
          at = rfl(at);
          if (at == 0 && lane == 0) ctr->overflow = 1;  // for the host
          at += (uint32_t)__popcll(m & __lanemask_lt());
          if (left && at < a->cfg.resume_cap) a->resume_out[at] = Resume{rt, rc, rs, re};
        }
        undone = false;
        entry = (uint32_t)min(entry + (uint64_t)63 * a->cfg.waves, (uint64_t)n_resume);
      } while (entry < n_resume);
    }
    bool resumed = false;
    while (entry < n_resume && !resumed) {
      const auto *in = as_const(a->resume_in) + entry;
      t = rfl(in->tile);
      col = rfl(in->col);
      slab = rfl(in->slab);
      end = rfl(in->end);
      resumed = t >= tile_lo && t < tile_hi;
      entry += a->cfg.waves;
    }
    if (!resumed && a->cfg.direct) {
      if (!fresh || a->cfg.n_resume_in) break;
      fresh = false;
      const uint32_t i = blockIdx.x / kXcds;  // one wave per workgroup
      const uint32_t k = ((i / kDirectDeal) * kXcds + blockIdx.x % kXcds) * kDirectDeal +
                         i % kDirectDeal;
      if (k >= n_tiles) break;
      t = tile_lo + k;
      if (full) {
        col = kTileStart;
        slab = end = 0;
        undone = true;
        continue;
      }
    } else if (!resumed) {
      if (full) break;
      uint32_t *cursors = &ctr->tile_next[a->cfg.cls][0][0];
      bool got = false;
      while (visit < kParts) {
        const uint32_t x = (xcd0 + visit / kSub) % kXcds, k = (sub0 + visit) % kSub;
        const uint32_t r0 = (uint32_t)(((uint64_t)n_tiles * x) / kXcds);
        const uint32_t len = (uint32_t)(((uint64_t)n_tiles * (x + 1)) / kXcds) - r0;
        // tiles of the region sub-cursor k owns: blocks k, k + kSub, ...
        const uint32_t rounds = len / (kSub * kDeal), rem = len - rounds * kSub * kDeal;
        const uint32_t owned =
            rounds * kDeal + min(kDeal, rem > k * kDeal ? rem - k * kDeal : 0u);
        uint32_t *cur = &cursors[(x * kSub + k) * 32];
        // a relaxed read first: exhausted sub-cursors cost no atomic
        uint32_t c = owned;
        if (lane == 0 &&
            __hip_atomic_load(cur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < owned)
          c = atomicAdd(cur, 1u);
        c = rfl(c);
        if (c < owned) {
          t = tile_lo + r0 + ((c / kDeal) * kSub + k) * kDeal + c % kDeal;
          got = true;
          break;
        }
        ++visit;
      }
      if (!got) break;
    }
    // decode the tile
    const uint32_t b = as_const(a->tile_block)[t];
    if (b >= a->cfg.n_blocks) break;
    const auto *blocks = as_const(a->blocks);
    const uint32_t *tables = a->tables;
    const uint32_t tile_cols = a->cfg.tile_cols;
    TileJob job;
    job.row0 = rfl(blocks[b].row0);
    job.row_end = min(rfl(blocks[b].row_end), a->cfg.n_rows);
    const uint32_t cbeg = rfl(blocks[b].col_begin);
    const uint32_t cend = rfl(blocks[b].col_end);
    const uint32_t k = t - rfl(blocks[b].tile_begin);
    const uint32_t task = rfl(blocks[b].task);
    const bool self = rfl(blocks[b].self) != 0;
    const auto *td = as_const(a->tasks) + task;
    job.task = task;
    job.slack = reinterpret_cast<const int32_t *>(tables + rfl(td->slack_off));
    job.cmin = tables + rfl(td->cmin_off);
    job.cmax = tables + rfl(td->cmax_off);
    job.sstart = as_const(a->sstart_cols) + rfl64(td->col_sstart_off);
    job.col_base = rfl(td->col_base);
    job.col_max = a->cfg.col_max_size;
    job.cosine = rfl(td->sim) == SSJ_SIM_COSINE;
    job.p = rfl(td->p);
    job.q = rfl(td->q);
    job.t = rfl((float)job.p / (float)job.q);
    uint32_t c0, c1;
    job.diag = false;
    if (self) {
      const uint32_t n_int = (job.row0 - cbeg + tile_cols - 1) / tile_cols;
      if (k < n_int) {
        c0 = cbeg + k * tile_cols;
        c1 = min(c0 + tile_cols, job.row0);
      } else {
        c0 = job.row0;
        c1 = cend;
        job.diag = true;
      }
    } else {
      c0 = cbeg + k * tile_cols;
      c1 = min(c0 + tile_cols, cend);
    }
    job.first = 0;
    job.end = 0;
    if (resumed && col != kTileStart) {
      c0 = col;
      job.first = slab;
      job.end = end;
    }
    job.c0 = c0;
    job.c1 = min(c1, a->cfg.n_cols);
    if (!run(job)) {
      // the queue is full: the tile resumes at the sink's point, and the wave takes no more
      stopped = undone = true;
      col = rfl(sink.fail_col);
      slab = rfl(sink.fail_slab);
      end = rfl(sink.fail_end);
    }
  }
  sink_pad(sink);
}

__device__ __forceinline__ void sink_init(Sink &sink, uint2 *stage, uint32_t *kept,
                                          uint32_t *rows) {
  sink.stage = stage;
  sink.kept = kept;
  sink.rows = rows;
  sink.fill = 0;
  sink.first_col = 0;
  sink.first_slab = 0;
  sink.first_end = 0;
  sink.fail_col = 0;
  sink.fail_slab = 0;
  sink.fail_end = 0;
  sink.stripe = wave_index() & (args()->cfg.stripes - 1);
  sink.pos = 0;
  sink.end = 0;
}

// Vector-ALU filter for one bitmap width (W words, R rows per lane, U
// columns per step).
template <int W, int R, int U, bool COS>
__global__ __launch_bounds__(kBlock) void k_filter(FilterArgs) {
  extern __shared__ uint2 stage[];  // kStage entries per wave
  Sink sink;
  sink_init(sink, stage + rfl(threadIdx.x >> 6) * kStage, nullptr, nullptr);
  tile_loop(sink, [&](const TileJob &jb) { return run_tile<W, R, U, COS>(jb, sink); });
}

// ---------------------------------------------------------------------------
// Matrix-core filter (b = 64, 128, 256, 512, 1024).
//
// With every bit of a bitmap mapped to +1 (set) or -1 (clear), the dot
// product of two such vectors over K bits is K - 2 popcount(b_r xor b_s), so
// the test of Theorem 1 reads dot >= T = K - 2 slack.  The values +-1 are
// exact in fp4 (e2m1) and the dot products are small integers, exact in the
// fp32 accumulator, so the decision is the same as the vector-ALU kernel's.
// One v_mfma_scale_f32_32x32x64_f8f6f4 scores 32 columns against 32 rows
// over 64 bits:
//   - MFMA rows (A) are 32 consecutive columns of the sweep (one step),
//     loaded per step from the column sign planes, the next step's while
//     the current one computes;
//   - MFMA columns (B) are 32 of the wave's rows, RT such row tiles, held in
//     registers for the whole tile;
//   - lane l holds row l%32 of every row tile and 16 of the step's columns,
//     8(v/4) + 4(l/32) + v%4 for v = 0..15.  Steps never cross a run's end (a
//     run's last step is partial, and the pairs of the columns past its end
//     are dropped), so one threshold per lane and row tile covers all 16
//     values: the max of the 16 dot products against T is the whole fast-path
//     test.  In a run of several sizes T is a bound, and the slow path tests
//     each pair that reaches it at its own sizes.
// The slow path stages the kept pairs in a fixed order (row tile, then v,
// then lane), so a step resumed after a full queue skips exactly the pairs
// it had written.

typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef float v16f_t __attribute__((ext_vector_type(16)));

constexpr float kNever = 1.0e9f;  // threshold of a row that no column of the group pairs with

template <int W, int RT>
struct MRows {
  uint4 sg[RT][W];  // this lane's half of every 64-bit block of its row in each row tile
  // dot threshold for the current run, for the fast test, which compares the bit patterns
  // of the dot products as integers: for a positive threshold those order
  // like the values (every value is an exact integer, +0 included, and the
  // negative ones fall below every positive pattern); a threshold of 0 or
  // less is below every pattern, so that every step goes to the exact test
  int32_t thr_bits[RT];
  uint32_t size[RT];
  uint32_t cmn[RT];
  uint32_t cmx[RT];
  uint32_t idx;     // this lane's row in row tile 0 (row tile rt: idx + 32 rt)
};

// The dot threshold a lane's thr_bits stand for.
__device__ __forceinline__ int32_t dot_threshold(int32_t bits) {
  return bits < INT32_MIN + (1 << 16) ? INT32_MIN - bits : (int32_t)__int_as_float(bits);
}
// ... and the other way: a threshold t of 0 or less becomes INT32_MIN - t, below
// every bit pattern of a dot product (INT32_MIN itself would be -0, which an
// accumulator that starts at +0 never holds).
__device__ __forceinline__ int32_t dot_threshold_bits(int32_t t) {
  return t > 0 ? __float_as_int((float)t) : INT32_MIN - max(t, -(1 << 15));
}

__device__ __forceinline__ v16f_t mfma_pm1(const uint4 &a, const uint4 &b, const v16f_t &c) {
  const v8i_t x = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
  const v8i_t y = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
  // formats 4/4: fp4 (e2m1) for A and B; scales 2^0 (e8m0 127)
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, c, 4, 4, 0, 127, 0, 127);
}

// This lane's half of set `col`'s sign planes, every block, or of set n's when !ok: the
// planes end in kSignPad sets of zeros, so every lane loads and no load sits
// behind a branch.
template <int W>
__device__ __forceinline__ void load_signs(const uint4 *__restrict__ planes, uint32_t n,
                                           uint32_t col, bool ok, uint32_t h, uint4 (&a)[W]) {
  const size_t c = ok ? col : n;
#pragma unroll
  for (int kb = 0; kb < W; ++kb) a[kb] = planes[((size_t)kb * (n + kSignPad) + c) * 2 + h];
}

// The columns j0 + (lane % 32) of one step: a uniform address (j0 is the
// same in every lane) plus the lane's byte offset loff = 32 (lane % 32) +
// 16 h.  No bounds test: the zero padding past set n - 1 covers loads up to
// 191 columns past a column below n, and the pairs of columns past the size
// group's end are dropped by the exact test.
template <int W>
__device__ __forceinline__ void load_cols(const uint4 *__restrict__ planes, uint32_t n,
                                          uint32_t j0, uint32_t loff, uint4 (&a)[W]) {
  // Opaque at 1024 bits: the compiler keeps loff widened to 64 bits, and the kernel has no
  // registers for it.  With this and the uniform values below in scalar registers
  // it uses no scratch memory: a reload in every step waited for all loads in
  // flight, the ring's among them (the 1024-bit class of a batch of 256 joins:
  // 4.31 -> 3.62 ms).
  if (W >= 16) asm volatile("" : "+v"(loff));
#pragma unroll
  for (int kb = 0; kb < W; ++kb) {
    const uint4 *p = planes + ((size_t)kb * (n + kSignPad) + j0) * 2;
    a[kb] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(p) + loff);
  }
}

// Stage one ballot mask of kept pairs (row `row` of the lanes' row tile is
// the caller's; column per lane): `skip` pairs are dropped first, `done`
// counts the step's pairs in order.
__device__ __forceinline__ bool stage_mask(unsigned long long m, uint32_t row, uint32_t col,
                                           uint32_t j0, uint32_t gend, uint32_t &skip,
                                           uint32_t &done, Sink &sink) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t cnt = (uint32_t)__popcll(m);
  if (skip) {
    if (skip >= cnt) {
      skip -= cnt;
      done += cnt;
      return true;
    }
    for (uint32_t x = 0; x < skip; ++x) m &= m - 1;  // drop the lowest `skip` lanes
    done += skip;
    cnt -= skip;
    skip = 0;
  }
  if (sink.fill + cnt > kStage && !flush(sink)) return false;
  if (sink.fill == 0) {
    sink.first_col = j0;
    sink.first_slab = done;
    sink.first_end = gend;
  }
  if ((m >> lane) & 1ull)
    sink.stage[sink.fill + (uint32_t)__popcll(m & __lanemask_lt())] = make_uint2(row, col);
  sink.fill += cnt;
  done += cnt;
  return true;
}

// Lane's values k (bit v: value v) that passed a bound, each tested exactly, one
// value per lane at a time, from the pair's sizes and bitmaps (b = 64).  rows: the
// lane's row, cols: the lane's first column, both in LDS (columns 8 (v / 4) + v % 4
// further on).
template <bool COS>
__device__ __forceinline__ uint32_t refine(uint32_t k, const uint32_t *rows, const uint32_t *cols,
                                           const TileJob &jb) {
  const uint32_t a = rows[0], lo = rows[kTwoRows], hi = rows[2 * kTwoRows];
  const uint32_t r0 = rows[3 * kTwoRows], r1 = rows[4 * kTwoRows];
#pragma unroll 1
  for (uint32_t todo = k; todo; todo &= todo - 1) {
    const uint32_t v = (uint32_t)__builtin_ctz(todo);
    const uint32_t *col = cols + 8u * (v >> 2) + (v & 3u);
    const uint32_t c = col[0];
    const int32_t h = __popc(r0 ^ col[64]) + __popc(r1 ^ col[128]);
    if (!(c >= lo && c <= hi && pair_kept<COS>(jb, a, c, h))) k &= ~(1u << v);
  }
  return k;
}

// Bits v (0 .. 15) whose column cb + 8 (v / 4) + v % 4 lies below `end`.
__device__ __forceinline__ uint32_t columns_below(uint32_t cb, uint32_t end) {
  const uint32_t left = end > cb ? min(end - cb, 32u) : 0u;
  const uint32_t whole = 4u * (left >> 3), some = min(left & 7u, 4u);
  return ((1u << whole) - 1u) | (((1u << some) - 1u) << whole);
}

// Stage the kept pairs of a step at columns j0 ...: bit rt of `hits` names the row
// tiles to look at, and sink.kept their lanes' kept values, 16 bits for each of
// the step's HALVES runs of 32 columns (bit v of a half: column 8 (v / 4) + 4 (lane /
// 32) + v % 4 of it), columns past the run's end or a diagonal tile's row among
// them; bound (HALVES = 2): they only passed a bound.  Few lanes with kept values
// (the usual case): the wave walks those lanes and their set bits, one pair at
// a time, in the order (lane, v).  Many: one ballot per value v stages whole masks, in the order
// (v, lane).  The choice depends only on the pairs kept, so a step resumed
// after a full queue takes the same order and skips exactly the `skip` pairs
// it had written.  (One rolled loop: unrolled over the row tiles it was most of
// the kernel's code, and every entry waited for instructions.)
template <int HALVES, bool COS>
__device__ __forceinline__ bool stage_step(uint32_t hits, uint32_t row_tile0, uint32_t j0,
                                           uint32_t gend, const TileJob &jb, uint32_t &skip,
                                           Sink &sink, bool bound = false) {
  constexpr uint32_t kFewLanes = 4;
  const uint32_t lane = threadIdx.x & 63;
  uint32_t done = 0;
#pragma unroll 1
  for (hits = rfl(hits); hits; hits &= hits - 1) {
    const uint32_t rt = (uint32_t)__builtin_ctz(hits);
    const uint32_t kept = sink.kept[64 * rt + lane];
    const uint32_t row0 = row_tile0 + 32u * rt;
#pragma unroll 1
    for (uint32_t s = 0; s < (uint32_t)HALVES; ++s) {
      uint32_t k = HALVES == 1 ? kept : (kept >> (16u * s)) & 0xFFFFu;
      const uint32_t js = j0 + 32u * s;
      const uint32_t cb = js + 4u * (lane >> 5), my_row = row0 + (lane & 31u);
      k &= columns_below(cb, jb.diag ? min(gend, my_row) : gend);
      if (HALVES == 2 && bound)
        k = refine<COS>(k, sink.rows + 32u * rt + (lane & 31u),
                        sink.rows + 5 * kTwoRows + (cb - j0), jb);
      unsigned long long lm = __ballot(k != 0);
      if ((uint32_t)__popcll(lm) > kFewLanes) {
#pragma unroll 1
        for (uint32_t v = 0; v < 16; ++v) {
          const unsigned long long m = __ballot((k >> v) & 1u);
          if (m && !stage_mask(m, my_row, cb + 8u * (v >> 2) + (v & 3u), j0, gend, skip, done,
                               sink))
            return false;
        }
        continue;
      }
      while (lm) {
        const uint32_t L = (uint32_t)__builtin_ctzll(lm);
        lm &= lm - 1;
        uint32_t kk = (uint32_t)__builtin_amdgcn_readlane((int)k, (int)L);
        const uint32_t row = row0 + (L & 31u);
        const uint32_t cL = js + 4u * (L >> 5);
        while (kk) {
          const uint32_t v = (uint32_t)__builtin_ctz(kk);
          kk &= kk - 1;
          if (skip) {
            --skip;
            ++done;
            continue;
          }
          if (sink.fill == kStage && !flush(sink)) return false;
          if (sink.fill == 0) {
            sink.first_col = j0;
            sink.first_slab = done;
            sink.first_end = gend;
          }
          if (lane == 0) sink.stage[sink.fill] = make_uint2(row, cL + 8u * (v >> 2) + (v & 3u));
          ++sink.fill;
          ++done;
        }
      }
    }
  }
  return true;
}

// Slow path of one step at columns [j0, j0 + 32) of a run: stage the kept pairs.
// Only row tiles whose best value reaches their threshold are looked at; their
// dot products are made again (the fast path does not keep them: registers
// are what limits the waves per SIMD).
template <int W, int RT, bool COS>
__device__ __forceinline__ bool emit_mfma(const MRows<W, RT> &rw, const uint4 (&a)[W],
                                          const int32_t (&mx)[RT], uint32_t j0,
                                          const ColRun &run, const TileJob &jb, uint32_t &skip,
                                          Sink &sink) {
  const uint32_t lane = threadIdx.x & 63;
  const bool bound = run.hi > run.lo || (COS && jb.cosine);  // the threshold is only a bound
  uint32_t hits = 0;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if (!__ballot(mx[rt] >= rw.thr_bits[rt])) continue;
    v16f_t d = {};
#pragma unroll
    for (int kb = 0; kb < W; ++kb) d = mfma_pm1(a[kb], rw.sg[rt][kb], d);
    const float thr = (float)dot_threshold(rw.thr_bits[rt]);
    uint32_t k = 0;  // bit v: value v kept (built by shifting: no wide constants)
#pragma unroll
    for (int v = 15; v >= 0; --v) k = (k << 1) | (d[v] >= thr ? 1u : 0u);
    if (bound) {
      const uint32_t cb = j0 + 4u * (lane >> 5), my_row = rw.idx + 32u * rt;
      k &= columns_below(cb, jb.diag ? min(run.end, my_row) : run.end);
      if (__ballot(k != 0)) {
        // each value that reaches the bound is tested at its own column's size,
        // one value per lane at a time, from a copy of the products in LDS (from
        // the bitmaps, W words a pair: +40 us in a 1024-bit class of 350 us)
        int16_t *dots = reinterpret_cast<int16_t *>(sink.rows);
#pragma unroll
        for (int v = 0; v < 16; ++v) dots[64 * v + lane] = (int16_t)d[v];
        __builtin_amdgcn_wave_barrier();
        const uint32_t *size_cols = args()->size_cols;
        for (uint32_t todo = k; todo; todo &= todo - 1) {
          const uint32_t v = (uint32_t)__builtin_ctz(todo);
          const uint32_t c = size_cols[cb + 8u * (v >> 2) + (v & 3u)];
          const int32_t dot = dots[64 * v + lane];
          if (!(c >= rw.cmn[rt] && c <= rw.cmx[rt] &&
                pair_kept<COS>(jb, rw.size[rt], c, (64 * W - dot) >> 1)))
            k &= ~(1u << v);
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
    sink.kept[64 * rt + lane] = k;
    hits |= 1u << rt;
  }
  __builtin_amdgcn_wave_barrier();
  return stage_step<1, COS>(hits, (uint32_t)__builtin_amdgcn_readlane((int)rw.idx, 0), j0,
                            run.end, jb, skip, sink);
}

// The dot products of the step's columns `a` with row tile rt.
template <int W, int RT>
__device__ __forceinline__ v16f_t products(const uint4 (&a)[W], const MRows<W, RT> &rw, int rt) {
  v16f_t t = {};
#pragma unroll
  for (int kb = 0; kb < W; ++kb) t = mfma_pm1(a[kb], rw.sg[rt][kb], t);
  return t;
}

// Largest of the 16 dot products of a lane (one row, 16 columns) as a bit
// pattern compared as an integer: a tree of 3-input maxima.
__device__ __forceinline__ int32_t max16(const v16f_t &x) {
  int32_t b[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) b[v] = __float_as_int(x[v]);
  int32_t m0 = max(max(b[0], b[1]), b[2]);
  int32_t m1 = max(max(b[3], b[4]), b[5]);
  int32_t m2 = max(max(b[6], b[7]), b[8]);
  int32_t m3 = max(max(b[9], b[10]), b[11]);
  int32_t m4 = max(max(b[12], b[13]), b[14]);
  m0 = max(max(m0, m1), m2);
  m3 = max(max(m3, m4), b[15]);
  return max(m0, m3);
}

// Fast path of one step: columns [j0, j0 + 32) (operands `a`) against the
// wave's rows.  Leaves each row tile's largest bit pattern (as an integer)
// in mx and returns whether one reaches its threshold (thr_bits).  Integer
// maxima: float maxima would first quiet possible signalling NaNs, two
// more instructions per row tile.
//
// The products run one row tile ahead of their reduction, across steps:
// product number k (row tile k mod RT of step k / RT) goes into
// accumulator k mod 3 and is reduced while product k + 1 runs on the
// matrix cores; the last row tile's reduction overlaps the first product
// of the next step (operands `an`, the next step's columns, already
// loaded).  K is the step's place in the three-step unrolled loop, so that
// every accumulator index is a constant; on entry accumulator (K RT) mod 3
// holds this step's first product.  When the sweep ends after this step,
// that last product is simply dropped.
template <int W, int RT, int K>
__device__ __forceinline__ bool fast_mfma(const uint4 (&a)[W], const uint4 (&an)[W],
                                          const MRows<W, RT> &rw, v16f_t (&acc)[3],
                                          int32_t (&mx)[RT]) {
  unsigned long long hit = 0;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    constexpr int base = K * RT;
    const int cur = (base + rt) % 3, nxt = (base + rt + 1) % 3;
    acc[nxt] = rt + 1 < RT ? products<W, RT>(a, rw, rt + 1) : products<W, RT>(an, rw, 0);
    __builtin_amdgcn_sched_barrier(0);
    mx[rt] = max16(acc[cur]);
    hit |= __ballot(mx[rt] >= rw.thr_bits[rt]);
    __builtin_amdgcn_sched_barrier(0);
  }
  // the next step's first product stays ahead of the branch that ends the
  // step (the compiler would otherwise sink it below, into the next step)
  asm volatile("" ::"v"(acc[(K * RT + RT) % 3]));
  return hit != 0;
}

// The steps of columns [j, g1) of one run; b0 and b1 hold (or are being
// loaded with) the columns of its first two steps.  Column loads run two
// steps ahead in a ring of three register buffers; the loop is unrolled by
// three so that the ring turns without register copies (a copy of a buffer
// still being loaded would wait for that load) and the accumulators of the
// fast path keep constant indices.  A step that keeps something leaves the
// loop for the one slow path, laid out once (instruction cache: the kernel
// stays small); the slow path turns the ring by register moves so that the
// loop goes on at the next step with the buffers already loaded.  Every
// branch leaves the loop, none enters it in the middle, and every buffer
// is read on both sides of each exit: the compiler keeps the ring in fixed
// registers and leaves the loads where they are.
template <int W, int RT, bool COS>
__device__ __forceinline__ bool sweep_mfma(const uint4 *__restrict__ sg_cols, uint32_t n_cols,
                                           const MRows<W, RT> &rw, uint4 (&b0)[W],
                                           uint4 (&b1)[W], uint32_t j, const ColRun &run,
                                           const TileJob &jb, uint32_t &skip, Sink &sink) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t loff = (lane & 31u) * 32u + (lane >> 5) * 16u;
  const uint32_t g1 = run.end;
  uint4 b2[W];
  int32_t mx[RT];
  v16f_t acc[3];
  uint32_t j0 = j;
  for (;;) {
    int phase;  // the ring buffer that holds the columns of step j0
    // The step's columns for the slow path, copied on the way out of the
    // loop from the one buffer that holds them: selecting among the three
    // would read the buffer whose load the step has just issued, and wait
    // for it (a whole memory round trip per slow-path entry).
    uint4 cur[W];
    acc[0] = products<W, RT>(b0, rw, 0);
    for (;;) {
      load_cols<W>(sg_cols, n_cols, j0 + 64, loff, b2);
      if (__builtin_expect(fast_mfma<W, RT, 0>(b0, b1, rw, acc, mx), 0)) {
        phase = 0;
#pragma unroll
        for (int kb = 0; kb < W; ++kb) cur[kb] = b0[kb];
        break;
      }
      skip = 0;
      if ((j0 += 32) >= g1) return true;
      load_cols<W>(sg_cols, n_cols, j0 + 64, loff, b0);
      if (__builtin_expect(fast_mfma<W, RT, 1>(b1, b2, rw, acc, mx), 0)) {
        phase = 1;
#pragma unroll
        for (int kb = 0; kb < W; ++kb) cur[kb] = b1[kb];
        break;
      }
      skip = 0;
      if ((j0 += 32) >= g1) return true;
      load_cols<W>(sg_cols, n_cols, j0 + 64, loff, b1);
      if (__builtin_expect(fast_mfma<W, RT, 2>(b2, b0, rw, acc, mx), 0)) {
        phase = 2;
#pragma unroll
        for (int kb = 0; kb < W; ++kb) cur[kb] = b2[kb];
        break;
      }
      skip = 0;
      if ((j0 += 32) >= g1) return true;
    }
    if (!emit_mfma<W, RT, COS>(rw, cur, mx, j0, run, jb, skip, sink)) return false;
    skip = 0;
    if ((j0 += 32) >= g1) return true;
    // b0 and b1 take the columns of steps j0 and j0 + 32
#pragma unroll
    for (int kb = 0; kb < W; ++kb) {
      const uint4 x0 = phase == 0 ? b1[kb] : phase == 1 ? b2[kb] : b0[kb];
      const uint4 x1 = phase == 0 ? b2[kb] : phase == 1 ? b0[kb] : b1[kb];
      b0[kb] = x0;
      b1[kb] = x1;
    }
  }
}

// One tile on the matrix cores: rows [row0, row_end) (at most 32*RT),
// columns [c0, c1).
template <int W, int RT, bool COS>
__device__ __forceinline__ bool run_tile_mfma(const TileJob &jb, Sink &sink) {
  const ArgPtr ka = args();
  const uint4 *__restrict__ sg_rows = ka->sg_rows, *__restrict__ sg_cols = ka->sg_cols;
  const uint32_t *__restrict__ size_rows = ka->size_rows, *__restrict__ size_cols = ka->size_cols;
  const uint32_t n_rows = ka->cfg.n_rows, n_cols = ka->cfg.n_cols;
  const uint32_t lane = threadIdx.x & 63, h = lane >> 5, jr = lane & 31;
  constexpr int32_t K = 64 * W;
  MRows<W, RT> rw;
  rw.idx = jb.row0 + jr;
  // No branches: every row's loads are in flight together (with a branch per row
  // tile each waited for the one before: b = 128, 256 and 512 classes of 20,000 ..
  // 32,000 tiles 750, 726, 284 -> 680, 686, 266 us; not measured by itself at b =
  // 1024, where the loads take the kernel's last registers).  Rows past the end read the last one's.
  const uint32_t last = jb.row_end - 1;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) rw.size[rt] = size_rows[min(rw.idx + 32u * rt, last)];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const uint32_t i = rw.idx + 32u * rt;
    load_signs<W>(sg_rows, n_rows, i, i <= last, h, rw.sg[rt]);
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    rw.cmn[rt] = jb.cmin[rw.size[rt]];
    rw.cmx[rt] = jb.cmax[rw.size[rt]];
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if (rw.idx + 32u * rt > last) {
      rw.size[rt] = 0;
      rw.cmn[rt] = 0xFFFFFFFFu;
      rw.cmx[rt] = 0;
    }
  }
  uint32_t skip = jb.first;
  uint32_t j = jb.c0;
  const uint32_t loff = jr * 32u + h * 16u;
  uint32_t c = j < jb.c1 ? as_const(size_cols)[j] : 0u;
  uint32_t resumed_end = jb.end;
  while (j < jb.c1) {
    // the run's first columns, its end and its thresholds are loaded
    // together (they need only j and c), the next run's first size while
    // this run is swept
    uint4 b0[W], b1[W];
    if (W < 16) {
      load_cols<W>(sg_cols, n_cols, j, loff, b0);
      load_cols<W>(sg_cols, n_cols, j + 32, loff, b1);
    }
    ColRun run = col_run(jb.sstart, jb.col_base, jb.col_max, c, j, jb.c1);
    if (resumed_end) {
      // resumed inside a run: its step ends where it did
      run.end = min(max(resumed_end, j + 1), jb.c1);
      run.hi = as_const(size_cols)[run.end - 1];
      resumed_end = 0;
    }
    if (run.end < jb.c1) c = as_const(size_cols)[run.end];
    bool any_ok = false;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const bool in_band = run.lo <= rw.cmx[rt] && run.hi >= rw.cmn[rt];
      // (slack[0] for a row outside the band: no branch, the loads go out together)
      const int32_t sl = run_slack<COS>(jb, in_band ? rw.size[rt] : 0u, run.lo,
                                        in_band ? min(run.hi, rw.cmx[rt]) : 0u);
      rw.thr_bits[rt] = in_band ? dot_threshold_bits(K - 2 * sl) : __float_as_int(kNever);
      any_ok |= in_band;
    }
    if (__ballot(any_ok)) {
      if (W >= 16) {  // no registers to hold them through the thresholds
        load_cols<W>(sg_cols, n_cols, j, loff, b0);
        load_cols<W>(sg_cols, n_cols, j + 32, loff, b1);
      }
      if (!sweep_mfma<W, RT, COS>(sg_cols, n_cols, rw, b0, b1, j, run, jb, skip, sink))
        return false;
    }
    skip = 0;
    j = run.end;
  }
  // the tile's staged pairs go out before the next tile
  return flush(sink, true);
}

// ---------------------------------------------------------------------------
// Two columns per accumulator (b = 64).
//
// There the reduction of the products, not the matrix cores, bounds the plain
// kernel: a product leaves 16 values per lane, 8 three-input maxima, 36 cycles of
// vector issue against 32 of the matrix cores (b = 64).  The K = 64 slots of a
// product are two blocks of 32 with a power-of-two scale each, so a product
// can score 32 bits of one column in block 0 and 32 bits of another in block 1:
// with scales 2^-1 and 2^15, and an accumulator that starts at C, 2 W chained
// products leave
//   C + d0 / 2 + 2^16 d1 / 2,
// d0 and d1 the dot products (even numbers) of columns j and j + 32 with the row.
// C is the float with bit pattern 0x4B404000 (1.5 2^23 + 2^14), so that the sum
// stays in [2^23, 2^24), where a float's pattern is its value plus a constant.
// (A single +-1/2 has no place there: that a block's sum arrives whole rests on how
// the matrix cores add, and on the test that checks every pair of dot products.)
// Its halves are 0x4B40 + d1 / 2 and 0x4000 + d0 / 2, two positive 16-bit floats
// that order like the dot products.  A tree of packed 3-input 16-bit maxima, the
// threshold (less one) among its inputs, reduces 32 pairs in the 8 instructions
// that 16 took, and a pair is kept exactly when the result differs from the
// threshold.
//
// Alone, in registers: 443 cycles per 12,288 pairs against 328 per 6,144; under
// load the clock falls (power) from 2.25 to 1.87 GHz, 4.3e13 -> 5.3e13 pairs/s.  In
// the 1,000,000-set join's b = 64 class 1.99 -> 1.72 ms, in a join of 4,000,000
// short sets 9.05 -> 7.85 ms.  At b = 128 the matrix cores bound the plain kernel
// as much as the reduction, and the larger state costs a wave per SIMD: 0.150 ->
// 0.198 ms in the 1,000,000-set join, 0.257 -> 0.284 in a query of 2,000 sets
// against 5,000,000; it keeps the plain kernel.
//
// A step is 64 columns: lane l holds column j0 + l, both halves of every 64-bit
// block; the row operand is the same in both halves of the wave.

typedef _Float16 h2_t __attribute__((ext_vector_type(2)));

constexpr uint32_t kFieldLo = 0x4000u, kFieldHi = 0x4B40u;

template <int W, int RT>
struct PRows {
  uint4 sg[RT][2 * W];  // every half block of the lane's row (lane % 32) in each row tile
  uint32_t thr[RT];     // packed: one less than the least kept value, in both halves
  // sizes and bands of the wave's rows in LDS (registers are what limits the
  // waves per SIMD, and they are needed once a run): size, cmin, cmax, and the
  // bitmap's low and high half
  uint32_t (*row)[kTwoRows];
};

// Packed threshold of the dot threshold t = 2 u (64 W + 2 or more: never).
template <int W>
__device__ __forceinline__ uint32_t pack_threshold(int32_t u) {
  u = min(max(u, -32 * W), 32 * W + 1);
  return ((kFieldHi + (uint32_t)(u - 1)) << 16) + kFieldLo + (uint32_t)(u - 1);
}

__device__ __forceinline__ v16f_t mfma_two(const uint4 &a, const uint4 &b, const v16f_t &c,
                                           int scale) {
  const v8i_t x = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
  const v8i_t y = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, c, 4, 4, 0, scale, 0, 127);
}

__device__ __forceinline__ h2_t max3(h2_t a, h2_t b, h2_t c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// Halfwise maximum of the 16 values and `thr`.
__device__ __forceinline__ uint32_t max17(const v16f_t &x, uint32_t thr) {
  h2_t b[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    // (by way of a float: bit-casting the element itself reads element 0)
    const float f = x[v];
    b[v] = __builtin_bit_cast(h2_t, f);
  }
  h2_t m0 = max3(b[0], b[1], b[2]), m1 = max3(b[3], b[4], b[5]), m2 = max3(b[6], b[7], b[8]);
  h2_t m3 = max3(b[9], b[10], b[11]), m4 = max3(b[12], b[13], b[14]);
  m0 = max3(m0, m1, m2);
  m3 = max3(m3, m4, b[15]);
  return __builtin_bit_cast(uint32_t, max3(m0, m3, __builtin_bit_cast(h2_t, thr)));
}

// The products of the step's columns with row tile rt; c: the start value.
template <int W, int RT>
__device__ __forceinline__ v16f_t products_two(const uint4 (&a)[2 * W], const PRows<W, RT> &rw,
                                               int rt, const v16f_t &c, int scale) {
  v16f_t t = mfma_two(a[0], rw.sg[rt][0], c, scale);
#pragma unroll
  for (int x = 1; x < 2 * W; ++x) t = mfma_two(a[x], rw.sg[rt][x], t, scale);
  return t;
}

// Columns j0 + lane of one step, as load_cols: a column below n plus at most
// kSignPad - 1.
template <int W>
__device__ __forceinline__ void load_cols_two(const uint4 *__restrict__ planes, uint32_t n,
                                              uint32_t j0, uint32_t loff, uint4 (&a)[2 * W]) {
  // (opaque: the compiler would keep planes + loff, 64 bits a lane, and spill it)
  asm volatile("" : "+v"(loff));
#pragma unroll
  for (int kb = 0; kb < W; ++kb) {
    const char *p = reinterpret_cast<const char *>(planes +
                                                   ((size_t)kb * (n + kSignPad) + j0) * 2) + loff;
    a[2 * kb] = *reinterpret_cast<const uint4 *>(p);
    a[2 * kb + 1] = *reinterpret_cast<const uint4 *>(p + 16);
  }
}

// Slow path of one step at columns [j0, j0 + 64), as emit_mfma, for the row tiles in
// the bits of `hits`: the packed products are made again and their halves give
// both columns' dot products.
template <int W, int RT, bool COS>
__device__ __forceinline__ bool emit_two(const PRows<W, RT> &rw, const uint4 (&a)[2 * W],
                                         uint32_t hits, int scale, uint32_t j0,
                                         const ColRun &run, const TileJob &jb, uint32_t &skip,
                                         Sink &sink) {
  const uint32_t lane = threadIdx.x & 63;
  const bool bound = run.hi > run.lo || (COS && jb.cosine);
  uint32_t size = 0;
  uint64_t bits = 0;
  if (bound && j0 + lane < run.end) {  // for the exact tests; in flight during the products
    const ArgPtr ka = args();
    size = ka->size_cols[j0 + lane];
    bits = ka->bm_cols[j0 + lane];
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if (!((hits >> rt) & 1u)) continue;
    v16f_t d;
#pragma unroll
    for (int v = 0; v < 16; ++v) d[v] = __uint_as_float((kFieldHi << 16) + kFieldLo);
#pragma unroll
    for (int x = 0; x < 2 * W; ++x) d = mfma_two(a[x], rw.sg[rt][x], d, scale);
    const uint32_t thr_hi = rw.thr[rt] | 0xFFFFu;
    const uint16_t thr_lo = (uint16_t)rw.thr[rt];
    uint32_t k0 = 0, k1 = 0;  // columns j0 .. and j0 + 32 ..
#pragma unroll
    for (int v = 15; v >= 0; --v) {
      const uint32_t p = __float_as_uint(d[v]);
      k0 = (k0 << 1) | ((uint16_t)p > thr_lo ? 1u : 0u);
      k1 = (k1 << 1) | (p > thr_hi ? 1u : 0u);
    }
    const uint32_t k = k0 | (k1 << 16);
    sink.kept[64 * rt + lane] = k;
  }
  if (bound) {
    uint32_t *cols = sink.rows + 5 * kTwoRows + lane;
    cols[0] = size;
    cols[64] = (uint32_t)bits;
    cols[128] = (uint32_t)(bits >> 32);
  }
  __builtin_amdgcn_wave_barrier();
  return stage_step<2, COS>(hits, jb.row0, j0, run.end, jb, skip, sink, bound);
}

// Fast path of one step, as fast_mfma: the products run one row tile ahead of
// their reduction, across steps, in two accumulators (RT is even, so every
// step starts in the first).
template <int W, int RT>
__device__ __forceinline__ uint32_t fast_two(const uint4 (&a)[2 * W], const uint4 (&an)[2 * W],
                                             const PRows<W, RT> &rw, const v16f_t &c, int scale,
                                             v16f_t (&acc)[2]) {
  static_assert(RT % 2 == 0, "steps start in accumulator 0");
  uint32_t hits = 0;  // bit rt: row tile rt keeps something
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int cur = rt & 1, nxt = cur ^ 1;
    acc[nxt] = rt + 1 < RT ? products_two<W, RT>(a, rw, rt + 1, c, scale)
                           : products_two<W, RT>(an, rw, 0, c, scale);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t m = max17(acc[cur], rw.thr[rt]);
    hits |= __ballot(m != rw.thr[rt]) ? 1u << rt : 0u;
    __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("" ::"v"(acc[0]));
  return hits;
}

// The steps of columns [j, run.end), as sweep_mfma.
template <int W, int RT, bool COS>
__device__ __forceinline__ bool sweep_two(const uint4 *__restrict__ sg_cols, uint32_t n_cols,
                                          const PRows<W, RT> &rw, int scale, uint4 (&b0)[2 * W],
                                          uint4 (&b1)[2 * W], uint32_t j, const ColRun &run,
                                          const TileJob &jb, uint32_t &skip, Sink &sink) {
  const uint32_t g1 = run.end, loff = (threadIdx.x & 63u) * 32u;
  uint4 b2[2 * W];
  v16f_t acc[2];
  uint32_t j0 = j;
  for (;;) {
    int phase;
    uint32_t hits;
    uint4 cur[2 * W];
    // the start value's pattern in every register, made anew after each slow
    // path, which needs the registers
    v16f_t c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = __uint_as_float((kFieldHi << 16) + kFieldLo);
    asm volatile("" : "+v"(c));
    acc[0] = products_two<W, RT>(b0, rw, 0, c, scale);
    for (;;) {
      load_cols_two<W>(sg_cols, n_cols, j0 + 128, loff, b2);
      if (__builtin_expect((hits = fast_two<W, RT>(b0, b1, rw, c, scale, acc)) != 0, 0)) {
        phase = 0;
#pragma unroll
        for (int x = 0; x < 2 * W; ++x) cur[x] = b0[x];
        break;
      }
      skip = 0;
      if ((j0 += 64) >= g1) return true;
      load_cols_two<W>(sg_cols, n_cols, j0 + 128, loff, b0);
      if (__builtin_expect((hits = fast_two<W, RT>(b1, b2, rw, c, scale, acc)) != 0, 0)) {
        phase = 1;
#pragma unroll
        for (int x = 0; x < 2 * W; ++x) cur[x] = b1[x];
        break;
      }
      skip = 0;
      if ((j0 += 64) >= g1) return true;
      load_cols_two<W>(sg_cols, n_cols, j0 + 128, loff, b1);
      if (__builtin_expect((hits = fast_two<W, RT>(b2, b0, rw, c, scale, acc)) != 0, 0)) {
        phase = 2;
#pragma unroll
        for (int x = 0; x < 2 * W; ++x) cur[x] = b2[x];
        break;
      }
      skip = 0;
      if ((j0 += 64) >= g1) return true;
    }
    if (!emit_two<W, RT, COS>(rw, cur, hits, scale, j0, run, jb, skip, sink)) return false;
    skip = 0;
    if ((j0 += 64) >= g1) return true;
    // b0 and b1 take the columns of steps j0 and j0 + 64
#pragma unroll
    for (int x = 0; x < 2 * W; ++x) {
      const uint4 x0 = phase == 0 ? b1[x] : phase == 1 ? b2[x] : b0[x];
      const uint4 x1 = phase == 0 ? b2[x] : phase == 1 ? b0[x] : b1[x];
      b0[x] = x0;
      b1[x] = x1;
    }
  }
}

// One tile, as run_tile_mfma.
template <int W, int RT, bool COS>
__device__ __forceinline__ bool run_tile_two(const TileJob &jb, Sink &sink) {
  static_assert(W == 1, "wider dot products leave the start value's range");
  const ArgPtr ka = args();
  const uint4 *__restrict__ sg_rows = ka->sg_rows, *__restrict__ sg_cols = ka->sg_cols;
  const uint32_t *__restrict__ size_rows = ka->size_rows, *__restrict__ size_cols = ka->size_cols;
  const uint32_t n_rows = ka->cfg.n_rows, n_cols = ka->cfg.n_cols;
  const uint32_t lane = threadIdx.x & 63, jr = lane & 31;
  const int scale = lane < 32 ? 127 - 1 : 127 + 15;
  static_assert(32 * RT <= kTwoRows, "rows fit their LDS arrays");
  PRows<W, RT> rw;
  rw.row = reinterpret_cast<uint32_t(*)[kTwoRows]>(sink.rows);
  // Rows 64 x + lane for the LDS arrays, without branches (see run_tile_mfma).
  const uint32_t last = jb.row_end - 1;
  uint32_t size[RT / 2], lo[RT / 2], hi[RT / 2];
  uint64_t bits[RT / 2];
#pragma unroll
  for (int x = 0; x < RT / 2; ++x) {
    const uint32_t i = min(jb.row0 + 64u * x + lane, last);
    size[x] = size_rows[i];
    bits[x] = ka->bm_rows[i];
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const uint32_t i = jb.row0 + 32u * rt + jr;
    load_cols_two<W>(sg_rows, n_rows, i <= last ? i : n_rows, 0, rw.sg[rt]);
  }
#pragma unroll
  for (int x = 0; x < RT / 2; ++x) {
    lo[x] = jb.cmin[size[x]];
    hi[x] = jb.cmax[size[x]];
  }
#pragma unroll
  for (int x = 0; x < RT / 2; ++x) {
    const uint32_t r = 64u * x + lane;
    const bool ok = jb.row0 + r <= last;
    rw.row[0][r] = ok ? size[x] : 0u;
    rw.row[1][r] = ok ? lo[x] : 0xFFFFFFFFu;
    rw.row[2][r] = ok ? hi[x] : 0u;
    rw.row[3][r] = (uint32_t)bits[x];
    rw.row[4][r] = (uint32_t)(bits[x] >> 32);
  }
  __builtin_amdgcn_wave_barrier();
  uint32_t skip = jb.first;
  uint32_t j = jb.c0;
  const uint32_t loff = lane * 32u;
  uint32_t c = j < jb.c1 ? as_const(size_cols)[j] : 0u;
  uint32_t resumed_end = jb.end;
  while (j < jb.c1) {
    uint4 b0[2 * W], b1[2 * W];
    load_cols_two<W>(sg_cols, n_cols, j, loff, b0);
    load_cols_two<W>(sg_cols, n_cols, j + 64, loff, b1);
    ColRun run = col_run(jb.sstart, jb.col_base, jb.col_max, c, j, jb.c1);
    if (resumed_end) {
      run.end = min(max(resumed_end, j + 1), jb.c1);
      run.hi = as_const(size_cols)[run.end - 1];
      resumed_end = 0;
    }
    if (run.end < jb.c1) c = as_const(size_cols)[run.end];
    bool any_ok = false;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const uint32_t x = 32u * rt + jr, hi = rw.row[2][x];
      const bool in_band = run.lo <= hi && run.hi >= rw.row[1][x];
      // (slack[0] for a row outside the band, as in run_tile_mfma; -1: never)
      const int32_t sl = run_slack<COS>(jb, in_band ? rw.row[0][x] : 0u, run.lo,
                                        in_band ? min(run.hi, hi) : 0u);
      rw.thr[rt] = pack_threshold<W>(32 * W - (in_band ? sl : -1));
      any_ok |= in_band;
    }
    if (__ballot(any_ok)) {
      if (!sweep_two<W, RT, COS>(sg_cols, n_cols, rw, scale, b0, b1, j, run, jb, skip, sink))
        return false;
    }
    skip = 0;
    j = run.end;
  }
  // the tile's staged pairs go out before the next tile
  return flush(sink, true);
}

// Widths whose kernel takes two columns per accumulator, and the waves per SIMD
// the register budget of a width aims at.
constexpr bool two_columns(int w) { return w == 1; }
constexpr int mfma_waves(int w) { return w <= 2 ? 3 : w <= 4 ? 2 : 1; }

// LDS bytes of a wave.
template <int W>
constexpr uint32_t mfma_wave_lds() {
  return kStage * sizeof(uint2) + 64 * kMaxRowTiles * sizeof(uint32_t) +
         (two_columns(W) ? kTwoWords * sizeof(uint32_t) : 1024 * sizeof(int16_t));
}

template <int W, int RT, bool COS>
__global__ __launch_bounds__(kBlock, mfma_waves(W)) void k_filter_mfma(FilterArgs) {
  static_assert(RT <= kMaxRowTiles, "kept values of every row tile");
  // per wave: kStage entries, kept values, the rows' sizes and bands or dot products
  extern __shared__ uint2 stage[];
  // The wave's number is uniform: left to the compiler the three addresses take vector
  // registers, which the kernel of 1024 bits has none of to spare.  (At 128 bits scalar
  // ones, moved to vector registers where they are used, cost a batch's class 4%.)
  uint32_t wave = threadIdx.x >> 6;
  if (W >= 16) wave = rfl(wave);
  uint2 *mine = stage + wave * (mfma_wave_lds<W>() / sizeof(uint2));
  Sink sink;
  sink_init(sink, mine, reinterpret_cast<uint32_t *>(mine + kStage),
            reinterpret_cast<uint32_t *>(mine + kStage + 32 * kMaxRowTiles));
  tile_loop(sink, [&](const TileJob &jb) {
    if constexpr (two_columns(W)) return run_tile_two<W, RT, COS>(jb, sink);
    else return run_tile_mfma<W, RT, COS>(jb, sink);
  });
}

template <int W, int R, int U, bool COS>
hipError_t launch_shape(dim3 grid, hipStream_t st, const FilterArgs &a) {
  hipLaunchKernelGGL((k_filter<W, R, U, COS>), grid, dim3(64 * a.cfg.block_waves),
                     a.cfg.block_waves * kStage * sizeof(uint2), st, a);
  return hipGetLastError();
}

template <int W, int RT, bool COS>
hipError_t launch_mfma(dim3 grid, hipStream_t st, const FilterArgs &a) {
  hipLaunchKernelGGL((k_filter_mfma<W, RT, COS>), grid, dim3(64 * a.cfg.block_waves),
                     a.cfg.block_waves * mfma_wave_lds<W>(), st, a);
  return hipGetLastError();
}

// Vector-ALU kernels: (padded words, rows per lane, columns per step)
#define SSJ_FILTER_SHAPES(X) \
  X(1, 4, 4)                 \
  X(2, 2, 4)                 \
  X(3, 2, 2)                 \
  X(4, 2, 2)                 \
  X(5, 1, 1)                 \
  X(6, 1, 1)                 \
  X(7, 1, 1)                 \
  X(8, 1, 1)                 \
  X(10, 1, 1)                \
  X(12, 1, 1)                \
  X(16, 1, 1)                \
  X(20, 1, 1)                \
  X(24, 1, 1)                \
  X(32, 1, 1)                \
  X(40, 1, 1)                \
  X(48, 1, 1)                \
  X(64, 1, 1)

// Matrix-core kernels: (words, row tiles of 32 per wave).  At b = 64 six row
// tiles (three waves per SIMD) beat four (four waves per SIMD): a column
// step's loads, loop control and tests serve six products instead of four.
// At b = 128 four row tiles (three waves per SIMD) and at b = 256 five (two
// waves per SIMD) are the most the registers allow at that occupancy; six,
// at one wave fewer per SIMD, were slower.  At b = 512 and 1024 a column step streams b/2 bytes of sign planes per
// column, shared by the 32 RT rows of the wave: four and two row tiles
// (one wave per SIMD, the register file's other half holding rows and
// column buffers) keep that stream within what L2 delivers, and beat the
// vector ALUs by 3.2x and 1.8x.  b = 2048 stays on the vector ALUs: its
// ring of column buffers alone would fill the registers.
#define SSJ_MFMA_SHAPES(X) \
  X(1, 6)                  \
  X(2, 4)                  \
  X(4, 5)                  \
  X(8, 4)                  \
  X(16, 2)

}  // namespace

uint32_t filter_padded_words(uint32_t words) {
#define X(w, r, u) \
  if (words <= (w)) return (w);
  SSJ_FILTER_SHAPES(X)
#undef X
  return 0;
}

FilterShape filter_shape(uint32_t padded_words, bool mfma) {
  FilterShape s{0, 0, false};
#define X(w, r, u)           \
  if (padded_words == (w)) { \
    s.words = (w);           \
    s.rows = 64 * (r);       \
  }
  SSJ_FILTER_SHAPES(X)
#undef X
  if (mfma) {
#define X(w, rt)                           \
  if (padded_words == (w)) {               \
    s.rows = 32 * (rt);                    \
    s.mfma = true;                         \
  }
    SSJ_MFMA_SHAPES(X)
#undef X
  }
  return s;
}

int filter_grid_blocks() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1024;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  return cus * 8;  // 32 waves per CU
}

uint32_t mfma_resident_waves(uint32_t words) {
  return (uint32_t)filter_grid_blocks() / 8 * 4 * (uint32_t)mfma_waves((int)words);
}

hipError_t launch_filter(uint32_t padded_words, bool cosine, const FilterArgs &args_in,
                         hipStream_t st) {
  FilterArgs a = args_in;
  // a persistent grid, but no more waves than the launch has tiles or resume
  // entries to hand out (small width classes would otherwise start thousands
  // of waves that find nothing to do); a direct launch has a wave for every
  // tile of its XCDs' regions, or for every resume entry
  const uint64_t n_tiles = a.cfg.tile_hi - a.cfg.tile_lo;
  const uint64_t waves_per_block = a.cfg.direct ? 1 : kBlock / 64;
  if (a.cfg.stripes == 0 || (a.cfg.stripes & (a.cfg.stripes - 1)) ||
      a.cfg.stripes > kQueueStripes)
    return hipErrorInvalidValue;
  dim3 grid;
  if (a.cfg.direct && a.cfg.n_resume_in == 0) {
    constexpr uint64_t kTurn = kXcds * kDirectDeal;
    grid = dim3((unsigned)(kTurn * ((n_tiles + kTurn - 1) / kTurn)));
  } else {
    // (A direct launch of the matrix-core kernel that resumes: no more waves than the GPU
    // holds.  Each costs a round that fills the queue two atomics on one address,
    // a slot reservation that fails and one of resume entries.)
    const uint64_t most = a.cfg.direct && a.sg_rows ? mfma_resident_waves(padded_words)
                                                    : (uint64_t)filter_grid_blocks() * (kBlock / 64);
    const uint64_t need = std::max<uint64_t>(
        a.cfg.direct ? a.cfg.n_resume_in : std::max<uint64_t>(n_tiles, a.cfg.n_resume_in), 1);
    grid = dim3((unsigned)std::min<uint64_t>(most / waves_per_block,
                                             (need + waves_per_block - 1) / waves_per_block));
  }
  a.cfg.block_waves = (uint32_t)waves_per_block;
  a.cfg.waves = grid.x * (uint32_t)waves_per_block;
  a.cfg.chunk = std::max(a.cfg.chunk, kFilterStage);
  if (a.sg_rows || a.sg_cols) {
    if (!a.sg_rows || !a.sg_cols) return hipErrorInvalidValue;
#define X(w, rt)                                                \
  if (padded_words == (w))                                      \
    return cosine ? launch_mfma<w, rt, true>(grid, st, a)       \
                  : launch_mfma<w, rt, false>(grid, st, a);
    SSJ_MFMA_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
  }
#define X(w, r, u)                                              \
  if (padded_words == (w))                                      \
    return cosine ? launch_shape<w, r, u, true>(grid, st, a)    \
                  : launch_shape<w, r, u, false>(grid, st, a);
  SSJ_FILTER_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace ssj
