// One-workgroup kernels for calls whose rows, or whose results, are few: the
// whole preparation of a small space in one launch, and the end of a join
// (counters to the host, and a short result list sorted and written there).
//
// What bounds them is latency: a small call spends its time on launches,
// copies and host waits, not on its few thousand sets.  Sorted by the general
// kernels, a space of 1,000 sets takes 10 launches, four copies and two host
// waits; here one launch and one wait.  Both kernels keep their keys in LDS
// and write what the host needs to page-locked memory, so that no copy is
// enqueued and the host only waits for the stream.
#include <cstddef>

#include "ssj_internal.h"

namespace ssj {
namespace {

constexpr int kThreads = 1024;
constexpr int kSmallWaves = kThreads / 64;

// Counters of a block sort: per wave and digit.
struct SortScratch {
  uint16_t cnt[kSmallWaves][256];
  uint32_t base[256];
  uint32_t wtot[4];
};

// Stable LSD radix sort, 8 bits per pass, of the n (at most 64 * kSmallWaves *
// ITEMS) elements 0 .. n - 1 whose keys key(x) are `bits` bits wide: every wave
// ranks its contiguous share, 64 keys at a time, peers with one digit found by
// eight ballots.  move(x, pos) copies element x to place pos of the other
// buffer, flip() swaps the buffers.  Every thread of the workgroup calls it.
template <int ITEMS, class Key, class Move, class Flip>
__device__ __forceinline__ void block_sort(uint32_t n, int bits, SortScratch &s, Key &&key,
                                           Move &&move, Flip &&flip) {
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t share = (n + kThreads - 1) / kThreads * 64;  // keys of a wave
  const unsigned long long below = __lanemask_lt();
  for (int shift = 0; shift < bits; shift += 8) {
    for (uint32_t i = threadIdx.x; i < kSmallWaves * 256; i += kThreads) (&s.cnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t dig[ITEMS], rank[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      dig[it] = rank[it] = 0;
      if ((uint32_t)it * 64 >= share) continue;  // the same in every thread
      const uint32_t x = w * share + it * 64 + lane;
      const bool valid = x < n;
      const uint32_t d = valid ? (uint32_t)(key(x) >> shift) & 0xFFu : 0u;
      unsigned long long peers = __ballot(valid);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const unsigned long long set = __ballot((d >> b) & 1u);
        peers &= ((d >> b) & 1u) ? set : ~set;
      }
      // the wave's count of the digit: every peer reads it before the highest of them
      // advances it, and the next 64 keys read it after that
      const uint32_t prior = s.cnt[w][d];
      __builtin_amdgcn_wave_barrier();
      dig[it] = d;
      rank[it] = prior + (uint32_t)__popcll(peers & below);
      if (valid && (peers >> lane) == 1ull)
        s.cnt[w][d] = (uint16_t)(prior + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // digit totals, the waves' offsets inside a digit, and the digits' bases
    uint32_t tot = 0, inc = 0;
    if (threadIdx.x < 256) {
#pragma unroll
      for (int v = 0; v < kSmallWaves; ++v) {
        const uint32_t c = s.cnt[v][threadIdx.x];
        s.cnt[v][threadIdx.x] = (uint16_t)tot;
        tot += c;
      }
      inc = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += v;
      }
      if (lane == 63) s.wtot[w] = inc;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
      uint32_t pre = 0;
      for (uint32_t v = 0; v < w; ++v) pre += s.wtot[v];
      s.base[threadIdx.x] = pre + inc - tot;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const uint32_t x = w * share + it * 64 + lane;
      if ((uint32_t)it * 64 < share && x < n)
        move(x, s.base[dig[it]] + s.cnt[w][dig[it]] + rank[it]);
    }
    __syncthreads();
    flip();
  }
}

// Number of the n ascending keys key(0) .. key(n - 1) below v.
template <class T, class Key>
__device__ __forceinline__ uint32_t lower_bound(uint32_t n, T v, Key &&key) {
  uint32_t lo = 0, hi = n;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (key(mid) < v) lo = mid + 1; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int bit_width(uint32_t v) { return 32 - __clz((int)v); }

__global__ __launch_bounds__(kThreads) void k_prepare_small(SmallSpace a) {
  __shared__ uint32_t k32[2][kSmallSets];
  __shared__ uint16_t idx[2][kSmallSets];
  __shared__ uint32_t sbase[kSmallSides];
  __shared__ SortScratch scratch;
  __shared__ uint32_t s_max, s_err;
  const uint32_t tid = threadIdx.x, n = a.n;
  for (uint32_t i = tid; i < sizeof(JoinCounters) / 16; i += kThreads)
    reinterpret_cast<uint4 *>(a.ctr)[i] = make_uint4(0, 0, 0, 0);
  for (uint32_t s = tid; s < a.n_sides; s += kThreads) {
    const SideDesc d = a.h_sides[s];
    a.d_sides[s] = d;
    sbase[s] = (uint32_t)d.base;
  }
  if (tid == 0) s_max = s_err = 0;
  __threadfence();  // d_sides is read back below
  __syncthreads();
  // sizes, offsets checked: the checks of k_set_sizes
  constexpr int kItems = kSmallSets / kThreads;
  uint32_t sz[kItems], sid[kItems], err = 0, mx = 0;
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const uint32_t g = it * kThreads + tid;
    sz[it] = sid[it] = 0;
    if (g >= n) continue;
    uint32_t lo = 0, hi = a.n_sides;  // the last side whose base is <= g
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (sbase[mid] <= g) lo = mid; else hi = mid;
    }
    sid[it] = lo;
    const SideDesc sd = a.d_sides[lo];
    const uint64_t k = g - sd.base;
    const uint64_t o0 = sd.offsets[k], o1 = sd.offsets[k + 1];
    if (k == 0 && o0 != 0) err |= kErrOffsets;
    if (k == sd.n - 1 && o1 != sd.n_tokens) err |= kErrOffsets;
    if (o1 < o0 || o1 > sd.n_tokens) err |= kErrOffsets;
    else sz[it] = (uint32_t)(o1 - o0);  // n_tokens fits 32 bits here
    mx = max(mx, sz[it]);
  }
  if (mx) atomicMax(&s_max, mx);
  if (err) atomicOr(&s_err, err);
  __syncthreads();
  const uint32_t max_size = s_max;
  const int size_bits = max(1, bit_width(max_size)), side_bits = bit_width(a.n_sides - 1);
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const uint32_t g = it * kThreads + tid;
    if (g >= n) continue;
    k32[0][g] = (sid[it] << size_bits) | sz[it];
    idx[0][g] = (uint16_t)g;
  }
  __syncthreads();
  uint32_t cur = 0;
  block_sort<kItems>(
      n, size_bits + side_bits, scratch, [&](uint32_t x) { return k32[cur][x]; },
      [&](uint32_t x, uint32_t pos) {
        k32[cur ^ 1][pos] = k32[cur][x];
        idx[cur ^ 1][pos] = idx[cur][x];
      },
      [&]() { cur ^= 1; });
  const uint32_t mask = (1u << size_bits) - 1;
  for (uint32_t x = tid; x < n; x += kThreads) {
    const uint32_t key = k32[cur][x], g = idx[cur][x], s = key >> size_bits;
    a.sizes[x] = key & mask;
    a.side_of[x] = s;
    a.perm[x] = g - sbase[s];
    a.rank[g] = x;
  }
  // group starts: sets of side s below (s, v), from the side's base
  const uint32_t stride = max_size + 2, entries = a.n_sides * stride;
  for (uint32_t e = tid; e < entries; e += kThreads) {
    const uint32_t s = e / stride, v = e - s * stride;
    const uint32_t end = s + 1 < a.n_sides ? sbase[s + 1] : n;
    const uint32_t pos =
        v > max_size ? end
                     : max(lower_bound(n, (s << size_bits) | v,
                                       [&](uint32_t x) { return k32[cur][x]; }),
                           sbase[s]);
    a.sstart[e] = pos - sbase[s];
    a.h_sstart[e] = pos - sbase[s];
  }
  if (tid == 0) {
    a.h_head->error = s_err;
    a.h_head->max_size = max_size;
    a.ctr->error = s_err;
  }
}

__global__ __launch_bounds__(kThreads) void k_finish(FinishArgs a) {
  __shared__ unsigned long long buf[2][kSmallResults];
  __shared__ SortScratch scratch;
  const uint32_t tid = threadIdx.x;
  constexpr uint32_t kWords = offsetof(JoinCounters, queue_next) / 4;
  const uint32_t *src = reinterpret_cast<const uint32_t *>(a.ctr);
  for (uint32_t i = tid; i < kWords; i += kThreads) a.h_ctr[i] = src[i];
  const unsigned long long count = a.ctr->results;
  if (a.ctr->error || a.ctr->overflow || count == 0 || count > a.max_results) return;
  const uint32_t n = (uint32_t)count;  // at most kSmallResults
  for (uint32_t x = tid; x < n; x += kThreads) buf[0][x] = a.keys[x];
  __syncthreads();
  uint32_t cur = 0;
  block_sort<kSmallResults / kThreads>(
      n, a.bits, scratch, [&](uint32_t x) { return buf[cur][x]; },
      [&](uint32_t x, uint32_t pos) { buf[cur ^ 1][pos] = buf[cur][x]; }, [&]() { cur ^= 1; });
  const int tshift = a.ib + a.jb;
  for (uint32_t x = tid; x < n; x += kThreads) {
    const unsigned long long k = buf[cur][x];
    ssj_pair pr;
    pr.i = (uint32_t)((k >> a.jb) & ((1ull << a.ib) - 1));
    pr.j = (uint32_t)(k & ((1ull << a.jb) - 1));
    a.h_pairs[x] = pr;
  }
  for (uint32_t t = tid; t <= a.n_tasks; t += kThreads)
    a.h_start[t] = t == a.n_tasks ? n
                   : t == 0       ? 0
                                  : lower_bound(n, (unsigned long long)t << tshift,
                                                [&](uint32_t x) { return buf[cur][x]; });
}

}  // namespace

hipError_t launch_prepare_small(const SmallSpace &a, hipStream_t st) {
  if (a.n == 0 || a.n > kSmallSets || a.n_sides == 0 || a.n_sides > kSmallSides)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_prepare_small, dim3(1), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_finish(const FinishArgs &a, hipStream_t st) {
  if (a.max_results > kSmallResults || a.ib < 1 || a.jb < 1 || a.ib > 32 || a.jb > 32 ||
      a.bits > 64)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_finish, dim3(1), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace ssj
