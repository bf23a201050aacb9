// Criticality, the top-n_keep select and the learned gate of the sparse
// injection (arXiv 2607.16305, Sec. 3.3, Eq. 9-10): the bodies shared by the stand-alone
// kernels (inject.hip) and by the launches that carry them beside the
// bucketing and the Level-2 scoring of small batches (bucket.hip, score.hip),
// so that all give the same bits.
//
//   row_sumsq    one wave streams a row of Delta once (NORM_UNROLL 16-byte
//                loads of a lane in flight) and returns its fp32 sum of
//                squares, accumulated in a fixed order; stored as its bit
//                pattern, it orders like the norm (non-negative floats order
//                like their bits, and the square root keeps the order);
//   select_layer one workgroup (1024, 512 or 256 threads): MSB-first radix
//                select of the n_keep-th largest key in at most four passes
//                (keys cached in LDS when they fit), then an order-preserving
//                compaction (ballots and prefix sums) of the kept token ids;
//   row_dot, gate_compact_layer  the learned SKA gate's logit z = Delta_i W_g
//                and the ascending compaction of its open rows (Eq. 9).
#pragma once

#include "common.h"

namespace lookme {

constexpr int NORM_UNROLL = 4;
constexpr int SEL_THREADS = 1024;
constexpr int SEL_WAVES = SEL_THREADS / WAVE;

// CN > 0: a layer's keys (n <= CN) are first copied to LDS, so that the four
// passes and the compaction read them there instead of from L2 (one global
// round trip instead of five).  Launchers take the smallest cache that holds
// n: the smaller ones leave room on the CU for the workgroups of a kernel that
// runs beside the select.
constexpr int SEL_CACHE_SMALL = 4096, SEL_CACHE_MID = 8192, SEL_CACHE_N = 32768;

template <int DT>
__device__ __forceinline__ float row_sumsq(const char* __restrict__ p, int chunks, int lane) {
  float acc0 = 0.f, acc1 = 0.f;
  // chunks past the row re-read its last chunk and are not summed (a
  // 4096-element bf16 row is two rounds)
  for (int c0 = lane; c0 < chunks; c0 += NORM_UNROLL * WAVE) {
    u32x4_t vv[NORM_UNROLL];
#pragma unroll
    for (int u = 0; u < NORM_UNROLL; ++u) {
      const int c = c0 + u * WAVE;
      vv[u] = ld16_nt(p + (int64_t)(c < chunks ? c : chunks - 1) * 16);
    }
#pragma unroll
    for (int u = 0; u < NORM_UNROLL; ++u) {
      if (c0 + u * WAVE >= chunks) continue;
      const u32x4_t v = vv[u];
      if constexpr (DT == DT_BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = bf16lo(v[e]), hi = bf16hi(v[e]);
          acc0 = fmaf(lo, lo, acc0);
          acc1 = fmaf(hi, hi, acc1);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float f = as_f32(v[e]);
          if (e & 1) acc1 = fmaf(f, f, acc1);
          else acc0 = fmaf(f, f, acc0);
        }
      }
    }
  }
  float acc = acc0 + acc1;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
  return acc;
}

// z = row . w (the SKA gate's logit of Eq. 9) by one wave: NORM_UNROLL 16-byte
// loads of the row and of w in flight per lane, fp32 fused multiply-adds in a
// fixed order, then the wave sum.
template <int DT>
__device__ __forceinline__ float row_dot(const char* __restrict__ p, const char* __restrict__ w,
                                         int chunks, int lane) {
  float acc = 0.f;
  for (int c0 = lane; c0 < chunks; c0 += NORM_UNROLL * WAVE) {
    u32x4_t dv[NORM_UNROLL], wv[NORM_UNROLL];
#pragma unroll
    for (int u = 0; u < NORM_UNROLL; ++u) {
      const int c = c0 + u * WAVE;
      const int cc = c < chunks ? c : chunks - 1;
      dv[u] = ld16_nt(p + (int64_t)cc * 16);
      wv[u] = ld16(w + (int64_t)cc * 16);
    }
#pragma unroll
    for (int u = 0; u < NORM_UNROLL; ++u) {
      if (c0 + u * WAVE >= chunks) continue;
      if constexpr (DT == DT_BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc = fmaf(bf16lo(dv[u][e]), bf16lo(wv[u][e]), acc);
          acc = fmaf(bf16hi(dv[u][e]), bf16hi(wv[u][e]), acc);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = fmaf(as_f32(dv[u][e]), as_f32(wv[u][e]), acc);
      }
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
  return acc;
}

// LDS words the select and the gate compaction work in (counts, scan
// partials, the located prefix).  The caller passes them: a kernel that
// also stages operands by direct-to-LDS loads keeps all of its LDS in one
// object (with several, the compiler puts a load wait before every LDS read
// that follows those loads).
constexpr int SEL_COPIES = 8;
struct SelLds {
  int hist[256 * SEL_COPIES];   // copy c of bin b at 8 b + c
  int wsum[SEL_WAVES];
  uint32_t prefix;
  int need;
  int total;
  int listed;
};

// Bits of m below the calling lane's.
__device__ __forceinline__ int bits_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// The open gates of one layer in ascending order (Eq. 9-10: z > 0; z = 0
// stays closed): a wave owns consecutive groups of 64 rows, whose signs are
// one ballot each (lane t keeps group t's), prefix sums of the counts over
// lanes and waves place them, and each group's open rows are written side by
// side; kept[count .. n) = -1 and *count = the number open.  Called by all
// THREADS threads of a workgroup.  One workgroup is bound by latency: eight
// coalesced loads of a wave in flight (23040 rows 18.1 -> 10.8 us; with 32
// rows a thread, each lane's loads had lines of their own).
template <int THREADS>
__device__ __forceinline__ void gate_compact_layer(const float* __restrict__ z, int64_t n,
                                                   int32_t* __restrict__ kept,
                                                   int32_t* __restrict__ count, SelLds& sl) {
  constexpr int WAVES = THREADS / WAVE, BATCH = 8;
  constexpr int64_t SPAN = (int64_t)THREADS * WAVE;   // rows a round: 64 groups a wave
  static_assert(WAVES <= SEL_WAVES, "scan partials");
  int* wsum = sl.wsum;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  int64_t base = 0;   // open rows in earlier rounds
  for (int64_t r0 = 0; r0 < n; r0 += SPAN) {
    const int64_t left = n - r0 < SPAN ? n - r0 : SPAN;
    const int per = (int)(((left + 63) / 64 + WAVES - 1) / WAVES);   // groups a wave, at most 64
    const int64_t w0 = r0 + (int64_t)wv * per * 64;
    uint64_t mine = 0;   // lane t: the open rows of group t
    for (int t0 = 0; t0 < per; t0 += BATCH) {
      float v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {   // every load issued, none under a branch
        const int64_t i = w0 + (t0 + u) * 64 + lane;
        v[u] = z[i < n ? i : n - 1];
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int64_t i = w0 + (t0 + u) * 64 + lane;
        const uint64_t m = __ballot(t0 + u < per && i < r0 + left && v[u] > 0.f);
        mine = lane == t0 + u ? m : mine;
      }
    }
    const int c = __popcll(mine);
    const int incl = wave_scan_incl(c);
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int64_t off = base;
    int total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      off += w < wv ? wsum[w] : 0;
      total += wsum[w];
    }
    for (int t = 0; t < per; ++t) {
      const uint64_t m = __shfl(mine, t, 64);
      const int64_t at = off + __shfl(incl - c, t, 64);
      if (m >> lane & 1) kept[at + bits_below(m)] = (int32_t)(w0 + t * 64 + lane);
    }
    base += total;
    __syncthreads();   // wsum is rewritten by the next round
  }
  for (int64_t i = base + tid; i < n; i += THREADS) kept[i] = -1;
  if (tid == 0) *count = (int32_t)base;
}

// LDS words of select_layer's key cache for CN keys.
constexpr int sel_cache_words(int cn) { return cn > 0 ? cn : 1; }

// The kept set of one layer: kept[0 .. n_keep) = the n_keep tokens of
// largest key (ties: lowest token), ascending.  Called by all THREADS (a
// multiple of 256) threads of a workgroup; cache: sel_cache_words(CN) words
// of LDS.  One workgroup is bound by its vector instructions and the latency
// of its LDS reads (32768 keys: 32 a thread), so: 32-bit indices, a wave's
// keys read side by side, bins in eight copies (a lane adds to copy lane mod
// 8: keys of one batch share few leading digits, and adds to one LDS word go
// one after the other), and once two digits are known the keys that share them
// are ranked directly, if they are few, instead of by two more passes over all
// keys.  32768 keys 41 -> 28 us, 4 x 23040 32 -> 19.  Few: the ranking compares
// each with each, 256 take about one of the passes they save (norms within 6%
// of one another: with up to 1024 ranked, 4 x 23040 keys took 32.5 us and 32768
// 47.0, with 256 26.5 and 33.2).  The positions stay below n_keep as long as
// the keys do not change during the launch; the comparison that makes sure of
// it takes 0.3 us of 4 x 23040 keys.
template <int CN, int THREADS = SEL_THREADS>
__device__ __forceinline__ void select_layer(const uint32_t* __restrict__ gkey, int64_t n64,
                                             int64_t n_keep64, int32_t* __restrict__ kept,
                                             uint32_t* cache, SelLds& sl) {
  constexpr bool CACHED = CN > 0;
  constexpr int WAVES = THREADS / WAVE, BATCH = 8;
  constexpr int LIST = 256;   // keys ranked directly, in the bins' words
  static_assert(THREADS % 256 == 0, "a thread per radix bin");
  static_assert(WAVES <= SEL_WAVES && LIST <= 256 * SEL_COPIES, "scan partials, list");
  int* hist = sl.hist;
  int* wsum = sl.wsum;
  if (n_keep64 == 0) return;
  const int n = (int)n64, n_keep = (int)n_keep64;   // at most 2^30 rows a call
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (CACHED) {
    for (int i0 = tid; i0 < n; i0 += THREADS * BATCH) {
      uint32_t v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int i = i0 + u * THREADS;
        v[u] = gkey[i < n ? i : n - 1];
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u)
        if (i0 + u * THREADS < n) cache[i0 + u * THREADS] = v[u];
    }
  }
  // the wave's keys [w0, w1), 64 side by side at a time
  const int per = ((n + 63) / 64 + WAVES - 1) / WAVES * 64;
  const int w0 = wv * per, w1 = w0 + per < n ? w0 + per : n;
  auto each = [&](auto&& f) {
    if constexpr (CACHED) {
      for (int i = w0 + lane; i < w1; i += WAVE) f(i, cache[i]);
    } else {
      for (int j = w0 + lane; j < w1; j += WAVE * BATCH) {
        uint32_t v[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) v[u] = gkey[j + u * WAVE < w1 ? j + u * WAVE : w1 - 1];
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
          if (j + u * WAVE < w1) f(j + u * WAVE, v[u]);
      }
    }
  };

  // ---- radix select (MSB first, 8 bits a pass): the n_keep-th largest T ----
  uint32_t prefix = 0, mask = 0;
  int need = n_keep;   // rank from the top still to be located
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    for (int b = tid; b < 256 * SEL_COPIES; b += THREADS) hist[b] = 0;
    __syncthreads();
    each([&](int, uint32_t k) {
      if ((k & mask) == prefix)
        atomicAdd(&hist[((k >> shift) & 255) * SEL_COPIES + (lane & (SEL_COPIES - 1))], 1);
    });
    __syncthreads();
    // thread t looks at bin 255 - t: cum = keys in bins >= that bin
    const int b = 255 - tid;
    int h = 0;
    if (tid < 256) {
#pragma unroll
      for (int c = 0; c < SEL_COPIES; ++c) h += hist[b * SEL_COPIES + c];
    }
    const int cum = block_scan_incl<4>(h, wsum);
    if (tid < 256 && cum - h < need && need <= cum) {
      sl.prefix = prefix | ((uint32_t)b << shift);
      sl.need = need - (cum - h);
      sl.total = h;
    }
    if (tid == 0) sl.listed = 0;
    __syncthreads();
    prefix = sl.prefix;
    need = sl.need;
    mask |= 255u << shift;
    const int left = sl.total;   // keys that share the digits found so far
    if (pass == 1 && left <= LIST) {
      // every one of them into a list, then each key's rank in it
      each([&](int, uint32_t k) {
        if ((k & mask) == prefix) {
          const int at = atomicAdd(&sl.listed, 1);
          if (at < LIST) hist[at] = (int)k;
        }
      });
      __syncthreads();
      for (int t = tid; t < left; t += THREADS) {
        const uint32_t x = (uint32_t)hist[t];
        int gt = 0, ge = 0;
        for (int j = 0; j < left; ++j) {
          const uint32_t y = (uint32_t)hist[j];
          gt += y > x;
          ge += y >= x;
        }
        if (gt < need && need <= ge) {   // equal keys store equal values
          sl.prefix = x;
          sl.total = need - gt;
        }
      }
      __syncthreads();
      prefix = sl.prefix;
      need = sl.total;
      break;
    }
  }
  const uint32_t T = prefix;   // kept: keys > T, plus the first `need` keys == T
  const int take_eq = need;

  // ---- order-preserving compaction: the waves' counts, then ballots ----
  int n_gt = 0, n_eq = 0;
  each([&](int, uint32_t k) {
    n_gt += k > T;
    n_eq += k == T;
  });
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    n_gt += __shfl_xor(n_gt, d, 64);
    n_eq += __shfl_xor(n_eq, d, 64);
  }
  __syncthreads();   // the list is read no more
  if (lane == 0) {
    hist[wv] = n_gt;
    hist[SEL_WAVES + wv] = n_eq;
  }
  __syncthreads();
  int g = 0, e = 0;   // keys above T (equal to T) before the wave's
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    g += w < wv ? hist[w] : 0;
    e += w < wv ? hist[SEL_WAVES + w] : 0;
  }
  g = __builtin_amdgcn_readfirstlane(g);
  e = __builtin_amdgcn_readfirstlane(e);
  each([&](int i, uint32_t k) {
    const uint64_t mg = __ballot(k > T), me = __ballot(k == T);
    if (k > T) {
      const int at = g + bits_below(mg) + min(e + bits_below(me), take_eq);
      if (at < n_keep) kept[at] = i;
    }
    if (me != 0) {
      const int eb = e + bits_below(me), at = g + bits_below(mg) + eb;
      if (k == T && eb < take_eq && at < n_keep) kept[at] = i;
      e += __popcll(me);
    }
    g += __popcll(mg);
  });
}

}  // namespace lookme
