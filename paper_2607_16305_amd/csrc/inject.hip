// Sparse injection (arXiv 2607.16305, Sec. 3.3, Eq. 9-10) and the residual
// add of Eq. 2: the criticality of token t is ||Delta_t||_2 (the size of the
// attention update that drives the SKA gate); the n_keep most critical tokens
// of every layer receive H[t, :d_v] += sum_i w_i * V[scene_t * P + p_i, :].
//
//   crit_norm   one wave per row streams Delta once (HBM-bound) and stores
//               the fp32 sum of squares as its bit pattern (non-negative
//               floats order like their bits, and the square root keeps the
//               order, so selecting on it selects on the norm);
//   crit_select one workgroup per layer: MSB-first radix select of the
//               n_keep-th largest key (keys cached in LDS when they fit), then
//               an order-preserving compaction of the kept token ids (crit.h);
//   ms_mix      one workgroup per kept token: the multi-scale router's mix of
//               the token's rows (multiscale.hip);
//   inject      one workgroup per kept token (one thread per 16-byte chunk of
//               a row, up to 256): coalesced loads of its k table rows (all
//               in flight together), fp32 weighted sum in a fixed order, one
//               rounding of H + sum, in-place store.  The table rows are read
//               with the normal cache policy: tokens of one scene pick many of
//               the same primitives (the Zipf batch's 104864 gathered rows are
//               30680 distinct ones), and the caches serve the repeats (with
//               the nontemporal hint the kernel took 44.7 us there, without
//               27.4 us; multi-scale 23.2 -> 19.0, 4-layer 73.3 -> 65.5).
#include "common.h"
#include "crit.h"
#include "kernels.h"

namespace lookme {

constexpr int NORM_WAVES = 4;
constexpr int64_t NORM_BACKGROUND_WGS = 256;
constexpr int INJ_THREADS = 256;

template <int DT>
__global__ __launch_bounds__(NORM_WAVES * WAVE) void crit_norm_kernel(
    const char* __restrict__ crit, int64_t rows, int64_t row_bytes,
    uint32_t* __restrict__ key) {
  const int lane = threadIdx.x & 63;
  for (int64_t r = (int64_t)blockIdx.x * NORM_WAVES + (threadIdx.x >> 6); r < rows;
       r += (int64_t)gridDim.x * NORM_WAVES) {
    const float acc = row_sumsq<DT>(crit + r * row_bytes, (int)(row_bytes / 16), lane);
    if (lane == 0) key[r] = as_u32(acc);
  }
}

template <int CN, int THREADS = SEL_THREADS>
__global__ __launch_bounds__(THREADS) void crit_select_kernel(
    const uint32_t* __restrict__ key_all, int64_t n, int64_t n_keep,
    int32_t* __restrict__ kept_all) {
  __shared__ uint32_t cache[sel_cache_words(CN)];
  __shared__ SelLds sl;
  const int layer = blockIdx.x;
  select_layer<CN, THREADS>(key_all + (int64_t)layer * n, n, n_keep,
                            kept_all + (int64_t)layer * n_keep, cache, sl);
}

// Rows of the injections whose kept id, scene or primitive index lay outside
// its range since the counter was last read (lookme_index_errors): such a
// row is not injected (in TO_R form its R row is written as zeros), so a
// caller's bad index is counted instead of adding some other row into H.
__device__ unsigned long long g_index_errors;

// TO_R: the weighted row sum R of kept row j is rounded to the storage
// dtype and written to row j of `hidden` (the fusion's or the multi-scale
// router's input, [rows, d_v]) instead of being added into H.  Layer l reads
// its kept list at kept + l * kept_batch (0: one list for all layers) and
// its scenes (in [0, S)) from scene l * scene_step of the table (multi-scale:
// scale l's partition).  With a count array only the first count entries of
// a kept list are used (count[l], or count[0] for a list shared by all
// layers).
template <int DT, int K, bool TO_R = false>
__global__ __launch_bounds__(INJ_THREADS) void inject_kernel(
    int64_t n, int64_t n_keep, const int32_t* __restrict__ kept_all,
    const int32_t* __restrict__ scene_all, const int32_t* __restrict__ prim_all,
    const float* __restrict__ w_all, const char* __restrict__ values, int S, int P, int k,
    int64_t v_bytes, char* __restrict__ hidden, int64_t h_bytes, int64_t kept_batch,
    int scene_step, const int32_t* __restrict__ count) {
  const int64_t j = blockIdx.x;
  const int64_t layer = j / n_keep;
  // counted lists (the learned gate): entries past the list's count are unused
  if (count != nullptr && j - layer * n_keep >= count[kept_batch != 0 ? layer : 0]) return;
  const int chunks = (int)(v_bytes / 16);
  // an index out of range: count the row once and leave it out (every
  // index below is uniform over the workgroup)
  auto reject = [&]() {
    if (threadIdx.x == 0) atomicAdd(&g_index_errors, 1ull);
    if constexpr (TO_R)
      for (int c = threadIdx.x; c < chunks; c += blockDim.x)
        st16(hidden + j * v_bytes + (int64_t)c * 16, u32x4_t{0, 0, 0, 0});
  };
  const int64_t t = kept_all[layer * kept_batch + (j - layer * n_keep)];
  if (t < 0 || t >= n) return reject();
  const int64_t row = layer * n + t;
  const int s0 = scene_all[row];
  if (s0 < 0 || s0 >= S) return reject();
  const int s = s0 + (int)layer * scene_step;
  int64_t vrow[K];
  float wt[K];
  bool bad = false;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (i < k) {
      const int p = prim_all[row * k + i];
      bad |= p < 0 || p >= P;
      vrow[i] = (int64_t)s * P + p;
      wt[i] = w_all[row * k + i];
    } else {
      vrow[i] = 0;
      wt[i] = 0.f;
    }
  }
  if (bad) return reject();
  char* h = TO_R ? hidden + j * v_bytes : hidden + row * h_bytes;
  for (int c = threadIdx.x; c < chunks; c += blockDim.x) {
    u32x4_t vv[K];
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (i < k) vv[i] = ld16(values + vrow[i] * v_bytes + (int64_t)c * 16);
    const u32x4_t hv = TO_R ? u32x4_t{0, 0, 0, 0} : ld16(h + (int64_t)c * 16);
    u32x4_t out;
    if constexpr (DT == DT_BF16) {
      float acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        if (i < k) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[2 * e] = fmaf(wt[i], bf16lo(vv[i][e]), acc[2 * e]);
            acc[2 * e + 1] = fmaf(wt[i], bf16hi(vv[i][e]), acc[2 * e + 1]);
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        out[e] = pack_bf16x2(bf16lo(hv[e]) + acc[2 * e], bf16hi(hv[e]) + acc[2 * e + 1]);
    } else {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < K; ++i) {
        if (i < k) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[e] = fmaf(wt[i], as_f32(vv[i][e]), acc[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        out[e] = as_u32(as_f32(hv[e]) + acc[e]);
    }
    st16(h + (int64_t)c * 16, out);
  }
}

// The multi-scale mix (Eq. 8) of one kept row j: the M scales' rows R^m (k
// table rows each, weighted and rounded as the gather form writes them),
// their products with the token's query, the softmax over the scales and the
// weighted sum added into the token's hidden row.  The R^m stay in LDS
// between their two uses: written to memory by a gather launch and read back
// twice they were 210 MB on 11520 rows of two scales, and the two launches
// took 91 + 38.5 us (the whole gated injection 237 -> 207 us).  Bound by the
// gather's traffic behind the caches, like the injection above; on few rows
// by its chain of dependent loads (kept row, scene, picks, values), so the
// scales of a row then go to thread groups of their own, side by side (50 bf16
// rows of four scales x 2048 24.1 -> 18.9 us), while that leaves the chip room
// for every workgroup; after that narrow workgroups run better (1500 such rows
// 71.2 us on four groups, 67.0 on one, 11520 408 and 372), down to two groups
// where the R^m of a row leave LDS for few workgroups a CU (8 scales x 3584:
// 11520 rows 1091 us on one group, 952 on two).  launch_multiscale has the rows
// that gather first (ms_gathers).
constexpr int MS_GROUP = 256;              // threads of a scale at most
constexpr int64_t MS_WIDE = 327680, MS_NARROW = 393216;   // threads of a launch
constexpr int64_t MS_CU_LDS = 160 * 1024, MS_CU_THREADS = 1280;
// threads of a row at most (k > 16 holds more loads in registers)
constexpr int ms_row_threads(int k) { return k > 16 ? 512 : 1024; }

template <int DT, int K>
__device__ __forceinline__ u32x4_t weighted_chunk(const char* __restrict__ values,
                                                  const int64_t (&vrow)[K], const float (&wt)[K],
                                                  int k, int64_t v_bytes, int c) {
  u32x4_t vv[K], out;
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (i < k) vv[i] = ld16(values + vrow[i] * v_bytes + (int64_t)c * 16);
  if constexpr (DT == DT_BF16) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (i < k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] = fmaf(wt[i], bf16lo(vv[i][e]), acc[2 * e]);
          acc[2 * e + 1] = fmaf(wt[i], bf16hi(vv[i][e]), acc[2 * e + 1]);
        }
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = pack_bf16x2(acc[2 * e], acc[2 * e + 1]);
  } else {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (i < k)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(wt[i], as_f32(vv[i][e]), acc[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = as_u32(acc[e]);
  }
  return out;
}

template <int DT>
__device__ __forceinline__ float chunk_dot(u32x4_t a, u32x4_t b, float acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (DT == DT_BF16) {
      acc = fmaf(bf16lo(a[e]), bf16lo(b[e]), acc);
      acc = fmaf(bf16hi(a[e]), bf16hi(b[e]), acc);
    } else {
      acc = fmaf(as_f32(a[e]), as_f32(b[e]), acc);
    }
  }
  return acc;
}

// groups x gs threads: group y takes scales y, y + groups, ...  A row whose
// token id is out of range is left alone and counted once a scale; a scale
// whose scene or a primitive is out of range has R^m = 0 and is counted.
template <int DT, int K>
__global__ __launch_bounds__(ms_row_threads(K)) void ms_mix_kernel(
    int64_t n, const int32_t* __restrict__ kept, const int32_t* __restrict__ scene_all,
    const int32_t* __restrict__ prim_all, const float* __restrict__ w_all,
    const char* __restrict__ values, int Sm, int P, int k, int M, int64_t v_bytes,
    const char* __restrict__ q, char* __restrict__ hidden, int64_t h_bytes, float inv_sqrt_d,
    const int32_t* __restrict__ count, int gs) {
  __shared__ float red[MS_MAX_SCALES][MS_GROUP / WAVE];
  extern __shared__ __attribute__((aligned(16))) char rows_lds[];   // [M, v_bytes]
  const int64_t j = blockIdx.x;
  if (count != nullptr && j >= *count) return;   // past a counted list's end
  const int tid = threadIdx.x, lane = tid & 63;
  const int groups = (int)blockDim.x / gs, nw = gs / WAVE;
  // the group (whole waves), and the thread's place in it
  const int y = __builtin_amdgcn_readfirstlane(tid / gs);
  const int gt = tid - y * gs, wv = gt >> 6;
  const int64_t t = kept[j];
  if (t < 0 || t >= n) {
    if (tid == 0) atomicAdd(&g_index_errors, (unsigned long long)M);
    return;
  }
  const int chunks = (int)(v_bytes / 16);
  const char* qrow = q + j * v_bytes;

  // scale m's table rows and weights (uniform over the group); false: an
  // index out of range
  auto picks = [&](int m, int64_t (&vrow)[K], float (&wt)[K]) {
    const int64_t row = (int64_t)m * n + t;
    const int s = scene_all[row];
    bool ok = s >= 0 && s < Sm;
    const int64_t base = ((int64_t)m * Sm + (ok ? s : 0)) * P;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      vrow[i] = base;
      wt[i] = 0.f;
      if (i < k) {
        const int p = prim_all[row * k + i];
        const bool in = p >= 0 && p < P;
        ok &= in;
        vrow[i] = base + (in ? p : 0);
        wt[i] = w_all[row * k + i];
      }
    }
    return ok;
  };

  for (int m = y; m < M; m += groups) {
    int64_t vrow[K];
    float wt[K], dot = 0.f;
    const bool ok = picks(m, vrow, wt);
    for (int c = gt; c < chunks; c += gs) {
      u32x4_t r = {0, 0, 0, 0};
      if (ok) {
        r = weighted_chunk<DT, K>(values, vrow, wt, k, v_bytes, c);
        dot = chunk_dot<DT>(ld16(qrow + (int64_t)c * 16), r, dot);
      }
      *reinterpret_cast<u32x4_t*>(rows_lds + m * v_bytes + c * 16) = r;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) dot += __shfl_xor(dot, d, 64);
    if (lane == 0) red[m][wv] = dot;
    if (!ok && gt == 0) atomicAdd(&g_index_errors, 1ull);
  }
  __syncthreads();
  float alpha[MS_MAX_SCALES];
  float top = -__builtin_inff();
#pragma unroll
  for (int m = 0; m < MS_MAX_SCALES; ++m) {
    alpha[m] = 0.f;
    if (m < M) {
      float v = 0.f;
      for (int w = 0; w < nw; ++w) v += red[m][w];
      alpha[m] = v * inv_sqrt_d;
      top = fmaxf(top, alpha[m]);
    }
  }
  float sum = 0.f;
#pragma unroll
  for (int m = 0; m < MS_MAX_SCALES; ++m) {
    if (m < M) {
      alpha[m] = expf(alpha[m] - top);
      sum += alpha[m];
    }
  }
#pragma unroll
  for (int m = 0; m < MS_MAX_SCALES; ++m) alpha[m] = alpha[m] / sum;

  char* h = hidden + t * h_bytes;
  for (int c = tid; c < chunks; c += blockDim.x) {
    const u32x4_t hv = ld16(h + (int64_t)c * 16);
    u32x4_t out;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < MS_MAX_SCALES; ++m) {
      if (m < M) {
        const u32x4_t rv = *reinterpret_cast<const u32x4_t*>(rows_lds + m * v_bytes + c * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (DT == DT_BF16) {
            acc[2 * e] = fmaf(alpha[m], bf16lo(rv[e]), acc[2 * e]);
            acc[2 * e + 1] = fmaf(alpha[m], bf16hi(rv[e]), acc[2 * e + 1]);
          } else {
            acc[e] = fmaf(alpha[m], as_f32(rv[e]), acc[e]);
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (DT == DT_BF16)
        out[e] = pack_bf16x2(bf16lo(hv[e]) + acc[2 * e], bf16hi(hv[e]) + acc[2 * e + 1]);
      else
        out[e] = as_u32(as_f32(hv[e]) + acc[e]);
    }
    st16(h + (int64_t)c * 16, out);
  }
}

hipError_t launch_ms_mix(int dt, int scales, int64_t n, int64_t n_keep, const int32_t* kept,
                         const int32_t* scene, const int32_t* prim, const float* w,
                         const void* values, int Sm, int P, int d_v, int k, const void* q,
                         int d_h, void* hidden, hipStream_t st, const int32_t* count) {
  const int64_t es = dt == DT_BF16 ? 2 : 4, vb = (int64_t)d_v * es;
  const int ch = (int)(vb / 16);
  const int gs = ch >= MS_GROUP ? MS_GROUP : (ch + 63) / 64 * 64;
  // a counted list has room for every row; about half of a gate is open
  const int64_t rows = count != nullptr ? (n_keep + 1) / 2 : n_keep;
  const int64_t room = (gs < MS_GROUP ? MS_NARROW : MS_WIDE) / (rows * gs);
  const int64_t fill = MS_CU_LDS / (scales * vb + 256) * gs < MS_CU_THREADS ? 2 : 1;
  int64_t groups = room > fill ? room : fill;
  if (groups > scales) groups = scales;
  if (groups > ms_row_threads(k) / gs) groups = ms_row_threads(k) / gs;
  const int64_t turns = (scales + groups - 1) / groups;
  groups = (scales + turns - 1) / turns;   // as even as the turns allow
  const float inv_sqrt_d = 1.0f / sqrtf((float)d_v);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_keep), dim3((unsigned)(gs * groups)),
                       (unsigned)(scales * vb), st, n, kept, scene, prim, w,
                       static_cast<const char*>(values), Sm, P, k, scales, vb,
                       static_cast<const char*>(q), static_cast<char*>(hidden), d_h * es,
                       inv_sqrt_d, count, gs);
  };
  if (dt != DT_BF16) launch(ms_mix_kernel<DT_F32, 8>);
  else if (k <= 8) launch(ms_mix_kernel<DT_BF16, 8>);
  else if (k <= 16) launch(ms_mix_kernel<DT_BF16, 16>);
  else launch(ms_mix_kernel<DT_BF16, 32>);
  return hipGetLastError();
}

template <int DT, bool TO_R = false>
static void launch_inject_k(int kk, dim3 grid, hipStream_t st, int64_t n, int64_t n_keep,
                            const int32_t* kept, const int32_t* scene, const int32_t* prim,
                            const float* w, const char* values, int S, int P, int64_t vb,
                            char* hidden, int64_t hb, int64_t kept_batch, int scene_step,
                            const int32_t* count = nullptr) {
  // as many whole waves as the row has 16-byte chunks (up to 256 threads):
  // narrow rows leave no thread idle, and the CU holds more workgroups
  const int ch = (int)(vb / 16);
  const int bs = ch >= INJ_THREADS ? INJ_THREADS : (ch + 63) / 64 * 64;
#define LOOKME_INJ(K_)                                                                \
  hipLaunchKernelGGL((inject_kernel<DT, K_, TO_R>), grid, dim3(bs), 0, st, n, n_keep, kept, \
                     scene, prim, w, values, S, P, kk, vb, hidden, hb, kept_batch, scene_step, \
                     count)
  if (kk <= 4) LOOKME_INJ(4);
  else if (kk <= 8) LOOKME_INJ(8);
  else if (kk <= 16) LOOKME_INJ(16);
  else LOOKME_INJ(32);
#undef LOOKME_INJ
}

hipError_t launch_crit_norm(int dt, int64_t rows, const void* crit, int d_c, uint32_t* key,
                            hipStream_t st, bool background) {
  if (rows == 0) return hipSuccess;
  const int es = dt == DT_BF16 ? 2 : 4;
  // a wave a row; in the background form 256 workgroups walk the rows, one
  // per CU, so that the norms leave the projection and routing running
  // beside them most of every CU (Zipf batch: those two 312 -> 289 us, the
  // step 2.248 -> 2.216 ms median, while the norms stretch from 107 to
  // ~185 us behind them)
  const int64_t g0 = (rows + NORM_WAVES - 1) / NORM_WAVES;
  const dim3 grid((unsigned)(background && g0 > NORM_BACKGROUND_WGS ? NORM_BACKGROUND_WGS : g0));
  if (dt == DT_BF16)
    hipLaunchKernelGGL(crit_norm_kernel<DT_BF16>, grid, dim3(NORM_WAVES * WAVE), 0, st,
                       static_cast<const char*>(crit), rows, (int64_t)d_c * es, key);
  else
    hipLaunchKernelGGL(crit_norm_kernel<DT_F32>, grid, dim3(NORM_WAVES * WAVE), 0, st,
                       static_cast<const char*>(crit), rows, (int64_t)d_c * es, key);
  return hipGetLastError();
}

hipError_t launch_crit_select(int layers, int64_t n, int64_t n_keep, const uint32_t* key,
                              int32_t* kept, hipStream_t st, bool background) {
  if (n == 0 || n_keep == 0) return hipSuccess;
  // beside the projection and routing of a second stream the large cache's
  // 132 KiB (and 16 waves) find no CU before those have ended, and the select
  // then runs into Level-2's start: 8 waves reading the keys from L2 fit
  // beside them (32768 tokens: select 122 -> 69 us beside the step's other
  // kernels, alone 32.9 us cached and 37.7 so).  Up to SEL_CACHE_MID keys the
  // cache leaves the room as well (4097 keys 20.7 -> 14.5 us alone, 8192 28.5
  // -> 15.4)
  if (background && n > SEL_CACHE_MID)
    hipLaunchKernelGGL((crit_select_kernel<0, SEL_THREADS / 2>), dim3(layers),
                       dim3(SEL_THREADS / 2), 0, st, key, n, n_keep, kept);
  else if (n <= SEL_CACHE_SMALL)
    hipLaunchKernelGGL(crit_select_kernel<SEL_CACHE_SMALL>, dim3(layers), dim3(SEL_THREADS), 0, st,
                       key, n, n_keep, kept);
  else if (n <= SEL_CACHE_MID)
    hipLaunchKernelGGL(crit_select_kernel<SEL_CACHE_MID>, dim3(layers), dim3(SEL_THREADS), 0, st,
                       key, n, n_keep, kept);
  else if (n <= SEL_CACHE_N)
    hipLaunchKernelGGL(crit_select_kernel<SEL_CACHE_N>, dim3(layers), dim3(SEL_THREADS), 0, st,
                       key, n, n_keep, kept);
  else
    hipLaunchKernelGGL(crit_select_kernel<0>, dim3(layers), dim3(SEL_THREADS), 0, st, key, n,
                       n_keep, kept);
  return hipGetLastError();
}

hipError_t take_index_errors(hipStream_t st, uint64_t* out) {
  static const unsigned long long zero = 0;
  unsigned long long v = 0;
  hipError_t e = hipMemcpyFromSymbolAsync(&v, HIP_SYMBOL(g_index_errors), sizeof(v), 0,
                                          hipMemcpyDeviceToHost, st);
  if (e == hipSuccess)
    e = hipMemcpyToSymbolAsync(HIP_SYMBOL(g_index_errors), &zero, sizeof(zero), 0,
                               hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e == hipSuccess) *out = v;
  return e;
}

hipError_t launch_inject_rows(int dt, int layers, int64_t n, int64_t n_keep, const int32_t* kept,
                              const int32_t* scene, const int32_t* prim, const float* w,
                              const void* values, int S, int P, int d_v, int k, void* hidden,
                              int d_h, hipStream_t st, const int32_t* count) {
  if (n == 0 || n_keep == 0) return hipSuccess;
  const int es = dt == DT_BF16 ? 2 : 4;
  const dim3 grid((unsigned)(layers * n_keep));
  if (dt == DT_BF16)
    launch_inject_k<DT_BF16>(k, grid, st, n, n_keep, kept, scene, prim, w,
                             static_cast<const char*>(values), S, P, (int64_t)d_v * es,
                             static_cast<char*>(hidden), (int64_t)d_h * es, n_keep, 0, count);
  else
    launch_inject_k<DT_F32>(k, grid, st, n, n_keep, kept, scene, prim, w,
                            static_cast<const char*>(values), S, P, (int64_t)d_v * es,
                            static_cast<char*>(hidden), (int64_t)d_h * es, n_keep, 0, count);
  return hipGetLastError();
}

hipError_t launch_gather_rows(int dt, int layers, int64_t n, int64_t n_keep, const int32_t* kept,
                              const int32_t* scene, const int32_t* prim, const float* w,
                              const void* values, int S, int P, int d_v, int k, void* r_out,
                              hipStream_t st, int64_t kept_batch, int scene_step,
                              const int32_t* count) {
  if (n == 0 || n_keep == 0) return hipSuccess;
  const int es = dt == DT_BF16 ? 2 : 4;
  const dim3 grid((unsigned)(layers * n_keep));
  if (dt == DT_BF16)
    launch_inject_k<DT_BF16, true>(k, grid, st, n, n_keep, kept, scene, prim, w,
                                   static_cast<const char*>(values), S, P, (int64_t)d_v * es,
                                   static_cast<char*>(r_out), 0, kept_batch, scene_step,
                                   count);
  else
    launch_inject_k<DT_F32, true>(k, grid, st, n, n_keep, kept, scene, prim, w,
                                  static_cast<const char*>(values), S, P, (int64_t)d_v * es,
                                  static_cast<char*>(r_out), 0, kept_batch, scene_step,
                                  count);
  return hipGetLastError();
}

}  // namespace lookme
