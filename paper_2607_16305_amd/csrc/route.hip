// Level-1 scene routing of large batches (arXiv 2607.16305, Sec. 3.2, Eq. 5)
// as a tiled product on the matrix cores with a fused arg max: scene[r] =
// argmax_s <q_r, K1[s]> + b[s], lowest s on exact ties; the scores are never
// written to memory.
//
// A workgroup owns 128 query rows and a range of 256-key tiles,
// computed on the phased loop of phase_gemm.h as one stream of K stages across
// all of its key tiles.  Each quadrant of a tile's last stage is folded (plus
// the bias, staged in LDS) into a running best per row while the next
// quadrant is multiplied; at the end the 4 lanes and then the 4 waves that
// share a row are merged in key order.  When a batch has few row blocks the
// key tiles are split over several workgroups and the partial arg maxima
// meet in route_partial (route_merge.h).
#include "common.h"
#include "kernels.h"
#include "phase_gemm.h"
#include "route_merge.h"

namespace lookme {

struct RouteDtlParams {
  const char* q;         // [rows, d_e]
  const char* keys;      // [S, d_e]
  const float* bias;     // [S] (the BIAS instantiation only)
  int64_t rows;
  int64_t k_bytes;       // d_e * elem size, a multiple of 128
  int S;
  int splits;            // key ranges per row block
  int tps;               // 256-key tiles per range
  int units;             // row blocks * splits
  int32_t* scene;
  uint64_t* part;
  int32_t* count;
};

// The stream of a unit's stages: key tile by key tile, every K stage of the
// query rows with each.  Both operands' lane offsets are 32-bit (a row block
// and a key tile are far below 4 GiB) from uniform bases.
template <class S>
struct RouteLoads {
  const char* q;       // first query row of the unit
  const char* keys;    // first key row of the table
  uint32_t oa[2][S::PA], ob[2][S::PB];
  int64_t k_bytes;
  int S_, nst, nt, kt0;
  int tile = 0, ks = 0;   // position of the stage that is loaded next
  // First key of tile t: a ragged last tile is moved back to end at the last
  // scene, so every key row it reads exists; its keys below t * 256 repeat
  // the previous tile's and are masked in the fold.  With fewer scenes than
  // a tile there is one tile, at 0.
  __device__ __forceinline__ int start(int t) const {
    return S_ < S::BN ? 0 : min(t * S::BN, S_ - S::BN);
  }
  __device__ __forceinline__ void a(int h, int, char* dst) const {
#pragma unroll
    for (int i = 0; i < S::PA; ++i) load_lds16_at(q, oa[h][i], ks * 128, dst + i * 1024);
  }
  __device__ __forceinline__ void b(int h, int, char* dst) const {
    const char* base = keys + (int64_t)start(kt0 + tile) * k_bytes;
#pragma unroll
    for (int i = 0; i < S::PB; ++i) load_lds16_at(base, ob[h][i], ks * 128, dst + i * 1024);
  }
  // past the unit's last stage it is read again, so that the waits keep
  // their counts
  __device__ __forceinline__ void next() {
    if (ks + 1 < nst) ++ks;
    else if (tile + 1 < nt) {
      ++tile;
      ks = 0;
    }
  }
};

template <int DT, bool BIAS>
__global__ __launch_bounds__(512, 2) void route_phase_kernel(RouteDtlParams a) {
  constexpr int MI = 2, NJ = 2;
  using S = PgShape<MI, NJ>;
  constexpr int W = S::W;
  static_assert(S::BM == ROUTE_DTL_ROWS && S::BN == ROUTE_DTL_KEYS, "tile shape");
  // All of the kernel's LDS is one object.  With several __shared__ objects
  // the compiler tags their accesses with alias scopes and then, finding the
  // stage buffers' direct-to-LDS loads and fragment reads in one scope, puts
  // a vmcnt(0) wait before the fragment reads.  The merge arrays and the
  // arrival flag reuse the stage buffers (after the last stage); the bias
  // table has its own words.
  constexpr int BIAS_OFF = 2 * S::BUF;
  constexpr int BIAS_BYTES = BIAS ? ROUTE_DTL_MAX_TPS * S::BN * 4 : 0;
  static_assert(4 * S::BM * 8 + 16 <= 2 * S::BUF, "merge arrays in the stage buffers");
  __shared__ __attribute__((aligned(1024))) char smem[BIAS_OFF + BIAS_BYTES];
  float* s_bias = reinterpret_cast<float*>(smem + BIAS_OFF);
  float (*m_s)[S::BM] = reinterpret_cast<float (*)[S::BM]>(smem);
  int (*m_i)[S::BM] = reinterpret_cast<int (*)[S::BM]>(smem + 4 * S::BM * 4);
  int* s_last = reinterpret_cast<int*>(smem + 4 * S::BM * 8);
  const int tid = threadIdx.x;

  const int u = xcd_remap(blockIdx.x, a.units);
  if (u < 0) return;
  // (the quotient comes out of vector instructions: said to be uniform, so
  // that what follows from it stays in scalar registers)
  const int rb = __builtin_amdgcn_readfirstlane(u / a.splits);
  const int split = __builtin_amdgcn_readfirstlane(u - rb * a.splits);
  const int64_t m0 = (int64_t)rb * S::BM;
  const int ntiles = (a.S + S::BN - 1) / S::BN;
  const int kt0 = split * a.tps, kt1 = min(ntiles, kt0 + a.tps);

  if constexpr (BIAS) {
    // the bias of the unit's keys (0 past the last scene: those keys are
    // masked by index anyway); visible after the loop's first barrier
    for (int i = tid; i < (kt1 - kt0) * S::BN; i += 512) {
      const int key = kt0 * S::BN + i;
      s_bias[i] = key < a.S ? a.bias[key] : 0.f;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  }

  PgLoop<DT, MI, NJ> L(smem, tid);
  RouteLoads<S> ld;
  ld.q = a.q + m0 * a.k_bytes;
  ld.keys = a.keys;
  ld.k_bytes = a.k_bytes;
  ld.S_ = a.S;
  ld.nst = (int)(a.k_bytes / 128);
  ld.nt = kt1 - kt0;
  ld.kt0 = kt0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < S::PA; ++i) {
      const int64_t r = min<int64_t>(m0 + h * S::HM + L.a_row(i), a.rows - 1) - m0;   // >= 0
      ld.oa[h][i] = (uint32_t)(r * a.k_bytes) + L.a_chunk(i) * 16;
    }
#pragma unroll
    for (int i = 0; i < S::PB; ++i) {
      // fewer scenes than a tile: rows past the last scene read it
      int r = h * S::HN + L.b_row(i);
      if (a.S < S::BN) r = min(r, a.S - 1);
      ld.ob[h][i] = (uint32_t)(r * a.k_bytes) + L.b_chunk(i) * 16;
    }
  }

  // running best of the lane's 2 MI rows (256-row blocks had no registers for
  // them: the loop spilled, and every reload waited for the loads before it)
  float bs[2][MI];
  int bi[2][MI];
#pragma unroll
  for (int qi = 0; qi < 2; ++qi)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      bs[qi][i] = -__builtin_inff();
      bi[qi][i] = -1;
    }
  f32x4_t acc[2][2][MI][NJ];
  int c_tile = 0, c_ks = 0;   // the stage that is multiplied
  // A quadrant of a complete tile: the lane holds W neighbouring keys of its
  // rows.  A row's keys come in increasing order, so a strict '>' keeps the
  // lowest on exact ties (a NaN is never taken).  Three vector instructions a
  // score where the tile has neither bias nor masked keys: with the mask
  // selected per score, a canonicalising maximum and ties compared it was
  // seven to eleven, and tiles of few K stages were bound by it (bf16 30000
  // rows x 4096 scenes x 64 42.1 -> 29.9 us, x 512 129.7 -> 113.8, 65536 x 4096
  // x 64 82.9 -> 58.7).
  auto fold_keys = [&](int qi, int qj, int key0, auto&& score) {
#pragma unroll
    for (int e = 0; e < W; ++e)
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const float v = score(acc[qi][qj][i][e >> 2][e & 3], e);
        const bool take = v > bs[qi][i];
        bi[qi][i] = take ? key0 + e : bi[qi][i];
        bs[qi][i] = take ? v : bs[qi][i];
      }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[qi][qj][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  auto fold = [&](int qi, int qj) {
    const int tile = __builtin_amdgcn_readfirstlane(kt0 + c_tile);
    const int key0 = ld.start(tile) + qj * S::HN + L.wc * 16 * NJ + W * L.g;
    const bool ragged = (tile + 1) * S::BN > a.S;
    if (BIAS || ragged) {
      float add[W];
#pragma unroll
      for (int e = 0; e < W; ++e) {
        const int key = key0 + e;
        add[e] = BIAS ? s_bias[max(key - kt0 * S::BN, 0)] : 0.f;
        // keys already scored by the previous tile, and rows past the last
        // scene
        if (ragged && (key < tile * S::BN || key >= a.S)) add[e] = -__builtin_inff();
      }
      fold_keys(qi, qj, key0, [&](float v, int e) { return v + add[e]; });
    } else {
      fold_keys(qi, qj, key0, [](float v, int) { return v; });
    }
  };
  L.run(ld.nt * ld.nst, ld, acc, [&](int, int q) {
    if (__builtin_amdgcn_readfirstlane(c_ks) == ld.nst - 1) {
      fold(q >> 1, q & 1);
    }
    if (q == 3) {
      const bool end = c_ks == ld.nst - 1;
      c_tile += end;
      c_ks = end ? 0 : c_ks + 1;
    }
  });
  __syncthreads();   // every wave is done with the stage buffers

  // merge the 4 lanes of a row (keys W g of every tile half), then the 4
  // waves that share rows, in key order
#pragma unroll
  for (int qi = 0; qi < 2; ++qi)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int d = 16; d < 64; d <<= 1) {
        const float os = __shfl_xor(bs[qi][i], d, 64);
        const int oi = __shfl_xor(bi[qi][i], d, 64);
        if (beats(os, oi, bs[qi][i], bi[qi][i])) {
          bs[qi][i] = os;
          bi[qi][i] = oi;
        }
      }
      if (L.g == 0) {
        const int row = qi * S::HM + L.wr * 16 * MI + 16 * i + L.n16;
        m_s[L.wc][row] = bs[qi][i];
        m_i[L.wc][row] = bi[qi][i];
      }
    }
  __syncthreads();
  const int nr = (int)min<int64_t>(S::BM, a.rows - m0);
  float best_s = -__builtin_inff();
  int best_i = -1;
  if (tid < S::BM) {
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (beats(m_s[w][tid], m_i[w][tid], best_s, best_i)) {
        best_s = m_s[w][tid];
        best_i = m_i[w][tid];
      }
  }
  if (a.splits == 1) {
    if (tid < nr) a.scene[m0 + tid] = best_i;
    return;
  }
  route_partial<S::BM>(a.part, a.count, a.splits, a.scene, rb, split, tid < S::BM ? tid : S::BM,
                       nr, best_s, best_i, s_last);
}

hipError_t launch_route_dtl(int dt, const void* q, const void* scene_keys, const float* bias,
                            int32_t* scene, int64_t rows, int d_e, int S, const RoutePlan& plan,
                            uint64_t* part, int32_t* count, hipStream_t st) {
  RouteDtlParams p{};
  p.q = static_cast<const char*>(q);
  p.keys = static_cast<const char*>(scene_keys);
  p.bias = bias;
  p.rows = rows;
  p.k_bytes = (int64_t)d_e * (dt == DT_BF16 ? 2 : 4);
  p.S = S;
  p.splits = plan.splits;
  p.tps = plan.per_split;
  p.units = (int)((rows + ROUTE_DTL_ROWS - 1) / ROUTE_DTL_ROWS * plan.splits);
  p.scene = scene;
  p.part = part;
  p.count = count;
  const dim3 grid((unsigned)((p.units + 7) / 8 * 8));
  if (dt == DT_BF16) {
    if (bias != nullptr) hipLaunchKernelGGL((route_phase_kernel<DT_BF16, true>), grid, dim3(512), 0, st, p);
    else hipLaunchKernelGGL((route_phase_kernel<DT_BF16, false>), grid, dim3(512), 0, st, p);
  } else {
    if (bias != nullptr) hipLaunchKernelGGL((route_phase_kernel<DT_F32, true>), grid, dim3(512), 0, st, p);
    else hipLaunchKernelGGL((route_phase_kernel<DT_F32, false>), grid, dim3(512), 0, st, p);
  }
  return hipGetLastError();
}

}  // namespace lookme
