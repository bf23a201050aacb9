// Small-tile product C = A B^T on the matrix cores for the MLP-shaped steps
// (the relevance MLP of Eq. 6, the SwiGLU fusion of Eq. 10 and the
// propagation of Eq. 11): 64 x 64
// output tiles, 4 waves in 2 x 2 (each 2 x 2 MFMA tiles), K in 128-byte
// stages loaded straight into LDS (dtl.h), a ring of NS stages, NS - 1 in
// flight while one is multiplied.  These products have few rows and long K,
// so the bytes in flight per CU over the loads' latency, not the matrix
// cores, set the pace: the ring is as deep as the grid's occupancy allows
// (launch_tile_gemm).
// blockIdx.y selects a batch (a layer) whose A, B and output start a fixed
// stride further.  With a count array, batch z has count[z] live rows (at
// most `rows`, which sizes the grid); the tiles beyond them do nothing.  Epilogues:
//
//   EPI_ACT     C + bias, ReLU, one rounding to the storage dtype, [rows, cols];
//   EPI_LOGIT   C + bias as float32, [rows, cols];
//   EPI_SWIGLU  the tile's B rows are 32 rows of B (gate) and the same 32 rows
//               of B2 (up): u = silu(gate) * up, rounded, [rows, cols] with
//               32 output columns a tile;
//   EPI_RESID   H[out_row(r), c] = round(H + C) with out_row(r) = z * n +
//               kept[z * kept_batch + r] (the kept token of row r of layer z);
//   EPI_ADD     round(C + res) with res [rows, cols], [rows, cols];
//   EPI_STORE   round(C), [rows, cols];
//   EPI_ACT_TAB C + tab[sel[row]] (a float32 row of [sel_rows, cols]: the
//               relevance MLP's per-scene half of the first layer, b1
//               included), ReLU, one rounding, [rows, cols].
//   EPI_Q       round(C), column c of row r at q[c / d_e][r][c % d_e] (the
//               query projection of all layers).
//
// With a_sel, row r of A is row a_sel[r] of a0 (the multi-scale router's
// queries: the kept tokens' hidden rows).
//
// Products with enough large tiles to fill the chip run on the phased kernel
// (phase_gemm.h); see launch_tile_gemm.

#pragma once

#include <type_traits>

#include "common.h"
#include "dtl.h"
#include "kernels.h"
#include "phase_gemm.h"

namespace lookme {

// TI: 16-row MFMA tiles a wave; 2 (64-row tiles), or 1 (32-row tiles) where
// that spreads a product over CUs that would have no workgroup.
template <int TI>
using TgShapeT = DtlShape<2, 2, TI, 2, 128>;
using TgShape = TgShapeT<2>;
constexpr int TG_KB = 128;

enum : int {
  EPI_ACT = 0, EPI_LOGIT = 1, EPI_SWIGLU = 2, EPI_RESID = 3, EPI_ADD = 4, EPI_STORE = 5,
  EPI_ACT_TAB = 6, EPI_Q = 7
};

struct TileGemmParams {
  const char* a0;           // [rows, K]
  const int32_t* a_sel;     // or null: [rows] row of a0 for each A row (clamped to [0, sel_rows))
  const int32_t* sel;       // EPI_ACT_TAB: [rows] row of tab (clamped to [0, sel_rows))
  const char* b;            // [cols, K] (EPI_SWIGLU: gate rows)
  const char* b2;           // EPI_SWIGLU: up rows [cols, K]
  const float* bias;        // [cols] or null (EPI_ACT, EPI_LOGIT)
  char* out;
  const int32_t* kept;      // EPI_RESID: kept list of batch z at kept + z * kept_batch
  const char* res;          // EPI_ADD: [rows, cols]
  const float* tab;         // EPI_ACT_TAB: [sel_rows, cols], row sel[r] added to row r
  const int32_t* count;     // or null: batch z uses only its first count[z * count_step]
                            // rows (a gate's counted kept list); tiles past them end at once
  int64_t rows;
  int64_t a_bytes;          // bytes between A rows
  int64_t k_bytes;          // K in bytes, a multiple of 128
  int64_t b_ld;             // bytes between B rows (0: k_bytes; a column slice of a wider B)
  int64_t a_batch, b_batch, out_batch;   // byte strides between batches
  int64_t n, kept_batch;    // EPI_RESID: tokens per layer, stride of the kept lists
  int64_t out_ld;           // EPI_RESID: bytes of an H row
  int sel_rows, cols, tiles;
  int col_major;            // tile ids run down the row tiles of a column block first
  int count_step;           // 1: a count per batch, 0: one count for all
  int batches;              // phased kernel: number of batches
  int d_e;                  // EPI_Q: columns of a layer (a multiple of 8)
};

// Origin of tile `tile`: row tiles of one column block are consecutive ids
// when col_major (so they land on one XCD and share its L2 copy of the B
// rows, which the larger operand then crosses HBM once), else the column
// tiles of one row block.
template <int TI>
__device__ __forceinline__ void tile_origin(const TileGemmParams& a, int tile, int tcols,
                                            int64_t* m0, int* n0) {
  constexpr int BM = TgShapeT<TI>::BM;
  if (a.col_major) {
    const int tiles_m = (int)((a.rows + BM - 1) / BM);
    *m0 = (int64_t)(tile % tiles_m) * BM;
    *n0 = (tile / tiles_m) * tcols;
  } else {
    const int tiles_n = (a.cols + tcols - 1) / tcols;
    *m0 = (int64_t)(tile / tiles_n) * BM;
    *n0 = (tile % tiles_n) * tcols;
  }
}

__device__ __forceinline__ float silu_f(float x) { return x / (1.f + expf(-x)); }

// Epilogue of the tile at (m0, n0) of batch z from the accumulators of
// thread tid: the lane holds rows m0 + wm + 16 i + 4 g + r and tile columns
// wn + 16 j + n16.  xch: 4096 floats of LDS (EPI_SWIGLU only).
template <int DT, int EPI, int TI>
__device__ __forceinline__ void tile_epilogue(const TileGemmParams& a,
                                              f32x4_t (&acc)[TI][2], int64_t z, int64_t m0,
                                              int n0, int tid, float* xch, int64_t rows,
                                              bool live) {
  constexpr int MI = TI, NJ = 2, WN = 2;
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  const int lane = tid & 63, wv = tid >> 6;
  const int n16 = lane & 15, g = lane >> 4;
  const int wm = (wv / WN) * 16 * MI, wn = (wv % WN) * 16 * NJ;
  if constexpr (EPI == EPI_SWIGLU) {
    // the up half (waves with wn = 32) passes its tile through LDS to the
    // gate half (wn = 0) of the same rows
    __syncthreads();   // every wave is done with the LDS the exchange reuses
    if (wn != 0) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            xch[(((wv / WN) * MI * NJ + i * NJ + j) * 4 + r) * WAVE + lane] = acc[i][j][r];
    }
    __syncthreads();
    if (wn != 0 || !live) return;
    char* U = a.out + z * a.out_batch;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = n0 + 16 * j + n16;
      if (col >= a.cols) continue;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t row = m0 + wm + 16 * i + 4 * g + r;
          if (row >= rows) continue;
          const float up = xch[(((wv / WN) * MI * NJ + i * NJ + j) * 4 + r) * WAVE + lane];
          const float u = silu_f(acc[i][j][r]) * up;
          char* dst = U + (row * a.cols + col) * ES;
          if constexpr (DT == DT_BF16)
            *reinterpret_cast<uint16_t*>(dst) = (uint16_t)f32_to_bf16_rne(u);
          else
            *reinterpret_cast<float*>(dst) = u;
        }
    }
  } else {
    if (!live) return;
    // every load (biases, kept rows, H or residual values) is issued before
    // the first store: as far as the compiler knows a store may alias a later
    // load, which would otherwise serialise the elements one round trip each.
    // The loads are unconditional, from addresses clamped into the operands
    // (a load under a branch gets a wait of its own where the paths meet).
    int col[NJ], ccol[NJ];
    float bias[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      col[j] = n0 + wn + 16 * j + n16;
      ccol[j] = col[j] < a.cols ? col[j] : a.cols - 1;
      bias[j] = 0.f;
      if constexpr (EPI == EPI_ACT || EPI == EPI_LOGIT)
        if (a.bias != nullptr) bias[j] = a.bias[ccol[j]];
    }
    int64_t orow[MI][4];   // output row: the tile row, or (EPI_RESID) its H row
    int64_t trow[MI][4];   // EPI_ACT_TAB: the row's table row
    bool rok[MI][4];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = m0 + wm + 16 * i + 4 * g + r;
        rok[i][r] = row < rows;
        orow[i][r] = rok[i][r] ? row : rows - 1;
        if constexpr (EPI == EPI_RESID) {
          int64_t t = a.kept[z * a.kept_batch + orow[i][r]];
          t = t < 0 ? 0 : (t >= a.n ? a.n - 1 : t);
          orow[i][r] = z * a.n + t;
        }
        if constexpr (EPI == EPI_ACT_TAB) {
          const int s = a.sel[orow[i][r]];
          trow[i][r] = s < 0 ? 0 : (s >= a.sel_rows ? a.sel_rows - 1 : s);
        }
      }
    float old[NJ][MI][4];   // EPI_RESID: H, EPI_ADD: the residual, EPI_ACT_TAB: the table
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          old[j][i][r] = 0.f;
          if constexpr (EPI == EPI_ACT_TAB)
            old[j][i][r] = a.tab[trow[i][r] * a.cols + ccol[j]];
          if constexpr (EPI == EPI_RESID || EPI == EPI_ADD) {
            const char* src = EPI == EPI_RESID
                                  ? a.out + orow[i][r] * a.out_ld + (int64_t)ccol[j] * ES
                                  : a.res + (orow[i][r] * a.cols + ccol[j]) * ES;
            if constexpr (DT == DT_BF16)
              old[j][i][r] = bf16lo(*reinterpret_cast<const uint16_t*>(src));
            else
              old[j][i][r] = *reinterpret_cast<const float*>(src);
          }
        }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (col[j] >= a.cols) continue;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!rok[i][r]) continue;
          const float c = acc[i][j][r] + bias[j];
          if constexpr (EPI == EPI_LOGIT) {
            reinterpret_cast<float*>(a.out)[orow[i][r] * a.cols + col[j]] = c;
            continue;
          }
          float v;
          char* dst;
          if constexpr (EPI == EPI_ACT || EPI == EPI_STORE) {
            v = EPI == EPI_ACT ? fmaxf(c, 0.f) : c;
            dst = a.out + (orow[i][r] * a.cols + col[j]) * ES;
          } else if constexpr (EPI == EPI_Q) {
            v = c;
            dst = a.out + (((int64_t)(col[j] / a.d_e) * a.rows + orow[i][r]) * a.d_e +
                           col[j] % a.d_e) * ES;
          } else if constexpr (EPI == EPI_ACT_TAB) {
            v = fmaxf(c + old[j][i][r], 0.f);
            dst = a.out + (orow[i][r] * a.cols + col[j]) * ES;
          } else if constexpr (EPI == EPI_ADD) {
            v = old[j][i][r] + c;
            dst = a.out + (orow[i][r] * a.cols + col[j]) * ES;
          } else {   // EPI_RESID
            v = old[j][i][r] + c;
            dst = a.out + orow[i][r] * a.out_ld + (int64_t)col[j] * ES;
          }
          if constexpr (DT == DT_BF16)
            *reinterpret_cast<uint16_t*>(dst) = (uint16_t)f32_to_bf16_rne(v);
          else
            *reinterpret_cast<float*>(dst) = v;
        }
    }
  }
}

// Tile (m0, n0) of batch z, computed by the four waves of threads tid = 0 ..
// 255 on a ring of NS stages at lds.  live: false for a tile that is computed
// beside another workgroup half's only to keep its barriers, and not stored.
template <int DT, int EPI, int NS, int TI>
__device__ __forceinline__ void tile_gemm_tile(const TileGemmParams& a,
                                               char (*lds)[TgShapeT<TI>::STAGE], int64_t z,
                                               int64_t m0, int n0, int tid, int64_t rows,
                                               bool live) {
  using S = TgShapeT<TI>;
  constexpr int MI = TI, NJ = 2, KB = TG_KB, KSL = KB / 64, WN = 2;
  constexpr int TCOLS = EPI == EPI_SWIGLU ? S::BN / 2 : S::BN;   // output columns a tile
  static_assert(NS >= 2, "a stage in flight while one is multiplied");
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n16 = lane & 15, g = lane >> 4;
  const int wm = (wv / WN) * 16 * MI, wn = (wv % WN) * 16 * NJ;
  const int nst = (int)(a.k_bytes / KB);
  const char* A0 = a.a0 + z * a.a_batch;
  const char* B0 = a.b + z * a.b_batch;

  // load b covers tile row trow (A rows first, then B rows).  Rows past the
  // edge are clamped (their outputs are not stored).
  const char* src[S::PER_WAVE];
  int sel[S::PER_WAVE];   // gathered rows, loaded together (one branch, no wait each)
  if (a.a_sel != nullptr) {
#pragma unroll
    for (int b = 0; b < S::PER_WAVE; ++b) {
      const int trow = (wv * S::PER_WAVE + b) * S::RPI + lane / S::LPR;
      int64_t r = m0 + (trow < S::BM ? trow : 0);
      r = r < rows ? r : rows - 1;
      sel[b] = a.a_sel[r];
    }
  }
#pragma unroll
  for (int b = 0; b < S::PER_WAVE; ++b) {
    const int trow = (wv * S::PER_WAVE + b) * S::RPI + lane / S::LPR;
    const int chunk = (lane % S::LPR) ^ blk_swz<KB>(trow & 15);
    if (trow < S::BM) {
      int64_t r = m0 + trow;
      r = r < rows ? r : rows - 1;
      if (a.a_sel != nullptr) {
        const int s = sel[b];
        r = s < 0 ? 0 : (s >= a.sel_rows ? a.sel_rows - 1 : s);
      }
      src[b] = A0 + r * a.a_bytes + chunk * 16;
    } else {
      int c = trow - S::BM;
      const char* base = B0;
      if constexpr (EPI == EPI_SWIGLU) {
        // rows 0..31 of the B part: gate rows, 32..63: the same up rows
        if (c >= TCOLS) {
          base = a.b2 + z * a.b_batch;
          c -= TCOLS;
        }
      }
      int r = n0 + c;
      r = r < a.cols ? r : a.cols - 1;
      src[b] = base + (int64_t)r * (a.b_ld != 0 ? a.b_ld : a.k_bytes) + chunk * 16;
    }
  }
  auto issue = [&](int i) {
    const int s = i < nst ? i : nst - 1;   // past the end: a harmless reload
    char* dst = lds[i % NS];
#pragma unroll
    for (int b = 0; b < S::PER_WAVE; ++b)
      load_lds16(src[b] + (int64_t)s * KB, dst + (wv * S::PER_WAVE + b) * 1024);
  };

  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  auto read = [&](int i, u32x4_t (&fa)[KSL][MI], u32x4_t (&fb)[KSL][NJ]) {
    const char* buf = lds[i % NS];
#pragma unroll
    for (int ks = 0; ks < KSL; ++ks) {
#pragma unroll
      for (int ii = 0; ii < MI; ++ii) fa[ks][ii] = read_frag<KB>(buf, wm + 16 * ii, ks, n16, g);
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb[ks][j] = read_frag<KB>(buf, S::BM + wn + 16 * j, ks, n16, g);
    }
  };
  auto mma = [&](const u32x4_t (&fa)[KSL][MI], const u32x4_t (&fb)[KSL][NJ]) {
#pragma unroll
    for (int ks = 0; ks < KSL; ++ks)
#pragma unroll
      for (int ii = 0; ii < MI; ++ii)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[ii][j] = mfma_chunk<DT>(fa[ks][ii], fb[ks][j], acc[ii][j]);
  };
  // this wave's loads of all but the `younger` most recent stages have
  // landed; the barrier makes every wave's visible and ends every read of
  // the buffer that the next loads fill (a plain s_barrier: the fence of
  // __syncthreads would wait for every load in flight)
  auto sync = [&](auto younger) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(younger)::value * S::PER_WAVE) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

#pragma unroll
  for (int i = 0; i < NS - 1; ++i) issue(i);
  if constexpr (NS == 2) {
    for (int i = 0; i < nst; ++i) {
      sync(std::integral_constant<int, 0>{});
      issue(i + 1);
      u32x4_t fa[KSL][MI], fb[KSL][NJ];
      read(i, fa, fb);
      mma(fa, fb);
    }
  } else {
    // one wave a SIMD (or two): nothing else hides a wave's LDS reads, so the
    // fragments of stage i + 1 are read while those of stage i are multiplied
    // (image fused injection 32.6 -> 30.4 us, propagated 100.6 -> 95.7; the
    // 32 KiB a stage that the four waves read from LDS bound it now)
    auto step = [&](int i, const u32x4_t (&ca)[KSL][MI], const u32x4_t (&cb)[KSL][NJ],
                    u32x4_t (&na)[KSL][MI], u32x4_t (&nb)[KSL][NJ]) {
      sync(std::integral_constant<int, NS - 3>{});   // stage i + 1 is in LDS
      read(i + 1, na, nb);
      issue(i + NS - 1);
      __builtin_amdgcn_sched_barrier(0);
      mma(ca, cb);
      __builtin_amdgcn_sched_barrier(0);
    };
    u32x4_t fa0[KSL][MI], fb0[KSL][NJ], fa1[KSL][MI], fb1[KSL][NJ];
    sync(std::integral_constant<int, NS - 2>{});
    read(0, fa0, fb0);
    int i = 0;
    for (; i + 1 < nst; i += 2) {
      step(i, fa0, fb0, fa1, fb1);
      step(i + 1, fa1, fb1, fa0, fb0);
    }
    if (i < nst) step(i, fa0, fb0, fa1, fb1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load into LDS outlives the wave

  tile_epilogue<DT, EPI, TI>(a, acc, z, m0, n0, tid, reinterpret_cast<float*>(&lds[0][0]), rows,
                             live);
}

template <int DT, int EPI, int NS, int TI = 2>
__global__ __launch_bounds__(256) void tile_gemm_kernel(TileGemmParams a) {
  using S = TgShapeT<TI>;
  constexpr int TCOLS = EPI == EPI_SWIGLU ? S::BN / 2 : S::BN;
  __shared__ __attribute__((aligned(1024))) char lds[NS][S::STAGE];
  const int64_t z = blockIdx.y;
  const int tile = xcd_remap(blockIdx.x, a.tiles);
  if (tile < 0) return;
  int64_t m0;
  int n0;
  tile_origin<TI>(a, tile, TCOLS, &m0, &n0);
  int64_t rows = a.rows;   // live rows of this batch
  if (a.count != nullptr) {
    const int64_t c = a.count[z * a.count_step];
    rows = c < 0 ? 0 : (c < a.rows ? c : a.rows);
    if (m0 >= rows) return;
  }
  tile_gemm_tile<DT, EPI, NS, TI>(a, lds, z, m0, n0, threadIdx.x, rows, true);
}

// ---------------------------------------------------------------------------
// The phased kernel (phase_gemm.h)
// ---------------------------------------------------------------------------
// 256 x 256 tiles, one workgroup a CU, in rounds of 256; when the last round
// would have at most 128 of them, each of these is cut into four 128 x 128
// tiles (same launch, after the others): a round of such quarters takes
// about a third of a whole tile's time, two of them still less than a round
// of whole tiles that leaves half of the chip idle.  (2304 x 2048 x 2048 for
// four layers, 288 tiles: 115 -> 85 us; 11520 x 1536 x 2048, 270: 100 -> 73.)
constexpr int PH_ROUND = 256;
struct PhasePlan {
  int whole, cut;   // tiles computed whole (the first ones), tiles cut in four
};
__host__ __device__ inline PhasePlan phase_plan(int tiles) {
  const int rem = tiles % PH_ROUND;
  const int cut = rem <= PH_ROUND / 2 ? rem : 0;
  return PhasePlan{tiles - cut, cut};
}

// One tile: rows from m0, output columns from n0 of batch z.  cols must be a
// multiple of 8, so that a lane's W columns are all inside or all outside and
// its 16-byte accesses are aligned.
template <int DT, int EPI, int MI, int NJ>
__device__ __forceinline__ void phase_tile(const TileGemmParams& a, char* lds, int64_t z,
                                           int64_t rows, int64_t m0, int n0) {
  using S = PgShape<MI, NJ>;
  constexpr int ES = DT == DT_BF16 ? 2 : 4, W = S::W;
  PgLoop<DT, MI, NJ> L(lds, threadIdx.x);
  PgLoads<S> ld;
  ld.last = (int)(a.k_bytes / 128) - 1;
  {
    // gathered rows (a_sel) count from the operand's first row, others from
    // the tile's
    ld.a_base = a.a0 + z * a.a_batch + (a.a_sel != nullptr ? 0 : m0 * a.a_bytes);
    const int64_t bld = a.b_ld != 0 ? a.b_ld : a.k_bytes;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < S::PA; ++q) {
        int64_t r = m0 + h * S::HM + L.a_row(q);
        r = r < rows ? r : rows - 1;
        if (a.a_sel != nullptr) {
          const int s = a.a_sel[r];
          r = s < 0 ? 0 : (s >= a.sel_rows ? a.sel_rows - 1 : s);
        } else {
          r -= m0;
        }
        ld.oa[h][q] = (uint32_t)(r * a.a_bytes) + L.a_chunk(q) * 16;
      }
      const int nh = n0 + (EPI == EPI_SWIGLU ? 0 : h * S::HN);   // first B row of the half
      const int first = nh < a.cols ? nh : a.cols - 1;
      ld.b_base[h] = (EPI == EPI_SWIGLU && h == 1 ? a.b2 : a.b) + z * a.b_batch + first * bld;
#pragma unroll
      for (int q = 0; q < S::PB; ++q) {
        int r = nh + L.b_row(q);
        r = r < a.cols ? r : a.cols - 1;
        ld.ob[h][q] = (uint32_t)((r - first) * bld) + L.b_chunk(q) * 16;
      }
    }
  }
  f32x4_t acc[2][2][MI][NJ];
  L.run(ld.last + 1, ld, acc, [](int, int) {});

  constexpr int QJ = EPI == EPI_SWIGLU ? 1 : 2;
  int col[QJ];
#pragma unroll
  for (int qj = 0; qj < QJ; ++qj) col[qj] = n0 + qj * S::HN + L.wc * 16 * NJ + W * L.g;
  const char* R = EPI == EPI_RESID ? a.out : a.res;
#pragma unroll
  for (int qi = 0; qi < 2; ++qi) {
    // every load of the half's rows before its first store: a store may alias
    // a later load as far as the compiler knows
    int64_t row[MI], orow[MI];
    int trow[MI];
    bool ok[MI];
    float old[MI][QJ][W];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      row[i] = m0 + qi * S::HM + L.wr * 16 * MI + 16 * i + L.n16;
      ok[i] = row[i] < rows;
      orow[i] = ok[i] ? row[i] : rows - 1;
      trow[i] = 0;
      if constexpr (EPI == EPI_RESID) {
        int64_t t = a.kept[z * a.kept_batch + orow[i]];
        t = t < 0 ? 0 : (t >= a.n ? a.n - 1 : t);
        orow[i] = z * a.n + t;
      }
      if constexpr (EPI == EPI_ACT_TAB) {
        const int s = a.sel[orow[i]];
        trow[i] = s < 0 ? 0 : (s >= a.sel_rows ? a.sel_rows - 1 : s);
      }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int qj = 0; qj < QJ; ++qj) {
        const int cc = col[qj] < a.cols ? col[qj] : a.cols - W;
        if constexpr (EPI == EPI_RESID)
          ld_cols<DT, W>(R + orow[i] * a.out_ld + (int64_t)cc * ES, old[i][qj]);
        else if constexpr (EPI == EPI_ADD)
          ld_cols<DT, W>(R + (orow[i] * a.cols + cc) * ES, old[i][qj]);
        else if constexpr (EPI == EPI_ACT_TAB)
          ld_cols<DT_F32, W>(reinterpret_cast<const char*>(a.tab + (int64_t)trow[i] * a.cols + cc),
                             old[i][qj]);
        else if constexpr (EPI == EPI_ACT || EPI == EPI_LOGIT)
#pragma unroll
          for (int e = 0; e < W; ++e) old[i][qj][e] = a.bias != nullptr ? a.bias[cc + e] : 0.f;
        else
#pragma unroll
          for (int e = 0; e < W; ++e) old[i][qj][e] = 0.f;
      }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if (!ok[i]) continue;
#pragma unroll
      for (int qj = 0; qj < QJ; ++qj) {
        if (col[qj] >= a.cols) continue;
        float v[W];
#pragma unroll
        for (int e = 0; e < W; ++e) {
          const float c = acc[qi][qj][i][e >> 2][e & 3];
          if constexpr (EPI == EPI_SWIGLU) v[e] = silu_f(c) * acc[qi][1][i][e >> 2][e & 3];
          else if constexpr (EPI == EPI_ACT || EPI == EPI_ACT_TAB) v[e] = fmaxf(c + old[i][qj][e], 0.f);
          else if constexpr (EPI == EPI_STORE || EPI == EPI_Q) v[e] = c;
          else v[e] = old[i][qj][e] + c;
        }
        if constexpr (EPI == EPI_LOGIT)
          st_cols<DT_F32, W>(a.out + (orow[i] * a.cols + col[qj]) * 4, v);
        else if constexpr (EPI == EPI_Q)
          st_cols<DT, W>(a.out + (((int64_t)(col[qj] / a.d_e) * a.rows + orow[i]) * a.d_e +
                                  col[qj] % a.d_e) * ES, v);
        else if constexpr (EPI == EPI_RESID)
          st_cols<DT, W>(a.out + orow[i] * a.out_ld + (int64_t)col[qj] * ES, v);
        else
          st_cols<DT, W>(a.out + z * a.out_batch + (orow[i] * a.cols + col[qj]) * ES, v);
      }
    }
  }
}

// A counted product with at most PH_FEW live tiles (512 of 64 x 64) runs on
// those instead, each on four waves: one a CU while there are that many CUs,
// then two (a half of the waves and of the LDS each).  A product's launch is
// chosen by its capacity, and a gate that opens few rows would leave most of
// the CUs idle and, in float32, the matrix cores of the others busy with
// padding (50 of 23040 rows open: float32 fused injection 193 -> 71 us,
// multi-scale 129 -> 47, bf16 24 -> 19; 500 open 199 -> 80, 137 -> 54, 29 -> 25).
// bf16 over several layers keeps the phased tiles: each 64 x 64 tile of a row
// block streams weights of its own, and the deeper pipeline is the better at
// that (four layers, 50 rows, 61 us against 74).
constexpr int PH_FEW = 32;

// Tiles are numbered batch by batch, inside a batch the column tiles of one
// row block after another (column-major was slower at every shape measured:
// 32768 x 512 x 4096 113 against 142 us), and dealt to the XCDs in contiguous
// ranges; with counts only the live row blocks are numbered, so that every
// XCD gets its share of them (numbered over all rows, a list that is half
// full left half of the XCDs idle).
template <int DT, int EPI>
__global__ __launch_bounds__(512, 2) void phase_gemm_kernel(TileGemmParams a) {
  using S = PgShape<4, 2>;
  constexpr int TCOLS = EPI == EPI_SWIGLU ? S::HN : S::BN;
  __shared__ __attribute__((aligned(1024))) char lds[2 * S::BUF];
  const int tn = (a.cols + TCOLS - 1) / TCOLS;
  auto live = [&](int z) -> int64_t {   // rows of batch z
    if (a.count == nullptr) return a.rows;
    const int64_t c = a.count[z * a.count_step];
    return c < 0 ? 0 : (c < a.rows ? c : a.rows);
  };
  // the batches' live rows in tiles of bm rows, tc tiles across
  auto count_tiles = [&](int bm, int tc) {
    if (a.count == nullptr || a.count_step == 0)
      return (int)((live(0) + bm - 1) / bm) * tc * a.batches;
    int t = 0;
    for (int z = 0; z < a.batches; ++z) t += (int)((live(z) + bm - 1) / bm) * tc;
    return t;
  };
  // batch, live rows, tile row and tile column of such a tile's number
  // (quotients come out of vector instructions: said to be uniform, so that
  // the operands' bases stay in scalar registers)
  auto find_tile = [&](int tile, int bm, int tc, int& z, int64_t& rows, int& tr, int& col) {
    z = 0;
    rows = live(0);
    if (a.count == nullptr || a.count_step == 0) {
      const int per = (int)((rows + bm - 1) / bm) * tc;
      z = __builtin_amdgcn_readfirstlane(tile / per);
      tile -= z * per;
    } else {
      for (int per = (int)((rows + bm - 1) / bm) * tc; tile >= per;
           per = (int)((rows + bm - 1) / bm) * tc) {
        tile -= per;
        rows = live(++z);
      }
    }
    tr = __builtin_amdgcn_readfirstlane(tile / tc);
    col = tile - tr * tc;
  };
  const int total = count_tiles(S::BM, tn);
  int z, tr, tc;
  int64_t rows;
  // (compiled for the products without counts too: without this path the
  // compiler spilled six registers of their float32 loop, and each reload
  // waited for every load in flight)
  if (a.count != nullptr && total <= PH_FEW && (DT == DT_F32 || a.batches == 1)) {
    using T = TgShapeT<2>;
    static_assert(S::BUF == 4 * T::STAGE, "a ring of four stages for each half");
    constexpr int TC = EPI == EPI_SWIGLU ? T::BN / 2 : T::BN;
    const int across = (a.cols + TC - 1) / TC;
    const int units = count_tiles(T::BM, across);
    char (*ring)[T::STAGE] = reinterpret_cast<char (*)[T::STAGE]>(lds);
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    if (units <= PH_ROUND) {
      // a CU each: the other four waves end (a barrier waits for the
      // surviving waves only), their LDS deepens the ring
      const int unit = __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, units));
      if (unit < 0 || half != 0) return;
      find_tile(unit, T::BM, across, z, rows, tr, tc);
      tile_gemm_tile<DT, EPI, 8, 2>(a, ring, z, (int64_t)tr * T::BM, tc * TC, threadIdx.x & 255,
                                    rows, true);
      return;
    }
    const int pair = __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, (units + 1) / 2));
    if (pair < 0) return;
    const bool own = 2 * pair + half < units;   // else the pair's first tile, not stored
    find_tile(own ? 2 * pair + half : 2 * pair, T::BM, across, z, rows, tr, tc);
    tile_gemm_tile<DT, EPI, 4, 2>(a, ring + 4 * half, z, (int64_t)tr * T::BM, tc * TC,
                                  threadIdx.x & 255, rows, own);
    return;
  }
  const PhasePlan pl = phase_plan(total);
  const int first_cut = (pl.whole + 7) / 8 * 8;   // workgroups of the whole tiles
  const bool whole = (int)blockIdx.x < first_cut;
  int tile = whole ? xcd_remap(blockIdx.x, pl.whole)
                   : xcd_remap((int)blockIdx.x - first_cut, 4 * pl.cut);
  if (tile < 0) return;
  tile = __builtin_amdgcn_readfirstlane(tile);
  const int quarter = tile & 3;
  if (!whole) tile = pl.whole + (tile >> 2);
  find_tile(tile, S::BM, tn, z, rows, tr, tc);
  int64_t m0 = (int64_t)tr * S::BM;
  int n0 = tc * TCOLS;
  if (whole) {
    phase_tile<DT, EPI, 4, 2>(a, lds, z, rows, m0, n0);
  } else {
    m0 += (quarter >> 1) * (S::BM / 2);
    n0 += (quarter & 1) * (TCOLS / 2);
    if (m0 < rows && n0 < a.cols) phase_tile<DT, EPI, 2, 1>(a, lds, z, rows, m0, n0);
  }
}

// output columns of a phased tile (a SwiGLU's gate and up columns share it)
template <int EPI>
constexpr int phase_cols() {
  return EPI == EPI_SWIGLU ? PgShape<4, 2>::HN : PgShape<4, 2>::BN;
}

template <int EPI>
static hipError_t launch_phase(int dt, TileGemmParams p, int batches, hipStream_t st) {
  constexpr int TCOLS = phase_cols<EPI>();
  const int64_t tiles = (p.rows + 255) / 256 * ((p.cols + TCOLS - 1) / TCOLS) * batches;
  p.batches = batches;
  const PhasePlan pl = phase_plan((int)tiles);
  // with counts the number of tiles is the device's: any number up to `tiles`
  // needs at most this many workgroups
  const int64_t grid = p.count != nullptr ? tiles + 3 * (PH_ROUND / 2) + 8
                                          : (pl.whole + 7) / 8 * 8 + 4 * pl.cut + 7;
  const dim3 g((unsigned)((grid + 7) / 8 * 8));
  if (dt == DT_BF16)
    hipLaunchKernelGGL((phase_gemm_kernel<DT_BF16, EPI>), g, dim3(512), 0, st, p);
  else
    hipLaunchKernelGGL((phase_gemm_kernel<DT_F32, EPI>), g, dim3(512), 0, st, p);
  return hipGetLastError();
}

// Launches the product over `batches` batches (blockIdx.y), tiles in the
// order that keeps the larger operand's rows on one XCD, with the deepest
// ring its grid's occupancy allows: 8 stages (128 KB of LDS) while every
// workgroup has a CU of its own (at most 256), 4 (64 KB) while all are
// resident at 2 a CU (at most 512), else 2 (32 KB, up to 5 a CU).
template <int EPI>
hipError_t launch_tile_gemm(int dt, TileGemmParams p, int batches, hipStream_t st) {
  // column-major tile order when B has at least as many rows as A
  p.col_major = (int64_t)p.cols * (EPI == EPI_SWIGLU ? 2 : 1) >= p.rows;
  // The phased kernel's lane offsets are 32-bit: rows below 8 MiB, gathered
  // rows inside 4 GiB.
  const bool near = p.a_bytes < (8 << 20) && p.k_bytes < (8 << 20) && p.b_ld < (8 << 20) &&
                    (p.a_sel == nullptr || p.sel_rows * p.a_bytes < ((int64_t)1 << 32));
  if (p.cols % 8 == 0 && near &&
      product_phased(dt, p.rows, p.cols, phase_cols<EPI>(), batches, p.k_bytes))
    return launch_phase<EPI>(dt, p, batches, st);
  if constexpr (EPI != EPI_SWIGLU) {
    // 32-row tiles while every one has a CU of its own and 64-row ones leave
    // half of the CUs idle: a CU's LDS traffic a stage (which bounds these)
    // falls from 48 to 36 KiB.  Image fused injection 30.3 -> 27.4 us,
    // propagated 95.7 -> 89.2 (same sums, same bits).
    const int tiles32 = (int)((p.rows + 31) / 32 * ((p.cols + 63) / 64));
    if ((int64_t)tiles32 * batches <= 256) {
      p.tiles = tiles32;
      const dim3 g((unsigned)((tiles32 + 7) / 8 * 8), (unsigned)batches);
      if (dt == DT_BF16)
        hipLaunchKernelGGL((tile_gemm_kernel<DT_BF16, EPI, 8, 1>), g, dim3(256), 0, st, p);
      else
        hipLaunchKernelGGL((tile_gemm_kernel<DT_F32, EPI, 8, 1>), g, dim3(256), 0, st, p);
      return hipGetLastError();
    }
  }
  const unsigned gx = (unsigned)((p.tiles + 7) / 8 * 8);
  const dim3 grid(gx, (unsigned)batches);
  const int64_t wgs = (int64_t)gx * batches;
  const int ns = wgs <= 256 ? 8 : (wgs <= 512 ? 4 : 2);
  if (dt == DT_BF16) {
    if (ns == 8)
      hipLaunchKernelGGL((tile_gemm_kernel<DT_BF16, EPI, 8>), grid, dim3(256), 0, st, p);
    else if (ns == 4)
      hipLaunchKernelGGL((tile_gemm_kernel<DT_BF16, EPI, 4>), grid, dim3(256), 0, st, p);
    else
      hipLaunchKernelGGL((tile_gemm_kernel<DT_BF16, EPI, 2>), grid, dim3(256), 0, st, p);
  } else {
    if (ns == 8)
      hipLaunchKernelGGL((tile_gemm_kernel<DT_F32, EPI, 8>), grid, dim3(256), 0, st, p);
    else if (ns == 4)
      hipLaunchKernelGGL((tile_gemm_kernel<DT_F32, EPI, 4>), grid, dim3(256), 0, st, p);
    else
      hipLaunchKernelGGL((tile_gemm_kernel<DT_F32, EPI, 2>), grid, dim3(256), 0, st, p);
  }
  return hipGetLastError();
}

}  // namespace lookme
