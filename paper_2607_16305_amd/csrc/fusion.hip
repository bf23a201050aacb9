// Sparse injection through the SwiGLU fusion of Eq. 10 (arXiv 2607.16305,
// Sec. 3.3): for the kept tokens of layer l, H <- round(H + f_l(R)) with
// f_l(R) = W_down (silu(W_gate R) * (W_up R)).  R (the weighted row sums,
// rounded) comes from launch_gather_rows; two products on the matrix cores
// (tile_gemm.h), batched over the layers (blockIdx.y):
//
//   gate/up   U = round(silu(R W_gate^T) * (R W_up^T)): every tile computes
//             32 columns of both products for the same rows and combines
//             them in its epilogue;
//   down      H[kept] = round(H[kept] + U W_down^T), written in place (the
//             kept list of the layer maps a product row to its token).
//
// The inter-layer propagation of Eq. 11 (launch_propagate) carries R from a
// LookME layer to the layers after it: R_j = round(R_{j-1} W_p^j + R_{j-1}),
// one product per layer (each needs the previous one), the residual added in
// the epilogue.
#include "common.h"
#include "kernels.h"
#include "tile_gemm.h"

namespace lookme {

// bf16: the phased kernel from 48 tiles of 256 x 256 on (192 quarters): 2304 x
// 2048 x 2048 for four layers 310 -> 149 us (gate/up) and 147 -> 85 us (down),
// 512 x 2048 x 2048 for four layers (64 tiles) 31 -> 24.5 us; below it too few
// of the CUs get one: 1024 x 2048 x 2048 (32 tiles) 17.2 us on 64 x 64 tiles,
// 18.0 phased, 512 x 2048 x 2048 13.2 and 16.5.  Short sums (K of at most 1 KiB
// a row) are over before the deeper pipeline pays, so they take it where most
// of a round is whole tiles (relevance lookups of 20011 rows, 158 tiles, 131.9
// us on 64 x 64 tiles and 129.1 phased; of 12000, 94 tiles, 125.2 and 132.2;
// 4000 x 2048 x 512, 128, 19.0 and 20.5).
// A last row or column tile that is mostly padding costs a whole one, and 64 x
// 64 tiles fill a last round better, so the outputs have to be worth the
// phased kernel's rounds: a round of whole tiles takes as long as `round` whole
// tiles' worth of 64 x 64 ones (float32, bound by the matrix cores on either,
// 195; bf16 90, short sums 125), a round of quarters `quarter` of that.  On 64 x
// 64 tiles and phased: bf16 16385 x 128 x 4096 38 and 57 us, 2 x 600 rows of a
// fused injection (d_v 1152, d_ff 1600) 38.9 and 43.0, 12000 x 640 x 640
// of short sums 67.6 and 76.9; 8192 x 320 x 4096 39.5 and 31.6; float32 131072 x
// 64 x 1024 168 and 483, x 256 632 and 500, 257 rows of four layers (d_v 2048,
// d_ff 4096) 601 and 694, 12000 x 1024 x 2048 (188 tiles) 462 and 469, 16385 x
// 768 x 2048 (193) 496 and 473, 4096 x 2048 x 2048 (128) 314 and 252.
bool product_phased(int dt, int64_t rows, int64_t cols, int tile_cols, int64_t batches,
                    int64_t k_bytes) {
  const bool f32 = dt != DT_BF16, brief = k_bytes <= 1024;
  const int64_t tiles = (rows + 255) / 256 * ((cols + tile_cols - 1) / tile_cols) * batches;
  if (!f32 && tiles < (brief ? 129 : 48)) return false;
  const int sub_cols = tile_cols / 4;
  const int64_t subs = (rows + 63) / 64 * ((cols + sub_cols - 1) / sub_cols) * batches;
  const PhasePlan pl = phase_plan((int)tiles);
  const double round = f32 ? 195. : brief ? 125. : 90., quarter = f32 ? 0.25 : 0.35;
  const double rounds = (pl.whole + PH_ROUND - 1) / PH_ROUND +
                        quarter * ((4 * pl.cut + PH_ROUND - 1) / PH_ROUND);
  return 16. * round * rounds < (double)subs;
}

hipError_t launch_fusion(int dt, const FusionFfn& f, int layers, int64_t n, int64_t n_keep,
                         const int32_t* kept, int64_t kept_batch, int d_v, const void* r, void* u,
                         void* hidden, hipStream_t st, const int32_t* count) {
  if (n == 0 || n_keep == 0) return hipSuccess;
  const int es = dt == DT_BF16 ? 2 : 4;
  const int64_t rt = (n_keep + TgShape::BM - 1) / TgShape::BM;

  TileGemmParams g1{};
  g1.a0 = static_cast<const char*>(r);
  g1.b = static_cast<const char*>(f.w_gate);
  g1.b2 = static_cast<const char*>(f.w_up);
  g1.out = static_cast<char*>(u);
  g1.rows = n_keep;
  g1.a_bytes = (int64_t)d_v * es;
  g1.k_bytes = g1.a_bytes;
  g1.a_batch = n_keep * g1.a_bytes;
  g1.b_batch = (int64_t)f.d_ff * g1.k_bytes;
  g1.out_batch = n_keep * (int64_t)f.d_ff * es;
  g1.cols = f.d_ff;
  g1.tiles = (int)(rt * ((f.d_ff + TgShape::BN / 2 - 1) / (TgShape::BN / 2)));
  g1.count = count;
  g1.count_step = kept_batch != 0 ? 1 : 0;
  hipError_t e = launch_tile_gemm<EPI_SWIGLU>(dt, g1, layers, st);
  if (e != hipSuccess) return e;

  TileGemmParams g2{};
  g2.a0 = static_cast<const char*>(u);
  g2.b = static_cast<const char*>(f.w_down);
  g2.out = static_cast<char*>(hidden);
  g2.kept = kept;
  g2.rows = n_keep;
  g2.a_bytes = (int64_t)f.d_ff * es;
  g2.k_bytes = g2.a_bytes;
  g2.a_batch = n_keep * g2.a_bytes;
  g2.b_batch = (int64_t)f.d_h * g2.k_bytes;
  g2.n = n;
  g2.kept_batch = kept_batch;
  g2.out_ld = (int64_t)f.d_h * es;
  g2.cols = f.d_h;
  g2.tiles = (int)(rt * ((f.d_h + TgShape::BN - 1) / TgShape::BN));
  g2.count = count;
  g2.count_step = g1.count_step;
  return launch_tile_gemm<EPI_RESID>(dt, g2, layers, st);
}

hipError_t launch_propagate(int dt, const void* w_p_t, int steps, int64_t n_keep, int d_v,
                            void* r, hipStream_t st, const int32_t* count) {
  if (n_keep == 0) return hipSuccess;
  const int64_t es = dt == DT_BF16 ? 2 : 4;
  const int64_t slice = n_keep * d_v * es;
  const int64_t rt = (n_keep + TgShape::BM - 1) / TgShape::BM;
  for (int j = 1; j <= steps; ++j) {
    TileGemmParams g{};
    g.a0 = static_cast<const char*>(r) + (j - 1) * slice;
    g.res = g.a0;
    g.b = static_cast<const char*>(w_p_t) + (int64_t)(j - 1) * d_v * d_v * es;
    g.out = static_cast<char*>(r) + j * slice;
    g.rows = n_keep;
    g.a_bytes = (int64_t)d_v * es;
    g.k_bytes = g.a_bytes;
    g.cols = d_v;
    g.tiles = (int)(rt * ((d_v + TgShape::BN - 1) / TgShape::BN));
    g.count = count;
    g.count_step = 0;
    const hipError_t e = launch_tile_gemm<EPI_ADD>(dt, g, 1, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lookme
