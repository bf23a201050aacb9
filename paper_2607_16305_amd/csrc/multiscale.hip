// Multi-scale image retrieval with the token-wise router (arXiv 2607.16305,
// Sec. 3.2, Eq. 8).  Each of the M scales was routed and looked up in its
// own scene partition of the table (scenes [m S/M, (m+1) S/M)); for every kept
// token t this file combines the M retrieved rows:
//
//   query      q_t = round(H[t] W_{h->e}) on the matrix cores (tile_gemm.h; the
//              A rows are the kept tokens' hidden states, gathered per row);
//   mix        R^m_t = round(sum_i w^m[t,i] V[partition m, scene^m_t, prim^m[t,i]])
//              for every scale, alpha = softmax_m(q_t . R^m_t / sqrt(d_v)), then
//              H[t, :d_v] = round(H[t, :d_v] + sum_m alpha_m R^m_t):
//              ms_mix_kernel (inject.hip), one workgroup per kept token.
#include "common.h"
#include "kernels.h"
#include "tile_gemm.h"

namespace lookme {

hipError_t launch_multiscale(int dt, int scales, int64_t n, int64_t n_keep, const int32_t* kept,
                             const int32_t* scene, const int32_t* prim, const float* w,
                             const void* values, int S, int P, int d_v, int k,
                             const void* w_he_t, int d_h, void* hidden, void* q,
                             hipStream_t st, const int32_t* count) {
  if (n == 0 || n_keep == 0) return hipSuccess;
  const int es = dt == DT_BF16 ? 2 : 4;
  // q = round(H[kept] W_he)
  TileGemmParams g{};
  g.a0 = static_cast<const char*>(hidden);
  g.a_sel = kept;
  g.sel_rows = (int)n;
  g.b = static_cast<const char*>(w_he_t);
  g.out = static_cast<char*>(q);
  g.rows = n_keep;
  g.a_bytes = (int64_t)d_h * es;
  g.k_bytes = g.a_bytes;
  g.cols = d_v;
  g.count = count;   // a counted list: rows past count[0] are skipped
  g.count_step = 0;
  g.tiles = (int)(((n_keep + TgShape::BM - 1) / TgShape::BM) *
                  ((d_v + TgShape::BN - 1) / TgShape::BN));
  const hipError_t e = launch_tile_gemm<EPI_STORE>(dt, g, 1, st);
  if (e != hipSuccess) return e;

  return launch_ms_mix(dt, scales, n, n_keep, kept, scene, prim, w, values, S / scales, P, d_v, k,
                       q, d_h, hidden, st, count);
}

}  // namespace lookme
