// Query projection v_e = v W_{v->e} (arXiv 2607.16305, Sec. 3.2, Level-1),
// for all layers at once: the per-layer matrices are stacked along the
// output dimension, so x is read once for every layer.
//
// C[M, N] = A[M, K] . B[N, K]^T with A = x [n, d_in], B = W^T stacked
// [layers * d_e, d_in]; C is rounded once to the storage dtype and scattered
// to q[layer, token, :].  Large batches run as a tile_gemm.h product, or on
// project_round_kernel where they are one round of 256 x 256 tiles.  The
// others are tiled on LDS here: a BM x BN output tile per 4 waves in a 2 x 2
// grid, 128-byte K stages double-buffered in LDS (rows padded by 16 bytes so
// the 16-byte fragment reads of 8 consecutive rows hit distinct banks), the
// global loads of the next D stages in flight while one is multiplied.
#include "common.h"
#include "kernels.h"
#include "tile_gemm.h"

namespace lookme {

constexpr int PJ_STAGE = 128;                // bytes of K per stage and row
constexpr int PJ_LD = PJ_STAGE + 16;         // padded LDS row pitch
constexpr int PJ_THREADS = 256;
constexpr int PJ_CPR = PJ_STAGE / 16;        // 16-byte chunks per row per stage

// Rounds a wave's accumulators once to the storage dtype and scatters them
// to q[layer, token, :]: the lane holds C[r0 + 16i + 4g + r][c0 + 16j + n16].
template <int DT, int MI, int NJ>
__device__ __forceinline__ void store_tile(const f32x4_t (&acc)[MI][NJ], char* __restrict__ Q,
                                           int64_t M, int N, int d_e, int64_t r0, int c0,
                                           int n16, int g) {
  constexpr int ES = DT == DT_BF16 ? 2 : 4;
  const int64_t layer_stride = M * d_e;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int col = c0 + 16 * j + n16;
    if (col >= N) continue;
    const int layer = col / d_e, jj = col % d_e;
    char* qcol = Q + ((int64_t)layer * layer_stride + jj) * ES;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = r0 + 16 * i + 4 * g + r;
        if (row < M) {
          if constexpr (DT == DT_BF16)
            *reinterpret_cast<uint16_t*>(qcol + row * d_e * ES) =
                (uint16_t)f32_to_bf16_rne(acc[i][j][r]);
          else
            *reinterpret_cast<float*>(qcol + row * d_e * ES) = acc[i][j][r];
        }
      }
    }
  }
}

// D: K stages whose global loads are in flight while one stage is multiplied
// (a ring of D register sets; every load is issued unconditionally, with
// its address clamped and its value zeroed when it lies outside the operand,
// so that the compiler's wait counts stay exact).  KG: groups of 4 waves that
// split K between them (group g takes stages g, g + KG, ...), each with its
// own LDS buffers; their partial tiles are summed through LDS in group order
// at the end, so a small M x N still keeps many loads in flight per tile.
template <int DT, int BM, int BN, int D, int KG>
__global__ __launch_bounds__(PJ_THREADS * KG) void project_kernel(
    const char* __restrict__ A, const char* __restrict__ B, char* __restrict__ Q, int64_t M,
    int N, int64_t k_bytes, int d_e, int tiles) {
  static_assert(D % 2 == 0, "the LDS buffer of a step is its parity");
  constexpr int MI = BM / 32, NJ = BN / 32;  // 16 x 16 MFMA tiles per wave
  constexpr int LA = BM * PJ_CPR / PJ_THREADS, LB = BN * PJ_CPR / PJ_THREADS;
  static_assert(LA >= 1 && LB >= 1, "a stage must cover every thread");
  __shared__ __attribute__((aligned(16))) char lds_a[KG][2][BM * PJ_LD];
  __shared__ __attribute__((aligned(16))) char lds_b[KG][2][BN * PJ_LD];
  const int tid = threadIdx.x & (PJ_THREADS - 1);
  const int kg = __builtin_amdgcn_readfirstlane(threadIdx.x / PJ_THREADS);
  const int lane = tid & 63, wv = tid >> 6;
  const int n16 = lane & 15, g = lane >> 4;
  const int wm = (wv >> 1) * (BM / 2), wn = (wv & 1) * (BN / 2);

  // tiles of one row block are neighbours in the work order and run on one
  // XCD, so their shared A rows come from that XCD's L2
  const int tiles_n = (N + BN - 1) / BN;
  const int tile = xcd_remap(blockIdx.x, tiles);
  if (tile < 0) return;
  const int64_t m0 = (int64_t)(tile / tiles_n) * BM;
  const int n0 = (tile % tiles_n) * BN;
  const int kchunks = (int)(k_bytes / 16);
  const int nstages = (int)((k_bytes + PJ_STAGE - 1) / PJ_STAGE);
  const int per_group = (nstages + KG - 1) / KG;
  const int nsteps = (per_group + D - 1) / D * D;   // padded: stages past K are zero

  u32x4_t ra[D][LA], rb[D][LB];
  auto gload = [&](u32x4_t (&a)[LA], u32x4_t (&b)[LB], int step) {
    const int stage = step * KG + kg;
#pragma unroll
    for (int r = 0; r < LA; ++r) {
      const int ci = tid + r * PJ_THREADS;
      const int kc = stage * PJ_CPR + ci % PJ_CPR;
      const int64_t am = m0 + ci / PJ_CPR;
      const bool ok = am < M && kc < kchunks;
      const u32x4_t v = ld16(A + (ok ? am * k_bytes + (int64_t)kc * 16 : 0));
      a[r] = ok ? v : u32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int r = 0; r < LB; ++r) {
      const int ci = tid + r * PJ_THREADS;
      const int kc = stage * PJ_CPR + ci % PJ_CPR;
      const int bn = n0 + ci / PJ_CPR;
      const bool ok = bn < N && kc < kchunks;
      const u32x4_t v = ld16(B + (ok ? (int64_t)bn * k_bytes + (int64_t)kc * 16 : 0));
      b[r] = ok ? v : u32x4_t{0, 0, 0, 0};
    }
  };
  auto lstore = [&](int buf, const u32x4_t (&a)[LA], const u32x4_t (&b)[LB]) {
#pragma unroll
    for (int r = 0; r < LA; ++r) {
      const int ci = tid + r * PJ_THREADS;
      st16(&lds_a[kg][buf][(ci / PJ_CPR) * PJ_LD + (ci % PJ_CPR) * 16], a[r]);
    }
#pragma unroll
    for (int r = 0; r < LB; ++r) {
      const int ci = tid + r * PJ_THREADS;
      st16(&lds_b[kg][buf][(ci / PJ_CPR) * PJ_LD + (ci % PJ_CPR) * 16], b[r]);
    }
  };

  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
#pragma unroll
    for (int s = 0; s < PJ_STAGE / 64; ++s) {
      u32x4_t fa[MI], fb[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i)
        fa[i] = *reinterpret_cast<const u32x4_t*>(
            &lds_a[kg][buf][(wm + 16 * i + n16) * PJ_LD + (4 * s + g) * 16]);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        fb[j] = *reinterpret_cast<const u32x4_t*>(
            &lds_b[kg][buf][(wn + 16 * j + n16) * PJ_LD + (4 * s + g) * 16]);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma_chunk<DT>(fa[i], fb[j], acc[i][j]);
    }
  };

  // prologue: steps 0..D-1 in flight, step 0 in LDS buffer 0
#pragma unroll
  for (int d = 0; d < D; ++d) {
    gload(ra[d], rb[d], d);
    asm volatile("" ::: "memory");   // keep the issue order: older steps first
  }
  lstore(0, ra[0], rb[0]);
  __syncthreads();
  for (int st = 0; st < nsteps; st += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      // set d held step st+d, already in LDS: refill it with step st+d+D
      gload(ra[d], rb[d], st + d + D);
      compute(d & 1);
      // step st+d+1 (register set (d+1)%D) into the other buffer, which was
      // last read in the previous step, finished by every wave before the
      // barrier that ended it
      lstore((d + 1) & 1, ra[(d + 1) % D], rb[(d + 1) % D]);
      __syncthreads();
    }
  }

  if constexpr (KG > 1) {
    // partial tiles of groups 1..KG-1 through their (now idle) LDS buffers,
    // added by group 0 in group order; lane-private slots, no bank pattern
    // matters for this one pass
    static_assert(MI * NJ * PJ_THREADS * 16 <= 2 * (BM + BN) * PJ_LD,
                  "partial tile fits the buffers");
    // the buffers of one group are lds_a[g] (both halves) then lds_b[g]:
    // not contiguous, so the partial tile is split over lds_a[g] and lds_b[g]
    auto slot = [&](int grp, int idx) -> f32x4_t* {
      constexpr int IN_A = 2 * BM * PJ_LD / 16;   // f32x4 slots in lds_a[grp]
      const int e = idx * 256 + tid;               // wave-interleaved, 16 B per lane
      return e < IN_A ? reinterpret_cast<f32x4_t*>(&lds_a[grp][0][0]) + e
                      : reinterpret_cast<f32x4_t*>(&lds_b[grp][0][0]) + (e - IN_A);
    };
    if (kg > 0) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) *slot(kg, i * NJ + j) = acc[i][j];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int o = 1; o < KG; ++o)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const f32x4_t p = *slot(o, i * NJ + j);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] += p[r];
        }
  }

  store_tile<DT, MI, NJ>(acc, Q, M, N, d_e, m0 + wm, n0 + wn, n16, g);
}

// One round of 256 x 256 tiles (at most one a CU), fed by direct global-to-LDS
// loads: 16 waves in 4 x 4, each 4 x 4 MFMA tiles, two 128-byte K stages (the
// loads of stage s + 1 fly during stage s).  Its waves take a quarter of a
// SIMD's registers less than the phased kernel's (tile_gemm.h) and so leave
// room for a wave of another stream's norms or select, which the phased
// kernel does not; see launch_project.  A load instruction fills 1 KB:
// neighbouring lanes read one row's contiguous bytes, whose 16-byte chunks
// are permuted by blk_swz so that the fragment reads hit distinct LDS banks.
constexpr int PR_WM = 4, PR_WN = 4, PR_MI = 4, PR_NJ = 4, PR_KB = 128;
using PrShape = DtlShape<PR_WM, PR_WN, PR_MI, PR_NJ, PR_KB>;

template <int DT>
__global__ __launch_bounds__(64 * PR_WM * PR_WN) void project_round_kernel(
    const char* __restrict__ A, const char* __restrict__ B, char* __restrict__ Q, int64_t M,
    int N, int64_t k_bytes, int d_e, int tiles) {
  using S = PrShape;
  constexpr int MI = PR_MI, NJ = PR_NJ, KB = PR_KB, KSL = KB / 64;
  __shared__ __attribute__((aligned(1024))) char lds[2][S::STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n16 = lane & 15, g = lane >> 4;
  const int wm = (wv / PR_WN) * 16 * MI, wn = (wv % PR_WN) * 16 * NJ;

  const int tiles_n = (N + S::BN - 1) / S::BN;
  const int tile = xcd_remap(blockIdx.x, tiles);
  if (tile < 0) return;
  const int64_t m0 = (int64_t)(tile / tiles_n) * S::BM;
  const int n0 = (tile % tiles_n) * S::BN;
  const int nst = (int)(k_bytes / KB);

  // load q of a stage covers tile rows [q RPI, q RPI + RPI) (A rows first,
  // then B rows).  Rows past the edge are clamped into the operand and feed
  // only outputs that are never stored.
  const char* src[S::PER_WAVE];
#pragma unroll
  for (int b = 0; b < S::PER_WAVE; ++b) {
    const int trow = (wv * S::PER_WAVE + b) * S::RPI + lane / S::LPR;
    const int chunk = (lane % S::LPR) ^ blk_swz<KB>(trow & 15);
    if (trow < S::BM) {
      int64_t r = m0 + trow;
      r = r < M ? r : M - 1;
      src[b] = A + r * k_bytes + chunk * 16;
    } else {
      int r = n0 + trow - S::BM;
      r = r < N ? r : N - 1;
      src[b] = B + (int64_t)r * k_bytes + chunk * 16;
    }
  }
  auto issue = [&](int stage) {
    const int s = stage < nst ? stage : nst - 1;   // past the end: a harmless reload
    char* dst = lds[stage & 1];
#pragma unroll
    for (int b = 0; b < S::PER_WAVE; ++b)
      load_lds16(src[b] + (int64_t)s * KB, dst + (wv * S::PER_WAVE + b) * 1024);
  };

  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  issue(0);
  for (int s = 0; s < nst; ++s) {
    // stage s has landed everywhere and every read of stage s - 1 (the other
    // buffer) has ended (a plain s_barrier: the empty asm keeps LDS accesses
    // on their side of it)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(s + 1);
    const char* buf = lds[s & 1];
    u32x4_t fa[KSL][MI], fb[KSL][NJ];
#pragma unroll
    for (int ks = 0; ks < KSL; ++ks) {
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[ks][i] = read_frag<KB>(buf, wm + 16 * i, ks, n16, g);
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb[ks][j] = read_frag<KB>(buf, S::BM + wn + 16 * j, ks, n16, g);
    }
#pragma unroll
    for (int ks = 0; ks < KSL; ++ks)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma_chunk<DT>(fa[ks][i], fb[ks][j], acc[i][j]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load into LDS outlives the wave
  store_tile<DT, MI, NJ>(acc, Q, M, N, d_e, m0 + wm, n0 + wn, n16, g);
}

template <int DT>
static void launch_round(const void* x, const void* wt, void* q, int64_t n, int N, int64_t kb,
                         int d_e, int tiles, hipStream_t st) {
  hipLaunchKernelGGL(project_round_kernel<DT>, dim3((unsigned)((tiles + 7) / 8 * 8)),
                     dim3(64 * PR_WM * PR_WN), 0, st, static_cast<const char*>(x),
                     static_cast<const char*>(wt), static_cast<char*>(q), n, N, kb, d_e, tiles);
}

template <int DT, int BM, int BN, int D, int KG>
static void launch_tiles(const void* x, const void* wt, void* q, int64_t n, int N, int64_t kb,
                         int d_e, hipStream_t st) {
  const int64_t tiles = ((n + BM - 1) / BM) * ((N + BN - 1) / BN);
  const int64_t slots = (tiles + 7) / 8 * 8;
  hipLaunchKernelGGL((project_kernel<DT, BM, BN, D, KG>), dim3((unsigned)slots),
                     dim3(PJ_THREADS * KG), 0,
                     st, static_cast<const char*>(x), static_cast<const char*>(wt),
                     static_cast<char*>(q), n, N, kb, d_e, (int)tiles);
}

// One nearly full round of large tiles leaves no CU to the norms and the
// select of a second stream, which then hold up the routing: beside them the
// phased kernel, whose tiles fill a CU's registers, made the step of 32768
// rows 2.235 ms, its 128 x 256 tiles in two rounds 2.169 (projection 150 us),
// project_round_kernel 2.147 (134 us).  Alone: 32768 x 512 x 4096 113 us
// phased, 122 here; 32768 x 512 x 2048 69.5 us on 128 x 256 tiles, 64.6 here;
// float32 616 us on 64 x 64 tiles, 567 here.  bf16 sums of at most 1 KiB of
// K are over before the phased pipeline is full, so half a round is enough
// for it there (5000 x 2048 x 512 26.9 us phased, 25.5 here; 16384 x 512 x
// 512 25.7 us on 64 x 64 tiles, 24.9 here).
// Tiles that are mostly padding leave that to the 64 x 64 ones (on those and
// here: float32 65536 x 64 x 2048 166 us and 521, x 192 466 and 521, 16384 x
// 896 540 and 519; bf16 32768 x 64 x 512 13.5 and 23.3, 16384 x 320 x 512
// 20.7 and 24.0, 8192 x 896 x 512 24.6 and 28.4).
bool project_one_round(int dt, int64_t n, int64_t cols, int64_t k_bytes) {
  const int64_t large = ((n + 255) / 256) * ((cols + 255) / 256);
  const int64_t filled = ((n + 63) / 64) * ((cols + 63) / 64) / 16;
  const bool brief = dt == DT_BF16 && k_bytes <= 1024;
  return k_bytes % PR_KB == 0 && large <= 256 && large > (brief ? 127 : 224) &&
         filled > (dt != DT_BF16 ? 200 : brief && large == 128 ? 112 : 100);
}

hipError_t launch_project(int dt, const void* x, const void* wt, void* q, int64_t n, int d_in,
                          int d_e, int layers, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int es = dt == DT_BF16 ? 2 : 4;
  const int N = layers * d_e;
  const int64_t kb = (int64_t)d_in * es;
  if (project_one_round(dt, n, N, kb)) {
    const int64_t large = ((n + 255) / 256) * ((N + 255) / 256);
    if (dt == DT_BF16) launch_round<DT_BF16>(x, wt, q, n, N, kb, d_e, (int)large, st);
    else launch_round<DT_F32>(x, wt, q, n, N, kb, d_e, (int)large, st);
    return hipGetLastError();
  }
  // The 32 x 64 tiles below split K over four wave groups, one workgroup a CU:
  // right while every tile has a CU of its own (1024 x 512 x 2048, 256 tiles:
  // 10.9 us against 12.1 on 64 x 64 tiles), slow after (2000 x 512 x 2048
  // 20.1 and 12.8 us, 4000 x 512 x 2048 40.1 and 16.6, 2000 x 2048 x 512 49.3
  // and 11.1).  float32 keeps them until the chip is full of 128 x 128 tiles:
  // its sums are stored as they are, and four partial sums err less than one.
  const int64_t tiles128 = ((n + 127) / 128) * ((N + 127) / 128);
  const int64_t tiles_k4 = ((n + 31) / 32) * ((N + 63) / 64);
  if (kb % TG_KB == 0 && (dt == DT_BF16 ? tiles_k4 > 256 : tiles128 >= 256)) {
    TileGemmParams p{};
    p.a0 = static_cast<const char*>(x);
    p.b = static_cast<const char*>(wt);
    p.out = static_cast<char*>(q);
    p.rows = n;
    p.a_bytes = kb;
    p.k_bytes = kb;
    p.cols = N;
    p.d_e = d_e;
    p.tiles = (int)(((n + TgShape::BM - 1) / TgShape::BM) * ((N + TgShape::BN - 1) / TgShape::BN));
    return launch_tile_gemm<EPI_Q>(dt, p, 1, st);
  }
  // else 32 x 64 tiles with K split over 4 wave groups
  if (dt == DT_BF16) launch_tiles<DT_BF16, 32, 64, 4, 4>(x, wt, q, n, N, kb, d_e, st);
  else launch_tiles<DT_F32, 32, 64, 4, 4>(x, wt, q, n, N, kb, d_e, st);
  return hipGetLastError();
}

}  // namespace lookme
