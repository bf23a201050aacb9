// Large products C = A B^T on the matrix cores, K in 128-byte stages: eight
// waves in 2 x 4 on a tile whose A and B rows are two halves each, so that a
// stage is four parts (A0, A1, B0, B1) and a wave owns 16 MI x 16 NJ outputs
// of every (A half, B half) quadrant.  The four quadrants of a stage are four
// phases; a phase multiplies one quadrant from registers, reads the part the
// next one needs from LDS and refills the part read one phase before with
// the stage after next:
//
//   phase  multiplies   reads       loads (global to LDS)
//   0      A0 x B0      B1(s)       B0(s + 2)
//   1      A0 x B1      A1(s)       B1(s + 2)
//   2      A1 x B1      A0(s + 1)   A1(s + 2)
//   3      A1 x B0      B0(s + 1)   A0(s + 3)
//
// Two stage buffers thus carry almost two stages of loads in flight (a part
// has seven phases to arrive), and no product waits for an LDS read of its
// own phase.  The loads are buffer loads (load_lds16_at): with 64-bit
// addresses each took vector instructions and two registers beside the 240
// that accumulators and fragments fill (23040 x 2048 x 2048 193.7 -> 185.5
// us, 1042 TFLOP/s; 32768 x 512 x 4096, a shape that the projection's own
// kernel takes beside another stream, 113 us, 1216).  What bounds it: without
// the loads 98 us of those 113, without the products 76, so the stage stream
// out of L2 and the LDS it shares with the fragment reads.  The weights' rows
// are MFMA operand A and the tokens' rows operand B, with the weight rows of
// the NJ tiles of a wave dealt so that a lane ends with 4 NJ neighbouring
// columns of one output row: the epilogues read and write 16 bytes a lane.
#pragma once

#include "common.h"
#include "dtl.h"

namespace lookme {

template <int MI, int NJ>
struct PgShape {
  static constexpr int HM = 32 * MI, HN = 64 * NJ;        // rows of an A (B) half
  static constexpr int BM = 2 * HM, BN = 2 * HN;
  static constexpr int PA = HM / 64, PB = HN / 64;        // 1 KiB loads a wave issues per part
  static constexpr int A_PART = HM * 128, B_PART = HN * 128;
  static constexpr int BUF = 2 * (A_PART + B_PART);
  static constexpr int W = 4 * NJ;                        // columns a lane holds side by side
  static_assert(MI % 2 == 0, "whole load shares");
};

// chunk c of row r of a part sits in slot c ^ pg_swz: the 16 rows of a
// fragment read take every slot twice.  A fragments (and B with one tile)
// read 16 consecutive rows; the B rows of tile j of two are 8 a + 4 j + b.
template <int NJ>
__device__ __forceinline__ int pg_swz(int r) {
  if constexpr (NJ == 2) return (r & 3) | (((r >> 3) & 1) << 2);
  else return r & 7;
}

// The accumulators of A B^T for the tile: acc[qi][qj][i][j] element r is
// row 16 MI wr + 16 i + n16 of A half qi and column 16 NJ wc + W g + 4 j + r
// of B half qj (wave (wr, wc), lane (g, n16)).  lds: 2 BUF bytes, all waves
// of the workgroup take part.  The loads come from the caller: ld.a(h, stage,
// dst) issues this wave's PA loads of A half h of a stage to dst (1 KiB
// each), ld.b the PB loads of a B half, and ld.next() ends a stage's loads.
template <int DT, int MI, int NJ>
struct PgLoop {
  using S = PgShape<MI, NJ>;
  char* lds;
  int lane, wv, n16, g, wr, wc;

  __device__ __forceinline__ PgLoop(char* l, int tid) : lds(l) {
    lane = tid & 63;
    wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    n16 = lane & 15;
    g = lane >> 4;
    wr = wv >> 2;
    wc = wv & 3;
  }
  // row (inside its half) of load q of an A (B) part, and the lane's chunk
  __device__ __forceinline__ int a_row(int q) const { return (wv * S::PA + q) * 8 + (lane >> 3); }
  __device__ __forceinline__ int b_row(int q) const { return (wv * S::PB + q) * 8 + (lane >> 3); }
  __device__ __forceinline__ int a_chunk(int q) const { return (lane & 7) ^ pg_swz<1>(a_row(q)); }
  __device__ __forceinline__ int b_chunk(int q) const { return (lane & 7) ^ pg_swz<NJ>(b_row(q)); }

  __device__ __forceinline__ char* a_dst(int h, int stage) const {
    return lds + (stage & 1) * S::BUF + h * S::A_PART + wv * S::PA * 1024;
  }
  __device__ __forceinline__ char* b_dst(int h, int stage) const {
    return lds + (stage & 1) * S::BUF + 2 * S::A_PART + h * S::B_PART + wv * S::PB * 1024;
  }
  __device__ __forceinline__ void read_a(int h, int stage, u32x4_t (&f)[2][MI]) const {
    const char* p = lds + (stage & 1) * S::BUF + h * S::A_PART + (wr * 16 * MI + n16) * 128;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int o = ((4 * ks + g) ^ pg_swz<1>(n16)) << 4;
#pragma unroll
      for (int i = 0; i < MI; ++i) f[ks][i] = *reinterpret_cast<const u32x4_t*>(p + i * 2048 + o);
    }
  }
  __device__ __forceinline__ void read_b(int h, int stage, u32x4_t (&f)[2][NJ]) const {
    const int r0 = NJ == 2 ? 8 * (n16 >> 2) + (n16 & 3) : n16;
    const char* p = lds + (stage & 1) * S::BUF + 2 * S::A_PART + h * S::B_PART +
                    (wc * 16 * NJ + r0) * 128;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int o = ((4 * ks + g) ^ pg_swz<NJ>(r0)) << 4;   // the same for both tiles
#pragma unroll
      for (int j = 0; j < NJ; ++j) f[ks][j] = *reinterpret_cast<const u32x4_t*>(p + j * 512 + o);
    }
  }
  static __device__ __forceinline__ void mma(const u32x4_t (&fa)[2][MI],
                                             const u32x4_t (&fb)[2][NJ],
                                             f32x4_t (&acc)[MI][NJ]) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma_chunk<DT>(fb[ks][j], fa[ks][i], acc[i][j]);
  }
  // ends a phase: this wave's LDS reads have returned and all but the V
  // youngest of its loads have landed; then the barrier (a plain s_barrier:
  // the fence of __syncthreads would wait for every load in flight)
  template <int V>
  static __device__ __forceinline__ void sync() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), in a form the compiler counts
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(V) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }

  // one stage; fb0 holds B0(s), fb1 receives B1(s) and then B0(s + 1)
  // (before phase k the part it reads is the oldest of the seven loaded
  // last: the six younger ones may be in flight).  done(q): quadrant q
  // (2 qi + qj) of the stage has been multiplied; called in order of q, beside
  // the products of the phase after it or (2 and 3) at the end.
  template <class Ld, class Done>
  __device__ __forceinline__ void stage(int s, Ld& ld, f32x4_t (&acc)[2][2][MI][NJ],
                                        u32x4_t (&fa0)[2][MI], u32x4_t (&fa1)[2][MI],
                                        u32x4_t (&fb0)[2][NJ], u32x4_t (&fb1)[2][NJ],
                                        Done&& done) const {
    constexpr int PA = S::PA, PB = S::PB;
    sync<4 * PA + 2 * PB>();
    read_b(1, s, fb1);
    ld.b(0, s + 2, b_dst(0, s + 2));
    mma(fa0, fb0, acc[0][0]);
    sync<3 * PA + 3 * PB>();
    read_a(1, s, fa1);
    ld.b(1, s + 2, b_dst(1, s + 2));
    mma(fa0, fb1, acc[0][1]);
    done(0);
    sync<2 * PA + 4 * PB>();
    read_a(0, s + 1, fa0);
    ld.a(1, s + 2, a_dst(1, s + 2));
    mma(fa1, fb1, acc[1][1]);
    done(1);
    sync<3 * PA + 3 * PB>();
    read_b(0, s + 1, fb1);
    ld.next();
    ld.a(0, s + 3, a_dst(0, s + 3));
    mma(fa1, fb0, acc[1][0]);
    done(2);
    done(3);
  }

  // done(s, q): see stage
  template <class Ld, class Done>
  __device__ __forceinline__ void run(int nst, Ld& ld, f32x4_t (&acc)[2][2][MI][NJ],
                                      Done&& done) const {
    constexpr int PA = S::PA, PB = S::PB;
#pragma unroll
    for (int qi = 0; qi < 2; ++qi)
#pragma unroll
      for (int qj = 0; qj < 2; ++qj)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) acc[qi][qj][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t fa0[2][MI], fa1[2][MI], fbx[2][NJ], fby[2][NJ];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      ld.a(0, s, a_dst(0, s));
      ld.b(0, s, b_dst(0, s));
      ld.b(1, s, b_dst(1, s));
      ld.a(1, s, a_dst(1, s));
      ld.next();
    }
    sync<3 * PA + 3 * PB>();   // A0(0) and B0(0) have landed
    read_a(0, 0, fa0);
    read_b(0, 0, fbx);
    sync<3 * PA + 3 * PB>();   // and every wave has read A0(0)
    ld.a(0, 2, a_dst(0, 2));
    int s = 0;
    for (; s + 1 < nst; s += 2) {
      stage(s, ld, acc, fa0, fa1, fbx, fby, [&](int q) { done(s, q); });
      stage(s + 1, ld, acc, fa0, fa1, fby, fbx, [&](int q) { done(s + 1, q); });
    }
    if (s < nst) stage(s, ld, acc, fa0, fa1, fbx, fby, [&](int q) { done(s, q); });
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // no load into LDS outlives the wave
  }
};

// The loads of one tile of A B^T: uniform bases (of the tile's A rows, of
// each B half) and 32-bit lane offsets of load q of a part of half h (row +
// chunk).  Past the last stage it is read again, so that the waits keep their
// counts.
template <class S>
struct PgLoads {
  const char* a_base;
  const char* b_base[2];
  uint32_t oa[2][S::PA], ob[2][S::PB];
  int last;
  __device__ __forceinline__ void a(int h, int stage, char* dst) const {
    const int k = (stage < last ? stage : last) * 128;
#pragma unroll
    for (int q = 0; q < S::PA; ++q) load_lds16_at(a_base, oa[h][q], k, dst + q * 1024);
  }
  __device__ __forceinline__ void b(int h, int stage, char* dst) const {
    const int k = (stage < last ? stage : last) * 128;
#pragma unroll
    for (int q = 0; q < S::PB; ++q) load_lds16_at(b_base[h], ob[h][q], k, dst + q * 1024);
  }
  __device__ __forceinline__ void next() const {}
};

// W neighbouring elements of a row as float32, and back with one rounding.
template <int DT, int W>
__device__ __forceinline__ void ld_cols(const char* p, float (&v)[W]) {
  if constexpr (DT == DT_BF16) {
    uint32_t u[W / 2];
    if constexpr (W == 8) {
      const u32x4_t t = ld16(p);
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = t[e];
    } else {
      const uint2 t = *reinterpret_cast<const uint2*>(p);
      u[0] = t.x;
      u[1] = t.y;
    }
#pragma unroll
    for (int e = 0; e < W / 2; ++e) {
      v[2 * e] = bf16lo(u[e]);
      v[2 * e + 1] = bf16hi(u[e]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < W / 4; ++q) {
      const f32x4_t t = *reinterpret_cast<const f32x4_t*>(p + 16 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * q + e] = t[e];
    }
  }
}
template <int DT, int W>
__device__ __forceinline__ void st_cols(char* p, const float (&v)[W]) {
  if constexpr (DT == DT_BF16) {
    uint32_t u[W / 2];
#pragma unroll
    for (int e = 0; e < W / 2; ++e) u[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
    if constexpr (W == 8) st16(p, u32x4_t{u[0], u[1], u[2], u[3]});
    else *reinterpret_cast<uint2*>(p) = make_uint2(u[0], u[1]);
  } else {
#pragma unroll
    for (int q = 0; q < W / 4; ++q)
      *reinterpret_cast<f32x4_t*>(p + 16 * q) =
          f32x4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
  }
}

}  // namespace lookme
