// MFMA tile core shared by the engine, the tile GEMM and the gradient
// contraction kernels (gfx950, wave64).
//
// A workgroup of 4 wave64 computes one 128x128 output tile; wave (wr, wc)
// owns the 64x64 quadrant (wr, wc) as 4x4 MFMA 16x16 sub-tiles.  Where a launch
// has too few tiles to fill the chip the tile is cut into 64x64 or 32x32 pieces, a
// workgroup each, and a wave owns 2x2 sub-tiles or one.  Every element sums its
// products in the same order in these forms (not where parts or waves share k).
// Whole tiles with float64 products take their operands through LDS (wg_gemm).
// Elsewhere (wave_gemm: pieces, thin tiles, float32 products) operand
// fragments are read straight from HBM/L2 in the MFMA 16x16x4 input layout
// (lane l supplies row l%16 and four consecutive k values starting at
// 4*(l/16)); the four MFMA k-steps of a 16-wide k chunk consume those four
// values, so each lane issues one contiguous 4-element load per sub-tile row
// per chunk and the next chunks are prefetched while the current one runs on
// the matrix cores.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lma {

typedef double dv4 __attribute__((ext_vector_type(4)));
typedef float fv4 __attribute__((ext_vector_type(4)));

template <typename T>
struct V4;
template <>
struct V4<double> { typedef dv4 type; };
template <>
struct V4<float> { typedef fv4 type; };

template <typename Tc>
struct Mfma;
template <>
struct Mfma<double> {
  typedef dv4 acc;
  __device__ static inline acc op(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // register v of lane l holds row (l/16) + 4v, column l%16 of the 16x16 tile
  __device__ static inline int row(int l, int v) { return (l >> 4) + 4 * v; }
};
template <>
struct Mfma<float> {
  typedef fv4 acc;
  __device__ static inline acc op(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // register v of lane l holds row 4*(l/16) + v, column l%16 of the 16x16 tile
  __device__ static inline int row(int l, int v) { return 4 * (l >> 4) + v; }
};

__device__ inline double k_exp(double x) { return exp(x); }
__device__ inline float k_exp(float x) { return expf(x); }
__device__ inline double k_sqrt(double x) { return sqrt(x); }
__device__ inline float k_sqrt(float x) { return sqrtf(x); }

// Workgroups are dealt round-robin to the 8 XCDs; remap so that consecutive
// work items (tiles of the same problem, which share the B operand) land on
// the same XCD and its L2.  The grid is padded to a multiple of 8.
__device__ inline int xcd_logical(int bid, int nb) {
  const int per = nb >> 3;
  return (bid & 7) * per + (bid >> 3);
}

// acc[ra][rb] += A[arow0 + 16 ra + i, k] * Bm[brow0 + 16 rb + j, k] over k in [k0, k1).
// Rows at or past anr / bnr are read from row 0 instead (always a valid
// address): they only feed output rows / columns that the callers either do
// not store or overwrite with their exact value (padding).  Loads are
// unconditional and rotate through PF+1 register slots, so the chunk in use
// never waits for the chunks in flight.
// PERMA feeds the A rows of each 16-row sub-tile in the order r(4a+b) = a+4b, which
// turns the float32 16x16 output layout into the float64 one (row l/16 + 4v).
// wave_gemm_fold (float32 accumulation, PERMA layout): every FOLD_ITERS steady
// iterations (FOLD_ITERS*(PF+1)*16 k, 144 by default) the float32 accumulators are
// added into the float64 ones and restarted from zero.  A single float32 chain over
// the thousands of k of a late column step loses accuracy linearly in k (about 10x a
// blocked float32 Cholesky at k ~ 3000); chains of 144 are more accurate than one.
constexpr int FOLD_ITERS = 3;
constexpr int FOLD_CHUNKS = FOLD_ITERS * 3;  // 16-wide chunks per fold with the prefetch depth of 2 that folding uses
template <typename Tin, typename Tc, bool PERMA, int PF, bool FOLD, int RA, int RB>
__device__ __forceinline__ void wave_gemm_impl(typename Mfma<Tc>::acc (&acc)[RA][RB],
                                               const Tin* __restrict__ A, int64_t lda, int anr,
                                               const Tin* __restrict__ Bm, int64_t ldb, int bnr,
                                               int k0, int k1, int arow0, int brow0, int lane,
                                               dv4 (&fold)[RA][RB]) {
  static_assert(!FOLD || (PERMA && std::is_same<Tc, float>::value), "folding needs the float64 output layout");
  typedef typename V4<Tin>::type vin;
  const int r16 = lane & 15, kq = (lane >> 4) << 2;
  const Tin* pa[RA];
  const Tin* pb[RB];
#pragma unroll
  for (int t = 0; t < RA; ++t) {
    const int ra = arow0 + t * 16 + (PERMA ? ((r16 >> 2) | ((r16 & 3) << 2)) : r16);
    pa[t] = A + (int64_t)(ra < anr ? ra : 0) * lda + k0 + kq;
  }
#pragma unroll
  for (int t = 0; t < RB; ++t) {
    const int rb = brow0 + t * 16 + r16;
    pb[t] = Bm + (int64_t)(rb < bnr ? rb : 0) * ldb + k0 + kq;
  }
  const int nc = (k1 - k0) >> 4;
  if (nc <= 0) return;
  vin sa[PF + 1][RA], sb[PF + 1][RB];
  // chunk x lives in slot x % (PF+1)
#define LMA_LOAD_CHUNK(X, SLOT)                                \
  {                                                            \
    const int off_ = (X) << 4;                                 \
    const int slot_ = (SLOT);                                  \
    _Pragma("unroll") for (int u_ = 0; u_ < RA; ++u_)          \
      sa[slot_][u_] = *(const vin*)(pa[u_] + off_);            \
    _Pragma("unroll") for (int u_ = 0; u_ < RB; ++u_)          \
      sb[slot_][u_] = *(const vin*)(pb[u_] + off_);            \
  }
#define LMA_MMA_SLOT(SLOT)                                                                 \
  {                                                                                        \
    const int slot_ = (SLOT);                                                              \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                        \
      _Pragma("unroll") for (int ra = 0; ra < RA; ++ra) {                                  \
        _Pragma("unroll") for (int rb = 0; rb < RB; ++rb) {                                \
          acc[ra][rb] = Mfma<Tc>::op((Tc)sa[slot_][ra][e], (Tc)sb[slot_][rb][e], acc[ra][rb]); \
        }                                                                                  \
      }                                                                                    \
    }                                                                                      \
  }
#define LMA_FOLD()                                                                    \
  if constexpr (FOLD) {                                                              \
    _Pragma("unroll") for (int a_ = 0; a_ < RA; ++a_) {                              \
      _Pragma("unroll") for (int b_ = 0; b_ < RB; ++b_) {                            \
        _Pragma("unroll") for (int v_ = 0; v_ < 4; ++v_) {                           \
          fold[a_][b_][v_] += (double)acc[a_][b_][v_];                               \
          acc[a_][b_][v_] = Tc(0);                                                   \
        }                                                                            \
      }                                                                              \
    }                                                                                \
  }
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (p < nc) LMA_LOAD_CHUNK(p, p)
  int c = 0;
  int since_fold = 0;
  // steady state: every prefetch is in range, no branches in the body
  for (; c + 2 * PF < nc; c += PF + 1) {
#pragma unroll
    for (int q = 0; q <= PF; ++q) {
      LMA_LOAD_CHUNK(c + q + PF, (q + PF) % (PF + 1))
      LMA_MMA_SLOT(q)
    }
    if constexpr (FOLD) {
      if (++since_fold == FOLD_ITERS) {
        since_fold = 0;
        LMA_FOLD()
      }
    }
  }
  // tail: at most 2*PF+1 chunks, slots known at compile time
#pragma unroll
  for (int t = 0; t <= 2 * PF; ++t) {
    if (c + t < nc) {
      if (c + t + PF < nc) LMA_LOAD_CHUNK(c + t + PF, (t + PF) % (PF + 1))
      LMA_MMA_SLOT(t % (PF + 1))
    }
  }
  LMA_FOLD()
#undef LMA_LOAD_CHUNK
#undef LMA_MMA_SLOT
#undef LMA_FOLD
}

// chunks in flight: a wave of fewer sub-tiles has fewer products per chunk to cover
// the latency of the next ones, and registers to spare
constexpr int pf_of(int sub) { return sub >= 4 ? 2 : sub == 2 ? 3 : 5; }

template <typename Tin, typename Tc, int RA, int RB>
__device__ __forceinline__ void wave_gemm(typename Mfma<Tc>::acc (&acc)[RA][RB],
                                          const Tin* __restrict__ A, int64_t lda, int anr,
                                          const Tin* __restrict__ Bm, int64_t ldb, int bnr,
                                          int k0, int k1, int arow0, int brow0, int lane) {
  dv4 unused[RA][RB];
  wave_gemm_impl<Tin, Tc, false, pf_of(RA > RB ? RA : RB), false>(acc, A, lda, anr, Bm, ldb, bnr, k0, k1, arow0, brow0,
                                                                 lane, unused);
}

// float32 products (PERMA layout) with the sums folded into the float64 accumulators fold
template <int RA, int RB>
__device__ __forceinline__ void wave_gemm_fold(fv4 (&acc)[RA][RB], const float* __restrict__ A, int64_t lda, int anr,
                                               const float* __restrict__ Bm, int64_t ldb, int bnr, int k0, int k1,
                                               int arow0, int brow0, int lane, dv4 (&fold)[RA][RB]) {
  wave_gemm_impl<float, float, true, 2, true>(acc, A, lda, anr, Bm, ldb, bnr, k0, k1, arow0, brow0, lane, fold);
}

// Accumulators start as the result of an MFMA of zero operands (exactly +0):
// started from constant zeros, the compiler keeps the loop-carried accumulators
// of a k loop in vector registers and copies all of them into the accumulation
// registers and back on every iteration; an MFMA result stays in place.
template <typename Tc, int RA, int RB>
__device__ inline void zero_acc(typename Mfma<Tc>::acc (&acc)[RA][RB]) {
#pragma unroll
  for (int a = 0; a < RA; ++a)
#pragma unroll
    for (int b = 0; b < RB; ++b) acc[a][b] = Mfma<Tc>::op(Tc(0), Tc(0), (typename Mfma<Tc>::acc){Tc(0), Tc(0), Tc(0), Tc(0)});
}

// ---------------------------------------------------------------------------
// whole 128 x 128 tile by one workgroup, float64 products, operands through LDS
// ---------------------------------------------------------------------------
// Stages of 16 k, double-buffered.  While a stage is multiplied, the next one goes
// from registers to the other buffer and the one after it is loaded (16 bytes a lane,
// whole 128-byte row pieces).  The one barrier of a stage lies between its two halves
// of 32 products; what the second half needs is in registers by then, and the first
// operands of the next stage are read under it, so neither the barrier nor the LDS
// latency shows.  Read from LDS the operands need half the registers that chunks in
// flight from memory need, so two workgroups fit on a CU.  The products of an element
// are summed in the same order as in wave_gemm.
// Measured with 4096 tiles of k = 4096 (peak 78.6 TFLOP/s): 63.0 for wave_gemm straight
// from memory with one workgroup per CU, 65.2 for two plain stages in LDS, 66.5 with
// the barrier between the halves, 71.9 with the LDS writes and loads dealt out among
// the products (matrix cores busy 92 %; 88 % over the whole-tile launches of an n=524288 step).  With 256 tiles, one per CU, both forms take
// the same time (668 and 679 us).
constexpr int SLD = 18;                                          // row stride in LDS: 16 rows touch every bank once
constexpr size_t WG_GEMM_LDS = 2 * 2 * 128 * SLD * sizeof(double);  // two stages of 128 + 128 rows
typedef double dv2 __attribute__((ext_vector_type(2)));

// Barrier of the workgroup that orders its LDS accesses only: loads from memory stay
// in flight.
__device__ inline void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Called by all 256 threads with the same arguments.  Rows at or past anr / bnr are
// read from row 0, as in wave_gemm; (row count) * ld * sizeof(Tin) is below 4 GiB.
template <typename Tin>
__device__ __forceinline__ void wg_gemm(dv4 (&acc)[4][4], const Tin* __restrict__ A, int64_t lda, int anr,
                                        const Tin* __restrict__ Bm, int64_t ldb, int bnr, int k0, int k1, double* sm) {
  constexpr int PER = 16 / sizeof(Tin);   // elements a lane loads at once
  constexpr int LPR = 16 / PER;           // lanes per row
  constexpr int RPI = 256 / LPR;          // rows per load of the workgroup
  constexpr int NL = 128 / RPI;           // loads per operand and stage
  typedef Tin vin __attribute__((ext_vector_type(PER)));
  const int nc = (k1 - k0) >> 4;
  if (nc <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wr = w >> 1, wc = w & 1;
  const int row = tid / LPR, col = tid % LPR * PER;
  uint32_t oa[NL], ob[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int r = row + i * RPI;
    oa[i] = (uint32_t)(((int64_t)(r < anr ? r : 0) * lda + col) * sizeof(Tin));
    ob[i] = (uint32_t)(((int64_t)(r < bnr ? r : 0) * ldb + col) * sizeof(Tin));
  }
  const char* pa = reinterpret_cast<const char*>(A + k0);
  const char* pb = reinterpret_cast<const char*>(Bm + k0);
  vin st[2 * NL];
  auto load = [&](int c) {
    const char* qa = pa + (int64_t)c * 16 * sizeof(Tin);
    const char* qb = pb + (int64_t)c * 16 * sizeof(Tin);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      st[i] = *reinterpret_cast<const vin*>(qa + oa[i]);
      st[NL + i] = *reinterpret_cast<const vin*>(qb + ob[i]);
    }
  };
  double* wp = sm + row * SLD + col;
  auto store = [&](int b) {
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) {
      double* q = wp + (b * 256 + i * RPI) * SLD;
#pragma unroll
      for (int e = 0; e < PER; e += 2) *reinterpret_cast<dv2*>(q + e) = (dv2){(double)st[i][e], (double)st[i][e + 1]};
    }
  };
  const double* ra = sm + (wr * 64 + (lane & 15)) * SLD + 4 * (lane >> 4);
  const double* rb = sm + (128 + wc * 64 + (lane & 15)) * SLD + 4 * (lane >> 4);
  dv2 f0[8], f1[8];
  auto frags = [&](dv2 (&f)[8], int b, int h) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f[t] = *reinterpret_cast<const dv2*>(ra + (b * 256 + 16 * t) * SLD + 2 * h);
      f[4 + t] = *reinterpret_cast<const dv2*>(rb + (b * 256 + 16 * t) * SLD + 2 * h);
    }
  };
  auto mul = [&](const dv2 (&f)[8]) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = Mfma<double>::op(f[x][e], f[4 + y][e], acc[x][y]);
  };
  // One stage: DEEP 2, two more stages follow; 1, one more; 0, the last.  The LDS writes
  // and the loads are dealt out among the products: issued in one go they hold up
  // their wave, and the other wave of the SIMD is often at the same place.
  auto stage = [&](int c, auto deep) {
    constexpr int DEEP = decltype(deep)::value;
    const int b = c & 1;
    frags(f1, b, 1);
    if constexpr (DEEP > 0) store(1 - b);
    if constexpr (DEEP > 1) load(c + 2);
    mul(f0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      if constexpr (DEEP > 0) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
      if constexpr (DEEP > 1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // load
    }
    if constexpr (DEEP > 0) {
      barrier_lds();
      frags(f0, 1 - b, 0);
    }
    mul(f1);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 1);
      if constexpr (DEEP > 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
    }
  };
  load(0);
  barrier_lds();  // the buffers may still be read by what came before
  store(0);
  barrier_lds();
  if (nc > 1) load(1);
  frags(f0, 0, 0);
  int c = 0;
  for (; c + 2 < nc; ++c) stage(c, std::integral_constant<int, 2>());
  if (c + 1 < nc) stage(c++, std::integral_constant<int, 1>());
  stage(c, std::integral_constant<int, 0>());
}

}  // namespace lma
