// Device kernels of the tiled Cholesky / triangular-solve engine (gfx950).
// The MFMA tile core (operand layout, prefetch pipeline) is in mfma_core.h.
#include "engine.h"
#include "mfma_core.h"

#include <algorithm>
#include <type_traits>

namespace lma {

// ---------------------------------------------------------------------------
// update: C_ij = K_ij - V_i V_j^T - sum_{k<j} L_ik L_jk^T for every item (p, i)
// ---------------------------------------------------------------------------
// SUB: MFMA sub-tiles per wave and side.  4: a workgroup computes the whole 128 x 128
// tile; 2 and 1: one of its 4 (16) pieces of 64 x 64 (32 x 32).  FIX: the products were
// formed by k_update_part; their a.nsplit parts are added in order.
template <typename T, bool MIXED, int SUB, bool FIX = false>
__global__ __launch_bounds__(NT, (std::is_same<T, double>::value && SUB == 4) ? 2 : 1) void k_update(StepArgs<T> a) {
  constexpr bool WG = std::is_same<T, double>::value && SUB == 4 && !FIX;  // operands through LDS
  constexpr int WS = 16 * SUB, QS = 2 * WS, NQ = TB / QS;  // rows of a wave, of a piece; pieces per side
  // covariance tile and V-part precision: float64 when T is double or MIXED
  typedef typename std::conditional<MIXED, double, T>::type TK;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * NQ * NQ) return;
  const WorkItem it = a.items[logical / (NQ * NQ)];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  const RowTile<T> rj = a.rt[pd.first + a.j];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int q0r = (logical / NQ) % NQ * QS, q0c = logical % NQ * QS;  // the piece's first row and column
  const bool diag = ri.is_j && (it.tile == a.j);
  if (q0r >= ri.nstore) return;         // no row of the piece is stored
  if (diag && q0c > q0r) return;        // above the diagonal: not read by the diagonal tile's kernel
  const int r0 = q0r + (w >> 1) * WS, c0 = q0c + (w & 1) * WS;  // the wave's
  const bool real = q0r < ri.nvalid && q0c < rj.nvalid;         // else padding only

  typename Mfma<TK>::acc accv[SUB][SUB];   // V_i V_j^T
  typename Mfma<T>::acc accl[SUB][SUB];    // sum_k L_ik L_jk^T (aliases accv when not MIXED)
  const bool band = ri.src == SRC_BAND;    // V part already inside the band entries
  const bool tband = ri.src == SRC_TBAND;  // likewise for test rows
  if (band || tband) {
    // Band rows start from minus their residual entries, so that the band reads
    // are in flight with the first operand loads instead of after the k loop;
    // the epilogue then stores -(accumulator).  Every lane issues its 64 reads
    // unconditionally (padding rows and columns read a valid entry of the tile and
    // are masked to zero), and the accumulators are started through an MFMA, as
    // in zero_acc, so that they stay in their register file.
    const int nvr = ri.nvalid, nvc = rj.nvalid;
    int64_t rowp[SUB][4], rowb[SUB][4], colq[SUB], colb[SUB];
#pragma unroll
    for (int cs = 0; cs < SUB; ++cs) {
      const int col = c0 + cs * 16 + (lane & 15);
      colq[cs] = rj.pt0 + (col < nvc ? col : nvc - 1);
      colb[cs] = tband ? 0 : a.brow[colq[cs]];
    }
#pragma unroll
    for (int rs = 0; rs < SUB; ++rs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = r0 + rs * 16 + Mfma<TK>::row(lane, v);
        rowp[rs][v] = ri.pt0 + (row < nvr ? row : nvr - 1);
        rowb[rs][v] = a.brow[rowp[rs][v]];
      }
#pragma unroll
    for (int rs = 0; rs < SUB; ++rs)
#pragma unroll
      for (int cs = 0; cs < SUB; ++cs) {
        typename Mfma<TK>::acc start;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = r0 + rs * 16 + Mfma<TK>::row(lane, v);
          const int col = c0 + cs * 16 + (lane & 15);
          const int64_t p = rowp[rs][v], q = colq[cs];
          const int64_t e = (tband || q <= p) ? rowb[rs][v] + q : colb[cs] + p;
          const TK kv = (TK)a.band[e];
          start[v] = (row < nvr && col < nvc) ? -kv : TK(0);
        }
        accv[rs][cs] = Mfma<TK>::op(TK(0), TK(0), start);
      }
  } else {
    zero_acc<TK>(accv);
  }
  if constexpr (MIXED) zero_acc<T>(accl);
  const TK* vi = MIXED ? (const TK*)ri.vt64 : (const TK*)ri.vt;
  const TK* vj = MIXED ? (const TK*)rj.vt64 : (const TK*)rj.vt;
  if (!FIX && real && !band && !tband && vi != nullptr && vj != nullptr && a.vlen > 0)
    if constexpr (WG)
      wg_gemm<TK>(accv, vi, a.vld, ri.nvalid, vj, a.vld, rj.nvalid, 0, a.vlen, reinterpret_cast<double*>(smem_raw));
    else
      wave_gemm<TK, TK>(accv, vi, a.vld, ri.nvalid, vj, a.vld, rj.nvalid, 0, a.vlen, r0, c0, lane);
  // factor columns kb .. j-1 (a row is zero left of its kbeg)
  const int kb = ri.kbeg > rj.kbeg ? ri.kbeg : rj.kbeg;
  if constexpr (FIX) {
    // several parts in flight (one after the other they took 1 us each)
    constexpr int FLY = SUB == 1 ? 8 : 2;
    const double* part = a.part + (int64_t)(logical / (NQ * NQ)) * a.nsplit * TB * TB;
    auto add = [&](auto np) {
      constexpr int NP = decltype(np)::value;
      double q[NP][SUB][SUB][4];
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int rs = 0; rs < SUB; ++rs)
#pragma unroll
          for (int cs = 0; cs < SUB; ++cs)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              q[p][rs][cs][v] =
                  part[p * TB * TB + (r0 + rs * 16 + Mfma<TK>::row(lane, v)) * TB + c0 + cs * 16 + (lane & 15)];
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int rs = 0; rs < SUB; ++rs)
#pragma unroll
          for (int cs = 0; cs < SUB; ++cs)
#pragma unroll
            for (int v = 0; v < 4; ++v) accv[rs][cs][v] += (TK)q[p][rs][cs][v];
      part += NP * TB * TB;
    };
    int p = 0;
    for (; p + FLY <= a.nsplit; p += FLY) add(std::integral_constant<int, FLY>());
    for (; p < a.nsplit; ++p) add(std::integral_constant<int, 1>());
  } else if (real && a.j > kb) {
    const T* pa = ri.panel + (int64_t)(kb - ri.kbeg) * TB;
    const T* pb = rj.panel + (int64_t)(kb - rj.kbeg) * TB;
    if constexpr (MIXED)  // float32 products, sums folded into the float64 accumulators
      wave_gemm_fold(accl, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, 0, (a.j - kb) * TB, r0, c0, lane,
                     accv);
    else if constexpr (WG)
      wg_gemm<T>(accv, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, 0, (a.j - kb) * TB,
                 reinterpret_cast<double*>(smem_raw));
    else
      wave_gemm<T, T>(accv, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, 0, (a.j - kb) * TB, r0, c0, lane);
  }

  const int d = a.d;
  TK* xr = reinterpret_cast<TK*>(smem_raw);  // [d][QS] row-side coordinates
  TK* xc = xr + d * QS;                      // [d][QS] column-side coordinates
  const bool kern = ri.src == SRC_KERNEL;
  if (WG && kern) __syncthreads();  // the operand stages lie where the coordinates go
  if (kern) {
    const TK* xsi = MIXED ? (const TK*)ri.xs64 : (const TK*)ri.xs;
    const TK* xsj = MIXED ? (const TK*)rj.xs64 : (const TK*)rj.xs;
    for (int idx = tid; idx < QS * d; idx += NT) {
      const int r = idx / d, t = idx - r * d;
      xr[t * QS + r] = q0r + r < ri.nvalid ? xsi[(int64_t)(q0r + r) * d + t] : TK(0);
      xc[t * QS + r] = q0c + r < rj.nvalid ? xsj[(int64_t)(q0c + r) * d + t] : TK(0);
    }
  }
  __syncthreads();
  const TK sf2 = (TK)a.sf2, sn2 = (TK)a.sn2;
  T* out = ri.panel + (int64_t)(a.j - ri.kbeg) * TB;
  const bool ident = ri.src == SRC_IDENT;
  const bool ident_here = ident && ri.kbeg == a.j;
#pragma unroll
  for (int rs = 0; rs < SUB; ++rs) {
    // squared distances of a 16-row strip, one coordinate at a time
    TK sq[SUB][4];
#pragma unroll
    for (int cs = 0; cs < SUB; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) sq[cs][v] = TK(0);
    if (kern && real) {
      for (int t = 0; t < d; ++t) {
        TK cv[SUB];
#pragma unroll
        for (int cs = 0; cs < SUB; ++cs) cv[cs] = xc[t * QS + c0 - q0c + cs * 16 + (lane & 15)];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const TK rv = xr[t * QS + r0 - q0r + rs * 16 + Mfma<TK>::row(lane, v)];
#pragma unroll
          for (int cs = 0; cs < SUB; ++cs) {
            const TK df = rv - cv[cs];
            sq[cs][v] += df * df;
          }
        }
      }
    }
#pragma unroll
    for (int cs = 0; cs < SUB; ++cs) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = r0 + rs * 16 + Mfma<TK>::row(lane, v);
        const int col = c0 + cs * 16 + (lane & 15);
        TK kv = TK(0);
        if (ident) {
          kv = (ident_here && row == col) ? TK(1) : TK(0);  // exact at padding too
        } else if (row < ri.nvalid && col < rj.nvalid) {
          if (kern) {
            kv = sf2 * k_exp(TK(-0.5) * sq[cs][v]);
            if (diag && row == col) kv += sn2;
          } else if (band || tband) {
            kv = TK(0);  // the residual entry started the accumulator (negated)
          } else if (ri.src == SRC_EXPLICIT) {
            kv = (TK)ri.expl[(int64_t)row * ri.eld + (int64_t)a.j * TB + col];
          } else {
            kv = row == 0 ? (TK)rj.cv[col] : TK(0);
          }
        } else if (diag && row == col) {
          kv = TK(1);
        }
        T val;
        if (row >= ri.nvalid || col >= rj.nvalid)
          val = (T)kv;  // padding: identity on the diagonal tile, zero elsewhere
        else if constexpr (MIXED)
          val = (T)(kv - accv[rs][cs][v]);  // accl was folded into accv
        else
          val = (T)(kv - accv[rs][cs][v]);
        if (row < ri.nstore) out[(int64_t)row * ri.ld + col] = val;
      }
    }
  }
}

// Part `piece` of a.nsplit of the sums over k of every item's tile, to the workspace.
// Where the tiles of a launch leave the last turn of the CUs nearly empty, or are
// fewer than the CUs, parts along k fill them at the full rate of whole tiles (64 x 64
// pieces reach half of it); k_update with FIX adds the parts.  In mixed precision the
// parts end where a float32 sum is folded, so only float64 sums are reordered.
template <typename T, bool MIXED>
__global__ __launch_bounds__(NT, (std::is_same<T, double>::value) ? 2 : 1) void k_update_part(StepArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * a.nsplit) return;
  const int piece = logical / a.nitems, item = logical - piece * a.nitems;
  const WorkItem it = a.items[item];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  const RowTile<T> rj = a.rt[pd.first + a.j];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r0 = (w >> 1) * 64, c0 = (w & 1) * 64;
  dv4 acc[4][4];
  zero_acc<double>(acc);
  const int kb = ri.kbeg > rj.kbeg ? ri.kbeg : rj.kbeg;
  // 16-wide chunks per indivisible step; wave_gemm_fold joins a last chunk of its own to
  // the group before it
  constexpr int U = MIXED ? FOLD_CHUNKS : 1;
  const int nc = (a.j - kb) * (TB / 16), nu = U > 1 && nc % U == 1 ? nc / U : (nc + U - 1) / U;
  const int k0 = 16 * U * (nu * piece / a.nsplit);
  const int k1 = piece + 1 < a.nsplit ? 16 * U * (nu * (piece + 1) / a.nsplit) : 16 * nc;
  const T* pa = ri.panel + (int64_t)(kb - ri.kbeg) * TB;
  const T* pb = rj.panel + (int64_t)(kb - rj.kbeg) * TB;
  if constexpr (MIXED) {
    fv4 accl[4][4];
    zero_acc<float>(accl);
    if (k1 > k0) wave_gemm_fold(accl, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, k0, k1, r0, c0, lane, acc);
  } else {
    if (k1 > k0)
      wg_gemm<T>(acc, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, k0, k1, reinterpret_cast<double*>(smem_raw));
  }
  double* out = a.part + ((int64_t)item * a.nsplit + piece) * TB * TB;
#pragma unroll
  for (int rs = 0; rs < 4; ++rs)
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        out[(r0 + rs * 16 + Mfma<double>::row(lane, v)) * TB + c0 + cs * 16 + (lane & 15)] = acc[rs][cs][v];
}

// ---------------------------------------------------------------------------
// thin tiles: at most 16 RS valid rows
// ---------------------------------------------------------------------------
// Bound: reading the other operand once.  A whole tile costs its 128 rows of products
// however few are real; here a workgroup takes 16 of the 128 columns and its 8 waves
// share the sums over k, so a launch of 60 tiles has 4000 waves with six chunks in flight
// each.  The waves' sums are added through LDS in order.
// Measured: test rows of 100 points (62 tiles of 1 to 14 rows, k up to 3000) 108 -> 45 us
// a launch, their products with the support rows 664 -> 250 us, their residual band (with
// tiles over several blocks) 506 -> 83; a prediction 3.41 -> 1.60 ms, covariance of 512
// points 2.73 -> 2.17 ms, fit and prediction of n=65536 34.8 -> 34.0 ms, mixed n=50021
// 53.2 -> 51.0, n=262144 all updates 690 -> 676.
template <int RS>
struct ThinShape {
  static constexpr int NW = 8, THREADS = 64 * NW, ELEMS = RS * 256;  // NW whatever RS is
};

// this wave's share of [k0, k1) in units of U chunks of 16; a last chunk of its own joins
// the unit before it (as the folds of wave_gemm_fold do)
template <int U, int NW>
__device__ inline void thin_share(int k0, int k1, int w, int* a, int* b) {
  const int nc = (k1 - k0) >> 4, nu = U > 1 && nc % U == 1 && nc > 1 ? nc / U : (nc + U - 1) / U;
  *a = k0 + 16 * U * (nu * w / NW);
  *b = w + 1 < NW ? k0 + 16 * U * (nu * (w + 1) / NW) : k0 + 16 * nc;
}

// red[w][row][16 columns] of this wave, then the barrier
template <int RS>
__device__ inline void thin_put(const dv4 (&acc)[RS][1], double* red, int w, int lane) {
#pragma unroll
  for (int rs = 0; rs < RS; ++rs)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      red[w * ThinShape<RS>::ELEMS + (rs * 16 + Mfma<double>::row(lane, v)) * 16 + (lane & 15)] = acc[rs][0][v];
  __syncthreads();
}
template <int RS>
__device__ inline double thin_sum(const double* red, int e) {
  double s = red[e];
#pragma unroll
  for (int w = 1; w < ThinShape<RS>::NW; ++w) s += red[w * ThinShape<RS>::ELEMS + e];
  return s;
}

// groups: row groups of 16 RS per tile; 1 for thin tiles (their other rows are zero).
// Launches of a few whole tiles take the same form: a 32 x 32 piece of such a tile was one
// serial chain over k on a quarter of its MFMA slots.  n = 16 tiles, k = 128 .. 1280: 9 ..
// 37 us as pieces, 5 .. 26 here (the rate is that of the operands from L2, 33 TFLOP/s).
template <typename T, bool MIXED, int RS>
__global__ __launch_bounds__(ThinShape<RS>::THREADS) void k_update_slim(StepArgs<T> a, int groups) {
  typedef typename std::conditional<MIXED, double, T>::type TK;
  static_assert(std::is_same<TK, double>::value, "sums in float64");
  constexpr int NW = ThinShape<RS>::NW, RG = 16 * RS;
  __shared__ double red[NW * ThinShape<RS>::ELEMS];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * 8 * groups) return;
  const WorkItem it = a.items[logical / (8 * groups)];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  const RowTile<T> rj = a.rt[pd.first + a.j];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = logical / 8 % groups * RG, c0 = logical % 8 * 16;
  const bool diag = ri.is_j && it.tile == a.j;
  if (r0 >= ri.nstore || (diag && c0 >= r0 + RG)) return;
  const bool real = r0 < ri.nvalid && c0 < rj.nvalid, band = ri.src == SRC_BAND || ri.src == SRC_TBAND;
  dv4 acc[RS][1];
  zero_acc<double>(acc);
  const double* vi = MIXED ? ri.vt64 : (const double*)ri.vt;
  const double* vj = MIXED ? rj.vt64 : (const double*)rj.vt;
  int k0, k1;
  if (real && !band && vi != nullptr && vj != nullptr && a.vlen > 0) {
    thin_share<1, NW>(0, a.vlen, w, &k0, &k1);
    wave_gemm<double, double>(acc, vi, a.vld, ri.nvalid, vj, a.vld, rj.nvalid, k0, k1, r0, c0, lane);
  }
  const int kb = ri.kbeg > rj.kbeg ? ri.kbeg : rj.kbeg;
  if (real && a.j > kb) {
    const T* pa = ri.panel + (int64_t)(kb - ri.kbeg) * TB;
    const T* pb = rj.panel + (int64_t)(kb - rj.kbeg) * TB;
    thin_share<MIXED ? FOLD_CHUNKS : 1, NW>(0, (a.j - kb) * TB, w, &k0, &k1);
    if constexpr (MIXED) {
      fv4 accl[RS][1];
      zero_acc<float>(accl);
      wave_gemm_fold(accl, pa, ri.ld, ri.nvalid, pb, rj.ld, rj.nstore, k0, k1, r0, c0, lane, acc);
    } else {
      wave_gemm<T, T>(acc, pa, ri.ld, ri.nvalid, pb, rj.ld, rj.nstore, k0, k1, r0, c0, lane);
    }
  }
  thin_put<RS>(acc, red, w, lane);
  T* out = ri.panel + (int64_t)(a.j - ri.kbeg) * TB + c0;
  const int stored = ri.nstore - r0 < RG ? ri.nstore - r0 : RG;
#pragma unroll 1
  for (int e = tid; e < stored * 16; e += ThinShape<RS>::THREADS) {
    const int row = r0 + (e >> 4), col = c0 + (e & 15);
    double val = 0.0;
    if (ri.src == SRC_IDENT) {
      val = ri.kbeg == a.j && row == col ? 1.0 : 0.0;
      if (row < ri.nvalid && col < rj.nvalid) val -= thin_sum<RS>(red, e);
    } else if (row < ri.nvalid && col < rj.nvalid) {
      if (band) {
        const int64_t p = ri.pt0 + row, q = rj.pt0 + col;
        val = (double)a.band[ri.src == SRC_TBAND || q <= p ? a.brow[p] + q : a.brow[q] + p];
      } else if (ri.src == SRC_KERNEL) {
        const double* x = (MIXED ? ri.xs64 : (const double*)ri.xs) + (int64_t)row * a.d;
        const double* y = (MIXED ? rj.xs64 : (const double*)rj.xs) + (int64_t)col * a.d;
        double sq = 0.0;
        for (int t = 0; t < a.d; ++t) {
          const double df = x[t] - y[t];
          sq += df * df;
        }
        val = a.sf2 * k_exp(-0.5 * sq);
        if (diag && row == col) val += a.sn2;
      } else if (ri.src == SRC_EXPLICIT) {
        val = (double)ri.expl[(int64_t)row * ri.eld + (int64_t)a.j * TB + col];
      } else {
        val = row == 0 ? (double)rj.cv[col] : 0.0;
      }
      val -= thin_sum<RS>(red, e);
    } else if (diag && row == col) {
      val = 1.0;  // padding: identity on the diagonal tile, zero elsewhere
    }
    out[(int64_t)row * ri.ld + (e & 15)] = (T)val;
  }
  if (groups == 1)
    for (int e = tid + 16 * RG; e < ri.nstore * 16; e += ThinShape<RS>::THREADS)
      out[(int64_t)(e >> 4) * ri.ld + (e & 15)] = T(0);
}

template <typename T, int RS>
__global__ __launch_bounds__(ThinShape<RS>::THREADS) void k_tile_gemm_slim(const GemmTerm<T>* __restrict__ terms,
                                                                           const GemmOut* __restrict__ outs, int nout,
                                                                           int groups) {
  constexpr int NW = ThinShape<RS>::NW;
  __shared__ double red[NW * ThinShape<RS>::ELEMS];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= nout * 8 * groups) return;
  const GemmOut o = outs[logical / (8 * groups)];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c0 = logical % 8 * 16;
  const int r0 = logical / 8 % groups * 16 * RS;
  if (c0 >= o.cols || r0 >= o.rows) return;
  dv4 acc[RS][1];
  zero_acc<double>(acc);
  for (int t = o.t0; t < o.t1; ++t) {
    if (t == o.tneg && t > o.t0) {
#pragma unroll
      for (int r = 0; r < RS; ++r) acc[r][0] = -acc[r][0];
    }
    const GemmTerm<T> tm = terms[t];
    int k0, k1;
    thin_share<1, NW>(tm.k0, tm.k1, w, &k0, &k1);
    wave_gemm<T, double>(acc, tm.a, tm.lda, tm.anr, tm.b, tm.ldb, tm.bnr, k0, k1, r0, c0, lane);
  }
  if (o.tneg == o.t1 && o.t1 > o.t0) {  // only subtracted terms
#pragma unroll
    for (int r = 0; r < RS; ++r) acc[r][0] = -acc[r][0];
  }
  thin_put<RS>(acc, red, w, lane);
  const int n = (o.rows - r0 < 16 * RS ? o.rows - r0 : 16 * RS) * 16;
  for (int e = tid; e < n; e += ThinShape<RS>::THREADS) {
    const int row = r0 + (e >> 4), col = c0 + (e & 15);
    if (col >= o.cols) continue;
    double* q = o.out + (int64_t)row * o.ld + col;
    double r = o.alpha * thin_sum<RS>(red, e);
    if (o.c) r += o.beta * o.c[(int64_t)row * o.ldc + col];
    *q = o.accumulate ? *q + r : r;
  }
}

template <typename T, int RS>
__global__ __launch_bounds__(ThinShape<RS>::THREADS) void k_band_thin(BandArgs<T> a) {
  constexpr int NW = ThinShape<RS>::NW;
  __shared__ double red[NW * ThinShape<RS>::ELEMS];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * 8) return;
  const BandItem it = a.items[logical / 8];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c0 = logical % 8 * 16;
  if (c0 >= it.nc) return;
  dv4 acc[RS][1];
  zero_acc<double>(acc);
  int k0, k1;
  thin_share<1, NW>(0, a.vlen, w, &k0, &k1);
  wave_gemm<double, double>(acc, a.Vr + it.p0 * a.vld, a.vld, it.nr, a.Vt + it.q0 * a.vld, a.vld, it.nc, k0, k1, 0, c0,
                            lane);
  thin_put<RS>(acc, red, w, lane);
  for (int e = tid; e < it.nr * 16; e += ThinShape<RS>::THREADS) {
    const int row = e >> 4, col = c0 + (e & 15);
    if (col >= it.nc) continue;
    const double* x = a.Xr + (it.p0 + row) * a.d;
    const double* y = a.Xs + (it.q0 + col) * a.d;
    double sq = 0.0;
    for (int t = 0; t < a.d; ++t) {
      const double df = x[t] - y[t];
      sq += df * df;
    }
    double kv = a.sf2 * k_exp(-0.5 * sq);
    if (a.noise && it.p0 + row == it.q0 + col) kv += a.sn2;
    const int64_t at = a.brow ? a.brow[it.p0 + row] + it.q0 : it.off + (int64_t)row * it.ld;
    a.band[at + col] = (T)(kv - thin_sum<RS>(red, e));
  }
}

// ---------------------------------------------------------------------------
// trsm: L_ij = C_ij L_jj^-T (in place) for every item (p, i), i != j
// ---------------------------------------------------------------------------
// The inverse is lower triangular: column block c (16 wide) of a row takes the first c + 1
// of its 8 blocks.  Rows are never split between waves, so a tile is replaced in place.
//
// k_trsm: a wave holds its 16 RW rows in registers (all of its loads in flight at once) and
// reads the inverse's 36 lower blocks from LDS, where they are staged once per workgroup
// (units of 16 bytes, placed so that a fragment's 16 rows touch every bank once); two
// workgroups on a CU.  Bound: reading and writing the tile (3000 tiles: 800 MB, 160 us at
// the rate of a copy).  With operands from memory and one wave per SIMD it took 259 us a
// launch at n=262144, 212 this way; n=65536 all launches 3.72 -> 3.08 ms, mixed n=50021
// 3.08 -> 2.66.  Sums in the same order as before, bit for bit.
//
// k_trsm_few: 16 rows per workgroup (strips of a tile that may hold rows), a wave per column block, operands from memory: the
// shortest chain where the chip is not filled.
template <typename T>
struct TrsmLds {
  static constexpr int PER = 16 / sizeof(T), UNITS = 16 / PER;  // elements per unit, units per block row
  static constexpr size_t BYTES = 36 * 256 * sizeof(T);
  // unit u of row r of a block
  __device__ static inline int at(int r, int u) {
    return r * UNITS + (u ^ (sizeof(T) == 8 ? (r >> 1) & 7 : (r >> 2) & 3));
  }
};

template <typename T, int RW>
__global__ __launch_bounds__(NT, 2) void k_trsm(StepArgs<T> a) {
  typedef TrsmLds<T> L;
  typedef T unit __attribute__((ext_vector_type(16 / sizeof(T))));
  typedef typename V4<T>::type vin;
  constexpr int RG = 64 * RW, NP = TB / RG;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  unit* inv = reinterpret_cast<unit*>(smem_raw);
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * NP) return;
  const WorkItem it = a.items[logical / NP];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  if (logical % NP * RG >= ri.nvalid) return;  // rows from nvalid on are zero and stay so
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r16 = lane & 15, q = lane >> 4;
  const int r0 = logical % NP * RG + w * 16 * RW;
  T* C = ri.panel + (int64_t)(a.j - ri.kbeg) * TB;
  const T* Li = a.invdiag + pd.invdiag_off + (int64_t)a.j * TB * TB;
  vin sa[RW][8];
#pragma unroll
  for (int rs = 0; rs < RW; ++rs) {
    const int row = r0 + rs * 16 + r16;
    const T* p = C + (int64_t)(row < ri.nstore ? row : 0) * ri.ld + 4 * q;
#pragma unroll
    for (int k = 0; k < 8; ++k) sa[rs][k] = *reinterpret_cast<const vin*>(p + 16 * k);
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int nu = (c + 1) * L::UNITS;
    for (int i = tid; i < 16 * nu; i += NT) {
      const int r = i / nu, u = i - r * nu;
      inv[(c * (c + 1) / 2 + u / L::UNITS) * 16 * L::UNITS + L::at(r, u % L::UNITS)] =
          *reinterpret_cast<const unit*>(Li + (c * 16 + r) * TB + u * L::PER);
    }
  }
  __syncthreads();
  if (r0 >= ri.nvalid) return;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    typename Mfma<T>::acc acc[RW][1];
    zero_acc<T>(acc);
#pragma unroll
    for (int k = 0; k <= c; ++k) {
      const unit* blk = inv + (c * (c + 1) / 2 + k) * 16 * L::UNITS;
      vin b;
      if constexpr (sizeof(T) == 8) {
        const unit b0 = blk[L::at(r16, 2 * q)], b1 = blk[L::at(r16, 2 * q + 1)];
        b = vin{b0[0], b0[1], b1[0], b1[1]};
      } else {
        b = blk[L::at(r16, q)];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int rs = 0; rs < RW; ++rs) acc[rs][0] = Mfma<T>::op(sa[rs][k][e], b[e], acc[rs][0]);
    }
#pragma unroll
    for (int rs = 0; rs < RW; ++rs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = r0 + rs * 16 + Mfma<T>::row(lane, v);
        if (row < ri.nstore) C[(int64_t)row * ri.ld + c * 16 + r16] = acc[rs][0][v];
      }
  }
}

template <typename T>
__global__ __launch_bounds__(2 * NT) void k_trsm_few(StepArgs<T> a, int strips) {
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * strips) return;
  const WorkItem it = a.items[logical / strips];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  if (logical % strips * 16 >= ri.nvalid) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // w / 8 is 0: written so, the row stays in a vector register and a launch takes 7.6 us
  // instead of 9.0 (111 registers for 122)
  const int r0 = logical % strips * 16 + w / 8 * 16, c0 = w % 8 * 16;
  T* C = ri.panel + (int64_t)(a.j - ri.kbeg) * TB;
  const T* Li = a.invdiag + pd.invdiag_off + (int64_t)a.j * TB * TB;
  typename Mfma<T>::acc acc[1][1];
  zero_acc<T>(acc);
  wave_gemm<T, T>(acc, C, ri.ld, ri.nstore, Li, TB, TB, 0, c0 + 16, r0, c0, lane);
  __syncthreads();  // every wave has consumed its reads of C before anyone overwrites it
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = r0 + Mfma<T>::row(lane, v);
    if (row < ri.nstore) C[(int64_t)row * ri.ld + c0 + (lane & 15)] = acc[0][0][v];
  }
}

// ---------------------------------------------------------------------------
// batched float64-accumulating tile GEMM
// ---------------------------------------------------------------------------
template <typename T, int SUB>
__global__ __launch_bounds__(NT, SUB == 4 ? 2 : 1) void k_tile_gemm(const GemmTerm<T>* __restrict__ terms,
                                                  const GemmOut* __restrict__ outs, int nout) {
  constexpr int WS = 16 * SUB, QS = 2 * WS, NQ = TB / QS;  // as in k_update
  extern __shared__ __align__(16) double sm[];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= nout * NQ * NQ) return;
  const GemmOut o = outs[logical / (NQ * NQ)];
  const int q0r = (logical / NQ) % NQ * QS, q0c = logical % NQ * QS;
  if (q0r >= o.rows || q0c >= o.cols) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = q0r + (w >> 1) * WS, c0 = q0c + (w & 1) * WS;
  typename Mfma<double>::acc acc[SUB][SUB];
  zero_acc<double>(acc);
  for (int t = o.t0; t < o.t1; ++t) {
    if (t == o.tneg && t > o.t0) {
#pragma unroll
      for (int a = 0; a < SUB; ++a)
#pragma unroll
        for (int b = 0; b < SUB; ++b) acc[a][b] = -acc[a][b];
    }
    const GemmTerm<T> tm = terms[t];
    if constexpr (SUB == 4)
      wg_gemm<T>(acc, tm.a, tm.lda, tm.anr, tm.b, tm.ldb, tm.bnr, tm.k0, tm.k1, sm);
    else
      wave_gemm<T, double>(acc, tm.a, tm.lda, tm.anr, tm.b, tm.ldb, tm.bnr, tm.k0, tm.k1, r0, c0, lane);
  }
  if (o.tneg == o.t1 && o.t1 > o.t0) {  // only subtracted terms
#pragma unroll
    for (int a = 0; a < SUB; ++a)
#pragma unroll
      for (int b = 0; b < SUB; ++b) acc[a][b] = -acc[a][b];
  }
#pragma unroll
  for (int rs = 0; rs < SUB; ++rs)
#pragma unroll
    for (int cs = 0; cs < SUB; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = r0 + rs * 16 + Mfma<double>::row(lane, v);
        const int col = c0 + cs * 16 + (lane & 15);
        if (row < o.rows && col < o.cols) {
          double* q = o.out + (int64_t)row * o.ld + col;
          double r = o.alpha * acc[rs][cs][v];
          if (o.c) r += o.beta * o.c[(int64_t)row * o.ldc + col];
          *q = o.accumulate ? *q + r : r;
        }
      }
}

// ---------------------------------------------------------------------------
// band: R_pq = K_pq + [p == q] sn2 - V_p . V_q on one 128 x 128 tile of the
// residual band (float64 arithmetic, one rounding to T on the store)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(NT, 2) void k_band(BandArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems) return;
  const BandItem it = a.items[logical];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wr = w >> 1, wc = w & 1;
  typename Mfma<double>::acc acc[4][4];
  zero_acc<double>(acc);
  wg_gemm<double>(acc, a.Vr + it.p0 * a.vld, a.vld, it.nr, a.Vt + it.q0 * a.vld, a.vld, it.nc, 0, a.vlen,
                  reinterpret_cast<double*>(smem_raw));
  __syncthreads();  // the operand stages lie where the coordinates go
  // coordinates of the tile's row and column points
  const int d = a.d;
  double* xr = reinterpret_cast<double*>(smem_raw);  // [d][TB]
  double* xc = xr + d * TB;
  for (int idx = tid; idx < TB * d; idx += NT) {
    const int r = idx / d, t = idx - r * d;
    xr[t * TB + r] = r < it.nr ? a.Xr[(it.p0 + r) * d + t] : 0.0;
    xc[t * TB + r] = r < it.nc ? a.Xs[(it.q0 + r) * d + t] : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int rs = 0; rs < 4; ++rs) {
    // squared distances of a 16-row strip, one coordinate at a time
    double sq[4][4];
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) sq[cs][v] = 0.0;
    for (int t = 0; t < d; ++t) {
      double cv[4];
#pragma unroll
      for (int cs = 0; cs < 4; ++cs) cv[cs] = xc[t * TB + wc * 64 + cs * 16 + (lane & 15)];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double rv = xr[t * TB + wr * 64 + rs * 16 + Mfma<double>::row(lane, v)];
#pragma unroll
        for (int cs = 0; cs < 4; ++cs) {
          const double df = rv - cv[cs];
          sq[cs][v] += df * df;
        }
      }
    }
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * 64 + rs * 16 + Mfma<double>::row(lane, v);
        const int col = wc * 64 + cs * 16 + (lane & 15);
        if (row < it.nr && col < it.nc) {
          double kv = a.sf2 * k_exp(-0.5 * sq[cs][v]);
          if (a.noise && it.p0 + row == it.q0 + col) kv += a.sn2;
          const int64_t at = a.brow ? a.brow[it.p0 + row] + it.q0 : it.off + (int64_t)row * it.ld;
          a.band[at + col] = (T)(kv - acc[rs][cs][v]);
        }
      }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
constexpr int NCU = 256;  // compute units
static inline int pad8(int n) { return ((n + 7) / 8) * 8; }

// Calls f(first, count) for pieces of n items that fit a launch (fewer than 2^32 threads; of
// a larger one only the remainder runs, without an error) with `threads` per item.  The
// forms that give a tile eight workgroups of 512 reach that with 1048576 tiles, which half a
// million windows of one or two points have.
template <class F>
static void in_launches(int64_t n, int64_t threads, F&& f) {
  const int64_t most = 0xffffffffll / threads & ~7ll;  // whole launches of a multiple of 8 workgroups
  for (int64_t i = 0; i < n; i += most) f(i, std::min(most, n - i));
}

// Pieces per tile side (1, 2 or 4) of a launch of n whole tiles with products of
// length k.  A whole tile gives its products the most reuse; pieces fill CUs that whole
// tiles leave idle, and overlap the covariance and the stores where products are short.
// Measured, us for 1 / 4 / 16 pieces a tile (d = 1):
//   float64, k = 3072: n = 8 384 / 176 / 90, 24 387 / 180 / 177, 64 388 / 186 / 342, 128 398 /
//   354 / 667, 136 397 / 517 / 751, 512 810 / 1368 / 2663 (two whole tiles share a CU)
//   mixed, k = 3072: n = 8 218 / 92 / 47, 64 220 / 99 / 179, 128 221 / 184 / 339, 136 222 / 265 / 380
//   k = 0: float64 n = 256 29 / 21 / 19, 1032 71 / 66 / 56; mixed 1032 93 / 58 / 56
//   k = 128: float64 n = 136 44 / 41 / 43, 1032 151 / 188 / 260; mixed 1032 144 / 115 / 140
//   k = 256: float64 n = 128 59 / 43 / 65, 1032 224 / 299 / 459; mixed 1032 194 / 171 / 234
//   k = 384: mixed n = 136 51 / 49 / 56, 512 99 / 113 / 176
// The line at k = 256 is right for mixed precision; in float64 it was drawn when a whole tile
// held a CU alone (n = 1032, k = 256: 324 / 310), and beyond n = 136 lies at 0 now.
static inline int split_of(int64_t n, int64_t k) {
  if (n <= 16 || (k == 0 && n <= NCU)) return 4;
  return n <= NCU / 2 || k <= 256 ? 2 : 1;
}

template <typename T, bool MIXED>
static void update_pieces(const StepArgs<T>& all, int64_t first, int64_t count, int split, hipStream_t st) {
  size_t lds = 2 * (size_t)all.d * (TB / split) * (MIXED ? sizeof(double) : sizeof(T));
  if (std::is_same<T, double>::value && split == 1) lds = std::max(lds, WG_GEMM_LDS);
  in_launches(count, split * split * NT, [&](int64_t i0, int64_t n) {
    StepArgs<T> a = all;
    a.items += first + i0;
    a.nitems = (int32_t)n;
    const dim3 grid(pad8(a.nitems * split * split));
    switch (split) {
      case 1: hipLaunchKernelGGL((k_update<T, MIXED, 4>), grid, dim3(NT), lds, st, a); break;
      case 2: hipLaunchKernelGGL((k_update<T, MIXED, 2>), grid, dim3(NT), lds, st, a); break;
      default: hipLaunchKernelGGL((k_update<T, MIXED, 1>), grid, dim3(NT), lds, st, a);
    }
  });
}

// A launch of n tiles with products of length k as `whole` tiles in full turns of the
// CUs, then the rest with its products in `parts` parts along k (1: whole).
struct UpdatePlan {
  int64_t whole;
  int parts;
  double us;
};

// Estimated times in us.  A turn of whole tiles is taken as 1.75 us per 16 k in float64
// (256 tiles alone take 2.1) and 1.05 in mixed precision (float32 products and their folds;
// 1.0 for half a turn, 1.3 for a full one); the parts are written and read once (128 KB
// each, 3.5 TB/s) and need a launch more.
// Measured over all launches (products of k_update, its parts and their sums): full GP
// n=16384 261 -> 201 ms, n=262144 728 -> 688, n=65536 22.4 -> 21.7, mixed n=50021 36.5 -> 31.3.
template <bool MIXED>
static UpdatePlan plan_update(int64_t n, int64_t k, int cap) {
  const double turn = (MIXED ? 1.05 : 1.75) * (double)(k / 16);
  UpdatePlan best{n, 1, turn * (double)((n + NCU - 1) / NCU)};
  for (int64_t whole = n / NCU * NCU; whole >= 0 && whole + 2 * NCU > n; whole -= NCU) {
    const int64_t rest = n - whole;
    for (int s = 2; s <= 32 && rest * s <= cap; ++s) {
      const double us = turn * (double)(whole / NCU) + turn * (double)((rest * s + NCU - 1) / NCU) / s +
                        2.0 * 131072.0 * (double)(rest * s) / 3.5e6 + (whole ? 12.0 : 8.0);
      if (us < best.us) best = UpdatePlan{whole, s, us};
    }
  }
  return best;
}

// Time of a launch of n tiles without thin ones, in us, on the same terms; the launch
// itself and the epilogue are left out.
template <bool MIXED>
static double update_us(int64_t n, int64_t k, bool can_part) {
  if (n <= 0) return 0.0;
  const int split = split_of(n, k);
  const double turn = (MIXED ? 1.05 : 1.75) * (double)(k / 16);
  const double pieces = split == 4 ? 0.245 * turn * (double)((16 * n + NCU - 1) / NCU)
                                   : split == 2 ? 0.48 * turn * (double)((4 * n + NCU - 1) / NCU) : 1e30;
  const double whole = can_part ? plan_update<MIXED>(n, k, PART_TILES).us : turn * (double)((n + NCU - 1) / NCU);
  return std::min(pieces, whole);
}

// A few whole tiles in the form of thin ones, in rs row groups of 16 per workgroup: as many
// workgroups as fit the CUs once.  Measured us per 128 k (float64; mixed precision 0.56 of
// it): n <= 4 0.72, 8 1.05, 16 2.05, 32 4.2; beyond 32 the pieces of split_of are faster
// (n = 48, k = 640 31 and 28 us).
static inline int slim_rs(int64_t n) { return n <= 4 ? 1 : n <= 8 ? 2 : 4; }
template <bool MIXED>
static double slim_us(int64_t n, int64_t k) {
  return (MIXED ? 0.56 : 1.0) * (n <= 4 ? 0.72 : n <= 8 ? 1.05 : n <= 16 ? 2.05 : 4.2) * (double)k / 128.0;
}

// row groups of 16 (1, 2 or 4) that hold `rows` rows
static inline int thin_rs(int rows) { return rows <= 16 ? 1 : rows <= 32 ? 2 : 4; }

// Time of n thin tiles with products of length k: the other operand from memory, or the
// products (256 cycles per row group and 16 k on each SIMD), and the launch.
template <typename T>
static double thin_us(int64_t n, int64_t k, int rs) {
  const double bytes = (double)n * TB * (double)k * sizeof(T) / 4.0e6;
  const double prod = (double)(n * 8) * (double)(k / 16) * 256.0 * rs / (1024.0 * 2400.0);
  return 6.0 + std::max(bytes, prod);
}

template <typename T, bool MIXED>
static void slim_launch(const StepArgs<T>& all, int rs, int groups, hipStream_t st) {
  in_launches(all.nitems, 8 * groups * ThinShape<1>::THREADS, [&](int64_t i0, int64_t n) {
    StepArgs<T> a = all;
    a.items += i0;
    a.nitems = (int32_t)n;
    const dim3 grid(pad8(8 * groups * a.nitems)), nt(ThinShape<1>::THREADS);
    switch (rs) {
      case 1: hipLaunchKernelGGL((k_update_slim<T, MIXED, 1>), grid, nt, 0, st, a, groups); break;
      case 2: hipLaunchKernelGGL((k_update_slim<T, MIXED, 2>), grid, nt, 0, st, a, groups); break;
      default: hipLaunchKernelGGL((k_update_slim<T, MIXED, 4>), grid, nt, 0, st, a, groups);
    }
  });
}

template <typename T, bool MIXED>
static void update_launches(const StepArgs<T>& a, hipStream_t st) {
  const int64_t n = a.nitems;
  const bool vpart = a.vlen > 0 && a.band == nullptr;  // some tiles have a V part before the factor's
  const int64_t k = (int64_t)a.j * TB + (vpart ? a.vlen : 0);
  if constexpr (MIXED || std::is_same<T, double>::value) {
    if (a.thin.n > 0) {
      // Thin tiles in a launch of their own where that is estimated to take less than
      // they add as whole tiles; always where the launch has no others.
      const int64_t full = n - a.thin.n;
      const int rs = thin_rs(a.thin.rows);
      const bool part = a.part != nullptr && !vpart && k > 256;
      StepArgs<T> b = a;
      b.thin = Thin{0, 0};
      if (full == 0 || update_us<MIXED>(n, k, part) - update_us<MIXED>(full, k, part) > thin_us<T>(a.thin.n, k, rs)) {
        b.nitems = (int32_t)full;
        if (full > 0) update_launches<T, MIXED>(b, st);
        b.items += full;
        b.nitems = a.thin.n;
        slim_launch<T, MIXED>(b, rs, 1, st);
      } else {
        update_launches<T, MIXED>(b, st);
      }
      return;
    }
  }
  const int split = split_of(n, k);
  if constexpr (MIXED || std::is_same<T, double>::value) {
    if (a.any_order && n <= 32 && slim_us<MIXED>(n, k) <= update_us<MIXED>(n, k, a.part != nullptr && !vpart && k > 256)) {
      const int rs = slim_rs(n);
      slim_launch<T, MIXED>(a, rs, 8 / rs, st);
      return;
    }
    if (a.part != nullptr && !vpart && k > 256) {
      const UpdatePlan p = plan_update<MIXED>(n, k, PART_TILES);
      // what the pieces of split_of would take
      const double turn = (MIXED ? 1.05 : 1.75) * (double)(k / 16);
      const double pieces = split == 4 ? 0.245 * turn : split == 2 ? 0.48 * turn * (double)((4 * n + NCU - 1) / NCU) : 1e30;
      if (p.parts > 1 && p.us < pieces) {
        StepArgs<T> b = a;
        update_pieces<T, MIXED>(a, 0, p.whole, 1, st);
        b.items += p.whole;
        b.nitems = (int32_t)(n - p.whole);
        b.nsplit = p.parts;
        hipLaunchKernelGGL((k_update_part<T, MIXED>), dim3(pad8(b.nitems * p.parts)), dim3(NT),
                           MIXED ? 0 : WG_GEMM_LDS, st, b);
        const size_t lds = 2 * (size_t)a.d * (TB / 2) * (MIXED ? sizeof(double) : sizeof(T));
        if (b.nitems <= 32)
          hipLaunchKernelGGL((k_update<T, MIXED, 1, true>), dim3(pad8(b.nitems * 16)), dim3(NT), lds / 2, st, b);
        else
          hipLaunchKernelGGL((k_update<T, MIXED, 2, true>), dim3(pad8(b.nitems * 4)), dim3(NT), lds, st, b);
        return;
      }
    }
  }
  // up to 64 tiles left over from full turns: a launch of their own, in pieces that fit
  // in half a turn
  const int64_t rest = split == 1 && n % NCU <= NCU / 4 ? n % NCU : 0;
  update_pieces<T, MIXED>(a, 0, n - rest, split, st);
  update_pieces<T, MIXED>(a, n - rest, rest, split_of(rest, k), st);
}

template <typename T>
void launch_update(const StepArgs<T>& a, bool mixed, hipStream_t st) {
  if (a.nitems <= 0) return;
  if constexpr (std::is_same<T, float>::value)
    if (mixed) {
      update_launches<T, true>(a, st);
      return;
    }
  update_launches<T, false>(a, st);
}

template <typename T>
void launch_trsm(const StepArgs<T>& a, hipStream_t st) {
  if (a.nitems <= 0) return;
  // Few rows: two workgroups per CU (n = 62 tiles of up to 14 rows 9 us, 14 with k_trsm; n =
  // 17 to 19 tiles 7.6 and 18).  Half tiles fill the CUs up to 256 tiles in float64 (all launches of a
  // full GP of n=16384 8.7 ms, 9.0 with a limit of 64, 9.4 without one); in float32, where
  // the stage is half as large, always (mixed n=50021 2.66 ms, 2.73 with a limit of 512).
  const int strips = a.thin.n == a.nitems ? (a.thin.rows + 15) / 16 : 8;  // all of them thin tiles
  if (a.nitems * strips <= 2 * NCU)
    hipLaunchKernelGGL((k_trsm_few<T>), dim3(pad8(strips * a.nitems)), dim3(2 * NT), 0, st, a, strips);
  else if (a.nitems <= NCU || std::is_same<T, float>::value)
    in_launches(a.nitems, 2 * NT, [&](int64_t i0, int64_t n) {
      StepArgs<T> b = a;
      b.items += i0;
      b.nitems = (int32_t)n;
      hipLaunchKernelGGL((k_trsm<T, 1>), dim3(pad8(2 * b.nitems)), dim3(NT), TrsmLds<T>::BYTES, st, b);
    });
  else if constexpr (std::is_same<T, double>::value)
    hipLaunchKernelGGL((k_trsm<T, 2>), dim3(pad8(a.nitems)), dim3(NT), TrsmLds<T>::BYTES, st, a);
}

template <typename T>
void launch_band(const BandArgs<T>& a, hipStream_t st) {
  if (a.nitems <= 0) return;
  const size_t lds = std::max(WG_GEMM_LDS, 2 * (size_t)a.d * TB * sizeof(double));
  BandArgs<T> b = a;
  b.nitems -= a.thin.n;
  if (b.nitems > 0) hipLaunchKernelGGL(k_band<T>, dim3(pad8(b.nitems)), dim3(NT), lds, st, b);
  if (a.thin.n <= 0) return;
  const BandItem* few = a.items + b.nitems;
  in_launches(a.thin.n, 8 * ThinShape<1>::THREADS, [&](int64_t i0, int64_t n) {
    b.items = few + i0;
    b.nitems = (int32_t)n;
    const dim3 grid(pad8(8 * b.nitems)), nt(ThinShape<1>::THREADS);
    switch (thin_rs(a.thin.rows)) {
      case 1: hipLaunchKernelGGL((k_band_thin<T, 1>), grid, nt, 0, st, b); break;
      case 2: hipLaunchKernelGGL((k_band_thin<T, 2>), grid, nt, 0, st, b); break;
      default: hipLaunchKernelGGL((k_band_thin<T, 4>), grid, nt, 0, st, b);
    }
  });
}

template <typename T>
static void tile_gemm_slim(const GemmTerm<T>* terms, const GemmOut* all, int nall, int rs, int groups, hipStream_t st) {
  in_launches(nall, 8 * groups * ThinShape<1>::THREADS, [&](int64_t i0, int64_t m) {
    const GemmOut* outs = all + i0;
    const int n = (int)m;
    const dim3 grid(pad8(8 * groups * n)), nt(ThinShape<1>::THREADS);
    switch (rs) {
      case 1: hipLaunchKernelGGL((k_tile_gemm_slim<T, 1>), grid, nt, 0, st, terms, outs, n, groups); break;
      case 2: hipLaunchKernelGGL((k_tile_gemm_slim<T, 2>), grid, nt, 0, st, terms, outs, n, groups); break;
      default: hipLaunchKernelGGL((k_tile_gemm_slim<T, 4>), grid, nt, 0, st, terms, outs, n, groups);
    }
  });
}

template <typename T>
void launch_tile_gemm(const GemmTerm<T>* terms, const GemmOut* outs, int nout, Thin thin, bool any_order,
                      hipStream_t st) {
  // thin outputs apart, unless the whole launch is small
  if (thin.n > 0 && (thin.n == nout || nout > 64)) {
    nout -= thin.n;
    tile_gemm_slim(terms, outs + nout, thin.n, thin_rs(thin.rows), 1, st);
  }
  if (nout <= 0) return;
  // measured, whole tiles / 4 pieces: float64 n = 48 204 / 75 us, n = 112 178 / 128, n = 176
  // 80 / 94; float32 operands leave the registers for three workgroups of pieces on a CU:
  // n = 240 863 / 755, n = 14240 8071 / 6637.  Up to 16 the waves share k.
  if (nout <= 16 && any_order)
    tile_gemm_slim(terms, outs, nout, slim_rs(nout), 8 / slim_rs(nout), st);
  else if (nout <= 16)  // 16 pieces: n = 14 31 us, 4 pieces 47
    hipLaunchKernelGGL((k_tile_gemm<T, 1>), dim3(pad8(16 * nout)), dim3(NT), 0, st, terms, outs, nout);
  else if (nout <= NCU / 2 || std::is_same<T, float>::value)
    in_launches(nout, 4 * NT, [&](int64_t i0, int64_t n) {
      hipLaunchKernelGGL((k_tile_gemm<T, 2>), dim3(pad8(4 * (int)n)), dim3(NT), 0, st, terms, outs + i0, (int)n);
    });
  else if constexpr (std::is_same<T, double>::value)
    hipLaunchKernelGGL((k_tile_gemm<T, 4>), dim3(pad8(nout)), dim3(NT), WG_GEMM_LDS, st, terms, outs, nout);
}

// Raise the dynamic-LDS limit of the kernels that need more than the default.
hipError_t engine_init() {
  hipError_t e = diag_init();
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_update<double, false, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(double)));
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_update<float, true, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(double)));
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_update<float, false, 4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(float)));
  if (e != hipSuccess) return e;
  for (const void* f : {(const void*)k_tile_gemm<double, 4>, (const void*)k_update_part<double, false>}) {
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)WG_GEMM_LDS);
    if (e != hipSuccess) return e;
  }
  for (const void* f : {(const void*)k_trsm<double, 1>, (const void*)k_trsm<double, 2>}) {
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)TrsmLds<double>::BYTES);
    if (e != hipSuccess) return e;
  }
  e = hipFuncSetAttribute((const void*)k_band<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(double)));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_band<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)(2 * 64 * TB * sizeof(double)));
}

template void launch_update<double>(const StepArgs<double>&, bool, hipStream_t);
template void launch_update<float>(const StepArgs<float>&, bool, hipStream_t);
template void launch_trsm<double>(const StepArgs<double>&, hipStream_t);
template void launch_trsm<float>(const StepArgs<float>&, hipStream_t);
template void launch_band<double>(const BandArgs<double>&, hipStream_t);
template void launch_band<float>(const BandArgs<float>&, hipStream_t);
template void launch_tile_gemm<double>(const GemmTerm<double>*, const GemmOut*, int, Thin, bool, hipStream_t);
template void launch_tile_gemm<float>(const GemmTerm<float>*, const GemmOut*, int, Thin, bool, hipStream_t);

}  // namespace lma
