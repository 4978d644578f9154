// Device kernels of the tiled Cholesky / triangular-solve engine (gfx950).
// The MFMA tile core (operand layout, prefetch pipeline) is in mfma_core.h.
#include "engine.h"
#include "mfma_core.h"

#include <type_traits>

namespace lma {

// ---------------------------------------------------------------------------
// update: C_ij = K_ij - V_i V_j^T - sum_{k<j} L_ik L_jk^T for every item (p, i)
// ---------------------------------------------------------------------------
template <typename T, bool MIXED>
__global__ __launch_bounds__(NT) void k_update(StepArgs<T> a) {
  // covariance tile and V-part precision: float64 when T is double or MIXED
  typedef typename std::conditional<MIXED, double, T>::type TK;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems) return;
  const WorkItem it = a.items[logical];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  const RowTile<T> rj = a.rt[pd.first + a.j];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wr = w >> 1, wc = w & 1;

  typename Mfma<TK>::acc accv[4][4];   // V_i V_j^T
  typename Mfma<T>::acc accl[4][4];    // sum_k L_ik L_jk^T (aliases accv when not MIXED)
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
    int64_t rowp[4][4], rowb[4][4], colq[4], colb[4];
#pragma unroll
    for (int cs = 0; cs < 4; ++cs) {
      const int col = wc * 64 + cs * 16 + (lane & 15);
      colq[cs] = rj.pt0 + (col < nvc ? col : nvc - 1);
      colb[cs] = tband ? 0 : a.brow[colq[cs]];
    }
#pragma unroll
    for (int rs = 0; rs < 4; ++rs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * 64 + rs * 16 + Mfma<TK>::row(lane, v);
        rowp[rs][v] = ri.pt0 + (row < nvr ? row : nvr - 1);
        rowb[rs][v] = a.brow[rowp[rs][v]];
      }
#pragma unroll
    for (int rs = 0; rs < 4; ++rs)
#pragma unroll
      for (int cs = 0; cs < 4; ++cs) {
        typename Mfma<TK>::acc r0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = wr * 64 + rs * 16 + Mfma<TK>::row(lane, v);
          const int col = wc * 64 + cs * 16 + (lane & 15);
          const int64_t p = rowp[rs][v], q = colq[cs];
          const int64_t e = (tband || q <= p) ? rowb[rs][v] + q : colb[cs] + p;
          const TK kv = (TK)a.band[e];
          r0[v] = (row < nvr && col < nvc) ? -kv : TK(0);
        }
        accv[rs][cs] = Mfma<TK>::op(TK(0), TK(0), r0);
      }
  } else {
    zero_acc<TK>(accv);
  }
  if constexpr (MIXED) zero_acc<T>(accl);
  const TK* vi = MIXED ? (const TK*)ri.vt64 : (const TK*)ri.vt;
  const TK* vj = MIXED ? (const TK*)rj.vt64 : (const TK*)rj.vt;
  if (!band && !tband && vi != nullptr && vj != nullptr && a.vlen > 0)
    wave_gemm<TK, TK>(accv, vi, a.vld, ri.nvalid, vj, a.vld, rj.nvalid, 0, a.vlen, wr * 64, wc * 64, lane);
  // factor columns kb .. j-1 (a row is zero left of its kbeg)
  const int kb = ri.kbeg > rj.kbeg ? ri.kbeg : rj.kbeg;
  if (a.j > kb) {
    const T* pa = ri.panel + (int64_t)(kb - ri.kbeg) * TB;
    const T* pb = rj.panel + (int64_t)(kb - rj.kbeg) * TB;
    if constexpr (MIXED)  // float32 products, sums folded into the float64 accumulators
      wave_gemm_fold(accl, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, 0, (a.j - kb) * TB, wr * 64, wc * 64, lane,
                     accv);
    else
      wave_gemm<T, T>(accv, pa, ri.ld, ri.nstore, pb, rj.ld, rj.nstore, 0, (a.j - kb) * TB, wr * 64, wc * 64, lane);
  }

  const int d = a.d;
  TK* xr = reinterpret_cast<TK*>(smem_raw);  // [d][TB] row-side coordinates
  TK* xc = xr + d * TB;                      // [d][TB] column-side coordinates
  const bool kern = ri.src == SRC_KERNEL;
  if (kern) {
    const TK* xsi = MIXED ? (const TK*)ri.xs64 : (const TK*)ri.xs;
    const TK* xsj = MIXED ? (const TK*)rj.xs64 : (const TK*)rj.xs;
    for (int idx = tid; idx < TB * d; idx += NT) {
      const int r = idx / d, t = idx - r * d;
      xr[t * TB + r] = r < ri.nvalid ? xsi[(int64_t)r * d + t] : TK(0);
      xc[t * TB + r] = r < rj.nvalid ? xsj[(int64_t)r * d + t] : TK(0);
    }
  }
  __syncthreads();
  const bool diag = ri.is_j && (it.tile == a.j);
  const TK sf2 = (TK)a.sf2, sn2 = (TK)a.sn2;
  T* out = ri.panel + (int64_t)(a.j - ri.kbeg) * TB;
  const bool ident = ri.src == SRC_IDENT;
  const bool ident_here = ident && ri.kbeg == a.j;
  // squared distances of the lane's 64 entries, one coordinate at a time
  TK sq[4][4][4];
#pragma unroll
  for (int rs = 0; rs < 4; ++rs)
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) sq[rs][cs][v] = TK(0);
  if (kern) {
    for (int t = 0; t < d; ++t) {
      TK cv[4];
#pragma unroll
      for (int cs = 0; cs < 4; ++cs) cv[cs] = xc[t * TB + wc * 64 + cs * 16 + (lane & 15)];
#pragma unroll
      for (int rs = 0; rs < 4; ++rs)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const TK rv = xr[t * TB + wr * 64 + rs * 16 + Mfma<TK>::row(lane, v)];
#pragma unroll
          for (int cs = 0; cs < 4; ++cs) {
            const TK df = rv - cv[cs];
            sq[rs][cs][v] += df * df;
          }
        }
    }
  }
#pragma unroll
  for (int rs = 0; rs < 4; ++rs) {
#pragma unroll
    for (int cs = 0; cs < 4; ++cs) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * 64 + rs * 16 + Mfma<TK>::row(lane, v);
        const int col = wc * 64 + cs * 16 + (lane & 15);
        TK kv = TK(0);
        if (ident) {
          kv = (ident_here && row == col) ? TK(1) : TK(0);  // exact at padding too
        } else if (row < ri.nvalid && col < rj.nvalid) {
          if (kern) {
            kv = sf2 * k_exp(TK(-0.5) * sq[rs][cs][v]);
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

// ---------------------------------------------------------------------------
// trsm: L_ij = C_ij L_jj^-T (in place) for every item (p, i), i != j
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(NT) void k_trsm(StepArgs<T> a) {
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems) return;
  const WorkItem it = a.items[logical];
  const ProbDesc pd = a.pd[it.p];
  const RowTile<T> ri = a.rt[pd.first + it.tile];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wr = w >> 1, wc = w & 1;
  T* C = ri.panel + (int64_t)(a.j - ri.kbeg) * TB;
  const T* Li = a.invdiag + pd.invdiag_off + (int64_t)a.j * TB * TB;
  typename Mfma<T>::acc acc[4][4];
  zero_acc<T>(acc);
  wave_gemm<T, T>(acc, C, ri.ld, ri.nstore, Li, TB, TB, 0, TB, wr * 64, wc * 64, lane);
  __syncthreads();  // every wave has consumed its reads of C before anyone overwrites it
#pragma unroll
  for (int rs = 0; rs < 4; ++rs)
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * 64 + rs * 16 + Mfma<T>::row(lane, v);
        const int col = wc * 64 + cs * 16 + (lane & 15);
        if (row < ri.nstore) C[(int64_t)row * ri.ld + col] = acc[rs][cs][v];
      }
}

// ---------------------------------------------------------------------------
// batched float64-accumulating tile GEMM
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(NT) void k_tile_gemm(const GemmTerm<T>* __restrict__ terms,
                                                  const GemmOut* __restrict__ outs, int nout) {
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= nout) return;
  const GemmOut o = outs[logical];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wr = w >> 1, wc = w & 1;
  typename Mfma<double>::acc acc[4][4];
  zero_acc<double>(acc);
  for (int t = o.t0; t < o.t1; ++t) {
    if (t == o.tneg && t > o.t0) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = -acc[a][b];
    }
    const GemmTerm<T> tm = terms[t];
    wave_gemm<T, double>(acc, tm.a, tm.lda, tm.anr, tm.b, tm.ldb, tm.bnr, tm.k0, tm.k1, wr * 64, wc * 64,
                         lane);
  }
  if (o.tneg == o.t1 && o.t1 > o.t0) {  // only subtracted terms
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = -acc[a][b];
  }
#pragma unroll
  for (int rs = 0; rs < 4; ++rs)
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * 64 + rs * 16 + Mfma<double>::row(lane, v);
        const int col = wc * 64 + cs * 16 + (lane & 15);
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
__global__ __launch_bounds__(NT) void k_band(BandArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems) return;
  const BandItem it = a.items[logical];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wr = w >> 1, wc = w & 1;
  // coordinates of the tile's row and column points
  const int d = a.d;
  double* xr = reinterpret_cast<double*>(smem_raw);  // [d][TB]
  double* xc = xr + d * TB;
  for (int idx = tid; idx < TB * d; idx += NT) {
    const int r = idx / d, t = idx - r * d;
    xr[t * TB + r] = r < it.nr ? a.Xr[(it.p0 + r) * d + t] : 0.0;
    xc[t * TB + r] = r < it.nc ? a.Xs[(it.q0 + r) * d + t] : 0.0;
  }
  typename Mfma<double>::acc acc[4][4];
  zero_acc<double>(acc);
  wave_gemm<double, double>(acc, a.Vr + it.p0 * a.vld, a.vld, it.nr, a.Vt + it.q0 * a.vld, a.vld, it.nc, 0, a.vlen,
                            wr * 64, wc * 64, lane);
  __syncthreads();
  // squared distances of the lane's 64 entries, one coordinate at a time (its 16
  // row and 4 column values of a coordinate are read from LDS once)
  double sq[4][4][4];
#pragma unroll
  for (int rs = 0; rs < 4; ++rs)
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) sq[rs][cs][v] = 0.0;
  for (int t = 0; t < d; ++t) {
    double cv[4];
#pragma unroll
    for (int cs = 0; cs < 4; ++cs) cv[cs] = xc[t * TB + wc * 64 + cs * 16 + (lane & 15)];
#pragma unroll
    for (int rs = 0; rs < 4; ++rs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double rv = xr[t * TB + wr * 64 + rs * 16 + Mfma<double>::row(lane, v)];
#pragma unroll
        for (int cs = 0; cs < 4; ++cs) {
          const double df = rv - cv[cs];
          sq[rs][cs][v] += df * df;
        }
      }
  }
#pragma unroll
  for (int rs = 0; rs < 4; ++rs)
#pragma unroll
    for (int cs = 0; cs < 4; ++cs)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * 64 + rs * 16 + Mfma<double>::row(lane, v);
        const int col = wc * 64 + cs * 16 + (lane & 15);
        if (row < it.nr && col < it.nc) {
          double kv = a.sf2 * k_exp(-0.5 * sq[rs][cs][v]);
          if (a.noise && it.p0 + row == it.q0 + col) kv += a.sn2;
          a.band[it.off + (int64_t)row * it.ld + col] = (T)(kv - acc[rs][cs][v]);
        }
      }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline int pad8(int n) { return ((n + 7) / 8) * 8; }

template <typename T>
void launch_update(const StepArgs<T>& a, bool mixed, hipStream_t st) {
  if (a.nitems <= 0) return;
  if constexpr (std::is_same<T, float>::value) {
    if (mixed) {
      const size_t lds = 2 * (size_t)a.d * TB * sizeof(double);
      hipLaunchKernelGGL((k_update<T, true>), dim3(pad8(a.nitems)), dim3(NT), lds, st, a);
      return;
    }
  }
  {
    const size_t lds = 2 * (size_t)a.d * TB * sizeof(T);
    hipLaunchKernelGGL((k_update<T, false>), dim3(pad8(a.nitems)), dim3(NT), lds, st, a);
  }
}

template <typename T>
void launch_trsm(const StepArgs<T>& a, hipStream_t st) {
  if (a.nitems <= 0) return;
  hipLaunchKernelGGL(k_trsm<T>, dim3(pad8(a.nitems)), dim3(NT), 0, st, a);
}

template <typename T>
void launch_band(const BandArgs<T>& a, hipStream_t st) {
  if (a.nitems <= 0) return;
  hipLaunchKernelGGL(k_band<T>, dim3(pad8(a.nitems)), dim3(NT), 2 * (size_t)a.d * TB * sizeof(double), st, a);
}

template <typename T>
void launch_tile_gemm(const GemmTerm<T>* terms, const GemmOut* outs, int nout, hipStream_t st) {
  if (nout <= 0) return;
  hipLaunchKernelGGL(k_tile_gemm<T>, dim3(pad8(nout)), dim3(NT), 0, st, terms, outs, nout);
}

// Raise the dynamic-LDS limit of the kernels that need more than the default.
hipError_t engine_init() {
  hipError_t e = diag_init();
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_update<double, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(double)));
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_update<float, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(double)));
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_update<float, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(2 * 64 * TB * sizeof(float)));
  if (e != hipSuccess) return e;
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
template void launch_tile_gemm<double>(const GemmTerm<double>*, const GemmOut*, int, hipStream_t);
template void launch_tile_gemm<float>(const GemmTerm<float>*, const GemmOut*, int, hipStream_t);

}  // namespace lma
