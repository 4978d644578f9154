// SE-ARD kernel-matrix times vector on 128 x 128 tiles (gfx950).
//
// One workgroup (4 wave64) per item, or per part of an item's column list: the item's
// row coordinates stay in LDS, each column tile is staged in LDS in turn, the cross
// products x_r . x_c come from v_mfma_f64_16x16x4f64 (one 16-column strip of up to four
// 16-row sub-tiles at a time, so that few accumulators are live; lane l supplies row
// l%16 and coordinate k4 + l/16 of a 4-wide step), and the epilogue forms
// d^2 = |x_r|^2 + |x_c|^2 - 2 x_r . x_c (all coordinates taken relative to the item's
// first row point), the covariance and its products with the column vectors, accumulated
// per row in registers.  Row sums are reduced in a fixed order (lane shuffles, the column
// shares of the waves, the parts), so results do not depend on scheduling.
//
// Bound: the exponentials on the vector units; before, the serial column list of an item
// (7 us per column tile of one wave per SIMD) with most of the chip idle.  Waves share a
// tile as 64 x 64 quadrants, or as 32 columns each where the item has at most 64 rows;
// 16-row sub-tiles without a row are left out.  Lists are cut into parts until the launch
// has KV_PIECES workgroups; k_kvec_end adds them.  With k_kv_weights, whole calls:
// prediction of 100 points 3.93 -> 3.41 ms, covariance of 512 3.34 -> 2.73, full GP of
// n=16384 with 4096 test points 236.8 -> 229.0, n=600 fit and prediction 917 -> 792 us.
#include "engine.h"
#include "kvec.h"
#include "mfma_core.h"
#include "misc.h"

#include <algorithm>

namespace lma {

__device__ inline double vdot_wave(const double* __restrict__ a, const double* __restrict__ b, int n, int lane) {
  double s0 = 0.0, s1 = 0.0;
  int k = lane;
  for (; k + 64 < n; k += 128) {
    s0 += a[k] * b[k];
    s1 += a[k + 64] * b[k + 64];
  }
  for (; k < n; k += 64) s0 += a[k] * b[k];
  double s = s0 + s1;
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  return s;
}

// The output row from its two sums (tid = row) and the two whitened dots.
__device__ inline void kv_row(const KvArgs& a, const KvItem& it, int r, double acc0, double acc1, double vd0,
                              double vd1) {
  if (a.mode == KV_CG) {
    if (r < it.nr) it.out0[r] = it.base0[r] - acc0;
  } else if (a.mode == KV_MEAN) {
    if (r < it.nr) it.out0[r] = a.mu + acc0 - vd0;
  } else {
    if (r < it.nr) {
      it.out0[r] = it.base0[r] - (acc0 + a.sn2 * it.self0[r] - vd0);
      if (it.flag) it.out1[r] = it.base0[r] - (acc1 + a.sn2 * it.self1[r] - vd1);
    } else {
      it.out0[r] = 0.0;
      if (it.flag) it.out1[r] = 0.0;
    }
  }
}

// PART: workgroup p of a.nsplit takes its share of the column list and leaves its row
// sums in a.part; otherwise the whole list and the output rows.
template <bool PART>
__global__ __launch_bounds__(256) void k_kvec(KvArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int d = a.d, dp = (d + 3) & ~3, ldx = dp + 1;
  double* xr = reinterpret_cast<double*>(smem_raw);  // [TB][ldx] row coordinates
  double* xc = xr + TB * ldx;                        // [TB][ldx] column coordinates
  double* nrm_r = xc + TB * ldx;                     // [TB]
  double* nrm_c = nrm_r + TB;                        // [TB]
  double* cv0 = nrm_c + TB;                          // [TB]
  double* cv1 = cv0 + TB;                            // [TB]
  double* red = cv1 + TB;                            // [2 sums][4 column shares][TB]
  double* vd = red + 8 * TB;                         // [2][TB] whitened-row dots
  const int nsplit = PART ? a.nsplit : 1;
  const int logical = xcd_logical(blockIdx.x, gridDim.x);
  if (logical >= a.nitems * nsplit) return;
  const KvItem it = a.items[logical / nsplit];
  const int piece = logical % nsplit, clen = it.c1 - it.c0;
  const int c_lo = it.c0 + (int)((int64_t)clen * piece / nsplit);
  const int c_hi = it.c0 + (int)((int64_t)clen * (piece + 1) / nsplit);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // the wave's share: rows from rbase (ng sub-tiles of 16), nrb strips of 16 columns from cbase
  const bool wide = it.nr > 64;
  const int rbase = wide ? (w >> 1) * 64 : 0, cbase = wide ? (w & 1) * 64 : w * 32, nrb = wide ? 4 : 2;
  const int nshare = wide ? 2 : 4, share = wide ? (w & 1) : w;
  const int ng = (it.nr - rbase + 15) / 16;  // sub-tiles ra >= ng hold no row (may be <= 0 or > 4)

  // coordinates relative to the item's first row point (distances are
  // translation invariant; small norms keep |x|^2 + |y|^2 - 2 x.y accurate)
  __shared__ double org[MAX_D];
  if (tid < d) org[tid] = it.nr > 0 ? it.x[tid] : 0.0;
  __syncthreads();
  for (int idx = tid; idx < TB * dp; idx += NT) {
    const int r = idx / dp, k = idx - r * dp;
    xr[r * ldx + k] = (r < it.nr && k < d) ? it.x[(int64_t)r * d + k] - org[k] : 0.0;
  }
  __syncthreads();
  if (tid < TB) {
    double s = 0.0;
    for (int k = 0; k < dp; ++k) s += xr[tid * ldx + k] * xr[tid * ldx + k];
    nrm_r[tid] = s;
  }
  double s0[4][4], s1[4][4];
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int v = 0; v < 4; ++v) s0[ra][v] = s1[ra][v] = 0.0;
  const double sf2 = a.sf2;

  for (int c = c_lo; c < c_hi; ++c) {
    const KvCol col = a.cols[c];
    __syncthreads();  // the previous column tile is consumed
    for (int r = tid >> 1; r < TB; r += NT / 2)
      for (int k = tid & 1; k < dp; k += 2)
        xc[r * ldx + k] = (r < col.nc && k < d) ? col.x[(int64_t)r * d + k] - org[k] : 0.0;
    if (tid < TB) {
      cv0[tid] = (col.v0 && tid < col.nc) ? col.v0[tid] : 0.0;
      cv1[tid] = (col.v1 && tid < col.nc) ? col.v1[tid] : 0.0;
    }
    __syncthreads();
    if (tid < TB) {
      double s = 0.0;
      for (int k = 0; k < dp; ++k) s += xc[tid * ldx + k] * xc[tid * ldx + k];
      nrm_c[tid] = s;
    }
    __syncthreads();  // column norms written
    if (ng <= 0) continue;
    // one 16-column strip at a time: its product tiles, then their covariance
    // entries (keeps 16 accumulators live instead of 64)
#pragma unroll 1
    for (int rb = 0; rb < nrb; ++rb) {
      dv4 acc[4];
#pragma unroll
      for (int ra = 0; ra < 4; ++ra) acc[ra] = Mfma<double>::op(0.0, 0.0, dv4{0.0, 0.0, 0.0, 0.0});
      const int cb = (cbase + rb * 16 + (lane & 15)) * ldx + (lane >> 4);
      for (int k4 = 0; k4 < dp; k4 += 4) {
        const double bf = xc[cb + k4];
#pragma unroll
        for (int ra = 0; ra < 4; ++ra) {
          if (ra >= ng) continue;
          const double af = xr[(rbase + ra * 16 + (lane & 15)) * ldx + k4 + (lane >> 4)];
          acc[ra] = Mfma<double>::op(af, bf, acc[ra]);
        }
      }
      const int cc = cbase + rb * 16 + (lane & 15);
      const double nc = nrm_c[cc], v0 = cv0[cc], v1 = cv1[cc];
#pragma unroll
      for (int ra = 0; ra < 4; ++ra) {
        if (ra >= ng) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int rr = rbase + ra * 16 + Mfma<double>::row(lane, v);
          double d2 = nrm_r[rr] + nc - 2.0 * acc[ra][v];
          d2 = d2 > 0.0 ? d2 : 0.0;
          const double kv = sf2 * exp(-0.5 * d2);
          s0[ra][v] += kv * v0;
          s1[ra][v] += kv * v1;
        }
      }
    }
  }

  // row sums: over the 16 column lanes, then over the waves' column shares
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double x0 = s0[ra][v], x1 = s1[ra][v];
      for (int o = 1; o < 16; o <<= 1) {
        x0 += __shfl_xor(x0, o);
        x1 += __shfl_xor(x1, o);
      }
      if ((lane & 15) == 0) {
        const int rr = rbase + ra * 16 + Mfma<double>::row(lane, v);
        red[share * TB + rr] = x0;
        red[(4 + share) * TB + rr] = x1;
      }
    }
  if constexpr (!PART) {
    // whitened-row dots (one wave per row)
    for (int r = w; r < TB; r += NT / 64) {
      double d0 = 0.0, d1 = 0.0;
      if (it.vt != nullptr && r < it.nr) {
        const double* vr = it.vt + (int64_t)r * a.sp;
        if (it.h0) d0 = vdot_wave(vr, it.h0, a.sp, lane);
        if (it.h1 && it.flag) d1 = vdot_wave(vr, it.h1, a.sp, lane);
      }
      if (lane == 0) {
        vd[r] = d0;
        vd[TB + r] = d1;
      }
    }
  }
  __syncthreads();
  if (tid < TB) {
    double acc0 = 0.0, acc1 = 0.0;
    if (wide || tid < 64)
      for (int q = 0; q < nshare; ++q) {
        acc0 += red[q * TB + tid];
        acc1 += red[(4 + q) * TB + tid];
      }
    if constexpr (PART) {
      double* out = a.part + (int64_t)logical * 2 * TB;
      out[tid] = acc0;
      out[TB + tid] = acc1;
    } else {
      kv_row(a, it, tid, acc0, acc1, vd[tid], vd[TB + tid]);
    }
  }
}

// Sums of the parts in order, and the output rows: one wave per row (lanes share the
// whitened dot), KV_ROWS rows per workgroup.
constexpr int KV_ROWS = 16;
__global__ __launch_bounds__(256) void k_kvec_end(KvArgs a) {
  const KvItem it = a.items[blockIdx.x / (TB / KV_ROWS)];
  const int r0 = blockIdx.x % (TB / KV_ROWS) * KV_ROWS;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double* part = a.part + (int64_t)(blockIdx.x / (TB / KV_ROWS)) * a.nsplit * 2 * TB;
  for (int r = r0 + w; r < r0 + KV_ROWS; r += NT / 64) {
    double d0 = 0.0, d1 = 0.0, s0 = 0.0, s1 = 0.0;
    if (r < it.nr) {
      if (it.vt != nullptr) {
        const double* vr = it.vt + (int64_t)r * a.sp;
        if (it.h0) d0 = vdot_wave(vr, it.h0, a.sp, lane);
        if (it.h1 && it.flag) d1 = vdot_wave(vr, it.h1, a.sp, lane);
      }
      // lane q holds part q (nsplit <= 64)
      if (lane < a.nsplit) {
        s0 = part[(int64_t)lane * 2 * TB + r];
        s1 = part[(int64_t)lane * 2 * TB + TB + r];
      }
      for (int o = 32; o > 0; o >>= 1) {
        s0 += __shfl_xor(s0, o);
        s1 += __shfl_xor(s1, o);
      }
    }
    if (lane == 0) kv_row(a, it, r, s0, s1, d0, d1);
  }
}

// Weights of the predictive mean over the training points of block q's span: the J
// vectors of windows q-B .. q minus the W vectors of all but the last, so that every
// training point is met once instead of once per window that holds it (of a full GP's
// last block 1088 column tiles become 128).
__global__ __launch_bounds__(256) void k_kv_weights(const KvWeights* __restrict__ items, const int64_t* __restrict__ tab,
                                                    const double* __restrict__ xJ, const double* __restrict__ xW,
                                                    double* __restrict__ out, int M, int B) {
  const KvWeights it = items[blockIdx.x];
  const int64_t* wstart = tab;
  const int64_t* wlen = tab + M;
  const int64_t* dstart = tab + 2 * (int64_t)M;
  const int64_t* dlen = tab + 3 * (int64_t)M;
  const int64_t* vec = tab + 6 * (int64_t)M;
  const int32_t* tw = reinterpret_cast<const int32_t*>(tab + 8 * (int64_t)M) + M;
  const int m0 = it.q > B ? it.q - B : 0;
  for (int64_t x = it.x0 + (int64_t)blockIdx.y * NT + threadIdx.x; x < it.x1; x += (int64_t)gridDim.y * NT) {
    double s = 0.0;
    for (int m = m0; m <= it.q; ++m) {
      const int64_t de = dstart[m] + dlen[m];
      if (x >= dstart[m] && x < de) {
        s += xJ[vec[m] + (int64_t)tw[m] * TB + (x - dstart[m])];
      } else if (x >= wstart[m] && x < wstart[m] + wlen[m]) {
        const int64_t e = vec[m] + (x - wstart[m]);
        s += xJ[e];
        if (m < it.q) s -= xW[e];
      }
    }
    out[it.out + (x - it.x0)] = s;
  }
}

__global__ void k_hq(const double* __restrict__ hJ, const double* __restrict__ hW, double* __restrict__ hq, int M,
                     int B, int sp) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)M * sp) return;
  const int q = (int)(e / sp), k = (int)(e - (int64_t)q * sp);
  double s = 0.0;
  for (int dl = 0; dl <= B && dl <= q; ++dl) {
    s += hJ[(int64_t)(q - dl) * sp + k];
    if (dl > 0) s -= hW[(int64_t)(q - dl) * sp + k];
  }
  hq[e] = s;
}

static size_t kvec_lds(int d) {
  const int ldx = ((d + 3) & ~3) + 1;
  return sizeof(double) * (size_t)(2 * TB * ldx + 14 * TB);
}

int kvec_split(int64_t nitems, int64_t longest) {
  if (nitems <= 0 || nitems >= KV_PIECES) return 1;
  return (int)std::max<int64_t>(1, std::min<int64_t>({(KV_PIECES + nitems - 1) / nitems, longest, 64}));
}

void launch_kvec(const KvArgs& a, hipStream_t st) {
  if (a.nitems <= 0) return;
  if (a.nsplit > 1 && a.part != nullptr) {
    hipLaunchKernelGGL(k_kvec<true>, dim3((a.nitems * a.nsplit + 7) / 8 * 8), dim3(NT), kvec_lds(a.d), st, a);
    hipLaunchKernelGGL(k_kvec_end, dim3(a.nitems * (TB / KV_ROWS)), dim3(NT), 0, st, a);
    return;
  }
  hipLaunchKernelGGL(k_kvec<false>, dim3((a.nitems + 7) / 8 * 8), dim3(NT), kvec_lds(a.d), st, a);
}

void launch_kv_weights(const KvWeights* items, int nitems, int64_t longest, const int64_t* tab, const double* xJ,
                       const double* xW, double* out, int M, int B, hipStream_t st) {
  if (nitems <= 0) return;
  const unsigned ny = (unsigned)std::max<int64_t>(1, std::min<int64_t>((longest + NT - 1) / NT, 1024));
  hipLaunchKernelGGL(k_kv_weights, dim3(nitems, ny), dim3(NT), 0, st, items, tab, xJ, xW, out, M, B);
}

void launch_hq(const double* hJ, const double* hW, double* hq, int M, int B, int sp, hipStream_t st) {
  const int64_t n = (int64_t)M * sp;
  hipLaunchKernelGGL(k_hq, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, hJ, hW, hq, M, B, sp);
}

hipError_t kvec_init() {
  hipError_t e = hipFuncSetAttribute((const void*)k_kvec<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)kvec_lds(MAX_D));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_kvec<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)kvec_lds(MAX_D));
}

}  // namespace lma
