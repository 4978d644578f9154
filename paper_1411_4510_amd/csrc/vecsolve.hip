// Vector solves with the stored window factors and the predictive mean.
//
// With g = Sigma_ddot_SS^-1 y_ddot_S and beta_X = R_X^-1 (c_X - K_XS g) for the
// windows X = J_m and the separators X = W_m, the predictive mean of Eq. (3)
// for u in test block q is
//   mu + k_u^T g + sum_{m=q-B..q} R_{u,J_m} beta_{J_m} - sum_{m=q-B..q-1} R_{u,W_m} beta_{W_m}.
// (Woodbury on Sigma_bar_DD = Q + R_bar and the signed window sum of
// R_bar_DD^-1 that the banded factor of Lemma 1 gives; the separator term of
// window q cancels against its own leading block.)  Only vector solves are
// needed, so they run in float64 arithmetic even on float32 factors.  The
// forward half is read off the whitened right-hand sides the factorisation
// already produced.  In mixed precision one refinement of beta against the
// float64 residual covariance and one global correction of g (whose residual
// is L_SS (sum_m V_{J_m} beta_{J_m} - V_{W_m} beta_{W_m}) - Sigma_SS g)
// restore float64-level accuracy of the mean.
#include "engine.h"
#include "misc.h"

namespace lma {

__device__ inline int64_t win_point(const WinTab& w, int m, int r, bool& valid) {
  const int tw = w.tw[m];
  if (r < tw * TB) {
    valid = r < w.wlen[m];
    return w.wstart[m] + r;
  }
  const int rr = r - tw * TB;
  valid = rr < w.dlen[m];
  return w.dstart[m] + rr;
}

__device__ inline int64_t jp_off(int i) { return (int64_t)TB * TB * i * (i + 1) / 2; }

__device__ inline double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ---------------------------------------------------------------------------
// triangular solves of one vector per window and separator
// ---------------------------------------------------------------------------
// Right-looking over the tiles, all windows in lock step, one launch per column
// tile: launch i subtracts the products with the tile solved before from every
// tile that is left (one workgroup per 128 x 128 factor tile), and the workgroup
// whose tile is next solves it at once with the inverted diagonal tile.  It alone
// touches that tile of the vector, so the solution replaces the vector in place.
// W_m's factor is the leading block of J_m's, so both vectors take part in one
// read of a tile.  A launch holds the windows that have a tile in it: 20000 windows of
// 2 points beside one of 8000 in mixed precision (B=0) took 95 ms, nearly all of it
// empty workgroups, with every window in each launch, and take 3.3 ms (the fit 135 -> 40).
// Bound: one read of the factors (HBM), and for few or narrow windows the launches.
// Measured against one workgroup per window walking its factor once for each vector:
// backward at n=16384, M=16, B=15 (6.3 GB of factors) 44.2 -> 2.6 ms, n=2048 92 -> 20 us
// (4 launches); forward and backward of a mixed fit (n=50021, B=3) 26.7 -> about 4 ms.
constexpr int SOLVE_NT = 512;
constexpr int SOLVE_W = SOLVE_NT / 64;
constexpr int SOLVE_R = TB / SOLVE_W;  // tile rows of a wave

template <typename TW>
struct Vec2;
template <>
struct Vec2<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <>
struct Vec2<double> { typedef double type __attribute__((ext_vector_type(2))); };

// The rows of this wave (SOLVE_R of them from row SOLVE_R * wave on) of a 128 x 128
// tile; each lane holds columns 2 lane and 2 lane + 1.
template <typename TW>
__device__ inline void load_rows(const TW* tile, int64_t ld, typename Vec2<TW>::type (&a)[SOLVE_R]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < SOLVE_R; ++r)
    a[r] = *(const typename Vec2<TW>::type*)(tile + (int64_t)(wv * SOLVE_R + r) * ld + 2 * lane);
}

// out[c] = sum_r a[r][c] x[r] over the 128 rows of the tile, for the threads c < 128
template <typename TW>
__device__ inline double mul_t(const typename Vec2<TW>::type (&a)[SOLVE_R], const double* x, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int r = 0; r < SOLVE_R; ++r) {
    const double xr = x[wv * SOLVE_R + r];
    s0 += (double)a[r][0] * xr;
    s1 += (double)a[r][1] * xr;
  }
  __syncthreads();
  red[wv * TB + 2 * lane] = s0;
  red[wv * TB + 2 * lane + 1] = s1;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x < TB)
#pragma unroll
    for (int q = 0; q < SOLVE_W; ++q) s += red[q * TB + threadIdx.x];
  return s;
}

// out[r] = sum_c a[r][c] x[c], for the threads r < 128
template <typename TW>
__device__ inline double mul_n(const typename Vec2<TW>::type (&a)[SOLVE_R], const double* x, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double x0 = x[2 * lane], x1 = x[2 * lane + 1];
  double v[SOLVE_R];
#pragma unroll
  for (int r = 0; r < SOLVE_R; ++r) v[r] = (double)a[r][0] * x0 + (double)a[r][1] * x1;
  // halve the rows held per lane with each exchange: lane bit b keeps the rows with that bit
#pragma unroll
  for (int n = SOLVE_R / 2, o = 32; n >= 1; n >>= 1, o >>= 1) {
    const bool hi = lane & o;
#pragma unroll
    for (int r = 0; r < n; ++r) {
      const double give = hi ? v[r] : v[r + n], keep = hi ? v[r + n] : v[r];
      v[r] = keep + __shfl_xor(give, o);
    }
  }
  double s = v[0];
#pragma unroll
  for (int o = 64 / SOLVE_R / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  __syncthreads();
  if ((lane & (64 / SOLVE_R - 1)) == 0) red[wv * SOLVE_R + lane / (64 / SOLVE_R)] = s;
  __syncthreads();
  return threadIdx.x < TB ? red[threadIdx.x] : 0.0;
}

// Step i of the solves with L^T (BWD, i = maxT .. 1: tile i is solved, tile i - 1
// comes next) or with L (i = 0 .. maxT - 1: tile i - 1 is solved, tile i comes next).
template <typename TW, bool BWD>
__global__ __launch_bounds__(SOLVE_NT) void k_solve_step(WinVecArgs<TW> a, int i, int y0) {
  __shared__ double xJ[TB], xW[TB];
  __shared__ double red[SOLVE_W * TB];
  typedef typename Vec2<TW>::type V2;
  const int m = a.order[blockIdx.x], tid = threadIdx.x;
  const WinTab& w = a.w;
  const int T = w.T[m], tw = w.tw[m];
  // the tile of the vector this workgroup updates, and whether there is a solved tile to subtract
  const int y = y0 + (int)blockIdx.y;
  const int tv = BWD ? i - 1 - y : i + y;
  const int ts = BWD ? i : i - 1;
  if (tv < 0 || tv >= T) return;
  const bool upd = BWD ? i < T : i > 0, next = y == 0;
  if (BWD && i > T) return;
  if (!upd && !next) return;
  const bool inW = tv < tw, updW = inW && (BWD ? i < tw : i > 0);
  const TW* base = a.panels + w.panel[m];
  double* vJ = a.vJ + w.vec[m] + (int64_t)tv * TB;
  double* vW = a.vW + w.vec[m] + (int64_t)tv * TB;
  V2 lt[SOLVE_R], li[SOLVE_R];
  if (upd) {
    const int tr = BWD ? ts : tv, tc = BWD ? tv : ts;
    load_rows<TW>(base + jp_off(tr) + (int64_t)tc * TB, (int64_t)(tr + 1) * TB, lt);
  }
  if (next) load_rows<TW>(a.invs + w.inv[m] + (int64_t)tv * TB * TB, TB, li);
  double rJ = 0.0, rW = 0.0;
  if (tid < TB) {
    rJ = vJ[tid];
    if (inW) rW = vW[tid];
  }
  if (upd) {
    const int64_t so = w.vec[m] + (int64_t)ts * TB;
    if (tid < TB) {
      xJ[tid] = a.vJ[so + tid];
      if (updW) xW[tid] = a.vW[so + tid];
    }
    __syncthreads();
    rJ -= BWD ? mul_t<TW>(lt, xJ, red) : mul_n<TW>(lt, xJ, red);
    if (updW) rW -= BWD ? mul_t<TW>(lt, xW, red) : mul_n<TW>(lt, xW, red);
  }
  if (next) {
    __syncthreads();
    if (tid < TB) {
      xJ[tid] = rJ;
      xW[tid] = rW;
    }
    __syncthreads();
    rJ = BWD ? mul_t<TW>(li, xJ, red) : mul_n<TW>(li, xJ, red);
    if (inW) rW = BWD ? mul_t<TW>(li, xW, red) : mul_n<TW>(li, xW, red);
  }
  if (tid < TB) {
    vJ[tid] = rJ;
    if (inW) vW[tid] = rW;
  }
}

// L_J^-1 (c_J - K_JS g) from the stored whitened right-hand sides:
// [p; z] - [Pi; Z] g  (its W_m prefix is L_11^-1 (c_W - K_WS g)).
template <typename TW>
__global__ __launch_bounds__(256) void k_ycp(WinVecArgs<TW> a) {
  const int m = blockIdx.x;
  const WinTab& w = a.w;
  const int T = w.T[m], tw = w.tw[m];
  const int col = blockIdx.y * blockDim.x + threadIdx.x;
  if (col >= T * TB) return;
  const int64_t ld = (int64_t)T * TB;
  const TW* R = a.panels + w.rhs[m];
  double s0 = (double)R[(int64_t)a.sp * ld + col], s1 = 0.0, s2 = 0.0, s3 = 0.0;
  int k = 0;
  for (; k + 3 < a.s; k += 4) {
    s0 -= (double)R[(int64_t)k * ld + col] * a.g[k];
    s1 -= (double)R[(int64_t)(k + 1) * ld + col] * a.g[k + 1];
    s2 -= (double)R[(int64_t)(k + 2) * ld + col] * a.g[k + 2];
    s3 -= (double)R[(int64_t)(k + 3) * ld + col] * a.g[k + 3];
  }
  for (; k < a.s; ++k) s0 -= (double)R[(int64_t)k * ld + col] * a.g[k];
  const double y = (s0 + s1) + (s2 + s3);
  const int64_t vo = w.vec[m];
  a.vJ[vo + col] = y;
  if (col < tw * TB) a.vW[vo + col] = y;
}

__device__ inline double tiled_L(const double* L, int r, int k) {
  const int ti = r / TB, tk = k / TB;
  return L[jp_off(ti) + (int64_t)(r - ti * TB) * (ti + 1) * TB + tk * TB + (k - tk * TB)];
}

// rho = L (H - L^T g), H = sum_m (hJ_m - hW_m) in block order; one workgroup
__global__ __launch_bounds__(256) void k_gres(GresArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* u = reinterpret_cast<double*>(smem_raw);  // [sp]
  const int sp = a.sp;
  for (int k = threadIdx.x; k < sp; k += blockDim.x) {
    double H = 0.0;
    for (int m = 0; m < a.M; ++m) H += a.hJ[(int64_t)m * sp + k] - a.hW[(int64_t)m * sp + k];
    double lg = 0.0;
    for (int r = k; r < sp; ++r) lg += tiled_L(a.L, r, k) * a.g[r];
    u[k] = H - lg;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < sp; r += blockDim.x) {
    double s = 0.0;
    for (int k = 0; k <= r; ++k) s += tiled_L(a.L, r, k) * u[k];
    a.rho[r] = s;
  }
}

// g += dg, t = L^T dg; one workgroup
__global__ __launch_bounds__(256) void k_gupdate(const double* L, const double* dg, double* g, double* t, int sp) {
  for (int k = threadIdx.x; k < sp; k += blockDim.x) {
    double lg = 0.0;
    for (int r = k; r < sp; ++r) lg += tiled_L(L, r, k) * dg[r];
    t[k] = lg;
    g[k] += dg[k];
  }
}

__global__ __launch_bounds__(256) void k_vdot(const double* Vt, const double* t, double* out, int64_t n, int sp) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;
  double s = 0.0;
  for (int k = lane; k < sp; k += 64) s += Vt[i * sp + k] * t[k];
  s = wave_sum(s);
  if (lane == 0) out[i] = s;
}

__global__ __launch_bounds__(256) void k_gather(WinTab w, const double* pt, double* vJ, double* vW) {
  const int m = blockIdx.x;
  const int T = w.T[m], tw = w.tw[m];
  const int r = blockIdx.y * blockDim.x + threadIdx.x;
  if (r >= T * TB) return;
  bool v;
  const int64_t p = win_point(w, m, r, v);
  const double x = v ? pt[p] : 0.0;
  const int64_t vo = w.vec[m];
  vJ[vo + r] = x;
  if (r < tw * TB) vW[vo + r] = x;
}

__global__ __launch_bounds__(256) void k_axpy2(double* vJ, double* vW, const double* xJ, const double* xW,
                                               double alpha, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    vJ[i] += alpha * xJ[i];
    vW[i] += alpha * xW[i];
  }
}

// h = V_X x, one workgroup per window and 64 columns of V: its 16 waves take every
// 16th row and the partial sums are added in wave order.  Bound: one read of the
// window's V rows.  With one thread walking all rows of a column the loads were a
// serial chain: 68 -> 13 us at n=2048, 2.5 ms -> 0.36 ms at n=16384 with B=15.
constexpr int H_W = 16;
__global__ __launch_bounds__(64 * H_W) void k_h(HArgs a) {
  __shared__ double red[2][H_W][64];
  const int m = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int k = blockIdx.y * 64 + lane;
  const WinTab& w = a.w;
  const int64_t vo = w.vec[m], wl = w.wlen[m], dl = w.dlen[m];
  double hj = 0.0, hw = 0.0;
  const double* V = a.Vt + w.wstart[m] * a.sp + k;
#pragma unroll 4
  for (int64_t r = wv; r < wl; r += H_W) {
    const double v = V[r * a.sp];
    hj += v * a.xJ[vo + r];
    hw += v * a.xW[vo + r];
  }
  V = a.Vt + w.dstart[m] * a.sp + k;
  const double* x = a.xJ + vo + (int64_t)w.tw[m] * TB;
#pragma unroll 4
  for (int64_t r = wv; r < dl; r += H_W) hj += V[r * a.sp] * x[r];
  red[0][wv][lane] = hj;
  red[1][wv][lane] = hw;
  __syncthreads();
  if (wv < 2) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < H_W; ++q) s += red[wv][q][lane];
    (wv == 0 ? a.hJ : a.hW)[(int64_t)m * a.sp + k] = s;
  }
}

template <typename TW>
void launch_ycp(const WinVecArgs<TW>& a, int M, int maxT, hipStream_t st) {
  hipLaunchKernelGGL(k_ycp<TW>, dim3(M, (maxT * TB + 255) / 256), dim3(256), 0, st, a);
}
// A workgroup without a tile takes 0.48 ns (20000 windows, maxT=63: 195M of them 95 ms),
// a launch about 4 us: launches are cut where they would hold more empty ones than this.
constexpr int64_t SOLVE_EMPTY = 8192;
template <typename TW>
void launch_fwd(const WinVecArgs<TW>& a, const int32_t* above, int maxT, hipStream_t st) {
  for (int i = 0; i < maxT; ++i) {
    const int ys = i > 0 ? maxT - i : 1;
    for (int y = 0, ny; y < ys; y += ny) {
      const int n = above[i + y];
      int64_t empty = 0;
      for (ny = 1; y + ny < ys && (empty += n - above[i + y + ny]) <= SOLVE_EMPTY;) ++ny;
      hipLaunchKernelGGL((k_solve_step<TW, false>), dim3(n, ny), dim3(SOLVE_NT), 0, st, a, i, y);
    }
  }
}
template <typename TW>
void launch_bwd(const WinVecArgs<TW>& a, const int32_t* above, int maxT, hipStream_t st) {
  for (int i = maxT; i > 0; --i) {
    // windows of i tiles start here with their last one; those of more subtract from all i
    const int n = above[i - 1], more = i < maxT ? above[i] : 0;
    const bool together = more > 0 && (int64_t)(n - more) * (i - 1) <= SOLVE_EMPTY;
    hipLaunchKernelGGL((k_solve_step<TW, true>), dim3(n, together ? i : 1), dim3(SOLVE_NT), 0, st, a, i, 0);
    if (more > 0 && !together)
      hipLaunchKernelGGL((k_solve_step<TW, true>), dim3(more, i - 1), dim3(SOLVE_NT), 0, st, a, i, 1);
  }
}
void launch_gres(const GresArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_gres, dim3(1), dim3(256), sizeof(double) * (size_t)a.sp, st, a);
}
void launch_gupdate(const double* L, const double* dg, double* g, double* t, int sp, hipStream_t st) {
  hipLaunchKernelGGL(k_gupdate, dim3(1), dim3(256), 0, st, L, dg, g, t, sp);
}
void launch_vdot(const double* Vt, const double* t, double* out, int64_t n, int sp, hipStream_t st) {
  hipLaunchKernelGGL(k_vdot, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, Vt, t, out, n, sp);
}
void launch_gather(const WinTab& w, const double* pt, double* vJ, double* vW, int M, int maxT, hipStream_t st) {
  hipLaunchKernelGGL(k_gather, dim3(M, (maxT * TB + 255) / 256), dim3(256), 0, st, w, pt, vJ, vW);
}
void launch_axpy2(double* vJ, double* vW, const double* xJ, const double* xW, double alpha, int64_t nvec,
                  hipStream_t st) {
  if (nvec <= 0) return;
  const int nb = (int)std::min<int64_t>((nvec + 255) / 256, 65536);
  hipLaunchKernelGGL(k_axpy2, dim3(nb), dim3(256), 0, st, vJ, vW, xJ, xW, alpha, nvec);
}
void launch_h(const HArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_h, dim3(a.M, a.sp / 64), dim3(64 * H_W), 0, st, a);
}
template void launch_ycp<double>(const WinVecArgs<double>&, int, int, hipStream_t);
template void launch_ycp<float>(const WinVecArgs<float>&, int, int, hipStream_t);
template void launch_fwd<double>(const WinVecArgs<double>&, const int32_t*, int, hipStream_t);
template void launch_fwd<float>(const WinVecArgs<float>&, const int32_t*, int, hipStream_t);
template void launch_bwd<double>(const WinVecArgs<double>&, const int32_t*, int, hipStream_t);
template void launch_bwd<float>(const WinVecArgs<float>&, const int32_t*, int, hipStream_t);

}  // namespace lma
