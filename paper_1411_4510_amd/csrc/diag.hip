// Diagonal tiles of the engine's column steps (gfx950): the Cholesky factor of
// the 128 x 128 tile (j, j), its log-diagonal, and the inverse of the factor for
// the triangular solves of the tiles below.  One workgroup per tile.
//
// The tile is factored and inverted in float64 for every storage type (the
// float32 window factors of the mixed mode included): the diagonal tiles of
// late column steps hold Schur complements near the noise level, and their
// factor and inverse feed every later tile.
//
// Two kernels.  Mixed-precision fits round the factor and the inverse of every
// window to float32, and which way an entry rounds depends on the last bits of the
// float64 result; they keep the order of operations of k_diag32 (and so does their
// Sigma_SS, whose factor the residual entries are formed with).  Float64 fits take
// k_diag16.
#include "engine.h"
#include "mfma_core.h"

#include <type_traits>

namespace lma {

// k_diag16 (float64 fits).  The serial chain of 128 pivots cannot be shortened, so
// it is kept in registers.  The 128 x 128 tile is cut into 16 x 16 blocks
// whose lower half lives in the accumulators of the four waves (block (i, j) with
// wave j mod 4).  For each block column kb the column goes to LDS as 16-wide rows;
// every lane then holds one row: lanes 0-15 of every wave the diagonal block (four copies, so the
// pivots need no barrier), lanes 16-47 the rows of two other blocks.  One pass over
// the 16 columns factors the diagonal block and solves all other rows against it,
// with the pivot row read by v_readlane.  The rows of block kb itself are rows of
// the identity, so what comes out for them is L_kk^-T: the inverse advances as
// right-hand-side rows b -> b L^-T of the same elimination, in the accumulator
// slots that the finished blocks of L leave (block (kb, j) of L^-T in the slot of
// block (j, kb) of L).  The trailing update of both is one MFMA product per slot.
// Two barriers per block column; they order LDS only, so the stores of the results
// (from LDS, in whole rows) drain behind the next block column.
// Measured per launch (one workgroup per diagonal tile): 205 us for 32 x 32 blocks with
// columns and sums as loops over LDS, 35 us in this form.  Bound: of the 35 us the pivot
// chain is 10; the rest is the sixteen barriers, the trips of a block column through LDS
// and the trailing products between them, one after the other.
constexpr int NB = 16;          // block edge
constexpr int NBK = TB / NB;    // blocks per tile side
constexpr int PLD = NB + 2;     // row stride of the panel in LDS (16-byte aligned rows)
static_assert(NBK == 8 && NT == 256, "block (i, j): slot (i, j >> 2) of wave j & 3");

// lane l's value of x, the same in every lane
__device__ inline double lane_value(double x, int l) {
  const int2 v = __builtin_bit_cast(int2, x);
  int2 r;
  r.x = __builtin_amdgcn_readlane(v.x, l);
  r.y = __builtin_amdgcn_readlane(v.y, l);
  return __builtin_bit_cast(double, r);
}

// 1/sqrt(d) of a positive d: the hardware's estimate (error about 2^-23) and one
// third-order step y (1 + e/2 + 3 e^2 / 8), e = 1 - d y^2.  For d = +inf the
// estimate is 0 and e NaN: the minimum makes the result 0.
__device__ inline double rsqrt_pos(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = __builtin_fmin(__builtin_fma(-(d * y), y, 1.0), 1.0);
  return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

__global__ __launch_bounds__(NT) void k_diag16(StepArgs<double> a, const int32_t* __restrict__ plist) {
  __shared__ __align__(16) double pin[TB * PLD];   // block column kb before its elimination
  __shared__ __align__(16) double pout[TB * PLD];  // the same rows solved
  __shared__ __align__(16) double dblk[NB * PLD];  // its diagonal block
  __shared__ __align__(16) double lkk[NB * PLD];   // and the factor of that
  __shared__ double piv[TB];
  __shared__ double lsum[NT / 64];
  const int p = plist[blockIdx.x];
  const ProbDesc pd = a.pd[p];
  const RowTile<double> rj = a.rt[pd.first + a.j];
  double* src = rj.panel + (int64_t)a.j * TB;
  double* inv = a.invdiag + pd.invdiag_off + (int64_t)a.j * TB * TB;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lh = lane >> 4;
  // slot (i, h) holds block (i, j), j = w + 4 h, if j <= i
  dv4 acc[NBK][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 4 * h; i < NBK; ++i)
      if (w + 4 * h <= i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[i][h][v] = src[(int64_t)(i * NB + lh + 4 * v) * rj.ld + (w + 4 * h) * NB + l16];
  int bad = 0;
  for (int kb = 0; kb < NBK; ++kb) {
    // ---- block column kb to LDS: blocks (i, kb) below the diagonal, the diagonal
    // block, and blocks (r, kb), r < kb, of the inverse rows (slots (kb, r))
    auto put = [&](double* dst, const dv4& c) {
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[(lh + 4 * v) * PLD + l16] = c[v];
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = w + 4 * h;
      if (j == kb) {
#pragma unroll
        for (int i = 4 * h; i < NBK; ++i) {
          if (i < kb) continue;
          put(i == kb ? dblk : pin + i * NB * PLD, acc[i][h]);
          acc[i][h] = (dv4){0.0, 0.0, 0.0, 0.0};  // from here on the slot of an inverse row block
        }
      } else if (j < kb) {
#pragma unroll
        for (int i = 4 * h; i < NBK; ++i)
          if (i == kb) put(pin + j * NB * PLD, acc[i][h]);
      }
    }
    if (w == ((kb + 1) & 3)) {  // block kb's own rows: the identity
      dv4 id;
#pragma unroll
      for (int v = 0; v < 4; ++v) id[v] = lh + 4 * v == l16 ? 1.0 : 0.0;
      put(pin + kb * NB * PLD, id);
    }
    barrier_lds();
    // ---- one row per lane
    const int t = 2 * w + ((lane >> 4) - 1);  // block of the rows in lanes 16..47
    const bool in_diag = lane < NB, live = lane >= NB && lane < 3 * NB;
    double x[NB];
    {
      const double* row = in_diag ? dblk + l16 * PLD : pin + ((live ? t : 0) * NB + l16) * PLD;
#pragma unroll
      for (int c = 0; c < NB; ++c) x[c] = row[c];
    }
    // a pivot that is not positive marks the problem; what follows from it is not used
    double d = lane_value(x[0], 0), y = rsqrt_pos(d);
    bad |= !(d > 0.0);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      x[k] *= y;
      if (k + 1 < NB) {  // the next pivot first: its root runs beside the other updates
        x[k + 1] = __builtin_fma(-x[k], lane_value(x[k], k + 1), x[k + 1]);
        d = lane_value(x[k + 1], k + 1);
        y = rsqrt_pos(d);
        bad |= !(d > 0.0);
      }
#pragma unroll
      for (int c = k + 2; c < NB; ++c) x[c] = __builtin_fma(-x[k], lane_value(x[k], c), x[c]);
      // keeps the updates of column k here: moved down, their pivot rows pile up in scalar registers
#pragma unroll
      for (int c = k + 1; c < NB; ++c) asm volatile("" : "+v"(x[c]));
    }
    if (w == 0 && in_diag) {
#pragma unroll
      for (int c = 0; c < NB; ++c) lkk[l16 * PLD + c] = x[c];
    }
    if (live) {
      double* o = pout + (t * NB + l16) * PLD;
#pragma unroll
      for (int c = 0; c < NB; ++c) o[c] = x[c];
    }
    barrier_lds();
    // ---- results: block column kb of L and rows kb of L^-1, zeros included
#pragma unroll
    for (int q = 0; q < TB * NB / 2 / NT; ++q) {
      const int idx = tid + q * NT, r = idx >> 3, c = 2 * (idx & 7), rk = r - kb * NB;
      dv2 v = *(const dv2*)((rk >= 0 && rk < NB ? lkk + rk * PLD : pout + r * PLD) + c);
      if (rk < NB) {
        v[0] = c <= rk ? v[0] : 0.0;
        v[1] = c + 1 <= rk ? v[1] : 0.0;
        if (c == (rk & ~1)) piv[r] = v[rk & 1];
      }
      *(dv2*)(src + (int64_t)r * rj.ld + kb * NB + c) = v;
    }
#pragma unroll
    for (int q = 0; q < NB * TB / NT; ++q) {
      const int idx = tid + q * NT, c = idx >> 7, r = idx & (TB - 1);
      const double v = pout[r * PLD + c];
      inv[(kb * NB + c) * TB + r] = r < (kb + 1) * NB ? v : 0.0;
    }
    // ---- trailing update: block (i, j) of L for j > kb, block (j, i) of L^-T for
    // j <= kb.  Slots that are done (i <= kb) or hold nothing (i < j) take part where
    // leaving them out would cost a branch: nothing reads them any more.
    const double* fr = pout + l16 * PLD + 4 * lh;
    auto update = [&](auto lo, auto hi, auto h) {
      constexpr int I0 = lo, I1 = hi, H = h;
      const int j = w + 4 * H;
      double fi[I1 - I0][4], fj[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) fj[e] = -fr[j * NB * PLD + e];
#pragma unroll
      for (int i = I0; i < I1; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) fi[i - I0][e] = fr[i * NB * PLD + e];
      if (j > kb) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = I0; i < I1; ++i) acc[i][H] = Mfma<double>::op(fi[i - I0][e], fj[e], acc[i][H]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = I0; i < I1; ++i) acc[i][H] = Mfma<double>::op(fj[e], fi[i - I0][e], acc[i][H]);
      }
    };
    typedef std::integral_constant<int, 0> c0;
    typedef std::integral_constant<int, 1> c1;
    typedef std::integral_constant<int, 4> c4;
    typedef std::integral_constant<int, NBK> c8;
    if (kb < 3) update(c1(), c4(), c0());
    if (kb < NBK - 1) {
      update(c4(), c8(), c0());
      update(c4(), c8(), c1());
    }
  }
  if (bad && tid == 0) a.status[p] = 1;
  // log-diagonal
  __syncthreads();
  double ls = 0.0;
  if (tid < TB && tid < rj.nvalid) ls = log(piv[tid]);
  for (int o = 32; o > 0; o >>= 1) ls += __shfl_xor(ls, o);
  if ((tid & 63) == 0) lsum[tid >> 6] = ls;
  __syncthreads();
  if (tid == 0) {
    const double tot = lsum[0] + lsum[1] + lsum[2] + lsum[3];
    a.logdiag[(int64_t)p * a.maxT + a.j] = (a.j >= pd.ld_from) ? tot : 0.0;
  }
}

// k_diag32 (mixed fits).  Both run on 32 x 32 blocks of the tile in LDS.  Factor, for
// each block column kb: right-looking columns, pivot root and reciprocal correctly
// rounded, the rows of the diagonal block scaled by the reciprocal and the rows below
// divided by the root; then the trailing lower triangle minus one sum over the 32
// columns.  Inverse (in place, X = L^-1): the four diagonal blocks, last column first,
// with the even and the odd terms of a sum added at its end; then block columns right
// to left: T_ib = sum_{k=jb+1..ib} X_ib,k L_k,jb and X_ib,jb = -T_ib X_jb,jb.
// The float64 matrix instruction is a chain of fused multiply-adds in order of k, so
// it forms those sums exactly as a loop over k does; the columns of a block run in
// registers, a row per lane (lanes 0-31 of every wave the diagonal block, lanes 32-63
// rows below it) with the pivot row by v_readlane.  Bound: the chain of 128 roots,
// reciprocals and divisions.  Measured per launch: 205 us (float32 tiles 220) with the
// columns and sums as loops over LDS, 60 us (64) in this form, with the same bits.
constexpr int DLD = TB + 1;      // row stride of the tile in LDS
constexpr int DB = 32;           // block edge
constexpr int DNB = TB / DB;     // blocks per tile side
constexpr int DT_LD = DB + 1;    // row stride of the block products' scratch

__device__ inline void wave_sync_lds() {
  // LDS writes of this wave are visible to its other lanes after this point
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__global__ __launch_bounds__(NT) void k_diag32(StepArgs<T> a, const int32_t* __restrict__ plist) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* A = reinterpret_cast<double*>(smem_raw);  // [TB][DLD]
  double* Tt = A + TB * DLD;                        // [DNB-1][DB][DT_LD] block products
  __shared__ double lsum[NT / 64];
  const int p = plist[blockIdx.x];
  const ProbDesc pd = a.pd[p];
  const RowTile<T> rj = a.rt[pd.first + a.j];
  T* src = rj.panel + (int64_t)a.j * TB;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lh = lane >> 4;
#pragma unroll 16
  for (int idx = tid; idx < TB * TB; idx += NT) {
    const int r = idx >> 7, c = idx & (TB - 1);
    const double v = (double)src[(int64_t)r * rj.ld + c];  // loaded above the diagonal too: no branch
    A[r * DLD + c] = c <= r ? v : 0.0;
  }
  __syncthreads();

  // ---- factor
  int bad = 0;
  for (int kb = 0; kb < DNB; ++kb) {
    const int b0 = kb * DB;
    {
      const bool in_diag = lane < DB;
      const int r = in_diag ? b0 + lane : b0 + DB + w * DB + (lane - DB);
      const bool live = r < TB;
      double* row = A + (live ? r : 0) * DLD + b0;
      double x[DB];
#pragma unroll
      for (int c = 0; c < DB; ++c) x[c] = row[c];
      auto pivot = [&](double d, double& root, double& ip) {
        const bool ok = d > 0.0;
        bad |= !ok;
        d = ok ? __builtin_fmin(d, 1.7976931348623157e308) : 1.0;  // keeps the residuals below defined
        // correctly rounded root and reciprocal from the reciprocal root by one residual
        // each (Markstein's theorems on division and square root)
        const double y = rsqrt_pos(d), g = d * y;
        root = __builtin_fma(__builtin_fma(-g, g, d), 0.5 * y, g);
        ip = __builtin_fma(y, __builtin_fma(-root, y, 1.0), y);
      };
      double root, ip;
      pivot(lane_value(x[0], 0), root, ip);
#pragma unroll
      for (int k = 0; k < DB; ++k) {
        const double up = x[k] * ip, below = __builtin_fma(__builtin_fma(-root, up, x[k]), ip, up);  // x / root
        x[k] = lane == k ? root : in_diag ? up : below;
        if (k + 1 < DB) {  // the next pivot first: its root and reciprocal run beside the other updates
          x[k + 1] = __builtin_fma(-x[k], lane_value(x[k], k + 1), x[k + 1]);
          pivot(lane_value(x[k + 1], k + 1), root, ip);
        }
#pragma unroll
        for (int c = k + 2; c < DB; ++c) x[c] = __builtin_fma(-x[k], lane_value(x[k], c), x[c]);
        // keeps the updates of column k here (see k_diag16)
#pragma unroll
        for (int c = k + 1; c < DB; ++c) asm volatile("" : "+v"(x[c]));
      }
      __syncthreads();  // every wave has read the diagonal block
      if (live && (w == 0 || !in_diag)) {
#pragma unroll
        for (int c = 0; c < DB; ++c) row[c] = (in_diag && c > lane) ? 0.0 : x[c];
      }
    }
    __syncthreads();
    // trailing lower triangle, one 16 x 16 block per wave at a time
    const int m16 = (TB - b0 - DB) / 16;
    for (int t = w; t < m16 * (m16 + 1) / 2; t += NT / 64) {
      int bi = 0;
      while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
      const int r0 = b0 + DB + 16 * bi, c0 = b0 + DB + 16 * (t - bi * (bi + 1) / 2);
      const double* pa = A + (r0 + l16) * DLD + b0 + lh;
      const double* pb = A + (c0 + l16) * DLD + b0 + lh;
      dv4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < DB / 4; ++e) acc = Mfma<double>::op(pa[4 * e], pb[4 * e], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + lh + 4 * v, c = c0 + l16;
        if (c <= r) A[r * DLD + c] -= acc[v];
      }
    }
    __syncthreads();
  }
  if (bad && tid == 0) a.status[p] = 1;
  // store L_jj and its log-diagonal
#pragma unroll 16
  for (int idx = tid; idx < TB * TB; idx += NT) {
    const int r = idx >> 7, c = idx & (TB - 1);
    src[(int64_t)r * rj.ld + c] = c <= r ? (T)A[r * DLD + c] : T(0);
  }
  {
    double ls = 0.0;
    if (tid < TB && tid < rj.nvalid) {
      // sqrt(DBL_MAX), 1.340780793e154, is the root of a pivot that was infinite (a variance beyond the range of
      // T): its factor has no finite determinant, and the fit is refused for that
      const double root = A[tid * DLD + tid];
      ls = root < 1.34078079299e154 ? log(root) : INFINITY;
    }
    for (int o = 32; o > 0; o >>= 1) ls += __shfl_xor(ls, o);
    if ((tid & 63) == 0) lsum[tid >> 6] = ls;
  }
  __syncthreads();  // the factor is stored and read before the inverse overwrites it
  if (tid == 0) {
    const double tot = lsum[0] + lsum[1] + lsum[2] + lsum[3];
    a.logdiag[(int64_t)p * a.maxT + a.j] = (a.j >= pd.ld_from) ? tot : 0.0;
  }

  // ---- inverse, diagonal blocks: wave w inverts block w, last column first:
  //   X_jj = 1/L_jj,  X_ij = -X_jj sum_{k=j+1..i} X_ik L_kj
  // lane (i, h) holds row i of X; h takes the terms k = j+1+h, j+3+h, ...
  {
    const int b0 = w * DB, il = lane & 31, h = lane >> 5;
    double* blk = A + b0 * DLD + b0;
    const double rec = 1.0 / blk[il * DLD + il];
    double x[DB];
#pragma unroll
    for (int c = 0; c < DB; ++c) x[c] = 0.0;
#pragma unroll
    for (int jj = DB - 1; jj >= 0; --jj) {
      const double xjj = lane_value(rec, jj);
      double sacc = 0.0;
      const double* col = blk + (jj + 1 + h) * DLD + jj;
#pragma unroll
      for (int k = jj + 1; k < DB; k += 2) {
        // the odd half's last term may lie past the block: its x is zero, its L not read
        const double xv = h ? (k + 1 < DB ? x[k + 1 < DB ? k + 1 : k] : 0.0) : x[k];
        const double lv = k + 1 < DB || h == 0 ? col[(k - jj - 1) * DLD] : 0.0;
        sacc = __builtin_fma(xv, lv, sacc);
      }
      sacc += __shfl_xor(sacc, 32);
      x[jj] = il > jj ? -xjj * sacc : il == jj ? xjj : 0.0;
      asm volatile("" : "+v"(x[jj]));
    }
    wave_sync_lds();  // every lane has read L
    if (h == 0)
#pragma unroll
      for (int c = 0; c < DB; ++c) blk[il * DLD + c] = x[c];
  }
  __syncthreads();
  // ---- inverse, block columns right to left
  for (int jb = DNB - 2; jb >= 0; --jb) {
    const int nb = DNB - 1 - jb;
    for (int t = w; t < 4 * nb; t += NT / 64) {
      const int q = t >> 2, ib = jb + 1 + q, si = (t >> 1) & 1, sj = t & 1;
      const double* pa = A + (ib * DB + 16 * si + l16) * DLD + lh;
      const double* pb = A + lh * DLD + jb * DB + 16 * sj + l16;
      dv4 acc = {0.0, 0.0, 0.0, 0.0};
      for (int k = (jb + 1) * DB; k < (ib + 1) * DB; k += DB)
#pragma unroll
        for (int e = 0; e < DB / 4; ++e) acc = Mfma<double>::op(pa[k + 4 * e], pb[(k + 4 * e) * DLD], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) Tt[(q * DB + 16 * si + lh + 4 * v) * DT_LD + 16 * sj + l16] = acc[v];
    }
    __syncthreads();
    for (int t = w; t < 4 * nb; t += NT / 64) {
      const int q = t >> 2, ib = jb + 1 + q, si = (t >> 1) & 1, sj = t & 1;
      const double* pa = Tt + (q * DB + 16 * si + l16) * DT_LD + lh;
      const double* pb = A + (jb * DB + lh) * DLD + jb * DB + 16 * sj + l16;
      dv4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < DB / 4; ++e) acc = Mfma<double>::op(pa[4 * e], pb[4 * e * DLD], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) A[(ib * DB + 16 * si + lh + 4 * v) * DLD + jb * DB + 16 * sj + l16] = -acc[v];
    }
    __syncthreads();
  }
  T* inv = a.invdiag + pd.invdiag_off + (int64_t)a.j * TB * TB;
#pragma unroll 16
  for (int idx = tid; idx < TB * TB; idx += NT) {
    const int r = idx >> 7, c = idx & (TB - 1);
    inv[idx] = c <= r ? (T)A[r * DLD + c] : T(0);
  }
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
constexpr size_t diag32_lds_bytes = sizeof(double) * (size_t)(TB * DLD + (DNB - 1) * DB * DT_LD);

template <>
void launch_diag<double>(const StepArgs<double>& a, const int32_t* plist, int np, hipStream_t st) {
  if (np <= 0) return;
  if (a.diag32)
    hipLaunchKernelGGL(k_diag32<double>, dim3(np), dim3(NT), diag32_lds_bytes, st, a, plist);
  else
    hipLaunchKernelGGL(k_diag16, dim3(np), dim3(NT), 0, st, a, plist);
}

template <>
void launch_diag<float>(const StepArgs<float>& a, const int32_t* plist, int np, hipStream_t st) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_diag32<float>, dim3(np), dim3(NT), diag32_lds_bytes, st, a, plist);
}

hipError_t diag_init() {
  const hipError_t e = hipFuncSetAttribute((const void*)k_diag32<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)diag32_lds_bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_diag32<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)diag32_lds_bytes);
}

}  // namespace lma
