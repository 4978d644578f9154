// Warm-start network (deep sets) on gfx950: forward, backward and Adam kernels
// and the lma_ds_* C ABI (include/lma_ds.h).
//
// Per-point layers run on the bfloat16 matrix cores (v_mfma_f32_16x16x32_bf16,
// float32 accumulation; lane l supplies row l%16 and eight consecutive k starting at
// 8*(l/16); output register v of lane l is row 4*(l/16)+v, column l%16).  A workgroup
// of 8 wave64 takes 64 points at a time and keeps everything between the features and
// its sums in LDS: the forward pass writes only the bfloat16 features and, per 128
// points, the column sums of the second layer; the backward pass computes both layers
// again from those features and the weights of the forward pass (a product more, and
// no activation of 512 bytes per point goes to memory and back, transposed or not)
// and accumulates all its weight gradients in registers over its points.  Bias, ReLU,
// the per-dataset mean and the head run in float32 on the vector units; every
// reduction has a fixed order, so results do not depend on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "lma_ds.h"
#include "runtime.h"

namespace lma {
namespace ds {

constexpr int W = 256;          // encoder / head width
constexpr int NF = LMA_DS_NFEAT;
constexpr int KF = 32;          // feature dimension padded for the k=32 MFMA
constexpr int NO = LMA_DS_NOUT;
constexpr int TR = 128;         // points per tile
constexpr int TP = 64;          // points a workgroup holds at a time
constexpr int ENT = 512;        // threads of an encoder workgroup: wave w owns units 32 w .. 32 w + 31
constexpr int MAXG = 256;       // workgroups (and partial sums) of the backward pass: one per CU
// row strides in LDS (bfloat16): 16-byte aligned, and 16 rows touch every bank once
constexpr int LU = W + 8;       // rows of units
constexpr int LP = TP + 8;      // rows of points
constexpr int LF = KF + 8;      // rows of features
// parameter offsets (float32 vector)
constexpr int64_t OW1 = 0, OB1 = OW1 + W * NF, OW2 = OB1 + W, OB2 = OW2 + W * W, OW3 = OB2 + W,
                  OB3 = OW3 + W * W, OW4 = OB3 + W, OB4 = OW4 + NO * W, NP = OB4 + NO;
static_assert(NP == LMA_DS_NPARAM, "parameter count");

typedef unsigned short u16;
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));

// round to nearest bfloat16, ties to even
__device__ inline u16 f2bf(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u16)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float bf2f(u16 h) { return __uint_as_float((uint32_t)h << 16); }
__device__ inline bf8 load8(const u16* p) { return __builtin_bit_cast(bf8, *(const uint4*)p); }
__device__ inline f4v mma(bf8 a, bf8 b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ inline uint2 pack4(const u16 (&h)[4]) {
  return make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
}

template <int A, int B>
__device__ inline void zero(f4v (&acc)[A][B]) {
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[a][b] = (f4v){0.f, 0.f, 0.f, 0.f};
}

// Encoder weights as the products read them.  Two copies: a parameter update writes
// the one the last forward pass did not use, so a backward pass that follows it still
// finds the weights its activations came from.
struct Enc {
  u16* W1b;      // [W][KF]  (k >= 17 zero)
  u16* W2b;      // [W][W]
  float* b1;     // [W]
  float* b2;     // [W]
};

struct Net {
  float* P;      // master parameters [NP]
  float* G;      // gradient [NP]
  float* M1;     // Adam first moment
  float* M2;     // Adam second moment
  u16* W2bT;     // [W][W]   transpose of the current W2
  u16* W3b;      // [W][W]
  u16* W4b;      // [NO][W]
};

struct Tiles {
  const int32_t* set;    // tile -> dataset
  const int32_t* valid;  // tile -> valid rows (0..128)
  const int64_t* tbeg;   // dataset -> first tile  [nsets+1]
  const float* ninv;     // dataset -> 1 / n_b
};

struct Acts {
  u16* Fb;         // [N][KF]    features of the last forward pass
  float* pool_part;// [ntiles][W]
  float* pool;     // [nsets][W]
  float* z3;       // [nsets][W]
  float* h3;       // [nsets][W]
  float* out;      // [nsets][NO]
  float* dp;       // [nsets][W]   dLoss/dpool, already divided by n_b
  float* dz3;      // [nsets][W]
  float* dout;     // [nsets][NO]
  float* wpart;    // per-workgroup partials of dW2, dW1, db2, db1
  float* lpart;    // per-dataset loss
};
constexpr int64_t WPART = (int64_t)W * W + W * NF + 2 * W;  // entries of one partial

// ---------------------------------------------------------------------------
// encoder
// ---------------------------------------------------------------------------
// First-layer fragments of a wave: its 32 units as matrix rows, and their biases in
// both output layouts (units along the registers, units along the lanes).
struct L1Frag {
  bf8 w[2];
  float bv[2][4], bc[2];
};
__device__ inline L1Frag load_l1(const Enc& e, int u0, int lane) {
  L1Frag f;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int u = u0 + 16 * s;
    f.w[s] = load8(e.W1b + (int64_t)(u + (lane & 15)) * KF + 8 * (lane >> 4));
    f.bc[s] = e.b1[u + (lane & 15)];
#pragma unroll
    for (int v = 0; v < 4; ++v) f.bv[s][v] = e.b1[u + 4 * (lane >> 4) + v];
  }
  return f;
}

// H1 = relu(F W1^T + b1) of the 64 points in LDS, the wave's 32 units: rows of units
// H [TP][LU], and (TRANS) rows of points HT [W][LP]
template <bool TRANS>
__device__ inline void layer1(const u16* F, const L1Frag& f, u16* H, u16* HT, int u0, int lane) {
  const int l16 = lane & 15, lh = lane >> 4;
#pragma unroll
  for (int ra = 0; ra < TP / 16; ++ra) {
    const bf8 a = load8(F + (16 * ra + l16) * LF + 8 * lh);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const f4v z = (f4v){0.f, 0.f, 0.f, 0.f};
      u16 h[4];
      const f4v t = mma(f.w[s], a, z);  // rows: units, columns: points
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = t[v] + f.bv[s][v];
        h[v] = f2bf(x > 0.f ? x : 0.f);
      }
      *(uint2*)(H + (16 * ra + l16) * LU + u0 + 16 * s + 4 * lh) = pack4(h);
      if constexpr (TRANS) {
        const f4v q = mma(a, f.w[s], z);  // rows: points, columns: units
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float x = q[v] + f.bc[s];
          h[v] = f2bf(x > 0.f ? x : 0.f);
        }
        *(uint2*)(HT + (u0 + 16 * s + l16) * LP + 16 * ra + 4 * lh) = pack4(h);
      }
    }
  }
}

// acc[ra][s] += rows 16 ra of X [TP][LU] (k = 0 .. W-1) times rows u0 + 16 s of Wt [W][W]
__device__ inline void points_times(f4v (&acc)[TP / 16][2], const u16* X, const u16* __restrict__ Wt, int u0, int lane) {
  const int l16 = lane & 15, lh = lane >> 4;
  const u16* w = Wt + (int64_t)(u0 + l16) * W + 8 * lh;
  const u16* x = X + l16 * LU + 8 * lh;
#pragma unroll 2
  for (int k = 0; k < W; k += 32) {
    bf8 b[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) b[s] = load8(w + 16 * s * W + k);
#pragma unroll
    for (int ra = 0; ra < TP / 16; ++ra) {
      const bf8 a = load8(x + 16 * ra * LU + k);
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[ra][s] = mma(a, b[s], acc[ra][s]);
    }
  }
}

// Forward: per 128-point tile the column sums of H2 = relu(H1 W2^T + b2) over the
// valid rows, points in LDS, the second layer's weights in registers for all tiles of
// the workgroup.  Bound: matrix cores and LDS reads about alike.  Measured at 64 sets
// of 4096 points: 342 us in two kernels that stored H1, its transpose and H2; 68 us now.
__global__ __launch_bounds__(ENT) void k_encode(Enc e, Acts a, Tiles tl, const float* __restrict__ feats, int ntiles) {
  __shared__ __align__(16) u16 F[TP * LF];
  __shared__ __align__(16) u16 H[TP * LU];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, u0 = 32 * w, l16 = lane & 15, lh = lane >> 4;
  const L1Frag f1 = load_l1(e, u0, lane);
  bf8 w2[2][W / 32];
  float b2[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    b2[s] = e.b2[u0 + 16 * s + l16];
#pragma unroll
    for (int k = 0; k < W / 32; ++k) w2[s][k] = load8(e.W2b + (int64_t)(u0 + 16 * s + l16) * W + 32 * k + 8 * lh);
  }
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int nvt = tl.valid[t];
    float sum[2] = {0.f, 0.f};
    for (int h = 0; h < TR / TP; ++h) {
      const int nv = nvt - h * TP;
      if (nv <= 0) break;
      const int64_t row0 = (int64_t)t * TR + h * TP;
      {  // four features of a point per thread
        const int r = tid >> 3, k = 4 * (tid & 7);
        u16 q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          q[i] = (r < nv && k + i < NF) ? f2bf(feats[(row0 + r) * NF + k + i]) : (u16)0;
        *(uint2*)(F + r * LF + k) = pack4(q);
        *(uint2*)(a.Fb + (row0 + r) * KF + k) = pack4(q);
      }
      __syncthreads();
      layer1<false>(F, f1, H, nullptr, u0, lane);
      __syncthreads();
      f4v acc[TP / 16][2];
      float cs[2] = {0.f, 0.f};
      zero(acc);
#pragma unroll
      for (int k = 0; k < W / 32; ++k)
#pragma unroll
        for (int ra = 0; ra < TP / 16; ++ra) {
          const bf8 x = load8(H + (16 * ra + l16) * LU + 32 * k + 8 * lh);
#pragma unroll
          for (int s = 0; s < 2; ++s) acc[ra][s] = mma(x, w2[s][k], acc[ra][s]);
        }
#pragma unroll
      for (int ra = 0; ra < TP / 16; ++ra)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float z = acc[ra][s][v] + b2[s];
            if (16 * ra + 4 * lh + v < nv && z > 0.f) cs[s] += z;
          }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        cs[s] += __shfl_xor(cs[s], 16);
        cs[s] += __shfl_xor(cs[s], 32);
        sum[s] += cs[s];
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (lane < 16) a.pool_part[(int64_t)t * W + u0 + 16 * s + lane] = sum[s];
  }
}

// Backward of the encoder over the 64-point pieces of this workgroup:
//   H1, Z2 again;  dZ2 = bf16(dp [Z2 > 0]) (zero on padding rows);
//   dZ1 = bf16(dZ2 W2) [H1 > 0];  dW2 += dZ2^T H1, dW1 += dZ1^T F, db += column sums.
// A product over the points needs its operands as rows of points, one over the units
// as rows of units, so H1 and dZ2 are held both ways and dZ1 (in H1's place) as rows
// of points.  Bound: matrix cores (832 instructions per 32 points), LDS, and the reads
// of W2 and its transpose from L2 for every piece.  Measured at 64 sets of 4096 points:
// 1420 us for the kernels that read and wrote the activations; 264 us now (the matrix
// instructions alone take 44).
constexpr size_t BWD_LDS = 2 * (size_t)(3 * W * LP + TP * LU + TP * LF + KF * LP);
__global__ __launch_bounds__(ENT) void k_encode_bwd(Enc e, Net net, Acts a, Tiles tl, int npiece) {
  extern __shared__ __align__(16) u16 sm[];
  u16* H1T = sm;             // [W][LP]
  u16* Z2T = H1T + W * LP;   // [W][LP]
  u16* H1 = Z2T + W * LP;    // [TP][LU], then
  u16* Z1T = H1;             // [W][LP]
  u16* Z2 = Z1T + W * LP;    // [TP][LU]
  u16* F = Z2 + TP * LU;     // [TP][LF]
  u16* FT = F + TP * LF;     // [KF][LP]
  static_assert(TP * LU <= W * LP, "H1 fits in dZ1's place");
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, u0 = 32 * w, l16 = lane & 15, lh = lane >> 4;
  const int o0 = 64 * (w >> 1), i0 = 128 * (w & 1);  // the wave's part of dW2
  float b2[2], db2[2] = {0.f, 0.f}, db1[2] = {0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 2; ++s) b2[s] = e.b2[u0 + 16 * s + l16];
  f4v g2[4][8], g1[2][2];
  zero(g2);
  zero(g1);
  const int p0 = (int)((int64_t)npiece * blockIdx.x / gridDim.x), p1 = (int)((int64_t)npiece * (blockIdx.x + 1) / gridDim.x);
  for (int p = p0; p < p1; ++p) {
    const int t = p / (TR / TP), nv = tl.valid[t] - p % (TR / TP) * TP;
    if (nv <= 0) continue;
    {
      const int r = tid >> 3, k = 4 * (tid & 7);
      const uint2 q = *(const uint2*)(a.Fb + ((int64_t)p * TP + r) * KF + k);
      *(uint2*)(F + r * LF + k) = q;
      FT[k * LP + r] = (u16)q.x;
      FT[(k + 1) * LP + r] = (u16)(q.x >> 16);
      FT[(k + 2) * LP + r] = (u16)q.y;
      FT[(k + 3) * LP + r] = (u16)(q.y >> 16);
    }
    const L1Frag f1 = load_l1(e, u0, lane);  // here and not outside: the registers are needed below
    u16 dz[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) dz[s] = f2bf(a.dp[(int64_t)tl.set[t] * W + u0 + 16 * s + l16]);
    __syncthreads();
    layer1<true>(F, f1, H1, H1T, u0, lane);
    __syncthreads();
    f4v acc[TP / 16][2];
    zero(acc);
    points_times(acc, H1, e.W2b, u0, lane);
#pragma unroll
    for (int ra = 0; ra < TP / 16; ++ra)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        u16 q[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * ra + 4 * lh + v;
          const float z = acc[ra][s][v] + b2[s];
          q[v] = (r < nv && f2bf(z > 0.f ? z : 0.f) != 0) ? dz[s] : (u16)0;
          Z2[r * LU + u0 + 16 * s + l16] = q[v];
          db2[s] += bf2f(q[v]);
        }
        *(uint2*)(Z2T + (u0 + 16 * s + l16) * LP + 16 * ra + 4 * lh) = pack4(q);
      }
    __syncthreads();
    zero(acc);
    points_times(acc, Z2, net.W2bT, u0, lane);
#pragma unroll
    for (int ra = 0; ra < TP / 16; ++ra)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint2 hq = *(const uint2*)(H1T + (u0 + 16 * s + l16) * LP + 16 * ra + 4 * lh);
        const u16 h[4] = {(u16)hq.x, (u16)(hq.x >> 16), (u16)hq.y, (u16)(hq.y >> 16)};
        u16 q[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          q[v] = h[v] != 0 ? f2bf(acc[ra][s][v]) : (u16)0;
          db1[s] += bf2f(q[v]);
        }
        *(uint2*)(Z1T + (u0 + 16 * s + l16) * LP + 16 * ra + 4 * lh) = pack4(q);
      }
#pragma unroll
    for (int k = 0; k < TP; k += 32) {
      bf8 x[4];
#pragma unroll
      for (int ra = 0; ra < 4; ++ra) x[ra] = load8(Z2T + (o0 + 16 * ra + l16) * LP + k + 8 * lh);
#pragma unroll
      for (int rb = 0; rb < 8; ++rb) {
        const bf8 y = load8(H1T + (i0 + 16 * rb + l16) * LP + k + 8 * lh);
#pragma unroll
        for (int ra = 0; ra < 4; ++ra) g2[ra][rb] = mma(x[ra], y, g2[ra][rb]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TP; k += 32)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bf8 x = load8(Z1T + (u0 + 16 * s + l16) * LP + k + 8 * lh);
#pragma unroll
        for (int c = 0; c < 2; ++c) g1[s][c] = mma(x, load8(FT + (16 * c + l16) * LP + k + 8 * lh), g1[s][c]);
      }
    __syncthreads();  // FT and dZ1 are read before the next piece overwrites them
  }
  float* part = a.wpart + blockIdx.x * WPART;
#pragma unroll
  for (int ra = 0; ra < 4; ++ra)
#pragma unroll
    for (int rb = 0; rb < 8; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[(o0 + 16 * ra + 4 * lh + v) * W + i0 + 16 * rb + l16] = g2[ra][rb][v];
  part += W * W;
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (16 * c + l16 < NF) part[(u0 + 16 * s + 4 * lh + v) * NF + 16 * c + l16] = g1[s][c][v];
  part += W * NF;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    db2[s] += __shfl_xor(db2[s], 16);
    db2[s] += __shfl_xor(db2[s], 32);
    db1[s] += __shfl_xor(db1[s], 16);
    db1[s] += __shfl_xor(db1[s], 32);
    if (lane < 16) {
      part[u0 + 16 * s + lane] = db2[s];
      part[W + u0 + 16 * s + lane] = db1[s];
    }
  }
}

// Sums of the partials in workgroup order -> dW2, dW1, db2, db1.  64 entries per
// workgroup; its four waves take a quarter of the partials each, eight loads in flight.
__global__ __launch_bounds__(256) void k_wgrad_reduce(Net net, Acts a, int npart) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  const int c0 = npart * w / 4, c1 = npart * (w + 1) / 4;
  float s = 0.f;
  if (e < WPART) {
    const float* p = a.wpart + e;
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p[(c + j) * WPART];
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; c < c1; ++c) s += p[c * WPART];
  }
  red[w][lane] = s;
  __syncthreads();
  if (w > 0 || e >= WPART) return;
  s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
  constexpr int64_t n2 = (int64_t)W * W, n1 = n2 + W * NF;
  const int64_t at = e < n2 ? OW2 + e : e < n1 ? OW1 + e - n2 : e < n1 + W ? OB2 + e - n1 : OB1 + e - n1 - W;
  net.G[at] = s;
}

// ---------------------------------------------------------------------------
// head
// ---------------------------------------------------------------------------
// mean over each dataset's tiles (in tile order), then the head in float32
__global__ __launch_bounds__(256) void k_head(Net net, Acts a, Tiles tl, float* __restrict__ out) {
  __shared__ float sp[W], sh[W];
  const int b = blockIdx.x, i = threadIdx.x;
  float s = 0.f;
#pragma unroll 8
  for (int64_t t = tl.tbeg[b]; t < tl.tbeg[b + 1]; ++t) s += a.pool_part[t * W + i];
  const float p = s * tl.ninv[b];
  a.pool[(int64_t)b * W + i] = p;
  sp[i] = p;
  __syncthreads();
  float z = net.P[OB3 + i];
#pragma unroll 4
  for (int k = 0; k < W; k += 8) {
    const uint4 q = *(const uint4*)(net.W3b + i * W + k);
    const uint32_t qw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) z += bf2f((u16)(qw[j >> 1] >> (16 * (j & 1)))) * sp[k + j];
  }
  a.z3[(int64_t)b * W + i] = z;
  const float h = z > 0.f ? z : 0.f;
  a.h3[(int64_t)b * W + i] = h;
  sh[i] = h;
  __syncthreads();
  if (i < NO) {
    float o = net.P[OB4 + i];
#pragma unroll 4
    for (int k = 0; k < W; k += 8) {
      const uint4 q = *(const uint4*)(net.W4b + i * W + k);
      const uint32_t qw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) o += bf2f((u16)(qw[j >> 1] >> (16 * (j & 1)))) * sh[k + j];
    }
    a.out[(int64_t)b * NO + i] = o;
    out[(int64_t)b * NO + i] = o;
  }
}

// per dataset: output gradient of the masked MSE, the head's layer gradients, and
// dLoss/dpool / n_b
__global__ __launch_bounds__(256) void k_head_bwd(Net net, Acts a, Tiles tl, const float* __restrict__ labels,
                                                  const float* __restrict__ masks, int nsets) {
  __shared__ float sdo[NO], sdz[W];
  const int b = blockIdx.x, i = threadIdx.x;
  if (i == 0) {
    float cnt = 0.f, l = 0.f;
    for (int j = 0; j < NO; ++j) cnt += masks[b * NO + j];
    for (int j = 0; j < NO; ++j) {
      const float r = (a.out[b * NO + j] - labels[b * NO + j]) * masks[b * NO + j];
      sdo[j] = 2.f * r / cnt / (float)nsets;
      l += r * r;
    }
    a.lpart[b] = l / cnt / (float)nsets;
  }
  __syncthreads();
  if (i < NO) a.dout[b * NO + i] = sdo[i];
  float dh = 0.f;
  for (int j = 0; j < NO; ++j) dh += bf2f(net.W4b[j * W + i]) * sdo[j];
  const float dz = a.z3[(int64_t)b * W + i] > 0.f ? dh : 0.f;
  sdz[i] = dz;
  a.dz3[(int64_t)b * W + i] = dz;
  __syncthreads();
  float dpv = 0.f;
#pragma unroll 16
  for (int r = 0; r < W; ++r) dpv += bf2f(net.W3b[r * W + i]) * sdz[r];
  a.dp[(int64_t)b * W + i] = dpv * tl.ninv[b];
}

// head gradients and the loss, summed over the datasets in order; 64 entries of one
// weight row (or of a bias) per wave
__global__ __launch_bounds__(256) void k_head_reduce(Net net, Acts a, int nsets, float* loss) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  constexpr int64_t n3 = (int64_t)W * W, nb3 = n3 + W, n4 = nb3 + NO * W, nh = n4 + NO;
  if (e == nh) {
    float s = 0.f;
    for (int b = 0; b < nsets; ++b) s += a.lpart[b];
    *loss = s;
  }
  if (e >= nh) return;
  const float* x;
  const float* y = nullptr;
  int64_t lx = W;
  if (e < n3) {
    x = a.dz3 + e / W;
    y = a.pool + e % W;
  } else if (e < nb3) {
    x = a.dz3 + (e - n3);
  } else if (e < n4) {
    x = a.dout + (e - nb3) / W;
    lx = NO;
    y = a.h3 + (e - nb3) % W;
  } else {
    x = a.dout + (e - n4);
    lx = NO;
  }
  float s = 0.f;
#pragma unroll 8
  for (int b = 0; b < nsets; ++b) s += y ? x[b * lx] * y[(int64_t)b * W] : x[b * lx];
  net.G[OW3 + e] = s;  // W3, b3, W4, b4 are contiguous in the parameter vector
}

// ---------------------------------------------------------------------------
// Adam and the weight copies the products read
// ---------------------------------------------------------------------------
// value v of parameter e into its copies
__device__ inline void put_copy(const Net& net, const Enc& c, int64_t e, float v) {
  if (e < OB1) {
    const int i = (int)(e / NF), k = (int)(e - (int64_t)i * NF);
    c.W1b[i * KF + k] = f2bf(v);
  } else if (e < OW2) {
    c.b1[e - OB1] = v;
  } else if (e < OB2) {
    const int64_t q = e - OW2;
    const u16 h = f2bf(v);
    c.W2b[q] = h;
    net.W2bT[(q % W) * W + q / W] = h;
  } else if (e < OW3) {
    c.b2[e - OB2] = v;
  } else if (e < OB3) {
    net.W3b[e - OW3] = f2bf(v);
  } else if (e >= OW4 && e < OB4) {
    net.W4b[e - OW4] = f2bf(v);
  }
}

__global__ void k_adam(Net net, Enc c, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= NP) return;
  const float g = net.G[e];
  const float m = b1 * net.M1[e] + (1.f - b1) * g;
  const float v = b2 * net.M2[e] + (1.f - b2) * g * g;
  net.M1[e] = m;
  net.M2[e] = v;
  const float p = net.P[e] - lr * (m / c1) / (sqrtf(v / c2) + eps);
  net.P[e] = p;
  put_copy(net, c, e, p);
}

__global__ void k_shadow(Net net, Enc c) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < NP) put_copy(net, c, e, net.P[e]);
}

// ---------------------------------------------------------------------------
// features of one dataset
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_ystats(const double* __restrict__ y, int64_t n, double* stats) {
  __shared__ double r1[256], r2[256];
  const int tid = threadIdx.x;
  double s = 0.0;
  for (int64_t i = tid; i < n; i += 256) s += y[i];
  r1[tid] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (tid < k) r1[tid] += r1[tid + k];
    __syncthreads();
  }
  const double mean = r1[0] / (double)n;
  double q = 0.0;
  for (int64_t i = tid; i < n; i += 256) q += (y[i] - mean) * (y[i] - mean);
  r2[tid] = q;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (tid < k) r2[tid] += r2[tid + k];
    __syncthreads();
  }
  if (tid == 0) {
    stats[0] = mean;
    stats[1] = 1.0 / sqrt(r2[0] / (double)n);
  }
}

__global__ void k_features(const double* __restrict__ X, const double* __restrict__ y, int64_t n, int d,
                           const double* __restrict__ stats, float* __restrict__ F) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * NF) return;
  const int64_t i = e / NF;
  const int k = (int)(e - i * NF);
  float v;
  if (k < 8) v = k < d ? (float)X[i * d + k] : 0.f;
  else if (k == 8) v = (float)((y[i] - stats[0]) * stats[1]);
  else v = (k - 9) < d ? 1.f : 0.f;
  F[e] = v;
}

}  // namespace ds
}  // namespace lma

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
using namespace lma;
using namespace lma::ds;
using lmart::Err;

struct lma_ds {
  int64_t max_rows = 0, max_sets = 0;
  char* mem = nullptr;
  Net net{};
  Enc enc[2]{};
  int cur = 0, fwd = 0;  // copies of the current parameters and of the last forward pass
  Acts act{};
  int32_t* d_set = nullptr;
  int32_t* d_valid = nullptr;
  int64_t* d_tbeg = nullptr;
  float* d_ninv = nullptr;
  float* d_loss = nullptr;
  double* d_stats = nullptr;
  int64_t nsets = 0, ntiles = 0, rows = 0;
  int64_t step = 0;
  bool have_fwd = false;
  // the copy a parameter update may overwrite, current from then on
  Enc& next_copy() {
    if (have_fwd) cur = 1 - fwd;
    return enc[cur];
  }
  std::vector<int32_t> h_set, h_valid;
  std::vector<int64_t> h_tbeg;
  std::vector<float> h_ninv;
  ~lma_ds() {
    if (mem) (void)hipFree(mem);
  }
};

namespace {

inline int64_t al(int64_t b) { return (b + 255) / 256 * 256; }
inline unsigned nb(int64_t n) { return (unsigned)((n + 255) / 256); }

template <class F>
lma_status guard(F&& f) {
  lmart::set_last_error("");
  try {
    f();
    return LMA_OK;
  } catch (const Err& e) {
    lmart::set_last_error(e.msg);
    return e.st;
  } catch (const std::bad_alloc&) {
    lmart::set_last_error("host allocation failed");
    return LMA_E_NOMEM;
  } catch (const std::exception& e) {
    lmart::set_last_error(std::string("internal error: ") + e.what());
    return LMA_E_INTERNAL;
  }
}

}  // namespace

extern "C" {

lma_status lma_ds_create(int64_t max_rows, int64_t max_sets, lma_ds** out) {
  return guard([&] {
    if (!out) throw Err{LMA_E_ARG, "out is NULL"};
    *out = nullptr;
    if (max_rows < TR || max_sets < 1) throw Err{LMA_E_ARG, "need max_rows >= 128 and max_sets >= 1"};
    std::unique_ptr<lma_ds> s(new lma_ds());
    const int64_t N = (max_rows + TR - 1) / TR * TR;
    const int64_t nt = N / TR, npart = std::min<int64_t>(MAXG, N / TP);
    s->max_rows = N;
    s->max_sets = max_sets;
    int64_t off = 0;
    auto take = [&](int64_t bytes) {
      const int64_t o = off;
      off += al(bytes);
      return o;
    };
    const int64_t oP = take(4 * NP), oG = take(4 * NP), oM1 = take(4 * NP), oM2 = take(4 * NP);
    const int64_t oW2T = take(2 * W * W), oW3 = take(2 * W * W), oW4 = take(2 * NO * W);
    int64_t oE[2][4];
    for (auto& e : oE) {
      e[0] = take(2 * W * KF);
      e[1] = take(2 * W * W);
      e[2] = take(4 * W);
      e[3] = take(4 * W);
    }
    const int64_t oFb = take(2 * KF * N);
    const int64_t oPP = take(4 * nt * W), oPool = take(4 * max_sets * W), oZ3 = take(4 * max_sets * W),
                  oH3 = take(4 * max_sets * W), oOut = take(4 * max_sets * NO), oDp = take(4 * max_sets * W),
                  oDz = take(4 * max_sets * W), oDo = take(4 * max_sets * NO);
    const int64_t oWp = take(4 * npart * WPART), oLp = take(4 * max_sets);
    const int64_t oSet = take(4 * nt), oVal = take(4 * nt), oTb = take(8 * (max_sets + 1)), oNi = take(4 * max_sets),
                  oLoss = take(8), oStats = take(16);
    void* mem = nullptr;
    if (hipMalloc(&mem, off) != hipSuccess || !mem) {
      (void)hipGetLastError();
      throw Err{LMA_E_NOMEM, "device allocation of the network workspace failed"};
    }
    s->mem = (char*)mem;
    char* b = s->mem;
    HIPCHK(hipMemset(b, 0, off));
    s->net = Net{(float*)(b + oP), (float*)(b + oG), (float*)(b + oM1), (float*)(b + oM2),
                 (u16*)(b + oW2T), (u16*)(b + oW3), (u16*)(b + oW4)};
    for (int i = 0; i < 2; ++i)
      s->enc[i] = Enc{(u16*)(b + oE[i][0]), (u16*)(b + oE[i][1]), (float*)(b + oE[i][2]), (float*)(b + oE[i][3])};
    HIPCHK(hipFuncSetAttribute((const void*)k_encode_bwd, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BWD_LDS));
    Acts& a = s->act;
    a.Fb = (u16*)(b + oFb);
    a.pool_part = (float*)(b + oPP);
    a.pool = (float*)(b + oPool);
    a.z3 = (float*)(b + oZ3);
    a.h3 = (float*)(b + oH3);
    a.out = (float*)(b + oOut);
    a.dp = (float*)(b + oDp);
    a.dz3 = (float*)(b + oDz);
    a.dout = (float*)(b + oDo);
    a.wpart = (float*)(b + oWp);
    a.lpart = (float*)(b + oLp);
    s->d_set = (int32_t*)(b + oSet);
    s->d_valid = (int32_t*)(b + oVal);
    s->d_tbeg = (int64_t*)(b + oTb);
    s->d_ninv = (float*)(b + oNi);
    s->d_loss = (float*)(b + oLoss);
    s->d_stats = (double*)(b + oStats);
    *out = s.release();
  });
}

void lma_ds_free(lma_ds* ds) { delete ds; }

lma_status lma_ds_set_params(lma_ds* ds, const float* params) {
  return guard([&] {
    if (!ds || !params) throw Err{LMA_E_ARG, "NULL argument"};
    HIPCHK(hipMemcpy(ds->net.P, params, 4 * NP, hipMemcpyHostToDevice));
    HIPCHK(hipMemset(ds->net.M1, 0, 4 * NP));
    HIPCHK(hipMemset(ds->net.M2, 0, 4 * NP));
    hipLaunchKernelGGL(k_shadow, dim3(nb(NP)), dim3(256), 0, 0, ds->net, ds->next_copy());
    HIPCHK(hipGetLastError());
    HIPCHK(hipDeviceSynchronize());
    ds->step = 0;
  });
}

lma_status lma_ds_get_params(lma_ds* ds, float* params) {
  return guard([&] {
    if (!ds || !params) throw Err{LMA_E_ARG, "NULL argument"};
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMemcpy(params, ds->net.P, 4 * NP, hipMemcpyDeviceToHost));
  });
}

lma_status lma_ds_features(lma_ds* ds, const double* X, const double* y, int64_t n, int32_t d, float* feats,
                           hipStream_t st) {
  return guard([&] {
    if (!ds || !X || !y || !feats) throw Err{LMA_E_ARG, "NULL argument"};
    if (n < 2 || d < 1 || d > 8) throw Err{LMA_E_ARG, "need n >= 2 and 1 <= d <= 8"};
    hipLaunchKernelGGL(k_ystats, dim3(1), dim3(256), 0, st, y, n, ds->d_stats);
    hipLaunchKernelGGL(k_features, dim3(nb(n * NF)), dim3(256), 0, st, X, y, n, (int)d, ds->d_stats, feats);
    HIPCHK(hipGetLastError());
  });
}

lma_status lma_ds_forward(lma_ds* ds, int64_t nsets, const int64_t* set_ptr, const int64_t* set_n,
                          const float* feats, float* out, hipStream_t st) {
  return guard([&] {
    if (!ds || !set_ptr || !set_n || !feats || !out) throw Err{LMA_E_ARG, "NULL argument"};
    if (nsets < 1 || nsets > ds->max_sets) throw Err{LMA_E_ARG, "nsets out of range"};
    if (set_ptr[0] != 0) throw Err{LMA_E_ARG, "set_ptr[0] must be 0"};
    for (int64_t b = 0; b < nsets; ++b) {
      if (set_ptr[b] % TR) throw Err{LMA_E_ARG, "set_ptr entries must be multiples of 128"};
      if (set_n[b] < 1 || set_ptr[b] + set_n[b] > set_ptr[b + 1])
        throw Err{LMA_E_ARG, "each set needs 1 <= set_n[b] <= set_ptr[b+1] - set_ptr[b]"};
    }
    const int64_t rows = (set_ptr[nsets] + TR - 1) / TR * TR;
    if (rows > ds->max_rows) throw Err{LMA_E_ARG, "more rows than the workspace holds"};
    ds->h_set.clear();
    ds->h_valid.clear();
    ds->h_tbeg.assign(nsets + 1, 0);
    ds->h_ninv.assign(nsets, 0.f);
    for (int64_t b = 0; b < nsets; ++b) {
      ds->h_tbeg[b] = (int64_t)ds->h_set.size();
      const int64_t nt = (set_ptr[b + 1] - set_ptr[b] + TR - 1) / TR;
      for (int64_t t = 0; t < nt; ++t) {
        ds->h_set.push_back((int32_t)b);
        const int64_t v = set_n[b] - t * TR;
        ds->h_valid.push_back((int32_t)(v < 0 ? 0 : (v > TR ? TR : v)));
      }
      ds->h_ninv[b] = 1.0f / (float)set_n[b];
    }
    ds->h_tbeg[nsets] = (int64_t)ds->h_set.size();
    const int64_t ntiles = (int64_t)ds->h_set.size();
    if (ntiles * TR != rows) throw Err{LMA_E_ARG, "set_ptr[nsets] must be a multiple of 128"};
    HIPCHK(hipMemcpyAsync(ds->d_set, ds->h_set.data(), 4 * ntiles, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(ds->d_valid, ds->h_valid.data(), 4 * ntiles, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(ds->d_tbeg, ds->h_tbeg.data(), 8 * (nsets + 1), hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(ds->d_ninv, ds->h_ninv.data(), 4 * nsets, hipMemcpyHostToDevice, st));
    ds->nsets = nsets;
    ds->ntiles = ntiles;
    ds->rows = rows;
    Tiles tl{ds->d_set, ds->d_valid, ds->d_tbeg, ds->d_ninv};
    const Acts& a = ds->act;
    // two workgroups fit on a CU
    hipLaunchKernelGGL(k_encode, dim3((unsigned)std::min<int64_t>(ntiles, 512)), dim3(ENT), 0, st, ds->enc[ds->cur], a, tl,
                       feats, (int)ntiles);
    hipLaunchKernelGGL(k_head, dim3(nsets), dim3(256), 0, st, ds->net, a, tl, out);
    HIPCHK(hipGetLastError());
    ds->fwd = ds->cur;
    ds->have_fwd = true;
  });
}

lma_status lma_ds_backward(lma_ds* ds, const float* labels, const float* masks, float* grad, double* loss,
                           hipStream_t st) {
  return guard([&] {
    if (!ds || !labels || !masks) throw Err{LMA_E_ARG, "NULL argument"};
    if (!ds->have_fwd) throw Err{LMA_E_ARG, "lma_ds_backward needs a preceding lma_ds_forward"};
    Tiles tl{ds->d_set, ds->d_valid, ds->d_tbeg, ds->d_ninv};
    const Acts& a = ds->act;
    const int nsets = (int)ds->nsets;
    const int64_t nh = (int64_t)W * W + W + NO * W + NO;
    hipLaunchKernelGGL(k_head_bwd, dim3(nsets), dim3(256), 0, st, ds->net, a, tl, labels, masks, nsets);
    hipLaunchKernelGGL(k_head_reduce, dim3(nb(nh + 1)), dim3(256), 0, st, ds->net, a, nsets, ds->d_loss);
    const int npiece = (int)(ds->rows / TP), npart = std::min(MAXG, npiece);
    hipLaunchKernelGGL(k_encode_bwd, dim3(npart), dim3(ENT), BWD_LDS, st, ds->enc[ds->fwd], ds->net, a, tl, npiece);
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((WPART + 63) / 64)), dim3(256), 0, st, ds->net, a, npart);
    HIPCHK(hipGetLastError());
    if (grad) HIPCHK(hipMemcpyAsync(grad, ds->net.G, 4 * NP, hipMemcpyDeviceToDevice, st));
    if (loss) {
      float l = 0.f;
      HIPCHK(hipMemcpyAsync(&l, ds->d_loss, 4, hipMemcpyDeviceToHost, st));
      HIPCHK(hipStreamSynchronize(st));
      *loss = l;
    }
  });
}

lma_status lma_ds_adam(lma_ds* ds, float lr, float beta1, float beta2, float eps, hipStream_t st) {
  return guard([&] {
    if (!ds) throw Err{LMA_E_ARG, "NULL argument"};
    ds->step += 1;
    const float c1 = 1.f - std::pow(beta1, (float)ds->step), c2 = 1.f - std::pow(beta2, (float)ds->step);
    hipLaunchKernelGGL(k_adam, dim3(nb(NP)), dim3(256), 0, st, ds->net, ds->next_copy(), lr, beta1, beta2, eps, c1, c2);
    HIPCHK(hipGetLastError());
  });
}

}  // extern "C"
