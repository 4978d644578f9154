// k-means steps of the block partitioner on gfx950 (include/lma_part.h).
//
// Nearest-centre assignment: one thread per point.  The centres are read with
// wave-uniform loads (every lane of a wave reads the same centre entry), eight
// centres per pass, so a lane keeps eight running sums in registers and reads
// each of its point's coordinates once per pass.  Each distance is summed over
// the coordinates in increasing order with separately rounded products and
// sums (contraction into fused multiply-adds is switched off), so the result
// is the same bit for bit as any plain evaluation in that order.  With few points
// (SPLIT_N) that is less than a workgroup per CU or a few, so the four waves of a
// workgroup take the same 64 points and a quarter of the passes each, and the
// smallest (distance, index) of the four wins.
//
// Centre update: the points are cut into chunks of 4096 consecutive indices.
// A workgroup takes one chunk and eight centres, lists the chunk's points of each
// of them in increasing index, and one thread per (centre, coordinate) adds its
// list in that order; a second kernel adds the chunk sums in chunk order and
// divides once by the count.  Every sum has a fixed order, so the update does
// not depend on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <vector>

#include "lma_part.h"
#include "misc.h"
#include "runtime.h"

namespace lma {
namespace part {

constexpr int NTA = 256;   // threads per workgroup, assignment
constexpr int CG = 8;      // centres per pass
constexpr int NTU = 64;    // threads per workgroup, combine
constexpr int CU = 8;      // centres per workgroup of the chunk sums
constexpr int64_t SPLIT_N = 262144;  // four workgroups of 256 points per CU
constexpr int MAX_K = 65536;
constexpr int64_t CHUNK = 4096;         // points per partial sum of the update
constexpr int64_t PART_BYTES = 1ll << 30;  // partial sums held at once

// Scratch of the allocation-free centre update (lma_kmeans_update_noalloc):
// one copy per GPU, held until the process ends.  Host code never passes the
// symbol itself to a kernel (on the host it is only a stand-in); it uses the
// device address that hipGetSymbolAddress returns for the current device.
constexpr int64_t NOALLOC_BYTES = 16ll << 20;
static __device__ __align__(256) char scratch[NOALLOC_BYTES];

// Measured at n=65536, k=64, d=8: 41 us whole, 14 us split.
template <bool SPLIT>
__global__ __launch_bounds__(NTA) void k_km_assign(const double* __restrict__ P, int64_t n, int d,
                                                   const double* __restrict__ C, int k, int32_t* __restrict__ label,
                                                   double* __restrict__ dist2) {
#pragma clang fp contract(off)
  const int w = SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int64_t i = SPLIT ? (int64_t)blockIdx.x * 64 + (threadIdx.x & 63) : (int64_t)blockIdx.x * NTA + threadIdx.x;
  if (!SPLIT && i >= n) return;
  const double* p = P + (i < n ? i : 0) * d;
  double best = INFINITY;
  int arg = 0;
  for (int c0 = w * CG; c0 < k; c0 += SPLIT ? 4 * CG : CG) {
    const int nc = k - c0 < CG ? k - c0 : CG;
    double acc[CG];
#pragma unroll
    for (int j = 0; j < CG; ++j) acc[j] = 0.0;
    const double* cb = C + (int64_t)c0 * d;
    for (int t = 0; t < d; ++t) {
      const double x = p[t];
#pragma unroll
      for (int j = 0; j < CG; ++j) {
        if (j < nc) {
          const double df = x - cb[j * d + t];
          const double sq = df * df;
          acc[j] = acc[j] + sq;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < CG; ++j)
      if (j < nc && acc[j] < best) {
        best = acc[j];
        arg = c0 + j;
      }
  }
  if constexpr (SPLIT) {
    // a wave that found no finite distance holds (+inf, 0): it wins only if every
    // wave holds it, which is the plain result for a point without one
    __shared__ double sb[4][64];
    __shared__ int sa[4][64];
    sb[w][threadIdx.x & 63] = best;
    sa[w][threadIdx.x & 63] = arg;
    __syncthreads();
    if (w > 0 || i >= n) return;
    for (int q = 1; q < 4; ++q) {
      const double v = sb[q][threadIdx.x];
      const int c = sa[q][threadIdx.x];
      if (v < best || (v == best && v < INFINITY && c < arg)) {
        best = v;
        arg = c;
      }
    }
  }
  label[i] = arg;
  if (dist2) dist2[i] = best;
}

// Sums of one chunk for CU centres.  Bound: the reads of the labels and the rows.
// Walking the chunk's labels once per 64 (centre, coordinate) pairs took 210 us at
// n=65536, k=64, d=8; the lists take 14 us.
__global__ __launch_bounds__(256) void k_km_partial(const double* __restrict__ P, int64_t n, int d,
                                                    const int32_t* __restrict__ label, int k, int64_t ch0,
                                                    int64_t nbx, int64_t b0, double* __restrict__ part,
                                                    int64_t* __restrict__ pcnt) {
  static_assert(CHUNK == 16 * 256 && CU == 8, "16 points per thread, eight 16-bit counters in two words");
  __shared__ __align__(16) uint8_t lab[CHUNK];  // centre of each point relative to c0, 255: another
  __shared__ uint16_t list[CHUNK];              // point offsets, by centre, in increasing order
  __shared__ uint64_t wsum[2][4];
  __shared__ int base[CU + 1];
  // block b (b0 and on) covers chunk ch0 + b / nbx and centres (b % nbx) * CU + 0..7
  const int64_t b = b0 + blockIdx.x, g = b / nbx;
  const int c0 = (int)(b - g * nbx) * CU;
  const int nc = k - c0 < CU ? k - c0 : CU;
  const int64_t i0 = (ch0 + g) * CHUNK;
  const int m = (int)(n - i0 < CHUNK ? n - i0 : CHUNK);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int o = j * 256 + tid;
    const uint32_t l = o < m ? (uint32_t)label[i0 + o] - (uint32_t)c0 : 255u;
    lab[o] = l < (uint32_t)nc ? (uint8_t)l : (uint8_t)255;
  }
  __syncthreads();
  // counts of this thread's 16 consecutive points: centre l in bits 16 (l % 4) of cnt[l / 4]
  const uint4 q4 = *(const uint4*)(lab + 16 * tid);
  const uint32_t qw[4] = {q4.x, q4.y, q4.z, q4.w};
  uint64_t cnt[2] = {0, 0};
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t l = (qw[j >> 2] >> (8 * (j & 3))) & 255u;
    if (l < 8) cnt[l >> 2] += 1ull << (16 * (l & 3));
  }
  // inclusive scan over the threads
  uint64_t inc[2] = {cnt[0], cnt[1]};
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t a = __shfl_up(inc[0], o), b = __shfl_up(inc[1], o);
    if (lane >= o) {
      inc[0] += a;
      inc[1] += b;
    }
  }
  if (lane == 63) {
    wsum[0][w] = inc[0];
    wsum[1][w] = inc[1];
  }
  __syncthreads();
  uint64_t tot[2] = {0, 0};
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (q < w) inc[h] += wsum[h][q];
      tot[h] += wsum[h][q];
    }
  if (tid <= CU) {
    int b = 0;
    for (int l = 0; l < tid; ++l) b += (int)((tot[l >> 2] >> (16 * (l & 3))) & 0xffffu);
    base[tid] = b;
  }
  __syncthreads();
  uint64_t pos[2] = {inc[0] - cnt[0], inc[1] - cnt[1]};
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t l = (qw[j >> 2] >> (8 * (j & 3))) & 255u;
    if (l < 8) {
      const int sh = 16 * (l & 3);
      list[base[l] + (int)((pos[l >> 2] >> sh) & 0xffffu)] = (uint16_t)(16 * tid + j);
      pos[l >> 2] += 1ull << sh;
    }
  }
  __syncthreads();
  for (int e = tid; e < nc * d; e += 256) {
    const int c = e / d, t = e - c * d;
    const double* col = P + i0 * d + t;
    double s = 0.0;
    int q = base[c];
    const int q1 = base[c + 1];
    for (; q + 8 <= q1; q += 8) {
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = col[(int)list[q + j] * d];
#pragma unroll
      for (int j = 0; j < 8; ++j) s = s + v[j];
    }
    for (; q < q1; ++q) s = s + col[(int)list[q] * d];
    part[g * (int64_t)k * d + (int64_t)c0 * d + e] = s;
  }
  if (tid < nc) pcnt[g * k + c0 + tid] = base[tid + 1] - base[tid];
}

__global__ __launch_bounds__(NTU) void k_km_combine(const double* __restrict__ part, const int64_t* __restrict__ pcnt,
                                                    int64_t nch, int k, int d, double* __restrict__ srun,
                                                    int64_t* __restrict__ crun, int first, int last,
                                                    double* __restrict__ C, int64_t* __restrict__ count) {
  const int64_t kd = (int64_t)k * d;
  const int64_t e = (int64_t)blockIdx.x * NTU + threadIdx.x;
  if (e >= kd) return;
  const int c = (int)(e / d), t = (int)(e - (int64_t)c * d);
  double s = first ? 0.0 : srun[e];
  int64_t cnt = first ? 0 : crun[e];
  for (int64_t g = 0; g < nch; ++g) {
    s = s + part[g * kd + e];
    cnt += pcnt[g * k + c];
  }
  if (!last) {
    srun[e] = s;
    crun[e] = cnt;
    return;
  }
  if (cnt > 0) C[e] = s / (double)cnt;
  if (count && t == 0) count[c] = cnt;
}

}  // namespace part
}  // namespace lma

namespace {

using lmart::Err;

void check_shape(const double* P, int64_t n, int32_t d, int32_t k) {
  if (n < 0) throw Err{LMA_E_ARG, "n < 0"};
  if (d < 1 || d > lma::MAX_D) throw Err{LMA_E_ARG, "need 1 <= d <= 64"};
  if (k < 1 || k > lma::part::MAX_K) throw Err{LMA_E_ARG, "need 1 <= k <= 65536"};
  if (n > 0 && !P) throw Err{LMA_E_ARG, "P is NULL"};
}

void assign(const double* P, int64_t n, int32_t d, const double* C, int32_t k, int32_t* label, double* dist2,
            hipStream_t st) {
  if (n == 0) return;
  const int64_t nb = (n + lma::part::NTA - 1) / lma::part::NTA;
  if (nb > 0x7fffffff) throw Err{LMA_E_ARG, "too many points"};
  if (n <= lma::part::SPLIT_N && k > lma::part::CG)
    hipLaunchKernelGGL(lma::part::k_km_assign<true>, dim3((unsigned)((n + 63) / 64)), dim3(lma::part::NTA), 0, st, P, n,
                       (int)d, C, (int)k, label, dist2);
  else
    hipLaunchKernelGGL(lma::part::k_km_assign<false>, dim3((unsigned)nb), dim3(lma::part::NTA), 0, st, P, n, (int)d, C,
                       (int)k, label, dist2);
  HIPCHK(hipGetLastError());
}

// Centre update in chunk order.  Chunks are processed in groups of `group`
// chunks whose partial sums sit at the start of the workspace `mem`; running
// sums (after them) carry the order across groups, so the result does not
// depend on the group size.  Returns the launch status; enqueues only.
hipError_t update_launch(const double* P, int64_t n, int32_t d, const int32_t* label, int32_t k, double* C,
                         int64_t* count, int64_t group, char* mem, hipStream_t st) {
  using namespace lma::part;
  const int64_t kd = (int64_t)k * d;
  const int64_t nch = n > 0 ? (n + CHUNK - 1) / CHUNK : 0;
  const int64_t per = (int64_t)sizeof(double) * kd + (int64_t)sizeof(int64_t) * k;
  const int64_t nbx = (kd + NTU - 1) / NTU, nbc = (k + CU - 1) / CU;
  double* part = reinterpret_cast<double*>(mem);
  int64_t* pcnt = reinterpret_cast<int64_t*>(mem + sizeof(double) * group * kd);
  double* srun = reinterpret_cast<double*>(mem + group * per);
  int64_t* crun = reinterpret_cast<int64_t*>(mem + group * per + sizeof(double) * kd);
  hipError_t err = hipSuccess;
  if (nch == 0) {
    hipLaunchKernelGGL(k_km_combine, dim3((unsigned)nbx), dim3(NTU), 0, st, part, pcnt, (int64_t)0, (int)k, (int)d,
                       srun, crun, 1, 1, C, count);
    err = hipGetLastError();
  }
  for (int64_t ch0 = 0; ch0 < nch && err == hipSuccess; ch0 += group) {
    const int64_t ng = std::min<int64_t>(group, nch - ch0);
    // a launch holds less than 2^32 threads
    for (int64_t b = 0; b < ng * nbc && err == hipSuccess; b += 0xffffff) {
      const dim3 blocks((unsigned)std::min<int64_t>(ng * nbc - b, 0xffffff));
      hipLaunchKernelGGL(k_km_partial, blocks, dim3(256), 0, st, P, n, (int)d, label, (int)k, ch0, nbc, b, part, pcnt);
      err = hipGetLastError();
    }
    if (err != hipSuccess) break;
    hipLaunchKernelGGL(k_km_combine, dim3((unsigned)nbx), dim3(NTU), 0, st, part, pcnt, ng, (int)k, (int)d, srun,
                       crun, ch0 == 0 ? 1 : 0, ch0 + ng >= nch ? 1 : 0, C, count);
    err = hipGetLastError();
  }
  return err;
}

// Bytes of partial sums per chunk, and of the running sums.
int64_t update_per_chunk(int32_t d, int32_t k) {
  return (int64_t)sizeof(double) * k * d + (int64_t)sizeof(int64_t) * k;
}
int64_t update_running(int32_t d, int32_t k) {
  return (int64_t)(sizeof(double) + sizeof(int64_t)) * k * d;
}

void check_launch_size(int64_t group, int32_t d, int32_t k) {
  const int64_t nbx = ((int64_t)k + lma::part::CU - 1) / lma::part::CU;
  if (group * nbx > 0x7fffffff) throw Err{LMA_E_ARG, "too many centres x coordinates for one launch"};
}

// `rounds` times (assign to label, then) the update, with one workspace from the
// library's device cache (partial sums of at most PART_BYTES at once), returned
// after a stream synchronisation.
void update(const double* P, int64_t n, int32_t d, int32_t* label, int32_t k, double* C, int64_t* count,
            hipStream_t st, int32_t rounds = 1, bool with_assign = false) {
  using namespace lma::part;
  const int64_t nch = n > 0 ? (n + CHUNK - 1) / CHUNK : 0;
  const int64_t per = update_per_chunk(d, k);
  int64_t cap = PART_BYTES;
  if (const char* env = std::getenv("LMA_KMEANS_PART_BYTES")) cap = std::max<long long>(1, std::atoll(env));
  const int64_t group = nch == 0 ? 0 : std::max<int64_t>(1, std::min<int64_t>(nch, cap / per));
  check_launch_size(group, d, k);
  struct Mem {  // given back after the stream has drained, also when a launch fails
    char* p;
    size_t bytes;
    hipStream_t st;
    hipError_t es = hipSuccess;
    void release() {
      if (!p) return;
      es = hipStreamSynchronize(st);
      lmart::devcache::put(p, bytes);
      p = nullptr;
    }
    ~Mem() { release(); }
  };
  const size_t bytes = (size_t)(group * per + update_running(d, k));
  Mem mem{static_cast<char*>(lmart::devcache::get(bytes)), bytes, st};
  if (!mem.p) throw Err{LMA_E_NOMEM, "device allocation for the centre update failed"};
  hipError_t err = hipSuccess;
  for (int32_t it = 0; it < rounds && err == hipSuccess; ++it) {
    if (with_assign) assign(P, n, d, C, k, label, nullptr, st);
    err = update_launch(P, n, d, label, k, C, count, group, mem.p, st);
  }
  mem.release();
  if (err != hipSuccess) throw Err{LMA_E_HIP, std::string("k-means update launch: ") + hipGetErrorString(err)};
  if (mem.es != hipSuccess) throw Err{LMA_E_HIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(mem.es)};
}

// Device address of the scratch array on the current device, looked up once
// per device (each GPU holds its own copy at its own address).
char* scratch_ptr() {
  static std::mutex mu;
  static std::vector<char*> ptrs;
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(mu);
  if ((int)ptrs.size() <= dev) ptrs.resize(dev + 1, nullptr);
  if (!ptrs[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(lma::part::scratch));
    if (e != hipSuccess || !ptr)
      throw Err{LMA_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)};
    ptrs[dev] = static_cast<char*>(ptr);
  }
  return ptrs[dev];
}

// The update in the fixed scratch array: no allocation and no synchronisation.
void update_noalloc(const double* P, int64_t n, int32_t d, const int32_t* label, int32_t k, double* C,
                    int64_t* count, hipStream_t st) {
  using namespace lma::part;
  const int64_t nch = n > 0 ? (n + CHUNK - 1) / CHUNK : 0;
  const int64_t per = update_per_chunk(d, k);
  const int64_t room = NOALLOC_BYTES - update_running(d, k);
  if (room < per)
    throw Err{LMA_E_ARG, "k * d too large for the allocation-free update: need 24 k d + 8 k <= " +
                             std::to_string(NOALLOC_BYTES) + " bytes"};
  const int64_t group = nch == 0 ? 0 : std::max<int64_t>(1, std::min<int64_t>(nch, room / per));
  check_launch_size(group, d, k);
  char* mem = scratch_ptr();
  const hipError_t err = update_launch(P, n, d, label, k, C, count, group, mem, st);
  if (err != hipSuccess) throw Err{LMA_E_HIP, std::string("k-means update launch: ") + hipGetErrorString(err)};
}

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

#pragma clang fp contract(off)
double host_sqdist(const double* a, const double* b, int d) {
  double acc = 0.0;
  for (int t = 0; t < d; ++t) {
    const double df = a[t] - b[t];
    const double sq = df * df;
    acc = acc + sq;
  }
  return acc;
}

void chain_order(const double* C, int k, int d, int32_t* order) {
  std::vector<double> mean(d, 0.0);
  for (int c = 0; c < k; ++c)
    for (int t = 0; t < d; ++t) mean[t] = mean[t] + C[(int64_t)c * d + t];
  for (int t = 0; t < d; ++t) mean[t] = mean[t] / (double)k;
  int cur = 0;
  double far = -1.0;
  for (int c = 0; c < k; ++c) {
    const double q = host_sqdist(C + (int64_t)c * d, mean.data(), d);
    if (q > far) {
      far = q;
      cur = c;
    }
  }
  std::vector<char> seen(k, 0);
  order[0] = cur;
  seen[cur] = 1;
  for (int step = 1; step < k; ++step) {
    int nxt = -1;
    double best = 0.0;
    for (int c = 0; c < k; ++c) {
      if (seen[c]) continue;
      const double q = host_sqdist(C + (int64_t)c * d, C + (int64_t)cur * d, d);
      if (nxt < 0 || q < best) {
        best = q;
        nxt = c;
      }
    }
    order[step] = nxt;
    seen[nxt] = 1;
    cur = nxt;
  }
}

}  // namespace

extern "C" {

lma_status lma_kmeans_assign(const double* P, int64_t n, int32_t d, const double* C, int32_t k, int32_t* label,
                             double* dist2, hipStream_t stream) {
  return guard([&] {
    check_shape(P, n, d, k);
    if (n > 0 && (!C || !label)) throw Err{LMA_E_ARG, "NULL array"};
    assign(P, n, d, C, k, label, dist2, stream);
  });
}

lma_status lma_kmeans_update(const double* P, int64_t n, int32_t d, const int32_t* label, int32_t k, double* C,
                             int64_t* count, hipStream_t stream) {
  return guard([&] {
    check_shape(P, n, d, k);
    if (!C || (n > 0 && !label)) throw Err{LMA_E_ARG, "NULL array"};
    update(P, n, d, const_cast<int32_t*>(label), k, C, count, stream);  // label is read only
  });
}

lma_status lma_kmeans_update_noalloc(const double* P, int64_t n, int32_t d, const int32_t* label, int32_t k,
                                     double* C, int64_t* count, hipStream_t stream) {
  return guard([&] {
    check_shape(P, n, d, k);
    if (!C || (n > 0 && !label)) throw Err{LMA_E_ARG, "NULL array"};
    update_noalloc(P, n, d, label, k, C, count, stream);
  });
}

lma_status lma_kmeans(const double* P, int64_t n, int32_t d, double* C, int32_t k, int32_t iters, int32_t* label,
                      double* dist2, hipStream_t stream) {
  return guard([&] {
    check_shape(P, n, d, k);
    if (iters < 0) throw Err{LMA_E_ARG, "iters < 0"};
    if (!C || (n > 0 && !label)) throw Err{LMA_E_ARG, "NULL array"};
    if (n > 0 && iters > 0) update(P, n, d, label, k, C, nullptr, stream, iters, true);
    assign(P, n, d, C, k, label, dist2, stream);
  });
}

lma_status lma_chain_order(const double* C, int32_t k, int32_t d, int32_t* order) {
  return guard([&] {
    if (d < 1 || d > lma::MAX_D) throw Err{LMA_E_ARG, "need 1 <= d <= 64"};
    if (k < 1) throw Err{LMA_E_ARG, "need k >= 1"};
    if (!C || !order) throw Err{LMA_E_ARG, "NULL array"};
    chain_order(C, k, d, order);
  });
}

}  // extern "C"
