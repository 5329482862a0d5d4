// fp32 kernels of the MLP workload: fully connected layer with ReLU (KARMA Sec. III-C,
// "Fully-Connected Layer", "ReLu Layer"), its backward, and the mean-squared-error loss.
//
// The workload's products are a few million multiply-adds (32 x 256 x 256): what bounds them is the chain of memory round
// trips and the launches, not arithmetic.  For these a workgroup computes one 16 x 16 tile, its four wavefronts each a
// quarter of the reduction with v_mfma_f32_16x16x4_f32 (fp32 products and sums), operands straight from global memory to
// registers, all of a wavefront's loads for 64 k in flight at once; the four partial tiles are added in order through LDS.
// Products with many tiles keep 32 x 32 tiles through LDS, which fetch an operand element half as often.  The backward
// pass of the former is one launch: the column sums of db, tiles of dx and tiles of dw, each reading dz = dy * (z > 0) as it loads.
// 32 x 256 x 256: forward 25.5 -> 5.6 us, backward 38 us in four launches -> 8.6 us in one (the 32 x 32 tile, stepped
// through LDS 16 k at a time, waits for memory 16 times in eight workgroups).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "karma.h"
#include "kernels.h"

namespace karma {

typedef __attribute__((ext_vector_type(4))) float f32x4;
constexpr int TS = 16;    // output tile edge
constexpr int TKW = 16;   // k per wavefront and step: four per quarter-wavefront
constexpr int AHEAD = 4;  // steps whose loads are in flight together

// An operand of `rows` rows and `K` reduction indices: element (r, k) lies at r * K + k (KC) or k * rows + r.
// z (may be null): elements whose z is not positive count as zero.
template <bool KC>
struct Operand {
  const float* p;
  const float* z;
  int rows, K;
  bool vec;   // KC: four consecutive k may be loaded at once
  __device__ __forceinline__ f32x4 load(int r, int k) const {   // elements (r, k .. k + 3), zero outside
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (r >= rows || k >= K) return v;
    if (KC && vec) {
      const size_t at = (size_t)r * K + k;
      v = *(const f32x4*)(p + at);
      if (z) {
        const f32x4 m = *(const f32x4*)(z + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = m[e] > 0.f ? v[e] : 0.f;
      }
      return v;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < K) {
        const size_t at = KC ? (size_t)r * K + k + e : (size_t)(k + e) * rows + r;
        v[e] = (!z || z[at] > 0.f) ? p[at] : 0.f;
      }
    return v;
  }
};

// One 16 x 16 tile of C[m,n] = sum_k A(m,k) B(n,k) by 256 threads; ep(m, n, value) once per element.
template <bool A_KC, bool B_KC, class Epilogue>
__device__ __forceinline__ void tile_f32(const Operand<A_KC>& A, const Operand<B_KC>& B, int m0, int n0, const Epilogue& ep,
                                         f32x4 (*part)[64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int K = A.K;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = wave * TKW; k0 < K; k0 += 4 * TKW * AHEAD) {
    f32x4 a[AHEAD], b[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {   // (k slots in the order 4 g + e for both operands: any order serves)
      a[u] = A.load(m0 + r, k0 + u * 4 * TKW + 4 * g);
      b[u] = B.load(n0 + r, k0 + u * 4 * TKW + 4 * g);
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][e], acc, 0, 0, 0);
  }
  part[wave][lane] = acc;
  __syncthreads();
  // element (4 g + wave, r) of the tile: one per thread
  const float* q = (const float*)part;
  const int at = lane * 4 + wave, n = n0 + r, m = m0 + 4 * g + wave;
  if (m < A.rows && n < B.rows) ep(m, n, ((q[at] + q[256 + at]) + q[512 + at]) + q[768 + at]);
}

__global__ __launch_bounds__(256) void linear_relu_fwd_kernel(Operand<true> X, Operand<true> W, const float* __restrict__ b,
                                                              float* __restrict__ z, float* __restrict__ y) {
  __shared__ f32x4 part[4][64];
  const int N = W.rows, across = (N + TS - 1) / TS;
  tile_f32(X, W, blockIdx.x / across * TS, blockIdx.x % across * TS, [&](int m, int n, float v) {
    v += b[n];
    z[(size_t)m * N + n] = v;
    y[(size_t)m * N + n] = v > 0.f ? v : 0.f;
  }, part);
}

// dx[m,k] = sum_n dz[m,n] w[n,k], dw[n,k] = sum_m dz[m,n] x[m,k], db[n] = sum_m dz[m,n] (rows in ascending order) and dz
// itself: the first `sums` workgroups take 256 columns of db and dz each (a serial walk over the rows, the longest chain
// of the launch where there are many), the next dx_tiles dx, the rest dw.
__global__ __launch_bounds__(256) void linear_relu_bwd_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                              const float* __restrict__ z, const float* __restrict__ dy,
                                                              float* __restrict__ dz, float* __restrict__ dx,
                                                              float* __restrict__ dw, float* __restrict__ db, int m, int n, int k,
                                                              int sums, int dx_tiles, bool vec) {
  __shared__ f32x4 part[4][64];
  const int across = (k + TS - 1) / TS, first = sums + dx_tiles;
  int id = blockIdx.x;
  if (id >= first) {
    id -= first;
    tile_f32(Operand<false>{dy, z, n, m, false}, Operand<false>{x, nullptr, k, m, false}, id / across * TS, id % across * TS,
             [&](int r, int c, float v) { dw[(size_t)r * k + c] = v; }, part);
    return;
  }
  if (id >= sums) {
    id -= sums;
    tile_f32(Operand<true>{dy, z, m, n, vec}, Operand<false>{w, nullptr, k, n, false}, id / across * TS, id % across * TS,
             [&](int r, int c, float v) { dx[(size_t)r * k + c] = v; }, part);
    return;
  }
  const int c = id * 256 + threadIdx.x;
  if (c >= n) return;
  float s = 0.f;
#pragma unroll 8
  for (int r = 0; r < m; ++r) {
    const size_t at = (size_t)r * n + c;
    const float v = z[at] > 0.f ? dy[at] : 0.f;
    dz[at] = v;
    s += v;
  }
  db[c] = s;
}

// ---- the same products for sizes that have workgroups enough without the split, where each operand element's trip is what
// counts: a 32 x 32 tile per workgroup, 16 k at a time through LDS, each of the 16 x 16 threads a 2 x 2 patch.
constexpr int TSL = 32, TKL = 16;

// C[m,n] = sum_k A(m,k) * B(n,k);  A row-major [M,K] (or [K,M] when A_T), B row-major [N,K] (or [K,N] when B_T).
template <bool A_T, bool B_T, class Epilogue>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* A, const float* B, int M, int N, int K, Epilogue ep) {
  __shared__ float As[TKL][TSL + 1];
  __shared__ float Bs[TKL][TSL + 1];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int m0 = blockIdx.y * TSL, n0 = blockIdx.x * TSL;
  float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
  for (int k0 = 0; k0 < K; k0 += TKL) {
    // 512 elements per operand tile, 2 per thread
    for (int e = threadIdx.x; e < TSL * TKL; e += 256) {
      int r, c;   // r: row within tile (m or n), c: k within step
      if (A_T) { r = e % TSL; c = e / TSL; } else { r = e / TKL; c = e % TKL; }
      int gm = m0 + r, gk = k0 + c;
      float v = 0.f;
      if (gm < M && gk < K) v = A_T ? A[(size_t)gk * M + gm] : A[(size_t)gm * K + gk];
      As[c][r] = v;
      if (B_T) { r = e % TSL; c = e / TSL; } else { r = e / TKL; c = e % TKL; }
      int gn = n0 + r;
      gk = k0 + c;
      v = 0.f;
      if (gn < N && gk < K) v = B_T ? B[(size_t)gk * N + gn] : B[(size_t)gn * K + gk];
      Bs[c][r] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TKL; ++k) {
      float a0 = As[k][ty], a1 = As[k][ty + 16], b0 = Bs[k][tx], b1 = Bs[k][tx + 16];
      acc[0][0] = fmaf(a0, b0, acc[0][0]);
      acc[0][1] = fmaf(a0, b1, acc[0][1]);
      acc[1][0] = fmaf(a1, b0, acc[1][0]);
      acc[1][1] = fmaf(a1, b1, acc[1][1]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int m = m0 + ty + 16 * i, n = n0 + tx + 16 * j;
      if (m < M && n < N) ep(m, n, acc[i][j]);
    }
}

struct EpBiasRelu {
  const float* b; float* z; float* y; int N;
  __device__ void operator()(int m, int n, float v) const {
    v += b[n];
    z[(size_t)m * N + n] = v;
    y[(size_t)m * N + n] = v > 0.f ? v : 0.f;
  }
};
struct EpStore {
  float* c; int N;
  __device__ void operator()(int m, int n, float v) const { c[(size_t)m * N + n] = v; }
};

// dz = dy * (z > 0)
__global__ void relu_mask_kernel(const float* z, const float* dy, float* dz, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dz[i] = z[i] > 0.f ? dy[i] : 0.f;
}

// db[n] = sum_m dz[m,n], rows in ascending order
__global__ void colsum_kernel(const float* __restrict__ dz, float* __restrict__ db, int M, int N) {
  int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  float s = 0.f;
  for (int m = 0; m < M; ++m) s += dz[(size_t)m * N + n];
  db[n] = s;
}

// stage 1 of the loss: dy and per-block partial sums of (y - t)^2
__global__ __launch_bounds__(256) void mse_partial_kernel(const float* __restrict__ y, const float* __restrict__ t,
                                                           float* __restrict__ dy, float* __restrict__ partial, size_t n) {
  __shared__ float red[256];
  float s = 0.f;
  const float scale = 2.0f / (float)n;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    float d = y[i] - t[i];
    s = fmaf(d, d, s);
    dy[i] = d * scale;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// stage 2: fixed-order sum of up to 1024 partials, scaled
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ partial, int count, float scale,
                                                            float* __restrict__ out) {
  __shared__ float red[256];
  float s = 0.f;
  for (int i = threadIdx.x; i < count; i += 256) s += partial[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0] * scale;
}

static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }
static inline dim3 large_tiles(int M, int N) { return dim3((N + TSL - 1) / TSL, (M + TSL - 1) / TSL); }
static inline size_t small_tiles(int M, int N) { return (size_t)((N + TS - 1) / TS) * ((M + TS - 1) / TS); }

// Which of the two tiles, by modelled times in us.  The small tile: 1.4 per 256 k of its chain, or 1 ns per workgroup and
// 13 (forward, 16-byte loads) to 40 ps per k; the large one: 0.95 per 16 k, or 1 ns per workgroup and 90 ps per k.  Over
// 494 sizes from 1 x 8 x 8 to 8192 x 8192 x 800 the choice is 0.5 % (forward) and 1.3 % (backward) behind the better one.
//   forward, small / large: 32 x 256 x 256 5.6 / 25.5, 2139 x 2923 x 641 634 / 297, 3483 x 3556 x 228 162 / 221
//   backward, one launch / four: 279 x 2955 x 60 99 / 346, 219 x 2566 x 6390 1206 / 624, 2858 x 2641 x 3406 8309 / 4227
constexpr size_t MOST_WORKGROUPS = 1u << 24;   // of 256 threads in one dimension of a grid, which holds fewer than 2^32
static double small_us(int M, int N, int K, double per_k) {
  return std::max(1.4 * ((K + 255) / 256), (double)small_tiles(M, N) * (1e-3 + per_k * K));
}
static double large_us(int M, int N, int K) {
  const dim3 t = large_tiles(M, N);
  return std::max(0.95 * ((K + TKL - 1) / TKL), (double)t.x * t.y * (1e-3 + 9e-5 * K));
}
static bool split_fwd(int m, int n, int k, bool vec) {
  return small_tiles(m, n) < MOST_WORKGROUPS && small_us(m, n, k, vec ? 1.3e-5 : 3.9e-5) <= large_us(m, n, k);
}
// (the walk of the column sums over the rows is on both sides; the ordered pass has three launches more, 9 us)
static bool split_bwd(int m, int n, int k, bool dx) {
  const double small = (dx ? small_us(m, k, n, n % 4 ? 4e-5 : 2e-5) : 0.0) + small_us(n, k, m, 3e-5);
  const double large = 9.0 + (dx ? large_us(m, k, n) : 0.0) + large_us(n, k, m);
  return small_tiles(m, k) + small_tiles(n, k) + (n + 255) / 256 < MOST_WORKGROUPS && small <= 1.1 * large;
}

int linear_relu_fwd_f32(const float* x, const float* w, const float* b, float* z, float* y, int m, int n, int k,
                        hipStream_t s) {
  const bool vec = k % 4 == 0 && aligned16(x) && aligned16(w);
  if (split_fwd(m, n, k, vec))
    hipLaunchKernelGGL(linear_relu_fwd_kernel, dim3((unsigned)small_tiles(m, n)), dim3(256), 0, s, (Operand<true>{x, nullptr, m, k, vec}),
                       (Operand<true>{w, nullptr, n, k, vec}), b, z, y);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<false, false, EpBiasRelu>), large_tiles(m, n), dim3(256), 0, s, x, w, m, n, k,
                       EpBiasRelu{b, z, y, n});
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

int linear_relu_bwd_f32(const float* x, const float* w, const float* z, const float* dy, float* dz, float* dx,
                        float* dw, float* db, int m, int n, int k, hipStream_t s) {
  const size_t mn = (size_t)m * n, mk = (size_t)m * k, nk = (size_t)n * k;
  // One launch, whose workgroups read and write side by side: only where no result lies over anything that others still
  // read.  (dz over dy is harmless: an element is replaced by itself or by the zero that it is read as.)
  auto meet = [](const float* p, size_t np, const float* q, size_t nq) { return p && q && p < q + nq && q < p + np; };
  auto over_inputs = [&](const float* out, size_t cnt) {
    return meet(out, cnt, x, mk) || meet(out, cnt, w, nk) || meet(out, cnt, z, mn) || meet(out, cnt, dy, mn);
  };
  const bool apart = !(meet(dz, mn, x, mk) || meet(dz, mn, w, nk) || meet(dz, mn, z, mn) || (dz != dy && meet(dz, mn, dy, mn))) &&
                     !over_inputs(dx, mk) && !over_inputs(dw, nk) && !over_inputs(db, n);
  if (apart && split_bwd(m, n, k, dx != nullptr)) {
    const int dx_tiles = dx ? (int)small_tiles(m, k) : 0, dw_tiles = (int)small_tiles(n, k), sums = (n + 255) / 256;
    hipLaunchKernelGGL(linear_relu_bwd_kernel, dim3(sums + dx_tiles + dw_tiles), dim3(256), 0, s, x, w, z, dy, dz, dx, dw, db, m, n, k,
                       sums, dx_tiles, n % 4 == 0 && aligned16(z) && aligned16(dy));
    return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
  }
  hipLaunchKernelGGL(relu_mask_kernel, dim3((unsigned)((mn + 255) / 256)), dim3(256), 0, s, z, dy, dz, mn);
  // dx[m,k] = sum_n dz[m,n] w[n,k]  -> A = dz [M,N] (reduction contiguous), B = w as [N,K] read transposed
  if (dx)
    hipLaunchKernelGGL((gemm_f32_kernel<false, true, EpStore>), large_tiles(m, k), dim3(256), 0, s, dz, w, m, k, n, EpStore{dx, k});
  // dw[n,k] = sum_m dz[m,n] x[m,k] -> both operands read transposed, reduction over m
  hipLaunchKernelGGL((gemm_f32_kernel<true, true, EpStore>), large_tiles(n, k), dim3(256), 0, s, dz, x, n, k, m, EpStore{dw, k});
  hipLaunchKernelGGL(colsum_kernel, dim3((n + 255) / 256), dim3(256), 0, s, dz, db, m, n);
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

int mse_f32(const float* y, const float* t, float* dy, float* loss, float* partial, size_t n, hipStream_t s) {
  int blocks = (int)std::min<size_t>(1024, (n + 255) / 256);
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(mse_partial_kernel, dim3(blocks), dim3(256), 0, s, y, t, dy, partial, n);
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, partial, blocks, 1.0f / (float)n, loss);
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

}  // namespace karma

using namespace karma;

extern "C" int karma_k_linear_relu_fwd_f32(const float* x, const float* w, const float* b, float* z, float* y,
                                           uint32_t m, uint32_t n, uint32_t k, void* stream) {
  if (!x || !w || !b || !z || !y || !m || !n || !k) return KARMA_E_INVAL;
  return linear_relu_fwd_f32(x, w, b, z, y, (int)m, (int)n, (int)k, (hipStream_t)stream);
}

extern "C" int karma_k_linear_relu_bwd_f32(const float* x, const float* w, const float* z, const float* dy,
                                           float* dz_ws, float* dx, float* dw, float* db, uint32_t m, uint32_t n,
                                           uint32_t k, void* stream) {
  if (!x || !w || !z || !dy || !dz_ws || !dw || !db || !m || !n || !k) return KARMA_E_INVAL;
  return linear_relu_bwd_f32(x, w, z, dy, dz_ws, dx, dw, db, (int)m, (int)n, (int)k, (hipStream_t)stream);
}

extern "C" int karma_k_mse_f32(const float* y, const float* t, float* dy, float* loss, float* partial_ws, uint64_t n,
                               void* stream) {
  if (!y || !t || !dy || !loss || !partial_ws || !n) return KARMA_E_INVAL;
  return mse_f32(y, t, dy, loss, partial_ws, (size_t)n, (hipStream_t)stream);
}
