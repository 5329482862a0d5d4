// fp32 kernels of the MLP workload: fully connected layer with ReLU (KARMA Sec. III-C,
// "Fully-Connected Layer", "ReLu Layer"), its backward, and the mean-squared-error loss.
//
// The products are a few million multiply-adds (32 x 256 x 256): what bounds them is the chain of memory round trips and
// the launches, not arithmetic.  A workgroup computes one 16 x 16 tile, its four wavefronts each a quarter of the
// reduction with v_mfma_f32_16x16x4_f32 (fp32 products and sums), operands straight from global memory to registers, all
// of a wavefront's loads for 64 k in flight at once; the four partial tiles are added in order through LDS.  The backward
// pass is one launch: tiles of dx, tiles of dw and the column sums of db, each reading dz = dy * (z > 0) as it loads.
// 32 x 256 x 256: forward 25.5 -> 5.6 us, backward 38 us in four launches -> 8.6 us in one (a
// 32 x 32 tile per workgroup stepped through LDS 16 k at a time waited for memory 16 times in eight workgroups).
#include <hip/hip_runtime.h>

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
// itself: workgroups 0 .. dx_tiles-1 take dx, the next dw_tiles dw, the rest 256 columns of db and dz each.
__global__ __launch_bounds__(256) void linear_relu_bwd_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                              const float* __restrict__ z, const float* __restrict__ dy,
                                                              float* __restrict__ dz, float* __restrict__ dx,
                                                              float* __restrict__ dw, float* __restrict__ db, int m, int n, int k,
                                                              int dx_tiles, int dw_tiles, bool vec) {
  __shared__ f32x4 part[4][64];
  int id = blockIdx.x;
  const int across = (k + TS - 1) / TS;
  if (id < dx_tiles) {
    tile_f32(Operand<true>{dy, z, m, n, vec}, Operand<false>{w, nullptr, k, n, false}, id / across * TS, id % across * TS,
             [&](int r, int c, float v) { dx[(size_t)r * k + c] = v; }, part);
    return;
  }
  id -= dx_tiles;
  if (id < dw_tiles) {
    tile_f32(Operand<false>{dy, z, n, m, false}, Operand<false>{x, nullptr, k, m, false}, id / across * TS, id % across * TS,
             [&](int r, int c, float v) { dw[(size_t)r * k + c] = v; }, part);
    return;
  }
  const int c = (id - dw_tiles) * 256 + threadIdx.x;
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

// dx alone, from dz
__global__ __launch_bounds__(256) void linear_relu_dx_kernel(const float* __restrict__ w, const float* __restrict__ dz,
                                                             float* __restrict__ dx, int m, int n, int k, bool vec) {
  __shared__ f32x4 part[4][64];
  const int across = (k + TS - 1) / TS, id = blockIdx.x;
  tile_f32(Operand<true>{dz, nullptr, m, n, vec}, Operand<false>{w, nullptr, k, n, false}, id / across * TS, id % across * TS,
           [&](int r, int c, float v) { dx[(size_t)r * k + c] = v; }, part);
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

int linear_relu_fwd_f32(const float* x, const float* w, const float* b, float* z, float* y, int m, int n, int k,
                        hipStream_t s) {
  const bool vec = k % 4 == 0;
  hipLaunchKernelGGL(linear_relu_fwd_kernel, dim3((unsigned)((n + TS - 1) / TS) * (unsigned)((m + TS - 1) / TS)), dim3(256), 0, s,
                     (Operand<true>{x, nullptr, m, k, vec && aligned16(x)}), (Operand<true>{w, nullptr, n, k, vec && aligned16(w)}), b, z, y);
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

int linear_relu_bwd_f32(const float* x, const float* w, const float* z, const float* dy, float* dz, float* dx,
                        float* dw, float* db, int m, int n, int k, hipStream_t s) {
  const int across = (k + TS - 1) / TS, dw_tiles = (n + TS - 1) / TS * across, sums = (n + 255) / 256;
  const int dx_tiles = dx ? (m + TS - 1) / TS * across : 0;
  const bool vec = n % 4 == 0 && aligned16(z) && aligned16(dy) && aligned16(dz);
  auto launch = [&](int first) {
    hipLaunchKernelGGL(linear_relu_bwd_kernel, dim3(first + dw_tiles + sums), dim3(256), 0, s, x, w, z, dy, dz, dx, dw, db, m, n, k,
                       first, dw_tiles, vec);
  };
  // dx written over its own inputs: everything else reads them first, and dx is made from dz
  auto meets = [&](const float* q) { return dx && dx < q + (size_t)m * n && q < dx + (size_t)m * k; };
  if (meets(dy) || meets(z)) {
    launch(0);
    hipLaunchKernelGGL(linear_relu_dx_kernel, dim3(dx_tiles), dim3(256), 0, s, w, dz, dx, m, n, k, vec);
  } else {
    launch(dx_tiles);
  }
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
