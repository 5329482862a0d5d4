// What happens to eight consecutive results of a bf16 product on their way to memory, shared by the GEMM kernels.
#pragma once
#include "device_utils.h"
#include "kernels.h"

namespace karma {

struct GemmEpilogue {
  void* C;                 // bf16 or fp32 [M][ldc]
  const bf16_t* bias;      // [N] or null
  const bf16_t* residual;  // [M][ldc] or null (bf16 output only)
  int ldc;
  int out_f32;             // store fp32 instead of bf16
  int accumulate;          // fp32 output only: C += result
  bf16_t* aux;             // [M][ldc]: octet<1> writes GELU(C) there, octet<2> multiplies the result by GELU'(aux) (bf16 C only)
  float* colsum;           // octet<2> only, or null: partial column sums of the result, a row of N per 64 (256 x 256 tile: 128) rows
  // eight consecutive columns n..n+7 of row m (n multiple of 8); cols = how many are inside the matrix
  // pre (when have_pre): the eight residual (or, ACT 2, pre-activation) values of this octet, fetched by the caller
  template <int ACT = 0>
  __device__ __forceinline__ void octet(int m, int n, int cols, const float4& lo, const float4& hi,
                                        bool have_pre = false, u32x4 pre = u32x4{0, 0, 0, 0}) const {
    float unused[8];
    octet<ACT>(m, n, cols, lo, hi, have_pre, pre, false, unused);
  }
  // do_sum (octet<2>, full octets): the eight results are also added to sum8
  template <int ACT>
  __device__ __forceinline__ void octet(int m, int n, int cols, const float4& lo, const float4& hi, bool have_pre, u32x4 pre,
                                        bool do_sum, float (&sum8)[8]) const {
    float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const size_t at = (size_t)m * ldc + n;
    if (cols == 8 && (ldc & 7) == 0) {
      if (bias) {
        u32x4 b = *(const u32x4*)(bias + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[2 * e] += __uint_as_float(b[e] << 16); v[2 * e + 1] += __uint_as_float(b[e] & 0xffff0000u); }
      }
      if (out_f32) {
        float4* c = (float4*)((float*)C + at);
        float4 o0 = make_float4(v[0], v[1], v[2], v[3]), o1 = make_float4(v[4], v[5], v[6], v[7]);
        if (accumulate) {
          float4 p0 = c[0], p1 = c[1];
          o0.x += p0.x; o0.y += p0.y; o0.z += p0.z; o0.w += p0.w;
          o1.x += p1.x; o1.y += p1.y; o1.z += p1.z; o1.w += p1.w;
        }
        c[0] = o0;
        c[1] = o1;
      } else {
        if (residual) {
          u32x4 r = have_pre ? pre : *(const u32x4*)(residual + at);
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[2 * e] += __uint_as_float(r[e] << 16); v[2 * e + 1] += __uint_as_float(r[e] & 0xffff0000u); }
        }
        if (ACT == 2) {
          u32x4 r = have_pre ? pre : *(const u32x4*)(aux + at);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[2 * e] *= gelu_grad_f(__uint_as_float(r[e] << 16));
            v[2 * e + 1] *= gelu_grad_f(__uint_as_float(r[e] & 0xffff0000u));
          }
          if (do_sum) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sum8[e] += v[e];
          }
        }
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = pack2(v[2 * e], v[2 * e + 1]);
        *(u32x4*)((bf16_t*)C + at) = o;
        if (ACT == 1) {   // the activation of the value as stored (what a separate pass over C would compute)
          u32x4 a2;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            a2[e] = pack2(gelu_f(__uint_as_float(o[e] << 16)), gelu_f(__uint_as_float(o[e] & 0xffff0000u)));
          *(u32x4*)(aux + at) = a2;
        }
      }
    } else {
      for (int e = 0; e < cols; ++e) {
        float x = v[e];
        if (bias) x += bf2f(bias[n + e]);
        if (out_f32) {
          float* c = (float*)C;
          c[at + e] = accumulate ? c[at + e] + x : x;
        } else {
          if (residual) x += bf2f(residual[at + e]);
          if (ACT == 2) x *= gelu_grad_f(bf2f(aux[at + e]));
          const bf16_t stored = f2bf(x);
          ((bf16_t*)C)[at + e] = stored;
          if (ACT == 1) aux[at + e] = f2bf(gelu_f(bf2f(stored)));
        }
      }
    }
  }
};

}  // namespace karma
