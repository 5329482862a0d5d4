// Launcher of the 64 x 64 tile of the bf16 product (gemm_slices.hip), for gemm_bf16.hip.
#pragma once
#include "gemm_epilogue.h"
#include "kernels.h"

namespace karma {

constexpr int SLICE_TILE = 64, SLICE_BK = 64, SLICE_WAVES = 4;

// One product of a launch: `items` workgroups, one for each (range of k, tile)
struct SliceWork {
  const bf16_t* A;
  const bf16_t* B;
  GemmEpilogue ep;
  float* partial;      // splits > 1: [splits][M][N]
  int M, N, K, lda, ldb;
  int splits, k_per_split;
};
inline int slice_items(const SliceWork& w) {
  return (w.M + SLICE_TILE - 1) / SLICE_TILE * ((w.N + SLICE_TILE - 1) / SLICE_TILE) * w.splits;
}
// The layouts and output stage of a product, as far as the kernel is compiled for them
struct SliceForm {
  bool a_kc, b_kc;
  int act;
};
// One product, or (second not null) two in one launch: an input gradient (first operand k-contiguous, the other strided, act 0
// or 2) and a weight gradient (both strided, act 0).  What gemm_ring_takes asks of the operands holds here too.
int gemm_slices_launch(const SliceWork& first, SliceForm form, const SliceWork* second, hipStream_t s);

}  // namespace karma
