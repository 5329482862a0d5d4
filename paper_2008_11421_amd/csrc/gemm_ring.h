// Launcher of the 128 x 128 tile of the bf16 product (gemm_ring.hip), for gemm_bf16.hip.
#pragma once
#include "gemm_epilogue.h"
#include "kernels.h"

namespace karma {

// One product of a gathered launch.  A strided convolution's input gradient is up to four of them: output pixels of
// one parity in each direction see one subset of the taps, as a stride-1 convolution of its own.
struct RingPhase {
  ConvGather cg;
  int M, K;              // pixels of this parity, taps * channels
  unsigned b_off;        // first element of its weights, [N][K] from there on
  unsigned magic_s;      // 2^32 / cg.S + 1, or 0 for a single column of taps
  int oy, ox;            // parity of its output pixels
  int pad_y, pad_x;      // padding, which may differ by direction between parities (cg.pad is not read)
};
struct RingConv {
  RingPhase p[4];
  int phases;
  int out_stride, oh, ow;   // output pixel (y, x) of a phase is pixel (y * out_stride + oy, x * out_stride + ox) of oh x ow
  unsigned magic_c;         // 2^32 / C + 1
};

constexpr int RING_TILE = 128, RING_BK = 64;
// the other tiles, for the gathered forms: 256 pixels x this many channels (conv_mode 1), or as many x 256 (conv_mode 2)
constexpr int RING_BROAD = 160, RING_SLIM = 64;

// Whether the operands' sizes and alignment are what the kernel's 16-byte pieces and 32-bit offsets need.
bool gemm_ring_takes(const GemmArgs& g);
// Launches the product over `splits` ranges of k_per_split (partials in g.ws when splits > 1; the caller adds them up).
// deep: four stages instead of two.  side: RING_TILE, RING_BROAD or RING_SLIM.
// rc: the gathered forms, else null.  ep.colsum is honoured with act 2.
int gemm_ring_launch(const GemmArgs& g, const GemmEpilogue& ep, int splits, int k_per_split, bool deep, int side, const RingConv* rc,
                     hipStream_t s);

}  // namespace karma
