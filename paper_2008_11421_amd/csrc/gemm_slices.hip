// The bf16 product with a 64 x 64 tile whose reduction is divided over the wavefronts of a workgroup: small products, which
// take their time from the trips to memory that follow one another and from how few compute units they reach.
//
// Each of the four wavefronts computes the whole tile over its own k-tiles of 64 (w, w + 4, ...), which it fetches into LDS
// for itself (two stages of 16 KiB, direct loads through buffer descriptors as in gemm_ring.hip): no barrier in the k-loop,
// eight k-tiles in flight per workgroup, and 64 x 64 results per wavefront keep it at one LDS read per MFMA.  The four partial
// tiles are added in LDS in the order of the wavefronts, so that no second launch adds them up.  Up to four k-tiles one stage
// is enough and two workgroups share a compute unit.
// A backward pass's two products of the same gradient run as one launch (SliceWork second): neither alone fills the chip.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>

#include "device_utils.h"
#include "gemm_slices.h"
#include "karma.h"

namespace karma {
namespace {

constexpr int BT = SLICE_TILE, BK = SLICE_BK, WAVES = SLICE_WAVES, KSTEPS = BK / 16;
constexpr int OP_BYTES = BT * BK * 2, STAGE = 2 * OP_BYTES, CH = OP_BYTES / 1024, LPT = 2 * CH;
constexpr int SP = BT + 4;                               // fp32 pitch of a partial tile
constexpr int PARTIALS = WAVES * BT * SP * 4;
constexpr int lds_bytes(int nst) { return nst * WAVES * STAGE > PARTIALS ? nst * WAVES * STAGE : PARTIALS; }

template <bool A_KC, bool B_KC, int ACT, int NST>
__device__ __forceinline__ void slice_item(const SliceWork& p, int item, unsigned char* smem) {
  const unsigned lds0 = (unsigned)(uintptr_t)((KARMA_LDS(unsigned char)*)smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lrow = lane & 31;
  const int M = p.M, N = p.N, K = p.K, splits = p.splits;
  const int tiles_m = (M + BT - 1) / BT, tiles_n = (N + BT - 1) / BT, total_tiles = tiles_m * tiles_n;
  const int split = item / total_tiles, id = item % total_tiles;
  const int band_sz = 8 * tiles_n, first_m = (id / band_sz) * 8, rows_in_band = min(tiles_m - first_m, 8);
  const int m0 = (first_m + (id % band_sz) % rows_in_band) * BT, n0 = ((id % band_sz) / rows_in_band) * BT;
  const int kb = split * p.k_per_split, klen = min(K, kb + p.k_per_split) - kb, KT = (klen + BK - 1) / BK;
  const int mine = KT > wave ? (KT - wave + WAVES - 1) / WAVES : 0;   // this wavefront's k-tiles

  // the output stage's per-element input, requested before anything else
  const GemmEpilogue& ep = p.ep;
  const int q = (lane & 3) | (((lane >> 3) & 1) << 2), rr = ((lane >> 2) & 1) | ((lane >> 4) << 1);
  const int n = n0 + q * 8;
  const bf16_t* ein = ACT == 2 ? ep.aux : (ep.out_f32 ? nullptr : ep.residual);
  const bool fetch_in = ein != nullptr && splits == 1 && (ep.ldc & 7) == 0 && n + 8 <= N;
  u32x4 pre[2];
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int m = m0 + pass * 32 + wave * 8 + rr;
    pre[pass] = fetch_in && m < M ? *(const u32x4*)(ein + (size_t)m * ep.ldc + n) : u32x4{0, 0, 0, 0};
  }

  // ---- global side: 1-KiB piece i of a tile is rows 8 i .. + 7 of a k-contiguous one (piece p of row r stored at
  // p ^ (r / 2) % 8) or k-rows 8 i .. + 7 of a strided one (piece p of k-row k stored at p ^ 4 (k / 2 % 2): four k-rows of
  // 32 columns then lie in different banks)
  auto piece_row = [&](int i) { return 8 * i + (lane >> 3); };
  auto piece_col = [&](bool kc, int i) {
    return kc ? ((lane & 7) ^ ((4 * (i & 1) + (lane >> 4)) & 7)) * 8 : ((lane & 7) ^ (((lane >> 4) & 1) << 2)) * 8;
  };
  unsigned a_off[CH], b_off[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    a_off[i] = (m0 + (A_KC ? piece_row(i) : piece_col(false, i)) < M)
                   ? (unsigned)(((size_t)piece_row(i) * p.lda + piece_col(A_KC, i)) * 2) : LOAD_NOTHING;
    b_off[i] = (n0 + (B_KC ? piece_row(i) : piece_col(false, i)) < N)
                   ? (unsigned)(((size_t)piece_row(i) * p.ldb + piece_col(B_KC, i)) * 2) : LOAD_NOTHING;
  }
  const bf16_t* a_base = p.A + (A_KC ? (size_t)m0 * p.lda + kb : (size_t)kb * p.lda + m0);
  const bf16_t* b_base = p.B + (B_KC ? (size_t)n0 * p.ldb + kb : (size_t)kb * p.ldb + n0);
  auto issue = [&](int j) {   // this wavefront's tile j
    const int t = wave + j * WAVES, left = klen - t * BK;
    const unsigned sa = lds0 + (wave * NST + (j & (NST - 1))) * STAGE, sb = sa + OP_BYTES;
    const u32x4 da = buffer_desc(a_base + (A_KC ? (size_t)t * BK : (size_t)t * BK * p.lda));
    const u32x4 db = buffer_desc(b_base + (B_KC ? (size_t)t * BK : (size_t)t * BK * p.ldb));
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      buffer_load_to_lds16(da, (left >= BK || (A_KC ? piece_col(true, i) : piece_row(i)) < left) ? a_off[i] : LOAD_NOTHING, sa + i * 1024);
      buffer_load_to_lds16(db, (left >= BK || (B_KC ? piece_col(true, i) : piece_row(i)) < left) ? b_off[i] : LOAD_NOTHING, sb + i * 1024);
    }
  };

  // ---- LDS side: fragment addresses as in gemm_ring.hip, strided tiles with 128-byte k-rows
  const int grp = lane >> 4, e4 = (lane >> 2) & 3, q4 = lane & 3;
  auto frag_base = [&](bool kc, int row0) -> unsigned {
    if (kc) return (unsigned)((row0 + lrow) * (BK * 2)) + (unsigned)(((lane >> 5) ^ ((lrow >> 1) & 7)) * 16);
    const int m = row0 + 16 * (grp & 1) + 4 * q4;
    return (unsigned)((8 * (grp >> 1) + e4) * (BT * 2) + ((m >> 3) ^ ((e4 >> 1) << 2)) * 16 + (m & 7) * 2);
  };
  unsigned a_fb[2], b_fb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    a_fb[i] = frag_base(A_KC, i * 32);
    b_fb[i] = frag_base(B_KC, i * 32);
  }
  auto read_one = [&](bool kc, unsigned tile, unsigned fb, int kk) -> bf16x8 {
    if (kc) return *(const KARMA_LDS(bf16x8)*)(uintptr_t)(tile + (fb ^ (unsigned)(kk << 5)));
    const unsigned at = tile + fb + (unsigned)(kk * 16 * (BT * 2));
    return read_tr_pair(at, at + 4 * (BT * 2));
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
  for (int j = 0; j < NST; ++j)
    if (j < mine) issue(j);
  for (int j = 0; j < mine; ++j) {
    if (NST > 1 && j + 1 < mine) wait_vm<LPT>();   // tile j has landed; the one after it need not have
    else wait_vm<0>();
    const unsigned ta = lds0 + (wave * NST + (j & (NST - 1))) * STAGE, tb = ta + OP_BYTES;
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      bf16x8 af[2], bf[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        bf[x] = read_one(B_KC, tb, b_fb[x], kk);
        af[x] = read_one(A_KC, ta, a_fb[x], kk);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int x = 0; x < 2; ++x) acc[i][x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[x], af[i], acc[i][x], 0, 0, 0);
    }
    if (j + NST < mine) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this stage's fragments are in registers
      issue(j + NST);
    }
  }

  // ---- the partial tiles, in LDS where the stages were; accumulators hold the transposed tile (a lane's quad is four
  // consecutive columns of a row)
  lds_barrier_visible();
  float* part = (float*)smem + wave * BT * SP;
  if (mine > 0 || wave == 0)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(float4*)(part + (i * 32 + lrow) * SP + x * 32 + g * 8 + (lane >> 5) * 4) =
              make_float4(acc[i][x][4 * g], acc[i][x][4 * g + 1], acc[i][x][4 * g + 2], acc[i][x][4 * g + 3]);
  lds_barrier_visible();
  const int parts = min(WAVES, KT);
  const bool col_sums = ACT == 2 && ep.colsum != nullptr && splits == 1;
  float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int row = pass * 32 + wave * 8 + rr, m = m0 + row;
    const float* src = (const float*)smem + row * SP + q * 8;
    float4 v = *(const float4*)src, u = *(const float4*)(src + 4);
#pragma unroll
    for (int w = 1; w < WAVES; ++w)
      if (w < parts) {
        const float4 a = *(const float4*)(src + w * BT * SP), b = *(const float4*)(src + w * BT * SP + 4);
        v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        u.x += b.x; u.y += b.y; u.z += b.z; u.w += b.w;
      }
    if (m < M && n < N) {
      if (splits > 1) {
        float* dst = p.partial + ((size_t)split * M + m) * N + n;
        const float vv[8] = {v.x, v.y, v.z, v.w, u.x, u.y, u.z, u.w};
        if (n + 8 <= N && (N & 3) == 0) { *(float4*)dst = v; *(float4*)(dst + 4) = u; }
        else for (int e = 0; e < N - n && e < 8; ++e) dst[e] = vv[e];
      } else {
        ep.template octet<ACT>(m, n, min(8, N - n), v, u, fetch_in, pre[pass], col_sums, cs);
      }
    }
  }
  if (col_sums) {
    // lanes that share a column octet differ in lane bits 2, 4 and 5; then the wavefronts, in their order
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      cs[e] += __shfl_xor(cs[e], 4, 64);
      cs[e] += __shfl_xor(cs[e], 16, 64);
      cs[e] += __shfl_xor(cs[e], 32, 64);
    }
    lds_barrier_visible();   // the partial tiles have been read
    float* sums = (float*)smem;
    if (rr == 0) {
      *(float4*)(sums + wave * BT + q * 8) = make_float4(cs[0], cs[1], cs[2], cs[3]);
      *(float4*)(sums + wave * BT + q * 8 + 4) = make_float4(cs[4], cs[5], cs[6], cs[7]);
    }
    lds_barrier_visible();
    if (tid < BT && n0 + tid < N)
      ep.colsum[(size_t)(m0 / BT) * N + n0 + tid] = ((sums[tid] + sums[BT + tid]) + sums[2 * BT + tid]) + sums[3 * BT + tid];
  }
}

// Items in eight contiguous ranges, one per XCD (workgroup ids go round-robin over them), as in gemm_ring.hip
__device__ __forceinline__ int xcd_item(int wg, int items) {
  const int per_xcd = (items + 7) / 8, item = (wg % 8) * per_xcd + wg / 8;
  return wg / 8 < per_xcd && item < items ? item : -1;
}

template <bool A_KC, bool B_KC, int ACT, int NST>
__global__ __launch_bounds__(256, 2) void gemm_slices_kernel(SliceWork p, int items) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_slices[];
  const int item = xcd_item((int)blockIdx.x, items);
  if (item >= 0) slice_item<A_KC, B_KC, ACT, NST>(p, item, smem_slices);
}
// first: an input gradient, in the first `wgs` workgroups (a multiple of eight); second: a weight gradient
template <int ACT, int NST>
__global__ __launch_bounds__(256, 2) void gemm_slices_pair_kernel(SliceWork first, int items, int wgs, SliceWork second, int items2) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_slices[];
  if ((int)blockIdx.x < wgs) {
    const int item = xcd_item((int)blockIdx.x, items);
    if (item >= 0) slice_item<true, false, ACT, NST>(first, item, smem_slices);
  } else {
    const int item = xcd_item((int)blockIdx.x - wgs, items2);
    if (item >= 0) slice_item<false, false, 0, NST>(second, item, smem_slices);
  }
}

int padded8(int items) { return (items + 7) / 8 * 8; }

template <bool AK, bool BKC, int ACT, int NST>
void launch_one(const SliceWork& p, hipStream_t s) {
  auto kern = gemm_slices_kernel<AK, BKC, ACT, NST>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(NST));
  const int items = slice_items(p);
  hipLaunchKernelGGL(kern, dim3((unsigned)padded8(items)), dim3(64 * WAVES), lds_bytes(NST), s, p, items);
}
template <int ACT, int NST>
void launch_pair(const SliceWork& a, const SliceWork& b, hipStream_t s) {
  auto kern = gemm_slices_pair_kernel<ACT, NST>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(NST));
  const int ia = slice_items(a), ib = slice_items(b), wgs = padded8(ia);
  hipLaunchKernelGGL(kern, dim3((unsigned)(wgs + padded8(ib))), dim3(64 * WAVES), lds_bytes(NST), s, a, ia, wgs, b, ib);
}
template <int NST>
void launch_form(const SliceWork& p, SliceForm f, const SliceWork* second, hipStream_t s) {
  if (second) {
    if (f.act == 2) launch_pair<2, NST>(p, *second, s);
    else launch_pair<0, NST>(p, *second, s);
  } else if (f.act == 1) launch_one<true, true, 1, NST>(p, s);
  else if (f.act == 2) launch_one<true, false, 2, NST>(p, s);
  else if (f.a_kc && f.b_kc) launch_one<true, true, 0, NST>(p, s);
  else if (f.a_kc) launch_one<true, false, 0, NST>(p, s);
  else if (f.b_kc) launch_one<false, true, 0, NST>(p, s);
  else launch_one<false, false, 0, NST>(p, s);
}

}  // namespace

int gemm_slices_launch(const SliceWork& first, SliceForm form, const SliceWork* second, hipStream_t s) {
  // the layouts of act 1 and 2 were checked by the caller
  if (second && !(form.a_kc && !form.b_kc && form.act != 1)) return KARMA_E_INVAL;
  const int longest = std::max(std::min(first.K, first.k_per_split), second ? std::min(second->K, second->k_per_split) : 0);
  if (longest <= WAVES * BK) launch_form<1>(first, form, second, s);
  else launch_form<2>(first, form, second, s);
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

}  // namespace karma
