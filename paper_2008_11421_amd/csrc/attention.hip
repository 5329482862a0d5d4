// Fused causal self-attention on the matrix cores, forward and backward.
// Attention(Q, K, V) = Softmax(Q K^T / sqrt(d_k)) V (KARMA Sec. III-C "Self-Attention
// Layer"), one head at a time, with the S x S score matrix never leaving the chip: only
// the output and one log-sum-exp per query are saved for backward.
//
// Data layout: qkv [batch][seq][3*hidden] bf16 with q | k | v in thirds and head j in
// columns j*D..(j+1)*D of each third; ctx [batch][seq][hidden]; lse, delta [batch][head][seq]
// fp32.  lse is kept in the base-2 domain of the scaled scores: lse2 = log2 sum_j
// 2^(s_ij * scale * log2 e).
//
// All three kernels compute score tiles in the orientation that puts the softmax/row
// quantities on the lane (not across lanes): a 32x32 MFMA result holds column l%32 in lane
// l and 16 rows in its registers, so with queries on the columns every per-query reduction
// is a loop over registers plus one exchange between the two half-waves, and the
// probabilities can be fed back as the k-operand of the next MFMA straight from registers.
// Reductions over tiles run in a fixed order; there are no atomics (dQ has its own pass).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "karma.h"
#include "device_utils.h"
#include "kernels.h"

namespace karma {

constexpr float LOG2E = 1.4426950408889634f;

// Tile sizes (keys per tile forward and for dQ, queries for dK/dV) and the workgroups per compute unit that the
// register allocation allows, from a sweep; small tiles need few registers and let the workgroups of a compute unit
// drift apart, so that one's MFMAs overlap the other's exponentials.  Per kernel, us (tile, workgroups):
//   32 x 16 heads x 1024 x 64:  forward (32, 4) 154, (64, 2) 141, (64, 3) 130, (64, 4) 138; dQ (32, 4) 200, (64, 2) 219,
//     (64, 4) 194; dK/dV (32, 2) 287, (32, 3) 267, (32, 4) 537, (64, 2) 284
//   8 x 24 heads x 1024 x 128:  forward (32, 2) 95, (64, 2) 103, (64, 3) 97; dQ (32, 2) 143, (64, 1) 141, (64, 2) 137;
//     dK/dV (32, 1) 268, (32, 2) 227, (64, 1) 243, (64, 2) 199
//   4 x 28 heads x 1024 x 152:  forward (32, 2) 75, (64, 2) 113; dQ (32, 1) 164, (32, 2) 105, (64, 2) 161;
//     dK/dV (32, 1) 224, (32, 2) 365, (64, 1) 181, (64, 2) 476
// The two larger head dimensions with tiles staged through registers, and transposed there: forward 208 and 165, dQ 276
// and 196 (+ 61 and 26 for delta), dK/dV 367 and 290.
// FWD_SLACK: by how many powers of two a query's maximum may grow before the forward pass rescales.  0 for the larger
// heads: with 8 (their forward in the sweep above; 0 takes 4 to 9 % longer, 91 -> 95 and 75 -> 79 us) the output was 2 to
// 14 % further from 64 bits, as a largest probability of one is exact in bf16.
// DKV_WGS_FEW: where there is no second workgroup for a compute unit, the kernel that may use all its registers
// (2 x 5 heads x 384 x 128: 28 -> 24 us).
// FWD_SPLIT_SEQ, BOTH_*: see the launchers (queries per tile, workgroups and groups of wavefronts of the joint backward launch).
template <int D>
struct AttnTiles;
template <>
struct AttnTiles<64> {
  static constexpr int FWD_KT = 64, FWD_WGS = 3, DQ_KT = 64, DQ_WGS = 4, DKV_QT = 32, DKV_WGS = 3, DKV_WGS_FEW = 3;
  static constexpr int FWD_SPLIT_SEQ = 512, BOTH_QT = 64, BOTH_WGS = 2, BOTH_GROUPS = 2;
  static constexpr float FWD_SLACK = 8.f;
};
template <>
struct AttnTiles<128> {
  static constexpr int FWD_KT = 64, FWD_WGS = 3, DQ_KT = 64, DQ_WGS = 2, DKV_QT = 64, DKV_WGS = 2, DKV_WGS_FEW = 1;
  static constexpr int FWD_SPLIT_SEQ = 512, BOTH_QT = 64, BOTH_WGS = 1, BOTH_GROUPS = 1;
  static constexpr float FWD_SLACK = 0.f;
};
template <>
struct AttnTiles<152> {
  static constexpr int FWD_KT = 32, FWD_WGS = 2, DQ_KT = 32, DQ_WGS = 2, DKV_QT = 64, DKV_WGS = 1, DKV_WGS_FEW = 1;
  static constexpr int FWD_SPLIT_SEQ = 256, BOTH_QT = 64, BOTH_WGS = 1, BOTH_GROUPS = 1;
  static constexpr float FWD_SLACK = 0.f;
};

// Head dimensions that are no multiple of 32 (152) run with padded columns: zeros in the tiles, so that they add
// nothing to any product, and the results' padded columns are not stored.  A tile lies in LDS as panels of 64 columns.
constexpr int padded_d(int d) { return (d + 31) / 32 * 32; }
constexpr int tile_bytes(int d, int rows) { return (d + 63) / 64 * rows * 128; }

// v_exp_f32: 2^x without the range fix-ups of exp2f (arguments here are <= 0 or -inf)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

union Frag {
  bf16x8 v;
  u32x4 u;
  u32x2 h[2];
};

// k-operand fragment from eight accumulator registers
__device__ __forceinline__ bf16x8 frag_regs(const f32x16& a, int s, float mul) {
  Frag f;
#pragma unroll
  for (int e = 0; e < 4; ++e) f.u[e] = pack2(a[8 * s + 2 * e] * mul, a[8 * s + 2 * e + 1] * mul);
  return f.v;
}

// Eight elements of a row starting at column col, zeros where the row (D columns) has ended
template <int D>
__device__ __forceinline__ bf16x8 row_frag(const bf16_t* row, int col) {
  Frag f;
  if (col < D) f.u = *(const u32x4*)(row + col);
  else f.u = u32x4{0, 0, 0, 0};
  return f.v;
}
// Sum over the 32 lanes of each half-wavefront, left in every lane: four data-parallel-primitive steps inside
// the rows of 16 lanes (swap neighbours, swap pairs, mirror the half row, mirror the row), one exchange across rows.
__device__ __forceinline__ float half_wave_sum(float v) {
  auto dpp_add = [](float x, auto ctrl) {
    const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false);
    return x + __int_as_float(y);
  };
  v = dpp_add(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1, 0, 3, 2]
  v = dpp_add(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2, 3, 0, 1]
  v = dpp_add(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
  v = dpp_add(v, std::integral_constant<int, 0x140>{});   // row_mirror
  return v + __shfl_xor(v, 16, 64);
}

// ------------------------------------------------------------------------------- forward
// grid (seq/128, heads, batch), 256 threads; wavefront w owns queries q0+32w .. q0+32w+31
// and walks the keys in tiles made of 32-key sub-tiles (those entirely after the
// wavefront's queries are skipped).
// Workgroup -> (tile, head, batch), L its number among nt * H * batches.  Workgroup ids go round-robin over the 8 XCDs;
// all tiles of one (batch, head) are given to the same XCD, so that head's K and V are fetched into one L2 only, and the
// heaviest tile of the causal triangle goes first (heavy_high: the last tile is the heaviest).  That holds for the first
// `local` (batch, head) pairs, a multiple of eight; the others are dealt tile by tile, heaviest tiles first.
__device__ __forceinline__ int workgroup_number() { return blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z); }
__device__ __forceinline__ void attn_block(int L, int nt, int H, int hb_total, int local, int& tile, int& head, int& b,
                                           bool heavy_high) {
  const int rest = hb_total - local;
  int t, hb;
  if (L < local * nt) {
    const int slot = L / 8;
    hb = (slot / nt) * 8 + L % 8;
    t = slot % nt;
  } else {
    const int at = L - local * nt;
    hb = local + at % rest;
    t = at / rest;
  }
  tile = heavy_high ? nt - 1 - t : t;
  head = hb % H;
  b = hb / H;
}

// ------------------------------------------------------------------------- operand tiles
// Every operand tile stays as it lies in memory, as panels of 64 columns ([rows][64], 128-byte rows), fetched
// straight into LDS by direct loads (two stages, one barrier per tile) and read either by rows (ds_read_b128: the
// operand whose reduction index is the head dimension) or transposed (ds_read_b64_tr_b16: the operand whose
// reduction index is the tile's row index), so no tile is loaded twice or transposed in registers.
// 16-byte piece p of row r is stored at piece p ^ swz64(r): row reads (16 consecutive rows,
// one piece) and transposing reads (4 rows x 4 pieces) are both free of bank conflicts.
__device__ __forceinline__ int swz64(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }

// Direct loads of a [ROWS][D] tile (row pitch ld elements in memory) by WAVES wavefronts, panel by panel: the
// per-lane byte offsets (row, swizzled piece) are computed once, a panel is then a uniform base pointer plus
// those offsets.  A last panel that the head fills only in part is loaded through a buffer descriptor, whose
// lanes beyond column D bring zeros (what lies there in memory is the next head).
template <int D, int ROWS, int WAVES>
struct TileLoader {
  static constexpr int CH = ROWS / 8 / WAVES;   // 1 KiB pieces (8 rows of a panel) per wavefront
  static constexpr int WHOLE = D / 64, TAIL = D % 64, PANEL = ROWS * 128;
  static_assert(CH >= 1 && ROWS % (8 * WAVES) == 0, "tile does not divide over the wavefronts");
  static_assert(TAIL % 8 == 0, "a row is made of 16-byte pieces");
  unsigned off[CH], off_tail[TAIL ? CH : 1];
  __device__ __forceinline__ void init(size_t ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int row = 8 * (wave * CH + i) + (lane >> 3), col = ((lane & 7) ^ swz64(row)) * 8;
      off[i] = (unsigned)(((size_t)row * ld + (size_t)col) * sizeof(bf16_t));
      if (TAIL) off_tail[i] = col < TAIL ? off[i] : LOAD_NOTHING;
    }
  }
  // tile: address of the tile's first row (the same in every lane); lds: byte address of the tile in LDS
  __device__ __forceinline__ void issue(const bf16_t* tile, unsigned lds, int wave) const {
#pragma unroll
    for (int p = 0; p < WHOLE; ++p)
#pragma unroll
      for (int i = 0; i < CH; ++i) load_to_lds16_s(tile + 64 * p, off[i], lds + p * PANEL + (wave * CH + i) * 1024);
    if constexpr (TAIL != 0) {
      const u32x4 desc = buffer_desc(tile + 64 * WHOLE);
#pragma unroll
      for (int i = 0; i < CH; ++i) buffer_load_to_lds16(desc, off_tail[i], lds + WHOLE * PANEL + (wave * CH + i) * 1024);
    }
  }
};

// per-lane address parts of the two fragment kinds
struct PanelFrag {
  unsigned row_off;      // row read: lane%32 * 128
  unsigned ko[4];        // row read: byte offset of the lane's piece for k-step ks (d = 16 ks + 8 g ..)
  unsigned tro[2][2];    // transposing read: [32-wide block of the transposed rows][first / second four k]
  __device__ __forceinline__ void init(int lane) {
    const int lrow = lane & 31, g = lane >> 5, grp = lane >> 4, e4 = (lane >> 2) & 3, q4 = lane & 3;
    row_off = (unsigned)(lrow * 128);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) ko[ks] = (unsigned)(((2 * ks + g) ^ swz64(lrow)) * 16);
    // the lane supplies (tile row = base + 4 g + 8 h + e4, columns 32 i + 16 (grp % 2) + 4 q4 ..): base is a
    // multiple of 16, so the swizzle of that row is known here
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int f = ((e4 >> 1) << 2) | ((g + 2 * h) & 3);
        const int piece = (4 * i + 2 * (grp & 1) + (q4 >> 1)) ^ f;
        tro[i][h] = (unsigned)((4 * g + 8 * h + e4) * 128 + piece * 16 + (q4 & 1) * 8);
      }
  }
  // rows r0 + lane%32 of the tile (of ROWS rows), k = d in [16 ks + 8 g, +8)
  template <int ROWS>
  __device__ __forceinline__ bf16x8 rows(unsigned tile, int r0, int ks) const {
    return *(const KARMA_LDS(bf16x8)*)(uintptr_t)(tile + (unsigned)((ks >> 2) * ROWS * 128 + r0 * 128) + row_off + ko[ks & 3]);
  }
  // transposed: MFMA row = column 32 i + lane%32 of the tile, k-slots = tile rows base + 4g + {0..3, 8..11}
  template <int ROWS>
  __device__ __forceinline__ bf16x8 cols(unsigned tile, int base, int i) const {
    const unsigned at = tile + (unsigned)((i >> 1) * ROWS * 128 + base * 128);
    return read_tr_pair(at + tro[i & 1][0], at + tro[i & 1][1]);
  }
};

// Walks a workgroup's tiles with SP groups of four wavefronts, group k on tiles k, k + SP, ...; each group has two stages
// of its own and its first tile has been requested.  The first n_full tiles need no masking; n_full and n are multiples of SP.
template <int SP, class Issue, class Step>
__device__ __forceinline__ void for_tiles(int n_full, int n, int group, Issue issue, Step step) {
  auto arrive = [&](int t) {
    wait_vm<0>();            // this wavefront's share of tile t has landed
    lds_barrier_visible();   // ... and everybody's; the tile before it is no longer read
    if (t + SP < n) issue(t + SP);
  };
  for (int t = group; t < n_full; t += SP) { arrive(t); step(t, std::true_type{}); }
  for (int t = n_full + group; t < n; t += SP) { arrive(t); step(t, std::false_type{}); }
}

// Adds the accumulators of the other groups of four wavefronts to group 0's, in the groups' order, through LDS (which holds
// no tile any more).  N registers per lane; mine(r) / theirs(r, v) read and add register r.
template <int SP, int N, class Mine, class Theirs>
__device__ __forceinline__ void join_groups(float* lds, int group, int tid, Mine mine, Theirs theirs) {
#pragma unroll
  for (int o = 1; o < SP; ++o) {
    lds_barrier_visible();
    if (group == o)
#pragma unroll
      for (int r = 0; r < N; ++r) lds[r * 256 + tid] = mine(r);
    lds_barrier_visible();
    if (group == 0)
#pragma unroll
      for (int r = 0; r < N; ++r) theirs(r, lds[r * 256 + tid]);
  }
}

// SP groups of four wavefronts share the workgroup's queries; group k takes the key tiles k, k + SP, ...
template <int D, int KT, int WGS, int SP>
__global__ __launch_bounds__(256 * SP, WGS) void attn_fwd_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ ctx,
                                                                   float* __restrict__ lse, int S, int H, int local) {
  constexpr int DP = padded_d(D), NMT = KT / 32, TILE = tile_bytes(D, KT), STAGE = 2 * TILE;   // stage = K tile | V tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_attn[];
  const int h = H * D;
  const size_t ld = 3 * (size_t)h;
  int tile, head, b;
  attn_block(workgroup_number(), S / 128, H, gridDim.y * gridDim.z, local, tile, head, b, true);
  const int q0 = tile * 128;
  const int group = SP > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  const unsigned lds0 = (unsigned)(uintptr_t)((KARMA_LDS(unsigned char)*)smem_attn) + group * 2 * STAGE;
  const int tid = threadIdx.x & 255, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lrow = lane & 31, g = lane >> 5;
  const bf16_t* base = qkv + (size_t)b * S * ld + (size_t)head * D;
  const bf16_t* Kg = base + h;
  const bf16_t* Vg = base + 2 * h;
  const int qbase = q0 + 32 * w, query = qbase + lrow;
  const float c = LOG2E * rsqrtf((float)D);
  PanelFrag fr;
  fr.init(lane);

  TileLoader<D, KT, 4> tl;
  tl.init(ld, w, lane);
  auto issue = [&](int kt) {
    const unsigned st = lds0 + (kt / SP & 1) * STAGE;
    tl.issue(Kg + (size_t)kt * KT * ld, st, w);
    tl.issue(Vg + (size_t)kt * KT * ld, st + TILE, w);
  };
  const int n_kt = (q0 + 128) / KT;
  static_assert(128 / KT % SP == 0, "the groups have as many tiles each");
  issue(group);

  bf16x8 qf[DP / 16];
#pragma unroll
  for (int ks = 0; ks < DP / 16; ++ks) qf[ks] = row_frag<D>(base + (size_t)query * ld, ks * 16 + g * 8);
  f32x16 o[DP / 32];
#pragma unroll
  for (int i = 0; i < DP / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  float m = -INFINITY, l = 0.f;   // m: running maximum of the raw scores (before the 1/sqrt(d) scale)

  // One key tile.  FULL: every key precedes every query of the workgroup (all tiles but the
  // last): no masking, no skipped sub-tiles, and the sub-tiles' MFMA chains are independent
  // instruction streams the scheduler can interleave with each other and with the exponentials.
  auto tile_step = [&](int kt, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    const int key0 = kt * KT;
    const unsigned Ks = lds0 + (kt / SP & 1) * STAGE, Vs = Ks + TILE;
    // sub-tiles this wavefront needs: keys key0 + 32*mt <= last query
    const int n_mt = FULL ? NMT : min(NMT, (qbase + 31 - key0) / 32 + 1);
    f32x16 s[NMT];
    float tmax = -INFINITY;
    if (FULL) {
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[mt][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < DP / 16; ++ks)
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt)
          s[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows<KT>(Ks, mt * 32, ks), qf[ks], s[mt], 0, 0, 0);
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[mt][r]);
    } else {
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt) {
        if (mt < n_mt) {
#pragma unroll
          for (int r = 0; r < 16; ++r) s[mt][r] = 0.f;
#pragma unroll
          for (int ks = 0; ks < DP / 16; ++ks) s[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows<KT>(Ks, mt * 32, ks), qf[ks], s[mt], 0, 0, 0);
          if (key0 + mt * 32 + 31 > qbase) {   // sub-tile touches the diagonal: mask keys after the query
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int key = key0 + mt * 32 + (r >> 2) * 8 + g * 4 + (r & 3);
              if (key > query) s[mt][r] = -INFINITY;
            }
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[mt][r]);
        }
      }
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    // The reference maximum m follows the true maximum lazily: the accumulators are rescaled only when
    // some query's maximum has grown by more than 2^FWD_SLACK in the exponent's domain; until then its
    // probabilities are computed against the old reference and may reach that (harmless in fp32
    // accumulators and in bf16, whose relative precision does not depend on the magnitude; but a largest
    // probability of one is exact in bf16).
    const float m_new = fmaxf(m, tmax);
    if (__any((m_new - m) * c > AttnTiles<D>::FWD_SLACK)) {
      // (a query of a group other than the first that has met only minus infinity: nothing to rescale, and no difference to take)
      const float alpha = SP > 1 && m_new == -INFINITY ? 1.f : fast_exp2((m - m_new) * c);
      l *= alpha;
#pragma unroll
      for (int i = 0; i < DP / 32; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] *= alpha;
      m = m_new;
    }
    // A group other than the first may have met no key of a query that counts: none at all, or only scores that are minus
    // infinity or so low that m * c, rounded, is far from them.  Its probabilities are then at most one, not infinite or NaN.
    const float mc = m * c, ms = m == -INFINITY ? 0.f : m;
    float psum = 0.f;
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt) {
      if (FULL || mt < n_mt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = fast_exp2(SP > 1 ? (s[mt][r] - ms) * c : fmaf(s[mt][r], c, -mc));
          s[mt][r] = p;
          psum += p;
        }
        // O^T += V^T P^T: the probabilities' k-slots are keys 16 st + 4 g + {0..3, 8..11}, which is
        // exactly what the transposing read delivers
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          bf16x8 pf = frag_regs(s[mt], st, 1.f);
#pragma unroll
          for (int i = 0; i < DP / 32; ++i) o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.cols<KT>(Vs, mt * 32 + st * 16, i), pf, o[i], 0, 0, 0);
        }
      }
    }
    l += psum;
  };
  const int n_full = q0 / KT;   // tiles whose keys all precede the workgroup's first query
  for_tiles<SP>(n_full, n_kt, group, issue, tile_step);
  l += __shfl_xor(l, 32, 64);
  if constexpr (SP > 1) {
    // the groups' sums against the larger of two references; group 0 has met every query's first key
    float* join = (float*)smem_attn;
#pragma unroll
    for (int x = 1; x < SP; ++x) {
      lds_barrier_visible();
      if (group == x) {
        join[tid] = m;
        join[256 + tid] = l;
#pragma unroll
        for (int i = 0; i < DP / 32; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) join[(2 + i * 16 + r) * 256 + tid] = o[i][r];
      }
      lds_barrier_visible();
      if (group == 0) {
        const float m2 = join[tid], m_new = fmaxf(m, m2);
        const float mine = fast_exp2((m - m_new) * c), theirs = m2 == -INFINITY ? 0.f : fast_exp2((m2 - m_new) * c);
        l = l * mine + join[256 + tid] * theirs;
#pragma unroll
        for (int i = 0; i < DP / 32; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[i][r] = o[i][r] * mine + join[(2 + i * 16 + r) * 256 + tid] * theirs;
        m = m_new;
      }
    }
    if (group != 0) return;
  }
  const float inv = 1.f / l;
  bf16_t* out = ctx + ((size_t)b * S + query) * h + (size_t)head * D;
#pragma unroll
  for (int i = 0; i < DP / 32; ++i)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      u32x2 v;
      v.x = pack2(o[i][rg * 4 + 0] * inv, o[i][rg * 4 + 1] * inv);
      v.y = pack2(o[i][rg * 4 + 2] * inv, o[i][rg * 4 + 3] * inv);
      if (DP == D || i * 32 + rg * 8 + g * 4 < D) *(u32x2*)(out + i * 32 + rg * 8 + g * 4) = v;
    }
  if (g == 0) lse[((size_t)b * H + head) * S + query] = m * c + log2f(l);
}

// ------------------------------------------------------------------ backward: delta
// delta[b][head][q] = sum_d dO[b][q][head*D + d] * O[b][q][head*D + d], in a launch of its own where dqkv lies over ctx
__global__ __launch_bounds__(256) void attn_delta_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                                                         float* __restrict__ delta, int S, int H, int D, size_t total) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;   // (b, q, head), head fastest
  if (i >= total) return;
  const int head = (int)(i % H);
  const size_t bq = i / H, q = bq % S, b = bq / S;
  const bf16_t* po = o + (bq * H + head) * D;
  const bf16_t* pd = dout + (bq * H + head) * D;
  float acc = 0.f;
  for (int v = 0; v < D; v += 8) {
    float a[8], d[8];
    unpack8(*(const u32x4*)(po + v), a);
    unpack8(*(const u32x4*)(pd + v), d);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(a[e], d[e], acc);
  }
  delta[(b * H + head) * S + q] = acc;
}

struct AttnBwd {
  const bf16_t* qkv;
  const bf16_t* o;      // the forward's output, or null: delta is there already
  const bf16_t* dout;
  const float* lse;
  float* delta;
  bf16_t* dqkv;
  float* colsum;        // or null
  int S, H, local;      // local: see attn_block
};

// ------------------------------------------------------------------ backward: dQ
// K and V tiles as they lie in memory; K is read by
// rows for the scores and transposed for dQ^T += K^T dS^T.
// It also computes delta[q] = sum_d dO[q][d] O[q][d] for its queries (each lane holds half a row of dO
// as MFMA fragments anyway) and stores it for the dK/dV pass; without `o` it takes delta as it finds it.
// L: the workgroup's number among hb_total * S / 128.
template <int D, int KT, int SP>
__device__ __forceinline__ void attn_bwd_dq(const AttnBwd& p, int L, int hb_total, unsigned char* smem_attn) {
  constexpr int DP = padded_d(D), NMT = KT / 32, TILE = tile_bytes(D, KT), STAGE = 2 * TILE;
  const bf16_t* __restrict__ const qkv = p.qkv;
  const bf16_t* __restrict__ const o = p.o;
  const bf16_t* __restrict__ const dout = p.dout;
  const float* __restrict__ const lse = p.lse;
  float* __restrict__ const delta = p.delta;
  bf16_t* __restrict__ const dqkv = p.dqkv;
  float* __restrict__ const colsum = p.colsum;
  const int S = p.S, H = p.H, h = H * D;
  const size_t ld = 3 * (size_t)h;
  int tile, head, b;
  attn_block(L, S / 128, H, hb_total, p.local, tile, head, b, true);
  const int q0 = tile * 128;
  const int group = SP > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  const unsigned lds0 = (unsigned)(uintptr_t)((KARMA_LDS(unsigned char)*)smem_attn) + group * 2 * STAGE;
  const int tid = threadIdx.x & 255, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lrow = lane & 31, g = lane >> 5;
  const bf16_t* base = qkv + (size_t)b * S * ld + (size_t)head * D;
  const bf16_t* Kg = base + h;
  const bf16_t* Vg = base + 2 * h;
  const int qbase = q0 + 32 * w, query = qbase + lrow;
  const float scale = rsqrtf((float)D), c = LOG2E * scale;
  PanelFrag fr;
  fr.init(lane);
  TileLoader<D, KT, 4> tl;
  tl.init(ld, w, lane);
  auto issue = [&](int kt) {
    const unsigned st = lds0 + (kt / SP & 1) * STAGE;
    tl.issue(Kg + (size_t)kt * KT * ld, st, w);
    tl.issue(Vg + (size_t)kt * KT * ld, st + TILE, w);
  };
  const int n_kt = (q0 + 128) / KT;
  static_assert(128 / KT % SP == 0, "the groups have as many tiles each");
  issue(group);

  bf16x8 qf[DP / 16], dof[DP / 16];
#pragma unroll
  for (int ks = 0; ks < DP / 16; ++ks) {
    qf[ks] = row_frag<D>(base + (size_t)query * ld, ks * 16 + g * 8);
    dof[ks] = row_frag<D>(dout + ((size_t)b * S + query) * h + (size_t)head * D, ks * 16 + g * 8);
  }
  const float my_lse = lse[((size_t)b * H + head) * S + query];
  float my_delta = 0.f;
  if (o) {
#pragma unroll
    for (int ks = 0; ks < DP / 16; ++ks) {
      Frag fo, fd;
      fo.v = row_frag<D>(o + ((size_t)b * S + query) * h + (size_t)head * D, ks * 16 + g * 8);
      fd.v = dof[ks];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        my_delta = fmaf(__uint_as_float(fo.u[e] << 16), __uint_as_float(fd.u[e] << 16), my_delta);
        my_delta = fmaf(__uint_as_float(fo.u[e] & 0xffff0000u), __uint_as_float(fd.u[e] & 0xffff0000u), my_delta);
      }
    }
    my_delta += __shfl_xor(my_delta, 32, 64);   // the other half of the row
    if (g == 0 && group == 0) delta[((size_t)b * H + head) * S + query] = my_delta;
  } else {
    my_delta = delta[((size_t)b * H + head) * S + query];
  }
  f32x16 dq[DP / 32];
#pragma unroll
  for (int i = 0; i < DP / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[i][r] = 0.f;

  auto tile_step = [&](int kt, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    const int key0 = kt * KT;
    const unsigned Ks = lds0 + (kt / SP & 1) * STAGE, Vs = Ks + TILE;
    const int n_mt = FULL ? NMT : min(NMT, (qbase + 31 - key0) / 32 + 1);
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt) {
      if (FULL || mt < n_mt) {
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < DP / 16; ++ks) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows<KT>(Ks, mt * 32, ks), qf[ks], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows<KT>(Vs, mt * 32, ks), dof[ks], dp, 0, 0, 0);
        }
        const bool diag = !FULL && key0 + mt * 32 + 31 > qbase;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float p = fast_exp2(fmaf(s[r], c, -my_lse));
          if (diag) {
            const int key = key0 + mt * 32 + (r >> 2) * 8 + g * 4 + (r & 3);
            if (key > query) p = 0.f;
          }
          s[r] = p * (dp[r] - my_delta);   // dS^T (before the 1/sqrt(d) factor)
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          bf16x8 dsf = frag_regs(s, st, scale);
#pragma unroll
          for (int i = 0; i < DP / 32; ++i) dq[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.cols<KT>(Ks, mt * 32 + st * 16, i), dsf, dq[i], 0, 0, 0);
        }
      }
    }
  };
  const int n_full = q0 / KT;   // tiles whose keys all precede the workgroup's first query
  for_tiles<SP>(n_full, n_kt, group, issue, tile_step);
  if constexpr (SP > 1) {
    join_groups<SP, DP / 2>((float*)smem_attn, group, tid, [&](int r) { return dq[r / 16][r % 16]; },
                            [&](int r, float v) { dq[r / 16][r % 16] += v; });
    if (group != 0) return;
  }

  bf16_t* out = dqkv + ((size_t)b * S + query) * ld + (size_t)head * D;
#pragma unroll
  for (int i = 0; i < DP / 32; ++i)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      u32x2 v;
      v.x = pack2(dq[i][rg * 4 + 0], dq[i][rg * 4 + 1]);
      v.y = pack2(dq[i][rg * 4 + 2], dq[i][rg * 4 + 3]);
      if (DP == D || i * 32 + rg * 8 + g * 4 < D) *(u32x2*)(out + i * 32 + rg * 8 + g * 4) = v;
    }
  // Column sums of dQ over this wavefront's 32 queries (the gradient of the QKV bias, first third): the
  // queries lie on the lanes of each half-wavefront, so five exchanges per register; one row of partial sums
  // per wavefront, [batch * S / 32][3 h], added up afterwards in a fixed order.
  if (colsum) {
    float* dst = colsum + ((size_t)b * (S / 32) + qbase / 32) * ld + (size_t)head * D;
#pragma unroll
    for (int i = 0; i < DP / 32; ++i)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          t[e] = half_wave_sum(dq[i][rg * 4 + e]);
        }
        if (lrow == 0 && (DP == D || i * 32 + rg * 8 + g * 4 < D)) *(float4*)(dst + i * 32 + rg * 8 + g * 4) = make_float4(t[0], t[1], t[2], t[3]);
      }
  }
}

// ------------------------------------------------------------------ backward: dK, dV
// Wavefront w owns keys k0+32w .. +31 and walks the query tiles at or after them.  Q and dO tiles lie as in
// memory, read by rows for S = Q K^T and dP = dO V^T and transposed for dV += P^T dO, dK += dS^T Q.
// OWN_DELTA: delta of a tile's queries is taken from their rows of O and dO here (256 / QT threads a query, fetched one tile
// ahead like the log-sum-exps), for launches that do not wait for the dQ pass.
template <int D, int QT, int SP, bool OWN_DELTA>
__device__ __forceinline__ void attn_bwd_dkv(const AttnBwd& p, int L, int hb_total, unsigned char* smem_attn) {
  constexpr int DP = padded_d(D), TILE = tile_bytes(D, QT), STAGE = 2 * TILE;   // stage = Q tile | dO tile
  const bf16_t* __restrict__ const qkv = p.qkv;
  const bf16_t* __restrict__ const dout = p.dout;
  const float* __restrict__ const lse = p.lse;
  const float* __restrict__ const delta = p.delta;
  bf16_t* __restrict__ const dqkv = p.dqkv;
  float* __restrict__ const colsum = p.colsum;
  const int S = p.S, H = p.H, h = H * D;
  const size_t ld = 3 * (size_t)h;
  int tile, head, b;
  attn_block(L, S / 128, H, hb_total, p.local, tile, head, b, false);
  const int k0 = tile * 128;
  const int group = SP > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  const unsigned lds0 = (unsigned)(uintptr_t)((KARMA_LDS(unsigned char)*)smem_attn) + group * 2 * STAGE;
  float* stat = (float*)(smem_attn + SP * 2 * STAGE) + group * 4 * QT;   // [2 stages][lse | delta][QT]
  const int tid = threadIdx.x & 255, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lrow = lane & 31, g = lane >> 5;
  const bf16_t* base = qkv + (size_t)b * S * ld + (size_t)head * D;
  const bf16_t* dOg = dout + (size_t)b * S * h + (size_t)head * D;
  const float* lse_g = lse + ((size_t)b * H + head) * S;
  const float* delta_g = delta + ((size_t)b * H + head) * S;
  const int kbase = k0 + 32 * w, key = kbase + lrow;
  const float scale = rsqrtf((float)D), c = LOG2E * scale;
  PanelFrag fr;
  fr.init(lane);
  TileLoader<D, QT, 4> tlq, tlo;   // Q rows lie 3 h apart, dO rows h
  tlq.init(ld, w, lane);
  tlo.init((size_t)h, w, lane);
  auto issue = [&](int t) {   // query tile t of this workgroup: queries k0 + QT t ..
    const unsigned st = lds0 + (t / SP & 1) * STAGE;
    const int qq = k0 + t * QT;
    tlq.issue(base + (size_t)qq * ld, st, w);
    tlo.issue(dOg + (size_t)qq * h, st + TILE, w);
  };
  const int n_t = (S - k0) / QT;

  bf16x8 kf[DP / 16], vf[DP / 16];
#pragma unroll
  for (int ks = 0; ks < DP / 16; ++ks) {
    kf[ks] = row_frag<D>(base + h + (size_t)key * ld, ks * 16 + g * 8);
    vf[ks] = row_frag<D>(base + 2 * h + (size_t)key * ld, ks * 16 + g * 8);
  }
  f32x16 dk[DP / 32], dv[DP / 32];
#pragma unroll
  for (int i = 0; i < DP / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dk[i][r] = 0.f; dv[i][r] = 0.f; }
  // per-query statistics of the next tile, in registers
  constexpr int TPQ = 256 / QT, VPT = OWN_DELTA ? (D / 8 + TPQ - 1) / TPQ : 1;
  const int dq_row = tid / TPQ, dq_part = tid % TPQ;
  float lse_r = 0.f, delta_r = 0.f;
  u32x4 o_r[VPT], do_r[VPT];
  auto fetch_stats = [&](int t) {
    const int qq = k0 + t * QT;
    if (tid < QT) {
      lse_r = lse_g[qq + tid];
      if (!OWN_DELTA) delta_r = delta_g[qq + tid];
    }
    if constexpr (OWN_DELTA) {
      const size_t at = ((size_t)b * S + qq + dq_row) * h + (size_t)head * D;
#pragma unroll
      for (int v = 0; v < VPT; ++v) {
        const int col = (dq_part + v * TPQ) * 8;
        o_r[v] = col < D ? *(const u32x4*)(p.o + at + col) : u32x4{0, 0, 0, 0};
        do_r[v] = col < D ? *(const u32x4*)(dout + at + col) : u32x4{0, 0, 0, 0};
      }
    }
  };
  auto store_stats = [&](int t) {   // (the buffer was last read two of this group's tiles ago)
    float* lse_s = stat + (t / SP & 1) * 2 * QT;
    if (tid < QT) lse_s[tid] = lse_r;
    if constexpr (!OWN_DELTA) {
      if (tid < QT) lse_s[QT + tid] = delta_r;
    } else {
      float sum = 0.f;
#pragma unroll
      for (int v = 0; v < VPT; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sum = fmaf(__uint_as_float(o_r[v][e] << 16), __uint_as_float(do_r[v][e] << 16), sum);
          sum = fmaf(__uint_as_float(o_r[v][e] & 0xffff0000u), __uint_as_float(do_r[v][e] & 0xffff0000u), sum);
        }
#pragma unroll
      for (int x = 1; x < TPQ; x *= 2) sum += __shfl_xor(sum, x, 64);
      if (dq_part == 0) lse_s[QT + dq_row] = sum;
    }
  };
  static_assert(128 / QT % SP == 0, "the groups have as many tiles each");
  fetch_stats(group);
  issue(group);

  auto tile_step = [&](int t, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    const int qq0 = k0 + t * QT;
    const float* lse_s = stat + (t / SP & 1) * 2 * QT;
    const float* delta_s = lse_s + QT;
    const unsigned Qs = lds0 + (t / SP & 1) * STAGE, Os = Qs + TILE;
    // sub-tiles of 32 queries; those entirely before this wavefront's keys contribute nothing
    const int first_mt = FULL ? 0 : max(0, (kbase - qq0) / 32);
#pragma unroll
    for (int mt = 0; mt < QT / 32; ++mt) {
      if (FULL || mt >= first_mt) {
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < DP / 16; ++ks) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows<QT>(Qs, mt * 32, ks), kf[ks], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows<QT>(Os, mt * 32, ks), vf[ks], dp, 0, 0, 0);
        }
        const bool diag = !FULL && qq0 + mt * 32 < kbase + 31;
        // p in s, dS in dp (in place); the per-query statistics come four at a time
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const int qb = mt * 32 + rg * 8 + g * 4;
          const float4 l4 = *(const float4*)(lse_s + qb);
          const float4 d4 = *(const float4*)(delta_s + qb);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dl[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = rg * 4 + e;
            float p = fast_exp2(fmaf(s[r], c, -lv[e]));
            if (diag && key > qq0 + qb + e) p = 0.f;
            s[r] = p;
            dp[r] = p * (dp[r] - dl[e]);
          }
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          bf16x8 pf = frag_regs(s, st, 1.f);
          bf16x8 dsf = frag_regs(dp, st, scale);
#pragma unroll
          for (int i = 0; i < DP / 32; ++i) {
            dv[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf, fr.cols<QT>(Os, mt * 32 + st * 16, i), dv[i], 0, 0, 0);
            dk[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dsf, fr.cols<QT>(Qs, mt * 32 + st * 16, i), dk[i], 0, 0, 0);
          }
        }
      }
    }
  };
  // the first 128 queries are the workgroup's own keys (the diagonal); all later tiles lie after them
  auto arrive = [&](int t) {
    store_stats(t);   // fetched one tile ago
    wait_vm<0>();
    lds_barrier_visible();
    if (t + SP < n_t) {
      issue(t + SP);
      fetch_stats(t + SP);
    }
  };
  for (int t = group; t < 128 / QT; t += SP) { arrive(t); tile_step(t, std::false_type{}); }
  for (int t = 128 / QT + group; t < n_t; t += SP) { arrive(t); tile_step(t, std::true_type{}); }
  if constexpr (SP > 1) {
    join_groups<SP, DP>((float*)smem_attn, group, tid, [&](int r) { return r < DP / 2 ? dk[r / 16][r % 16] : dv[(r - DP / 2) / 16][r % 16]; },
                        [&](int r, float v) {
                          if (r < DP / 2) dk[r / 16][r % 16] += v;
                          else dv[(r - DP / 2) / 16][r % 16] += v;
                        });
    if (group != 0) return;
  }

  // dk[i][r]: key = kbase + (r/4)*8 + 4g + r%4, d = i*32 + lane%32
#pragma unroll
  for (int i = 0; i < DP / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int kk = kbase + (r >> 2) * 8 + g * 4 + (r & 3);
      bf16_t* row = dqkv + ((size_t)b * S + kk) * ld + (size_t)head * D + i * 32 + lrow;
      if (DP == D || i * 32 + lrow < D) {
        row[h] = f2bf(dk[i][r]);
        row[2 * h] = f2bf(dv[i][r]);
      }
    }
  // Column sums of dK and dV over this wavefront's 32 keys (second and third third of the QKV bias gradient):
  // a lane holds 16 keys of one column in its registers, the other half-wavefront the other 16.
  if (colsum) {
    float* dst = colsum + ((size_t)b * (S / 32) + kbase / 32) * ld + (size_t)head * D;
#pragma unroll
    for (int i = 0; i < DP / 32; ++i) {
      float sk = 0.f, sv = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) { sk += dk[i][r]; sv += dv[i][r]; }
      sk += __shfl_xor(sk, 32, 64);
      sv += __shfl_xor(sv, 32, 64);
      if (g == 0 && (DP == D || i * 32 + lrow < D)) {
        dst[h + i * 32 + lrow] = sk;
        dst[2 * h + i * 32 + lrow] = sv;
      }
    }
  }
}

template <int D, int KT, int WGS>
__global__ __launch_bounds__(256, WGS) void attn_bwd_dq_kernel(AttnBwd p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_attn[];
  attn_bwd_dq<D, KT, 1>(p, workgroup_number(), gridDim.y * gridDim.z, smem_attn);
}
template <int D, int QT, int WGS>
__global__ __launch_bounds__(256, WGS) void attn_bwd_dkv_kernel(AttnBwd p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_attn[];
  attn_bwd_dkv<D, QT, 1, false>(p, workgroup_number(), gridDim.y * gridDim.z, smem_attn);
}
// Both passes in one launch of twice as many workgroups, the longer dK/dV ones first
template <int D, int KT, int QT, int WGS, int SP, bool OWN_DELTA>
__global__ __launch_bounds__(256 * SP, WGS) void attn_bwd_both_kernel(AttnBwd p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_attn[];
  const int hb = gridDim.y * gridDim.z, n = p.S / 128 * hb, L = workgroup_number();
  if (L < n) attn_bwd_dkv<D, QT, SP, OWN_DELTA>(p, L, hb, smem_attn);
  else attn_bwd_dq<D, KT, SP>(p, L - n, hb, smem_attn);
}

// ------------------------------------------------------------------------------ launchers
static inline int ok() { return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP; }

// How many (batch, head) pairs stay on one XCD each, of pairs with nt tiles: all whole groups of eight; but none where the number
// is no multiple of eight and up to four workgroups for a compute unit, which all start at once, would leave one of them
// with a fifth more tiles than dealing all pairs tile by tile does.  (A unit's workgroups are 32 tiles of its XCD apart, one
// eighth of the units: with 11 tiles these are neighbours.)  us, rounds of all workgroups -> local -> this: forward 51 pairs of 11
// tiles, heads of 64 35.6 -> 39.8 -> 31.4, 13 of 31, heads of 128 106 -> 121 -> 100, backward 46 of 13, heads of 64 127 -> 130 -> 112; 85 of 9,
// heads of 64, forward 34.4 -> 30.1, as it is.
static int local_pairs(int nt, int pairs) {
  const int cus = compute_units(), apart = std::max(1, cus / 8), each = (int)(((long)nt * pairs + cus - 1) / cus);
  if (pairs % 8 == 0 || each < 2 || each > 4) return pairs / 8 * 8;
  int most = 0, even = 0;
  for (int t = 0; t < nt; ++t) {
    int sum = 0;
    for (int i = 0; i < each; ++i) sum += nt - (t + apart * i) % nt;
    most = std::max(most, sum);
  }
  for (int i = 0; i < each; ++i) even += std::max(1, nt - cus * i / pairs);
  return most * 5 >= even * 6 ? 0 : pairs / 8 * 8;
}

template <int D, int KT, int WGS, int SP>
static void launch_fwd_as(dim3 grid, hipStream_t s, const bf16_t* qkv, bf16_t* ctx, float* lse, int seq, int heads) {
  // two stages of (K tile, V tile) per group; the other groups' sums on their way to group 0
  constexpr int lds = std::max(SP * 2 * 2 * tile_bytes(D, KT), SP > 1 ? (2 + padded_d(D) / 2) * 1024 : 0);
  auto kern = attn_fwd_kernel<D, KT, WGS, SP>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  hipLaunchKernelGGL(kern, grid, dim3(256 * SP), lds, s, qkv, ctx, lse, seq, heads, local_pairs((int)grid.x, (int)(grid.y * grid.z)));
}
template <int D>
static void launch_fwd(dim3 grid, hipStream_t s, const bf16_t* qkv, bf16_t* ctx, float* lse, int seq, int heads) {
  using T = AttnTiles<D>;
  // Where no compute unit has a second workgroup, two groups of wavefronts share the key tiles of one: each walks half of
  // them and the other's MFMAs fill its gaps.  From a sweep, us, one group -> two: 1 x 16 heads x 1024 x 64 16.6 -> 14.4,
  // 2 x 16 x 512 x 64 10.1 -> 9.6, 1 x 8 x 1024 x 128 25.6 -> 22.2, 2 x 5 x 384 x 152 17.2 -> 15.1, 1 x 18 x 1536 x 152
  // 63.5 -> 48.1.  On short sequences adding the groups up takes longer than that saves (4 x 256 x 4 x 64 6.5 -> 6.9, 2 x 5
  // x 384 x 128 12.1 -> 12.6, 1 x 4 x 128 x 152 8.3 -> 9.2), and with two workgroups for a unit nothing is idle (8 x 16 x
  // 512 x 64 14.6 -> 15.6).
  const size_t wgs = (size_t)grid.x * grid.y * grid.z;
  if (wgs <= (size_t)compute_units() && seq >= T::FWD_SPLIT_SEQ) launch_fwd_as<D, T::FWD_KT, 2, 2>(grid, s, qkv, ctx, lse, seq, heads);
  else launch_fwd_as<D, T::FWD_KT, T::FWD_WGS, 1>(grid, s, qkv, ctx, lse, seq, heads);
}

int attention_fwd(const bf16_t* qkv, bf16_t* ctx, float* lse, int batch, int seq, int heads, int d, hipStream_t s) {
  if (seq % 128 || (d != 64 && d != 128 && d != 152) || batch <= 0 || heads <= 0) return KARMA_E_INVAL;
  dim3 grid(seq / 128, heads, batch);
  if (d == 64) launch_fwd<64>(grid, s, qkv, ctx, lse, seq, heads);
  else if (d == 128) launch_fwd<128>(grid, s, qkv, ctx, lse, seq, heads);
  else launch_fwd<152>(grid, s, qkv, ctx, lse, seq, heads);
  return ok();
}

template <int D, int KT, int QT, int WGS, int SP>
static void launch_bwd_both(dim3 grid, hipStream_t s, const AttnBwd& p) {
  constexpr int dq = SP * 2 * 2 * tile_bytes(D, KT), dkv = SP * (2 * 2 * tile_bytes(D, QT) + 2 * 2 * QT * 4);
  constexpr int lds = std::max({dq, dkv, SP > 1 ? padded_d(D) * 1024 : 0});
  auto kern = p.o ? attn_bwd_both_kernel<D, KT, QT, WGS, SP, true> : attn_bwd_both_kernel<D, KT, QT, WGS, SP, false>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  grid.x *= 2;
  hipLaunchKernelGGL(kern, grid, dim3(256 * SP), lds, s, p);
}
template <int D>
static void launch_bwd(dim3 grid, hipStream_t s, const AttnBwd& p) {
  using T = AttnTiles<D>;
  // Few workgroups: both passes in one launch, side by side on the chip; the dK/dV pass then takes delta from O and dO
  // itself, which larger grids would pay for again and again.  From a sweep, us, two launches -> one (with the column sums'):
  //   heads of 64, two groups of wavefronts per workgroup: 4 x 4 heads x 256 26.2 -> 15.7, 1 x 16 x 1024 60.0 -> 31.9,
  //     1 x 16 x 1536 81.5 -> 44.6 (one group 53.7; 4 x 16 x 512: two groups 32.0, one 25.2)
  //   heads of 64, one group: 4 x 12 x 384 33.2 -> 22.0, 2 x 16 x 1024 60.7 -> 39.4, 8 x 16 x 512 50.3 -> 47.5,
  //     32 x 16 x 1024 422 -> 497
  //   heads of 128: 2 x 5 x 384 43.3 -> 28.8, 1 x 8 x 1024 81.2 -> 55.4, 2 x 16 x 768 68.8 -> 56.1, 3 x 16 x 512 54.0 -> 56.3
  //   heads of 152: 2 x 5 x 384 50.4 -> 33.1, 1 x 15 x 1536 145 -> 110, 3 x 16 x 512 68.7 -> 74.6
  const size_t wgs = (size_t)grid.x * grid.y * grid.z, cus = (size_t)compute_units();
  if (wgs * 2 <= cus || (wgs * 4 <= cus * 3 && p.S >= 640)) return launch_bwd_both<D, T::DQ_KT, T::BOTH_QT, T::BOTH_WGS, T::BOTH_GROUPS>(grid, s, p);
  if constexpr (D == 64) {
    if (wgs <= 2 * cus) return launch_bwd_both<D, 64, 64, 2, 1>(grid, s, p);
  }
  constexpr int l1 = 2 * 2 * tile_bytes(D, T::DQ_KT);                             // two stages of (K tile, V tile)
  constexpr int l2 = 2 * 2 * tile_bytes(D, T::DKV_QT) + 2 * 2 * T::DKV_QT * 4;    // two stages of (Q tile, dO tile) + their lse, delta
  auto kq = attn_bwd_dq_kernel<D, T::DQ_KT, T::DQ_WGS>;
  const bool few = wgs <= cus;   // no second workgroup for one of them
  auto kkv = few ? attn_bwd_dkv_kernel<D, T::DKV_QT, T::DKV_WGS_FEW> : attn_bwd_dkv_kernel<D, T::DKV_QT, T::DKV_WGS>;
  (void)hipFuncSetAttribute((const void*)kq, hipFuncAttributeMaxDynamicSharedMemorySize, l1);
  (void)hipFuncSetAttribute((const void*)kkv, hipFuncAttributeMaxDynamicSharedMemorySize, l2);
  hipLaunchKernelGGL(kq, grid, dim3(256), l1, s, p);
  hipLaunchKernelGGL(kkv, grid, dim3(256), l2, s, p);
}

size_t attention_bwd_colsum_bytes(int batch, int seq, int heads, int d) {
  return (size_t)batch * (seq / 32) * 3 * heads * d * sizeof(float);
}

// colsum_partial (may be null) with room for attention_bwd_colsum_bytes: the kernels leave one row of column sums of
// dqkv per 32 tokens there and *colsum_rows is set to the number of rows (colsum_finish adds them up: the gradient of
// the QKV bias).
int attention_bwd(const bf16_t* qkv, const bf16_t* ctx, const bf16_t* dctx, const float* lse, float* delta,
                  bf16_t* dqkv, int batch, int seq, int heads, int d, hipStream_t s, float* colsum_partial,
                  int* colsum_rows) {
  if (seq % 128 || (d != 64 && d != 128 && d != 152) || batch <= 0 || heads <= 0) return KARMA_E_INVAL;
  dim3 grid(seq / 128, heads, batch);
  float* sums = colsum_rows ? colsum_partial : nullptr;
  const size_t tokens = (size_t)batch * seq, width = (size_t)heads * d;
  if (dqkv < ctx + tokens * width && ctx < dqkv + tokens * 3 * width) {   // gradients over the outputs: these are read first
    const size_t total = tokens * heads;
    hipLaunchKernelGGL(attn_delta_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, ctx, dctx, delta, seq, heads, d, total);
    ctx = nullptr;
  }
  const AttnBwd p{qkv, ctx, dctx, lse, delta, dqkv, sums, seq, heads, local_pairs(seq / 128, batch * heads)};
  if (d == 64) launch_bwd<64>(grid, s, p);
  else if (d == 128) launch_bwd<128>(grid, s, p);
  else launch_bwd<152>(grid, s, p);
  if (sums) *colsum_rows = batch * (seq / 32);
  return ok();
}

}  // namespace karma

using namespace karma;

extern "C" int karma_k_attention_fwd_bf16(const void* qkv, void* ctx, float* lse, uint32_t batch, uint32_t seq,
                                          uint32_t heads, uint32_t d, void* stream) {
  if (!qkv || !ctx || !lse) return KARMA_E_INVAL;
  return attention_fwd((const bf16_t*)qkv, (bf16_t*)ctx, lse, (int)batch, (int)seq, (int)heads, (int)d,
                       (hipStream_t)stream);
}

extern "C" int karma_k_attention_bwd_bf16(const void* qkv, const void* ctx, const void* dctx, const float* lse,
                                          float* delta_ws, void* dqkv, uint32_t batch, uint32_t seq, uint32_t heads,
                                          uint32_t d, void* stream) {
  if (!qkv || !ctx || !dctx || !lse || !delta_ws || !dqkv) return KARMA_E_INVAL;
  return attention_bwd((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta_ws, (bf16_t*)dqkv,
                       (int)batch, (int)seq, (int)heads, (int)d, (hipStream_t)stream, nullptr, nullptr);
}

// The same with the column sums of dqkv (the QKV bias gradient) from the kernels.
// ws: batch * seq / 32 * 3 * heads * d floats.
extern "C" int karma_k_attention_bwd_colsum_bf16(const void* qkv, const void* ctx, const void* dctx, const float* lse,
                                                 float* delta_ws, void* dqkv, float* colsum_out, float* ws, uint64_t ws_bytes,
                                                 uint32_t batch, uint32_t seq, uint32_t heads, uint32_t d, void* stream) {
  if (!qkv || !ctx || !dctx || !lse || !delta_ws || !dqkv || !colsum_out || !ws) return KARMA_E_INVAL;
  const int rows = (int)(batch * seq), cols = (int)(3 * heads * d);
  if (ws_bytes < std::max(attention_bwd_colsum_bytes((int)batch, (int)seq, (int)heads, (int)d), colsum_ws_bytes(rows, cols)))
    return KARMA_E_OOM;
  // partial sums over what the kernels still read: the sums are taken from dqkv afterwards
  const size_t used = attention_bwd_colsum_bytes((int)batch, (int)seq, (int)heads, (int)d), tensor = (size_t)rows * heads * d * sizeof(bf16_t);
  auto meets = [&](const void* p, size_t bytes) { return (const char*)ws < (const char*)p + bytes && (const char*)p < (const char*)ws + used; };
  const size_t stats = (size_t)rows * heads * sizeof(float);
  const bool over = meets(qkv, 3 * tensor) || meets(ctx, tensor) || meets(dctx, tensor) || meets(lse, stats) || meets(delta_ws, stats);
  int parts = 0;
  int st = attention_bwd((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta_ws, (bf16_t*)dqkv,
                         (int)batch, (int)seq, (int)heads, (int)d, (hipStream_t)stream, over ? nullptr : ws, over ? nullptr : &parts);
  if (st) return st;
  if (over) return colsum_bf16((const bf16_t*)dqkv, colsum_out, ws, rows, cols, (hipStream_t)stream);
  return colsum_finish(ws, parts, cols, colsum_out, (hipStream_t)stream);
}
