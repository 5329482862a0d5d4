// The bf16 product with a 128 x 128 tile: what the 256 x 256 kernel of gemm_bf16.hip leaves half of the chip idle for.
//
// A workgroup is four wavefronts of 64 x 64 and computes one (tile, range of k).  Operand tiles go global -> LDS directly
// into a ring of NST stages and are read as in the 256 x 256 kernel (XOR-swizzled 16-byte pieces, transposing reads for
// strided operands).  All loads go through a buffer descriptor: pieces outside the matrix, beyond the range of k or on a
// convolution's padding are lanes beyond the descriptor's record count, which bring zeros without a branch, so the number
// of outstanding loads is known on ragged shapes too and NST - 1 tiles stay in flight.
//   NST 2: two workgroups per compute unit (64 KB each); one multiplies while the other waits or writes out.
//   NST 4: one per compute unit, for grids that do not fill the chip: with nobody to hide behind, a k-tile's trip from
//          memory (about 2 us cold) is covered by three more tiles in flight instead.
// Measured, kernel before -> this one (gemm_bf16.hip's plan chooses): 1024 x 1024 x 256 12.3 -> 7.7 us, 3000 x 2344 x 1416
// 58.5 -> 34 us (590 TFLOP/s), 2048^3 50 -> 23 us (750 TFLOP/s); 3 x 3 convolutions 8 x 64 x 64 x 256 -> 256 80 -> 45 us
// (860 TFLOP/s).  With the chip full it multiplies at 900 to 1000 TFLOP/s: each wavefront reads 16 bytes of LDS per lane and
// MFMA, which with 64 x 64 per wavefront is all that LDS delivers; from about two rounds of large tiles on those are ahead
// (4096^3: 132 against 108 us).
// A stride-2 convolution's input gradient runs by parity of the output pixel: each parity meets a quarter of the taps (3 x 3:
// 4, 2, 2 and 1), so a quarter of the multiplications of gathering every tap for every pixel and masking three in four.
// 32 x 57 x 57, 3 x 3, 96 -> 192 channels, forward and backward with normalisation: 282 -> 123 us.
#include <hip/hip_runtime.h>
#include <cstdint>

#include "karma.h"
#include "device_utils.h"
#include "gemm_epilogue.h"
#include "gemm_ring.h"
#include "kernels.h"

namespace karma {
namespace {

struct NoConv {};
template <int CONV>
using ConvArg = std::conditional_t<CONV != 0, RingConv, NoConv>;

// The tile of a workgroup of WGM x WGN wavefronts, WGS of which (workgroups) share a compute unit
template <int BM_, int BN_, int WGM_, int WGN_, int WGS_>
struct Shape {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, WGS = WGS_;
};
using Square = Shape<RING_TILE, RING_TILE, 2, 2, 2>;
using Wide = Shape<256, RING_BROAD, 4, 1, 1>;   // wavefronts of 64 x 160
using Tall = Shape<RING_BROAD, 256, 1, 4, 1>;   // wavefronts of 160 x 64
using Slim = Shape<256, RING_SLIM, 4, 1, 2>;    // wavefronts of 64 x 64, as Square's
using Flat = Shape<RING_SLIM, 256, 1, 4, 2>;

// Where a strided operand tile of T columns keeps what.  In LDS a k-row is T / 8 pieces of 16 bytes; a transposing read takes
// four k-rows times four pieces at once, which have to lie in different banks: a row of 160 columns sees to that by itself,
// the others exchange pieces by the k-row.  256 columns: a lane would meet two columns in turn, as 1 KiB is two
// k-rows, so rows are placed such that a wavefront's all have the same k / 2 % 2.
template <int T>
struct Strided {
  static constexpr int PPR = T / 8, CH = T * RING_BK * 2 / 1024 / 4;
  static_assert(T == 64 || T == 128 || T == 160 || T == 256, "a layout below");
  // k-row and first column of lane `lane` of wavefront `wave`'s piece i
  static __device__ __forceinline__ int row(int wave, int i, int lane) {
    if (T == 256) return 32 * (wave >> 1) + 4 * i + 2 * (wave & 1) + (lane >> 5);
    return ((wave * CH + i) * 64 + lane) / PPR;
  }
  static __device__ __forceinline__ int col(int wave, int i, int lane) {
    const int k = row(wave, i, lane), p = T == 256 ? lane & 31 : ((wave * CH + i) * 64 + lane) % PPR;
    return (p ^ swizzle(k)) * 8;
  }
  static __device__ __forceinline__ int swizzle(int k) {
    return T == 160 ? 0 : T == 64 ? (k >> 1 & 1) << 2 : (k & 3) << 2;
  }
  // byte address in the tile of column m, k = 8 half + e (half 0 or 1, e below 4); k + 4 lies NEXT further, k-step kk at step(kk)
  static constexpr int NEXT = (T == 256 ? 2 : 4) * T * 2;
  static __device__ __forceinline__ unsigned at(int half, int e, int m) {
    const int r = T == 256 ? 16 * (e >> 1) + 4 * half + (e & 1) : 8 * half + e;
    return (unsigned)(r * T * 2 + ((m >> 3) ^ swizzle(e)) * 16 + (m & 7) * 2);
  }
  static __device__ __forceinline__ constexpr unsigned step(int kk) {
    return (unsigned)((T == 256 ? 32 * (kk >> 1) + 8 * (kk & 1) : 16 * kk) * T * 2);
  }
};

template <bool A_KC, bool B_KC, int ACT, int CONV, int NST, class SH>
__global__ __launch_bounds__(256, SH::WGS) void gemm_ring_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, int M_, int N,
                                                           int K_, int lda, int ldb, int splits, int k_per_split, GemmEpilogue ep,
                                                           float* __restrict__ partial, ConvArg<CONV> rc) {
  static_assert(CONV == 0 || (CONV == 1 && A_KC && B_KC) || (CONV == 2 && !A_KC && !B_KC), "the gathered forms");
  constexpr int BM = SH::BM, BN = SH::BN, BK = RING_BK, KSTEPS = BK / 16, WTM = BM / SH::WGM, WTN = BN / SH::WGN, TM = WTM / 32, TN = WTN / 32;
  static_assert(SH::WGM * SH::WGN == 4 && WTM % 32 == 0 && WTN % 32 == 0, "four wavefronts");
  constexpr int A_BYTES = BM * BK * 2, STAGE = (BM + BN) * BK * 2;
  constexpr int CH_A = BM * BK * 2 / 4096, CH_B = BN * BK * 2 / 4096, LPT = CH_A + CH_B;   // 1-KiB pieces per wavefront
  constexpr int SP = WTN + 4;
  static_assert(4 * 32 * SP * 4 <= NST * STAGE && (NST - 1) * LPT < 64, "strip fits; outstanding loads can be counted");
  static_assert(CONV != 1 || CH_A % 2 == 0, "a lane meets two values of k");
  static_assert(CONV != 2 || BN == 128 || BN == 256, "a lane meets one column");
  static_assert(SH::WGS == 1 || NST == 2 || NST == 4, "as the waits below");
  static_assert(ACT != 2 || WTN == 64, "column sums: a lane's octets lie in the same columns");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned lds0 = (unsigned)(uintptr_t)((KARMA_LDS(unsigned char)*)smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / SH::WGN, wn = wave % SH::WGN, lrow = lane & 31;
  int M = M_, K = K_;
  if constexpr (CONV == 1) {
    M = rc.p[blockIdx.y].M;
    K = rc.p[blockIdx.y].K;
    B += rc.p[blockIdx.y].b_off;
    ldb = K;
  }
  // work item: as in gemm_bf16.hip, eight contiguous ranges of (split, tile), one per XCD, tiles in bands of 8 tile rows
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN, total_tiles = tiles_m * tiles_n;
  const int total_items = total_tiles * splits, per_xcd = (total_items + 7) / 8;
  const int item = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per_xcd || item >= total_items) return;
  const int split = item / total_tiles, id = item % total_tiles;
  const int band_sz = 8 * tiles_n, first_m = (id / band_sz) * 8, rows_in_band = min(tiles_m - first_m, 8);
  const int m0 = (first_m + (id % band_sz) % rows_in_band) * BM, n0 = ((id % band_sz) / rows_in_band) * BN;
  const int kb = split * k_per_split, klen = min(K, kb + k_per_split) - kb, KT = (klen + BK - 1) / BK;

  // ---- global side: 1-KiB piece i of wavefront w is piece g = w * CH + i of the tile: rows 8 g .. + 7 of a k-contiguous
  // one (eight 16-byte pieces per row, piece p of row r stored at p ^ (r / 2) % 8), or the k-rows of a strided one that
  // Strided says.
  auto kc_row = [&](int g) { return 8 * g + (lane >> 3); };
  auto kc_col = [&](int g) { return ((lane & 7) ^ ((4 * (g & 1) + (lane >> 4)) & 7)) * 8; };
  using SA = Strided<BM>;
  using SB = Strided<BN>;
  auto a_row = [&](int i) { return A_KC ? kc_row(wave * CH_A + i) : SA::row(wave, i, lane); };
  auto a_col = [&](int i) { return A_KC ? kc_col(wave * CH_A + i) : SA::col(wave, i, lane); };
  auto b_row = [&](int i) { return B_KC ? kc_row(wave * CH_B + i) : SB::row(wave, i, lane); };
  auto b_col = [&](int i) { return B_KC ? kc_col(wave * CH_B + i) : SB::col(wave, i, lane); };
  unsigned a_off[CH_A], b_off[CH_B];
#pragma unroll
  for (int i = 0; i < CH_A; ++i)
    if (CONV != 1) a_off[i] = (m0 + (A_KC ? a_row(i) : a_col(i)) < M) ? (unsigned)(((size_t)a_row(i) * lda + a_col(i)) * 2) : LOAD_NOTHING;
#pragma unroll
  for (int i = 0; i < CH_B; ++i)
    if (CONV != 2) b_off[i] = (n0 + (B_KC ? b_row(i) : b_col(i)) < N) ? (unsigned)(((size_t)b_row(i) * ldb + b_col(i)) * 2) : LOAD_NOTHING;
  const bf16_t* a_base = CONV == 1 ? A : A + (A_KC ? (size_t)m0 * lda + kb : (size_t)kb * lda + m0);
  const bf16_t* b_base = CONV == 2 ? B : B + (B_KC ? (size_t)n0 * ldb + kb : (size_t)kb * ldb + n0);

  // The gathered tensor's geometry, in registers once: read where it is used it would be fetched from the kernel's arguments
  // again and again in the k-loop, each time waited for.
  struct Geometry { int H, W, C, S, Ho, Wo, stride, transposed; unsigned magic_s, magic_c; } cg{};
  if constexpr (CONV != 0) {
    const RingPhase& ph = rc.p[CONV == 1 ? blockIdx.y : 0];
    auto keep = [](auto v) { return (decltype(v))__builtin_amdgcn_readfirstlane((int)v); };
    cg = Geometry{keep(ph.cg.H), keep(ph.cg.W), keep(ph.cg.C), keep(ph.cg.S), keep(ph.cg.Ho), keep(ph.cg.Wo), keep(ph.cg.stride),
                  keep(ph.cg.transposed), keep(ph.magic_s), keep(rc.magic_c)};
  }
  // CONV 1: input position of tap (0, 0) for this lane's CH_A pixels and its element offset (modulo 2^32)
  int ch0[CONV == 1 ? CH_A : 1], cw0[CONV == 1 ? CH_A : 1];
  unsigned cpix[CONV == 1 ? CH_A : 1];
  // CONV 2: this lane's tap and channel are fixed; its CH_B pixels advance by BK per k-tile
  int gr = 0, gs = 0, gho[CONV == 2 ? CH_B : 1], gwo[CONV == 2 ? CH_B : 1];
  unsigned goff[CONV == 2 ? CH_B : 1];
  int adv_h = 0, adv_w = 0;
  unsigned adv_off = 0, row_off = 0, img_off = 0;
  bool g_in = false;
  if constexpr (CONV == 1) {
    const unsigned grid = (unsigned)(cg.Ho * cg.Wo);
    const int pad_y = rc.p[blockIdx.y].pad_y, pad_x = rc.p[blockIdx.y].pad_x;
#pragma unroll
    for (int i = 0; i < CH_A; ++i) {
      const unsigned row = (unsigned)(m0 + a_row(i)), img = row / grid, rem = row - img * grid;
      const int ho = (int)(rem / (unsigned)cg.Wo), wo = (int)rem - ho * cg.Wo;
      const int h = cg.transposed ? ho + pad_y : ho * cg.stride - pad_y, w = cg.transposed ? wo + pad_x : wo * cg.stride - pad_x;
      ch0[i] = (int)row < M ? h : -(1 << 20);     // (rows outside the matrix: no tap lies inside the tensor)
      cw0[i] = w;
      cpix[i] = (((unsigned)((int)img * cg.H + h)) * (unsigned)cg.W + (unsigned)w) * (unsigned)cg.C;
    }
  }
  if constexpr (CONV == 2) {
    const RingPhase& ph = rc.p[0];
    const int n = n0 + b_col(0);                  // (the same for every i)
    g_in = n < N;
    const int tap = (int)__umulhi((unsigned)n, cg.magic_c), c = n - tap * cg.C;
    const int r = cg.magic_s ? (int)__umulhi((unsigned)tap, cg.magic_s) : tap, sx = tap - r * cg.S;
    gr = r - ph.pad_y;
    gs = sx - ph.pad_x;
    const unsigned grid = (unsigned)(cg.Ho * cg.Wo);
#pragma unroll
    for (int i = 0; i < CH_B; ++i) {
      const unsigned p = (unsigned)(kb + b_row(i)), img = p / grid, rem = p - img * grid;
      gho[i] = (int)(rem / (unsigned)cg.Wo);
      gwo[i] = (int)rem - gho[i] * cg.Wo;
      goff[i] = ((((unsigned)((int)img * cg.H + gho[i] * cg.stride + gr)) * (unsigned)cg.W + (unsigned)(gwo[i] * cg.stride + gs)) *
                     (unsigned)cg.C + (unsigned)c) * 2u;
    }
    const int d_img = BK / (int)grid, d_rem = BK % (int)grid;
    adv_h = d_rem / cg.Wo;
    adv_w = d_rem % cg.Wo;
    adv_off = (((unsigned)(d_img * cg.H + adv_h * cg.stride)) * (unsigned)cg.W + (unsigned)(adv_w * cg.stride)) * (unsigned)cg.C * 2u;
    row_off = (unsigned)((cg.stride * cg.W - cg.Wo * cg.stride) * cg.C) * 2u;                  // a row on, Wo pixels back
    img_off = (unsigned)((cg.H - cg.Ho * cg.stride) * cg.W) * (unsigned)cg.C * 2u;             // an image on, Ho rows back
  }

  // A tile's loads, piece by piece.  What a tile's pieces share comes from begin_a / begin_b.
  unsigned a_to = 0, b_to = 0, c_delta[2] = {0u, 0u};
  int a_left = 0, b_left = 0, c_r[2] = {0, 0}, c_s[2] = {0, 0};
  bool c_in[2] = {false, false};
  auto begin_a = [&](int t, int stage) {
    a_to = lds0 + stage * STAGE + wave * (CH_A * 1024);
    a_left = klen - t * BK;   // k from this tile's first one on
    if constexpr (CONV == 1) {
#pragma unroll
      for (int par = 0; par < 2; ++par) {   // a lane's pieces lie at two values of k
        const int col = a_col(par), k = kb + t * BK + col;
        const int tap = (int)__umulhi((unsigned)k, cg.magic_c), c = k - tap * cg.C;
        c_r[par] = cg.magic_s ? (int)__umulhi((unsigned)tap, cg.magic_s) : tap;
        c_s[par] = tap - c_r[par] * cg.S;
        if (cg.transposed) { c_r[par] = -c_r[par]; c_s[par] = -c_s[par]; }
        c_delta[par] = (unsigned)((c_r[par] * cg.W + c_s[par]) * cg.C + c);
        c_in[par] = col < a_left;
      }
      return buffer_desc(A);
    } else {
      return buffer_desc(a_base + (A_KC ? (size_t)t * BK : (size_t)t * BK * lda));
    }
  };
  auto piece_a = [&](int i, const u32x4& a_desc) {
    if constexpr (CONV == 1) {
      const int par = i & 1;   // (& and not &&: no branches)
      const bool ok = c_in[par] & ((unsigned)(ch0[i] + c_r[par]) < (unsigned)cg.H) & ((unsigned)(cw0[i] + c_s[par]) < (unsigned)cg.W);
      buffer_load_to_lds16(a_desc, ok ? (cpix[i] + c_delta[par]) * 2u : LOAD_NOTHING, a_to + i * 1024);
    } else {
      buffer_load_to_lds16(a_desc, (A_KC ? a_col(i) : a_row(i)) < a_left ? a_off[i] : LOAD_NOTHING, a_to + i * 1024);
    }
  };
  auto begin_b = [&](int t, int stage) {
    b_to = lds0 + stage * STAGE + A_BYTES + wave * (CH_B * 1024);
    b_left = klen - t * BK;
    return buffer_desc(CONV == 2 ? B : b_base + (B_KC ? (size_t)t * BK : (size_t)t * BK * ldb));
  };
  auto piece_b = [&](int i, const u32x4& b_desc) {
    if constexpr (CONV == 2) {
      const bool ok = g_in & (b_row(i) < b_left) & ((unsigned)(gho[i] * cg.stride + gr) < (unsigned)cg.H) &
                      ((unsigned)(gwo[i] * cg.stride + gs) < (unsigned)cg.W);
      buffer_load_to_lds16(b_desc, ok ? goff[i] : LOAD_NOTHING, b_to + i * 1024);
      // the pixel this lane fetches for the next k-tile
      gwo[i] += adv_w;
      const bool cw = gwo[i] >= cg.Wo;
      gwo[i] -= cw ? cg.Wo : 0;
      gho[i] += adv_h + (cw ? 1 : 0);
      const bool chh = gho[i] >= cg.Ho;
      gho[i] -= chh ? cg.Ho : 0;
      goff[i] += adv_off + (cw ? row_off : 0u) + (chh ? img_off : 0u);
    } else {
      buffer_load_to_lds16(b_desc, (B_KC ? b_col(i) : b_row(i)) < b_left ? b_off[i] : LOAD_NOTHING, b_to + i * 1024);
    }
  };
  auto issue_a = [&](int t, int stage) {
    const u32x4 d = begin_a(t, stage);
#pragma unroll
    for (int i = 0; i < CH_A; ++i) piece_a(i, d);
  };
  auto issue_b = [&](int t, int stage) {
    const u32x4 d = begin_b(t, stage);
#pragma unroll
    for (int i = 0; i < CH_B; ++i) piece_b(i, d);
  };

  // ---- LDS side: fragment addresses as in the 256 x 256 kernel
  const int grp = lane >> 4, e4 = (lane >> 2) & 3, q4 = lane & 3;
  auto kc_frag = [&](int row0) { return (unsigned)((row0 + lrow) * (BK * 2)) + (unsigned)(((lane >> 5) ^ ((lrow >> 1) & 7)) * 16); };
  unsigned a_fb[TM], b_fb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_fb[i] = A_KC ? kc_frag(wm * WTM + i * 32) : SA::at(grp >> 1, e4, wm * WTM + i * 32 + 16 * (grp & 1) + 4 * q4);
#pragma unroll
  for (int j = 0; j < TN; ++j) b_fb[j] = B_KC ? kc_frag(wn * WTN + j * 32) : SB::at(grp >> 1, e4, wn * WTN + j * 32 + 16 * (grp & 1) + 4 * q4);
  auto read_kc = [&](unsigned tile, unsigned fb, int kk) { return *(const KARMA_LDS(bf16x8)*)(uintptr_t)(tile + (fb ^ (unsigned)(kk << 5))); };
  bf16x8 af[2][TM], bfr[2][TN];
  auto read_b = [&](int buf, int stage, int kk, int x) {
    const unsigned tb = lds0 + stage * STAGE + A_BYTES;
    bfr[buf][x] = B_KC ? read_kc(tb, b_fb[x], kk) : read_tr_pair(tb + b_fb[x] + SB::step(kk), tb + b_fb[x] + SB::step(kk) + SB::NEXT);
  };
  auto read_a = [&](int buf, int stage, int kk, int x) {
    const unsigned ta = lds0 + stage * STAGE;
    af[buf][x] = A_KC ? read_kc(ta, a_fb[x], kk) : read_tr_pair(ta + a_fb[x] + SA::step(kk), ta + a_fb[x] + SA::step(kk) + SA::NEXT);
  };
  auto read_frags = [&](int buf, int stage, int kk) {
#pragma unroll
    for (int x = 0; x < (TM > TN ? TM : TN); ++x) {
      if (x < TN) read_b(buf, stage, kk, x);
      if (x < TM) read_a(buf, stage, kk, x);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // wait until at most `tiles` of the youngest tiles' loads are outstanding
  auto wait_tiles = [&](int tiles) {
    if (NST > 3 && tiles >= 3) wait_vm<(NST > 3 ? 3 : 0) * LPT>();
    else if (NST > 2 && tiles == 2) wait_vm<(NST > 2 ? 2 : 0) * LPT>();
    else if (tiles == 1) wait_vm<LPT>();
    else wait_vm<0>();
  };
  int st = 0;
  if constexpr (SH::WGS == 1) {
    // One wavefront per SIMD: what it does beside its MFMAs is done in their shadow, some of the next step's fragments and of
    // a tile's loads after each.  A tile's first operand is requested during the last step of the tile whose stage it takes,
    // the second during the step after that; beyond the range's last tile the requests go on and bring zeros, so that how
    // many are outstanding is always the same.
    constexpr int Q = TM * TN;
#pragma unroll
    for (int t = 0; t < NST; ++t) {
      issue_a(t, t);
      if (t + 1 < NST) issue_b(t, t);
    }
    wait_vm<(NST - 2) * LPT + CH_A>();
    lds_barrier_visible();
    read_frags(0, 0, 0);
    for (int t = 0; t < KT; ++t) {
      const int stn = st + 1 == NST ? 0 : st + 1, stp = st == 0 ? NST - 1 : st - 1;
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        const int nb = (kk + 1) & 1, nst = kk + 1 < KSTEPS ? st : stn, nk = kk + 1 < KSTEPS ? kk + 1 : 0;
        u32x4 desc{};
        if (kk == KSTEPS - 1) desc = begin_a(t + NST, st);
        if (kk == 0) desc = begin_b(t + NST - 1, stp);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int i = q / TN, j = q % TN;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk & 1][j], af[kk & 1][i], acc[i][j], 0, 0, 0);
#pragma unroll
          for (int f = q * (TM + TN) / Q; f < (q + 1) * (TM + TN) / Q; ++f) {
            if (f < TN) read_b(nb, nst, nk, f);
            else read_a(nb, nst, nk, f - TN);
          }
          if (kk == KSTEPS - 1) {
#pragma unroll
            for (int f = q * CH_A / Q; f < (q + 1) * CH_A / Q; ++f) piece_a(f, desc);
          }
          if (kk == 0) {
#pragma unroll
            for (int f = q * CH_B / Q; f < (q + 1) * CH_B / Q; ++f) piece_b(f, desc);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (kk == KSTEPS - 2) {
          // the next tile has landed, for every wavefront (those behind it may be on their way); past the barrier nobody
          // reads this stage any more
          wait_vm<(NST - 2) * LPT>();
          lds_barrier_visible();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      st = stn;
    }
    wait_vm<0>();   // (the requests beyond the last tile)
  } else {
#pragma unroll
  for (int t = 0; t < NST; ++t)
    if (t < KT) { issue_a(t, t); issue_b(t, t); }
  wait_tiles(min(NST, KT) - 1);
  lds_barrier_visible();
  if (KT > 0) read_frags(0, 0, 0);
  for (int t = 0; t < KT; ++t) {
    const int stn = st + 1 == NST ? 0 : st + 1;
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      if (kk + 1 < KSTEPS) read_frags((kk + 1) & 1, st, kk + 1);
      else read_frags(0, stn, 0);   // the next tile's first step (not used after the last tile)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk & 1][j], af[kk & 1][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (kk == KSTEPS - 2 && t + 1 < KT) {
        // the next tile has landed, for every wavefront; past the barrier nobody reads this stage any more (the last
        // step's fragments have been fetched), so the tile NST further on goes into it
        wait_tiles(min(NST - 2, KT - t - 2));
        lds_barrier_visible();
        if (t + NST < KT) issue_a(t + NST, st);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (kk == KSTEPS - 1 && t + NST < KT) {
        issue_b(t + NST, st);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    st = stn;
  }
  }
  lds_barrier_visible();   // every wavefront's reads are done (and no load is in flight): the strips may overlay the stages

  // ---- epilogue as in gemm_bf16.hip: the accumulators hold the transposed tile; each wavefront parks a 32-row strip in its
  // own fp32 patch of LDS and reads it back row-contiguously
  float* strip = (float*)smem + wave * 32 * SP;
  // Octet and row of a lane in a pass: for 64 columns eight consecutive lanes read two rows' worth of alternate 16-byte units
  // (no bank is met twice) and keep their columns from pass to pass; else one octet after the other.
  constexpr int QPR = WTN / 8, PASSES = QPR / 2;
  auto octet_of = [&](int pass) { return WTN == 64 ? (lane & 3) | (((lane >> 3) & 1) << 2) : (pass * 64 + lane) % QPR; };
  auto row_of = [&](int pass) { return WTN == 64 ? pass * 8 + (((lane >> 2) & 1) | ((lane >> 4) << 1)) : (pass * 64 + lane) / QPR; };
  auto col_of = [&](int pass) { return n0 + wn * WTN + octet_of(pass) * 8; };
  const bf16_t* ein = ACT == 2 ? ep.aux : (ep.out_f32 ? nullptr : ep.residual);
  const bool fetches = ein != nullptr && splits == 1 && (ep.ldc & 7) == 0;
  auto out_row = [&](int m) {   // row of C that row m of this product is
    if constexpr (CONV == 1) {
      if (rc.out_stride == 1) return m;
      const RingPhase& ph = rc.p[blockIdx.y];
      const unsigned grid = (unsigned)(ph.cg.Ho * ph.cg.Wo), img = (unsigned)m / grid, rem = (unsigned)m - img * grid;
      const int y = (int)(rem / (unsigned)ph.cg.Wo), x = (int)rem - y * ph.cg.Wo;
      return ((int)img * rc.oh + y * rc.out_stride + ph.oy) * rc.ow + x * rc.out_stride + ph.ox;
    } else {
      return m;
    }
  };
  u32x4 pre[PASSES];
  auto fetch = [&](int i, int pass) {
    const int m = m0 + wm * WTM + i * 32 + row_of(pass), n = col_of(pass);
    return fetches && m < M && n + 8 <= N ? *(const u32x4*)(ein + (size_t)out_row(m) * ep.ldc + n) : u32x4{0, 0, 0, 0};
  };
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) pre[pass] = fetch(0, pass);
  const bool col_sums = ACT == 2 && ep.colsum != nullptr && splits == 1;
  float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(float4*)(strip + lrow * SP + j * 32 + g * 8 + (lane >> 5) * 4) =
            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int row = row_of(pass), q = octet_of(pass), m = m0 + wm * WTM + i * 32 + row, n = col_of(pass);
      const float4 v = *(const float4*)(strip + row * SP + q * 8);
      const float4 u = *(const float4*)(strip + row * SP + q * 8 + 4);
      if (splits > 1) {
        if (m < M && n < N) {
          float* dst = partial + ((size_t)split * M + m) * N + n;
          const float vv[8] = {v.x, v.y, v.z, v.w, u.x, u.y, u.z, u.w};
          if (n + 8 <= N && (N & 3) == 0) { *(float4*)dst = v; *(float4*)(dst + 4) = u; }
          else for (int e = 0; e < N - n && e < 8; ++e) dst[e] = vv[e];
        }
      } else {
        const u32x4 cur = pre[pass];
        if (i + 1 < TM) pre[pass] = fetch(i + 1, pass);
        if (m < M && n < N) ep.template octet<ACT>(out_row(m), n, min(8, N - n), v, u, fetches && n + 8 <= N, cur, col_sums, cs);
      }
    }
  }
  if (col_sums) {
    // lanes that share a column octet differ in lane bits 2, 4 and 5 (the row they take in a pass)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      cs[e] += __shfl_xor(cs[e], 4, 64);
      cs[e] += __shfl_xor(cs[e], 16, 64);
      cs[e] += __shfl_xor(cs[e], 32, 64);
    }
    const int n = col_of(0);
    if (row_of(0) == 0 && n < N) {
      float* dst = ep.colsum + ((size_t)(m0 / BM) * SH::WGM + wm) * N + n;
      *(float4*)dst = make_float4(cs[0], cs[1], cs[2], cs[3]);
      *(float4*)(dst + 4) = make_float4(cs[4], cs[5], cs[6], cs[7]);
    }
  }
}

template <bool AK, bool BKC, int ACT, int CONV, int NST, class SH>
void launch(const GemmArgs& g, const GemmEpilogue& ep, int splits, int k_per_split, const RingConv* rc, hipStream_t s) {
  constexpr int lds = NST * (SH::BM + SH::BN) * RING_BK * 2;
  static_assert(lds * SH::WGS <= 160 * 1024 || NST > 2, "the stages fit");
  auto kern = gemm_ring_kernel<AK, BKC, ACT, CONV, NST, SH>;
  if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  int rows = g.M, phases = 1;
  ConvArg<CONV> arg{};
  if constexpr (CONV != 0) {
    arg = *rc;
    if constexpr (CONV == 1) {
      phases = rc->phases;
      rows = 0;
      for (int p = 0; p < phases; ++p) rows = rows > rc->p[p].M ? rows : rc->p[p].M;
    }
  }
  const int tiles = ((rows + SH::BM - 1) / SH::BM) * ((g.N + SH::BN - 1) / SH::BN);
  hipLaunchKernelGGL(kern, dim3((unsigned)((tiles * splits + 7) / 8 * 8), (unsigned)phases), dim3(256), lds, s, g.A, g.B, g.M, g.N, g.K,
                     g.lda, g.ldb, splits, k_per_split, ep, (float*)g.ws, arg);
}

template <int NST>
void launch_form(const GemmArgs& g, const GemmEpilogue& ep, int splits, int k_per_split, const RingConv* rc, hipStream_t s) {
  if (g.conv_mode == 1) launch<true, true, 0, 1, NST, Square>(g, ep, splits, k_per_split, rc, s);
  else if (g.conv_mode == 2) launch<false, false, 0, 2, NST, Square>(g, ep, splits, k_per_split, rc, s);
  else if (g.act == 1) launch<true, true, 1, 0, NST, Square>(g, ep, splits, k_per_split, rc, s);      // the layouts were checked by the caller
  else if (g.act == 2) launch<true, false, 2, 0, NST, Square>(g, ep, splits, k_per_split, rc, s);
  else if (g.a_kc && g.b_kc) launch<true, true, 0, 0, NST, Square>(g, ep, splits, k_per_split, rc, s);
  else if (g.a_kc) launch<true, false, 0, 0, NST, Square>(g, ep, splits, k_per_split, rc, s);
  else if (g.b_kc) launch<false, true, 0, 0, NST, Square>(g, ep, splits, k_per_split, rc, s);
  else launch<false, false, 0, 0, NST, Square>(g, ep, splits, k_per_split, rc, s);
}

}  // namespace

bool gemm_ring_takes(const GemmArgs& g) {
  if (((uintptr_t)g.A % 16) || ((uintptr_t)g.B % 16)) return false;
  // 16-byte pieces are whole and aligned
  if (g.conv_mode != 1 && (g.lda % 8 || (g.a_kc ? g.K % 8 : g.M % 8))) return false;
  if (g.conv_mode != 2 && (g.ldb % 8 || (g.b_kc ? g.K % 8 : g.N % 8))) return false;
  // offsets inside a tile are 32-bit byte counts
  if (g.conv_mode != 1 && (uint64_t)g.lda * 2 * RING_TILE >= (1ull << 31)) return false;
  if (g.conv_mode != 2 && (uint64_t)g.ldb * 2 * RING_TILE >= (1ull << 31)) return false;
  if (g.conv_mode) {
    const ConvGather& cg = g.conv;
    const long pixels = (long)cg.Ho * cg.Wo;
    const uint64_t images = (uint64_t)((g.conv_mode == 1 ? g.M : g.K) / pixels);
    // the tensor is addressed by 32-bit byte offsets below LOAD_NOTHING; (tap, channel) come from reciprocals (2^32 / C + 1:
    // exact below 2^32 / C); heights and widths stay far from the mark of a row outside
    if (images * cg.H * cg.W * cg.C * 2 >= (1ull << 32) || (uint64_t)cg.R * cg.S * cg.C * cg.C >= (1ull << 31)) return false;
    if (cg.H >= (1 << 16) || cg.W >= (1 << 16) || cg.Ho >= (1 << 16) || cg.Wo >= (1 << 16) || cg.pad >= (1 << 10) || cg.R >= (1 << 10) || cg.S >= (1 << 10))
      return false;
    if (cg.transposed && cg.stride > 1 && !cg.phased) return false;
  }
  return true;
}

int gemm_ring_launch(const GemmArgs& g, const GemmEpilogue& ep, int splits, int k_per_split, bool deep, int side, const RingConv* rc,
                     hipStream_t s) {
  if (side == RING_BROAD && g.conv_mode == 1) launch<true, true, 0, 1, 3, Wide>(g, ep, splits, k_per_split, rc, s);
  else if (side == RING_BROAD && g.conv_mode == 2) launch<false, false, 0, 2, 3, Tall>(g, ep, splits, k_per_split, rc, s);
  else if (side == RING_SLIM && g.conv_mode == 1) launch<true, true, 0, 1, 2, Slim>(g, ep, splits, k_per_split, rc, s);
  else if (side == RING_SLIM && g.conv_mode == 2) launch<false, false, 0, 2, 2, Flat>(g, ep, splits, k_per_split, rc, s);
  else if (side != RING_TILE) return KARMA_E_INVAL;
  else if (deep) launch_form<4>(g, ep, splits, k_per_split, rc, s);
  else launch_form<2>(g, ep, splits, k_per_split, rc, s);
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

}  // namespace karma
