// bf16 GEMM on the CDNA4 matrix cores: C[M,N] = sum_k A(m,k) B(n,k), fp32 accumulation.
// This is the dense contraction behind every fully connected layer of the transformer
// workloads (KARMA Sec. III-C "Fully-Connected Layer": |X| x |Y| multiply-adds) and its
// two gradients (dX = dY W, dW = dY^T X).
//
// Operands may have the reduction index contiguous ("k-contiguous": A[M][K], B[N][K]) or
// strided (A[K][M], B[K][N]); strided tiles are transposed in registers on their way into
// LDS, so the MFMA loop always reads 16-byte k-runs.  v_mfma_f32_32x32x16_bf16 does the arithmetic; the workgroup ->
// tile map keeps each XCD's L2 on a compact patch of C.  Four kernels: the direct-load one below (256 x 256 tiles,
// persistent), gemm_ring.hip (128 x 128, what does not fill the chip with the large tile, and other tiles for convolutions),
// gemm_slices.hip (64 x 64, small products), and for sizes and alignments none of these takes the first one here, which
// stages tiles through registers; gemm_bf16_launch chooses.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>
#include <mutex>

#include "karma.h"
#include "device_utils.h"
#include "gemm_epilogue.h"
#include "gemm_ring.h"
#include "gemm_slices.h"
#include "kernels.h"

namespace karma {

// Persistent kernel: each workgroup walks the work items (output tile x k-split) of its
// XCD's range.  Per item: the first k-tile is already in registers (loaded while the previous
// item's results were being written out), the main loop is software-pipelined by hand
// (fragments of step kk+1 are read from LDS while the MFMAs of step kk run; the next
// k-tile's global loads are issued at the top and parked in LDS half way through), and the
// results leave through a per-wavefront LDS strip so that stores are row-contiguous.  The
// stores are not waited for: they drain while the next item computes.
// CONV 1: A is an NHWC tensor gathered through a convolution (rows = output pixels, forward
// and input-gradient passes); CONV 2: B is (reduction index = output pixels, weight gradient).
template <int BM, int BN, int BK, int WGM, int WGN, bool A_KC, bool B_KC, int CONV = 0, int ACT = 0>
__global__ __launch_bounds__(WGM* WGN * 64, (BM <= 128 && BN <= 128 ? 2 : 1)) void gemm_bf16_kernel(const bf16_t* __restrict__ A,
                                                                   const bf16_t* __restrict__ B, int M, int N, int K,
                                                                   int lda, int ldb, int tiles_m, int tiles_n,
                                                                   int splits, int k_per_split, GemmEpilogue ep,
                                                                   float* __restrict__ partial, ConvGather cg) {
  static_assert(CONV == 0 || (CONV == 1 && A_KC) || (CONV == 2 && !B_KC), "which operand a convolution gathers");
  constexpr int T = WGM * WGN * 64;
  constexpr int PITCH = BK + LDS_PAD;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int KSTEPS = BK / 16;
  static_assert(KSTEPS % 2 == 0 && KSTEPS >= 4, "fragment double buffer alternates per step; tiles are parked before the barrier of step KSTEPS-2");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* As = (bf16_t*)smem;          // [2][BM][PITCH]
  bf16_t* Bs = As + 2 * BM * PITCH;    // [2][BN][PITCH]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int lrow = lane & 31, lk = (lane >> 5) * 8;
  const int total_tiles = tiles_m * tiles_n;
  const int total_items = total_tiles * splits;

  // Work items are numbered split-major (item = split * tiles + tile) and cut into 8 equal
  // contiguous ranges, one per XCD: workgroup ids go round-robin over the XCDs, so workgroup
  // b serves range b % 8, starting at position b / 8 and advancing by gridDim.x / 8.  What
  // runs together on one XCD is then a compact patch of tiles inside one k-split (tiles are
  // walked in bands of 8 tile rows), so its L2 fetches every operand panel about once.
  const int per_xcd = (total_items + 7) / 8;
  const int xcd_first = (int)(blockIdx.x % 8) * per_xcd;
  const int xcd_step = (int)gridDim.x / 8;
  auto decode = [&](int pos, int& m0, int& n0, int& kb, int& ke, int& split) {
    const int item = xcd_first + pos;
    split = item / total_tiles;
    const int id = item % total_tiles;
    constexpr int BAND = 8;
    const int band_sz = BAND * tiles_n;
    const int first_m = (id / band_sz) * BAND;
    const int rows_in_band = min(tiles_m - first_m, BAND);
    m0 = (first_m + (id % band_sz) % rows_in_band) * BM;
    n0 = ((id % band_sz) / rows_in_band) * BN;
    kb = split * k_per_split;
    ke = min(K, kb + k_per_split);
  };
  auto valid = [&](int pos) { return pos < per_xcd && xcd_first + pos < total_items; };

  TileMover<BM, BK, T, A_KC> ma;
  TileMover<BN, BK, T, B_KC> mb;
  auto load_a = [&](int row0, int k0, int k_end, bool whole) {
    if (CONV == 1) ma.load_conv(A, cg, row0, k0, M, k_end, tid);
    else ma.load(A, lda, row0, k0, M, k_end, tid, whole);
  };
  auto load_b = [&](int row0, int k0, int k_end, bool whole) {
    if (CONV == 2) mb.load_conv(B, cg, row0, k0, N, k_end, tid);
    else mb.load(B, ldb, row0, k0, N, k_end, tid, whole);
  };
  bf16x8 af[2][TM], bfr[2][TN];
  auto read_frags = [&](int buf, int cur, int kk) {
    const bf16_t* as = As + cur * BM * PITCH + (wm * WTM + lrow) * PITCH + lk + kk * 16;
    const bf16_t* bs = Bs + cur * BN * PITCH + (wn * WTN + lrow) * PITCH + lk + kk * 16;
#pragma unroll
    for (int i = 0; i < TM; ++i) af[buf][i] = *(const bf16x8*)(as + i * 32 * PITCH);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[buf][j] = *(const bf16x8*)(bs + j * 32 * PITCH);
  };

  int pos = blockIdx.x / 8;
  if (!valid(pos)) return;
  int m0, n0, kb, ke, split;
  decode(pos, m0, n0, kb, ke, split);
  bool full = m0 + BM <= M && n0 + BN <= N && (ke - kb) % BK == 0;
  load_a(m0, kb, ke, full);
  load_b(n0, kb, ke, full);

  for (;;) {
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    lds_barrier();   // every wavefront is done with the previous item's tiles
    ma.store(As, tid);
    mb.store(Bs, tid);
    lds_barrier();
    read_frags(0, 0, 0);
    const int KT = (ke - kb + BK - 1) / BK;
    // the second k-tile starts its trip right away: a tile's loads are issued one whole
    // tile time before they are parked in LDS (half way through the tile before it is used)
    if (KT > 1) {
      load_a(m0, kb + BK, ke, full);
      load_b(n0, kb + BK, ke, full);
    }
    for (int kt = 0; kt < KT; ++kt) {
      const int cur = kt & 1;
      const bool more = kt + 1 < KT;
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        // fragments of the next step; the last step already reads the next tile (the barrier
        // after the step before it has made that tile visible and retired this one)
        if (kk + 1 < KSTEPS) read_frags((kk + 1) & 1, cur, kk + 1);
        else if (more) read_frags(0, cur ^ 1, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk & 1][j], af[kk & 1][i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // The next tile is parked in LDS half way through the current one and its registers
        // are refilled at once with the tile after next.  Transposed tiles, whose LDS writes
        // are slower, go in two halves (A after step 0, B after step 1) so that the eight
        // wavefronts' writes do not all land in the same step.
        constexpr int A_AT = 0;
        constexpr int B_AT = A_KC ? 0 : 1;
        if (kk == A_AT && more) {
          ma.store(As + (cur ^ 1) * BM * PITCH, tid);
          if (A_AT != B_AT && kt + 2 < KT) load_a(m0, kb + (kt + 2) * BK, ke, full);
        }
        if (kk == B_AT && more) {
          mb.store(Bs + (cur ^ 1) * BN * PITCH, tid);
          if (kt + 2 < KT) {
            if (A_AT == B_AT) load_a(m0, kb + (kt + 2) * BK, ke, full);
            load_b(n0, kb + (kt + 2) * BK, ke, full);
          }
        }
        if ((kk == A_AT || kk == B_AT) && more) __builtin_amdgcn_sched_barrier(0);
        if (kk == KSTEPS - 2) lds_barrier();
      }
    }
    lds_barrier();   // the last tile's reads are done: LDS is free for the epilogue

    // where the results of this item go
    const int out_m0 = m0, out_n0 = n0, out_split = split;
    // start fetching the next item's first k-tile before writing this one out
    pos += xcd_step;
    const bool have_next = valid(pos);
    if (have_next) {
      decode(pos, m0, n0, kb, ke, split);
      full = m0 + BM <= M && n0 + BN <= N && (ke - kb) % BK == 0;
      load_a(m0, kb, ke, full);
      load_b(n0, kb, ke, full);
    }

    // Epilogue through LDS (the operand tiles are dead now: the k-loop ended on a barrier).
    // The MFMAs ran with the operands exchanged, so each accumulator holds the transposed
    // tile: register r of lane l is column (r/4)*8 + (l/32)*4 + r%4 of row l%32, i.e. four
    // consecutive columns per register quad.  Each wavefront parks one 32-row strip of its
    // tile in its own fp32 [32][WTN] patch of LDS with 16-byte writes, then reads it back so
    // that a run of lanes stores one contiguous piece of a row (stores that scatter 16-byte
    // pieces over 32 rows are several times slower).  The patch is private to the wavefront,
    // whose LDS operations execute in order: no barrier in here.
    constexpr int SP = WTN + 4;   // fp32 pitch of the strip
    static_assert((size_t)WGM * WGN * 32 * SP * 4 <= (size_t)2 * (BM + BN) * PITCH * 2, "strip does not fit the tile LDS");
    float* strip = (float*)smem + wave * 32 * SP;
    constexpr int QPR = WTN / 8;              // octets per strip row
    constexpr int RPI = 64 / QPR;             // rows covered per pass of the wavefront
    static_assert(QPR >= 4 && 64 % QPR == 0 && RPI % 2 == 0 && 32 % RPI == 0, "strip read-out does not tile");
    // lane -> (octet q, row rr) such that eight consecutive lanes read two rows' worth of
    // alternate 16-byte units (conflict-free with the odd pitch in 16-byte units)
    const int q = (lane & 3) | (((lane >> 3) % (QPR / 4)) << 2);
    const int rr = ((lane >> 2) & 1) | ((lane / (2 * QPR)) << 1);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(float4*)(strip + lrow * SP + j * 32 + g * 8 + (lane >> 5) * 4) =
              make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
      const int n = out_n0 + wn * WTN + q * 8;
#pragma unroll
      for (int pass = 0; pass < 32 / RPI; ++pass) {
        const int row = pass * RPI + rr;
        const int m = out_m0 + wm * WTM + i * 32 + row;
        const float4 v = *(const float4*)(strip + row * SP + q * 8);
        const float4 u = *(const float4*)(strip + row * SP + q * 8 + 4);
        if (m < M && n < N) {
          if (splits > 1) {
            float* dst = partial + ((size_t)out_split * M + m) * N + n;
            const float vv[8] = {v.x, v.y, v.z, v.w, u.x, u.y, u.z, u.w};
            if (n + 8 <= N && (N & 3) == 0) { *(float4*)dst = v; *(float4*)(dst + 4) = u; }
            else for (int e = 0; e < N - n && e < 8; ++e) dst[e] = vv[e];
          } else {
            ep.template octet<ACT>(m, n, min(8, N - n), v, u);
          }
        }
      }
    }
    if (!have_next) break;
  }
}

// ---------------------------------------------------------------------------------------
// The same product for shapes made of whole tiles, with the two gfx950 additions that take
// the operand tiles off the vector-register path:
//  * global_load_lds_dwordx4 copies 16 bytes per lane from global memory straight into LDS
//    (lane l's piece lands at M0 + 16*l): no staging registers, no ds_write burst in which
//    all eight wavefronts stall at once, and the loads are waited for only at the single
//    barrier per k-tile;
//  * ds_read_b64_tr_b16 reads a strided operand (k-rows of m-contiguous elements) out of LDS
//    already transposed into the MFMA's 8-consecutive-k-per-lane layout, so strided tiles
//    need no register transposes either.
// LDS holds two stages of (A tile, B tile) without padding; bank conflicts are avoided by
// choosing which 16-byte piece of global memory each lane fetches (an XOR swizzle of the
// piece index with low bits of the row), undone in the fragment addresses.
// The tile stream is continuous across work items: while the last k-tile of an item is being
// multiplied, the first k-tile of the next item is already landing in the other stage; the
// epilogue's fp32 strip aliases the stage of the last tile (plus a small margin).
// EDGE: the matrix need not be made of whole tiles.  Loads go through a buffer descriptor: lanes whose piece of an operand
// tile lies outside the matrix are beyond its record count and bring zeros, so that the products they enter vanish, and a
// wavefront issues as many loads for every tile, without a branch; results outside the matrix are not stored.
// CONV 1 (with EDGE, both operands k-contiguous): A is an NHWC tensor gathered through a convolution, rows =
// pixels of the grid cg.Ho x cg.Wo, k = (tap, channel).  A 16-byte piece is eight channels of one (pixel, tap), so
// the direct load takes it from wherever the convolution reads it, and pieces that fall on padding (or on the
// holes of a strided convolution's gradient) come as zeros like pieces outside the matrix.  The pixel of each
// of a lane's rows is decoded once per work item; per k-tile only (tap, channel) of the lane's two k offsets are
// (multiplications by reciprocals: magic_c = 2^32 / C + 1, magic_s = 2^32 / S + 1, exact for the sizes admitted).
// CONV 2 (with EDGE, both operands strided): B is gathered, k = pixels of the grid cg.Ho x cg.Wo, n = (tap, channel):
// the weight gradient.  A lane's four k-rows are four pixels that change with every k-tile: each is decoded per tile
// (image by a float reciprocal with an exact correction, row and column by reciprocal multiplication: magic_w =
// 2^32 / Wo + 1, inv_grid = 1 / (Ho * Wo)).
template <int BM, int BN, int BK, int WGM, int WGN, bool A_KC, bool B_KC, int ACT = 0, bool EDGE = false, int CONV = 0>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void gemm_bf16_dl_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                                         int M, int N, int K, int lda, int ldb, int tiles_m,
                                                                         int tiles_n, int splits, int k_per_split,
                                                                         GemmEpilogue ep, float* __restrict__ partial,
                                                                         ConvGather cg, unsigned magic_c, unsigned magic_s,
                                                                         unsigned magic_w, float inv_grid) {
  static_assert(CONV == 0 || (CONV == 1 && A_KC && B_KC && EDGE && ACT == 0) || (CONV == 2 && !A_KC && !B_KC && EDGE && ACT == 0),
                "the gathered forms");
  constexpr int WAVES = WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int KSTEPS = BK / 16;
  static_assert(BK == 64 && KSTEPS == 4, "swizzles below are written for 128-byte k-rows");
  static_assert(BM == 256 && BN == 256, "strided swizzle assumes 512-byte k-rows");
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int CH_A = A_BYTES / 1024 / WAVES, CH_B = B_BYTES / 1024 / WAVES;   // 1 KiB pieces per wavefront
  constexpr int LPT = CH_A + CH_B;                                               // direct loads per lane per k-tile
  constexpr int SP = WTN + 4;
  constexpr int STRIP = WAVES * 32 * SP * 4;
  constexpr int EXTRA = STRIP > STAGE ? STRIP - STAGE : 0;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [EXTRA][stage 0][stage 1][EXTRA]
  const unsigned lds0 = (unsigned)(uintptr_t)((KARMA_LDS(unsigned char)*)smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int lrow = lane & 31;
  const int total_tiles = tiles_m * tiles_n;
  const int total_items = total_tiles * splits;
  const int per_xcd = (total_items + 7) / 8;
  const int xcd_first = (int)(blockIdx.x % 8) * per_xcd;
  const int xcd_step = (int)gridDim.x / 8;
  auto decode = [&](int pos, int& m0, int& n0, int& kb, int& ke, int& split) {
    const int item = xcd_first + pos;
    split = item / total_tiles;
    const int id = item % total_tiles;
    constexpr int BAND = 8;
    const int band_sz = BAND * tiles_n;
    const int first_m = (id / band_sz) * BAND;
    const int rows_in_band = min(tiles_m - first_m, BAND);
    m0 = (first_m + (id % band_sz) % rows_in_band) * BM;
    n0 = ((id % band_sz) / rows_in_band) * BN;
    kb = split * k_per_split;
    ke = min(K, kb + k_per_split);
  };
  auto valid = [&](int pos) { return pos < per_xcd && xcd_first + pos < total_items; };

  // ---- global side of the direct loads.  A wavefront moves CH 1-KiB pieces per operand and
  // k-tile; piece i of wavefront w is rows 32w + 8i .. +7 of a k-contiguous tile (eight
  // 16-byte pieces per 128-byte row) or k-rows 8w + 2i, +1 of a strided one (32 pieces per
  // 512-byte k-row).  The lane at LDS piece p of a row fetches global piece p ^ swizzle(row):
  //   k-contiguous: swizzle = (row / 2) % 8     strided: swizzle = (k % 4) * 4
  // Both depend on i only through its parity, so two column offsets per lane suffice.
  static_assert((BM / WAVES) % 16 == 0 && (BN / WAVES) % 16 == 0 && (BK / WAVES) % 4 == 0, "swizzle parity per piece");
  const int a_row = A_KC ? wave * (BM / WAVES) + (lane >> 3) : wave * (BK / WAVES) + (lane >> 5);
  const int b_row = B_KC ? wave * (BN / WAVES) + (lane >> 3) : wave * (BK / WAVES) + (lane >> 5);
  // byte offset of each of this lane's pieces from the tile's first element; a tile is then a uniform
  // base address (scalar registers) plus these, and issuing it costs no vector arithmetic
  unsigned a_off[CH_A], b_off[CH_B];
#pragma unroll
  for (int i = 0; i < (CH_A > CH_B ? CH_A : CH_B); ++i) {
    const int odd = i & 1;
    const int kc_col = ((lane & 7) ^ ((4 * odd + (lane >> 4)) & 7)) * 8;
    const int st_col = ((lane & 31) ^ ((2 * odd + (lane >> 5)) << 2)) * 8;
    if (i < CH_A) a_off[i] = (unsigned)(((size_t)(a_row + i * (A_KC ? 8 : 2)) * lda + (A_KC ? kc_col : st_col)) * sizeof(bf16_t));
    if (i < CH_B) b_off[i] = (unsigned)(((size_t)(b_row + i * (B_KC ? 8 : 2)) * ldb + (B_KC ? kc_col : st_col)) * sizeof(bf16_t));
  }
  // element offset of an item's k-tile 0 (the same in every lane)
  auto a_origin = [&](int m0, int kb) { return A_KC ? (size_t)m0 * lda + kb : (size_t)kb * lda + m0; };
  auto b_origin = [&](int n0, int kb) { return B_KC ? (size_t)n0 * ldb + kb : (size_t)kb * ldb + n0; };
  // EDGE: where piece i of this lane lies inside a tile: (row of the operand, k) for a k-contiguous tile,
  // (k, first of its eight rows) for a strided one; `rows` is how many rows the operand has from the tile's
  // first row on, `ks` how many k are left from the tile's first k on
  auto piece_inside = [&](bool kc, int rowbase, int i, int rows, int ks) {
    const int odd = i & 1;
    if (kc) {
      const int r = rowbase + i * 8, k = ((lane & 7) ^ ((4 * odd + (lane >> 4)) & 7)) * 8;
      return (r < rows) & (k < ks);
    }
    const int k = rowbase + i * 2, r = ((lane & 31) ^ ((2 * odd + (lane >> 5)) << 2)) * 8;
    return (r < rows) & (k < ks);
  };
  auto fetch_piece = [&](const bf16_t* base, const u32x4& desc, unsigned off, unsigned lds, bool inside) {
    if (!EDGE) load_to_lds16_s(base, off, lds);
    else buffer_load_to_lds16(desc, inside ? off : LOAD_NOTHING, lds);
  };
  // CONV: where the pixels of this lane's CH_A rows lie, for the item whose tiles are being issued (dec_m0)
  // one register per row: image << 20 | (h0 + CBIAS) << 10 | (w0 + CBIAS), (h0, w0) = top-left input position of
  // the pixel's window (or, transposed, the pixel's own position plus the padding); image 4095 = row outside the matrix
  constexpr int CBIAS = 64;   // keeps the packed coordinates non-negative
  unsigned c_pix[CONV ? CH_A : 1], c_pix_next[CONV ? CH_A : 1];   // of the current item's rows, of the next item's
  const int c_shift = cg.transposed && cg.stride == 2 ? 1 : 0, c_sign = cg.transposed ? -1 : 1;
  auto conv_decode = [&](int m0x, unsigned (&pix)[CONV ? CH_A : 1]) {
    const int grid = cg.Ho * cg.Wo;
#pragma unroll
    for (int i = 0; i < CH_A; ++i) {
      const int row = m0x + a_row + 8 * i;
      const int img = row / grid, rem = row - img * grid;
      const int ho = rem / cg.Wo, wo = rem - ho * cg.Wo;
      const int h0 = cg.transposed ? ho + cg.pad : ho * cg.stride - cg.pad;
      const int w0 = cg.transposed ? wo + cg.pad : wo * cg.stride - cg.pad;
      pix[i] = ((unsigned)(row < M ? img : 4095) << 20) | ((unsigned)(h0 + CBIAS) << 10) | (unsigned)(w0 + CBIAS);
    }
  };
  // m0 / n0: the tile's first row of the operand; k0: the item's first k; kend: its last k + 1 (EDGE only)
  // nxt (CONV): the tile belongs to the next item (whose rows were decoded into c_pix_next)
  auto issue_a = [&](int stage, size_t ao, int t, int m0 = 0, int k0 = 0, int kend = 0, bool nxt = false) {
    const unsigned sa = lds0 + EXTRA + stage * STAGE + wave * (CH_A * 1024);
    if constexpr (CONV == 1) {
      const u32x4 desc = buffer_desc(A);
#pragma unroll
      for (int i = 0; i < CH_A; ++i) {
        // (tap, channel) of this piece's k; recomputed per piece: a few multiplications against registers held
        // across the MFMA steps
        const int k = k0 + t * BK + ((lane & 7) ^ ((4 * (i & 1) + (lane >> 4)) & 7)) * 8;
        const int tap = (int)__umulhi((unsigned)k, magic_c);
        const int ch = k - tap * cg.C;
        const int r = (int)__umulhi((unsigned)tap, magic_s), sx = tap - r * cg.S;
        const unsigned px = nxt ? c_pix_next[i] : c_pix[i];
        const int img = (int)(px >> 20), h0 = (int)((px >> 10) & 1023u) - CBIAS, w0 = (int)(px & 1023u) - CBIAS;
        // (transposed: taps count backwards, and where the stride leaves holes only whole positions are in the tensor)
        const int th = h0 + r * c_sign, tw = w0 + sx * c_sign, hi = th >> c_shift, wi = tw >> c_shift;
        const bool ok = (k < kend) & (img != 4095) & !((th | tw) & c_shift) & ((unsigned)hi < (unsigned)cg.H) &
                        ((unsigned)wi < (unsigned)cg.W);   // (& and not &&: no branches)
        const unsigned off = (unsigned)(((img * cg.H + hi) * cg.W + wi) * cg.C + ch) * 2u;
        fetch_piece(A, desc, off, sa + i * 1024, ok);
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    const bf16_t* pa = A + ao + (A_KC ? (size_t)t * BK : (size_t)t * BK * lda);
    const u32x4 desc = buffer_desc(pa);
#pragma unroll
    for (int i = 0; i < CH_A; ++i)
      fetch_piece(pa, desc, a_off[i], sa + i * 1024, !EDGE || piece_inside(A_KC, a_row, i, M - m0, kend - k0 - t * BK));
  };
  auto issue_b = [&](int stage, size_t bo, int t, int n0 = 0, int k0 = 0, int kend = 0) {
    const unsigned sb = lds0 + EXTRA + stage * STAGE + A_BYTES + wave * (CH_B * 1024);
    if constexpr (CONV == 2) {
      const int grid = cg.Ho * cg.Wo;
      const u32x4 desc = buffer_desc(B);
#pragma unroll
      for (int i = 0; i < CH_B; ++i) {
        // n = (tap, channel) of this piece's eight columns
        const int n = n0 + ((lane & 31) ^ ((2 * (i & 1) + (lane >> 5)) << 2)) * 8;
        const int tap = (int)__umulhi((unsigned)n, magic_c);
        const int ch = n - tap * cg.C;
        const int r = (int)__umulhi((unsigned)tap, magic_s), sx = tap - r * cg.S;
        // its k-row is one pixel
        const int p = k0 + t * BK + b_row + 2 * i;
        int img = (int)((float)p * inv_grid);
        int rem = p - img * grid;
        if (rem < 0) { --img; rem += grid; }
        if (rem >= grid) { ++img; rem -= grid; }
        const int ho = (int)__umulhi((unsigned)rem, magic_w), wo = rem - ho * cg.Wo;
        const int hi = ho * cg.stride - cg.pad + r, wi = wo * cg.stride - cg.pad + sx;
        const bool ok = (p < kend) & (n < N) & ((unsigned)hi < (unsigned)cg.H) & ((unsigned)wi < (unsigned)cg.W);
        const unsigned off = (unsigned)(((img * cg.H + hi) * cg.W + wi) * cg.C + ch) * 2u;
        fetch_piece(B, desc, off, sb + i * 1024, ok);
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    const bf16_t* pb = B + bo + (B_KC ? (size_t)t * BK : (size_t)t * BK * ldb);
    const u32x4 desc = buffer_desc(pb);
#pragma unroll
    for (int i = 0; i < CH_B; ++i)
      fetch_piece(pb, desc, b_off[i], sb + i * 1024, !EDGE || piece_inside(B_KC, b_row, i, N - n0, kend - k0 - t * BK));
  };
  auto issue = [&](int stage, size_t ao, size_t bo, int t, int m0 = 0, int n0 = 0, int k0 = 0, int kend = 0, bool nxt = false) {
    issue_a(stage, ao, t, m0, k0, kend, nxt);
    issue_b(stage, bo, t, n0, k0, kend);
  };

  // ---- LDS side: fragment addresses (bytes from the start of the operand's tile).
  // k-contiguous: lane reads 16 bytes: row = block row + lane%32, piece (lane/32 + 2*kk) ^ swizzle.
  // strided: two transposing 8-byte reads (k + 0..3 and k + 4..7); in each group of 16 lanes,
  // lane 4e+q supplies k-row e, columns 4q..4q+3, and receives column (its index in the group),
  // k-rows 0..3: lane group g covers block rows 16*(g%2).. and k offset 8*(g/2).
  const int grp = lane >> 4, e4 = (lane >> 2) & 3, q4 = lane & 3;
  auto frag_base = [&](bool kc, int wrow0, int blk) -> unsigned {
    if (kc) return (unsigned)((wrow0 + blk * 32 + lrow) * (BK * 2));
    const int m = wrow0 + blk * 32 + 16 * (grp & 1) + 4 * q4;
    const int piece = (m >> 3) ^ (e4 << 2);
    return (unsigned)((8 * (grp >> 1) + e4) * (BM * 2) + piece * 16 + (m & 7) * 2);
  };
  const unsigned kc_k0 = (unsigned)(((lane >> 5) ^ ((lrow >> 1) & 7)) * 16);   // piece for kk = 0; kk flips bits 5-6
  unsigned a_fb[TM], b_fb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_fb[i] = frag_base(A_KC, wm * WTM, i) + (A_KC ? kc_k0 : 0u);
#pragma unroll
  for (int j = 0; j < TN; ++j) b_fb[j] = frag_base(B_KC, wn * WTN, j) + (B_KC ? kc_k0 : 0u);
  bf16x8 af[2][TM], bfr[2][TN];
  auto read_one = [&](bool kc, unsigned tile_lds, unsigned fb, int kk) -> bf16x8 {
    if (kc) return *(const KARMA_LDS(bf16x8)*)(uintptr_t)(tile_lds + (fb ^ (unsigned)(kk << 5)));
    const unsigned at = tile_lds + fb + (unsigned)(kk * 16 * (BM * 2));
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((KARMA_LDS(s16x4_t)*)(uintptr_t)at);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((KARMA_LDS(s16x4_t)*)(uintptr_t)(at + 4 * (BM * 2)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read_frags = [&](int buf, int stage, int kk) {
    const unsigned ta = lds0 + EXTRA + stage * STAGE, tb = ta + A_BYTES;
    // in the order the MFMAs below want them: (a0, b0), (a0, b1), (a1, ...), ...
#pragma unroll
    for (int x = 0; x < (TM > TN ? TM : TN); ++x) {
      if (x < TN) bfr[buf][x] = read_one(B_KC, tb, b_fb[x], kk);
      if (x < TM) af[buf][x] = read_one(A_KC, ta, a_fb[x], kk);
    }
  };

  int pos = blockIdx.x / 8;
  if (!valid(pos)) return;
  int m0, n0, kb, ke, split;
  decode(pos, m0, n0, kb, ke, split);
  size_t ao = a_origin(m0, kb), bo = b_origin(n0, kb);
  int s0 = 0;   // stage of the current item's first k-tile
  if constexpr (CONV == 1) conv_decode(m0, c_pix);
  issue(s0, ao, bo, 0, m0, n0, kb, ke);

  for (;;) {
    const int KT = EDGE ? (ke - kb + BK - 1) / BK : (ke - kb) / BK;
    // the next item, whose first k-tile is fetched while this one is still computing
    int m0n = 0, n0n = 0, kbn = 0, ken = 0, splitn = 0;
    const bool have_next = valid(pos + xcd_step);
    size_t aon = 0, bon = 0;
    if (have_next) {
      decode(pos + xcd_step, m0n, n0n, kbn, ken, splitn);
      aon = a_origin(m0n, kbn);
      bon = b_origin(n0n, kbn);
      if constexpr (CONV == 1) conv_decode(m0n, c_pix_next);
    }
    lds_barrier_visible();   // the previous item's strip (which overlays stage s0 ^ 1) has been read out by every wavefront
    if (KT > 1) issue(s0 ^ 1, ao, bo, 1, m0, n0, kb, ke);
    else if (have_next) issue(s0 ^ 1, aon, bon, 0, m0n, n0n, kbn, ken, true);
    if (KT > 1 || have_next) wait_vm<LPT>();   // everything older than the loads just issued: tile 0 has landed
    else wait_vm<0>();
    lds_barrier_visible();
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    read_frags(0, s0, 0);
    int st = s0;
    for (int kt = 0; kt < KT; ++kt) {
      const bool more = kt + 1 < KT;
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        if (kk + 1 < KSTEPS) read_frags((kk + 1) & 1, st, kk + 1);
        else read_frags(0, st ^ 1, 0);   // the next tile's first step (not used after the item's last tile)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk & 1][j], af[kk & 1][i], acc[i][j], 0, 0, 0);
        // one LDS read in the shadow of each MFMA
#pragma unroll
        for (int r = 0; r < TM + TN; ++r) {
          if (r < TM * TN) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if constexpr (TM * TN > TM + TN) __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - (TM + TN), 0);
        __builtin_amdgcn_sched_barrier(0);
        if (kk == KSTEPS - 2 && more) {
          // The next k-tile (issued one tile ago) must have landed, for every wavefront; past
          // the barrier nobody reads this stage any more (the last step's fragments were
          // fetched before this step's MFMAs), so the tile after next goes into it at once.
          wait_vm<0>();
          lds_barrier_visible();
          if (kt + 2 < KT) issue_a(st, ao, kt + 2, m0, kb, ke);
          else if (have_next) issue_a(st, aon, 0, m0n, kbn, ken, true);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (kk == KSTEPS - 1 && more) {
          if (kt + 2 < KT) issue_b(st, bo, kt + 2, n0, kb, ke);
          else if (have_next) issue_b(st, bon, 0, n0n, kbn, ken);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      st ^= 1;
    }
    lds_barrier_visible();   // the last tile's reads are done: its stage is free for the strip

    // Epilogue as in the kernel above: accumulators hold the transposed tile; each wavefront
    // parks a 32-row strip in its own fp32 patch of LDS and reads it back row-contiguously.
    float* strip = (float*)(smem + ((st ^ 1) == 0 ? 0 : EXTRA + STAGE)) + wave * 32 * SP;
    constexpr int QPR = WTN / 8;
    constexpr int RPI = 64 / QPR;
    static_assert(QPR >= 4 && 64 % QPR == 0 && RPI % 2 == 0 && 32 % RPI == 0, "strip read-out does not tile");
    const int q = (lane & 3) | (((lane >> 3) % (QPR / 4)) << 2);
    const int rr = ((lane >> 2) & 1) | ((lane / (2 * QPR)) << 1);
    // The output stage's per-element input (the residual, or with ACT 2 the saved pre-activation) is
    // fetched one strip ahead, octet by octet as the previous strip's octets are consumed, so that its
    // latency hides behind a whole strip's trip through LDS at the price of one vector per pass.
    constexpr int PASSES = 32 / RPI;
    const bf16_t* ein = ACT == 2 ? ep.aux : (ep.out_f32 ? nullptr : ep.residual);
    const bool fetch_in = ein != nullptr && splits == 1 && (ep.ldc & 7) == 0;
    const int n = n0 + wn * WTN + q * 8;
    auto fetch = [&](int i, int pass) {
      const int m = m0 + wm * WTM + i * 32 + pass * RPI + rr;
      if (EDGE && (m >= M || n >= N)) return u32x4{0, 0, 0, 0};
      return *(const u32x4*)(ein + (size_t)m * ep.ldc + n);
    };
    u32x4 pre[PASSES];
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) pre[pass] = fetch_in ? fetch(0, pass) : u32x4{0, 0, 0, 0};
    // column sums of this wavefront's part of the tile (the bias gradient of the layer whose input gradient
    // this product is): every octet of a lane lies in the same eight columns
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
        const int row = pass * RPI + rr;
        const int m = m0 + wm * WTM + i * 32 + row;
        const float4 v = *(const float4*)(strip + row * SP + q * 8);
        const float4 u = *(const float4*)(strip + row * SP + q * 8 + 4);
        const bool inside = !EDGE || (m < M && n < N);
        if (splits > 1) {
          if (inside) {
            float* dst = partial + ((size_t)split * M + m) * N + n;
            *(float4*)dst = v;
            *(float4*)(dst + 4) = u;
          }
        } else {
          const u32x4 cur = pre[pass];
          if (fetch_in && i + 1 < TM) pre[pass] = fetch(i + 1, pass);
          // (rows outside the matrix were multiplied from zeroed operand rows: they add nothing to the column sums)
          if (inside) ep.template octet<ACT>(m, n, 8, v, u, fetch_in, cur, col_sums, cs);
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
      if (rr == 0 && (!EDGE || n < N)) {
        float* dst = ep.colsum + ((size_t)(m0 / BM) * WGM + wm) * N + n;
        *(float4*)dst = make_float4(cs[0], cs[1], cs[2], cs[3]);
        *(float4*)(dst + 4) = make_float4(cs[4], cs[5], cs[6], cs[7]);
      }
    }
    if (!have_next) break;
    pos += xcd_step;
    m0 = m0n; n0 = n0n; kb = kbn; ke = ken; split = splitn;
    ao = aon; bo = bon;
    if constexpr (CONV == 1) {
#pragma unroll
      for (int i = 0; i < CH_A; ++i) c_pix[i] = c_pix_next[i];
    }
    s0 = st;
  }
}

// out = sum over splits (ascending) of partial[s], then the epilogue's conversions
__global__ void splitk_reduce_kernel(const float* __restrict__ partial, int splits, size_t mn, GemmEpilogue ep, int N) {
  size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= mn) return;
  const int cnt = (int)min((size_t)4, mn - i);
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < splits; ++s)
    for (int e = 0; e < cnt; ++e) v[e] += partial[(size_t)s * mn + i + e];
  // rows are dense (ldc == N) in the split-k path, so element i is (i / N, i % N)
  for (int e = 0; e < cnt; ++e) {
    const size_t at = i + e;
    float x = v[e];
    if (ep.bias) x += bf2f(ep.bias[at % N]);
    if (ep.out_f32) {
      float* c = (float*)ep.C;
      c[at] = ep.accumulate ? c[at] + x : x;
    } else {
      if (ep.residual) x += bf2f(ep.residual[at]);
      ((bf16_t*)ep.C)[at] = f2bf(x);
    }
  }
}

// The same reduction for many splits of a small result (weight gradients of convolutions:
// a few thousand elements, up to 256 splits): eight slices of threads each add every eighth
// partial in ascending order, then the slices are added in ascending order.  The association
// is fixed, so results are reproducible (it differs from the kernel above, which is used for
// few splits: the choice depends on the split count only).
__global__ __launch_bounds__(256) void splitk_reduce_sliced_kernel(const float* __restrict__ partial, int splits, size_t mn,
                                                                    GemmEpilogue ep, int N) {
  __shared__ float red[8][32][4];
  const int q = threadIdx.x & 31, slice = threadIdx.x >> 5;
  const size_t i = ((size_t)blockIdx.x * 32 + q) * 4;
  const int cnt = i < mn ? (int)min((size_t)4, mn - i) : 0;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = slice; s < splits; s += 8)
    for (int e = 0; e < cnt; ++e) v[e] += partial[(size_t)s * mn + i + e];
#pragma unroll
  for (int e = 0; e < 4; ++e) red[slice][q][e] = v[e];
  __syncthreads();
  if (slice != 0 || cnt == 0) return;
  for (int k = 1; k < 8; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += red[k][q][e];
  for (int e = 0; e < cnt; ++e) {
    const size_t at = i + e;
    float x = v[e];
    if (ep.bias) x += bf2f(ep.bias[at % N]);
    if (ep.out_f32) {
      float* c = (float*)ep.C;
      c[at] = ep.accumulate ? c[at] + x : x;
    } else {
      if (ep.residual) x += bf2f(ep.residual[at]);
      ((bf16_t*)ep.C)[at] = f2bf(x);
    }
  }
}

// Both reductions for rows of whole octets: 32 bytes of a partial per thread, four partials in flight, the epilogue's
// vector form.  SLICES threads share an octet (1, or 8 from 16 splits on); the orders of the sums are those above.
// With the scalar form -> with this one, product and reduction: 3000 x 2344 x 1416 in 2 ranges 63 -> 54 us,
// 1024 x 256 x 1024 in 4 ranges 13.2 -> 11.0 us.
template <int SLICES>
__global__ __launch_bounds__(256) void splitk_reduce_octets_kernel(const float* __restrict__ partial, int splits, size_t mn,
                                                                    GemmEpilogue ep, int N) {
  constexpr int PER = 256 / SLICES;
  __shared__ float4 red[SLICES > 1 ? SLICES : 1][PER][2];
  const int q = threadIdx.x % PER, slice = threadIdx.x / PER;
  const unsigned o = blockIdx.x * PER + q;
  const bool in = (size_t)o * 8 < mn;
  float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
  auto add = [](float4& a, const float4& b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; };
  if (in) {
    const float* src = partial + (size_t)o * 8;
    int s = slice;
    for (; s + 3 * SLICES < splits; s += 4 * SLICES) {
      float4 a[4], b[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4* p = (const float4*)(src + (size_t)(s + k * SLICES) * mn);
        a[k] = p[0];
        b[k] = p[1];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) { add(lo, a[k]); add(hi, b[k]); }
    }
    for (; s < splits; s += SLICES) {
      const float4* p = (const float4*)(src + (size_t)s * mn);
      add(lo, p[0]);
      add(hi, p[1]);
    }
  }
  if constexpr (SLICES > 1) {
    red[slice][q][0] = lo;
    red[slice][q][1] = hi;
    __syncthreads();
    if (slice != 0) return;
    for (int k = 1; k < SLICES; ++k) { add(lo, red[k][q][0]); add(hi, red[k][q][1]); }
  }
  if (in) {
    const unsigned per_row = (unsigned)N / 8u, m = o / per_row;
    ep.octet<0>((int)m, (int)(o - m * per_row) * 8, 8, lo, hi);
  }
}

static int g_cus = 0;
int compute_units() {
  if (!g_cus) {
    int dev = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess) g_cus = p.multiProcessorCount;
    if (g_cus <= 0) g_cus = 256;
  }
  return g_cus;
}

static void launch_reduce(const GemmArgs& g, const GemmEpilogue& ep, int splits, hipStream_t s) {
  const size_t mn = (size_t)g.M * g.N;
  if (g.N % 8 == 0 && mn < (1ull << 32)) {
    const unsigned octets = (unsigned)(mn / 8);
    if (splits >= 16)
      hipLaunchKernelGGL(splitk_reduce_octets_kernel<8>, dim3((octets + 31) / 32), dim3(256), 0, s, (const float*)g.ws, splits, mn, ep, g.N);
    else
      hipLaunchKernelGGL(splitk_reduce_octets_kernel<1>, dim3((octets + 255) / 256), dim3(256), 0, s, (const float*)g.ws, splits, mn, ep, g.N);
  } else if (splits >= 16)
    hipLaunchKernelGGL(splitk_reduce_sliced_kernel, dim3((unsigned)((mn / 4 + 31) / 32 + 1)), dim3(256), 0, s,
                       (const float*)g.ws, splits, mn, ep, g.N);
  else
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((mn / 4 + 255) / 256 + 1)), dim3(256), 0, s,
                       (const float*)g.ws, splits, mn, ep, g.N);
}

template <int BM, int BN, int BK, int WGM, int WGN, bool EDGE>
static void launch_direct(const GemmArgs& g, hipStream_t s, dim3 grid, dim3 block, int tiles_m, int tiles_n, int splits,
                          int k_per_split, const GemmEpilogue& ep) {
  if constexpr (BM == 256 && BN == 256 && BK == 64) {
    constexpr int STAGE = (BM + BN) * BK * 2, STRIP = WGM * WGN * 32 * (BN / WGN + 4) * 4;
    constexpr int EXTRA = STRIP > STAGE ? STRIP - STAGE : 0;
    const int lds = 2 * STAGE + 2 * EXTRA;
#define KARMA_DL_LAUNCH(AK, BKC, ACT)                                                                             \
  do {                                                                                                            \
    auto kern = gemm_bf16_dl_kernel<BM, BN, BK, WGM, WGN, AK, BKC, ACT, EDGE>;                                    \
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);                \
    hipLaunchKernelGGL(kern, grid, block, lds, s, g.A, g.B, g.M, g.N, g.K, g.lda, g.ldb, tiles_m, tiles_n, splits, \
                       k_per_split, ep, (float*)g.ws, g.conv, 0u, 0u, 0u, 0.f);                                   \
  } while (0)
    if (g.conv_mode) {
      if constexpr (EDGE) {
        const unsigned magic_c = (unsigned)((1ull << 32) / (unsigned)g.conv.C + 1), magic_s = (unsigned)((1ull << 32) / (unsigned)g.conv.S + 1);
        const unsigned magic_w = (unsigned)((1ull << 32) / (unsigned)g.conv.Wo + 1);
        const float inv_grid = 1.0f / (float)(g.conv.Ho * g.conv.Wo);
        if (g.conv_mode == 1) {
          auto kern = gemm_bf16_dl_kernel<BM, BN, BK, WGM, WGN, true, true, 0, true, 1>;
          (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
          hipLaunchKernelGGL(kern, grid, block, lds, s, g.A, g.B, g.M, g.N, g.K, g.lda, g.ldb, tiles_m, tiles_n, splits,
                             k_per_split, ep, (float*)g.ws, g.conv, magic_c, magic_s, magic_w, inv_grid);
        } else {
          auto kern = gemm_bf16_dl_kernel<BM, BN, BK, WGM, WGN, false, false, 0, true, 2>;
          (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
          hipLaunchKernelGGL(kern, grid, block, lds, s, g.A, g.B, g.M, g.N, g.K, g.lda, g.ldb, tiles_m, tiles_n, splits,
                             k_per_split, ep, (float*)g.ws, g.conv, magic_c, magic_s, magic_w, inv_grid);
        }
      }
    } else if (g.act == 1) KARMA_DL_LAUNCH(true, true, 1);          // the layouts were checked by the caller
    else if (g.act == 2) KARMA_DL_LAUNCH(true, false, 2);
    else if (g.a_kc && g.b_kc) KARMA_DL_LAUNCH(true, true, 0);
    else if (g.a_kc && !g.b_kc) KARMA_DL_LAUNCH(true, false, 0);
    else if (!g.a_kc && g.b_kc) KARMA_DL_LAUNCH(false, true, 0);
    else KARMA_DL_LAUNCH(false, false, 0);
#undef KARMA_DL_LAUNCH
  }
}

// How a product is cut up: tile and number of ranges of the reduction
struct GemmPlan {
  int tile;     // 256: the direct-load kernel above, 128 and 160 (RING_BROAD): gemm_ring.hip, 64: gemm_slices.hip
  int splits;
  bool deep;    // 128: four stages
  double us;    // modelled time
};

// Modelled time of a launch of the 64 x 64 tile in us: `items` workgroups of kt k-tiles each.  Up to four k-tiles two
// workgroups share a compute unit; from there on one has it to itself and its wavefronts take every fourth k-tile.
//   us, this tile / the better of the other two with its ranges added up: 1024 x 256 x 256 4.9 / 6.4, 1024 x 1024 x 256
//   5.2 / 6.6, 1024 x 256 x 1024 6.9 / 10.6, 64 x 2048 x 1000 7.0 / 10.4, 1024 x 1024 x 1024 7.6 / 11.5, 64 x 1000 x 2048 in
//   four ranges 8.1 / 10.1; 4096 x 1024 x 256 10.3 / 7.4, 2048 x 1024 x 1024 13.1 / 12.0, 2048 x 2048 x 2048 34 / 21
// SLICES_MAX_KT: as far as this was measured; a workgroup fetches as many bytes per k-tile as it multiplies 64 x 64 by.
// SLICES_TILE_MORE: where one round follows another, those of the next already fetching: 1352 x 816 x 2008 in 286 workgroups 23.2
// us, 21.0 on the 128 x 128 tile; 64 x 544 x 137384 in 693 38 and 34.
constexpr double SLICES_BASE = 1.4, SLICES_ROUND = 2.8, SLICES_TILE = 0.68, SLICES_TILE_MORE = 0.95;
constexpr int SLICES_MAX_KT = 32;
static double slices_us(long items, int kt, int cus) {
  if (kt <= SLICE_WAVES) {
    const long rounds = (items + 2l * cus - 1) / (2l * cus), rest = items - (rounds - 1) * 2l * cus;
    return SLICES_BASE + SLICES_ROUND + SLICES_TILE + 3.9 * (rounds - 1) + 0.33 * kt * std::max(0.0, (double)(rest - cus) / cus);
  }
  const long rounds = (items + cus - 1) / cus;
  return SLICES_BASE + rounds * (SLICES_ROUND + (rounds > 1 ? SLICES_TILE_MORE : SLICES_TILE) * ((kt + SLICE_WAVES - 1) / SLICE_WAVES));
}

// The same for a convolution's gathers on 256 pixels x 160 channels, one workgroup per compute unit ...
static double broad_us(long items, double kt, int cus) {
  const long full = items / cus, rest = items % cus;
  return 12.5 + 14.5 * (full + (rest ? 1 : 0) - 1) + kt * (full * 1.14 + (rest ? 0.95 + 0.19 * rest / cus : 0.0));
}
// ... and on 128 x 128, two of them
constexpr double SQUARE_GATHER = 1.15, SQUARE_GATHER_LONE = 0.85;
static double square_gather_us(long items, double kt, int cus) {
  const long full = items / (2l * cus), rest = items % (2l * cus);
  const double f = (double)rest / cus, alone = f <= 1.0 ? 0.45 + 0.15 * f : 0.8 + 0.2 * (f - 1.0);
  const double last = !rest ? 0.0 : !full ? alone : SQUARE_GATHER_LONE + (1.0 - SQUARE_GATHER_LONE) * std::max(0.0, f - 1.0);
  return 5.5 + 2.5 * (full + (rest ? 1 : 0) - 1) + kt * SQUARE_GATHER * (full + last);
}

// The cheapest of the tiles, and the number of ranges, by their modelled times in microseconds.  A round is one work
// item for every place on the chip (one per compute unit with the 256 tile, two with the 128 tile); a k-tile of 64 costs,
// in a full round and with the places of the last one partly empty, what was measured on 500 products from 64 x 1000 x
// 2048 to 8192 x 3072 x 3072 and 470 convolutions: 1.5 us down to 1.25 us for the large tile (2.0 to 1.4 where its first
// operand is gathered), 1.0 us for two workgroups of the small tile per compute unit, 0.45 to 0.6 us for one that has the
// unit to itself with four stages, 0.75 with two, 15 % more where it gathers.  The choice is 0.5 % (products, weight
// gradients) and 0.3 % (gathered first operand) behind the better tile, and no size measured was more than 5 % slower than
// with the large tile alone.  Rows of C that are no whole octets are stored element by element, unless the reduction is
// divided.  Dividing it costs a launch and two trips of M x N floats per range through memory at 5 TB/s.
//   4096 x 1024 x 1024: 256 tile, 8 ranges 46.7 us -> 128 tile 13.9 us     3072 x 3072 x 8192: 275 -> 181 us
//   3000 x 2344 x 1416: 58.5 -> 34 us     4096 x 4096 x 4096: 108 us with the 256 tile, 132 us with the 128 tile
//   4808 x 1824 x 2032 (570 small tiles, 152 large ones): 55 us with the 256 tile, 73 us with the 128 tile
//   5 x 5 convolution, stride 2, 30 x 93 x 93, 232 -> 232 channels: 190 us and 225 us
// Convolutions also have 256 pixels x 160 channels (weight gradients 160 x 256), one workgroup per compute unit: 1.14 us a
// k-tile, and 14.5 us more for every round, which begins and ends with nobody to hide behind.  us, the better of the others ->
// this one, 3 x 3: 256 x 32 x 32 x 160 -> 160 216 -> 159, 256 x 8 x 8 x 640 -> 640 153 -> 115, 256 x 16 x 16 x 320 -> 320
// 144 -> 128, its weight gradient 155 -> 138 (with room for 10 ranges; the wide residual network's records have room for 8, and
// their weight gradients of 160 channels and more stay on 128 x 128); 8 x 128 x 128 x 128 -> 128 50 -> 68, 16 x 30 x 30 x 192 -> 192 24 -> 39.
// And 256 x 64 (weight gradients 64 x 256), two workgroups per compute unit: 1.5 and 1.18 us a k-tile.  us, the better of the
// others (for 64 channels until then 256 x 64 with eight wavefronts) -> this one, 3 x 3 but for the last: 8 x 256 x 256 x 64
// -> 64 74.7 -> 69.2, 64 -> 8 (input gradient) 93 -> 59, weight gradients 8 x 256 x 256 x 64 -> 64 95 -> 76 and from 128
// channels 155 -> 115; 7 x 7 at stride 2, 64 x 224 x 224 x 8 -> 64 87 -> 78, weight gradient 99 -> 73, input gradient 698 -> 409.
// Its 256 pixels against 128 of the square tile are what the L2s have to hold until the next tap reads them again: 47 x 113 x
// 113 x 232 -> 40, 7 x 7, 2183 us, 1669 on 128 x 128; 18 x 91 x 91 x 200 -> 8 109 and 84; 27 x 142 x 142 x 104 -> 16, 5 x 5, 102 and 75; but
// 93 x 119 x 119 x 160 -> 48 464 and 572.  Of 583 convolutions to at most 64 channels that factor leaves 6 more than 3 % slower
// than on the tiles that there were before, without it 137 (by up to 36 %); of 148 to 136 and more on 256 x 160 the 7 % leave 3, without
// them 7 (by up to 8 %).
// The calculation itself takes 0.4 to 1.9 us on the host.
constexpr double L2_BYTES = 8.0 * (4 << 20);
static GemmPlan plan_product(const GemmArgs& g, bool large, bool small, bool may_split) {
  const int cus = compute_units(), k_tiles = (g.K + 63) / 64;
  const double full256 = g.conv_mode == 1 ? 2.0 : 1.5, alone256 = g.conv_mode == 1 ? 1.4 : 1.25;
  const double gather128 = g.conv_mode == 1 ? SQUARE_GATHER : 1.0, lone128 = g.conv_mode == 1 ? SQUARE_GATHER_LONE : 0.75;
  const double ragged = g.M % 256 || g.N % 256 || g.K % 64 ? 1.05 : 1.0;
  const double by_element = g.N % 8 || g.ldc % 8 ? std::min(1.0, g.M / 128.0) : 0.0;
  GemmPlan best{0, 1, false, 1e30}, square = best;
  const int max_splits = may_split ? std::min(256, std::max(1, g.K / (4 * 64))) : 1;
  for (int tile : {64, 128, RING_BROAD, 256}) {
    const bool gathers = tile == RING_BROAD || (tile == RING_SLIM && g.conv_mode);   // 256 on one side
    const bool taken = tile == 256 ? large : small && (tile == 128 || (gathers ? g.conv_mode : g.N % 8 == 0 && g.ldc % 8 == 0));
    // (sums in the order they always had: only unsplit gathers, see below, are free to take another tile)
    if (g.keep_sums && (gathers ? g.conv_mode != 1 : tile == SLICE_TILE)) continue;
    if (!taken || (tile == RING_SLIM && g.conv_mode == 1 && g.N > RING_SLIM)) continue;   // (beyond 64 channels its gathers are read twice)
    const int rows = gathers && g.conv_mode == 1 ? 256 : tile, cols = gathers && g.conv_mode == 2 ? 256 : tile;
    const long tiles = (long)((g.M + rows - 1) / rows) * ((g.N + cols - 1) / cols);
    GemmPlan own{tile, 1, false, 1e30};   // the best number of ranges with this tile ...
    double late = 0.0;                    // ... and what its k-tiles take beyond two workgroups' pace
    for (int sp = 1; sp <= (gathers && g.keep_sums ? 1 : max_splits); ++sp) {
      if (sp > 1 && ((uint64_t)sp * g.M * g.N * sizeof(float) > g.ws_bytes || tiles * sp > 8l * cus)) break;
      const int kt = (k_tiles + sp - 1) / sp;
      const long items = tiles * sp, places = tile >= RING_BROAD ? cus : 2l * cus, full = items / places, rest = items % places;
      const long rounds = full + (rest ? 1 : 0);
      const double f = (double)rest / cus;   // workgroups per compute unit in the last round
      double us, more = 0.0;
      if (tile == RING_SLIM && g.conv_mode) {
        // pixels are read again for the tap after the next `stride` ones: by then gone where the chip's do not fit its L2s
        const int apart = g.conv_mode == 1 && !g.conv.transposed ? g.conv.stride : 1;
        const double fill = g.conv_mode == 1 ? std::min(items, places) * 256.0 * g.conv.C * 2 * apart / L2_BYTES : 0.0;
        const double again = 1.0 + std::min(0.8, 1.5 * std::max(0.0, fill - 1.0));
        const double slim = again * (g.conv_mode == 1 ? 1.5 : 1.18), lone = again * (g.conv_mode == 1 ? 0.75 : 0.85);   // (full, and next to alone)
        us = 5.5 + 2.5 * (rounds - 1) + kt * (full * slim + (!rest ? 0.0 : f <= 1.0 ? lone + 0.15 * f : lone + 0.15 + (slim - lone - 0.15) * (f - 1.0)));
      } else if (tile == 64) {
        if (kt > SLICES_MAX_KT) continue;
        us = slices_us(items, kt, cus) + 0.4 + 0.09 * kt;   // (by which the small tile's figure below is too high at few k-tiles)
      } else if (tile == RING_BROAD) {
        us = (g.conv_mode == 1 ? 1.07 : 1.0) * broad_us(items, kt, cus);   // (in doubt the other tiles)
      } else if (tile == 256) {
        us = 9.0 + 4.0 * (rounds - 1) + ragged * kt * (full * full256 + (rest ? alone256 + (full256 - alone256) * f : 0.0));
      } else {
        const double last = !rest ? 0.0 : f <= 1.0 ? 0.45 + 0.15 * f : 0.8 + 0.2 * (f - 1.0);
        const double slow = !rest || !full ? last : lone128 + (1.0 - lone128) * std::max(0.0, f - 1.0);
        us = 5.5 + 2.5 * (rounds - 1) + kt * (full + last);
        more = kt * (gather128 * (full + slow) - (full + last));
        if (sp == 1) us += by_element * (14.0 + 17.5 * (rounds - 1));
      }
      if (sp > 1) us += 3.5 + (double)sp * g.M * g.N * 8.0 / 5e6;
      // (four stages instead of two: 1000 x 1000 x 4000 in 33 us instead of 47, one k-tile in flight per workgroup having
      // nobody to hide behind; below 24 k-tiles per item there is no difference)
      if (us < own.us) {
        own = GemmPlan{tile, sp, items <= cus && kt >= 24, us};
        late = more;
      }
    }
    own.us += late;
    if (own.us < best.us) best = own;
    if (!gathers && own.us < square.us) square = own;
  }
  // keep_sums: ranges only as the two square tiles would have them.  A tile alone doesn't change a sum, its ranges do.  A step of
  // 4 bottleneck blocks, 64 images of 224 x 224: 4535 us so, 4458 us free, but by then 2 % of its update apart at small batches.
  if (g.keep_sums && square.splits > 1 && square.us < 1e30) return square;
  return best;
}

// Rows m0 .. m0 + m - 1 and columns n0 .. n0 + n - 1 of a product
static GemmArgs block_of(const GemmArgs& g, int m0, int m, int n0, int n) {
  GemmArgs b = g;
  const size_t at = (size_t)m0 * g.ldc + n0;
  b.M = m;
  b.N = n;
  b.A += g.a_kc ? (size_t)m0 * g.lda : (size_t)m0;
  b.B += g.b_kc ? (size_t)n0 * g.ldb : (size_t)n0;
  b.C = g.out_f32 ? (void*)((float*)g.C + at) : (void*)((bf16_t*)g.C + at);
  if (g.bias) b.bias += n0;
  if (g.residual) b.residual += at;
  if (g.aux) b.aux = (bf16_t*)g.aux + at;
  return b;
}
// What the large tile's piece offsets and loads need of a dense product
static bool large_tile_takes(const GemmArgs& g) {
  // (a lane's piece offsets inside a tile are kept as 32-bit byte counts; tiles that hang over the matrix pay for a
  // whole tile)
  return g.M % 8 == 0 && g.N % 8 == 0 && g.K % 8 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 && ((uintptr_t)g.A % 16) == 0 &&
         ((uintptr_t)g.B % 16) == 0 && g.ldc % 8 == 0 && (uint64_t)g.lda * 2 * 256 < (1ull << 31) &&
         (uint64_t)g.ldb * 2 * 256 < (1ull << 31) && g.M >= 256 && g.N >= 256 && g.K >= 128;
}

static GemmEpilogue epilogue_of(const GemmArgs& g) {
  return GemmEpilogue{g.C, g.bias, g.residual, g.ldc, g.out_f32, g.accumulate, (bf16_t*)g.aux, nullptr};
}
// Column sums of the result, `rows` partial rows of them, where the caller asked for them and gave room
static void take_colsum(const GemmArgs& g, int rows, GemmEpilogue& ep) {
  if (g.act != 2 || !g.colsum_partial || !g.colsum_rows || g.ldc != g.N || g.N % 8 || (size_t)rows * g.N * sizeof(float) > g.colsum_bytes) return;
  ep.colsum = g.colsum_partial;
  *g.colsum_rows = rows;
}
// k per range: whole k-tiles, and the number of ranges that are then not empty
static int range_length(int K, int& splits) {
  const int len = ((K + splits - 1) / splits + 63) / 64 * 64;
  splits = (K + len - 1) / len;
  return len;
}
static int finish(const GemmArgs& g, const GemmEpilogue& ep, int splits, hipStream_t s) {
  if (splits > 1) launch_reduce(g, ep, splits, s);
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

// The direct-load kernel with the 256 x 256 tile; eligibility was checked by the caller.
static int launch_large(const GemmArgs& g, int splits, hipStream_t s) {
  constexpr int BM = 256, BN = 256, BK = 64, WGM = 2, WGN = 4;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int k_per_split = range_length(g.K, splits);
  GemmEpilogue ep = epilogue_of(g);
  if (splits == 1) take_colsum(g, tiles_m * WGM, ep);
  // a multiple of 8 workgroups, at most what runs at once: the kernel deals work items out per XCD
  const dim3 grid(std::min((tiles_m * tiles_n * splits + 7) / 8 * 8, std::max(8, compute_units() / 8 * 8))), block(WGM * WGN * 64);
  if (!g.conv_mode && g.M % BM == 0 && g.N % BN == 0 && g.K % BK == 0)
    launch_direct<BM, BN, BK, WGM, WGN, false>(g, s, grid, block, tiles_m, tiles_n, splits, k_per_split, ep);
  else
    launch_direct<BM, BN, BK, WGM, WGN, true>(g, s, grid, block, tiles_m, tiles_n, splits, k_per_split, ep);
  return finish(g, ep, splits, s);
}

// The register-staged kernel's work: its tile leaves room for `places` workgroups on the chip at a time
struct GeneralPlan {
  int tiles_m, tiles_n, places, splits;
};
static GeneralPlan plan_general(const GemmArgs& g, int tile) {
  GeneralPlan p{(g.M + tile - 1) / tile, (g.N + tile - 1) / tile, compute_units() * (tile == 128 ? 2 : 1), 1};
  const int tiles = p.tiles_m * p.tiles_n;
  // split the reduction when the tiles alone cannot fill the chip (weight gradients: small M x N, K = tokens); partial
  // sums are reduced in a fixed order afterwards
  if (g.ws && g.ldc == g.N && tiles < p.places && !g.act) {
    // the split count that best fills whole rounds of the chip, fewer splits preferred: every split writes and re-reads
    // an M x N fp32 partial, which is weighed against the operand bytes of the whole product
    const int max_splits = std::min(256, std::max(1, g.K / (4 * 64)));
    const double per_split = std::min(0.01, 0.5 * (8.0 * g.M * g.N) / (2.0 * ((double)g.M + g.N) * g.K));
    double best = -1.0;
    for (int sp = 1; sp <= max_splits; ++sp) {
      if (sp > 1 && (size_t)sp * g.M * g.N * sizeof(float) > g.ws_bytes) break;
      const int items = tiles * sp, rounds = (items + p.places - 1) / p.places;
      const double score = (double)items / ((double)rounds * p.places) - per_split * sp;
      if (score > best) { best = score; p.splits = sp; }
    }
  }
  return p;
}

// Modelled time in us: what a round costs beside its k-tiles (more where the rows of C are no whole octets and are stored
// element by element), and a k-tile in a full round and in one with few of the places taken, with the number of strided
// operands, which are transposed on their way.  Fitted to 250 sizes, within 17 % (rms); the choice by it is 0.5 % behind
// the better tile.
static double general_us(const GemmArgs& g, const GeneralPlan& p, int tile) {
  const bool scalar = g.N % 8 != 0, large = tile == 256;
  const int strided = !g.a_kc + !g.b_kc;
  const long items = (long)p.tiles_m * p.tiles_n * p.splits, full = items / p.places, rest = items % p.places;
  const int kt = ((g.K + 63) / 64 + p.splits - 1) / p.splits;
  const double first = large ? (scalar ? 41.0 : 10.0) : (scalar ? 19.5 : 5.5);
  const double next = large ? (scalar ? 46.5 : 10.5) : (scalar ? 22.0 : 4.5);
  const double k_full = large ? 2.15 : 1.25 + 0.27 * strided, k_few = large ? 1.65 + 0.26 * strided : 0.72 + 0.32 * strided;
  double us = first + next * (full + (rest ? 1 : 0) - 1) + kt * (full * k_full + (rest ? k_few + (k_full - k_few) * rest / p.places : 0.0));
  if (p.splits > 1) us += 3.5 + (double)p.splits * g.M * g.N * 8.0 / 5e6;
  return us;
}

template <int BM, int BN, int WGM, int WGN>
static int launch_general(const GemmArgs& g, int splits, hipStream_t s) {
  constexpr int BK = 64;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN, tiles = tiles_m * tiles_n;
  const int cus = compute_units() * (BM == 128 ? 2 : 1);
  const int k_per_split = range_length(g.K, splits);
  const size_t lds = (size_t)2 * (BM + BN) * (BK + LDS_PAD) * sizeof(bf16_t);
  GemmEpilogue ep = epilogue_of(g);
  const dim3 grid(std::min((tiles * splits + 7) / 8 * 8, std::max(8, cus / 8 * 8))), block(WGM * WGN * 64);
#define KARMA_GEMM_LAUNCH(AK, BKC, CV, ACT)                                                             \
  do {                                                                                                  \
    auto kern = gemm_bf16_kernel<BM, BN, BK, WGM, WGN, AK, BKC, CV, ACT>;                               \
    if (lds > 64 * 1024) (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    hipLaunchKernelGGL(kern, grid, block, lds, s, g.A, g.B, g.M, g.N, g.K, g.lda, g.ldb, tiles_m, tiles_n, splits,  \
                       k_per_split, ep, (float*)g.ws, g.conv);                                          \
  } while (0)
  constexpr bool CONVS = BM == 128;   // the gathered forms exist for the small tile only
  if (g.conv_mode) {
    if constexpr (CONVS) {
      if (g.conv_mode == 1) KARMA_GEMM_LAUNCH(true, true, 1, 0);
      else KARMA_GEMM_LAUNCH(false, false, 2, 0);
    } else {
      return KARMA_E_INVAL;
    }
  } else if (g.act == 1) KARMA_GEMM_LAUNCH(true, true, 0, 1);
  else if (g.act == 2) KARMA_GEMM_LAUNCH(true, false, 0, 2);
  else if (g.a_kc && g.b_kc) KARMA_GEMM_LAUNCH(true, true, 0, 0);
  else if (g.a_kc && !g.b_kc) KARMA_GEMM_LAUNCH(true, false, 0, 0);
  else if (!g.a_kc && g.b_kc) KARMA_GEMM_LAUNCH(false, true, 0, 0);
  else KARMA_GEMM_LAUNCH(false, false, 0, 0);
#undef KARMA_GEMM_LAUNCH
  return finish(g, ep, splits, s);
}

thread_local GemmTimer* g_gemm_timer = nullptr;

// The 64 x 64 tile
static SliceWork slice_work(const GemmArgs& g, int& splits) {
  const int k_per_split = range_length(g.K, splits);
  SliceWork w{g.A, g.B, epilogue_of(g), (float*)g.ws, g.M, g.N, g.K, g.lda, g.ldb, splits, k_per_split};
  if (splits == 1) take_colsum(g, (g.M + SLICE_TILE - 1) / SLICE_TILE, w.ep);
  return w;
}
static int launch_slices(const GemmArgs& g, int splits, hipStream_t s) {
  const SliceWork w = slice_work(g, splits);
  const int st = gemm_slices_launch(w, SliceForm{g.a_kc, g.b_kc, g.act}, nullptr, s);
  return st == KARMA_OK ? finish(g, w.ep, splits, s) : st;
}

// The 128 x 128 tile: geometry of the gathered forms, then the launch
static int launch_ring(const GemmArgs& g, int splits, bool deep, int side, hipStream_t s) {
  const int k_per_split = range_length(g.K, splits);
  GemmEpilogue ep = epilogue_of(g);
  if (splits == 1) take_colsum(g, 2 * ((g.M + RING_TILE - 1) / RING_TILE), ep);
  RingConv rc{};
  if (g.conv_mode) {
    const ConvGather& cg = g.conv;
    auto magic = [](int d) { return d > 1 ? (unsigned)((1ull << 32) / (unsigned)d + 1) : 0u; };
    rc.magic_c = magic(cg.C);
    rc.out_stride = 1;
    if (cg.transposed && cg.stride == 2) {
      const int images = g.M / (cg.Ho * cg.Wo);
      unsigned at = 0;
      rc.out_stride = 2;
      rc.oh = cg.Ho;
      rc.ow = cg.Wo;
      for (int oy = 0; oy < 2; ++oy)
        for (int ox = 0; ox < 2; ++ox) {
          const DgradTaps ty = dgrad_taps(cg.R, cg.pad, oy), tx = dgrad_taps(cg.S, cg.pad, ox);
          const int rows = (cg.Ho - oy + 1) / 2, cols = (cg.Wo - ox + 1) / 2, k = ty.count * tx.count * cg.C;
          if (rows > 0 && cols > 0) {
            RingPhase& p = rc.p[rc.phases++];
            p.cg = ConvGather{cg.H, cg.W, cg.C, rows, cols, ty.count, tx.count, 1, 0, 1};
            p.pad_y = ty.shift;
            p.pad_x = tx.shift;
            p.M = images * rows * cols;
            p.K = k;
            p.b_off = at;
            p.magic_s = magic(tx.count);
            p.oy = oy;
            p.ox = ox;
          }
          at += (unsigned)k * (unsigned)g.N;
        }
    } else {
      rc.phases = 1;
      rc.p[0] = RingPhase{cg, g.M, g.K, 0u, magic(cg.S), 0, 0, cg.pad, cg.pad};
    }
  }
  const int st = gemm_ring_launch(g, ep, splits, k_per_split, deep, side, g.conv_mode ? &rc : nullptr, s);
  return st == KARMA_OK ? finish(g, ep, splits, s) : st;
}

// One launch of a product (with the sum of its ranges): what gemm_choose decides and launch_piece carries out
struct Piece {
  GemmArgs g;
  uint32_t kernel;   // KARMA_PRODUCT_*
  int splits;
  bool deep;    // the 128 x 128 tile: four stages
  double us = 0.0;   // modelled, where the tile was chosen by that
};
static Piece planned(const GemmArgs& g, const GemmPlan& p) {
  const uint32_t of64 = !g.conv_mode ? KARMA_PRODUCT_SLICES : g.conv_mode == 1 ? KARMA_PRODUCT_NARROW : KARMA_PRODUCT_FLAT;
  return Piece{g, p.tile == 256 ? KARMA_PRODUCT_LARGE : p.tile == 128 ? KARMA_PRODUCT_SMALL : p.tile == 64 ? of64 : KARMA_PRODUCT_BROAD, p.splits, p.deep, p.us};
}
static int launch_piece(const Piece& p, hipStream_t s) {
  switch (p.kernel) {
    case KARMA_PRODUCT_LARGE: return launch_large(p.g, p.splits, s);
    case KARMA_PRODUCT_SMALL: return launch_ring(p.g, p.splits, p.deep, RING_TILE, s);
    case KARMA_PRODUCT_BROAD: return launch_ring(p.g, p.splits, false, RING_BROAD, s);
    case KARMA_PRODUCT_NARROW:
    case KARMA_PRODUCT_FLAT: return launch_ring(p.g, p.splits, false, RING_SLIM, s);
    case KARMA_PRODUCT_SLICES: return launch_slices(p.g, p.splits, s);
    case KARMA_PRODUCT_STAGED_LARGE: return launch_general<256, 256, 2, 4>(p.g, p.splits, s);
    default: return launch_general<128, 128, 2, 2>(p.g, p.splits, s);
  }
}

// Operands whose sizes or alignment do not allow 16-byte pieces (4-element runs), and gradients of convolutions with a
// stride above 2: tiles go through registers, of the size whose modelled time is the shorter.  us, 256 / 128: 3940 x 3084 x
// 16304 both operands strided 617 / 934, 2836 x 4540 x 5848 254 / 309, 1156 x 5484 x 8136 with a workspace 191 / 258;
// 2288 x 536 x 776 33 / 16.5, 132 x 236 x 776 60 / 33.
static Piece choose_general(const GemmArgs& g) {
  const GeneralPlan small = plan_general(g, 128);
  if (!g.conv_mode && g.M > 128 && g.N > 128) {
    const GeneralPlan large = plan_general(g, 256);
    if (general_us(g, large, 256) < general_us(g, small, 128)) return Piece{g, KARMA_PRODUCT_STAGED_LARGE, large.splits, false};
  }
  return Piece{g, KARMA_PRODUCT_STAGED_SMALL, small.splits, false};
}

// A product whose large tiles leave a last round nearly empty, cut in two along its columns or rows: as many whole tiles
// as fill the rounds before it, and the rest with the tile and number of ranges that suit it.  Taken where the model says
// that it saves 4 % and a launch (3 us).  us, whole -> cut, without / with a workspace for the rest's ranges:
//   4096 x 4256 x 17024 (272 tiles on 256 compute units): 795 -> 681 / 492      4096 x 4256 x 4256: 187 -> 161 / 143
//   8192 x 3072 x 12288 (one and a half rounds): 549 -> 515 / 497               8192 x 9216 x 3072: 385 -> 372
//   12768 x 4256 x 4096: 439 -> 407
// From 1024 k on: below, writing the tiles out is most of a round, and the model puts that too low (412776 x 560 x 216:
// 290 -> 325, 4512 x 8128 x 680: 72, 68 with the small tile throughout).
static bool plan_cut(const GemmArgs& g, double whole_us, Piece* part) {
  const int cus = compute_units(), tm = (g.M + 255) / 256, tn = (g.N + 255) / 256;
  const long whole_rounds = (long)tm * tn / cus * cus;      // tiles in them
  double best_us = 0.96 * whole_us;
  bool found = false;
  for (int rows = 0; rows < 2; ++rows) {
    const long keep = whole_rounds / (rows ? tn : tm);      // rows or columns of tiles that stay
    if (keep < 1 || keep * 256 >= (rows ? g.M : g.N)) continue;
    const int cut = (int)keep * 256;
    const GemmArgs a = rows ? block_of(g, 0, cut, 0, g.N) : block_of(g, 0, g.M, 0, cut);
    const GemmArgs b = rows ? block_of(g, cut, g.M - cut, 0, g.N) : block_of(g, 0, g.M, cut, g.N - cut);
    if (!large_tile_takes(a) || !gemm_ring_takes(b)) continue;
    // (partial results are dense and are added up octet by octet into rows ldc apart)
    const bool may_split = b.ws && !b.act && b.N % 8 == 0 && b.ldc % 8 == 0 && (uint64_t)b.M * b.N < (1ull << 32);
    const GemmPlan pa = plan_product(a, true, false, false), pb = plan_product(b, large_tile_takes(b), true, may_split);
    const double us = pa.us + pb.us + 3.0;
    if (us >= best_us) continue;
    best_us = us;
    part[0] = planned(a, pa);
    part[1] = planned(b, pb);
    found = true;
  }
  return found;
}

// Checks the arguments and decides how the product is carried out: one piece, or two.  Host only.
static int gemm_choose(const GemmArgs& g, Piece* piece, int* pieces) {
  *pieces = 1;
  if (!g.A || !g.B || !g.C || g.M <= 0 || g.N <= 0 || g.K <= 0) return KARMA_E_INVAL;
  // 16-byte k-runs (k-contiguous) or 8-byte row runs (strided) must stay aligned and whole
  if ((g.a_kc || g.b_kc) && g.K % 8) return KARMA_E_INVAL;   // strided operands take any K: every k-row is bounds-checked
  if (g.conv_mode != 1 && (g.a_kc ? (g.lda % 8) : (g.lda % 4 || g.M % 4))) return KARMA_E_INVAL;
  if (g.conv_mode != 2 && (g.b_kc ? (g.ldb % 8) : (g.ldb % 4 || g.N % 4))) return KARMA_E_INVAL;
  if (g.conv_mode < 0 || g.conv_mode > 2) return KARMA_E_INVAL;
  if (g.accumulate && !g.out_f32) return KARMA_E_INVAL;
  if (g.act < 0 || g.act > 2 || (g.act && (!g.aux || g.out_f32 || g.residual || g.conv_mode))) return KARMA_E_INVAL;
  // the fused forms exist for the layouts of the feed-forward layer: forward x W1^T (both operands
  // k-contiguous), backward dy W2 (second operand strided)
  if ((g.act == 1 && !(g.a_kc && g.b_kc)) || (g.act == 2 && !(g.a_kc && !g.b_kc))) return KARMA_E_INVAL;
  if (g.residual && g.out_f32) return KARMA_E_INVAL;
  if (g.conv_mode) {
    const ConvGather& cg = g.conv;
    if (g.conv_mode == 1 ? !(g.a_kc && g.b_kc) : (g.a_kc || g.b_kc)) return KARMA_E_INVAL;
    if (cg.C % 8 || cg.H <= 0 || cg.W <= 0 || cg.Ho <= 0 || cg.Wo <= 0 || cg.R <= 0 || cg.S <= 0 || cg.stride <= 0 || cg.pad < 0)
      return KARMA_E_INVAL;
    // the gathered operand's index ranges must be what the convolution spans
    const long pixels = (long)cg.Ho * cg.Wo, taps_c = (long)cg.R * cg.S * cg.C;
    if (g.conv_mode == 1 ? (g.M % pixels || g.K != taps_c) : (g.K % pixels || g.N != taps_c)) return KARMA_E_INVAL;
    if (cg.phased && (g.conv_mode != 1 || !cg.transposed || cg.stride != 2 || !gemm_ring_takes(g))) return KARMA_E_INVAL;
  }
  const bool small = gemm_ring_takes(g);
  if (g.conv_mode && g.conv.phased) {
    const ConvGather& cg = g.conv;
    // by parity of the pixel: four products of a quarter of the rows, and of a quarter of the taps on average.  The broad tile where it
    // leaves less than 0.7 of the columns to multiply, fills the chip twice and is modelled to be faster by a tenth: 256 x 32 x 32 x 160
    // from 320 channels, 3 x 3, 131 -> 120 us, 31 x 160 x 160 x 160 from 264, 7 x 7, 1347 -> 1009; 7 x 168 x 168 x 160 from 16, 3 x 3, 48 and
    // 60, 84 x 82 x 82 x 152 from 128, 1 x 1, 103 and 124 (of 51 one is left 5 % slower, without the model 37); 320 from 640 channels
    // (0.83 of the columns) 97 and 99
    const int cus = compute_units();
    const double kt = g.K / (4.0 * 64.0);
    const long wide = 4l * ((g.M / 4 + 255) / 256) * ((g.N + RING_BROAD - 1) / RING_BROAD);
    const long square = 4l * ((g.M / 4 + 127) / 128) * ((g.N + RING_TILE - 1) / RING_TILE);
    const bool broad = (g.N + RING_BROAD - 1) / RING_BROAD * RING_BROAD * 10 < (g.N + RING_TILE - 1) / RING_TILE * RING_TILE * 7 && wide >= 2 * cus &&
                       1.1 * broad_us(wide, kt, cus) < square_gather_us(square, kt, cus);
    // Up to 64 columns the slim tile, where it has a workgroup for every compute unit: 64 x 224 x 224 x 8 from 64 channels, 7 x 7,
    // 698 -> 409 us; not for the longest reductions, least where channels are no whole cache lines (5 x 236 x 236 x 8 from 320, 7 x 7,
    // 311 -> 214; 21 x 227 x 227 x 32 from 264 898 and 1139, 21 x 182 x 182 x 40 from 424 1029 and 1259).
    const bool slim = g.N <= RING_SLIM && 4l * ((g.M / 4 + 255) / 256) >= cus && g.K <= (cg.C % 64 ? 8192 : 16384);
    piece[0] = Piece{g, slim ? KARMA_PRODUCT_NARROW : broad ? KARMA_PRODUCT_BROAD : KARMA_PRODUCT_SMALL, 1, false};
    return KARMA_OK;
  }
  bool may_split = g.ws && g.ldc == g.N && !g.act;
  bool large;
  if (g.conv_mode) {
    const ConvGather& cg = g.conv;
    const long pixels = (long)cg.Ho * cg.Wo;
    // What the direct-load kernel's gathers assume: piece offsets are 32-bit byte counts, packed coordinates ten bits wide,
    // strides 1 and 2; (tap, channel) from reciprocals.  A gathered second operand: pixels * Wo < 2^32, the
    // reciprocal multiplication by magic_w = 2^32 / Wo + 1 being exact for every n with n * (magic_w * Wo - 2^32) < 2^32,
    // and that excess is at most Wo.
    const uint64_t gathered_bytes = (uint64_t)((g.conv_mode == 1 ? g.M : g.K) / pixels) * cg.H * cg.W * cg.C * 2;
    large = g.ldc % 8 == 0 && cg.H * cg.stride + cg.pad + 64 < 1024 && cg.W * cg.stride + cg.pad + 64 < 1024 &&
            gathered_bytes < (1ull << 32) && ((uintptr_t)g.A % 16) == 0 && ((uintptr_t)g.B % 16) == 0 &&
            (cg.S > 1 || cg.R == 1) && (cg.Wo > 1 || cg.Ho == 1);   // (no reciprocal of 1 in 32 bits)
    if (g.conv_mode == 1)
      large = large && g.K >= 128 && g.N % 8 == 0 && cg.stride <= 2 && cg.Ho + cg.pad + 64 < 1024 && cg.Wo + cg.pad + 64 < 1024 &&
              g.M / pixels < 4095 && (uint64_t)g.K * cg.C < (1ull << 31) && (uint64_t)g.ldb * 2 * 256 < (1ull << 31);
    else
      large = large && g.M >= 64 && g.N >= 512 && g.K >= 4096 && g.M % 8 == 0 && g.lda % 8 == 0 && g.ws != nullptr &&
              (uint64_t)g.N * cg.C < (1ull << 31) && (uint64_t)pixels * cg.Wo < (1ull << 32) && g.K < (1 << 24) &&
              (uint64_t)g.lda * 2 * 256 < (1ull << 31);
    // Sums that keep their order: those of 64 channels on large images have never been divided
    if (g.keep_sums && g.conv_mode == 1 && large && g.N == 64 && (g.M + 255) / 256 >= 384) may_split = false;
    // below 128 output channels most of the large tile is empty
    if (g.conv_mode == 1 && g.N < 128) large = false;
  } else {
    large = large_tile_takes(g);
  }
  if (!large && !small) {
    piece[0] = choose_general(g);
    return KARMA_OK;
  }
  // Results whose rows are no whole octets do without the large tile's direct loads.  From 0.3 TFLOP on the register-staged
  // large tile is ahead of the small one all the same: 3280 x 4331 x 12184 433 / 488 us, 7346 x 9171 x 8224 1479 / 1607,
  // 2701 x 7687 x 6112 (0.25) 257 / 193.
  if (!g.conv_mode && !large && g.N % 8 && g.M > 128 && g.N > 128 && (double)g.M * g.N * g.K >= 1.5e11) {
    piece[0] = Piece{g, KARMA_PRODUCT_STAGED_LARGE, plan_general(g, 256).splits, false};
    return KARMA_OK;
  }
  // One k-tile, one column of tiles and more than a round of them: nothing to pipeline within an item, and the staged
  // kernel's workgroups, which stay for several, fetch the next item before they write one out.  us, small / staged:
  // 1954597 x 64 x 32 158 / 124, 475061 x 40 x 32 36 / 31, 224225 x 32 x 48 18 / 16; 242215 x 88 x 72 26 / 28.
  if (!g.conv_mode && g.a_kc && g.b_kc && g.K <= 64 && g.N <= 128 && (g.M + 127) / 128 > 2 * compute_units()) {
    piece[0] = Piece{g, KARMA_PRODUCT_STAGED_SMALL, 1, false};
    return KARMA_OK;
  }
  const GemmPlan p = plan_product(g, large, small, may_split);
  if (large && small && !g.conv_mode && !g.colsum_partial && g.K >= 1024 && plan_cut(g, p.us, piece)) *pieces = 2;
  else piece[0] = planned(g, p);
  return KARMA_OK;
}

static int gemm_bf16_launch(const GemmArgs& g, hipStream_t s) {
  Piece piece[2];
  int pieces = 0, st = gemm_choose(g, piece, &pieces);
  for (int i = 0; i < pieces && st == KARMA_OK; ++i) st = launch_piece(piece[i], s);
  return st;
}

// A product as gemm_choose would have it carried out
struct Choice {
  Piece piece[2];
  int pieces = 0;
};

// Both gradients of a layer in one launch of the 64 x 64 tile where that is modelled to be the shorter way by 5 %: one workgroup
// per compute unit, those of dx first, those of dw as units become free; beside other work a round of k-tiles takes
// SLICES_TILE_MORE.  Of 700 layers of transformers (widths from 128 to 1280, 128 to 24576 tokens) 291 take
// it: 1.56 times as fast as the two products with tiles of their own up to 32 k-tiles, 1.33 up to 48, 1.15 up to 64, and three
// of them more than 3 % slower (41.1 / 38.8, 39.1 / 37.9, 59.1 / 52.4 us).  us, one launch / two: 1024 x 256 x 256 8 / 16,
// 640 x 2560 x 640 (rows, n, k) 17.1 / 22.3, 2304 x 2560 x 640 35.9 / 43.9, 3200 x 512 x 128 13.7 / 17.8.  An estimate that shared the
// work out evenly had taken 481, 113 of them slower, by up to 1.6: 6912 x 768 x 256 31.4 / 24.0, 3840 x 3040 x 760 100 / 62.
// PAIR_MAX_KT: beyond it gains and losses were alike (27 layers, 0.82 to 1.35).
constexpr int PAIR_MAX_KT = 64;
static bool pair_of_slices(const GemmArgs& dx, const GemmArgs& dw, const Choice (&own)[2]) {
  if (!dx.a_kc || dx.b_kc || dx.act == 1 || dw.a_kc || dw.b_kc || dw.act || dx.conv_mode || dw.conv_mode) return false;
  const GemmArgs* g[2] = {&dx, &dw};
  double apart = 0.0, each[2];
  long items[2];
  for (int i = 0; i < 2; ++i) {
    if (own[i].pieces != 1) return false;
    // (products of which one alone fills the chip are better off with tiles of their own)
    const Piece& p = own[i].piece[0];
    if (p.kernel != KARMA_PRODUCT_SLICES && p.kernel != KARMA_PRODUCT_SMALL) return false;
    const int kt = (g[i]->K + SLICE_BK - 1) / SLICE_BK;
    if (kt > PAIR_MAX_KT) return false;
    apart += p.us;
    items[i] = (long)((g[i]->M + SLICE_TILE - 1) / SLICE_TILE) * ((g[i]->N + SLICE_TILE - 1) / SLICE_TILE);
    each[i] = SLICES_ROUND + SLICES_TILE_MORE * ((kt + SLICE_WAVES - 1) / SLICE_WAVES);
  }
  // dx leaves `late` units busy until `then`, the others from `now` on take dw's workgroups, and so on
  const long cus = compute_units(), late = items[0] % cus;
  double now = items[0] / cus * each[0], then = now + each[0], end = late ? then : now;
  for (long left = items[1]; left > 0;) {
    const bool first = !late || now <= then;
    double& at = first ? now : then;
    left -= first ? cus - late : late;
    at += each[1];
    end = std::max(end, at);
    if (SLICES_BASE + end >= 0.95 * apart) return false;
  }
  return SLICES_BASE + end < 0.95 * apart;
}

static int gemm_pair_choose(const GemmArgs& dx, const GemmArgs& dw, Choice (&own)[2], bool* together) {
  int st = gemm_choose(dx, own[0].piece, &own[0].pieces);
  if (st == KARMA_OK) st = gemm_choose(dw, own[1].piece, &own[1].pieces);
  *together = st == KARMA_OK && pair_of_slices(dx, dw, own);
  return st;
}

static int gemm_pair_launch(const GemmArgs& dx, const GemmArgs& dw, hipStream_t s) {
  Choice own[2];
  bool together = false;
  int st = gemm_pair_choose(dx, dw, own, &together);
  if (together) {
    int one = 1;
    const SliceWork a = slice_work(dx, one), b = slice_work(dw, one);
    return gemm_slices_launch(a, SliceForm{true, false, dx.act}, &b, s);
  }
  for (const Choice& c : own)
    for (int i = 0; i < c.pieces && st == KARMA_OK; ++i) st = launch_piece(c.piece[i], s);
  return st;
}

// Launches with events around them when the caller samples them
template <class Launch>
static int timed(double flops, hipStream_t s, Launch launch) {
  GemmTimer* t = g_gemm_timer;
  if (!t) return launch();
  if (t->stride > 1 && (t->seq++ % t->stride) != t->phase % t->stride) return launch();
  while (t->events->size() < *t->used + 2) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return KARMA_E_HIP;
    t->events->push_back(e);
  }
  if (hipEventRecord((*t->events)[*t->used], s) != hipSuccess) return KARMA_E_HIP;
  const int st = launch();
  if (hipEventRecord((*t->events)[*t->used + 1], s) != hipSuccess) return KARMA_E_HIP;
  *t->used += 2;
  t->flops->push_back(flops);
  return st;
}

int gemm_bf16(const GemmArgs& g, hipStream_t s) {
  return timed(2.0 * g.M * g.N * g.K, s, [&] { return gemm_bf16_launch(g, s); });
}
int gemm_bf16_pair(const GemmArgs& dx, const GemmArgs& dw, hipStream_t s) {
  return timed(2.0 * dx.M * dx.N * dx.K + 2.0 * dw.M * dw.N * dw.K, s, [&] { return gemm_pair_launch(dx, dw, s); });
}

int gemm_plan(const GemmArgs& g, karma_product_part* parts, uint32_t* n, bool tiles) {
  Piece piece[2];
  int pieces = 0;
  const int st = gemm_choose(g, piece, &pieces);
  if (st != KARMA_OK) return st;
  for (int i = 0; i < pieces; ++i) {
    int splits = piece[i].splits;
    (void)range_length(piece[i].g.K, splits);   // (ranges are whole k-tiles: the last may come to nothing)
    const uint32_t kernel = !tiles && piece[i].kernel >= KARMA_PRODUCT_SLICES ? KARMA_PRODUCT_SMALL : piece[i].kernel;
    parts[i] = karma_product_part{kernel, (uint32_t)piece[i].g.M, (uint32_t)piece[i].g.N, (uint32_t)splits};
  }
  *n = (uint32_t)pieces;
  return KARMA_OK;
}

}  // namespace karma

using namespace karma;

extern "C" int karma_k_gemm_gelu_bf16(const void* a, const void* b, void* c, const void* bias, void* aux, uint32_t m,
                                      uint32_t n, uint32_t k, uint32_t flags, uint32_t mode, void* stream) {
  if (mode != KARMA_GEMM_GELU_FWD && mode != KARMA_GEMM_GELU_BWD) return KARMA_E_INVAL;
  if (flags & (KARMA_GEMM_OUT_F32 | KARMA_GEMM_ACCUMULATE)) return KARMA_E_INVAL;
  GemmArgs g{};
  g.A = (const bf16_t*)a;
  g.B = (const bf16_t*)b;
  g.C = c;
  g.bias = (const bf16_t*)bias;
  g.M = (int)m; g.N = (int)n; g.K = (int)k;
  g.a_kc = !(flags & KARMA_GEMM_A_STRIDED);
  g.b_kc = !(flags & KARMA_GEMM_B_STRIDED);
  g.lda = g.a_kc ? (int)k : (int)m;
  g.ldb = g.b_kc ? (int)k : (int)n;
  g.ldc = (int)n;
  g.act = (int)mode;
  g.aux = aux;
  return gemm_bf16(g, (hipStream_t)stream);
}

// The backward product with GELU' and the column sums of its result (fused where the shape allows)
extern "C" int karma_k_gemm_gelu_bwd_colsum_bf16(const void* a, const void* b, void* c, const void* aux, float* colsum_out,
                                                 float* ws, uint64_t ws_bytes, uint32_t m, uint32_t n, uint32_t k,
                                                 void* stream) {
  if (!a || !b || !c || !aux || !colsum_out || !ws) return KARMA_E_INVAL;
  if (ws_bytes < colsum_ws_bytes((int)m, (int)n)) return KARMA_E_OOM;
  GemmArgs g{};
  g.A = (const bf16_t*)a;
  g.B = (const bf16_t*)b;
  g.C = c;
  g.M = (int)m; g.N = (int)n; g.K = (int)k;
  g.a_kc = true;
  g.b_kc = false;
  g.lda = (int)k;
  g.ldb = (int)n;
  g.ldc = (int)n;
  g.act = 2;
  g.aux = const_cast<void*>(aux);
  int rows = 0;
  g.colsum_partial = ws;
  g.colsum_bytes = colsum_ws_bytes((int)m, (int)n);
  g.colsum_rows = &rows;
  int st = gemm_bf16(g, (hipStream_t)stream);
  if (st) return st;
  if (rows) return colsum_finish(ws, rows, (int)n, colsum_out, (hipStream_t)stream);
  return colsum_bf16((const bf16_t*)c, colsum_out, ws, (int)m, (int)n, (hipStream_t)stream);
}

static GemmArgs product_args(const void* a, const void* b, void* c, const void* bias, const void* residual, uint32_t m, uint32_t n,
                             uint32_t k, uint32_t flags, void* ws, uint64_t ws_bytes) {
  GemmArgs g{};
  g.A = (const bf16_t*)a;
  g.B = (const bf16_t*)b;
  g.C = c;
  g.bias = (const bf16_t*)bias;
  g.residual = (const bf16_t*)residual;
  g.M = (int)m; g.N = (int)n; g.K = (int)k;
  g.a_kc = !(flags & KARMA_GEMM_A_STRIDED);
  g.b_kc = !(flags & KARMA_GEMM_B_STRIDED);
  g.lda = g.a_kc ? (int)k : (int)m;
  g.ldb = g.b_kc ? (int)k : (int)n;
  g.ldc = (int)n;
  g.out_f32 = (flags & KARMA_GEMM_OUT_F32) != 0;
  g.accumulate = (flags & KARMA_GEMM_ACCUMULATE) != 0;
  g.ws = ws;
  g.ws_bytes = ws ? (size_t)ws_bytes : 0;
  return g;
}

extern "C" int karma_k_gemm_bf16(const void* a, const void* b, void* c, const void* bias, const void* residual,
                                 uint32_t m, uint32_t n, uint32_t k, uint32_t flags, void* ws, uint64_t ws_bytes,
                                 void* stream) {
  return gemm_bf16(product_args(a, b, c, bias, residual, m, n, k, flags, ws, ws_bytes), (hipStream_t)stream);
}

extern "C" int karma_k_gemm_plan(uint32_t m, uint32_t n, uint32_t k, uint32_t flags, uint32_t gelu_mode, uint32_t misaligned,
                                 uint64_t ws_bytes, karma_product_part* parts_out, uint32_t* n_out) {
  if (!parts_out || !n_out || gelu_mode > KARMA_GEMM_GELU_BWD) return KARMA_E_INVAL;
  void* const somewhere = (void*)(uintptr_t)(4096 + (misaligned ? 8 : 0));   // (addresses are only looked at)
  GemmArgs g = product_args(somewhere, somewhere, somewhere, nullptr, nullptr, m, n, k, flags & ~KARMA_PLAN_TILES,
                            ws_bytes ? somewhere : nullptr, ws_bytes);
  g.act = (int)gelu_mode;
  g.aux = gelu_mode ? somewhere : nullptr;
  return gemm_plan(g, parts_out, n_out, (flags & KARMA_PLAN_TILES) != 0);
}

// dx = dy w (with aux: times GELU'(aux)) and dw = dy^T x
static void linear_bwd_products(const void* dy, const void* w, const void* x, void* dx, void* dw, const void* aux, void* ws, uint64_t ws_bytes,
                                uint32_t rows, uint32_t n, uint32_t k, uint32_t flags, GemmArgs (&g)[2]) {
  const bool room = !aux;   // (GELU' is taken in the output stage of an undivided product)
  g[0] = product_args(dy, w, dx, nullptr, nullptr, rows, k, n, KARMA_GEMM_B_STRIDED, room ? ws : nullptr, ws_bytes);
  g[1] = product_args(dy, x, dw, nullptr, nullptr, n, k, rows, KARMA_GEMM_A_STRIDED | KARMA_GEMM_B_STRIDED | flags, ws, ws_bytes);
  g[0].act = aux ? 2 : 0;
  g[0].aux = const_cast<void*>(aux);
}

extern "C" int karma_k_linear_bwd_bf16(const void* dy, const void* w, const void* x, void* dx, void* dw, const void* aux, float* colsum_out,
                                       void* ws, uint64_t ws_bytes, uint32_t rows, uint32_t n, uint32_t k, uint32_t flags, void* stream) {
  if ((flags & ~(KARMA_GEMM_OUT_F32 | KARMA_GEMM_ACCUMULATE)) || (colsum_out && !aux)) return KARMA_E_INVAL;
  const size_t sums = colsum_out ? (colsum_ws_bytes((int)rows, (int)k) + 255) / 256 * 256 : 0;
  if (colsum_out && (!ws || ws_bytes < sums)) return KARMA_E_OOM;
  if (!ws) ws_bytes = 0;
  void* const rest = ws_bytes > sums ? (char*)ws + sums : nullptr;
  GemmArgs g[2];
  linear_bwd_products(dy, w, x, dx, dw, aux, rest, rest ? ws_bytes - sums : 0, rows, n, k, flags, g);
  int parts = 0;
  if (colsum_out) {
    g[0].colsum_partial = (float*)ws;
    g[0].colsum_bytes = colsum_ws_bytes((int)rows, (int)k);
    g[0].colsum_rows = &parts;
  }
  const int st = gemm_bf16_pair(g[0], g[1], (hipStream_t)stream);
  if (st || !colsum_out) return st;
  if (parts) return colsum_finish((float*)ws, parts, (int)k, colsum_out, (hipStream_t)stream);
  return colsum_bf16((const bf16_t*)dx, colsum_out, (float*)ws, (int)rows, (int)k, (hipStream_t)stream);
}

extern "C" int karma_k_linear_bwd_plan(uint32_t rows, uint32_t n, uint32_t k, uint32_t gelu, uint32_t flags, uint64_t ws_bytes, uint32_t* together_out) {
  if (!together_out || (flags & ~(KARMA_GEMM_OUT_F32 | KARMA_GEMM_ACCUMULATE))) return KARMA_E_INVAL;
  void* const somewhere = (void*)(uintptr_t)4096;   // (addresses are only looked at)
  GemmArgs g[2];
  linear_bwd_products(somewhere, somewhere, somewhere, somewhere, somewhere, gelu ? somewhere : nullptr, ws_bytes ? somewhere : nullptr, ws_bytes, rows,
                      n, k, flags, g);
  Choice own[2];
  bool together = false;
  const int st = gemm_pair_choose(g[0], g[1], own, &together);
  *together_out = together ? 1u : 0u;
  return st;
}

// ---- the product for callers that cannot allocate -------------------------------------------
// The split-reduction workspace lives in a file-scope device array instead of a caller's buffer.
// In host code the array's name is only a handle: the device address comes from
// hipGetSymbolAddress, once per device (each GPU holds its own copy at its own address).
namespace {
constexpr size_t STATIC_WS_BYTES = KARMA_GEMM_STATIC_WS_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_WS_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on the current device, or nullptr (HIP error).
void* static_ws() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" int karma_k_gemm_bf16_static_ws(const void* a, const void* b, void* c, const void* bias, const void* residual,
                                           uint32_t m, uint32_t n, uint32_t k, uint32_t flags, void* stream) {
  // two partial results must fit, or the workspace could not serve any split
  if ((uint64_t)m * n * sizeof(float) * 2 > STATIC_WS_BYTES) return KARMA_E_OOM;
  void* ws = static_ws();
  if (!ws) return KARMA_E_HIP;
  return karma_k_gemm_bf16(a, b, c, bias, residual, m, n, k, flags, ws, STATIC_WS_BYTES, stream);
}
