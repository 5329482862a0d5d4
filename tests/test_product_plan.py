"""The choice of kernel, ranges and cut of a bf16 product (karma_k_gemm_plan, karma_k_conv2d_plan), over the whole range of
sizes, layouts and workspaces: parts cover the product once, partial sums fit the workspace, and a kernel is given only
what it takes."""
import random

import pytest

import paper_2008_11421_amd as K

A, B = K.GEMM_A_STRIDED, K.GEMM_B_STRIDED


def log_int(rng, lo, hi, step=1):
    return max(lo, int(2 ** rng.uniform(lo.bit_length() - 1, hi.bit_length() - 1)) // step * step)


def check(parts, m, n, k, ws, may_split, pieces16, gathered=False):
    assert 1 <= len(parts) <= 2
    if len(parts) == 1:
        assert parts[0][1:3] == (m, n)
    else:       # cut along whole large tiles; the first part is whole rounds of them, undivided
        (k0, m0, n0, s0), (_, m1, n1, _) = parts
        assert k0 == K.PRODUCT_LARGE and s0 == 1
        assert (m0 == m1 == m and n0 + n1 == n and n0 % 256 == 0) or (n0 == n1 == n and m0 + m1 == m and m0 % 256 == 0)
    for kernel, pm, pn, splits in parts:
        assert 1 <= splits <= max(1, (k + 63) // 64)
        assert splits == 1 or (may_split and splits * pm * pn * 4 <= ws)
        if not pieces16:
            assert kernel in (K.PRODUCT_STAGED_SMALL, K.PRODUCT_STAGED_LARGE)
        if kernel == K.PRODUCT_LARGE and not gathered:
            assert pm >= 256 and pn >= 256 and k >= 128 and pm % 8 == 0 and pn % 8 == 0 and k % 8 == 0
        if kernel == K.PRODUCT_STAGED_LARGE:
            assert pm > 128 and pn > 128 and not gathered


def test_products_over_the_whole_range():
    rng = random.Random(11)
    seen = set()
    for _ in range(3000):
        flags, mode = rng.choice([(0, 0), (A, 0), (B, 0), (A | B, 0), (0, K.GEMM_GELU_FWD), (B, K.GEMM_GELU_BWD)])
        step = rng.choice([1, 4, 8, 8, 256])
        m = log_int(rng, 1, 40000, max(step, 4) if flags & A else step)
        n = log_int(rng, 1, 40000, max(step, 4) if flags & B else step)
        m, n = max(m, 4 if flags & A else 1), max(n, 4 if flags & B else 1)
        k = max(8, log_int(rng, 8, 40000, rng.choice([8, 64])))
        misaligned, ws = rng.random() < 0.2, rng.choice([0, 4 * m * n, 8 * m * n, 64 << 20])
        parts = K.gemm_plan(m, n, k, flags, mode, misaligned, ws)
        pieces16 = not misaligned and (not flags & A or m % 8 == 0) and (not flags & B or n % 8 == 0)
        check(parts, m, n, k, ws, mode == 0, pieces16)
        seen.add((parts[0][0], len(parts), parts[-1][3] > 1))
    assert {kernel for kernel, _, _ in seen} == {K.PRODUCT_STAGED_SMALL, K.PRODUCT_STAGED_LARGE, K.PRODUCT_SMALL, K.PRODUCT_LARGE}
    assert any(pieces == 2 for _, pieces, _ in seen) and any(divided for _, _, divided in seen)


def test_convolutions_over_the_whole_range():
    rng = random.Random(12)
    seen = set()
    for _ in range(3000):
        c = K.ConvShape(log_int(rng, 1, 256), log_int(rng, 1, 600), log_int(rng, 1, 600), log_int(rng, 8, 1024, 8), log_int(rng, 8, 1024, 8),
                        *([rng.choice([1, 2, 3, 3, 5, 7])] * 2), rng.choice([1, 1, 2, 2, 3]), rng.choice([0, 0, 1, 3]))
        ho, wo = (c.h + 2 * c.pad - c.r) // c.stride + 1, (c.w + 2 * c.pad - c.s) // c.stride + 1
        if c.h + 2 * c.pad < c.r or c.w + 2 * c.pad < c.s or max(c.n * c.h * c.w, c.n * ho * wo) >= 1 << 26:
            continue
        plain = c.r == 1 and c.stride == 1 and c.pad == 0
        for which, (m, n, k) in enumerate([(c.n * ho * wo, c.c_out, c.r * c.s * c.c_in), (c.n * c.h * c.w, c.c_in, c.r * c.s * c.c_out),
                                           (c.c_out, c.r * c.s * c.c_in, c.n * ho * wo)]):
            ws = rng.choice([0, 16 * c.c_out * c.r * c.s * c.c_in * 4])
            parts = K.conv_plan(c, which, ws)
            check(parts, m, n, k, ws, True, True if plain else parts[0][0] >= K.PRODUCT_SMALL, gathered=not plain)
            bytes_gathered = 2 * c.n * (ho * wo * c.c_out if which == K.CONV_DGRAD else c.h * c.w * c.c_in)
            if not plain and (bytes_gathered >= 1 << 32 or (which == K.CONV_DGRAD and c.stride == 3)):
                assert parts[0][0] == K.PRODUCT_STAGED_SMALL
            seen.add((which, parts[0][0]))
    assert {(w, k) for w in range(3) for k in (K.PRODUCT_STAGED_SMALL, K.PRODUCT_SMALL, K.PRODUCT_LARGE)} <= seen


@pytest.mark.parametrize("args", [(8, 8, 12, 0), (6, 8, 8, A), (8, 6, 8, B), (0, 8, 8, 0), (8, 8, 8, A, K.GEMM_GELU_FWD), (8, 8, 8, 0, K.GEMM_GELU_BWD)])
def test_what_a_product_refuses_its_plan_refuses(args):
    with pytest.raises(Exception):
        K.gemm_plan(*args)


def test_known_routes():
    # the last round of large tiles nearly empty: cut along columns, the rest divided where there is room
    assert K.gemm_plan(4096, 4256, 17024) == [(K.PRODUCT_LARGE, 4096, 4096, 1), (K.PRODUCT_SMALL, 4096, 160, 1)]
    assert K.gemm_plan(4096, 4256, 17024, ws_bytes=64 << 20)[1][3] > 1
    assert K.gemm_plan(32768, 4096, 1024) == [(K.PRODUCT_LARGE, 32768, 4096, 1)]
    assert K.gemm_plan(64, 1000, 2048)[0][0] == K.PRODUCT_SMALL
    assert K.gemm_plan(132, 236, 776, misaligned=True)[0][0] == K.PRODUCT_STAGED_SMALL
    assert K.gemm_plan(3940, 3084, 16304, A | B)[0][0] == K.PRODUCT_STAGED_LARGE
    # 64 output channels on large images
    assert K.conv_plan(K.ConvShape(8, 256, 256, 64, 64, 3, 3, 1, 1), K.CONV_FWD)[0][0] == K.PRODUCT_NARROW
    # a stride-2 input gradient by parity, and one whose tensor is beyond 32-bit offsets
    assert K.conv_plan(K.ConvShape(32, 57, 57, 96, 192, 3, 3, 2, 1), K.CONV_DGRAD) == [(K.PRODUCT_SMALL, 32 * 57 * 57, 96, 1)]


def test_tiles_that_leave_a_round_nearly_empty_are_not_split_finer():
    """Sizes on which the small tile had been taken and was slower than the large one by 15 to 30 %."""
    for m, n, k in [(4808, 1824, 2032), (1360, 6024, 10400), (5072, 1600, 1320), (1504, 5584, 3184)]:
        assert K.gemm_plan(m, n, k)[0][0] == K.PRODUCT_LARGE
    assert K.conv_plan(K.ConvShape(30, 93, 93, 232, 232, 5, 5, 2, 0), K.CONV_FWD)[0][0] == K.PRODUCT_LARGE
    # rows that are stored element by element: divided where that avoids it, through registers where the product is huge
    assert K.gemm_plan(77, 2647, 616, ws_bytes=64 << 20)[0][3] > 1
    assert K.gemm_plan(7346, 9171, 8224)[0][0] == K.PRODUCT_STAGED_LARGE
    assert K.gemm_plan(2701, 7687, 6112)[0][0] == K.PRODUCT_SMALL


def test_one_k_tile_and_one_column_of_tiles():
    for m, n, k, kernel in [(475061, 40, 32, K.PRODUCT_STAGED_SMALL), (65537, 128, 64, K.PRODUCT_STAGED_SMALL), (65536, 128, 64, K.PRODUCT_SMALL),
                            (475061, 136, 32, K.PRODUCT_SMALL), (475061, 40, 72, K.PRODUCT_SMALL)]:
        assert K.gemm_plan(m, n, k)[0][0] == kernel
    assert K.gemm_plan(475064, 40, 32, B)[0][0] == K.PRODUCT_SMALL


def test_short_reductions_are_not_cut():
    assert K.gemm_plan(412776, 560, 216) == [(K.PRODUCT_LARGE, 412776, 560, 1)]
    assert all(len(K.gemm_plan(m, n, k)) == 1 for m, n, k in [(4512, 8128, 680), (6296, 5624, 840), (4096, 4256, 1016)])
    assert len(K.gemm_plan(4096, 4256, 1024)) == 2


def test_products_that_keep_their_sums():
    """64 channels on large images are not divided, whatever the model of times says; weight gradients and small products are
    divided as the 128 x 128 and 256 x 256 tiles are, whatever other tile a free product takes."""
    keep, room = K.CONV_KEEP_SUMS, 1 << 30
    for args in [(49, 47, 47, 560, 64, 7, 7, 1, 3), (6, 272, 272, 648, 64, 7, 7, 2, 3), (64, 224, 224, 8, 64, 7, 7, 2, 3), (64, 56, 56, 64, 64, 3, 3, 1, 1)]:
        shape = K.ConvShape(*args)
        m = args[0] * ((args[1] + 2 * args[8] - args[5]) // args[7] + 1) ** 2
        (_, rows, cols, splits), = K.conv_plan(shape, K.CONV_FWD | keep, room)
        assert rows == m > 383 * 256 and (cols, splits) == (64, 1)
    shape = K.ConvShape(2, 228, 228, 64, 1328, 7, 7, 1, 3)
    assert K.conv_plan(shape, K.CONV_DGRAD | keep, room)[0][3] == 1
    # (ranges of the square tiles, ranges where the order is free)
    for args, which, kept, free in [((64, 56, 56, 64, 64, 3, 3, 1, 1), K.CONV_WGRAD, 102, 166), ((64, 224, 224, 8, 64, 7, 7, 2, 3), K.CONV_WGRAD, 128, 256),
                                    ((8, 56, 56, 64, 256, 1, 1, 1, 0), K.CONV_WGRAD, 79, 49), ((4, 14, 14, 256, 256, 3, 3, 1, 1), K.CONV_FWD, 6, 6)]:
        assert [K.conv_plan(K.ConvShape(*args), w, room)[0][3] for w in (which | keep, which)] == [kept, free]
    with pytest.raises(Exception):
        K.conv_plan(shape, 3 | keep)


def test_pairs_of_gradients():
    """One launch for small layers, not where the products alone are known to be faster, nor beyond 64 k-tiles."""
    ask = lambda rows, n, k, gelu=False, flags=0: K.linear_bwd_together(rows, n, k, gelu, flags, 8 * n * k * 4)
    assert ask(1024, 256, 256) and ask(1024, 1024, 256) and ask(1024, 256, 1024, True) and ask(640, 2560, 640) and ask(3200, 512, 128)
    assert ask(1024, 2048, 256, False, K.GEMM_OUT_F32 | K.GEMM_ACCUMULATE)
    for rows, n, k in [(6912, 768, 256), (8960, 768, 192), (3840, 3040, 760), (4864, 2560, 640), (8192, 960, 320), (6144, 192, 192), (4160, 64, 64),
                       (64, 4160, 64), (8192, 3072, 3072)]:
        assert not ask(rows, n, k)
    for bad in [(0, 8, 8), (8, 4, 8), (8, 8, 10)]:
        with pytest.raises(Exception):
            ask(*bad)
    with pytest.raises(Exception):
        ask(8, 8, 8, False, K.GEMM_A_STRIDED)


def test_tiles_told_apart():
    """With PLAN_TILES the kernels that are PRODUCT_SMALL otherwise have names of their own, and nothing else changes."""
    rng = random.Random(13)
    seen = set()
    for _ in range(1000):
        m, n, k, flags, ws = log_int(rng, 8, 8000, 8), log_int(rng, 8, 8000, 8), log_int(rng, 8, 8000, 8), rng.choice([0, A, B, A | B]), rng.choice([0, 64 << 20])
        c = K.ConvShape(log_int(rng, 1, 256), *[rng.randint(7, 128)] * 2, log_int(rng, 8, 320, 8), log_int(rng, 8, 320, 8), *[rng.choice([1, 3, 7])] * 2, rng.choice([1, 2]), 3)
        which = rng.randrange(3)
        for ask, f, own in [(lambda f: K.gemm_plan(m, n, k, f, 0, False, ws), flags, {K.PRODUCT_SLICES}),
                            (lambda f: K.conv_plan(c, f, ws), which, {K.PRODUCT_BROAD, K.PRODUCT_FLAT} if which == K.CONV_WGRAD else {K.PRODUCT_BROAD})]:
            for plain, told in zip(ask(f), ask(f | K.PLAN_TILES)):
                assert plain[1:] == told[1:] and (plain[0] == told[0] or (plain[0] == K.PRODUCT_SMALL and told[0] in own)), (plain, told)
                seen.add(told[0])
    assert {K.PRODUCT_SLICES, K.PRODUCT_BROAD, K.PRODUCT_FLAT} <= seen


def test_rounds_of_small_tiles():
    """Many k-tiles in more than one round of workgroups are slower on 64 x 64 than on 128 x 128, in one round faster."""
    for m, n, k in [(1352, 816, 2008), (2224, 744, 1960), (1032, 1424, 1752)]:
        assert K.gemm_plan(m, n, k, A | B | K.PLAN_TILES)[0][0] == K.PRODUCT_SMALL
    assert K.gemm_plan(1024, 1024, 2008, A | B | K.PLAN_TILES)[0][0] == K.PRODUCT_SLICES


def fwd(*a):
    return K.conv_plan(K.ConvShape(*a), K.CONV_FWD | K.PLAN_TILES)[0][0]


def back(*a):
    return K.conv_plan(K.ConvShape(*a), K.CONV_DGRAD | K.PLAN_TILES)[0][0]


def test_gathers_beyond_the_caches():
    """256 x 64 is slower than 128 x 128 where the L2 caches do not hold what its workgroups read again for the next tap."""
    assert back(47, 113, 113, 40, 232, 7, 7, 1, 3) == fwd(27, 142, 142, 104, 16, 5, 5, 2, 2) == back(18, 91, 91, 8, 200, 3, 3, 1, 1) == K.PRODUCT_SMALL
    assert fwd(93, 119, 119, 160, 48, 3, 3, 1, 1) == fwd(8, 256, 256, 64, 64, 3, 3, 1, 1) == K.PRODUCT_NARROW


def test_input_gradients_by_parity():
    """256 x 160 is slower than 128 x 128 with few taps and channels, 256 x 64 with very many."""
    assert back(7, 168, 168, 160, 16, 3, 3, 2, 1) == back(84, 82, 82, 152, 128, 1, 1, 2, 0) == K.PRODUCT_SMALL
    assert back(31, 160, 160, 160, 264, 7, 7, 2, 3) == back(256, 32, 32, 160, 320, 3, 3, 2, 1) == K.PRODUCT_BROAD
    assert back(21, 182, 182, 40, 424, 7, 7, 2, 3) == back(21, 227, 227, 32, 264, 7, 7, 2, 3) == K.PRODUCT_SMALL
    assert back(5, 236, 236, 8, 320, 7, 7, 2, 3) == back(64, 224, 224, 8, 64, 7, 7, 2, 3) == K.PRODUCT_NARROW
