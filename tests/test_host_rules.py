"""The host side's rules that need no GPU (csrc/host_rules.h), compiled alone with the
host compiler: which operands the direct loads take and which grids a launch, how long a tile takes with k whole or in
ranges, which lists' products depend on each other, what of a list runs when one of its products fails, and which networks train on
the step kernel."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1706_10086_amd", "csrc")


@pytest.fixture(scope="module")
def R(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rules") / "host_rules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(HERE, "host_rules.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    i64 = ctypes.c_int64
    lib.grid_fits_c.argtypes = [i64, i64]
    lib.list_grid_fits_c.argtypes = [i64, i64]
    lib.may_hold_c.argtypes = [i64, i64, i64]
    lib.direct_loads_c.argtypes = [i64] * 11
    lib.list_joins_c.argtypes = [i64] * 9
    i32 = ctypes.c_int
    lib.step_blocks_c.argtypes = [i32, i32, i32, i64, i32]
    lib.tile_time_c.argtypes = [i32, i32, i64, i64, i64, i64, i64, i32]
    lib.tile_time_c.restype = ctypes.c_double
    lib.tile_taken_c.argtypes = [i32, i32, i64, i64, i64, i64, i32]
    lib.tile_c.argtypes = [i32, i32, *[ctypes.POINTER(ctypes.c_int32)] * 3]
    return lib


@pytest.mark.parametrize("threads", [64, 256, 512])
def test_grid_counts_work_items_in_32_bits(R, threads):
    edge = (1 << 32) // threads
    assert R.grid_fits_c(edge - 1, threads) and R.grid_fits_c(1, threads)
    assert not R.grid_fits_c(edge, threads) and not R.grid_fits_c(1 << 40, threads)


def test_a_full_list_of_the_largest_products_fits_a_grid(R):
    """56 products of the most 32 x 32 tiles that may share a launch: their work-items
    (256 to a tile) stay below 2^32."""
    most = max(t for t in range(299000, 300200) if R.list_grid_fits_c(32 * t, 4))
    assert most * 56 * 256 < 1 << 32 <= (most + 1) * 56 * 256
    # the same count in two dimensions, and sizes at a tile's edge
    assert R.list_grid_fits_c(32 * most - 31, 32) and not R.list_grid_fits_c(32 * most + 1, 1)
    assert R.list_grid_fits_c(1024, 1024) and not R.list_grid_fits_c(1 << 27, 4)


def dependent(R, spans):
    n = len(spans)
    b, e = ((ctypes.c_int64 * n)(*[s[i] for s in spans]) for i in (0, 1))
    w = (ctypes.c_int32 * n)(*[int(s[2]) for s in spans])
    return bool(R.dependent_c(n, b, e, w))


def test_dependent_products_are_found(R):
    """Against every pair: a written span that meets another one, in any order of the
    list, at shared and touching ends and with one inside the other."""
    cuts = [0, 4, 5, 8, 9, 12]
    spans = [(a, b, w) for a, b in itertools.combinations(cuts, 2) for w in (False, True)]
    meets = lambda x, y: x[0] < y[1] and y[0] < x[1]  # noqa: E731
    seen = set()
    for some in itertools.permutations(spans, 3):
        want = any(meets(x, y) and (x[2] or y[2]) for x, y in itertools.combinations(some, 2))
        assert dependent(R, some) == want, some
        seen.add(want)
    assert seen == {True, False}
    assert not dependent(R, [(0, 4, True)]) and not dependent(R, [(0, 4, False)] * 5)


def window(R, what, group_rc=0):
    n = len(what)
    order = (ctypes.c_int32 * n)()
    ran, told = ctypes.c_int(), ctypes.c_int()
    rc = R.window_c(n, (ctypes.c_int32 * n)(*what), group_rc, order, ctypes.byref(ran),
                    ctypes.byref(told))
    return rc, list(order[:ran.value]), told.value


@pytest.mark.parametrize("what,group_rc,rc,ran,told", [
    ([0, 1, 0, 1, 1], 0, 0, [0, 2, 1, 3, 4], -1),
    ([1, 1], 0, 0, [0, 1], -1),
    ([0, 0], 0, 0, [0, 1], -1),
    # a failure leaves what came before it done and what comes after it undone
    ([1, 0, 1, -7, 1, 0], 0, -7, [1, 0, 2], 1),
    ([1, -3], 0, -3, [0], 0),
    ([-3, 1, 0], 0, -3, [], 0),
    # the first error is the one reported
    ([1, 0, -7], -9, -7, [1, 0], 1),
    ([1, 0], -9, -9, [1, 0], -1),
])
def test_a_failing_product_leaves_the_ones_before_it_done(R, what, group_rc, rc, ran, told):
    assert window(R, what, group_rc) == (rc, ran, told)


@pytest.mark.parametrize("dims,rows,blocks", [
    # the tile-choice network, the smallest sets, one tile of rows more
    ((6, 64, 247), 13600, 213), ((6, 64, 247), 1, 1), ((6, 64, 247), 65, 2), ((6, 100, 247), 65, 3),
    ((6, 64, 247), 1 << 20, 256), ((32, 128, 247), 500, 16), ((6, 64, 768), 1, 1),
    # many outputs on few rows (times at host_rules.h), and rows enough for them
    ((6, 64, 769), 768, 0), ((6, 64, 769), 769, 13), ((6, 64, 4096), 4095, 0),
    ((6, 64, 4096), 13600, 213), ((6, 128, 2048), 500, 0), ((6, 128, 2048), 8192, 256),
    # more than 64 hidden units: rounds x outputs at and past the line
    ((6, 128, 1024), 16384, 256), ((6, 128, 1025), 16384, 0), ((6, 128, 2048), 8193, 0),
    ((6, 65, 256), 65536, 256), ((6, 65, 257), 65536, 0), ((6, 64, 4096), 1 << 20, 256),
    # widths the kernel does not hold
    ((33, 64, 20), 90, 0), ((6, 129, 20), 90, 0),
])
def test_networks_on_the_step_kernel(R, dims, rows, blocks):
    assert R.step_blocks_c(*dims, rows, 256) == blocks


def tile(R, f32, i):
    v = [ctypes.c_int32() for _ in range(3)]
    R.tile_c(f32, i, *[ctypes.byref(x) for x in v])
    return tuple(x.value for x in v)


def pick(R, f32, m, n, k, S, kc):
    times = {i: R.tile_time_c(f32, i, m, n, k, S, kc, 256) for i in range(6)
             if R.tile_taken_c(f32, i, m, n, k, S, 256)}
    return tile(R, f32, min(times, key=times.get))


@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("i", range(6))
def test_time_of_ranges(R, f32, i):
    """A last range as long as the others counts as one of them (the time of a product
    of as many times the rows, whose tiles are as many); a shorter one costs no more, and
    costs nothing but its start where it fits beside the full ones."""
    bm, bn, bk = tile(R, f32, i)
    for tiles in (1, 40, 100, 128, 200, 300, 700):
        for S in (2, 3, 5, 16):
            kc = 1024
            time = lambda k: R.tile_time_c(f32, i, tiles * bm, bn, k, S, kc, 256)  # noqa: E731
            full = time(S * kc)
            assert full == R.tile_time_c(f32, i, S * tiles * bm, bn, kc, 1, kc, 256)
            ks = [(S - 1) * kc + r for r in (1, bk, 100, 256, 500, 512, 513, 1000, kc)]
            times = [time(k) for k in ks]
            assert times == sorted(times) and times[-1] == full
            if S * tiles <= 256:
                assert times[0] == full


# FP32 products whose last range is short (times of the six tiles at 256 compute units)
@pytest.mark.parametrize("m,n,k,S,kc,slow", [
    (1441, 488, 5140, 5, 1280, (64, 128, 32)),      # 101 99 80 83 86 89 us
    (2433, 336, 4636, 4, 1280, (64, 128, 32)),      # 103 101 90 89 91 92
    (10061, 120, 3328, 3, 1280, (64, 128, 32)),     # 108 106 96 95 98 101
    (1126, 836, 4344, 4, 1280, (64, 128, 32)),      # 103 101 87 91 95 97
])
def test_a_short_last_range_leaves_the_smaller_tiles_ahead(R, m, n, k, S, kc, slow):
    assert (S - 1) * kc < k < S * kc
    assert pick(R, 1, m, n, S * kc, S, kc) == slow
    assert pick(R, 1, m, n, k, S, kc) != slow


@pytest.mark.parametrize("f32,m,n,k", [(0, 722, 4414, 32), (0, 7462, 446, 2), (0, 834, 2120, 109),
                                       (0, 1038, 3158, 95), (1, 247, 12851, 45), (1, 1330, 1468, 27)])
def test_short_products_of_one_round_leave_the_wide_tiles(R, f32, m, n, k):
    """Products that the wide tiles' estimates undercut, each 4-20 % slower there."""
    times = [R.tile_time_c(f32, i, m, n, k, 1, k, 256) for i in range(6)]
    assert tile(R, f32, times.index(min(times)))[1] == 128
    assert pick(R, f32, m, n, k, 1, k)[1] < 128


def test_where_the_wide_tiles_are_left_out(R):
    """Whole products of at most 512 k whose 64 x 64 tiles are resident at once (four to a
    compute unit); ranges of k, longer and larger products keep every tile."""
    for f32 in (0, 1):
        for i in range(6):
            wide = tile(R, f32, i)[1] == 128
            taken = lambda *a: bool(R.tile_taken_c(f32, i, *a, 256))  # noqa: E731
            assert taken(2048, 2048, 512, 1) == (not wide)
            assert taken(1, 1, 1, 1) == (not wide)
            assert taken(2048, 2048, 513, 1) and taken(2048, 2049, 512, 1)
            assert taken(2049, 2048, 512, 1) and taken(256, 256, 4096, 8)


def test_a_workspace_is_given_up_only_for_one_that_fits(R):
    """100 bytes held, 120 wanted: grown with 20 free, kept with 19; what is held needs
    no free memory."""
    assert R.may_hold_c(100, 20, 120) and not R.may_hold_c(100, 19, 120)
    assert R.may_hold_c(120, 0, 120) and R.may_hold_c(0, 120, 120) and not R.may_hold_c(0, 119, 120)


BASE = 1 << 20


@pytest.mark.parametrize("es", [8, 4])
def test_what_the_direct_loads_take(R, es):
    loads = lambda m=64, n=64, k=64, A=BASE, lda=64, B=BASE, ldb=64: bool(  # noqa: E731
        R.direct_loads_c(es, 128, 128, 32, m, n, k, A, lda, B, ldb))
    assert loads() and loads(1, 16 // es, 1)
    assert not loads(n=16 // es - 1) and not loads(m=0) and not loads(k=0)
    assert loads(A=BASE + 4) and loads(B=BASE + 12)
    assert not loads(A=BASE + 2) and not loads(B=BASE + 1)
    # 128 rows of A, 32 of B and a row's 128 elements below 2^31 bytes
    edge = (1 << 31) // (128 * es)
    assert loads(lda=edge - 1) and not loads(lda=edge)
    edge = ((1 << 31) // es - 128) // 32
    assert loads(ldb=edge - 1) and not loads(ldb=edge)


@pytest.mark.parametrize("es", [8, 4])
def test_plans_and_lists_under_gpu_test_take_both_paths(R, es):
    """The shapes of the GPU tests that compare a default plan and a list with products in
    turn: some of them are for the direct loads and some are not, and the list has more
    products that share launches than one launch takes."""
    off = 4 if es == 4 else 8
    plan = [(1, 1, 1), (70, 1, 33), (65, 2, 64), (20, 3, 17), (129, 5, 40), (64, 64, 48), (63, 65, 1),
            (200, 333, 77), (333, 200, 130), (17, 1000, 5), (1000, 17, 250)]
    direct = [bool(R.direct_loads_c(es, 64, 64, 32 if es == 4 else 16, m, n, k, BASE + off * (n % 2),
                                    k + (m + n) % 3, BASE + off * (m % 4), n + k % 2))
              for m, n, k in plan]
    assert direct == [n >= 16 // es for _, n, _ in plan] and set(direct) == {True, False}
    rng = np.random.RandomState(5)
    shapes = [tuple(int(2.0 ** rng.uniform(0, 8)) for _ in range(3)) for _ in range(130)]
    shapes += [(700, 650, 600), (33, 2, 9), (40, 1, 40), (1, 1, 1)]
    joins = [bool(R.list_joins_c(es, m, n, k, BASE + off, k + 2, BASE + off, n + 1, n + 4))
             for m, n, k in shapes]
    assert sum(joins) > 56 and not all(joins)


def test_which_products_share_launches(R):
    joins = lambda m, n, k, ld=0: bool(R.list_joins_c(8, m, n, k, BASE, max(k, ld), BASE, n, n))  # noqa: E731
    assert joins(1000, 1000, 2000) and not joins(1000, 1000, 2001)        # 4e9 operations
    assert joins(100, 100, 100, (1 << 21) - 1) and not joins(100, 100, 100, 1 << 21)
    assert not joins(100, 1, 100) and not joins(1 << 27, 2, 1)
