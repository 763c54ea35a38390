"""The host side's rules that need no GPU (csrc/host_rules.h), compiled alone with the
host compiler: which grids a launch may take, which lists' products depend on each
other, what of a list runs when one of its products fails, and which networks train on
the step kernel."""
import ctypes
import itertools
import os
import subprocess

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
    i32 = ctypes.c_int
    lib.step_blocks_c.argtypes = [i32, i32, i32, i64, i32]
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
