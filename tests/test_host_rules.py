"""The host side's rules that need no GPU (csrc/host_rules.h), compiled alone with the
host compiler: which grids a launch may take."""
import ctypes
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
