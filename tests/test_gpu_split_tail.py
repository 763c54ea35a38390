"""The split tail of the slice emulations: tiles beyond whole rounds of the compute
units (or a small product's only tiles) have their k cut between work-groups.  The level
sums are exact integers in any order, so every result is bitwise the oracle's."""
import numpy as np
import pytest

import synth
from test_gpu_split import FMT, dev, gpu_split, orc, say  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402

# one tile, a few ragged ones (k past a multiple of every chunk and range), and one
# tile more than a 256-unit card has compute units (int8 128 x 64 tiles, bf16 64 x 128,
# FP8 64 x 64), whose last is ragged
CASES = [(mg.SPLIT_INT8, (1, 1, 4097)), (mg.SPLIT_INT8, (150, 190, 3001)),
         (mg.SPLIT_INT8, (128 * 256 + 5, 60, 701)),
         (mg.SPLIT_BF16, (1, 1, 4097)), (mg.SPLIT_BF16, (150, 190, 3001)),
         (mg.SPLIT_BF16, (64 * 256 + 5, 120, 2101)),
         (mg.SPLIT_FP8, (1, 1, 4097)), (mg.SPLIT_FP8, (150, 190, 3001)),
         (mg.SPLIT_FP8, (64 * 256 + 5, 60, 1001))]


@pytest.mark.parametrize("beta", [0.0, -0.5])
@pytest.mark.parametrize("dtype,shape", CASES)
def test_tail_bitwise_equal_to_oracle(dev, orc, dtype, shape, beta):  # noqa: F811
    m, n, k = shape
    fmt, S = FMT[dtype]
    say(f"split tail {mg.DTYPE_NAMES[dtype]} {shape} beta={beta}")
    A = synth.wide_range((m, k), 11)
    B = synth.wide_range((k, n), 12)
    C = synth.uniform_pm1((m, n), 13)
    got = gpu_split(dev, A, B, C, 1.25, beta, dtype)
    rows = np.unique(np.r_[0:min(m, 200), max(0, m - 200):m])
    want = orc.split_gemm(1.25, A[rows], B, beta, C[rows], fmt=fmt, S=S, nthreads=8)
    assert np.array_equal(got[rows], want)
