"""Products of less than one or two k-steps on the direct-load tiles, where FP32 tiles run
only the groups of 8 k that hold values: the values of the register-staged 64 x 64 x 16 configuration
(every tile sums k in the same order; equality needs no tolerance), also of products that
underflow to zero (whose sign depends on the zeros a configuration pads k with: k = 16
fills its k-step and half of a k-step of 32), on outputs of one tile to thousands, with
NaN around the operands."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402


def embedded(rows, cols, pad, off, tdt, dev, gen, scale):
    ld = cols + pad
    buf = torch.full((off + (rows - 1) * ld + cols,), float("nan"), device=dev, dtype=tdt)
    v = torch.as_strided(buf, (rows, cols), (ld, 1), off)
    v.copy_((torch.rand((rows, cols), device=dev, dtype=tdt, generator=gen) * 2 - 1) * scale)
    return v


@pytest.mark.parametrize("dtype", [mg.F64, mg.F32])
@pytest.mark.parametrize("mn", [(40, 70), (700, 901), (3001, 1000), (2047, 7000)])
def test_short_k(dtype, mn):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n = mn
    dev = torch.device("cuda:0")
    tdt, tiny = (torch.float64, 1e-170) if dtype == mg.F64 else (torch.float32, 1e-25)
    two_stage = [c for c in mg.configs(dtype) if c.as_tuple() == (64, 64, 16, 4, 2, 1, 0)][0]
    g = torch.Generator(device=dev)
    for k in (1, 2, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 40, 63, 64, 65):
        for scale in (1.0, tiny):
            print(f"short k dtype={mg.DTYPE_NAMES[dtype]} {m}x{n}x{k} scale {scale}", flush=True)
            g.manual_seed(m + n + k)
            A = embedded(m, k, k % 3, 1, tdt, dev, g, scale)
            B = embedded(k, n, k % 2, k % 4, tdt, dev, g, scale)
            C = [torch.full((m, n), float("nan"), device=dev, dtype=tdt) for _ in range(2)]
            mg.gemm(A, B, C[0])
            mg.gemm(A, B, C[1], cfg=two_stage)
            torch.cuda.synchronize()
            assert bool(torch.isfinite(C[0]).all()) and bool((C[0] == 0).all()) == (scale == tiny)
            assert torch.equal(C[0], C[1]), k
