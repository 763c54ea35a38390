"""The sum of the partial planes of a product whose k is cut, for every number of planes
(2 to 16, one kernel each): integer values keep every partial sum exact in both types, so
the result is the exact product whatever the order; C is read only with beta != 0 and
written nowhere else."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402


@pytest.mark.parametrize("dtype", [mg.F64, mg.F32])
@pytest.mark.parametrize("S,n", [(S, 64) for S in range(2, 17)] + [(4, 4), (4, 68), (4, 128), (4, 132)])
def test_every_number_of_planes(dtype, S, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # 256 // S tiles of 128 x 128, each in S ranges, fill 256 compute units once; the
    # sum takes 4, 4, 2, 2 and 1 rows to a work-group at n = 4, 64, 68, 128 and 132
    m, k = 128 * (256 // S // -(-n // 128)) - 5, 256 * S * -(-8 // S)
    print(f"split sum dtype={mg.DTYPE_NAMES[dtype]} {m}x{n}x{k} S={S}", flush=True)
    assert mg.choice(m, n, k, dtype)[1] == S
    tdt = torch.float64 if dtype == mg.F64 else torch.float32
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(S)
    A, B, C = (torch.randint(-3, 4, s, device=dev, generator=g).to(tdt)
               for s in ((m, k), (k, n), (m, n)))
    want = A.double() @ B.double()
    buf = torch.full((m, n + 4), float("nan"), device=dev, dtype=tdt)
    for alpha, beta in ((1.0, 0.0), (2.0, -1.0)):
        if beta:
            buf[:, :n] = C
        mg.gemm(A, B, buf[:, :n], alpha, beta)
        torch.cuda.synchronize()
        assert torch.equal(buf[:, :n].double(), alpha * want + beta * C.double())
        assert bool(torch.isnan(buf[:, n:]).all())
