"""Outputs of so many tiles that the smallest direct-load tiles' work-items pass the 2^32
of a grid (2^24 tiles): products of one k, whose elements are single rounded products, so
equality with the elementwise product needs no tolerance."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mg.lib()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    yield torch.device("cuda:0")
    torch.cuda.empty_cache()


def column(m, dev, seed):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    return torch.rand((m, 1), device=dev, dtype=torch.float32, generator=g) * 2 - 1


# 2^24 tiles of 64 x 32 at m = 2^30 (one work-item too many), one tile less, one more
@pytest.mark.parametrize("m", [(1 << 30) - 64, 1 << 30, (1 << 30) + 1])
def test_product_of_2_24_tiles(dev, m):
    print(f"large grid m={m}", flush=True)
    A, B = column(m, dev, 1), column(4, dev, 2).view(1, 4)
    C = torch.full((m, 4), float("nan"), device=dev, dtype=torch.float32)
    mg.gemm(A, B, C)
    torch.cuda.synchronize()
    for i in range(0, m, 1 << 28):
        assert torch.equal(C[i:i + (1 << 28)], A[i:i + (1 << 28)] * B)


def test_default_plan_of_more_than_2_24_tiles(dev):
    """17 problems of 2^20 - 1 tile rows: more tiles than a grid of one work-group per
    tile may hold, few enough for a tile map."""
    m = (1 << 26) - 64
    print(f"large plan 17 x {m}", flush=True)
    A = column(m, dev, 3)
    Bs = [column(4, dev, 10 + i).view(1, 4) for i in range(17)]
    Cs = [torch.full((m, 4), float("nan"), device=dev, dtype=torch.float32) for _ in range(17)]
    plan = mg.BatchedPlan([A] * 17, Bs, Cs)
    assert plan.info()["tiles"] == 17 * ((1 << 20) - 1)
    plan.execute()
    torch.cuda.synchronize()
    for b, c in zip(Bs, Cs):
        assert torch.equal(c, A * b)
    plan.destroy()


def test_list_of_products_of_many_tiles(dev):
    """Products of 2^22 tiles of 32 x 32 each, too many of them to share launches, beside
    small ones that do."""
    m = 1 << 27
    print(f"large list 8 x {m}", flush=True)
    A, small = column(m, dev, 5), column(100, dev, 6)
    Bs = [column(4, dev, 20 + i).view(1, 4) for i in range(16)]
    As = [A if i % 2 else small for i in range(16)]
    Cs = [torch.full((a.shape[0], 4), float("nan"), device=dev, dtype=torch.float32) for a in As]
    mg.set_stream(torch.cuda.current_stream())
    mg.gemm_batched(As, Bs, Cs)
    torch.cuda.synchronize()
    for a, b, c in zip(As, Bs, Cs):
        assert torch.equal(c, a * b)
