"""The direct-load tiles behind the built-in choice: bit for bit the two-stage
kernel's results (every tile sums k in the same order) on rows of any alignment --
odd leading dimensions, bases off the 16-byte grid, rows shorter than a tile whose
last load unit runs past them, partial and whole last k-steps -- with NaN in every
byte around the operands, which neither the zero padding of k nor a clamped load may
let in, and C written nowhere else.  Equality of bits needs no tolerance; products
whose k is cut (another sum order) are held to gamma_{k+2} of the FP64 reference."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mg.lib()
    return torch.device("cuda:0")


def embedded(rows, cols, pad, off, tdt, dev, gen):
    """rows x cols uniform values with leading dimension cols + pad, starting `off`
    elements into a NaN buffer that ends with the last element."""
    ld = cols + pad
    buf = torch.full((off + (rows - 1) * ld + cols,), float("nan"), device=dev, dtype=tdt)
    v = torch.as_strided(buf, (rows, cols), (ld, 1), off)
    v.copy_(torch.rand((rows, cols), device=dev, dtype=tdt, generator=gen) * 2 - 1)
    return buf, v


# (m, n, k, pad of A, pad of B, offset of A, offset of B): tile edges and
# remainders, rows shorter than one load unit's multiple, k below, at and past one
# k-step, outputs from one tile to thousands (so that the choice takes every tile)
SHAPES = [(1, 2, 1, 0, 0, 0, 0), (1, 4, 16, 0, 0, 1, 1), (5, 5, 64, 0, 0, 0, 0),
          (33, 3, 32, 1, 0, 1, 0), (64, 7, 33, 0, 0, 0, 1), (31, 33, 31, 3, 1, 1, 3),
          (65, 63, 127, 0, 0, 0, 0), (200, 1, 50, 0, 0, 0, 0), (300, 129, 300, 1, 5, 3, 1),
          (513, 511, 96, 0, 0, 0, 0), (777, 1030, 250, 1, 0, 0, 2), (1500, 1501, 130, 0, 0, 1, 0),
          (2048, 2050, 64, 0, 0, 0, 0), (3001, 2999, 70, 0, 1, 0, 0), (6000, 130, 99, 0, 0, 0, 0),
          (100, 9000, 40, 2, 3, 0, 1)]


@pytest.mark.parametrize("dtype", [mg.F64, mg.F32])
@pytest.mark.parametrize("shape", SHAPES)
def test_direct_tiles_bitwise(dev, dtype, shape):
    m, n, k, pa, pb, oa, ob = shape
    print(f"direct tiles dtype={mg.DTYPE_NAMES[dtype]} {shape}", flush=True)
    tdt = torch.float64 if dtype == mg.F64 else torch.float32
    g = torch.Generator(device=dev)
    g.manual_seed(m * 31 + n * 7 + k)
    _, A = embedded(m, k, pa, oa, tdt, dev, g)
    _, B = embedded(k, n, pb, ob, tdt, dev, g)
    bufs = [embedded(m, n, 3, 1, tdt, dev, g) for _ in range(2)]
    bufs[1][0].copy_(bufs[0][0])
    before = bufs[0][0].clone()
    two_stage = [c for c in mg.configs(dtype) if c.as_tuple() == (64, 64, 16, 4, 2, 1, 0)][0]
    mg.gemm(A, B, bufs[0][1], 1.5, 0.5)
    mg.gemm(A, B, bufs[1][1], 1.5, 0.5, cfg=two_stage)
    torch.cuda.synchronize()
    got, want = bufs[0][1], bufs[1][1]
    assert bool(torch.isfinite(got).all())
    _, splits = mg.choice(m, n, k, dtype, lda=k + pa, ldb=n + pb)
    assert splits == 1 and torch.equal(got, want)
    # outside the m x n elements the C buffer keeps its NaN
    outside = torch.ones_like(before, dtype=torch.bool)
    torch.as_strided(outside, (m, n), (n + 3, 1), 1).fill_(False)
    assert bool(torch.isnan(bufs[0][0][outside]).all())


@pytest.mark.parametrize("dtype", [mg.F64, mg.F32])
@pytest.mark.parametrize("shape", [(300, 129, 5007, 0, 0, 0, 0), (64, 65, 2561, 1, 1, 1, 0),
                                   (256, 512, 8192, 0, 0, 0, 0)])
def test_direct_tiles_long_k(dev, dtype, shape):
    m, n, k, pa, pb, oa, ob = shape
    print(f"direct tiles, long k dtype={mg.DTYPE_NAMES[dtype]} {shape}", flush=True)
    tdt, u = (torch.float64, 2.0 ** -53) if dtype == mg.F64 else (torch.float32, 2.0 ** -24)
    g = torch.Generator(device=dev)
    g.manual_seed(m + n + k)
    _, A = embedded(m, k, pa, oa, tdt, dev, g)
    _, B = embedded(k, n, pb, ob, tdt, dev, g)
    _, C = embedded(m, n, 0, 0, tdt, dev, g)
    A64, B64, C64 = (x.double().cpu().numpy() for x in (A, B, C))
    mg.gemm(A, B, C, 1.5, 0.5)
    torch.cuda.synchronize()
    err = np.abs(C.double().cpu().numpy() - (1.5 * (A64 @ B64) + 0.5 * C64))
    gam = lambda v: (k + 2) * v / (1 - (k + 2) * v)  # noqa: E731
    # the reference's own rounding adds its gamma with the FP64 unit
    bound = (gam(u) + gam(2.0 ** -53)) * (1.5 * np.abs(A64) @ np.abs(B64) + 0.5 * np.abs(C64))
    assert np.all(err <= bound)


@pytest.mark.parametrize("dtype", [mg.F64, mg.F32])
def test_default_plan_mixes_direct_and_register_staged(dev, dtype):
    """A plan without configurations: problems the direct loads take (any alignment)
    beside rows of fewer elements than one load unit, which they cannot; bit for bit
    the 64 x 64 x 16 configuration per problem, in one configuration group."""
    tdt = torch.float64 if dtype == mg.F64 else torch.float32
    g = torch.Generator(device=dev)
    g.manual_seed(17)
    shapes = [(m, n, k, (m + n) % 3, k % 2, n % 2, m % 4) for m, n, k in
              [(1, 1, 1), (70, 1, 33), (65, 2, 64), (20, 3, 17), (129, 5, 40), (64, 64, 48),
               (63, 65, 1), (200, 333, 77), (333, 200, 130), (17, 1000, 5), (1000, 17, 250)]]
    As = [embedded(m, k, pa, oa, tdt, dev, g)[1] for m, n, k, pa, pb, oa, ob in shapes]
    Bs = [embedded(k, n, pb, ob, tdt, dev, g)[1] for m, n, k, pa, pb, oa, ob in shapes]
    Cs = [embedded(m, n, pa, ob, tdt, dev, g)[1] for m, n, k, pa, pb, oa, ob in shapes]
    want = [c.clone() for c in Cs]
    cfg = [c for c in mg.configs(dtype) if c.as_tuple() == (64, 64, 16, 4, 2, 1, 0)][0]
    plan = mg.BatchedPlan(As, Bs, Cs, 1.25, -0.5)
    info = plan.info()
    assert info["buckets"] == 1
    assert info["tiles"] == sum(-(-m // 64) * -(-n // 64) for m, n, *_ in shapes)
    plan.execute()
    for a, b, c in zip(As, Bs, want):
        mg.gemm(a, b, c, 1.25, -0.5, cfg=cfg)
    torch.cuda.synchronize()
    for s, c, w in zip(shapes, Cs, want):
        print(f"default plan dtype={mg.DTYPE_NAMES[dtype]} {s}", flush=True)
        assert torch.equal(c, w), s
    plan.destroy()


@pytest.mark.parametrize("dtype", [mg.F64, mg.F32])
def test_lists_share_launches(dev, dtype):
    """gemm_batched: more products than one launch takes, with empty ones, alpha = 0, a
    split of k and rows shorter than a load unit among them, give the bits of gemm
    called in turn; so do lists whose products depend on each other (a result read as
    A, as B, rewritten, or interleaved with another's rows)."""
    tdt = torch.float64 if dtype == mg.F64 else torch.float32
    g = torch.Generator(device=dev)
    g.manual_seed(23)
    rng = np.random.RandomState(5)
    shapes = [tuple(int(2.0 ** rng.uniform(0, 8)) for _ in range(3)) for _ in range(130)]
    shapes += [(100, 60, 5000), (64, 64, 4096), (700, 650, 600), (33, 2, 9), (40, 1, 40), (1, 1, 1)]
    As = [embedded(m, k, i % 3, i % 2, tdt, dev, g)[1] for i, (m, n, k) in enumerate(shapes)]
    Bs = [embedded(k, n, i % 2, i % 4, tdt, dev, g)[1] for i, (m, n, k) in enumerate(shapes)]
    Cs = [embedded(m, n, i % 5, 0, tdt, dev, g)[1] for i, (m, n, k) in enumerate(shapes)]
    As.append(torch.zeros((0, 8), device=dev, dtype=tdt))
    Bs.append(torch.zeros((8, 4), device=dev, dtype=tdt))
    Cs.append(torch.zeros((0, 4), device=dev, dtype=tdt))
    alphas = [0.0 if i == 3 else 1.25 for i in range(len(As))]
    want = [c.clone() for c in Cs]
    print(f"list of {len(As)} dtype={mg.DTYPE_NAMES[dtype]}", flush=True)
    mg.set_stream(torch.cuda.current_stream())
    mg.gemm_batched(As, Bs, Cs, alphas, -0.5)
    for a, b, c, al in zip(As, Bs, want, alphas):
        mg.gemm(a, b, c, al, -0.5)
    torch.cuda.synchronize()
    for i, (c, w) in enumerate(zip(Cs, want)):
        assert torch.equal(c, w), (i, tuple(c.shape))

    def chain():
        x = [torch.rand((48, 48), device=dev, dtype=tdt, generator=g) for _ in range(5)]
        wide = torch.rand((48, 96), device=dev, dtype=tdt, generator=g)
        l, r = wide[:, :48], wide[:, 48:]
        # x[2] is read as A, then as B, then rewritten; the halves of `wide` interleave
        return x + [wide], [(x[0], x[1], x[2]), (x[2], x[1], x[3]), (x[0], x[2], x[4]),
                            (x[1], x[0], x[2]), (x[0], x[1], l), (x[1], x[0], r)]

    for lo, hi in ((0, 2), (0, 3), (0, 6), (1, 4), (4, 6)):
        bufs, probs = chain()
        probs = probs[lo:hi]
        saved = [b.clone() for b in bufs]
        print(f"dependent list {lo}:{hi}", flush=True)
        mg.gemm_batched(*zip(*probs), 1.0, 0.5)
        torch.cuda.synchronize()
        got = [b.clone() for b in bufs]
        for b, s in zip(bufs, saved):
            b.copy_(s)
        for a, b, c in probs:
            mg.gemm(a, b, c, 1.0, 0.5)
        torch.cuda.synchronize()
        for b, w in zip(got, bufs):
            assert torch.equal(b, w), (lo, hi)
