"""A large product from host memory keeps the reported configuration, whose tiles read
less over the host link: on the direct-load tiles of device-resident operands FP32 8192^3
took three times as long.  The default and the configuration named, in turn, best of
three: no more than twice apart, and the same bits."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402


def test_large_product_from_host_memory():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 8192
    cfg, splits = mg.choice(n, n, n, mg.F32)
    assert splits == 1
    bufs = [mg.HostBuffer(4 * n * n) for _ in range(3)]
    for i, b in enumerate(bufs[:2]):
        b.array((n, n), "float32")[:] = (torch.arange(n * n, dtype=torch.float32) % (7 + i) - 3).view(n, n).numpy()
    stream = torch.cuda.current_stream()

    def run(c):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        rc = mg.gemm_ex_raw(n, n, n, 1.0, bufs[0].dev, n, bufs[1].dev, n, 0.0, bufs[2].dev, n, mg.F32, c,
                            stream.cuda_stream)
        e[1].record()
        torch.cuda.synchronize()
        assert rc == 0
        return e[0].elapsed_time(e[1]), torch.from_numpy(bufs[2].array((n, n), "float32")).clone()

    best = {}
    results = []
    for _ in range(3):
        for name, c in (("default", None), ("named", cfg)):
            ms, out = run(c)
            print(f"host memory {name} {ms:.1f} ms", flush=True)
            best[name] = min(ms, best.get(name, ms))
            results.append(out)
    assert all(torch.equal(r, results[0]) for r in results[1:])
    assert best["default"] <= 2.0 * best["named"]
    for b in bufs:
        b.free()
