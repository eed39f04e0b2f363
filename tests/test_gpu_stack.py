"""Batched calls take several slices per pass through a plan's second
workspace; every slice equals its own call bit for bit, at batches below, at
and past the workspace's slices, where it holds only one or a few, and where
it cannot be allocated (first call under stream capture)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from radon_inputs import uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Plan  # noqa: E402

DEV = "cuda:0"


def _inputs(batch, n, nv, nd, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn((batch, n, n), generator=g, device=DEV), torch.randn((batch, nv, nd), generator=g, device=DEV))


# 64: eight slices, odd view count (odd distance of the ray spectra); 48 x 80, W = 8
# and 4; 1024: four slices fit; 2048: one
@pytest.mark.parametrize("n,nv,nd,W,batch", [(64, 31, 64, 6, 1), (64, 31, 64, 6, 8), (64, 300, 64, 6, 11),
                                             (48, 7, 80, 4, 3), (128, 50, 96, 8, 9), (1024, 9, 1024, 6, 6),
                                             (2048, 3, 2048, 6, 2)])
def test_stacked_slices_equal_single_calls(n, nv, nd, W, batch):
    print(f"stack n={n} nv={nv} nd={nd} W={W} batch={batch}", flush=True)
    plan = Plan(n, uniform_angles(nv), nd, W=W)
    x, y = _inputs(batch, n, nv, nd, n + batch)
    for _ in range(2):
        f, a = plan.forward_batched(x), plan.adjoint_batched(y)
        for b in range(batch):
            assert torch.equal(f[b], plan.forward(x[b])) and torch.equal(a[b], plan.adjoint(y[b]))


def test_stack_under_capture_and_profiling():
    print("stack under capture", flush=True)
    n, nv, batch = 64, 20, 5
    plan = Plan(n, uniform_angles(nv), n)
    x, y = _inputs(batch, n, nv, n, 3)
    want = torch.stack([plan.forward(x[b]) for b in range(batch)])
    before = plan.info()["device_bytes"]
    out = torch.zeros((batch, nv, n), device=DEV)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.forward_batched(x, out=out)          # may not allocate: one slice at a time
    assert plan.info()["device_bytes"] == before
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(plan.forward_batched(x), want)      # eager, with the second workspace
    assert plan.info()["device_bytes"] > before
    plan.set_profiling(True)
    plan.adjoint_batched(y)
    assert plan.stage_times()["A1_ray_fft"][1] == batch        # a stage time stays one slice's
    plan.set_profiling(False)
