"""Uneven batches on either side of the sizes up to which the launches of different
lengths run on one branch and on two: every slice equals its own call bit for bit, on
replays too, whatever number of branches is asked for."""
import pytest

torch = pytest.importorskip("torch")

from radon_inputs import uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Batch, Plan  # noqa: E402

DEV = "cuda:0"


# 4.2, 5.1 and 9.2 million pixels; six sides; one slice; one length
@pytest.mark.parametrize("shapes,asked", [([(1536, 5), (1280, 9), (512, 20)], 4), ([(1536, 5), (1280, 9), (1024, 20)], 4),
                                          ([(1536, 5), (1280, 9), (1024, 20)], 1), ([(2560, 3)], 4),
                                          ([(2560, 4), (1280, 9), (1024, 20)], 4),
                                          ([(64, 9), (80, 9), (96, 9), (128, 9), (160, 9), (192, 9)], 4),
                                          ([(1536, 5), (1536, 9)], 16)])
def test_batch_branches(shapes, asked):
    print(f"batch branches {shapes} {asked}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(asked)
    plans = [Plan(n, uniform_angles(v), n) for n, v in shapes]
    x = [torch.randn((n, n), generator=gen, device=DEV) for n, _ in shapes]
    y = [torch.randn((v, n), generator=gen, device=DEV) for n, v in shapes]
    batch = Batch(plans, n_branches=asked)
    f, a = [torch.empty_like(t) for t in y], [torch.empty_like(t) for t in x]
    for rep in range(3):
        for t in f + a:
            t.fill_(float("nan"))
        batch.forward(x, f)
        batch.adjoint(y, a)
        torch.cuda.synchronize()
        for p, xi, yi, fi, ai in zip(plans, x, y, f, a):
            assert torch.equal(fi, p.forward(xi)) and torch.equal(ai, p.adjoint(yi)), rep
    assert batch.graphs_recorded() == 2
