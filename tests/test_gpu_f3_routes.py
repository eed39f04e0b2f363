"""Forward interpolation on either side of the lines between reading the grid directly and
staging it: the same bits as an uneven batch, which always stages, and as the calls of
single slices. Views just below and above each line: points = slices views (n + 1) W^2
against 6e6 (W = 8: 9e6) up to 512^2 pixels in all, 3.5e6 + 1.25 pixels (W = 8: 3e6 +
2.5 pixels) above."""
import pytest

torch = pytest.importorskip("torch")

from radon_inputs import uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Batch, Plan  # noqa: E402

DEV = "cuda:0"


def _line(n, W, slices):
    pixels = slices * n * n
    if pixels <= 512 * 512:
        limit = 9e6 if W == 8 else 6e6
    else:
        limit = 3e6 + 2.5 * pixels if W == 8 else 3.5e6 + 1.25 * pixels
    return int(limit / (slices * (n + 1) * W * W))


@pytest.mark.parametrize("n,W,slices", [(64, 4, 1), (64, 6, 1), (64, 8, 1), (40, 6, 1), (640, 4, 1), (640, 6, 1),
                                        (640, 8, 1), (64, 6, 8), (128, 4, 5), (128, 8, 3), (512, 6, 4), (512, 8, 2)])
@pytest.mark.parametrize("side", [-1, 2])
def test_either_side_of_the_line(n, W, slices, side):
    nv = _line(n, W, slices) + side
    print(f"f3 routes n={n} W={W} slices={slices} nv={nv}", flush=True)
    plan = Plan(n, uniform_angles(nv), n, W=W)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n + W)
    x = torch.randn((slices, n, n), generator=gen, device=DEV)
    got = plan.forward_batched(x)
    batch = Batch([plan])
    want = torch.empty((nv, n), device=DEV)
    for b in range(slices):
        batch.forward([x[b]], [want])
        torch.cuda.synchronize()
        assert torch.isfinite(want).all() and float(want.abs().max()) > 0
        assert torch.equal(got[b], want) and torch.equal(plan.forward(x[b]), want), b
