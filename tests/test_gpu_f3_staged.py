"""The staged forward interpolation of one plan, which calls with few samples do not take:
every kernel width and tile size, items shorter than a tile's samples and as many as
fit, ragged geometries and several slices per pass, against the FP64 gridding oracle.
The view counts lie 4 to 20% above the line from which a plan stages (6e6 points, views
(n_det + 1) W^2, and 9e6 with W = 8)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.grid import grid_forward  # noqa: E402
from radon_inputs import random_image, uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Batch, Plan  # noqa: E402

DEV = "cuda:0"
TOL = 1e-5     # float32 transforms of these lengths, as for every decomposition


def _rel(a, ref):
    return np.linalg.norm(a.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("W,nv", [(4, 6001), (6, 2700), (8, 2301)])
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_tiles_and_items(W, nv, tile):
    n = 64
    x, ang = random_image(17, n), uniform_angles(nv)
    ref = grid_forward(x.astype(np.float64), ang, n, W=W)
    xd = torch.from_numpy(x).to(DEV)
    outs = []
    for chunk in (256, 2048):
        print(f"staged n={n} W={W} nv={nv} tile={tile} chunk={chunk}", flush=True)
        plan = Plan(n, ang, n, W=W, tuning={"tile": tile, "f3_chunk": chunk})
        outs.append((plan.forward(xd), plan.info()["n_fitems"]))
        assert _rel(outs[-1][0], ref) <= TOL, chunk
    assert outs[0][1] > outs[1][1]          # shorter items, more of them


# 40 rows take tiles of 8 only; an odd view count; detectors unlike the side
@pytest.mark.parametrize("n,nv,nd,W", [(40, 3601, 48, 6), (48, 7001, 64, 4), (192, 621, 256, 8), (96, 3501, 48, 8)])
def test_ragged(n, nv, nd, W):
    print(f"staged n={n} nv={nv} nd={nd} W={W}", flush=True)
    x, ang = random_image(18, n), uniform_angles(nv) + 0.01
    plan = Plan(n, ang, nd, W=W)
    assert _rel(plan.forward(torch.from_numpy(x).to(DEV)), grid_forward(x.astype(np.float64), ang, nd, W=W)) <= TOL


# three slices pass the line that one does not
@pytest.mark.parametrize("W,nv,tile", [(4, 2101, 16), (6, 951, 32), (8, 801, 8), (8, 801, 32)])
def test_several_slices(W, nv, tile):
    n, batch = 64, 3
    print(f"staged stack W={W} nv={nv} tile={tile}", flush=True)
    ang = uniform_angles(nv)
    plan = Plan(n, ang, n, W=W, tuning={"tile": tile})
    x = [random_image(20 + b, n) for b in range(batch)]
    xd = torch.stack([torch.from_numpy(v).to(DEV) for v in x])
    got = plan.forward_batched(xd)
    for b in range(batch):
        assert _rel(got[b], grid_forward(x[b].astype(np.float64), ang, n, W=W)) <= TOL, b
        assert torch.equal(got[b], plan.forward(xd[b])), b


def test_wide_kernel_at_a_large_size():
    print("staged 1536 x 361 x 1280, W = 8", flush=True)
    plan = Plan(1536, uniform_angles(361), 1280, W=8)
    x = torch.from_numpy(random_image(19, 1536)).to(DEV)
    want = torch.empty((361, 1280), device=DEV)
    batch = Batch([plan])
    batch.forward([x], [want])
    torch.cuda.synchronize()
    assert torch.equal(plan.forward(x), want)
    ref = grid_forward(x.cpu().numpy().astype(np.float64), uniform_angles(361), 1280, W=8)
    assert _rel(want, ref) <= TOL
