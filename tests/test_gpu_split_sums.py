"""Strips whose visits fill several spreading items: their partial sums are
added by the pass that reads the grid next. The adjoint against the FP64
gridding oracle with few to many partial sums per tile, every tile size, alone,
stacked and in an uneven batch; a grid left dirty by a forward changes nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.grid import grid_adjoint  # noqa: E402
from radon_inputs import random_image, random_sinogram, uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Batch, Plan  # noqa: E402

DEV = "cuda:0"


# float32 transforms of these lengths: 1e-5, as for every tuned decomposition
@pytest.mark.parametrize("n,nv,nd,W,tile,chunk", [(64, 300, 64, 6, 8, 64), (64, 300, 64, 6, 16, 512),
                                                  (64, 300, 64, 8, 32, 64), (40, 200, 48, 4, 8, 64),
                                                  (16, 90, 16, 6, 16, 64), (256, 400, 256, 6, 32, 0)])
def test_split_sums_vs_oracle(n, nv, nd, W, tile, chunk):
    print(f"split sums n={n} nv={nv} nd={nd} W={W} tile={tile} chunk={chunk}", flush=True)
    ang = uniform_angles(nv)
    y = random_sinogram(31, nv, nd)
    plan = Plan(n, ang, nd, W=W, tuning={"tile": tile, "a2_chunk": chunk})
    assert plan.info()["n_slots"] > 0
    yd = torch.from_numpy(y).to(DEV)
    a = plan.adjoint(yd)
    ref = grid_adjoint(y.astype(np.float64), ang, n, W=W)
    got = a.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
    plan.forward(torch.from_numpy(random_image(32, n)).to(DEV))
    assert torch.equal(plan.adjoint(yd), a)
    stacked = plan.adjoint_batched(torch.stack([yd, 2 * yd, yd]))
    assert torch.equal(stacked[0], a) and torch.equal(stacked[1], 2 * a) and torch.equal(stacked[2], a)
    batch = Batch([plan, Plan(48, uniform_angles(17), 48)])
    out = [torch.empty_like(a), torch.empty((48, 48), device=DEV)]
    batch.adjoint([yd, torch.zeros((17, 48), device=DEV)], out)
    torch.cuda.synchronize()
    assert torch.equal(out[0], a) and not out[1].any()
