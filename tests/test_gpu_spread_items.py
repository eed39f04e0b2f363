"""The most visits of a spreading item: a value that the caller sets is kept, the default
is the value that the plan reports, and with either the adjoint agrees with the FP64
gridding oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.grid import grid_adjoint  # noqa: E402
from radon_inputs import random_sinogram, uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Plan  # noqa: E402

DEV = "cuda:0"


# small plans with strips of more than 256 visits; one without (48 rows, 10 views);
# one with too many partial sums, one with too many items for 256
@pytest.mark.parametrize("n,nv,W,default", [(64, 90, 6, 256), (128, 180, 6, 256), (96, 150, 8, 256), (48, 10, 6, 512),
                                            (512, 720, 6, 512), (2048, 180, 6, 512)])
def test_visits_per_item(n, nv, W, default):
    print(f"visits per item n={n} nv={nv} W={W}", flush=True)
    ang = uniform_angles(nv)
    plan = Plan(n, ang, n, W=W)
    assert plan.tuning()["a2_chunk"] == default
    y = random_sinogram(41, nv, n)
    yd = torch.from_numpy(y).to(DEV)
    a = plan.adjoint(yd)
    again = Plan(n, ang, n, W=W, tuning=plan.tuning())           # what the plan reports builds the same plan
    assert again.info()["n_items"] == plan.info()["n_items"] and torch.equal(again.adjoint(yd), a)
    ref = grid_adjoint(y.astype(np.float64), ang, n, W=W) if n <= 128 else None
    items = []
    for chunk in (64, 256, 300, 512):
        p = Plan(n, ang, n, W=W, tuning={"a2_chunk": chunk})
        assert p.tuning()["a2_chunk"] == chunk
        items.append(p.info()["n_items"])
        if ref is not None:     # float32 transforms of these lengths: 1e-5, as for every decomposition
            got = p.adjoint(yd).cpu().numpy().astype(np.float64)
            assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref), chunk
    assert items == sorted(items, reverse=True)
    assert plan.info()["n_items"] == items[1 if default == 256 else 3]
    if default == 256:
        assert items[1] > items[2] > items[3]    # 300 and 512 are kept, not cut to 256
