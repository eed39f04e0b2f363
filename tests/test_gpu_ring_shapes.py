"""Ring filter over the splits of its sums: few and many views (one and several
chunks of views, short last chunks), detector counts from 8 to 4096, buffers
that are not 16-byte aligned, and in place."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.solver import ring_filter  # noqa: E402
from radon_inputs import random_sinogram, uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Plan  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("nv,N", [(1, 8), (3, 12), (127, 20), (128, 320), (129, 32), (700, 96), (1025, 128), (1300, 40),
                                  (5, 4096)])
def test_ring_filter_shapes(nv, N):
    print(f"ring filter views={nv} n_det={N}", flush=True)
    y = random_sinogram(nv + N, nv, N) + np.random.default_rng(N).normal(0, 0.5, N).astype(np.float32)[None, :]
    ref = ring_filter(y.astype(np.float64))
    # float64 sums, one rounding of the result to float32 (2^-24 of a value of at most |y| + |ring|)
    bound = 2.0 ** -24 * (np.abs(y).max() * 3) + 1e-30
    plan = Plan(8, uniform_angles(nv), N)
    yd = torch.from_numpy(y).to(DEV)
    out = plan.ring_filter(yd)
    assert np.abs(out.cpu().numpy() - ref).max() <= bound
    assert torch.equal(plan.ring_filter_noalloc(yd), out)
    for shift in (1, 2):                                     # 4 and 8 bytes past a 16-byte boundary
        raw = torch.empty(nv * N + shift, device=DEV)
        ys = raw[shift:].view(nv, N)
        ys.copy_(yd)
        assert torch.equal(plan.ring_filter(ys), out)
        plan.ring_filter(ys, out=ys)                         # in place
        assert torch.equal(ys, out)
    plan.close()
