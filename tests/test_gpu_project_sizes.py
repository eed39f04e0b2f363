"""l1-ball projection at the edges of its launches: one block and its last
piece, the last block of the one-round launches and the first second round;
values of one digit at every level, and values that differ in their last bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.solver import project_l1 as oracle_project_l1  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import project_l1  # noqa: E402


@pytest.mark.parametrize("n", [8188, 8192, 8196, 256 * 8192 - 4, 256 * 8192, 256 * 8192 + 4])
@pytest.mark.parametrize("kind", ["equal", "close", "spread"])
def test_project_l1_launch_edges(kind, n):
    print(f"projection {kind} n={n}", flush=True)
    rng = np.random.default_rng(n)
    if kind == "equal":
        v = np.full(n, 1.9999999, dtype=np.float32)      # all low bits set, one value
    elif kind == "close":
        v = (np.float32(1.5).view(np.uint32) + rng.integers(0, 3000, n).astype(np.uint32)).view(np.float32).copy()
    else:
        v = (rng.standard_normal(n) * 10.0 ** rng.uniform(-6, 6, n)).astype(np.float32)
    v[-1] = -v[-1]
    a = np.abs(v.astype(np.float64))
    vd = torch.from_numpy(v).to("cuda:0")
    for frac in (0.001, 0.5, 0.999):
        tau = frac * float(a.sum())
        out, lam = project_l1(vd, tau)
        ref = oracle_project_l1(v.astype(np.float64), tau)
        # one float32 rounding of the largest value, as at every other size
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= 2e-7 * a.max()
        assert abs(np.maximum(a - lam, 0).sum() - tau) <= 1e-9 * tau
