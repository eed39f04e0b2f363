"""A shortage of memory when a batched call asks for the plan's second workspace: that
call takes its slices one by one, with the same results, and the next call that
finds memory takes them together."""
import os

import pytest

torch = pytest.importorskip("torch")

from radon_inputs import uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Plan  # noqa: E402

DEV = "cuda:0"


def _plan_whose_next_allocation_fails(n, ang, nd):
    """The allocations of a plan's building fail one after another until it is built:
    the one meant to fail is then the first made after it."""
    try:
        for k in range(1, 200):
            os.environ["RADON_TEST_FAIL_ALLOC"] = str(k)
            try:
                return Plan(n, ang, nd)
            except Exception:   # noqa: BLE001 (out of memory, as asked)
                continue
    finally:
        os.environ.pop("RADON_TEST_FAIL_ALLOC", None)
    raise AssertionError("no plan was built")


@pytest.mark.parametrize("first", ["forward", "adjoint"])
def test_workspace_is_asked_for_again(first):
    print(f"stack after a failed allocation, {first} first", flush=True)
    n, nv, batch = 64, 20, 5
    plan = _plan_whose_next_allocation_fails(n, uniform_angles(nv), n)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(9)
    x = torch.randn((batch, n, n), generator=gen, device=DEV)
    y = torch.randn((batch, nv, n), generator=gen, device=DEV)
    calls = {"forward": (plan.forward_batched, plan.forward, x), "adjoint": (plan.adjoint_batched, plan.adjoint, y)}
    many, one, arg = calls[first]
    want = torch.stack([one(arg[b]) for b in range(batch)])
    built = plan.info()["device_bytes"]
    assert torch.equal(many(arg), want) and plan.info()["device_bytes"] == built      # no memory: one by one
    assert torch.equal(many(arg), want) and plan.info()["device_bytes"] > built       # asked for again
    grown = plan.info()["device_bytes"]
    for m, o, a in calls.values():
        assert torch.equal(m(a), torch.stack([o(a[b]) for b in range(batch)]))
    assert plan.info()["device_bytes"] == grown
