"""The first batched call of a plan allocates its second workspace; a capture that is
under way on another stream, of this thread or of another, is not disturbed by it."""
import threading

import pytest

torch = pytest.importorskip("torch")

from radon_inputs import uniform_angles  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import Plan  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("threaded", [False, True])
@pytest.mark.parametrize("direction", ["forward", "adjoint"])
def test_first_batched_call_beside_a_capture(direction, threaded):
    print(f"stack beside a capture {direction} threaded={threaded}", flush=True)
    n, nv, batch = 64, 20, 4
    plan = Plan(n, uniform_angles(nv), n)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    if direction == "forward":
        x, out = torch.randn((batch, n, n), generator=gen, device=DEV), torch.zeros((batch, nv, n), device=DEV)
        one, many = plan.forward, plan.forward_batched
    else:
        x, out = torch.randn((batch, nv, n), generator=gen, device=DEV), torch.zeros((batch, n, n), device=DEV)
        one, many = plan.adjoint, plan.adjoint_batched
    want = torch.stack([one(x[b]) for b in range(batch)])
    before = plan.info()["device_bytes"]
    z, other = torch.zeros(8, device=DEV), torch.cuda.Stream()
    torch.cuda.synchronize()
    errors = []

    def call():
        try:
            with torch.cuda.device(DEV), torch.cuda.stream(other):
                many(x, out=out)
        except Exception as e:   # noqa: BLE001 (shown below)
            errors.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        z.add_(1)
        if threaded:
            t = threading.Thread(target=call)
            t.start()
            t.join()
        else:
            call()
        z.add_(1)
    assert not errors, errors
    torch.cuda.synchronize()
    assert torch.equal(out, want) and plan.info()["device_bytes"] > before
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, torch.full_like(z, 2.0 * (k + 1)))
        assert torch.equal(many(x), want)
