"""Weight gradients whose last round of 64 x 64 channel workgroups is split over
smaller ones: a round of at most a quarter of the CUs (32 x 32 channels), of up to
half of them (32 x 64), a full last round and one above half (not split); ragged
images, the last tiles partly outside."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1009_1380_amd import cnn_conv_test  # noqa: E402

DEV = "cuda:0"


# 128 x 128 channels are four workgroups per chunk of 64 tiles: 64 chunks fill 256 CUs
@pytest.mark.parametrize("chunks", [64, 65, 80, 81, 96, 97])
def test_weight_gradient_last_round(chunks):
    C, H, W = 128, 8 * chunks - 3, 509
    print(f"weight gradient, {chunks} chunks", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chunks)
    x16, g16 = (torch.randn((1, C, H, W), generator=gen, device=DEV).to(torch.bfloat16) for _ in range(2))
    w = torch.zeros((C, C, 3, 3), device=DEV)
    gw = cnn_conv_test(x16.view(torch.int16), w, gout16=g16.view(torch.int16))[3]
    x = torch.zeros((C, H + 2, W + 2), dtype=torch.float64, device=DEV)
    x[:, 1:-1, 1:-1] = x16[0].double()
    g = g16[0].double().reshape(C, H * W)
    for dy in range(3):
        for dx in range(3):
            ref = g @ x[:, dy:dy + H, dx:dx + W].reshape(C, H * W).t().contiguous()
            err = (gw[:, :, dy, dx].double() - ref).norm() / ref.norm()
            # float32 sums of 512 steps per chunk and at most 97 chunks: a few 1e-7
            assert float(err) <= 1e-5, (dy, dx)
