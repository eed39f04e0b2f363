"""Warm-start convolutions and network where their pixel tiles, channel blocks
and pixel chunks end: sizes off the 16 x 16, 16 x 8 and 16 x 4 output tiles and
the 8 x 8 tiles of the weight gradient, single tiles, single-pixel levels,
channel counts off the 16-channel chunk, and enough pixels for several chunks."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import torch.nn.functional as Fn  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle.cnn import CHANNELS  # noqa: E402
from paper_1009_1380_amd import WarmStartNet, cnn_conv_test  # noqa: E402
from test_gpu_cnn import DEV, _emulated_network, _random_params, bf16_bits, from_bits, note, rel  # noqa: E402


@pytest.mark.parametrize("B,Cin,Cout,H,W", [(1, 64, 128, 17, 33), (1, 16, 64, 1, 1), (3, 24, 40, 9, 47),
                                            (1, 64, 32, 75, 31), (2, 1, 32, 33, 15), (2, 32, 1, 31, 17),
                                            (1, 64, 64, 136, 128), (8, 32, 32, 5, 3)])
def test_conv_at_tile_edges(B, Cin, Cout, H, W):
    note(f"conv B={B} Cin={Cin} Cout={Cout} H={H} W={W}")
    rng = np.random.default_rng(B * 1000 + Cin + Cout + H)
    x, x16 = bf16_bits(rng.standard_normal((B, Cin, H, W)))
    w, _ = bf16_bits(rng.standard_normal((Cout, Cin, 3, 3)) / np.sqrt(Cin * 9))
    g, g16 = bf16_bits(rng.standard_normal((B, Cout, H, W)))
    xt = torch.as_tensor(x).requires_grad_(True)
    wt = torch.as_tensor(w).requires_grad_(True)
    conv = Fn.conv2d(xt, wt, None, padding=1)
    conv.backward(torch.as_tensor(g))
    out32, _, gin, gw, gb = cnn_conv_test(x16, torch.as_tensor(w, dtype=torch.float32).to(DEV), gout16=g16)
    # float32 sums of exact products: at most a few hundred roundings of 2^-24 add up
    assert rel(out32.cpu().numpy(), conv.detach().numpy()) <= 1e-5
    assert rel(gw.cpu().numpy(), wt.grad.numpy()) <= 1e-5
    assert np.abs(gb.cpu().numpy() - g.sum(axis=(0, 2, 3))).max() <= 1e-5 * np.abs(g).sum(axis=(0, 2, 3)).max()
    assert rel(from_bits(gin), xt.grad.numpy()) <= 4e-3      # one bfloat16 rounding, at most 2^-8 each


@pytest.mark.parametrize("B,H,W", [(1, 8, 8), (2, 72, 40), (1, 24, 136)])
def test_network_at_tile_edges(B, H, W):
    """Against the float32 emulation of the bfloat16 storage points. A sum in
    another order flips an occasional rounding (2^-8 of a value); were every
    value flipped, the rms difference would still be below 2^-8."""
    note(f"network B={B} H={H} W={W}")
    net = WarmStartNet(B, H, W, seed=3)
    p = _random_params(net, scale_last=1.0, seed=H + W)
    net.set_params(p)
    rng = np.random.default_rng(H * W)
    x = rng.standard_normal((B, H, W)).astype(np.float32)
    t = rng.standard_normal((B, H, W)).astype(np.float32)
    y = net.forward(torch.from_numpy(x).to(DEV)).cpu().numpy()
    loss = net.train_step(torch.from_numpy(x).to(DEV), torch.from_numpy(t).to(DEV), 0.0)
    g = net.get_grads()
    ye, le, ge = _emulated_network(p, x, t)
    assert rel(y - x, ye - x) <= 2 ** -8 and abs(loss - le) <= 2 ** -8 * le
    off = 0
    for ci, co in CHANNELS:
        n = co * ci * 9 + co
        assert rel(g[off:off + n], ge[off:off + n]) <= 2 ** -7, (ci, co)
        off += n
