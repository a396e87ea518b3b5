"""The corrector network's tiled kernels where tiles go wrong: a grid of one
tile (its halo is itself), one tile high or wide, several per block; and batches
that split into groups.  Layers against the FP64 oracle on BF16-exact inputs,
held as in the other parity tests to FP32 accumulation, 1e-5 of the max norm; a
batch's gradient against its samples' one by one, the same bound where the loss's
1 / batch is a power of two.  Elsewhere that factor moves the BF16 roundings of
dz (2^-9 each, on both sides): 2^-8.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cnn
from paper_0710_5912_amd import inputs

pytestmark = pytest.mark.gpu

le = pytest.importorskip("paper_0710_5912_amd.le")
torch = pytest.importorskip("torch")

GRIDS = [(16, 16), (16, 128), (128, 16), (256, 256)]


def bf16_bits(x):
    r = cnn.bf16_round(x)
    return (np.asarray(r, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16), r


def dev(a, dtype=torch.float32):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30))


def make(H, W):
    n = le.Net(H, W)
    p = inputs.cnn_init_params(3) + np.random.default_rng(1).uniform(-0.02, 0.02, cnn.nparams())
    n.set_params(p.astype(np.float32), [1.0, 1.0, 1.0, 1.0])
    layers = [(cnn.bf16_round(Wl), b)
              for Wl, b in cnn.unpack(p.astype(np.float32).astype(np.float64))]
    return n, layers


@pytest.mark.parametrize("layer", [0, 1, 3])
@pytest.mark.parametrize("H,W", GRIDS)
def test_layer(H, W, layer):
    print(f"case {H}x{W} layer {layer}", flush=True)
    cin, cout = cnn.LAYERS[layer]
    P = H * W
    n, layers = make(H, W)
    Wl, b = layers[layer]
    rng = np.random.default_rng(60 + layer)
    bits, a = bf16_bits(rng.standard_normal((P, cin)))
    _, dz = bf16_bits(rng.standard_normal((P, cout)))
    zprev = rng.standard_normal((P, cin)).astype(np.float32)
    a_c, dz_c = a.T.reshape(cin, H, W), dz.T.reshape(cout, H, W)
    a_d = dev(bits.view(np.int16), torch.int16)

    z = torch.empty((P, cout), dtype=torch.float32, device="cuda")
    ao = torch.empty((P, cout), dtype=torch.int16, device="cuda")
    n.layer_fwd(layer, a_d, z, ao if layer < 3 else None)
    got = z.cpu().numpy().astype(np.float64).T.reshape(cout, H, W)
    assert rel(got, cnn.conv3x3(a_c, Wl, b)) <= 1e-5

    dw = torch.empty(9 * cin * cout + cout, dtype=torch.float32, device="cuda")
    dzp = torch.empty((P, cin), dtype=torch.float32, device="cuda") if layer else None
    n.layer_bwd(layer, dev(dz), a_d, dev(zprev) if layer else None, dzp, dw)
    dW, db = cnn.conv3x3_dw(dz_c, a_c)
    g = dw.cpu().numpy().astype(np.float64)
    assert rel(g[:dW.size], dW.ravel()) <= 1e-5
    assert rel(g[dW.size:], db) <= 1e-5
    if layer:
        ref = cnn.conv3x3_dx(dz_c, Wl) * cnn.silu_grad(
            zprev.astype(np.float64).T.reshape(cin, H, W))
        assert rel(dzp.cpu().numpy().astype(np.float64).T.reshape(cin, H, W), ref) <= 1e-5
    n.close()


# 2^20 pixels are one group: 1030 samples of 32 x 32 are two, the second short
@pytest.mark.parametrize("H,W,B", [(16, 16, 4), (32, 16, 64), (64, 64, 5), (32, 32, 1030)])
def test_batch_is_the_sum_of_its_samples(H, W, B):
    print(f"case {H}x{W} batch {B}", flush=True)
    n, _ = make(H, W)
    gen = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((B, 2, H, W), device="cuda", generator=gen)
    t = torch.randn((B, 2, H, W), device="cuda", generator=gen)
    loss, g = n.grad(x, t, B, want_grad=True)
    parts = [n.grad(x[k:k + 1].contiguous(), t[k:k + 1].contiguous(), 1, want_grad=True)
             for k in range(B)]
    assert abs(loss - np.mean([p[0] for p in parts])) <= 1e-12 * loss
    assert rel(g, np.mean([p[1].astype(np.float64) for p in parts], axis=0)) <= \
        (1e-5 if B & (B - 1) == 0 else 2.0 ** -8)
    again = n.grad(x, t, B, want_grad=True)
    assert again[0] == loss and np.array_equal(again[1], g)
    n.close()
