"""The 2x2 stride-2 conv at the edges of each of its tiles, against the product
in 64 bits."""
import pytest
import torch

import paper_2404_03617_amd as cf
from paper_2404_03617_amd import synth

pytestmark = pytest.mark.gpu


# few pixels: 32 x 64 tiles (one pixel; one past a tile; K of two steps and of
# 24); many: 64 x 128, and 128 x 64 where 128 does not divide the outputs
@pytest.mark.parametrize("N,H,W,Cin,Cout", [(1, 2, 2, 32, 64), (3, 2, 22, 96, 192), (2, 6, 10, 384, 128),
                                            (7, 60, 62, 32, 256), (7, 62, 58, 64, 192), (97, 16, 18, 160, 128)])
@pytest.mark.parametrize("dtype,u", [("f16", 2.0 ** -11), ("bf16", 2.0 ** -8)])
@pytest.mark.parametrize("affine", [True, False])
def test_downsample_tiles(N, H, W, Cin, Cout, dtype, u, affine):
    print(N, H, W, Cin, Cout, dtype, flush=True)
    x = synth.activations(21, N, H, W, Cin, dtype)
    p = synth.down_params(21, 0, Cin, Cout, dtype, scales="uniform")
    if not affine:
        p = {"wd": p["wd"]}
    y = cf.downsample_forward(x.cuda(), {k: v.cuda() for k, v in p.items()}).cpu().double()
    a = x.double().reshape(N, H // 2, 2, W // 2, 2, Cin).permute(0, 1, 3, 2, 4, 5).reshape(-1, 4 * Cin)
    w = p["wd"].double().reshape(Cout, -1)
    s = p["sd"].double() if affine else 1.0
    b = p["bd"].double() if affine else 0.0
    ref = (a @ w.t() * s + b).reshape(y.shape)
    # fp32 sums of 4 Cin exact products, scale and bias, then one rounding
    size = ((a.abs() @ w.abs().t()) * s + abs(b)).reshape(y.shape)
    bound = 1.01 * (u * ref.abs() + (4 * Cin + 2) * 2.0 ** -24 * size) + 2.0 ** -24
    assert ((y - ref).abs() <= bound).all()
