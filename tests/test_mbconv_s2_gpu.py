"""Parity of the fused stride-2 MBConv + Squeeze & Excitation kernel (Fig.
f:mbconv with stride 2, Sec. 5.4: BlurPool with the Triangle-3 filter after
the grouped conv, squeeze over the down-sampled map, project to K channels,
no residual) on the GPU with the fp64 oracle.

Gate: max |gpu - oracle| <= 2e-2 * max |oracle| over the whole output (the
sampled images at batch 128); fp16 cases also meet the diagnostic bound
DIAG_F16.  Covers one to sixteen hidden groups per image, the smallest image
(2 x 2: one output pixel, every tap reflected), odd sizes (the last output
row and column read a reflected row and column), one output column, K below,
equal to and above C, R from 1 to 64, both I/O dtypes and both launch modes,
null scales and biases, zero project weights (no residual: y = b3), a
workspace for two images at a time, image independence, determinism,
workspace reuse across shapes (stride 1 and 2 sharing one workspace) and
the four 16 x 16 stride-2 rows of the paper's speed-projection tables at
batch 128."""
import sys

import pytest
import torch

import oracle
import paper_2404_03617_amd as cf
from paper_2404_03617_amd import synth
from paper_2404_03617_amd.workloads import MBCONV_S2_WORKLOADS

from _util import DIAG_F16, assert_close, guarded_ws, to_dev, untouched

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def make(seed, N, H, W, C, E, R, K, dtype="f16", scales="uniform", bias_std=0.5):
    x = synth.activations(seed, N, H, W, C, dtype)
    p = synth.mbconv_params(seed, 0, C, E, R, dtype, scales=scales, bias_std=bias_std, K=K)
    return x, p


def ref(x, p):
    return oracle.mbconv_s2_forward(synth.to_f64(x), synth.params_f64(p))


def run(x, p, **kw):
    """The kernel on x (CPU tensor) with its own workspace; returns (y, ws)."""
    N, H, W, C = x.shape
    EC, R, K = p["w1"].shape[0], p["wr"].shape[0], p["w2"].shape[0]
    need = cf.mbconv_s2_workspace_bytes(N, H, W, C, EC // C, R, K, x.dtype)
    assert need > 0
    ws = guarded_ws(need)
    y = cf.mbconv_s2_forward(x.cuda(), to_dev(p), ws=ws, **kw)
    torch.cuda.synchronize()
    return y, ws


SWEEP = [
    # C, E, R, K, N, H, W
    (16, 4, 4, 32, 2, 6, 6),       # one hidden group
    (32, 2, 8, 16, 3, 7, 9),       # odd sizes: 4 x 5 outputs, reflected last row and column
    (48, 4, 12, 64, 2, 16, 16),    # C % 32 == 16; the 8-wave kernel
    (64, 4, 16, 48, 3, 11, 13),    # ragged pixel tile of the full-resolution map
    (64, 2, 16, 16, 2, 2, 2),      # the smallest image: one output pixel
    (80, 4, 1, 32, 2, 3, 16),      # R = 1; two output rows of eight
    (96, 2, 24, 96, 2, 16, 2),     # one output column
    (128, 4, 32, 128, 2, 16, 16),  # the paper's 16 x 16 -> 8 x 8 row, C = K = 128
    (128, 2, 32, 256, 2, 8, 8),    # K = 2C
    (160, 4, 40, 160, 2, 16, 16),
    (256, 4, 64, 256, 2, 5, 7),    # sixteen hidden groups
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", SWEEP, ids=lambda c: "C%d_E%d_R%d_K%d_N%d_%dx%d" % c)
def test_mbconv_s2_matches_oracle(case, dtype):
    C, E, R, K, N, H, W = case
    say("mbconv_s2", case, dtype)
    x, p = make(181, N, H, W, C, E, R, K, dtype)
    y, ws = run(x, p)
    assert tuple(y.shape) == (N, (H + 1) // 2, (W + 1) // 2, K)
    assert untouched(ws)
    assert_close(y, ref(x, p), what="mbconv_s2 %s %s" % (case, dtype), diag=DIAG_F16 if dtype == "f16" else None)
    # the ordinary launch of the same grid gives the same bits
    ye, wse = run(x, p, launch="exclusive")
    assert untouched(wse)
    assert torch.equal(ye, y)


def test_mbconv_s2_null_scales_and_biases():
    x, p = make(182, 2, 9, 9, 64, 4, 16, 32, scales="none", bias_std=None)
    assert all(p[k] is None for k in ("s1", "b1", "s2", "b2", "br", "be", "s3", "b3"))
    y, _ = run(x, p)
    assert_close(y, ref(x, p), what="mbconv_s2 null scale/bias", diag=DIAG_F16)


def test_mbconv_s2_zero_project_weights_give_the_bias():
    """No residual: with W2 = 0 every output pixel is b3 rounded to the I/O
    dtype (the stride-1 block would return x + b3)."""
    x, p = make(183, 3, 8, 8, 64, 4, 16, 48)
    p["w2"] = torch.zeros_like(p["w2"])
    y, _ = run(x, p)
    exp = p["b3"].to(x.dtype).expand(3, 4, 4, 48)
    assert torch.equal(y.cpu(), exp)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_mbconv_s2_small_workspace_matches_bitwise(dtype):
    """A workspace for two images at a time gives the same bits as the default
    call; one byte less is refused."""
    N, H, W, C, E, R, K = 6, 16, 16, 128, 4, 32, 128
    x, p = make(184, N, H, W, C, E, R, K, dtype)
    y, _ = run(x, p)
    pd = to_dev(p)
    full = cf.mbconv_s2_workspace_bytes(N, H, W, C, E, R, K, x.dtype)
    # reserved bytes, squeeze shares, the down-sampled conv output of two images
    G = E * C // 64
    one_slot = 256 + 2048 * 128 + ((N * G * R * 4 + 255) // 256) * 256 + 2 * 8 * 8 * E * C * 2
    assert one_slot <= full
    ws = guarded_ws(one_slot)
    y1 = cf.mbconv_s2_forward(x.cuda(), pd, ws=ws)
    torch.cuda.synchronize()
    assert untouched(ws)
    assert torch.equal(y1, y)
    small = torch.zeros(one_slot - 1, dtype=torch.uint8, device="cuda")
    with pytest.raises(cf.CFError) as ei:
        cf.mbconv_s2_forward(x.cuda(), pd, ws=small)
    assert ei.value.status == cf.CF_ERR_WORKSPACE


def test_mbconv_s2_images_are_independent_and_deterministic():
    N, H, W, C, E, R, K = 9, 8, 8, 128, 4, 32, 128
    x, p = make(185, N, H, W, C, E, R, K)
    xd, pd = x.cuda(), to_dev(p)
    y = cf.mbconv_s2_forward(xd, pd)
    assert torch.equal(y, cf.mbconv_s2_forward(xd, pd))
    x2 = xd.clone()
    x2[4] = synth.activations(186, 1, H, W, C)[0].cuda()
    y2 = cf.mbconv_s2_forward(x2, pd)
    torch.cuda.synchronize()
    assert torch.equal(y[:4], y2[:4]) and torch.equal(y[5:], y2[5:])
    assert not torch.equal(y[4], y2[4])


SAMPLE = [0, 37, 90, 127]


@pytest.mark.parametrize("name", list(MBCONV_S2_WORKLOADS))
def test_mbconv_s2_paper_projection_shapes(name):
    """The four 16 x 16 stride-2 rows of the paper's speed projections at
    batch 128 (the benchmark's own inputs); the oracle checks four images
    spread over the batch (the images are independent, pinned above)."""
    w = MBCONV_S2_WORKLOADS[name]
    say("mbconv_s2 workload", name)
    x = synth.activations(w["seed"], w["N"], w["H"], w["W"], w["C"], w["dtype"])
    p = synth.mbconv_params(w["seed"], 0, w["C"], w["E"], w["R"], w["dtype"], K=w["K"])
    y, ws = run(x, p)
    assert untouched(ws)
    assert torch.isfinite(y.float()).all()
    assert_close(y.cpu()[SAMPLE], ref(x[SAMPLE], p), what=name, diag=DIAG_F16)


def test_mbconv_s2_workspace_shared_with_stride_one_calls():
    """One workspace serves a sequence of stride-1 and stride-2 calls of
    different shapes and batch sizes (none touches its reserved bytes): each
    output equals, bit for bit, the output with a fresh workspace."""
    calls = [(2, 128, 4, 32, 128, 6, 16, 16), (1, 128, 4, 32, 128, 6, 16, 16), (2, 64, 2, 16, 16, 20, 4, 4),
             (2, 256, 4, 64, 256, 3, 5, 7), (1, 64, 2, 16, 64, 20, 4, 4), (2, 128, 4, 32, 128, 6, 16, 16)]
    need = 0
    for s, C, E, R, K, N, H, W in calls:
        need = max(need, cf.mbconv_s2_workspace_bytes(N, H, W, C, E, R, K) if s == 2 else
                   cf.mbconv_workspace_bytes(N, H, W, C, E, R))
    ws = guarded_ws(need)
    for i, (s, C, E, R, K, N, H, W) in enumerate(calls):
        say("shared workspace call", i, (s, C, E, R, K, N, H, W))
        x, p = make(190 + i, N, H, W, C, E, R, K)
        xd, pd = x.cuda(), to_dev(p)
        fwd = cf.mbconv_s2_forward if s == 2 else cf.mbconv_forward
        for _ in range(2):
            y = fwd(xd, pd, ws=ws)
            torch.cuda.synchronize()
            assert untouched(ws)
            assert torch.equal(y, fwd(xd, pd))
