"""Parity of the fused stride-2 ConvFirst kernel (Fig. f:convfirst-block (c)
in the reading the App. A counts fix: grouped conv C -> C, BlurPool of the
conv output and of the input, both concatenated into the expand, project to
K, no residual) on the GPU with the fp64 oracle.

Gate: max |gpu - oracle| <= 2e-2 * max |oracle| over the whole output (the
sampled images at batch 128); fp16 cases also meet DIAG_F16.  Covers every
supported C (16, 24, 32, 48, 64: 2C of 32, 48, 64, 96, 128 expand channels,
one padded), R an odd multiple of 16, K a multiple of 8 but not of 16, the
smallest image (2 x 2), odd sizes (reflected last row and column), rows of
one, two and several 16-pixel units with a partial last one, all three
activations, both dtypes, null scales and biases, zero project weights (no
residual: y = b2), image independence, determinism and the seven stride-2
ConvFirst rows of the paper's speed-projection tables at batch 128."""
import sys

import pytest
import torch

import oracle
import paper_2404_03617_amd as cf
from paper_2404_03617_amd import synth
from paper_2404_03617_amd.workloads import CONVFIRST_S2_WORKLOADS

from _util import DIAG_F16, assert_close, to_dev

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def make(seed, N, H, W, C, R, K, dtype="f16", scales="uniform", bias_std=0.5):
    x = synth.activations(seed, N, H, W, C, dtype)
    p = synth.convfirst_s2_params(seed, 0, C, R, K, dtype, scales=scales, bias_std=bias_std)
    return x, p


def ref(x, p, act="relu"):
    return oracle.convfirst_s2_forward(synth.to_f64(x), synth.params_f64(p), act)


def run(x, p, act="relu"):
    y = cf.convfirst_s2_forward(x.cuda(), to_dev(p), act=act)
    torch.cuda.synchronize()
    return y


SWEEP = [
    # C, R, K, N, H, W
    (16, 96, 32, 2, 9, 11),     # odd sizes: 5 x 6 outputs
    (24, 144, 48, 2, 8, 8),     # 2C = 48 expand channels (K step half padding), R = 9 tiles of 16
    (32, 192, 48, 1, 6, 70),    # three units per row, the last of three pixels
    (48, 288, 72, 2, 7, 5),     # K % 16 == 8
    (64, 384, 96, 1, 12, 34),   # 2C = 128, two units per row
    (16, 32, 16, 2, 2, 2),      # the smallest image: one output pixel
    (32, 64, 8, 3, 3, 33),      # K = 8, 17 output columns (a unit of one pixel)
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", SWEEP, ids=lambda c: "C%d_R%d_K%d_N%d_%dx%d" % c)
def test_convfirst_s2_matches_oracle(case, dtype):
    C, R, K, N, H, W = case
    say("convfirst_s2", case, dtype)
    x, p = make(281, N, H, W, C, R, K, dtype)
    for act in ("relu", "gelu", "none"):
        y = run(x, p, act)
        assert tuple(y.shape) == (N, (H + 1) // 2, (W + 1) // 2, K)
        assert_close(y, ref(x, p, act), what="convfirst_s2 %s %s %s" % (case, dtype, act),
                     diag=DIAG_F16 if dtype == "f16" else None)


def test_convfirst_s2_null_scales_and_biases():
    x, p = make(282, 2, 10, 9, 32, 64, 32, scales="none", bias_std=None)
    assert all(p[k] is None for k in ("s0", "b0", "s1", "b1", "s2", "b2"))
    assert_close(run(x, p), ref(x, p), what="convfirst_s2 null scale/bias", diag=DIAG_F16)


def test_convfirst_s2_zero_project_weights_give_the_bias():
    x, p = make(283, 2, 8, 8, 16, 32, 24)
    p["w2"] = torch.zeros_like(p["w2"])
    y = run(x, p)
    assert torch.equal(y.cpu(), p["b2"].to(x.dtype).expand(2, 4, 4, 24))


def test_convfirst_s2_images_are_independent_and_deterministic():
    N, H, W, C, R, K = 5, 12, 40, 32, 64, 48
    x, p = make(284, N, H, W, C, R, K)
    xd, pd = x.cuda(), to_dev(p)
    y = cf.convfirst_s2_forward(xd, pd)
    assert torch.equal(y, cf.convfirst_s2_forward(xd, pd))
    x2 = xd.clone()
    x2[2] = synth.activations(285, 1, H, W, C)[0].cuda()
    y2 = cf.convfirst_s2_forward(x2, pd)
    torch.cuda.synchronize()
    assert torch.equal(y[:2], y2[:2]) and torch.equal(y[3:], y2[3:])
    assert not torch.equal(y[2], y2[2])


SAMPLE = [0, 77, 127]


@pytest.mark.parametrize("name", list(CONVFIRST_S2_WORKLOADS))
def test_convfirst_s2_paper_projection_shapes(name):
    """The stride-2 ConvFirst rows of the paper's speed projections at batch
    128 (the benchmark's own inputs); the oracle checks three images spread
    over the batch (the images are independent, pinned above)."""
    w = CONVFIRST_S2_WORKLOADS[name]
    say("convfirst_s2 workload", name)
    x = synth.activations(w["seed"], w["N"], w["H"], w["W"], w["C"], w["dtype"])
    p = synth.convfirst_s2_params(w["seed"], 0, w["C"], w["R"], w["K"], w["dtype"])
    y = run(x, p, w["act"])
    assert torch.isfinite(y.float()).all()
    assert_close(y.cpu()[SAMPLE], ref(x[SAMPLE], p, w["act"]), what=name, diag=DIAG_F16)


@pytest.mark.parametrize("case", [
    # C, R, K, N, H, W: enough tiles for four-row tiles in every plan
    (16, 96, 32, 40, 37, 66),     # staged weights, two workgroups per CU, ragged rows and columns
    (24, 144, 48, 90, 14, 70),    # two-row tiles, two workgroups per CU
    (32, 192, 56, 90, 14, 70),    # four-row tiles with the weights, K % 16 == 8
    (48, 272, 64, 90, 14, 70),    # four-row tiles, weights from L2, R % 32 == 16
    (64, 1024, 128, 100, 9, 70),  # the largest R and K: two-row tiles, weights from L2
    (48, 288, 64, 3, 9, 70),      # few tiles: two rows with the weights
], ids=lambda c: "C%d_R%d_K%d_N%d_%dx%d" % c)
def test_convfirst_s2_every_tile_plan(case):
    C, R, K, N, H, W = case
    say("convfirst_s2 plan", case)
    x, p = make(286, N, H, W, C, R, K)
    y = run(x, p)
    pick = sorted({0, N // 2, N - 1})
    assert_close(y.cpu()[pick], ref(x[pick], p), what="convfirst_s2 plan %s" % (case,), diag=DIAG_F16)


@pytest.mark.parametrize("case", [(16, 48, 32, 2, 12, 40), (48, 272, 64, 90, 14, 70), (48, 288, 64, 2, 14, 70)],
                         ids=lambda c: "C%d_R%d_K%d_N%d_%dx%d" % c)
def test_convfirst_s2_infinite_hidden_values_stay_infinite(case):
    """The last eight hidden channels overflow fp16 at some pixels: with their
    project weights positive the outputs there are +inf, whether the K steps
    past R (R % 32 == 16, or the end of a batch of steps) repeat them or not,
    and the outputs elsewhere are what they are without the overflow."""
    C, R, K, N, H, W = case
    say("convfirst_s2 overflow", case)
    x, p = make(287, N, H, W, C, R, K, scales="none", bias_std=None)
    p["w2"][:, R - 8:] = p["w2"][:, R - 8:].abs().clamp_min(2.0 ** -6)
    p["s1"] = torch.ones(R)
    calm = run(x, p)
    p["s1"][R - 8:] = 3.0e5
    y = run(x, p)
    assert not y.isnan().any()
    hit = y.isinf()
    assert (y[hit] > 0).all() and 0.05 < hit.float().mean() < 1.0
    # pixels none of whose overflowing channels is positive
    p["w2"][:, R - 8:] = 0
    p["s1"][R - 8:] = 1.0
    none = run(x, p)
    zero = (calm == none).all(-1)
    assert not hit[zero].any() and torch.equal(y[zero], calm[zero])
