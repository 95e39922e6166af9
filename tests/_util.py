"""Shared helpers for the tests: seeded inputs, oracle calls, error metrics."""
import numpy as np
import torch

import oracle
from paper_2404_03617_amd import synth

# max |gpu - ref| <= TOL * max |ref|, for fp16 and bf16 I/O alike
TOL = 2e-2
# Diagnostic bound for fp16 I/O, not the gate: the kernels keep the depth-wise
# output and the hidden values in fp16 and accumulate in fp32, which puts
# max|err| / max|ref| near 1e-3; a dropped bias, a wrong scale or a misplaced
# fragment that the loose gate could absorb shows up well above this.
DIAG_F16 = 5e-3


def make_block(seed, N, H, W, C, E, k, dtype="f16", scales="uniform", bias_std=1.0, layer=0):
    x = synth.activations(seed, N, H, W, C, dtype)
    p = synth.block_params(seed, layer, C, E, k, dtype, scales=scales, bias_std=bias_std)
    return x, p


def to_dev(p, dev="cuda"):
    return {k: (None if v is None else v.to(dev)) for k, v in p.items()}


def oracle_block(x, p, act="gelu", images=None):
    xs = x if images is None else x[list(images)]
    return oracle.block_forward(synth.to_f64(xs), synth.params_f64(p), act=act)


def rel_err(gpu, ref):
    g = gpu.detach().to("cpu").to(torch.float64).numpy() if isinstance(gpu, torch.Tensor) else gpu
    err = np.abs(g - ref)
    return float(err.max() / max(np.abs(ref).max(), 1e-30)), float(err.max()), float(np.abs(ref).max())


def assert_close(gpu, ref, tol=TOL, what="", diag=None):
    """The parity gate (and, when `diag` is given, the tighter diagnostic
    bound).  Prints the measured ratio so every run records it."""
    r, e, m = rel_err(gpu, ref)
    print("  %s: max|err|/max|ref| = %.2e (max|ref| %.3g)" % (what, r, m), flush=True)
    assert r <= tol, "%s: max|err|=%.3e max|ref|=%.3e ratio=%.3e > %.1e" % (what, e, m, r, tol)
    if diag is not None:
        assert r <= diag, "%s: diagnostic bound: ratio %.3e > %.1e" % (what, r, diag)
    return r


def log_uniform(seed, tid, n, lo, hi):
    """Per-channel scales spread over several decades (folded batch norms)."""
    return synth.to_f32(np.exp(synth.draw_uniform(seed, tid, (n,), np.log(lo), np.log(hi))))


def block_c(x, p, act="gelu"):
    """cf_block_forward itself: no scratch memory, so no hidden groups (and for
    a handful of pixels at C >= 128 the slice kernel)."""
    import ctypes

    import paper_2404_03617_amd as cf

    N, H, W, C = x.shape
    keep = []
    bp = cf._block_struct(x, p, keep)
    y = torch.empty_like(x)
    cf._check(cf.lib().cf_block_forward(x.data_ptr(), y.data_ptr(), ctypes.byref(bp), N, H, W, C,
                                        p["w1"].shape[0] // C, p["dw_w"].shape[0], cf.DTYPES[x.dtype], cf.ACTS[act],
                                        torch.cuda.current_stream().cuda_stream))
    return y


RESERVED = 256 + 2048 * 128  # bytes at the start of an MBConv workspace that no call touches
_PAD = 4096


def guarded_ws(nbytes):
    """An MBConv workspace of nbytes full of 0xA5, and as much behind it."""
    return torch.full((nbytes + _PAD,), 0xA5, dtype=torch.uint8, device="cuda")[:nbytes]


def untouched(ws):
    """Whether the reserved bytes of a guarded_ws and those behind it are as
    they were."""
    whole = torch.empty(0, dtype=torch.uint8, device="cuda").set_(ws.untyped_storage())
    return bool((whole[:RESERVED] == 0xA5).all()) and bool((whole[ws.numel():] == 0xA5).all())
