"""Calls on a stream of the caller's: their scratch memory and new outputs come
from that stream's pool, and the outputs are those of the default stream."""
import sys

import pytest
import torch

import paper_2404_03617_amd as cf
from paper_2404_03617_amd import synth

from _util import make_block, to_dev

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def calls(out):
    """name -> call of the stream, with an output of the caller's or without"""
    x, p = make_block(95, 4, 14, 14, 256, 4, 3)
    x, p, q = x.cuda(), to_dev(p), to_dev(make_block(95, 4, 14, 14, 256, 4, 3, layer=1)[1])
    x5, p5 = make_block(95, 1, 7, 7, 512, 4, 3, "bf16")
    x5, p5 = x5.cuda(), to_dev(p5)
    xm = synth.activations(95, 2, 12, 10, 64).cuda()
    m, m2 = (to_dev(synth.mbconv_params(95, i, 64, 4, 16)) for i in range(2))
    m2 = dict(m2, w2=m2["w2"][:64].contiguous())
    r, g = to_dev(make_block(95, 4, 7, 7, 512, 4, 3)[1]), to_dev(synth.gblock_params(95, 0, 64, 4, 3))
    y, y5, ym = torch.empty_like(x), torch.empty_like(x5), torch.empty_like(xm)
    yh = torch.empty(2, 6, 5, 64, dtype=xm.dtype, device="cuda")
    if not out:
        y = y5 = ym = yh = None
    d = {"wd": torch.randn(512, 2, 2, 256).half().cuda() / 32, "sd": None, "bd": None}
    more = {} if out else {
        "down": lambda s: cf.downsample_forward(x, d, stream=s),
        "stack": lambda s: cf.stack_forward(x, [("block", p), ("down", d), ("block", r)], stream=s),
        "gblock": lambda s: cf.gblock_forward(xm, g, stream=s),
    }
    return {
        **more,
        "block c256": lambda s: cf.block_forward(x, p, out=y, stream=s),
        "block c512": lambda s: cf.block_forward(x5, p5, out=y5, stream=s),
        "stage": lambda s: cf.stage_forward(x, [p, q], out=y, stream=s),
        "microbatch": lambda s: cf.stage_forward_microbatch(x, [p, q], micro_batch=3, out=y, stream=s),
        "unfused": lambda s: cf.block_forward_unfused(x, p, out=y, stream=s),
        "split": lambda s: cf.block_forward_split(x5, p5, groups=4, out=y5, stream=s),
        "mbconv": lambda s: cf.mbconv_forward(xm, m, out=ym, stream=s),
        "mbconv_s2": lambda s: cf.mbconv_s2_forward(xm, m2, out=yh, stream=s),
    }


SCRATCH = ["block c256", "block c512", "stage", "microbatch", "unfused", "split", "mbconv", "mbconv_s2"]


@pytest.mark.parametrize("name,out", [(n, True) for n in SCRATCH] +
                         [(n, False) for n in SCRATCH + ["down", "stack", "gblock"]])
def test_call_on_a_side_stream(name, out, monkeypatch):
    say("side stream", name, out)
    call = calls(out)[name]
    want = call(None).clone()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    empty, at = torch.empty, []
    monkeypatch.setattr(torch, "empty", lambda *a, **k: (at.append(torch.cuda.current_stream()), empty(*a, **k))[1])
    got = call(side)
    monkeypatch.undo()
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(got, want)
    assert at and all(s == side for s in at), at
    assert torch.cuda.current_stream() == torch.cuda.default_stream()


def test_any_object_with_a_stream_handle_will_do():
    class Handle:
        def __init__(self, stream):
            self.cuda_stream = stream.cuda_stream

    side = torch.cuda.Stream()
    x, p = make_block(95, 1, 7, 7, 256, 4, 3)
    x, p = x.cuda(), to_dev(p)
    want = cf.block_forward(x, p).clone()
    torch.cuda.synchronize()
    for call in (cf.block_forward, cf.block_autotune, lambda x, p, stream: cf.stage_forward(x, [p], stream=stream)):
        got = call(x, p, stream=Handle(side))
        torch.cuda.current_stream().wait_stream(side)
        assert (got - want).abs().max() <= 2e-2 * want.abs().max()


@pytest.mark.parametrize("fork", [False, True], ids=["capture_stream", "forked_stream"])
def test_calls_with_a_stream_inside_a_capture(fork):
    """A call whose stream is the one being captured, or one forked from it:
    scratch memory and a new output come from the graph's pool, and every
    replay gives what the eager call gives for the input at that time."""
    x, p = make_block(94, 4, 14, 14, 256, 4, 3)
    xd, pd = x.cuda(), to_dev(p)
    inputs = [xd.clone(), synth.activations(92, 4, 14, 14, 256).cuda()]
    refs = [cf.block_forward(v, pd).clone() for v in inputs]
    own, side = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=own):
        on = side if fork else own
        if fork:
            side.wait_stream(own)
        y = cf.block_forward(xd, pd, stream=on)
        z = cf.stage_forward(xd, [pd, pd], stream=on)
        if fork:
            own.wait_stream(side)
    for i in (0, 1, 1, 0):
        xd.copy_(inputs[i])
        g.replay()
        other = cf.stage_forward(inputs[i], [pd, pd])
        torch.cuda.synchronize()
        assert torch.equal(y, refs[i]) and torch.equal(z, other), "replay of input %d" % i
