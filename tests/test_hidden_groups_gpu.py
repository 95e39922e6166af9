"""Hidden groups of wide blocks over few pixels: the workspace behind the
ping-pong buffer holds fp32 partials, one per group, and the reduction adds
exactly those that were written.  The workspace is filled with NaN first, so a
partial that no workgroup wrote shows in every output; it is as large as
cf_stage_workspace_bytes says, or has room for a given number of groups, among
them counts that the hidden chunks do not fill (12 chunks over 8 groups make 6
groups of two)."""
import ctypes
import sys

import pytest
import torch

import paper_2404_03617_amd as cf

from _util import DIAG_F16, assert_close, make_block, oracle_block, to_dev

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def chunk(C):
    """Hidden channels that a workgroup of the FFN kernel takes at a time."""
    return 32 if C == 512 else 64


def run(x, p, room, microbatch=None, act="gelu"):
    """One block through the C entry point with `room` bytes of workspace full
    of NaN (a stage of one block needs none).  Returns (y, partials written)."""
    N, H, W, C = x.shape
    E, k = p["w1"].shape[0] // C, p["dw_w"].shape[0]
    keep = []
    bp = cf._block_struct(x, p, keep)
    ws = torch.full((max(room, 256),), 0xFF, dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    a = (x.data_ptr(), y.data_ptr(), ws.data_ptr(), room, ctypes.byref(bp), 1, N, H, W, C, E, k)
    if microbatch is None:
        cf._check(cf.lib().cf_stage_forward(*a, cf.DTYPES[x.dtype], cf.ACTS[act], None))
    else:
        cf._check(cf.lib().cf_stage_forward_microbatch(*a, microbatch, cf.DTYPES[x.dtype], cf.ACTS[act], None))
    torch.cuda.synchronize()
    m = N if microbatch is None else min(N, microbatch)
    one = m * H * W * C * 4
    parts = ws[:room // one * one].view(torch.float32).view(-1, one // 4)
    return y, int((~parts.isnan().any(1)).sum())


CASES = [
    # C, E, k, N, H, W
    (256, 1, 3, 1, 7, 7), (256, 3, 3, 1, 14, 14), (256, 3, 5, 3, 14, 14), (256, 5, 3, 2, 14, 14),
    (256, 7, 7, 4, 14, 14), (512, 3, 3, 2, 7, 5), (512, 4, 3, 1, 7, 7),
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "C%d_E%d_k%d_N%d_%dx%d" % c)
def test_reduction_adds_only_partials_that_were_written(case, dtype):
    C, E, k, N, H, W = case
    x, p = make_block(91, N, H, W, C, E, k, dtype)
    ref = oracle_block(x, p)
    xd, pd = x.cuda(), to_dev(p)
    chunks = E * C // chunk(C)
    one = N * H * W * C * 4
    recommended = cf.lib().cf_stage_workspace_bytes(1, N, H, W, C, cf.DTYPES[x.dtype])
    for room in (recommended,) + tuple(g * one for g in (2, 3, 5, 7, 9, 14, 23)):
        if room < 2 * one:  # nothing recommended: C = 512 in bf16
            continue
        say("hidden groups", case, dtype, "room for", room // one)
        y, written = run(xd, pd, room)
        # chunks dealt in equal parts to at most that many groups, none empty
        tiles = -(-N * H * W // (64 if C == 512 else 32))
        g = min(room // one, chunks // 2 if C == 512 else chunks, (16 << 20) // one,
                torch.cuda.get_device_properties(0).multi_processor_count // tiles)
        per = -(-chunks // g)
        assert written == -(-chunks // per), (written, room // one)
        assert_close(y.cpu(), ref, what="groups %s %s room %d" % (case, dtype, room // one),
                     diag=DIAG_F16 if dtype == "f16" else None)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_microbatch_reduction_adds_only_partials_that_were_written(dtype):
    N, H, W, C, E, k, m = 3, 9, 11, 256, 3, 3, 2  # micro-batches of 2 and 1
    x, p = make_block(92, N, H, W, C, E, k, dtype)
    ref = oracle_block(x, p)
    xd, pd = x.cuda(), to_dev(p)
    for groups in (2, 5, 8):
        say("hidden groups, micro-batches", dtype, groups)
        y, written = run(xd, pd, groups * m * H * W * C * 4, microbatch=m)
        assert written >= 2
        assert_close(y.cpu(), ref, what="micro-batch groups %d %s" % (groups, dtype))


@pytest.mark.parametrize("case", [(256, 4, 3, 1, 7, 7), (256, 4, 7, 1, 8, 8), (256, 2, 5, 4, 4, 4), (512, 4, 3, 1, 7, 7),
                                  (512, 4, 5, 1, 5, 9), (512, 2, 7, 2, 4, 4), (256, 4, 7, 2, 5, 11), (256, 2, 3, 1, 8, 16)],
                         ids=lambda c: "C%d_E%d_k%d_N%d_%dx%d" % c)
def test_fp16_gelu_over_few_pixels_is_that_of_fp32(case):
    """fp16 blocks over up to 128 pixels keep the depth-wise sums and the GELU in
    fp32, with or without hidden groups: what is left is the rounding of D, of
    the hidden values and of y, each within 2^-11 of its value (2^-11 / sqrt 3 on
    average), so the relative error stays below 2^-11.  The packed-fp16 GELU of
    the large batches gives 7.5e-4 to 8.2e-4 here."""
    C, E, k, N, H, W = case
    x, p = make_block(93, N, H, W, C, E, k, "f16", bias_std=0.1)
    ref = torch.from_numpy(oracle_block(x, p))
    say("fp32 GELU", case)
    y = cf.block_forward(x.cuda(), to_dev(p)).cpu().double()
    err = float((y - ref).norm() / ref.norm())
    print("  relative error %.2e" % err, flush=True)
    assert err < 2.0 ** -11


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", [(1, 4, 4, 3), (1, 4, 8, 1), (1, 5, 13, 3), (1, 5, 13, 7), (2, 14, 14, 3),  # none
                                  (1, 2, 2, 3), (1, 3, 11, 3), (1, 8, 8, 1), (1, 4, 4, 5)],
                         ids=lambda c: "N%d_%dx%d_k%d" % c)
def test_four_chunks_are_not_split_where_that_loses(case, dtype):
    """C = 256, E = 1: groups over at most 64 pixels, for k <= 3 not from 5 to 32;
    without, the workspace stays as it was."""
    N, H, W, k = case
    P = N * H * W
    x, p = make_block(97, N, H, W, 256, 1, k, dtype)
    say("E = 1", case, dtype)
    y, written = run(x.cuda(), to_dev(p), 8 * P * 1024)
    assert written == (4 if P <= 64 and (k >= 5 or P <= 4 or P > 32) else 0)
    assert_close(y.cpu(), oracle_block(x, p), what="E = 1 %s %s" % (case, dtype),
                 diag=DIAG_F16 if dtype == "f16" else None)


@pytest.mark.parametrize("N", [2, 24])
def test_stage_too_wide_for_the_two_launch_block_keeps_its_groups(N):
    """C = 512, E = 8 in fp16: the hidden layer is split over four groups
    (N = 2: the small-batch kernel, N = 24: the streaming one) whose partials
    the workspace of the recommended size holds; the run without room for them
    gives the same up to the order of the sums."""
    H, W, C, E, k = 7, 7, 512, 8, 3
    x, p = make_block(96, N, H, W, C, E, k, "f16")
    ref = oracle_block(x, p)
    say("wide groups", N)
    xd, pd = x.cuda(), to_dev(p)
    y, written = run(xd, pd, cf.lib().cf_stage_workspace_bytes(1, N, H, W, C, cf.DTYPES[x.dtype]))
    assert written == 4
    assert_close(y.cpu(), ref, what="E = 8 stage, groups", diag=DIAG_F16)
    y, _ = run(xd, pd, 0)
    assert_close(y.cpu(), ref, what="E = 8 stage, no room", diag=DIAG_F16)
