"""Performance cases of the library: what a program that runs ConvFirst
networks on one GPU calls, from a single image to a batch of 128.

A case is a dict of plain values.  ``kind`` names the public entry point:

  block          block_forward          depth-wise conv, FFN, residual
  stage          stage_forward          `depth` blocks of one shape
  down           downsample_forward     2x2 stride-2 conv between stages
  stack          stack_forward          a whole network: stages and down-sampling
  stack_graph    capture_stack          the same, replayed as one HIP graph
  gblock         gblock_forward         the paper's block (grouped conv, ReLU)
  stem_gblock    stem_gblock_forward    image stem fused into the first block
  convfirst_s2   convfirst_s2_forward   stride-2 ConvFirst block with BlurPool
  mbconv         mbconv_forward         MBConv with Squeeze & Excitation
  mbconv_s2      mbconv_s2_forward      the stride-2 MBConv block

Activations are N(0, 1), weights N(0, 1/fan_in), biases N(0, 0.1^2) and the
scales of the folded batch norms U(0.5, 1.5).  Outputs and workspaces are
buffers that the program keeps between calls, as the entry points offer.
"""
import math

import torch

import paper_2404_03617_amd as cf
from paper_2404_03617_amd import roofline

DEPTHS, WIDTHS = "2-2-6-2", "64-128-256-512"


def listed():
    return [
        # One small image: what a call costs when there is next to no work.
        dict(name="block_n1_14x14_c64", kind="block", N=1, H=14, W=14, C=64, E=4, k=3, dtype="f16", act="gelu"),
        # The last stage of a network on one image, bf16: every weight is read for 49 pixels.
        dict(name="block_n1_7x7_c512_bf16", kind="block", N=1, H=7, W=7, C=512, E=4, k=3, dtype="bf16", act="gelu"),
        # First and third stage of a network at batch 128 (the two single-block benchmark shapes).
        dict(name="block_n128_56x56_c64", kind="block", N=128, H=56, W=56, C=64, E=4, k=3, dtype="f16", act="gelu"),
        dict(name="block_n128_14x14_c256_k7", kind="block", N=128, H=14, W=14, C=256, E=4, k=7, dtype="f16",
             act="gelu"),
        # bf16 weights and an image whose sizes no tile divides (a detector's feature map).
        dict(name="block_n24_27x35_c128_bf16", kind="block", N=24, H=27, W=35, C=128, E=4, k=3, dtype="bf16",
             act="gelu"),
        # A whole four-stage network: a throughput batch, and a serving batch replayed as a graph.
        dict(name="stack_n128", kind="stack", N=128, H=56, W=56, depths=DEPTHS, widths=WIDTHS, E=4, k=3, dtype="f16",
             act="gelu"),
        dict(name="stack_graph_n4", kind="stack_graph", N=4, H=56, W=56, depths=DEPTHS, widths=WIDTHS, E=4, k=3,
             dtype="f16", act="gelu"),
        # The paper's block where it is most efficient in the paper's kernel table.
        dict(name="gblock_n128_64x64_c64_e6", kind="gblock", N=128, H=64, W=64, C=64, E=6, k=3, dtype="f16",
             act="relu"),
        # The first layers of the paper's network: image in, first block out.
        dict(name="stem_gblock_n128_256x256_c16", kind="stem_gblock", N=128, H=256, W=256, C=16, E=3, k=3,
             dtype="f16", act="relu"),
        # A stage transition of the early stages.
        dict(name="convfirst_s2_n128_64x64_c48", kind="convfirst_s2", N=128, H=64, W=64, C=48, R=288, K=64,
             dtype="f16", act="relu"),
        # The late stages of the paper's networks: MBConv with Squeeze & Excitation, and its stride-2 form.
        dict(name="mbconv_n128_16x16_c192", kind="mbconv", N=128, H=16, W=16, C=192, E=4, R=48, dtype="f16"),
        dict(name="mbconv_s2_n128_16x16_c128", kind="mbconv_s2", N=128, H=16, W=16, C=128, E=4, R=32, K=128,
             dtype="f16"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more call of the same entry points: image sizes around those of the
    network stage that has the channel count, batches from 1 to 128, both I/O
    dtypes, and no more work than the batch-128 blocks listed above."""
    kind = rng.choice(["block"] * 4 + ["stage"] * 2 + ["gblock"] * 3 + ["convfirst_s2"] * 2 + ["mbconv"] * 2 +
                      ["mbconv_s2", "stem_gblock", "down"])
    c = dict(kind=kind, N=_log(rng, 1, 128), dtype=rng.choice(["f16", "f16", "f16", "bf16"]))
    if kind in ("block", "stage"):
        c["C"] = rng.choice([64, 64, 128, 128, 256, 256, 512])
        side = 3584 // c["C"]
        c.update(E=rng.choice([2, 3, 4, 4, 4, 6]), k=3 if c["C"] == 512 else rng.choice([3, 3, 3, 5, 7]),
                 act=rng.choice(["gelu"] * 3 + ["relu"]))
        if kind == "stage":
            c.update(k=3, depth=rng.choice([2, 3, 4, 6]))
        cap = 2.8e10 if c["dtype"] == "f16" and c["C"] < 512 else 1e10
    elif kind == "gblock":
        c["C"] = rng.choice([16, 32, 48, 64, 80, 96, 112])
        side = 128 if c["C"] == 16 else 64 if c["C"] <= 64 else 32
        c.update(E=rng.choice([3, 4, 6, 6]), k=3, act=rng.choice(["relu"] * 3 + ["gelu"]))
        cap = 6e10
    elif kind == "convfirst_s2":
        c["C"] = rng.choice([16, 24, 32, 48, 64])
        side = 128 if c["C"] <= 32 else 64
        c.update(R=6 * c["C"], K=rng.choice([32, 48, 64, 72, 96]), act="relu")
        cap = 3.5e10
    elif kind in ("mbconv", "mbconv_s2"):
        c["C"] = rng.choice([128, 144, 160, 192, 256])
        side = 16
        c.update(E=4, R=c["C"] // 4)
        if kind == "mbconv_s2":
            c["K"] = rng.choice([128, 160, 192, 256])
        cap = 4e10
    elif kind == "stem_gblock":
        c["C"] = rng.choice([16, 32])
        side = 256
        c.update(E=3, k=3, act="relu")
        cap = 4e10
    else:
        c["C"] = rng.choice([64, 128, 256])
        side = 3584 // c["C"]
        c["K"] = 2 * c["C"]
        cap = 2.8e10
    lo = max(7, side // 2)
    hi = side if kind in ("mbconv", "mbconv_s2") else side + side // 4
    c["H"] = rng.choice([side, rng.randint(lo, hi)])
    c["W"] = rng.choice([c["H"], rng.randint(lo, hi)])
    if kind == "down":
        c["H"], c["W"] = c["H"] & ~1, c["W"] & ~1
    while c["N"] > 1 and work(c)["flops"] > cap:
        c["N"] = max(1, int(c["N"] * min(0.95, cap / work(c)["flops"])))
    return c


def _ints(s):
    return tuple(int(v) for v in s.split("-"))


class _Draw:
    """Tensors on the GPU from one seed, in the order they are asked for."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = torch.float16 if dtype == "f16" else torch.bfloat16

    def normal(self, shape, fan_in=1):
        t = torch.randn(shape, generator=self.g, device="cuda")
        return (t * (1.0 / fan_in) ** 0.5).to(self.dtype)

    def scale(self, n):
        return torch.rand(n, generator=self.g, device="cuda") + 0.5

    def bias(self, n):
        return torch.randn(n, generator=self.g, device="cuda") * 0.1

    def block(self, C, E, k):
        EC = E * C
        return {"dw_w": self.normal((k, k, C), k * k), "s0": self.scale(C), "b0": self.bias(C),
                "w1": self.normal((EC, C), C), "s1": self.scale(EC), "b1": self.bias(EC),
                "w2": self.normal((C, EC), EC), "s2": self.scale(C), "b2": self.bias(C)}

    def gblock(self, C, E):
        p = self.block(C, E, 3)
        del p["dw_w"]
        p["gw_w"] = self.normal((3, 3, C, 8), 72)
        return p

    def down(self, Cin, Cout):
        return {"wd": self.normal((Cout, 2, 2, Cin), 4 * Cin), "sd": self.scale(Cout), "bd": self.bias(Cout)}

    def stem(self, C):
        return {"sw": self.normal((C, 3, 3, 3), 27), "ss": self.scale(C), "sb": self.bias(C)}

    def convfirst_s2(self, C, R, K):
        return {"gw_w": self.normal((3, 3, C, 8), 72), "s0": self.scale(C), "b0": self.bias(C),
                "w1": self.normal((R, 2 * C), 2 * C), "s1": self.scale(R), "b1": self.bias(R),
                "w2": self.normal((K, R), R), "s2": self.scale(K), "b2": self.bias(K)}

    def mbconv(self, C, E, R, K):
        EC = E * C
        return {"w1": self.normal((EC, C), C), "s1": self.scale(EC), "b1": self.bias(EC),
                "gw_w": self.normal((3, 3, EC, 8), 72), "s2": self.scale(EC), "b2": self.bias(EC),
                "wr": self.normal((R, EC), EC), "br": self.bias(R), "we": self.normal((EC, R), R),
                "be": self.bias(EC), "w2": self.normal((K, EC), EC), "s3": self.scale(K), "b3": self.bias(K)}

    def stack(self, depths, widths, E, k):
        layers = []
        for s, (d, c) in enumerate(zip(depths, widths)):
            if s:
                layers.append(("down", self.down(widths[s - 1], c)))
            layers += [("block", self.block(c, E, k)) for _ in range(d)]
        return layers


def _inputs(case, seed):
    """(x, parameters): the tensors of one case."""
    d, c = _Draw(seed, case["dtype"]), case
    kind = c["kind"]
    if kind in ("stack", "stack_graph"):
        widths = _ints(c["widths"])
        x = d.normal((c["N"], c["H"], c["W"], widths[0]))
        return x, d.stack(_ints(c["depths"]), widths, c["E"], c["k"])
    x = d.normal((c["N"], c["H"], c["W"], 3 if kind == "stem_gblock" else c["C"]))
    if kind == "block":
        return x, d.block(c["C"], c["E"], c["k"])
    if kind == "stage":
        return x, [d.block(c["C"], c["E"], c["k"]) for _ in range(c["depth"])]
    if kind == "down":
        return x, d.down(c["C"], c["K"])
    if kind == "gblock":
        return x, d.gblock(c["C"], c["E"])
    if kind == "stem_gblock":
        return x, (d.stem(c["C"]), d.gblock(c["C"], c["E"]))
    if kind == "convfirst_s2":
        return x, d.convfirst_s2(c["C"], c["R"], c["K"])
    return x, d.mbconv(c["C"], c["E"], c["R"], c["K"] if kind == "mbconv_s2" else c["C"])


def prepare(case, seed):
    x, p = _inputs(case, seed)
    N, H, W = x.shape[:3]
    kind, new = case["kind"], lambda *s: torch.empty(s, dtype=x.dtype, device=x.device)
    s = dict(kind=kind, x=x, p=p, act=case.get("act"))
    if kind in ("stack", "stack_graph"):
        widths = _ints(case["widths"])
        s["bufs"] = [new(N, H, W, widths[0])]  # one per stage and per down-sampling step
        for i, c in list(enumerate(widths))[1:]:
            s["bufs"] += [new(N, H >> i, W >> i, c) for _ in range(2)]
        if kind == "stack_graph":
            s["graph"] = cf.capture_stack(x, p, s["bufs"], act=s["act"])
    elif kind in ("block", "stage", "gblock", "mbconv"):
        s["y"] = torch.empty_like(x)
    elif kind == "down":
        s["y"] = new(N, H // 2, W // 2, case["K"])
    else:
        s["y"] = new(N, (H + 1) // 2, (W + 1) // 2, case["C"] if kind == "stem_gblock" else case["K"])
    if kind == "stage":
        need = cf.lib().cf_stage_workspace_bytes(case["depth"], N, H, W, case["C"], cf.DTYPES[x.dtype])
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=x.device)
    elif kind == "mbconv":
        need = cf.mbconv_workspace_bytes(N, H, W, case["C"], case["E"], case["R"], x.dtype)
        s["ws"] = torch.zeros(need, dtype=torch.uint8, device=x.device)
    elif kind == "mbconv_s2":
        need = cf.mbconv_s2_workspace_bytes(N, H, W, case["C"], case["E"], case["R"], case["K"], x.dtype)
        s["ws"] = torch.zeros(need, dtype=torch.uint8, device=x.device)
    return s


def run(state):
    s = state
    kind = s["kind"]
    if kind == "block":
        return cf.block_forward(s["x"], s["p"], act=s["act"], out=s["y"])
    if kind == "stage":
        return cf.stage_forward(s["x"], s["p"], act=s["act"], out=s["y"], ws=s["ws"])
    if kind == "down":
        return cf.downsample_forward(s["x"], s["p"], out=s["y"])
    if kind == "stack":
        return cf.stack_forward(s["x"], s["p"], act=s["act"], bufs=s["bufs"])
    if kind == "stack_graph":
        s["graph"].replay()
        return s["bufs"][-1]
    if kind == "gblock":
        return cf.gblock_forward(s["x"], s["p"], act=s["act"], out=s["y"])
    if kind == "stem_gblock":
        return cf.stem_gblock_forward(s["x"], s["p"][0], s["p"][1], act=s["act"], out=s["y"])
    if kind == "convfirst_s2":
        return cf.convfirst_s2_forward(s["x"], s["p"], act=s["act"], out=s["y"])
    if kind == "mbconv":
        return cf.mbconv_forward(s["x"], s["p"], out=s["y"], ws=s["ws"])
    return cf.mbconv_s2_forward(s["x"], s["p"], out=s["y"], ws=s["ws"])


def work(case):
    """Operations by the paper's rule (convolutions and matrix products) and
    every input, weight and output byte once."""
    c, r = case, roofline
    kind, N, H, W = c["kind"], c["N"], c["H"], c["W"]
    if kind in ("stack", "stack_graph"):
        ks = r.stack_kernels(N, H, W, _ints(c["depths"]), _ints(c["widths"]), c["E"], c["k"])
        flops = sum(n for _, n, _ in ks)
        depths, widths = _ints(c["depths"]), _ints(c["widths"])
        weights = sum(d * r.block_weight_bytes(w, c["E"], c["k"]) for d, w in zip(depths, widths))
        weights += sum(r.down_bytes(0, 0, 0, a, b) for a, b in zip(widths, widths[1:]))
        last = len(widths) - 1
        return dict(flops=flops, bytes=weights + 2 * N * (H * W * widths[0] + (H >> last) * (W >> last) * widths[-1]))
    if kind == "block":
        return dict(flops=r.block_flops(N, H, W, c["C"], c["E"], c["k"]),
                    bytes=r.block_bytes_fused(N, H, W, c["C"], c["E"], c["k"]))
    if kind == "stage":
        return dict(flops=c["depth"] * r.block_flops(N, H, W, c["C"], c["E"], c["k"]),
                    bytes=4 * N * H * W * c["C"] + c["depth"] * r.block_weight_bytes(c["C"], c["E"], c["k"]))
    if kind == "down":
        return dict(flops=r.down_flops(N, H, W, c["C"], c["K"]), bytes=r.down_bytes(N, H, W, c["C"], c["K"]))
    if kind == "gblock":
        return dict(flops=r.gblock_flops(N, H, W, c["C"], c["E"]), bytes=r.gblock_bytes_fused(N, H, W, c["C"], c["E"]))
    if kind == "stem_gblock":
        h, w = (H + 1) // 2, (W + 1) // 2
        return dict(flops=r.stem_flops(N, H, W, c["C"]) + r.gblock_flops(N, h, w, c["C"], c["E"]),
                    bytes=r.stem_gblock_bytes_fused(N, H, W, c["C"], c["E"]))
    if kind == "convfirst_s2":
        return dict(flops=r.convfirst_s2_flops(N, H, W, c["C"], c["R"], c["K"]),
                    bytes=r.convfirst_s2_bytes_fused(N, H, W, c["C"], c["R"], c["K"]))
    if kind == "mbconv":
        return dict(flops=r.mbconv_flops(N, H, W, c["C"], c["E"], c["R"]),
                    bytes=r.mbconv_bytes_fused(N, H, W, c["C"], c["E"], c["R"]))
    return dict(flops=r.mbconv_s2_flops(N, H, W, c["C"], c["E"], c["R"], c["K"]),
                bytes=r.mbconv_s2_bytes_fused(N, H, W, c["C"], c["E"], c["R"], c["K"]))


def tolerance(case):
    """About four times the largest distance from exact() seen over the listed
    and 300 drawn cases: the rounding of the activations and hidden values to
    the I/O dtype (and, in fp16, of the GELU polynomial)."""
    rel, most = TOLERANCES[case["kind"].split("_graph")[0]][case["dtype"]]
    return {"rel": rel, "max": most}


TOLERANCES = {
    "block": {"f16": (4e-3, 3e-2), "bf16": (1e-2, 6e-2)},
    "stage": {"f16": (7e-3, 4e-2), "bf16": (2.6e-2, 0.15)},
    "down": {"f16": (8e-4, 2e-3), "bf16": (7e-3, 1.6e-2)},
    "stack": {"f16": (8e-3, 5e-2)},
    "gblock": {"f16": (1.2e-3, 1.2e-2), "bf16": (1e-2, 7e-2)},
    "stem_gblock": {"f16": (1.5e-3, 1.2e-2), "bf16": (1.2e-2, 8e-2)},
    "convfirst_s2": {"f16": (1.6e-3, 1.2e-2), "bf16": (1.2e-2, 9e-2)},
    "mbconv": {"f16": (9e-4, 4e-3), "bf16": (7e-3, 2.6e-2)},
    "mbconv_s2": {"f16": (1.4e-3, 8e-3), "bf16": (1.1e-2, 6e-2)},
}


# ---------------------------------------------------------------- 64-bit reference

def _f64(t):
    if isinstance(t, dict):
        return {k: _f64(v) for k, v in t.items()}
    return t.double()


def _act(u, act):
    return u * 0.5 * (1 + torch.erf(u * 0.5 ** 0.5)) if act == "gelu" else u.clamp_min(0) if act == "relu" else u


def _shift(x, i, j, H, W):
    """x [N, H, W, C] moved so that [n, h, w] holds pixel (h + i, w + j), zero outside."""
    m = max(abs(i), abs(j))
    xp = torch.nn.functional.pad(x, (0, 0, m, m, m, m))
    return xp[:, m + i:m + i + H, m + j:m + j + W]


def _dw(x, w):
    k = w.shape[0]
    y = torch.zeros_like(x)
    for i in range(k):
        for j in range(k):
            y += _shift(x, i - k // 2, j - k // 2, *x.shape[1:3]) * w[i, j]
    return y


def _grouped(x, w):
    """3x3 conv of group width 8: x [N, H, W, C], w [3, 3, C, 8]."""
    N, H, W, C = x.shape
    y = torch.zeros(C // 8, N * H * W, 8, dtype=x.dtype, device=x.device)
    for i in range(3):
        for j in range(3):
            xs = _shift(x, i - 1, j - 1, H, W).reshape(N * H * W, C // 8, 8).transpose(0, 1).contiguous()
            y += torch.bmm(xs, w[i, j].reshape(C // 8, 8, 8).transpose(1, 2).contiguous())
    return y.transpose(0, 1).reshape(N, H, W, C)


def _ffn(d, p, act):
    h = _act(torch.nn.functional.linear(d, p["w1"]) * p["s1"] + p["b1"], act)
    return torch.nn.functional.linear(h, p["w2"]) * p["s2"] + p["b2"]


def _blur(x):
    """Triangle-3 with one reflected pixel, stride 2."""
    xp = torch.nn.functional.pad(x.permute(0, 3, 1, 2), (1, 1, 1, 1), mode="reflect").permute(0, 2, 3, 1)
    H, W = (x.shape[1] + 1) // 2, (x.shape[2] + 1) // 2
    t = (0.25, 0.5, 0.25)
    return sum(t[a] * t[b] * xp[:, a:a + 2 * H - 1:2, b:b + 2 * W - 1:2] for a in range(3) for b in range(3))


def _ref(kind, x, p, act):
    if kind == "block":
        return x + _ffn(_dw(x, p["dw_w"]) * p["s0"] + p["b0"], p, act)
    if kind == "gblock":
        return x + _ffn(_grouped(x, p["gw_w"]) * p["s0"] + p["b0"], p, act)
    if kind == "down":
        N, H, W, C = x.shape
        s = x.reshape(N, H // 2, 2, W // 2, 2, C).permute(0, 1, 3, 2, 4, 5).reshape(N, H // 2, W // 2, 4 * C)
        return torch.nn.functional.linear(s, p["wd"].reshape(p["wd"].shape[0], -1)) * p["sd"] + p["bd"]
    if kind == "stem":
        N, H, W = x.shape[:3]
        h, w = (H + 1) // 2, (W + 1) // 2
        xp = torch.nn.functional.pad(x, (0, 0, 1, 2, 1, 2))
        taps = [xp[:, a:a + 2 * h - 1:2, b:b + 2 * w - 1:2] for a in range(3) for b in range(3)]
        y = torch.nn.functional.linear(torch.cat(taps, -1), p["sw"].reshape(p["sw"].shape[0], 27))
        return (y * p["ss"] + p["sb"]).clamp_min(0)
    if kind == "convfirst_s2":
        d = _grouped(x, p["gw_w"]) * p["s0"] + p["b0"]
        return _ffn(torch.cat([_blur(d), _blur(x)], -1), p, act)
    silu = torch.nn.functional.silu
    u = silu(torch.nn.functional.linear(x, p["w1"]) * p["s1"] + p["b1"])
    v = silu(_grouped(u, p["gw_w"]) * p["s2"] + p["b2"])
    if kind == "mbconv_s2":
        v = _blur(v)
    z = (torch.nn.functional.linear(v.mean((1, 2)), p["wr"]) + p["br"]).clamp_min(0)
    g = torch.sigmoid(torch.nn.functional.linear(z, p["we"]) + p["be"])
    y = torch.nn.functional.linear(v * g[:, None, None], p["w2"]) * p["s3"] + p["b3"]
    return x + y if kind == "mbconv" else y


def exact(case, seed):
    x, p = _inputs(case, seed)
    kind, act = case["kind"], case.get("act")
    if kind in ("stack", "stack_graph"):
        steps = [(k, _f64(q)) for k, q in p]
    elif kind == "stage":
        steps = [("block", _f64(q)) for q in p]
    elif kind == "stem_gblock":
        steps = [("stem", _f64(p[0])), ("gblock", _f64(p[1]))]
    else:
        steps = [(kind, _f64(p))]
    out = []
    for part in x.split(8):  # a few images at a time: the 64-bit hidden layer of a batch is large
        y = _f64(part)
        for k, q in steps:
            y = _ref(k, y, q, act)
        out.append(y)
    return torch.cat(out)
