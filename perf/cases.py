"""Performance cases: the calls a program that serves sliced models makes, over the sizes it
makes them at.

Each case is one pass through the package's public entry points: the boundary codec
(``mopar_boundary_encode`` / ``mopar_boundary_decode``), one slice of a model
(``SlicedModel.slice_forward``, a slice being what the method deploys on its own) or a whole
sliced forward (``SlicedModel.forward``, codecs at every cut).  The models are the five
workloads of the repository's benchmark and single stages of them, at batch sizes, image
sizes and sequence lengths around theirs, odd ones included.

``exact`` evaluates the same operators on the same inputs and weights with plain torch in
float64, nothing rounded in between.
"""
from __future__ import annotations

import math

import torch

import paper_2404_02445_amd as P

DEV = "cuda"
TDT = {"f32": torch.float32, "bf16": torch.bfloat16}
ESZ = {"f32": 4, "bf16": 2, "i32": 4}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # a whole small float32 model on one image, three slices, AE codecs: latency and launches
        dict(name="tiny_cnn_b1", kind="tiny_cnn", n=1, hw=32),
        # ResNet-50 as the benchmark serves it: a whole sliced forward of 8 images
        dict(name="resnet50_b8", kind="resnet50", n=8, hw=224),
        # the benchmark's image batch through one bottleneck block of ResNet-50's first stage
        dict(name="bottleneck_s1_b8", kind="bottleneck", n=8, hw=56, mid=64, stride=1),
        # the strided block that opens ResNet-50's last stage, a larger batch
        dict(name="bottleneck_s4_down_b24", kind="bottleneck", n=24, hw=14, mid=512, stride=2),
        # VGG-16's third block: three wide 3x3 convs and a pool, 16 images
        dict(name="vgg_block3_b16", kind="conv_block", n=16, hw=56, cin=128, c=256, convs=3),
        # image intake: NCHW float32 to the 7x7 stem conv and its pool, 32 images
        dict(name="stem_b32", kind="stem", n=32, hw=224),
        # VGG-16's last slice: three linear layers over few rows (weights from HBM), k = 8
        dict(name="classifier_b16", kind="classifier", n=16, hw=7, c=512, fc=4096),
        # one BERT-base encoder layer at the benchmark's batch, bf16
        dict(name="encoder_b32_s128", kind="encoder", dt="bf16", n=32, s=128, heads=12),
        # the same layer in float32 on a few ragged sequences
        dict(name="encoder_f32_b4_s77", kind="encoder", dt="f32", n=4, s=77, heads=12),
        # one LSTM layer of the language model: 64 sequences of 128 steps
        dict(name="lstm_b64_t128", kind="lstm", dt="bf16", n=64, t=128, e=1024, h=1024),
        # its vocabulary projection in 8 sub-slices: the largest product
        dict(name="vocab_projection_8192", kind="projection", rows=8192, k=1024, n_out=32000),
        # the hand-off between two slices: a sequence activation encoded and decoded
        dict(name="codec_seq_64x128x1024", kind="codec", dt="bf16", shape_n=64, shape_h=128, shape_w=0, c=1024),
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny_cnn", "resnet50", "bottleneck", "bottleneck", "conv_block", "conv_block", "stem",
                       "classifier", "encoder", "encoder", "lstm", "lstm", "projection", "projection",
                       "codec", "codec"])
    if kind == "tiny_cnn":
        return dict(kind=kind, n=_log(rng, 1, 32), hw=rng.randint(24, 64))
    if kind == "resnet50":
        return dict(kind=kind, n=_log(rng, 1, 16), hw=rng.randint(97, 224))
    if kind == "bottleneck":
        st = rng.randint(0, 3)
        hw = rng.randint((40, 20, 10, 5)[st], (64, 32, 16, 8)[st])
        stride = rng.choice([1, 1, 2])
        return dict(kind=kind, n=_log(rng, 1, 48), hw=hw * (2 if stride == 2 else 1), mid=64 << st, stride=stride)
    if kind == "conv_block":
        st = rng.randint(0, 3)
        return dict(kind=kind, n=_log(rng, 1, 16), hw=rng.randint(56 >> st, 224 >> st),
                    cin=rng.choice([64, 64 << st]), c=64 << st, convs=rng.randint(1, 3))
    if kind == "stem":
        return dict(kind=kind, n=_log(rng, 1, 48), hw=rng.randint(96, 256))
    if kind == "classifier":
        return dict(kind=kind, n=_log(rng, 1, 64), hw=rng.randint(4, 7), c=rng.choice([128, 256, 512]),
                    fc=rng.choice([1024, 2048, 4096]))
    if kind == "encoder":
        dt = rng.choice(["bf16", "bf16", "bf16", "f32"])
        return dict(kind=kind, dt=dt, n=_log(rng, 1, 64 if dt == "bf16" else 16), s=rng.randint(7, 128),
                    heads=rng.choice([4, 8, 12, 12]))
    if kind == "lstm":
        dt = rng.choice(["bf16", "bf16", "bf16", "f32"])
        if dt == "f32":
            return dict(kind=kind, dt=dt, n=_log(rng, 1, 32), t=_log(rng, 4, 48), e=256, h=rng.choice([256, 512]))
        return dict(kind=kind, dt=dt, n=_log(rng, 1, 128), t=_log(rng, 4, 200),
                    e=rng.choice([256, 512, 1024]), h=rng.choice([256, 512, 640, 1024]))
    if kind == "projection":
        return dict(kind=kind, rows=_log(rng, 1, 8192), k=rng.choice([512, 768, 1024]),
                    n_out=rng.randint(4000, 32000))
    if rng.random() < 0.5:
        return dict(kind="codec", dt=rng.choice(["bf16", "bf16", "f32"]), shape_n=_log(rng, 1, 128),
                    shape_h=rng.randint(5, 128), shape_w=0, c=rng.choice([256, 512, 768, 1024]))
    st = rng.randint(0, 3)
    return dict(kind="codec", dt=rng.choice(["bf16", "bf16", "f32"]), shape_n=_log(rng, 1, 32),
                shape_h=rng.randint(28 >> st, 64 >> st), shape_w=rng.randint(28 >> st, 64 >> st), c=256 << st)


# ---------------------------------------------------------------------------
# model descriptions (what SlicedModel takes): shapes first, values drawn by fill()
# ---------------------------------------------------------------------------

class Net:
    def __init__(self, dtype):
        self.dtype, self.tensors, self.ops, self.layers = dtype, [], [], []
        self.weights, self.wspec = {}, []              # wspec: (name, shape, std, mean)
        self.input_tid, self.output_tid, self.slicing = 0, -1, {}

    def tensor(self, shape, dtype=None):
        self.tensors.append(dict(shape=tuple(shape), dtype=dtype or self.dtype))
        return len(self.tensors) - 1

    def node(self, name):
        self.layers.append(name)

    def shape(self, t):
        return self.tensors[t]["shape"]

    def weight(self, shape, std, mean=0.0):
        name = f"w{len(self.wspec)}"
        self.wspec.append((name, tuple(shape), std, mean))
        return name

    def op(self, out, **kw):
        kw.update(layer=len(self.layers) - 1, out=out)
        kw.setdefault("branch", 0)
        kw.setdefault("pos", 1 + sum(o["layer"] == kw["layer"] for o in self.ops))
        kw.setdefault("rd", False)
        self.ops.append(kw)
        self.output_tid = out
        return out

    def conv(self, x, cout, k, stride, pad, act="relu", res=None, rd=False, **kw):
        n, c, h, w = self.shape(x)
        out = self.tensor((n, cout, (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1))
        return self.op(out, kind="conv", inputs=[x] + ([] if res is None else [res]), cout=cout, kh=k, kw=k,
                       stride=stride, pad=pad, act=act, rd=rd, w=self.weight((cout, c, k, k), math.sqrt(2 / (c * k * k))),
                       b=self.weight((cout,), 0.1), **kw)

    def linear(self, x, nout, act="none", res=None, rd=False, std=None):
        s = self.shape(x)
        nin, lead = (s[1] * s[2] * s[3], s[:1]) if len(s) == 4 else (s[-1], s[:-1])
        return self.op(self.tensor(lead + (nout,)), kind="linear", inputs=[x] + ([] if res is None else [res]),
                       nout=nout, nin=nin, act=act, rd=rd,
                       w=self.weight((nout, nin), std or math.sqrt(2 / nin)), b=self.weight((nout,), 0.05))

    def maxpool(self, x, k, stride, pad):
        n, c, h, w = self.shape(x)
        out = self.tensor((n, c, (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1))
        return self.op(out, kind="maxpool", inputs=[x], k=k, stride=stride, pad=pad)

    def avgpool(self, x):
        return self.op(self.tensor(self.shape(x)[:2]), kind="avgpool", inputs=[x])

    def layernorm(self, x):
        f = self.shape(x)[-1]
        return self.op(self.tensor(self.shape(x)), kind="layernorm", inputs=[x], eps=1e-12,
                       g=self.weight((f,), 0.1, 1.0), beta=self.weight((f,), 0.1))

    def attention(self, qkv, heads):
        b, s, f3 = self.shape(qkv)
        return self.op(self.tensor((b, s, f3 // 3)), kind="attention", inputs=[qkv], heads=heads, head_dim=64,
                       scale=0.125)

    def lstm(self, x, h):
        b, t, e = self.shape(x)
        s = 0.9 / math.sqrt(h)
        return self.op(self.tensor((b, t, h)), kind="lstm", inputs=[x], hidden=h, w_ih=self.weight((4 * h, e), s),
                       w_hh=self.weight((4 * h, h), s), b_ih=self.weight((4 * h,), s), b_hh=self.weight((4 * h,), s))

    def fill(self, gen):
        """Draw every weight (in the model dtype's values); float32 arrays as SlicedModel packs them."""
        for name, shape, std, mean in self.wspec:
            w = torch.randn(shape, generator=gen, device=DEV) * std + mean
            self.weights[name] = w.to(TDT[self.dtype]).float().cpu().numpy()
        return self


def _tiny_cnn(c):
    net = Net("f32")
    x = net.tensor((c["n"], 3, c["hw"], c["hw"]), "f32")
    for i, ch in enumerate((16, 16, 32, 32, 64, 64)):
        net.node(f"conv{i + 1}")
        x = net.conv(x, ch, 3, 1, 1, rd=i == 5)
        if i % 2:
            net.node(f"pool{i // 2 + 1}")
            x = net.maxpool(x, 2, 2, 0)
    net.node("fc")
    net.linear(x, 10)
    k = [0] * len(net.layers)
    k[7] = 2
    return net, dict(n_slices=3, allowed_cut=None, elim_tau=0.05, k_override=k)


def _bottleneck(net, x, mid, stride, project):
    a = net.conv(x, mid, 1, 1, 0, branch=1, pos=1)
    b = net.conv(a, mid, 3, stride, 1, rd=True, branch=1, pos=2)
    sc = net.conv(x, 4 * mid, 1, stride, 0, act="none", branch=2, pos=1) if project else x
    return net.conv(b, 4 * mid, 1, 1, 0, res=sc, branch=1, pos=3)


def _resnet50(c):
    net = Net("bf16")
    x = net.tensor((c["n"], 3, c["hw"], c["hw"]), "f32")
    net.node("stem")
    x = net.maxpool(net.conv(x, 64, 7, 2, 3), 3, 2, 1)
    cuts, k = [], [0]
    for s, blocks in enumerate((3, 4, 6, 3)):
        for b in range(blocks):
            net.node(f"s{s + 1}b{b + 1}")
            x = _bottleneck(net, x, 64 << s, 2 if s and b == 0 else 1, b == 0)
            k.append(4)
        cuts.append(len(net.layers) - 1)
    net.node("head")
    net.linear(net.avgpool(x), 1000)
    cuts = cuts[:-1]
    allowed = [int(j in cuts) for j in range(len(net.layers) - 1)]
    return net, dict(n_slices=4, allowed_cut=allowed, elim_tau=0.05, k_override=k + [0])


def _after_stub(dtype, n, c, hw):
    """A net whose first node (an 8-channel 1x1 conv, never run) hands over an n x c x hw x hw image:
    the slice under test is the one after it and takes that activation as its input."""
    net = Net(dtype)
    x = net.tensor((n, 8, hw, hw), "f32")
    net.node("previous")
    x = net.conv(x, c, 1, 1, 0)
    net.node("slice")
    return net, x


def _net(c):
    """The model of a case, and its planner options (None: the last node is the slice, k given)."""
    kind = c["kind"]
    if kind == "tiny_cnn":
        return _tiny_cnn(c)
    if kind == "resnet50":
        return _resnet50(c)
    if kind == "bottleneck":
        wide = 4 * c["mid"]
        net, x = _after_stub("bf16", c["n"], wide // 2 if c["stride"] == 2 else wide, c["hw"])
        _bottleneck(net, x, c["mid"], c["stride"], c["stride"] == 2)
        return net, 4
    if kind == "conv_block":
        net, x = _after_stub("bf16", c["n"], c["cin"], c["hw"])
        for _ in range(c["convs"]):
            x = net.conv(x, c["c"], 3, 1, 1)
        net.maxpool(x, 2, 2, 0)
        return net, 1
    if kind == "stem":
        net = Net("bf16")
        x = net.tensor((c["n"], 3, c["hw"], c["hw"]), "f32")
        net.node("slice")
        net.maxpool(net.conv(x, 64, 7, 2, 3), 3, 2, 1)
        return net, 1
    if kind == "classifier":
        net, x = _after_stub("bf16", c["n"], c["c"], c["hw"])
        x = net.linear(x, c["fc"], "relu", rd=True)
        net.linear(net.linear(x, c["fc"], "relu"), 1000)
        return net, 8
    if kind == "encoder":
        f = 64 * c["heads"]
        net = Net(c["dt"])
        x = net.tensor((c["n"], c["s"], f))
        net.node("slice")
        std = 1.1 / math.sqrt(f)
        a = net.attention(net.linear(x, 3 * f, std=std), c["heads"])
        a = net.layernorm(net.linear(a, f, res=x, std=std))
        h = net.linear(a, 4 * f, "gelu", rd=True, std=std)
        net.layernorm(net.linear(h, f, res=a, rd=True, std=std))
        return net, 4
    if kind == "lstm":
        net = Net(c["dt"])
        x = net.tensor((c["n"], c["t"], c["e"]))
        net.node("slice")
        net.lstm(x, c["h"])
        return net, 1
    if kind == "projection":
        net = Net("bf16")
        x = net.tensor((1, c["rows"], c["k"]))
        net.node("slice")
        net.linear(x, c["n_out"], rd=True, std=1 / math.sqrt(c["k"]))
        return net, 8
    raise ValueError(kind)


def _codec_shape(c):
    if c["shape_w"]:
        return (c["shape_n"], c["c"], c["shape_h"], c["shape_w"])
    return (c["shape_n"], c["shape_h"], c["c"])


def _codec_weights(c, cc, dtype, gen):
    """Encoder and decoder of a boundary with c channels and cc code channels."""
    t = lambda *s, std: (torch.randn(s, generator=gen, device=DEV) * std).to(TDT[dtype])
    return [t(cc, c, std=math.sqrt(1 / c)), t(cc, std=0.1), t(c, cc, std=math.sqrt(1 / cc)), t(c, std=0.1)]


def _input(net, whole, gen):
    """The input of a pass: the model input, or the activation the previous slice handed over
    (channels-last; after a ReLU, so no negative values)."""
    t = net.tensors[net.input_tid]
    if not whole and len(net.layers) == 2:
        n, c, h, w = net.shape(net.ops[0]["out"])
        return torch.randn((n, h, w, c), generator=gen, device=DEV).relu().to(TDT[net.dtype])
    x = torch.randn(t["shape"], generator=gen, device=DEV)
    return x if len(t["shape"]) == 4 else x.to(TDT[net.dtype])


def _out_shape(net):
    s = net.shape(net.output_tid)
    return s if len(s) != 4 else (s[0], s[2], s[3], s[1])


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


# ---------------------------------------------------------------------------
# prepare, run
# ---------------------------------------------------------------------------

def prepare(case, seed):
    gen = _generator(seed)
    if case["kind"] == "codec":
        shape, dt = _codec_shape(case), case["dt"]
        w = _codec_weights(case["c"], case["c"] // 8, dt, gen)
        pos = math.prod(shape) // case["c"]
        x = torch.randn((pos, case["c"]), generator=gen, device=DEV).relu().to(TDT[dt])
        return dict(kind="codec", shape=shape, dt=dt, x=x, w=w, y=torch.empty_like(x),
                    codec=P.make_codec("ae", case["c"], case["c"] // 8, *w),
                    code=torch.empty((pos, case["c"] // 8), dtype=TDT[dt], device=DEV))
    net, opts = _net(case)
    net.fill(gen)
    sm = P.SlicedModel(net, device=DEV)
    whole = isinstance(opts, dict)
    st = dict(kind="whole" if whole else "slice", sm=sm, s=0)
    if whole:
        st["plan"] = plan = P.mopar_plan_slices(sm.profile(), **opts)
        cuts = sm.boundary_tensors(plan)
        st["w"] = [_codec_weights(net.shape(t)[1], net.shape(t)[1] // 8, net.dtype, gen) for t in cuts]
        st["codecs"], st["keep"] = sm.codecs(plan, "raw")
        for i, t in enumerate(cuts):
            st["codecs"][i] = P.make_codec("ae", net.shape(t)[1], net.shape(t)[1] // 8, *st["w"][i])
        st["codes"] = sm.alloc_codes(plan, st["codecs"])
        st["code_vals"] = [b.view(TDT[net.dtype]).reshape(-1, net.shape(t)[1] // 8) for b, t in zip(st["codes"], cuts)]
    elif len(net.layers) == 2:
        st["plan"], st["s"] = P.make_plan(2, [0, 1], [1, opts]), 1
    else:
        st["plan"] = P.make_plan(1, [0], [opts])
    st["ws"] = sm.alloc_workspace(st["plan"])
    st["x"] = _input(net, whole, gen)
    st["out"] = torch.empty(_out_shape(net), dtype=TDT[net.dtype], device=DEV)
    return st


def run(state):
    if state["kind"] == "codec":
        P.mopar_boundary_encode(state["codec"], state["shape"], state["dt"], state["x"], state["code"])
        P.mopar_boundary_decode(state["codec"], state["shape"], state["dt"], state["code"], state["y"])
        return state["code"], state["y"]
    sm = state["sm"]
    if state["kind"] == "whole":
        sm.forward(state["plan"], state["x"], state["out"], state["codecs"], state["codes"], state["ws"])
        return state["out"], *state["code_vals"]          # the logits, and what every cut handed over
    return sm.slice_forward(state["plan"], state["s"], state["x"], state["out"], state["ws"])


# ---------------------------------------------------------------------------
# work, tolerance
# ---------------------------------------------------------------------------

def work(case):
    """Weights, the pass's input and its output once; the multiply-adds of the contractions."""
    if case["kind"] == "codec":
        pos, c, e = math.prod(_codec_shape(case)) // case["c"], case["c"], ESZ[case["dt"]]
        # x read, code written and read, y written, both weight matrices read
        return dict(bytes=e * (2 * pos * c + 2 * pos * c // 8 + 2 * c * c // 8), flops=4 * pos * c * (c // 8))
    net, opts = _net(case)
    e = ESZ[net.dtype]
    skip = 1 if not isinstance(opts, dict) and len(net.layers) == 2 else 0     # the stub node does not run
    first = net.ops[skip]
    nbytes = math.prod(net.shape(first["inputs"][0])) * (e if skip else ESZ[net.tensors[0]["dtype"]])
    nbytes += e * (math.prod(net.shape(net.output_tid)) + sum(math.prod(w[1]) for w in net.wspec[2 * skip:]))
    flops = 0
    for op in net.ops[skip:]:
        out = net.shape(op["out"])
        if op["kind"] == "conv":
            flops += 2 * math.prod(out) * net.shape(op["inputs"][0])[1] * op["kh"] * op["kw"]
        elif op["kind"] == "linear":
            flops += 2 * math.prod(out) * op["nin"]
        elif op["kind"] == "attention":
            flops += 4 * math.prod(out) * out[1]
        elif op["kind"] == "lstm":
            flops += 8 * math.prod(out) * (net.shape(op["inputs"][0])[2] + op["hidden"])
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """About four times the distance measured between these passes and ``exact``: in bf16 1.7e-3
    (one layer) to 3.7e-3 (an encoder layer), at most 1.9e-2 at one value; for a whole ResNet-50,
    whose roundings travel through every later layer and the codecs, 2.7e-3 at the logits and up
    to 7.6e-3 at the last cut's code; in float32 3e-7 to 7e-7 (3e-6 at one value), with room for
    the hardware exponential in the cells and the softmax."""
    if case["kind"] == "tiny_cnn" or case.get("dt") == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    if case["kind"] == "resnet50":
        return {"rel": 3e-2, "max": 0.25}
    return {"rel": 1.2e-2, "max": 8e-2}


# ---------------------------------------------------------------------------
# the same passes in float64
# ---------------------------------------------------------------------------

def _f64(a):
    return torch.as_tensor(a, device=DEV).double()


def _conv64(x, w, b, stride, pad):
    n, c, h, wd = x.shape
    co, _, k, _ = w.shape
    ho, wo = (h + 2 * pad - k) // stride + 1, (wd + 2 * pad - k) // stride + 1
    cols = w.reshape(co, -1)
    y = [cols @ torch.nn.functional.unfold(x[i:i + 1], k, padding=pad, stride=stride)[0] for i in range(n)]
    return torch.stack(y).reshape(n, co, ho, wo) + b.reshape(1, -1, 1, 1)


def _act64(y, act):
    return y.relu() if act == "relu" else torch.nn.functional.gelu(y) if act == "gelu" else y


def _op64(net, op, val):
    W = net.weights
    x = val[op["inputs"][0]]
    res = val[op["inputs"][1]] if len(op["inputs"]) > 1 else 0.0
    kind = op["kind"]
    if kind == "conv":
        return _act64(_conv64(x, _f64(W[op["w"]]), _f64(W[op["b"]]), op["stride"], op["pad"]) + res, op["act"])
    if kind == "linear":
        if x.dim() == 4:
            x = x.reshape(x.shape[0], -1)
        return _act64(x @ _f64(W[op["w"]]).T + _f64(W[op["b"]]) + res, op["act"])
    if kind == "maxpool":
        return torch.nn.functional.max_pool2d(x, op["k"], op["stride"], op["pad"])
    if kind == "avgpool":
        return x.mean((2, 3))
    if kind == "layernorm":
        return torch.nn.functional.layer_norm(x, x.shape[-1:], _f64(W[op["g"]]), _f64(W[op["beta"]]), op["eps"])
    if kind == "attention":
        b, s, f3 = x.shape
        q, k, v = (t.reshape(b, s, op["heads"], 64).transpose(1, 2).contiguous() for t in x.split(f3 // 3, -1))
        p = torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) * op["scale"], -1)
        return torch.matmul(p, v).transpose(1, 2).reshape(b, s, f3 // 3)
    if kind == "lstm":
        b, t, _ = x.shape
        gx = x @ _f64(W[op["w_ih"]]).T + _f64(W[op["b_ih"]]) + _f64(W[op["b_hh"]])
        whh = _f64(W[op["w_hh"]]).T.contiguous()
        h = c = torch.zeros((b, op["hidden"]), dtype=torch.float64, device=DEV)
        hs = []
        for i in range(t):
            gi, gf, gg, go = (gx[:, i] + h @ whh).chunk(4, -1)
            c = torch.sigmoid(gf) * c + torch.sigmoid(gi) * torch.tanh(gg)
            h = torch.sigmoid(go) * torch.tanh(c)
            hs.append(h)
        return torch.stack(hs, 1)
    raise ValueError(kind)


def exact(case, seed):
    gen = _generator(seed)
    if case["kind"] == "codec":
        we, be, wd, bd = (w.double() for w in _codec_weights(case["c"], case["c"] // 8, case["dt"], gen))
        pos = math.prod(_codec_shape(case)) // case["c"]
        x = torch.randn((pos, case["c"]), generator=gen, device=DEV).relu().to(TDT[case["dt"]]).double()
        code = x @ we.T + be
        return code, code @ wd.T + bd
    net, opts = _net(case)
    net.fill(gen)
    whole = isinstance(opts, dict)
    stub = not whole and len(net.layers) == 2
    codecs, codes = {}, []
    if whole:                                          # the plan only says where the codecs sit
        sm = P.SlicedModel(net, device=DEV)
        plan = P.mopar_plan_slices(sm.profile(), **opts)
        for t in sm.boundary_tensors(plan):
            codecs[t] = [w.double() for w in _codec_weights(net.shape(t)[1], net.shape(t)[1] // 8, net.dtype, gen)]
    x = _input(net, whole, gen)
    val = {net.ops[0]["out"]: x.double().permute(0, 3, 1, 2)} if stub else {net.input_tid: x.double()}
    if len(net.tensors[0]["shape"]) == 4 and not stub:
        val[0] = x.to(TDT[net.dtype]).double()         # the first conv reads the image in the model dtype
    for op in net.ops[1 if stub else 0:]:
        y = _op64(net, op, val)
        if op["out"] in codecs:
            we, be, wd, bd = codecs[op["out"]]
            code = y.movedim(1, -1) @ we.T + be
            codes.append(code.reshape(-1, code.shape[-1]))
            y = ((code @ wd.T) + bd).movedim(-1, 1)
        val[op["out"]] = y
    y = val[net.output_tid]
    y = y.permute(0, 2, 3, 1).contiguous() if y.dim() == 4 else y
    return (y, *codes) if whole else y
