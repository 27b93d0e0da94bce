"""Timed cases of the measure -> route -> execute path.

Every case is a dict of plain values.  `prepare` makes what a program holds
before the call (inputs, weights, packed weights, buffers, an Engine, a
captured graph), `run` is one pass through the public calls, `work` the bytes
and operations the pass cannot do without, `exact` the same outputs in
float64 by plain torch.  Sizes are those of the layer tables (ResNet-50,
MobileNetV2, the FFN blocks), of the FC sweep and of the tests, and generic
ones around them.

Kinds:
  fc        one FC operator, sparoa_fc_measured
  fc_batch  a list of FC operators, sparoa_fc_ops_run
  conv      one conv layer whose input nobody measured: sparoa_measure_sparsity
            and sparoa_conv2d_routed
  stack     layers through driver.Engine.forward_routed, called layer by layer
            or replayed from a HIP graph (`graph`): FFN blocks, a ResNet
            bottleneck, a MobileNetV2 inverted residual, an image stem with
            its max pool, or a whole network

Gaussian inputs stand for normalised images and linear (un-activated) layers,
ReLU'd ones for post-activation tensors; FC sweep inputs carry zeros i.i.d. or
in 16 x 16 blocks, and a padded batch holds zeros in its unused samples.
"""
import torch

from paper_2511_19457_amd import abi, stacks
from paper_2511_19457_amd.driver import Engine

_DT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_SPARSITY_THR = 0.5
_RIDGE = {"bf16": 315.0, "f16": 315.0, "f32": 20.0}   # FLOP/byte
_FC_SPARSITY_THR = 0.81    # the FC sweep's calibrated thresholds are 0.80 .. 0.83


# ------------------------------------------------------------------- cases

def listed():
    return [
        # one projection of one token: the smallest call, all latency
        dict(name="fc_token", kind="fc", m=1, k=1024, n=1024, dtype="bf16", rho=0.5, pattern="iid"),
        # the FC sweep: 24 operators, one weight matrix each, m = 1, 8, 64,
        # i.i.d. and block zeros at 0, .5, .8, .95
        dict(name="fc_sweep", kind="fc_batch", ops=24, ms="1,8,64", k=4096, n=4096, dtype="bf16"),
        # two transformer FFN blocks over 2048 tokens
        dict(name="ffn_2048", kind="stack", net="ffn", tokens=2048, hidden=768, inner=3072,
             blocks=2, dtype="f16", graph=False),
        # ResNet-50 stage 1 identity bottleneck, batch 32: large images, few channels
        dict(name="bottleneck_56", kind="stack", net="bottleneck", n=32, h=56, w=56, cin=256,
             width=64, stride=1, dtype="bf16", graph=False),
        # ResNet-50 stage 3 identity bottleneck, batch 32: small images, many channels
        dict(name="bottleneck_14", kind="stack", net="bottleneck", n=32, h=14, w=14, cin=1024,
             width=256, stride=1, dtype="bf16", graph=True),
        # a downsampling bottleneck with its projection, odd batch and image, fp16
        dict(name="bottleneck_odd", kind="stack", net="bottleneck", n=5, h=45, w=39, cin=256,
             width=128, stride=2, dtype="f16", graph=True),
        # MobileNetV2 inverted residual (expand, depthwise, project), batch 32
        dict(name="inverted_56", kind="stack", net="inverted", n=32, h=56, w=56, cin=24, cout=24,
             expand=6, stride=1, dtype="f16", graph=True),
        # ResNet-50's image stem and max pool, batch 32
        dict(name="stem_224", kind="stack", net="stem", n=32, h=224, w=224, cout=64, ksize=7,
             pool=True, dtype="bf16", graph=False),
        # the single fp32 conv of the tests: measure, route, execute
        dict(name="conv_f32", kind="conv", n=1, h=56, w=56, cin=64, cout=64, ksize=3, stride=1,
             dtype="f32", filled=1),
        # a wide 3x3 conv over large images: the largest call, compute bound
        dict(name="conv_wide", kind="conv", n=32, h=56, w=56, cin=256, cout=256, ksize=3, stride=1,
             dtype="bf16", filled=32),
        # a batch padded to 32 with 8 samples in use: the zero-skip path
        dict(name="conv_padded", kind="conv", n=32, h=28, w=28, cin=128, cout=128, ksize=3,
             stride=1, dtype="bf16", filled=8),
        # a whole network on one image, replayed from a graph: latency
        dict(name="resnet50_b1", kind="stack", net="resnet50", n=1, dtype="bf16", graph=True),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    dt = rng.choice(("bf16", "f16"))
    kind = rng.choice(("fc", "fc", "fc_batch", "ffn", "bottleneck", "bottleneck", "inverted",
                       "inverted", "stem", "conv", "conv", "conv", "network"))
    if kind == "fc":
        return dict(kind="fc", m=_log(rng, 1, 512), k=8 * _log(rng, 32, 1024),
                    n=_log(rng, 64, 8192), dtype=dt, rho=rng.choice((0.0, 0.5, 0.8, 0.95)),
                    pattern=rng.choice(("iid", "block")))
    if kind == "fc_batch":
        return dict(kind="fc_batch", ops=rng.randint(3, 24),
                    ms=",".join(str(_log(rng, 1, 64)) for _ in range(3)),
                    k=8 * _log(rng, 64, 512), n=_log(rng, 512, 4096), dtype=dt)
    if kind == "ffn":
        hidden = 8 * rng.randint(32, 128)
        return dict(kind="stack", net="ffn", tokens=_log(rng, 64, 4096), hidden=hidden,
                    inner=4 * hidden, blocks=rng.randint(1, 2), dtype=dt,
                    graph=rng.random() < 0.5)
    if kind == "bottleneck":
        width = rng.choice((64, 128, 256, 512, 8 * rng.randint(6, 64)))
        h = _log(rng, 7, 60)
        w = max(7, min(60, h + rng.randint(-6, 6)))
        cap = max(1, min(32, int(1.8e9 / (h * w * width * width)),
                         32 * 56 * 56 * 64 // (h * w * width)))
        return dict(kind="stack", net="bottleneck", n=_log(rng, 1, cap), h=h, w=w,
                    cin=rng.choice((2, 4)) * width, width=width, stride=rng.choice((1, 2)),
                    dtype=dt, graph=rng.random() < 0.5)
    if kind == "inverted":
        h = _log(rng, 7, 112)
        w = max(7, min(112, h + rng.randint(-9, 9)))
        cin = 8 * rng.randint(2, 20)
        cap = max(1, min(32, 32 * 112 * 112 * 24 // (h * w * cin)))
        return dict(kind="stack", net="inverted", n=_log(rng, 1, cap), h=h, w=w, cin=cin,
                    cout=rng.choice((cin, 8 * rng.randint(2, 40))), expand=rng.choice((1, 6)),
                    stride=rng.choice((1, 2)), dtype=dt, graph=rng.random() < 0.5)
    if kind == "stem":
        h = rng.randint(90, 256)
        return dict(kind="stack", net="stem", n=_log(rng, 1, 32), h=h,
                    w=max(90, min(256, h + rng.randint(-20, 20))), cout=rng.choice((32, 64)),
                    ksize=rng.choice((3, 7)), pool=rng.random() < 0.5, dtype=dt,
                    graph=rng.random() < 0.5)
    if kind == "conv":
        dt = rng.choice(("bf16", "f16", "f32"))
        h = _log(rng, 7, 60)
        w = max(7, min(60, h + rng.randint(-6, 6)))
        cin, cout = _log(rng, 12, 512), _log(rng, 12, 512)
        if rng.random() < 0.7:
            cin, cout = 8 * -(-cin // 8), 8 * -(-cout // 8)
        k = rng.choice((1, 3, 3))
        most = 6e9 if dt == "f32" or cin % 8 else 5e10
        cap = max(1, min(32, int(most / (2.0 * h * w * cin * cout * k * k))))
        n = _log(rng, 1, cap)
        return dict(kind="conv", n=n, h=h, w=w, cin=cin, cout=cout, ksize=k,
                    stride=rng.choice((1, 1, 2)), dtype=dt,
                    filled=n if rng.random() < 0.6 else rng.randint(1, n))
    net = rng.choice(("resnet50", "mobilenet_v2"))
    return dict(kind="stack", net=net, n=_log(rng, 1, 4 if net == "resnet50" else 12),
                dtype="bf16" if net == "resnet50" else "f16", graph=True)


# ------------------------------------------------------------------ inputs

def _gen(seed, i=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + i) % (1 << 62))
    return g


def _normal(shape, dtype, gen, std=1.0):
    return torch.empty(shape, device="cuda").normal_(0.0, std, generator=gen).to(dtype)


def _relu_normal(shape, dtype, gen):
    return torch.empty(shape, device="cuda").normal_(0.0, 1.0, generator=gen).relu_().to(dtype)


def _sparse(m, k, rho, pattern, dtype, gen):
    """|N(0, 1)| with zeros i.i.d. at rate rho, or as 16 x 16 blocks."""
    v = torch.empty(m, k, device="cuda").normal_(0.0, 1.0, generator=gen).abs_().add_(1e-3)
    if pattern == "block":
        z = torch.rand(-(-m // 16), -(-k // 16), device="cuda", generator=gen) < rho
        z = z.repeat_interleave(16, 0)[:m].repeat_interleave(16, 1)[:, :k]
    else:
        z = torch.rand(m, k, device="cuda", generator=gen) < rho
    return v.masked_fill_(z, 0.0).to(dtype)


def _batch_ops(case):
    """(m, rho, pattern) of each operator of an FC batch."""
    ms = [int(v) for v in case["ms"].split(",")]
    mix = [(m, rho, pat) for m in ms for pat in ("iid", "block") for rho in (0.0, 0.5, 0.8, 0.95)]
    return [mix[i * len(mix) // case["ops"]] for i in range(case["ops"])]


def _fc_inputs(m, k, n, rho, pattern, dtype, gen):
    x = _sparse(m, k, rho, pattern, dtype, gen)
    return x, _normal((n, k), dtype, gen, k ** -0.5)


def _layers(case):
    net = case["net"]
    if net == "resnet50":
        return stacks.resnet50(case["n"])
    if net == "mobilenet_v2":
        return stacks.mobilenet_v2(case["n"])
    if net == "ffn":
        return stacks.ffn(case["tokens"], case["hidden"], case["inner"], case["blocks"])
    n, h, w, s = case["n"], case["h"], case["w"], case.get("stride", 2)
    ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
    relu, relu6, none = stacks.ACT_RELU, stacks.ACT_RELU6, stacks.ACT_NONE
    conv = stacks.conv
    if net == "bottleneck":
        cin, width = case["cin"], case["width"]
        out = [conv("c1", 0, n, cin, h, w, width, 1, 1, 0, relu),
               conv("c2", 1, n, width, h, w, width, 3, s, 1, relu)]
        short = 0
        if s != 1 or cin != 4 * width:
            out.append(conv("proj", 0, n, cin, h, w, 4 * width, 1, s, 0, none))
            short = 3
        out.append(conv("c3", 2, n, width, ho, wo, 4 * width, 1, 1, 0, relu, res=short))
        return out
    if net == "inverted":
        cin, cout, hid = case["cin"], case["cout"], case["cin"] * case["expand"]
        out = []
        if case["expand"] != 1:
            out.append(conv("expand", 0, n, cin, h, w, hid, 1, 1, 0, relu6))
        out.append(conv("dw", len(out), n, hid, h, w, hid, 3, s, 1, relu6, groups=hid))
        out.append(conv("project", len(out), n, hid, ho, wo, cout, 1, 1, 0, none,
                        res=0 if s == 1 and cin == cout else None))
        return out
    if net == "stem":
        k, c = case["ksize"], case["cout"]
        out = [conv("stem", 0, n, 3, h, w, c, k, 2, k // 2, relu)]
        if case["pool"]:
            _, ho, wo, _ = stacks.output_shape(out[0])
            out.append(stacks.Layer("maxpool", "maxpool", 1,
                                    dict(n=n, c=c, h=ho, w=wo, k=3, s=2, p=1)))
        return out
    raise ValueError(net)


def _weight_shape(layer):
    s = layer.shape
    if layer.kind == "fc":
        return (s["n"], s["k"]), s["k"]
    if layer.kind == "maxpool":
        return None, 0
    cg = s["cin"] // s["groups"]
    return (s["cout"], s["kh"], s["kw"], cg), s["kh"] * s["kw"] * cg


def _stack_inputs(case, seed):
    layers, dtype = _layers(case), _DT[case["dtype"]]
    # images, FFN residual streams and linear bottlenecks are signed; a
    # ResNet bottleneck reads a ReLU'd tensor
    make = _relu_normal if case["net"] == "bottleneck" else _normal
    x = make(stacks.input_shape(layers), dtype, _gen(seed))
    ws = []
    for i, layer in enumerate(layers):
        shape, fan_in = _weight_shape(layer)
        ws.append(None if shape is None
                  else _normal(shape, dtype, _gen(seed, i + 1), (2.0 / fan_in) ** 0.5))
    return layers, x, ws


def _conv_inputs(case, seed):
    dtype = _DT[case["dtype"]]
    x = _relu_normal((case["n"], case["h"], case["w"], case["cin"]), dtype, _gen(seed))
    x[case["filled"]:] = 0
    k = case["ksize"]
    w = _normal((case["cout"], k, k, case["cin"]), dtype, _gen(seed, 1),
                (2.0 / (k * k * case["cin"])) ** 0.5)
    return x, w, _normal((case["cout"],), dtype, _gen(seed, 2), 0.1)


# ----------------------------------------------------------------- prepare

class _Fc:
    """Buffers of one FC operator."""

    def __init__(self, m, k, n, rho, pattern, dtype, gen, act):
        self.x, self.w = _fc_inputs(m, k, n, rho, pattern, dtype, gen)
        self.bias = _normal((n,), dtype, gen, 0.1)
        self.desc = abi.fc_desc(m, k, n, dtype, has_bias=1)
        self.act = act
        light = abi.sparoa_op_intensity_fc(self.desc)["intensity"] < 315.0
        family = abi.PATH_DENSE_BW if light else abi.PATH_DENSE_MFMA
        self.wp = None
        if abi.sparoa_fc_uses_packed(self.desc, family):
            self.wp = torch.empty(abi.sparoa_fc_packed_bytes(self.desc) // 2, dtype=dtype,
                                  device="cuda")
            abi.sparoa_fc_pack_weights(self.desc, self.w, self.wp)
        br, bc = abi.sparoa_fc_skip_block(self.desc, family | 1)
        self.counts = torch.zeros(4, dtype=torch.int64, device="cuda")
        self.mask = torch.zeros(abi.sparoa_mask_words(m, k, br, bc), dtype=torch.int32,
                                device="cuda")
        ws = max(abi.sparoa_fc_workspace_size(self.desc, family | p) for p in (0, 1))
        self.ws = torch.empty(max(16, ws), dtype=torch.uint8, device="cuda")
        self.path = torch.zeros(1, dtype=torch.int32, device="cuda")
        self.y = torch.empty(m, n, dtype=dtype, device="cuda")

    def outputs(self):
        return [self.y, self.counts, self.path]


def prepare(case, seed):
    kind, dtype = case["kind"], _DT[case["dtype"]]
    if kind == "fc":
        return dict(kind=kind, op=_Fc(case["m"], case["k"], case["n"], case["rho"],
                                      case["pattern"], dtype, _gen(seed), abi.ACT_RELU))
    if kind == "fc_batch":
        ops = [_Fc(m, case["k"], case["n"], rho, pat, dtype, _gen(seed, i), abi.ACT_NONE)
               for i, (m, rho, pat) in enumerate(_batch_ops(case))]
        arr = abi.fc_op_array([
            abi.fc_op(o.desc, o.x, o.w, o.wp, o.bias, None, o.act, o.counts, o.mask, o.y, o.ws,
                      o.path) for o in ops])
        return dict(kind=kind, ops=ops, arr=arr)
    if kind == "conv":
        x, w, bias = _conv_inputs(case, seed)
        k = case["ksize"]
        d = abi.conv_desc(case["n"], case["cin"], case["h"], case["w"], case["cout"], k, k,
                          case["stride"], case["stride"], k // 2, k // 2, dtype=dtype, has_bias=1)
        ridge = _RIDGE[case["dtype"]]
        light = abi.sparoa_op_intensity_conv(d)["intensity"] < ridge
        family = abi.PATH_DENSE_BW if light else abi.PATH_DENSE_MFMA
        rows, cols = case["n"] * case["h"] * case["w"], case["cin"]
        br, bc = abi.sparoa_conv2d_skip_block(d, family | 1)
        ws = max(abi.sparoa_conv2d_workspace_size(d, family | p) for p in (0, 1))
        ho, wo = ((case[a] - 1) // case["stride"] + 1 for a in ("h", "w"))
        return dict(
            kind=kind, desc=d, x=x, w=w, bias=bias, rows=rows, cols=cols, br=br, bc=bc,
            ridge=ridge, counts=torch.zeros(4, dtype=torch.int64, device="cuda"),
            mask=torch.zeros(abi.sparoa_mask_words(rows, cols, br, bc), dtype=torch.int32,
                             device="cuda"),
            ws=torch.empty(max(16, ws), dtype=torch.uint8, device="cuda"),
            path=torch.zeros(1, dtype=torch.int32, device="cuda"),
            y=torch.empty(case["n"], ho, wo, case["cout"], dtype=dtype, device="cuda"))
    layers, x, ws = _stack_inputs(case, seed)
    eng = Engine(layers, dtype, "cuda", weights=ws)
    graph = None
    if case["graph"]:
        eng.forward_routed(x)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            eng.forward_routed(x)
    return dict(kind=kind, eng=eng, x=x, graph=graph, whole=len(layers) > 8)


# --------------------------------------------------------------------- run

def run(state):
    kind = state["kind"]
    if kind == "fc":
        o = state["op"]
        abi.sparoa_fc_measured(o.desc, _FC_SPARSITY_THR, 315.0, abi.ROUTE_BLOCK, o.x, o.w, o.wp,
                               o.bias, None, o.act, o.counts, o.mask, o.y, o.ws, o.path)
        return o.outputs() + [o.mask]
    if kind == "fc_batch":
        abi.sparoa_fc_ops_run(state["arr"], _FC_SPARSITY_THR, 315.0)
        return dict(y=[o.y for o in state["ops"]], counts=[o.counts for o in state["ops"]],
                    path=[o.path for o in state["ops"][:12]])
    if kind == "conv":
        s = state
        abi.sparoa_measure_sparsity(s["x"], s["rows"], s["cols"], s["br"], s["bc"], 0, s["counts"],
                                    s["mask"])
        abi.sparoa_conv2d_routed(s["desc"], _SPARSITY_THR, s["ridge"], abi.ROUTE_BLOCK,
                                 s["counts"], s["x"], s["w"], s["bias"], None, abi.ACT_RELU,
                                 s["mask"], s["y"], s["ws"], s["path"])
        return dict(y=s["y"], counts=s["counts"], mask=s["mask"], path=s["path"])
    eng = state["eng"]
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        eng.forward_routed(state["x"])
    # a whole network hands over its last activation, a block every layer's
    return [eng.acts[-1]] if state["whole"] else eng.acts[1:]


# ------------------------------------------------------------ work, limits

def _size(case):
    return _DT[case["dtype"]].itemsize


def _fc_work(m, k, n, rho, pattern, size):
    """Bytes and operations of one FC: an input column that is zero in every
    row needs no weights (at the sparsities that take the skip path)."""
    if pattern == "block":
        live = 1.0 - rho ** (-(-m // 16))
    else:
        live = 1.0 - rho ** m
    if 1.0 - live < _FC_SPARSITY_THR or m > 64:
        live = 1.0
    return size * (m * k + live * k * n + n + m * n), 2.0 * m * n * k * live


def work(case):
    kind, size = case["kind"], _size(case)
    if kind == "fc":
        b, f = _fc_work(case["m"], case["k"], case["n"], case["rho"], case["pattern"], size)
        return {"bytes": b, "flops": f}
    if kind == "fc_batch":
        each = [_fc_work(m, case["k"], case["n"], rho, pat, size)
                for m, rho, pat in _batch_ops(case)]
        return {"bytes": sum(e[0] for e in each), "flops": sum(e[1] for e in each)}
    if kind == "conv":
        n, cin, cout, k = case["n"], case["cin"], case["cout"], case["ksize"]
        ho, wo = ((case[a] - 1) // case["stride"] + 1 for a in ("h", "w"))
        live = case["filled"]
        return {"bytes": size * (n * case["h"] * case["w"] * cin + cout * k * k * cin + cout +
                                 n * ho * wo * cout),
                "flops": 2.0 * live * ho * wo * cout * cin * k * k}
    # a stack: input, weights and every output that `run` hands over, once
    layers = _layers(case)
    numel = lambda shape: int(torch.Size(shape).numel())  # noqa: E731
    total, flops = numel(stacks.input_shape(layers)), 0.0
    for i, layer in enumerate(layers):
        out = numel(stacks.output_shape(layer))
        if len(layers) <= 8 or i == len(layers) - 1:
            total += out
        shape, fan_in = _weight_shape(layer)
        if shape is not None:
            total += numel(shape)
            flops += 2.0 * out * fan_in
    return {"bytes": size * total, "flops": flops}


def tolerance(case):
    """Another order of the fp32 sums moves an output by one step of its
    storage type now and then, and in a stack such a step travels on.  About
    four times the error seen against float64: 1.7e-3 (bf16) and 2.1e-4
    (fp16) for one layer, 3e-3 and 4e-4 for a block, 6.4e-3 for ResNet-50."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] != "stack":
        return {"rel": 7e-3 if case["dtype"] == "bf16" else 1e-3}
    if case["net"] in ("resnet50", "mobilenet_v2"):
        return {"rel": 3e-2}
    return {"rel": 1.2e-2 if case["dtype"] == "bf16" else 2e-3}


# ------------------------------------------------------------------- exact

def _act64(y, act):
    if act == abi.ACT_RELU:
        return y.clamp_(min=0.0)
    return y.clamp_(0.0, 6.0) if act == abi.ACT_RELU6 else y


def _conv64(x, w, stride, pad, groups=1):
    """NHWC conv in float64, one product per kernel tap."""
    n, h, wd, c = x.shape
    cout, kh, kw, cg = w.shape
    ho, wo = (h + 2 * pad - kh) // stride + 1, (wd + 2 * pad - kw) // stride + 1
    xp = torch.zeros(n, h + 2 * pad, wd + 2 * pad, c, dtype=torch.float64, device=x.device)
    xp[:, pad:pad + h, pad:pad + wd] = x
    y = torch.zeros(n * ho * wo, cout, dtype=torch.float64, device=x.device)
    for r in range(kh):
        for s in range(kw):
            t = xp[:, r:r + (ho - 1) * stride + 1:stride, s:s + (wo - 1) * stride + 1:stride]
            t = t.reshape(n * ho * wo, c)
            tap = w[:, r, s].double()
            if groups == 1:
                y.addmm_(t, tap.t())
            else:
                y.addcmul_(t, tap.reshape(1, c))
    return y.view(n, ho, wo, cout)


def _pool64(x, s):
    return torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), s["k"], s["s"],
                                          s["p"]).permute(0, 2, 3, 1).contiguous()


def _fc64(x, w, bias):
    return torch.addmm(bias.double(), x.double(), w.double().t())


def exact(case, seed):
    kind, dtype = case["kind"], _DT[case["dtype"]]
    if kind == "fc":
        gen = _gen(seed)
        x, w = _fc_inputs(case["m"], case["k"], case["n"], case["rho"], case["pattern"], dtype, gen)
        bias = _normal((case["n"],), dtype, gen, 0.1)
        return [_fc64(x, w, bias).clamp_(min=0.0), None, None, None]
    if kind == "fc_batch":
        ys = []
        for i, (m, rho, pat) in enumerate(_batch_ops(case)):
            gen = _gen(seed, i)
            x, w = _fc_inputs(m, case["k"], case["n"], rho, pat, dtype, gen)
            ys.append(_fc64(x, w, _normal((case["n"],), dtype, gen, 0.1)))
        return dict(y=ys, counts=None, path=None)
    if kind == "conv":
        x, w, bias = _conv_inputs(case, seed)
        y = _conv64(x.double(), w, case["stride"], case["ksize"] // 2)
        return dict(y=_act64(y.add_(bias.double()), abi.ACT_RELU), counts=None, mask=None,
                    path=None)
    layers, x, ws = _stack_inputs(case, seed)
    acts = [x.double()]
    for layer, w in zip(layers, ws):
        s, src = layer.shape, acts[layer.src]
        if layer.kind == "maxpool":
            acts.append(_pool64(src, s))
            continue
        if layer.kind == "fc":
            y = src @ w.double().t()
        else:
            y = _conv64(src, w, s["sh"], s["ph"], s["groups"])
        if layer.res is not None:
            y = y.add_(acts[layer.res])
        acts.append(_act64(y, layer.act))
    return [acts[-1]] if len(layers) > 8 else acts[1:]
