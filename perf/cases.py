"""The work that a user of the library has it do, as cases that can be timed and compared.

A case is one pass through the public entry points of paper_2609_28358_amd.mxconv
or through one of its whole training steps (workloads.py).  Its "kind":

  layer   one convolution trained on its own: quantize X and W, forward, quantize
          G_Y, input and weight gradient, full-precision results in the caller's
          layout (mxconv_quantize*, _fwd, _backward or _dgrad + _wgrad; optionally
          the explicit im2col and stochastically rounded gradients)
  nvfp    the same layer on the paper's two-level NVFP operands
  hidden  a hidden layer of a SiLU network on stored codes: quantize W, the forward
          with the quantizing epilogue, the quantized sum of its consumers'
          gradients, the input gradient with the quantizing epilogue, the deferred
          weight gradient and its reduction
  merge   a layer behind a concatenation: the parts joined (one of them upsampled),
          a 1x1 convolution over them, and its backward pass
  stem    an image quantized into a kept buffer, the first convolution and its
          weight gradient
  net     the YOLOv8n-shaped backbone + neck, forward and backward, one HIP graph
  replay  the quantized-latent-replay training step, one HIP graph

"batch" is the number of samples; sizes are those of the repository's benchmark,
network description and tests, and generic odd ones.
"""
import functools
import math

import torch

from paper_2609_28358_amd import mxconv as mx
from paper_2609_28358_amd import synth
from paper_2609_28358_amd import workloads

DEV = "cuda:0"
FMT = {"e4m3": mx.E4M3, "e2m1": mx.E2M1, "e2m3": mx.E2M3, "e3m2": mx.E3M2}
# bits of an element; mantissa bits, smallest exponent, largest value
BITS = {mx.E4M3: 8, mx.E2M1: 4, mx.E2M3: 6, mx.E3M2: 6}
GRID = {mx.E4M3: (3, -6, 448.0, 8), mx.E2M1: (1, 0, 6.0, 2), mx.E2M3: (3, 0, 7.5, 2), mx.E3M2: (2, -2, 28.0, 4)}
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
LAYOUT = {"nchw": mx.NCHW, "nhwc": mx.NHWC, "cbf": mx.CBF}


# ---------------------------------------------------------------- the cases
def _conv(kind, batch, cin, cout, h, w, k, s, **more):
    return dict(kind=kind, batch=batch, cin=cin, cout=cout, h=h, w=w, k=k, s=s, **more)


def listed():
    named = {
        # the smallest call that the package's smoke test makes: latency of a plain layer
        "layer_fp8_n2_32to32_8": _conv("layer", 2, 32, 32, 8, 8, 3, 1, fmt="e4m3", xfmt="e4m3", src="f32",
                                       layout="nchw", sr=False, col=False),
        # the layer sweep's 3x3 layer, with its explicit im2col
        "layer_fp8_n32_64to64_56": _conv("layer", 32, 64, 64, 56, 56, 3, 1, fmt="e4m3", xfmt="e4m3", src="f32",
                                         layout="cbf", sr=False, col=True),
        # odd sizes, channels that fill no block, plain layouts, gradients rounded as the paper rounds them
        "layer_fp4_n96_48to80_35x27": _conv("layer", 96, 48, 80, 35, 27, 3, 1, fmt="e2m1", xfmt="e2m1", src="f32",
                                            layout="nchw", sr=True, col=False),
        # a batch below 32 (batch block 16): a C2f 3x3 of the network at batch 16
        "layer_fp8_n16_32to32_80": _conv("layer", 16, 32, 32, 80, 80, 3, 1, fmt="e4m3", xfmt="e4m3", src="bf16",
                                         layout="nchw", sr=False, col=False),
        # FP4 weights and gradients, FP6 activations (MicroQonv+), a 40x40 stage of the network
        "layer_fp46_n64_128to128_40": _conv("layer", 64, 128, 128, 40, 40, 3, 1, fmt="e2m1", xfmt="e3m2", src="bf16",
                                            layout="cbf", sr=False, col=False),
        # the paper's own NVFP4, the layer sweep's 3x3 layer
        "nvfp4_n32_64to64_56": _conv("nvfp", 32, 64, 64, 56, 56, 3, 1, fmt="e2m1", xfmt="e2m1", src="f32"),
        # a downsampling layer of the network (64 -> 128, 80 -> 40), bf16 tensors between layers
        "hidden_fp4_n64_64to128_80_s2": _conv("hidden", 64, 64, 128, 80, 80, 3, 2, fmt="e2m1", src="bf16", terms=2,
                                              sr=False),
        # a wide layer where the products dominate, MXFP8
        "hidden_fp8_n128_256to256_16": _conv("hidden", 128, 256, 256, 16, 16, 3, 1, fmt="e4m3", src="f32", terms=1,
                                             sr=False),
        # the neck's merge at 40x40: an upsampled 256-channel part and a 128-channel one
        "merge_fp4_n64_256u_128to64_40": _conv("merge", 64, 256, 64, 40, 40, 1, 1, fmt="e2m1", src="bf16", skip=128),
        # the network's first layer, half its batch
        "stem_fp4_n32_3to16_640": _conv("stem", 32, 3, 16, 640, 640, 3, 2, fmt="e2m1", src="bf16"),
        # the quantized-latent-replay step
        "replay_fp4_n128": dict(kind="replay", batch=128, fmt="e2m1", src="bf16"),
        # the headline: the whole training step
        "net_fp4_n64_640": dict(kind="net", batch=64, size=640, fmt="e2m1", src="bf16"),
    }
    return [dict(case, name=name) for name, case in named.items()]


def _log(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "nvfp", "hidden", "hidden", "hidden", "merge", "merge", "stem",
                       "replay", "net"])
    if kind == "net":
        # whole steps train in MXFP4
        return dict(kind="net", batch=rng.choice([32, 64]), size=32 * rng.randint(3, 14), fmt="e2m1",
                    src=rng.choice(["bf16", "f32"]))
    if kind == "replay":
        return dict(kind="replay", batch=32 * rng.randint(2, 5), fmt="e2m1", src=rng.choice(["bf16", "f32"]))
    while True:
        batch = 32 * rng.randint(1, 4)
        h = _log(rng, 7, 160)
        w = h if rng.random() < 0.5 else max(5, int(h * rng.uniform(0.6, 1.4)))
        cin, cout = _log(rng, 16, 384, 8), _log(rng, 16, 384, 8)
        k, s = rng.choice([(3, 1), (3, 1), (3, 2), (1, 1), (1, 1)])
        fmt = rng.choice(["e2m1", "e2m1", "e4m3"])
        src = rng.choice(["f32", "bf16"])
        if kind == "stem":
            h = 16 * rng.randint(4, 26)
            w = 16 * rng.randint(4, 26)
            case = _conv("stem", batch, 3, rng.choice([16, 32]), h, w, 3, 2, fmt=fmt, src="bf16")
        elif kind == "merge":
            h, w = max(4, h // 2 * 2), max(4, w // 2 * 2)
            case = _conv("merge", batch, cin, cout, h, w, 1, 1, fmt=fmt, src=src, skip=_log(rng, 16, 256, 8))
        elif kind == "hidden":
            case = _conv("hidden", batch, cin, cout, h, w, k, s, fmt=fmt, src=src, terms=rng.randint(1, 3),
                         sr=rng.random() < 0.25)
        elif kind == "nvfp":
            fmt, xfmt = rng.choice([("e2m1", "e2m1"), ("e2m1", "e2m1"), ("e4m3", "e4m3"), ("e2m3", "e2m3")])
            case = _conv("nvfp", batch, cin, cout, h, w, k, s, fmt=fmt, xfmt=xfmt, src="f32")
        else:
            fmt, xfmt = rng.choice([("e2m1", "e2m1"), ("e2m1", "e2m1"), ("e4m3", "e4m3"), ("e4m3", "e4m3"),
                                    ("e2m3", "e2m3"), ("e2m1", "e3m2")])
            layout = rng.choice(["cbf", "cbf", "nchw", "nhwc"])
            sr = rng.random() < 0.3
            col = layout == "cbf" and rng.random() < 0.2
            if layout != "cbf" and fmt == xfmt and fmt != "e2m3" and rng.random() < 0.4:
                batch, k = rng.choice([2, 4, 8, 16]), rng.choice([1, 3, 5])
            case = _conv("layer", batch, cin, cout, h, w, k, s, fmt=fmt, xfmt=xfmt, src=src, layout=layout, sr=sr, col=col)
        if work(case)["bytes"] <= 8e8 and work(case)["flops"] <= 3e11:
            return case


def _cv(case):
    """The convolution; a merge's input channels are its parts' whole blocks."""
    cin = case["cin"]
    if case["kind"] == "merge":
        cin = 32 * (-(-case["cin"] // 32) + -(-case["skip"] // 32))
    return synth.conv_dict(case["batch"], cin, case["cout"], case["h"], case["w"], case["k"], case["s"])


# ---------------------------------------------------------------- inputs, on the GPU from the seed
def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 64 + k)
    return g


def _normal(shape, std, seed, k, dtype=torch.float32):
    return (torch.randn(shape, generator=_gen(seed, k), device=DEV) * std).to(dtype)


def _feature(shape, seed, k, dtype=torch.float32):
    return torch.nn.functional.silu(_normal(shape, 1.0, seed, k)).to(dtype)


def _kaiming(cv, seed, k, dtype):
    return _normal((cv["cout"], cv["cin"], cv["kh"], cv["kw"]), math.sqrt(2.0 / (cv["cin"] * cv["kh"] * cv["kw"])), seed, k,
                   dtype)


def _cbf_shape(n, c, h, w):
    return (n // 32, h, w, c, 32)


def _stored(shape, layout):
    n, c, h, w = shape
    return {"nchw": (n, c, h, w), "nhwc": (n, h, w, c)}.get(layout) or _cbf_shape(n, c, h, w)


def _workspace(cv, fmt):
    return torch.empty(max(16, mx.wgrad_workspace_bytes(cv, fmt)), dtype=torch.uint8, device=DEV)


def _graph(calls):
    """The step's calls captured once, as the benchmark launches them."""
    fns = [c[1] for c in calls]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for f in fns:
            f()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for f in fns:
            f()
    return graph


def prepare(case, seed):
    kind = case["kind"]
    dt = DTYPE[case["src"]]
    fmt = FMT[case["fmt"]]
    st = dict(case=case, kind=kind, seed=seed, dt=dt, fmt=fmt, xfmt=FMT[case.get("xfmt", case["fmt"])])
    if kind == "net":
        step = workloads.NetStep(workloads.yolo_net(case["size"]), case["batch"], fmt, DEV, seed=seed % 100000 * 100000,
                                 master=dt)
        return dict(st, step=step, graph=_graph(step.calls()))
    if kind == "replay":
        step = workloads.QlrStep(DEV, fmt, buffer=256, batch=case["batch"], seed=seed % 100000 * 100000, master=dt)
        return dict(st, step=step, graph=_graph(step.calls()))
    cv = _cv(case)
    n, h, w, cin, cout = cv["n"], cv["h"], cv["w"], cv["cin"], cv["cout"]
    ho, wo = synth.out_hw(cv)
    st.update(cv=cv, w=_kaiming(cv, seed, 1, dt), xshape=(n, cin, h, w), yshape=(n, cout, ho, wo))
    fbf = mx.FN_BF16 if dt == torch.bfloat16 else 0
    if kind in ("layer", "nvfp"):
        layout = case.get("layout", "cbf")
        st["layout"] = LAYOUT[layout]
        st["out"] = mx.CBF if layout == "cbf" else mx.NCHW
        st["x"] = _feature(_stored(st["xshape"], layout), seed, 0, dt)
        st["gy"] = _normal(_stored(st["yshape"], layout), 1e-3, seed, 2, dt)
        if kind == "layer" and case["col"]:
            c = mx.conv_struct(cv)
            st["col"] = tuple(torch.empty(f(c, st["xfmt"]), dtype=torch.uint8, device=DEV)
                              for f in (mx.lib().mxconv_im2col_codes_bytes, mx.lib().mxconv_im2col_scales_bytes))
    elif kind == "stem":
        st["x"] = torch.rand(st["xshape"], generator=_gen(seed, 0), device=DEV).to(dt)
        st["gq"] = mx.quantize(_normal(_cbf_shape(*st["yshape"]), 1e-3, seed, 2, dt), mx.ACT, fmt, mx.CBF, st["yshape"])
        st["xq"] = mx.MxTensor.empty(mx.ACT, fmt, st["xshape"], DEV)
        st["xq"].codes.zero_()
        st["wq"] = mx.quantize(st["w"], mx.WEIGHT, fmt)
    else:
        st["terms"] = [_normal(_cbf_shape(*st["yshape"]), 1e-3, seed, 10 + k, dt) for k in range(case.get("terms", 1))]
        if kind == "hidden":
            st["z"] = _normal(_cbf_shape(*st["xshape"]), 1.0, seed, 0, dt)
            st["xq"] = mx.quantize(torch.nn.functional.silu(st["z"]), mx.ACT, fmt, mx.CBF, st["xshape"])
        else:
            shapes = ((n, case["cin"], h // 2, w // 2), (n, case["skip"], h, w))
            st["pq"] = [mx.quantize(_feature(_cbf_shape(*s), seed, 4 + k), mx.ACT, fmt, mx.CBF, s)
                        for k, s in enumerate(shapes)]
            st["gxl"] = mx.CBF_BF16 if fbf else mx.CBF
    if kind in ("stem", "hidden", "merge"):
        st["fn"] = mx.FN_SILU | fbf
        st["y"] = torch.empty(_cbf_shape(*st["yshape"]), dtype=dt, device=DEV)
        st["ws"] = _workspace(cv, fmt)
        st["gw"] = torch.empty(tuple(st["w"].shape), dtype=torch.float32, device=DEV)
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    return _RUN[st["kind"]](st)


def _run_layer(st):
    case, cv, fmt, xfmt, lay = st["case"], st["cv"], st["fmt"], st["xfmt"], st["layout"]
    if lay == mx.CBF:
        xi = (st["x"], mx.ACT, xfmt, mx.CBF, st["xshape"], None)
        qx, qw = mx.quantize_multi([xi + ((cv,) + st["col"],) if "col" in st else xi,
                                    (st["w"], mx.WEIGHT, fmt, mx.NCHW, tuple(st["w"].shape), None)])
    else:
        qx = mx.quantize(st["x"], mx.ACT, xfmt, lay, st["xshape"])
        qw = mx.quantize(st["w"], mx.WEIGHT, fmt)
    y = mx.fwd(cv, qw, qx, layout=st["out"])
    if case["sr"]:
        qg = mx.quantize_sr(st["gy"], mx.ACT, fmt, st["seed"] + 7, lay, st["yshape"])
    else:
        qg = mx.quantize(st["gy"], mx.ACT, fmt, lay, st["yshape"])
    if fmt == xfmt:
        gx, gw = mx.backward(cv, qw, qg, qx, layout=st["out"])
    else:
        gx = mx.dgrad(cv, qw, qg, layout=st["out"])
        gw = mx.wgrad(cv, qg, qx)
    out = dict(y=y, gx=gx, gw=gw, xc=qx.codes, xs=qx.scales, wc=qw.codes, gc=qg.codes, gs=qg.scales)
    if "col" in st:
        out.update(cc=st["col"][0], cs=st["col"][1])
    return out


def _run_nvfp(st):
    cv = st["cv"]
    qx = mx.nvfp_quantize(st["x"], mx.ACT, st["xfmt"], mx.CBF, st["xshape"])
    qw = mx.nvfp_quantize(st["w"], mx.WEIGHT, st["fmt"])
    y = mx.nvfp_fwd(cv, qw, qx, layout=mx.CBF)
    qg = mx.nvfp_quantize(st["gy"], mx.ACT, st["fmt"], mx.CBF, st["yshape"])
    gx = mx.nvfp_dgrad(cv, qw, qg, layout=mx.CBF)
    gw = mx.nvfp_wgrad(cv, qg, qx)
    return dict(y=y, gx=gx, gw=gw, xc=qx.codes, xs=qx.scales, gc=qg.codes, gs=qg.scales)


def _run_hidden(st):
    cv, fmt = st["cv"], st["fmt"]
    qw = mx.quantize(st["w"], mx.WEIGHT, fmt)
    qy = mx.fwd_quant(cv, qw, st["xq"], fn=st["fn"] | mx.FN_PRE_OUT, act_out=st["y"])
    sr = st["seed"] + 7 if st["case"]["sr"] else None
    qg = mx.quantize_sum([(t, cv["cout"], 0, 0) for t in st["terms"]], st["yshape"], fmt, fn=st["fn"], z=st["y"], sr_seed=sr)
    qgx = mx.dgrad_quant(cv, qw, qg, fn=st["fn"], z=st["z"], sr_seed=sr)
    mx.wgrad(cv, qg, st["xq"], out=st["gw"], workspace=st["ws"], deferred=True)
    mx.wgrad_reduce_multi([(cv, fmt, st["ws"], st["gw"])])
    return dict(y=st["y"], gw=st["gw"], yc=qy.codes, ys=qy.scales, gc=qg.codes, gs=qg.scales, gxc=qgx.codes, gxs=qgx.scales)


def _run_merge(st):
    cv, fmt = st["cv"], st["fmt"]
    qw = mx.quantize(st["w"], mx.WEIGHT, fmt)
    qx = mx.concat_cbf([(st["pq"][0], 1), (st["pq"][1], 0)])
    qy = mx.fwd_quant(cv, qw, qx, fn=st["fn"] | mx.FN_PRE_OUT, act_out=st["y"])
    qg = mx.quantize_sum([(st["terms"][0], cv["cout"], 0, 0)], st["yshape"], fmt, fn=st["fn"], z=st["y"])
    gx, gw = mx.backward(cv, qw, qg, qx, layout=st["gxl"], gw_out=st["gw"], workspace=st["ws"])
    # the upsampled part's producer gets the sum over its 2x2 copies
    n, c, h, w = st["pq"][0].shape
    qu = mx.quantize_sum([(gx, cv["cin"], 0, 1)], (n, c, h, w), fmt, fn=mx.FN_BF16 if st["dt"] == torch.bfloat16 else 0)
    return dict(y=st["y"], gx=gx, gw=gw, yc=qy.codes, ys=qy.scales, gc=qg.codes, gs=qg.scales, uc=qu.codes, us=qu.scales)


def _run_stem(st):
    cv, fmt = st["cv"], st["fmt"]
    mx.quantize(st["x"], mx.ACT, fmt, out=st["xq"], keep_pad=True)
    qy = mx.fwd_quant(cv, st["wq"], st["xq"], fn=st["fn"] | mx.FN_PRE_OUT, act_out=st["y"])
    mx.wgrad(cv, st["gq"], st["xq"], out=st["gw"], workspace=st["ws"])
    return dict(y=st["y"], gw=st["gw"], xc=st["xq"].codes, xs=st["xq"].scales, yc=qy.codes, ys=qy.scales)


def _run_net(st):
    st["graph"].replay()
    s = st["step"]
    out = {"gw." + k: v for k, v in s.gw.items()}
    for o in s.net.outputs:
        out["y." + o] = s.y[o]
        out["c." + o] = s.t[o].codes
        out["s." + o] = s.t[o].scales
    return out


def _run_replay(st):
    st["graph"].replay()
    s = st["step"]
    return dict(gw=s.gw, y=s.y, c=[t.codes for t in s.x], s=[t.scales for t in s.x], g=[t.codes for t in s.gy])


_RUN = dict(layer=_run_layer, nvfp=_run_nvfp, hidden=_run_hidden, merge=_run_merge, stem=_run_stem, net=_run_net,
            replay=_run_replay)


# ---------------------------------------------------------------- what a pass cannot do without
def _mxb(fmt, n, c, h, w, act=True, real=False):
    """Bytes of the codes and scales; real: of a single block's real channels only."""
    cp, bn = -(-c // 32) * 32, 32 if n >= 32 or not act else n
    np_ = n if act else -(-n // 32) * 32
    rows = c if real and c < 32 else cp
    return np_ * h * w * rows * BITS[fmt] / 8.0 + np_ // bn * h * w * (cp // 32)


@functools.lru_cache(maxsize=None)
def _net_convs(size):
    net = workloads.yolo_net(size)
    return net, [n for n in net.nodes if n["kind"] == "conv"]


def work(case):
    kind, n = case["kind"], case["batch"]
    fmt = FMT[case["fmt"]]
    xfmt = FMT[case.get("xfmt", case["fmt"])]
    es = 2.0 if case["src"] == "bf16" else 4.0
    if kind == "net":
        # a training pass reads the image and the weights, keeps each convolution's pre-activation and codes for
        # the backward pass, and hands each gradient on once: every such tensor is written once and read once
        net, convs = _net_convs(case["size"])
        by = 0.0
        fl = 0.0
        for t in convs:
            el = n * t["c"] * t["h"] * t["w"]
            wsize = t["cout"] * t["cin_real"] * t["k"] * t["k"]
            by += 2 * es * el + 4 * _mxb(fmt, n, t["c"], t["h"], t["w"]) + 2.0 * wsize + 4.0 * wsize
            fl += workloads.real_flops(t, n) * (2 if net.node(t["src"])["kind"] == "input" else 3)
        img = net.nodes[0]
        return dict(bytes=by + 2.0 * n * img["c"] * img["h"] * img["w"], flops=fl)
    if kind == "replay":
        by, fl = 4.0 * 32 * 3 * 128 * 128, 0.0
        for ci, co in workloads.QlrStep.BACK:
            f = 2.0 * n * ci * co * 9 * 256
            fl += f * (2 if ci == 128 else 3)
            by += 2 * es * n * co * 256 + 4 * _mxb(fmt, n, co, 16, 16) + 6.0 * ci * co * 9
        h = 64
        for ci, co in workloads.QlrStep.FRONT:
            fl += 2.0 * 32 * co * h * h * ci * 9
            by += 2 * _mxb(fmt, 32, co, h, h)
            h //= 2
        return dict(bytes=by, flops=fl)
    cv = _cv(case)
    cin, cout, h, w, k = cv["cin"], cv["cout"], cv["h"], cv["w"], cv["kh"]
    ho, wo = synth.out_hw(cv)
    f = 2.0 * n * cout * ho * wo * cin * k * k
    xe, ye, we = n * cin * h * w, n * cout * ho * wo, cout * cin * k * k
    xb, gb = _mxb(xfmt, n, cin, h, w), _mxb(fmt, n, cout, ho, wo)
    wb = _mxb(fmt, cout, cin, k, k, act=False)
    if kind in ("layer", "nvfp"):
        # the sources read, the codes that the user gets, the three full-precision results
        by = es * (xe + we + ye) + xb + wb + gb + 4.0 * (ye + xe + we)
        if case.get("col"):
            by += _mxb(xfmt, n, cin, ho, wo) * k * k
        return dict(bytes=by, flops=3 * f)
    if kind == "stem":
        xr = _mxb(xfmt, n, cin, h, w, real=True)
        return dict(bytes=es * xe + xr + 2 * gb + es * ye + 4.0 * we + wb, flops=2 * f)
    if kind == "hidden":
        by = es * we + wb + xb + gb + es * ye * (1 + case["terms"]) + gb + es * xe + xb + 4.0 * we
        return dict(bytes=by, flops=3 * f)
    pb = _mxb(fmt, n, case["cin"], h // 2, w // 2)
    by = es * we + wb + pb + _mxb(fmt, n, case["skip"], h, w) + gb + 2 * es * ye + gb + es * xe + 4.0 * we + pb
    return dict(bytes=by, flops=3 * f)


# ---------------------------------------------------------------- agreement
def tolerance(case):
    kind = case["kind"]
    if kind in ("layer", "nvfp"):
        # exact codes in, exact products, fp32 sums: only the order of the additions is free (measured against 64 bits:
        # at most 1.1e-7, and 7e-7 for the largest)
        return {"rel": 1e-6, "max": 5e-6, "differ": 0.0}
    if kind in ("net", "replay"):
        # FP4 products sum exactly in fp32, so equal roundings give equal codes; one changed code of the image
        # changes most of the codes behind it, so more than this would say nothing
        return {"rel": 2e-2, "max": 0.5, "differ": 5e-3}
    # SiLU's exponential to an ulp decides a tie of the next codes now and then (measured against 64 bits: 2e-4 of a
    # weight gradient, 1.2e-3 of a small one); a bf16 result moves by its last bit
    return {"rel": 5e-3, "max": 5e-2, "differ": 1e-3}


# ---------------------------------------------------------------- the same in 64 bits, without this repository's code
def _round(v, fmt):
    mb, emin, top, _ = GRID[fmt]
    _, e = torch.frexp(v.abs())
    q = torch.exp2((e.double() - 1).clamp_min(emin) - mb)
    r = torch.round(v / q) * q
    return torch.where(v == 0, torch.zeros_like(v), r.clamp(-top, top))


def _blocks(x, bn, cb):
    """(n, c, h, w) with both sides padded to whole blocks, as (nb, bn, cbk, cb, h, w)."""
    n, c, h, w = x.shape
    x = torch.nn.functional.pad(x, (0, 0, 0, 0, 0, -c % cb, 0, -n % bn))
    return x.reshape(x.shape[0] // bn, bn, x.shape[1] // cb, cb, h, w)


def _mx_values(x, fmt, bn):
    n, c, h, w = x.shape
    b = _blocks(x.double(), bn, 32)
    amax = b.abs().amax(dim=(1, 3), keepdim=True)
    _, e = torch.frexp(amax)
    s = torch.exp2((e.double() - 1 - GRID[fmt][3]).clamp(-127, 127))
    s = torch.where(amax == 0, torch.ones_like(s), s)
    v = _round(b / s, fmt) * s
    return v.reshape(-1, v.shape[2] * 32, h, w)[:n, :c]


def _nv_values(x, fmt):
    """The format's own fp32 steps (they decide the codes), then exact values."""
    n, c, h, w = x.shape
    b = _blocks(x.float(), 8, 8)
    top = torch.tensor(GRID[fmt][2], device=x.device)
    t = b.abs().max() / (448.0 * top)
    r = (b.abs().amax(dim=(1, 3), keepdim=True) / (t * top)).double()
    bs = _round(r, mx.E4M3).float()
    v = _round(torch.where(bs == 0, torch.zeros_like(b), b / (bs * t)).double(), fmt) * bs.double() * t.double()
    return v.reshape(-1, v.shape[2] * 8, h, w)[:n, :c]


def _nchw(t, shape, layout):
    if layout == mx.CBF:
        return t.permute(0, 4, 3, 1, 2).reshape(shape)
    return t.permute(0, 3, 1, 2) if layout == mx.NHWC else t


def _to(t, layout):
    n, c, h, w = t.shape
    return t.reshape(n // 32, 32, c, h, w).permute(0, 3, 4, 2, 1).contiguous() if layout == mx.CBF else t.contiguous()


def _taps(cv, x):
    """For each tap, its rows of the padded input: (kh, kw, (cin, n*ho*wo))."""
    ho, wo = synth.out_hw(cv)
    xp = torch.nn.functional.pad(x, (cv["pw"],) * 2 + (cv["ph"],) * 2)
    for a in range(cv["kh"]):
        for b in range(cv["kw"]):
            t = xp[:, :, a:a + (ho - 1) * cv["sh"] + 1:cv["sh"], b:b + (wo - 1) * cv["sw"] + 1:cv["sw"]]
            yield a, b, t.transpose(0, 1).reshape(x.shape[1], -1)


def _conv64(cv, w, x):
    ho, wo = synth.out_hw(cv)
    y = torch.zeros((cv["cout"], cv["n"] * ho * wo), dtype=torch.float64, device=x.device)
    for a, b, t in _taps(cv, x):
        y += torch.mm(w[:, :, a, b].contiguous(), t)
    return y.reshape(cv["cout"], cv["n"], ho, wo).transpose(0, 1)


def _wgrad64(cv, g, x):
    gf = g.transpose(0, 1).reshape(cv["cout"], -1)
    gw = torch.empty((cv["cout"], cv["cin"], cv["kh"], cv["kw"]), dtype=torch.float64, device=x.device)
    for a, b, t in _taps(cv, x):
        gw[:, :, a, b] = torch.mm(gf, t.t().contiguous())
    return gw


def _dgrad64(cv, w, g):
    ho, wo = synth.out_hw(cv)
    gf = g.transpose(0, 1).reshape(cv["cout"], -1)
    gx = torch.zeros((cv["cin"], cv["n"], cv["h"] + 2 * cv["ph"], cv["w"] + 2 * cv["pw"]), dtype=torch.float64,
                     device=g.device)
    for a in range(cv["kh"]):
        for b in range(cv["kw"]):
            t = torch.mm(w[:, :, a, b].t().contiguous(), gf).reshape(cv["cin"], cv["n"], ho, wo)
            gx[:, :, a:a + (ho - 1) * cv["sh"] + 1:cv["sh"], b:b + (wo - 1) * cv["sw"] + 1:cv["sw"]] += t
    return gx[:, :, cv["ph"]:cv["ph"] + cv["h"], cv["pw"]:cv["pw"] + cv["w"]].transpose(0, 1)


def exact(case, seed):
    """The full-precision results in 64 bits; codes are whole numbers and have none.  Stochastically rounded
    gradients and whole networks have no such value here."""
    kind = case["kind"]
    if kind in ("net", "replay"):
        return None
    st = prepare(case, seed)
    cv, fmt, xfmt = st["cv"], st["fmt"], st["xfmt"]
    bn = synth.batch_block(cv["n"])
    w = _mx_values(st["w"], fmt, 32) if kind != "nvfp" else _nv_values(st["w"], fmt)
    if kind in ("layer", "nvfp"):
        lay, out = st["layout"], st["out"]
        x, g = _nchw(st["x"], st["xshape"], lay), _nchw(st["gy"], st["yshape"], lay)
        if kind == "nvfp":
            x, g = _nv_values(x, xfmt), _nv_values(g, fmt)
        else:
            x, g = _mx_values(x, xfmt, bn), _mx_values(g, fmt, bn)
        sr = case.get("sr", False)
        got = dict(y=_to(_conv64(cv, w, x), out), gx=None if sr else _to(_dgrad64(cv, w, g), out),
                   gw=None if sr else _wgrad64(cv, g, x), xc=None, xs=None, gc=None, gs=None)
        if kind == "layer":
            got["wc"] = None
        if "col" in st:
            got.update(cc=None, cs=None)
        return got
    if kind == "stem":
        x = _mx_values(st["x"], fmt, 32)
        g = _mx_values(_nchw(_normal(_cbf_shape(*st["yshape"]), 1e-3, seed, 2, st["dt"]), st["yshape"], mx.CBF), fmt, 32)
        return dict(y=_to(_conv64(cv, w, x), mx.CBF), gw=_wgrad64(cv, g, x), xc=None, xs=None, yc=None, ys=None)
    if kind == "hidden":
        x = _mx_values(_nchw(torch.nn.functional.silu(st["z"]), st["xshape"], mx.CBF), fmt, 32)
    else:
        n, h, wd = cv["n"], cv["h"], cv["w"]
        parts = []
        for k, s in enumerate(((n, case["cin"], h // 2, wd // 2), (n, case["skip"], h, wd))):
            v = _mx_values(_nchw(_feature(_cbf_shape(*s), seed, 4 + k), s, mx.CBF), fmt, 32)
            v = torch.nn.functional.pad(v, (0, 0, 0, 0, 0, -s[1] % 32))
            parts.append(v.repeat_interleave(2, 2).repeat_interleave(2, 3) if k == 0 else v)
        x = torch.cat(parts, 1)
    y = _conv64(cv, w, x)
    z = y.to(st["dt"]).double()
    sg = torch.sigmoid(z)
    total = sum(_nchw(t, st["yshape"], mx.CBF).double() for t in st["terms"])
    g = _mx_values(total * sg * (1 + z * (1 - sg)), fmt, 32)
    got = dict(y=_to(y, mx.CBF), gw=None if case.get("sr") else _wgrad64(cv, g, x), yc=None, ys=None, gc=None, gs=None)
    if kind == "hidden":
        return dict(got, gxc=None, gxs=None)
    return dict(got, gx=_to(_dgrad64(cv, w, g), mx.CBF), uc=None, us=None)
