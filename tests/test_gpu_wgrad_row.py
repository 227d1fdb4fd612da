"""The kernel-row weight gradient (3-wide kernels, batch block 32) at the edges
of its tiles: one column, an odd number of output rows, rows and columns of
padding wider than the input, unequal row and column strides, kernels of one
and five rows, channels that fill no block, tiles of 32 x 32 and 64 x 64, one
split and many -- against the oracle, within 1e-5 of the sum of absolute
products, and mxconv_backward equal to it bit for bit."""
import numpy as np
import pytest
import torch

import mx_tolerance as mxt
import oracle
import wgrad_plan
from paper_2609_28358_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SAMPLES = 3000


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_28358_amd import mxconv
    mxconv.lib()
    return mxconv


def _cv(n, cin, cout, h, w, kh=3, sh=1, sw=1, ph=1, pw=1):
    return dict(n=n, cin=cin, cout=cout, h=h, w=w, kh=kh, kw=3, sh=sh, sw=sw, ph=ph, pw=pw)


LAYERS = [
    _cv(32, 3, 16, 31, 33, sw=2, sh=2),              # the stem's shape, odd sizes
    _cv(32, 32, 32, 1, 1),                           # one pixel: every tap but the middle in the padding
    _cv(96, 24, 20, 5, 1),                           # one column, an odd number of rows over three groups
    _cv(32, 16, 32, 3, 4, pw=2, ph=2),               # padding on both sides of every row
    _cv(64, 40, 24, 9, 7, kh=1, ph=0),               # one kernel row, two channel blocks against one
    _cv(32, 33, 65, 12, 11, kh=5, sh=2, sw=1, ph=2),
    _cv(32, 32, 64, 10, 13, sh=1, sw=2, pw=0),
    _cv(32, 8, 8, 40, 57),                           # many splits, some waves past the end
    _cv(64, 70, 72, 33, 63),                         # 64 x 64 tiles, the third block of each side alone
    _cv(64, 70, 72, 65, 64, sh=2, sw=2),
    _cv(32, 70, 72, 67, 64),                         # 64 x 64 tiles, the last row pair half empty
    _cv(32, 70, 72, 133, 129, sh=2, sw=2),
]
# 64 x 64 tiles: these layers, the strided ones in FP8 only
WIDE = {8: False, 9: True, 10: False, 11: True}


def _operands(mx, cv, fg, fx, seed, x=None, gy=None):
    if x is None:
        x, _, gy = synth.layer_inputs(cv, seed, kind="sweep")
    q = [mx.quantize(synth.nchw_to_cbf(t, 32).to(DEV), mx.ACT, f, layout=mx.CBF, shape=tuple(t.shape))
         for t, f in ((gy, fg), (x, fx))]
    o = [oracle.quantize(t.numpy(), oracle.NCHW, oracle.ACT, f, *t.shape) for t, f in ((gy, fg), (x, fx))]
    return q, o


@pytest.mark.parametrize("fg,fx", [(0, 0), (1, 1), (2, 2), (1, 3)])
@pytest.mark.parametrize("k", range(len(LAYERS)))
def test_against_oracle(mx, k, fg, fx):
    cv = LAYERS[k]
    (qg, qx), (og, ox) = _operands(mx, cv, fg, fx, 900 + k)
    gw = torch.full((cv["cout"], cv["cin"], cv["kh"], 3), 9.0, device=DEV)
    ws = torch.full((max(16, mx.wgrad_workspace_bytes(cv, mx.pair(fg, fx))),), 255, dtype=torch.uint8, device=DEV)
    mx.wgrad(cv, qg, qx, out=gw, workspace=ws)
    dims = tuple(gw.shape)
    rng = np.random.default_rng(k)
    idx = (np.stack(np.meshgrid(*[np.arange(d) for d in dims], indexing="ij"), -1).reshape(-1, 4)
           if np.prod(dims) <= SAMPLES else np.stack([rng.integers(0, d, SAMPLES) for d in dims], 1))
    r, s = oracle.wgrad_at(cv, fg if fg == fx else (fg, fx), og, ox, idx)
    got = gw.cpu().numpy()[tuple(idx.T)]
    err = mxt.gemm_err(got, r, s)
    assert err <= 1.0, f"layer {k}: error is {err:.3f} of the allowed bound"
    if fg == fx:
        w = synth.kaiming(cv["cout"], cv["cin"], cv["kh"], 3, 1)
        qw = mx.quantize(w.to(DEV), mx.WEIGHT, fg)
        if cv["sh"] == cv["sw"] or fg < 2:
            gw2 = mx.backward(cv, qw, qg, qx)[1]
            torch.cuda.synchronize()
            assert torch.equal(gw, gw2), f"layer {k}: backward's weight gradient differs"


@pytest.mark.parametrize("fg,fx", [(0, 0), (1, 1), (2, 2), (1, 3)])
def test_layers_reach_their_tiles(mx, fg, fx):
    for k, cv in enumerate(LAYERS):
        plan = wgrad_plan.row_plan(cv, fg, fx)
        if k in WIDE:
            assert (plan is not None and plan[0] == 2) == (fg == 0 or not WIDE[k]), (k, plan)
        else:
            assert plan is not None and plan[0] == 1, (k, plan)
        assert mx.wgrad_workspace_bytes(cv, mx.pair(fg, fx)) == wgrad_plan.workspace_bytes(cv, fg, fx)
    odd = [k for k in WIDE if (LAYERS[k]["n"] // 32 * synth.out_hw(LAYERS[k])[0]) % 2]
    assert {WIDE[k] for k in odd} == {False, True}


@pytest.mark.parametrize("fg,fx", [(0, 0), (1, 1), (2, 2), (1, 3)])
@pytest.mark.parametrize("sw", [1, 2])
def test_walks_of_every_length(mx, fg, fx, sw):
    """Waves whose walk ends at each slot of the operand ring: one to nine
    columns, row pairs complete and half empty."""
    for w in range(1, 10):
        for h in (2, 3):
            cv = _cv(32, 24, 20, h, w, sh=1, sw=sw)
            (qg, qx), (og, ox) = _operands(mx, cv, fg, fx, 500 + 10 * w + h)
            gw = mx.wgrad(cv, qg, qx)
            dims = tuple(gw.shape)
            idx = np.stack(np.meshgrid(*[np.arange(d) for d in dims], indexing="ij"), -1).reshape(-1, 4)
            r, s = oracle.wgrad_at(cv, fg if fg == fx else (fg, fx), og, ox, idx)
            assert mxt.gemm_err(gw.cpu().numpy()[tuple(idx.T)], r, s) <= 1.0, (w, h)


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("cv", [_cv(32, 24, 24, 6, 5), _cv(64, 70, 72, 33, 63)], ids=["32x32", "64x64"])
def test_a_nan_reaches_its_taps_only(mx, fmt, cv):
    """A non-finite X pixel in the first column meets the taps whose window
    covers it, not the ones that would reach it from outside the output."""
    x, _, gy = synth.layer_inputs(cv, 77, kind="sweep")
    x[0, 1, :, 0] = float("nan")                     # column 0, every row: taps 0 and 1 of each kernel row
    (qg, qx), _ = _operands(mx, cv, fmt, fmt, 0, x, gy)
    gw = mx.wgrad(cv, qg, qx).cpu()
    assert torch.isnan(gw[:, :32, :, :2]).all()      # the whole 32-channel block shares the NaN scale
    assert not torch.isnan(gw[:, :, :, 2]).any()
    assert not torch.isnan(gw[:, 32:]).any()


@pytest.mark.parametrize("fmt,n,cin,cout,h,sw", [(0, 192, 3, 16, 640, 2), (1, 736, 24, 8, 430, 1)])
def test_tensors_past_two_gib(mx, fmt, n, cin, cout, h, sw):
    """Codes of 2 GiB and more, in launches of some batch groups each: against
    the sum, in 64 bits, of the groups' own gradients."""
    cv = _cv(n, cin, cout, h, h, sh=sw, sw=sw)
    assert wgrad_plan.row_plan(cv, fmt, fmt) is not None
    gen = torch.Generator(device=DEV).manual_seed(n)
    ho, wo = synth.out_hw(cv)

    def tensor(c, hh, ww):
        q = mx.MxTensor.empty(mx.ACT, fmt, (n, c, hh, ww), DEV)
        q.codes.random_(0, 0x7F, generator=gen).bitwise_and_(0x7F if fmt == 0 else 0x77)   # positive, no NaN
        q.scales.random_(118, 124, generator=gen)
        return q
    qx, qg = tensor(cin, h, h), tensor(cout, ho, wo)
    assert max(qx.codes.numel(), qg.codes.numel()) >= 1 << 31
    gw = mx.wgrad(cv, qg, qx)
    ng = n // 32
    one = dict(cv, n=32)
    ref = torch.zeros(gw.shape, dtype=torch.float64, device=DEV)
    for g in range(ng):
        part = [mx.MxTensor(t.codes[g * (t.codes.numel() // ng):(g + 1) * (t.codes.numel() // ng)].clone(),
                            t.scales[g * (t.scales.numel() // ng):(g + 1) * (t.scales.numel() // ng)].clone(),
                            mx.ACT, fmt, (32,) + t.shape[1:]) for t in (qg, qx)]
        ref += mx.wgrad(one, *part).double()
    assert bool(((gw.double() - ref).abs() <= 1e-5 * ref).all())   # positive products: their sum is the bound's scale
