"""GPU parity of the network-step operations against the oracle.

mxconv_concat_cbf: codes and scales bit for bit equal to oracle.concat_cbf
(channel concatenation and 2x nearest upsampling on whole MX blocks), into
garbage-filled outputs, for several batch blocks and both formats.

mxconv_quantize_sum: the fp32 values it quantized (returned through `vals`)
against oracle.gradient_sum in fp64 -- within the rounding of at most eight
fp32 additions of the terms plus SiLU' in fp32 (1e-6 of the sum of absolute
terms times |fn'|, plus 1e-6 relative) -- and its codes and scales bit for
bit equal to the oracle quantizer applied to those values (both sides take
the rounding decision on the same numbers).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_28358_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_28358_amd import mxconv
    mxconv.lib()
    return mxconv


def _garbage(t):
    t.random_(0, 256)
    return t


CONCAT_CASES = [
    # n, h, w, parts: (channels, up)
    (32, 6, 4, [(40, 0), (16, 1), (32, 0)]),
    (64, 8, 10, [(64, 1), (128, 0)]),
    (16, 5, 7, [(32, 0), (48, 0), (16, 0), (96, 0)]),
    (32, 40, 40, [(256, 1), (128, 0)]),                     # the neck's first concatenation, one group
    (8, 4, 4, [(32, 1)]),
]


@pytest.mark.parametrize("fmt", [0, 1], ids=["e4m3", "e2m1"])
@pytest.mark.parametrize("case", CONCAT_CASES, ids=lambda c: f"n{c[0]}_{c[1]}x{c[2]}_{len(c[3])}parts")
def test_concat(mx, fmt, case):
    n, h, w, parts = case
    xs, qs, ops = [], [], []
    for k, (c, up) in enumerate(parts):
        hk, wk = (h // 2, w // 2) if up else (h, w)
        x = synth.silu_normal((n, c, hk, wk), 50 + k)
        q = mx.quantize(x.to(DEV), mx.ACT, fmt)
        qs.append((q, up))
        ox = oracle.quantize(x.numpy(), oracle.NCHW, oracle.ACT, fmt, n, c, hk, wk)
        ops.append((ox[0], ox[1], c, up))
    tot = sum(-(-c // 32) for c, _ in parts)
    out = mx.MxTensor.empty(mx.ACT, fmt, (n, 32 * tot, h, w), DEV)
    _garbage(out.codes), _garbage(out.scales)
    y = mx.concat_cbf(qs, out=out)
    torch.cuda.synchronize()
    rc, rs = oracle.concat_cbf(ops, fmt, n, h, w)
    assert np.array_equal(y.scales.cpu().numpy(), rs)
    assert np.array_equal(y.codes.cpu().numpy(), rc)


def test_concat_errors(mx):
    import ctypes
    L = mx.lib()
    x = mx.quantize(synth.silu_normal((32, 32, 4, 4), 1).to(DEV), mx.ACT, 0)
    good = (mx.MxcPart * 1)(mx.MxcPart(x.codes.data_ptr(), x.scales.data_ptr(), 1, 0))
    bad_up = (mx.MxcPart * 1)(mx.MxcPart(x.codes.data_ptr(), x.scales.data_ptr(), 1, 1))
    out = mx.MxTensor.empty(mx.ACT, 0, (32, 32, 4, 4), DEV)
    P = ctypes.c_void_p
    assert L.mxconv_concat_cbf(0, 32, 4, 4, 0, good, P(out.codes.data_ptr()), P(out.scales.data_ptr()), None) == -2
    assert L.mxconv_concat_cbf(0, 32, 4, 4, 5, good, P(out.codes.data_ptr()), P(out.scales.data_ptr()), None) == -2
    assert L.mxconv_concat_cbf(0, 32, 5, 4, 1, bad_up, P(out.codes.data_ptr()), P(out.scales.data_ptr()), None) == -3
    assert L.mxconv_concat_cbf(0, 32, 4, 4, 1, good, None, P(out.scales.data_ptr()), None) == -1
    assert L.mxconv_concat_cbf(0, 33, 4, 4, 1, good, P(out.codes.data_ptr()), P(out.scales.data_ptr()), None) == -3


SUM_CASES = [
    # n, c, h, w, terms: (c_src, c_off, down), fn
    (32, 32, 6, 5, [(32, 0, 0)], 0),
    (32, 48, 4, 6, [(96, 16, 0), (48, 0, 0)], 2),
    (64, 16, 5, 4, [(48, 32, 1), (16, 0, 0), (32, 16, 0)], 2),   # a 16-channel part: padded block
    (32, 64, 3, 3, [(64, 0, 0), (128, 64, 1), (64, 0, 0), (192, 0, 0)], 2),
    (32, 40, 7, 9, [(40, 0, 0), (80, 40, 0)], 0),
    (32, 48, 4, 6, [(96, 16, 0), (48, 0, 1)], 1),                # ReLU
    (32, 3, 5, 7, [(3, 0, 0), (8, 5, 0), (3, 0, 0), (4, 1, 0)], 2),   # four plain terms, few channels
    (64, 41, 4, 3, [(41, 0, 0), (64, 8, 0), (41, 0, 0)], 0),
]


@pytest.mark.parametrize("fmt", [0, 1], ids=["e4m3", "e2m1"])
@pytest.mark.parametrize("case", SUM_CASES, ids=lambda c: f"n{c[0]}c{c[1]}_{c[2]}x{c[3]}_{len(c[4])}terms_fn{c[5]}")
def test_quantize_sum(mx, fmt, case):
    n, c, h, w, tdesc, fn = case
    terms_gpu, terms_o, terms_abs = [], [], []
    for k, (c_src, c_off, down) in enumerate(tdesc):
        hs, ws = (2 * h, 2 * w) if down else (h, w)
        g = synth.normal((n, c_src, hs, ws), 1e-3 * (k + 1), 70 + k)
        gc = synth.nchw_to_cbf(g, 32)
        terms_gpu.append((gc.to(DEV), c_src, c_off, down))
        flat = gc.numpy().reshape(-1)
        terms_o.append((flat, c_src, c_off, down))
        terms_abs.append((np.abs(flat), c_src, c_off, down))
    z = synth.normal((n, c, h, w), 2.0, 90)
    zc = synth.nchw_to_cbf(z, 32)
    vals = torch.full((n // 32, h, w, c, 32), float("nan"), device=DEV)
    out = mx.MxTensor.empty(mx.ACT, fmt, (n, c, h, w), DEV)
    _garbage(out.codes), _garbage(out.scales)
    g = mx.quantize_sum(terms_gpu, (n, c, h, w), fmt, fn=fn, z=zc.to(DEV) if fn else None, out=out, vals=vals)
    torch.cuda.synchronize()
    v = synth.cbf_to_nchw(vals.cpu(), n, c, h, w, 32).numpy()
    ref = oracle.gradient_sum(terms_o, fn, zc.numpy().reshape(-1), n, c, h, w)
    sabs = oracle.gradient_sum(terms_abs, oracle.FN_NONE, None, n, c, h, w)
    gscale = np.abs(oracle.act_grad(z.numpy(), fn))
    tol = 1e-6 * sabs * np.maximum(1.0, gscale) + 1e-6 * np.abs(ref)
    assert np.all(np.abs(v - ref) <= tol), float(np.max(np.abs(v - ref) / np.maximum(tol, 1e-300)))
    rc, rs = oracle.quantize(v.astype(np.float32), oracle.NCHW, oracle.ACT, fmt, n, c, h, w)
    assert np.array_equal(g.scales.cpu().numpy(), rs)
    assert np.array_equal(g.codes.cpu().numpy(), rc)


def test_quantize_sum_errors(mx):
    t = torch.zeros((1, 4, 4, 32, 32), device=DEV)
    ok = [(t, 32, 0, 0)]
    with pytest.raises(mx.MxconvError, match="code -3"):
        mx.quantize_sum([(t, 32, 16, 0)], (32, 32, 4, 4), 0)          # slice past the source's channels
    with pytest.raises(mx.MxconvError, match="code -3"):
        mx.quantize_sum(ok, (16, 32, 4, 4), 0)                       # batch block 16
    with pytest.raises(mx.MxconvError, match="code -2"):
        mx.quantize_sum(ok, (32, 32, 4, 4), 2)                       # FP6 not offered
    with pytest.raises(mx.MxconvError, match="code -1"):
        mx.quantize_sum(ok, (32, 32, 4, 4), 0, fn=mx.FN_SILU)        # SiLU' needs z


@pytest.mark.parametrize("sr", [None, 5], ids=["rne", "sr"])
@pytest.mark.parametrize("bf", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("fmt", [0, 1], ids=["e4m3", "e2m1"])
@pytest.mark.parametrize("c,nt,fn", [(1, 1, 2), (8, 2, 2), (9, 3, 1), (40, 3, 2), (72, 2, 0)])
def test_quantize_sum_plain_as_any(mx, c, nt, fn, fmt, bf, sr):
    """Plain terms, any number of them and rows that hold no channel, against the
    form that takes any terms (reached by a 2x2 patch sum of zeros)."""
    dt = torch.bfloat16 if bf else torch.float32
    cbf = lambda ch, std, seed: synth.nchw_to_cbf(synth.normal((64, ch, 5, 3), std, seed), 32).to(dt).to(DEV)
    terms = [(cbf(c + 8 * k, 1e-3, 50 + k), c + 8 * k, 8 * k, 0) for k in range(nt)]
    patch = [(torch.zeros((2, 10, 6, c, 32), dtype=dt, device=DEV), c, 0, 1)]
    z = cbf(c, 2.0, 60)
    got = []
    for ts in (terms, terms + patch):
        vals = torch.full((2, 5, 3, c, 32), float("nan"), device=DEV)
        out = mx.MxTensor.empty(mx.ACT, fmt, (64, c, 5, 3), DEV)
        _garbage(out.codes), _garbage(out.scales)
        mx.quantize_sum(ts, (64, c, 5, 3), fmt, fn=fn | (mx.FN_BF16 if bf else 0), z=z if fn else None, out=out,
                        vals=vals, sr_seed=sr)
        got.append((out.codes, out.scales, vals))
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("sr", [None, 5], ids=["rne", "sr"])
@pytest.mark.parametrize("bf", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("fmt", [0, 1], ids=["e4m3", "e2m1"])
@pytest.mark.parametrize("c,nt,fn", [(8, 1, 2), (16, 2, 2), (17, 1, 1), (48, 2, 0), (72, 1, 2)])
def test_quantize_sum_few_terms_as_many(mx, c, nt, fn, fmt, bf, sr):
    """One or two plain terms take a path of their own: the same codes, scales
    and values as the path for any terms (three or more; the further ones zero)."""
    dt = torch.bfloat16 if bf else torch.float32
    cbf = lambda ch, std, seed: synth.nchw_to_cbf(synth.normal((64, ch, 5, 3), std, seed), 32).to(dt).to(DEV)
    terms = [(cbf(c + 8 * k, 1e-3, 30 + k), c + 8 * k, 8 * k, 0) for k in range(nt)]
    zero = [(torch.zeros_like(terms[0][0]), c, 0, 0)] * (3 - nt)
    z = cbf(c, 2.0, 40)
    got = []
    for ts in (terms, terms + zero):
        vals = torch.full((2, 5, 3, c, 32), float("nan"), device=DEV)
        out = mx.MxTensor.empty(mx.ACT, fmt, (64, c, 5, 3), DEV)
        _garbage(out.codes), _garbage(out.scales)
        mx.quantize_sum(ts, (64, c, 5, 3), fmt, fn=fn | (mx.FN_BF16 if bf else 0), z=z if fn else None, out=out,
                        vals=vals, sr_seed=sr)
        got.append((out.codes, out.scales, vals))
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a, b)
