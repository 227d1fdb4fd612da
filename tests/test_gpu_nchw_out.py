"""The batch-block-32 forward and input gradient into NCHW outputs: every
element equals the channel-batch-first output's, bit for bit, over the tile
shapes (4, 8 and 16 pixels, one and two row blocks), strides, pixel segments
that end inside a tile and channels that end inside a block; nothing else of
the buffer is written."""
import pytest
import torch

from paper_2609_28358_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

LAYERS = [
    (synth.conv_dict(32, 40, 24, 7, 9, 3, 1), 0),          # few tiles: one pixel per wave
    (synth.conv_dict(64, 70, 100, 21, 19, 3, 1), 0),
    (synth.conv_dict(32, 33, 65, 23, 30, 1, 1), 1),
    (synth.conv_dict(64, 16, 20, 33, 35, 3, 1), 1),        # one row block: 16 pixels (8 at stride 2)
    (synth.conv_dict(64, 24, 17, 34, 37, 3, 2), 1),
    (synth.conv_dict(32, 64, 48, 20, 26, 3, 2), 0),
    (synth.conv_dict(32, 64, 40, 11, 10, 3, 1), 2),
    (synth.conv_dict(64, 3, 16, 34, 37, 3, 2), 1),         # few rows: 3 (16 wide tiles), 1, 5, 33 and 8
    (synth.conv_dict(64, 1, 5, 30, 33, 1, 1), 1),
    (synth.conv_dict(32, 5, 3, 9, 10, 3, 1), 0),
    (synth.conv_dict(32, 33, 1, 17, 19, 3, 2), 0),
    (synth.conv_dict(32, 8, 35, 20, 21, 3, 1), 2),
]


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_28358_amd import mxconv
    mxconv.lib()
    return mxconv


@pytest.mark.parametrize("k", range(len(LAYERS)))
def test_nchw_is_cbf_permuted(mx, k):
    cv, fmt = LAYERS[k]
    x, w, gy = (t.to(DEV) for t in synth.layer_inputs(cv, 700 + k, kind="sweep"))
    qx, qw, qg = mx.quantize(x, mx.ACT, fmt), mx.quantize(w, mx.WEIGHT, fmt), mx.quantize(gy, mx.ACT, fmt)
    gw = torch.empty(w.shape, device=DEV)

    def both(call, shape):
        n = x.new_empty(shape).numel()
        buf = torch.full((n + 512,), 3.5, device=DEV)
        out = buf[256:256 + n].view(shape)
        call(mx.NCHW, out)
        ref = synth.cbf_to_nchw(call(mx.CBF, None), *shape, 32)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert (buf[:256] == 3.5).all() and (buf[256 + n:] == 3.5).all()

    both(lambda lay, out: mx.fwd(cv, qw, qx, layout=lay, out=out), tuple(gy.shape))
    both(lambda lay, out: mx.dgrad(cv, qw, qg, layout=lay, out=out), tuple(x.shape))
    both(lambda lay, out: mx.backward(cv, qw, qg, qx, layout=lay, gx_out=out, gw_out=gw)[0], tuple(x.shape))
