"""The reduction of split-K partial sums, several layers in one launch: random
partials in the workspaces, against the stated order in fp32 (below 64 splits
four running sums per column, from 64 on sixteen, then a pairwise tree), bit
for bit, and nothing written past a layer's gradient."""
import pytest
import torch

from paper_2609_28358_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# one column block to many, splits on both sides of 64, channels inside a block
LAYERS = [
    synth.conv_dict(32, 32, 1, 40, 40, 1, 1),
    synth.conv_dict(64, 16, 16, 80, 80, 3, 1),
    synth.conv_dict(32, 3, 16, 64, 64, 3, 2),
    synth.conv_dict(64, 48, 80, 35, 27, 3, 1),
    synth.conv_dict(32, 70, 33, 9, 7, 3, 1),
    synth.conv_dict(64, 96, 64, 20, 20, 1, 1),
    synth.conv_dict(64, 128, 128, 20, 20, 3, 1),
]


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_28358_amd import mxconv
    mxconv.lib()
    return mxconv


def _reference(ws, cv):
    """The gradient from the partials [split][Cout_p][tap * Cin_p + ci]."""
    cop, cip = -(-cv["cout"] // 32) * 32, -(-cv["cin"] // 32) * 32
    p = ws.view(torch.float32).view(-1, cop, cv["kh"] * cv["kw"], cip)
    nr = 16 if p.shape[0] >= 64 else 4
    s = [torch.zeros_like(p[0]) for _ in range(nr)]
    for k in range(p.shape[0]):
        s[k % nr] = s[k % nr] + p[k]
    while len(s) > 1:
        s = [s[i] + s[i + 1] for i in range(0, len(s), 2)]
    g = s[0][:cv["cout"], :, :cv["cin"]].permute(0, 2, 1)
    return p.shape[0], g.reshape(cv["cout"], cv["cin"], cv["kh"], cv["kw"])


@pytest.mark.parametrize("fmt", [0, 1], ids=["e4m3", "e2m1"])
def test_reduce_order_and_extent(mx, fmt):
    items, guards, refs, splits = [], [], [], []
    gen = torch.Generator(device=DEV).manual_seed(5)
    for cv in LAYERS:
        need = mx.wgrad_workspace_bytes(cv, fmt)
        if not need:
            continue
        ws = torch.randn(need // 4, generator=gen, device=DEV).view(torch.uint8)
        count = cv["cout"] * cv["cin"] * cv["kh"] * cv["kw"]
        buf = torch.full((count + 64,), 7.0, device=DEV)
        guards.append(buf)
        items.append((cv, fmt, ws, buf[:count].view(cv["cout"], cv["cin"], cv["kh"], cv["kw"])))
        n, r = _reference(ws, cv)
        splits.append(n)
        refs.append(r)
    assert min(splits) < 64 <= max(splits)
    mx.wgrad_reduce_multi(items)
    torch.cuda.synchronize()
    for (cv, _, _, gw), buf, ref in zip(items, guards, refs):
        assert torch.equal(gw, ref)
        assert bool((buf[ref.numel():] == 7.0).all())
    for it, ref in zip(items, refs):                 # each alone: the same bits
        it[3].fill_(0.0)
        mx.wgrad_reduce_multi([it])
    torch.cuda.synchronize()
    for it, ref in zip(items, refs):
        assert torch.equal(it[3], ref)
