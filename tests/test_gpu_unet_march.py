"""The 3x3x3 convolution at the edges of its work split: the z march of up to
32 input channels (columns of 16 x 16 or 16 x 8 voxels, marches of 2 to 32
planes) and the output-channel split of the others, against the FP64 oracle;
the fused ends of the network against the calls that they stand for, bit for
bit."""
import ctypes

import numpy as np
import pytest

import synth
from oracle import unet as U
from test_gpu_unet import P, _bf, _bf16_close, _lib, _np, _p, _rel, _s  # noqa: F401 (P: fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _conv(L, n, d, h, w, x0, c0, x1, c1, wt, b, cout):
    out = torch.full((n, d, h, w, cout), float("nan"), dtype=torch.bfloat16, device="cuda")
    L.check(L.lib().ctmi_conv3d_bf16_fwd(n, d, h, w, _p(x0), c0, x0.shape[-1], _p(x1), c1, x1.shape[-1] if c1 else 8,
                                         _p(wt), _p(b), cout, 1, _p(out), cout, _s()))
    return out


# one voxel, one march and one more plane, columns cut in x and y, both tensors of
# a concatenation, rows wider than their channels; from 48 channels on the tiles
@pytest.mark.parametrize("n,d,h,w,c0,ld0,c1,cout", [
    (1, 1, 1, 1, 16, 16, 0, 16),
    (2, 3, 16, 16, 16, 16, 0, 32),
    (1, 5, 17, 15, 16, 40, 0, 16),
    (1, 2, 9, 17, 16, 24, 16, 16),
    (1, 4, 8, 33, 32, 32, 0, 64),
    (3, 1, 7, 16, 32, 48, 0, 128),
    (1, 3, 9, 17, 48, 48, 0, 32),
    (2, 2, 8, 16, 32, 32, 32, 64),
])
def test_conv3_split_edges(P, n, d, h, w, c0, ld0, c1, cout):  # noqa: F811
    L = _lib()
    x0 = synth.bf16_values((n, d, h, w, c0), 11)
    x1 = synth.bf16_values((n, d, h, w, c1), 12) if c1 else None
    wt = synth.bf16_values((cout, 27, c0 + c1), 13, -0.2, 0.2)
    b = synth.bf16_values((cout,), 14, -0.5, 0.5)
    wide = np.full((n, d, h, w, ld0), 1e30, np.float32)
    wide[..., :c0] = x0
    got = _conv(L, n, d, h, w, _bf(wide), c0, _bf(x1) if c1 else None, c1, _bf(wt), torch.from_numpy(b).cuda(), cout)
    want = np.maximum(U.conv3(np.concatenate([x0, x1], -1) if c1 else x0, wt, b), 0.0)
    assert not np.isnan(_np(got)).any()
    _bf16_close(_np(got), want)


@pytest.mark.parametrize("cin,cout", [(16, 16), (16, 32), (32, 16), (32, 32)])
def test_march_length_does_not_matter(P, cin, cout):  # noqa: F811
    """A volume that is marched in the longest pieces and thin slabs of it give
    the same bits (every output is the same sum, whatever the split)."""
    L = _lib()
    d, h, w = 67, 264, 528
    g = torch.Generator(device="cuda").manual_seed(15)
    x = torch.randn((1, d, h, w, cin), generator=g, device="cuda").to(torch.bfloat16)
    wt = (0.1 * torch.randn((cout, 27, cin), generator=g, device="cuda")).to(torch.bfloat16)
    b = torch.randn(cout, generator=g, device="cuda")
    full = _conv(L, 1, d, h, w, x, cin, None, 0, wt, b, cout)
    for z0, z1 in ((0, 5), (29, 36), (61, d)):
        slab = _conv(L, 1, z1 - z0, h, w, x[:, z0:z1].contiguous(), cin, None, 0, wt, b, cout)
        lo, hi = (0 if z0 == 0 else 1), (z1 - z0 if z1 == d else z1 - z0 - 1)
        assert torch.equal(slab[:, lo:hi].view(torch.int16), full[:, z0 + lo:z0 + hi].view(torch.int16))


@pytest.mark.parametrize("n,d,h,w", [(1, 1, 1, 1), (1, 3, 5, 7), (2, 33, 18, 50), (1, 34, 16, 16), (4, 64, 64, 64)])
def test_fused_ends_are_the_separate_calls(P, n, d, h, w):  # noqa: F811
    L = _lib()
    g = torch.Generator(device="cuda").manual_seed(16)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    x, b, hb = rnd(n, d, h, w), rnd(16), rnd(1)
    w1, w2, hw = (0.2 * rnd(16, 27, 16)).to(torch.bfloat16), (0.1 * rnd(16, 27, 16)).to(torch.bfloat16), rnd(16).to(torch.bfloat16)
    x16 = torch.empty((n, d, h, w, 16), dtype=torch.bfloat16, device="cuda")
    L.check(L.lib().ctmi_unet_pack_input(_p(x), x.numel(), _p(x16), _s()))
    a = _conv(L, n, d, h, w, x16, 16, None, 0, w1, b, 16)
    a2 = torch.full_like(a, float("nan"))
    L.check(L.lib().ctmi_unet_conv_first(n, d, h, w, _p(x), _p(w1), _p(b), 1, _p(a2), 16, _s()))
    assert torch.equal(a.view(torch.int16), a2.view(torch.int16))
    last = _conv(L, n, d, h, w, a, 16, None, 0, w2, b, 16)
    want, got = torch.empty_like(x), torch.full_like(x, float("nan"))
    L.check(L.lib().ctmi_unet_head(x.numel(), _p(x), _p(last), 16, 16, _p(hw), _p(hb), _p(want), _s()))
    L.check(L.lib().ctmi_unet_conv_head(n, d, h, w, _p(a), 16, _p(w2), _p(b), 1, _p(x), _p(hw), _p(hb), _p(got), _s()))
    assert torch.equal(got, want)


def test_forward_with_and_without_the_cache(P):  # noqa: F811
    """The inference path (fused ends) and the training forward give the same bits."""
    net = P.UNet(seed=3)
    x = torch.randn((2, 16, 24, 32), device="cuda", generator=torch.Generator(device="cuda").manual_seed(17))
    out = net.forward(x)
    kept = net.forward(x, keep=True)
    assert torch.equal(out, kept[0] if isinstance(kept, tuple) else kept)


# one voxel; one tile; a few tiles per split with every axis cut; fewer tiles than
# splits over many channel pairs; rows wider than their channels
@pytest.mark.parametrize("n,d,h,w,cin,ld,cout", [
    (1, 1, 1, 1, 16, 16, 16),
    (1, 2, 8, 16, 16, 24, 32),
    (2, 63, 65, 41, 16, 16, 16),
    (4, 8, 8, 8, 64, 80, 128),
])
def test_conv3_wgrad_split_edges(P, n, d, h, w, cin, ld, cout):  # noqa: F811
    L = _lib()
    x = synth.bf16_values((n, d, h, w, cin), 21)
    dz = synth.bf16_values((n, d, h, w, cout), 22)
    wide = np.full((n, d, h, w, ld), 1e30, np.float32)
    wide[..., :cin] = x
    ws = torch.full((L.lib().ctmi_conv3d_wgrad_workspace_bytes(n, d, h, w, cin, cout) // 4,), float("nan"), device="cuda")
    dw, db = torch.ones((cout, 27, cin), device="cuda"), torch.ones(cout, device="cuda")
    tx, tdz = _bf(wide), _bf(dz)
    wdw, wdb = U.conv3_wgrad(x, dz)
    for acc in (1, 0):
        L.check(L.lib().ctmi_conv3d_bf16_wgrad(n, d, h, w, _p(tx), cin, ld, None, 0, 8, _p(tdz), cout, cout, _p(dw),
                                               _p(db), acc, _p(ws), ws.numel() * 4, _s()))
        assert _rel(dw.cpu().numpy().astype(np.float64) - acc, wdw) < 1e-5
        assert _rel(db.cpu().numpy().astype(np.float64) - acc, wdb) < 1e-5


# one voxel; several rounds of chunks per workgroup with the last one cut; one
# chunk of many channels
@pytest.mark.parametrize("n,d,h,w,cin,cout", [(1, 1, 1, 1, 32, 16), (1, 32, 33, 35, 32, 16), (1, 4, 4, 4, 128, 64)])
def test_up2_wgrad_with_bias(P, n, d, h, w, cin, cout):  # noqa: F811
    L = _lib()
    x = synth.bf16_values((n, d, h, w, cin), 23)
    g = synth.bf16_values((n, 2 * d, 2 * h, 2 * w, cout), 24)
    ws = torch.full((L.lib().ctmi_upsample2_wgrad_workspace_bytes(n, d, h, w, cin, cout) // 4,), float("nan"), device="cuda")
    dw, db = torch.ones((cout, 8, cin), device="cuda"), torch.ones(cout, device="cuda")
    tx, tg = _bf(x), _bf(g)
    wdw, wdb = U.up2_wgrad(x, g)
    for acc in (1, 0):
        L.check(L.lib().ctmi_upsample2_wgrad(n, d, h, w, _p(tx), cin, cin, _p(tg), cout, cout, _p(dw), _p(db), acc,
                                             _p(ws), ws.numel() * 4, _s()))
        assert _rel(dw.cpu().numpy().astype(np.float64) - acc, wdw) < 1e-5
        assert _rel(db.cpu().numpy().astype(np.float64) - acc, wdb) < 1e-5


@pytest.mark.parametrize("nv", [1, 257, 140001])   # 1, 2 and 512 blocks of partial sums
def test_head_loss_sums(P, nv):  # noqa: F811
    L = _lib()
    rng = np.random.Generator(np.random.PCG64(25))
    out, tgt = rng.random(nv).astype(np.float32), rng.random(nv).astype(np.float32)
    act, hw = synth.bf16_values((nv, 16), 26), synth.bf16_values((16,), 27, -0.5, 0.5)
    ws = torch.empty(L.lib().ctmi_unet_head_workspace_bytes() // 8 + 2, dtype=torch.float64, device="cuda")
    sums, dhead = torch.empty(18, dtype=torch.float64, device="cuda"), torch.empty(17, device="cuda")
    dz = torch.empty((nv, 16), dtype=torch.bfloat16, device="cuda")
    tout, ttgt, tact, thw = torch.from_numpy(out).cuda(), torch.from_numpy(tgt).cuda(), _bf(act), _bf(hw)
    L.check(L.lib().ctmi_unet_head_mse_bwd(nv, _p(tout), _p(ttgt), _p(tact), 16, _p(thw), _p(dz), 16, _p(sums),
                                           _p(dhead), _p(ws), ws.numel() * 8, _s()))
    loss, g = U.mse_loss(out.astype(np.float64), tgt)
    s = sums.cpu().numpy()
    assert abs(s[17] / nv - loss) < 1e-6 * loss
    assert _rel(s[:16], g @ act) < 1e-5 and abs(s[16] - g.sum()) < 1e-5 * np.abs(g).sum()
    assert _rel(dhead.cpu().numpy(), s[:17]) < 1e-6


# the up-convolution at both sides of its channel split (fewer than 256 workgroups of
# 64 voxels, or not), forward and data gradient, against the oracle
@pytest.mark.parametrize("n,d,h,w,cin,cout", [(1, 1, 1, 1, 32, 16), (2, 5, 7, 9, 128, 64), (1, 26, 25, 26, 64, 32),
                                              (1, 33, 32, 33, 32, 16), (1, 33, 32, 33, 64, 64), (1, 33, 32, 33, 128, 16)])
def test_up2_split_edges(P, n, d, h, w, cin, cout):  # noqa: F811
    L = _lib()
    lib = L.lib()
    x = synth.bf16_values((n, d, h, w, cin), 31)
    wt = synth.bf16_values((cout, 8, cin), 32, -0.3, 0.3)
    b = synth.bf16_values((cout,), 33, -0.5, 0.5)
    out = torch.full((n, 2 * d, 2 * h, 2 * w, cout), float("nan"), dtype=torch.bfloat16, device="cuda")
    tx, tw, tb = _bf(x), _bf(wt), torch.from_numpy(b).cuda()
    L.check(lib.ctmi_upsample2(n, d, h, w, _p(tx), cin, cin, _p(tw), _p(tb), cout, _p(out), cout, _s()))
    _bf16_close(_np(out), U.up2(x, wt, b))
    gr = synth.bf16_values((n, 2 * d, 2 * h, 2 * w, cout), 34)
    below = synth.bf16_values((n, d, h, w, cin), 35)
    dx = torch.full((n, d, h, w, cin), float("nan"), dtype=torch.bfloat16, device="cuda")
    tg, tbel = _bf(gr), _bf(below)
    L.check(lib.ctmi_upsample2_dgrad(n, d, h, w, _p(tg), cout, cout, _p(tw), cin, _p(tbel), cin, _p(dx), cin, _s()))
    _bf16_close(_np(dx), U.up2_dgrad(gr, wt) * (below > 0))
