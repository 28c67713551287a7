"""The float32 matrix-core kernels (windows of 3 and 5): forward, log of the softmax denominator and
all six gradients against the CPU oracle where their tiling can go wrong: maps of one and two
columns (runs of pixels that touch hundreds of rows), runs that end inside a row, several column
strips with a narrower last one, head sizes that are no multiple of four or of a staged step, both
block shapes (few pixels: channels shared between waves), both layouts, both element types.

Tolerances: float32 1e-5 of the largest entry (the operator's); bfloat16 activations 2e-2 of
max(1, largest entry) for the rounded outputs, and 1e-5 for the kernel and bias gradients, which
stay float32 from exact inputs."""
import numpy as np
import pytest
import torch

import paper_2304_04237_amd as sa
from paper_2304_04237_amd import synth
from oracle import slide_oracle as oracle

pytestmark = pytest.mark.gpu

GRAD_NAMES = "dq dk dv dwk dwv dbias".split()

SHAPES = [
    # B, H, W, C, heads, ksize, dtype, channels-last
    (1, 5, 1, 6, 1, 3, "f32", False), (1, 300, 1, 4, 1, 5, "f32", False), (2, 150, 2, 9, 3, 3, "f32", False),
    (1, 1, 1, 1, 1, 3, "f32", False), (2, 1, 70, 8, 1, 5, "f32", False), (1, 14, 14, 64, 2, 3, "f32", False),
    (1, 9, 125, 40, 1, 3, "f32", False), (1, 9, 121, 20, 1, 5, "f32", True), (2, 13, 63, 33, 1, 3, "f32", False),
    (2, 13, 61, 64, 2, 5, "f32", False), (64, 33, 62, 8, 1, 3, "f32", False), (40, 33, 29, 12, 1, 5, "f32", True),
    (40, 33, 29, 14, 2, 3, "f32", True), (4, 63, 63, 24, 1, 3, "f32", False), (40, 200, 125, 4, 1, 3, "f32", False), (33, 61, 31, 16, 2, 5, "f32", False),
    (40, 30, 27, 24, 2, 5, "bf16", False), (1, 28, 28, 64, 2, 5, "bf16", False), (2, 17, 19, 64, 1, 3, "bf16", True),
    (64, 40, 67, 40, 1, 3, "bf16", False),
]


def _check(name, got, want, tol, floor):
    got = got.detach().double().cpu().numpy()
    assert got.shape == want.shape, name
    err = float(np.abs(got - want).max())
    bound = tol * max(floor, float(np.abs(want).max()))
    assert err <= bound, "%s: max abs err %.3e > %.3e" % (name, err, bound)


@pytest.mark.parametrize("two_branch", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_against_oracle(shape, two_branch):
    B, H, W, C, heads, ks, dtype, last = shape
    print("float32 matrix-core case", shape, two_branch, flush=True)
    if dtype == "f32" or last:      # (the channels-last forward of these shapes follows the rule of float32)
        narrow = ks == 3 and C // heads <= 8 and B * heads * H * W <= 8192
        assert sa.slide_attn_fwd_variant(B, H, W, C, heads, ks, 0) == (10 if narrow else 11)
    if dtype == "f32" or ks == 5:
        assert sa.slide_attn_bwd_variant(B, H, W, C, heads, ks, 0 if dtype == "f32" else 1) == 11
    dev = torch.device("cuda:0")
    dd = synth.make_inputs(B, H, W, C, heads, ks, dtype, seed=300 + H + W + C, with_dout=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    lay = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if last else (lambda t: t)
    back = (lambda t: t.permute(0, 3, 1, 2)) if last else (lambda t: t)
    q, k, v, do = (lay(dd[n].to(dev).to(tdt)) for n in ("q", "k", "v", "dout"))
    bias = dd["bias"].to(dev)
    wk_l, wv_l = dd["wk_learned"].to(dev), dd["wv_learned"].to(dev)
    wk, wv = sa.slide_reparam(wk_l), sa.slide_reparam(wv_l)
    lse = torch.full((B, heads, H, W), float("nan"), dtype=torch.float32, device=dev)
    if last:
        out = sa.slide_attn_fwd_nhwc(q, k, v, wk, wv, bias, heads, ks, lse=lse)
        w = (wk_l, wv_l) if two_branch else (wk, wv)
        grads = sa.slide_attn_bwd_nhwc(do, q, k, v, *w, bias, heads, ks, two_branch=two_branch)
    elif two_branch:
        out = sa.slide_attn_fwd_two_branch(q, k, v, wk_l, wv_l, bias, heads, ks, lse=lse)
        grads = sa.slide_attn_bwd_two_branch(do, q, k, v, wk_l, wv_l, bias, heads, ks)
    else:
        out = sa.slide_attn_fwd(q, k, v, wk, wv, bias, heads, ks, lse=lse)
        grads = sa.slide_attn_bwd(do, q, k, v, wk, wv, bias, heads, ks)
    torch.cuda.synchronize()
    n = {x: dd[x].double().numpy() for x in ("q", "k", "v", "dout", "bias")}
    wkn, wvn = wk.double().cpu().numpy(), wv.double().cpu().numpy()
    ref, ref_lse = oracle.fwd(n["q"], n["k"], n["v"], wkn, wvn, n["bias"], heads, ks, return_lse=True)
    refg = oracle.bwd(n["dout"], n["q"], n["k"], n["v"], wkn, wvn, n["bias"], heads, ks)
    exact = dtype == "f32"
    # planar bf16: window 3 with heads of up to 32 channels, and the forward of window 5 with heads of 32,
    # run on the half-precision kernels
    half = not exact and ks == 3 and not last and C // heads <= 32
    half_fwd = half or (not exact and ks == 5 and not last and C // heads == 32)
    _check("out", back(out), ref, 1e-5 if exact else 2e-2, 0.0 if exact else 1.0)
    _check("lse", lse, ref_lse, 1e-5 if not half_fwd else 2e-2, 1.0)
    for name, got, want in zip(GRAD_NAMES, grads, refg):
        param = name in ("dwk", "dwv", "dbias")
        got = got if param else back(got)
        if exact or (param and not half):
            _check(name, got, want, 1e-5, 0.0)
        else:
            _check(name, got, want, 2e-2, 1.0)


@pytest.mark.parametrize("shape", [(1, 8, 2715, 4, 1, 5, "f32", False), (1, 32, 3600, 4, 1, 3, "f32", False), (1, 40, 3010, 8, 2, 5, "bf16", False)])
def test_strips_of_wide_maps(shape):
    """Widths whose strips of equal width would leave a last one of a few columns."""
    test_against_oracle(shape, False)


@pytest.mark.parametrize("shape", [
    # narrow maps with heads beyond those that the general forward serves; both block forms at the same number of pixels
    (1, 5, 1, 9, 1, 3, "f32", False), (2, 150, 2, 27, 3, 3, "f32", False), (1, 1, 1, 10, 1, 3, "f32", True),
    (1, 63, 63, 32, 8, 3, "f32", False), (1, 61, 63, 80, 8, 3, "f32", True), (1, 31, 33, 80, 8, 3, "bf16", True), (1, 62, 61, 24, 8, 5, "f32", False),
    # the general forward: up to eight channels per head on few pixels
    (1, 31, 33, 64, 8, 3, "f32", True), (2, 15, 13, 12, 4, 3, "bf16", False),
])
def test_narrow_heads_and_maps(shape):
    test_against_oracle(shape, True)


@pytest.mark.parametrize("shape", [(2, 13, 27, 64, 2, 3, "bf16"), (1, 9, 21, 24, 2, 5, "f32"), (40, 33, 29, 16, 1, 3, "f32"), (4, 30, 63, 128, 2, 5, "bf16")])
def test_channels_last_at_any_element(shape):
    """Four channels are loaded and stored at once, at any element's address: tensors one element past an aligned one, NaN
    around the inputs, a pattern around the output that stays."""
    B, H, W, C, heads, ks, dtype = shape
    print("channels last, unaligned", shape, flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    dd = synth.make_inputs(B, H, W, C, heads, ks, dtype, seed=31)

    def placed(t, fill):
        buf = torch.full((t.numel() + 9,), fill, dtype=tdt, device="cuda")
        view = buf[1:1 + t.numel()].view(t.shape)
        view.copy_(t)
        return buf, view
    q, k, v = (placed(dd[n].permute(0, 2, 3, 1).to(tdt), float("nan"))[1] for n in ("q", "k", "v"))
    buf, out = placed(torch.zeros(B, H, W, C), 7.0)
    wk, wv = (sa.slide_reparam(dd[n].cuda()) for n in ("wk_learned", "wv_learned"))
    bias = dd["bias"].cuda()
    sa.slide_attn_fwd_nhwc(q, k, v, wk, wv, bias, heads, ks, out=out)
    aligned = sa.slide_attn_fwd_nhwc(*(x.clone() for x in (q, k, v)), wk, wv, bias, heads, ks)
    torch.cuda.synchronize()
    assert (buf[:1] == 7.0).all() and (buf[1 + out.numel():] == 7.0).all()
    n = {x: dd[x].double().numpy() for x in ("q", "k", "v", "bias")}
    ref = oracle.fwd(n["q"], n["k"], n["v"], wk.double().cpu().numpy(), wv.double().cpu().numpy(), n["bias"], heads, ks)
    _check("out", out.permute(0, 3, 1, 2), ref, 1e-5 if dtype == "f32" else 2e-2, 0.0 if dtype == "f32" else 1.0)
    if W not in range(32, 65, 8):        # (the streaming kernel takes aligned tensors of those widths)
        assert torch.equal(out, aligned)


@pytest.mark.parametrize("ks", [3, 5])
@pytest.mark.parametrize("shape", [(2, 21, 23, 12, 2), (34, 40, 33, 12, 2)])     # both block forms
def test_infinite_values_stay_in_reach(shape, ks):
    """One infinite element of k, v or dO: results of other batch items, of other heads and of pixels that do not see it are
    those without it, bit by bit; kernel gradients of the other head too."""
    B, H, W, C, heads = shape
    print("infinite values", shape, ks, flush=True)
    dd = synth.make_inputs(B, H, W, C, heads, ks, "f32", seed=41, with_dout=True)
    base = {n: dd[n].cuda() for n in ("dout", "q", "k", "v")}
    wk, wv = (sa.slide_reparam(dd[n].cuda()) for n in ("wk_learned", "wv_learned"))
    bias = dd["bias"].cuda()

    def results(a):
        return (sa.slide_attn_fwd(a["q"], a["k"], a["v"], wk, wv, bias, heads, ks),
                *sa.slide_attn_bwd(a["dout"], a["q"], a["k"], a["v"], wk, wv, bias, heads, ks))
    want = results(base)
    i, j, c, reach = 10, 11, 2, 2 * (ks // 2)
    for name in ("k", "v", "dout"):
        acts = {n: t.clone() for n, t in base.items()}
        acts[name][1, c, i, j] = float("inf")
        for what, got, clean in list(zip("out dq dk dv".split(), results(acts), want)):
            touched = torch.zeros_like(got, dtype=torch.bool)
            touched[1, :C // heads, max(0, i - reach):i + reach + 1, max(0, j - reach):j + reach + 1] = True
            assert torch.equal(got[~touched], clean[~touched]), (name, what)
        for what, got, clean in list(zip("dwk dwv".split(), results(acts)[4:6], want[4:6])):
            assert torch.equal(got[C // heads:], clean[C // heads:]), (name, what)
