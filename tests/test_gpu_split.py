"""Backward of bf16 activations with a 5x5 window on the kernels that split float32 operands in 16-bit terms, against the CPU
oracle where their tiling can go wrong: one pixel, one column, one row, planes that share a run of 256 pixels, several
column strips, rows of odd length, heads that are no whole quad or block of 32 channels, more than one block of them, more
column groups than waves, activations at odd addresses, activations far from one.

Tolerances: the rounded gradients 2e-2 of max(1, largest entry) as everywhere; kernel and bias gradients 1e-5 of the
largest entry, what float32 arithmetic gives (the split terms hold all 24 bits)."""
import pytest
import torch

import numpy as np
import paper_2304_04237_amd as sa
from paper_2304_04237_amd import synth
from oracle import slide_oracle as oracle

pytestmark = pytest.mark.gpu

NAMES = "dq dk dv dwk dwv dbias".split()
SHAPES = [
    # B, H, W, C, heads
    (1, 1, 1, 3, 1), (2, 1, 1, 4, 1), (3, 1, 9, 10, 2), (5, 9, 1, 6, 1), (2, 2, 3, 5, 1), (7, 5, 4, 8, 2), (3, 14, 14, 64, 2),
    (2, 28, 28, 32, 1), (9, 30, 37, 32, 1), (1, 19, 61, 33, 1), (1, 7, 130, 40, 1), (2, 31, 45, 64, 1), (1, 13, 60, 24, 1), (40, 6, 11, 8, 1),
]


def _inputs(shape, seed):
    B, H, W, C, heads = shape
    dev = torch.device("cuda:0")
    dd = synth.make_inputs(B, H, W, C, heads, 5, "bf16", seed=seed, with_dout=True)
    acts = [dd[n].to(dev).bfloat16() for n in ("dout", "q", "k", "v")]
    wk, wv = (sa.slide_reparam(dd[n].to(dev)) for n in ("wk_learned", "wv_learned"))
    return acts, wk, wv, dd["bias"].to(dev), [dd[n].to(dev) for n in ("wk_learned", "wv_learned")]


def _odd(t):
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    out = buf[1:].view(t.shape)
    out.copy_(t)
    return out


def _compare(grads, acts, wk, wv, bias, heads, floor=1.0):
    want = oracle.bwd(*[x.double().cpu().numpy() for x in (*acts, wk, wv, bias)], heads, 5)
    for name, got, w in zip(NAMES, grads, want):
        got = got.double().cpu().numpy()
        assert got.shape == w.shape, name
        err, top = float(np.abs(got - w).max()), float(np.abs(w).max())
        bound = 1e-5 * top if name in ("dwk", "dwv", "dbias") else 2e-2 * max(floor, top)
        assert err <= bound, "%s: max abs err %.3e > %.3e" % (name, err, bound)


@pytest.mark.parametrize("shape", SHAPES)
def test_against_oracle(shape):
    heads = shape[4]
    print("split kernels", shape, flush=True)
    acts, wk, wv, bias, learned = _inputs(shape, 300 + sum(shape))
    _compare(sa.slide_attn_bwd(*[_odd(a) for a in acts], wk, wv, bias, heads, 5), acts, wk, wv, bias, heads)
    _compare(sa.slide_attn_bwd_two_branch(*acts, *learned, bias, heads, 5), acts, wk, wv, bias, heads)


@pytest.mark.parametrize("size", [1e-12, 1e10])
def test_gradients_of_any_size(size):
    """dO a power of two away from one: every gradient but da's softmax is linear in it, so the results are the same numbers."""
    shape = (2, 9, 13, 32, 1)
    acts, wk, wv, bias, _ = _inputs(shape, 41)
    factor = 2.0 ** round(np.log2(size))
    plain = sa.slide_attn_bwd(*acts, wk, wv, bias, 1, 5)
    scaled = sa.slide_attn_bwd(acts[0] * factor, *acts[1:], wk, wv, bias, 1, 5)
    for name, a, b in zip(NAMES, plain, scaled):
        assert torch.equal(a.float() * factor, b.float()), name


# An outlier of q and dO whose window of v is zero (no gradient of its logits), one of k and v that only pixels without dO
# see, in one tile: every term with an outlier is zero, and what is left are sums of ordinary numbers.
@pytest.mark.parametrize("power", [10, 14, 18, 24])
def test_ordinary_terms_beside_outliers(power):
    """Kernel gradients, entry by entry: a float32 sum rounds each of its steps by 2^-24 of what it has so far, at most the sum
    of the magnitudes; an entry's value passes at most 25 taps, 32 channels, 25 shifts, 48 pixel steps."""
    H, W, C, r = 4, 28, 32, 2
    acts, wk, wv, bias, _ = _inputs((1, H, W, C, 1), 45)
    dout, q, k, v = acts
    big = 2.0 ** power
    for t, j in ((q, 3), (dout, 3), (k, 20), (v, 20)):
        t[0, :, 1, j] *= big
    v[0, :, :, 1:6] = 0.0
    dout[0, :, :, 18:23] = 0.0
    grads = sa.slide_attn_bwd(*acts, wk, wv, bias, 1, 5)
    d64, q64, k64, v64, wk64, wv64, b64 = (x.double().cpu() for x in (*acts, wk, wv, bias))

    def windows(x):                                                 # [C, S, H * W]
        return torch.nn.functional.unfold(x, 5, padding=r).view(C, 25, H * W)

    kw, vw, qf, df = windows(k64), windows(v64), q64.view(C, -1), d64.view(C, -1)
    flat = lambda w: w.view(C, 25, 25)
    scale = C ** -0.5
    a = torch.softmax(scale * torch.einsum("cp,cst,ctp->sp", qf, flat(wk64), kw) + b64.view(25, 1), 0)
    da = torch.einsum("cp,cst,ctp->sp", df, flat(wv64), vw)
    dl = a * (da - (a * da).sum(0))
    size = a * (da.abs() + (a * da.abs()).sum(0))                   # what dl's own rounding is measured by
    for name, got, p, mag, x, y, f in (("dwk", grads[3], dl, size, qf, kw, scale), ("dwv", grads[4], a, a, df, vw, 1.0)):
        want = f * torch.einsum("sp,cp,ctp->cst", p, x, y)
        bound = f * torch.einsum("sp,cp,ctp->cst", mag, x.abs(), y.abs()) * (25 + 32 + 25 + 48) * 2.0 ** -24
        err = (got.double().cpu().view(C, 25, 25) - want).abs()
        worst = float((err / bound.clamp_min(1e-300)).max())
        print("2^%d %s: worst error / bound %.3g" % (power, name, worst), flush=True)
        assert worst <= 1.0, "%s: %.3g times the bound" % (name, worst)


@pytest.mark.parametrize("shape", [(4, 27, 27, 96, 3), (8, 28, 28, 64, 2), (2, 45, 45, 64, 1)])
def test_kernel_gradients_round_no_more_than_float32_kernels(shape):
    """The same numbers as float32 activations run on the float32 matrix instructions: the split kernels' results may be no further
    from 64 bits than theirs."""
    heads = shape[4]
    acts, wk, wv, bias, _ = _inputs(shape, 47)
    want = oracle.bwd(*[x.double().cpu().numpy() for x in (*acts, wk, wv, bias)], heads, 5)
    error = []
    for x in (acts, [t.float() for t in acts]):
        grads = sa.slide_attn_bwd(*x, wk, wv, bias, heads, 5)
        error.append([float(np.linalg.norm(g.double().cpu().numpy() - w) / np.linalg.norm(w)) for g, w in zip(grads[3:], want[3:])])
    print(shape, "split", ["%.2e" % e for e in error[0]], "float32", ["%.2e" % e for e in error[1]], flush=True)
    for name, split, plain in zip(NAMES[3:], *error):
        assert split <= plain, name


def test_infinite_key_reaches_its_window_only():
    shape = (1, 11, 17, 8, 1)
    acts, wk, wv, bias, _ = _inputs(shape, 42)
    acts[2][0, 3, 5, 8] = float("inf")
    dq, dk, dv = sa.slide_attn_bwd(*acts, wk, wv, bias, 1, 5)[:3]
    for t, reach in ((dq, 2), (dk, 4), (dv, 4)):            # (dk and dv of a pixel see the pixels whose windows it is in)
        bad = ~torch.isfinite(t[0]).all(0).cpu()
        ii, jj = torch.meshgrid(torch.arange(11), torch.arange(17), indexing="ij")
        near = torch.maximum((ii - 5).abs(), (jj - 8).abs()) <= reach
        assert not (bad & ~near).any()
        assert bad[5, 8]


@pytest.mark.parametrize("W", [3, 20, 21, 33])
def test_infinite_value_reaches_no_other_tap(W):
    """An infinite v in the last column: the kernel gradient of a tap that never reads that column stays finite."""
    acts, wk, wv, bias, _ = _inputs((1, 6, W, 8, 1), 43)
    acts[3][:, :, :, -1] = float("inf")
    dwv = sa.slide_attn_bwd(*acts, wk, wv, bias, 1, 5)[4].view(8, 25, 5, 5)
    assert torch.isfinite(dwv[:, :, :, :2]).all()
    assert not torch.isfinite(dwv[:, :, :, 2]).any()


def test_gradients_are_added():
    acts, wk, wv, bias, learned = _inputs((3, 11, 18, 40, 2), 44)
    once = sa.slide_attn_bwd_two_branch(*acts, *learned, bias, 2, 5)
    twice = [torch.full_like(g, 3.0) for g in once]
    sa.slide_attn_bwd_two_branch(*acts, *learned, bias, 2, 5, outputs=twice, accumulate=True)
    for name, a, b in list(zip(NAMES, twice, once))[3:]:
        assert torch.equal(a, b + 3.0), name


def _rounds_once(name, got, want):
    """bf16 results: 2^-9 of each entry, and float32 sums before."""
    got = got.double().cpu().numpy()
    err = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    print(name, "%.2e" % err, flush=True)
    assert err <= 2.0 ** -9 + 1e-5, "%s: %.2e" % (name, err)


@pytest.mark.parametrize("power", [20, 40, 80])
def test_ordinary_weights_beside_large_ones(power):
    """One tap in every channel's kernels is large, at a shift that the bias masks: its terms are zero, the others ordinary."""
    acts, wk, wv, bias, _ = _inputs((2, 9, 13, 32, 1), 48)
    for w in (wk, wv):
        w.view(32, 25, 25)[:, 7, 11] = 2.0 ** power
    bias.view(25)[7] = -1e30
    grads = sa.slide_attn_bwd(*acts, wk, wv, bias, 1, 5)
    want = oracle.bwd(*[x.double().cpu().numpy() for x in (*acts, wk, wv, bias)], 1, 5)
    for i in (0, 1, 2):
        _rounds_once(NAMES[i], grads[i], want[i])


@pytest.mark.parametrize("lead", [10.0, 25.0, 60.0])
def test_small_attention_beside_a_saturated_shift(lead):
    """One shift takes nearly all attention and has no value kernel: dv is made of the others' attention, e^-lead each."""
    acts, wk, wv, bias, _ = _inputs((2, 9, 13, 32, 1), 49)
    for w in (wk, wv):
        w.view(32, 25, 25)[:, 7] = 0.0
    bias.view(25)[7] = lead
    grads = sa.slide_attn_bwd(*acts, wk, wv, bias, 1, 5)
    want = oracle.bwd(*[x.double().cpu().numpy() for x in (*acts, wk, wv, bias)], 1, 5)
    for i in (0, 1, 2):
        _rounds_once(NAMES[i], grads[i], want[i])


@pytest.mark.parametrize("shape", [(1, 1, 1, 3, 1), (40, 28, 28, 8, 1), (8, 45, 45, 8, 1), (30, 30, 37, 40, 2)])
def test_smaller_workspace_runs_on_float32_kernels(shape):
    """What the same sizes need in float32 is enough, as it was before the split kernels; a byte less is refused."""
    B, H, W, C, heads = shape
    acts, wk, wv, bias, _ = _inputs(shape, 50)
    need = sa.slide_attn_workspace_bytes(B, H, W, C, heads, 5, torch.float32, True)
    assert need < sa.slide_attn_workspace_bytes(B, H, W, C, heads, 5, torch.bfloat16, True)
    workspace = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    grads = sa.slide_attn_bwd(*acts, wk, wv, bias, heads, 5, workspace=workspace)
    _compare(grads, acts, wk, wv, bias, heads)
    split = sa.slide_attn_bwd(*acts, wk, wv, bias, heads, 5)
    assert shape[:3] == (1, 1, 1) or not torch.equal(grads[3], split[3])        # (other kernels, other roundings)
    with pytest.raises(sa.SlideAttnError):
        sa.slide_attn_bwd(*acts, wk, wv, bias, heads, 5, workspace=workspace[:-1])
    tokens = [a.permute(0, 2, 3, 1).contiguous() for a in acts]
    need = -need // 256 * -256 + 7 * (-2 * B * C * H * W // 256 * -256)
    workspace = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    again = sa.slide_attn_bwd_nhwc(*tokens, wk, wv, bias, heads, 5, workspace=workspace)
    for name, a, b in zip(NAMES, grads, again):
        assert torch.equal(a, b if b.dim() != 4 or name in ("dwk", "dwv") else b.permute(0, 3, 1, 2)), name
    with pytest.raises(sa.SlideAttnError):
        sa.slide_attn_bwd_nhwc(*tokens, wk, wv, bias, heads, 5, workspace=workspace[:-1])
