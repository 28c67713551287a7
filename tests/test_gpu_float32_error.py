"""Rounding of the float32 path against 64 bits, merged kernels: the matrix-core kernels' results may be no further
from the operator than one float32 multiply-add at a time in the plain order: a channel's window first, channels dealt to
eight sums that are added in pairs, one sum over the shifts.  The plain order is computed here in numpy for sampled pixels (a
float32 multiply-add is a float64 one rounded once more), so the bound is a count of the roundings and no guess; 4 % on top
for the device's expf, which the model rounds correctly."""
import numpy as np
import pytest
import torch

import paper_2304_04237_amd as sa
from paper_2304_04237_amd import synth
from oracle import slide_oracle as oracle

pytestmark = pytest.mark.gpu

f32, f64 = np.float32, np.float64


def _fma(a, b, c):
    return (a.astype(f64) * b.astype(f64) + c.astype(f64)).astype(f32)


def _windows(x, ks, where):
    """[n, C, S] window of every sampled pixel (b, i, j)."""
    r = ks // 2
    padded = np.pad(x, ((0, 0), (0, 0), (r, r), (r, r)))
    b, i, j = where.T
    return np.stack([padded[b, :, i + p, j + t] for p in range(ks) for t in range(ks)], axis=2)


def _shifted32(w, win):
    """sum over taps of w[c,s,t] win[n,c,t], float32, tap by tap."""
    acc = np.zeros(win.shape, f32)
    for t in range(win.shape[2]):
        acc = _fma(np.broadcast_to(w[None, :, :, t], acc.shape), np.broadcast_to(win[:, :, t:t + 1], acc.shape), acc)
    return acc


def _plain_order32(q, kw, vw, wk, wv, bias, heads):
    n, C, S = kw.shape
    d = C // heads
    ks = _shifted32(wk, kw).reshape(n, heads, d, S)
    qh = np.broadcast_to(q.reshape(n, heads, d, 1), ks.shape)
    lanes = [np.zeros((n, heads, S), f32) for _ in range(8)]
    for c in range(d):
        lanes[c % 8] = _fma(qh[:, :, c], ks[:, :, c], lanes[c % 8])
    while len(lanes) > 1:
        lanes = [lanes[e] + lanes[e + 1] for e in range(0, len(lanes), 2)]
    scale = f32(1) / np.sqrt(f32(d))
    logit = _fma(np.full_like(lanes[0], scale), lanes[0], np.broadcast_to(bias, lanes[0].shape))
    e = np.exp((logit - logit.max(axis=2, keepdims=True)).astype(f64)).astype(f32)
    den = np.zeros(e.shape[:2], f32)
    for s in range(S):
        den = den + e[:, :, s]
    a = e * (f32(1) / den)[:, :, None]
    vs = _shifted32(wv, vw).reshape(n, heads, d, S)
    out = np.zeros((n, heads, d), f32)
    for s in range(S):
        out = _fma(np.broadcast_to(a[:, :, None, s], out.shape), vs[:, :, :, s], out)
    return out.reshape(n, C)


def _exact(q, kw, vw, wk, wv, bias, heads):
    n, C, S = kw.shape
    d = C // heads
    ks = np.einsum("cst,nct->ncs", wk, kw)
    vs = np.einsum("cst,nct->ncs", wv, vw)
    logit = (q[:, :, None] * ks).reshape(n, heads, d, S).sum(2) / np.sqrt(d) + bias
    a = np.exp(logit - logit.max(axis=2, keepdims=True))
    a /= a.sum(axis=2, keepdims=True)
    return (a[:, :, None] * vs.reshape(n, heads, d, S)).sum(3).reshape(n, C)


# (blocks of 256 pixels and of 64 whose channels the waves share; heads of one and of several groups of four quads)
@pytest.mark.parametrize("shape", [(64, 32, 32, 64, 2, 3), (128, 32, 32, 64, 1, 3), (64, 32, 32, 64, 2, 5), (4, 32, 32, 64, 2, 3), (4, 32, 32, 128, 1, 5)])
def test_forward_rounds_no_more_than_the_plain_order(shape):
    B, H, W, C, heads, ks = shape
    print("float32 error", shape, flush=True)
    g = torch.Generator().manual_seed(11)
    q, k, v = (torch.randn((B, C, H, W), generator=g) for _ in range(3))
    S = ks * ks
    eye = torch.eye(S).view(1, S, ks, ks)
    wk, wv = (torch.randn((C, S, ks, ks), generator=g) * synth.KERNEL_STD + eye for _ in range(2))
    bias = torch.randn((heads, S), generator=g) * synth.BIAS_STD
    out = sa.slide_attn_fwd(*(x.cuda() for x in (q, k, v, wk, wv, bias)), heads, ks).cpu().numpy()
    rng = np.random.default_rng(5)
    where = np.stack([rng.integers(0, m, 1500) for m in (B, H, W)], axis=1)
    b, i, j = where.T
    qs = q.numpy()[b, :, i, j]
    kw, vw = (_windows(x.numpy(), ks, where) for x in (k, v))
    w32 = [x.numpy().reshape(C, S, S) for x in (wk, wv)]
    exact = _exact(qs.astype(f64), kw.astype(f64), vw.astype(f64), *(w.astype(f64) for w in w32), bias.numpy().astype(f64), heads)
    plain = _plain_order32(qs, kw, vw, *w32, bias.numpy(), heads)
    error = [np.linalg.norm(x - exact) / np.linalg.norm(exact) for x in (out[b, :, i, j], plain)]
    assert error[0] <= 1.04 * error[1], "%.3e, plain order %.3e" % tuple(error)
    print("%.3e, plain order %.3e" % tuple(error))


@pytest.mark.parametrize("shape", [(32, 28, 28, 128, 32, 3), (16, 28, 28, 64, 16, 5), (1, 31, 30, 8, 2, 5)])
def test_kernel_gradients_are_no_long_running_sums(shape):
    """Many heads, so that few blocks share a head's pixels and each sums thousands of them.  A running sum of n terms of
    either sign rounds like n / 2 roundings of its result, each 0.41 * 2^-24 of it (root mean square).  Groups of at
    most 64 pixels, their totals, the walkers and the chunks come to no more than 60 such roundings; the terms bring the
    error of a and dl with them, which dv and dk show.  One running sum per walker: 196 roundings here."""
    B, H, W, C, heads, ks = shape
    print("float32 kernel gradients", shape, flush=True)
    dd = synth.make_inputs(B, H, W, C, heads, ks, "f32", seed=21, with_dout=True)
    wk, wv = (sa.slide_reparam(dd[n].cuda()) for n in ("wk_learned", "wv_learned"))
    acts = [dd[n].cuda() for n in ("dout", "q", "k", "v")]
    bias = dd["bias"].cuda()
    grads = sa.slide_attn_bwd(*acts, wk, wv, bias, heads, ks)
    ref = oracle.bwd(*(x.double().cpu().numpy() for x in (*acts, wk, wv, bias)), heads, ks)
    dq, dk, dv, dwk, dwv, dbias = (float(np.linalg.norm(g.double().cpu().numpy() - r) / np.linalg.norm(r)) for g, r in zip(grads, ref))
    print("dk %.2e dv %.2e dwk %.2e dwv %.2e dbias %.2e" % (dk, dv, dwk, dwv, dbias))
    chain = 60 ** 0.5 * 0.41 * 2.0 ** -24
    assert dwk <= np.hypot(dk, chain)
    assert dwv <= np.hypot(dv, chain)
