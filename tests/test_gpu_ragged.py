"""The 3x3 half-precision kernels on maps whose rows are no multiple of 8 pixels (rows start at any even address,
the last 16-byte piece of a row runs into the next one, that of the last row past the tensor's end):
forward, log of the softmax denominator and activation gradients against the CPU oracle.  Rows
shorter than one piece, one and several column tiles with a narrower last one, single rows, tiles
that are no whole passes, more tiles than compute units and fewer, pointers one element past an
aligned address, both forms of the kernels.

Tolerance: 2e-2 of max(1, largest entry), the operator's for bfloat16.  The tensors are followed by
NaN in memory: a value read past a row's end must not reach a result."""
import numpy as np
import pytest
import torch

import paper_2304_04237_amd as sa
from paper_2304_04237_amd import synth
from oracle import slide_oracle as oracle

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, H, W, C, heads
    (1, 1, 9, 32, 1), (2, 5, 7, 32, 1), (1, 14, 14, 64, 2), (2, 28, 28, 64, 2), (1, 33, 63, 32, 1), (3, 9, 65, 64, 2),
    (1, 12, 77, 32, 1), (1, 21, 131, 96, 3), (1, 1, 333, 32, 1), (40, 17, 28, 128, 4), (300, 15, 14, 64, 2), (90, 30, 50, 32, 1),
]


def _placed(t, shift):
    """The same values `shift` elements past an aligned address, NaN before and after them."""
    buf = torch.full((t.numel() + 64,), float("nan"), dtype=t.dtype, device=t.device)
    out = buf[shift:shift + t.numel()].view(t.shape)
    out.copy_(t)
    return out


def _check(name, got, want):
    got = got.detach().double().cpu().numpy()
    err = float(np.abs(got - want).max())
    bound = 2e-2 * max(1.0, float(np.abs(want).max()))
    assert err <= bound, "%s: max abs err %.3e > %.3e" % (name, err, bound)


@pytest.mark.parametrize("shift, two_branch", [(0, False), (0, True), (1, False)])
@pytest.mark.parametrize("shape", SHAPES)
def test_against_oracle(shape, shift, two_branch):
    B, H, W, C, heads = shape
    print("ragged rows", shape, shift, two_branch, flush=True)
    assert sa.slide_attn_fwd_variant(B, H, W, C, heads, 3, 1) == (22 if W >= 8 else 20)
    assert sa.slide_attn_bwd_variant(B, H, W, C, heads, 3, 1, shift == 0) == (11 if shift else 20)
    dev = torch.device("cuda:0")
    dd = synth.make_inputs(B, H, W, C, heads, 3, "bf16", seed=900 + H + W, with_dout=True)
    do, q, k, v = (_placed(dd[n].to(dev).to(torch.bfloat16), shift) for n in ("dout", "q", "k", "v"))
    bias = dd["bias"].to(dev)
    wk_l, wv_l = dd["wk_learned"].to(dev), dd["wv_learned"].to(dev)
    wk, wv = sa.slide_reparam(wk_l), sa.slide_reparam(wv_l)
    # what lies around the output stays as it was
    around = torch.full((q.numel() + 64,), 7.0, dtype=torch.bfloat16, device=dev)
    out = around[shift:shift + q.numel()].view(q.shape)
    lse = torch.full((B, heads, H, W), float("nan"), dtype=torch.float32, device=dev)
    if two_branch:
        sa.slide_attn_fwd_two_branch(q, k, v, wk_l, wv_l, bias, heads, 3, out=out, lse=lse)
        grads = sa.slide_attn_bwd_two_branch(do, q, k, v, wk_l, wv_l, bias, heads, 3)
    else:
        sa.slide_attn_fwd(q, k, v, wk, wv, bias, heads, 3, out=out, lse=lse)
        grads = sa.slide_attn_bwd(do, q, k, v, wk, wv, bias, heads, 3)
    no_lse = (sa.slide_attn_fwd_two_branch(q, k, v, wk_l, wv_l, bias, heads, 3) if two_branch
              else sa.slide_attn_fwd(q, k, v, wk, wv, bias, heads, 3))
    torch.cuda.synchronize()
    assert torch.equal(no_lse, out)
    assert (around[:shift] == 7.0).all() and (around[shift + q.numel():] == 7.0).all()
    n = [x.double().cpu().numpy() for x in (do, q, k, v, wk, wv, bias)]
    ref, ref_lse = oracle.fwd(*n[1:], heads, 3, return_lse=True)
    _check("out", out, ref)
    _check("lse", lse, ref_lse)
    for name, got, want in zip("dq dk dv dwk dwv dbias".split(), grads, oracle.bwd(*n, heads, 3)):
        _check(name, got, want)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("shape", [(1, 1, 1, 32, 1), (1, 2, 2, 32, 1), (3, 4, 4, 64, 2), (1, 1, 15, 32, 1), (1, 1, 17, 64, 2)])
def test_last_pieces_of_tiny_tensors(shape, shift):
    """Most 16-byte pieces of these run past the tensor's end, by up to seven elements."""
    test_against_oracle(shape, shift, False)


@pytest.mark.parametrize("two_branch", [False, True])
@pytest.mark.parametrize("shape", [(2, 15, 14, 64, 2), (3, 9, 65, 64, 2), (1, 21, 131, 96, 3)])
def test_kernels_that_are_not_16_byte_aligned(shape, two_branch):
    """The pipelined kernel loads the kernels 16 bytes at a time; others take one tile per block, here in column tiles of
    even shares."""
    B, H, W, C, heads = shape
    print("ragged rows, unaligned kernels", shape, two_branch, flush=True)
    dd = synth.make_inputs(B, H, W, C, heads, 3, "bf16", seed=950 + W)
    q, k, v = (dd[n].cuda().to(torch.bfloat16) for n in ("q", "k", "v"))
    bias = dd["bias"].cuda()
    merged = [sa.slide_reparam(dd[n].cuda()) for n in ("wk_learned", "wv_learned")]
    given = [dd[n].cuda() for n in ("wk_learned", "wv_learned")] if two_branch else merged
    wk, wv = (_placed(w, 1) for w in given)
    lse = torch.full((B, heads, H, W), float("nan"), dtype=torch.float32, device="cuda")
    fwd = sa.slide_attn_fwd_two_branch if two_branch else sa.slide_attn_fwd
    out = fwd(q, k, v, wk, wv, bias, heads, 3, lse=lse)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.fwd(*(x.double().cpu().numpy() for x in (q, k, v, *merged, bias)), heads, 3, return_lse=True)
    _check("out", out, ref)
    _check("lse", lse, ref_lse)
