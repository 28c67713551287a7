"""Channels-last backward on the streaming kernels, which read and write [B, H, W, C] themselves: the same bits as the planar
backward on permuted tensors, on every width that they take (blocks of 16 pixels that are whole, half and empty), bands
of one row to many, one to three heads; pointers off a 16-byte boundary still take the layout changes and the tiles."""
import pytest
import torch

import paper_2304_04237_amd as sa
from paper_2304_04237_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [  # B, H, W, C, heads (the last does not fit the dk/dv ring and takes the layout changes)
    (64, 32, 32, 64, 2), (1, 12, 40, 64, 2), (3, 28, 48, 96, 3), (1, 56, 56, 64, 2), (5, 7, 56, 32, 1), (70, 5, 40, 64, 2), (2, 9, 32, 32, 1),
]


@pytest.mark.parametrize("two_branch", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_same_bits_as_planar(shape, two_branch):
    B, H, W, C, heads = shape
    print("channels-last backward", shape, two_branch, flush=True)
    assert sa.slide_attn_bwd_variant(B, H, W, C, heads, 3, torch.bfloat16) == (26 if shape == SHAPES[-1] else 27)
    dev = torch.device("cuda:0")
    d = synth.make_inputs(B, H, W, C, heads, 3, "bf16", seed=61, with_dout=True)
    acts = [d[n].to(dev).bfloat16() for n in ("dout", "q", "k", "v")]
    w = [d[n].to(dev) for n in ("wk_learned", "wv_learned")]
    if not two_branch:
        w = [sa.slide_reparam(x) for x in w]
    bias = d["bias"].to(dev)
    back = sa.slide_attn_bwd_two_branch if two_branch else sa.slide_attn_bwd
    want = back(*acts, *w, bias, heads, 3)
    tokens = [a.permute(0, 2, 3, 1).contiguous() for a in acts]
    got = sa.slide_attn_bwd_nhwc(*tokens, *w, bias, heads, 3, two_branch=two_branch)
    for name, a, b in zip("dq dk dv dwk dwv dbias".split(), got, want):
        assert torch.equal(a, b.permute(0, 2, 3, 1) if name in ("dq", "dk", "dv") else b), name
    odd = []
    for t in tokens:
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=dev)
        odd.append(buf[1:].view(t.shape).copy_(t))
    again = sa.slide_attn_bwd_nhwc(*odd, *w, bias, heads, 3, two_branch=two_branch)
    for name, a, b in zip("dq dk dv dwk dwv dbias".split(), again, got):    # (copies are aligned: the same kernels, planar)
        assert torch.equal(a, b), name
