"""GPU parity of the wave-split product (conv_ks_impl.h) and of the launches it shares with the weight gradient: the three tile sizes,
pixels and channels that end inside a tile, fewer, as many and more chunks than waves, several taps in a chunk, chunks that span taps,
residue classes with and without taps, the post-operations and the fold on the side."""
import numpy as np
import pytest
import torch

from paper_2305_11624_amd import binding as B
from paper_2305_11624_amd import synth
from paper_2305_11624_amd.runner import BlockRun
from paper_2305_11624_amd.synth import BlockShape

from helpers import compare, oracle_block, routes

pytestmark = pytest.mark.gpu

SHAPES = [
    #  N  Cin  H   W   Cout k  s  p
    (1, 8, 1, 1, 8, 1, 1, 0),          # one pixel, one granule
    (1, 64, 5, 7, 40, 1, 1, 0),        # one chunk: one wave has work
    (2, 448, 5, 3, 72, 1, 1, 0),       # seven, eight and nine chunks
    (2, 512, 4, 4, 32, 1, 1, 0),
    (1, 576, 8, 4, 33 * 8, 1, 1, 0),
    (1, 24, 9, 7, 104, 3, 1, 1),       # chunks that span taps, a tap's channels in three granules
    (3, 136, 11, 13, 56, 3, 1, 1),
    (2, 16, 13, 9, 200, 5, 1, 2),      # four taps a chunk
    (5, 512, 7, 7, 512, 3, 1, 1),      # 32 x 32 tiles, 72 chunks
    (20, 512, 7, 7, 512, 3, 1, 1),     # 64 x 32
    (6, 256, 19, 17, 256, 3, 1, 1),    # ... ragged; both gradients on 128 x 64 tiles
    (5, 72, 27, 33, 136, 3, 1, 1),     # 64 x 64 tiles, ragged both ways; both gradients too
    (12, 256, 14, 16, 256, 3, 1, 1),   # ... the last tile's pixels ragged
    (45, 376, 5, 37, 40, 1, 1, 0),     # ... six chunks, the last not full
    (40, 736, 6, 5, 16, 5, 1, 0),      # ... in the input gradient, with a fold-back on the side
    (7, 1024, 15, 15, 256, 1, 1, 0),
    (3, 512, 9, 7, 512, 3, 2, 1),      # four residue classes
    (2, 64, 11, 14, 96, 1, 2, 0),      # three of them without a tap
    (4, 40, 12, 10, 48, 4, 2, 1),
    (2, 32, 16, 17, 48, 2, 3, 0),      # nine: not one launch
    (4, 128, 23, 21, 128, 3, 2, 0),
]


@pytest.mark.parametrize("keep", [True, False], ids=["keeps_w", "keeps_nothing"])
@pytest.mark.parametrize("n,cin,h,w,cout,k,s,p", SHAPES)
def test_block(n, cin, h, w, cout, k, s, p, keep):
    inp = synth.make_inputs(BlockShape("ks", n, cin, h, w, cout, k, s, p, "bf16", n + 5 * h + w), bias=True)
    inp["x"] = torch.clamp(inp["x"], min=0)
    ref = oracle_block(inp)
    r = BlockRun(inp, keep_folded=keep, poison=True, act=B.ACT_RELU_OUT | B.ACT_RELU_IN)
    r.step()
    ref["Z"] = np.maximum(ref["Z"], 0)
    ref["dX"] = ref["dX"] * (inp["x"].double().numpy() > 0)
    compare(r.results(), ref, "bf16", tag="keep %s" % keep)
    if keep:   # w' = bf16(float(W) s), whichever launch folds
        wf = torch.empty_like(r.w_folded)
        B.convbn_fold(r.desc, r.W, r.b, r.gamma, r.beta, r.mean, r.var, None, wf, None)
        torch.cuda.synchronize()
        assert torch.equal(wf, r.w_folded)


@pytest.mark.parametrize("dims,fwd,bwd", [
    ((1, 64, 5, 7, 40, 1, 1, 0), "ks 32x32", "pair ks 32x32"), ((20, 512, 7, 7, 512, 3, 1, 1), "ks 64x32", "fused, ks 64x32"),
    ((5, 512, 7, 7, 512, 3, 1, 1), "ks 32x32", "pair ks 64x32"), ((5, 72, 27, 33, 136, 3, 1, 1), "ks 64x64", "pair ks 64x64"),
    ((12, 256, 14, 16, 256, 3, 1, 1), "ks 64x64", "pair win 128x64"), ((45, 376, 5, 37, 40, 1, 1, 0), "ks 64x64", "win, win 128x128"),
    ((40, 736, 6, 5, 16, 5, 1, 0), "ks 32x32", "win, ks 64x64 + fold-back"), ((2, 32, 16, 17, 48, 2, 3, 0), "ks 32x32", "win, ks 32x32 + fold-back"),
])
def test_shapes_reach_what_they_are_for(dims, fwd, bwd):
    assert dims in SHAPES
    f, b = routes(BlockShape("ks", *dims, "bf16", 1))
    assert f == fwd and b.startswith(bwd)


@pytest.mark.parametrize("n,cin,h,w,cout,k,s,p", [(3, 136, 11, 13, 56, 3, 1, 1), (2, 64, 11, 14, 96, 1, 2, 0)])
def test_addends(n, cin, h, w, cout, k, s, p):
    shape = BlockShape("ks", n, cin, h, w, cout, k, s, p, "bf16", 3)
    inp = synth.make_inputs(shape)
    g = torch.Generator().manual_seed(5)
    add_in = torch.randn((n, h, w, cin), generator=g).bfloat16().cuda()
    add_out = torch.randn((n, shape.Hout, shape.Wout, cout), generator=g).bfloat16().cuda()
    r = BlockRun(inp, poison=True, act=B.ACT_ADD_IN | B.ACT_ADD_OUT, add_in=add_in, add_out=add_out)
    r.step()
    plain = BlockRun(inp, poison=True)
    plain.step()
    B.convbn_aux_eltwise(B.OP_ADD, plain.dx, add_in)
    B.convbn_aux_eltwise(B.OP_ADD, plain.z, add_out)
    torch.cuda.synchronize()
    assert torch.equal(r.dx, plain.dx) and torch.equal(r.z, plain.z)
