"""GPU parity of the window product and the window weight gradient (conv_win.hip, wgrad_win.hip, and both as one launch): channel counts that end inside a 64-channel chunk or a channel tile,
one and several taps per chunk, pixel tails, few chunks against the depth of its ring, pixel slices, residue classes of a strided input
gradient with few or no taps (and more than four of them), the post-operations on positions no tap reaches, and the
fold on the side of forward launches (also of the pointwise product)."""
import numpy as np
import pytest
import torch

from paper_2305_11624_amd import binding as B
from paper_2305_11624_amd import synth
from paper_2305_11624_amd.synth import BlockShape

from helpers import compare, oracle_block, routes

pytestmark = pytest.mark.gpu

SHAPES = [
    BlockShape("win_8_channels", 2, 8, 5, 7, 8, 3, 1, 1, "bf16", 921),                # eight taps in a chunk
    BlockShape("win_one_chunk", 3, 24, 9, 5, 72, 1, 1, 0, "bf16", 922),               # one chunk
    BlockShape("win_72_136", 2, 72, 17, 19, 136, 3, 1, 1, "bf16", 923),
    BlockShape("win_200_56_5x5", 1, 200, 11, 13, 56, 5, 1, 2, "bf16", 924),
    BlockShape("win_many_tiles_ragged", 24, 40, 33, 31, 232, 3, 1, 1, "bf16", 925),   # 128 x 128 tiles
    BlockShape("win_stride2_64", 5, 64, 23, 18, 64, 3, 2, 1, "bf16", 926),
    BlockShape("win_stride2_512", 9, 512, 14, 13, 512, 3, 2, 1, "bf16", 927),         # weight larger than the activations
    BlockShape("win_stride2_1x1", 4, 192, 13, 15, 320, 1, 2, 0, "bf16", 928),         # three classes without a tap
    BlockShape("win_stride3_2x2", 2, 32, 16, 17, 48, 2, 3, 0, "bf16", 929),           # nine classes, five without a tap
    BlockShape("win_stride2_wide", 40, 128, 30, 30, 256, 3, 2, 1, "bf16", 930),       # 128-pixel tiles of 64 (forward) and 128 channels
    BlockShape("win_stride2_256", 90, 128, 30, 30, 256, 3, 2, 1, "bf16", 944),        # 256-pixel tiles (from 160 on: 80 x 2, and 4 x 80), the last ragged
    BlockShape("win_small_1x1", 2, 256, 9, 11, 1024, 1, 1, 0, "bf16", 931),
    BlockShape("gm_fold_aside", 7, 128, 28, 28, 512, 1, 1, 0, "bf16", 932),           # pointwise product, folds on the side
    BlockShape("gm_long_runs", 40, 256, 30, 33, 192, 1, 1, 0, "bf16", 933),
    BlockShape("gm_two_stages_3_chunks", 21, 192, 31, 33, 256, 1, 1, 0, "bf16", 941),
    BlockShape("gm_two_stages_4_chunks", 9, 256, 24, 25, 1024, 1, 1, 0, "bf16", 942),
    BlockShape("ww_one_pixel", 1, 8, 1, 1, 16, 1, 1, 0, "bf16", 934),
    BlockShape("ww_64_64_tile", 3, 64, 13, 10, 64, 1, 1, 0, "bf16", 935),             # 390 pixels: four slices, the last ragged
    BlockShape("ww_128_64_tile", 2, 56, 9, 15, 120, 1, 1, 0, "bf16", 936),
    BlockShape("ww_64_128_tile", 2, 24, 16, 8, 48, 3, 1, 1, "bf16", 937),
    BlockShape("ww_alone", 30, 136, 29, 31, 264, 1, 1, 0, "bf16", 938),               # too many workgroups for one launch of both
    BlockShape("ww_alone_5x5", 12, 96, 27, 26, 72, 5, 2, 2, "bf16", 939),
    BlockShape("pair_3x3_256", 3, 256, 13, 14, 256, 3, 1, 1, "bf16", 940),
    # the product's own tiles (the shapes above that have few pixels are wave-split): whole chunks of a tap and chunks across taps, rings of
    # three, four and six, one chunk and less, ragged pixels and channels
    BlockShape("win_ring6_flat_one_chunk", 33, 8, 20, 26, 8, 1, 1, 0, "bf16", 945),
    BlockShape("win_ring6_flat", 24, 8, 41, 30, 8, 2, 1, 0, "bf16", 946),             # ... input gradient too
    BlockShape("win_ring6_one_chunk", 13, 64, 31, 54, 80, 1, 2, 0, "bf16", 947),
    BlockShape("win_ring6", 43, 192, 58, 27, 8, 1, 2, 0, "bf16", 948),
    BlockShape("win_ring3_flat_one_chunk", 39, 8, 15, 57, 8, 1, 1, 0, "bf16", 949),
    BlockShape("win_ring3_flat", 40, 8, 22, 54, 8, 2, 1, 0, "bf16", 950),
    BlockShape("win_ring3_one_chunk", 45, 64, 28, 27, 232, 1, 2, 0, "bf16", 951),
    BlockShape("win_ring3", 58, 128, 27, 38, 136, 1, 2, 0, "bf16", 952),              # ... input gradient: three classes without a tap
    BlockShape("win_128_flat", 17, 72, 32, 39, 8, 2, 1, 0, "bf16", 953),              # 128 x 128 tiles: input gradient
    BlockShape("win_128_flat_fwd", 26, 8, 41, 20, 72, 1, 1, 0, "bf16", 954),
    BlockShape("win_128", 45, 72, 19, 38, 64, 2, 2, 1, "bf16", 955),
    BlockShape("win_128_one_chunk_fwd", 45, 64, 30, 43, 208, 1, 2, 0, "bf16", 956),
    BlockShape("win_256", 47, 88, 21, 57, 64, 2, 2, 1, "bf16", 957),
    BlockShape("win_no_tap", 33, 144, 22, 52, 8, 1, 2, 0, "bf16", 958),
    BlockShape("win_stride_beyond_image", 2, 64, 5, 4, 64, 3, 65536, 1, "bf16", 943),   # twenty classes of one position, most without a tap
]
BOTH = B.ACT_RELU_OUT | B.ACT_RELU_IN


@pytest.mark.parametrize("name,fwd,bwd", [
    ("win_many_tiles_ragged", "win 128x128", "win, win 128x64 + fold-back"), ("win_stride2_wide", "win 128x64", "win, win 128x128 + fold-back"),
    ("win_stride2_256", "win 256x128", "win, win 256x128 + fold-back"), ("win_ring6_flat_one_chunk", "win 128x64", "pair"),
    ("win_ring6_flat", "win 128x64", "win, win 128x64 + fold-back"), ("win_ring6_one_chunk", "win 128x64", "pair"),
    ("win_ring6", "win 128x64", "win, win 128x64 + fold-back"), ("win_ring3_flat_one_chunk", "win 128x64", "win, win 128x64 + fold-back"),
    ("win_ring3_flat", "win 128x64", "win, win 128x64 + fold-back"), ("win_ring3_one_chunk", "win 128x64", "pair"),
    ("win_ring3", "win 128x64", "win, win 128x64 + fold-back"), ("win_128_flat", "win 128x64", "win, win 128x128 + fold-back"),
    ("win_128_flat_fwd", "win 128x128", "pair"), ("win_128", "win 128x64", "win, win 128x128 + fold-back"),
    ("win_128_one_chunk_fwd", "win 128x128", "pair"), ("win_256", "ks 64x64", "win, win 256x128 + fold-back"),
    ("win_no_tap", "ks 64x32", "win, win 128x64 + fold-back"),
])
def test_shapes_reach_what_they_are_for(name, fwd, bwd):
    f, b = routes(next(s for s in SHAPES if s.name == name))
    assert f == fwd and b.startswith(bwd)


@pytest.mark.parametrize("keep", [True, False], ids=["keeps_w", "keeps_nothing"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_block(shape, keep):
    from paper_2305_11624_amd.runner import BlockRun
    inp = synth.make_inputs(shape, bias=True)
    inp["x"] = torch.clamp(inp["x"], min=0)
    ref = oracle_block(inp)
    run = BlockRun(inp, mode="tune", keep_folded=keep, poison=True, act=BOTH)
    run.step()
    got = run.results()
    ref["Z"] = np.maximum(ref["Z"], 0)
    ref["dX"] = ref["dX"] * (inp["x"].double().numpy() > 0)
    compare(got, ref, "bf16", tag=shape.name)
    if keep:   # w' = bf16(float(W) s), whichever launch folds
        w = torch.empty_like(run.w_folded)
        B.convbn_fold(run.desc, run.W, run.b, run.gamma, run.beta, run.mean, run.var, None, w, None)
        torch.cuda.synchronize()
        assert torch.equal(w, run.w_folded)


@pytest.mark.parametrize("name", ["win_stride2_1x1", "win_no_tap"])
def test_addend_reaches_positions_no_tap_does(name):
    from paper_2305_11624_amd.runner import BlockRun
    shape = next(s for s in SHAPES if s.name == name)
    inp = synth.make_inputs(shape)
    add = torch.randn((shape.N, shape.Hin, shape.Win, shape.Cin), generator=torch.Generator().manual_seed(5)).bfloat16().cuda()
    run = BlockRun(inp, mode="tune", poison=True, act=B.ACT_ADD_IN, add_in=add)
    run.step()
    plain = BlockRun(inp, mode="tune", poison=True)
    plain.step()
    B.convbn_aux_eltwise(B.OP_ADD, plain.dx, add)
    torch.cuda.synchronize()
    assert torch.equal(run.dx, plain.dx)


@pytest.mark.parametrize("name", ["win_72_136", "win_stride2_wide", "gm_fold_aside", "gm_two_stages_4_chunks"])
def test_forward_rounds_once(name):
    """Z = s (w (*) X) + b' with s and b' in the epilogue: fp32 up to the one rounding to bf16 on the way out, which is at
    most 2^-9 of a value, hence of the 2-norm (1e-5: the fp32 sums).  A product of the rounded w' is further off (2.3e-3)."""
    from paper_2305_11624_amd.runner import BlockRun
    inp = synth.make_inputs(next(s for s in SHAPES if s.name == name), bias=True)
    run = BlockRun(inp, mode="tune", poison=True)
    run.forward()
    ref = oracle_block(inp, need_dx=False)["Z"]
    err = np.linalg.norm(run.results()["Z"].numpy() - ref) / np.linalg.norm(ref)
    assert err <= 2.0 ** -9 + 1e-5, err
