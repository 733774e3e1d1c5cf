"""GPU parity of the fold-back where it rides in the input gradient's launch (64 to 512 threads a channel, channels that do not fill a
workgroup; transposed blocks: rows and shared copies, odd numbers of workgroups) and of rows that are no multiple of four elements, as columns of four and of one."""
import pytest

from paper_2305_11624_amd import synth
from paper_2305_11624_amd.runner import BlockRun, TconvRun
from paper_2305_11624_amd.synth import BlockShape

from helpers import compare, oracle_block, oracle_tconv_block, routes

pytestmark = pytest.mark.gpu

SHAPES = [
    #  N  Cin  H   W   Cout k  s  p
    (20, 256, 30, 33, 64, 1, 1, 0, "bf16", "win, gm + fold-back"),     # pointwise product: many copies of short rows
    (24, 64, 41, 40, 192, 1, 1, 0, "bf16", "win, gm + fold-back"),     # sixteen columns a row
    (12, 512, 17, 19, 640, 1, 1, 0, "bf16", "win, gm + fold-back"),    # few copies, 128 columns
    (41, 2048, 6, 6, 512, 1, 1, 0, "bf16", "win, gm + fold-back"),     # long rows: four columns at once on 128 x 128 tiles
    (5, 1024, 20, 17, 256, 1, 1, 0, "bf16", "win, gm + fold-back"),    # ... two on 128 x 64
    (10, 1024, 19, 19, 256, 1, 1, 0, "bf16", "gm, win, fold-back"),    # a launch of its own behind a full round of tiles
    # residue classes; rows longer than a channel's threads, channels that fill no workgroup
    (40, 128, 30, 30, 264, 3, 2, 1, "bf16", "win, win 128x128 + fold-back"),
    (40, 96, 31, 40, 40, 3, 1, 1, "bf16", "win, win 128x128 + fold-back"),
    (30, 128, 28, 17, 136, 3, 2, 1, "bf16", "win, win 128x64 + fold-back"),
    (42, 600, 30, 6, 64, 2, 2, 0, "bf16", "win, win 256x128 + fold-back"),
    (21, 128, 28, 28, 128, 3, 1, 1, "bf16", "sq, st + fold-back"),     # the deep-layer kernel
    (2, 1032, 7, 6, 16, 5, 2, 0, "bf16", "win, ks 32x32 + fold-back"),   # wave-split tiles
    (4, 992, 6, 16, 8, 5, 2, 0, "bf16", "win, ks 64x32 + fold-back"),
    (40, 736, 6, 5, 16, 5, 1, 0, "bf16", "win, ks 64x64 + fold-back"),
    (3, 128, 37, 41, 128, 3, 1, 1, "bf16", "pair win 128x64 win 64x128, fold-back"),   # launches of their own, behind both gradients
    (38, 1024, 9, 9, 2048, 1, 2, 0, "bf16", "pair win 128x64 win 128x128, fold-back"),
    (24, 256, 13, 13, 256, 3, 1, 1, "bf16", "pair win 128x64 win 128x128, fold-back"),
    (9, 3, 24, 24, 32, 3, 2, 1, "bf16", "stem, stem + fold-back"),     # first layers: 27 and 75 elements a row
    (6, 3, 33, 52, 64, 5, 2, 2, "bf16", "stem, stem + fold-back"),
    (1, 3, 8, 8, 32, 1, 1, 0, "bf16", "stem, stem, fold-back"),        # three elements a row
    (4, 3, 40, 40, 16, 3, 1, 1, "f32", "pair wave, fold-back"), (2, 5, 9, 11, 7, 1, 1, 0, "f32", "pair wave, fold-back"),
    (1, 2, 6, 5, 3, 1, 1, 0, "f32", "pair wave, fold-back"),
]


@pytest.mark.parametrize("n,cin,h,w,cout,k,s,p,dtype,route", SHAPES)
def test_parameter_gradients(n, cin, h, w, cout, k, s, p, dtype, route):
    shape = BlockShape("fb", n, cin, h, w, cout, k, s, p, dtype, 3 * h + w)
    assert routes(shape)[1] == route
    inp = synth.make_inputs(shape, bias=True)
    ref = oracle_block(inp)
    for keep in (True, False):
        r = BlockRun(inp, poison=True, keep_folded=keep)
        r.step()
        compare(r.results(), ref, dtype, tag="keep %s" % keep)


@pytest.mark.parametrize("over", ["dz", "w_folded"])
def test_gradient_over_an_operand(over):
    """dW may take the place of what the input gradient reads: it is written behind it then."""
    inp = synth.make_inputs(BlockShape("fb", 20, 256, 30, 33, 64, 1, 1, 0, "bf16", 7))
    ref = oracle_block(inp)
    r = BlockRun(inp, poison=True)
    r.forward()
    r.dW = getattr(r, over).flatten()[:r.dW.numel()].view(r.dW.shape)
    r.backward()
    compare(r.results(), ref, "bf16", keys=("dX", "dW", "dgamma", "dbeta"), tag=over)


TCONV = [
    #  N  Cin  H   W   Cout k  s  p
    (1, 64, 5, 7, 32, 4, 2, 1),       # eight rows a workgroup
    (3, 512, 14, 14, 256, 4, 2, 1),   # thirty-two
    (2, 72, 30, 23, 40, 4, 2, 1),     # the copies shared by the threads of sixteen column groups
    (2, 128, 40, 41, 64, 4, 2, 1),    # ... of sixty-four
    (1, 24, 9, 5, 8, 3, 2, 1),
    (2, 16, 6, 6, 12, 4, 2, 1),       # not a multiple of eight: launches of their own
]


@pytest.mark.parametrize("n,cin,h,w,cout,k,s,p", TCONV)
def test_transposed(n, cin, h, w, cout, k, s, p):
    inp = synth.make_tconv_inputs(BlockShape("fbt", n, cin, h, w, cout, k, s, p, "bf16", h + w), bias=True)
    ref = oracle_tconv_block(inp)
    for keep in (True, False):
        r = TconvRun(inp, poison=True, keep_folded=keep)
        r.step()
        compare(r.results(), ref, "bf16", tag="keep %s" % keep)


@pytest.mark.parametrize("over", ["dz", "w_folded"])
def test_transposed_gradient_over_an_operand(over):
    inp = synth.make_tconv_inputs(BlockShape("fbt", 9, 64, 14, 13, 32, 4, 2, 1, "bf16", 5))
    ref = oracle_tconv_block(inp)
    r = TconvRun(inp, poison=True)
    r.forward()
    r.dW = getattr(r, over).flatten()[:r.dW.numel()].view(r.dW.shape)
    r.backward()
    compare(r.results(), ref, "bf16", keys=("dX", "dW", "dgamma", "dbeta"), tag=over)


@pytest.mark.parametrize("n,cin,h,w,cout,k,s,p", [
    (1, 24, 9, 5, 8, 3, 2, 1),        # rows, 27 workgroups of 256 threads: the last has nothing beside it
    (1, 40, 6, 5, 16, 3, 2, 1),       # ... 45
    (2, 72, 30, 23, 40, 4, 2, 1),     # copies shared
])
def test_transposed_gradient_in_place_of_the_weight(n, cin, h, w, cout, k, s, p):
    """dW may take the place of W: every row is read by the threads that write it, and by no others."""
    inp = synth.make_tconv_inputs(BlockShape("fbt", n, cin, h, w, cout, k, s, p, "bf16", 11))
    ref = oracle_tconv_block(inp)
    for keep in (True, False):
        r = TconvRun(inp, poison=True, keep_folded=keep)
        r.forward()
        r.dW = r.W
        r.backward()
        compare(r.results(), ref, "bf16", keys=("dX", "dW", "dgamma", "dbeta"), tag="keep %s" % keep)
