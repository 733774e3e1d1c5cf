"""GPU parity of the first-layer kernels (at most four input channels): the unrolled 7x7 / stride-2 RGB case at the edges of its
tiles, the general kernels beside it, and a ReLU behind the block."""
import pytest

from paper_2305_11624_amd import binding as B, synth
from paper_2305_11624_amd.runner import BlockRun
from paper_2305_11624_amd.synth import BlockShape

from helpers import compare, oracle_block

pytestmark = pytest.mark.gpu

SHAPES = [
    #  N  Cin  H    W   Cout k  s  p
    (1, 3, 8, 8, 64, 7, 2, 3),        # one tile of a few pixels, fewer tiles than XCDs
    (2, 3, 37, 260, 64, 7, 2, 3),     # two tiles a row, the second of two pixels; an odd number of rows
    (3, 3, 64, 256, 64, 7, 2, 3),     # whole tiles
    (2, 3, 30, 44, 64, 7, 2, 0),      # no padding
    (2, 3, 21, 24, 32, 7, 2, 3),      # one fragment of output channels
    (2, 3, 20, 28, 40, 7, 2, 3),      # a second fragment of 8 channels
    (2, 3, 22, 24, 56, 7, 2, 3),      # ... of 24
    (2, 3, 20, 28, 72, 7, 2, 3),      # three fragments: the input padded to 8 channels
    (2, 3, 18, 36, 104, 7, 2, 3),     # four, the last of 8 channels
    (3, 2, 21, 34, 128, 4, 2, 1),     # ... of a 4-channel copy of the input
    (2, 3, 19, 21, 64, 7, 2, 3),      # rows that are no whole groups of four pixels
    (2, 3, 24, 24, 64, 3, 2, 1),
    (2, 1, 23, 20, 64, 5, 1, 2), (2, 2, 17, 19, 40, 4, 2, 1), (2, 4, 18, 18, 64, 8, 2, 3), (1, 3, 16, 16, 128, 7, 1, 3)]


@pytest.mark.parametrize("n,cin,h,w,cout,k,s,p", SHAPES)
def test_first_layer(n, cin, h, w, cout, k, s, p):
    shape = BlockShape("first", n, cin, h, w, cout, k, s, p, "bf16", h + w + k)
    inp = synth.make_inputs(shape, bias=h % 2 == 0)
    ref = oracle_block(inp)
    keys = ("Z", "dX", "dW", "db", "dgamma", "dbeta", "Wf")
    for keep in (True, False):
        r = BlockRun(inp, poison=True, keep_folded=keep)
        r.step()
        compare(r.results(), ref, "bf16", keys=keys if keep else keys[:-1], tag="keep %s" % keep)
    r = BlockRun(inp, poison=True, act=B.ACT_RELU_OUT)
    r.step()
    compare(r.results(), dict(ref, Z=ref["Z"].clip(min=0)), "bf16", keys=keys, tag="relu")
