"""GPU parity of the fp32 path (reduction split over a workgroup's waves): sizes around the 32 pixel x 32 channel tile,
the 16-channel operand stage (whole, half, channel counts that are not multiples of 4), fewer reduction steps than
waves, strides with residue classes no tap reaches, and pixel slices of the weight gradient with ragged ends."""
import pytest

from paper_2305_11624_amd import synth
from paper_2305_11624_amd.synth import BlockShape

from helpers import compare, oracle_block

pytestmark = pytest.mark.gpu

SHAPES = [
    BlockShape("wave_one_pixel", 1, 4, 1, 1, 4, 1, 1, 0, "f32", 901),            # one step: seven waves have none
    BlockShape("wave_31_pixels", 1, 16, 31, 1, 32, 1, 1, 0, "f32", 902),
    BlockShape("wave_33_pixels_33_channels", 1, 20, 33, 1, 33, 1, 1, 0, "f32", 903),   # 20 = a stage and a half one
    BlockShape("wave_12_28_channels", 3, 12, 9, 10, 28, 3, 1, 1, "f32", 904),    # the last stage of a tap more / less than half full
    BlockShape("wave_odd_channels", 2, 9, 11, 7, 57, 3, 1, 1, "f32", 905),       # element-wise operand loads
    BlockShape("wave_stride2", 3, 40, 15, 14, 24, 3, 2, 1, "f32", 906),
    BlockShape("wave_stride2_1x1", 2, 32, 13, 12, 64, 1, 2, 0, "f32", 907),      # three of four classes have no taps
    BlockShape("wave_stride3_5x5", 2, 8, 17, 16, 12, 5, 3, 2, "f32", 908),       # single-tap groups
    BlockShape("wave_ragged_slices", 5, 96, 13, 17, 96, 3, 1, 1, "f32", 909),    # 1105 pixels
    BlockShape("wave_pad0_wide", 8, 64, 30, 29, 96, 3, 1, 0, "f32", 910),
    BlockShape("wave_stride_beyond_image", 2, 64, 5, 4, 64, 3, 65536, 1, "f32", 911),   # twenty classes of one position, most without a tap
]


@pytest.mark.parametrize("keep", [True, False], ids=["keeps_w", "keeps_nothing"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_fp32_block(shape, keep):
    from paper_2305_11624_amd.runner import BlockRun
    inp = synth.make_inputs(shape, bias=True)
    run = BlockRun(inp, mode="tune", keep_folded=keep, poison=True)
    run.step()
    compare(run.results(), oracle_block(inp), "f32", tag=shape.name)
