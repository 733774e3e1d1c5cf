"""GPU parity of the fp32 path (reduction split over a workgroup's waves): sizes around the 32 pixel x 32 channel tile,
the 16-channel operand stage (whole, half, channel counts that are not multiples of 4), fewer reduction steps than
waves, strides with residue classes no tap reaches, and pixel slices of the weight gradient with ragged ends."""
import pytest
import torch

from paper_2305_11624_amd import binding as B
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


def _taps(s):
    """Per tap (i, j): the output rows and columns that it reaches the image from, and the input's."""
    for i in range(s.k):
        for j in range(s.k):
            def inside(n_in, n_out, t):
                o = [q for q in range(n_out) if 0 <= q * s.stride + t - s.pad < n_in]
                return (slice(o[0], o[-1] + 1), slice(o[0] * s.stride + t - s.pad, o[-1] * s.stride + t - s.pad + 1, s.stride)) if o else None
            h, w = inside(s.Hin, s.Hout, i), inside(s.Win, s.Wout, j)
            if h and w:
                yield (i, j), (h[0], w[0]), (h[1], w[1])


@pytest.mark.parametrize("cin,stride", [(16, 1), (16, 2), (6, 1)])
def test_infinities_reach_no_position_through_the_padding(cin, stride):
    """A tap in the padding takes no part in a sum: an infinite weight or gradient makes exactly those outputs infinite or
    NaN that it does in the definition."""
    s = BlockShape("wave_inf", 2, cin, 11, 10, 40, 3, stride, 1, "f32", 912)
    g = torch.Generator().manual_seed(s.seed)
    x, w = torch.randn(2, 11, 10, cin, generator=g).double(), torch.randn(40, 3, 3, cin, generator=g).double()
    dz = torch.randn(2, s.Hout, s.Wout, 40, generator=g).double()
    w[3, 0, 0, 1] = w[37, 2, 1, 2] = float("inf")
    w[5, 2, 2, 0] = float("nan")
    dzi = dz.clone()
    dzi[0, 0, 3, 7] = float("inf")
    dzi[1, s.Hout - 1, s.Wout - 1, 33] = -float("inf")
    z, dx, dw = torch.zeros_like(dz), torch.zeros_like(x), torch.zeros_like(w)
    for (i, j), (oh, ow), (ih, iw) in _taps(s):
        z[:, oh, ow] += torch.einsum("nhwc,oc->nhwo", x[:, ih, iw], w[:, i, j])
        dx[:, ih, iw] += torch.einsum("nhwo,oc->nhwc", dz[:, oh, ow], w[:, i, j])
        dw[:, i, j] += torch.einsum("nhwo,nhwc->oc", dzi[:, oh, ow], x[:, ih, iw])
    d = B.desc_from_shape(s)
    dev = lambda t: t.float().contiguous().cuda()
    gz, gdx = torch.empty(z.shape, device="cuda"), torch.empty(dx.shape, device="cuda")
    part = torch.empty((B.convbn_wgrad_parts(d),) + tuple(w.shape), device="cuda")
    r = torch.empty((B.convbn_rsum_parts(d), 40), device="cuda")
    B.convbn_conv_fprop(d, dev(x), dev(w), None, gz)
    B.convbn_conv_dgrad(d, dev(dz), dev(w.permute(3, 1, 2, 0)), gdx)
    B.convbn_conv_wgrad(d, dev(x), dev(dzi), part, r)
    torch.cuda.synchronize()
    for name, got, want in (("z", gz, z), ("dx", gdx, dx), ("dw", part.double().sum(0), dw)):
        got = got.double().cpu()
        assert not want.isfinite().all() and torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf()), name
        ok = want.isfinite()
        assert (got[ok] - want[ok]).abs().max() <= 1e-4 * want[ok].abs().max(), name
