"""What is timed when this library's speed is followed from one version to the next.

A case is one pass of a user's program through the public entry points: a ConvBN block in Tune mode, forward and
backward (`runner.BlockRun` and its depthwise, grouped and transposed siblings, which hold the buffers that a training
loop holds), or the forward pass of the chained ResNet-50 backbone.  Gradients are compared block by block: in a chained
bf16 backbone they depend on ReLU decisions that one rounding can turn over, so no two correct versions agree on them.
"""
import torch

from paper_2305_11624_amd import binding as B
from paper_2305_11624_amd.resnet50 import ResNet50
from paper_2305_11624_amd.runner import BlockRun, DepthwiseRun, GroupedRun, TconvRun
from paper_2305_11624_amd.synth import BlockShape, tconv_out

# the activation bits that a bottleneck unit's blocks carry (ReLU behind / in front, residual sum behind / in front)
PLAIN = 0
FIRST = B.ACT_RELU_OUT                                          # first block: its input feeds the shortcut too
MIDDLE = B.ACT_RELU_OUT | B.ACT_RELU_IN
LAST = B.ACT_RELU_IN | B.ACT_ADD_OUT | B.ACT_RELU_OUT           # max(z + shortcut, 0)
ENTRY = B.ACT_RELU_OUT | B.ACT_RELU_IN | B.ACT_ADD_IN           # dx + the shortcut's gradient, masked


def _block(kind, N, Cin, H, W, Cout, k, stride, pad, dtype="bf16", groups=1, bias=False, act=PLAIN, name=None):
    c = dict(kind=kind, N=N, Cin=Cin, H=H, W=W, Cout=Cout, k=k, stride=stride, pad=pad, dtype=dtype, groups=groups,
             bias=bias, act=act)
    return dict(c, name=name) if name else c


def _backbone(N, image, name=None):
    c = dict(kind="backbone", N=N, image=image)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest block in single precision: launches and host work
        _block("block", 2, 16, 16, 16, 32, 3, 1, 1, dtype="f32", name="f32_16"),
        # a 3x3 layer in single precision, the paper's own precision, at a detector's batch
        _block("block", 8, 64, 28, 28, 64, 3, 1, 1, dtype="f32", name="f32_28"),
        # ResNet-50, first stage: the pointwise reduction, bound by memory
        _block("block", 32, 256, 56, 56, 64, 1, 1, 0, name="pointwise_56"),
        # ResNet-50, first stage: many pixels, few channels
        _block("block", 32, 64, 56, 56, 64, 3, 1, 1, name="conv3_56"),
        # ResNet-50, last stage: few pixels, many channels; w' is larger than the output and is not kept
        _block("block", 64, 512, 7, 7, 512, 3, 1, 1, name="conv3_7"),
        # ResNet-50's first layer with the gradient of the images (adversarial examples need it)
        _block("block", 32, 3, 224, 224, 64, 7, 2, 3, name="stem_224"),
        # a small ragged layer with a convolution bias and a ReLU behind it: no size fits a tile
        _block("block", 5, 72, 27, 33, 136, 3, 1, 1, bias=True, act=FIRST, name="ragged_27x33"),
        # a mobile network's depthwise layer
        _block("depthwise", 32, 144, 56, 56, 144, 3, 1, 1, name="depthwise_56"),
        # an aggregated-transform network's grouped layer, 8 channels a group
        _block("grouped", 32, 256, 28, 28, 256, 3, 1, 1, groups=32, name="grouped_28"),
        # an encoder-decoder network's 4x4 / 2 up-sampling
        _block("tconv", 32, 512, 14, 14, 256, 4, 2, 1, name="tconv_14"),
        # all 53 blocks, forward (validation, feature extraction): an ordinary batch, and a large one
        _backbone(32, 224, name="backbone_32"),
        _backbone(128, 224, name="backbone_128"),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _side(rng, side):
    """A feature map's side around `side`: images from about half to twice the usual area, odd ones among them."""
    return max(5, int(round(side * rng.uniform(0.72, 1.45))))


def _layer(rng):
    """A layer of a bottleneck network: any stage, any of the unit's four blocks, any batch up to 64."""
    stage = rng.randrange(4)
    width, side = 64 << stage, _side(rng, 56 >> stage)
    n, ragged = _log(rng, 1, 64), rng.random() < 0.5
    h, w = side, _side(rng, 56 >> stage) if ragged else side
    which = rng.choice(["reduce", "conv3", "conv3", "expand", "down3", "shortcut"])
    if which == "reduce":
        return _block("block", n, 4 * width, h, w, width, 1, 1, 0, act=rng.choice([PLAIN, FIRST, ENTRY]))
    if which == "conv3":
        return _block("block", n, width, h, w, width, 3, 1, 1, act=rng.choice([PLAIN, MIDDLE]))
    if which == "expand":
        return _block("block", n, width, h, w, 4 * width, 1, 1, 0, act=rng.choice([PLAIN, LAST]))
    if which == "down3":
        return _block("block", n, width, h, w, width, 3, 2, 1, act=rng.choice([PLAIN, MIDDLE]))
    return _block("block", n, 2 * width, h, w, 4 * width, 1, 2, 0)


def draw(rng):
    kind = rng.choice(["layer"] * 8 + ["first", "ragged", "ragged", "f32", "f32", "depthwise", "depthwise", "grouped",
                                       "grouped", "tconv", "tconv", "backbone", "backbone"])
    if kind == "layer":
        return _layer(rng)
    if kind == "first":
        side = rng.randrange(96, 289, 4) if rng.random() < 0.7 else rng.randrange(97, 289, 2)
        return _block("block", _log(rng, 1, 32), 3, side, side, rng.choice([32, 64]), *rng.choice([(7, 2, 3), (3, 2, 1)]))
    if kind == "ragged":
        k = rng.choice([1, 3, 3, 5])
        return _block("block", _log(rng, 1, 16), 8 * rng.randrange(2, 33), rng.randrange(7, 50), rng.randrange(7, 50),
                      8 * rng.randrange(2, 33), k, rng.choice([1, 1, 2]), k // 2, bias=rng.random() < 0.5,
                      act=rng.choice([PLAIN, FIRST]))
    if kind == "f32":
        k = rng.choice([1, 3, 3])
        cin, cout, h, w = _log(rng, 8, 96), _log(rng, 8, 96), rng.randrange(7, 33), rng.randrange(7, 33)
        n = max(1, min(8, int(230e6 / (cin * cout * k * k * h * w))))   # at most what the listed layer multiplies
        return _block("block", _log(rng, 1, n), cin, h, w, cout, k, rng.choice([1, 1, 2]), k // 2, dtype="f32",
                      bias=rng.random() < 0.5)
    if kind == "depthwise":
        c, side = rng.choice([(32, 112), (96, 112), (144, 56), (192, 28), (384, 14), (576, 14), (960, 7)])
        return _block("depthwise", _log(rng, 1, 32), c, _side(rng, side), _side(rng, side), c, 3, rng.choice([1, 1, 2]), 1)
    if kind == "grouped":
        stage = rng.randrange(4)
        c, side = 128 << stage, 56 >> stage
        return _block("grouped", _log(rng, 1, 32), c, _side(rng, side), _side(rng, side), c, 3, rng.choice([1, 1, 2]), 1,
                      groups=32)
    if kind == "tconv":
        cin, side = rng.choice([(64, 56), (128, 56), (256, 28), (512, 14)])
        return _block("tconv", _log(rng, 1, 32), cin, _side(rng, side), _side(rng, side), cin // 2,
                      *rng.choice([(2, 2, 0), (4, 2, 1)]))
    image = rng.randrange(64, 449, 8) + rng.choice([0, 0, 1])
    return _backbone(_log(rng, 1, max(1, min(128, int(128 * 224 * 224 / image ** 2)))), image)


def _shape(c):
    return BlockShape("case", c["N"], c["Cin"], c["H"], c["W"], c["Cout"], c["k"], c["stride"], c["pad"], c["dtype"])


class _State:
    pass


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*size):
        return torch.randn(*size, generator=g, device="cuda")

    def uniform(n, lo, hi):
        return torch.rand(n, generator=g, device="cuda") * (hi - lo) + lo

    st = _State()
    st.kind = case["kind"]
    if case["kind"] == "backbone":
        st.net = ResNet50(case["N"], case["image"], mode="tune", group_units=True)
        st.x = normal(case["N"], case["image"], case["image"], 3).to(torch.bfloat16)
        return st
    s = _shape(case)
    groups = case["groups"]
    if case["kind"] == "tconv":
        ho, wo = tconv_out(s)
        w_size, fan_in = (s.Cin, s.Cout, s.k, s.k), s.Cin * s.k * s.k / s.stride ** 2
    else:
        ho, wo = s.Hout, s.Wout
        cg = 1 if case["kind"] == "depthwise" else s.Cin // groups
        w_size, fan_in = (s.Cout, cg, s.k, s.k), cg * s.k * s.k
    x = normal(s.N, s.Cin, s.Hin, s.Win)
    if case["act"] & B.ACT_RELU_IN:   # the input is a ReLU's output
        x = x.clamp_min_(0)
    inp = dict(shape=s, x=x, W=normal(*w_size) * (2.0 / fan_in) ** 0.5, gamma=uniform(s.Cout, 0.5, 1.5),
               beta=normal(s.Cout) * 0.1, rmean=normal(s.Cout) * 0.1, rvar=uniform(s.Cout, 0.5, 2.0),
               dy=normal(s.N, s.Cout, ho, wo), b=normal(s.Cout) * 0.1 if case["bias"] else None, eps=1e-5)
    if case["kind"] == "block":
        dt = torch.bfloat16 if s.dtype == "bf16" else torch.float32
        add_out = normal(s.N, ho, wo, s.Cout).to(dt) if case["act"] & B.ACT_ADD_OUT else None
        add_in = normal(s.N, s.Hin, s.Win, s.Cin).to(dt) if case["act"] & B.ACT_ADD_IN else None
        # w' is kept between the passes unless it is larger than the output
        st.run = BlockRun(inp, keep_folded=s.P <= s.A_z, act=case["act"], add_out=add_out, add_in=add_in)
    elif case["kind"] == "grouped":
        st.run = GroupedRun(dict(inp, groups=groups))
    else:
        st.run = (DepthwiseRun if case["kind"] == "depthwise" else TconvRun)(inp)
    return st


def run(state):
    if state.kind == "backbone":
        return state.net.forward(state.x)
    r = state.run
    r.step()
    return dict(z=r.z, w_folded=r.w_folded, dx=r.dx, dW=r.dW, db=r.db, dgamma=r.dgamma, dbeta=r.dbeta)


def work(case):
    if case["kind"] == "backbone":
        from paper_2305_11624_amd.synth import resnet50_blocks
        shapes = resnet50_blocks(case["N"], case["image"])
        # the images in, the weights in and w' out, every block's output out (backward needs it) and in again
        return {"bytes": 2.0 * (shapes[0].A_x + sum(2 * s.P + 2 * s.A_z for s in shapes)),
                "flops": float(sum(s.fwd_flop for s in shapes))}
    s = _shape(case)
    e = s.elem_bytes
    taps = s.k * s.k
    if case["kind"] == "tconv":
        ho, wo = tconv_out(s)
        z, p, macs = s.N * ho * wo * s.Cout, s.Cin * s.Cout * taps, s.N * s.Hin * s.Win * s.Cin * s.Cout * taps
    else:
        cg = 1 if case["kind"] == "depthwise" else s.Cin // case["groups"]
        z, p, macs = s.A_z, s.Cout * cg * taps, s.A_z * cg * taps
    keep = 1 if case["kind"] != "block" or s.P <= s.A_z else 0
    adds = (z if case["act"] & B.ACT_ADD_OUT else 0) + (s.A_x if case["act"] & B.ACT_ADD_IN else 0)
    # x, dz, w and the addends in; z, dx, dw and the kept w' out; nine vectors
    return {"bytes": float(e * (2 * s.A_x + 2 * z + (2 + keep) * p + adds) + 36 * s.Cout), "flops": 6.0 * macs}


def tolerance(case):
    if case["kind"] == "backbone":
        return {"rel": 2e-2}   # 53 layers, each rounded to bf16
    return {"rel": 1e-5, "max": 1e-3} if case["dtype"] == "f32" else {"rel": 1e-2}
