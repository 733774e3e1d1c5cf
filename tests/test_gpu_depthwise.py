"""GPU parity of the depthwise ConvBN block (one filter per channel), Tune mode and the Eval comparison path,
against the fp64 Eval-mode definition of the CPU oracle, through the C ABI."""
import pytest
import torch

from paper_2305_11624_amd import binding as B, synth
from paper_2305_11624_amd.synth import BlockShape

from helpers import compare, oracle_dw_block

pytestmark = pytest.mark.gpu

KEYS = ("Z", "dX", "dW", "db", "dgamma", "dbeta", "Wf")
EVAL_KEYS = ("Z", "dX", "dW", "db", "dgamma", "dbeta", "Y")


def _run(inp, **kw):
    from paper_2305_11624_amd.runner import DepthwiseRun
    r = DepthwiseRun(inp, poison=True, **kw)
    r.step()
    return r.results()


SHAPES = [
    #          name          N  C   H   W   C  k s p
    BlockShape("d32_3x3", 2, 6, 9, 8, 6, 3, 1, 1, "f32", 91),
    BlockShape("d32_3x3_s2", 2, 5, 9, 9, 5, 3, 2, 1, "f32", 92),
    BlockShape("d32_5x5", 1, 4, 11, 10, 4, 5, 1, 2, "f32", 93),
    # bf16, channel counts of inverted-residual / ghost modules; several slices and a ragged tail in every dimension
    BlockShape("d_3x3", 3, 144, 28, 28, 144, 3, 1, 1, "bf16", 94),
    BlockShape("d_3x3_s2", 2, 96, 29, 27, 96, 3, 2, 1, "bf16", 95),
    BlockShape("d_5x5", 2, 72, 14, 14, 72, 5, 1, 2, "bf16", 96),       # more window positions than one pass accumulates
    BlockShape("d_5x5_s2", 2, 40, 17, 17, 40, 5, 2, 2, "bf16", 97),
    BlockShape("d_wide", 2, 960, 7, 7, 960, 3, 1, 1, "bf16", 98),
    BlockShape("d_odd_ch", 2, 20, 9, 9, 20, 3, 1, 1, "bf16", 99),      # channels not a multiple of 8: scalar path
    BlockShape("d_1x1", 2, 32, 6, 6, 32, 1, 1, 0, "bf16", 100),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_shapes(shape):
    inp = synth.make_dw_inputs(shape, bias=shape.dtype == "f32" or shape.name in ("d_3x3_s2", "d_5x5"))
    ref = oracle_dw_block(inp)
    compare(_run(inp), ref, shape.dtype, keys=KEYS, tag=shape.name)
    compare(_run(inp, mode="eval"), ref, shape.dtype, keys=EVAL_KEYS, tag=shape.name + "/eval")


def test_refold_input_gradient_only_and_wide_scale():
    shape = BlockShape("d_refold", 2, 64, 12, 12, 64, 3, 1, 1, "bf16", 101)
    inp = synth.make_dw_inputs(shape, wide_scale=True, bias=True)
    ref = oracle_dw_block(inp)
    compare(_run(inp), ref, "bf16", keys=KEYS, tag="d_wide_scale")
    compare(_run(inp, keep_folded=False), ref, "bf16", keys=KEYS[:-1], tag="d_refold")
    res = _run(inp, params=False)
    compare(res, ref, "bf16", keys=("Z", "dX"), tag="d_dx_only")
    assert res["dW"] is None and res["dgamma"] is None


@pytest.mark.parametrize("s,p", [(1, 1), (1, 0), (1, 2), (2, 1), (2, 0)])
def test_refolding_reproduces_the_kept_filter(s, p):
    """The filter that backward folds again is the one forward keeps (rounded to bf16 once): dX is the same bit for bit, with the
    weight gradient beside it and on its own."""
    shape = BlockShape("d_refold", 3, 40, 17, 14, 40, 3, s, p, "bf16", 11 + 3 * s + p)
    inp = synth.make_dw_inputs(shape, wide_scale=True)
    kept = _run(inp)["dX"]
    assert torch.equal(kept, _run(inp, keep_folded=False)["dX"])
    assert torch.equal(kept, _run(inp, keep_folded=False, params=False)["dX"])
    assert torch.equal(kept, _run(inp, params=False)["dX"])


# the sweep of the 3x3 kernels: every padding it takes, odd and even sides, strips with a remainder, one channel group and
# several workgroups of channels, fewer positions than threads, strides
SWEEP = [(n, c, h, w, s, p) for n, c, h, w, s, p in [
    (1, 8, 3, 3, 1, 0), (1, 8, 1, 1, 1, 1), (2, 16, 5, 4, 1, 2), (3, 264, 13, 11, 1, 1), (1, 520, 31, 7, 1, 0),
    (2, 32, 57, 63, 1, 1), (40, 96, 29, 30, 1, 1), (2, 24, 9, 10, 1, 2), (1, 8, 3, 3, 2, 0), (1, 8, 1, 2, 2, 1),
    (2, 16, 5, 4, 2, 2), (3, 264, 13, 10, 2, 1), (2, 40, 14, 15, 2, 0), (2, 32, 57, 64, 2, 1), (24, 96, 28, 29, 2, 1),
    (2, 24, 8, 11, 2, 2),
    # paddings above the window: dZ's first and last rows and columns meet no x
    (2, 24, 9, 7, 1, 3), (1, 8, 1, 1, 1, 4), (9, 72, 21, 30, 1, 5), (2, 24, 9, 8, 2, 3), (1, 8, 2, 1, 2, 4), (9, 72, 21, 30, 2, 5)]]


@pytest.mark.parametrize("n,c,h,w,s,p", SWEEP)
def test_row_sweep(n, c, h, w, s, p):
    shape = BlockShape("d_sweep", n, c, h, w, c, 3, s, p, "bf16", 7 * c + h + w + p)
    inp = synth.make_dw_inputs(shape, bias=(h + w) % 2 == 0)
    ref = oracle_dw_block(inp)
    compare(_run(inp), ref, "bf16", keys=KEYS, tag=str((n, c, h, w, s, p)))
    compare(_run(inp, keep_folded=False, need_dx=False), ref, "bf16", keys=("Z", "dW", "db", "dgamma", "dbeta"), tag="no dx")
    compare(_run(inp, keep_folded=False, params=False), ref, "bf16", keys=("dX",), tag="dx only")
    compare(_run(inp, mode="eval"), ref, "bf16", keys=EVAL_KEYS, tag="eval")


@pytest.mark.parametrize("s", [1, 2])
@pytest.mark.parametrize("ph,pw", [(1, 0), (0, 2), (2, 1), (1, 4), (5, 1), (3, 0)])
def test_uneven_paddings(ph, pw, s):
    """Rows and columns padded differently, all four gradients at once and dX or dW alone, against fp64 on the host."""
    import torch.nn.functional as F
    n, c, h, w = 3, 24, 11, 18
    g = torch.Generator().manual_seed(17 * ph + pw)
    r = lambda *size: torch.randn(*size, generator=g).to(torch.bfloat16).double()
    x, wt, gamma, var = r(n, c, h, w).requires_grad_(), r(c, 1, 3, 3).requires_grad_(), r(c), r(c).abs() + 0.5
    beta, mean = r(c), r(c)
    scale = gamma / (var + 1e-5).sqrt()
    y = F.conv2d(x, wt, None, s, (ph, pw), groups=c)
    z = (y - mean[:, None, None]) * scale[:, None, None] + beta[:, None, None]
    dz = r(*z.shape)
    z.backward(dz)
    ref = dict(Z=z.detach(), dX=x.grad, dW=wt.grad, dbeta=dz.sum((0, 2, 3)),
               dgamma=(dz * ((y.detach() - mean[:, None, None]) / (var + 1e-5).sqrt()[:, None, None])).sum((0, 2, 3)))
    ref = {k: v.numpy() for k, v in ref.items()}
    d = B.make_desc(n, c, h, w, c, 3, 3, s, ph, pad_w=pw)
    act, vec = (lambda t: B.act_to_device(t.detach().float(), torch.bfloat16, "cuda")), (lambda t: t.float().cuda())
    xd, wd, dzd = act(x), wt.detach().reshape(c, 3, 3).to(torch.bfloat16).cuda(), act(dz)
    nan = lambda like: torch.full_like(like, float("nan"))
    ws = [torch.empty(max(16, B.convbn_dw_workspace_bytes(d, B.MODE_TUNE, p)), dtype=torch.uint8, device="cuda")
          for p in (B.PASS_FWD, B.PASS_BWD)]
    zd, wf = nan(dzd), torch.empty(3, 3, c, dtype=torch.bfloat16, device="cuda")
    B.convbn_dw_tune_fwd(d, xd, wd, None, vec(gamma), vec(beta), vec(mean), vec(var), zd, wf, ws[0])
    for need_dx, params in ((True, True), (True, False), (False, True)):
        dx, dw, dga, dbe = (nan(t) for t in (xd, wd, vec(gamma), vec(beta)))
        B.convbn_dw_tune_bwd(d, xd, wd, None, vec(gamma), vec(mean), vec(var), wf, dzd, dx if need_dx else None,
                             dw if params else None, None, dga if params else None, dbe if params else None, ws[1])
        got = dict(Z=B.act_from_device(zd))
        if need_dx:
            got["dX"] = B.act_from_device(dx)
        if params:
            got.update(dW=dw.double().cpu().reshape(c, 1, 3, 3), dgamma=dga.double().cpu(), dbeta=dbe.double().cpu())
        compare(got, ref, "bf16", keys=list(got), tag=str((ph, pw, s)))


@pytest.mark.parametrize("s", [1, 2])
@pytest.mark.parametrize("where", ["x", "dy"])
def test_infinity_stays_with_the_taps_that_touch_it(where, s):
    """An infinite value in the last row and column meets fewer than nine taps: dW is finite at the others."""
    h = 13
    shape = BlockShape("d_inf", 2, 16, h, h, 16, 3, s, 1, "bf16", 3)
    inp = synth.make_dw_inputs(shape)
    t = inp[where].clone()
    t[1, 5, -1, -1] = float("inf")
    finite = torch.isfinite(_run(dict(inp, **{where: t}))["dW"])
    assert finite[[c for c in range(16) if c != 5]].all()
    # x[h-1] meets dZ[h + 1 - i]: taps 1, 2 (stride 2 with an odd side: tap 1);  dZ[last] meets x[last + i - 1]: taps 0, 1
    hit = ([1] if s == 2 else [1, 2]) if where == "x" else [0, 1]
    for i in range(3):
        for j in range(3):
            assert bool(finite[5, 0, i, j]) == (i not in hit or j not in hit), (i, j)


@pytest.mark.parametrize("s", [1, 2])
def test_large_outputs(s):
    """Outputs of 16 MB and more leave through other stores: 32 images at once give what two calls of 16 give, bit for bit."""
    from paper_2305_11624_amd.runner import DepthwiseRun
    c, h = 96, 64 * s
    g = torch.Generator(device="cuda").manual_seed(7)
    normal = lambda *size: torch.randn(*size, generator=g, device="cuda")
    x, dy = normal(32, c, h, h), normal(32, c, 64, 64)
    inp = dict(W=normal(c, 1, 3, 3), gamma=normal(c), beta=normal(c), rmean=normal(c), rvar=normal(c).abs() + 0.5, b=None, eps=1e-5)
    z, dx = [], []
    for a, b in ((0, 32), (0, 16), (16, 32)):
        shape = BlockShape("large", b - a, c, h, h, c, 3, s, 1, "bf16")
        r = DepthwiseRun(dict(inp, shape=shape, x=x[a:b], dy=dy[a:b]), poison=True)
        r.step()
        z.append(r.z)
        dx.append(r.dx)
    assert z[0].nbytes >= 16 << 20 > z[1].nbytes
    assert torch.equal(z[0], torch.cat(z[1:])) and torch.equal(dx[0], torch.cat(dx[1:]))


def test_full_size_layer():
    """A depthwise layer at network size: 144 channels, 56x56, N = 32 (an inverted-residual stage), sampled against
    the oracle run on the first two images (the block is independent across images except for the parameter gradients,
    which are compared on a two-image problem of their own)."""
    shape = BlockShape("d_full", 32, 144, 56, 56, 144, 3, 1, 1, "bf16", 102)
    inp = synth.make_dw_inputs(shape)
    res = _run(inp)
    small = {k: (v[:2] if k in ("x", "dy") else v) for k, v in inp.items()}
    small["shape"] = BlockShape("d_full2", 2, 144, 56, 56, 144, 3, 1, 1, "bf16", 102)
    ref = oracle_dw_block(small)
    compare({k: res[k][:2] for k in ("Z", "dX")}, ref, "bf16", keys=("Z", "dX"), tag="d_full[:2]")
    compare(_run(small), ref, "bf16", keys=KEYS, tag="d_full2")


def test_errors():
    d = B.make_desc(2, 16, 8, 8, 32, 3, 3, 1, 1)     # Cin != Cout
    assert B.convbn_dw_workspace_bytes(d, B.MODE_TUNE, B.PASS_FWD) == 0
    x = torch.zeros(4096, device="cuda", dtype=torch.bfloat16)
    v = torch.zeros(32, device="cuda")
    assert B.convbn_dw_tune_fwd(d, x, x, None, v, v, v, v, x, None, x, check=False) == B.ERR_SHAPE
    d = B.make_desc(2, 16, 8, 8, 16, 3, 3, 1, 1)
    assert B.convbn_dw_tune_fwd(d, x, x, None, v, v, v, v, x, None, None, check=False) == B.ERR_WORKSPACE
