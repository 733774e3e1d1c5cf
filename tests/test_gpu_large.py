"""GPU parity of large tensors.  Beyond 2 GiB, which the kernels with 32-bit byte offsets decline: bf16 runs the implicit GEMM
(conv_igemm.hip), fp32 one thread per output (conv_direct.hip).  One 3x3 block, Tune mode; three images are compared,
one of them across the 2 GiB line, against the definition in fp64, and the others' input gradient is zero.  Depthwise
blocks beyond 1 GiB, which take several launches, by images or by bands of an image's rows, and first layers whose one image
is beyond 1 GiB on one side or the other, and a grouped block there: everything against fp64."""
import pytest
import torch
import torch.nn.functional as F

from paper_2305_11624_amd import binding as B

from helpers import TOL

pytestmark = pytest.mark.gpu

N, H, W, K = 33, 2050, 2047, 3
IMAGES = (0, 31, 32)   # (16 bytes a pixel: the 2 GiB line is in image 31)
ROWS = (slice(0, 8), slice(H // 2, H // 2 + 8), slice(H - 8, H))   # rows that have a gradient: sums short enough for fp32


@pytest.mark.parametrize("dtype,cin,cout", [("bf16", 8, 8), ("f32", 4, 4)])
def test_block_beyond_2_gib(dtype, cin, cout):
    g = torch.Generator(device="cuda").manual_seed(951)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    d = B.make_desc(N, cin, H, W, cout, K, K, 1, 1, dtype=B.BF16 if dtype == "bf16" else B.F32)
    normal = lambda *size: torch.randn(*size, generator=g, device="cuda")
    x, dz = torch.empty((N, H, W, cin), dtype=dt, device="cuda"), torch.zeros((N, H, W, cout), dtype=dt, device="cuda")
    assert x.nbytes > 1 << 31 and x[31].data_ptr() - x.data_ptr() < 1 << 31 < x[32].data_ptr() - x.data_ptr()
    for n in range(N):
        x[n] = normal(H, W, cin)
    for n in IMAGES:
        for r in ROWS:
            dz[n, r] = normal(8, W, cout)
    w = (normal(cout, K, K, cin) * 0.2).to(dt)
    gamma, var = torch.rand(cout, generator=g, device="cuda") + 0.5, torch.rand(cout, generator=g, device="cuda") + 0.5
    b, beta, mean = normal(cout), normal(cout), normal(cout)
    nan = lambda like: torch.full_like(like, float("nan"))
    z, dx, dw, wf = nan(dz), nan(x), nan(w), torch.empty((cin, K, K, cout), dtype=dt, device="cuda")
    db, dgamma, dbeta = nan(b), nan(gamma), nan(beta)
    ws = [torch.empty(max(16, B.convbn_workspace_bytes(d, B.MODE_TUNE, p)), dtype=torch.uint8, device="cuda")
          for p in (B.PASS_FWD, B.PASS_BWD)]
    print(dtype, "forward", flush=True)
    B.convbn_tune_fwd(d, x, w, b, gamma, beta, mean, var, z, wf, ws[0])
    torch.cuda.synchronize()
    print(dtype, "backward", flush=True)
    B.convbn_tune_bwd(d, x, w, b, gamma, mean, var, wf, dz, dx, dw, db, dgamma, dbeta, ws[1])
    torch.cuda.synchronize()

    def close(got, ref, what):
        err = (got.double() - ref).abs().max() / ref.abs().max()
        assert err <= TOL[dtype], (what, err.item())

    wd, isd = w.double(), 1.0 / (var.double() + d.eps).sqrt()
    s = gamma.double() * isd
    taps = [(i, j) for i in range(K) for j in range(K)]
    pad = lambda t: F.pad(t.double(), (0, 0, 1, 1, 1, 1))
    rdw, rdgamma, r = torch.zeros_like(wd), torch.zeros_like(s), torch.zeros_like(s)
    for n in IMAGES:
        xp, zp = pad(x[n]), pad(dz[n])
        y = torch.zeros((H * W, cout), dtype=torch.float64, device="cuda")
        rdx = torch.zeros((H * W, cin), dtype=torch.float64, device="cuda")
        for i, j in taps:
            xt = xp[i:i + H, j:j + W].reshape(-1, cin)
            y += xt @ wd[:, i, j].t().contiguous()
            rdx += zp[2 - i:2 - i + H, 2 - j:2 - j + W].reshape(-1, cout) @ (wd[:, i, j] * s[:, None])
            for q in ROWS:
                xq = xp[q.start + i:q.stop + i, j:j + W].reshape(-1, 1, cin)
                rdw[:, i, j] += (dz[n, q].double().reshape(-1, cout, 1) * xq).sum(0) * s[:, None]
        y += b.double() - mean.double()
        close(z[n].reshape(-1, cout), y * s + beta.double(), ("Z", n))
        close(dx[n].reshape(-1, cin), rdx, ("dX", n))
        for q in ROWS:
            dzq = dz[n, q].double().reshape(-1, cout)
            rdgamma += (dzq * y[q.start * W:q.stop * W]).sum(0) * isd
            r += dzq.sum(0)
    close(dw, rdw, "dW")
    close(dgamma, rdgamma, "dgamma")
    close(dbeta, r, "dbeta")
    close(db, r * s, "db")
    for n in range(1, 31):
        assert not dx[n].any(), n


@pytest.mark.parametrize("n,h,w,s,p", [(5, 3101, 3003, 1, 1), (5, 3101, 3003, 2, 1),   # three images and two
                                       (1, 6100, 6003, 1, 1), (1, 6100, 6003, 2, 1), (1, 6100, 6003, 1, 3),
                                       (2, 6101, 6003, 2, 0)])                         # bands of one image
def test_depthwise_block_beyond_1_gib(n, h, w, s, p):
    g = torch.Generator(device="cuda").manual_seed(h + s)
    c, bf = 16, torch.bfloat16
    d = B.make_desc(n, c, h, w, c, K, K, s, p)
    ho, wo = (h + 2 * p - K) // s + 1, (w + 2 * p - K) // s + 1
    normal = lambda *size: torch.randn(*size, generator=g, device="cuda")
    x, dz = normal(n, h, w, c).to(bf), normal(n, ho, wo, c).to(bf)
    assert x.nbytes > 1 << 30 and (n == 5 or x[0].nbytes > 1 << 30)
    wt = normal(c, K, K).to(bf)
    gamma, var = torch.rand(c, generator=g, device="cuda") + 0.5, torch.rand(c, generator=g, device="cuda") + 0.5
    b, beta, mean = normal(c), normal(c), normal(c)
    nan = lambda like: torch.full_like(like, float("nan"))
    z, dx, dw, wf = nan(dz), nan(x), nan(wt), torch.empty((K, K, c), dtype=bf, device="cuda")
    db, dgamma, dbeta = nan(b), nan(gamma), nan(beta)
    ws = [torch.empty(max(16, B.convbn_dw_workspace_bytes(d, B.MODE_TUNE, q)), dtype=torch.uint8, device="cuda")
          for q in (B.PASS_FWD, B.PASS_BWD)]
    ws[1].fill_(255)   # (NaNs: every slice has to be written)
    print("forward", flush=True)
    B.convbn_dw_tune_fwd(d, x, wt, b, gamma, beta, mean, var, z, wf, ws[0])
    torch.cuda.synchronize()
    print("backward", flush=True)
    B.convbn_dw_tune_bwd(d, x, wt, b, gamma, mean, var, wf, dz, dx, dw, db, dgamma, dbeta, ws[1])
    torch.cuda.synchronize()

    def close(got, ref, what):
        err = (got.double() - ref).abs().max() / ref.abs().max()
        assert err <= TOL["bf16"], (what, err.item())

    isd = 1.0 / (var.double() + d.eps).sqrt()
    scale, wd = gamma.double() * isd, wt.double()
    rdw, rdgamma, r = torch.zeros_like(wd), torch.zeros_like(scale), torch.zeros_like(scale)
    for i in range(n):
        xp, zd = F.pad(x[i].double(), (0, 0, p, p, p, p)), dz[i].double()
        dxp, y = torch.zeros_like(xp), torch.zeros_like(zd)
        for u in range(K):
            for v in range(K):
                at = (slice(u, u + (ho - 1) * s + 1, s), slice(v, v + (wo - 1) * s + 1, s))
                y += xp[at] * wd[:, u, v]
                dxp[at] += zd * (wd[:, u, v] * scale)
                rdw[:, u, v] += (zd * xp[at]).sum((0, 1)) * scale
        y += b.double() - mean.double()
        close(z[i], y * scale + beta.double(), ("Z", i))
        close(dx[i], dxp[p:p + h, p:p + w], ("dX", i))
        rdgamma += (zd * y).sum((0, 1)) * isd
        r += zd.sum((0, 1))
    close(dw, rdw, "dW")
    close(dgamma, rdgamma, "dgamma")
    close(dbeta, r, "dbeta")
    close(db, r * scale, "db")


@pytest.mark.parametrize("h,w,cin,cout,k", [(6000, 6004, 3, 64, 7), (6001, 5999, 3, 64, 7),   # dZ; read as it is, and widened
                                            (11700, 11600, 3, 32, 3)])                        # x
def test_first_layer_beyond_1_gib(h, w, cin, cout, k):
    g = torch.Generator(device="cuda").manual_seed(h)
    bf, s, p = torch.bfloat16, 2, k // 2
    d = B.make_desc(1, cin, h, w, cout, k, k, s, p)
    ho, wo = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
    normal = lambda *size: torch.randn(*size, generator=g, device="cuda")
    x, dz = normal(1, h, w, cin).to(bf), normal(1, ho, wo, cout).to(bf)
    assert dz.nbytes > 1 << 30 or h * w * 8 > 1 << 30
    wt = (normal(cout, k, k, cin) * 0.2).to(bf)
    gamma, var = torch.rand(cout, generator=g, device="cuda") + 0.5, torch.rand(cout, generator=g, device="cuda") + 0.5
    b, beta, mean = normal(cout), normal(cout), normal(cout)
    nan = lambda like: torch.full_like(like, float("nan"))
    z, dx, dw, wf = nan(dz), nan(x), nan(wt), torch.empty((cin, k, k, cout), dtype=bf, device="cuda")
    db, dgamma, dbeta = nan(b), nan(gamma), nan(beta)
    ws = [torch.empty(max(16, B.convbn_workspace_bytes(d, B.MODE_TUNE, q)), dtype=torch.uint8, device="cuda")
          for q in (B.PASS_FWD, B.PASS_BWD)]
    print("forward", flush=True)
    B.convbn_tune_fwd(d, x, wt, b, gamma, beta, mean, var, z, wf, ws[0])
    torch.cuda.synchronize()
    print("backward", flush=True)
    B.convbn_tune_bwd(d, x, wt, b, gamma, mean, var, wf, dz, dx, dw, db, dgamma, dbeta, ws[1])
    torch.cuda.synchronize()

    def close(got, ref, what):
        err = (got.double() - ref).abs().max() / ref.abs().max()
        assert err <= TOL["bf16"], (what, err.item())

    isd = 1.0 / (var.double() + d.eps).sqrt()
    scale, wd = gamma.double() * isd, wt.double()
    xp, zd = F.pad(x[0].double(), (0, 0, p, p, p, p)), dz[0].double().reshape(-1, cout)
    dxp, y, rdw = torch.zeros_like(xp), torch.zeros_like(zd), torch.zeros_like(wd)
    for i in range(k):
        for j in range(k):
            at = (slice(i, i + (ho - 1) * s + 1, s), slice(j, j + (wo - 1) * s + 1, s))
            xt = xp[at].reshape(-1, cin)
            y += xt @ wd[:, i, j].t().contiguous()
            dxp[at] += (zd @ (wd[:, i, j] * scale[:, None])).reshape(ho, wo, cin)
            for c in range(cin):
                rdw[:, i, j, c] = (zd * xt[:, c:c + 1]).sum(0) * scale
    y += b.double() - mean.double()
    r = zd.sum(0)
    rdgamma = (zd * y).sum(0) * isd
    close(z.reshape(-1, cout), y * scale + beta.double(), "Z")
    close(dx[0], dxp[p:p + h, p:p + w], "dX")
    close(dw, rdw, "dW")
    close(dgamma, rdgamma, "dgamma")
    close(dbeta, r, "dbeta")
    close(db, r * scale, "db")


@pytest.mark.parametrize("s", [1, 2])
def test_grouped_block_beyond_1_gib(s):
    g = torch.Generator(device="cuda").manual_seed(s)
    n, h, w, c, groups, p, bf = 2, 3000, 2900, 32, 8, 1, torch.bfloat16
    cg = c // groups
    d = B.make_desc(n, c, h, w, c, K, K, s, p)
    ho, wo = (h + 2 * p - K) // s + 1, (w + 2 * p - K) // s + 1
    normal = lambda *size: torch.randn(*size, generator=g, device="cuda")
    x, dz = normal(n, h, w, c).to(bf), normal(n, ho, wo, c).to(bf)
    assert x.nbytes > 1 << 30
    wt = (normal(c, K, K, cg) * 0.3).to(bf)
    gamma, var = torch.rand(c, generator=g, device="cuda") + 0.5, torch.rand(c, generator=g, device="cuda") + 0.5
    b, beta, mean = normal(c), normal(c), normal(c)
    nan = lambda like: torch.full_like(like, float("nan"))
    z, dx, dw, wf = nan(dz), nan(x), nan(wt), torch.empty((cg, K, K, c), dtype=bf, device="cuda")
    db, dgamma, dbeta = nan(b), nan(gamma), nan(beta)
    ws = [torch.empty(max(16, B.convbn_grouped_workspace_bytes(d, groups, B.MODE_TUNE, q)), dtype=torch.uint8, device="cuda")
          for q in (B.PASS_FWD, B.PASS_BWD)]
    print("forward", flush=True)
    B.convbn_grouped_tune_fwd(d, groups, x, wt, b, gamma, beta, mean, var, z, wf, ws[0])
    torch.cuda.synchronize()
    print("backward", flush=True)
    B.convbn_grouped_tune_bwd(d, groups, x, wt, b, gamma, mean, var, wf, dz, dx, dw, db, dgamma, dbeta, ws[1])
    torch.cuda.synchronize()

    def close(got, ref, what):
        err = (got.double() - ref).abs().max() / ref.abs().max()
        assert err <= TOL["bf16"], (what, err.item())

    isd = 1.0 / (var.double() + d.eps).sqrt()
    scale, wd = gamma.double() * isd, wt.double()
    rdw, rdgamma, r = torch.zeros_like(wd), torch.zeros_like(scale), torch.zeros_like(scale)
    for m in range(n):
        xp, zd = F.pad(x[m].double(), (0, 0, p, p, p, p)), dz[m].double()
        dxp, y = torch.zeros_like(xp), torch.zeros_like(zd)
        for i in range(K):
            for j in range(K):
                rows, cols = slice(i, i + (ho - 1) * s + 1, s), slice(j, j + (wo - 1) * s + 1, s)
                for k in range(groups):
                    ch = slice(k * cg, (k + 1) * cg)
                    xt = xp[rows, cols, ch]
                    for o in range(k * cg, (k + 1) * cg):
                        y[..., o] += (xt * wd[o, i, j]).sum(-1)
                        dxp[rows, cols, ch] += zd[..., o:o + 1] * (wd[o, i, j] * scale[o])
                        rdw[o, i, j] += (zd[..., o:o + 1] * xt).sum((0, 1)) * scale[o]
        y += b.double() - mean.double()
        close(z[m], y * scale + beta.double(), ("Z", m))
        close(dx[m], dxp[p:p + h, p:p + w], ("dX", m))
        rdgamma += (zd * y).sum((0, 1)) * isd
        r += zd.sum((0, 1))
    close(dw, rdw, "dW")
    close(dgamma, rdgamma, "dgamma")
    close(dbeta, r, "dbeta")
    close(db, r * scale, "db")
