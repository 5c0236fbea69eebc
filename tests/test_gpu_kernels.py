"""Kernels behind a rule on sizes, each at the sizes where it can go wrong (edges
of its tiles, remainders, the smallest and largest of its range), against plain
torch in 64 bits on the same rounded inputs.

Tolerances are relative to the sums of absolute values: a sum of n products in
working precision u, in any order, is within (n + 2) u of that; the bounds below
use that with a factor 4 for the activation and the operand that feeds it.
"""
import math

import pytest
import torch

from paper_1812_04352_amd import lp as L

pytestmark = pytest.mark.gpu
EPS = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}
DT = {"f32": torch.float32, "f64": torch.float64}


def act(z, a):
    if a == "tanh":
        return torch.tanh(z)
    if a == "relu":
        return torch.clamp(z, min=0.0)
    if a == "identity":
        return z
    return torch.where(z.abs() <= 0.1, (2.5 * z + 0.5) * z + 0.025, torch.clamp(z, min=0.0))


def dact(z, a):
    if a == "tanh":
        return 1.0 - torch.tanh(z) ** 2
    if a == "relu":
        return (z > 0).to(z.dtype)
    if a == "identity":
        return torch.ones_like(z)
    return torch.where(z.abs() <= 0.1, 5.0 * z + 0.5, (z > 0).to(z.dtype))


def rnd(seed, *shape, dtype=torch.float32, std=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64) * std).to(dtype)


def within(got, ref, scale, bound, what):
    """|got - ref| <= bound * scale elementwise (scale: the sums of absolute values)."""
    d = (got.double() - ref).abs()
    worst = float((d / (scale + 1e-300)).max())
    assert worst <= bound, f"{what}: {worst:.3e} of the absolute sum, bound {bound:.3e}"


# tiles of 32 x 32 with 512-byte pieces of the features (forward); an example per thread up
# to 8 features, else 1 to 16 features per lane and 8 or 16 waves (gradient)
@pytest.mark.parametrize("dtype,act_name,B,q,nf", [
    ("f32", "tanh", 1, 8, 1), ("f32", "relu", 31, 16, 2), ("f32", "smoothrelu", 33, 32, 127), ("f32", "tanh", 129, 32, 128),
    ("f32", "identity", 100, 64, 129), ("f32", "tanh", 257, 220, 220), ("f32", "tanh", 70, 8, 513),
    ("f32", "tanh", 37, 8, 1023), ("f32", "relu", 1500, 32, 1024),
    ("f64", "tanh", 1, 8, 1), ("f64", "smoothrelu", 65, 16, 63), ("f64", "tanh", 257, 32, 65), ("f64", "tanh", 33, 8, 1024),
    ("f64", "tanh", 5000, 8, 2), ("f64", "smoothrelu", 4097, 16, 3), ("f32", "relu", 4096, 8, 8), ("f32", "tanh", 1025, 16, 9),
    ("f64", "tanh", 130, 16, 128), ("f64", "tanh", 129, 16, 200), ("f64", "smoothrelu", 100, 8, 513),
])
def test_dense_opening(dtype, act_name, B, q, nf):
    p = L.problem(dtype, "dense", act_name, 1, B, q)
    y, Lw, lam = (rnd(k, *s, dtype=DT[dtype], std=d) for k, s, d in
                  ((1, (B, nf), 1.0), (2, (q, nf), nf ** -0.5), (3, (B, q), 1.0)))
    u0, dL = torch.full((B, q), float("nan"), device="cuda", dtype=DT[dtype]), torch.empty_like(Lw)
    L.lp_open_forward(p, L.LP_OPEN_DENSE_ACT, nf, y, Lw, u0)
    L.lp_open_grad(p, L.LP_OPEN_DENSE_ACT, nf, y, Lw, lam, dL)
    y, Lw, lam = y.double(), Lw.double(), lam.double()
    z, za = y @ Lw.T.contiguous(), y.abs() @ Lw.abs().T.contiguous()
    within(u0, act(z, act_name), za + 0.025, 4 * (nf + 8) * EPS[dtype], "u0")
    s = dact(z, act_name) * lam
    # sigma' changes by at most 5 |dz|; a ReLU site within rounding of zero may go either way
    scale = (lam.abs() * (1.0 + 5.0 * za)).T.contiguous() @ y.abs()
    bound = 4 * (nf + B + 8) * EPS[dtype]
    if act_name == "relu":
        open_sites = (z.abs() <= 4 * (nf + 8) * EPS[dtype] * za).double() * lam.abs()
        scale = scale + (open_sites.T.contiguous() @ y.abs()) / bound
    within(dL, s.T.contiguous() @ y, scale, bound, "dL")


@pytest.mark.parametrize("act_name,B,H,W", [("tanh", 1, 2, 7), ("smoothrelu", 3, 4, 9), ("tanh", 37, 28, 28),
                                            ("identity", 5, 12, 13), ("tanh", 2, 28, 3), ("smoothrelu", 150, 6, 4)])
def test_conv_opening_gradient(act_name, B, H, W):
    p = L.problem("f32", "conv3x3", act_name, 1, B, 8, H, W)
    y, Lw, lam = rnd(1, B, 1, H, W), rnd(2, 8, 1, 3, 3, std=0.3), rnd(3, B, 8, H, W)
    dL = torch.empty_like(Lw)
    L.lp_open_grad(p, L.LP_OPEN_CONV_ACT, H * W, y, Lw, lam, dL)
    y, Lw, lam = y.double(), Lw.double(), lam.double()
    pad = torch.nn.functional.pad(y[:, 0], (1, 1, 1, 1))
    taps = torch.stack([pad[:, i:i + H, j:j + W] for i in range(3) for j in range(3)])  # [9][B][H][W]
    z = torch.tensordot(Lw.reshape(8, 9), taps, 1).transpose(0, 1)
    za = torch.tensordot(Lw.abs().reshape(8, 9), taps.abs(), 1).transpose(0, 1)
    s = dact(z, act_name) * lam
    ref = torch.stack([(s * t[:, None]).sum((0, 2, 3)) for t in taps], 1)
    scale = torch.stack([(lam.abs() * (1.0 + 5.0 * za) * t.abs()[:, None]).sum((0, 2, 3)) for t in taps], 1)
    within(dL.reshape(8, 9), ref, scale, 4 * (9 + 8 + 32) * EPS["f32"], "dL")


# staged in LDS up to 64 KB, one workgroup (or wave) per example beyond
@pytest.mark.parametrize("layer,B,C,H,W,nc", [("dense", 1, 8, 1, 1, 1), ("dense", 67, 220, 1, 1, 64),
                                             ("conv3x3", 1, 8, 12, 13, 10), ("conv3x3", 9, 8, 28, 28, 64),
                                             ("conv3x3", 6, 8, 28, 28, 1), ("conv3x3", 5, 8, 20, 27, 17)])
def test_head_and_accuracy(layer, B, C, H, W, nc):
    p = L.problem("f32", layer, "tanh", 1, B, C, H, W)
    q = C * H * W
    u, Wc, mu = rnd(1, B, q), rnd(2, nc, q, std=q ** -0.5), rnd(3, nc)
    c = torch.zeros(B, nc, device="cuda")
    c[torch.arange(B), torch.arange(B) % nc] = 1.0
    J, acc = (torch.zeros(1, device="cuda", dtype=torch.float64) for _ in range(2))
    lam, dW, dmu, ws = torch.empty_like(u), torch.empty_like(Wc), torch.empty_like(mu), L.alloc_workspace(p)
    L.lp_loss_terminal(p, nc, u, Wc, mu, c, J, lam, dW, dmu, ws)
    L.lp_accuracy(p, nc, u, Wc, mu, c, acc, ws)
    u, Wc, mu, c = u.double(), Wc.double(), mu.double(), c.double()
    z = u @ Wc.T.contiguous() + mu
    d = (torch.softmax(z, 1) - c) / B
    torch.testing.assert_close(J[0], -(c * torch.log_softmax(z, 1)).sum() / B, rtol=1e-12, atol=1e-12)
    for got, ref, s in ((lam, d @ Wc, d.abs() @ Wc.abs()), (dW, d.T.contiguous() @ u, d.abs().T.contiguous() @ u.abs()),
                        (dmu, d.sum(0), d.abs().sum(0))):
        within(got, ref, s, 2 * EPS["f32"], "head")  # summed in fp64, rounded once
    assert float(acc) == float((z.argmax(1) == c.argmax(1)).double().mean())


NARROW = [("f64", 8), ("f64", 16), ("f64", 32), ("f32", 8), ("f32", 16)]


def dense_problem(dtype, q, act_name, N, B, seed=0, h=0.05):
    p = L.problem(dtype, "dense", act_name, N, B, q, h=h)
    # weights at an odd offset of a flat vector: element alignment is all that is promised
    flat = rnd(seed + 1, 1 + N * q * q, dtype=DT[dtype], std=0.5 * q ** -0.5)
    K, b = flat[1:].view(N, q, q), rnd(seed + 2, 1 + N * q, dtype=DT[dtype], std=0.1)[1:].view(N, q)
    U = torch.full((N + 1, B, q), float("nan"), device="cuda", dtype=DT[dtype])
    Lam = torch.full_like(U, float("nan"))
    U[0], Lam[N] = rnd(seed + 3, B, q, dtype=DT[dtype]), rnd(seed + 4, B, q, dtype=DT[dtype])
    return p, K, b, U, Lam


def serial_reference(K, b, U, Lam, a, h):
    """Trajectory, adjoint, gradient and residual norms in 64 bits, layer by layer."""
    K, b, N = K.double(), b.double(), K.shape[0]
    u = [U[0].double()]
    for n in range(N):
        u.append(u[-1] + h * act(u[-1] @ K[n].T.contiguous() + b[n], a))
    lam, dK, db = [Lam[N].double()], [], []
    for n in reversed(range(N)):
        s = dact(u[n] @ K[n].T.contiguous() + b[n], a) * lam[0]
        dK.insert(0, h * (s.T.contiguous() @ u[n]))
        db.insert(0, h * s.sum(0))
        lam.insert(0, lam[0] + h * (s @ K[n]))
    return torch.stack(u), torch.stack(lam), torch.stack(dK), torch.stack(db)


# tiles of 16 examples per wave, 64 per sweep workgroup; smooth activations (no sites
# that rounding decides). The error of N = 6 layers grows by at most (1 + 5 h |K|)^2
# per layer, far below 16 here, so 16 (N (q + 8)) u bounds it; the gradient adds B terms.
@pytest.mark.parametrize("B", [1, 15, 17, 64, 129])
@pytest.mark.parametrize("dtype,q", NARROW)
def test_narrow_dense_layers(dtype, q, B):
    for a in ("tanh", "smoothrelu", "identity"):
        N, h = 6, 0.05
        p, K, b, U, Lam = dense_problem(dtype, q, a, N, B)
        dK, db, ws = torch.empty_like(K), torch.empty_like(b), L.alloc_workspace(p)
        L.lp_serial_forward(p, K, b, U)
        L.lp_serial_adjoint(p, K, b, U, Lam)
        L.lp_gradient(p, K, b, U, Lam, dK, db, ws)
        ref = serial_reference(K, b, U, Lam, a, h)
        bound = 16 * N * (q + 8) * EPS[dtype]
        for got, r, n in ((U, ref[0], 0), (Lam, ref[1], 0), (dK, ref[2], B), (db, ref[3], B)):
            e = float((got.double() - r).norm() / r.norm())
            assert e <= bound + 4 * n * EPS[dtype], (a, e, bound)
        # residuals of a perturbed pair against the definition
        V, M = U + 1e-3 * rnd(7, *U.shape, dtype=DT[dtype]), Lam + 1e-3 * rnd(8, *U.shape, dtype=DT[dtype])
        z = torch.bmm(V[:-1].double(), K.double().transpose(1, 2).contiguous()) + b.double()[:, None]
        rs = V[:-1].double() + h * act(z, a) - V[1:].double()
        ra = M[1:].double() + h * torch.bmm(dact(z, a) * M[1:].double(), K.double().contiguous()) - M[:-1].double()
        for which, r in ((L.LP_STATE, rs), (L.LP_ADJOINT, ra)):
            got = L.lp_residual_norm(p, which, K, b, V, M, ws)
            assert abs(got - float(r.norm())) <= bound * float(V.double().norm() + M.double().norm())


# two tiles per wave from 8192 pairs of tiles per sweep on (256 intervals x 32 here):
# examples are independent, so a part of the batch solved alone gives the same bits
@pytest.mark.parametrize("dtype,q", NARROW)
def test_narrow_two_tiles_per_wave(dtype, q):
    N, B = 1024, 1037
    p, K, b, U, Lam = dense_problem(dtype, q, "tanh", N, B, h=0.005)
    mg = L.mgrit(cf=4, max_levels=3, max_iter=2)

    def solve(U0, LN):
        ps = L.problem(dtype, "dense", "tanh", N, U0.shape[0], q, h=0.005)
        u, lam = (torch.full((N + 1,) + U0.shape, float("nan"), device="cuda", dtype=DT[dtype]) for _ in range(2))
        u[0], lam[N] = U0, LN
        ws = L.alloc_workspace(ps, mg)
        L.lp_mgrit_forward(ps, mg, K, b, u, ws)
        L.lp_mgrit_adjoint(ps, mg, K, b, u, lam, ws)
        return u, lam

    u, lam = solve(U[0], Lam[N])
    assert bool(torch.isfinite(u).all()) and bool(torch.isfinite(lam).all())
    for part in (slice(0, 33), slice(1000, 1037)):
        us, ls = solve(U[0][part].contiguous(), Lam[N][part].contiguous())
        assert torch.equal(us, u[:, part]) and torch.equal(ls, lam[:, part])


# width 220: two, four or six tiles of 16 examples per workgroup by the number of
# workgroups (six from 512 on, four from 256 on); parts of a batch give the same bits
@pytest.mark.parametrize("act_name,record", [("smoothrelu", True), ("relu", True), ("tanh", False)])
def test_wide_tiles_per_workgroup(act_name, record):
    N, B, q, h = 1024, 200, 220, 0.005
    _, K, b, U, Lam = dense_problem("f32", q, act_name, N, B, h=h)
    mg = L.mgrit(cf=4, max_levels=3, max_iter=1)

    def solve(U0, LN):
        p = L.problem("f32", "dense", act_name, N, U0.shape[0], q, h=h)
        u, lam = (torch.full((N + 1,) + U0.shape, float("nan"), device="cuda") for _ in range(2))
        u[0], lam[N] = U0, LN
        ws, rec = L.alloc_workspace(p, mg), L.alloc_dsig(p) if record else None
        L.lp_mgrit_forward(p, mg, K, b, u, ws, dsig=rec)
        L.lp_mgrit_adjoint(p, mg, K, b, u, lam, ws, dsig=rec)
        return u, lam

    u, lam = solve(U[0], Lam[N])
    assert bool(torch.isfinite(u).all()) and bool(torch.isfinite(lam).all())
    for part in (slice(0, 37), slice(185, 200)):
        us, ls = solve(U[0][part].contiguous(), Lam[N][part].contiguous())
        assert torch.equal(us, u[:, part]) and torch.equal(ls, lam[:, part])


@pytest.mark.parametrize("B", [1, 31, 65, 129])
def test_wide_layers(B):
    N, q, h = 4, 220, 0.05
    for a in ("tanh", "smoothrelu", "identity"):
        p, K, b, U, Lam = dense_problem("f32", q, a, N, B)
        ref = serial_reference(K, b, U, Lam, a, h)
        for record in (True, False):
            rec = L.alloc_dsig(p) if record else None
            dK, db, ws = torch.empty_like(K), torch.empty_like(b), L.alloc_workspace(p)
            L.lp_serial_forward(p, K, b, U, dsig=rec)
            L.lp_serial_adjoint(p, K, b, U, Lam, dsig=rec)
            L.lp_gradient(p, K, b, U, Lam, dK, db, ws, dsig=rec)
            bound = 16 * N * (q + 8) * EPS["f32"]
            for got, r, n in ((U, ref[0], 0), (Lam, ref[1], 0), (dK, ref[2], B), (db, ref[3], B)):
                e = float((got.double() - r).norm() / r.norm())
                assert e <= bound + 4 * n * EPS["f32"], (a, record, e, bound)


# convolution sweeps read their products from a split image in LDS: odd widths, the
# narrowest and the largest images, ghost lanes in the last tile
@pytest.mark.parametrize("H,W", [(2, 1), (4, 9), (12, 13), (28, 28), (30, 28)])
def test_conv_layers(H, W):
    N, B, h = 4, 3, 0.1
    for a in ("tanh", "smoothrelu", "identity"):
        p = L.problem("f32", "conv3x3", a, N, B, 8, H, W, h=h)
        K, b = rnd(1, N, 8, 8, 3, 3, std=0.15), rnd(2, N, 8, std=0.1)
        U, Lam = (torch.full((N + 1, B, 8, H, W), float("nan"), device="cuda") for _ in range(2))
        U[0], Lam[N] = rnd(3, B, 8, H, W), rnd(4, B, 8, H, W)
        Kd, bd = K.double().cpu(), b.double().cpu()[:, None, :, None, None]
        u = [U[0].double().cpu()]
        for n in range(N):
            u.append(u[-1] + h * act(torch.conv2d(u[-1], Kd[n], padding=1) + bd[n], a))
        lam, dK = [Lam[N].double().cpu()], []
        for n in reversed(range(N)):
            s = dact(torch.conv2d(u[n], Kd[n], padding=1) + bd[n], a) * lam[0]
            dK.insert(0, h * torch.nn.grad.conv2d_weight(u[n], Kd[n].shape, s, padding=1))
            lam.insert(0, lam[0] + h * torch.nn.grad.conv2d_input(s.shape, Kd[n], s, padding=1))
        u, lam, dK = torch.stack(u), torch.stack(lam), torch.stack(dK)
        for record in (True, False):
            rec = L.alloc_dsig(p) if record else None
            gK, gb, ws = torch.empty_like(K), torch.empty_like(b), L.alloc_workspace(p)
            L.lp_serial_forward(p, K, b, U, dsig=rec)
            L.lp_serial_adjoint(p, K, b, U, Lam, dsig=rec)
            L.lp_gradient(p, K, b, U, Lam, gK, gb, ws, dsig=rec)
            # 72-term products over N layers (growth below 16), then sums over the pixels
            bound = 16 * N * (72 + 8) * EPS["f32"]
            for got, r, n in ((U, u, 0), (Lam, lam, 0), (gK, dK, B * H * W)):
                e = float((got.double().cpu() - r).norm() / r.norm())
                assert e <= bound + 4 * n * EPS["f32"], (a, record, e, bound)


# Residual norms on the matrix cores: a wave takes 16 examples, a workgroup 64 through a
# run of 1 to 8 layers (by ntiles N / 4096), the last run being shorter. Against the
# definition in 64 bits: an entry's error is at most (q + 8) u of its terms, which the
# states bound (h |K| < 1 here), so (q + 8) u (|V| + |M|) bounds the norm's.
@pytest.mark.parametrize("q", [32, 64])
@pytest.mark.parametrize("N,B", [(3, 1), (6, 17), (5, 64), (130, 129), (1027, 700), (1027, 2047)])
def test_dense_residual_runs(q, N, B):
    for a in ("tanh", "smoothrelu", "identity"):
        p, K, b, _, _ = dense_problem("f32", q, a, N, B, h=0.05)
        V, M = rnd(7, N + 1, B, q, dtype=torch.float32), rnd(8, N + 1, B, q, dtype=torch.float32)
        ws = L.alloc_workspace(p)
        rs = ra = 0.0
        for n in range(N):
            u, k = V[n].double(), K[n].double()
            z = u @ k.T.contiguous() + b[n].double()
            rs += float((u + 0.05 * act(z, a) - V[n + 1].double()).square().sum())
            lam = M[n + 1].double()
            ra += float((lam + 0.05 * (dact(z, a) * lam) @ k - M[n].double()).square().sum())
        scale = float(V.double().norm() + M.double().norm())
        for which, r in ((L.LP_STATE, rs), (L.LP_ADJOINT, ra)):
            got = L.lp_residual_norm(p, which, K, b, V, M, ws)
            assert abs(got - r ** 0.5) <= (q + 8) * EPS["f32"] * scale, (a, which)


# narrow widths: a wave takes 1 to 16 tiles of 16 examples (by N ceil(B/64) / 8192), the last
# run being ragged; the bound is that of the runs of layers above
@pytest.mark.parametrize("dtype,q", NARROW)
@pytest.mark.parametrize("N,B", [(1024, 1037), (64, 20011), (3, 190001)])
def test_narrow_residual_runs(dtype, q, N, B):
    for a in ("tanh", "smoothrelu"):
        p, K, b, _, _ = dense_problem(dtype, q, a, N, 1, h=0.05)
        p = L.problem(dtype, "dense", a, N, B, q, h=0.05)
        V, M = (rnd(k, N + 1, B, q, dtype=DT[dtype]) for k in (7, 8))
        ws, rs, ra = L.alloc_workspace(p), 0.0, 0.0
        for n in range(N):
            u, k, lam = V[n].double(), K[n].double(), M[n + 1].double()
            z = u @ k.T.contiguous() + b[n].double()
            rs += float((u + 0.05 * act(z, a) - V[n + 1].double()).square().sum())
            ra += float((lam + 0.05 * (dact(z, a) * lam) @ k - M[n].double()).square().sum())
        scale = float(V.double().norm() + M.double().norm())
        for which, r in ((L.LP_STATE, rs), (L.LP_ADJOINT, ra)):
            got = L.lp_residual_norm(p, which, K, b, V, M, ws)
            assert abs(got - r ** 0.5) <= (q + 8) * EPS[dtype] * scale, (a, which)


# the residual's tanh is accurate relative to its value, also near zero: a zero state and
# zero weights leave r = h tanh(b), whose norm is off by the few ulp of one tanh
@pytest.mark.parametrize("dtype,q", [("f32", 8), ("f32", 16), ("f32", 32), ("f32", 64), ("f32", 220), ("f64", 16)])
@pytest.mark.parametrize("size", [1e-6, 1e-3, 0.3])
def test_residual_of_small_tanh(dtype, q, size):
    N, B = 3, 50
    p = L.problem(dtype, "dense", "tanh", N, B, q, h=1.0)
    K, b = torch.zeros(N, q, q, device="cuda", dtype=DT[dtype]), rnd(1, N, q, dtype=DT[dtype], std=size)
    U = torch.zeros(N + 1, B, q, device="cuda", dtype=DT[dtype])
    got = L.lp_residual_norm(p, L.LP_STATE, K, b, U, None, L.alloc_workspace(p))
    ref = B ** 0.5 * float(torch.tanh(b.double()).norm())
    assert abs(got - ref) <= 8 * EPS[dtype] * ref


# one launch up to 8192 elements, partial sums above: fp64 sums of up to 2^17 products
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [0, 1, 1023, 1025, 8191, 8192, 8193, 131073])
def test_vec_dot_sizes(dtype, n):
    x, y = rnd(1, n, dtype=DT[dtype]), rnd(2, n, dtype=DT[dtype])
    out = torch.full((1 + L.LP_DOT_PARTIALS,), float("nan"), device="cuda", dtype=torch.float64)
    L.lp_vec_dot(x, y, out)
    ref = (x.double() * y.double()).cpu()
    assert abs(float(out[0]) - math.fsum(ref.tolist())) <= 32 * EPS["f64"] * float(ref.abs().sum())


# serial solves with the operands of 4 (width 32) or 1 and 2 (width 64) layers in flight:
# depths below, at and beside the rings' lengths; 16 examples per wave; weights through LDS
# above 4096 (width 64) and 8192 examples. The bound is the narrow layers' above.
@pytest.mark.parametrize("q", [32, 64])
@pytest.mark.parametrize("N,batches", [(1, (1, 16, 33)), (2, (33,)), (3, (33,)), (4, (33,)), (5, (4097, 8193)),
                                       (9, (33, 4096, 8193))])
def test_dense_serial_depths(q, N, batches):
    for B in batches:
        for a in ("tanh", "smoothrelu", "identity"):
            p, K, b, U, Lam = dense_problem("f32", q, a, N, B)
            L.lp_serial_forward(p, K, b, U)
            L.lp_serial_adjoint(p, K, b, U, Lam)
            ref = serial_reference(K, b, U, Lam, a, 0.05)
            rec = L.alloc_dsig(p) if L.lp_dsig_bytes(p) else None
            if rec is not None:  # other kernels by the same rule: the same states, the adjoint to rounding
                V, M = U.clone(), Lam.clone()
                V[1:] = M[:-1] = float("nan")
                L.lp_serial_forward(p, K, b, V, dsig=rec)
                L.lp_serial_adjoint(p, K, b, V, M, dsig=rec)
                assert torch.equal(V, U)
                assert float((M.double() - ref[1]).norm() / ref[1].norm()) <= 16 * N * (q + 8) * EPS["f32"], (a, B)
            for got, r in ((U, ref[0]), (Lam, ref[1])):
                e = float((got.double() - r).norm() / r.norm())
                assert e <= 16 * N * (q + 8) * EPS["f32"], (a, B, e)
