"""Infinite, NaN and very large operands in the families that run split bf16 products.
Width 220: results as fp32 arithmetic gives them, and the other examples' bits
untouched. The reference is the definition in 64 bits, rounded to 32 (products beyond
the range of fp32 become infinite in both). 3x3 convolutions: NaN, which nothing swallows."""
import pytest
import torch

from paper_1812_04352_amd import lp as L

pytestmark = pytest.mark.gpu
INF, BIG = float("inf"), 3.4e38  # BIG is finite in fp32 and beyond the largest bf16 value, 3.39e38


def act(z, a):
    if a == "tanh":
        return torch.tanh(z)
    return torch.where(z > 0, z, torch.zeros_like(z)) if a == "relu" else z


def dact(z, a):
    if a == "tanh":
        return 1.0 - torch.tanh(z) ** 2
    return (z > 0).to(z.dtype) if a == "relu" else torch.ones_like(z)


def f32(x):
    return x.float().double()


def same(got, ref, what):
    got, ref = got.double().cpu(), f32(ref).cpu()
    assert bool((got.isnan() == ref.isnan()).all()), what
    fin = ref.isfinite()
    assert bool((got[ref.isinf()] == ref[ref.isinf()]).all()), what
    if fin.any():
        assert float((got[fin] - ref[fin]).abs().max()) <= 1e-5 * float(ref[fin].abs().max()), what


def normal(seed, *shape, std=1.0):
    return torch.randn(*shape, generator=torch.Generator().manual_seed(seed)).mul_(std).cuda()


@pytest.mark.parametrize("where", ["state", "weight", "bias"])
@pytest.mark.parametrize("value", [INF, -INF, BIG, float("nan")])
@pytest.mark.parametrize("a", ["tanh", "relu", "identity"])
def test_wide_layers(a, value, where):
    N, B, q, h = 1, 40, 220, 0.5
    p = L.problem("f32", "dense", a, N, B, q, h=h)
    # (small weights beside BIG, so that no sum overflows on the way)
    K, b = normal(1, N, q, q, std=1e-4 if value == BIG else 0.05), normal(2, N, q, std=0.1)
    U0, LN = normal(3, B, q), normal(4, B, q)
    bad = torch.zeros(B, dtype=torch.bool)
    if where == "state":
        U0[17, 219] = value
        LN[21, 3] = value
        bad[17] = bad[21] = True
    elif where == "weight":
        K[0, 33, 0] = value
        bad[:] = True
    else:
        b[0, 7] = value
        bad[:] = True

    def solve(U0, LN, record):
        U, Lam = torch.zeros(N + 1, B, q, device="cuda"), torch.zeros(N + 1, B, q, device="cuda")
        U[0], Lam[N] = U0, LN
        rec = L.alloc_dsig(p) if record and L.lp_dsig_bytes(p) else None
        L.lp_serial_forward(p, K, b, U, dsig=rec)
        L.lp_serial_adjoint(p, K, b, U, Lam, dsig=rec)
        return U, Lam

    Kd, bd, u, lam = K[0].double().cpu(), b[0].double().cpu(), U0.double().cpu(), LN.double().cpu()
    z = f32(u @ Kd.T) + bd
    ref = f32(u + h * act(z, a))
    s = f32(dact(z, a) * lam)
    adj = f32(lam + h * f32(s @ Kd))
    for record in (True, False):
        U, Lam = solve(U0, LN, record)
        same(U[1], ref, ("state", record))
        same(Lam[0], adj, ("adjoint", record))
        if where == "state":  # the other examples' results are those of a batch without such values
            Uf, Lf = solve(torch.where(U0.isfinite() & (U0.abs() < 1e38), U0, 0), torch.where(LN.isfinite() & (LN.abs() < 1e38), LN, 0), record)
            assert torch.equal(U[1][~bad.cuda()], Uf[1][~bad.cuda()])
            assert torch.equal(Lam[0][~bad.cuda()], Lf[0][~bad.cuda()])
    # a residual with such a value is reported, not passed over
    if where == "state" and value != BIG:
        with pytest.raises(L.LpError) as e:
            L.lp_residual_norm(p, L.LP_STATE, K, b, solve(U0, LN, False)[0], None, L.alloc_workspace(p))
        assert e.value.status == L.LP_ENONFINITE
        with pytest.raises(L.LpError):  # clear the device's flag
            L.lp_check_finite()


# A split product with an operand that is not finite, or beyond the largest bf16 value, is
# NaN, and the state shows it with every activation (also ReLU, which gives 0 for NaN by
# comparison): the residual reports it. The image's own pixels beside it, and the other
# images' bits, are untouched.
@pytest.mark.parametrize("where", ["state", "weight"])
@pytest.mark.parametrize("value", [INF, -INF, BIG, float("nan")])
@pytest.mark.parametrize("a", ["tanh", "relu", "smoothrelu", "identity"])
@pytest.mark.parametrize("H,W", [(28, 28), (12, 13)])
def test_conv_layers(H, W, a, value, where):
    N, B, C = 1, 5, 8
    p = L.problem("f32", "conv3x3", a, N, B, C, H, W, h=0.5)
    K, b = normal(1, N, C, C, 3, 3, std=0.1), normal(2, N, C, std=0.1)
    U0, LN = normal(3, B, C, H, W), normal(4, B, C, H, W)
    U0f, LNf = U0.clone(), LN.clone()
    y, x = H // 2, W // 2
    if where == "state":
        U0[1, 5, y, x] = value
        LN[3, :, y, x] = value  # (in every channel: sigma' may be zero in some)
    else:
        K[0, 6, 1, 1, 1] = value

    def solve(U0, LN, record):
        U, Lam = torch.zeros(N + 1, B, C, H, W, device="cuda"), torch.zeros(N + 1, B, C, H, W, device="cuda")
        U[0], Lam[N] = U0, LN
        rec = L.alloc_dsig(p) if record and L.lp_dsig_bytes(p) else None
        L.lp_serial_forward(p, K, b, U, dsig=rec)
        L.lp_serial_adjoint(p, K, b, U, Lam, dsig=rec)
        return U, Lam

    ws = L.alloc_workspace(p)
    for record in (True, False):
        U, Lam = solve(U0, LN, record)
        if where == "state":  # the 3 x 3 pixels around it, all channels; and no pixel four rows or two columns away
            assert not U[1, 1, :, y - 1:y + 2, x - 1:x + 2].isfinite().any()
            assert U[1, 1, :, :y - 4].isfinite().all() and U[1, 1, :, :, x + 2:].isfinite().all()
            assert value == BIG or not Lam[0, 3, :, y, x].isfinite().any()
            Uf, Lf = solve(U0f, LNf, record)
            for got, ref, others in ((U[1], Uf[1], [0, 2, 3, 4]), (Lam[0], Lf[0], [0, 2, 4])):
                assert torch.equal(got[others], ref[others])
        else:  # the channel that the weight feeds
            assert not U[1, :, 6].isfinite().any() and U[1, :, [0, 1, 2, 3, 4, 5, 7]].isfinite().all()
            assert value == BIG or not Lam[0, :, 1].isfinite().all()
        for which in (L.LP_STATE, L.LP_ADJOINT)[:1 if value == BIG else 2]:  # (sigma' times BIG may be in range)
            with pytest.raises(L.LpError) as e:
                L.lp_residual_norm(p, which, K, b, U, Lam, ws)
            assert e.value.status == L.LP_ENONFINITE
    with pytest.raises(L.LpError):  # clear the device's flag
        L.lp_check_finite()
