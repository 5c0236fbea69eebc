"""A ReLU site within rounding of zero is decided once: in the families that run split
bf16 products (3x3 convolutions, width 220) every kernel that evaluates a layer forms
its pre-activation with the same arithmetic, so the gradient that recomputes sigma'
agrees bit for bit with the one that reads the solve's record. The gradient of a dense
opening decides its sites as the opening layer did."""
import pytest
import torch

from paper_1812_04352_amd import lp as L

pytestmark = pytest.mark.gpu


def near_zero(K, u, last):
    """u with its last feature (or channel) set so that the first output's products sum to zero."""
    u[:, last] = 0.0
    k = K[0].double().flatten(1).sum(1) if K.dim() == 4 else K[0].double()
    u[:, last] = (-(u.double().flatten(2)[..., 0] if u.dim() == 4 else u.double()) @ k / k[last]).to(u.dtype).reshape(
        (-1,) + (1,) * (u.dim() - 2))
    return u


# images constant per channel: an inner pixel's pre-activation is the sum of u_c times
# the sum of the nine weights, which the last channel cancels to rounding
@pytest.mark.parametrize("H,W", [(28, 28), (12, 13), (20, 27)])
def test_conv_gradient_decides_sites_as_the_solve(H, W):
    g = torch.Generator(device="cuda").manual_seed(3)
    B, C = 256, 8
    p = L.problem("f32", "conv3x3", "relu", 1, B, C, H, W, h=2.0 ** 20)
    K, b = torch.randn(1, C, C, 3, 3, generator=g, device="cuda"), torch.zeros(1, C, device="cuda")
    U, Lam = torch.zeros(2, B, C, H, W, device="cuda"), torch.randn(2, B, C, H, W, generator=g, device="cuda")
    U[0] = near_zero(K[0], torch.randn(B, C, 1, 1, generator=g, device="cuda"), C - 1)
    ws, rec = L.alloc_workspace(p), L.alloc_dsig(p)
    L.lp_serial_forward(p, K, b, U, dsig=rec)
    # the step is long, so that relu(z) shows beside the state
    z = (U[1, :, 0, 1:-1, 1:-1] - U[0, :, 0, 1:-1, 1:-1]).amax((1, 2)) / 2.0 ** 20
    assert float(z.max()) < 1e-4 and 0.02 < float((z > 0).double().mean()) < 0.98  # the sites are at zero
    out = []
    for r in (rec, None):
        dK, db = torch.empty_like(K), torch.empty_like(b)
        L.lp_gradient(p, K, b, U, Lam, dK, db, ws, dsig=r)
        out.append((dK, db))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_wide_gradient_decides_sites_as_the_solve():
    q = 220
    g = torch.Generator(device="cuda").manual_seed(4)
    B = 512
    p = L.problem("f32", "dense", "relu", 1, B, q, h=2.0 ** 20)
    K, b = torch.randn(1, q, q, generator=g, device="cuda"), torch.zeros(1, q, device="cuda")
    U, Lam = torch.zeros(2, B, q, device="cuda"), torch.randn(2, B, q, generator=g, device="cuda")
    U[0] = near_zero(K[0], torch.randn(B, q, generator=g, device="cuda"), q - 1)
    ws, rec = L.alloc_workspace(p), L.alloc_dsig(p)
    L.lp_serial_forward(p, K, b, U, dsig=rec)
    z = (U[1, :, 0] - U[0, :, 0]) / 2.0 ** 20
    assert float(z.max()) < 1e-3 and 0.02 < float((z > 0).double().mean()) < 0.98
    out = []
    for r in (rec, None):
        dK, db = torch.empty_like(K), torch.empty_like(b)
        L.lp_gradient(p, K, b, U, Lam, dK, db, ws, dsig=r)
        out.append((dK, db))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


# an example per thread (nf <= 8), then 1, 2, 4, 8, 16 features per lane
@pytest.mark.parametrize("dtype,nf", [("f32", 7), ("f32", 9), ("f32", 64), ("f32", 100), ("f32", 220), ("f32", 512),
                                      ("f32", 1024), ("f64", 16), ("f64", 130)])
def test_opening_gradient_decides_sites_as_the_layer(dtype, nf):
    g = torch.Generator(device="cuda").manual_seed(5)
    dt, B, q = {"f32": torch.float32, "f64": torch.float64}[dtype], 500, 8
    p = L.problem(dtype, "dense", "relu", 1, B, q)
    y, Lw, lam = (torch.randn(*s, generator=g, device="cuda", dtype=torch.float64).to(dt) for s in ((B, nf), (q, nf), (B, q)))
    y[:, -1] = 0.0
    y[:, -1] = (-(y.double() @ Lw[0].double()) / Lw[0, -1].double()).to(dt)  # the first row's z is zero to rounding
    u0, dL = torch.empty(B, q, device="cuda", dtype=dt), torch.empty_like(Lw)
    L.lp_open_forward(p, L.LP_OPEN_DENSE_ACT, nf, y, Lw, u0)
    L.lp_open_grad(p, L.LP_OPEN_DENSE_ACT, nf, y, Lw, lam, dL)
    assert 0.02 < float((u0[:, 0] > 0).double().mean()) < 0.98  # the sites are at zero
    s = (u0 > 0).double() * lam.double()
    ref, scale = s.T.contiguous() @ y.double(), s.abs().T.contiguous() @ y.double().abs()
    # products and at most 8 terms at a time in the type, the rest in 64 bits (B terms)
    bound = 16 * torch.finfo(dt).eps + B * 2.0 ** -52
    assert float(((dL.double() - ref).abs() / (scale + 1e-300)).max()) <= bound
