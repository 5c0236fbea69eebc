"""Kernels behind a rule on sizes, each at the sizes where it can go wrong (edges
of its tiles, remainders, the smallest and largest of its range), against plain
torch in 64 bits on the same rounded inputs.

Tolerances are relative to the sums of absolute values: a sum of n products in
working precision u, in any order, is within (n + 2) u of that; the bounds below
use that with a factor 4 for the activation and the operand that feeds it.
"""
import pytest
import torch

from paper_1812_04352_amd import lp as L

pytestmark = pytest.mark.gpu
U = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}
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


# tiles of 32 x 32 with 512-byte pieces of the features (forward); tiles of 4 .. 128
# examples by feature count and 1024 threads (gradient)
@pytest.mark.parametrize("dtype,act_name,B,q,nf", [
    ("f32", "tanh", 1, 8, 1), ("f32", "relu", 31, 16, 2), ("f32", "smoothrelu", 33, 32, 127), ("f32", "tanh", 129, 32, 128),
    ("f32", "identity", 100, 64, 129), ("f32", "tanh", 257, 220, 220), ("f32", "tanh", 70, 8, 513),
    ("f32", "tanh", 37, 8, 1023), ("f32", "relu", 1500, 32, 1024),
    ("f64", "tanh", 1, 8, 1), ("f64", "smoothrelu", 65, 16, 63), ("f64", "tanh", 257, 32, 65), ("f64", "tanh", 33, 8, 1024),
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
    within(u0, act(z, act_name), za + 0.025, 4 * (nf + 8) * U[dtype], "u0")
    s = dact(z, act_name) * lam
    # sigma' changes by at most 5 |dz|; a ReLU site within rounding of zero may go either way
    scale = (lam.abs() * (1.0 + 5.0 * za)).T.contiguous() @ y.abs()
    bound = 4 * (nf + B + 8) * U[dtype]
    if act_name == "relu":
        open_sites = (z.abs() <= 4 * (nf + 8) * U[dtype] * za).double() * lam.abs()
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
    within(dL.reshape(8, 9), ref, scale, 4 * (9 + 8 + 32) * U["f32"], "dL")


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
        within(got, ref, s, 2 * U["f32"], "head")  # summed in fp64, rounded once
    assert float(acc) == float((z.argmax(1) == c.argmax(1)).double().mean())
