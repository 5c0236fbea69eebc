"""The precision of the split bf16 products (width 220, 3x3 convolutions): no less than
that of an fp32 sum, which rounds with every product as the fp32 matrix instructions do,
and without a bias over the layers.

A layer of the identity with a long step shows its product: U1 = U0 + h z with h z far
above U0. The fp32 sum is formed here, one product after the other, and passes through the
same last step."""
import pytest
import torch

from paper_1812_04352_amd import lp as L

pytestmark = pytest.mark.gpu
H_LONG = 2.0 ** 20


def normal(seed, *shape, std=1.0):
    return torch.randn(*shape, generator=torch.Generator().manual_seed(seed)).mul_(std).cuda()


def solve(layer, K, u, C, H, W, adjoint):
    p = L.problem("f32", layer, "identity", 1, u.shape[0], C, H, W, h=H_LONG)
    b = torch.zeros(1, C, device="cuda")
    X = torch.zeros(2, *u.shape, device="cuda")
    if adjoint:
        X[1] = u
        L.lp_serial_adjoint(p, K, b, torch.zeros_like(X), X)
        return X[0]
    X[0] = u
    L.lp_serial_forward(p, K, b, X)
    return X[1]


def error(x1, u, z):
    return float(((x1.double() - u.double()) / H_LONG - z).norm() / z.norm())


def last_step(u, z32):
    return (u.double() + H_LONG * z32.double()).float()


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("positive", [False, True])
def test_wide_product_against_fp32_sums(adjoint, positive):
    q, B = 220, 300
    K, u = normal(1, 1, q, q, std=0.1), normal(2, B, q)
    if positive:
        K, u = K.abs(), u.abs()
    A = K[0].T.contiguous() if adjoint else K[0]
    z = u.double() @ A.double().T.contiguous()
    acc = torch.zeros(B, q, device="cuda")
    for k in range(q):
        acc = (acc.double() + u[:, k:k + 1].double() * A[:, k].double()).float()
    got = error(solve("dense", K, u, q, 1, 1, adjoint), u, z)
    ref = error(last_step(u, acc), u, z)
    assert got <= 1.05 * ref, (got, ref)
    assert got <= 4e-7


def taps(x):
    H, W = x.shape[-2:]
    pad = torch.nn.functional.pad(x, (1, 1, 1, 1))
    return [pad[..., i:i + H, j:j + W] for i in range(3) for j in range(3)]


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("H,W", [(28, 28), (12, 13)])
def test_conv_product_against_fp32_sums(H, W, adjoint, positive):
    B, C = 8, 8
    K, u = normal(1, 1, C, C, 3, 3, std=0.1), normal(2, B, C, H, W)
    if positive:
        K, u = K.abs(), u.abs()
    A = K[0].flip(2, 3).transpose(0, 1).contiguous() if adjoint else K[0]
    z, acc = 0.0, torch.zeros(B, C, H, W, device="cuda")
    for c in range(C):
        for t, x in enumerate(taps(u)):
            part = x[:, c:c + 1].double() * A[:, c, t // 3, t % 3].double()[None, :, None, None]
            z = z + part
            acc = (acc.double() + part).float()
    got = error(solve("conv3x3", K, u, C, H, W, adjoint), u, z)
    ref = error(last_step(u, acc), u, z)
    assert got <= 1.05 * ref, (got, ref)
    assert got <= 3e-7


# The matrix instruction's accumulation rounds towards minus infinity, and the layers' signs
# cancel it: the mean over layers and values of the increments' relative error. Without the
# signs it is -8.7e-9 at width 220. (The rounding of the state itself is unbiased, 1e-6 of
# an increment: 5e-10 in the mean of three million values.)
@pytest.mark.parametrize("layer,N,B,C,H,W,most", [("dense", 64, 200, 220, 1, 1, 2e-9), ("conv3x3", 64, 40, 8, 28, 28, 1e-9)])
def test_layers_have_no_common_bias(layer, N, B, C, H, W, most):
    conv = layer == "conv3x3"
    p = L.problem("f32", layer, "identity", N, B, C, H, W, h=1.0)
    K = normal(1, *((N, C, C, 3, 3) if conv else (N, C, C))).abs()
    K *= 0.1 / K.flatten(2).sum(2).mean() / (1 if not conv else C) * (C if conv else 1)
    b = torch.zeros(N, C, device="cuda")
    U = torch.zeros(N + 1, B, C, H, W, device="cuda") if conv else torch.zeros(N + 1, B, C, device="cuda")
    U[0] = normal(2, *U.shape[1:]).abs() + 0.5
    L.lp_serial_forward(p, K, b, U)
    mean = []
    for n in range(N):
        u = U[n].double()
        if conv:
            z = sum(torch.tensordot(x, K[n, :, :, t // 3, t % 3].double(), ([1], [1])).permute(0, 3, 1, 2)
                    for t, x in enumerate(taps(u)))
        else:
            z = u @ K[n].double().T.contiguous()
        mean.append(float(((U[n + 1].double() - u) / z - 1.0).mean()))
    mean = torch.tensor(mean, dtype=torch.float64)
    assert abs(float(mean.mean())) <= most
