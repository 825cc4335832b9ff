"""Arithmetic of the Gram route against Eq. 2's products in bf16, as a model on the CPU (matrices rounded to 16 bits where the kernels store
them, fp32 sums): groups of two and three iterations in f16 are closer to 64 bits than the products as they are written in bf16."""
import pytest
import torch

A, B, C = 3.4445, -4.7750, 2.0315
SCALE_A, SCALE_P, SCALE_X = 2.0 ** 13, 2.0 ** 9, 2.0 ** 13       # as in muon_plan.h


def bf16(x):
    return x.bfloat16().float()


def f16(x, scale):
    return (x * scale).half().float() / scale


def mirrored(x):
    return torch.triu(x) + torch.triu(x, 1).T


def exact(u):
    x = u.double() / u.double().norm()
    for _ in range(5):
        g = x @ x.T
        x = A * x + (B * g + C * (g @ g)) @ x
    return x


def written(x, s):
    eye = torch.eye(len(x))
    for k in range(5):
        g = bf16((x @ x.T) * (s * s if k == 0 else 1.0))
        x = bf16(bf16(B * g + C * (g @ g) + A * eye) @ x * (s if k == 0 else 1.0))
    return x


def gram_route(x, s, groups=(2, 3), mirror=mirrored):
    """A product is L R^T and takes its addend transposed, as in the kernels: the same unless a matrix is not quite symmetric."""
    eye = torch.eye(len(x))
    for n, steps in enumerate(groups):
        first, last = n == 0, n == len(groups) - 1
        g = f16((x @ x.T) * (s * s if first else 1.0), SCALE_A)
        q = p = f16(B * g.T + C * (g @ g.T) + A * eye, SCALE_P)
        g = mirror(f16(mirror(f16(p @ g.T, SCALE_A)) @ p.T, SCALE_A))
        for j in range(1, steps):
            d = f16(B * g.T + C * (g @ g.T), SCALE_P)
            q = A * q.T + d @ q.T
            q = mirror(bf16(q) if first and j == steps - 1 else f16(q, SCALE_P))
            if j < steps - 1:
                t = mirror(f16(A * g.T + d @ g.T, SCALE_A))
                g = mirror(f16(A * t.T + t @ d.T, SCALE_A))
        x = q @ x * (s if first else 1.0)
        x = bf16(x) if last else f16(x, SCALE_X)
    return x


def matrix(kind, m, n, seed):
    gen = torch.Generator().manual_seed(seed)
    u = torch.randn(m, n, generator=gen)
    if kind == "outliers":
        return torch.where(torch.rand(m, n, generator=gen) < 0.01, 100.0 * u, u)
    if kind == "decay":                                          # singular values that fall like 1 / i
        a, _, b = torch.linalg.svd(u, full_matrices=False)
        return (a / torch.arange(1, m + 1)) @ b
    return u


@pytest.mark.parametrize("kind", ["gauss", "outliers", "decay"])
@pytest.mark.parametrize("m,n", [(128, 512), (256, 1024), (384, 3072)])     # (the route's smallest: 384 x 3072)
def test_the_route_is_closer_to_64_bits(kind, m, n):
    u = matrix(kind, m, n, 31 + m)
    ref, x, s = exact(u), bf16(u), 1.0 / float(u.norm())
    err = [float((o.double() - ref).norm() / ref.norm()) for o in (written(x, s), gram_route(x, s))]
    print(kind, m, n, err)
    assert err[1] <= err[0]
    assert kind == "decay" or err[1] < 0.75 * err[0]


def test_groups_need_a_symmetric_gram_matrix():
    """Without the mirrored triangle the asymmetry that rounding leaves in T and A is amplified by every further iteration."""
    u = matrix("gauss", 256, 1024, 3)
    ref, x, s = exact(u), bf16(u), 1.0 / float(u.norm())
    err = [float((gram_route(x, s, mirror=m).double() - ref).norm() / ref.norm()) for m in (mirrored, lambda v: v)]
    print(err)
    assert err[0] < 5e-3 and err[1] > 2 * err[0]
