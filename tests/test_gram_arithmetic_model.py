"""Arithmetic of the Gram route against Eq. 2's products in bf16, as a model on the CPU (matrices rounded to 16 bits where the kernels store
them, fp32 sums): the first iteration in bf16 and groups of two in f16 are closer to 64 bits than the products as they are written in bf16,
on inputs of full rank and on inputs that fill a few directions only."""
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


def exact(u, steps=5):
    x = u.double() / u.double().norm()
    for _ in range(steps):
        g = x @ x.T
        x = A * x + (B * g + C * (g @ g)) @ x
    return x


def written(x, s, steps=5):
    eye = torch.eye(len(x))
    for k in range(steps):
        g = bf16((x @ x.T) * (s * s if k == 0 else 1.0))
        x = bf16(bf16(B * g + C * (g @ g) + A * eye) @ x * (s if k == 0 else 1.0))
    return x


def gram_route(x, s, mirror=mirrored, steps=5):
    """A product is L R^T and takes its addend transposed, as in the kernels: the same unless a matrix is not quite symmetric."""
    eye = torch.eye(len(x))
    g = bf16((x @ x.T) * (s * s))
    x = f16(bf16(B * g + C * (g @ g) + A * eye) @ x * s, SCALE_X)
    left = steps - 1
    while left:
        group = min(left, 2)
        left -= group
        g = f16(x @ x.T, SCALE_A)
        q = f16(B * g.T + C * (g @ g.T) + A * eye, SCALE_P)
        if group == 2:
            g = mirror(f16(mirror(f16(q @ g.T, SCALE_A)) @ q.T, SCALE_A))
            q = mirror(f16(A * q.T + f16(B * g.T + C * (g @ g.T), SCALE_P) @ q.T, SCALE_P))
        x = q @ x
        x = f16(x, SCALE_X) if left else bf16(x)
    return x


def matrix(kind, m, n, seed):
    gen = torch.Generator().manual_seed(seed)
    u = torch.randn(m, n, generator=gen)
    if kind == "outliers":
        return torch.where(torch.rand(m, n, generator=gen) < 0.01, 100.0 * u, u)
    if kind == "decay":                                          # singular values that fall like 1 / i
        a, _, b = torch.linalg.svd(u, full_matrices=False)
        return (a / torch.arange(1, m + 1)) @ b
    if kind.startswith("columns"):                               # zero outside the first few columns
        few = int(kind[len("columns"):])
        return torch.cat([u[:, :few], torch.zeros(m, n - few)], 1)
    if kind == "equal columns":
        return u[:, :1].expand(m, n).contiguous()
    if kind == "fading columns":                                 # scales that fall over ten decades
        return u * torch.logspace(0, -10, n)
    return u


@pytest.mark.parametrize("steps", [4, 5, 10])
@pytest.mark.parametrize("kind", ["gauss", "outliers", "decay", "columns1", "columns2", "columns16", "columns48", "columns96", "equal columns",
                                  "fading columns"])
@pytest.mark.parametrize("m,n", [(128, 512), (256, 1024), (384, 3072)])     # (the route's smallest: 384 x 3072)
def test_the_route_is_closer_to_64_bits(kind, m, n, steps):
    u = matrix(kind, m, n, 31 + m)
    ref, x, s = exact(u, steps), bf16(u), 1.0 / float(u.norm())
    err = [float((o.double() - ref).norm() / ref.norm()) for o in (written(x, s, steps), gram_route(x, s, steps=steps))]
    print(kind, m, n, steps, err)
    assert err[1] <= err[0]
    assert kind == "decay" or err[1] < 0.75 * err[0]


@pytest.mark.parametrize("kind", ["gauss", "columns16"])
def test_the_mirrored_triangle_costs_little(kind):
    """T, A and Q are symmetric up to rounding.  One triangle is put in the place of the other so that a result does not depend on the
    tile that holds it; left as they are they would be no closer on inputs of full rank, and a third closer where errors repeat."""
    u = matrix(kind, 256, 1024, 3)
    ref, x, s = exact(u), bf16(u), 1.0 / float(u.norm())
    err = [float((o.double() - ref).norm() / ref.norm()) for o in (written(x, s), gram_route(x, s), gram_route(x, s, mirror=lambda v: v))]
    print(err)
    assert err[1] < 1.5 * err[2] and err[1] < 0.75 * err[0]
