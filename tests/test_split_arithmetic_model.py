"""Where the split-bf16 tolerances come from: a numpy model of the arithmetic (every iterate and temporary kept as p bf16
planes, every product of Eq. 2 taken over the plane pairs i + j < p - with two planes the polynomial takes the pair (1,1) as
well, whole or in the tile's own pieces of K -, summed in fp32 in the kernels' orders, results formed in fp32 and split
again), run against the fp64 oracle.  No GPU and no library code is involved; the model states what the library's rounding
points are, the parity tests check that the library stays inside the same bars."""
import numpy as np
import pytest

from oracle import muon_oracle as orc

A_, B_, C_ = 3.4445, -4.7750, 2.0315


def bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


def split(x, planes):
    rest, out = np.asarray(x, np.float32).copy(), []
    for _ in range(planes):
        h = bf16(rest)
        out.append(h.astype(np.float64))
        rest = (rest - h).astype(np.float32)          # exact: the rounding error of an fp32 value is an fp32 value
    return out


def product(left, right, planes):
    acc = np.zeros((left[0].shape[0], right[0].shape[0]))
    for i in range(planes):
        for j in range(planes - i):
            acc += left[i] @ right[j].T
    return acc


def product_in_order(left, right, planes, order):
    """The same in fp32, 16 terms of K at a time: "one": one accumulator takes the pairs piece of 64 by piece, plane 0 first;
    "three": the leading pair in two, of even and odd pieces, the other pairs in a third; "pair by pair": one accumulator
    takes the whole K of a pair at a time, the smallest pairs first."""
    k = left[0].shape[1]
    acc = np.zeros((3, left[0].shape[0], right[0].shape[0]), np.float32)
    pairs = sorted(((i, j) for i in range(planes) for j in range(planes - i)), key=lambda ij: max(ij))
    def add(c, i, j, k0):
        acc[c] += (left[i][:, k0:k0 + 16] @ right[j][:, k0:k0 + 16].T).astype(np.float32)
    if order == "pair by pair":
        for i, j in sorted(pairs, key=lambda ij: -sum(ij)):
            for k0 in range(0, k, 16):
                add(0, i, j, k0)
        return acc[0].astype(np.float64)
    for piece in range(0, k, 64):
        for i, j in pairs:
            c = 0 if order == "one" else piece // 64 % 2 if i + j == 0 else 2
            for k0 in range(piece, min(piece + 64, k), 16):
                add(c, i, j, k0)
    return acc[2].astype(np.float64) + (acc[0] + acc[1]).astype(np.float64)


def pair_11(a1, own):
    """The pair (1,1) of the polynomial: whole, or only over the k in the rows' and the columns' own tile of side `own`."""
    if own is None:
        return a1 @ a1
    tile = np.arange(len(a1)) // own
    block = np.where(tile[:, None] == tile[None, :], a1, 0.0)
    twice = block @ a1 + a1 @ block
    return np.where(tile[:, None] == tile[None, :], twice / 2, twice)


def model(u, planes, steps=5, pair="whole", multiply=None):
    multiply = multiply or product
    s = 1.0 / np.linalg.norm(u)
    x = split(u, planes)                               # stored un-normalised; s enters in the first two epilogues
    for it in range(steps):
        s2, s1 = (s * s, s) if it == 0 else (1.0, 1.0)
        a = split((s2 * multiply(x, x, planes)).astype(np.float32), planes)
        aa = multiply(a, a, planes)
        if planes == 2 and pair != "left out":
            aa = aa + pair_11(a[1], None if pair == "whole" else pair)
        b = split((C_ * aa + B_ * sum(a)).astype(np.float32), planes)
        xt = [p.T for p in x]
        x = split((s1 * (multiply(b, xt, planes) + A_ * sum(x))).astype(np.float32), planes)
    return sum(x)


@pytest.mark.parametrize("shape", [(96, 160), (128, 256), (256, 512)])
def test_error_level_of_each_plane_count(shape):
    rng = np.random.default_rng(shape[0])
    u = bf16(rng.standard_normal(shape) * 1e-3).astype(np.float64)
    ref = orc.newton_schulz(u, steps=5)
    err = {p: np.linalg.norm(model(u, p) - ref) / np.linalg.norm(ref) for p in (1, 2, 3)}
    assert 3e-3 < err[1] < 2e-2          # plain bf16: the 2e-2 bar
    assert 3e-6 < err[2] < 6e-5          # two planes: below the 1e-4 bar with room for fp32 accumulation order
    assert err[3] < 1e-6                 # three planes: fp32-class; the library's 1e-5 bar is set by its fp32 sums
    assert err[2] < err[1] / 100 and err[3] < err[2] / 30


def test_dropping_a_cross_term_is_visible():
    """The pair list matters: with two planes and only the hi*hi product the result is no better than plain bf16."""
    rng = np.random.default_rng(5)
    u = bf16(rng.standard_normal((96, 160)) * 1e-3).astype(np.float64)
    ref = orc.newton_schulz(u, steps=5)

    def hi_only(left, right, planes):
        return left[0] @ right[0].T

    global product
    full = product
    try:
        product = hi_only
        crippled = np.linalg.norm(model(u, 2) - ref) / np.linalg.norm(ref)
    finally:
        product = full
    assert crippled > 2e-3


def relative_errors(shape, models):
    """Root mean square over seeds of each model's relative error."""
    total = np.zeros(len(models))
    for seed in range(3):
        rng = np.random.default_rng(100 * seed + shape[0])
        u = bf16(rng.standard_normal(shape) * 1e-3).astype(np.float64)
        ref = orc.newton_schulz(u, steps=5)
        total += [(np.linalg.norm(m(u) - ref) / np.linalg.norm(ref)) ** 2 for m in models]
    return np.sqrt(total / 3)


@pytest.mark.parametrize("shape", [(128, 256), (256, 256), (192, 420), (320, 704), (63, 1030)])
def test_own_pieces_hold_what_the_pair_11_is_worth(shape):
    """Two planes: leaving (1,1) out of the polynomial costs up to half of the error again (most where the spectrum is narrow,
    so that A is nearly a multiple of the identity).  The part of its sums that does not average is in the diagonal of A: taken
    over an eighth of the matrix, the pieces of the tile's own rows and columns, the pair is worth what it is worth whole."""
    side = max(8, shape[0] // 8)
    out, whole, own = relative_errors(shape, [lambda u: model(u, 2, pair="left out"), lambda u: model(u, 2),
                                              lambda u: model(u, 2, pair=side)])
    assert whole < 1.002 * out and abs(own - whole) < 0.02 * whole
    if shape[1] > 1.5 * shape[0] and shape[0] > 128:
        assert out > 1.1 * whole and out > 1.1 * own


@pytest.mark.parametrize("planes,shape", [(2, (128, 256)), (2, (96, 1024)), (3, (96, 320))])
def test_order_of_the_terms(planes, shape):
    """fp32 sums in any of the kernels' orders: two planes within 2 % of exact sums, three planes within a third of their
    bar, where three accumulators are never worse than one."""
    err = relative_errors(shape, [lambda u: model(u, planes)] + [
        lambda u, order=order: model(u, planes, multiply=lambda l, r, p: product_in_order(l, r, p, order))
        for order in ("one", "three", "pair by pair")])
    if planes == 2:
        assert (abs(err[1:] - err[0]) < 0.02 * err[0]).all(), err
    else:
        assert (err[1:] < 3e-6).all() and err[2] <= err[1], err
