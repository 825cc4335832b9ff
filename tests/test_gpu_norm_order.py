"""The sum of squares behind the Frobenius norm is added up in an order that belongs to the matrix, not to the way a kernel
distributes the matrix over its threads: the norm's last bits decide bf16 roundings of the whole iteration, so a new
distribution must not make another result.  The order, per 64 x 64 tile: 16 consecutive columns of a row are a chain of
fp32 fma; the 64 chains of 16 consecutive rows (four of a row side by side) are a tree, the farthest added first; the
four results (0 + 1) + (2 + 3).  The tiles' sums are added in double."""
import numpy as np
import pytest
import torch

from paper_2502_16982_amd import binding

pytestmark = pytest.mark.gpu

EPS = 1e-7


def fma32(a, b, c):
    # the product of two fp32 values is exact in 64 mantissa bits
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(np.float32)


def tile_sum(t):
    """t: 64 x 64 fp32, zero beyond the matrix."""
    t = t.reshape(64, 4, 16)
    c = np.zeros((64, 4), np.float32)
    for i in range(16):
        c = fma32(t[:, :, i], t[:, :, i], c)
    v = c.reshape(4, 64)
    while v.shape[1] > 1:
        half = v.shape[1] // 2
        v = v[:, :half] + v[:, half:]
    v = v[:, 0]
    return (v[0] + v[1]) + (v[2] + v[3])


def norm_scalar(u):
    rows, cols = u.shape
    pad = np.zeros((-(-rows // 64) * 64, -(-cols // 64) * 64), np.float32)
    pad[:rows, :cols] = u
    parts = [tile_sum(pad[r:r + 64, c:c + 64]) for r in range(0, pad.shape[0], 64) for c in range(0, pad.shape[1], 64)]
    assert len(parts) <= 256
    v = np.zeros(256)
    v[:len(parts)] = parts
    while len(v) > 1:
        v = v[:len(v) // 2] + v[len(v) // 2:]
    return np.float32(1.0 / (np.sqrt(v[0]) + EPS))


@pytest.mark.parametrize("g_dtype", [torch.float32, torch.bfloat16])
def test_norm_is_summed_in_the_stated_order(g_dtype):
    dev = torch.device("cuda:0")
    gen = torch.Generator().manual_seed(97)
    shapes = [(64, 64)] * 24 + [(1, 70), (70, 1), (63, 65), (100, 130), (130, 100), (257, 511), (512, 320), (33, 1000)]
    tensors, u = [], []
    for shape in shapes:
        g = (torch.randn(shape, generator=gen) * torch.exp(torch.randn(shape, generator=gen))).to(g_dtype)
        g[0, 0] = 1.0                                          # O there is the scalar itself
        u.append(g.float().numpy())
        tensors.append((torch.zeros(shape, device=dev), g.to(dev), torch.zeros(shape, device=dev)))
    # no iteration: O = U / (||U|| + eps) as it is stored, U = G (zero momentum)
    st = binding.MuonStepper(tensors, ns_dtype="f32")
    st.step(binding.default_hparams(lr=0.0, weight_decay=0.0, nesterov=0, ns_steps=0, eps=EPS))
    torch.cuda.synchronize()
    got = [st.read_update(i)[0, 0].item() for i in range(len(shapes))]
    st.close()
    want = [float(norm_scalar(x)) for x in u]
    wrong = [(s, a, b) for s, a, b in zip(shapes, got, want) if a != b]
    assert not wrong, (len(wrong), wrong[:4])
