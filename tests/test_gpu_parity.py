"""GPU parity: the HIP library, called through its C ABI, against the fp64 oracle on the same seeded
buffers.  Tolerances: relative Frobenius error of O <= 1e-4 (fp32 Newton-Schulz) / <= 2e-2 (bf16
Newton-Schulz with fp32 accumulation); momentum and weight update elementwise <= 1e-6 relative to the
magnitude of the terms (fp32); bf16 weights within half an ulp plus that fp32 error of the exact result, and
different from the rounded fp64 result on a small fraction only (double rounding)."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2502_16982_amd import binding, workloads  # noqa: E402
from tests import gpu_util as U  # noqa: E402


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()   # a missing library must fail loudly, not skip
    return torch.device("cuda:0")


def assert_records(recs, tol_fro):
    for r in recs:
        print(r, flush=True)
        assert r["o_finite"], r
        assert r["o_rel_fro"] <= tol_fro, r
        assert r["o_blk_max"] <= U.BLOCK_FACTOR * tol_fro, r
        assert r["o_elem_max"] <= U.ELEM_FACTOR * tol_fro, r
        assert r["m_err"] <= U.TOL_ELEM, r
        w = r["w"]
        if "max_rel" in w:
            assert w["max_rel"] <= U.TOL_ELEM, r
        else:
            assert w["max_excess"] <= 1.0 and w["frac_off"] <= 1e-3, r


# ---------------------------------------------------------------------------------------------
# fp32 path
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("nesterov", [0, 1])
def test_single_128x256_f32(dev, nesterov):
    wl = workloads.workload("single_128x256_f32")
    assert_records(U.run_and_compare(wl, dev, hp_over={"nesterov": nesterov}), U.TOL_F32_FRO)


def test_f32_ragged_shapes_two_steps(dev):
    shapes = [(1, 1), (1, 7), (7, 1), (3, 5), (65, 64), (100, 130), (130, 100), (200, 333)]
    wl = workloads.custom("ragged_f32", shapes, w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32",
                          w_std=1.0, g_std=1.0, seed_base=11)
    assert_records(U.run_and_compare(wl, dev, steps=2), U.TOL_F32_FRO)


def test_f32_path_with_bf16_buffers(dev):
    wl = workloads.custom("mixed", [(96, 200), (256, 64)], w_dtype=torch.bfloat16, g_dtype=torch.bfloat16, ns_dtype="f32",
                          seed_base=12)
    assert_records(U.run_and_compare(wl, dev, steps=2), U.TOL_F32_FRO)


# ---------------------------------------------------------------------------------------------
# bf16 path: small sizes spanning several tiles and ragged tails, both tile shapes, both orientations
# ---------------------------------------------------------------------------------------------
def test_bf16_ragged_shapes(dev):
    shapes = [(1, 1), (1, 9), (5, 3), (64, 64), (130, 130), (200, 333), (333, 200), (257, 511), (384, 128), (128, 640)]
    wl = workloads.custom("ragged_bf16", shapes, seed_base=21)
    assert_records(U.run_and_compare(wl, dev, steps=2), U.TOL_BF16_FRO)


def test_bf16_fp32_buffers_and_plain_momentum(dev):
    wl = workloads.custom("bf16ns_f32buf", [(300, 500), (512, 256)], w_dtype=torch.float32, g_dtype=torch.float32,
                          w_std=1.0, g_std=1.0, seed_base=22)
    assert_records(U.run_and_compare(wl, dev, steps=3, hp_over={"nesterov": 0}), U.TOL_BF16_FRO)


@pytest.mark.parametrize("copies", [1, 9])
def test_bf16_large_tile_shapes(dev, copies):
    """Sides that 256 x 256 tiles cover: three matrices alone run in smaller tiles, a list of them in the large ones."""
    shapes = [(1024, 1024), (1024, 1536), (1280, 1024)] * copies
    assert (min(U.coarse_tiles(shapes, "bf16")) > 0) == (copies > 1)
    wl = workloads.custom("tile256", shapes, seed_base=23)
    recs = U.run_and_compare(wl, dev, check=range(len(shapes) - 3, len(shapes)), steps=2)
    assert_records(recs, U.TOL_BF16_FRO)


def test_bf16_outliers(dev):
    wl = workloads.custom("outliers", [(512, 1024), (768, 768)], outlier_frac=0.01, outlier_mult=100.0, seed_base=24)
    assert_records(U.run_and_compare(wl, dev), U.TOL_BF16_FRO)


@pytest.mark.parametrize("ns_steps", [0, 1, 2, 5, 10])
def test_ns_step_counts(dev, ns_steps):
    wl32 = workloads.custom("steps32", [(96, 160), (160, 96)], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32",
                            w_std=1.0, g_std=1.0, seed_base=26)
    assert_records(U.run_and_compare(wl32, dev, hp_over={"ns_steps": ns_steps}), U.TOL_F32_FRO)
    wl = workloads.custom("steps", [(192, 320), (320, 192)], seed_base=25)
    recs = U.run_and_compare(wl, dev, hp_over={"ns_steps": ns_steps})
    if ns_steps == 10:
        # Known gap of the plain bf16 arithmetic, stated in include/muon.h: the 2e-2 bar holds for N <= 5.  The quintic
        # is expansive around its fixed point (|f'(0.868)| = 1.58), so bf16 rounding noise keeps growing with the
        # iteration count: measured 2.2-2.3e-2 here.  The run must still be sane (finite, within 5e-2); the parity
        # claim for N = 10 is made by MUON_BF16X2 (test_split_step_counts) and fails here by design.
        for r in recs:
            print(r, flush=True)
            assert r["o_finite"] and r["o_rel_fro"] <= 5e-2 and r["m_err"] <= U.TOL_ELEM, r
        if max(r["o_rel_fro"] for r in recs) > U.TOL_BF16_FRO:
            pytest.xfail("plain bf16 Newton-Schulz at N = 10 misses the 2e-2 bar (%.2e): documented range is N <= 5"
                         % max(r["o_rel_fro"] for r in recs))
        return
    assert_records(recs, 5e-3 if ns_steps == 0 else U.TOL_BF16_FRO)


def test_other_coefficients_and_hyperparameters(dev):
    wl = workloads.custom("coef", [(128, 256)], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32",
                          w_std=1.0, g_std=1.0, seed_base=27)
    over = {"a": 2.0, "b": -1.5, "c": 0.5, "lr": 0.3, "weight_decay": 0.01, "momentum": 0.5, "rms_scale": 0.4, "eps": 0.0}
    assert_records(U.run_and_compare(wl, dev, steps=2, hp_over=over), U.TOL_F32_FRO)


def test_bf16_six_steps_track_the_oracle(dev):
    """Six consecutive steps with fresh gradients, both orientations and a padded shape: every step is compared with
    the oracle run on the library's own state of the step before (momentum and weights carried on the device)."""
    wl = workloads.custom("six", [(256, 384), (384, 256), (200, 520), (512, 512)], seed_base=43)
    recs = U.run_and_compare(wl, dev, steps=6, want_rms=True)
    assert len(recs) == 6 * 4
    assert_records(recs, U.TOL_BF16_FRO)
    for r in recs:
        assert abs(r["rms_gpu"] - r["rms_ref"]) <= 2e-3 * r["rms_ref"], r


def test_coefficient_schedule(dev):
    """Iteration k of Eq. 2 with its own (a, b, c): three steps with the paper's triple, then two with the textbook
    order-5 Newton-Schulz polynomial (15, -10, 3)/8; also checks that the order of the triples is honoured."""
    paper = (3.4445, -4.7750, 2.0315)
    polish = (15.0 / 8.0, -10.0 / 8.0, 3.0 / 8.0)
    sched = [paper, paper, paper, polish, polish]
    wl = workloads.custom("sched", [(192, 320), (320, 192), (256, 256)], seed_base=41)
    assert_records(U.run_and_compare(wl, dev, hp_over={"coeff_schedule": sched}), U.TOL_BF16_FRO)
    assert_records(U.run_and_compare(wl, dev, hp_over={"coeff_schedule": sched[::-1]}), U.TOL_BF16_FRO)
    wl32 = workloads.custom("sched32", [(96, 160), (160, 96)], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32",
                            w_std=1.0, g_std=1.0, seed_base=42)
    assert_records(U.run_and_compare(wl32, dev, steps=2, hp_over={"coeff_schedule": sched}), U.TOL_F32_FRO)
    assert_records(U.run_and_compare(wl32, dev, hp_over={"coeff_schedule": sched[::-1]}), U.TOL_F32_FRO)
    # an even number of iterations leaves O in the other ping-pong buffer
    assert_records(U.run_and_compare(wl32, dev, hp_over={"coeff_schedule": sched[:4]}), U.TOL_F32_FRO)


@pytest.mark.parametrize("mode", [binding.MUON_SCALE_BASELINE, binding.MUON_SCALE_UPDATE_NORM])
def test_update_scaling_variants(dev, mode):
    """Eq. 5 (0.2 sqrt(H)) and Eq. 6 (0.2 O / RMS(O)) of section 3.1, fp32 and bf16 weights, both orientations."""
    over = {"scale_mode": mode, "hidden_size": 192.0, "lr": 0.05}
    wl = workloads.custom("variants", [(192, 320), (320, 192), (100, 100)], seed_base=28)
    assert_records(U.run_and_compare(wl, dev, steps=2, hp_over=over), U.TOL_BF16_FRO)
    wl32 = workloads.custom("variants32", [(96, 160), (160, 96)], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32",
                            w_std=1.0, g_std=1.0, seed_base=29)
    assert_records(U.run_and_compare(wl32, dev, steps=2, hp_over=over), U.TOL_F32_FRO)
    if mode == binding.MUON_SCALE_UPDATE_NORM:
        # the applied update has RMS exactly rms_scale: W0 = 0, lambda = 0, lr = 1  ->  RMS(W1) = 0.2
        w = torch.zeros(200, 136, device=dev)
        g = torch.randn(200, 136, device=dev)
        m = torch.zeros_like(w)
        for ns, ns_steps in (("f32", 5), ("bf16", 5), ("bf16", 0)):
            w.zero_(); m.zero_()
            st = binding.MuonStepper([(w, g, m)], ns_dtype=ns)
            st.step(binding.default_hparams(lr=1.0, weight_decay=0.0, scale_mode=mode, ns_steps=ns_steps))
            torch.cuda.synchronize()
            assert float(w.double().pow(2).mean().sqrt()) == pytest.approx(0.2, rel=2e-6)
            st.close()
        # an all-zero update stays zero (factor 0, no NaN)
        w.fill_(1.0); m.zero_()
        st = binding.MuonStepper([(w, torch.zeros_like(g), m)], ns_dtype="f32")
        st.step(binding.default_hparams(lr=0.5, weight_decay=0.0, scale_mode=mode))
        torch.cuda.synchronize()
        assert torch.equal(w, torch.ones_like(w))
        st.close()


# ---------------------------------------------------------------------------------------------
# split-bf16 paths (two / three bf16 planes per matrix on the matrix cores): the fp32 path's bar and better
# ---------------------------------------------------------------------------------------------
SPLIT = ["bf16x2", "bf16x3"]


@pytest.mark.parametrize("ns", SPLIT)
def test_split_ragged_shapes(dev, ns):
    shapes = [(1, 1), (1, 9), (5, 3), (64, 64), (130, 130), (200, 333), (333, 200), (257, 511), (384, 128), (128, 640)]
    wl = workloads.custom("ragged_" + ns, shapes, ns_dtype=ns, seed_base=51)
    assert_records(U.run_and_compare(wl, dev, steps=2), U.TOL_SPLIT_FRO[ns])


@pytest.mark.parametrize("ns", SPLIT)
@pytest.mark.timeout(600)
def test_split_large_tiles_and_strips(dev, ns):
    # sides that are even and odd multiples of 128, both orientations, fp32 and bf16 buffers: up to here planes stay in
    # 128-wide tiles
    shapes = [(1024, 1024), (1024, 1536), (1280, 1024), (384, 640), (640, 1152)]
    assert U.coarse_tiles(shapes, ns) == [0, 0]
    wl = workloads.custom("tiles_" + ns, shapes, ns_dtype=ns, seed_base=52)
    assert_records(U.run_and_compare(wl, dev, steps=2), U.TOL_SPLIT_FRO[ns])
    # coarse entries, 256 x 256 and 512 x 128 strips, and a small matrix in the fine launch beside them
    shapes = [(3200, 3200), (200, 333), (3328, 3200)]
    assert min(U.coarse_tiles(shapes, ns)) > 0
    wl = workloads.custom("large_" + ns, shapes, ns_dtype=ns, seed_base=59)
    assert_records(U.run_and_compare(wl, dev, check=[1, 2]), U.TOL_SPLIT_FRO[ns])
    wl = workloads.custom("tiles32_" + ns, [(300, 500), (512, 256)], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype=ns,
                          w_std=1.0, g_std=1.0, seed_base=53)
    assert_records(U.run_and_compare(wl, dev, steps=3, hp_over={"nesterov": 0}), U.TOL_SPLIT_FRO[ns])


@pytest.mark.parametrize("ns", SPLIT)
@pytest.mark.parametrize("ns_steps", [0, 1, 2, 10])
def test_split_step_counts(dev, ns, ns_steps):
    wl = workloads.custom("steps_" + ns, [(192, 320), (320, 192)], ns_dtype=ns, seed_base=54)
    assert_records(U.run_and_compare(wl, dev, hp_over={"ns_steps": ns_steps}, want_rms=True), U.TOL_SPLIT_FRO[ns])


@pytest.mark.parametrize("ns", SPLIT)
def test_split_outliers_schedule_and_variants(dev, ns):
    wl = workloads.custom("outl_" + ns, [(512, 1024), (768, 768)], ns_dtype=ns, outlier_frac=0.01, outlier_mult=100.0, seed_base=55)
    assert_records(U.run_and_compare(wl, dev), U.TOL_SPLIT_FRO[ns])
    paper = (3.4445, -4.7750, 2.0315)
    polish = (15.0 / 8.0, -10.0 / 8.0, 3.0 / 8.0)
    wl = workloads.custom("sched_" + ns, [(192, 320), (320, 192), (256, 256)], ns_dtype=ns, seed_base=56)
    assert_records(U.run_and_compare(wl, dev, hp_over={"coeff_schedule": [paper, paper, paper, polish, polish]}),
                   U.TOL_SPLIT_FRO[ns])
    over = {"scale_mode": binding.MUON_SCALE_UPDATE_NORM, "lr": 0.05}
    recs = U.run_and_compare(wl, dev, steps=2, hp_over=over, want_rms=True)
    assert_records(recs, U.TOL_SPLIT_FRO[ns])
    for r in recs:
        assert r["rms_gpu"] == pytest.approx(r["rms_ref"], rel=1e-5)


def test_split_is_closer_to_the_oracle_than_bf16(dev):
    """Same inputs through the three matrix-core paths: each added plane buys orders of magnitude."""
    errs = {}
    for ns in ("bf16", "bf16x2", "bf16x3"):
        wl = workloads.custom("ladder", [(512, 768), (768, 512)], ns_dtype=ns, seed_base=57)
        errs[ns] = max(r["o_rel_fro"] for r in U.run_and_compare(wl, dev))
    print(errs, flush=True)
    assert errs["bf16x2"] < errs["bf16"] / 50 and errs["bf16x3"] < errs["bf16x2"] / 10


def test_split_bitwise_repeatable_with_poisoned_workspace(dev):
    wl = workloads.custom("repeat_split", [(384, 640), (640, 384)], ns_dtype="bf16x2", seed_base=58)
    outs = []
    for trial in range(2):
        tensors = workloads.make_all(wl, dev)
        st = binding.MuonStepper(tensors, ns_dtype="bf16x2")
        if trial == 1:
            tail = st.workspace[st.workspace_bytes // 2:]
            tail.fill_(255)
        hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
        st.step(hp)
        st.step(hp)
        torch.cuda.synchronize()
        outs.append([t.clone() for trip in tensors for t in (trip[0], trip[2])] + [st.read_update(i) for i in range(2)])
        st.close()
    for x, y in zip(*outs):
        assert torch.equal(x, y)


# ---------------------------------------------------------------------------------------------
# degenerate inputs
# ---------------------------------------------------------------------------------------------
def test_zero_gradient_only_decays(dev):
    for ns in ("f32", "bf16"):
        w = torch.randn(70, 90, device=dev)
        w0 = w.clone()
        g = torch.zeros_like(w)
        m = torch.zeros_like(w)
        st = binding.MuonStepper([(w, g, m)], ns_dtype=ns)
        st.step(binding.default_hparams(lr=0.02, weight_decay=0.1, eps=1e-7))
        torch.cuda.synchronize()
        assert torch.equal(m, torch.zeros_like(m))
        assert torch.count_nonzero(st.read_update(0)).item() == 0
        ref = U.to64(w0) * (1 - 0.02 * 0.1)
        assert np.max(np.abs(U.to64(w) - ref) / np.abs(ref)) <= 1e-6
        # eps = 0 and an all-zero U must not produce NaN
        st.step(binding.default_hparams(lr=0.02, weight_decay=0.0, eps=0.0))
        torch.cuda.synchronize()
        assert torch.isfinite(w).all()
        st.close()


@pytest.mark.parametrize("ns", ["bf16", "bf16x2", "f32"])
def test_extreme_aspect_ratios(dev, ns):
    """One-row / one-column matrices and a 130 x 33000 one: iterates that are almost all padding, K loops of 500+ slabs."""
    tol = {"bf16": U.TOL_BF16_FRO, "bf16x2": U.TOL_SPLIT_FRO["bf16x2"], "f32": U.TOL_F32_FRO}[ns]
    wl = workloads.custom("extreme_" + ns, [(1, 70000), (70000, 1), (130, 33000)], ns_dtype=ns, seed_base=61)
    assert_records(U.run_and_compare(wl, dev, steps=2), tol)


@pytest.mark.parametrize("ns", ["bf16", "bf16x2", "f32"])
def test_largest_dimensions(dev, ns):
    """The largest row / column counts the interface accepts (2^20), both orientations: tile indices at the top of their
    range, K loops of 16384 slabs.  Gaussian gradient except for three 64-wide bands (first, middle and last K slab of
    the Gram product) scaled by 128, each carrying as much energy as all the rest, so that a slab dropped or read twice
    where a boundary could go wrong moves O by tens of percent.  Four equal singular values make the relative error of
    O that of ONE number, which the five iterations amplify about 5 times (nothing averages out): an emulation of ideal
    bf16 storage on Gaussian 4 x 2^20 gives 3e-2, of two planes 5e-5.  The test therefore asserts a structural bound
    (1e-1 bf16, 3e-4 two planes) and reports the case as an expected failure when the parity bar of the arithmetic
    (2e-2, 1e-4) is missed - the documented range of MUON_BF16 / MUON_BF16X2 excludes it; the fp32 path keeps 1e-4.  (Inputs with only a few distinct values are another matter
    at this length: a matrix-core accumulator is one chain of K / 16 fp32 additions whose rounding errors then all
    point the same way - 1e-2 in O for a +-2^-10 sign matrix with two or three planes alike.)"""
    big = 1 << 20
    # structural bound (a dropped or doubled slab moves O by tens of percent) and the parity bar of the arithmetic
    sane = {"bf16": 1e-1, "bf16x2": 3e-4, "f32": U.TOL_F32_FRO}[ns]
    bar = {"bf16": U.TOL_BF16_FRO, "bf16x2": U.TOL_SPLIT_FRO["bf16x2"], "f32": U.TOL_F32_FRO}[ns]
    worst = 0.0
    for shape in ((4, big), (big, 4)):
        gen = torch.Generator(device=dev).manual_seed(62 + shape[0] % 7)
        g = torch.randn(shape, generator=gen, device=dev) * 1e-3
        gl = g if shape[1] == big else g.t()
        for start in (0, big // 2 - 64, big - 64):
            gl[:, start:start + 64] *= 128.0
        g = g.to(torch.bfloat16)
        w = (torch.randn(shape, generator=gen, device=dev) * 0.02).to(torch.bfloat16)
        m = torch.zeros(shape, device=dev)
        w0, g0 = U.to64(w), U.to64(g)
        hp, d = U.hp_from(workloads.Hyper(), lr=0.02, weight_decay=0.1)
        st = binding.MuonStepper([(w, g, m)], ns_dtype=ns)
        st.step(hp)
        torch.cuda.synchronize()
        W, M, O = U.oracle_step(w0, g0, np.zeros(shape), d)
        o_gpu = U.to64(st.read_update(0))
        err = U.rel_fro(o_gpu, O)
        worst = max(worst, err)
        print({"ns": ns, "shape": shape, "o_rel_fro": err}, flush=True)
        assert torch.equal(m, g.float())
        assert err <= sane, (shape, err)
        chk = U.check_weight_update(w, w0, o_gpu, d)
        assert chk["max_excess"] <= 1.0 and chk["frac_off"] <= 1e-3, chk
        st.close()
    if worst > bar:
        # Known gap, stated in include/muon.h: with a handful of rows and K = 2^20 nothing averages out (see above);
        # measured 2.2-2.9e-2 (bf16) and 0.8-1.1e-4 (two planes) against bars of 2e-2 and 1e-4.
        pytest.xfail("4 x 2^20 with %s: %.2e exceeds the %.0e bar of the arithmetic (documented range)" % (ns, worst, bar))


def _structured_cases():
    """Matrices the method treats specially (Newton-Schulz acts on singular values only, section 2.1): fed as the
    gradient with zero momentum, so that U is the matrix itself up to the factor 1 + mu."""
    rng = np.random.default_rng(71)
    cases = {}
    q, _ = np.linalg.qr(rng.standard_normal((1024, 256)))
    cases["orthonormal_rows_256x1024"] = q.T                              # all singular values equal
    cases["orthonormal_cols_1024x256"] = q
    cases["diagonal_256"] = np.diag(np.geomspace(1e-3, 1.0, 256) * np.where(np.arange(256) % 3 == 0, -1.0, 1.0))
    cases["identical_rows_192x320"] = np.tile(rng.standard_normal((1, 320)), (192, 1))          # rank 1
    cases["rank_deficient_256x384"] = rng.standard_normal((256, 96)) @ rng.standard_normal((96, 384))   # rank 96 of 256
    return cases


@pytest.mark.parametrize("ns", ["bf16", "bf16x2", "f32"])
@pytest.mark.parametrize("case", ["orthonormal_rows_256x1024", "orthonormal_cols_1024x256", "diagonal_256",
                                  "identical_rows_192x320", "rank_deficient_256x384"])
def test_structured_inputs(dev, ns, case):
    """Equal singular values, a diagonal matrix, rank one and rank deficiency, through every arithmetic.
    Rank-deficient inputs have exact zeros among their singular values, which the quintic amplifies 3.4445-fold per
    iteration: whatever a path's rounding (2^-9 bf16 storage, 2^-17 two planes, 2^-21 fp32 accumulation) puts into the null
    space grows up to 485-fold in five iterations.  For them O is therefore compared on the row and column space of
    the input at the path's bar, and the null-space part is checked against that amplification bound."""
    mat = _structured_cases()[case]
    tol = {"bf16": U.TOL_BF16_FRO, "bf16x2": U.TOL_SPLIT_FRO["bf16x2"], "f32": U.TOL_F32_FRO}[ns]
    g = torch.tensor(mat, dtype=torch.float32, device=dev).contiguous()
    w = torch.zeros_like(g)
    m = torch.zeros_like(g)
    g64 = U.to64(g)
    hp, d = U.hp_from(workloads.Hyper(), lr=0.02, weight_decay=0.0, eps=0.0)
    st = binding.MuonStepper([(w, g, m)], ns_dtype=ns)
    st.step(hp)
    torch.cuda.synchronize()
    W, M, O = U.oracle_step(np.zeros_like(g64), g64, np.zeros_like(g64), d)
    o_gpu = U.to64(st.read_update(0))
    st.close()
    assert np.isfinite(o_gpu).all()
    assert U.momentum_error(U.to64(m), M, np.zeros_like(g64), g64, d["momentum"]) <= U.TOL_ELEM
    low_rank = case.startswith(("identical_rows", "rank_deficient"))
    if not low_rank:
        err = U.rel_fro(o_gpu, O)
        print({"case": case, "ns": ns, "o_rel_fro": err, **U.block_errors(o_gpu, O)}, flush=True)
        assert err <= tol, (case, ns, err)
        if case.startswith("diagonal"):
            off = o_gpu - np.diag(np.diag(o_gpu))
            assert np.count_nonzero(off) == 0          # zeros stay exact zeros in every arithmetic
        return
    # projectors onto the row and column space of the input, from its SVD.  The input reaches both sides rounded to
    # fp32, which fills its null space with singular values around 1e-7 of the largest: the oracle amplifies those
    # to 5e-5 at most, so "rank" means the singular values above 1e-5 of the largest.
    u, sv, vt = np.linalg.svd(g64, full_matrices=False)
    r = int((sv > 1e-5 * sv[0]).sum())
    assert r == {"identical_rows_192x320": 1, "rank_deficient_256x384": 96}[case]
    pu, pv = u[:, :r] @ u[:, :r].T, vt[:r].T @ vt[:r]
    inside = pu @ o_gpu @ pv
    outside = (o_gpu - inside) - (O - pu @ O @ pv)      # beyond what the oracle itself has there (5e-5 of the fp32 input)
    err_in = U.rel_fro(inside, pu @ O @ pv)
    # relative noise an iteration puts into its iterate: storage rounding for the matrix-core paths (2^-9, 2^-17); for
    # the fp32 path the fp32 accumulation of the products over K <= 1024 terms, about sqrt(K) 2^-24 <= 2^-21
    storage = {"bf16": 2.0 ** -9, "bf16x2": 2.0 ** -17, "f32": 2.0 ** -21}[ns]
    # ||outside||_F: the noise of the first iterate (Frobenius norm 1) is at most `storage` and grows
    # 3.4445^5-fold; what later iterations inject grows less (sum of the geometric series: factor 1.41)
    bound_out = 3.4445 ** 5 * storage * 1.5
    print({"case": case, "ns": ns, "rank": r, "o_rel_fro_range": err_in, "null_norm": float(np.linalg.norm(outside)),
           "null_bound": bound_out, "o_norm": float(np.linalg.norm(O))}, flush=True)
    assert np.linalg.norm(outside) <= bound_out, (case, ns, float(np.linalg.norm(outside)), bound_out)
    if ns == "bf16" and tol < err_in <= 5e-2:
        # Known gap of the plain bf16 arithmetic, stated in include/muon.h: when all rows are multiples of one row,
        # every rounding error repeats in every row and nothing averages out over the Gram product; a numpy model of
        # the arithmetic gives 2.2e-2 for identical rows (1.4e-2 with the a X term kept as an fp32 addend).
        pytest.xfail("bf16 Newton-Schulz on %s: %.2e on the range of the input exceeds 2e-2 (documented range)" % (case, err_in))
    assert err_in <= tol, (case, ns, err_in)


@pytest.mark.parametrize("ns", ["bf16", "bf16x2", "f32"])
def test_momentum_zero_ignores_a_nonzero_buffer(dev, ns):
    """mu = 0 makes M_t = G whatever M_{t-1} held (section 2.1's recurrence): a momentum buffer of garbage-sized values
    must leave no trace, in M or in O."""
    wl = workloads.custom("mu0_" + ns, [(192, 320), (320, 192)], ns_dtype=ns, seed_base=72)
    tensors = workloads.make_all(wl, dev)
    for _, _, m in tensors:
        m.normal_(0.0, 50.0)
    hp, d = U.hp_from(wl.hyper, momentum=0.0)
    host = [[U.to64(t) for t in trip] for trip in tensors]
    st = binding.MuonStepper(tensors, ns_dtype=ns)
    st.step(hp)
    torch.cuda.synchronize()
    tol = {"bf16": U.TOL_BF16_FRO, "bf16x2": U.TOL_SPLIT_FRO["bf16x2"], "f32": U.TOL_F32_FRO}[ns]
    for i, (w0, g0, m0) in enumerate(host):
        assert torch.equal(tensors[i][2], tensors[i][1].float())
        W, M, O = U.oracle_step(w0, g0, m0, d)
        assert U.rel_fro(U.to64(st.read_update(i)), O) <= tol
    st.close()


@pytest.mark.parametrize("ns", ["bf16", "bf16x2", "f32"])
@pytest.mark.parametrize("g_std", [1e-12, 1e8])
@pytest.mark.parametrize("eps", [0.0, 1e-7])
def test_gradient_scale_invariance(dev, ns, g_std, eps):
    """X_0 = U / ||U||_F does not depend on the scale of U (section 2.1).  The library stores the un-normalised U in
    the iteration's dtype and applies 1 / ||U||_F^2 and 1 / ||U||_F in the first Gram and apply epilogues, so both
    the sum of squares and those factors must stay inside fp32: gradients of standard deviation 1e-12 and 1e+8, both
    orientations, with the paper's formula (eps = 0) and with the default eps (which is not small against
    ||U||_F = 1e-12 * sqrt(A B), so the oracle's O shrinks accordingly - same formula both sides)."""
    tol = {"bf16": U.TOL_BF16_FRO, "bf16x2": U.TOL_SPLIT_FRO["bf16x2"], "f32": U.TOL_F32_FRO}[ns]
    wl = workloads.custom("scale_%s_%g" % (ns, g_std), [(192, 320), (320, 192)], w_dtype=torch.float32, g_dtype=torch.float32,
                          ns_dtype=ns, w_std=1.0, g_std=g_std, seed_base=73)
    recs = U.run_and_compare(wl, dev, hp_over={"eps": eps})
    for r in recs:
        print(r, flush=True)
        assert r["o_finite"] and r["o_rel_fro"] <= tol and r["m_err"] <= U.TOL_ELEM, r


def test_last_round_of_a_persistent_launch_in_the_fine_launch(dev):
    """26 matrices of 1024 x 1024: the symmetric launches have 26 x 10 = 256 + 4 tiles of equal K, so they are
    persistent and the planner issues the last 4 plain tiles (of the last matrices) as sixteen 128 x 128 tiles in the
    fine launch; 64 x (1024 x 2048) does the same to the apply product (64 x 32 = 2048 tiles: nothing left over) and
    65 of them leave 32 over.  Every matrix that can hold a moved tile is compared with the oracle."""
    wl = workloads.custom("sym_tail", [(1024, 1024)] * 26, seed_base=91)
    assert_records(U.run_and_compare(wl, dev, check=[0, 23, 24, 25]), U.TOL_BF16_FRO)
    wl = workloads.custom("apply_tail", [(1024, 2048)] * 65, seed_base=92)
    assert_records(U.run_and_compare(wl, dev, check=[0, 62, 63, 64]), U.TOL_BF16_FRO)


def test_lr_zero_leaves_weights_bitwise(dev):
    wl = workloads.custom("lr0", [(100, 300)], seed_base=31)
    (w, g, m), = workloads.make_all(wl, dev)
    w0 = w.clone()
    st = binding.MuonStepper([(w, g, m)])
    st.step(binding.default_hparams(lr=0.0, weight_decay=0.1))
    torch.cuda.synchronize()
    assert torch.equal(w, w0)
    assert torch.allclose(m, g.float())     # mu * 0 + G
    st.close()


def test_bitwise_repeatable_and_workspace_poison(dev):
    wl = workloads.custom("repeat", [(384, 640), (640, 384), (256, 256)], seed_base=32)
    outs = []
    for trial in range(2):
        tensors = workloads.make_all(wl, dev)
        st = binding.MuonStepper(tensors)
        if trial == 1:
            # garbage in the Newton-Schulz temporaries must not leak into the result
            tail = st.workspace[st.workspace_bytes // 2:]
            tail.view(torch.float32 if tail.numel() % 4 == 0 else torch.uint8).fill_(float("nan") if tail.numel() % 4 == 0 else 255)
        hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
        st.step(hp)
        st.step(hp)
        torch.cuda.synchronize()
        outs.append([t.clone() for trip in tensors for t in (trip[0], trip[2])] + [st.read_update(i) for i in range(3)])
        st.close()
    for x, y in zip(*outs):
        assert torch.equal(x, y)


def test_checkpoint_resume_is_bitwise(dev):
    wl = workloads.custom("resume", [(200, 264)], seed_base=33)
    (w, g, m), = workloads.make_all(wl, dev)
    g2 = workloads.make_gradient(wl, 0, 1, dev)
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    st = binding.MuonStepper([(w, g, m)])
    st.step(hp)
    torch.cuda.synchronize()
    w_ck, m_ck = w.clone(), m.clone()
    g.copy_(g2)
    st.step(hp)
    torch.cuda.synchronize()
    st.close()
    # resume from the copies in fresh buffers and a fresh context
    st2 = binding.MuonStepper([(w_ck, g2, m_ck)])
    st2.step(hp)
    torch.cuda.synchronize()
    assert torch.equal(w_ck, w) and torch.equal(m_ck, m)
    st2.close()


def test_update_rms_output_and_lemma1(dev):
    wl = workloads.custom("rms", [(256, 512), (512, 256), (100, 100)], seed_base=34)
    recs = U.run_and_compare(wl, dev, want_rms=True)
    for r in recs:
        assert r["rms_gpu"] == pytest.approx(r["rms_ref"], rel=1e-5)
        A, B = r["shape"]
        assert 0.6 <= r["rms_gpu"] * np.sqrt(max(A, B)) <= 1.25      # Lemma 1 band


def test_pointer_changes_between_steps(dev):
    wl = workloads.custom("ptrs", [(128, 192), (192, 128)], seed_base=35)
    t1 = workloads.make_all(wl, dev)
    t2 = [tuple(x.clone() for x in trip) for trip in t1]
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    st = binding.MuonStepper(t1)
    st.step(hp)
    st.set_tensors(t2)          # same shapes, different buffers
    st.step(hp)
    torch.cuda.synchronize()
    for a, b in zip(t1, t2):
        assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
    st.close()


def test_error_codes_with_a_live_context(dev):
    wl = workloads.custom("err", [(64, 96)], seed_base=36)
    tensors = workloads.make_all(wl, dev)
    st = binding.MuonStepper(tensors)
    L = binding.lib()
    hp = binding.default_hparams()
    two = binding.param_array([(64, 96), (64, 96)], [1, 1], [1, 1])
    assert L.muon_step(st.ctx, two, 2, C.byref(hp), None, None) == -3
    wrong = binding.param_array([(64, 97)], [1], [1])
    wrong[0].w, wrong[0].g, wrong[0].m = st.params[0].w, st.params[0].g, st.params[0].m
    assert L.muon_step(st.ctx, wrong, 1, C.byref(hp), None, None) == -3
    nul = binding.param_array([(64, 96)], [1], [1])
    assert L.muon_step(st.ctx, nul, 1, C.byref(hp), None, None) == -1
    odd = binding.param_array([(64, 96)], [1], [1])
    odd[0].w, odd[0].g, odd[0].m = st.params[0].w + 1, st.params[0].g, st.params[0].m
    assert L.muon_step(st.ctx, odd, 1, C.byref(hp), None, None) == -7
    bad = binding.default_hparams(ns_steps=-1)
    assert L.muon_step(st.ctx, st.params, 1, C.byref(bad), None, None) == -1
    bad = binding.default_hparams(lr=float("nan"))
    assert L.muon_step(st.ctx, st.params, 1, C.byref(bad), None, None) == -1
    bad = binding.default_hparams(scale_mode=3)
    assert L.muon_step(st.ctx, st.params, 1, C.byref(bad), None, None) == -1
    bad = binding.default_hparams(scale_mode=binding.MUON_SCALE_BASELINE, hidden_size=0.0)
    assert L.muon_step(st.ctx, st.params, 1, C.byref(bad), None, None) == -1
    bad = binding.default_hparams(reserved=1)
    assert L.muon_step(st.ctx, st.params, 1, C.byref(bad), None, None) == -1
    bad = binding.default_hparams(coeff_schedule=[(3.4445, -4.7750, 2.0315), (1.0, float("inf"), 0.0)])
    assert bad.ns_steps == 2
    assert L.muon_step(st.ctx, st.params, 1, C.byref(bad), None, None) == -1
    dst = torch.empty(64, 96, device=dev)
    assert L.muon_debug_read_update(st.ctx, 0, C.c_void_p(dst.data_ptr()), 0, None) == -6   # no step yet
    assert L.muon_debug_read_update(st.ctx, 5, C.c_void_p(dst.data_ptr()), 0, None) == -1
    st.close()
    # a workspace that holds the tables but not the largest matrix
    p = binding.param_array([(512, 512)], [1], [1])
    need = binding.muon_workspace_bytes(p, 1, binding.MUON_BF16)
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    ctx = C.c_void_p(None)
    assert L.muon_init(C.byref(ctx), p, 1, 1, C.c_void_p(ws.data_ptr()), need - 4096) == -4


def test_chunked_workspace_matches_resident(dev):
    shapes = [(256, 384)] * 5 + [(384, 256)] * 3
    wl = workloads.custom("chunks", shapes, seed_base=37)
    res = {}
    for label, cap in (("resident", 0), ("chunked", 1)):
        tensors = workloads.make_all(wl, dev)
        st = binding.MuonStepper(tensors, max_workspace_bytes=cap)
        res[label + "_chunks"] = binding.muon_plan_chunks(st.ctx)
        hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
        st.step(hp)
        st.step(hp)
        torch.cuda.synchronize()
        res[label] = [t.clone() for trip in tensors for t in (trip[0], trip[2])]
        if label == "chunked":
            with pytest.raises(binding.MuonError):
                st.read_update(0)
            st.read_update(len(shapes) - 1)
        st.close()
    assert res["resident_chunks"] == 1 and res["chunked_chunks"] == len(shapes)
    for x, y in zip(res["resident"], res["chunked"]):
        assert torch.equal(x, y)


def test_runs_on_a_side_stream(dev):
    wl = workloads.custom("stream", [(256, 256)], seed_base=38)
    t1 = workloads.make_all(wl, dev)
    t2 = [tuple(x.clone() for x in trip) for trip in t1]
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    s1 = binding.MuonStepper(t1)
    s1.step(hp)
    torch.cuda.synchronize()
    side = torch.cuda.Stream(device=dev)
    s2 = binding.MuonStepper(t2)
    s2.step(hp, stream=side)
    side.synchronize()
    assert torch.equal(t1[0][0], t2[0][0]) and torch.equal(t1[0][2], t2[0][2])
    s1.close()
    s2.close()
