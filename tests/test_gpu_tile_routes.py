"""The planner gives a product 256-, 128-, 64- or 32-wide tiles by how much work a launch holds.  Every tile adds an output
element's products in the same order, so in plain bf16 a matrix must come out with the same bits whichever tiles computed
it: alone (64-wide), in a short list (128-wide) and in a list long enough for 256-wide tiles and strips (plain bf16 only at
these sides).  With several planes an element of a symmetric product and its mirror image add the plane pairs in different orders (fp32 rounding,
about 1e-7 of A per product), and the tile decides which of the two is kept: there the results agree to a tenth of the
path's own bar."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2502_16982_amd import binding, workloads  # noqa: E402
from tests import gpu_util as U  # noqa: E402
from tests.gpu_util import coarse_tiles, table_sizes  # noqa: E402
from tests import plan_routes  # noqa: E402
from tests.plan_routes import fine_forms  # noqa: E402
from tests.test_gpu_parity import assert_records  # noqa: E402


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("ns", ["bf16", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("shape,short,long", [((640, 1408), 12, 130), ((1408, 640), 12, 130), ((1024, 1024), 10, 60)])
def test_same_bits_from_every_tile(dev, ns, shape, short, long):
    wl = workloads.custom("routes", [shape] * long, ns_dtype=ns, seed_base=310)
    first = workloads.make_matrix(wl, 0, dev)
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    results = []
    for n in (1, short, long):
        tensors = [tuple(t.clone() for t in first) for _ in range(n)]
        st = binding.MuonStepper(tensors, ns_dtype=ns)
        st.step(hp)
        torch.cuda.synchronize()
        # the same matrix everywhere in the list: first, last and one in the middle
        for i in {0, n // 2, n - 1}:
            results.append((st.read_update(i), tensors[i][0], tensors[i][2]))
        st.close()
    assert coarse_tiles([shape], ns) == [0, 0] and (min(coarse_tiles([shape] * long, ns)) > 0) == (ns == "bf16")
    for o, w, m in results[1:]:
        assert torch.equal(m, results[0][2])
        if ns == "bf16":
            assert torch.equal(o, results[0][0]) and torch.equal(w, results[0][1])
        else:
            assert U.rel_fro(U.to64(o), U.to64(results[0][0])) <= 0.1 * U.TOL_SPLIT_FRO[ns]


@pytest.mark.parametrize("ns,tol", [("bf16", U.TOL_BF16_FRO), ("bf16x2", U.TOL_SPLIT_FRO["bf16x2"]), ("bf16x3", U.TOL_SPLIT_FRO["bf16x3"])])
def test_64_wide_tiles_at_their_edges(dev, ns, tol):
    """K of one, two, three and many pairs of slabs, both orientations, one padded row or column short of a tile."""
    shapes = [(128, 128), (65, 127), (129, 256), (256, 129), (127, 384), (128, 1024), (1024, 128), (320, 577)]
    wl = workloads.custom("edges64_" + ns, shapes, ns_dtype=ns, seed_base=320)
    assert coarse_tiles(shapes, ns) == [0, 0]
    assert_records(U.run_and_compare(wl, dev, steps=2, want_rms=True), tol)


@pytest.mark.parametrize("shape", [(100, 130), (128, 256), (256, 300), (384, 200), (130, 520), (40, 900), (300, 1100)])
def test_same_bits_from_waves_and_both_rings(dev, shape):
    """Plain bf16: alone a matrix of these sizes runs as one wave per 32 x 32; in longer lists as 64-wide blocks with a ring of
    four slabs, then of three, then in 128-wide tiles, the apply product (K-major operand) and the symmetric ones each in
    every form.  K of 2, 4, 6 and more slabs; the norm added up by one wave, by a block, and by its own launch."""
    wl = workloads.custom("waves", [shape], seed_base=345)
    first = workloads.make_matrix(wl, 0, dev)
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    results, seen = [], {"sym": set(), "apply": set()}
    sym, _, app = table_sizes([shape], "bf16", 0)
    for n in sorted({1, -(-40 // app), -(-40 // sym), -(-100 // app), -(-100 // sym), 400}):
        gram, poly, apply = fine_forms([shape] * n, "bf16")
        seen["sym"] |= {gram, poly}
        seen["apply"].add(apply)
        tensors = [tuple(t.clone() for t in first) for _ in range(n)]
        st = binding.MuonStepper(tensors)
        for _ in range(2):
            st.step(hp)
        torch.cuda.synchronize()
        results += [(n, i, st.read_update(i), tensors[i][0], tensors[i][2]) for i in {0, n // 2, n - 1}]
        st.close()
    assert all({"waves", "ring4", "quarters"} <= forms and forms & {"whole", "-"} for forms in seen.values()), seen
    for n, i, o, w, m in results[1:]:
        assert torch.equal(o, results[0][2]) and torch.equal(w, results[0][3]) and torch.equal(m, results[0][4]), (n, i)


@pytest.mark.parametrize("ns", ["bf16x2", "bf16x3"])
@pytest.mark.parametrize("shapes,forms", [
    ([(129, 256), (300, 140), (65, 1200)], ["ring4", "ring4", "ring4"]),
    ([(200, 384), (384, 200), (100, 700)] * 14, ["quarters", "quarters", "quarters"]),
    ([(300, 700)] * 6 + [(700, 300)] * 6 + [(128, 2048)] * 8, ["ring4", "quarters", "quarters"]),
    ([(128, 1100)] * 260, ["quarters", "quarters", "whole"]),
])
def test_planes_in_every_form_of_a_short_launch(dev, ns, shapes, forms):
    """64-wide blocks with either ring, alone and where 128-wide ones would leave their last round badly filled, lists that mix K."""
    assert fine_forms(shapes, ns) == forms
    wl = workloads.custom("forms_" + ns, shapes, ns_dtype=ns, seed_base=327)
    n = len(shapes)
    assert_records(U.run_and_compare(wl, dev, check=sorted({0, 1, 2, n - 3, n - 2, n - 1}), steps=2, want_rms=True), U.TOL_SPLIT_FRO[ns])


@pytest.mark.parametrize("ns", ["bf16x2", "bf16x3"])
def test_planes_in_128_wide_tiles_at_their_edges(dev, ns):
    """More entries than a launch in quarters holds.  K of one and of several pairs of pieces (the loop not run, run once, run
    several times), both orientations, one padded row or column short of a tile."""
    shapes = [(128, 128), (127, 384), (384, 129), (257, 640)]
    copies = 60 if ns == "bf16x2" else 110
    assert fine_forms(shapes * copies, ns) == ["whole"] * 3 and coarse_tiles(shapes * copies, ns) == [0, 0]
    wl = workloads.custom("edges128_" + ns, shapes * copies, ns_dtype=ns, seed_base=325)
    n = len(wl.shapes)
    assert_records(U.run_and_compare(wl, dev, check=list(range(4)) + list(range(n - 4, n)), steps=2, want_rms=True), U.TOL_SPLIT_FRO[ns])


@pytest.mark.parametrize("copies", [1, 40])
def test_f32_products_whole_and_in_quarters(dev, copies):
    """fp32 path: K of two 32-wide slabs (two of a block's four waves have none) up to several rounds of the ring, ragged
    edges, both orientations; alone every launch runs in quarters, in 40 copies the longer ones run whole.  Bar: a tenth
    of the path's (a dot product of K <= 1024 fp32 terms is good to about 1e-6; five iterations amplify that by < 5)."""
    shapes = [(64, 64), (1, 65), (63, 130), (130, 63), (100, 320), (320, 257), (384, 1000)]
    wl = workloads.custom("f32_routes", shapes * copies, w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32",
                          w_std=1.0, g_std=1.0, seed_base=330)
    n = len(wl.shapes)
    assert_records(U.run_and_compare(wl, dev, check=list(range(n - len(shapes), n)), steps=2, want_rms=True), 0.1 * U.TOL_F32_FRO)


@pytest.mark.parametrize("shape,long", [((100, 320), 120), ((384, 1000), 30), ((520, 130), 70), ((130, 4300), 60)])
def test_f32_bits_do_not_depend_on_the_list(dev, shape, long):
    """fp32 path: the order of a dot product's terms belongs to K alone.  A matrix comes out with the same bits alone (quarters),
    in a list long enough for whole entries, beside a matrix whose K is over 4096 (accumulators with a second level; the last
    shape needs them itself), and in a workspace that holds a part of the list."""
    wl = workloads.custom("f32_lists", [shape], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32", seed_base=335)
    first = workloads.make_matrix(wl, 0, dev)
    far = (torch.randn(40, 5000, device=dev), torch.randn(40, 5000, device=dev), torch.zeros(40, 5000, device=dev))
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    assert min(table_sizes([shape] * long, "f32", 0)) > 320         # more than a launch that runs in quarters holds
    results = []
    for n, extra, parts in ((1, 0, 1), (1, 1, 1), (long, 0, 1), (long, 1, 1), (long, 0, 5)):
        tensors = [tuple(t.clone() for t in first) for _ in range(n)] + [tuple(t.clone() for t in far)] * extra
        whole = binding.MuonStepper(tensors, ns_dtype="f32").workspace_bytes
        st = binding.MuonStepper(tensors, ns_dtype="f32", max_workspace_bytes=0 if parts == 1 else whole // parts)
        assert (binding.muon_plan_chunks(st.ctx) > 1) == (parts > 1)
        st.step(hp)
        torch.cuda.synchronize()
        results += [(n, extra, parts, i, tensors[i][0], tensors[i][2]) for i in {0, n // 2, n - 1}]
        st.close()
    for n, extra, parts, i, w, m in results[1:]:
        assert torch.equal(m, results[0][5]) and torch.equal(w, results[0][4]), (n, extra, parts, i)


@pytest.mark.parametrize("dtypes", [(torch.bfloat16, torch.bfloat16), (torch.float32, torch.bfloat16), (torch.bfloat16, torch.float32)])
def test_elementwise_passes_at_odd_widths_and_addresses(dev, dtypes):
    """Widths around the 4- and 8-element pieces and the 64-wide tile, buffers that start one element off every wider
    alignment, in guarded memory: M and W agree with the oracle and nothing outside the matrices changes."""
    shapes = [(1, 1), (3, 5), (65, 63), (64, 65), (130, 7), (33, 257), (100, 1001), (16, 320), (97, 64), (31, 72)]
    wl = workloads.custom("odd", shapes, w_dtype=dtypes[0], g_dtype=dtypes[1], seed_base=340)
    hp, d = U.hp_from(wl.hyper)
    tensors, flats = [], []
    for i, (a, b) in enumerate(shapes):
        views = []
        for t in workloads.make_matrix(wl, i, dev):
            flat = torch.full((a * b + 66,), 7.0, dtype=t.dtype, device=dev)
            flat[33:33 + a * b] = t.reshape(-1)
            flats.append((flat, a * b))
            views.append(flat[33:33 + a * b].view(a, b))
        tensors.append(tuple(views))
    host = [tuple(U.to64(t) for t in trip) for trip in tensors]
    st = binding.MuonStepper(tensors)
    st.step(hp)
    torch.cuda.synchronize()
    for i, (w0, g0, m0) in enumerate(host):
        _, m_ref, _ = U.oracle_step(w0, g0, m0, d)
        assert U.momentum_error(U.to64(tensors[i][2]), m_ref, m0, g0, d["momentum"]) <= U.TOL_ELEM
        rec = U.check_weight_update(tensors[i][0], w0, U.to64(st.read_update(i)), d)
        assert rec.get("max_rel", 0.0) <= U.TOL_ELEM and rec.get("max_excess", 0.0) <= 1.0, (shapes[i], rec)
        assert torch.equal(tensors[i][1].double().cpu(), torch.from_numpy(g0))
    for flat, n in flats:
        assert (flat[:33] == 7).all() and (flat[33 + n:] == 7).all()
    st.close()


@pytest.mark.timeout(600)
def test_update_of_a_long_list_of_odd_widths(dev):
    """More than 64 M elements of bf16 weights in rows that end inside a 128-byte line: the weight update without its hint."""
    wl = workloads.custom("long_odd", [(1025, 1025)] * 64 + [(1031, 999)], seed_base=360)
    assert_records(U.run_and_compare(wl, dev, check=[0, 63, 64]), U.TOL_BF16_FRO)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("ns", ["bf16x2", "bf16x3"])
def test_planes_in_coarse_tiles_and_strips(dev, ns):
    """With several planes only large matrices get coarse entries (256 x 256 and, where the side is an odd multiple of 128, 512 x 128,
    each run as four 128 x 128 blocks); one of the two is iterated on its transpose."""
    shapes = [(3200, 3328), (3328, 3200)]
    assert min(coarse_tiles(shapes, ns)) > 0
    wl = workloads.custom("strips_" + ns, shapes, ns_dtype=ns, seed_base=350)
    assert_records(U.run_and_compare(wl, dev), U.TOL_SPLIT_FRO[ns])


@pytest.mark.timeout(600)
def test_planes_in_both_launches_of_a_product(dev):
    """Two planes, 2 x 136 symmetric tiles of one K: 256 stay in the coarse launch, the last 16, all of the second matrix, go to
    the fine launch as four 128 x 128 entries each."""
    shapes = [(4096, 4096)] * 2
    assert table_sizes(shapes, "bf16x2", 1) == [256, 256, 512] and table_sizes(shapes, "bf16x2", 0) == [64, 64, 0]
    wl = workloads.custom("planes_tail", shapes, ns_dtype="bf16x2", seed_base=355)
    assert_records(U.run_and_compare(wl, dev, check=[1]), U.TOL_SPLIT_FRO["bf16x2"])


def scalar_two_planes(u, pair, steps=5, a=3.4445, b=-4.7750, c=2.0315, eps=1e-7):
    """What two-plane arithmetic makes of a diagonal matrix: every product of the iteration is a scalar one (float64 vector u of
    the diagonal; `pair`: with (1,1) in the polynomial)."""
    def split(x):
        x = x.float()
        h = x.bfloat16().float()
        return h.double(), (x - h).bfloat16().double()

    s = 1.0 / (u.norm() + eps)
    x = split(u)
    for it in range(steps):
        s2, s1 = (s * s, s) if it == 0 else (1.0, 1.0)
        g = split(s2 * (x[0] * x[0] + 2 * x[0] * x[1]))
        poly = split(c * (g[0] * g[0] + 2 * g[0] * g[1] + (g[1] * g[1] if pair else 0.0)) + b * (g[0] + g[1]))
        x = split(s1 * (x[0] * poly[0] + x[0] * poly[1] + x[1] * poly[0] + a * (x[0] + x[1])))
    return x[0] + x[1]


@pytest.mark.timeout(600)
@pytest.mark.parametrize("shape,copies,coarse", [((3200, 3328), 2, True), ((3328, 3200), 2, True), ((1024, 1100), 12, False), ((300, 500), 1, False)])
def test_two_planes_polynomial_takes_the_last_pair_on_the_diagonal(dev, shape, copies, coarse):
    """A diagonal matrix runs the scalar iteration on every element: O must be the one with the pair (1,1), whichever tile
    the polynomial runs in (coarse ones take the pair in their own pieces of K alone).  The library's fp32 norm and products
    round the second plane of some elements the other way, which is seen as a fifth of the distance to the iteration
    without the pair; without it the two distances would change places."""
    assert (coarse_tiles([shape] * copies, "bf16x2")[0] > 0) == coarse
    m = min(shape)
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    d = torch.empty(m, device=dev).uniform_(0.7e-3, 1.4e-3, generator=gen)
    g = torch.zeros(shape, device=dev)
    g[torch.arange(m), torch.arange(m)] = d
    tensors = [(torch.zeros(shape, device=dev), g.clone(), torch.zeros(shape, device=dev)) for _ in range(copies)]
    st = binding.MuonStepper(tensors, ns_dtype="bf16x2")
    st.step(binding.default_hparams(lr=0.02, weight_decay=0.1, momentum=0.95, nesterov=1, eps=1e-7))
    o = st.read_update(copies - 1).double()
    st.close()
    diag = o[torch.arange(m), torch.arange(m)]
    assert float((o - torch.zeros_like(o).index_put((torch.arange(m, device=dev),) * 2, diag)).abs().max()) == 0.0
    u = (torch.tensor(0.95, device=dev) * d + d).double()
    far = {pair: float(((diag - scalar_two_planes(u, pair)) / diag).square().mean().sqrt()) for pair in (True, False)}
    print("rms distance from the scalar iteration with / without the pair:", far[True], far[False], flush=True)
    assert far[True] < 0.5 * far[False]


@pytest.mark.timeout(600)
def test_large_two_plane_polynomial_costs_what_the_gram_product_costs(dev):
    """Square matrices in coarse tiles: Gram product and polynomial are the same three plane pairs over the same tiles.  The
    polynomial's addend and its fourth pair in the tile's own pieces (4 of 64 here) are 2 to 6 % more; the pair over the whole of K
    was 25 %."""
    shapes = [(4096, 4096)] * 3
    assert min(coarse_tiles(shapes, "bf16x2")) > 0
    wl = workloads.custom("poly_cost", shapes, ns_dtype="bf16x2", seed_base=365)
    st = binding.MuonStepper(workloads.make_all(wl, dev), ns_dtype="bf16x2")
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    ratios = []
    for k in range(6):
        binding.muon_profile_enable(st.ctx, True)
        st.step(hp)
        torch.cuda.synchronize()
        r = binding.muon_profile_read(st.ctx, reset=True)
        if k:
            ratios.append(r["poly"][0] / r["gram"][0])
    st.close()
    print("polynomial / Gram product:", sorted(ratios), flush=True)
    assert sorted(ratios)[2] < 1.15


@pytest.mark.parametrize("shape,copies", [((256, 300), 64), ((384, 400), 30), ((1024, 1000), 7), ((1152, 1300), 2), ((1300, 3000), 2)])
def test_same_bits_from_the_128_wide_ring(dev, shape, copies):
    """Plain bf16: in lists of about one 128-wide entry per compute unit (the symmetric products, the apply product or both) blocks have a
    ring of four slabs.  K of four slabs (the loop not run) and more, with and without the addend, the norm folded or not, tiles on
    the diagonal; the same bits as alone and in a list too long for it."""
    wl = workloads.custom("ring128", [shape], seed_base=347)
    first = workloads.make_matrix(wl, 0, dev)
    hp = binding.default_hparams(lr=0.02, weight_decay=0.1)
    sym, _, app = table_sizes([shape], "bf16", 0)
    results = []
    lengths = sorted({1, copies, 230 // sym, 250 // app, -(-260 // sym) * 2} - {0})
    assert "ring128" in {f for n in lengths for f in fine_forms([shape] * n, "bf16")}
    for n in lengths:
        tensors = [tuple(t.clone() for t in first) for _ in range(n)]
        st = binding.MuonStepper(tensors)
        for _ in range(2):
            st.step(hp)
        torch.cuda.synchronize()
        results += [(n, i, st.read_update(i), tensors[i][0], tensors[i][2]) for i in sorted({0, n // 2, n - 1})]
        st.close()
    for n, i, o, w, m in results[1:]:
        assert torch.equal(o, results[0][2]) and torch.equal(w, results[0][3]) and torch.equal(m, results[0][4]), (n, i)


@pytest.mark.parametrize("shape,lengths,product", [((512, 512), (1, 12, 13), "apply"), ((512, 4160), (1, 14, 15), "gram")])
def test_f32_bits_where_the_last_entries_run_in_quarters(dev, shape, lengths, product):
    """13 of 512 x 512: 832 entries of the apply product, 64 more than three per compute unit hold; one alone; 12, exactly one round.  15 of
    512 x 4160: 540 entries of the Gram product, whose sums over K > 4096 have two levels and two places per compute unit; 14, none over."""
    assert [plan_routes.tails([shape] * n)[product] > 0 for n in lengths] == [False, False, True]
    wl = workloads.custom("f32_tail", [shape], w_dtype=torch.float32, g_dtype=torch.float32, ns_dtype="f32", seed_base=349)
    first = workloads.make_matrix(wl, 0, dev)
    results = []
    for n in lengths:
        tensors = [tuple(t.clone() for t in first) for _ in range(n)]
        st = binding.MuonStepper(tensors, ns_dtype="f32")
        st.step(binding.default_hparams(lr=0.02, weight_decay=0.1))
        torch.cuda.synchronize()
        results += [(n, i, tensors[i][0], tensors[i][2]) for i in sorted({0, n // 2, n - 1})]
        st.close()
    for n, i, w, m in results[1:]:
        assert torch.equal(w, results[0][2]) and torch.equal(m, results[0][3]), (n, i)
