"""Host logic of the launch planner, without a GPU: muon_plan_only builds the plan muon_init would build and
muon_plan_tiles hands out its tile tables; the tests check that every product's tiles cover exactly the output they
must, once, whatever the shape mix, the arithmetic and the chunking."""
import numpy as np
import pytest

from paper_2502_16982_amd import binding

SHAPE_SETS = {
    "ragged": [(1, 1), (1, 9), (5, 3), (64, 64), (130, 130), (200, 333), (333, 200), (257, 511), (384, 128), (128, 640)],
    "tiles256": [(1024, 1024), (1024, 1536), (1280, 1024), (384, 640), (640, 1152)],
    "moe_expert": [(2048, 1408), (2048, 1408), (1408, 2048)],
    "block": [(4096, 4096), (4096, 11008), (11008, 4096)],
    # the whole 4096-wide block: its 3088 apply tiles are 12 x 256 + 16, so 16 of them move to the fine launch
    "block_full": [(4096, 4096)] * 4 + [(4096, 11008)] * 2 + [(11008, 4096)],
    "many_small": [(256, 384)] * 40 + [(384, 256)] * 30,
    # 26 x 10 symmetric tiles = 256 + 4 and 26 x 16 apply tiles = 256 + 160: the 4 go to the fine launch, the 160 stay
    "sym_tail": [(1024, 1024)] * 26,
    "extreme": [(4, 1 << 20), (1 << 20, 4), (1, 70000)],
}


def plan(shapes, ns, max_bytes=0):
    n = len(shapes)
    p = binding.param_array(shapes, [1] * n, [1] * n)
    need = binding.muon_workspace_bytes(p, n, ns, max_bytes)
    return binding.muon_plan_only(p, n, ns, need), p


def assert_full_coverage(ctx, shapes, ns, label=""):
    """Every output cell of every product is covered by a tile; a cell is covered twice only where the last
    512 x 128 tile of a column strip was shifted to end at the matrix edge (both tiles then write the same values).
    Works over all chunks of the plan: a matrix's tiles are all in the chunk the plan puts it in."""
    desc = [binding.muon_plan_describe(ctx, i) for i in range(len(shapes))]
    mc = ns != binding.MUON_F32
    chunks = binding.muon_plan_chunks(ctx)
    for product in ("gram", "poly", "apply", "apply_last"):
        sym = product in ("gram", "poly")
        cover, strip_cover = {}, {}
        for i, d in enumerate(desc):
            fine = d["tile_n"]
            tm, tn = d["m_pad"] // fine, d["n_pad"] // fine
            # output grid in fine cells: m x m for the symmetric products; X'^T (n x m) on the matrix cores, X' else
            cover[i] = np.zeros((tm, tm) if sym else ((tn, tm) if mc else (tm, tn)), dtype=np.int32)
            strip_cover[i] = np.zeros_like(cover[i])
        for chunk in range(chunks):
            for level in (0, 1):
                for mat, r0, c0, rows, cols, blocks in binding.muon_plan_tiles(ctx, chunk, product, level):
                    assert desc[mat]["chunk"] == chunk
                    fine = desc[mat]["tile_n"]
                    if not mc:
                        assert level == 0 and (rows, cols) == (64, 64)
                    elif level == 0:
                        assert (rows, cols) == (128, 128)
                    else:
                        assert (rows, cols) in ((256, 256), (512, 128))
                    assert r0 % fine == 0 and c0 % fine == 0 and r0 % 64 == 0 and c0 % 64 == 0
                    # plain bf16: a 256-tile on the diagonal of a symmetric product is computed from its upper triangle
                    halved = ns == binding.MUON_BF16 and sym and (rows, cols) == (256, 256) and r0 == c0
                    assert blocks == (36 if halved else rows * cols // 1024) or not mc
                    grid = cover[mat]
                    assert 0 <= r0 and r0 + rows <= grid.shape[0] * fine and 0 <= c0 and c0 + cols <= grid.shape[1] * fine
                    if sym:
                        assert c0 + cols > r0       # touches the diagonal or lies above it
                    sl = (slice(r0 // fine, (r0 + rows) // fine), slice(c0 // fine, (c0 + cols) // fine))
                    grid[sl] += 1
                    if (rows, cols) == (512, 128):
                        assert c0 + cols == grid.shape[1] * fine    # strips are the last 128 columns
                        strip_cover[mat][sl] += 1
        for i, grid in cover.items():
            twice = grid > 1
            assert (grid[twice] == 2).all() and (strip_cover[i][twice] == 2).all(), (label, product, shapes[i])
            assert twice.sum() <= 3, (label, product, shapes[i])    # at most one shifted tile: < 512 rows of overlap
            if sym:
                upper = np.triu(np.ones_like(grid))
                assert (grid[upper == 1] >= 1).all(), (label, product, shapes[i])
                # below the diagonal only what a diagonal 256-tile computes along with its upper part
                r = 256 // desc[i]["tile_n"] if mc else 1
                blocks_i, blocks_j = np.nonzero(np.tril(grid, -1))
                assert all(bi // r == bj // r for bi, bj in zip(blocks_i, blocks_j)), (label, product, shapes[i])
            else:
                assert (grid >= 1).all(), (label, product, shapes[i])


@pytest.mark.parametrize("ns", [binding.MUON_BF16, binding.MUON_BF16X2, binding.MUON_F32])
@pytest.mark.parametrize("name", sorted(SHAPE_SETS))
def test_every_output_tile_is_computed(name, ns):
    shapes = SHAPE_SETS[name]
    ctx, _ = plan(shapes, ns)
    try:
        assert binding.muon_plan_chunks(ctx) == 1
        assert_full_coverage(ctx, shapes, ns, name)
    finally:
        binding.lib().muon_destroy(ctx)


@pytest.mark.parametrize("seed", range(12))
def test_random_shape_lists_are_covered_in_every_chunking(seed):
    """Seeded random lists (dimensions from 1 to 3000, many of them multiples of 128 or 256 so that strips, moved
    tiles and fine leftovers all occur; sometimes many copies of one shape, which makes the launches persistent),
    planned once with room for everything and once with a workspace that forces several chunks."""
    rng = np.random.RandomState(1000 + seed)
    def dim():
        k = rng.randint(4)
        return int(rng.randint(1, 3000)) if k == 0 else int(128 * rng.randint(1, 24)) if k == 1 else int(256 * rng.randint(1, 12)) if k == 2 else int(64 * rng.randint(1, 40))
    shapes = [(dim(), dim()) for _ in range(int(rng.randint(1, 10)))]
    if seed % 3 == 0:
        shapes += [(int(256 * rng.randint(2, 6)), int(256 * rng.randint(2, 6)))] * int(rng.randint(20, 70))
    ns = [binding.MUON_BF16, binding.MUON_BF16X2, binding.MUON_F32][seed % 3 if seed % 3 != 0 else 0]
    n = len(shapes)
    p = binding.param_array(shapes, [1] * n, [1] * n)
    full = binding.muon_workspace_bytes(p, n, ns, 0)
    least = binding.muon_workspace_bytes(p, n, ns, 1)
    for ws in (full, least + (full - least) // 3):
        ctx = binding.muon_plan_only(p, n, ns, ws)
        try:
            assert_full_coverage(ctx, shapes, ns, "random%d" % seed)
        finally:
            binding.lib().muon_destroy(ctx)


@pytest.mark.parametrize("seed", range(6))
def test_random_lists_of_large_matrices_with_planes_are_covered(seed):
    """Several planes get coarse tiles, strips and moved tails only where matrices are large: sides up to 5000, one list in
    three of one shape (whose last round moves)."""
    rng = np.random.RandomState(2000 + seed)
    def dim():
        return int([rng.randint(3072, 5000), 128 * rng.randint(24, 40), 256 * rng.randint(12, 20)][rng.randint(3)])
    shapes = [(dim(), dim())] * int(rng.randint(2, 5)) if seed % 3 == 0 else \
        [(dim(), dim()) for _ in range(int(rng.randint(2, 4)))] + [(int(rng.randint(1, 1000)), int(rng.randint(1, 1000)))]
    ns = [binding.MUON_BF16X2, binding.MUON_BF16X3][seed % 2]
    n = len(shapes)
    p = binding.param_array(shapes, [1] * n, [1] * n)
    full = binding.muon_workspace_bytes(p, n, ns, 0)
    ctx = binding.muon_plan_only(p, n, ns, full)
    try:
        assert len(binding.muon_plan_tiles(ctx, 0, "gram", 1)) > 0 and len(binding.muon_plan_tiles(ctx, 0, "apply", 1)) > 0
        assert_full_coverage(ctx, shapes, ns, "planes%d" % seed)
    finally:
        binding.lib().muon_destroy(ctx)


def test_orientation_padding_and_tile_sizes():
    shapes = [(2048, 1408), (1408, 2048), (100, 130), (4096, 4096), (384, 640)]
    ctx, _ = plan(shapes, binding.MUON_BF16)
    try:
        d = [binding.muon_plan_describe(ctx, i) for i in range(5)]
        assert [x["transposed"] for x in d] == [1, 0, 0, 0, 0]
        assert [(x["m"], x["n"]) for x in d] == [(1408, 2048), (1408, 2048), (100, 130), (4096, 4096), (384, 640)]
        assert [(x["m_pad"], x["n_pad"]) for x in d] == [(1408, 2048), (1408, 2048), (128, 256), (4096, 4096), (384, 640)]
        assert [x["tile_m"] for x in d] == [256, 256, 128, 256, 256] and all(x["tile_n"] == 128 for x in d)
        # 1408 = 5 x 256 + 128: fifteen 256-tiles on or above the diagonal and the last 128 columns as three
        # 512 x 128 tiles (rows 0, 512 and, shifted to end at the edge, 896), all in the coarse launch
        gram = [t for t in binding.muon_plan_tiles(ctx, 0, "gram", 1) if t[0] == 0]
        assert sorted(t[1:5] for t in gram if t[3:5] == (512, 128)) == [(0, 1280, 512, 128), (512, 1280, 512, 128), (896, 1280, 512, 128)]
        assert len([t for t in gram if t[3:5] == (256, 256)]) == 15
        assert sorted(t[5] for t in gram if t[3:5] == (256, 256)) == [36] * 5 + [64] * 10
        assert not [t for t in binding.muon_plan_tiles(ctx, 0, "gram", 0) if t[0] == 0]
        app = [t for t in binding.muon_plan_tiles(ctx, 0, "apply", 1) if t[0] == 0]
        assert len([t for t in app if t[3:5] == (256, 256)]) == 8 * 5
        assert sorted(t[1] for t in app if t[3:5] == (512, 128)) == [0, 512, 1024, 1536]
        assert not [t for t in binding.muon_plan_tiles(ctx, 0, "apply", 0) if t[0] == 0]
        # 384 x 640 is too low for a 512-row strip tile: 128 x 128 tiles take what the 256-tiles leave
        gram = [t for t in binding.muon_plan_tiles(ctx, 0, "gram", 1) if t[0] == 4]
        assert [t[3:] for t in gram] == [(256, 256, 36)]
        assert len([t for t in binding.muon_plan_tiles(ctx, 0, "gram", 0) if t[0] == 4]) == 3
        # apply output is X'^T, 640 x 384: two 256-tiles, a 512 x 128 pair over the last 128 columns (rows 0 and 128),
        # and the last 128 rows beside them in two 128 x 128 tiles
        app = [t for t in binding.muon_plan_tiles(ctx, 0, "apply", 1) if t[0] == 4]
        assert sorted(t[1:5] for t in app if t[3:5] == (512, 128)) == [(0, 256, 512, 128), (128, 256, 512, 128)]
        assert sorted(t[1:5] for t in binding.muon_plan_tiles(ctx, 0, "apply", 0) if t[0] == 4) == [(512, 0, 128, 128), (512, 128, 128, 128)]
    finally:
        binding.lib().muon_destroy(ctx)


def test_described_tile_is_one_the_plan_uses():
    for shapes, ns in (([(1024, 1024)], binding.MUON_BF16), ([(4096, 4096), (100, 130), (384, 640)], binding.MUON_BF16),
                       ([(1024, 1024)] * 48, binding.MUON_BF16X2), ([(512, 512)], binding.MUON_F32)):
        ctx, _ = plan(shapes, ns)
        try:
            for i in range(len(shapes)):
                used = {t[3] for product in ("gram", "poly", "apply") for level in (0, 1)
                        for t in binding.muon_plan_tiles(ctx, 0, product, level) if t[0] == i}
                d = binding.muon_plan_describe(ctx, i)
                assert d["tile_m"] == (256 if used & {256, 512} else d["tile_n"]), (shapes, i, used)
        finally:
            binding.lib().muon_destroy(ctx)


def test_chunked_plan_keeps_each_matrix_in_one_chunk():
    shapes = [(256, 384)] * 5 + [(384, 256)] * 3
    n = len(shapes)
    p = binding.param_array(shapes, [1] * n, [1] * n)
    small = binding.muon_workspace_bytes(p, n, binding.MUON_BF16, 1)       # room for one matrix at a time
    ctx = binding.muon_plan_only(p, n, binding.MUON_BF16, small)
    try:
        chunks = binding.muon_plan_chunks(ctx)
        assert chunks == n
        seen = set()
        for c in range(chunks):
            mats = {t[0] for level in (0, 1) for t in binding.muon_plan_tiles(ctx, c, "apply", level)}
            assert len(mats) == 1 and not (mats & seen)
            assert {binding.muon_plan_describe(ctx, m)["chunk"] for m in mats} == {c}
            seen |= mats
        assert seen == set(range(n))
    finally:
        binding.lib().muon_destroy(ctx)


def test_plan_only_contexts_are_rejected_by_device_entry_points():
    import ctypes as C
    ctx, p = plan([(128, 256)], binding.MUON_BF16)
    L = binding.lib()
    try:
        hp = binding.default_hparams()
        assert L.muon_step(ctx, p, 1, C.byref(hp), None, None) == -1
        assert L.muon_debug_read_update(ctx, 0, C.c_void_p(256), 0, None) == -1
        assert L.muon_profile_enable(ctx, 1) == -1
        assert L.muon_plan_tiles(ctx, 1, 0, 0, None, 0) == -1      # no such chunk
        assert L.muon_plan_tiles(ctx, 0, 4, 0, None, 0) == -1
        assert L.muon_plan_tiles(ctx, 0, 0, 2, None, 0) == -1
    finally:
        L.muon_destroy(ctx)
    ctx = C.c_void_p(None)
    assert L.muon_plan_only(C.byref(ctx), p, 1, binding.MUON_BF16, 16) == -4
    assert ctx.value is None


def closed_form_executed_flops(m, n):
    """Matrix-core flops one Newton-Schulz iteration issues for an m x n matrix (m <= n, multiples of 128, m >= 512)
    under the planner's tiling: 256-tiles on and above the diagonal for the symmetric products, 256-tiles for the
    apply product, and 512-row tiles over the 128-wide strip an odd multiple of 128 leaves."""
    cm, cn, odd = m // 256, n // 256, (m // 128) % 2
    # diagonal 256-tiles: the 36 upper-triangle blocks of their 64
    sym_area = cm * (cm - 1) // 2 * 256 * 256 + cm * 36 * 1024 + odd * -(-m // 512) * 512 * 128
    app_area = cn * cm * 256 * 256 + odd * -(-n // 512) * 512 * 128 + ((n // 128) % 2) * 2 * cm * 128 * 128
    return 2 * (sym_area * n + sym_area * m + app_area * m)


def test_last_round_of_a_persistent_launch_goes_to_the_fine_launch():
    """Launches whose tiles all run the same K are persistent, one block per compute unit (256 when no device is
    asked): when the table is a few tiles longer than a multiple of that, those tiles are issued as four 128 x 128
    tiles each in the fine launch, and every block of the coarse launch gets the same number of tiles."""
    shapes = SHAPE_SETS["block_full"]
    ctx, _ = plan(shapes, binding.MUON_BF16)
    try:
        coarse = binding.muon_plan_tiles(ctx, 0, "apply", 1)
        fine = binding.muon_plan_tiles(ctx, 0, "apply", 0)
        assert len(coarse) == 3072 and len(fine) == 64
        assert all(t[3:5] == (128, 128) for t in fine)
        # whole 256 x 256 tiles: the four quarters of each moved tile are all there
        corners = {(t[0], t[1] // 256, t[2] // 256) for t in fine}
        assert len(corners) == 16
        for m, i, j in corners:
            assert {(m, 256 * i + a, 256 * j + b) for a in (0, 128) for b in (0, 128)} <= {t[:3] for t in fine}
        # the symmetric launches mix K = 4096 and K = 11008 in the Gram product: not persistent, nothing moved
        assert len(binding.muon_plan_tiles(ctx, 0, "gram", 1)) == 7 * 136
        assert len(binding.muon_plan_tiles(ctx, 0, "gram", 0)) == 0
    finally:
        binding.lib().muon_destroy(ctx)
    # 96 tiles over a multiple of 256 are too many to be worth a second launch: left alone
    ctx, _ = plan(SHAPE_SETS["block"], binding.MUON_BF16)
    try:
        assert len(binding.muon_plan_tiles(ctx, 0, "apply", 1)) == 1632
        assert len(binding.muon_plan_tiles(ctx, 0, "apply", 0)) == 0
    finally:
        binding.lib().muon_destroy(ctx)


@pytest.mark.parametrize("name", ["dense12_w1024", "block_w4096", "moe_bank_66x2048x1408"])
def test_bench_counts_the_flops_the_plan_issues(name):
    """bench.py's executed-flop figure is summed over the planner's tile tables; it must equal the closed form of the
    tiling for the benchmark shapes."""
    import bench
    from paper_2502_16982_amd import workloads
    wl = workloads.workload(name)
    want = sum(closed_form_executed_flops(min(a, b), max(a, b)) for a, b in wl.shapes)
    assert bench.executed_ns_flops(wl, 1) == want
    assert bench.executed_ns_flops(wl, 5) == 5 * want
    # symmetry saves between a quarter and a third of the nominal count on these shapes
    assert 0.62 < want / wl.ns_flops(1) < 0.78


@pytest.mark.parametrize("shape,product", [((4096, 4096), "gram"), ((4096, 11008), "apply"), ((11008, 4096), "apply")])
def test_tiles_that_run_together_on_a_die_share_operand_panels(shape, product):
    """Entry b of a tile table runs on accelerator die b % 8 (workgroups are handed out round-robin), one tile per
    compute unit, 32 at a time.  A die's sequence is a contiguous run of a blocked order of the tile grid (4 x 8 or
    8 x 4 blocks), so any 32 consecutive tiles of it lie in at most two blocks and touch at most 2 x 12 operand panels
    in that die's L2, against 33 for a row-major run; the first die's first 32 tiles are one whole block."""
    ctx, _ = plan([shape], binding.MUON_BF16)
    try:
        tiles = [t for t in binding.muon_plan_tiles(ctx, 0, product, 1) if t[3:5] == (256, 256)]
        worst = 0
        for die in range(8):
            seq = tiles[die::8]
            width = min(32, len(seq))
            for start in range(0, len(seq) - width + 1, width):
                block = seq[start:start + width]
                worst = max(worst, len({t[1] for t in block}) + len({t[2] for t in block}))
        assert worst <= 24, worst
        if product == "apply":
            first = tiles[0::8][:32]
            assert len({t[1] for t in first}) + len({t[2] for t in first}) == 12
    finally:
        binding.lib().muon_destroy(ctx)


def coarse_counts(shapes, ns):
    ctx, _ = plan(shapes, ns)
    try:
        return tuple(len(binding.muon_plan_tiles(ctx, 0, product, 1)) for product in ("gram", "apply"))
    finally:
        binding.lib().muon_destroy(ctx)


@pytest.mark.parametrize("ns,shapes,gram,apply", [
    # plain bf16: below one full round of coarse tiles only small matrices are quicker in fine tiles
    (binding.MUON_BF16, [(1024, 1024)] * 16, False, True),
    (binding.MUON_BF16, [(2048, 2048)] * 4, True, True),
    (binding.MUON_BF16, [(1536, 2048)] * 8, False, True),
    (binding.MUON_BF16, [(1792, 2048)] * 6, True, True),
    (binding.MUON_BF16, [(1536, 1536)] * 4, False, True),
    (binding.MUON_BF16, [(1280, 2560)] * 3, False, True),
    (binding.MUON_BF16, [(256, 8192)] * 5, False, False),
    # planes: large matrices, and long K loops in well-filled rounds
    (binding.MUON_BF16X2, [(1024, 1024)] * 48, False, False),
    (binding.MUON_BF16X2, [(1024, 4096)] * 24, False, False),
    (binding.MUON_BF16X2, [(1536, 8192)] * 6, False, False),
    (binding.MUON_BF16X2, [(1536, 8192)] * 12, True, True),
    (binding.MUON_BF16X2, [(1280, 10240)] * 8, False, False),
    (binding.MUON_BF16X2, [(1536, 6144)] * 12, True, False),
    (binding.MUON_BF16X2, [(2048, 2048)] * 7, False, True),
    (binding.MUON_BF16X2, [(2688, 3200)] * 7, False, True),
    (binding.MUON_BF16X2, [(2048, 8192)] * 4, True, True),
    (binding.MUON_BF16X2, [(2560, 10240)] * 4, True, True),
    (binding.MUON_BF16X2, [(2816, 11008)] * 4, False, True),
    (binding.MUON_BF16X2, [(4096, 4096)], True, True),
    (binding.MUON_BF16X3, [(2048, 2048)] * 7, True, True),
    (binding.MUON_BF16X3, [(2048, 4096)] * 7, True, True),
    (binding.MUON_BF16X3, [(2560, 2560)] * 4, True, True),
    (binding.MUON_BF16X3, [(1024, 4096)] * 24, False, False),
    # lists that mix K, and one that only has a small matrix beside the large ones
    (binding.MUON_BF16X2, [(2048, 2816)] * 3 + [(2944, 8832)] * 3, False, True),
    (binding.MUON_BF16X3, [(2048, 8192)] * 7 + [(1024, 1024)] * 4, False, True),
    (binding.MUON_BF16X3, [(2560, 10240)] * 4 + [(2560, 2560)] * 4, True, True),
    (binding.MUON_BF16X3, [(2048, 2816)] * 3 + [(2944, 8832)] * 3, False, True),
    (binding.MUON_BF16X2, [(2048, 8192)] * 4 + [(256, 256)], True, True),
    (binding.MUON_BF16X2, [(2304, 3840)] * 11, True, True),
])
def test_coarse_tiles_where_they_were_measured_to_be_quicker(ns, shapes, gram, apply):
    assert tuple(c > 0 for c in coarse_counts(shapes, ns)) == (gram, apply)


def test_one_more_matrix_does_not_move_all_the_others():
    """The choice between the launches goes by what the coarse tiles are like on average, not by the list's extremes."""
    for ns in (binding.MUON_BF16X2, binding.MUON_BF16X3):
        assert coarse_counts([(1024, 1024)] * 48, ns) == (0, 0)
        assert coarse_counts([(1024, 1024)] * 48 + [(3072, 3072)], ns) == (0, 0)
    assert coarse_counts([(1024, 1024)] * 16, binding.MUON_BF16) == (0, 256)
    assert coarse_counts([(1024, 1024)] * 16 + [(16, 2100)], binding.MUON_BF16)[0] == 0


@pytest.mark.parametrize("ns,shapes,forms", [
    # plain bf16: waves up to 24 entries, up to 36 with K <= 1024; the longer ring by the work, entries of the longest K
    ("bf16", [(512, 512)] * 2, ["waves", "waves", "waves"]),                      # 20, 20, 32 of K = 512
    ("bf16", [(512, 640)] * 2, ["waves", "waves", "ring4"]),                      # apply: 40
    ("bf16", [(640, 1024)] * 2, ["waves", "waves", "quarters"]),                  # 30, 30 of K = 1024 and 640; apply: 80
    ("bf16", [(640, 1152)] * 2, ["ring4", "waves", "quarters"]),
    ("bf16", [(128, 300)] * 36, ["waves", "waves", "quarters"]),
    ("bf16", [(128, 300)] * 37, ["ring4", "ring4", "quarters"]),
    ("bf16", [(128, 300)] * 68, ["ring4", "ring4", "whole"]),
    ("bf16", [(128, 300)] * 69, ["quarters", "quarters", "whole"]),
    ("bf16", [(1024, 1024), (256, 8000), (256, 8000), (256, 8000)], ["ring4", "ring4", "quarters"]),   # Gram product: 45 entries, the work of 14; apply: 442, of 159
    ("bf16", [(1000, 3001)] * 2 + [(777, 777)] * 2 + [(63, 4097)] * 2, ["ring4", "quarters", "whole"]),    # 130, of 67
    # two planes: up to three quarters of the compute units, and a little more than all of them up to K = 2048
    ("bf16x2", [(128, 300)] * 64, ["ring4", "ring4", "quarters"]),
    ("bf16x2", [(128, 300)] * 65, ["quarters", "quarters", "quarters"]),
    # Gram product: 80 entries, the work of 22; apply: 472, the work of 302, with a block's fixed cost of 399; 344, of 259 and 308
    ("bf16x2", [(300, 700)] * 6 + [(700, 300)] * 6 + [(128, 4096)] * 8, ["ring4", "quarters", "whole"]),
    ("bf16x2", [(300, 700)] * 6 + [(700, 300)] * 6 + [(128, 2048)] * 8, ["ring4", "quarters", "quarters"]),
    ("bf16x2", [(128, 384)] * 192, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(128, 384)] * 193, ["whole", "quarters", "whole"]),
    ("bf16x2", [(128, 384)] * 257, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(128, 256)] * 256, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(128, 256)] * 160, ["quarters", "quarters", "quarters"]),
    ("bf16x2", [(128, 256)] * 161, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(128, 128)] * 320, ["quarters", "quarters", "quarters"]),
    ("bf16x2", [(128, 128)] * 321, ["whole", "whole", "whole"]),
    ("bf16x2", [(128, 2048)] * 300, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(128, 2176)] * 300, ["whole", "quarters", "whole"]),
    # apply product, entries of a longer K and of K = 128: 270 and 72, the work of 294 of 384 (322); 240 and 168, of 296 (360), and of
    # 274 of 640
    ("bf16x2", [(384, 640)] * 18 + [(16, 768)] * 12, ["quarters", "quarters", "quarters"]),
    ("bf16x2", [(592, 384)] * 16 + [(16, 768)] * 28, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(1984, 592)] * 3 + [(16, 768)] * 28, ["quarters", "ring4", "whole"]),
    # the longer ring by work: two planes up to 51, three up to 40
    ("bf16x2", [(250, 2048)] * 17 + [(16, 128)] * 14, ["quarters", "quarters", "whole"]),
    ("bf16x2", [(250, 2048)] * 16 + [(16, 128)] * 48, ["ring4", "quarters", "whole"]),
    ("bf16x3", [(250, 2048)] * 13 + [(16, 128)] * 32, ["quarters", "quarters", "quarters"]),
    ("bf16x3", [(250, 2048)] * 12 + [(16, 128)] * 64, ["ring4", "quarters", "quarters"]),
    # three planes: half of the compute units, more with a short K; a badly filled last round, by K
    ("bf16x3", [(128, 256)] * 512, ["quarters"] * 3),                             # full rounds of K = 128 and 256
    ("bf16x3", [(128, 256)] * 513, ["quarters", "quarters", "whole"]),            # apply: 1026, more than 1024
    ("bf16x3", [(128, 384)] * 200, ["quarters"] * 3),
    ("bf16x3", [(128, 384)] * 201, ["whole", "quarters", "quarters"]),
    ("bf16x3", [(128, 384)] * 435, ["quarters", "quarters", "whole"]),            # Gram product: 0.8496 of two rounds
    ("bf16x3", [(128, 384)] * 436, ["whole", "quarters", "whole"]),
    ("bf16x3", [(128, 896)] * 150, ["quarters", "quarters", "whole"]),
    ("bf16x3", [(128, 896)] * 151, ["whole", "quarters", "whole"]),
    ("bf16x3", [(128, 4096)] * 128, ["quarters", "quarters", "whole"]),
    ("bf16x3", [(128, 4096)] * 129, ["whole", "quarters", "whole"]),
    ("bf16x3", [(128, 1024)] * 409, ["quarters", "quarters", "whole"]),
    ("bf16x3", [(128, 1024)] * 410, ["whole", "quarters", "whole"]),
    ("bf16x3", [(128, 2048)] * 332, ["quarters", "quarters", "whole"]),
    ("bf16x3", [(128, 2048)] * 333, ["whole", "quarters", "whole"]),
    ("bf16x3", [(128, 4096)] * 291, ["quarters", "quarters", "whole"]),
    ("bf16x3", [(128, 4096)] * 292, ["whole", "quarters", "whole"]),
    # Gram product, K = 640 and 128: 215 and 108 entries, the work of 237, of 275 with a block's fixed cost: a second round, badly
    # filled; 215 and 40 of 223 and 238: one round
    ("bf16x3", [(128, 600)] * 215 + [(128, 128)] * 108, ["quarters", "quarters", "whole"]),
    ("bf16x3", [(128, 600)] * 215 + [(128, 128)] * 40, ["whole", "quarters", "whole"]),
])
def test_blocks_of_the_fine_launches(ns, shapes, forms):
    """The lines between 128-wide blocks, 64-wide ones with either ring and single waves."""
    from tests.plan_routes import fine_forms
    assert fine_forms(shapes, ns) == forms


@pytest.mark.parametrize("ns,count,coarse,fine", [
    ("bf16x2", 4, 512, 128), ("bf16x2", 6, 768, 192), ("bf16x2", 8, 1088, 0),
    ("bf16x3", 4, 512, 128), ("bf16x3", 6, 816, 0), ("bf16x3", 8, 1088, 0), ("bf16", 8, 1024, 256)])
def test_planes_move_a_tail_only_where_it_runs_in_quarters(ns, count, coarse, fine):
    """136 symmetric tiles for each 4096 x 4096: 32, 48 or 64 are beyond a multiple of 256.  With planes they go to the fine launch
    where four entries for each still run as 64-wide blocks; persistent launches (plain bf16) move up to 64."""
    from tests.plan_routes import routes
    tables, _ = routes([(4096, 4096)] * count, ns)
    for product in ("gram", "poly"):
        assert tables[product, 1][0] == coarse and tables[product, 0][0] == fine
        assert fine == 0 or ns == "bf16" or tables[product, 0][1] != "whole"


@pytest.mark.parametrize("ns,shapes,fold", [
    # one wave per 32 x 32: four partials (64 x 64 tiles of the padded matrix) per lane
    ("bf16", [(64, 8192)], True), ("bf16", [(64, 8193)], False), ("bf16", [(512, 2048)], True), ("bf16", [(512, 2049)], False),
    # blocks of four waves: four per thread
    ("bf16", [(64, 8193)] * 25, True), ("bf16", [(64, 32768)] * 25, True), ("bf16", [(64, 32769)] * 25, False),
    ("bf16x2", [(64, 32768)], True), ("bf16x2", [(64, 32769)], False), ("f32", [(64, 65536)], True), ("f32", [(64, 65537)], False),
    # no quarters, no fold
    ("bf16", [(128, 128)] * 177, False)])
def test_norm_is_folded_up_to_four_partials_per_thread(ns, shapes, fold):
    from tests.plan_routes import routes
    assert routes(shapes, ns)[1] == fold


def test_bench_counts_the_plane_pairs_that_are_multiplied():
    """Two planes: three products a block, and the polynomial's fourth over the whole of K in fine tiles, over the block's own rows
    and columns in coarse ones, whose blocks below the diagonal and in two strips count once.  Three planes: six products."""
    import bench
    from paper_2502_16982_amd import workloads
    block = 2 * 128 * 128

    def count(shapes, ns):
        return bench.executed_ns_flops(workloads.custom("count", shapes, ns_dtype=ns), 1, ns)

    def sides(s):
        return s * (s + 1) // 2

    # 1024 x 1280, all fine: 36 blocks on and above the diagonal, 80 of X'^T
    assert count([(1024, 1280)], "bf16x2") == block * (36 * (3 * 1280 + 4 * 1024) + 80 * 3 * 1024)
    assert count([(1024, 1280)], "bf16x3") == block * 6 * (36 * (1280 + 1024) + 80 * 1024)
    # 4096^2 and, with strips, two of 3200 x 3328, all coarse
    for m, n, copies in ((4096, 4096, 1), (3200, 3328, 2)):
        tm, tn = m // 128, n // 128
        gram, apply = sides(tm) * n, tm * tn * m
        assert count([(m, n)] * copies, "bf16x3") == copies * block * 6 * (gram + sides(tm) * m + apply)
        own = tm * 128 + (sides(tm) - tm) * 256
        assert count([(m, n)] * copies, "bf16x2") == copies * block * (3 * (gram + sides(tm) * m + apply) + own)
