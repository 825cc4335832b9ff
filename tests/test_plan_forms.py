"""Which launches the lists of the GPU tests take, from the planner on the host: the forms that those tests mean to run."""
import pytest

from tests import plan_routes
from tests.test_gpu_gram_route import ALONE, BESIDE, PAIRED

FORMS = {"waves", "quarters", "ring4", "ring128", "whole"}


def test_the_128_wide_ring_is_reached_by_every_product():
    """Lists of test_same_bits_from_the_128_wide_ring."""
    forms = [plan_routes.fine_forms([s] * n, "bf16") for s, n in [((256, 300), 64), ((384, 400), 30), ((1024, 1000), 7), ((1152, 1300), 2)]]
    assert [{f[i] == "ring128" for f in forms} for i in range(3)] == [{True, False}] * 3
    assert plan_routes.routes([(256, 300)] * 64, "bf16")[1] and not plan_routes.routes([(256, 300)] * 90, "bf16")[1]      # folds the norm


def test_fp32_entries_behind_full_rounds():
    assert plan_routes.tails([(512, 512)] * 13) == {"gram": 0, "poly": 0, "apply": 64}
    assert plan_routes.tails([(512, 4160)] * 15)["gram"] == 28         # two places per compute unit
    assert not any(plan_routes.tails([(512, 512)] * n)["apply"] for n in (12, 14)) and not any(plan_routes.tails([(448, 512)] * 15).values())


def test_launches_of_the_gram_route():
    alone = [plan_routes.pair_routes(shapes) for shapes, _ in ALONE]
    for product in ("gram", "sym"):
        forms = {r["pairs"].get(("none", product), (0, "-"))[1] for r in alone}
        assert forms >= {"waves", "quarters", "ring4", "ring128"}, (product, forms)
    assert any(r["coarse"][1][0] > 0 for r in alone) and any(r["coarse"][1][1] > 0 for r in alone)
    both = [plan_routes.pair_routes(s) for s in [b[0] for b in BESIDE] + PAIRED]
    assert {form for r in both for (i, j), (_, form) in r["pairs"].items() if i != "none" and j != "none"} >= FORMS
    assert any(r["shared"] for r in both)
    assert {p for r in both for p in r["beside"]} == {(i, p) for i in (0, 1) for p in ("gram", "sym", "apply")}
    assert {r["lone"][1] for r in both if r["lone"]} >= {"quarters", "ring128", "whole"}
    joint = [r["joint"] for r in both]                                  # both apply products from one table, strips among them
    assert {n > 0 for n, _ in joint} == {True, False} and {s for n, s in joint if n} == {True, False}
    assert {tuple(c[1] > 0 for c in r["coarse"]) for r in both if r["joint"][0]} >= {(True, False), (False, True), (True, True)}
    few = plan_routes.pair_routes(PAIRED[3])                            # an apply product in fine tiles, symmetric ones with coarse tiles
    assert few["coarse"][0][1] == 0 and few["coarse"][1][0] > 0 and few["lone"][2] == "whole"


@pytest.mark.parametrize("full,beside", [([(1024, 1024)] * 8 + [(640, 2560)], True), ([(2048, 2048)] * 8 + [(1024, 4096)], False)])
def test_only_idle_compute_units_take_the_other_group_in(full, beside):
    """An apply product of 128 coarse tiles is fine altogether; one of 512, two full rounds, leaves nothing idle."""
    r = plan_routes.pair_routes(full)
    assert (r["coarse"][0][1] == 0) == beside and not r["beside"]
