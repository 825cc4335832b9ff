"""The kernels the planner picks for a list of matrices, from the planner itself, on the host (plan_routes_main.cpp)."""
import functools
import os
import shutil
import subprocess
import tempfile

from paper_2502_16982_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PRODUCTS = ("gram", "poly", "apply")


@functools.lru_cache(maxsize=None)
def program():
    gxx = shutil.which("g++")
    assert gxx, "g++ not found"
    folder = tempfile.TemporaryDirectory()
    exe = os.path.join(folder.name, "plan_routes")
    build = subprocess.run([gxx, "-std=c++17", "-O1", os.path.join(ROOT, "paper_2502_16982_amd", "csrc", "muon_plan.cpp"),
                            os.path.join(ROOT, "tests", "plan_routes_main.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    return exe, folder                 # the folder lives as long as the cache


@functools.lru_cache(maxsize=None)
def _routes(shapes, ns, compute_units):
    run = subprocess.run([program()[0], str(binding.NS_DTYPES[ns]), str(compute_units)] + [str(v) for s in shapes for v in s],
                         capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, (run.returncode, run.stderr)
    lines = [line.split() for line in run.stdout.splitlines()]
    fold = [bool(int(line[1])) for line in lines if line[0] == "fold"]
    tables = {(line[1], int(line[2])): (int(line[3]), line[4]) for line in lines if line[0] == "0"}
    tails = {line[1]: int(line[5]) for line in lines if line[0] == "0" and line[2] == "0"}
    pairs = {"pairs": {(line[2], line[3]): (int(line[4]), line[5]) for line in lines if line[0] == "pair" and line[1] == "0"},
             "coarse": [tuple(int(v) for v in line[3:]) for line in lines if line[0] == "coarse" and line[1] == "0"],
             "lone": next(((int(line[2]), line[3], line[4]) for line in lines if line[0] == "lone" and line[1] == "0"), None),
             "shared": next((int(line[2]) for line in lines if line[0] == "shared" and line[1] == "0"), 0),
             "joint": next(((int(line[2]), bool(int(line[3]))) for line in lines if line[0] == "joint" and line[1] == "0"), (0, False)),
             "beside": {(int(line[2]), line[3]) for line in lines if line[0] == "beside" and line[1] == "0"}}
    return tables, fold[0], tails, pairs


def routes(shapes, ns, compute_units=256):
    """{(product, level): (entries, form)} of a list planned whole, form one of "whole", "quarters" (64-wide blocks, ring of
    three), "ring4" (of four), "waves" (32-wide), "ring128" (128-wide, ring of four); and whether the first Gram launch adds up the norm.
    Empty for lists with matrices of the Gram route (pair_routes)."""
    return _routes(tuple(tuple(s) for s in shapes), ns, compute_units)[:2]


def tails(shapes, ns="f32", compute_units=256):
    """{product: last entries of its fine launch that run in quarters behind it}."""
    return _routes(tuple(tuple(s) for s in shapes), ns, compute_units)[2]


def pair_routes(shapes, compute_units=256):
    """Of a list with matrices of the Gram route, planned whole.  "pairs": {(product of the others, product of theirs): (entries, form) of the
    fine launch}, "coarse": coarse entries of the symmetric and of the apply products of either group, "lone": entries and forms of their symmetric
    products without the others', "shared": entries of the table of both, "joint": those of both apply products' and whether strips are among them,
    "beside": {(group, product)} that share the other's apply launch."""
    return _routes(tuple(tuple(s) for s in shapes), "bf16", compute_units)[3]


def fine_forms(shapes, ns):
    """Form of the fine launch of each product, in order; "-" where it has none."""
    tables, _ = routes(shapes, ns)
    return [tables[p, 0][1] if tables[p, 0][0] else "-" for p in PRODUCTS]
