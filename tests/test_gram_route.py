"""The Gram route of plain bf16 (two iterations at a time on the Gram matrix) without a GPU: its line and tables from the
planner under sanitizers, and the LDS waits in the generated code of its kernels."""
import os
import shutil
import subprocess

import pytest

from tests import asm_lds_hazards as hz
from tests.test_kmajor_asm_hazards import compile_to_asm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tables_of_the_gram_route(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "gram_route")
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall", "-Wextra",
                            os.path.join(ROOT, "paper_2502_16982_amd", "csrc", "muon_plan.cpp"), os.path.join(ROOT, "tests", "gram_route_main.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    run = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    assert run.returncode == 0 and "gram route ok" in run.stdout, run.stdout + run.stderr


def scratch_of(lines):
    """Scratch instructions of a kernel, and those in the loops over K (8 and more MFMAs between a label and the nearest branch back to it,
    within 600 lines of code and without an inner loop)."""
    text = [t for _, t in lines]
    at = {t[:-1]: i for i, t in enumerate(text) if t.endswith(":")}
    loops = []
    for i, t in enumerate(text):
        to = t.split()[-1] if t.startswith(("s_branch", "s_cbranch")) else None
        if to in at and at[to] < i and sum("v_mfma" in x for x in text[at[to]:i]) >= 8:
            loops.append((at[to], i))
    inner = [(a, b) for a, b in loops if b - a < 600 and not any((c, d) != (a, b) and a <= c and d <= b for c, d in loops)]
    assert inner
    spills = [i for i, t in enumerate(text) if t.startswith("scratch_")]
    return len(spills), sum(a <= i <= b for i in spills for a, b in inner)


def test_generated_code_of_the_paired_kernels_waits_for_every_lds_read_it_uses(tmp_path_factory):
    kernels = {k: v for k, v in hz.split_kernels(compile_to_asm(tmp_path_factory, "kernels_gemm_pair.hip")).items() if "ns_pair" in k}
    assert len(kernels) == 12        # fine, 128-wide ring, 64-wide with two rings, lone waves, shared symmetric, shared apply, beside K-major coarse tiles of bf16 and f16, coarse in
                                     # f16, K-major coarse of bf16 and f16
    # registers spilled around the epilogues of the kernels that hold several coarse bodies, none in a loop over K
    most = {"ns_pair_sym_kernel": 32, "ns_pair_apply_kernel": 8, "ns_pair_beside_kernel": 8, "ns_pair_coarse_kernel": 4}
    for name, lines in kernels.items():
        spilled, in_loops = scratch_of(lines)
        print(name, spilled, in_loops)
        assert spilled <= next((n for k, n in most.items() if k in name), 0) and in_loops == 0, (name, spilled, in_loops)
        assert any("v_mfma_f32_32x32x16_f16" in t for _, t in lines) or "Lb1E" in name and "4Bf16" in name or "pair_apply" in name, name
        assert hz.check_kernel(lines) == [], name


def test_generated_code_of_the_128_wide_ring_waits_for_every_lds_read_it_uses(tmp_path_factory):
    kernels = {k: v for k, v in hz.split_kernels(compile_to_asm(tmp_path_factory, "kernels_gemm_bf16.hip")).items() if "ns_ring128" in k}
    assert len(kernels) == 2         # {k-contiguous, K-major}
    for name, lines in kernels.items():
        assert not any("scratch_" in t for _, t in lines), name          # no spills
        assert hz.check_kernel(lines) == [], name
