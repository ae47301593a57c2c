"""The rectangular GEMM tiles, on the host: their stage schedule (tests/rect_schedule_check.cpp) and, from the metadata of
the library as built here, their register allocation."""
import os
import re
import subprocess

import pytest

from test_kernel_registers import LIB, READELF, _kernels, forms

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12526_amd", "csrc")
HEADER = os.path.join(CSRC, "mom_gemm_rect_schedule.h")


def _build_and_run(tmp_path, include_dir):
    exe = os.path.join(str(tmp_path), "rect_schedule_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", include_dir, "-I", CSRC, "-o", exe,
                    os.path.join(ROOT, "tests", "rect_schedule_check.cpp")], check=True)
    return subprocess.run([exe], capture_output=True, text=True)


def test_schedule_as_shipped_passes(tmp_path):
    r = _build_and_run(tmp_path, CSRC)
    assert r.returncode == 0 and ": ok" in r.stdout, r.stdout


@pytest.mark.parametrize("old,new,says", [
    ("int barrier_row() { return 1; }", "int barrier_row() { return 2; }", "landed"),
    ("(slots(MB, NB, WGT) == 3 ? NB : 0);", "(slots(MB, NB, WGT) == 3 ? NB : 0) + 1;", "landed"),
    ("OuterRead{row - 1, 1}", "OuterRead{row, 1}", "refilled"),
    ("const int p = (row + OB - 1) % OB * IB + pair;", "const int p = row % OB * IB + pair;", "loaded"),
    ("return j < n ? Load{f, j} : Load{1 - f, j - n};", "return j < n ? Load{f, j} : Load{1 - f, j - n + 1};", "index"),
    ("if (i == 4 && slots(MB, NB, f) == 2) return {1 - f, 2};", "if (i == 4 && slots(MB, NB, f) == 2) return {f, 2};", "slot"),
])
def test_a_planted_mistake_is_caught(tmp_path, old, new, says):
    """Planted in a copy of the header, on the CPU."""
    inc = os.path.join(str(tmp_path), "inc")
    os.makedirs(inc)
    text = open(HEADER).read()
    assert text.count(old) == 1, f"header text changed: {old}"
    with open(os.path.join(inc, "mom_gemm_rect_schedule.h"), "w") as f:
        f.write(text.replace(old, new))
    r = _build_and_run(tmp_path, inc)
    assert r.returncode != 0 and says in r.stdout, r.stdout[-2000:]


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
def test_acc_registers_hold_the_accumulators_and_nothing_else(tmp_path):
    if not os.path.exists(LIB):
        from paper_2504_12526_amd import build
        build.build()
    seen = []
    for name, v in _kernels(tmp_path).items():
        m = re.search(r"16gemm_rect_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", name)
        if m:
            seen.append(tuple(int(x) for x in m.groups()))
            assert v["agpr"] == 4 * (int(m[2]) // 32) * (int(m[3]) // 32), (name, v)
            assert not (v["vgpr_spill_count"] or v["sgpr_spill_count"] or v["private_segment_fixed_size"]), (name, v)
    # (projection, token rows, weight rows, non-temporal weights): every form of the lists, and no other
    want = [(0, *f, 0) for f in forms("MOM_RECT_FORMS_DOWN")] + [(1, *f, nt) for f in forms("MOM_RECT_FORMS_GATEUP") for nt in (0, 1)]
    assert sorted(seen) == sorted(want)
