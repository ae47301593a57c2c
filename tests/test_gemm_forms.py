"""The short GEMM forms and the rule that picks one, checked on the host (tests/gemm_forms_check.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12526_amd", "csrc")
HEADER = os.path.join(CSRC, "mom_gemm_forms.h")


def _build_and_run(tmp_path, include_dir):
    exe = os.path.join(str(tmp_path), "gemm_forms_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", include_dir, "-o", exe,
                    os.path.join(ROOT, "tests", "gemm_forms_check.cpp")], check=True)
    return subprocess.run([exe], capture_output=True, text=True)


def test_forms_and_choice(tmp_path):
    r = _build_and_run(tmp_path, CSRC)
    assert r.returncode == 0 and ": ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("old,new,says", [
    # the 256-row tiles priced on a grid of more tiles than they run on
    ("        const TileGrid g = tile_grid(M, N, false, f);\n        const double t = launch_time(g,",
     "        const TileGrid g = tile_grid(M + M / 4, N, false, f);\n        const double t = launch_time(g,", "rounds, 256 x"),
    # the last, shorter token tile forgotten
    ("const uint32_t tm = ((uint32_t)M + f.tm - 1) / f.tm,", "const uint32_t tm = M < f.tm ? 1 : (uint32_t)M / f.tm,", "rows of M="),
    # a step in the time of a launch: neighbouring row counts alternate between forms
    ("last < 0.72 ? (0.72 - last) / 0.32 : 0;", "last < 0.72 ? (M & 1) : 0;", "between two runs of"),
    # W_down taken to be in the cache whatever the gate/up launch before it does, and that launch in more than one group
    ("weights_once(gateup.grid.tiles_m, K, N, true) && weights_fit(N, K)", "weights_fit(N, K)", "W_down kept"),
    ("one_group = to_pass_by(M, N, K, more);", "one_group = false;", "W_down displaced"),
    # the last, shorter group of token tiles walked as a whole one
    ("const int gsz = tiles_m - first_m < group_m ? tiles_m - first_m : group_m;", "const int gsz = group_m;", "of M="),
    # the rows of W_up behind those of a whole tile instead of half a one
    ("half * HR + src, src}", "half * TN + src, src}", "block of"),
    # a wait that lets one load too many of the stage be on its way, that forgets the other stage of its group, and that waits for more than it needs
    ("n = r + (ahead - r) * loads;", "n = r + (ahead - r) * loads + 1;", "waited for at"),
    ("n = r + (ahead - r) * loads;", "n = ahead * loads + 0 * r;", "waited for at"),
    ("return nstg - 2 - t % group; }", "return nstg - 3 - t % group; }", "waited for at"),
    # a group requested one stage early: into a slot that is still to be read
    ("t % group == group - 1 ? t + nstg - group + 1 : -1", "t % group == group - 1 ? t + nstg - group + 2 : -1", "slot of stage"),
])
def test_a_planted_mistake_is_caught(tmp_path, old, new, says):
    """Planted in a copy of the header, on the CPU."""
    inc = os.path.join(str(tmp_path), "inc")
    os.makedirs(inc)
    text = open(HEADER).read()
    assert text.count(old) == 1, f"header text changed: {old}"
    with open(os.path.join(inc, "mom_gemm_forms.h"), "w") as f:
        f.write(text.replace(old, new))
    r = _build_and_run(tmp_path, inc)
    assert r.returncode != 0 and says in r.stdout, r.stdout[-2000:]
