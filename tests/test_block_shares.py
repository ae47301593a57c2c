"""Several workgroups per block of token rows, each a share of the output columns: the shares on the host (tests/block_share_check.cpp), the bits on
the GPU."""
import os
import subprocess

import pytest
import torch

from paper_2504_12526_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12526_amd", "csrc")


@pytest.mark.parametrize("old,new", [("", ""),
                                     ("share = (groups + parts - 1) / parts;", "share = groups / parts;"),          # a last part too many, the ninth
                                     ("return ((uint32_t)H / 32 + share - 1) / (uint32_t)share;", "return (uint32_t)H / 32 / (uint32_t)share;")])
def test_shares(tmp_path, old, new):
    text = open(os.path.join(CSRC, "mom_gemm_forms.h")).read()
    assert not old or text.count(old) == 1, old
    with open(os.path.join(str(tmp_path), "mom_gemm_forms.h"), "w") as f:
        f.write(text.replace(old, new) if old else text)
    exe = os.path.join(str(tmp_path), "block_share_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", str(tmp_path), "-o", exe, os.path.join(ROOT, "tests", "block_share_check.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert (r.returncode == 0) == (not old), r.stdout


# one share; two of four groups; last shares of fewer (160 columns: 4 and 1 groups, 1056: 5 ... and 3); an odd contraction; 16 and 32 rows per block
@pytest.mark.gpu
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("S,H,I", [(40, 128, 96), (512, 256, 1024), (33, 160, 224), (100, 1056, 96), (700, 1056, 160), (17, 1024, 32), (2100, 288, 96)])
def test_shares_give_the_bits_of_the_full_tiles(S, H, I, rows):
    from test_gpu_short_forms import _full_tiles, _inputs
    t = _inputs(S, H, I, S + H, 0.05)
    ref = _full_tiles(*t)[0]
    out, ws = torch.full_like(t[0], float("nan")), torch.full((S * I,), float("nan"), dtype=torch.bfloat16, device="cuda")
    try:
        binding.mom_debug_force_block(rows)
        binding.mom_mlp_prefill(*t, 0, out, ws)
        torch.cuda.synchronize()
    finally:
        binding.mom_debug_force_block(0)
    assert bool(torch.isnan(ws).all())                 # blocks it is
    assert torch.equal(out.view(torch.int16), ref)
