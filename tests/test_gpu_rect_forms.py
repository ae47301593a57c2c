"""The rectangular GEMM tiles on the GPU: every form against the 256 x 256 tiles bit for bit, with token and weight rows around
the edges of its tiles, contractions of a half stage only, one, two and several turns of the rings, and a half stage behind them."""
import os
import re

import pytest
import torch

from paper_2504_12526_amd import binding, synth
from test_gpu_short_forms import _full_tiles, _inputs, _run

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_TEXT = open(os.path.join(ROOT, "paper_2504_12526_amd", "csrc", "mom_gemm_forms.h")).read()
FORMS = sorted({tuple(int(v) for v in f.split(",")) for t in re.findall(r"#define MOM_RECT_FORMS_\w+\(X\)((?:.*\\\n)*.*\n)", _TEXT)
                for f in re.findall(r"X\(([\d, ]+)\)", t)})


@pytest.fixture
def rect_form():
    yield binding.mom_debug_force_rect_form
    binding.mom_debug_force_rect_form(0, 0)
    binding.mom_debug_force_short_form(0, 0)
    binding.mom_debug_force_gemm_form(0, 0, 0)


@pytest.mark.parametrize("tm,tn", FORMS)
def test_form_gives_the_bits_of_the_full_tiles(tm, tn, rect_form):
    # I = 32, 64, 96, 160, ...: down with 0, 1, 1, 2, ... whole stages; H likewise for gate/up
    for S, H, I in ((1, 32, 64), (tm - 1, 64, 32), (tm + 1, 96, tn), (2 * tm, tn, 160), (2 * tm + 5, 448, tn + 32),
                    (4 * tm + 3, 1056, tn // 2 + 32 - tn // 2 % 32), (tm + 9, 3 * tn + 32, 480)):
        H, I = H + -H % 32, I + -I % 32
        t = _inputs(S, H, I, S + H, 0.05)
        ref = _full_tiles(*t)
        rect_form(tm, tn)
        got = _run(*t)
        torch.cuda.synchronize()
        rect_form(0, 0)
        assert torch.equal(got[1], ref[1]), f"intermediate S={S} H={H} I={I}"
        assert torch.equal(got[0], ref[0]), f"out S={S} H={H} I={I}"


@pytest.mark.parametrize("tm,tn", FORMS)
def test_form_with_non_temporal_weights(tm, tn, rect_form):
    # a layer of 336 MiB: one or two token tiles read their gate/up weights past the Infinity Cache
    wl = synth.Workload("large", S=2 * tm, H=8192, I=7168, mini_seq=0, seed=7, w_std=0.02)
    x, *w = synth.mlp_inputs(wl, device="cuda")
    for S, mini_seq in ((tm - 3, 0), (2 * tm, tm + 5)):
        t = (x[:S].contiguous(), *w)
        ref = _full_tiles(*t)
        rect_form(tm, tn)
        got = _run(*t, mini_seq)
        torch.cuda.synchronize()
        rect_form(0, 0)
        assert torch.equal(got[0], ref[0]), f"S={S} mini_seq={mini_seq}"


def test_rows_where_the_choice_takes_them(rect_form):
    # as chosen, at the production contraction lengths: one and several rounds, either projection
    for name in ("llama3_8b_32k", "qwen25_7b_256k"):
        x, *w = synth.mlp_inputs(synth.WORKLOADS[name], device="cuda", S=3000)
        for S in (97, 180, 288, 384, 450, 600, 700, 1300, 2300, 3000):
            t = (x[:S].contiguous(), *w)
            ref = _full_tiles(*t)
            got = _run(*t)
            torch.cuda.synchronize()
            assert torch.equal(got[1], ref[1]) and torch.equal(got[0], ref[0]), f"{name} S={S}"


def test_forced_rect_form_validation(rect_form):
    for f in ((48, 16), (0, 64), (-160, 160), (256, 256)):
        assert binding.lib().mom_debug_force_rect_form(*f) == binding.MOM_ERR_SHAPE
