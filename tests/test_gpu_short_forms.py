"""The GEMM forms for few token rows on the GPU: every form against the 256-row tiles bit for bit at the edges of its
tiles, over several groups of token tiles, with every length of the final, shorter stage, and with weights by non-temporal
loads; the library's own choice at production contraction lengths."""
import os
import re

import pytest
import torch

import oracle
from paper_2504_12526_amd import binding, synth

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_TEXT = open(os.path.join(ROOT, "paper_2504_12526_amd", "csrc", "mom_gemm_forms.h")).read()
_SHAPES = {d: sorted({tuple(int(v) for v in f.split(",")[:2]) for f in re.findall(r"X\(([\d, ]+)\)", t)})
           for d, t in re.findall(r"#define MOM_SHORT_FORMS_(DOWN|GATEUP)\(X\)((?:.*\\\n)*.*\n)", _TEXT)}
FORMS = sorted(set(_SHAPES["DOWN"] + _SHAPES["GATEUP"]))


@pytest.fixture
def short_form():
    yield binding.mom_debug_force_short_form
    binding.mom_debug_force_short_form(0, 0)
    binding.mom_debug_force_gemm_form(0, 0, 0)


def _inputs(S, H, I, seed, std):
    wl = synth.Workload("short", S=S, H=H, I=I, mini_seq=0, seed=seed, w_std=std)
    return synth.mlp_inputs(wl, device="cuda")


def _run(x, wg, wu, wd, mini_seq=0):
    """out and the intermediate (of the last mini-sequence), both poisoned before."""
    S, I = x.shape[0], wg.shape[0]
    out = torch.full_like(x, float("nan"))
    ws = torch.full(((mini_seq or S) * I,), float("nan"), dtype=torch.bfloat16, device=x.device)
    binding.mom_mlp_prefill(x, wg, wu, wd, mini_seq, out, ws)
    return out.view(torch.int16), ws.view(torch.int16)


def _full_tiles(*t):
    binding.mom_debug_force_short_form(0, 0)
    binding.mom_debug_force_gemm_form(256, 5, 256)
    r = _run(*t)
    binding.mom_debug_force_gemm_form(0, 0, 0)
    return r


@pytest.mark.parametrize("tm,tn", FORMS)
def test_form_gives_the_bits_of_the_full_tiles(tm, tn, short_form):
    # rows around one and two token tiles and over two and three groups of four of them; K = 32 (nothing but a final
    # stage) ... several turns of the ring, with final stages of 32 ... 224 elements; columns that end inside a tile
    for S, H, I in ((1, 64, 32), (tm - 1 or 1, 32, 96), (tm, 160, 224), (tm + 1, 288, 352), (2 * tm + 5, 1056, 480),
                    (2 * tm - 3, 736, 2080), (4 * tm + 1, 160, 288), (4 * tm + tm // 2 + 3, 352, 416), (9 * tm + 7, 96, 160)):
        t = _inputs(S, H, I, S + H, 0.05)
        ref = _full_tiles(*t)
        short_form(tm, tn)
        got = _run(*t)
        torch.cuda.synchronize()
        assert torch.equal(got[1], ref[1]), f"intermediate S={S} H={H} I={I}"
        assert torch.equal(got[0], ref[0]), f"out S={S} H={H} I={I}"


@pytest.fixture(scope="module")
def large_layer():
    """Weights of 336 MiB, which a launch of few token tiles reads past the Infinity Cache."""
    wl = synth.Workload("large", S=1024, H=8192, I=7168, mini_seq=0, seed=7, w_std=0.02)
    return synth.mlp_inputs(wl, device="cuda")


@pytest.mark.parametrize("tm,tn", _SHAPES["GATEUP"])
def test_gate_up_form_with_non_temporal_weights(tm, tn, large_layer, short_form):
    # a call of one mini-sequence: at most two token tiles; of several: four, the last mini-sequence shorter
    x, *w = large_layer
    for S, mini_seq in ((1, 0), (tm + 5, 0), (min(4 * tm + 9, 1024), min(4 * tm - 3, 600))):
        t = (x[:S].contiguous(), *w)
        ref = _full_tiles(*t)
        short_form(tm, tn)
        got = _run(*t, mini_seq)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]), f"out S={S} mini_seq={mini_seq}"
        if not mini_seq:
            assert torch.equal(got[1], ref[1]), f"intermediate S={S}"


@pytest.mark.parametrize("H,I", [(96, 466080), (224, 199808), (352, 127136), (736, 60832), (1120, 40000), (4128, 10880)])
def test_non_temporal_weights_at_every_end_of_a_group_of_stages(H, I, short_form):
    # rows shorter than the ring, and ends in the first and in the second stage of a group, whole and shorter; weights of 256 MiB and more
    assert 6 * H * I > 256 << 20
    x, *w = _inputs(140, H, I, H, 0.05)
    for S in (1, 61, 140):
        t = (x[:S].contiguous(), *w)
        ref = _full_tiles(*t)
        for tm, tn in _SHAPES["GATEUP"]:
            if S > 2 * tm:
                continue                                        # three token tiles read plain weights
            short_form(tm, tn)
            got = _run(*t)
            torch.cuda.synchronize()
            assert torch.equal(got[1], ref[1]) and torch.equal(got[0], ref[0]), f"{tm}x{tn} S={S}"


def test_the_second_ring_of_the_64_row_gate_up_form(large_layer, short_form):
    # chosen at these sizes, with weights by non-temporal and by plain loads (tests/gemm_forms_check.cpp says so)
    x, wg, wu, wd = large_layer
    for S, I in ((33, 7168), (61, 7168), (100, 3584)):
        t = (x[:S].contiguous(), wg[:I].contiguous(), wu[:I].contiguous(), wd[:, :I].contiguous())
        ref = _full_tiles(*t)
        got = _run(*t)
        torch.cuda.synchronize()
        assert torch.equal(got[1], ref[1]) and torch.equal(got[0], ref[0]), f"S={S} I={I}"
        r = oracle.mlp_rows(*(synth.bits(a) for a in (t[0][:8], *t[1:])))
        g = got[0][:8].view(torch.bfloat16).float().cpu().numpy()
        assert abs(g - r).max() <= 2e-2 * abs(r).max()          # the bar of the parity tests


@pytest.mark.parametrize("name", ["llama3_8b_32k", "qwen25_7b_256k"])
def test_few_token_rows_at_production_contraction_lengths(name, short_form):
    wl = synth.WORKLOADS[name]
    x, wg, wu, wd = synth.mlp_inputs(wl, device="cuda", S=2048)
    for S in (1, 16, 17, 40, 61, 80, 128, 150, 192, 224, 256, 317, 512, 900, 1000, 1536, 1800, 2048):
        t = (x[:S].contiguous(), wg, wu, wd)
        ref = _full_tiles(*t)
        got = _run(*t)
        torch.cuda.synchronize()
        assert torch.equal(got[1], ref[1]) and torch.equal(got[0], ref[0]), f"S={S}"
        if S == 40:
            r = oracle.mlp_rows(*(synth.bits(a) for a in t))
            g = got[0].view(torch.bfloat16).float().cpu().numpy()
            assert abs(g - r).max() <= 2e-2 * abs(r).max()      # the bar of the parity tests


def test_forced_short_form_validation(short_form):
    L = binding.lib()
    for f in ((48, 16), (0, 64), (-16, 16), (256, 256)):
        assert L.mom_debug_force_short_form(*f) == binding.MOM_ERR_SHAPE
