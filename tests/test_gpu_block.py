"""Whole blocks of token rows in one launch, the intermediate in LDS: the bits of the tile kernels, row counts around whole blocks,
contractions with and without a half unit, fewer row groups than wavefronts and row groups that leave some wavefronts idle."""
import pytest
import torch

from paper_2504_12526_amd import binding, synth
from test_gpu_short_forms import _full_tiles, _inputs

pytestmark = pytest.mark.gpu


@pytest.fixture
def block():
    yield binding.mom_debug_force_block
    binding.mom_debug_force_block(0)


def _call(t, mini_seq):
    S, I = t[0].shape[0], t[1].shape[0]
    out = torch.full_like(t[0], float("nan"))
    ws = torch.full(((mini_seq or S) * I,), float("nan"), dtype=torch.bfloat16, device="cuda")
    binding.mom_mlp_prefill(*t, mini_seq, out, ws)
    torch.cuda.synchronize()
    return out.view(torch.int16), ws


@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("S,H,I", [(1, 32, 32), (15, 64, 96), (16, 96, 64), (17, 32, 480), (33, 160, 224), (65, 288, 352),
                                   (100, 480, 1184), (512, 256, 1024), (31, 1056, 1984), (40, 2016, 32)])
def test_block_gives_the_bits_of_the_full_tiles(S, H, I, rows, block):
    t = _inputs(S, H, I, S + H, 0.05)
    ref = _full_tiles(*t)[0]
    block(rows)
    got, ws = _call(t, 0)
    assert torch.equal(got, ref)
    # the workspace is not needed: it is as it was, unless the layer is too large for blocks of so many rows
    fits = 2 * rows * (H + I + 16) + 65536 <= 163840 or (rows == 16 and 32 * (H + I + 16) + 49152 <= 163840)
    assert bool(torch.isnan(ws).all()) == fits


@pytest.mark.parametrize("S,H,I,C", [(512, 256, 1024, 128), (4099, 256, 1024, 100), (8200, 256, 1024, 512), (2001, 1056, 2080, 100)])
def test_chosen_for_several_mini_sequences(S, H, I, C):
    t = _inputs(S, H, I, S + C, 0.05)
    got, ws = _call(t, C)
    assert bool(torch.isnan(ws).all())                 # blocks it is
    assert torch.equal(got, _call(t, 0)[0])
    events = [torch.cuda.Event(enable_timing=True) for _ in range(1 + 2 * (-(-S // C)))]
    for e in events:
        e.record()
    out = torch.full_like(t[0], float("nan"))
    binding.mom_mlp_prefill_events(*t, C, out, torch.empty(C * I * 2, dtype=torch.uint8, device="cuda"), events)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), got)     # kernel by kernel, as ever
