"""mom_mlp_prefill_static and mom_mlp_prefill_pipelined take more rows at a time than mini_seq: the bits of mom_mlp_prefill, and
nothing written behind the workspace that the call asks for."""
import pytest
import torch

from paper_2504_12526_amd import binding, synth

pytestmark = pytest.mark.gpu


def _case(S, H, I, seed):
    t = synth.mlp_inputs(synth.Workload("passes", S=S, H=H, I=I, mini_seq=0, seed=seed, w_std=0.05), device="cuda")
    ref = torch.full_like(t[0], float("nan"))
    ws = torch.empty(binding.mom_mlp_workspace_bytes(S, H, I, 0), dtype=torch.uint8, device="cuda")
    binding.mom_mlp_prefill(*t, 0, ref, ws)
    return t, ref.view(torch.int16)


# one pass, two with a last one of a single row, of both halves, several; a mini-sequence of 14 rounds and more stays one
@pytest.mark.parametrize("S,H,I,C", [(101, 64, 96, 100), (200, 96, 224, 100), (201, 64, 160, 100), (777, 160, 352, 150),
                                     (5, 32, 32, 1), (9000, 64, 16384, 7200)])
def test_pipelined(S, H, I, C):
    t, ref = _case(S, H, I, S + C)
    need = binding.mom_mlp_pipelined_workspace_bytes(S, H, I, C)
    ws = torch.full((need + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    out = torch.full_like(t[0], float("nan"))
    side, events = torch.cuda.Stream(), [torch.cuda.Event() for _ in range(5)]
    for e in events:
        e.record()
    binding.mom_mlp_prefill_pipelined(*t, C, out, ws[:need], torch.cuda.current_stream(), side, events)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref)
    assert bool((ws[need:] == 0x5a).all())


# the array holds 1024 rows at I = 32768: one pass, whole passes and a short one, mini_seq kept where the gain is too small
@pytest.mark.parametrize("S,C", [(1024, 100), (1025, 1), (2500, 500), (2500, 700), (1500, 1024)])
def test_static(S, C):
    t, ref = _case(S, 64, 32768, S + C)
    out = torch.full_like(t[0], float("nan"))
    binding.mom_mlp_prefill_static(*t, C, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref)
