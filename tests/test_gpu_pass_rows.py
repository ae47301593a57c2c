"""mom_mlp_prefill_static and mom_mlp_prefill_pipelined take more rows at a time than mini_seq: as many passes as their rules say
(two kernels each, by the nodes of the graph a call is captured into), the bits of mom_mlp_prefill, the rows of the workspace that are
theirs and nothing behind it."""
import pytest
import torch

from graph_nodes import KERNEL, node_types
from paper_2504_12526_amd import binding, synth

pytestmark = pytest.mark.gpu

FILL = 0x5a5a


def _case(S, H, I, seed):
    t = synth.mlp_inputs(synth.Workload("passes", S=S, H=H, I=I, mini_seq=0, seed=seed, w_std=0.05), device="cuda")
    ref = torch.full_like(t[0], float("nan"))
    ws = torch.empty(binding.mom_mlp_workspace_bytes(S, H, I, 0), dtype=torch.uint8, device="cuda")
    binding.mom_mlp_prefill(*t, 0, ref, ws)
    return t, ref.view(torch.int16)


# layers too large for blocks of rows (H + I > 8192).  Both halves at once: one pass, two with a last one of a single row, of both
# halves, several; three of 512 rows instead of two of 600 and one of 150; a mini-sequence of 14 rounds and more stays one.
@pytest.mark.parametrize("S,H,I,C,rows", [(101, 64, 8192, 100, 101), (200, 96, 8224, 100, 200), (201, 64, 8192, 100, 200),
                                          (777, 160, 8352, 150, 300), (1000, 32, 8192, 100, 200), (5, 32, 8192, 1, 2),
                                          (1350, 4096, 14336, 300, 512), (9000, 64, 16384, 7200, 7200)])
def test_pipelined(S, H, I, C, rows):
    t, ref = _case(S, H, I, S + C)
    need = binding.mom_mlp_pipelined_workspace_bytes(S, H, I, C)
    ws = torch.full((need // 2 + 2048,), FILL, dtype=torch.int16, device="cuda")
    out = torch.full_like(t[0], float("nan"))
    side, events = torch.cuda.Stream(), [torch.cuda.Event() for _ in range(5)]
    for e in events:
        e.record()

    def call(stream):
        binding.mom_mlp_prefill_pipelined(*t, C, out, ws[:need // 2], stream, side, events)

    assert node_types(call) == [KERNEL] * (2 * -(-S // rows))
    call(torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref)
    assert not bool((ws.view(-1)[(rows - 1) * I: rows * I] == FILL).all())         # the last row of a pass
    assert bool((ws[rows * I:] == FILL).all())


# the array holds 1024 rows at I = 32768: one pass, whole passes and a short one, mini_seq kept where the gain is too small
@pytest.mark.parametrize("S,C,passes", [(1024, 100, 1), (1025, 1, 2), (2500, 500, 3), (2500, 700, 4), (1500, 1024, 2)])
def test_static(S, C, passes):
    t, ref = _case(S, 64, 32768, S + C)
    out = torch.full_like(t[0], float("nan"))
    binding.mom_init()
    assert node_types(lambda stream: binding.mom_mlp_prefill_static(*t, C, out, stream=stream)) == [KERNEL] * (2 * passes)
    binding.mom_mlp_prefill_static(*t, C, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref)
