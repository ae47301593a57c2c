"""Passes of more rows than the workspace holds, the rest of their intermediate in the rows of `out` that are still to come: the rules on
the host (tests/longer_passes_check.cpp), the bits and what is written on the GPU."""
import os
import subprocess

import pytest
import torch

from paper_2504_12526_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12526_amd", "csrc")
GUARD = 4096


def _check(tmp_path, include_dir):
    exe = os.path.join(str(tmp_path), "longer_passes_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", include_dir, "-o", exe,
                    os.path.join(ROOT, "tests", "longer_passes_check.cpp")], check=True)
    return subprocess.run([exe], capture_output=True, text=True)


def test_rows_and_places(tmp_path):
    r = _check(tmp_path, CSRC)
    assert r.returncode == 0 and ": ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("old,new,says", [
    ("return C / down.tm * down.tm;", "return C;", "split"),                                    # a token tile of the down launch in both pieces
    ("- kSpareAlign / 2) / (H + I)", ") / (H + I)", "rows "),                                   # no room for the alignment
    ("if (t < least && rows <= most_rows(left, H, I, p.split))", "if (t < least)", "rows "),      # room counted for more rows in the workspace
    ("if (t + 0.9 * p.time()", "if (t + 3.0 * p.time()", "in blocks"),                           # longer passes given up too early
])
def test_a_planted_mistake_is_caught(tmp_path, old, new, says):
    text = open(os.path.join(CSRC, "mom_gemm_forms.h")).read()
    assert text.count(old) == 1, old
    with open(os.path.join(str(tmp_path), "mom_gemm_forms.h"), "w") as f:
        f.write(text.replace(old, new))
    r = _check(tmp_path, str(tmp_path))
    assert r.returncode == 1 and "FAILED" in r.stdout and says in r.stdout, r.stdout + r.stderr


def _case(S, H, I, C, offset=0):
    """Inputs, the result of one pass, and guarded buffers for out (offset elements further) and workspace."""
    t = synth.mlp_inputs(synth.Workload("longer", S=S, H=H, I=I, mini_seq=0, seed=S + C, w_std=0.03), device="cuda")
    ref = torch.full_like(t[0], float("nan"))
    binding.mom_mlp_prefill(*t, 0, ref, torch.empty(S * I * 2, dtype=torch.uint8, device="cuda"))
    whole = torch.full((S * H + 2 * GUARD + offset,), 0x5a5a, dtype=torch.int16, device="cuda")
    out = whole[GUARD + offset: GUARD + offset + S * H].view(torch.bfloat16).view(S, H)
    ws = torch.full((C * I + GUARD,), 0x5a5a, dtype=torch.int16, device="cuda")
    return t, ref.view(torch.int16), whole, out, ws


def _assert_result(ref, whole, out, ws, used, what):
    torch.cuda.synchronize()
    lo = (out.data_ptr() - whole.data_ptr()) // 2
    assert torch.equal(out.view(torch.int16), ref), what
    assert bool((whole[:lo] == 0x5a5a).all()) and bool((whole[lo + out.numel():] == 0x5a5a).all()), what
    assert bool((ws[used:] == 0x5a5a).all()), what


# rows in the workspace: none (C below a token tile), some, most; a last pass of one row and of a whole mini-sequence; gate/up of two widths and in
# rectangular tiles; an odd contraction; out at 16 bytes past a 256-byte line
@pytest.mark.gpu
@pytest.mark.parametrize("S,H,I,C,offset", [(4101, 1056, 2080, 256, 0), (2048, 1056, 2080, 300, 8), (3001, 2048, 8192, 100, 0), (6216, 2048, 5632, 777, 72),
                                            (2600, 4096, 14336, 128, 8), (4096, 4096, 14336, 512, 0), (4101, 3584, 18944, 256, 8), (5000, 3584, 9728, 512, 120),
                                            (9005, 1024, 4096, 1500, 0)])
def test_bits_and_what_is_written(S, H, I, C, offset):
    from graph_nodes import KERNEL, node_types
    t, ref, whole, out, ws = _case(S, H, I, C, offset)
    binding.mom_mlp_prefill(*t, C, out, ws[:C * I])
    _assert_result(ref, whole, out, ws, C * I, "plain")
    out.view(torch.int16).fill_(0x5a5a)
    nodes = node_types(lambda stream: binding.mom_mlp_prefill(*t, C, out, ws[:C * I], stream=stream))
    assert set(nodes) == {KERNEL} and len(nodes) % 2 == 0 and len(nodes) < 2 * -(-S // C)          # longer passes it is
    events = [torch.cuda.Event(enable_timing=True) for _ in range(1 + 2 * -(-S // C))]
    for e in events:
        e.record()
    binding.mom_mlp_prefill_events(*t, C, out, ws[:C * I], events)                                # one at a time
    _assert_result(ref, whole, out, ws, C * I, "events")


@pytest.mark.gpu
@pytest.mark.parametrize("S,H,I,C", [(3001, 1056, 2080, 512), (12000, 1056, 2080, 256), (3000, 2048, 8192, 256)])
def test_out_in_host_memory_holds_results_only(S, H, I, C):
    """... which would go through the link for every column tile: as many launches as mini-sequences take."""
    from graph_nodes import KERNEL, node_types
    t, ref, _, device_out, ws = _case(S, H, I, C)
    out = torch.zeros((S, H), dtype=torch.bfloat16, pin_memory=True)

    def nodes(out):
        return node_types(lambda stream: binding.mom_mlp_prefill(*t, C, out, ws[:C * I], stream=stream))

    assert len(nodes(device_out)) < 2 * -(-S // C)                 # where it is the device's, longer passes or blocks
    blocks = nodes(out) == [KERNEL]                                # (these hold nothing there either)
    assert blocks or nodes(out) == [KERNEL] * (2 * -(-S // C))
    binding.mom_mlp_prefill(*t, C, out, ws[:C * I])
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref.cpu())


@pytest.mark.gpu
@pytest.mark.parametrize("form", [("gemm", 256, 5, 224), ("gemm", 256, 5, 160), ("gemm", 128, 0, 0), ("rect", 192, 256), ("rect", 160, 160), ("rect", 224, 160),
                                  ("short", 96, 64), ("short", 160, 128), ("short", 48, 32), ("short", 80, 64)])
def test_pieces_in_every_kind_of_tile(form):
    # workspaces of 400 rows, of which 256, 256, (down not forced), 384, 320, 224, 384, 320, 384 and 400 are whole tiles of the down launch, and of 130,
    # none or 96, 96 and 80
    from graph_nodes import node_types
    S, H, I = 4500, 1056, 2080
    t, ref, whole, out, ws = _case(S, H, I, 400, 8)
    force = {"gemm": binding.mom_debug_force_gemm_form, "rect": binding.mom_debug_force_rect_form, "short": binding.mom_debug_force_short_form}[form[0]]
    try:
        force(*form[1:])
        for c in (400, 130):
            out.view(torch.int16).fill_(0x5a5a)
            ws.fill_(0x5a5a)

            def call(stream):
                binding.mom_mlp_prefill(*t, c, out, ws[:c * I], stream=stream)

            assert len(node_types(call)) < 2 * -(-S // c), f"{form} C={c}: no longer pass"
            call(torch.cuda.current_stream())
            _assert_result(ref, whole, out, ws, c * I, f"{form} C={c}")
    finally:
        force(*([0] * len(form[1:])))


@pytest.mark.gpu
def test_two_streams():
    from graph_nodes import node_types
    S, H, I, C = 5000, 1056, 2080, 300
    t, ref, whole, out, ws = _case(S, H, I, 2 * C, 8)
    side, events = torch.cuda.Stream(), [torch.cuda.Event() for _ in range(5)]
    for e in events:
        e.record()

    def call(stream):
        binding.mom_mlp_prefill_pipelined(*t, C, out, ws[:2 * C * I], stream, side, events)

    assert len(node_types(call)) < 2 * -(-S // (2 * C))                    # fewer than two mini-sequences at a time take
    call(torch.cuda.current_stream())
    _assert_result(ref, whole, out, ws, 2 * C * I, "pipelined")


@pytest.mark.gpu
@pytest.mark.parametrize("S,H,I,C", [(4797, 4096, 14336, 2340), (8169, 4096, 14336, 2340)])
def test_static(S, H, I, C):
    from graph_nodes import node_types
    t, ref, whole, out, _ = _case(S, H, I, 1, 8)
    binding.mom_init()

    def call(stream):
        binding.mom_mlp_prefill_static(*t, C, out, stream=stream)

    fit = binding.MOM_STATIC_WORKSPACE_BYTES // (2 * I)
    assert 2 < len(node_types(call)) < 2 * -(-S // fit)                    # fewer than the array's rows at a time take
    call(torch.cuda.current_stream())
    torch.cuda.synchronize()
    lo = (out.data_ptr() - whole.data_ptr()) // 2
    assert torch.equal(out.view(torch.int16), ref)
    assert bool((whole[:lo] == 0x5a5a).all()) and bool((whole[lo + out.numel():] == 0x5a5a).all())


@pytest.mark.gpu
def test_captured():
    S, H, I, C = 5000, 1056, 2080, 300
    t, ref, whole, out, ws = _case(S, H, I, C, 8)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.mom_mlp_prefill(*t, C, out, ws[:C * I])
    for r in range(3):
        t[0].mul_(-0.5)
        binding.mom_mlp_prefill(*t, 0, (want := torch.empty_like(out)), torch.empty(S * I * 2, dtype=torch.uint8, device="cuda"))
        out.view(torch.int16).fill_(0x5a5a)
        ws.fill_(0x5a5a)
        torch.cuda.synchronize()
        graph.replay()
        _assert_result(want.view(torch.int16), whole, out, ws, C * I, f"replay {r}")
