"""An error of the HIP runtime that the program has left behind is neither taken for an error of a call nor taken away by it: the
runtime keeps it through calls that succeed."""
import pytest
import torch

from graph_nodes import hip as _runtime
from paper_2504_12526_amd import binding, synth

pytestmark = pytest.mark.gpu


def _recorded(**kw):
    e = torch.cuda.Event(**kw)
    e.record()
    return e


@pytest.fixture(scope="module")
def hip():
    return _runtime()


@pytest.fixture(scope="module")
def calls():
    """name -> (call, the tensors it writes, event it records)"""
    wl = synth.Workload("errors", S=300, H=256, I=1024, mini_seq=100, w_std=0.05)
    t = synth.mlp_inputs(wl, device="cuda")
    large = synth.mlp_inputs(synth.Workload("errors", S=300, H=4096, I=6144, mini_seq=0), device="cuda")     # rectangular tiles
    ws = torch.empty(300 * 6144 * 2, dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    events = [_recorded() for _ in range(5)]
    made = {}

    def mlp(name, of, run):
        out = torch.empty_like(of[0])
        made[name] = (lambda: run(of, out), [out], None)

    mlp("prefill", t, lambda t, out: binding.mom_mlp_prefill(*t, 0, out, ws, check=False))
    mlp("prefill in blocks", t, lambda t, out: binding.mom_mlp_prefill(*t, 100, out, ws, check=False))
    mlp("prefill of a large layer", large, lambda t, out: binding.mom_mlp_prefill(*t, 0, out, ws, check=False))
    mlp("static", t, lambda t, out: binding.mom_mlp_prefill_static(*t, 100, out, check=False))
    mlp("pipelined", t, lambda t, out: binding.mom_mlp_prefill_pipelined(*t, 100, out, ws, torch.cuda.current_stream(), side, events, check=False))
    last, x = torch.empty(256, dtype=torch.bfloat16, device="cuda"), t[0][-1].clone()
    made["last"] = (lambda: binding.mom_mlp_last(x, *t[1:], last, ws, check=False), [last], None)
    logits = torch.empty(1024, dtype=torch.float32, device="cuda")
    made["head"] = (lambda: binding.mom_lmhead_last(x, t[1], logits, check=False), [logits], None)
    for name, n in (("reload by a kernel", 4096), ("reload by copies", 4095), ("large reload", 1 << 20)):
        host = torch.randint(-32768, 32767, (2 * n,), dtype=torch.int16).pin_memory().view(torch.bfloat16)
        k, v = (torch.empty(n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        done = _recorded(enable_timing=True)
        made[name] = (lambda host=host, k=k, v=v, done=done: binding.mom_kv_reload(host, k, v, side, done, check=False), [k, v], done)
    return made


@pytest.mark.parametrize("name", ["prefill", "prefill in blocks", "prefill of a large layer", "static", "pipelined", "last", "head",
                                  "reload by a kernel", "reload by copies", "large reload"])
def test_call_after_an_error_of_the_program(name, hip, calls):
    call, outs, done = calls[name]
    binding.mom_init()
    assert call() == binding.MOM_OK
    torch.cuda.synchronize()
    want = [o.clone() for o in outs]
    for o in outs:
        o.zero_()
    torch.cuda.synchronize()
    before = _recorded(enable_timing=True)
    torch.cuda.synchronize()
    error = hip.hipSetDevice(12345)                     # refused on the host: no such device
    assert error != 0 and hip.hipPeekAtLastError() == error
    rc = call()
    left = hip.hipGetLastError()
    torch.cuda.synchronize()
    assert rc == binding.MOM_OK
    assert left == error
    assert all(torch.equal(o.view(torch.int16), w.view(torch.int16)) for o, w in zip(outs, want))
    assert done is None or before.elapsed_time(done) > 0      # recorded by this call
