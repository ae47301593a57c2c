"""KV-cache reload by a kernel and by copies: the bytes, and none beside them, at the edges of the kernel's passes, of the sizes at
which the one or the other is taken and of its alignment; which of them is taken, captured and not; beside other work and errors."""
import ctypes

import pytest
import torch

from graph_nodes import KERNEL, MEMCPY, hip, node_types
from paper_2504_12526_amd import binding, synth

pytestmark = pytest.mark.gpu

PASS = 16 * 256 * 4 * 16          # bytes
LARGEST = 256 << 10               # bytes each of the kernel's range under stream capture (elsewhere 1 MiB, and any behind work)
GUARD = 64                         # elements on either side


def _reload(each, offset, seed):
    n = each // 2
    g = torch.Generator().manual_seed(seed)
    host = torch.randint(-32768, 32767, (2 * n + offset,), dtype=torch.int16, generator=g).pin_memory()
    bufs = [torch.full((n + 2 * GUARD + offset,), 77 + i, dtype=torch.int16, device="cuda") for i in range(2)]
    k, v = (b[GUARD + offset: GUARD + offset + n].view(torch.bfloat16) for b in bufs)
    src = host[offset:].view(torch.bfloat16)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    binding.mom_kv_reload(src, k, v, side)
    side.synchronize()
    for i, b in enumerate(bufs):
        got = b.cpu()
        lo = GUARD + offset
        assert torch.equal(got[lo: lo + n], host[offset + i * n: offset + (i + 1) * n])
        assert bool((got[:lo] == 77 + i).all()) and bool((got[lo + n:] == 77 + i).all())


@pytest.mark.parametrize("each", [16, 32, 4096, 8192 - 16, 8192, 8192 + 16, PASS // 2 - 16, PASS // 2, PASS // 2 + 16, PASS - 16,
                                  LARGEST - 16, LARGEST, LARGEST + 16, 4 * LARGEST])
def test_bytes(each):
    _reload(each, 0, each % 1000)


@pytest.mark.parametrize("each,offset", [(2, 0), (14, 0), (4098, 0), (4096, 1), (4096, 8), (65536, 3)])
def test_odd_sizes_and_alignments(each, offset):
    _reload(each, offset, each + offset)


# passes of the kernel's 48 wavefronts (64 threads, four loads of 16 bytes), K ending and V beginning inside one, and some MiB
WAVES_PASS = 48 * 64 * 4 * 16


@pytest.mark.parametrize("each", [WAVES_PASS // 2 - 16, WAVES_PASS // 2 + 16, WAVES_PASS - 16, WAVES_PASS, WAVES_PASS + 16, 5 * WAVES_PASS // 2 + 48,
                                  7 * WAVES_PASS - 1024, (4 << 20) - 16, (4 << 20) + 4112, 16 << 20])
def test_bytes_of_several_passes(each):
    _reload(each, 0, each % 999)


def test_a_large_reload_only_enqueues():
    """The calling thread is not held until the work ahead of the reload is done."""
    n = 2 << 20
    main, ahead = torch.cuda.current_stream(), torch.cuda.Event()
    t = synth.mlp_inputs(synth.Workload("ahead", S=8192, H=2048, I=8192, mini_seq=0, seed=4), device="cuda")
    out, ws = torch.empty_like(t[0]), torch.empty(8192 * 8192 * 2, dtype=torch.uint8, device="cuda")
    sides = [(torch.cuda.Stream(), torch.zeros(2 * n, dtype=torch.int16).pin_memory(), *(torch.zeros(n, dtype=torch.int16, device="cuda") for _ in range(2)))
             for _ in range(3)]
    torch.cuda.synchronize()                                    # (the zeros are there before another stream writes)

    def reload(side, host, k, v):
        binding.mom_kv_reload(host.view(torch.bfloat16), k.view(torch.bfloat16), v.view(torch.bfloat16), side)

    for s in sides:                                             # (the first reload maps the pages)
        reload(*s)
    torch.cuda.synchronize()
    for i, (_, host, _, _) in enumerate(sides):                 # other bytes than those that are there now
        host.copy_(torch.randint(-32768, 32767, (2 * n,), dtype=torch.int16, generator=torch.Generator().manual_seed(i)))
    for _ in range(24):                                         # some 15 ms
        binding.mom_mlp_prefill(*t, 0, out, ws, stream=main)
    ahead.record(main)
    for s in sides:
        s[0].wait_event(ahead)
        reload(*s)
    assert not ahead.query()
    torch.cuda.synchronize()
    for _, host, k, v in sides:
        assert bool((host != 0).any()) and torch.equal(k.cpu(), host[:n]) and torch.equal(v.cpu(), host[n:])


def _some_work():
    """call(): some milliseconds on the current stream."""
    t = synth.mlp_inputs(synth.Workload("ahead", S=8192, H=2048, I=8192, mini_seq=0, seed=4), device="cuda")
    out, ws = torch.empty_like(t[0]), torch.empty(8192 * 8192 * 2, dtype=torch.uint8, device="cuda")
    return lambda: [binding.mom_mlp_prefill(*t, 0, out, ws) for _ in range(6)]


def _buffers(each):
    host = torch.randint(-32768, 32767, (each,), dtype=torch.int16).pin_memory().view(torch.bfloat16)
    k, v = (torch.zeros(each // 2, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    return host, k, v


def _assert_bytes(host, k, v):
    torch.cuda.synchronize()
    assert torch.equal(torch.cat([k, v]).view(torch.int16).cpu(), host.view(torch.int16))


def test_what_an_eager_reload_takes():
    """The kernel up to 1 MiB each and behind work that is still to be done; copies, which take nothing from the kernels beside them, on a
    stream that is ready."""
    from torch.profiler import ProfilerActivity, profile
    work, side = _some_work(), torch.cuda.Stream()
    cases = [(each, behind) for each in (16, 1 << 20, (1 << 20) + 16, 16 << 20) for behind in (False, True)]
    buffers = {each: _buffers(each) for each, _ in cases}
    taken = []
    for each, behind in cases:
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            if behind:
                work()
                side.wait_stream(torch.cuda.current_stream())
            binding.mom_kv_reload(*buffers[each], side)
            torch.cuda.synchronize()
        names = [e.name for e in p.events()]
        taken.append((any("kv_reload_kernel" in n for n in names), any("Memcpy HtoD" in n for n in names)))
        _assert_bytes(*buffers[each])
    for (each, behind), (kernel, copies) in zip(cases, taken):
        assert (kernel, copies) == ((True, False) if each <= 1 << 20 or behind else (False, True)), f"{each} bytes each, behind work: {behind}"


@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("each", [4096, 512 << 10, 4 << 20])
def test_a_capture_on_another_stream_goes_on(each, behind):
    runtime, vp = hip(), ctypes.c_void_p
    work, side, captured = _some_work(), torch.cuda.Stream(), torch.cuda.Stream()
    buffers, graph, mode = _buffers(each), vp(), ctypes.c_int(-1)
    if behind:
        work()
        side.wait_stream(torch.cuda.current_stream())
    assert runtime.hipStreamBeginCapture(vp(captured.cuda_stream), 0) == 0           # global: no call that it forbids, on any stream
    rc = binding.mom_kv_reload(*buffers, side, check=False)
    end = runtime.hipStreamEndCapture(vp(captured.cuda_stream), ctypes.byref(graph))
    assert (rc, end) == (binding.MOM_OK, 0)
    assert runtime.hipGraphDestroy(graph) == 0
    mode.value = 2
    assert runtime.hipThreadExchangeStreamCaptureMode(ctypes.byref(mode)) == 0
    was, back = mode.value, ctypes.c_int(mode.value)
    assert runtime.hipThreadExchangeStreamCaptureMode(ctypes.byref(back)) == 0 and was == 0       # the thread's mode is what it was
    _assert_bytes(*buffers)


def test_an_error_of_the_program_stays_behind_work():
    runtime, work, side = hip(), _some_work(), torch.cuda.Stream()
    buffers = _buffers(4 << 20)
    work()
    side.wait_stream(torch.cuda.current_stream())
    error = runtime.hipSetDevice(12345)
    assert error != 0 and runtime.hipPeekAtLastError() == error
    rc = binding.mom_kv_reload(*buffers, side, check=False)
    left = runtime.hipGetLastError()
    assert rc == binding.MOM_OK and left == error
    _assert_bytes(*buffers)


def test_overlapping_buffers_are_copied_one_after_the_other():
    host = torch.randint(-32768, 32767, (2 * 4096,), dtype=torch.int16).pin_memory()
    buf = torch.zeros(4096 + 64, dtype=torch.int16, device="cuda")
    binding.mom_kv_reload(host.view(torch.bfloat16), buf[:4096].view(torch.bfloat16), buf[64:].view(torch.bfloat16), torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(buf.cpu(), torch.cat([host[:64], host[4096:]]))


def test_captured():
    n = 40000
    host = torch.zeros(2 * n, dtype=torch.int16).pin_memory()
    k, v = (torch.zeros(n, dtype=torch.int16, device="cuda") for _ in range(2))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        binding.mom_kv_reload(host.view(torch.bfloat16), k.view(torch.bfloat16), v.view(torch.bfloat16), side)
    for r in range(4):
        host.copy_(torch.arange(2 * n).add_(r * 7919).to(torch.int16))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(k.cpu(), host[:n]) and torch.equal(v.cpu(), host[n:])
        k.zero_()
        v.zero_()


@pytest.mark.parametrize("each,offset,kernel", [(16, 0, True), (4096, 8, True), (LARGEST, 0, True), (LARGEST + 16, 0, False),
                                                (4098, 0, False), (4096, 1, False)])
def test_which_of_them_a_reload_takes(each, offset, kernel):
    n = each // 2
    host = torch.zeros(2 * n + offset, dtype=torch.int16).pin_memory()[offset:].view(torch.bfloat16)
    k, v = (torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    assert node_types(lambda stream: binding.mom_kv_reload(host, k, v, stream)) == ([KERNEL] if kernel else [MEMCPY, MEMCPY])


def test_buffers_that_end_before_the_bytes_do_are_refused():
    """... also where another allocation follows: its bytes stay."""
    runtime, each = hip(), 65536
    host = torch.zeros(each * 4, dtype=torch.uint8).pin_memory()
    pointers = [ctypes.c_void_p() for _ in range(64)]
    for p in pointers:
        assert runtime.hipMalloc(ctypes.byref(p), ctypes.c_size_t(each)) == 0
    try:
        at = sorted(p.value for p in pointers)
        a, b = next((a, b) for a, b in zip(at, at[1:]) if b == a + each)          # nothing lies between the two
        for p in (a, b):
            assert runtime.hipMemset(ctypes.c_void_p(p), 0x33, ctypes.c_size_t(each)) == 0
        other = torch.empty(2 * each, dtype=torch.uint8, device="cuda")
        for k, v in ((a, other.data_ptr()), (other.data_ptr(), a)):
            rc = binding.lib().mom_kv_reload(ctypes.c_void_p(host.data_ptr()), ctypes.c_void_p(k), ctypes.c_void_p(v),
                                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), 2 * each, None)
            runtime.hipGetLastError()
            torch.cuda.synchronize()
            assert rc == binding.MOM_ERR_HIP
        got = torch.empty(each, dtype=torch.uint8)
        assert runtime.hipMemcpy(ctypes.c_void_p(got.data_ptr()), ctypes.c_void_p(b), ctypes.c_size_t(each), 2) == 0
        assert bool((got == 0x33).all())
    finally:
        for p in pointers:
            assert runtime.hipFree(p) == 0


@pytest.mark.parametrize("flags", [0, 0x40000000, 0x80000000])          # default, coherent, non-coherent
def test_host_memory_written_between_reloads(flags):
    runtime, n, p = hip(), 32768, ctypes.c_void_p()
    assert runtime.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(2 * n), ctypes.c_uint(flags)) == 0
    try:
        k, v = (torch.empty(n, dtype=torch.uint8, device="cuda") for _ in range(2))
        for r in range(6):
            ctypes.memset(p.value, 17 * r + 1, 2 * n)
            assert binding.lib().mom_kv_reload(p, ctypes.c_void_p(k.data_ptr()), ctypes.c_void_p(v.data_ptr()),
                                               ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), n, None) == binding.MOM_OK
            assert bool((k == 17 * r + 1).all()) and bool((v == 17 * r + 1).all())
        torch.cuda.synchronize()
    finally:
        assert runtime.hipHostFree(p) == 0
