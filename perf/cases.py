"""The work that programs have this library do, as measurable cases.

A case is one call (or the few calls that belong together) through the public entry points of
`paper_2504_12526_amd.binding`, on the layer shapes of the model families the library is benchmarked on:

    llama   H = 4096, I = 14336, V = 128256      (Llama-3-8B-shaped; the Mistral-7B-shaped layer is the same)
    qwen    H = 3584, I = 18944, V = 152064      (Qwen2.5-7B-shaped)
    tiny    H = 256,  I = 1024,  V = 4096        (the small correctness workload)
    odd     H = 1056, I = 2080,  V = 32001       (multiples of 32 but not of 64, a ragged vocabulary)

Kinds:
    prefill    one MLP layer over S tokens in mini-sequences of `mini_seq` rows; `entry` says through which of
               the three drivers: "plain" (the caller's workspace), "static" (the library's own workspace) or
               "two_stream" (double-buffered on two streams)
    last       the last-token branch: one-token MLP, then the LM head
    offload    one layer of a prefill: K and V to pinned host memory on a side stream under the MLP
    reload     the step before decoding: K and V back to the device on a side stream beside the one-token MLP
"""
import torch

from paper_2504_12526_amd import binding, synth

LAYERS = {"llama": (4096, 14336, 128256), "qwen": (3584, 18944, 152064), "tiny": (256, 1024, 4096),
          "odd": (1056, 2080, 32001)}
KV_HEADS, HEAD_DIM = 8, 128


def _prefill(name, layer, S, mini_seq, entry="plain"):
    return {"name": name, "kind": "prefill", "layer": layer, "S": S, "mini_seq": mini_seq, "entry": entry}


def listed():
    return [
        # the small correctness workload: eight launches of a few workgroups each, all latency
        _prefill("tiny_512", "tiny", 512, 128),
        # one short chat turn: few rows against all the weights
        _prefill("turn_61", "llama", 61, 0),
        # a short prompt, odd length, through the entry point that brings its own workspace
        _prefill("prompt_317_static", "qwen", 317, 2048, "static"),
        # an ordinary prompt, shorter than one mini-sequence
        _prefill("prompt_1000", "llama", 1000, 4096),
        # chunked prefill at the chunk size the paper compares against
        _prefill("chunk_512", "llama", 8192, 512),
        # small mini-sequences on two streams
        _prefill("two_stream_1024", "llama", 16384, 1024, "two_stream"),
        # the headline configuration
        _prefill("llama_32k", "llama", 32768, 4096),
        # a long prompt whose length divides into nothing: mini-sequences of 8192, 8192 and 3627 rows
        _prefill("qwen_20011", "qwen", 20011, 8192),
        # a long context, the largest call
        _prefill("llama_128k", "llama", 131072, 8192),
        # the last token of a prefill (and every decoded one): each weight read once
        {"name": "last_token_llama", "kind": "last", "layer": "llama"},
        # one layer of a prefill with its KV cache leaving for host memory meanwhile
        {"name": "offload_16k", "kind": "offload", "layer": "llama", "S": 16384, "mini_seq": 4096},
        # the cache of one layer coming back before decoding
        {"name": "reload_8k", "kind": "reload", "layer": "llama", "S": 8192},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["prefill"] * 6 + ["last"] * 2 + ["offload", "reload"])
    if kind == "last":
        # any vocabulary: padded, sharded over devices, odd
        return {"kind": "last", "layer": rng.choice(["llama", "qwen", "tiny", "odd"]), "V": _log_int(rng, 1001, 152064)}
    if kind == "reload":
        return {"kind": "reload", "layer": rng.choice(["llama", "llama", "odd"]), "S": _log_int(rng, 16, 32768)}
    layer = rng.choice(["llama", "llama", "qwen", "qwen", "tiny", "odd"])
    if kind == "offload":
        return {"kind": "offload", "layer": layer, "S": _log_int(rng, 256, 32768), "mini_seq": rng.choice([1024, 2048, 4096, 8192])}
    mini_seq = rng.choice([0, 128, 256, 512, 1024, 2048, 4096, 8192, 16384, _log_int(rng, 100, 16384)])
    # at most 64 mini-sequences of small calls, and never more than the largest listed call
    most = 16384 if mini_seq == 0 else min(64 * mini_seq, 100000)
    S = _log_int(rng, 1, most)
    entry = rng.choice(["plain", "plain", "static", "two_stream"])
    if entry == "static":
        rows = binding.MOM_STATIC_WORKSPACE_BYTES // (2 * LAYERS[layer][1])
        mini_seq = min(mini_seq, rows) if mini_seq else 0
        if mini_seq == 0:
            S = min(S, rows)
    return {"kind": "prefill", "layer": layer, "S": S, "mini_seq": mini_seq, "entry": entry}


def _shape(case):
    H, I, V = LAYERS[case["layer"]]
    return H, I, case.get("V", V)


def _inputs(case, seed):
    """The tensors of the path's inputs, by name (device tensors; unit-RMS activations, weights of the usual spread)."""
    H, I, V = _shape(case)
    kind, dev = case["kind"], "cuda"
    t = {"W_gate": synth.normal_bf16("W_gate", (I, H), seed, 0.02, dev),
         "W_up": synth.normal_bf16("W_up", (I, H), seed, 0.02, dev),
         "W_down": synth.normal_bf16("W_down", (H, I), seed, 0.02, dev)}
    if kind in ("last", "reload"):
        t["x_last"] = synth.normal_bf16("x_last", (H,), seed, 1.0, dev)
    else:
        t["x"] = synth.normal_bf16("x", (case["S"], H), seed, 1.0, dev, rms_norm_rows=True)
    if kind == "last":
        t["W_lm"] = synth.normal_bf16("W_lm", (V, H), seed, 0.02, dev)
    if kind in ("offload", "reload"):
        for n in ("k", "v"):
            t[n] = synth.normal_bf16(n, (case["S"], KV_HEADS, HEAD_DIM), seed, 1.0, dev)
    return t


def _event():
    e = torch.cuda.Event()
    e.record()                       # the handle exists from the first record on
    return e


def prepare(case, seed):
    H, I, V = _shape(case)
    kind = case["kind"]
    binding.mom_init()
    st = _inputs(case, seed)
    st["case"] = case
    if kind in ("last", "reload"):
        st["out"] = torch.empty(H, dtype=torch.bfloat16, device="cuda")
        st["ws"] = torch.empty(I * 2, dtype=torch.uint8, device="cuda")
        if kind == "last":
            st["logits"] = torch.empty(V, dtype=torch.float32, device="cuda")
    else:
        S, C, entry = case["S"], case["mini_seq"], case.get("entry", "plain")
        st["out"] = torch.empty((S, H), dtype=torch.bfloat16, device="cuda")
        if entry == "two_stream":
            st["ws"] = torch.empty(binding.mom_mlp_pipelined_workspace_bytes(S, H, I, C), dtype=torch.uint8, device="cuda")
            st["side"] = torch.cuda.Stream()
            st["events"] = [_event() for _ in range(5)]
        elif entry == "plain":
            st["ws"] = torch.empty(binding.mom_mlp_workspace_bytes(S, H, I, C), dtype=torch.uint8, device="cuda")
    if kind in ("offload", "reload"):
        st["side"] = torch.cuda.Stream()
        st["order"], st["done"] = _event(), _event()
        n = st["k"].numel()
        st["host"] = torch.empty(2 * n, dtype=torch.bfloat16, pin_memory=True)
        if kind == "reload":
            st["host"][:n].copy_(st["k"].view(-1))
            st["host"][n:].copy_(st["v"].view(-1))
            st["k"], st["v"] = torch.empty_like(st["k"]), torch.empty_like(st["v"])
    torch.cuda.synchronize()
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    main = torch.cuda.current_stream()
    if kind == "prefill":
        entry, args = case["entry"], (st["x"], st["W_gate"], st["W_up"], st["W_down"], case["mini_seq"], st["out"])
        if entry == "static":
            binding.mom_mlp_prefill_static(*args, stream=main)
        elif entry == "two_stream":
            binding.mom_mlp_prefill_pipelined(*args, st["ws"], main, st["side"], st["events"])
        else:
            binding.mom_mlp_prefill(*args, st["ws"], stream=main)
        return {"out": st["out"]}
    if kind == "last":
        binding.mom_mlp_last(st["x_last"], st["W_gate"], st["W_up"], st["W_down"], st["out"], st["ws"], stream=main)
        binding.mom_lmhead_last(st["out"], st["W_lm"], st["logits"], stream=main)
        return {"out": st["out"], "logits": st["logits"]}
    if kind == "offload":
        binding.mom_kv_offload(st["k"], st["v"], st["host"], st["side"], producer_stream=main,
                               order_event=st["order"], done_event=st["done"])
        binding.mom_mlp_prefill(st["x"], st["W_gate"], st["W_up"], st["W_down"], case["mini_seq"], st["out"], st["ws"],
                                stream=main)
        main.wait_event(st["done"])
        return {"out": st["out"], "host": st["host"].view(torch.int16)}
    st["side"].wait_stream(main)     # the old contents of k and v are no longer read
    binding.mom_kv_reload(st["host"], st["k"], st["v"], st["side"], done_event=st["done"])
    binding.mom_mlp_last(st["x_last"], st["W_gate"], st["W_up"], st["W_down"], st["out"], st["ws"], stream=main)
    main.wait_event(st["done"])
    return {"out": st["out"], "k": st["k"].view(torch.int16), "v": st["v"].view(torch.int16)}


def work(case):
    H, I, V = _shape(case)
    kind = case["kind"]
    rows = case["S"] if kind in ("prefill", "offload") else 1
    b = 2 * 3 * H * I + 2 * 2 * rows * H                 # the weights, the tokens in and out
    f = 6 * rows * H * I
    if kind == "last":
        b += 2 * V * H + 4 * V
        f += 2 * V * H
    if kind in ("offload", "reload"):
        b += 2 * 2 * case["S"] * KV_HEADS * HEAD_DIM * 2     # K and V read once and written once
    return {"bytes": b, "flops": f}


def tolerance(case):
    # bf16 results of fp32 sums, the intermediate rounded once to bf16.  The same with the sums in another order
    # (plain float32 matrix products) differs by up to 4.4e-4 in norm and by one bf16 unit, 2^-7 of a value, at
    # most: four times that.  Bytes that are only moved, and the whole numbers they are seen as, stay the same.
    return {"rel": 1.8e-3, "max": 3.2e-2, "differ": 0.0}


def _mlp64(x, t):
    out = torch.empty((x.shape[0], t["W_down"].shape[0]), dtype=torch.float64, device=x.device)
    wg, wu, wd = (t[n].double().t().contiguous() for n in ("W_gate", "W_up", "W_down"))
    for r in range(0, x.shape[0], 8192):
        xr = x[r:r + 8192].double()
        g = xr @ wg
        h = g / (1.0 + torch.exp(-g))
        del g
        h *= xr @ wu
        out[r:r + 8192] = h @ wd
        del h
    return out


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "prefill":
        return {"out": _mlp64(t["x"], t)}
    if kind == "last":
        # the head multiplies the token the MLP handed on, which is a bf16 tensor
        out = _mlp64(t["x_last"].view(1, -1), t)
        last = out.to(torch.bfloat16).double()
        logits = torch.cat([last @ t["W_lm"][r:r + 16384].double().t().contiguous() for r in range(0, t["W_lm"].shape[0], 16384)], 1)
        return {"out": out.view(-1), "logits": logits.view(-1)}
    if kind == "offload":
        return {"out": _mlp64(t["x"], t), "host": torch.cat([t["k"].view(-1), t["v"].view(-1)]).cpu().view(torch.int16)}
    return {"out": _mlp64(t["x_last"].view(1, -1), t).view(-1), "k": t["k"].view(torch.int16), "v": t["v"].view(torch.int16)}
