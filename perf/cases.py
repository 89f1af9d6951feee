"""What users of the stage library have it do: training iterations of one pipeline stage, and whole iterations
of the V-shaped bidirectional schedule, through the C ABI (`bp_stage_*`, `bp_run_schedule`).

One pass is one training iteration as a user's loop runs it: clear the gradients, take every micro-batch
forward and backward through the stage (or the whole schedule over them), and read all parameter gradients
back into the pinned host buffers that the optimizer works on.  Outputs: the activations handed to the next
stage, the input gradients handed to the previous one, and every parameter gradient.

A case is a dict of plain values:
  kind        "stage" (forward / backward calls) or "iteration" (bp_run_schedule)
  dtype       "bf16" or "f32" (storage type)          causal   GPT-style mask, else BERT-style
  layers, hidden, heads, seq, batch (sequences per micro-batch), micro (micro-batches per iteration)
  min_len     BERT-style key padding: valid lengths uniform on min_len..seq; 0: no padding
  ahead       forwards one micro-batch ahead on a stream of their own (bp_opts.forward_ahead)
  lean        reduced stash (bp_opts.stash_recompute)
  devices     "iteration" only: virtual devices D; the object holds 2 D chunks of `layers` layers
"""
import math
import weakref

import numpy as np
import torch

import paper_2410_19367_amd as bp

TENSORS = tuple(bp.TENSOR_IDS)            # ln1_g, ln1_b, wqkv, ... in the order of their ids


def _case(name, kind="stage", dtype="bf16", causal=True, layers=1, hidden=1024, heads=16, seq=1024, batch=1,
          micro=8, min_len=0, ahead=True, lean=False, devices=0):
    return {"name": name, "kind": kind, "dtype": dtype, "causal": causal, "layers": layers, "hidden": hidden,
            "heads": heads, "seq": seq, "batch": batch, "micro": micro, "min_len": min_len, "ahead": ahead,
            "lean": lean, "devices": devices}


def listed():
    return [
        # a toy stage in fp32, as run first to check an installation or a schedule: nothing but launches
        _case("f32_toy_h128", dtype="f32", layers=2, hidden=128, heads=2, seq=64, batch=2, micro=4, ahead=False),
        # a small bf16 stage on short sequences: latency and launch counts
        _case("bf16_small_h256", layers=2, hidden=256, heads=4, seq=192, batch=2, micro=4, ahead=False),
        # a debugging / reference run in fp32 at a width that real models have
        _case("f32_mid_h768", dtype="f32", layers=2, hidden=768, heads=12, seq=512, batch=2, micro=4, ahead=False),
        # GPT-style stage, micro-batches of one long sequence
        _case("gpt_h2048_s2048", layers=2, hidden=2048, heads=16, seq=2048, batch=1, micro=16),
        # BERT-style stage with padded sequences of 256..512 tokens
        _case("bert_h1024_s512", causal=False, layers=3, hidden=1024, heads=16, seq=512, batch=8, micro=8, min_len=256),
        # the widest GPT-style layer (the largest case); single products fill the chip: the plain call order
        _case("gpt_h5120_s2048", layers=1, hidden=5120, heads=40, seq=2048, batch=2, micro=16, ahead=False),
        # a whole bidirectional iteration, four virtual devices, sixteen micro-batches
        _case("vsched_h1024_d4", kind="iteration", layers=1, hidden=1024, heads=16, seq=1024, batch=1, micro=16,
              ahead=False, devices=4),
        # heads of width 40 (the BERT-64 stage shape), padded keys
        _case("bert_h2560_d40", causal=False, layers=2, hidden=2560, heads=64, seq=512, batch=4, micro=16, min_len=256),
        # heads of width 96 (the GPT-96 stage shape), short micro-batches, many of them
        _case("gpt_h3072_d96", layers=2, hidden=3072, heads=32, seq=1024, batch=1, micro=32),
        # sequences whose length is no multiple of any tile, width a multiple of 64 only
        _case("gpt_h1600_s1000", layers=2, hidden=1600, heads=25, seq=1000, batch=1, micro=8),
        # odd padded length, as a bucketed text batch has it
        _case("bert_h768_s333", causal=False, layers=2, hidden=768, heads=12, seq=333, batch=6, micro=8, min_len=100),
        # long context with the reduced stash: attention and activation memory
        _case("gpt_h1024_s6144", layers=2, hidden=1024, heads=16, seq=6144, batch=1, micro=2, lean=True),
    ]


# ---------------------------------------------------------------- sizes

def _chunks(c):
    return 2 * c["devices"] if c["kind"] == "iteration" else 1


def _flops(c):
    """Forward + backward of all micro-batches: three products per linear layer and 12 T S H for the attention
    (half of it under the causal mask), nothing recomputed."""
    T, H, S = c["batch"] * c["seq"], c["hidden"], c["seq"]
    attn = 12.0 * T * S * H * (0.5 if c["causal"] else 1.0)
    if c["min_len"]:
        attn *= 0.5 * (c["min_len"] + S) / S       # masked keys need no work
    return _chunks(c) * c["layers"] * c["micro"] * (72.0 * T * H * H + attn)


def work(c):
    T, H = c["batch"] * c["seq"], c["hidden"]
    e = 4 if c["dtype"] == "f32" else 2
    params = _chunks(c) * c["layers"] * 12.0 * H * H
    acts = c["micro"] * T * H * e * (2.0 if c["kind"] == "iteration" else 4.0)     # inputs and targets, or x, z, dz, dx
    return {"bytes": params * (e + 4.0) + acts, "flops": _flops(c)}


# ---------------------------------------------------------------- more cases of the same ranges

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_flops(c) for c in listed())
    while True:
        kind = rng.choices(("bf16", "ragged", "f32", "iteration"), (4, 3, 2, 2))[0]
        d = rng.choice((40, 64, 64, 96, 128))
        if kind == "f32":
            H = max(2, round(_log_int(rng, 128, 1024) / d)) * d
            c = _case("", dtype="f32", layers=rng.randint(1, 2), hidden=H, heads=H // d, seq=_log_int(rng, 48, 700),
                      batch=rng.randint(1, 3), micro=rng.randint(2, 4), causal=rng.random() < 0.6, ahead=False)
            limit = 1.5e12
        elif kind == "iteration":
            H = max(2, round(_log_int(rng, 256, 1536) / d)) * d
            D = rng.choice((2, 4))
            c = _case("", kind="iteration", layers=1, hidden=H, heads=H // d, seq=32 * rng.randint(4, 32), batch=1,
                      micro=D * rng.randint(1, 4), causal=True, ahead=False, devices=D)
            limit = most / 4
        else:
            H = max(2, round(_log_int(rng, 256, 4096 if kind == "bf16" else 2048) / d)) * d
            S = 64 * _log_int(rng, 2, 64) if kind == "bf16" else _log_int(rng, 64, 1500)
            c = _case("", layers=rng.randint(1, 3), hidden=H, heads=H // d, seq=S,
                      batch=rng.randint(1, max(1, min(8, 4096 // S))), micro=rng.randint(2, 16),
                      causal=rng.random() < 0.6, ahead=rng.random() < 0.6, lean=rng.random() < 0.2)
            limit = most / 2 if kind == "bf16" else most / 10
        if not c["causal"] and rng.random() < 0.7:
            c["min_len"] = max(1, c["seq"] // rng.randint(2, 4))
        del c["name"]
        if _flops(c) <= limit:
            return c


# ---------------------------------------------------------------- a stage and its buffers

class State:
    """A stage object with its parameters set, the device tensors of one iteration and the pinned host
    buffers its gradients are read into."""


def _destroy(handle):
    bp.bp_stage_destroy(handle)


def _param_shape(name, H):
    return {"wqkv": (H, 3 * H), "bqkv": (3 * H,), "wo": (H, H), "w1": (H, 4 * H), "b1": (4 * H,),
            "w2": (4 * H, H)}.get(name, (H,))


def _parameter(name, H, gen):
    """N(0, 0.02) matrices and biases, LayerNorm parameters scattered around (1, 0)."""
    v = torch.randn(_param_shape(name, H), device="cuda", generator=gen)
    if name in ("ln1_g", "ln2_g"):
        return 1.0 + 0.1 * v
    return v * (0.1 if name in ("ln1_b", "ln2_b") else 0.02)


def prepare(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    H, shape = c["hidden"], (c["micro"], c["batch"], c["seq"], c["hidden"])
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    s = State()
    s.case = c
    s.handle = bp.bp_stage_init_ex(c["layers"], H, c["heads"], c["seq"], c["batch"], c["causal"], n_chunks=_chunks(c),
                                   dtype=bp.BP_F32 if c["dtype"] == "f32" else bp.BP_BF16,
                                   max_inflight=2 if c["kind"] == "stage" else 0,
                                   stash_recompute=int(c["lean"]), forward_ahead=int(c["ahead"]))
    weakref.finalize(s, _destroy, s.handle)
    host = {n: torch.empty(_param_shape(n, H), pin_memory=True) for n in TENSORS}
    for chunk in range(_chunks(c)):
        for layer in range(c["layers"]):
            for n in TENSORS:
                host[n].copy_(_parameter(n, H, gen))
                bp.bp_stage_set_param(s.handle, chunk, layer, bp.TENSOR_IDS[n], host[n].numpy())
    if c["min_len"]:
        for mb in range(c["micro"]):
            lens = torch.randint(c["min_len"], c["seq"] + 1, (c["batch"],), device="cuda", generator=gen)
            bp.bp_stage_set_seqlens(s.handle, mb, lens.cpu().numpy().astype(np.int32))
    s.x = torch.randn(shape, device="cuda", generator=gen).to(dt)
    s.y = torch.randn(shape, device="cuda", generator=gen).to(dt)      # output gradients, or the loss targets
    if c["kind"] == "stage":
        s.z, s.dx = torch.empty_like(s.x), torch.empty_like(s.x)
    else:
        s.order = bp.bp_schedule_generate(c["devices"], c["micro"])
    s.grads = {n: torch.empty((_chunks(c), c["layers"]) + _param_shape(n, H), pin_memory=True) for n in TENSORS}
    return s


def _read_gradients(s):
    get = bp.lib().bp_stage_get_grad
    for chunk in range(_chunks(s.case)):
        for layer in range(s.case["layers"]):
            for n in TENSORS:
                g = s.grads[n][chunk, layer]
                rc = get(s.handle, chunk, layer, bp.TENSOR_IDS[n], g.data_ptr(), g.numel())
                if rc != bp.BP_OK:
                    raise bp.BitPipeError(rc, bp.bp_last_error())


def run(s):
    c, h = s.case, s.handle
    if c["kind"] == "iteration":
        loss = bp.bp_run_schedule(h, s.order, c["devices"], s.x, s.y)
        _read_gradients(s)
        return {"loss": loss, **s.grads}
    bp.bp_stage_zero_grad(h)
    n = c["micro"]
    if c["ahead"]:                      # F(0) F(1) B(0) F(2) B(1) ...
        bp.bp_stage_forward(h, 0, 0, s.x[0], s.z[0])
    for mb in range(n):
        nxt = mb + 1 if c["ahead"] else mb
        if nxt < n:
            bp.bp_stage_forward(h, 0, nxt, s.x[nxt], s.z[nxt])
        bp.bp_stage_backward(h, 0, mb, s.y[mb], s.dx[mb])
    if c["ahead"]:
        bp.bp_stage_wait_forward(h)
    _read_gradients(s)
    return {"z": s.z, "dx": s.dx, **s.grads}


def tolerance(c):
    """Measured against the same iteration in 64 bits, over all outputs: f32 rel 1.2e-6, max 1.3e-5; bf16 stages
    rel 4e-3 to 8e-3 (the widest), max 8e-2 (q and k columns of the first causal rows); schedule iterations, whose
    outputs are sums over many micro-batches, rel 1.6e-3, max 1.5e-2."""
    if c["dtype"] == "f32":
        return {"rel": 5e-6, "max": 6e-5}
    if c["kind"] == "iteration":
        return {"rel": 6e-3, "max": 6e-2}
    return {"rel": 1.5e-2, "max": 0.25}
