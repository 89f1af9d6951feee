"""GPU parity of the stage forward/backward against the fp64 oracle, through the C ABI."""
import numpy as np
import pytest

import synth_inputs as si
from tests import harness as hz

pytestmark = pytest.mark.gpu


def test_cfg0_tiny_gpt_fp32_full():
    """Tiny GPT-style stage in fp32: all 4 micro-batches, gradients accumulated; bound 1e-4."""
    errs = hz.run_fwd_bwd_parity(si.CONFIGS[0])
    print({k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("name,kw", [
    ("gpt_d64", dict(layers=2, hidden=256, heads=4, seq=192, microbatch=2, causal=True)),
    ("gpt_d128_ragged", dict(layers=2, hidden=256, heads=2, seq=200, microbatch=1, causal=True)),
    ("bert_d64_padded", dict(layers=2, hidden=256, heads=4, seq=160, microbatch=3, causal=False,
                             len_lo=40, len_hi=160)),
    ("bert_full_len", dict(layers=1, hidden=128, heads=2, seq=96, microbatch=2, causal=False)),
    ("bert_d40_padded", dict(layers=2, hidden=320, heads=8, seq=128, microbatch=2, causal=False,
                             len_lo=40, len_hi=128)),
    ("gpt_d96", dict(layers=2, hidden=384, heads=4, seq=192, microbatch=1, causal=True)),
])
def test_small_bf16_stages(name, kw):
    cfg = si.scaled(si.CONFIGS[1], name="small_" + name, n_micro=2, **kw)
    errs = hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1)
    worst = max(errs.items(), key=lambda kv: kv[1])
    print(name, "worst", worst)


@pytest.mark.parametrize("stash_recompute,wgrad_group,causal", [(0, 0, True), (1, 2, True), (0, 3, False)])
def test_forward_ahead_small_stages(stash_recompute, wgrad_group, causal):
    """Forwards on their own stream, one micro-batch ahead of the backwards (F0 F1 B0 F2 B1 ...), no
    synchronisation in between: outputs, input gradients and accumulated parameter gradients against
    the oracle, with the full and the reduced stash and with weight-gradient groups that end inside
    and at the end of the run."""
    kw = dict(layers=2, hidden=256, heads=4, seq=192, microbatch=2, causal=causal)
    if not causal:
        kw.update(len_lo=40, len_hi=192)
    cfg = si.scaled(si.CONFIGS[1], name="small_ahead", n_micro=5, **kw)
    hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1, sync_each=False, forward_ahead=True,
                          stash_recompute=stash_recompute, wgrad_group=wgrad_group)


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_forward_ahead_any_lead_gives_the_same_bits(seed):
    """Forwards up to three micro-batches ahead of the backwards, in a random but valid interleaving
    (backwards in micro-batch order, so the weight-gradient groups form the same way), three iterations
    on one object so that stash slots and group buffers are reused across the streams: every output and
    gradient equals, bit for bit, what the same object type gives in the plain order on one stream."""
    import torch
    rng = np.random.default_rng(seed)
    kw = [dict(layers=2, hidden=256, heads=4, seq=128, microbatch=2, causal=True),
          dict(layers=1, hidden=384, heads=4, seq=192, microbatch=1, causal=True),
          dict(layers=2, hidden=256, heads=2, seq=128, microbatch=3, causal=False, len_lo=30, len_hi=128)][seed]
    n_micro = 7
    cfg = si.scaled(si.CONFIGS[1], name="ahead_rand", n_micro=n_micro, **kw)
    params = si.make_params(cfg, seed, 0.1)
    ins = [(hz.to_dev(si.make_activation(cfg, "act_in", mb, seed), cfg.dtype),
            hz.to_dev(si.make_activation(cfg, "grad_out", mb, seed), cfg.dtype)) for mb in range(n_micro)]

    def calls(lead):
        order, f, b = [], 0, 0
        while b < n_micro:
            can_f = f < n_micro and f - b < lead
            if can_f and (f == b or rng.random() < 0.6):
                order.append(("F", f)); f += 1
            else:
                order.append(("B", b)); b += 1
        return order

    def run(forward_ahead, lead):
        with hz.GpuStage(cfg, max_inflight=4, wgrad_group=[3, 0, 2][seed], stash_recompute=int(seed == 1),
                         forward_ahead=forward_ahead) as g:
            g.load_params(params)
            for mb in range(n_micro):
                lens = si.make_seqlens(cfg, mb, seed)
                if lens is not None:
                    g.bp.bp_stage_set_seqlens(g.h, mb, lens)
            for it in range(3):
                g.bp.bp_stage_zero_grad(g.h)
                zs, dxs = {}, {}
                for kind, mb in calls(lead):
                    if kind == "F":
                        zs[mb] = g.forward(0, mb, ins[mb][0])
                    else:
                        dxs[mb] = g.backward(0, mb, ins[mb][1])
                g.bp.bp_stage_wait_forward(g.h)
            torch.cuda.synchronize()
            outs = [(hz.to_host(zs[mb]), hz.to_host(dxs[mb])) for mb in range(n_micro)]
            grads = {(l, n): g.grad(0, l, n) for l in range(cfg.layers) for n in si.PARAM_NAMES}
        return outs, grads

    outs_a, grads_a = run(1, 3)
    outs_b, grads_b = run(0, 1)
    for mb in range(n_micro):
        assert np.array_equal(outs_a[mb][0], outs_b[mb][0]), f"act_out[{mb}]"
        assert np.array_equal(outs_a[mb][1], outs_b[mb][1]), f"grad_in[{mb}]"
    for k in grads_a:
        assert np.array_equal(grads_a[k], grads_b[k]), k


class _EarlyReads:
    """Iterations on two chunks (four for a schedule) whose gradients are worth reading early, with other inputs in
    every iteration: what a read right behind the last call gives is compared with what an object gives that is
    synchronised before every step."""

    def __init__(self, n_micro=4, wgrad_group=4, stash_recompute=0, forward_ahead=0, n_chunks=2, layers=2):
        self.opts = dict(max_inflight=n_chunks * 2, wgrad_group=wgrad_group, stash_recompute=stash_recompute,
                         forward_ahead=forward_ahead)
        self.cfg = si.scaled(si.CONFIGS[1], name="read_early", layers=layers, hidden=1024, heads=8, seq=256, microbatch=4,
                             causal=True, n_chunks=n_chunks, n_micro=n_micro)
        self.params = si.make_params(self.cfg, 0, 0.1)
        self.names = [(c, l, n) for c in range(n_chunks) for l in range(layers) for n in si.PARAM_NAMES]

    def data(self, role, mb, it):
        return hz.to_dev(si.make_activation(self.cfg, role, mb, it), self.cfg.dtype)

    def stage(self):
        g = hz.GpuStage(self.cfg, **self.opts)
        g.load_params(self.params)
        return g

    def iteration(self, g, it, direction=lambda mb: 0, sync=False):
        import torch
        n = self.cfg.n_micro
        ins = [(self.data("act_in", mb, it), self.data("grad_out", mb, it)) for mb in range(n)]
        torch.cuda.synchronize()
        step = torch.cuda.synchronize if sync else (lambda: None)
        g.bp.bp_stage_zero_grad(g.h)
        keep = []                                   # (outputs stay allocated until the caller has read)
        def forward(mb):
            for c in range(self.cfg.n_chunks):
                keep.append(g.forward(c, mb, ins[mb][0])); step()
        lead = 1 if self.opts["forward_ahead"] else 0
        if lead:
            forward(0)
        for mb in range(n):
            if mb + lead < n:
                forward(mb + lead)
            for c in range(self.cfg.n_chunks):
                keep.append(g.backward(c, mb, ins[mb][1], direction(mb))); step()
        g.bp.bp_stage_wait_forward(g.h)
        return ins, keep

    def reference(self, it, **kw):
        import torch
        with self.stage() as g:
            keep = self.iteration(g, it, sync=True, **kw)
            g.grad(*self.names[-1])                 # completes the open groups
            torch.cuda.synchronize()
            return {k: g.grad(*k) for k in self.names}


def _assert_same(got, ref, what):
    for k in got:
        assert np.array_equal(got[k], ref[k]), (what, k)


@pytest.mark.parametrize("n_micro,wgrad_group,stash_recompute,forward_ahead", [
    (4, 4, 0, 0), (8, 4, 0, 0), (5, 2, 0, 0), (3, 1, 0, 0), (4, 4, 1, 0), (4, 4, 0, 1), (6, 2, 0, 1), (5, 4, 1, 1)])
@pytest.mark.parametrize("backwards", [False, True])
def test_gradients_read_while_others_are_computed(n_micro, wgrad_group, stash_recompute, forward_ahead, backwards):
    """bp_stage_get_grad waits for the tensor it copies and not for the weight-gradient GEMMs behind it: read
    right after the last call, in either order of the tensors, on two chunks and in two iterations over different
    inputs, every gradient has the bits of a synchronised run."""
    e = _EarlyReads(n_micro, wgrad_group, stash_recompute, forward_ahead)
    with e.stage() as g:
        for it in range(2):
            keep = e.iteration(g, it)
            got = {k: g.grad(*k) for k in (e.names[::-1] if backwards else e.names)}
            _assert_same(got, e.reference(it), it)


@pytest.mark.parametrize("forward_ahead", [0, 1])
def test_next_iteration_while_gradients_are_still_computed(forward_ahead):
    """One tensor read, the gradients cleared and the next iteration issued at once, while weight gradients of the
    one before still run; then once more with the launches timed (one stream) and once after that."""
    e = _EarlyReads(forward_ahead=forward_ahead)
    with e.stage() as g:
        keep, first = [], []
        for it in range(4):
            if it == 2:
                g.bp.bp_prof_enable(g.h, 1)
            elif it == 3:
                g.bp.bp_prof_enable(g.h, 0)
            keep.append(e.iteration(g, it))
            first.append({e.names[0]: g.grad(*e.names[0])})
        last = {k: g.grad(*k) for k in e.names}
    refs = [e.reference(it) for it in range(4)]
    for it in range(4):
        _assert_same(first[it], refs[it], it)
    _assert_same(last, refs[3], "last")


@pytest.mark.parametrize("forward_ahead,layers", [(0, 2), (1, 1), (0, 3)])
def test_open_group_dropped_and_its_buffers_used_again_at_once(forward_ahead, layers):
    """Three micro-batches of a group of four, cleared and started over several times without a wait: the buffers of
    a dropped group go to the next backwards while column reductions that read them may still run."""
    e = _EarlyReads(n_micro=3, wgrad_group=4, forward_ahead=forward_ahead, layers=layers)
    with e.stage() as g:
        keep = [e.iteration(g, it) for it in range(4)]
        got = {k: g.grad(*k) for k in e.names}
    _assert_same(got, e.reference(3), "last")


@pytest.mark.parametrize("n_micro,n_chunks,layers", [(16, 1, 2), (26, 1, 2), (17, 2, 1), (33, 1, 1)])
def test_kept_groups_give_the_bits_of_given_groups(n_micro, n_chunks, layers):
    """Groups of eight by default and one micro-batch ahead: complete groups are kept (two of 8 x 1024 tokens, a third
    makes the oldest multiply).  Their GEMMs add up in the same order as with a group size of eight given, where none
    is kept: the same bits, also when iterations are cleared unread, and the memory they take is bounded."""
    import paper_2410_19367_amd as bp
    kept, given = [_EarlyReads(n_micro=n_micro, wgrad_group=w, forward_ahead=1, n_chunks=n_chunks, layers=layers) for w in (0, 8)]
    got = []
    for e in (kept, given):
        with e.stage() as g:
            bp.bp_stage_reset_peak_bytes(g.h)
            one = bp.bp_stage_stash_bytes(g.h) + layers * e.cfg.T * (e.cfg.F + 5 * e.cfg.hidden) * 2
            results = []
            alive = [e.iteration(g, 0)]
            results.append({k: g.grad(*k) for k in e.names})
            alive += [e.iteration(g, 1), e.iteration(g, 2)]     # the first of these is cleared unread
            results.append({k: g.grad(*k) for k in e.names})
            got.append(results)
            most = bp.bp_stage_held_bytes(g.h)["peak_total"] / one / n_chunks
            assert most <= (16 + 8 + 2 if e is kept else 8 + 2), most
    for a, b in zip(*got):
        _assert_same(a, b, "kept")


def test_kept_groups_give_way_when_memory_is_short():
    """With room on the device for a few stashes only, groups are not kept: nothing fails that went through without
    keeping, and the bits stay.  (Groups that are kept when the room goes: the next test.)"""
    import torch
    e = _EarlyReads(n_micro=26, wgrad_group=0, forward_ahead=1, n_chunks=1, layers=2)
    peaks, results = [], []
    for room in (None, 8):                          # stashes with their buffers
        with e.stage() as g:
            torch.cuda.synchronize()
            torch.cuda.empty_cache()
            one = g.bp.bp_stage_stash_bytes(g.h) + 2 * e.cfg.T * (e.cfg.F + 5 * e.cfg.hidden) * 2
            # inputs and outputs of the iteration, left in torch's cache
            io = [hz.empty_like_dev((e.cfg.microbatch, e.cfg.seq, e.cfg.hidden), e.cfg.dtype) for _ in range(6 * e.cfg.n_micro)]
            hog = None
            if room:
                hog = torch.empty(torch.cuda.mem_get_info()[0] - room * one, dtype=torch.uint8, device="cuda")
            del io
            keep = e.iteration(g, 0)
            peaks.append(g.bp.bp_stage_held_bytes(g.h)["peak_total"])
            results.append({k: g.grad(*k) for k in e.names})
            del hog, keep
            torch.cuda.empty_cache()
    assert peaks[1] < peaks[0], peaks               # fewer stashes were held
    ref, got = results
    _assert_same(got, ref, "short of memory")


@pytest.mark.parametrize("layers", [1, 2])
@pytest.mark.parametrize("what", ["group buffer", "parameter"])
def test_memory_runs_out_while_a_group_is_kept(what, layers):
    """The device fills up after a group of eight has been kept: the next group buffer, or the temporary of a parameter
    that is set, takes the place of what is kept, and every gradient has the bits of the same groups given."""
    import torch
    n_micro = 16
    cfg = si.scaled(si.CONFIGS[1], name="runs_out", layers=layers, hidden=3072, heads=24, seq=512, microbatch=4, causal=True,
                    n_chunks=1, n_micro=n_micro)
    params = si.make_params(cfg, 0, 0.1, bulk=True)
    names = [(0, l, n) for l in range(layers) for n in si.PARAM_NAMES]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    shape = (n_micro, cfg.microbatch, cfg.seq, cfg.hidden)
    x, go = [torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2)]
    z, dx = torch.empty_like(x), torch.empty_like(x)
    group_buffer, spare = layers * 9 * cfg.T * cfg.hidden * 2, 48 << 20
    assert min(group_buffer, 4 * cfg.hidden * cfg.F) > 2 * spare

    def run(wgrad_group, fill_at):
        hog = []
        with hz.GpuStage(cfg, wgrad_group=wgrad_group, max_inflight=3) as g:
            g.load_params(params)
            for mb in range(n_micro + 1):
                if mb < n_micro:
                    g.bp.bp_stage_forward(g.h, 0, mb, x[mb], z[mb])
                if mb == 0:
                    continue
                if mb - 1 == fill_at:
                    # the forwards' stashes first, so that what is short is the buffer (or the temporary) alone
                    torch.cuda.synchronize()
                    held = g.bp.bp_stage_held_bytes(g.h)
                    assert held["group_stash"] >= 8 * g.bp.bp_stage_stash_bytes(g.h), held
                    rest = torch.empty(spare, dtype=torch.uint8, device="cuda")
                    size = torch.cuda.mem_get_info()[0]
                    while size > 20 << 20:          # until nothing larger is to be had (the free size is an estimate)
                        try:
                            hog.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
                        except torch.cuda.OutOfMemoryError:
                            size //= 2
                    del rest
                    torch.cuda.empty_cache()
                    if what == "parameter":
                        g.bp.bp_stage_set_param(g.h, 0, layers - 1, g.bp.TENSOR_IDS["w1"], params[0][layers - 1]["w1"])
                g.bp.bp_stage_backward(g.h, 0, mb - 1, go[mb - 1], dx[mb - 1])
                if mb - 1 == fill_at:
                    held = g.bp.bp_stage_held_bytes(g.h)
                    assert held["group_stash"] <= 2 * g.bp.bp_stage_stash_bytes(g.h), held
            return {k: g.grad(*k) for k in names}

    ref = run(8, -1)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    try:
        got = run(0, 9)
    finally:
        torch.cuda.empty_cache()                    # the others leave
    _assert_same(got, ref, "ran out")


@pytest.mark.parametrize("hidden,dtype", [(64, "f32"), (1024, "bf16"), (4096, "bf16"), (4104, "bf16")])
def test_gradients_read_into_pinned_memory(hidden, dtype):
    """Small tensors are written to pinned host memory by a kernel, others copied: the same values as in pageable
    memory, at any offset of whole floats, with nothing around them touched (sizes on both sides of 16 KB)."""
    import torch
    import paper_2410_19367_amd as bp
    cfg = si.scaled(si.CONFIGS[1], name="pinned", layers=1, hidden=hidden, heads=1 if hidden == 64 else hidden // 8 if hidden == 4104 else 8, seq=16,
                    microbatch=1, n_micro=1, dtype=dtype)
    vectors = [n for n in si.PARAM_NAMES if n not in ("wqkv", "wo", "w1", "w2")]
    with hz.GpuStage(cfg) as g:
        g.forward(0, 0, hz.to_dev(si.make_activation(cfg, "act_in", 0, 0), cfg.dtype))
        g.backward(0, 0, hz.to_dev(si.make_activation(cfg, "grad_out", 0, 0), cfg.dtype))
        for n in vectors:
            ref = g.grad(0, 0, n).ravel()
            for off in (0, 1, 7):
                buf = torch.full((ref.size + 16,), 7.0, pin_memory=True)
                rc = bp.lib().bp_stage_get_grad(g.h, 0, 0, bp.TENSOR_IDS[n], buf.data_ptr() + 4 * off, ref.size)
                assert rc == bp.BP_OK
                got = buf.numpy()
                assert np.array_equal(got[off:off + ref.size], ref), (n, off)
                assert np.all(got[:off] == 7) and np.all(got[off + ref.size:] == 7), (n, off)


@pytest.mark.parametrize("stash_recompute", [0, 1])
def test_parameters_set_while_gradients_are_still_computed(stash_recompute):
    """Parameters set right after the first read: the gradients still to come are those of the old ones (the
    weight gradients of the reduced stash read LayerNorm parameters and b1 when they run)."""
    e = _EarlyReads(stash_recompute=stash_recompute)
    ref = e.reference(0)
    with e.stage() as g:
        keep = e.iteration(g, 0)
        got = {e.names[0]: g.grad(*e.names[0])}
        for c, l, n in e.names:
            g.bp.bp_stage_set_param(g.h, c, l, g.bp.TENSOR_IDS[n], np.full(si.param_shape(e.cfg, n), 0.5, np.float32))
        got.update({k: g.grad(*k) for k in e.names[1:]})
        _assert_same(got, ref, "old parameters")


def test_schedule_while_gradients_are_still_computed():
    """A whole schedule iteration right after the first read: its gradients are those of an object that has done
    nothing else."""
    import torch
    e = _EarlyReads(n_chunks=4, layers=1)
    runs = []
    for before in (False, True):
        with e.stage() as g:
            if before:
                keep = e.iteration(g, 0)
                g.grad(*e.names[0])
            order = g.bp.bp_schedule_generate(2, e.cfg.n_micro)
            x = torch.stack([e.data("act_in", mb, 7) for mb in range(e.cfg.n_micro)])
            y = torch.stack([e.data("target", mb, 7) for mb in range(e.cfg.n_micro)])
            g.bp.bp_run_schedule(g.h, order, 2, x, y)
            runs.append({k: g.grad(*k) for k in e.names})
    _assert_same(runs[1], runs[0], "schedule")


def test_two_directions_read_while_gradients_are_still_computed():
    """Micro-batches 0, 1, 4, 5 in one direction, the others in the other: a read gives direction 0 alone; after the
    merge both, as a synchronised object gives them."""
    import torch
    e = _EarlyReads(n_micro=8, wgrad_group=2)
    direction = lambda mb: mb // 2 % 2
    merged, first = [], []
    for sync in (True, False):
        with e.stage() as g:
            keep = e.iteration(g, 0, direction=direction, sync=sync)
            first.append({k: g.grad(*k) for k in e.names})
            g.bp.bp_stage_merge_directions(g.h)
            merged.append({k: g.grad(*k) for k in e.names})
    _assert_same(first[1], first[0], "direction 0")
    _assert_same(merged[1], merged[0], "both")


@pytest.mark.parametrize("hidden,group,early", [(1024, 4, True), (1024, 2, True), (256, 4, False)])
def test_peak_of_held_memory_counts_the_complete_group(hidden, group, early):
    """With gradients worth reading early (16 MB and more in a chunk) the call that completes a weight-gradient
    group writes into a group buffer like the others: at the peak the object holds `group` stashes and as many
    buffers of dz, du, dy, dqkv; else the last micro-batch has its stash only."""
    import paper_2410_19367_amd as bp
    cfg = si.scaled(si.CONFIGS[1], name="held", layers=2, hidden=hidden, heads=4, seq=128, microbatch=2, causal=True, n_micro=group)
    assert early == (cfg.layers * 12 * hidden * hidden * 4 >= 16 << 20)
    with hz.GpuStage(cfg, max_inflight=2, wgrad_group=group) as g:
        g.load_params(si.make_params(cfg, 0, 0.1))
        bp.bp_stage_reset_peak_bytes(g.h)
        stash = bp.bp_stage_stash_bytes(g.h)
        buffer = cfg.layers * cfg.T * (cfg.F + 5 * hidden) * 2
        for mb in range(group):
            g.forward(0, mb, hz.to_dev(si.make_activation(cfg, "act_in", mb, 0), cfg.dtype))
            g.backward(0, mb, hz.to_dev(si.make_activation(cfg, "grad_out", mb, 0), cfg.dtype))
        held = bp.bp_stage_held_bytes(g.h)
        assert (held["live_stash"], held["group_stash"], held["group_grads"]) == (0, 0, 0)
        assert held["peak_total"] == group * stash + (group if early else group - 1) * buffer


def test_group_completed_while_a_stash_is_live_multiplies_at_once():
    """F0 F1 B0 F2 B1 F3 B2 B3 in groups of two: B1 completes a group while the stash of F2 is live, so more backwards
    follow and its weight gradients start beside its own chain, without a group buffer; B3 is the last one.
    The most that is held is then at F2: its stash, that of F1, that of the waiting B0 and B0's buffer."""
    import paper_2410_19367_amd as bp
    cfg = si.scaled(si.CONFIGS[1], name="held_ahead", layers=2, hidden=1024, heads=4, seq=128, microbatch=2, causal=True, n_micro=4)
    with hz.GpuStage(cfg, max_inflight=2, wgrad_group=2, forward_ahead=1) as g:
        g.load_params(si.make_params(cfg, 0, 0.1))
        bp.bp_stage_reset_peak_bytes(g.h)
        xs = [hz.to_dev(si.make_activation(cfg, "act_in", mb, 0), cfg.dtype) for mb in range(4)]
        dys = [hz.to_dev(si.make_activation(cfg, "grad_out", mb, 0), cfg.dtype) for mb in range(4)]
        g.forward(0, 0, xs[0])
        for mb in range(4):
            if mb + 1 < 4:
                g.forward(0, mb + 1, xs[mb + 1])
            g.backward(0, mb, dys[mb])
        bp.bp_stage_wait_forward(g.h)
        buffer = cfg.layers * cfg.T * (cfg.F + 5 * cfg.hidden) * 2
        assert bp.bp_stage_held_bytes(g.h)["peak_total"] == 3 * bp.bp_stage_stash_bytes(g.h) + buffer


def test_small_fp32_bert_padded():
    cfg = si.scaled(si.CONFIGS[0], name="small_f32_bert", causal=False, len_lo=10, len_hi=64,
                    microbatch=3, n_micro=2)
    hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1)


def test_state_errors():
    import paper_2410_19367_amd as bp
    cfg = si.scaled(si.CONFIGS[0], name="state", layers=1)
    with hz.GpuStage(cfg, max_inflight=2) as g:
        x = hz.to_dev(si.make_activation(cfg, "act_in", 0), cfg.dtype)
        out = hz.empty_like_dev(tuple(x.shape), cfg.dtype)
        with pytest.raises(bp.BitPipeError) as e:
            bp.bp_stage_backward(g.h, 0, 0, x, out)
        assert e.value.code == bp.BP_ESTATE
        bp.bp_stage_forward(g.h, 0, 0, x, out)
        with pytest.raises(bp.BitPipeError) as e:
            bp.bp_stage_forward(g.h, 0, 0, x, out)
        assert e.value.code == bp.BP_ESTATE
        bp.bp_stage_forward(g.h, 0, 1, x, out)
        with pytest.raises(bp.BitPipeError) as e:      # max_inflight = 2
            bp.bp_stage_forward(g.h, 0, 2, x, out)
        assert e.value.code == bp.BP_ESTATE
        with pytest.raises(bp.BitPipeError) as e:
            bp.bp_stage_forward(g.h, 1, 0, x, out)
        assert e.value.code == bp.BP_EINVAL
        with pytest.raises(bp.BitPipeError) as e:
            bp.bp_stage_set_seqlens(g.h, 0, np.array([3, 3], dtype=np.int32))
        assert e.value.code == bp.BP_ESTATE       # causal stage
        bp.bp_stage_backward(g.h, 0, 1, x, out)
        bp.bp_stage_backward(g.h, 0, 0, x, out)
        with pytest.raises(bp.BitPipeError):
            bp.bp_stage_set_param(g.h, 0, 0, bp.TENSOR_IDS["wo"], np.zeros(7, dtype=np.float32))
    with pytest.raises(bp.BitPipeError) as e:
        bp.bp_stage_init(1, 100, 3, 8, 1, 1)
    assert e.value.code == bp.BP_ESHAPE


def test_zero_grad_semantics_across_iterations():
    """The clear between iterations: gradients read right after it are zero, an iteration after it
    reproduces the oracle's single-iteration gradients (nothing left over from the iteration
    before, nothing lost from the first micro-batch), and a second chunk that never ran a
    backward reads as zero."""
    cfg = si.scaled(si.CONFIGS[1], name="small_clear", layers=2, hidden=256, heads=2, seq=128,
                    microbatch=2, n_micro=3, n_chunks=2)
    params = si.make_params(cfg, 3, 0.1)
    orc = hz.make_oracle(cfg, params)
    with hz.GpuStage(cfg) as g:
        g.load_params(params)

        def iteration(seed, with_oracle):
            for mb in range(cfg.n_micro):
                x = si.make_activation(cfg, "act_in", mb, seed)
                go = si.make_activation(cfg, "grad_out", mb, seed)
                g.forward(0, mb, hz.to_dev(x, cfg.dtype))
                g.backward(0, mb, hz.to_dev(go, cfg.dtype))
                if with_oracle:
                    orc.forward(0, mb, x)
                    orc.backward(0, mb, go)

        iteration(11, False)                    # leaves non-zero gradients behind
        assert np.abs(g.grad(0, 1, "w1")).max() > 0
        g.bp.bp_stage_zero_grad(g.h)
        for name in si.PARAM_NAMES:
            assert not g.grad(0, 0, name).any(), name
        iteration(12, True)
        for l in range(cfg.layers):
            for name in si.PARAM_NAMES:
                err = hz.rel_err(g.grad(0, l, name), orc.get_grad(0, l, name))
                assert err <= hz.TOL[cfg.dtype], (l, name, err)
                assert not g.grad(1, l, name).any(), ("chunk 1 never ran", l, name)


@pytest.mark.parametrize("group,n_micro", [(1, 5), (2, 5), (3, 5), (4, 5), (5, 5), (8, 5), (8, 9)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_grouped_weight_gradients(group, n_micro, dtype):
    """Weight gradients computed over groups of 1..8 backward calls: the micro-batches give
    complete groups plus a remainder (or no complete group at all) that only the gradient
    read-out flushes; activations, input gradients and all accumulated gradients must match the
    oracle either way."""
    base = si.CONFIGS[1] if dtype == "bf16" else si.CONFIGS[0]
    cfg = si.scaled(base, name=f"small_group{group}_{n_micro}", layers=2, hidden=256, heads=2, seq=128,
                    microbatch=2, n_micro=n_micro, dtype=dtype, causal=True)
    hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1, wgrad_group=group)


def test_grouped_weight_gradients_interleaved_chunks_and_directions():
    """Groups are kept per (chunk, direction): backward calls of two chunks and both directions
    interleave, with more stashes alive than any one group holds, and a clear in the middle of
    a group discards that group's waiting contributions."""
    cfg = si.scaled(si.CONFIGS[1], name="small_group_mix", layers=1, hidden=256, heads=2, seq=128,
                    microbatch=1, n_micro=5, n_chunks=2)
    params = si.make_params(cfg, 5, 0.1)
    orc = hz.make_oracle(cfg, params)
    with hz.GpuStage(cfg, max_inflight=12, wgrad_group=3) as g:
        g.load_params(params)
        xs = {mb: si.make_activation(cfg, "act_in", mb, 5) for mb in range(cfg.n_micro)}
        gos = {mb: si.make_activation(cfg, "grad_out", mb, 5) for mb in range(cfg.n_micro)}
        # a waiting contribution that the clear must discard
        g.forward(0, 0, hz.to_dev(xs[0], cfg.dtype))
        g.backward(0, 0, hz.to_dev(gos[0], cfg.dtype), direction=0)
        g.bp.bp_stage_zero_grad(g.h)
        for c in range(2):
            for mb in range(cfg.n_micro):
                g.forward(c, mb, hz.to_dev(xs[mb], cfg.dtype))
                orc.forward(c, mb, xs[mb])
        for mb in range(cfg.n_micro):
            for c in (1, 0):
                d = (mb + c) % 2
                g.backward(c, mb, hz.to_dev(gos[mb], cfg.dtype), direction=d)
                orc.backward(c, mb, gos[mb], d)
        # get_grad reads the direction-0 accumulators
        for c in range(2):
            for name in si.PARAM_NAMES:
                err = hz.rel_err(g.grad(c, 0, name), orc.grads[0][c][0][name])
                assert err <= hz.TOL[cfg.dtype], (c, name, err)
        # the sum of the two replicas (Section 3.4): direction 1 is added into direction 0, once
        for rep in range(2):
            g.bp.bp_stage_merge_directions(g.h)
            for c in range(2):
                for name in si.PARAM_NAMES:
                    want = orc.grads[0][c][0][name] + orc.grads[1][c][0][name]
                    err = hz.rel_err(g.grad(c, 0, name), want)
                    assert err <= hz.TOL[cfg.dtype], (rep, c, name, err)


@pytest.mark.parametrize("group", [1, 3, 5])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_lean_stash_recomputes_ln_and_gelu_outputs(group, dtype):
    """stash_recompute = 1 keeps 10 instead of 16 [T,H]-sized tensors per layer (Table 2's activation
    memory M_a) and rebuilds the LayerNorm and GELU outputs for the weight gradients: same
    activations, input gradients and accumulated gradients as the oracle, with and without
    grouped weight gradients (five micro-batches: complete groups and a flushed remainder)."""
    import paper_2410_19367_amd as bp
    base = si.CONFIGS[1] if dtype == "bf16" else si.CONFIGS[0]
    cfg = si.scaled(base, name=f"small_lean{group}", layers=2, hidden=256, heads=2, seq=128,
                    microbatch=2, n_micro=5, dtype=dtype, causal=True)
    hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1, wgrad_group=group, stash_recompute=1)
    with hz.GpuStage(cfg) as full, hz.GpuStage(cfg, stash_recompute=1) as lean:
        esz = 2 if dtype == "bf16" else 4
        T, H, F = cfg.T, cfg.hidden, cfg.F
        saved = bp.bp_stage_stash_bytes(full.h) - bp.bp_stage_stash_bytes(lean.h)
        assert saved == cfg.layers * (2 * T * H + T * F) * esz          # a, m and g of every layer
        # 16 T H elements per layer plus the row statistics and the softmax log-sum-exp
        stats = (4 * T + cfg.microbatch * cfg.heads * cfg.seq) * 4
        assert bp.bp_stage_stash_bytes(full.h) == cfg.layers * (16 * T * H * esz + stats)
        assert bp.bp_stage_stash_bytes(lean.h) == cfg.layers * (10 * T * H * esz + stats)


def _random_small_configs(n, seed):
    """Seeded draw of small stage shapes that land on different kernel paths: aligned and ragged
    GEMMs, head widths 32..128 (some padded), causal / padded-bidirectional, MLP widths that are
    and are not multiples of 128, all weight-gradient group sizes, lean and full stash."""
    import random
    rng = random.Random(seed)
    out = []
    for i in range(n):
        d = rng.choice([32, 40, 64, 96, 128])
        heads = rng.choice([1, 2, 3, 4])
        hidden = d * heads
        causal = rng.random() < 0.5
        seq = rng.choice([64, 128, 192, 100, 72]) if d in (64, 128) or rng.random() < 0.7 else rng.choice([64, 128])
        mb = rng.choice([1, 2, 3])
        mlp = rng.choice([4 * hidden, 2 * hidden, 3 * hidden + 8, 512])
        kw = dict(layers=rng.choice([1, 2]), hidden=hidden, heads=heads, seq=seq, microbatch=mb, causal=causal,
                  mlp=mlp, n_micro=rng.choice([1, 2, 3, 5]))
        if not causal and rng.random() < 0.7:
            kw.update(len_lo=max(1, seq // 4), len_hi=seq)
        out.append((i, kw, rng.choice([1, 2, 3, 4]), rng.choice([0, 1])))
    return out


@pytest.mark.parametrize("idx,kw,group,lean", _random_small_configs(16, 20241127))
def test_random_small_stage_configs(idx, kw, group, lean):
    cfg = si.scaled(si.CONFIGS[1], name=f"small_rand{idx}", **kw)
    errs = hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1, wgrad_group=group, stash_recompute=lean, seed=idx)
    worst = max(errs.items(), key=lambda kv: kv[1])
    print(idx, kw, "group", group, "lean", lean, "worst", worst)


@pytest.mark.parametrize("kw,group,lean", [
    # T = 231 tokens (odd), width a multiple of 8 only, MLP deep enough for K slices: edge tiles in every GEMM form
    # with the fused GELU epilogues, token segments that end inside a slice
    (dict(layers=2, hidden=520, heads=13, seq=77, microbatch=3, causal=True, n_micro=4), 3, 0),
    (dict(layers=1, hidden=320, heads=5, seq=333, microbatch=2, causal=False, n_micro=2, len_lo=20, len_hi=333), 0, 1),
    # MLP so deep that the data-side products of its second matrix are cut along K, aligned and not
    (dict(layers=1, hidden=256, heads=4, seq=77, microbatch=3, causal=True, n_micro=2, mlp=4104), 2, 0),
    (dict(layers=1, hidden=256, heads=4, seq=128, microbatch=2, causal=True, n_micro=2, mlp=6144), 2, 0),
    # fp32: fused GELU epilogues with edge tiles
    (dict(layers=2, hidden=200, heads=5, seq=77, microbatch=3, causal=True, n_micro=4, dtype="f32"), 3, 0),
])
def test_ragged_stage(kw, group, lean):
    cfg = si.scaled(si.CONFIGS[1], name="small_ragged_edges", **kw)
    hz.run_fwd_bwd_parity(cfg, ln_jitter=0.1, wgrad_group=group, stash_recompute=lean)
