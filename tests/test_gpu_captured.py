"""Calls that the caller captures into a HIP graph and replays: what a replay does may not depend on what the host knew when
the call was recorded."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def context(cfg, weights, stream=None):
    from paper_1811_03115_amd import binding
    ctx = binding.Context(binding.config_from_workload(cfg), stream=stream)
    ctx.bpd_load_weights(weights)
    return ctx


def capture(stream, call):
    """A graph of what `call` enqueues on `stream`."""
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        call()
    return g


def replay(g, stream):
    with torch.cuda.stream(stream):
        g.replay()


def snapshot(ctx):
    st = ctx.bpd_get_stats()
    return [np.array(v) for v in ctx.bpd_get_state()] + [np.array(v) for v in ctx.bpd_get_output()] + [np.array([st.steps, st.seq_steps, st.accepted_total, st.finished])]


def same(a, b, what):
    for u, v in zip(a, b):
        np.testing.assert_array_equal(u, v, err_msg=what)


def job(cfg, seed):
    """Sources and budgets: one sequence ends in every other step from the second on, at two tokens a step."""
    src, n = wl.make_sources(cfg)
    budget = np.minimum(4 * np.arange(1, cfg.batch + 1), cfg.max_out).astype(np.int32)
    return src, n, np.random.default_rng(seed).permutation(budget)


# one row tile; several, of a width without and with kernels of a constant K; two-phase scoring
@pytest.mark.parametrize("d,F,k,B,two_phase", [(128, 512, 3, 4, False), (192, 384, 5, 6, False), (128, 512, 4, 9, False), (128, 512, 5, 7, True)])
def test_step_captured_after_a_sequence_has_ended(d, F, k, B, two_phase):
    cfg = wl.Config("captured", 80, 1, 2, d, d // 64, F, 272, k, B, 7, 4 * B, "bf16", -1, src_len_kind="lognormal")
    weights = wl.make_weights(cfg)
    stream = torch.cuda.Stream()
    ref, cap = context(cfg, weights), context(cfg, weights, stream)
    src, n, budget = job(cfg, B)
    two = torch.full((B,), 2, dtype=torch.int32, device="cuda")
    acc = torch.zeros((2, B), dtype=torch.int32, device="cuda")
    for c in (ref, cap):
        c.bpd_set_two_phase(two_phase)
        c.bpd_encode(src, n, budget)
        for _ in range(2):
            c.bpd_step(k, two)
    assert ref.bpd_get_state()[3].sum() == 1
    same(snapshot(ref), snapshot(cap), "before the capture")
    g = capture(stream, lambda: cap.bpd_step_static(k, two, acc[1]))
    same(snapshot(ref), snapshot(cap), "recorded, not run")
    for s in range(2 * B - 1):
        ref.bpd_step(k, two, acc[0])
        replay(g, stream)
        same(snapshot(ref), snapshot(cap), f"replay {s}")
        torch.cuda.synchronize()
        assert acc[0].tolist() == acc[1].tolist()
        if s == B:                                         # a direct step in between
            ref.bpd_step(k, two)
            cap.bpd_step_static(k, two)
    assert ref.bpd_get_state()[3].all()


@pytest.mark.parametrize("dtype,d,F,host", [("bf16", 128, 512, False), ("bf16", 192, 384, False), ("bf16", 128, 512, True), ("f32", 64, 256, False), ("f32", 64, 1024, True)])
def test_captured_encode(dtype, d, F, host):
    """A captured encode takes what its arrays hold at each replay, and direct encodes go on before the first replay and
    between replays."""
    cfg = wl.Config("captured", 84, 1, 2, d, d // (64 if dtype == "bf16" else 16), F, 272, 4, 3, 20, 12, dtype, 2)
    weights = wl.make_weights(cfg, std=0.1)
    stream = torch.cuda.Stream()
    ref, cap = context(cfg, weights), context(cfg, weights, stream)
    rng = np.random.default_rng(d)
    arrays = [np.zeros((3, 20), np.int32), np.ones(3, np.int32), np.ones(3, np.int32)]
    if not host:
        arrays = [torch.from_numpy(a).cuda() for a in arrays]

    def fill():
        n = rng.integers(1, 21, 3).astype(np.int32)
        new = [rng.integers(3, cfg.vocab, (3, 20)).astype(np.int32), n, rng.integers(1, 13, 3).astype(np.int32)]
        for a, v in zip(arrays, new):
            if host:
                a[...] = v
            else:
                a.copy_(torch.from_numpy(v))
        torch.cuda.synchronize()
        return new

    fill()
    g = capture(stream, lambda: cap.bpd_encode(*arrays))
    for s in range(6):
        new = fill()
        if s in (0, 1, 3):                                 # direct encodes of other sources, from host memory
            other = [np.roll(new[0], 1, 0), np.roll(new[1], 1), np.roll(new[2], 1)]
            for c in (ref, cap):
                c.bpd_encode(*other)
            same(snapshot(ref), snapshot(cap), f"direct encode before replay {s}")
        ref.bpd_encode(*new)
        replay(g, stream)
        same(snapshot(ref), snapshot(cap), f"replay {s}")
        for t in range(2):
            ref.bpd_step(3)
            cap.bpd_step_static(3)                         # (its scratch is one array per GPU: not both contexts at a time)
            same(snapshot(ref), snapshot(cap), f"step {t} after replay {s}")


@pytest.mark.parametrize("dtype,d,F,eos,B", [("bf16", 128, 512, 2, 1), ("bf16", 128, 512, -1, 3), ("bf16", 192, 384, 2, 6), ("f32", 64, 256, 2, 2)])
def test_direct_calls_between_replays(dtype, d, F, eos, B):
    """Decodes and steps that are called directly find what replays have left, not what the host last knew: tokens to come, the
    sequences still in use, a block embedded ahead of time."""
    cfg = wl.Config("captured", 85, 1, 2, d, d // (64 if dtype == "bf16" else 16), F, 272, 4, B, 9, 24, dtype, eos)
    weights = wl.make_weights(cfg, std=0.1)
    stream = torch.cuda.Stream()
    ref, cap = context(cfg, weights), context(cfg, weights, stream)
    rng = np.random.default_rng(d + B)
    src = torch.zeros((B, 9), dtype=torch.int32, device="cuda")
    n = torch.full((B,), 9, dtype=torch.int32, device="cuda")
    budget = torch.from_numpy(rng.integers(9, 25, B).astype(np.int32)).cuda()
    two = torch.full((B,), 2, dtype=torch.int32, device="cuda")

    def fill():
        src.copy_(torch.from_numpy(rng.integers(3, cfg.vocab, (B, 9)).astype(np.int32)))
        torch.cuda.synchronize()

    fill()
    encode = capture(stream, lambda: cap.bpd_encode(src, n, budget))
    replay(encode, stream)
    step = capture(stream, lambda: cap.bpd_step(3, two))
    P_dev = torch.zeros((B, 4), dtype=torch.int32, device="cuda")
    proposals = capture(stream, lambda: cap.bpd_set_proposals(P_dev))

    def decode(c, sched=None):
        ids, lens, st = c.bpd_decode(3, sched)
        return [ids, lens, np.array([st.steps, st.accepted_total, st.finished])]

    for rep in range(4):
        for c in (ref, cap):                               # a whole decode: the host knows that all sequences have ended
            c.bpd_encode(src, n, budget)
        same(decode(ref), decode(cap), "direct")
        fill()
        ref.bpd_encode(src, n, budget)
        replay(encode, stream)
        for s in range(rep):                               # replayed and direct steps in turn
            ref.bpd_step(3, two)
            if s % 2:
                cap.bpd_step(3, two)
            else:
                replay(step, stream)
            same(snapshot(ref), snapshot(cap), f"step {s}, time {rep}")
        P = ref.bpd_get_state()[0]
        if rep % 2:                                        # other proposals, then a replayed step
            P = ((P + 7) % cfg.vocab).astype(np.int32)
            ref.bpd_set_proposals(P)
            if rep == 3:
                P_dev.copy_(torch.from_numpy(P))
                torch.cuda.synchronize()
                replay(proposals, stream)
            else:
                cap.bpd_set_proposals(P)
            ref.bpd_step(3, two)
            replay(step, stream)
            same(snapshot(ref), snapshot(cap), f"after new proposals, time {rep}")
        same(decode(ref), decode(cap), f"after replays, time {rep}")
        same(snapshot(ref), snapshot(cap), f"after replays, time {rep}")
