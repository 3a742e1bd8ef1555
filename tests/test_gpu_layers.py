"""All decoder layers as one kernel: a job of up to 16 rows per XCD (d = 512, d_ff = 2048), or one block of up to 16 or of 17 .. 64 rows on the whole chip (d =
1024, d_ff = 4096).  Rows and slots at their limits, long caches, whose attention several workgroups may share, groups that are not full, and sequences that end."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as wl
from harness import TOL, LockStep, gpu_context

pytestmark = pytest.mark.gpu


def config(k, B, S, out, layers=2, d=512, **kw):
    return wl.Config("layers", 75, 1, layers, d, d // 64, 4 * d, 272, k, B, S, out, "bf16", 2, src_len_kind="lognormal", **kw)


def lockstep(cfg, steps, budgets=None):
    weights = wl.make_weights(cfg)
    ctx = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    budgets = np.full(cfg.batch, cfg.max_out, np.int32) if budgets is None else budgets
    ls = LockStep(cfg, weights, ctx, src, n, budgets, sample=sorted({0, cfg.batch // 2, cfg.batch - 1}))
    for _ in range(steps):
        ls.step(imposed=np.full(cfg.batch, cfg.k, np.int32))


# (k, batch): one row; 16 rows of one sequence, of two and of three with one to spare; a last job that is not full; four slots per job
@pytest.mark.parametrize("k,B,S", [(1, 1, 1), (16, 1, 33), (16, 8, 3), (8, 16, 5), (8, 9, 40), (5, 24, 3), (4, 32, 3), (1, 27, 5), (3, 5, 140)])
def test_rows_and_slots(k, B, S):
    lockstep(config(k, B, S, 3 * k + 4), 3)


# one row, rows of one wave, of two and of three of a helper's rounds; two to four slots, which the attentions share places for from three on
@pytest.mark.parametrize("k,B,S", [(1, 1, 1), (4, 1, 33), (10, 1, 3), (16, 1, 140), (8, 2, 5), (5, 3, 40), (4, 4, 3), (1, 4, 70)])
def test_wide_rows_and_slots(k, B, S):
    lockstep(config(k, B, S, 3 * k + 4, d=1024), 3)


# two to four row tiles, one row of the second, third and fourth, all slots and rows there can be; up to four slots the attentions have members of their own,
# from nine on a member has two heads or more
@pytest.mark.parametrize("k,B,S", [(16, 3, 33), (9, 2, 5), (8, 5, 50), (11, 3, 3), (6, 8, 140), (10, 4, 20), (3, 6, 1), (5, 7, 70), (7, 7, 5), (16, 4, 40), (4, 16, 3), (2, 9, 130), (5, 11, 9)])
def test_tall_rows_and_slots(k, B, S):
    lockstep(config(k, B, S, 3 * k + 4, d=1024), 3)


# groups of fewer workgroups than places, and one that waits until its time is up; d = 1024: fewer XCDs, too
@pytest.mark.parametrize("group,k,B,d", [(1, 7, 2, 512), (5, 8, 16, 512), (31, 10, 3, 512), (33, 4, 9, 512),
                                         (5, 10, 1, 1024), (31, 4, 4, 1024), (33, 7, 2, 1024), (32 + 64 * 3, 5, 3, 1024), (3 + 64, 3, 1, 1024),
                                         (5, 10, 4, 1024), (33, 6, 8, 1024), (32 + 64 * 3, 8, 5, 1024), (3 + 64, 9, 2, 1024), (7, 4, 14, 1024)])
def test_groups(group, k, B, d, monkeypatch):
    monkeypatch.setenv("BPD_LAYERS_GROUP", str(group))
    lockstep(config(k, B, 5, 3 * k + 4, d=d), 3)


@pytest.mark.parametrize("k,B,d", [(4, 9, 512), (6, 13, 512), (4, 4, 1024), (6, 8, 1024)])
def test_ended_sequences(k, B, d):
    lockstep(config(k, B, 4, 4 * k + 1, d=d), 4, np.array([1 + (5 * b) % (4 * k + 1) for b in range(B)], np.int32))


# Blocks beyond the kernels of all layers whose cross-attention projects the queries of two sequences per workgroup: an odd sequence, one row and sixteen, one key
# and 128, sequences that end (a pair of which one or none goes on)
@pytest.mark.parametrize("k,B,S,d,ended", [(10, 9, 33, 1024, False), (16, 12, 128, 1024, False), (3, 31, 1, 1024, True), (10, 32, 64, 1024, True), (8, 17, 40, 512, False), (5, 40, 128, 512, True), (9, 64, 7, 512, True)])
def test_two_sequences_per_workgroup(k, B, S, d, ended):
    budgets = np.array([1 + (7 * (b // 2) + 3 * (b % 3)) % (4 * k) for b in range(B)], np.int32) if ended else None
    lockstep(config(k, B, S, 4 * k + 1, layers=1, d=d), 4 if ended else 2, budgets)


# ... in blocks of other kernels: LayerNorm folded into the weights of what follows (more than 640 rows, or a depth without kernels of constant K), or its statistics left behind by what goes
# before (up to 128 rows)
@pytest.mark.parametrize("k,B,S,d,F,ended", [(11, 60, 40, 512, 2048, False), (16, 41, 128, 512, 2048, True), (12, 63, 7, 512, 1024, True), (10, 20, 33, 1024, 1280, True), (4, 11, 64, 1024, 1280, False)])
def test_two_sequences_per_workgroup_of_other_blocks(k, B, S, d, F, ended):
    budgets = np.array([1 + (7 * (b // 2) + 3 * (b % 3)) % (4 * k) for b in range(B)], np.int32) if ended else None
    lockstep(dataclasses.replace(config(k, B, S, 4 * k + 1, layers=2, d=d), d_ff=F), 4 if ended else 2, budgets)


# Their queries have the bits of the separate kernels up to the rows whose LayerNorm those take inside the query projection (d = 512: 256, 1024: 32; sums in the same order): room for
# sources of 160 tokens takes the separate kernels, and states and scores are the same
@pytest.mark.parametrize("k,B,S,d,F", [(1, 17, 33, 512, 2048), (8, 20, 40, 512, 2048), (4, 64, 100, 512, 1024), (1, 32, 128, 1024, 4096), (2, 16, 64, 1024, 1024), (3, 10, 9, 1024, 2048)])
def test_two_sequences_per_workgroup_bits(k, B, S, d, F):
    cfg = wl.Config("pairs", 81, 1, 2, d, d // 64, F, 528, k, B, 160, 3 * k + 4, "bf16", 2)
    weights = wl.make_weights(cfg)
    src, n = (a[:, :S] if a.ndim > 1 else np.minimum(a, S - np.arange(B) % max(1, S // 2)).astype(np.int32) for a in wl.make_sources(cfg))
    src = np.ascontiguousarray(np.where(np.arange(S)[None, :] < n[:, None], src, cfg.pad_id)).astype(np.int32)
    seen = []
    for room in (160, S):
        w = dict(weights, pos_src=np.ascontiguousarray(weights["pos_src"][:room]))
        ctx = gpu_context(dataclasses.replace(cfg, max_src=room), w)
        ctx.bpd_encode(src, n, np.full(B, cfg.max_out, np.int32))
        seen.append([np.asarray(ctx.bpd_get_state()[0])] + [ctx.bpd_debug_step_logits(r).cpu().numpy().copy() for r in sorted({1, k})])
    for separate, pairs in zip(*seen):
        np.testing.assert_array_equal(pairs, separate)


# caches of more keys than a workgroup takes in one round, of more than 1024, which three workgroups share, two slots per job, a window.  Both ways the logits
# are within TOL of the oracle's (shown above and for the kernel chain elsewhere), so within twice that of each other.
@pytest.mark.parametrize("k,B,out,steps,local,d", [(16, 1, 400, 20, 0, 512), (10, 3, 700, 60, 0, 512), (16, 8, 1100, 66, 0, 512), (8, 16, 600, 60, 0, 512), (9, 2, 700, 70, 256, 512),
                                                   (16, 2, 300, 9, 40, 512), (16, 1, 900, 50, 0, 1024), (8, 2, 1100, 125, 0, 1024), (10, 1, 300, 25, 64, 1024), (10, 3, 700, 60, 0, 1024), (6, 8, 300, 40, 64, 1024)])
def test_long_caches(k, B, out, steps, local, d, monkeypatch):
    cfg = config(k, B, 35, out, layers=1, d=d, local_q=local, local_m=local)
    weights = wl.make_weights(cfg)
    ctx = gpu_context(cfg, weights)
    monkeypatch.setenv("BPD_LAYERS_GROUP", "0")
    ref = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    rng = np.random.default_rng(k)
    whole = torch.full((B,), k, dtype=torch.int32, device="cuda")
    for c in (ctx, ref):
        c.bpd_encode(src, n, np.full(B, out, np.int32))
    for s in range(steps):
        tok = torch.from_numpy(rng.integers(3, 272, (B, cfg.k)).astype(np.int32)).cuda()
        for c in (ctx, ref):
            c.bpd_set_proposals(tok)
            if s + 1 < steps:
                c.bpd_step(k, whole)
    a, b = (c.bpd_debug_step_logits(k).double().cpu().numpy() for c in (ctx, ref))
    assert np.isfinite(a).all() and np.abs(a - b).max() <= 2 * TOL["bf16"], np.abs(a - b).max()


@pytest.mark.parametrize("k,B,d", [(8, 8, 512), (8, 2, 1024), (8, 5, 1024)])
def test_two_streams(k, B, d):
    """Contexts on streams of their own, decoding at the same time: the workgroups of both launches share the CUs."""
    import threading
    cfg = config(k, B, 9, 60, d=d)
    weights = wl.make_weights(cfg)
    src, n = wl.make_sources(cfg)
    budgets = np.full(B, 60, np.int32)
    sched = np.random.default_rng(3).integers(1, k + 1, (60, B)).astype(np.int32)
    torch.cuda.synchronize()
    out = [None, None, None]

    def run(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            ctx = gpu_context(cfg, weights)
            for _ in range(4):
                ctx.bpd_encode(src, n, budgets)
                ids, lens, stats = ctx.bpd_decode(k, sched)
            out[i] = (np.asarray(ids).tolist(), np.asarray(lens).tolist(), stats.steps)

    run(2)
    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert out[0] == out[2] and out[1] == out[2]


# which kernels run is a matter of the source that was encoded, not of what the context has room for: the same scores to the last bit
@pytest.mark.parametrize("k,B", [(10, 1), (8, 5)])
def test_room_for_longer_sources(k, B):
    import dataclasses
    cfg = config(k, B, 20, 60, d=1024)
    weights = wl.make_weights(cfg)
    src, n = wl.make_sources(cfg)
    two = torch.full((B,), 2, dtype=torch.int32, device="cuda")
    scores = []
    for room in (20, 1100):
        pos = np.zeros((room, 1024), np.float32)
        pos[:20] = weights["pos_src"]
        ctx = gpu_context(dataclasses.replace(cfg, max_src=room), dict(weights, pos_src=pos))
        ctx.bpd_encode(src, n)
        for _ in range(3):
            ctx.bpd_step(k, two)
        scores.append(ctx.bpd_debug_step_logits(k))
    assert torch.equal(*scores)


def words_of(ctx, dtype):
    """The workspace in rows of 256 bytes, at which its arrays start."""
    start = -ctx.workspace.data_ptr() % 256
    return ctx.workspace[start:start + (ctx.workspace.numel() - start) // 256 * 256].view(dtype).view(-1, 256 // dtype.itemsize)


def cleared_context(cfg, weights, monkeypatch):
    """A context in a workspace that held nothing of an earlier one's."""
    with monkeypatch.context() as m:
        m.setattr(torch, "empty", torch.zeros)
        return gpu_context(cfg, weights)


# A wait inside a kernel that ran out leaves a word behind the counters; here the test puts it there.  Everything that hands out results says so until the next
# encode, which (recorded before, or not) and whose steps then go kernel by kernel: the scores are those of a context that always did.
@pytest.mark.parametrize("k,B,d,encodes", [(8, 3, 512, 1), (10, 1, 1024, 9), (8, 4, 1024, 1)])
def test_a_wait_that_ran_out(k, B, d, encodes, monkeypatch):
    from paper_1811_03115_amd import binding
    cfg = config(k, B, 9, 60, d=d)
    weights = wl.make_weights(cfg)
    ctx = cleared_context(cfg, weights, monkeypatch)
    monkeypatch.setenv("BPD_LAYERS_GROUP", "0")
    ref = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    two = torch.full((B,), 2, dtype=torch.int32, device="cuda")
    tok = torch.from_numpy(np.random.default_rng(k).integers(3, 272, (B, k)).astype(np.int32)).cuda()

    def scores(c):
        c.bpd_encode(src, n, np.full(B, 60, np.int32))
        for _ in range(3):
            c.bpd_set_proposals(tok)
            c.bpd_step(k, two)
        c.bpd_set_proposals(tok)
        return c.bpd_debug_step_logits(k).cpu()

    want = scores(ref)
    for _ in range(encodes):
        assert not torch.equal(scores(ctx), want)
    st = ctx.bpd_get_stats()
    counters = torch.tensor([st.seq_steps, st.accepted_total, st.finished, *st.hist, st.steps], device="cuda")
    rows = words_of(ctx, torch.int64)
    at = (rows[:, :21] == counters).all(1).nonzero().flatten()
    assert len(at) == 1
    rows[at[0], 31] = 1
    torch.cuda.synchronize()
    assert torch.isnan(ctx.bpd_debug_step_logits(k)).all()
    for call in (ctx.bpd_get_stats, ctx.bpd_get_state, ctx.bpd_get_output, lambda: ctx.bpd_decode(k), ctx.bpd_get_state):
        with pytest.raises(binding.BpdError, match="wait ran out") as e:
            call()
        assert e.value.code == -5
    assert torch.equal(scores(ctx), want)
    ctx.bpd_get_state()


# The opt-in kernel's word is one of its own, behind the map of workgroups to XCDs (1024 words, the first 256 of them round and round): told once, then it is off
def test_a_wait_of_the_stack_kernel_that_ran_out(monkeypatch):
    from paper_1811_03115_amd import binding
    monkeypatch.setenv("BPD_DECODER_STACK", "1")
    cfg = config(4, 1, 9, 20, d=128)
    ctx = cleared_context(cfg, wl.make_weights(cfg), monkeypatch)
    src, n = wl.make_sources(cfg)
    ctx.bpd_encode(src, n)
    ctx.bpd_step(4)
    ctx.bpd_get_stats()
    words = words_of(ctx, torch.int32)
    round_robin = ((words[:, :8].sort(1).values == torch.arange(8, device="cuda")).all(1) & (words[:, 8:] == words[:, :-8]).all(1)).nonzero().flatten().tolist()
    first = [r for r in round_robin if r + 3 in round_robin and r - 1 not in round_robin]
    assert len(first) == 1
    words[first[0] + 16, 0] = 7
    torch.cuda.synchronize()
    with pytest.raises(binding.BpdError, match=r"wait ran out \(code 7\)"):
        ctx.bpd_get_stats()
    ctx.bpd_get_stats()
    ctx.bpd_get_output()


# one kernel per captured step, replayed with other work of the program's between the replays: every replay finds the words that the workgroups count in cleared
@pytest.mark.parametrize("k,B,d", [(6, 5, 512), (5, 20, 512), (9, 1, 1024), (7, 4, 1024), (8, 7, 1024)])
def test_captured_steps(k, B, d):
    from test_gpu_captured import capture, context, replay, same, snapshot
    cfg = config(k, B, 9, 60, d=d)
    weights = wl.make_weights(cfg)
    stream = torch.cuda.Stream()
    ref, cap = context(cfg, weights), context(cfg, weights, stream)
    src, n = wl.make_sources(cfg)
    two = torch.full((B,), 2, dtype=torch.int32, device="cuda")
    acc = torch.zeros((2, B), dtype=torch.int32, device="cuda")
    for c in (ref, cap):
        c.bpd_encode(src, n, np.full(B, 60, np.int32))
        c.bpd_step(k, two)
    g = capture(stream, lambda: cap.bpd_step_static(k, two, acc[1]))
    same(snapshot(ref), snapshot(cap), "recorded, not run")
    for s in range(6):
        ref.bpd_step(k, two, acc[0])
        replay(g, stream)
        torch.cuda.synchronize()
        torch.randn(1 << 20, device="cuda").sum().item()
        same(snapshot(ref), snapshot(cap), f"replay {s}")
        if s == 3:                                         # a direct step in between
            ref.bpd_step(k, two)
            cap.bpd_step(k, two)
    assert acc[0].tolist() == acc[1].tolist() == [2] * B


# Steps past the end of every sequence: no row is in use.  With 98 .. 128 rows the GEMM behind the layers kernel has tiles that then end at once, and still the words that workgroups
# count in have to be cleared: the next source is decoded as by a context that has seen nothing else.
@pytest.mark.parametrize("k,B,captured", [(16, 8, False), (14, 7, False), (16, 7, True), (5, 8, False)])
def test_steps_past_the_end(k, B, captured):
    from test_gpu_captured import capture
    cfg = config(k, B, 9, 40)
    weights = wl.make_weights(cfg)
    src, n = wl.make_sources(cfg)
    other = np.where(src > 0, 271 - src, 0).astype(np.int32)
    budgets = np.full(B, 40, np.int32)
    sched = np.random.default_rng(k).integers(1, k + 1, (40, B)).astype(np.int32)

    def results(c):
        c.bpd_encode(other, n, budgets)
        first = c.bpd_get_state()[0]
        ids, lens, _ = c.bpd_decode(k, sched)
        c.bpd_encode(other, n, budgets)
        c.bpd_step(k, whole)
        return first, ids, lens, c.bpd_debug_step_logits(k).cpu().numpy()

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        whole = torch.full((B,), k, dtype=torch.int32, device="cuda")
        ctx, ref = gpu_context(cfg, weights), gpu_context(cfg, weights)
        ctx.bpd_encode(src, n, budgets)
        if captured:
            g = capture(stream, lambda: ctx.bpd_step_static(k, whole))
        else:
            ctx.bpd_decode(k, sched)
        for _ in range(6 if captured else 3):
            g.replay() if captured else ctx.bpd_step(k, whole)
            ctx.bpd_get_stats()
        assert ctx.bpd_get_state()[3].all()
        for got, want in zip(results(ctx), results(ref)):
            np.testing.assert_array_equal(got, want)


# Sources of ragged batches without their padding: lengths that the host has; with lengths on the device the encoder computes the padding, too.  A tile of 16 rows (skinny
# kernels), one sequence in more room than it needs, tiles with rows of no sequence, widths with and without kernels of constant K, more than 128 keys, more rows than those
# kernels take; widths below 512 with padding beyond those kernels, and with many places.  Both ways the logits are within TOL of the oracle's, so within twice that of each other.
@pytest.mark.parametrize("d,S,lens", [(320, 9, [1, 3, 9]), (320, 60, [5, 60, 30, 2]), (128, 40, [1, 1, 40]), (512, 140, [16, 17, 1, 33, 140]), (1024, 128, [27]),
                                      (1024, 140, [140, 100, 60, 90, 3]), (512, 48, [15 + b % 17 for b in range(33)]), (128, 40, [9 + b for b in range(17)]),
                                      (128, 96, [20 + b for b in range(44)]), (320, 60, [1 + 2 * b for b in range(28)]), (512, 21, [9, 1, 5]), (1024, 14, [10, 2, 3]), (128, 12, [3 + b % 10 for b in range(30)])])
def test_packed_sources(d, S, lens):
    B, k = len(lens), 3
    cfg = config(k, B, S, 8, layers=2, d=d)
    weights = wl.make_weights(cfg)
    rng = np.random.default_rng(d + S)
    src = rng.integers(3, 272, (B, S)).astype(np.int32)
    n = np.array(lens, np.int32)
    tok = torch.from_numpy(rng.integers(3, 272, (B, k)).astype(np.int32)).cuda()
    got = []
    ctx = gpu_context(cfg, weights)
    for lengths in (n, torch.from_numpy(n).cuda(), n):
        ctx.bpd_encode(src, lengths, np.full(B, 8, np.int32))
        ctx.bpd_set_proposals(tok)
        got.append(ctx.bpd_debug_step_logits(k).cpu().numpy())
    assert np.abs(got[0] - got[1]).max() <= 2 * TOL["bf16"]
    assert (got[0] == got[2]).all()


# Source rows without padding, several row tiles a workgroup of the encoder's attention: a last tile that is not full, a last workgroup with fewer; and so many rows that the GEMM
# of the long K takes one round of 256-column tiles (3640 and 4100 rows)
@pytest.mark.parametrize("d,batch,S", [(1024, 28, 130), (1024, 41, 100), (512, 64, 81), (512, 70, 128), (1024, 33, 49)])
def test_many_source_rows(d, batch, S):
    cfg = dataclasses.replace(config(2, batch, S, 6, layers=1, d=d), src_len_kind="fixed")
    lockstep(cfg, 1)
