"""Kernels and launch paths of small blocks: GEMMs with a constant K at the edges of their row and column tiles, attention at
the edges of its key groups, whole decodes in one workgroup, and steps that are recorded and replayed as graphs."""
import numpy as np
import pytest

import workloads as wl
from harness import LockStep, gpu_context

pytestmark = pytest.mark.gpu


def lockstep(cfg, steps, sched=None, std=0.02):
    weights = wl.make_weights(cfg, std=std)
    ctx = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    ls = LockStep(cfg, weights, ctx, src, n, np.full(cfg.batch, cfg.max_out, np.int32), sample=sorted({0, cfg.batch // 2, cfg.batch - 1}))
    for s in range(steps):
        ls.step(imposed=np.full(cfg.batch, cfg.k, np.int32) if sched is None else sched[s])
    return ls


# (d, F, k, batch): rows 1, 15 .. 17, 33, 127 .. 129 of each width; F = 3072 and 4096 leave K slices; 768 columns are three quarters of 1024
@pytest.mark.parametrize("d,F,k,B", [(128, 512, 1, 1), (256, 1024, 5, 3), (512, 2048, 16, 1), (512, 512, 1, 17), (768, 3072, 11, 3), (1024, 4096, 16, 2), (1024, 4096, 3, 11),
                                     (512, 2048, 1, 127), (256, 512, 8, 16), (1024, 1024, 3, 43)])
def test_row_blocks(d, F, k, B):
    cfg = wl.Config("rows", 70, 1, 2, d, d // 64, F, 272, k, B, 3, 2 * k + 4, "bf16", 2, src_len_kind="lognormal")
    lockstep(cfg, 2)


# source rows on both sides of where the encoder leaves the kernels with a constant K: 320 (beyond d = 512) and 640
@pytest.mark.parametrize("d,F,B,S", [(1024, 1024, 10, 32), (1024, 1024, 11, 30), (512, 512, 20, 32), (512, 512, 21, 31), (768, 512, 9, 36)])
def test_encoder_rows(d, F, B, S):
    cfg = wl.Config("rows", 74, 2, 1, d, d // 64, F, 272, 2, B, S, 8, "bf16", 2)
    lockstep(cfg, 1)


# encoders of more rows, whose large tiles finish whole 32 or 64 columns of a wave: lengths that are and are not multiples of 8 keys, rows past the last whole tile, columns past it
# (d = 320, 576), ragged batches
@pytest.mark.parametrize("d,F,B,S,ragged", [(512, 2048, 8, 96, False), (512, 1024, 7, 101, False), (1024, 4096, 9, 120, False), (384, 1536, 13, 56, False), (320, 1280, 9, 88, False),
                                            (576, 576, 11, 72, False), (1024, 2048, 20, 104, False), (1024, 1024, 40, 128, True), (512, 2048, 64, 128, True), (768, 1536, 48, 100, True), (1024, 2048, 64, 72, True), (640, 1280, 50, 128, True), (384, 768, 64, 128, True)])
def test_encoder_large_tiles(d, F, B, S, ragged):
    cfg = wl.Config("rows", 75, 2, 1, d, d // 64, F, 272, 2, B, S, 8, "bf16", 2, src_len_kind="lognormal" if ragged else "fixed")
    lockstep(cfg, 1)


# LayerNorm folded into weights of K = 256, which the tiles of 64 columns walk in one chunk: the row statistics that the first wave puts together are for all four.  (d_ff 640 and more
# than 640 rows: no kernels of constant K.)  Every sequence's scores
@pytest.mark.parametrize("F,k,B", [(640, 10, 60), (640, 9, 17), (1024, 13, 50)])
def test_folded_weights_of_one_chunk(F, k, B):
    cfg = wl.Config("fold", 82, 1, 2, 256, 4, F, 272, k, B, 5, 2 * k + 4, "bf16", 2, src_len_kind="lognormal")
    weights = wl.make_weights(cfg)
    ctx = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    ls = LockStep(cfg, weights, ctx, src, n, np.full(B, cfg.max_out, np.int32), sample=range(B))
    for _ in range(2):
        ls.step(imposed=np.full(B, k, np.int32))


# K slices of the encoder (F > 2048) of more source rows than the decoder ever has: up to 192 rows leave some
@pytest.mark.parametrize("d,F,B,S", [(1024, 4096, 1, 17), (1024, 4096, 4, 48), (768, 3072, 1, 70), (512, 4096, 1, 193)])
def test_encoder_slices(d, F, B, S):
    cfg = wl.Config("rows", 76, 2, 1, d, d // 64, F, 272, 1, B, S, 8, "bf16", 2)
    lockstep(cfg, 1)


# rank among vocabularies of less than a thread's first 32 floats each, exactly those, and 16 tokens more
@pytest.mark.parametrize("V,k,B", [(16, 3, 2), (272, 16, 1), (32768, 4, 2), (32784, 5, 3)])
def test_top_n_vocabularies(V, k, B):
    cfg = wl.Config("rank", 77, 1, 1, 128, 2, 512, V, k, B, 7, 4 * k + 8, "bf16", 2, src_len_kind="lognormal")
    weights = wl.make_weights(cfg)
    ctx = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    ls = LockStep(cfg, weights, ctx, src, n, np.full(B, cfg.max_out, np.int32), sample=list(range(B)))
    for top in (2, V // 3, V - 1):
        ls.step(top_n=top, check_logits=False)


# scores of head 1 out of the one pass over the vocabulary, by each of its kernels: up to 16 rows (2 and 4 heads), 18 and 100
# streamed, staged in LDS, a width of no whole 64, fp32 past the
# one-workgroup kernels
@pytest.mark.parametrize("d,V,k,B,dtype", [(512, 4112, 2, 1, "bf16"), (128, 272, 4, 1, "bf16"), (512, 20496, 3, 2, "bf16"), (1024, 16400, 5, 4, "bf16"),
                                           (512, 1040, 7, 3, "bf16"), (96, 272, 5, 2, "bf16"), (64, 5008, 3, 3, "f32")])
def test_top_n_kept_scores(d, V, k, B, dtype):
    cfg = wl.Config("kept", 78, 1, 1, d, d // (64 if d % 64 == 0 and dtype == "bf16" else 16), 2 * d, V, k, B, 7, 4 * k + 8, dtype, 2, src_len_kind="lognormal")
    weights = wl.make_weights(cfg)
    ctx = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    ls = LockStep(cfg, weights, ctx, src, n, np.full(B, cfg.max_out, np.int32), sample=list(range(B)))
    for top in (2, V // 3, V - 1):
        ls.step(top_n=top, check_logits=False)


# lengths of the caches on both sides of 32, 128 and 256 keys (a group, four waves, eight waves), sources likewise
@pytest.mark.parametrize("k,S,out", [(1, 1, 34), (7, 31, 40), (5, 33, 135), (16, 129, 150), (13, 200, 270)])
def test_key_groups(k, S, out):
    cfg = wl.Config("keys", 71, 1, 1, 128, 2, 512, 272, k, 2, S, out, "bf16", 2)
    lockstep(cfg, max(3, out // k))


# fp32, one workgroup: widths with and without a LayerNorm of its own, vocabularies of one block to more than a workgroup's columns, row
# counts past a quad, heads that do not fit LDS together
@pytest.mark.parametrize("d,F,V,k,S,L", [(32, 32, 16, 1, 1, 1), (64, 256, 272, 4, 17, 2), (96, 384, 832, 9, 33, 2), (64, 512, 1040, 16, 5, 1), (128, 512, 2000, 5, 16, 1)])
def test_small_models(d, F, V, k, S, L):
    cfg = wl.Config("small", 72, L, L, d, d // 16, F, V, k, 2, S, 3 * k + 70, "f32", 2, src_kind="uniform3", src_len_kind="lognormal")
    lockstep(cfg, 5, std=0.08)


@pytest.mark.parametrize("B,eos,local", [(1, 2, 0), (3, -1, 0), (2, -1, 40)])
def test_replayed_steps(B, eos, local):
    """Decodes and encodes on one context, over and over with other sources and schedules, against steps launched one by one."""
    cfg = wl.Config("replay", 73, 2, 2, 128, 2, 512, 272, 4, B, 9, 150, "bf16", eos, local_q=local, local_m=local)
    weights = wl.make_weights(cfg)
    ctx, ref = gpu_context(cfg, weights), gpu_context(cfg, weights)
    rng = np.random.default_rng(B)
    for rep in range(6):
        S = 9 - rep % 2
        src = rng.integers(3, cfg.vocab, (B, S)).astype(np.int32)
        n = np.full(B, S, np.int32)
        sched = rng.integers(1, cfg.k + 1, (cfg.max_out, B)).astype(np.int32) if rep != 3 else None
        eps = 1 if rep == 4 else 0
        for c in (ctx, ref):
            c.bpd_set_acceptance(eps, 1)
            c.bpd_encode(src, n)
        ids, lens, st = ctx.bpd_decode(cfg.k, sched)
        steps = 0
        while not np.all(ref.bpd_get_state()[3]):
            ref.bpd_step(cfg.k, None if sched is None else sched[steps])
            steps += 1
        ids2, lens2 = ref.bpd_get_output()
        assert lens.tolist() == lens2.tolist() and (np.asarray(ids) == np.asarray(ids2)).all()
        assert st.steps == steps
        for a, b in zip(ctx.bpd_get_state(), ref.bpd_get_state()):
            assert (np.asarray(a) == np.asarray(b)).all()


# d, F, k, S, longest output: caches past which steps go out launch by launch (about 1000 keys); sources of two tiles, which one
# workgroup encodes, and of three, which it does not; 16 rows, launch by launch from the start
@pytest.mark.parametrize("d,F,k,S,out", [(64, 256, 4, 32, 1300), (64, 256, 8, 33, 500), (32, 64, 16, 16, 120)])
def test_small_models_leave_the_one_workgroup(d, F, k, S, out):
    """Small fp32 models by the rule against launches throughout (what timing a phase makes of it): same tokens, scores to
    fp32 rounding, in steps that change over in mid-sequence and in whole decodes."""
    from paper_1811_03115_amd import binding
    from test_gpu_slots import saying
    cfg = wl.Config("small", 75, 2, 2, d, d // 16, F, 256, k, 2, S, out, "f32", -1)
    w, said = saying(cfg, 9)
    ctx, ref = gpu_context(cfg, w), gpu_context(cfg, w)
    ref.bpd_profile_enable(binding.PHASE_ACCEPT)
    src, n = wl.make_sources(cfg)
    n[-1] = max(1, S - 5)
    full = np.full(2, k, np.int32)
    for c in (ctx, ref):
        c.bpd_encode(src, n)
    for s in range((out - k) // k):
        for c in (ctx, ref):
            c.bpd_step(k, full)
        if s % 60 == 3:
            a, b = ctx.bpd_debug_step_logits(k), ref.bpd_debug_step_logits(k)
            assert float((a - b).abs().max()) <= 1e-4, s
            for u, v in zip(ctx.bpd_get_state(), ref.bpd_get_state()):
                assert (np.asarray(u) == np.asarray(v)).all(), s
    for budget in (out, 20):
        for c in (ctx, ref):
            c.bpd_encode(src, n, np.full(2, budget, np.int32))
        got, want = ctx.bpd_decode(k), ref.bpd_decode(k)
        assert got[1].tolist() == want[1].tolist() == [budget] * 2 and (got[0] == want[0]).all()
        assert got[2].steps == want[2].steps
