"""Batches of unequal lengths: rows of ended sequences leave the steps (slots are dealt again by every accept kernel).
The position table says the token of each position louder than anything else, so the whole decode can be replayed on the
host whatever kernels the shrinking batch goes through."""
import numpy as np
import pytest

import workloads as wl
from harness import gpu_context

pytestmark = pytest.mark.gpu


def saying(cfg, seed):
    """Weights under which every head's arg-max at target position t is said[t]."""
    w = wl.make_weights(cfg, seed=seed)
    said = np.random.default_rng(seed).integers(3, cfg.vocab, w["pos_tgt"].shape[0]).astype(np.int32)
    w["pos_tgt"] = wl.round_bf16(w["emb"][said] * np.float32(4 * np.sqrt(cfg.d_model)))
    return w, said


def replay(said, sched, budget, steps):
    """[tokens per sequence] after at most `steps` steps."""
    out = []
    for b, n in enumerate(budget):
        got, tok = [], said[0]
        for s in range(steps):
            a = min(int(sched[s, b]), int(n) - len(got))
            if a <= 0:
                break
            got += [tok] * a
            tok = said[len(got)]
        out.append(got)
    return out


@pytest.mark.parametrize("B,d,k,two_phase,top_n", [(2, 64, 4, False, 1), (3, 128, 5, False, 1), (17, 64, 8, False, 1), (33, 128, 5, True, 1), (70, 64, 3, False, 2),
                                                    (130, 64, 2, True, 1)])
def test_ragged_batches(B, d, k, two_phase, top_n):
    cfg = wl.Config("slots", 60, 1, 2, d, d // 64, 2 * d, 528, k, B, 7, 40, "bf16", 2, src_len_kind="lognormal")
    w, said = saying(cfg, 5 + B)
    src, n = wl.make_sources(cfg)
    rng = np.random.default_rng(B)
    budget = rng.integers(1, cfg.max_out + 1, B).astype(np.int32)
    budget[0], budget[-1] = 1, cfg.max_out
    sched = rng.integers(1, k + 1, (cfg.max_out, B)).astype(np.int32)
    ctx = gpu_context(cfg, w)
    ctx.bpd_set_two_phase(two_phase)
    ctx.bpd_set_top_n(top_n)
    whole = replay(said, sched, budget, cfg.max_out)

    def check(ids, lens, expect):
        assert lens.tolist() == [len(e) for e in expect]
        for b, e in enumerate(expect):
            assert ids[b, :len(e)].tolist() == e, b

    for _ in range(2):                                     # the second decode starts from the slots the first one left
        ctx.bpd_encode(src, n, budget)
        ids, lens, st = ctx.bpd_decode(k, sched)
        check(ids, lens, whole)
        assert st.finished == B and st.accepted_total == int(budget.sum())
    # a decode in pieces, with single steps and a table of scores between them
    ctx.bpd_encode(src, n, budget)
    ctx.bpd_decode(k, sched[:3])
    for s in range(3, 6):
        acc = np.zeros(B, np.int32)
        ctx.bpd_step(k, sched[s], acc)
    P, A, j, fin = ctx.bpd_get_state()
    expect = replay(said, sched, budget, 6)
    assert j.tolist() == [len(e) for e in expect]
    assert fin.tolist() == [int(len(e) == b) for e, b in zip(expect, budget)]
    top = ctx.bpd_debug_step_logits(k).argmax(-1).cpu().numpy()           # ended sequences are scored as well
    for b in range(B):
        assert (top[b] == said[j[b] + 1:j[b] + 1 + k, None]).all(), b
    ids, lens, st = ctx.bpd_decode(k, sched[6:])
    check(ids, lens, whole)
    assert st.finished == B


@pytest.mark.parametrize("B,k", [(6, 4), (9, 2), (5, 5)])
def test_two_phase_table_when_few_sequences_are_left(B, k):
    """The table of two-phase scoring is column 1 and row k-hat, all else -1, for every batch of more than 16 block rows: also in
    steps that sequences have left until the live ones have 16 rows or fewer."""
    cfg = wl.Config("slots", 61, 1, 2, 128, 2, 512, 528, k, B, 7, 40, "bf16", 2, src_len_kind="lognormal")
    w, said = saying(cfg, B)
    src, n = wl.make_sources(cfg)
    budget = np.array([4 + 6 * b for b in range(B)], np.int32).clip(1, cfg.max_out)
    sched = np.random.default_rng(B).integers(1, k + 1, (cfg.max_out, B)).astype(np.int32)
    ctx = gpu_context(cfg, w)
    ctx.bpd_set_two_phase(True)
    steps = 0
    ctx.bpd_encode(src, n, budget)
    while steps < cfg.max_out:
        ctx.bpd_decode(k, sched[steps:steps + 3])
        steps += 3
        P, A, j, fin = ctx.bpd_get_state()
        for b in range(B):
            rows = [r for r in range(k) if (A[b, r, 1:k] >= 0).all()]
            assert len(rows) == 1, (steps, b, A[b])
            assert (A[b, :k, 0] >= 0).all() and (np.delete(A[b, :k, 1:k], rows[0], 0) == -1).all(), (steps, b, A[b])
            assert P[b, :k].tolist() == A[b, rows[0], :k].tolist()
        if fin.all():
            break
    assert fin.all()
