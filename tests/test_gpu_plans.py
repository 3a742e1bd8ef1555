"""Encodes and steps that are recorded once they have come often enough, and replayed: every setting that they depend on has a
recording of its own, and recordings that are given up for others change nothing."""
import numpy as np
import pytest

import workloads as wl
from harness import gpu_context

pytestmark = pytest.mark.gpu


def test_settings_do_not_share_recorded_steps():
    """(distance_eps, min_block, top_n, query block, memory): each after one that a narrower key took for the same."""
    cfg = wl.Config("plans", 81, 1, 2, 128, 2, 512, 272, 4, 1, 9, 80, "bf16", -1)
    weights = wl.make_weights(cfg, std=0.12)                # tokens that depend on what is seen and accepted
    ctx, ref = gpu_context(cfg, weights), gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    settings = [(4096 * 8, 1, 1, 0, 0), (0, 1, 1, 8, 0), (4096 * 8, 1, 1, 8, 0), (0, 1, 1, 16, 0), (0, 1, 1, 8, 1), (0, 3, 1, 8, 0), (0, 1, 3, 8, 0), (0, 1, 1, 0, 0)]
    seen = {}
    for rep in range(2):
        for eps, least, top, q, mem in settings:
            for c in (ctx, ref):
                c.bpd_set_acceptance(eps, least)
                c.bpd_set_top_n(top)
                c.bpd_set_local_attention(q, mem)
                c.bpd_encode(src, n)
            ids, lens, st = ctx.bpd_decode(cfg.k)
            steps = 0
            while not ref.bpd_get_state()[3].all():
                ref.bpd_step(cfg.k)
                steps += 1
            what = f"eps {eps} min {least} top {top} local {q}, {mem}"
            assert st.steps == steps, what
            for a, b in zip([ids, lens, *ctx.bpd_get_state()], [*ref.bpd_get_output(), *ref.bpd_get_state()]):
                np.testing.assert_array_equal(a, b, err_msg=what)
            seen[what] = (ids.tobytes(), steps)
    first, second = list(seen.values())[:2]
    assert first != second and len(set(seen.values())) >= 4  # (otherwise nothing would show)


def test_more_settings_than_recordings_are_kept():
    """Recordings are given up for newer ones, and the decodes go on as before."""
    cfg = wl.Config("plans", 82, 1, 1, 128, 2, 512, 272, 4, 1, 5, 16, "bf16", -1)
    weights = wl.make_weights(cfg, std=0.12)
    ctx, ref = gpu_context(cfg, weights), gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    for rep in range(3):
        for eps in range(30):
            for c in (ctx, ref):
                c.bpd_set_acceptance(eps, 1)
                c.bpd_encode(src, n)
            ids, lens, st = ctx.bpd_decode(cfg.k)
            while not ref.bpd_get_state()[3].all():
                ref.bpd_step(cfg.k)
            for a, b in zip([ids, lens, *ctx.bpd_get_state()], [*ref.bpd_get_output(), *ref.bpd_get_state()]):
                np.testing.assert_array_equal(a, b, err_msg=f"eps {eps}, time {rep}")


def test_recorded_encodes():
    """Few source lengths often enough to be recorded, many others in between, and again; the sources are others every time.
    The reference times a phase, under which nothing is recorded."""
    from paper_1811_03115_amd import binding
    cfg = wl.Config("plans", 83, 2, 1, 128, 2, 512, 272, 4, 2, 40, 8, "bf16", 2)
    weights = wl.make_weights(cfg, std=0.12)
    ctx, ref = gpu_context(cfg, weights), gpu_context(cfg, weights)
    ref.bpd_profile_enable(binding.PHASE_ACCEPT)
    rng = np.random.default_rng(6)
    for lengths in ([3, 17, 40] * 10, range(1, 41), [3, 17, 40] * 10, [9, 10] * 9):
        for S in lengths:
            src = rng.integers(3, cfg.vocab, (2, S)).astype(np.int32)
            n = np.array([S, rng.integers(1, S + 1)], np.int32)
            for c in (ctx, ref):
                c.bpd_encode(src, n)
            for a, b in zip(ctx.bpd_get_state(), ref.bpd_get_state()):
                np.testing.assert_array_equal(a, b, err_msg=f"source length {S}")
            assert (ctx.bpd_debug_step_logits(1) == ref.bpd_debug_step_logits(1)).all(), S
