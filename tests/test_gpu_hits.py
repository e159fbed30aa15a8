"""The ordered fetch from the hit words that the test itself keeps, at every entry width
(rows of 5 to 64 words), in both modes and through the scheduled kernel; with gaps among
the ids and ids issued between test and fetch, after records were lost, and after the
words were given up for want of memory.  The record set and its order are exact."""
import numpy as np
import pytest

import oracle
from gpu_helpers import new_context
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu


def _check(ctx, flags, want):
    assert ctx.test(flags | gss.GSS_TEST_SORTED) == len(want)
    assert (ctx.fetch_reports(len(want)) == want).all()


@pytest.mark.parametrize("slots", [320, 512, 960, 1024, 2048, 3136, 4096])
def test_hit_words(slots):
    rng = np.random.default_rng(slots)
    row = max(8, 1 << (slots // 64 - 1).bit_length())
    V, n = 300, (1 << 18) // row + 77  # more cells than one workgroup orders
    lits, offs = gen.random_clauses(rng, rng.integers(1, 9, n), V)
    vals = gen.assignments_bernoulli(rng, slots, V, 0.7)
    more, moffs = gen.random_clauses(rng, rng.integers(1, 5, 100), V)
    gone = np.arange(0, n, 3, dtype=np.uint32)
    with new_context(V, slots) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        for mode, flag in (("falsified", 0), ("trigger", gss.GSS_TEST_TRIGGER)):
            print(f"hit words {slots} {mode}", flush=True)
            _check(ctx, flag, oracle.report_set(oracle.masks(lits, offs, vals, mode=mode)))
        masks = oracle.masks(lits, offs, vals)
        want = oracle.report_set(masks)
        assert ctx.test(gss.GSS_TEST_SORTED) == len(want)
        ctx.remove_clauses(gone)
        ctx.add_clauses(more, moffs)
        assert (ctx.fetch_reports(len(want)) == want).all()  # the test's records, not the store's
        assert (ctx.fetch_reports(77) == want[:77]).all()
        masks[gone] = 0
        masks = np.concatenate([masks, oracle.masks(more, moffs, vals)])
        _check(ctx, 0, oracle.report_set(masks))  # bits of removed clauses are cleared
        ctx.priority_enable()
        ctx.priority_mark(np.zeros(len(masks), dtype=np.uint8))
        _check(ctx, gss.GSS_TEST_SCHEDULED, oracle.report_set(masks))


def test_hit_words_after_lost_records():
    rng = np.random.default_rng(3)
    V, n, slots = 200, 40_000, 1024
    lits, offs = gen.random_clauses(rng, rng.integers(1, 4, n), V)
    vals = gen.assignments_bernoulli(rng, slots, V, 0.8)
    want = oracle.report_set(oracle.masks(lits, offs, vals))
    with new_context(V, slots, report_capacity=1) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        with pytest.raises(gss.GssError) as e:
            ctx.test(gss.GSS_TEST_SORTED | gss.GSS_TEST_NO_REGROW)
        assert e.value.code == gss.GSS_ERR_REPORT_OVERFLOW
        kept = ctx.fetch_reports(len(want))
        assert 0 < len(kept) < len(want)
        assert (kept == want[np.isin(want, kept)]).all()
        _check(ctx, 0, want)  # grows and repeats the test


def test_hit_words_given_up():
    rng = np.random.default_rng(4)
    V, n = 1_000, 200_000
    lits = (rng.integers(1, V + 1, (n, 3)) * rng.choice([-1, 1], (n, 3))).astype(np.int32).ravel()
    offs = np.arange(0, 3 * n + 1, 3, dtype=np.int64)
    vals = gen.assignments_bernoulli(rng, 1, V, 0.6)
    want = oracle.report_set(oracle.masks(lits, offs, vals))

    def filled(**kw):
        ctx = new_context(V, 4096, **kw)
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        return ctx

    with filled() as ctx:
        ctx.test()
        ctx.fetch_reports(len(want))
        ctx.priority_enable()
        full = ctx.store_info()["device_bytes"]
    with filled(hbm_budget_bytes=full + n * 8 // 2) as ctx:  # room for half the words
        ctx.test()
        ctx.fetch_reports(len(want))
        assert ctx.test(gss.GSS_TEST_SORTED) == len(want)
        ctx.priority_enable()
        assert (ctx.fetch_reports(len(want)) == want).all()
        _check(ctx, 0, want)  # without them
