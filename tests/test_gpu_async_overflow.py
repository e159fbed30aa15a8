"""Asynchronous tests whose report segments overflow while changes are queued behind
them: the wait does not repeat the test."""
import numpy as np
import pytest

import oracle
from gpu_helpers import mismatch_summary, new_context, reports_to_dense
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu


def _overflowing(seed, slots=64):
    """Binary clauses with far more hits than the smallest segments hold."""
    rng = np.random.default_rng(seed)
    V, n = 200, 20_000
    lits, offs = gen.random_clauses(rng, np.full(n, 2, dtype=np.int64), V)
    vals = gen.assignments_bernoulli(rng, slots, V, 0.6)
    want = oracle.masks(lits, offs, vals)
    assert int(np.count_nonzero(want)) > 16 * (n // 64 + 64) * (slots // 64)
    return V, n, lits, offs, vals, want


def test_bad_update_behind_an_overflowing_test_is_the_next_tests():
    """The update with an invalid value is queued behind the test that overflows: the
    wait reports the overflow, and the first test begun after the update reports it."""
    import torch
    V, n, lits, offs, vals, want = _overflowing(1)
    vs = np.arange(1, 9, dtype=np.uint32)
    bad = torch.full((8, 64), 3, dtype=torch.int8, device="cuda")
    with new_context(V, 64, report_capacity=1) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        ctx.test_async()
        ctx.set_var_values_async(0, vs, bad)
        with pytest.raises(gss.GssError) as e:
            ctx.test_wait()
        assert e.value.code == gss.GSS_ERR_REPORT_OVERFLOW
        assert ctx.stats()["last_reports"] == int(np.count_nonzero(want))
        with pytest.raises(gss.GssError) as e:
            ctx.test()
        assert e.value.code == gss.GSS_ERR_INVALID_ARG
        # nothing of it was applied, and it is reported once
        got = reports_to_dense(ctx.fetch_reports(ctx.test()), n, 1)
        assert np.array_equal(got, want), mismatch_summary(got, want)
