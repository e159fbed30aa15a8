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


def _check_kept(ctx, want, ordered):
    """The records that fitted: fewer than all, each a real one, none twice."""
    total = int(np.count_nonzero(want))
    r = ctx.fetch_reports(total)
    assert 0 < len(r) < total
    got = reports_to_dense(r, *want.shape)
    assert np.array_equal(got[got != 0], want[got != 0])
    if ordered:
        key = r["clause_id"].astype(np.int64) * want.shape[1] + r["word"]
        assert (np.diff(key) > 0).all()


# one word a row: ordered from marked cells; eight: from the test's hit words when it fits
@pytest.mark.parametrize("slots", [64, 512])
@pytest.mark.parametrize("flags", [0, gss.GSS_TEST_SORTED])
def test_records_that_fitted_are_kept(slots, flags):
    V, n, lits, offs, vals, want = _overflowing(2, slots)
    total = int(np.count_nonzero(want))
    print(f"kept {slots} {flags}", flush=True)
    with new_context(V, slots, report_capacity=1) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        for again in (False, True):  # the second time with the grown segments: nothing is lost
            ctx.test_async(flags)
            f = sum((vals[b] == -1).astype(np.uint64) << np.uint64(b) for b in range(64))
            t = sum((vals[b] == 1).astype(np.uint64) << np.uint64(b) for b in range(64))
            ctx.update_words(0, np.arange(1, V + 1, dtype=np.uint32), f, t)
            if not again:
                with pytest.raises(gss.GssError) as e:
                    ctx.test_wait()
                assert e.value.code == gss.GSS_ERR_REPORT_OVERFLOW and ctx.stats()["last_reports"] == total
                _check_kept(ctx, want, flags)
                _check_kept(ctx, want, flags)  # fetched again
            else:
                assert ctx.test_wait() == total
                got = reports_to_dense(ctx.fetch_reports(total), n, slots // 64)
                assert np.array_equal(got, want), mismatch_summary(got, want)


@pytest.mark.parametrize("behind", ["change", "bad update before"])
def test_batch_records_that_fitted_are_kept(behind):
    """A batched test that is not repeated: a member changed behind the launch, or a
    queued update was refused."""
    import torch
    stream = torch.cuda.Stream()
    stores = []
    for i in range(2):
        V, n, lits, offs, vals, want = _overflowing(10 + i)
        ctx = new_context(V, 64, stream=stream, report_capacity=1)
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        stores.append((ctx, vals, want))
    vs = np.arange(1, 9, dtype=np.uint32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    with gss.Batch([s[0] for s in stores]) as batch:
        if behind == "change":
            batch.test_async()
            stores[0][0].set_var_values_async(0, vs, dev(stores[0][1][:, :8].T))
            code = gss.GSS_ERR_REPORT_OVERFLOW
        else:
            stores[0][0].set_var_values_async(0, vs, dev(np.full((8, 64), 3, np.int8)))
            batch.test_async()
            code = gss.GSS_ERR_INVALID_ARG
        with pytest.raises(gss.GssError) as e:
            batch.wait()
        assert e.value.code == code
        for ctx, _, want in stores:
            _check_kept(ctx, want, False)
        for ctx, c, (_, _, want) in zip([s[0] for s in stores], batch.test(), stores):
            assert int(c) == int(np.count_nonzero(want))
            got = reports_to_dense(ctx.fetch_reports(int(c)), *want.shape)
            assert np.array_equal(got, want), mismatch_summary(got, want)
    for s in stores:
        s[0].close()
