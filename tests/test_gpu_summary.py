"""The summary that the test kernel's last workgroup writes: grids of one workgroup, of
fewer and more than the arrival groups, and of the whole device; run after run on the
same words; with one overflowing segment (the exact count is reported, the segments
grow, the records come whole); unordered fetches, whose offsets are made on demand."""
import numpy as np
import pytest

import oracle
from gpu_helpers import mismatch_summary, new_context, reports_to_dense
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 257, 256 * 31, 256 * 32, 256 * 33 + 1, 700_000])
def test_summary_over_grids(n):
    print(f"summary {n}", flush=True)
    rng = np.random.default_rng(n)
    V = 500
    lits, offs = gen.random_clauses(rng, rng.integers(2, 5, n), V)
    vals = gen.assignments_bernoulli(rng, 64, V, 0.5)
    want = oracle.masks(lits, offs, vals)
    hits = int(np.count_nonzero(want))
    with new_context(V, 64) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        for flags in (0, gss.GSS_TEST_AGGREGATE, gss.GSS_TEST_SORTED, gss.GSS_TEST_DENSE, 0):
            got_n = ctx.test(flags)
            assert got_n == (0 if flags & gss.GSS_TEST_DENSE else hits)
        for _ in range(2):
            got = reports_to_dense(ctx.fetch_reports(got_n), n, 1)
            assert np.array_equal(got, want), mismatch_summary(got, want)
        assert ctx.stats()["last_kernel_ms"] > 0 and ctx.stats()["timed_launches"] >= 5


def test_one_overflowing_segment():
    """All hits in one tile: a single segment overflows."""
    V, n = 300, 40_000
    lits = np.full(n, 2, np.int32)  # never F
    lits[:600] = 1                  # F in every slot; unit clauses in one class, sorted by lead: neighbouring tiles
    offs = np.arange(n + 1)
    vals = np.zeros((1024, V), np.int8)
    vals[:, 0] = -1
    vals[:, 1] = 1
    with new_context(V, 1024, report_capacity=1024) as ctx:  # 16 records a segment
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        with pytest.raises(gss.GssError) as e:
            ctx.test(gss.GSS_TEST_NO_REGROW)
        assert e.value.code == gss.GSS_ERR_REPORT_OVERFLOW and ctx.stats()["last_reports"] == 600 * 16
        assert ctx.test() == 600 * 16
        r = gss.sort_reports(ctx.fetch_reports(600 * 16))
        assert (r["clause_id"] == np.repeat(np.arange(600), 16)).all() and (r["mask"] == 2**64 - 1).all()
        assert ctx.test() == 600 * 16  # the words were reset
