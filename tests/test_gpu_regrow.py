"""A scheduled test whose report segments overflow: its list of slots is in another order
in each run, so that the repeat after the growth can give one wavefront more records
than any had before.  No record is lost all the same."""
import numpy as np
import pytest

from gpu_helpers import new_context
from paper_2012_03119_amd import gss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", range(3))
def test_scheduled_regrow(seed):
    rng = np.random.default_rng(seed)
    V, n, block = 64, 37 * 8192, 8192
    vals = np.ones((1024, V), dtype=np.int8)
    lits = np.ones((n, 2), dtype=np.int32)  # true everywhere
    lits[:, 1] = 2
    hits = []
    for k in range(5):  # sixteen clauses false everywhere, at one place of three blocks of slots
        for b in rng.choice(37, 3, replace=False):
            at = b * block + 1024 * k
            lits[at: at + 16] = (-1, -2)
            hits.append(at + np.arange(16))
    want = 16 * np.unique(np.concatenate(hits)).size
    print(f"scheduled regrow {seed}", flush=True)
    with new_context(V, 1024, report_capacity=1) as ctx:
        ctx.add_clauses(lits.ravel(), np.arange(0, 2 * n + 1, 2, dtype=np.int64))
        ctx.set_assignments(0, vals)
        ctx.priority_enable()
        ctx.priority_mark(np.zeros(n, dtype=np.uint8))
        assert ctx.test(gss.GSS_TEST_SCHEDULED) == want
        r = ctx.fetch_reports(want)
        assert len(r) == want and (r["mask"] == np.uint64(2**64 - 1)).all()
        assert len(np.unique(r["clause_id"].astype(np.int64) * 16 + r["word"])) == want
