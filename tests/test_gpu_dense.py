"""Dense tests after removals, additions and under a schedule: rows of removed clauses
and of clauses sitting out are zero, whatever the table held before; rows into host
and device memory, at an odd address too."""
import numpy as np
import pytest

import oracle
from gpu_helpers import mismatch_summary, new_context
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [64, 448, 1024])
def test_dense_rows_after_changes(slots):
    import torch
    rng = np.random.default_rng(slots)
    V, n = 600, 3_000
    lits, offs = gen.random_clauses(rng, rng.integers(1, 20, n), V)
    vals = gen.assignments_bernoulli(rng, slots, V, 0.8)
    want = oracle.masks(lits, offs, vals)
    W = slots // 64
    every = np.arange(n, dtype=np.uint32)
    with new_context(V, slots) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        ctx.test(gss.GSS_TEST_DENSE)
        got = ctx.fetch_masks(every)
        assert np.array_equal(got, want), mismatch_summary(got, want)
        raw = torch.zeros(n * W * 8 + 16, dtype=torch.uint8, device="cuda")
        for shift in (0, 4, 8):  # straight into the caller's memory, or through the stage
            raw.zero_()
            torch.cuda.synchronize()
            rc = gss.load_library().gss_fetch_masks(ctx.ctx, every.ctypes.data, n, raw.data_ptr() + shift)
            assert rc == gss.GSS_OK
            dev = raw[shift:shift + n * W * 8].cpu().numpy().tobytes()
            assert dev == want.tobytes()
        gone = rng.choice(n, 500, replace=False).astype(np.uint32)
        ctx.remove_clauses(gone)  # after the test: its rows are still there, and not shown
        want[gone] = 0
        assert np.array_equal(ctx.fetch_masks(every), want)
        ctx.set_assignments(0, -vals)
        want = oracle.masks(lits, offs, -vals)
        want[gone] = 0
        ctx.test(gss.GSS_TEST_DENSE)
        assert np.array_equal(ctx.fetch_masks(every), want)
        # a scheduled dense test: low clauses sit out three runs in four
        ctx.priority_enable()
        low = rng.random(n) < 0.5
        ctx.priority_mark(low.astype(np.uint8))
        run = ctx.priority_info()["run"]
        ctx.test(gss.GSS_TEST_DENSE | gss.GSS_TEST_SCHEDULED)
        want[low & ((run + every) % 4 != 0)] = 0
        assert np.array_equal(ctx.fetch_masks(every), want)
