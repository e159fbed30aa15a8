"""Staged rows at the 64 KiB cap, on both sides of the rule that joins long survivors
(two tiles per SIMD): every row width, both modes, ordered records, and the scheduled
kernel.  Masks are exact."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_dense, mismatch_summary, new_context
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu

LONG = (13, 17, 28, 33, 64, 65, 129, 300, 513)


def _workload(rng, n, V, vals):
    """Short clauses and a few long ones hit in one slot, or hit but for the last literal."""
    lits, offs = gen.random_clauses(rng, rng.integers(2, 9, n - 4 * len(LONG)), V)
    parts, lens = [lits], [np.diff(offs)]
    for length in LONG:
        for kind in range(4):
            row = vals[rng.integers(0, len(vals))]
            pick = rng.permutation(np.flatnonzero(row))[:length]
            c = -(pick + 1) * row[pick].astype(np.int64)
            if kind == 3:
                c[-1] = -c[-1]
            parts.append(c)
            lens.append([length])
    return np.concatenate(parts).astype(np.int32), np.concatenate([[0], np.cumsum(np.concatenate(lens))]).astype(np.int64)


@pytest.mark.parametrize("few", [True, False])
@pytest.mark.parametrize("slots", [64, 128, 256, 512, 1024, 2048, 4096])
def test_staged_at_the_cap(slots, few):
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    words = slots // 64
    per_tile = 64 if words <= 4 else 256 // words
    tiles = 20 if few else 8 * n_cu + 1
    n, V = tiles * per_tile, 2_000
    rng = np.random.default_rng(slots + few)
    vals = gen.assignments_bernoulli(rng, slots, V, 0.8)
    lits, offs = _workload(rng, n, V, vals)
    with new_context(V, slots, hot_vars=V) as ctx:  # more than fit: the cap
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        hot, stored = ctx.rank_vars()
        assert 0 < hot <= stored
        for mode, flag in (("trigger", gss.GSS_TEST_TRIGGER), ("falsified", 0)):
            want = oracle.masks(lits, offs, vals, mode=mode)
            for extra in (0, gss.GSS_TEST_SORTED):
                print(f"staged {slots} few={few} {mode} {extra}", flush=True)
                got = gpu_dense(ctx, n, flag | extra)
                assert np.array_equal(got, want), mismatch_summary(got, want)
            r = ctx.fetch_reports()
            assert (np.diff(r["clause_id"].astype(np.int64) * words + r["word"]) > 0).all()
        ctx.priority_enable()
        ctx.priority_mark(np.zeros(n, dtype=np.uint8))
        got = gpu_dense(ctx, n, gss.GSS_TEST_SCHEDULED)
        assert np.array_equal(got, want), mismatch_summary(got, want)
