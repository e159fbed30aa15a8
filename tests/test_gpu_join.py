"""Long clauses that stay live: the wavefront joins them, its lane groups taking
different literals.  Clauses of lengths around the steps of every lane-group count,
falsified in one slot, falsified but for their last literal, or with one Undef
literal, among short ones; every row width, both modes, with and without early exit,
through the plain, the scheduled and the batched kernel.  Masks are exact."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_dense, mismatch_summary, new_context, reports_to_dense
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu

LENGTHS = (13, 14, 16, 17, 20, 28, 29, 32, 33, 44, 64, 65, 76, 77, 129, 300, 513, 1100)


def _workload(slots, seed):
    rng = np.random.default_rng(seed)
    V = 3_000
    vals = gen.assignments_bernoulli(rng, slots, V, 0.8)
    clauses = [rng.choice(V, size=int(n), replace=False) + 1 for n in rng.integers(2, 9, 1500)]
    clauses = [c * rng.choice([-1, 1], c.size) for c in clauses]
    for n in LENGTHS:
        for kind in ("hit", "hit", "last", "undef", "undef2"):
            row = vals[rng.integers(0, slots)]
            pick = rng.permutation(np.flatnonzero(row))[:n]
            lits = -(pick + 1) * row[pick].astype(np.int64)
            if kind == "last":
                lits[-1] = -lits[-1]
            elif kind != "hit":  # one or two literals Undef in that slot, anywhere
                free = rng.permutation(np.flatnonzero(row == 0))[: 1 if kind == "undef" else 2]
                lits[rng.permutation(n)[: free.size]] = free + 1
            clauses.append(lits)
    order = rng.permutation(len(clauses))
    clauses = [clauses[i] for i in order]
    offs = np.concatenate([[0], np.cumsum([len(c) for c in clauses])]).astype(np.int64)
    return V, np.concatenate(clauses).astype(np.int32), offs, vals


@pytest.mark.parametrize("slots", [64, 128, 192, 512, 1024, 2048, 4096, 4160])
def test_long_survivors(slots):
    V, lits, offs, vals = _workload(slots, slots)
    n = len(offs) - 1
    with new_context(V, slots) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        for mode, flag in (("falsified", 0), ("trigger", gss.GSS_TEST_TRIGGER)):
            want = oracle.masks(lits, offs, vals, mode=mode)
            for extra in (0, gss.GSS_TEST_NO_EARLY_EXIT, gss.GSS_TEST_COUNT):
                print(f"join {slots} {mode} {extra}", flush=True)
                got = gpu_dense(ctx, n, flag | extra)
                assert np.array_equal(got, want), mismatch_summary(got, want)
        if slots <= 4096:  # the scheduled kernel, every clause on its turn
            ctx.priority_enable()
            ctx.priority_mark(np.zeros(n, dtype=np.uint8))
            got = gpu_dense(ctx, n, gss.GSS_TEST_SCHEDULED)
            want = oracle.masks(lits, offs, vals)
            assert np.array_equal(got, want), mismatch_summary(got, want)


@pytest.mark.parametrize("mode", ["falsified", "trigger"])
def test_long_survivors_batched(mode):
    import torch
    flag = gss.GSS_TEST_TRIGGER if mode == "trigger" else 0
    stream = torch.cuda.Stream()
    stores = []
    for i, slots in enumerate((64, 128, 256, 512, 1024, 2048, 4096)):
        V, lits, offs, vals = _workload(slots, 50 + i)
        ctx = new_context(V, slots, stream=stream)
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        stores.append((ctx, lits, offs, vals))
    with gss.Batch([s[0] for s in stores]) as batch:
        counts = batch.test(flag)
        for (ctx, lits, offs, vals), c in zip(stores, counts):
            print(f"join batched {mode} {ctx.max_slots}", flush=True)
            got = reports_to_dense(ctx.fetch_reports(int(c)), len(offs) - 1, ctx.n_words)
            want = oracle.masks(lits, offs, vals, mode=mode)
            assert np.array_equal(got, want), mismatch_summary(got, want)
    for s in stores:
        s[0].close()
