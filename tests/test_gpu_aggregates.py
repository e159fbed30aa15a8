"""Aggregate bits kept in step by every kind of update: full sets, small and large
var-major deltas (host, device, queued), packed words, the active set, cleared slots,
with renumbered variables.  After each update the tests with the aggregate pre-test, in
both modes and in either order, equal the oracle.  Every row width, one and several
chunks, a variable count that leaves the last wavefront's variables ragged."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_dense, mismatch_summary, new_context
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu

A, T = gss.GSS_TEST_AGGREGATE, gss.GSS_TEST_TRIGGER


@pytest.mark.parametrize("slots,hot", [(64, 0), (128, 0), (256, 4), (320, 0), (1024, 16), (2048, 0), (4096, 0), (4160, 0)])
def test_aggregates_follow_updates(slots, hot):
    import torch
    rng = np.random.default_rng(slots)
    V, W = 1_237, slots // 64
    lits, offs = gen.random_clauses(rng, gen.lengths_geometric(rng, 1500, 0.3, 1, 12), V)
    n = len(offs) - 1
    vals = np.concatenate([gen.assignments_table1(rng, 64, V) for _ in range(W)])
    active = np.zeros(slots, bool)

    with new_context(V, slots, hot_vars=hot) as ctx:
        ctx.add_clauses(lits, offs)

        def check(what, order):
            for mode in order:
                print(f"aggregates {slots} {what} {mode}", flush=True)
                want = oracle.masks(lits, offs, vals, active=active, mode=mode)
                got = gpu_dense(ctx, n, A | (T if mode == "trigger" else 0))
                assert np.array_equal(got, want), f"{what}: " + mismatch_summary(got, want)

        ctx.set_assignments(0, vals)
        active[:] = True
        check("full set", ("falsified", "trigger"))
        for step, k in enumerate((1, 7, 130, V, 40, 65)):
            vs = np.sort(rng.choice(V, k, replace=False)).astype(np.uint32) + 1
            first, m = (0, slots) if step % 2 == 0 else (11, min(slots - 11, 90))
            new = rng.choice(np.array([-1, 0, 0, 1], np.int8), (k, m))
            if step % 3 == 0:
                ctx.set_var_values(first, vs, new)
            elif step % 3 == 1:
                ctx.set_var_values(first, vs, torch.from_numpy(new).cuda())
            else:
                ctx.set_var_values_async(first, vs, torch.from_numpy(new).cuda())
            vals[first:first + m, vs - 1] = new.T
            check(f"delta of {k}", ("trigger", "falsified") if step % 2 else ("falsified", "trigger"))
        for w in (0, W - 1):
            vs = np.sort(rng.choice(V, 90, replace=False)).astype(np.uint32) + 1
            new = rng.choice(np.array([-1, 0, 1], np.int8), (64, 90))
            f = np.ascontiguousarray(np.packbits(new.T == -1, axis=1, bitorder="little")).view(np.uint64).ravel()
            t = np.ascontiguousarray(np.packbits(new.T == 1, axis=1, bitorder="little")).view(np.uint64).ravel()
            ctx.update_words(w, vs, f, t)
            vals[64 * w:64 * w + 64, vs - 1] = new
            check(f"word {w}", ("trigger", "falsified"))
        active[:] = rng.random(slots) < 0.7
        ctx.set_active(np.packbits(active, bitorder="little").view(np.uint64))
        check("active set", ("trigger", "falsified"))
        ctx.clear_slots(3, 50)
        vals[3:53] = 0
        active[3:53] = False
        check("cleared slots", ("falsified", "trigger"))
        # a queued delta that fails its check changes nothing
        bad = torch.full((2, slots), 3, dtype=torch.int8, device="cuda")
        active[:] = True
        ctx.set_active(np.packbits(active, bitorder="little").view(np.uint64))
        ctx.set_var_values_async(0, np.array([5, 9], np.uint32), bad)
        with pytest.raises(gss.GssError):
            ctx.test(A | T)
        check("refused delta", ("trigger", "falsified"))
