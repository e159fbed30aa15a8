"""The ordered fetch (GSS_TEST_SORTED) at the sizes where its two ways can go wrong:
cells of one word and of a rounded-up number of words, stores just below and above
a packing block, few and many records, and a store whose cells outnumber its
records so far that the radix sort takes over, with one and with several chunks of
digit counts.  The record set and its order are exact."""
import numpy as np
import pytest

import oracle
from gpu_helpers import new_context
from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,slots", [(3, 64), (63, 64), (65_535, 64), (65_600, 64), (21_846, 192), (1_000, 4_160)])
def test_ranked_order(n, slots):
    print(f"ranked order {n} clauses {slots} slots", flush=True)
    rng = np.random.default_rng(n + slots)
    V = 400
    lits, offs = gen.random_clauses(rng, rng.integers(1, 5, n), V)
    vals = gen.assignments_bernoulli(rng, slots, V, 0.5)
    masks = oracle.masks(lits, offs, vals)
    want = oracle.report_set(masks)
    with new_context(V, slots) as ctx:
        ctx.add_clauses(lits, offs)
        ctx.set_assignments(0, vals)
        assert ctx.test(gss.GSS_TEST_SORTED) == len(want)
        assert (ctx.fetch_reports(len(want)) == want).all()
        # after removals and additions the ids have gaps and grow
        gone = np.arange(0, n, 3, dtype=np.uint32)
        ctx.remove_clauses(gone)
        more, moffs = gen.random_clauses(rng, rng.integers(1, 5, 100), V)
        ctx.add_clauses(more, moffs)
        masks[gone] = 0
        want = oracle.report_set(np.concatenate([masks, oracle.masks(more, moffs, vals)]))
        assert ctx.test(gss.GSS_TEST_SORTED) == len(want)
        assert (ctx.fetch_reports(len(want)) == want).all()
        assert (ctx.fetch_reports(max(1, len(want) // 2)) == want[: max(1, len(want) // 2)]).all()


@pytest.mark.parametrize("n_slots", [1, 2])
def test_radix_order_of_a_sparse_result(n_slots):
    """3.3 M clauses x 64 words are 211 M cells: with fewer than 300 000 records the
    radix sort orders them (about 90 000 records: up to 32 tiles, one chunk or two of
    counts; about 180 000: several chunks)."""
    print(f"radix order {n_slots} slots", flush=True)
    rng = np.random.default_rng(5 + n_slots)
    V, n = 1_000, 3_300_000
    lits = (rng.integers(1, V + 1, (n, 3)) * rng.choice([-1, 1], (n, 3))).astype(np.int32)
    offs = np.arange(0, 3 * n + 1, 3, dtype=np.int64)
    vals = gen.assignments_bernoulli(rng, n_slots, V, 0.6)
    hit = oracle.masks(lits.ravel(), offs, vals)[:, 0]  # bit k: slot k
    at = [64 * (12 * k + 3) + 7 * k for k in range(n_slots)]  # one slot in each of several words
    want = [np.array([(i, s // 64, 1 << (s % 64)) for i in np.flatnonzero((hit >> np.uint64(k)) & np.uint64(1))],
                     dtype=gss.REPORT_DTYPE) for k, s in enumerate(at)]
    want = gss.sort_reports(np.concatenate(want))
    assert 131_072 * (n_slots - 1) < len(want) < 300_000 // (3 - n_slots)
    with new_context(V, 4096) as ctx:
        ctx.add_clauses(lits.ravel(), offs)
        for k, s in enumerate(at):
            ctx.set_assignments(s, vals[k:k + 1])
        assert ctx.test(gss.GSS_TEST_SORTED) == len(want)
        assert (ctx.fetch_reports(len(want)) == want).all()
        assert (ctx.fetch_reports(1000) == want[:1000]).all()
