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


@pytest.mark.parametrize("n,slots", [(3, 64), (63, 64), (9_000, 64), (65_535, 64), (65_600, 64), (21_846, 192), (1_000, 4_160)])
def test_ranked_order(n, slots):
    import torch
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
        dev = torch.zeros((len(want), 2), dtype=torch.int64, device="cuda")
        assert gss.gss_fetch_reports_into(ctx.ctx, dev.data_ptr(), len(want)) == len(want)
        assert (dev.cpu().numpy().view(want.dtype).reshape(-1) == want).all()


def _sparse_problem(n, n_slots, max_slots):
    """n clauses of three literals, n_slots assignments spread over the words: the
    records are one a hit."""
    rng = np.random.default_rng(5 + n_slots)
    V = 1_000
    lits = (rng.integers(1, V + 1, (n, 3)) * rng.choice([-1, 1], (n, 3))).astype(np.int32)
    offs = np.arange(0, 3 * n + 1, 3, dtype=np.int64)
    vals = gen.assignments_bernoulli(rng, n_slots, V, 0.6)
    hit = oracle.masks(lits.ravel(), offs, vals)[:, 0]  # bit k: slot k
    at = [64 * ((max_slots // 64 - 1) * k // max(1, n_slots - 1)) + 5 * k for k in range(n_slots)]
    want = [np.array([(i, s // 64, 1 << (s % 64)) for i in np.flatnonzero((hit >> np.uint64(k)) & np.uint64(1))],
                     dtype=gss.REPORT_DTYPE) for k, s in enumerate(at)]
    return V, lits, offs, vals, at, gss.sort_reports(np.concatenate(want))


def _check_sparse(V, lits, offs, vals, at, want, max_slots):
    with new_context(V, max_slots) as ctx:
        ctx.add_clauses(lits.ravel(), offs)
        for k, s in enumerate(at):
            ctx.set_assignments(s, vals[k:k + 1])
        assert ctx.test(gss.GSS_TEST_SORTED) == len(want)
        assert (ctx.fetch_reports(len(want)) == want).all()
        assert (ctx.fetch_reports(1000) == want[:1000]).all()


@pytest.mark.parametrize("n,n_slots", [(70_000, 2), (400_000, 9)])
def test_ranked_order_of_a_sparse_result(n, n_slots):
    """Few records among the cells of 64 words a clause: bit cells."""
    print(f"sparse ranked order {n} x {n_slots}", flush=True)
    p = _sparse_problem(n, n_slots, 4096)
    assert 1000 < len(p[-1]) < n * 64 // 240
    _check_sparse(*p, 4096)


@pytest.mark.parametrize("n_slots", [3, 11])
def test_radix_order(n_slots):
    """600 000 clauses x 4096 words are 2.46 G cells, beyond the ranked order's: the
    radix sort orders them (about 50 000 records: up to 32 tiles, one launch for the
    scan; about 180 000: the scan in chunks)."""
    print(f"radix order {n_slots} slots", flush=True)
    p = _sparse_problem(600_000, n_slots, 262_144)
    assert (131_072 < len(p[-1])) == (n_slots == 11)
    _check_sparse(*p, 262_144)
