"""Device outputs against the caller's stream: a fetch into device memory writes it on
the context's stream, behind what torch's current stream still does with it."""
import numpy as np
import pytest

from paper_2012_03119_amd import gen, gss

pytestmark = pytest.mark.gpu


def test_fetch_waits_for_the_callers_stream():
    """Copies of a buffer are queued on torch's stream behind long work; the records
    fetched into that buffer arrive only after the copies have read it."""
    import torch
    w = gen.tiny(3)
    with gss.Context(w.n_vars, 64) as ctx:
        ctx.add_clauses(w.lits, w.offsets)
        ctx.set_assignments(0, w.values)
        n = ctx.test()
        buf = torch.full((n, 2), -7, dtype=torch.int64, device="cuda")
        work = torch.ones(1 << 28, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        for _ in range(20):  # about 5 ms
            work.add_(1)
        copy = buf.clone()
        assert gss.gss_fetch_reports_into(ctx.ctx, buf.data_ptr(), n) == n
        assert bool((copy == -7).all())
        got = buf.cpu().numpy().view(gss.REPORT_DTYPE).reshape(-1)
        want = ctx.fetch_reports(n)
        assert np.array_equal(got, want)
