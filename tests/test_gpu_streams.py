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


def _small(ctx, w):
    ctx.add_clauses(w.lits, w.offsets)
    ctx.set_assignments(0, w.values)
    n = ctx.test()
    want = ctx.fetch_reports(n)  # (staging is allocated)
    return n, want


@pytest.mark.parametrize("call", ["masks", "forward"])
def test_masks_and_forward_wait_for_the_callers_stream(call):
    """The same for mask rows, and for the network, whose features also are still
    being written when the call is made."""
    import torch
    w = gen.tiny(8)
    rng = np.random.default_rng(8)
    params = rng.standard_normal(gss.MLP_PARAMS).astype(np.float32) * 0.1
    feats = rng.random((4096, 12), dtype=np.float32)
    with gss.Context(w.n_vars, 64) as ctx:
        ids = ctx.add_clauses(w.lits, w.offsets)
        ctx.set_assignments(0, w.values)
        ctx.test(gss.GSS_TEST_DENSE)
        src = torch.from_numpy(feats).cuda()
        x = torch.zeros_like(src)
        if call == "masks":
            want, buf = ctx.fetch_masks(ids), torch.full((len(ids), 1), -7, dtype=torch.int64, device="cuda")
        else:
            want, buf = gss.gss_mlp_forward(ctx.ctx, params, feats), torch.full((4096,), -7.0, device="cuda")
        work = torch.ones(1 << 28, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        for _ in range(20):  # about 5 ms
            work.add_(1)
        x.copy_(src)
        copy = buf.clone()
        if call == "masks":
            gss.gss_fetch_masks_into(ctx.ctx, ids, buf.data_ptr())
            got = buf.cpu().numpy().view(np.uint64)
        else:
            gss.gss_mlp_forward_into(ctx.ctx, params, x.data_ptr(), 4096, buf.data_ptr())
            got = buf.cpu().numpy()
        assert bool((copy == -7).all())
        assert np.array_equal(got, want)


def test_host_output_does_not_wait_for_the_callers_stream():
    """A fetch into host memory returns while torch's current stream still runs."""
    import torch
    w = gen.tiny(4)
    with gss.Context(w.n_vars, 64) as ctx:
        n, want = _small(ctx, w)
        buf = np.empty(n, dtype=gss.REPORT_DTYPE)
        work = torch.ones(1 << 28, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        for _ in range(800):  # about 200 ms
            work.add_(1)
        assert gss.gss_fetch_reports_into(ctx.ctx, buf.ctypes.data, n) == n
        assert not torch.cuda.current_stream().query()
        assert np.array_equal(buf, want)
        torch.cuda.synchronize()


def test_device_outputs_while_the_callers_stream_is_captured():
    """Tests and fetches into device memory between the captured calls of another
    stream: that stream cannot be waited for, and the capture goes on."""
    import torch
    w = gen.tiny(5)
    with gss.Context(w.n_vars, 64) as ctx:
        n, want = _small(ctx, w)
        a = torch.full((n, 2), -7, dtype=torch.int64, device="cuda")
        b = torch.full((n, 2), -7, dtype=torch.int64, device="cuda")
        x = torch.zeros(1000, device="cuda")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, capture_error_mode="relaxed"):
            x.add_(1)
            assert gss.gss_fetch_reports_into(ctx.ctx, a.data_ptr(), n) == n
            assert ctx.test_noalloc(0, b) == n
            x.add_(1)
        for k in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert bool((x == 2 * (k + 1)).all())
        for buf in (a, b):
            assert np.array_equal(gss.sort_reports(buf.cpu().numpy().view(gss.REPORT_DTYPE).reshape(-1)),
                                  gss.sort_reports(want))


@pytest.mark.parametrize("own", [True, False])
def test_statistics_while_a_stream_is_captured(own):
    """The last test's kernel time is read when the statistics are asked for: not
    during a capture of the context's own stream, but after it; during a capture of
    another stream without disturbing that."""
    import torch
    w = gen.tiny(6)
    stream = torch.cuda.Stream()
    with gss.Context(w.n_vars, 64, stream=stream) as ctx:
        n, _ = _small(ctx, w)
        x = torch.zeros(1000, device="cuda")
        torch.cuda.synchronize()
        ctx.reset_stats()
        assert ctx.test() == n
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream if own else None, capture_error_mode="thread_local"):
            x.add_(1)
            assert ctx.stats()["last_reports"] == n
        g.replay()
        torch.cuda.synchronize()
        assert bool((x == 1).all())
        s = ctx.stats()
        assert s["timed_launches"] == 1 and s["last_kernel_ms"] > 0


def test_timed_tests_queued_while_another_stream_is_captured():
    """A test queued during the capture of another stream, with the time of the test
    before it not read yet."""
    import torch
    w = gen.tiny(7)
    with gss.Context(w.n_vars, 64) as ctx:
        n, _ = _small(ctx, w)
        x = torch.zeros(1000, device="cuda")
        torch.cuda.synchronize()
        ctx.reset_stats()
        assert ctx.test() == n
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, capture_error_mode="thread_local"):
            x.add_(1)
            ctx.test_async()
        assert ctx.test_wait() == n
        g.replay()
        torch.cuda.synchronize()
        assert bool((x == 1).all())
        assert ctx.stats()["timed_launches"] == 2
