"""gss_set_assignments at the edges of its packing kernel: variable counts around a
lane's four and a wavefront's 256, rows at every alignment, slot ranges that begin and
end inside words, more words than a workgroup takes, device and host values.  Unit
clauses of both signs of every variable show both plane rows in full."""
import numpy as np
import pytest

from gpu_helpers import new_context
from paper_2012_03119_amd import gss

pytestmark = pytest.mark.gpu


def _rows(values, active, n_words):
    """Masks of the unit clauses v and -v, [2 V][n_words]: the active slots where each is F."""
    out = np.zeros((2 * values.shape[1], n_words * 64), dtype=bool)
    out[0::2, : values.shape[0]] = ((values == -1) & active[:, None]).T
    out[1::2, : values.shape[0]] = ((values == 1) & active[:, None]).T
    return np.packbits(out, axis=1, bitorder="little").view(np.uint64)


@pytest.mark.parametrize("V", [1, 3, 6, 255, 256, 257, 1031])
@pytest.mark.parametrize("slots", [64, 192, 1216])
def test_packed_rows(V, slots):
    import torch
    rng = np.random.default_rng(V * slots)
    lits = np.stack([np.arange(1, V + 1), -np.arange(1, V + 1)], axis=1).astype(np.int32).ravel()
    have = np.zeros((slots, V), np.int8)
    active = np.zeros(slots, bool)
    spans = [(0, slots), (5, slots - 9), (63, 1), (slots - 3, 3), (17, 40)] + ([(63, 66), (64, 128)] if slots > 64 else [])
    with new_context(V, slots) as ctx:
        ids = ctx.add_clauses(lits, np.arange(2 * V + 1))
        for k, (first, n) in enumerate(spans[1:] + spans[:1] + spans[1:]):
            new = rng.integers(-1, 2, (n, V)).astype(np.int8)
            print(f"pack V {V} slots {slots} first {first} n {n} {'host' if k % 3 == 0 else 'device'}", flush=True)
            if k % 3 == 0:
                ctx.set_assignments(first, new)
            else:  # at every alignment
                raw = torch.zeros(n * V + 16, dtype=torch.int8, device="cuda")
                dev = raw[k % 7: k % 7 + n * V].view(n, V)
                dev.copy_(torch.from_numpy(new))
                torch.cuda.synchronize()
                ctx.set_assignments(first, dev)
            have[first:first + n] = new
            active[first:first + n] = True
            ctx.test(gss.GSS_TEST_DENSE)
            assert np.array_equal(ctx.fetch_masks(ids), _rows(have, active, slots // 64))
        bad = torch.zeros((slots, V), dtype=torch.int8, device="cuda")
        bad[-1, -1] = 2
        with pytest.raises(gss.GssError) as e:  # applies nothing
            ctx.set_assignments(0, bad)
        assert e.value.code == gss.GSS_ERR_INVALID_ARG
        ctx.test(gss.GSS_TEST_DENSE)
        assert np.array_equal(ctx.fetch_masks(ids), _rows(have, active, slots // 64))
