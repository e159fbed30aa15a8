"""The calls whose speed this repository watches: clause tests over the range of
stores and slot counts it is used at, the updates that come between them, and the
network of the learned priority.

A case is a dict of plain values; its ``kind`` names what a program does in one
pass:

* ``plain``    a delta of some variables, the test, its ordered records (``trigger``
               tests Definition 1 in full).  With ``host`` the delta and the records
               are host arrays, as of a small caller; otherwise both stay on the GPU.
* ``words``    packed deltas of some solver threads' words, the test with the
               aggregate pre-test, its ordered records: a round of a served store.
* ``wide``     a delta on rows of more than 4096 slots and the test with the
               aggregate of aggregates.
* ``batch``    deltas of several stores and one batched test of all of them, the
               records merged into a table per store.
* ``fresh``    every assignment replaced, then the test.
* ``dense``    a delta and the test whose result is one mask row per clause.
* ``learned``  a scheduled test, its observation and the rescoring of the clauses
               that changed.
* ``churn``    new clauses in, old ones out, the test.
* ``forward``  the network's probabilities of a set of clauses.
* ``train``    a few Adam steps of the network (forward, backward, update).

Records are asked for in (clause id, word) order: the unordered list's order is
unspecified.  Clause lengths, assignment densities, deltas and Table 1 words follow
``paper_2012_03119_amd/gen.py`` and ``bench.py``.
"""
import math

import numpy as np
import torch

from paper_2012_03119_amd import gen, gss

MIX = ((0.5, 2, 10), (0.4, 11, 50), (0.1, 51, 300))  # gen.LENGTH_MIX
MEAN_LEN = 0.5 * 6 + 0.4 * 30.5 + 0.1 * 175.5
ALL = 2**64 - 1
# the eight stores of the batched benchmark: clauses, variables, slots
STORES = ((100_000, 50_000, 64), (250_000, 100_000, 128), (500_000, 200_000, 256), (1_000_000, 500_000, 512),
          (1_500_000, 750_000, 1024), (2_000_000, 1_000_000, 512), (2_500_000, 1_500_000, 256), (3_000_000, 2_000_000, 256))


def listed():
    return [
        # the smallest program: a few thousand variables, one 64-slot group, host arrays both ways
        dict(name="tiny", kind="plain", clauses=20_000, vars=2_000, slots=64, trigger=False, host=True),
        # the paper's scale: millions of clauses, 1024 assignments, 5% of the variables flipped between rounds
        dict(name="paper", kind="plain", clauses=4_000_000, vars=1_000_000, slots=1024, trigger=False, host=False),
        # Definition 1 in full on a mid-size store; 320 slots leave part of each plane row unused
        dict(name="trigger", kind="plain", clauses=1_000_000, vars=250_000, slots=320, trigger=True, host=False),
        # 32 solver threads' words of correlated assignments, an eighth of them sending a snapshot a round
        dict(name="words", kind="words", clauses=2_000_000, vars=300_000, slots=2048, trigger=False),
        # the largest slot counts: four super-groups of 64 words over a compact variable set
        dict(name="wide", kind="wide", clauses=500_000, vars=25_000, slots=16384, trigger=True),
        # uneven independent stores in one launch (the batched benchmark's, a quarter of their sizes)
        dict(name="batch", kind="batch", quarter=True, scale=0.25),
        # a solver restart: every assignment of every slot is new
        dict(name="fresh", kind="fresh", clauses=300_000, vars=250_000, slots=1024),
        # a caller that wants masks, not records; a ragged slot count and an odd store size
        dict(name="dense", kind="dense", clauses=700_001, vars=150_011, slots=448),
        # the learned schedule's round: the test of the clauses it picks, observation, rescoring
        dict(name="learned", kind="learned", clauses=2_000_000, vars=300_000, slots=1024),
        # clauses learned and clauses deleted between two runs
        dict(name="churn", kind="churn", clauses=400_000, vars=200_000, slots=512, batch=20_000),
        # scoring of a large store's features
        dict(name="forward", kind="forward", n=500_000),
        # training of the priority network on logged samples
        dict(name="train", kind="train", n=65_536, batch=1024, steps=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "plain", "words", "wide", "batch", "fresh", "dense", "learned", "churn", "forward",
                       "train"])
    if kind == "plain":
        # from the tiny store to a quarter of the paper's, odd sizes and ragged slot counts included
        n = _log(rng, 15_000, 1_000_000)
        host = n < 60_000 and rng.random() < 0.5
        return dict(kind=kind, clauses=n, vars=_log(rng, max(2_000, n // 20), max(3_000, n // 2)),
                    slots=64 * _log(rng, 1, 4 if host else 40), trigger=rng.random() < 0.3, host=host)
    if kind == "words":
        return dict(kind=kind, clauses=_log(rng, 100_000, 2_000_000), vars=_log(rng, 20_000, 300_000),
                    slots=64 * rng.randint(8, 40), trigger=rng.random() < 0.3)
    if kind == "wide":
        return dict(kind=kind, clauses=_log(rng, 50_000, 500_000), vars=_log(rng, 5_000, 25_000),
                    slots=64 * _log(rng, 70, 256), trigger=rng.random() < 0.5)
    if kind == "batch":
        return dict(kind=kind, quarter=rng.random() < 0.5, scale=round(math.exp(rng.uniform(math.log(0.02), math.log(0.25))), 4))
    if kind == "fresh":
        return dict(kind=kind, clauses=_log(rng, 30_000, 300_000), vars=_log(rng, 3_000, 250_000), slots=64 * _log(rng, 1, 16))
    if kind == "dense":
        return dict(kind=kind, clauses=_log(rng, 20_000, 700_000), vars=_log(rng, 5_000, 150_000), slots=64 * _log(rng, 1, 16))
    if kind == "learned":
        return dict(kind=kind, clauses=_log(rng, 100_000, 2_000_000), vars=_log(rng, 20_000, 300_000),
                    slots=64 * rng.randint(4, 16))
    if kind == "churn":
        return dict(kind=kind, clauses=_log(rng, 50_000, 400_000), vars=_log(rng, 10_000, 200_000), slots=64 * _log(rng, 1, 16),
                    batch=_log(rng, 200, 20_000))
    if kind == "forward":
        return dict(kind=kind, n=_log(rng, 1_000, 500_000))
    return dict(kind=kind, n=_log(rng, 8_192, 65_536), batch=_log(rng, 64, 4096), steps=rng.randint(4, 16))


# ---- inputs ------------------------------------------------------------------

def _clauses(g, n, n_vars):
    """Device literals and offsets of n clauses: the length mix, uniform variables and signs."""
    u = torch.rand(n, generator=g, device="cuda")
    r = torch.rand(n, generator=g, device="cuda")
    lens = torch.zeros(n, dtype=torch.int64, device="cuda")
    edge = 0.0
    for p, lo, hi in MIX:
        sel = (u >= edge) & (u < edge + p)
        lens = torch.where(sel, lo + (r * (hi - lo + 1)).long().clamp(max=hi - lo), lens)
        edge += p
    lens.clamp_(min=2)
    offs = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=offs[1:])
    total = int(offs[-1])
    lits = torch.randint(1, n_vars + 1, (total,), generator=g, device="cuda", dtype=torch.int32)
    sign = torch.randint(0, 2, (total,), generator=g, device="cuda", dtype=torch.int32)
    return lits * (2 * sign - 1), offs, lens


def _values(g, slots, n_vars):
    """Slot-major truth values: a slot's assigned fraction is uniform in [0.3, 0.9], T and F are equally likely."""
    out = torch.empty((slots, n_vars), dtype=torch.int8, device="cuda")
    for s in range(0, slots, 64):
        m = min(64, slots - s)
        half = torch.rand((m, 1), generator=g, device="cuda").mul_(0.3).add_(0.15)
        x = torch.rand((m, n_vars), generator=g, device="cuda")
        out[s:s + m] = (x < half).to(torch.int8) - (x > 1 - half).to(torch.int8)
    return out


def _plant(g, lits, offs, lens, values, n_planted):
    """Makes about n_planted clauses falsified by one slot each: their literals are redrawn among the variables
    assigned in that slot, with the signs that are F there."""
    n = offs.numel() - 1
    pick = torch.randperm(n, generator=g, device="cuda")[:n_planted]
    slot = torch.randint(0, values.shape[0], (pick.numel(),), generator=g, device="cuda")
    at = torch.repeat_interleave(torch.arange(pick.numel(), device="cuda"), lens[pick])
    first = torch.cumsum(lens[pick], 0) - lens[pick]
    pos = offs[pick][at] + (torch.arange(at.numel(), device="cuda") - first[at])
    slot = slot[at]
    var = torch.randint(0, values.shape[1], (at.numel(),), generator=g, device="cuda")
    val = values[slot, var].int()
    for _ in range(12):
        new = torch.randint(0, values.shape[1], (at.numel(),), generator=g, device="cuda")
        var = torch.where(val == 0, new, var)
        val = values[slot, var].int()
    lits[pos] = torch.where(val == 0, lits[pos], -(var.int() + 1) * val)


def _table1(rng, n):
    """F and T words of n variables in one 64-slot word: a value subset with the ratios of Table 1 each, then every
    slot a value of it."""
    p = np.cumsum([w for _, w in gen.TABLE1_SUBSETS])
    pick = np.searchsorted(p / p[-1], rng.random(n), side="right").clip(max=6)
    x = rng.integers(0, ALL, n, dtype=np.uint64, endpoint=True)
    y = rng.integers(0, ALL, n, dtype=np.uint64, endpoint=True)
    zero, ones = np.zeros(n, np.uint64), np.full(n, ALL, np.uint64)
    # the subsets in order: T, F, TF, U, TU, FU, TFU
    f = np.choose(pick, [zero, ones, x, zero, zero, x, x & ~y])
    t = np.choose(pick, [ones, zero, ~x, zero, x, zero, y & ~x])
    return f, t


def _hierarchical(rng, words, n_vars):
    """F and T words [words][n_vars]: per 64 words a Table 1 subset a variable, of which each word keeps 70%."""
    f = np.empty((words, n_vars), np.uint64)
    t = np.empty((words, n_vars), np.uint64)
    masks = np.array([sum({1: 1, -1: 2, 0: 4}[v] for v in sub) for sub, _ in gen.TABLE1_SUBSETS])
    p = np.cumsum([w for _, w in gen.TABLE1_SUBSETS])
    for w in range(words):
        if w % 64 == 0:
            base = masks[np.searchsorted(p / p[-1], rng.random(n_vars), side="right").clip(max=6)]
        r = rng.integers(0, 1000, (3, n_vars)) < 700
        mask = base & (r[0] * 1 | r[1] * 2 | r[2] * 4)
        mask = np.where(mask == 0, base & -base, mask)
        x = rng.integers(0, ALL, n_vars, dtype=np.uint64, endpoint=True)
        y = rng.integers(0, ALL, n_vars, dtype=np.uint64, endpoint=True)
        zero, ones = np.zeros(n_vars, np.uint64), np.full(n_vars, ALL, np.uint64)
        # subset masks 0..7: T = 1, F = 2, U = 4
        t[w] = np.choose(mask, [zero, ones, zero, x, zero, x, zero, y & ~x])
        f[w] = np.choose(mask, [zero, zero, ones, ~x, zero, zero, x, x & ~y])
    return f, t


def _features(rng, n):
    """Features and labels as the learned priority logs them: length, LBD, age, source, eight hit counts of which most
    are zero."""
    length = rng.integers(2, 120, n)
    x = np.zeros((n, 12), np.float32)
    x[:, 0] = np.log1p(length)
    x[:, 1] = np.log1p(2 + rng.random(n) * (length - 2))
    x[:, 2] = np.log1p(rng.integers(0, 200, n))
    x[:, 3] = rng.integers(0, 32, n) / 31
    busy = rng.random(n) < 0.3
    x[:, 4:] = np.log1p(rng.poisson(2.0, (n, 8)) * (busy[:, None] & (rng.random((n, 8)) < 0.5)))
    y = (rng.random(n) < np.where(busy, 0.6, 0.03)).astype(np.float32)
    return x, y


def _params(rng):
    p = np.zeros(5057, np.float32)
    p[:768] = rng.uniform(-1, 1, 768) * math.sqrt(6 / 12)
    p[832:4928] = rng.uniform(-1, 1, 4096) * math.sqrt(6 / 64)
    p[4992:5056] = rng.uniform(-1, 1, 64) * math.sqrt(6 / 64)
    p[768:832] = rng.uniform(-0.1, 0.1, 64)
    p[4928:4992] = rng.uniform(-0.1, 0.1, 64)
    return p


def _host(t):
    return t.cpu().numpy()


def _vars(rng, n_vars, fraction):
    k = max(1, int(round(fraction * n_vars)))
    return np.sort(rng.choice(n_vars, size=k, replace=False)).astype(np.uint32) + 1


def _store(case, g, rng, stream=None, flips=0.05):
    """A context holding the case's clauses and assignments, and two values of the delta a pass applies in turn: the
    listed variables' values flipped, and as they were."""
    n, v, s = case["clauses"], case["vars"], case["slots"]
    lits, offs, lens = _clauses(g, n, v)
    values = _values(g, s, v)
    _plant(g, lits, offs, lens, values, n // 100)
    ctx = gss.Context(v, s, stream=stream)
    ctx.add_clauses(_host(lits), _host(offs))
    ctx.set_assignments(0, values)
    vs = _vars(rng, v, flips)
    old = values[:, torch.from_numpy(vs.astype(np.int64) - 1).cuda()].t().contiguous()
    return ctx, vs, [-old, old]


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind = case["kind"]
    st = dict(case=case, turn=0)
    if kind in ("plain", "dense"):
        st["ctx"], st["vars"], st["new"] = _store(case, g, rng)
        st["ids"] = np.arange(case["clauses"], dtype=np.uint32)
        if case.get("host"):
            st["new"] = [_host(x) for x in st["new"]]
    elif kind == "fresh":
        st["ctx"], _, _ = _store(case, g, rng)
        st["values"] = [_values(g, case["slots"], case["vars"]) for _ in range(2)]
    elif kind == "words":
        n, v, words = case["clauses"], case["vars"], case["slots"] // 64
        lits, offs, _ = _clauses(g, n, v)
        ctx = gss.Context(v, case["slots"])
        ctx.add_clauses(_host(lits), _host(offs))
        every = np.arange(1, v + 1, dtype=np.uint32)
        for w in range(words):
            ctx.update_words(w, every, *_table1(rng, v))
        ctx.set_active(np.full(words, ALL, np.uint64))
        # a snapshot redraws 5% of a thread's variables, in runs of 64
        st["deltas"] = []
        for _ in range(2 * max(1, words // 8)):
            block = rng.choice((v + 63) // 64, size=max(1, v // 64 // 20), replace=False)
            vs = (np.sort(block)[:, None] * 64 + np.arange(1, 65)).ravel()
            vs = vs[vs <= v].astype(np.uint32)
            st["deltas"].append((vs, *_table1(rng, vs.size)))
        st["ctx"] = ctx
    elif kind == "wide":
        n, v, words = case["clauses"], case["vars"], case["slots"] // 64
        lits, offs, _ = _clauses(g, n, v)
        ctx = gss.Context(v, case["slots"])
        ctx.add_clauses(_host(lits), _host(offs))
        f, t = _hierarchical(rng, words, v)
        every = np.arange(1, v + 1, dtype=np.uint32)
        for w in range(words):
            ctx.update_words(w, every, f[w], t[w])
        ctx.set_active(np.full(words, ALL, np.uint64))
        vs = _vars(rng, v, 0.02)
        st["new"] = []
        for _ in range(2):  # other variables' values, slot by slot
            src = rng.permutation(v)[:vs.size]
            bits = [np.unpackbits(x[:, src].T.copy().view(np.uint8), axis=1, bitorder="little") for x in (f, t)]
            st["new"].append(torch.from_numpy(bits[1].astype(np.int8) - bits[0].astype(np.int8)).cuda())
        st["ctx"], st["vars"] = ctx, vs
    elif kind == "batch":
        stream = torch.cuda.Stream()
        st["stores"] = []
        for n, v, s in STORES if case["quarter"] else STORES[::-1]:
            # either the benchmark's stores or their sizes dealt the other way round over the slot counts
            sub = dict(clauses=max(1, int(n * case["scale"])), vars=max(300, int(v * case["scale"])),
                       slots=s if case["quarter"] else 64 * max(1, 17 - s // 64))
            ctx, vs, new = _store(sub, g, rng, stream=stream)
            st["stores"].append((sub, ctx, vs, new))
        st["batch"] = gss.Batch([x[1] for x in st["stores"]])
    elif kind == "learned":
        ctx, st["vars"], st["new"] = _store(case, g, rng)
        n = case["clauses"]
        ctx.priority_enable(n_sources=32, seed=seed)
        ids = np.arange(n, dtype=np.uint32)
        ctx.priority_set_clause_info(ids, 2 + 10 * rng.random(n).astype(np.float32), rng.integers(0, 32, n).astype(np.uint32))
        ctx.priority_score(0.0)
        st["sample"] = np.sort(rng.choice(n, size=min(n, 4096), replace=False)).astype(np.uint32)
        score = ctx.priority_fetch(st["sample"])[1]
        ctx.priority_score(float(np.quantile(score, 0.8)))  # four fifths of the clauses are low
        st["ctx"] = ctx
    elif kind == "churn":
        st["ctx"], _, _ = _store(case, g, rng)
        st["in"] = []
        for _ in range(4):
            lits, offs, _ = _clauses(g, case["batch"], case["vars"])
            st["in"].append((_host(lits), _host(offs).astype(np.uint64)))
        st["out"] = rng.permutation(case["clauses"])[:case["batch"]].astype(np.uint32)
    else:
        x, y = _features(rng, case["n"])
        st["ctx"] = gss.Context(64, 64)
        st["params"] = _params(rng)
        if kind == "forward":
            st["x"] = torch.from_numpy(x).cuda()
        else:
            st["x"], st["y"] = x, y
            st["order"] = np.concatenate([rng.permutation(case["n"]) for _ in range(1 + case["batch"] * case["steps"] // case["n"])])
            st["order"] = st["order"][:case["batch"] * case["steps"]].astype(np.uint32)
    if "clauses" in case:
        # a buffer for the records of a pass: by the clauses' hit rate, or one word in 25 on correlated words
        per = 0.04 * (case["slots"] / 64) if kind in ("words", "wide") else 1.25 * _p_hit(case["slots"], case.get("trigger", False))
        cap = min(1 << 24, 4096 + int(per * case["clauses"]))
        st["buf"] = np.zeros((cap, 2), np.int64) if case.get("host") else torch.zeros((cap, 2), dtype=torch.int64, device="cuda")
    return st


# ---- one pass ----------------------------------------------------------------

def _fetch(ctx, buf):
    """The last test's records, as many as the program's buffer holds: how many, and (clause id and word, mask) each."""
    ptr = buf.ctypes.data if isinstance(buf, np.ndarray) else buf.data_ptr()
    return dict(n=gss.gss_fetch_reports_into(ctx.ctx, ptr, buf.shape[0]), records=buf)


def run(st):
    case, turn = st["case"], st["turn"]
    kind, ctx = case["kind"], st.get("ctx")
    st["turn"] = turn + 1
    flags = gss.GSS_TEST_SORTED | (gss.GSS_TEST_TRIGGER if case.get("trigger") else 0)
    if kind == "plain" and case["host"]:
        ctx.set_var_values(0, st["vars"], st["new"][turn % 2])
        ctx.test(flags)
        return _fetch(ctx, st["buf"])
    if kind == "plain":
        ctx.set_var_values_async(0, st["vars"], st["new"][turn % 2])
        ctx.test(flags)
        return _fetch(ctx, st["buf"])
    if kind == "fresh":
        ctx.set_assignments(0, st["values"][turn % 2])
        ctx.test(flags)
        return _fetch(ctx, st["buf"])
    if kind == "dense":
        ctx.set_var_values_async(0, st["vars"], st["new"][turn % 2])
        ctx.test(gss.GSS_TEST_DENSE)
        out = torch.empty((case["clauses"], ctx.n_words), dtype=torch.int64, device="cuda")
        rc = gss.load_library().gss_fetch_masks(ctx.ctx, st["ids"].ctypes.data, st["ids"].size, out.data_ptr())
        if rc != gss.GSS_OK:
            raise gss.GssError(rc, "gss_fetch_masks")
        return out
    if kind == "words":
        words = case["slots"] // 64
        k = max(1, words // 8)
        for i in range(k):
            at = (turn * k + i) % len(st["deltas"])
            ctx.update_words((at * words // len(st["deltas"])) % words, *st["deltas"][at])
        ctx.test(flags | gss.GSS_TEST_AGGREGATE)
        return _fetch(ctx, st["buf"])
    if kind == "wide":
        ctx.set_var_values(0, st["vars"], st["new"][turn % 2])
        ctx.test(flags | gss.GSS_TEST_AGGREGATE)
        return _fetch(ctx, st["buf"])
    if kind == "batch":
        for _, c, vs, new in st["stores"]:
            c.set_var_values_async(0, vs, new[turn % 2])
        counts = st["batch"].test(gss.GSS_TEST_GRAPH)
        out = []
        for (sub, c, _, _), n in zip(st["stores"], counts):
            r = torch.empty((int(n), 2), dtype=torch.int64, device="cuda")
            gss.gss_fetch_reports_into(c.ctx, r.data_ptr(), int(n))
            key = (r[:, 0] & 0xFFFFFFFF) * c.n_words + (r[:, 0] >> 32)
            out.append(torch.zeros(sub["clauses"] * c.n_words, dtype=torch.int64, device="cuda").index_put_((key,), r[:, 1]))
        return out
    if kind == "learned":
        ctx.set_var_values_async(0, st["vars"], st["new"][turn % 2])
        ctx.test(flags | gss.GSS_TEST_SCHEDULED)
        got = _fetch(ctx, st["buf"])
        ctx.priority_observe()
        return dict(got, low=ctx.priority_update(), activity=ctx.priority_activity(st["sample"]))
    if kind == "churn":
        ids = ctx.add_clauses(*st["in"][turn % 4])
        ctx.remove_clauses(st["out"])
        st["out"] = ids
        ctx.test(flags)
        return dict(_fetch(ctx, st["buf"]), ids=ids.astype(np.int64))
    if kind == "forward":
        out = torch.empty(case["n"], dtype=torch.float32, device="cuda")
        rc = gss.load_library().gss_mlp_forward(ctx.ctx, st["params"].ctypes.data, st["x"].data_ptr(), case["n"], out.data_ptr())
        if rc != gss.GSS_OK:
            raise gss.GssError(rc, "gss_mlp_forward")
        return out
    params, losses = gss.gss_mlp_train(ctx.ctx, st["params"], st["x"], st["y"], st["order"], batch=case["batch"], lr=1e-3)
    return dict(params=params, losses=losses)


# ---- what a pass cannot do without -------------------------------------------

def _p_hit(slots, trigger=False):
    """Records a clause brings on average: words of 64 slots where it is hit, under the drawn assignments."""
    f = np.linspace(0.15, 0.45, 64)[:, None]  # probability that a literal is F in a slot
    total = 0.0
    for p, lo, hi in MIX:
        k = np.arange(lo, hi + 1)[None, :]
        hit = f ** k
        if trigger:
            hit = hit + k * f ** (k - 1) * (1 - 2 * f)
        total += p * (1 - (1 - hit.mean(0).clip(max=1)) ** 64).mean()
    return total * slots / 64


def work(case):
    kind = case["kind"]
    if kind == "forward":
        return dict(bytes=case["n"] * 52 + 5057 * 4, flops=2 * 4928 * case["n"])
    if kind == "train":
        k = case["batch"] * case["steps"]
        return dict(bytes=case["n"] * 52 + 4 * k + 2 * 5057 * 4 + 4 * case["steps"], flops=6 * 4928 * k)
    if kind == "batch":
        subs = [dict(clauses=n * case["scale"], vars=max(300, v * case["scale"]), slots=s if case["quarter"] else 64 * max(1, 17 - s // 64))
                for n, v, s in (STORES if case["quarter"] else STORES[::-1])]
    else:
        subs = [case]
    total = 0.0
    for c in subs:
        n, v, s = c["clauses"], c["vars"], c["slots"]
        total += n * (4 * MEAN_LEN + 8) + v * s / 4  # codes, metadata, both planes
        if kind == "fresh":
            total += v * s * 1.25  # the values in, the planes out
        elif kind == "words":
            total += max(1, s // 64 // 8) * v * 0.05 * 36
        elif kind == "churn":
            total += c["batch"] * (8 * MEAN_LEN + 24)
        else:
            total += v * (0.02 if kind == "wide" else 0.05) * s * 1.25
        if kind == "dense":
            total += n * s / 8
        elif kind not in ("words", "wide"):  # few records there: the clauses that fire on correlated assignments
            total += 16 * n * _p_hit(s, c.get("trigger", False))
    return dict(bytes=total, flops=0)


# ---- references --------------------------------------------------------------

def _unpack(p):
    return p[:768].reshape(12, 64), p[768:832], p[832:4928].reshape(64, 64), p[4928:4992], p[4992:5056], p[5056]


def exact(case, seed):
    """The network's outputs in 64 bits; every other kind's outputs are whole numbers (and activities, which count)."""
    if case["kind"] not in ("forward", "train"):
        return None
    rng = np.random.default_rng(seed)
    x, y = _features(rng, case["n"])
    p = _params(rng).astype(np.float64)
    if case["kind"] == "forward":
        w1, b1, w2, b2, w3, b3 = _unpack(p)
        h = np.maximum(np.maximum(x.astype(np.float64) @ w1 + b1, 0) @ w2 + b2, 0)
        return torch.from_numpy(1 / (1 + np.exp(-(h @ w3 + b3))))
    order = np.concatenate([rng.permutation(case["n"]) for _ in range(1 + case["batch"] * case["steps"] // case["n"])])
    x, y = x.astype(np.float64), y.astype(np.float64)
    lr, b1_, b2_, eps = (float(np.float32(v)) for v in (1e-3, 0.9, 0.999, 1e-8))
    m, v, losses = np.zeros(5057), np.zeros(5057), []
    for k in range(case["steps"]):
        at = order[k * case["batch"]:(k + 1) * case["batch"]]
        w1, b1, w2, b2, w3, b3 = _unpack(p)
        a, n = x[at], len(at)
        h1 = np.maximum(a @ w1 + b1, 0)
        h2 = np.maximum(h1 @ w2 + b2, 0)
        z = h2 @ w3 + b3
        losses.append((np.maximum(z, 0) + np.log1p(np.exp(-np.abs(z))) - y[at] * z).mean())
        d3 = (1 / (1 + np.exp(-z)) - y[at]) / n
        d2 = d3[:, None] * w3 * (h2 > 0)
        d1 = d2 @ w2.T * (h1 > 0)
        g = np.concatenate([(a.T @ d1).ravel(), d1.sum(0), (h1.T @ d2).ravel(), d2.sum(0), h2.T @ d3, [d3.sum()]])
        m = b1_ * m + (1 - b1_) * g
        v = b2_ * v + (1 - b2_) * g * g
        p = p - lr * (m / (1 - b1_ ** (k + 1))) / (np.sqrt(v / (1 - b2_ ** (k + 1))) + eps)
    return dict(params=p, losses=np.array(losses))
