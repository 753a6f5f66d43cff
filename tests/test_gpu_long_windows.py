"""Windows at the edges of the longer analyses: batches of more windows than
compute units (those of up to 32768 tokens two to a unit, the rest after them),
token ranks by radix sort, and single windows whose stages are separate kernels
(first sort by several tokens at once, large units split by one workgroup or
many).  Rows against the oracle, active suffix counts against its rounds."""
import numpy as np
import pytest

import oracle
from paper_2406_18111_amd import synth

pytestmark = pytest.mark.gpu


def _rows(r):
    return np.stack([r["row_start"], r["row_len"], r["row_count"]], 1).astype(np.int64).reshape(-1, 3)


def _as3(rows):
    return np.stack([rows[k] for k in rows.dtype.names], 1).astype(np.int64).reshape(-1, 3)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_18111_amd import Context
    c = Context(0)
    yield c
    c.close()


def _active(t):
    return int(oracle.suffix_array(t, return_active=True)[1].sum()) if len(t) > 1 else 0


def _distinct(rng, n, d):
    """n tokens, d distinct."""
    return np.concatenate([rng.permutation(d), rng.integers(0, d, n - d)]).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)


def test_large_batch(ctx):
    rng = np.random.default_rng(11)
    low = rng.integers(0, 2, (4, 12000)).astype(np.uint64)  # four high bytes that tie, low ones that differ
    tied = (low[0] << np.uint64(56)) | (low[1] << np.uint64(48)) | (low[2] << np.uint64(40)) | (low[3] << np.uint64(32))
    base = [synth.loop_stream(k, int(rng.integers(0, 400)), 20, 64, 0.05) for k in range(20)]
    base += [synth.loop_stream(k, n, 60, 500, 0.05) for k, n in enumerate((4096, 4097, 8193, 32767, 32768, 32769, 50000, 65536))]
    base += [_distinct(rng, n, d) for n, d in ((20000, 6144), (20000, 6145), (32768, 12000), (33000, 8193), (40000, 39000), (4097, 4097))]
    base += [tied | rng.permutation(12000).astype(np.uint64), np.full(32768, 3, np.uint64), rng.integers(0, 2, 30000).astype(np.uint64)]
    refs = [_rows(oracle.find_repeats(w, 3)) for w in base]
    active = [_active(w) for w in base]
    for times in (1, 44):  # one launch, and two (the sum of the windows keeps the chip busy long enough)
        pick = rng.permutation(np.repeat(np.arange(len(base)), times))
        toks = np.concatenate([base[k] for k in pick])
        off = np.zeros(len(pick) + 1, dtype=np.uint64)
        off[1:] = np.cumsum([len(base[k]) for k in pick])
        for graphs in (True, False):
            try:
                ctx.set_graphs(graphs)
                for rep in range(2):
                    print("times", times, "graphs", graphs, "rep", rep, flush=True)
                    rows, oo = ctx.analyze_batch(toks, off, 3)
                    rows = _as3(rows)
                    for w, k in enumerate(pick):
                        assert np.array_equal(rows[int(oo[w]):int(oo[w + 1])], refs[k]), (rep, w, len(base[k]))
                    c = ctx.counters()
                    assert c["active_sum"] - len(toks) == sum(active[k] for k in pick)
                    assert c["sigma"] == times * sum(len(np.unique(w)) for w in base)
            finally:
                ctx.set_graphs(True)


def test_batch_of_all_distinct_tokens(ctx):
    """65536 distinct tokens in one window: ranks that 16 bits do not hold."""
    rng = np.random.default_rng(12)
    wins = [rng.permutation(65536).astype(np.uint64), np.resize(np.arange(9, dtype=np.uint64), 5000), rng.permutation(65535).astype(np.uint64)]
    toks = np.concatenate(wins)
    off = np.array([0, 65536, 70536, 136071], dtype=np.uint64)
    rows, oo = ctx.analyze_batch(toks, off, 2)
    for w in range(3):
        assert np.array_equal(_as3(rows[int(oo[w]):int(oo[w + 1])]), _rows(oracle.find_repeats(wins[w], 2)))


@pytest.mark.parametrize("n,values", [(32769, 2), (40000, 1), (65536, 3), (65537, 15), (65537, 16), (70000, 255), (90001, 256),
                                      (131072, 65535), (131075, 16385), (140000, 70000)])
@pytest.mark.parametrize("bits", (32, 64))
def test_long_single_window(ctx, n, values, bits):
    """Alphabets around the widths at which 16, 8, 4, 2 or 1 tokens fit the
    first key, random with a run and a repeated part (units on both sides of
    what one workgroup splits)."""
    rng = np.random.default_rng(n + values)
    t = rng.integers(0, values, n).astype(np.uint64)
    t[n // 5: n // 5 + n // 9] = values - 1
    t[n // 2: n // 2 + n // 7] = t[:n // 7]
    t = t * np.uint64(0x9E3779B97F4A7C15) if bits == 64 else t.astype(np.uint32)
    rows, occ = ctx.analyze(t, 6, occurrences=True)
    ref = oracle.find_repeats(t.astype(np.uint64), 6)
    assert np.array_equal(_as3(rows), _rows(ref)) and len(occ) == int(ref["row_count"].sum())
    act = oracle.suffix_array(t.astype(np.uint64), return_active=True)[1]
    c, r = ctx.counters(), ctx.rounds()
    assert c["active_sum"] - n == int(act.sum())
    assert c["sigma"] == (len(np.unique(t)) if bits == 64 else 0)


@pytest.mark.parametrize("kind", ("runs", "period"))
def test_units_of_mostly_one_key(ctx, kind):
    """Above 2^22 tokens, where a unit of mostly one key is taken apart around
    it: runs of the smallest, a middle and the largest value (entries leave on
    either side), a loop of period 3 (the key is another group's)."""
    n = (1 << 22) + 4097
    rng = np.random.default_rng(5)
    t = rng.integers(0, 4, n).astype(np.uint32)
    if kind == "runs":
        for at, length, value in ((7, 200000, 0), (300000, n // 2, 2), (3000000, 400000, 3), (3500000, 100000, 2)):
            t[at: at + length] = value
    else:
        t[100000: 100000 + n // 2] = np.resize(np.array([1, 0, 2], np.uint32), n // 2)
        t[n - 300000:] = 1
    rows = ctx.analyze(t, 64)
    ref = oracle.find_repeats(t.astype(np.uint64), 64)
    assert np.array_equal(_as3(rows), _rows(ref))
    act = oracle.suffix_array(t.astype(np.uint64), return_active=True)[1]
    assert ctx.counters()["active_sum"] - n == int(act.sum())


@pytest.mark.parametrize("n", (1 << 20, (1 << 20) + 1, (1 << 20) + 273))
def test_block_minima_over_several_levels(ctx, n):
    """Either side of the size up to which one workgroup takes every level of
    block minima above the first: repeats from a few tokens that occur in every
    block to one half of the window, so that the walks use all levels."""
    rng = np.random.default_rng(n)
    t = rng.integers(0, 1 << 14, n).astype(np.uint32)
    t[n // 2: n // 2 + n // 3] = t[: n // 3]
    t[rng.integers(0, n - 4, 50000)[:, None] + np.arange(4)] = np.array([5, 6, 7, 8], np.uint32)
    rows = ctx.analyze(t, 3)
    ref = oracle.find_repeats(t.astype(np.uint64), 3)
    assert np.array_equal(_as3(rows), _rows(ref))


@pytest.mark.parametrize("cap", (64, 2, 3, 4, 5))
@pytest.mark.parametrize("half", (False, True))
@pytest.mark.parametrize("n", (33000, 60001, 131071))
def test_last_selection_rounds(ctx, n, half, cap):
    """Few symbols, so that some thousands of candidates stay undecided for
    several rounds: the rounds of the whole chip, those of one workgroup from 1024
    candidates on, and the round cap before, at and inside these."""
    rng = np.random.default_rng(n)
    t = rng.integers(0, 4, n).astype(np.uint32)
    if half:
        t[n // 3: n // 3 + n // 2] = 0
    ref = oracle.find_repeats(t.astype(np.uint64), 4)
    rows = ctx.analyze(t, 4)
    full = ctx.rounds()["sel_live"]
    try:
        ctx.set_selection_round_cap(cap)
        rows2 = ctx.analyze(t, 4)
        live = ctx.rounds()["sel_live"]
    finally:
        ctx.set_selection_round_cap(64)
    assert np.array_equal(_as3(rows), _rows(ref)) and np.array_equal(_as3(rows2), _rows(ref))
    assert len(full) > 3 and all(a > b for a, b in zip(full[1:], full[2:]))
    assert live[:cap] == full[:cap]


@pytest.mark.parametrize("n", (270, 777, 4095, 5000, 8192, 8193, 20011, 32768))
@pytest.mark.parametrize("period", (1, 7, 500))
@pytest.mark.parametrize("bits", (32, 64))
def test_periodic_windows(ctx, n, period, bits):
    """LCPs of up to the whole window at every position: a loop without a
    substitution, and with two that part it."""
    t = np.resize(np.random.default_rng(period).permutation(500)[:period].astype(np.uint32), n)
    parted = t.copy()
    parted[n // 3] += 1
    parted[n - n // 5] += 1
    for u in (t, parted):
        rows, occ = ctx.analyze(u.astype(np.uint64) if bits == 64 else u, 5, occurrences=True)
        ref = oracle.find_repeats(u.astype(np.uint64), 5)
        assert np.array_equal(_as3(rows), _rows(ref)) and len(occ) == int(ref["row_count"].sum())


def test_batch_of_periodic_windows(ctx):
    wins = []
    for k, n in enumerate((65536, 65535, 50001, 32769, 32768, 9000, 3000, 300, 40) * 2):
        t = np.resize(np.arange(1 + 37 * k, dtype=np.uint64), n)
        if k % 2:
            t[n // 2] = np.uint64(1 << 40)
        wins.append(t)
    off = np.zeros(len(wins) + 1, np.uint64)
    off[1:] = np.cumsum([len(t) for t in wins])
    rows, oo = ctx.analyze_batch(np.concatenate(wins), off, 5)
    for w, t in enumerate(wins):
        assert np.array_equal(_as3(rows[int(oo[w]):int(oo[w + 1])]), _rows(oracle.find_repeats(t, 5))), len(t)


@pytest.mark.parametrize("values", [12, 14, 20, 22, 28, 44, 60])
def test_repeated_calls_of_one_context(values):
    """Each round's outcome is the host's to read once the round has written it,
    whatever the calls before it left behind: a few tokens' worth of groups longer
    than a tile, whose count earlier calls report, over enough calls for the runs'
    numbers to come past a quarter of it."""
    import torch
    from paper_2406_18111_amd import Context
    t = np.random.default_rng(values).integers(0, values, 1 << 17).astype(np.uint32)
    ref = oracle.suffix_array(t.astype(np.uint64))
    dev = torch.from_numpy(t.view(np.int32)).cuda()
    with Context(0) as c:
        for call in range(10):
            sa, _ = c.suffix_array_dev(dev)
            assert np.array_equal(sa.cpu().numpy().astype(np.int64), ref), (values, call)
