"""Windows analysed by one workgroup each (alone up to 32768 tokens, in batches
up to 65536): rows, occurrences and counters against the oracle and against the
stage-by-stage analysis (set_window_greedy(False)), at the edges of the
workgroup sizes (256, 512 and 1024 threads with 4 or 8 tokens each, then arrays
in the workspace)."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2406_18111_amd import _lib, synth

pytestmark = pytest.mark.gpu

TOP = np.uint64(np.iinfo(np.uint64).max)
EDGES = (2, 3, 63, 64, 65, 255, 257, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 5000, 8191, 8192, 8193, 12345, 32767, 32768)


def _streams(n):
    rng = np.random.default_rng(n)
    some = synth.loop_stream(n, n, 37, 64, 0.05)
    with_top = some.copy()
    with_top[rng.integers(0, n, max(1, n // 9))] = TOP
    return {"loop": some, "top": with_top, "run": np.full(n, TOP), "distinct": rng.permutation(n).astype(np.uint64) << np.uint64(40),
            "binary": rng.integers(0, 2, n).astype(np.uint64), "period": np.tile(np.arange(7, dtype=np.uint64), n // 7 + 1)[:n]}


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


@pytest.mark.parametrize("n", EDGES)
def test_short_window(ctx, n):
    import torch
    for name, t in _streams(n).items():
        for m in ((1, 5) if n <= 8193 else (2,)):
            print("n", n, name, "min_len", m, flush=True)
            ref = oracle.find_repeats(t, m)
            occ_ref = np.stack([ref["occ_start"], ref["occ_len"], ref["occ_row"]], 1).astype(np.int64).reshape(-1, 3)
            rows, occ = ctx.analyze(t, m, occurrences=True)
            c, r = ctx.counters(), ctx.rounds()
            assert np.array_equal(_as3(rows), _rows(ref)) and np.array_equal(_as3(occ), occ_ref)
            d, docc = ctx.analyze_dev(torch.from_numpy(t.view(np.int64)).cuda(), m, occurrences=True)
            assert np.array_equal(d.cpu().numpy(), _as3(rows)) and np.array_equal(docc.cpu().numpy(), occ_ref)
            try:
                ctx.set_window_greedy(False)
                assert np.array_equal(ctx.analyze(t, m), rows)
                old = ctx.counters()
            finally:
                ctx.set_window_greedy(True)
            for k in ("rounds", "candidates", "candidates_dedup", "accepted", "rows", "active_sum", "sigma"):
                assert c[k] == old[k], (k, c, old)
            assert sum(r["sa_active"]) == c["active_sum"]


@pytest.mark.parametrize("n", (5, 1000, 3001, 8192, 9001, 32768))
def test_short_window_u32(ctx, n):
    import torch
    t = np.random.default_rng(n).integers(0, 4, n).astype(np.uint32) * np.uint32(0x3FFFFFFF)
    for m in (1, 3):
        ref = oracle.find_repeats(t.astype(np.uint64), m)
        assert np.array_equal(_as3(ctx.analyze(t, m)), _rows(ref))
        d, _ = ctx.analyze_dev(torch.from_numpy(t.view(np.int32)).cuda(), m)
        assert np.array_equal(d.cpu().numpy(), _rows(ref))


def test_short_window_output_sizes(ctx):
    """Too small a row or occurrence buffer reports the counts and writes nothing."""
    import torch
    lib = _lib.load()
    t, m = synth.config0()
    ref = oracle.find_repeats(t, m)
    nr, no = len(ref["row_start"]), len(ref["occ_start"])
    dev = torch.from_numpy(t.view(np.int64)).cuda()
    for cr, co, ok in ((nr, no, True), (nr - 1, no, False), (nr, no - 1, False), (0, 0, False)):
        rows = torch.full((nr + 1, 3), -7, dtype=torch.int32, device="cuda")
        occ = torch.full((no + 1, 3), -7, dtype=torch.int32, device="cuda")
        a, b = ctypes.c_uint32(0), ctypes.c_uint32(0)
        rc = lib.apo_analyze_window_dev(ctx._h, _lib._dev_ptr(dev), 64, len(t), m, _lib._dev_ptr(rows), cr, ctypes.byref(a),
                                        _lib._dev_ptr(occ), co, ctypes.byref(b), None)
        assert rc == (_lib.APO_OK if ok else _lib.APO_ERANGE) and a.value == nr and b.value == no
        assert bool((rows[cr if ok else 0:] == -7).all()) and bool((occ[co if ok else 0:] == -7).all())


@pytest.mark.parametrize("longest", (900, 2048, 4096, 8192))
def test_short_window_batch(ctx, longest):
    """Batches of short windows, empty and one-token ones among them: every
    lane and graph setting gives each window's own rows."""
    rng = np.random.default_rng(longest)
    wins = [np.zeros(0, np.uint64), np.array([5], np.uint64)]
    for k, n in enumerate([longest] + [int(x) for x in rng.integers(2, longest, 30)]):
        wins.append(list(_streams(n).values())[k % 6])
    wins.append(np.zeros(0, np.uint64))
    toks = np.concatenate(wins)
    off = np.zeros(len(wins) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([len(w) for w in wins])
    for m in (1, 6):
        refs = [_rows(oracle.find_repeats(w, m)) for w in wins]
        act = sum(int(oracle.suffix_array(w, return_active=True)[1].sum()) for w in wins if len(w) > 1)
        for lanes, graphs in ((3, True), (3, False), (1, True), (1, False)):
            print("longest", longest, "min_len", m, "lanes", lanes, "graphs", graphs, flush=True)
            try:
                ctx.set_lanes(lanes)
                ctx.set_graphs(graphs)
                for rep in range(2):
                    rows, oo = ctx.analyze_batch(toks, off, m)
                    for w in range(len(wins)):
                        assert np.array_equal(_as3(rows[int(oo[w]):int(oo[w + 1])]), refs[w]), (rep, w, len(wins[w]))
                    c = ctx.counters()
                    assert c["rows"] == len(rows) and c["active_sum"] - len(toks) == act
                    assert c["sigma"] == sum(len(np.unique(w)) for w in wins)
            finally:
                ctx.set_lanes(3)
                ctx.set_graphs(True)


def test_long_window_batch(ctx):
    """Windows of up to 65536 tokens beside short ones, at the largest sizes
    and the least and most repetitive inputs; then with a window of more
    distinct tokens than the hash table takes (8192, the largest value aside)."""
    rng = np.random.default_rng(7)
    many = synth.loop_stream(5, 20000, 300, 4096, 0.05)
    at = np.concatenate([rng.permutation(8192).astype(np.uint64), rng.integers(0, 8192, 3000).astype(np.uint64), [TOP]])
    over = np.concatenate([at, np.array([8192], np.uint64)])
    base = [synth.loop_stream(3, 65536, 211, 4096, 0.05), np.full(65536, 7, np.uint64), many, at,
            np.tile(np.arange(3, dtype=np.uint64), 22000)[:65535], rng.integers(0, 2, 40001).astype(np.uint64),
            synth.loop_stream(4, 3000, 40, 64, 0.05), np.zeros(0, np.uint64), synth.loop_stream(6, 8192, 40, 64, 0.05)]
    for wins, lanes in ((base, 3), (base, 1), (base[::-1] + [over], 3)):
        toks = np.concatenate(wins).astype(np.uint64)
        off = np.zeros(len(wins) + 1, dtype=np.uint64)
        off[1:] = np.cumsum([len(w) for w in wins])
        refs = [_rows(oracle.find_repeats(w, 4)) for w in wins]
        act = sum(int(oracle.suffix_array(w, return_active=True)[1].sum()) for w in wins if len(w) > 1)
        for graphs in (True, False):
            print("windows", [len(w) for w in wins], "lanes", lanes, "graphs", graphs, flush=True)
            try:
                ctx.set_lanes(lanes)
                ctx.set_graphs(graphs)
                for rep in range(2):
                    rows, oo = ctx.analyze_batch(toks, off, 4)
                    for w in range(len(wins)):
                        assert np.array_equal(_as3(rows[int(oo[w]):int(oo[w + 1])]), refs[w]), (rep, w, len(wins[w]))
                    assert ctx.counters()["active_sum"] - len(toks) == act
            finally:
                ctx.set_lanes(3)
                ctx.set_graphs(True)


def test_window_over_the_distinct_limit(ctx):
    """A lone window of more than 8192 distinct tokens."""
    t = np.concatenate([np.arange(8193, dtype=np.uint64) << np.uint64(33)] * 2)
    rows, occ = ctx.analyze(t, 3, occurrences=True)
    assert np.array_equal(_as3(rows), _rows(oracle.find_repeats(t, 3))) and len(occ) == 2
