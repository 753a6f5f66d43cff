"""The routes that a batch can take: a workgroup per window, or stage by stage where
a window is longer than 65536 tokens (in lanes, captured or host-driven).  Rows
against the oracle; what else a call reports, against what it did."""
import numpy as np
import pytest

import oracle
from paper_2406_18111_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_18111_amd import Context
    with Context(0) as c:
        yield c


def _pack(wins):
    import torch
    off = np.zeros(len(wins) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([len(w) for w in wins])
    return torch.from_numpy(np.concatenate(wins).astype(np.uint64).view(np.int64)).cuda(), off


def _refs(wins, m):
    out = []
    for w in wins:
        r = oracle.find_repeats(w, m)
        out.append(np.stack([r["row_start"], r["row_len"], r["row_count"]], 1).astype(np.int64).reshape(-1, 3))
    return out


def _check(got, refs, what=None):
    rows, off = got
    rows = rows.cpu().numpy().astype(np.int64)
    for w, ref in enumerate(refs):
        assert np.array_equal(rows[int(off[w]):int(off[w + 1])], ref), (what, w)


def _loops(lens, seed=0):
    return [synth.loop_stream(seed + k, n, 10 + 7 * k, 64, 0.05).astype(np.uint64) for k, n in enumerate(lens)]


def test_stage_times_of_a_workgroup_per_window(ctx):
    """The longest time that a window took in each stage: of the first run of a
    shape, of its replays, and of a run without graphs."""
    wins = _loops([300, 5000, 20000, 9000])
    dev, off = _pack(wins)
    refs = _refs(wins, 4)
    for graphs in (True, True, False):
        ctx.set_graphs(graphs)
        _check(ctx.analyze_batch_dev(dev, off, 4), refs)
        ms = ctx.stage_ms()
        assert all(0 < v < 100 for v in ms.values()), (graphs, ms)


def test_tuning_times_the_kernels_that_it_tunes(ctx):
    """The tile and the digit width are the stage-by-stage kernels': a tuned batch
    goes stage by stage while it is timed, whatever its windows' lengths (which a
    captured run shows by reporting no stage times), and not afterwards."""
    wins = _loops([3000, 5000, 20000, 9000])
    dev, off = _pack(wins)
    refs = _refs(wins, 4)
    for lanes in (3, 1):
        ctx.set_lanes(lanes)
        _check(ctx.analyze_batch_dev(dev, off, 4), refs)
        assert any(ctx.stage_ms().values())
        ctx.tune_batch(dev, off, 4, reps=1)
        assert not any(ctx.stage_ms().values()), lanes
        for rep in range(2):  # and no graph of the timed form is left over
            _check(ctx.analyze_batch_dev(dev, off, 4), refs)
            assert any(ctx.stage_ms().values()), (lanes, rep)


def test_a_capturing_stream_is_refused(ctx):
    """A batch reads counters on the host, which a stream that the caller is
    capturing cannot do: the call is refused before anything is enqueued, the
    caller's capture goes on, and the context keeps its graphs."""
    import torch
    from paper_2406_18111_amd import ApoError, _lib
    wins = _loops([3000, 5000, 700])
    dev, off = _pack(wins)
    refs = _refs(wins, 4)
    _check(ctx.analyze_batch_dev(dev, off, 4), refs)
    x = torch.zeros(8, device="cuda")
    s = torch.cuda.Stream()
    for lanes in (3, 1):
        ctx.set_lanes(lanes)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s, capture_error_mode="thread_local"):
            x += 1
            with pytest.raises(ApoError) as e:
                ctx.analyze_batch_dev(dev, off, 4, stream=s)
            assert e.value.code == _lib.APO_EDEVICE
        g.replay()
        g.replay()
        torch.cuda.synchronize()
    assert x.tolist() == [4.0] * 8
    before = ctx.graph_stats()["replays"]
    for _ in range(3):
        _check(ctx.analyze_batch_dev(dev, off, 4), refs)
    assert ctx.graph_stats()["replays"] >= before + 2


def test_lanes_where_one_workspace_does_not_fit(ctx):
    """A batch whose one workspace (of the next power of two tokens) finds no
    device memory is analysed in lanes, whose smaller ones do."""
    import torch
    total, lanes = 12_000_000, 3
    lens = [20000] * (total // 20000)
    base = _loops([20000] * 10)
    wins = [base[k % 10] for k in range(len(lens))]
    dev, off = _pack(wins)
    refs10 = _refs(base, 25)
    lib = ctx._lib
    one = lib.apo_workspace_bytes(total, len(wins))
    per_lane = lib.apo_workspace_bytes(1 << 22, len(wins))
    room = (one + lanes * per_lane) // 2
    assert lanes * per_lane + (1 << 30) < room < one - (1 << 30)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hog = []
    try:
        while torch.cuda.mem_get_info()[0] > room + (64 << 20):
            hog.append(torch.empty(torch.cuda.mem_get_info()[0] - room, dtype=torch.uint8, device="cuda"))
            assert len(hog) < 8
        for rep in range(2):
            got = ctx.analyze_batch_dev(dev, off, 25)
            _check(got, [refs10[k % 10] for k in range(len(wins))], rep)
    finally:
        hog.clear()
        torch.cuda.empty_cache()
    _check(ctx.analyze_batch_dev(dev, off, 25), [refs10[k % 10] for k in range(len(wins))])
    assert any(ctx.stage_ms().values())  # a workgroup per window again, now that there is room


@pytest.mark.parametrize("windows", [1, 2, 5])
def test_windows_of_65536_distinct_tokens(ctx, windows):
    """More ranks than 16 bits hold, and nothing that repeats: no rows, beside
    windows that have some, in one run (which reports its stage times)."""
    rng = np.random.default_rng(9)
    all_distinct = rng.permutation(1 << 16).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    top = all_distinct.copy()
    top[77] = np.uint64(np.iinfo(np.uint64).max)
    one_twice = all_distinct.copy()
    one_twice[40000:40003] = one_twice[100:103]
    wins = [all_distinct, one_twice, top, _loops([65536])[0], all_distinct][:windows]
    dev, off = _pack(wins)
    refs = _refs(wins, 3)
    active = sum(int(oracle.suffix_array(w, return_active=True)[1].sum()) for w in wins)
    for graphs in (True, True, False):
        ctx.set_graphs(graphs)
        _check(ctx.analyze_batch_dev(dev, off, 3), refs, graphs)
        c = ctx.counters()
        assert c["sigma"] == sum(len(np.unique(w)) for w in wins)
        assert c["active_sum"] - int(off[-1]) == active, c
        if windows > 1:
            assert any(ctx.stage_ms().values())


@pytest.mark.parametrize("windows", [4096, 4097, 8193, 150000])
def test_many_small_windows(ctx, windows):
    """Rows packed in window order for any number of windows (up to 4096 each
    finds its place on its own), and what is counted over all of them."""
    rng = np.random.default_rng(windows)
    base = _loops(rng.integers(0, 60, 40), seed=3) + [np.zeros(0, np.uint64), np.full(33, 7, np.uint64)]
    refs, sigma = _refs(base, 3), [len(np.unique(w)) for w in base]
    active = [int(oracle.suffix_array(w, return_active=True)[1].sum()) if len(w) > 1 else 0 for w in base]
    pick = rng.integers(0, len(base), windows)
    if windows == 8193:
        pick[50:-50] = len(base) - 2  # more windows than tokens
    dev, off = _pack([base[k] for k in pick])
    want = np.concatenate([refs[k] for k in pick])
    counts = np.cumsum([0] + [len(refs[k]) for k in pick])
    for graphs in (True, True, False):
        ctx.set_graphs(graphs)
        rows, oo = ctx.analyze_batch_dev(dev, off, 3)
        assert np.array_equal(oo.astype(np.int64), counts)
        assert np.array_equal(rows.cpu().numpy().astype(np.int64), want)
        c = ctx.counters()
        assert c["rows"] == len(want) and c["sigma"] == sum(sigma[k] for k in pick)
        assert c["active_sum"] - int(off[-1]) == sum(active[k] for k in pick)


def test_time_grows_with_the_number_of_windows_only(ctx):
    """Four times the windows take some four times as long (rows placed by adding up
    all counts before each window's took 12 times), the shortest of three runs each."""
    import time
    import torch
    took = []
    for windows in (500000, 2000000):
        dev = torch.tensor([1, 2, 3, 4], device="cuda").repeat(2 * windows)
        off = np.arange(windows + 1, dtype=np.uint64) * np.uint64(8)
        ts = []
        for _ in range(4):
            t0 = time.perf_counter()
            rows, oo = ctx.analyze_batch_dev(dev, off, 2)
            ts.append(time.perf_counter() - t0)
        assert np.array_equal(oo, np.arange(windows + 1)) and torch.equal(rows[:2], rows[-2:])
        assert rows[0].tolist() == [0, 4, 2]
        took.append(min(ts[1:]))
    assert took[1] < 7 * took[0], took


@pytest.mark.parametrize("longest", [4096, 4097, 8192])
def test_many_windows_beside_one_somewhat_longer(ctx, longest):
    """Windows of up to 8192 tokens share compute units in twos where they are many:
    at the edges of that form's two analyses, with as many distinct tokens as its
    table takes and one more, and beside windows of a few tokens."""
    rng = np.random.default_rng(longest)
    mix = np.uint64(0x9E3779B97F4A7C15)
    base = _loops([4095, longest - 1, longest, 300, 30, 1, 0, 2], seed=5)
    base += [np.concatenate([rng.permutation(d), rng.integers(0, d, longest - d)]).astype(np.uint64) * mix
             for d in (6144, 6145, longest) if d <= longest]
    base += [np.full(longest, 3, np.uint64), np.tile(np.arange(7, dtype=np.uint64), longest)[:longest]]
    refs = _refs(base, 2)
    pick = np.concatenate([np.repeat(np.arange(len(base)), 100), rng.integers(4, 8, 3000)])
    rng.shuffle(pick)
    dev, off = _pack([base[k] for k in pick])
    want = np.concatenate([refs[k] for k in pick])
    for rep in range(3):
        rows, oo = ctx.analyze_batch_dev(dev, off, 2)
        assert np.array_equal(oo.astype(np.int64), np.cumsum([0] + [len(refs[k]) for k in pick]))
        assert np.array_equal(rows.cpu().numpy().astype(np.int64), want), rep


@pytest.mark.parametrize("n", [25600, 25601, 32768, 65536, 65537])
def test_the_only_window_of_a_batch(ctx, n):
    """One window in a batch, and one request at a time at the server, around the
    length up to which it takes one workgroup: with and without graphs, from
    device and host tokens."""
    from paper_2406_18111_amd import Context
    rng = np.random.default_rng(n)
    wins = [_loops([n])[0], np.tile(np.arange(100, dtype=np.uint64), n // 100 + 1)[:n],
            rng.integers(0, 1 << 40, n).astype(np.uint64),
            np.concatenate([np.zeros(n // 2, np.uint64), rng.integers(0, 4, n - n // 2).astype(np.uint64)])]
    refs = [_refs([w], 8) for w in wins]
    active = [int(oracle.suffix_array(w, return_active=True)[1].sum()) for w in wins]
    for k, w in enumerate(wins):
        dev, off = _pack([w])
        for graphs in (True, True, False):
            ctx.set_graphs(graphs)
            _check(ctx.analyze_batch_dev(dev, off, 8), refs[k], k)
            c = ctx.counters()
            assert c["active_sum"] - n == active[k] and c["rows"] == len(refs[k][0]), (k, c)
            assert c["sigma"] == len(np.unique(w)), (k, c)
        rows, _ = ctx.analyze_batch(w, off, 8)
        assert np.array_equal(np.stack([rows[f] for f in rows.dtype.names], 1).astype(np.int64), refs[k][0]), k
    with Context(0) as srv:
        srv.server_start(slots=1)
        for k, w in enumerate(wins):
            ticket, got = srv.submit(w, 8), None
            while got is None:
                got = srv.fetch(ticket)
            rows = got[0]
            assert np.array_equal(np.stack([rows[f] for f in rows.dtype.names], 1).astype(np.int64), refs[k][0]), k
        srv.server_stop()


@pytest.mark.parametrize("n", [25600, 25601, 50000, 65536])
def test_few_long_windows_that_give_up_their_workgroups(ctx, n):
    """Two or three windows, one of which keeps its suffixes grouped (alone, beside
    others that would finish, and beside a short one): rows and counts whichever form
    the batch ends up in, through a graph, its replays, no graph, and the server."""
    from paper_2406_18111_amd import Context
    rng = np.random.default_rng(n)
    loop, other = _loops([n, n - 1000], seed=9)
    periodic = np.tile(np.arange(100, dtype=np.uint64), n // 100 + 1)[:n]
    run = np.concatenate([rng.integers(0, 4, n // 4), np.zeros(n // 2, np.int64), rng.integers(0, 4, n // 4)]).astype(np.uint64)
    distinct = rng.permutation(n).astype(np.uint64)
    short, none = _loops([3000])[0], np.zeros(0, np.uint64)
    batches = [[periodic, loop], [loop, run, other], [short, periodic], [none, run, none], [distinct, periodic[:-7], distinct],
               [loop, other, distinct], [np.full(n, 5, np.uint64), run]]
    for wins in batches:
        dev, off = _pack(wins)
        refs = _refs(wins, 8)
        active = sum(int(oracle.suffix_array(w, return_active=True)[1].sum()) for w in wins if len(w) > 1)
        for graphs in (True, True, True, False):
            ctx.set_graphs(graphs)
            _check(ctx.analyze_batch_dev(dev, off, 8), refs, graphs)
            c = ctx.counters()
            assert c["active_sum"] - int(off[-1]) == active and c["rows"] == sum(len(r) for r in refs), c
    with Context(0) as srv:
        srv.server_start(slots=1)
        for wins in batches:
            tickets = [srv.submit(w, 8) for w in wins]
            for ticket, ref in zip(tickets, _refs(wins, 8)):
                got = None
                while got is None:
                    got = srv.fetch(ticket)
                assert np.array_equal(np.stack([got[0][f] for f in got[0].dtype.names], 1).astype(np.int64), ref)
        srv.server_stop()


# ---- stage by stage: batches with a window of more than 65536 tokens

FORMS = [(3, False), (2, False), (1, False), (3, True), (2, True), (1, True)]  # lanes, graphs


def _long(seed=1, n=66000):
    """A window that sends its batch stage by stage: few distinct tokens and pairs."""
    return synth.loop_stream(seed, n, 40, 64, 0.05).astype(np.uint64)


def _each_form(ctx, wins, m, check=None, forms=FORMS):
    dev, off = _pack(wins)
    refs = _refs(wins, m)
    for lanes, graphs in forms:
        ctx.set_lanes(lanes)
        ctx.set_graphs(graphs)
        for rep in range(3 if graphs else 1):
            _check(ctx.analyze_batch_dev(dev, off, m), refs, (lanes, graphs, rep))
            if check:
                check(ctx.counters(), lanes)


@pytest.mark.parametrize("over", [(), (4097,), (6000, 4097)])
def test_stage_batch_window_ranks(ctx, over):
    """Windows at the bound of the per-window token ranks (4096 distinct tokens,
    the largest value aside), and over it, where the shared table ranks them."""
    from test_gpu_batch_serve import _distinct_window
    rng = np.random.default_rng(22)
    wins = [_distinct_window(rng, d, mx) for d, mx in ((1, False), (700, False), (4095, True), (4096, False), (4096, True))]
    wins += [_long()] + [_distinct_window(rng, d, True) for d in over]
    sigma = sum(len(np.unique(w)) for w in wins)

    def check(c, lanes):
        if not over:
            assert c["sigma"] == sigma
    _each_form(ctx, wins, 2, check)


@pytest.mark.parametrize("order", range(3))
def test_stage_batch_pair_ranks(ctx, order):
    """The first two doubling rounds from the windows' own pair ranks, in the lanes
    whose windows all have at most 8192 distinct adjacent pairs (picked by the host
    in host-driven lanes, on the device in sync-free ones and graphs)."""
    from test_gpu_batch_serve import _oracle_active, _pair_lane_windows, _pairs_window
    rng = np.random.default_rng(34)
    at, over = _pairs_window(rng, 8192), _pairs_window(rng, 8193)
    loops = _loops([3000, 9000, 700, 5000], seed=50)
    wins = [loops + [at, _long()], loops[:2] + [over, _long()] + loops[2:] + [at], [_long(2), over, at, _long()] + loops][order]
    active = sum(_oracle_active(w) for w in wins)
    total = sum(len(w) for w in wins)

    def check(c, lanes):
        assert c["active_sum"] - total == active
        assert c["pair_windows"] == _pair_lane_windows(wins, lanes, over), (c, lanes)
    _each_form(ctx, wins, 3, check)


@pytest.mark.parametrize("seed", [8, 9])
def test_stage_batch_random(ctx, seed):
    """Random windows around those bounds, tiny ones and the largest token value among them."""
    from test_gpu_batch_serve import _oracle_active, _pair_mix_windows
    wins = _pair_mix_windows(seed, 14)
    wins.insert(5, _long(seed))
    active, total = sum(_oracle_active(w) for w in wins), sum(len(w) for w in wins)

    def check(c, lanes):
        assert c["active_sum"] - total == active
    _each_form(ctx, wins, 3, check)


def test_stage_lanes_never_get_only_empty_windows(ctx):
    """Empty windows join a lane that has tokens: behind the long one, before it, and
    where a lane's first boundary lands past it."""
    e = np.zeros(0, np.uint64)
    heads = _loops([17, 100, 2047], seed=70)
    for wins in (heads + [_long(), e], [_long()] + [e] * 5, [e] * 3 + [_long()] + heads + [e] * 3,
                 [heads[0][:5], heads[0][:3], heads[2], heads[0][:1], heads[1], _long(), e]):
        _each_form(ctx, wins, 3)
        stats = ctx.graph_stats()
    assert stats["captures"] >= 8 and stats["replays"] >= 16  # none of them fell back to host-driven lanes


def test_stage_lane_graph_replays(ctx):
    """Three lanes as branches of one graph: replays on tokens rewritten in place,
    on other window boundaries of the same shape, with eager work in between."""
    import torch
    ctx.set_lanes(3)
    lens_a, lens_b = [70100, 100, 66000, 4200, 69000, 1200], [100, 70100, 4200, 66000, 1200, 69000]
    a, b = _loops(lens_a, seed=80), _loops(lens_b, seed=90)
    dev, off_a = _pack(a)
    _, off_b = _pack(b)
    refs = [_refs(w, 4) for w in (a, b)]
    eager = _refs(a[3:4], 4)[0]
    for rep, which in enumerate((0, 0, 1, 0, 1, 1)):
        dev.copy_(torch.from_numpy(np.concatenate((a, b)[which]).view(np.int64)))
        _check(ctx.analyze_batch_dev(dev, (off_a, off_b)[which], 4), refs[which], rep)
        rows = ctx.analyze(a[3], 4)
        assert np.array_equal(np.stack([rows[f] for f in rows.dtype.names], 1).astype(np.int64), eager)
        torch.zeros(1 << 20, device="cuda").add_(1)
    assert ctx.graph_stats() == {"captures": 1, "replays": 5}
    c = _loops([66000, 300, 70000, 20], seed=100)
    dev_c, off_c = _pack(c)
    _check(ctx.analyze_batch_dev(dev_c, off_c, 4), _refs(c, 4), "another shape")
    assert ctx.graph_stats()["captures"] == 2


def test_stage_batch_of_the_batched_workload(ctx):
    """Windows of the batched workload stage by stage: beside a long one, and without
    it while a kernel is timed."""
    wins, m = synth.config3(num_windows=40)
    wins = [w.astype(np.uint64) for w in wins]
    _each_form(ctx, wins[:20] + [_long()] + wins[20:], m)
    ctx.profile_kernel(1)
    _each_form(ctx, wins, m, forms=FORMS[:3])
    assert ctx.kernel_profile()["launches"] > 0
    ctx.profile_kernel(0)


def test_stage_batch_needing_many_selection_rounds(ctx):
    """Block families need more greedy rounds than a sync-free run enqueues (windows
    past the per-window greedy's 2^17 tokens go through the rounds): such a run, or such
    a lane, is finished host-driven."""
    blocks = []
    for k in range(1, 60):
        blocks += [0] * k + [1]
    blocks = np.array(blocks, dtype=np.uint64)
    wins = [blocks, _long(3, 140000), synth.config0()[0].astype(np.uint64), _long(4, 132000), blocks]
    _each_form(ctx, wins, 1)
