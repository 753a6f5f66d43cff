"""Repeat-finding workloads, from one ruler slice of a task stream to a whole batch or serving burst.

Every case goes through the entry points a program uses: a window of host or device tokens, a packed batch of
windows, the continuous-batching server, and the trace finder on top of it.  The token streams are the
repository's own generators (paper_2406_18111_amd/synth.py) or generic ones, seeded.
"""
import math

import numpy as np
import torch

from paper_2406_18111_amd import _lib, synth

_CTX = {}


def _context(server=False):
    """A program keeps one context per GPU for its analyses, and one whose server runs."""
    key = "server" if server else "direct"
    if key not in _CTX:
        _CTX[key] = _lib.Context()
        if server:
            _CTX[key].server_start(slots=3)
    return _CTX[key]


def listed():
    return [
        # the shortest ruler slice of the trace finder: one block of 250 tasks, minimum trace length 25, host tokens
        dict(name="slice_250", do="window", n=250, stream="loop", body=30, alphabet=64, p_sub=0.02, min_len=25, bits=64,
             api="host", occ=False),
        # the longest ruler slice: the whole history buffer of 5000 tasks, with the occurrence list
        dict(name="history_5000", do="window", n=5000, stream="nested", min_len=25, bits=64, api="host", occ=True),
        # the repository's smallest configuration (config0): 4096 tokens on the device
        dict(name="loop_4096", do="window", n=4096, stream="loop", body=50, alphabet=64, p_sub=0.05, min_len=8, bits=64,
             api="dev", occ=False),
        # 32-bit tokens over a tiny alphabet: short repeats everywhere, the most candidates per token; odd size
        dict(name="symbols_u32_3001", do="window", n=3001, stream="symbols", alphabet=4, min_len=3, bits=32, api="dev",
             occ=True),
        # a window as long as the serving trace's median, odd size
        dict(name="loop_30011", do="window", n=30011, stream="loop", body=211, alphabet=4096, p_sub=0.05, min_len=8,
             bits=64, api="dev", occ=False),
        # a long serving window on its own
        dict(name="nested_131071", do="window", n=131071, stream="nested", min_len=16, bits=64, api="dev", occ=False),
        # config1: one window of 2^20 tokens
        dict(name="nested_1048576", do="window", n=1 << 20, stream="nested", min_len=16, bits=64, api="dev", occ=False),
        # config2: the adversarial window, 2^24 32-bit tokens, half of them one run of one value
        dict(name="half_run_u32_16777216", do="window", n=1 << 24, stream="half", alphabet=4, min_len=32, bits=32,
             api="dev", occ=False),
        # one ruler slice from each of 64 task streams, packed into one batch of host tokens
        dict(name="batch_64_slices", do="batch", windows=64, lo=250, hi=5000, alphabet=64, p_sub=0.02, min_len=25,
             api="host"),
        # config3: the batched workload
        dict(name="batch_4096", do="batch", windows=4096, lo=256, hi=65536, alphabet=4096, p_sub=0.05, min_len=8,
             api="dev"),
        # a burst of the serving trace (config4): windows of 2^10 to 2^20 tokens submitted together, rows fetched as they come
        dict(name="serve_48", do="serve", requests=48, lo=1024, hi=1 << 20, min_len=16),
        # the trace finder over one task stream: a slice analysed after every block of 250 tasks
        dict(name="tracer_20_blocks", do="tracer", blocks=20, block=250, capacity=5000, min_len=25),
    ]


def _log(rng, lo, hi):
    """A whole number, uniform over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["window", "window", "window", "batch", "serve", "tracer"])
    if kind == "window":
        stream = rng.choice(["loop", "loop", "nested", "symbols", "half"])
        c = dict(do="window", n=_log(rng, 100, 1 << 20), stream=stream, min_len=rng.choice([4, 8, 16, 25, 32]),
                 bits=rng.choice([64, 64, 32]), api=rng.choice(["host", "dev"]), occ=rng.random() < 0.4)
        if stream == "loop":
            c.update(body=rng.randint(10, 500), alphabet=rng.choice([64, 1024, 4096]),
                     p_sub=rng.choice([0.0, 0.01, 0.05, 0.2]))
        elif stream in ("symbols", "half"):
            c.update(alphabet=rng.choice([2, 4, 16]))
        return c
    if kind == "batch":
        lo = _log(rng, 16, 1024)
        hi = _log(rng, 2 * lo, 65536)
        return dict(do="batch", windows=min(_log(rng, 2, 2048), (16 << 20) // hi), lo=lo, hi=hi,
                    alphabet=rng.choice([64, 4096]), p_sub=rng.choice([0.02, 0.05]), min_len=rng.choice([4, 8, 25]),
                    api=rng.choice(["host", "dev"]))
    if kind == "serve":
        return dict(do="serve", requests=rng.randint(3, 48), lo=_log(rng, 256, 4096), hi=_log(rng, 8192, 1 << 19),
                    min_len=rng.choice([8, 16, 25]))
    return dict(do="tracer", blocks=rng.randint(4, 40), block=rng.randint(100, 500), capacity=rng.randint(2000, 8000),
                min_len=rng.choice([10, 25]))


def _stream(case, n, seed):
    kind = case["stream"]
    if kind == "loop":
        t = synth.loop_stream(seed, n, case["body"], case["alphabet"], case["p_sub"])
    elif kind == "nested":
        t = synth.NestedLoopSource(seed).take(n)
    else:
        s = synth.Stream(seed, 8)
        t = s.below(case["alphabet"], n).astype(np.uint64)
        if kind == "half":  # half the window is one run
            at = int(s.below(n - n // 2 + 1, 1)[0])
            t[at: at + n // 2] = 0
    return (t & np.uint64(0xFFFFFFFF)).astype(np.uint32) if case["bits"] == 32 else t


def _to_gpu(t):
    return torch.from_numpy(t.view(np.int64 if t.dtype == np.uint64 else np.int32)).cuda()


def _inputs(case, seed):
    """The case's host tokens: one array, or for a batch or burst the list of its windows."""
    if case["do"] == "window":
        return _stream(case, case["n"], 5000 + seed)
    if case["do"] == "batch":
        out = []
        for w in range(case["windows"]):
            s = 1000 + 5003 * seed + w
            st = synth.Stream(s, 7)
            n = case["lo"] * (case["hi"] / case["lo"]) ** float(st.unit(1)[0])
            body = 10 + int(st.below(491, 1)[0])
            out.append(synth.loop_stream(s, max(case["lo"], min(case["hi"], int(n))), body, case["alphabet"], case["p_sub"]))
        return out
    if case["do"] == "serve":
        u = synth.Stream(4242 + seed, 7).unit(case["requests"])
        sizes = [int(case["lo"] * (case["hi"] / case["lo"]) ** float(x)) for x in u]
        return [synth.NestedLoopSource(2000 + 64 * seed + k).take(n) for k, n in enumerate(sizes)]
    return synth.NestedLoopSource(3000 + seed).take(case["blocks"] * case["block"])


def prepare(case, seed):
    t = _inputs(case, seed)
    st = dict(case=case, ctx=_context(server=case["do"] in ("serve", "tracer")))
    if case["do"] == "window":
        st["tokens"] = _to_gpu(t) if case["api"] == "dev" else t
    elif case["do"] == "batch":
        off = np.zeros(len(t) + 1, dtype=np.uint64)
        off[1:] = np.cumsum([len(w) for w in t])
        packed = np.concatenate(t)
        st["tokens"], st["offsets"] = (_to_gpu(packed) if case["api"] == "dev" else packed), off
    else:
        st["tokens"] = t
    return st


def _wait(get):
    while True:
        got = get()
        if got is not None:
            return got


def run(state):
    case, ctx, t = state["case"], state["ctx"], state["tokens"]
    if case["do"] == "window":
        analyze = ctx.analyze_dev if case["api"] == "dev" else ctx.analyze
        got = analyze(t, case["min_len"], occurrences=case["occ"])
        got = [x for x in got if x is not None] if isinstance(got, tuple) else [got]
        return [_keep(state, k, x, case["n"] // case["min_len"]) for k, x in enumerate(got)]
    if case["do"] == "batch":
        analyze = ctx.analyze_batch_dev if case["api"] == "dev" else ctx.analyze_batch
        rows, off = analyze(t, state["offsets"], case["min_len"])
        return [_keep(state, 0, rows, case["windows"] * case["hi"] // case["min_len"]), off.astype(np.int64)]
    if case["do"] == "serve":
        tickets = [ctx.submit(w, case["min_len"], stream_id=k) for k, w in enumerate(t)]
        rows = [_wait(lambda: ctx.fetch(k))[0] for k in tickets]
        room = case["requests"] * case["hi"] // case["min_len"]
    else:
        tracer = _lib.Tracer(ctx, block_tokens=case["block"], capacity=case["capacity"], min_len=case["min_len"])
        slices = 0
        for b in range(case["blocks"]):
            slices += tracer.push(t[b * case["block"]: (b + 1) * case["block"]])
        rows = [_wait(tracer.poll)[2] for _ in range(slices)]
        tracer.close()
        room = case["blocks"] * case["capacity"] // case["min_len"]
    return [_keep(state, 0, np.concatenate(rows), room), np.array([len(r) for r in rows], dtype=np.int64)]


def _keep(state, k, rows, room):
    """Output k's rows moved into the buffer the program keeps for them: `room` rows, the unused ones zero."""
    if ("rows", k) not in state:
        like = dict(dtype=torch.int32, device="cuda") if isinstance(rows, torch.Tensor) else None
        state["rows", k] = torch.zeros((room, 3), **like) if like else np.zeros((room, 3), dtype=np.int32)
    out = state["rows", k]
    out[: len(rows)] = rows if isinstance(rows, torch.Tensor) else np.ascontiguousarray(rows).view(np.int32).reshape(len(rows), 3)
    return out


def work(case):
    """Tokens read once; rows written once (loop streams keep about one row per 32 tokens)."""
    if case["do"] == "window":
        n, width = case["n"], case["bits"] // 8
        rows = n // 32 * (2 if case["occ"] else 1)
    else:
        width = 8
        if case["do"] == "tracer":
            # ruler slices: after block i the last block * 2^(trailing zeros of i) tokens, at most the history
            n = sum(min(case["block"] * (i & -i), case["capacity"], case["block"] * i) for i in range(1, case["blocks"] + 1))
        else:
            count = case["windows"] if case["do"] == "batch" else case["requests"]
            n = int(count * (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"]))
        rows = n // 32
    return {"bytes": float(n * width + 12 * rows), "flops": 0.0}


def _literal(tokens, min_len):
    """Algorithm 2 written out over Python lists: rows (start, length, count) and occurrences (start, length, row)."""
    s = [int(x) for x in tokens]
    n = len(s)
    sa = sorted(range(n), key=lambda i: s[i:])
    found = []
    for a, b in zip(sa, sa[1:]):
        p, d, lo = 0, abs(a - b), min(a, b)
        while max(a, b) + p < n and s[a + p] == s[b + p]:
            p += 1
        if p <= d:
            length, starts = p, (a, b)
        else:
            length = (p + d) // 2
            length -= length % d
            starts = (lo, lo + length)
        if length >= min_len:
            found += [(-length, tuple(s[lo: lo + length]), x) for x in starts]
    found.sort()
    taken = bytearray(n)
    rows, occ, index = [], [], {}
    for neg, sub, x in found:
        end = x - neg
        if taken[x] or taken[end - 1]:
            continue
        taken[x:end] = b"\x01" * -neg
        if sub not in index:
            index[sub] = len(rows)
            rows.append([x, -neg, 0])
        rows[index[sub]][2] += 1
        occ.append([x, -neg, index[sub]])
    return np.array(rows, dtype=np.int32).reshape(-1, 3), np.array(occ, dtype=np.int32).reshape(-1, 3)


def exact(case, seed):
    def padded(rows, room):
        return np.concatenate([rows, np.zeros((room - len(rows), 3), dtype=np.int32)])

    if case["do"] == "window" and case["n"] <= 5000 and case["stream"] != "half":
        rows, occ = _literal(_inputs(case, seed), case["min_len"])
        return [padded(x, case["n"] // case["min_len"]) for x in ((rows, occ) if case["occ"] else (rows,))]
    if case["do"] == "batch" and case["windows"] * case["hi"] <= 400000 and case["hi"] <= 5000:
        rows = [_literal(w, case["min_len"])[0] for w in _inputs(case, seed)]
        off = np.cumsum([0] + [len(r) for r in rows]).astype(np.int64)
        return [padded(np.concatenate(rows), case["windows"] * case["hi"] // case["min_len"]), off]
    return None
