"""Timed cases of the matcher: what a program does with it, through its public
entry points, from the smallest call to the largest.

A case is one pass over inputs that are already where the entry point takes
them (device tensors for the scans, host arrays for the dispatch and the
request server), with the automaton built and the output buffers kept.

The matcher reports an unordered match set.  Every pass therefore also writes
the set into a table with one entry per text byte, the id of the keyword that
starts there (-1: none), as a program that annotates its text does: one
``scatter_`` on the device or one indexed store on the host.  The keyword sets
are free of prefixes of one another, so at most one keyword starts at an
offset and the table holds the whole set.  Device buffers of the asynchronous
calls start out pointing at a spare last entry of the table, so slots past the
match count write there.

Texts are drawn on the device from the seed, with a keyword planted at a random
place of every ``gap`` bytes, the densities of the repository's own workloads.
"""

import math

import numpy as np
import torch

import paper_1412_7789_amd as pf

KIB, MIB, GIB = 1 << 10, 1 << 20, 1 << 30

# Keyword sets: number, shortest, longest, byte range, share of keywords that
# start with 4 to 12 bytes of another one, and the text's bytes per planted
# keyword.  All but "short" are the sets that the tests and the benchmark use;
# "short" stands for token lists whose shortest entries have two bytes (the
# filter's shorter prefixes).
SETS = {
    "tiny": (64, 4, 12, 0x61, 0x7A, 0.0, 524),
    "short": (200, 2, 8, 0x20, 0x7E, 0.0, 4096),
    "sweep": (1000, 8, 32, 0x20, 0x7E, 0.0, 4096),
    "batched": (2000, 8, 32, 0x20, 0x7E, 0.0, 4096),
    "large": (20000, 16, 64, 0x00, 0xFF, 0.30, 65536),
    "served_500": (500, 8, 64, 0x00, 0xFF, 0.0, 65536),
    "served_5000": (5000, 8, 64, 0x00, 0xFF, 0.0, 65536),
    "served_20000": (20000, 8, 64, 0x00, 0xFF, 0.0, 65536),
    "served_50000": (50000, 8, 64, 0x00, 0xFF, 0.0, 65536),
}
SERVED = ("served_500", "served_5000", "served_20000", "served_50000")
ALPHA = bytes(range(0x61, 0x7B))
LINE = ALPHA * 5 + b"\n"


def listed():
    return [
        # A request of one packet or record: launches and latency are all of it.
        dict(name="call_1k", kind="call", set="sweep", n=KIB, shift=0, entry="sync"),
        # A small dictionary over a document, many matches.
        dict(name="tiny_1m", kind="call", set="tiny", n=MIB, shift=0, entry="sync"),
        # The paper's own experiment at its largest size: five permutations of
        # the alphabet in repeated alphabet lines, a match every 26 bytes.
        dict(name="paper_671k", kind="paper", patterns=5, lines=5125, entry="sync"),
        # A text inside a larger buffer, at an odd address and of an odd size,
        # enqueued without waiting.
        dict(name="sweep_4m_odd", kind="call", set="sweep", n=4 * MIB + 5, shift=3, entry="async"),
        # The largest served request against the largest resident automaton.
        dict(name="served50k_64m", kind="call", set="served_50000", n=64 * MIB, shift=0, entry="async"),
        # Short tokens: two-byte prefixes, every offset tested, dense matches.
        dict(name="short_64m", kind="call", set="short", n=64 * MIB, shift=0, entry="sync"),
        # The headline scan: a 1 GiB text against 1000 printable keywords.
        dict(name="sweep_1g", kind="call", set="sweep", n=GIB, shift=0, entry="sync"),
        # The same size against 20000 binary keywords, tables beyond LDS.
        dict(name="large_1g", kind="call", set="large", n=GIB, shift=0, entry="sync"),
        # Thousands of texts of uneven length in one call, counts per text.
        dict(name="batch_4096", kind="batch", set="batched", texts=4096, median=8192, per_text=True, entry="sync"),
        # A small batch as a server forms it, enqueued without waiting.
        dict(name="batch_64", kind="batch", set="served_5000", texts=64, median=8192, per_text=False, entry="async"),
        # Host text in, host matches out, above the CPU/GPU crossover.
        dict(name="dispatch_256k", kind="dispatch", set="sweep", n=256 * KIB),
        # Requests of uneven size in flight at once on four resident automata.
        dict(name="served_mix", kind="served", requests=24, size_hi=4 * MIB),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.5:
        name = rng.choice(sorted(SETS))
        top = {"short": 64 * MIB, "tiny": 64 * MIB}.get(name, GIB)
        return dict(kind="call", set=name, n=_log_uniform(rng, KIB, top), shift=rng.choice((0, 0, rng.randrange(16))),
                    entry=rng.choice(("sync", "async", "noalloc")))
    if u < 0.7:
        return dict(kind="batch", set=rng.choice(("batched", "sweep") + SERVED), texts=_log_uniform(rng, 2, 4096),
                    median=_log_uniform(rng, 256, 8192), per_text=rng.random() < 0.5, entry=rng.choice(("sync", "async")))
    if u < 0.85:
        return dict(kind="dispatch", set=rng.choice(("sweep", "batched") + SERVED), n=_log_uniform(rng, KIB, 16 * MIB))
    if u < 0.95:
        return dict(kind="paper", patterns=rng.choice((5, 10)), lines=_log_uniform(rng, 10, 5125),
                    entry=rng.choice(("sync", "async")))
    return dict(kind="served", requests=rng.randrange(4, 25), size_hi=_log_uniform(rng, 64 * KIB, 4 * MIB))


# ---- inputs -------------------------------------------------------------------

def _prefix_free(kws):
    """The keywords none of which starts another one."""
    order = sorted(range(len(kws)), key=kws.__getitem__)
    keep = set(order)
    for a, b in zip(order, order[1:]):
        if kws[b].startswith(kws[a]):
            keep.discard(a)
    return [kws[i] for i in sorted(keep)]


def _keywords(name, seed):
    n, lo, hi, b0, b1, shared, _ = SETS[name]
    rng = np.random.default_rng([seed, 1])
    lens = rng.integers(lo, hi + 1, size=n)
    ends = np.cumsum(lens)
    flat = rng.integers(b0, b1 + 1, size=int(ends[-1]), dtype=np.uint8).tobytes()
    kws = [flat[e - m:e] for e, m in zip(ends.tolist(), lens.tolist())]
    free = n - int(shared * n)
    for i in range(free, n):
        donor = kws[int(rng.integers(0, free))]
        m = min(int(rng.integers(4, 13)), len(donor), len(kws[i]))
        kws[i] = donor[:m] + kws[i][m:]
    return _prefix_free(sorted(set(kws), key=kws.index) if len(set(kws)) < n else kws)


def _paper_keywords(patterns, seed):
    rng = np.random.default_rng([seed, 2])
    alpha = np.frombuffer(ALPHA, dtype=np.uint8)
    kws = [ALPHA, ALPHA[7:] + ALPHA[:7]]         # the identity, and a rotation of it
    while len(kws) < patterns:
        k = rng.permutation(alpha).tobytes()
        if k not in kws:
            kws.append(k)
    return kws


def _text(name, kws, n, seed, device, planted_by=None):
    """Random bytes of the set's range with one keyword per `gap` bytes (one
    in a shorter text)."""
    _, _, longest, b0, b1, _, gap = SETS[name]
    gap = min(gap, n)
    g = torch.Generator(device=device).manual_seed(seed)
    text = torch.randint(b0, b1 + 1, (n,), dtype=torch.uint8, device=device, generator=g)
    for lists in (planted_by or [kws]):
        rng = np.random.default_rng([seed, 3, len(lists)])
        cells = n // gap
        pids = rng.integers(0, len(lists), size=cells)
        lens = np.array([len(k) for k in lists])[pids]
        at = np.arange(cells, dtype=np.int64) * gap + (rng.random(cells) * (gap - longest)).astype(np.int64)
        firsts = np.cumsum(lens) - lens
        where = np.repeat(at - firsts, lens) + np.arange(int(lens.sum()))
        what = np.frombuffer(b"".join(lists[p] for p in pids.tolist()), dtype=np.uint8)
        text[torch.from_numpy(where).to(device)] = torch.from_numpy(what.copy()).to(device)
    return text


def _single(case, seed, device):
    """(keywords, text) of a case with one text."""
    if case["kind"] == "paper":
        kws = _paper_keywords(case["patterns"], seed)
        text = torch.frombuffer(bytearray(LINE * case["lines"]), dtype=torch.uint8).to(device)
        # another seed starts at another byte of the line
        return kws, torch.roll(text, -(seed % len(LINE)))
    kws = _keywords(case["set"], seed)
    return kws, _text(case["set"], kws, case["n"], seed, device)


def _batch_starts(case):
    """Starts of packed texts of log-normal lengths: the case's, not the seed's."""
    rng = np.random.default_rng([case["texts"], case["median"]])
    lens = np.exp(rng.normal(math.log(case["median"]), 2.1, size=case["texts"]))
    lens = np.clip(np.rint(lens), 64, 4 * MIB).astype(np.int64)
    starts = np.zeros(case["texts"] + 1, dtype=np.int64)
    np.cumsum(lens, out=starts[1:])
    return starts


def _batch(case, seed, device):
    """(keywords, packed texts, text starts) of a batch."""
    kws, starts = _keywords(case["set"], seed), _batch_starts(case)
    return kws, _text(case["set"], kws, int(starts[-1]), seed, device), starts


def _request_lengths(case):
    """Log-uniform request sizes: the case's, not the seed's."""
    rng = np.random.default_rng([case["requests"], case["size_hi"]])
    return np.exp(rng.uniform(math.log(KIB), math.log(case["size_hi"]), size=case["requests"])).astype(np.int64)


def _requests(case, seed, device):
    """(keyword lists, pool, automaton, start and length of every request)."""
    lists = [_keywords(name, seed + 7 * i) for i, name in enumerate(SERVED)]
    rng = np.random.default_rng([seed, 5])
    k, lens = case["requests"], _request_lengths(case)
    which = rng.integers(0, len(lists), size=k)
    pool_n = 2 * case["size_hi"]
    pool = _text(SERVED[0], None, pool_n, seed, device, planted_by=lists)
    at = (rng.random(k) * (pool_n - lens + 1)).astype(np.int64)
    return lists, pool, which, at, lens


def _capacity(case, n):
    if case["kind"] == "paper":
        return n // 12 + 1024
    if case["set"] == "short":
        return n // 64 + 1024
    return 2 * n // SETS[case["set"]][6] + 1024


def prepare(case, seed):
    dev = torch.device("cuda")
    s = {"kind": case["kind"], "entry": case.get("entry")}
    if case["kind"] in ("call", "paper"):
        kws, text = _single(case, seed, dev)
        n, shift = text.numel(), case.get("shift", 0)
        if shift:
            buf = torch.empty(n + 16, dtype=torch.uint8, device=dev)
            buf[shift:shift + n] = text
            text = buf[shift:shift + n]
        cap = _capacity(case, n)
        s.update(a=pf.Automaton(kws), text=text, count=torch.zeros(1, dtype=torch.int64, device=dev),
                 off=torch.full((cap,), n, dtype=torch.int64, device=dev),
                 pid=torch.full((cap,), -1, dtype=torch.int32, device=dev),
                 tags=torch.full((n + 1,), -1, dtype=torch.int32, device=dev))
    elif case["kind"] == "batch":
        kws, texts, starts = _batch(case, seed, dev)
        n = texts.numel()
        cap = _capacity(case, n)
        s.update(a=pf.Automaton(kws), text=texts, starts=torch.from_numpy(starts).to(dev),
                 count=torch.zeros(1, dtype=torch.int64, device=dev),
                 tid=torch.zeros(cap, dtype=torch.int32, device=dev),
                 off=torch.full((cap,), n, dtype=torch.int64, device=dev),
                 pid=torch.full((cap,), -1, dtype=torch.int32, device=dev),
                 per=torch.zeros(case["texts"], dtype=torch.int64, device=dev) if case["per_text"] else None,
                 tags=torch.full((n + 1,), -1, dtype=torch.int32, device=dev))
    elif case["kind"] == "dispatch":
        kws, text = _single(case, seed, dev)
        host = torch.empty(text.numel(), dtype=torch.uint8, pin_memory=True)
        host.copy_(text)
        s.update(a=pf.Automaton(kws), host=host, text=host.numpy(),
                 tags=np.full(text.numel(), -1, dtype=np.int32))
    else:
        lists, pool, which, at, lens = _requests(case, seed, dev)
        host = torch.empty(pool.numel(), dtype=torch.uint8, pin_memory=True)
        host.copy_(pool)
        server = pf.Server()
        for kws in lists:
            server.add_automaton(pf.Automaton(kws))
        flat = host.numpy()
        base = np.cumsum(lens) - lens
        s.update(server=server, host=host, base=base.tolist(), automata=which.tolist(),
                 texts=[flat[o:o + m] for o, m in zip(at.tolist(), lens.tolist())],
                 tags=np.full(int(lens.sum()), -1, dtype=np.int32))
    return s


# ---- one pass -------------------------------------------------------------------

def run(s):
    kind, entry, tags = s["kind"], s["entry"], s["tags"]
    if kind in ("call", "paper"):
        if entry == "sync":
            n = s["a"].match_into(s["text"], s["off"], s["pid"])
            tags.scatter_(0, s["off"][:n], s["pid"][:n])
            return {"count": n, "tags": tags}
        call = s["a"].match_async if entry == "async" else s["a"].match_async_noalloc
        call(s["text"], s["off"], s["pid"], s["count"])
        tags.scatter_(0, s["off"], s["pid"])
        return {"count": s["count"], "tags": tags}
    if kind == "batch":
        if entry == "sync":
            n = s["a"].match_batch_into(s["text"], s["starts"], s["tid"], s["off"], s["pid"], s["per"])
            tid, off, pid = s["tid"][:n], s["off"][:n], s["pid"][:n]
        else:
            s["a"].match_batch_async(s["text"], s["starts"], s["tid"], s["off"], s["pid"], s["count"], s["per"])
            n, tid, off, pid = s["count"], s["tid"], s["off"], s["pid"]
        tags.scatter_(0, s["starts"].index_select(0, tid).add_(off), pid)
        out = {"count": n, "tags": tags}
        if s["per"] is not None:
            out["per_text"] = s["per"]
        return out
    if kind == "dispatch":
        off, pid, _ = s["a"].match_dispatch(s["text"])
        tags[off] = pid
        return {"count": len(off), "tags": tags}
    server = s["server"]
    ids = [server.submit(a, t) for a, t in zip(s["automata"], s["texts"])]
    counts = []
    for i, base in zip(ids, s["base"]):
        off, pid, _ = server.wait(i)
        tags[off + base] = pid
        counts.append(len(off))
    return {"counts": counts, "tags": tags}


# ---- what a pass cannot do without, and its results ------------------------------

def work(case):
    """Every text byte read once, every match (offset and id) written once."""
    if case["kind"] == "paper":
        n = case["lines"] * len(LINE)
        return {"bytes": n + 12 * (n // 14), "flops": 0}
    if case["kind"] == "batch":
        n = int(_batch_starts(case)[-1])
        return {"bytes": n + 16 * (n // SETS[case["set"]][6]) + 8 * case["texts"], "flops": 0}
    if case["kind"] == "served":
        n = int(_request_lengths(case).sum())
        return {"bytes": n + 12 * (n // 65536), "flops": 0}
    return {"bytes": case["n"] + 12 * (case["n"] // SETS[case["set"]][6]), "flops": 0}


def _find_all(kws, text, tags):
    """Writes every occurrence of every keyword in `text` (bytes) into tags."""
    count = 0
    for p, k in enumerate(kws):
        at = text.find(k)
        while at >= 0:
            tags[at] = p
            count += 1
            at = text.find(k, at + 1)
    return count


def exact(case, seed):
    """The same outputs from plain substring search on the host, where that
    takes a few seconds; the results are whole numbers."""
    small = case["kind"] == "paper" or (case["kind"] in ("call", "dispatch") and case["n"] <= MIB
                                        and SETS[case["set"]][0] <= 1000)
    if not small:
        return None
    kws, text = _single(case, seed, torch.device("cuda"))
    data = text.cpu().numpy().tobytes()
    tags = np.full(len(data) + (case["kind"] != "dispatch"), -1, dtype=np.int32)
    count = _find_all(kws, data, tags)
    if case.get("entry", "sync") != "sync":
        count = np.array([count], dtype=np.int64)
    return {"count": count, "tags": tags}
