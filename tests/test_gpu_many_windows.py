"""Keyword sets with more 4-byte windows than the window tables are built for:
the 4-byte-window map works without its table, candidates being looked up in
the prefix table, as every other map does."""

import numpy as np
import pytest

from oracle import Oracle
from tests.helpers import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shortest,strides", [(8, (0, 1, 2, 4)), (6, (0, 2))])
def test_large_sets_at_every_stride_and_map(shortest, strides):
    import paper_1412_7789_amd as pf
    assert torch.cuda.is_available()
    rng = np.random.default_rng(shortest)
    pool = rng.integers(0, 256, size=4 << 20, dtype=np.uint8)
    kws = [bytes(pool[o:o + n]) for o, n in zip(rng.integers(0, len(pool) - 40, size=70_000),
                                                rng.integers(shortest, 33, size=70_000))]
    kws += [b"a" * (shortest - 1) + b"b", b"a" * shortest + b"bc"]
    a = pf.Automaton(kws)
    assert a.info()["n_quads2"] > 131_072
    # parts of the pool (matches at every alignment), random bytes, and runs
    # that are a candidate at every offset and a match at none
    text = np.concatenate([pool[:300_001], rng.integers(0, 256, size=200_003, dtype=np.uint8),
                           np.full(100_000, ord("a"), dtype=np.uint8), np.frombuffer(b"bcaaabc", dtype=np.uint8)])
    o = Oracle(kws)
    exp = o.match(text)
    cuts = np.array([0, 1, 150_000, 150_000, 299_990, 520_000, len(text)], dtype=np.int64)
    want = [o.match(text[s:e]) for s, e in zip(cuts[:-1], cuts[1:])]
    d = torch.zeros(len(text) + 16, dtype=torch.uint8, device="cuda")[3:3 + len(text)]
    d.copy_(torch.from_numpy(text))
    for stride in strides:
        for f in (0, 1, 4, 5, 6) if stride else (0,):
            for segs in (1, 2, 4):
                cfg = pf.launch_config(policy=1, filter=f, stride=stride, segs=segs)
                off, pid = a.match(d, launch=cfg, capacity=len(exp[0]))
                assert_same((off.cpu().numpy(), pid.cpu().numpy()), exp, f"stride {stride} filter {f} segs {segs}")
                tid, off, pid, per = (x.cpu().numpy() for x in a.match_batch(d, torch.from_numpy(cuts).cuda(), launch=cfg))
                for t, w in enumerate(want):
                    assert_same((off[tid == t], pid[tid == t]), w, f"text {t} stride {stride} filter {f} segs {segs}")
    # enough runs that waves go on in slow mode
    waves = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    run = np.full(3 * waves * 2176 * 2 + 777, ord("a"), dtype=np.uint8)
    run[rng.integers(0, len(run), size=5000)] = ord("b")
    exp = o.match(run)
    d = torch.from_numpy(run).cuda()
    for stride in strides[1:]:
        for segs in (1, 4):
            cfg = pf.launch_config(policy=1, filter=6, stride=stride, segs=segs, block=256)
            off, pid = a.match(d, launch=cfg, capacity=len(exp[0]) + 8)
            assert_same((off.cpu().numpy(), pid.cpu().numpy()), exp, f"run, stride {stride} segs {segs}")


def test_two_segments_need_eight_mebibytes_without_a_window_table():
    """Two segments per step from 3 MiB on leave waves without one; where every
    offset may be a candidate (no window table) they wait for 8 MiB."""
    import paper_1412_7789_amd as pf
    assert torch.cuda.is_available()
    rng = np.random.default_rng(5)
    acgt = np.frombuffer(b"ACGT", dtype=np.uint8)
    text = acgt[rng.integers(0, 4, size=(8 << 20) + 5)]
    short = sorted({bytes(acgt[rng.integers(0, 4, size=int(n))]) for n in rng.integers(4, 7, size=20)})
    long = sorted({bytes(rng.integers(0, 256, size=12, dtype=np.uint8)) for _ in range(500)})
    for kws, at in ((long, 3 << 20), (short, 8 << 20)):
        a = pf.Automaton(kws)
        assert [a.default_launch(n)["segs"] for n in (1 << 20, at - 1, at, 64 << 20)] == [1, 1, 2, 2]
    d, o = torch.from_numpy(text).cuda(), Oracle(short)
    for n in ((3 << 20) + 1, (8 << 20) - 1, len(text)):
        off, pid = a.match(d[:n])
        assert_same((off.cpu().numpy(), pid.cpu().numpy()), o.match(text[:n]), f"{n} bytes")
