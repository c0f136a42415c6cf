"""Slow mode: waves whose hit records run out leave the streaming loop and walk
the rest of their text as they find hits.  The texts are sized by the records
there are: more hits than all waves together can keep, so some wave must
refuse a drain (most do, about half way), and the last, ragged chunks are
scanned in slow mode too.  Few hits are matches, so that whole match sets can be
compared with the oracle's."""

import sys

import numpy as np
import pytest

from oracle import oracle_match
from tests.helpers import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

pf = None
RECORDS = 128 + 2 * 1024        # a wave keeps this many: 128 in LDS, the rest in its region
WAVES = 4                       # per block of 256 threads; such blocks take a CU's whole LDS


def setup_module(module):
    global pf
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1412_7789_amd as _pf
    _pf.load()
    pf = _pf


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def make_text(n, seed):
    """Runs of 'a' between lone 'b's some hundred bytes apart, which make the
    queueing rounds uneven, so that a refusal finds part of a group queued."""
    rng = np.random.default_rng(seed)
    text = np.full(n, ord("a"), dtype=np.uint8)
    text[rng.integers(0, n, size=n // 300)] = ord("b")
    return text


# shortest keyword -> keywords that runs of 'a' nearly match: a hit at every
# tested place, a match only beside a 'b'
SETS = {
    "window table": [b"aaaaaaab", b"aaaaaaaaab", b"baaaaaaab", b"aaabaaaa", b"aaaaaaab", b"a" * 40 + b"b"],
    "seven bytes": [b"aaaaaab", b"baaaaaab", b"aabaaaa"],
    "five bytes": [b"aaaab", b"baaab", b"aabaa"],
    "three bytes": [b"aab", b"aaaab", b"baab"],
    "two bytes": [b"ba", b"aaab"],
    "one byte": [b"b", b"aaab"],
}
# shortest keyword, sampling stride, filters
CASES = [("window table", 4, (6, 4, 5)), ("window table", 2, (6, 2, 3)), ("window table", 1, (2,)),
         ("seven bytes", 4, (1, 4)), ("five bytes", 2, (5, 3)), ("three bytes", 1, (1, 4)),
         ("two bytes", 1, (3,)), ("one byte", 1, (2,))]


def key(tid, off, pid):
    return np.sort((tid.astype(np.int64) << 40) | (off.astype(np.int64) << 8) | pid)


@pytest.mark.parametrize("kind,stride,filters", CASES, ids=[f"{k}-stride{s}" for k, s, _ in CASES])
def test_more_hits_than_records(kind, stride, filters):
    kws = SETS[kind]
    waves = WAVES * torch.cuda.get_device_properties(0).multi_processor_count
    n = (2 * waves * RECORDS * stride & ~4095) - 4096 + 1533     # ends in a chunk's second segment, mid-word
    text = make_text(n, stride)
    # places a hit is certain: tested ones inside a run of at least 12 bytes
    run = np.ones(n, dtype=bool)
    for at in np.flatnonzero(text == ord("b")):
        run[max(0, at - 12):at + 12] = False
    assert int(run.sum()) // stride > waves * RECORDS * 3 // 2
    a = pf.Automaton(kws)
    buf = torch.zeros(n + 64, dtype=torch.uint8, device="cuda")
    exp = oracle_match(kws, text)
    rng = np.random.default_rng(7)
    cuts = np.sort(np.concatenate([[0, n, n // 2, n // 2], rng.integers(0, n, size=23)])).astype(np.int64)
    want = [oracle_match(kws, text[s:e]) for s, e in zip(cuts[:-1], cuts[1:])]
    want_n = np.array([len(w[0]) for w in want])
    want_key = key(np.repeat(np.arange(len(want)), want_n), np.concatenate([w[0] for w in want]),
                   np.concatenate([w[1] for w in want]))
    bounds = torch.from_numpy(cuts).cuda()
    for f in filters:
        for segs in (1, 2, 4):
            cfg = pf.launch_config(policy=1, filter=f, stride=stride, segs=segs, block=256)
            shift = (5 * segs + f) % 16
            t = buf[shift:shift + n]
            t.copy_(torch.from_numpy(text))
            say("slow mode", kind, stride, f, segs, n)
            off, pid = a.match(t, launch=cfg, capacity=len(exp[0]))
            assert_same((off.cpu().numpy(), pid.cpu().numpy()), exp, f"filter {f} segs {segs}")
            assert a.count(t, launch=cfg) == len(exp[0])
            tid, off, pid, per = (x.cpu().numpy() for x in a.match_batch(t, bounds, launch=cfg, capacity=len(want_key)))
            assert np.array_equal(key(tid, off, pid), want_key), f"batch, filter {f} segs {segs}"
            assert np.array_equal(per, want_n)


def test_text_ending_in_each_segment():
    """A wave in slow mode reads its last chunk one segment at a time: texts
    that end in every segment of it, at its edges and in the middle, followed by
    bytes that would go on with a keyword."""
    kws = SETS["window table"]
    waves = WAVES * torch.cuda.get_device_properties(0).multi_processor_count
    full = 4 * waves * RECORDS * 4 // 3 & ~4095
    text = make_text(full + 4096, 3)
    a = pf.Automaton(kws)
    t = torch.from_numpy(text).cuda()
    off_all, pid_all = oracle_match(kws, text)
    end_all = off_all + np.array([len(k) for k in kws])[pid_all]
    for segs, stride, f in ((4, 4, 6), (2, 4, 4), (4, 2, 6)):
        for extra in [1, 3, 4, 1023, 1024, 1025, 2047, 2049, 3071, 3073, 4095]:
            n = full + extra
            cfg = pf.launch_config(policy=1, filter=f, stride=stride, segs=segs, block=256)
            say("ends at", extra, segs, stride)
            off, pid = a.match(t[:n], launch=cfg, capacity=len(off_all))
            keep = end_all <= n
            assert_same((off.cpu().numpy(), pid.cpu().numpy()), (off_all[keep], pid_all[keep]), f"{n} segs {segs}")


@pytest.mark.parametrize("stride,segs", [(4, 1), (4, 2), (4, 4), (2, 2)])
def test_more_hits_than_records_with_chained_windows(stride, segs):
    """The same with windows that lie on several keywords' paths, which keep one
    entry for each."""
    from paper_1412_7789_amd import _lib as L
    kws = [b"aaaaaaab", b"aaaaaaaaaab", b"aaaaaaaaab", b"baaaaaaab"]
    table = L.AC_TABLE_WINDOW4_KEYS if stride == 4 else L.AC_TABLE_WINDOW2_KEYS
    assert len(pf.Plan(kws).export(table, np.uint32)) > 0
    waves = WAVES * torch.cuda.get_device_properties(0).multi_processor_count
    n = 2 * waves * RECORDS * stride + 1533
    text = make_text(n, segs)
    exp = oracle_match(kws, text)
    cuts = np.array([0, n // 3, n // 3 + 1, n // 2, n], dtype=np.int64)
    want = [oracle_match(kws, text[s:e]) for s, e in zip(cuts[:-1], cuts[1:])]
    a, t = pf.Automaton(kws), torch.from_numpy(text).cuda()
    cfg = pf.launch_config(policy=1, filter=6, stride=stride, segs=segs, block=256)
    off, pid = a.match(t, launch=cfg, capacity=len(exp[0]))
    assert_same((off.cpu().numpy(), pid.cpu().numpy()), exp, "single")
    tid, off, pid, per = (x.cpu().numpy() for x in a.match_batch(t, torch.from_numpy(cuts).cuda(), launch=cfg))
    for k, w in enumerate(want):
        assert_same((off[tid == k], pid[tid == k]), w, f"text {k}")
