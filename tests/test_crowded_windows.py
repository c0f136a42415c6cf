"""Keyword sets whose 4-byte windows lie on many keyword paths (small alphabets,
words, a middle that many keywords share): the window table is left out where
most windows are like that, and a few such windows in another set get one entry
for each position, walked from the root, instead of one for each path."""

import numpy as np
import pytest

import paper_1412_7789_amd as pf
from oracle import Oracle
from paper_1412_7789_amd import _lib as L
from tests.helpers import assert_same
from tests.test_builder import _window_slots

DIGITS, ACGT = b"0123456789", b"ACGT"


def letters(rng, alphabet, n):
    return np.frombuffer(alphabet, dtype=np.uint8)[rng.integers(0, len(alphabet), size=n)]


def draw(rng, alphabet, n, lo, hi):
    return sorted({bytes(letters(rng, alphabet, int(k))) for k in rng.integers(lo, hi + 1, size=n)})


def some_shared(rng):
    """5000 random keywords and 40 with one middle: 20 first letters, 2 endings."""
    kws = [bytes(rng.integers(0, 256, size=int(n), dtype=np.uint8)) for n in rng.integers(8, 40, size=5000)]
    return kws + [bytes([c]) + b"erver[" + b"%d" % i for c in b"abcdefghijklmnopqrst" for i in (10, 11)]


def tables(kws):
    plan = pf.Plan(kws)
    return [(plan.export(k, np.uint32), plan.export(e, np.int32).reshape(-1, 4)) for k, e in (
        (L.AC_TABLE_WINDOW2_KEYS, L.AC_TABLE_WINDOW2_ENTRIES), (L.AC_TABLE_WINDOW4_KEYS, L.AC_TABLE_WINDOW4_ENTRIES))]


@pytest.mark.parametrize("alphabet,n,lo,hi,have", [
    (DIGITS, 5000, 8, 12, (True, True)), (DIGITS, 30_000, 8, 12, (False, False)),
    (ACGT, 100, 10, 30, (True, True)), (ACGT, 2000, 12, 12, (False, False)),
])
def test_no_table_where_windows_are_crowded(alphabet, n, lo, hi, have):
    rng = np.random.default_rng(n)
    kws = draw(rng, alphabet, n, lo, hi)
    assert tuple(len(keys) > 0 for keys, _ in tables(kws)) == have


def test_crowded_windows_among_others_are_shared():
    """No chain of entries is longer than 8; the shared middle's windows have
    exactly one entry for each position they occur at, which compares nothing and
    goes on from the root, and every other window keeps its paths."""
    kws = some_shared(np.random.default_rng(3))
    for (keys, ent), stride in zip(tables(kws), (2, 4)):
        assert len(keys)
        paths = {}
        for k in kws:
            for j in range(1, stride + 1):
                paths.setdefault(int.from_bytes(k[j:j + 4], "little"), {}).setdefault(j, set()).add(k[:j + 4])
        shared = 0
        for x, at in paths.items():
            i, = (s for s in _window_slots(keys, x) if int(keys[s]) == x)
            chain = []
            while True:
                _, n, what, link = (int(v) for v in ent[i])
                chain.append((link & 7, n, what, bool(link & 8)))
                link = (link & 0xFFFFFFFF) >> 4
                if link == 0:
                    break
                i = link - 1
            assert len(chain) <= 2 * stride
            if sum(map(len, at.values())) > 2 * stride:
                shared += 1
                assert sorted(chain) == [(j, 0, 0, True) for j in sorted(at)]
            else:
                assert sorted(j for j, _, _, _ in chain) == sorted(j for j, p in at.items() for _ in p)
                assert all(n >= j + 4 for j, n, _, _ in chain)
        assert shared == stride        # "erve", "rver", "ver[" and "er[1" at positions 1 .. stride


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["shared middle", "digits", "acgt", "acgt few"])
def test_matches_with_crowded_windows(kind):
    """Whole match sets, single texts at every alignment and length around their
    ends and a batch cut inside keywords, for default and explicit launches."""
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(17)
    if kind == "shared middle":
        kws = some_shared(rng)
        parts = [kws[int(i)] for i in rng.integers(len(kws) - 40, len(kws), size=3000)]
        parts += [bytes([c]) + b"erver[" for c in b"abcdzyx"] * 200 + [kws[int(i)] for i in rng.integers(0, 5000, size=1000)]
        text = np.frombuffer(b"".join(parts[int(i)] for i in rng.permutation(len(parts))), dtype=np.uint8)
    else:
        alphabet, n, lo, hi = {"digits": (DIGITS, 30_000, 8, 12), "acgt": (ACGT, 2000, 8, 12),
                               "acgt few": (ACGT, 100, 8, 30)}[kind]
        kws = draw(rng, alphabet, n, lo, hi)
        text = letters(rng, alphabet, 300_000).copy()
        for at in rng.integers(0, len(text) - 40, size=500):
            k = np.frombuffer(kws[int(rng.integers(len(kws)))], dtype=np.uint8)
            text[at:at + len(k)] = k
    a, o = pf.Automaton(kws), Oracle(kws)
    buf = torch.from_numpy(np.concatenate([np.zeros(16, np.uint8), text, np.zeros(16, np.uint8)])).cuda()
    exp = o.match(text)
    cuts = np.sort(np.concatenate([[0, len(text)], rng.integers(0, len(text), size=99)])).astype(np.int64)
    want = [o.match(text[s:e]) for s, e in zip(cuts[:-1], cuts[1:])]
    launches = [None] + [dict(policy=1, stride=s, filter=f, segs=g) for s, f, g in
                         ((4, 6, 2), (4, 4, 1), (4, 5, 4), (2, 6, 4), (2, 3, 2), (1, 2, 2))]
    for cfg in launches:
        launch = pf.launch_config(**cfg) if cfg else None
        off, pid = a.match(buf[16:16 + len(text)], launch=launch, capacity=len(exp[0]))
        assert_same((off.cpu().numpy(), pid.cpu().numpy()), exp, f"{kind} {cfg}")
        tid, off, pid, per = (x.cpu().numpy() for x in a.match_batch(
            buf[16:16 + len(text)], torch.from_numpy(cuts).cuda(), launch=launch, capacity=len(exp[0])))
        for t, w in enumerate(want):
            assert_same((off[tid == t], pid[tid == t]), w, f"{kind} {cfg} text {t}")
        for start in range(0, 40, 3):
            for n in (1, 7, 8, 9, 15, 16, 33, 1023, 1031):
                part = text[start:start + n]
                off, pid = a.match(buf[16 + start:16 + start + n], launch=launch, capacity=8 * n)
                assert_same((off.cpu().numpy(), pid.cpu().numpy()), o.match(part), f"{kind} {cfg} {start}+{n}")


def test_a_few_keywords_in_one_window():
    """Sets of under 16 paths keep their tables while no window lies on more than
    2 * stride of them."""
    few = [b"aaaaaaaa", b"aaaaaaaab", b"baaaaaaaa"]                       # "aaaa": 8 paths, 4 at stride 2
    assert [len(k) > 0 for k, _ in tables(few)] == [True, True]
    assert [len(k) > 0 for k, _ in tables(few + [b"aaabaaaa"])] == [True, False]   # 9 paths at stride 4


@pytest.mark.gpu
def test_crowded_windows_of_zeros_at_the_texts_end():
    """What lies past a text's end reads as zeros: keywords crowded in a window of
    zeros, in texts that end before, inside and after one."""
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(23)
    kws = [bytes(rng.integers(1, 256, size=int(n), dtype=np.uint8)) for n in rng.integers(8, 40, size=5000)]
    kws += [bytes([c]) + bytes(7) + bytes([d]) for c in range(1, 21) for d in (0, 1)]
    assert all(len(keys) for keys, _ in tables(kws))
    a, o = pf.Automaton(kws), Oracle(kws)
    text = np.concatenate([rng.integers(0, 21, size=2000, dtype=np.uint8)] +
                          [np.frombuffer(kws[5000 + i] + bytes(i % 5), dtype=np.uint8) for i in range(40)])
    buf = torch.zeros(len(text) + 64, dtype=torch.uint8, device="cuda")
    buf[16:16 + len(text)] = torch.from_numpy(text).cuda()
    for stride, segs in ((0, 0), (4, 1), (4, 4), (2, 2)):
        launch = pf.launch_config(policy=1, stride=stride, segs=segs)
        for n in range(len(text) - 70, len(text) + 1):
            for start in (0, 5):
                off, pid = a.match(buf[16 + start:16 + n], launch=launch, capacity=200)
                assert_same((off.cpu().numpy(), pid.cpu().numpy()), o.match(text[start:n]), f"{stride} {segs} {start} {n}")
        cuts = np.concatenate([[0], np.arange(len(text) - 300, len(text) + 1, 3), [len(text)]]).astype(np.int64)
        tid, off, pid, per = (x.cpu().numpy() for x in a.match_batch(
            buf[16:16 + len(text)], torch.from_numpy(cuts).cuda(), launch=launch))
        for t in range(len(cuts) - 1):
            assert_same((off[tid == t], pid[tid == t]), o.match(text[cuts[t]:cuts[t + 1]]), f"{stride} {segs} text {t}")
