"""Texts with more matches than a wave's or a block's match stage holds: counts,
whole match sets and the first part of them, around the stages' sizes."""

import numpy as np
import pytest

from oracle import Oracle
from tests.helpers import as_pairs, assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (keywords, bytes from one occurrence to the next that no keyword spans)
SETS = {"prefix table": ([b"a"], b"a."), "two ids": ([b"a", b"a"], b"a."),
        "window table": ([b"abcdefgh"], b"abcdefgh"), "nested": ([b"abcdefgh", b"abcdefghi"], b"abcdefghi.......")}


@pytest.fixture(scope="module")
def pf():
    import paper_1412_7789_amd as _pf
    assert torch.cuda.is_available()
    _pf.load()
    return _pf


@pytest.mark.parametrize("kind", list(SETS))
def test_around_the_waves_stage(pf, kind):
    """One wave scans one chunk of 4 KiB; its stage holds 126 matches and is
    written out between rounds of 64 hits."""
    kws, step = SETS[kind]
    a, o = pf.Automaton(kws), Oracle(kws)
    launch = pf.launch_config(policy=1, segs=4)
    for m in (0, 1, 62, 63, 64, 65, 125, 126, 127, 128, 129, 189, 190, 191, 192, 193, 252, 255, 256, 257, 511, 2048):
        if m * len(step) > 4096:
            continue
        text = np.frombuffer(step * m + b"." * (4096 - m * len(step)), dtype=np.uint8)
        exp = as_pairs(*o.match(text))
        t = torch.from_numpy(text.copy()).cuda()
        assert a.count(t, launch=launch) == len(exp[0])
        off, pid = a.match(t, launch=launch, capacity=len(exp[0]) + 3)
        assert_same((off.cpu().numpy(), pid.cpu().numpy()), exp, f"{kind} {m}")
        for cap in {1, len(exp[0]) // 2, len(exp[0]) - 1}:
            if not 0 < cap < len(exp[0]):
                continue
            off = torch.full((cap + 1,), -7, dtype=torch.int64, device="cuda")
            pid = torch.full((cap + 1,), -7, dtype=torch.int32, device="cuda")
            assert a.match_into(t, off[:cap], pid[:cap], launch=launch) == len(exp[0])
            got = set(zip(off.tolist()[:cap], pid.tolist()[:cap]))
            assert len(got) == cap and got <= set(zip(exp[0].tolist(), exp[1].tolist()))
            assert off[cap] == -7 and pid[cap] == -7


@pytest.mark.parametrize("kind", list(SETS))
@pytest.mark.parametrize("per_text", [True, False])
def test_around_the_blocks_stage(pf, kind, per_text):
    """One block scans a batch of 64 KiB; its stage holds 3072 matches and is
    written out between rounds of 1024 hits."""
    kws, step = SETS[kind]
    a, o = pf.Automaton(kws), Oracle(kws)
    launch = pf.launch_config(policy=1, segs=4)
    for m in (2047, 2048, 2049, 3071, 3072, 3073, 4095, 4096, 4097, 5120, 6143, 6144, 6145, 8192, 32768):
        if m * len(step) > 65536:
            continue
        text = np.frombuffer(step * m + b"." * (65536 - m * len(step)), dtype=np.uint8)
        cuts = np.array([0, 0, 7, 30_001, 30_002, 65_000, 65536], dtype=np.int64)
        want = [as_pairs(*o.match(text[s:e])) for s, e in zip(cuts[:-1], cuts[1:])]
        total = sum(len(w[0]) for w in want)
        t, c = torch.from_numpy(text.copy()).cuda(), torch.from_numpy(cuts).cuda()
        tid = torch.empty(total + 1, dtype=torch.int32, device="cuda")
        off = torch.empty(total + 1, dtype=torch.int64, device="cuda")
        pid = torch.empty(total + 1, dtype=torch.int32, device="cuda")
        per = torch.full((len(want),), -1, dtype=torch.int64, device="cuda") if per_text else None
        got = a.match_batch_into(t, c, tid, off, pid, per_text=per, launch=launch)
        assert got == total
        if per_text:
            assert per.tolist() == [len(w[0]) for w in want]
        tid, off, pid = (x[:total].cpu().numpy() for x in (tid, off, pid))
        for k, w in enumerate(want):
            assert_same((off[tid == k], pid[tid == k]), w, f"{kind} {m} text {k}")


def test_more_matches_of_one_text_than_32_bits_count(pf):
    """A million keyword ids at each of 4400 offsets, all in one block: the
    text's count is exact past 2^32 (the other texts have none)."""
    n_ids, n = 1_000_000, 4400
    a = pf.Automaton([b"a"] * n_ids)
    t = torch.full((n,), ord("a"), dtype=torch.uint8, device="cuda")
    c = torch.tensor([0, 0, n, n], dtype=torch.int64, device="cuda")
    none32 = torch.empty(0, dtype=torch.int32, device="cuda")
    none64 = torch.empty(0, dtype=torch.int64, device="cuda")
    per = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    assert a.match_batch_into(t, c, none32, none64, none32, per_text=per) == n * n_ids
    assert per.tolist() == [0, n * n_ids, 0]
