"""The size limit of the exact window table (CPU only): its entries are linked
by 28-bit indices, so a table that would need more is left out as a whole
instead of losing the paths past the limit.  The builder's own function is
compiled into a small program and given limits around a table's size."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
PROGRAM = r"""
#include "plan.cpp"
#include <cstdio>
using namespace pfac;

// `windows` distinct windows with `share` paths each: the entries built under
// `limit`, and whether every path is reached from its window
static void run(uint32_t windows, uint32_t share, size_t limit) {
    std::vector<uint64_t> pairs;
    for (uint32_t w = 0; w < windows; ++w)
        for (uint32_t k = 0; k < share; ++k) pairs.push_back(uint64_t(w * 2654435761u) << 32 | (w * share + k));
    std::stable_sort(pairs.begin(), pairs.end(), [](uint64_t a, uint64_t b) { return a >> 32 < b >> 32; });
    WindowTable W;
    const bool ok = build_windows(pairs, [](int32_t s) { return WindowEntry{s, 8, s, 1u}; }, W, limit);
    size_t reached = 0;
    for (size_t i = 0; i < W.keys.size(); ++i)
        if (W.entries[i].len)
            for (size_t j = i;; j = (W.entries[j].link >> 4) - 1) {
                ++reached;
                if (!(W.entries[j].link >> 4)) break;
            }
    std::printf("%d %d %zu %zu %zu\n", ok, W.bits, W.keys.size(), W.entries.size(), reached);
}

int main() {
    std::printf("%zu\n", kMaxWindowEntries);
    run(1000, 1, 2048);     // 2048 slots: fits
    run(1000, 1, 2047);     // one too few
    run(1000, 5, 6048);     // 2048 slots and 4000 linked entries: fits
    run(1000, 5, 6047);
    run(1, 5000, 16 + 4999);
    run(1, 5000, 16 + 4998);
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("window_limit")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                    f"-I{ROOT}/paper_1412_7789_amd/csrc", str(d / "main.cpp"), "-o", str(d / "main")],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([str(d / "main")], check=True, capture_output=True, text=True).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


def test_a_table_past_the_limit_is_left_out(lines):
    empty = [0, 0, 0, 0, 0]
    assert lines[1:] == [[1, 11, 2048, 2048, 1000], empty, [1, 11, 2048, 6048, 5000], empty,
                         [1, 4, 16, 5015, 5000], empty]


def test_the_limit_is_what_a_link_can_hold(lines):
    (limit,) = lines[0]
    last = limit - 1                     # the last entry's index
    assert ((last + 1) << 4) & 0xFFFFFFFF == (last + 1) << 4
    assert ((last + 2) << 4) & 0xFFFFFFFF != (last + 2) << 4


@pytest.mark.parametrize("n,alphabet,tables", [
    (60_000, 256, (True, True)),      # 120,000 windows at stride 2, 240,000 at stride 4
    (66_000, 256, (False, False)),    # 132,000 and 264,000
    (100_000, 40, (True, False)),     # at most 64,000 3-byte windows: stride 2 is a default
], ids=["both", "neither", "stride 2"])
def test_tables_exist_where_default_launches_use_them(n, alphabet, tables):
    """Both tables would take 20 bytes of device memory per slot; the 4-byte
    windows' maps and counts are there either way."""
    import numpy as np

    import paper_1412_7789_amd as pf
    from paper_1412_7789_amd import _lib as L

    rng = np.random.default_rng(n)
    kws = [bytes(k) for k in rng.integers(0, alphabet, size=(n, 8), dtype=np.uint8)]
    plan = pf.Plan(kws)
    info = plan.info()
    for stride, (keys, entries), wanted, windows in (
            (2, (L.AC_TABLE_WINDOW2_KEYS, L.AC_TABLE_WINDOW2_ENTRIES), tables[0], info["n_quads2"]),
            (4, (L.AC_TABLE_WINDOW4_KEYS, L.AC_TABLE_WINDOW4_ENTRIES), tables[1], info["n_quads4"])):
        assert windows == len({k[j:j + 4] for k in kws for j in range(1, stride + 1)})
        assert (len(plan.export(keys, np.uint32)) > windows) == wanted
        assert (len(plan.export(entries, np.int32)) > 0) == wanted
        pair = plan.export(L.AC_TABLE_FILTER_BASE + 6 * (stride // 2) + L.AC_FILTER_PAIR20, np.uint8)
        assert len(pair) == 1 << 17
