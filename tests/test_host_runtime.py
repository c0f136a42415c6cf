"""Host code of the GPU entry points on a HIP runtime made of host memory
(CPU only): small programs include the library's host sources and stand in for
the kernel launches, so what a call leaves behind can be set up and read."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

# stands in for kernels.hip: a scan counts with the CPU matcher the way the
# kernel does, adding to the count word and handing it out at the end
PRELUDE = r"""
#include "fake_hip.hpp"
#include "plan.cpp"
#include "host_match.cpp"
#include "capi.cpp"
#include "serve.cpp"
#include <cstdio>

namespace pfac {
void resolve_launch(const ac_automaton *, int64_t, bool, ac_launch &cfg) {
    if (!cfg.policy) cfg.policy = AC_POLICY_FILTERED;
}
int64_t scan_regions(const ac_automaton *, const uint8_t *, int64_t, const ac_launch &) { return 32; }
int64_t widest_scan_regions(int, int64_t) { return 32; }
int launch_probe_read(const uint8_t *, int64_t, uint32_t *, hipStream_t, std::string &) { return AC_OK; }
int launch_zero(unsigned long long *count, unsigned long long *words, int64_t *per_text, int32_t n_texts, hipStream_t,
                std::string &) {
    *count = 0;
    if (words) words[0] = words[kScanCount] = 0;
    for (int32_t t = 0; per_text && t < n_texts; ++t) per_text[t] = 0;
    return AC_OK;
}
int launch_scan(const ac_automaton *a, const ScanArgs &S, const ac_launch &, const HitScratch &, hipStream_t,
                std::string &, const KernelTiming *) {
    if (S.n <= 0) return AC_OK;
    if (S.near_cap > 0) {
        // the pinned arrays' entries arrive at once, later, in part later, or never
        std::vector<int64_t> off(size_t(S.near_cap));
        std::vector<int32_t> pid(size_t(S.near_cap));
        const int64_t n = std::min(S.near_cap, host_match(a->host, S.text, S.n, off.data(), pid.data(), S.near_cap, 1));
        auto put = [=](int64_t i0, int64_t i1) {
            for (int64_t i = i0; i < i1; ++i) {
                __atomic_store_n(S.near_pid + i, pid[size_t(i)], __ATOMIC_RELAXED);
                __atomic_store_n(S.near_off + i, off[size_t(i)], __ATOMIC_RELAXED);
            }
        };
        switch (fake::late) {
            case 0: put(0, n); break;
            case 1: fake::later([=] { put(0, n); }); break;
            case 2: put(0, n - 1); fake::later([=] { put(n - 1, n); }); break;
            case 3: put(1, n); fake::later([=] { put(0, 1); }); break;
            case 4: put(0, n / 2); fake::later([=] { put(n / 2, n); }); break;
            default: put(0, n / 2);
        }
    }
    int64_t n = 0;
    for (int32_t t = 0; t < (S.text_off ? S.n_texts : 1); ++t) {
        const int64_t at = S.text_off ? S.text_off[t] : 0, end = S.text_off ? S.text_off[t + 1] : S.n;
        const int64_t room = S.near_cap > 0 ? 0 : std::max<int64_t>(0, S.cap - n);
        const int64_t m = host_match(a->host, S.text + at, end - at, S.out_off + n, S.out_pid + n, room, 1);
        for (int64_t i = n; S.out_tid && i < std::min(n + m, S.cap); ++i) S.out_tid[i] = t;
        n += m;
    }
    *S.count += uint64_t(n);
    if (S.done && S.done[0] != 0) return AC_OK;      // counts of another scan: no block is the last
    if (S.dev_count) { *S.dev_count = *S.count; *S.count = 0; }
    if (S.host_count) { S.host_count[0] = *S.count; S.host_count[1] = report_tag(*S.count, S.host_seq); }
    return AC_OK;
}
}  // namespace pfac
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (%s)\n", __LINE__, #c, ac_last_error()); return 1; } } while (0)
const uint8_t *kText = reinterpret_cast<const uint8_t *>("abcdefgh-abcdefgh-abcdefgh");
const int64_t kLen = 26;
ac_automaton *make() {
    const int64_t offs[2] = {0, 8};
    ac_automaton *a = nullptr;
    return ac_build_csr(kText, offs, 1, nullptr, &a) == AC_OK ? a : nullptr;
}
"""


def run(tmp_path, source, prelude=PRELUDE):
    (tmp_path / "main.cpp").write_text(prelude + source)
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_1412_7789_amd/csrc", f"-I{ROOT}/tests",
                    str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main"), "-lpthread"], check=True)
    res = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr


def test_counts_left_by_overlapping_scans_are_cleared(tmp_path):
    """Asynchronous scans count in words of their scratch that are zero between
    scans.  Scans that overlapped against the rules may leave something
    there; an asynchronous call of an empty text puts the words back to
    zero, the array's of ac_match_async_noalloc and a stream's, and a
    synchronous call that clears its count does so for its stream's."""
    run(tmp_path, r"""
int main() {
    ac_automaton *a = make();
    CHECK(a);
    int64_t count = -1;
    CHECK(ac_match_async_noalloc(a, kText, kLen, nullptr, nullptr, &count, nullptr) == AC_OK && count == 3);
    scratch_words[0] = 5;
    scratch_words[kScanCount] = 7;
    CHECK(ac_match_async_noalloc(a, kText, 0, nullptr, nullptr, &count, nullptr) == AC_OK && count == 0);
    CHECK(ac_match_async_noalloc(a, kText, kLen, nullptr, nullptr, &count, nullptr) == AC_OK && count == 3);

    CHECK(ac_match_async(a, kText, kLen, nullptr, nullptr, &count, nullptr) == AC_OK && count == 3);
    CountSlot &slot = g_slots.begin()->second;
    auto poison = [&] { slot.hs.words[0] = 5; slot.hs.words[kScanCount] = 7; };
    poison();
    CHECK(ac_match_async(a, kText, 0, nullptr, nullptr, &count, nullptr) == AC_OK && count == 0);
    CHECK(ac_match_async(a, kText, kLen, nullptr, nullptr, &count, nullptr) == AC_OK && count == 3);

    poison();
    slot.stale = true;
    CHECK(ac_match(a, kText, kLen, nullptr, nullptr) == 3);
    CHECK(ac_match_async(a, kText, kLen, nullptr, nullptr, &count, nullptr) == AC_OK && count == 3);
    CHECK(ac_match(a, kText, kLen, nullptr, nullptr) == 3);
    ac_free(a);
    return 0;
}
""")


def test_server_goes_on_after_a_failed_allocation(tmp_path):
    """A request whose buffers cannot be allocated fails with AC_ENOMEM; the
    stream's buffers that were given up for it are allocated again for the next
    one: the text's, and each of the match arrays' (a re-scan that needs more)."""
    run(tmp_path, r"""
int main() {
    ac_automaton *a = make();
    CHECK(a);
    ac_server_opts o{};
    o.n_streams = 1;
    o.max_batch_bytes = 4096;
    o.max_batch_texts = 4;
    o.matches_per_kib = 1;
    ac_server *s = nullptr;
    CHECK(ac_server_create(&o, &s) == AC_OK);
    CHECK(ac_server_add_automaton(s, a) == 0);
    std::vector<uint8_t> text;
    ac_request_result r{};
    auto serve = [&](int64_t len) {
        const int64_t id = ac_server_submit(s, 0, text.data(), len);
        return id < 0 ? int(id) : ac_server_wait(s, id, &r);
    };
    text.assign(1 << 20, '.');
    std::memcpy(text.data(), "abcdefgh", 8);
    fake::fail_in = 0;
    CHECK(serve(1 << 20) == AC_ENOMEM);
    CHECK(serve(1000) == AC_OK && r.count == 1 && r.offset[0] == 0);
    CHECK(serve(1 << 20) == AC_OK && r.count == 1);
    for (size_t at = 0; at < text.size(); at += 8) std::memcpy(text.data() + at, "abcdefgh", 8);
    for (int array = 0; array < 3; ++array) {
        const int64_t len = int64_t(1) << (15 + array);
        fake::fail_in = array;
        CHECK(serve(len) == AC_ENOMEM);
        CHECK(serve(800) == AC_OK && r.count == 100 && r.pattern_id[99] == 0);
        CHECK(serve(len) == AC_OK && r.count == len / 8);
    }
    ac_server_destroy(s);
    ac_free(a);
    return 0;
}
""")


def test_matches_that_arrive_after_their_count(tmp_path):
    """A kernel's stores to pinned memory may reach the host after the count that
    reports them.  A dispatched call waits for each entry, whether the last ones
    come late or the first, and never returns what an earlier call left; if the
    stream ends without them the call fails, and the next one works."""
    run(tmp_path, r"""
int main() {
    ac_automaton *a = make();
    CHECK(a);
    ac_set_dispatch_threshold(a, 0);
    std::vector<uint8_t> text(60000, '.');
    std::vector<int64_t> off(8000);
    std::vector<int32_t> pid(8000);
    auto call = [&] { return ac_match_dispatch(a, text.data(), int64_t(text.size()), off.data(), pid.data(), 8000, nullptr, nullptr); };
    for (int round = 0; round < 12; ++round) {
        // round + 1 bytes between the matches, so every round has other ones
        std::fill(text.begin(), text.end(), '.');
        int64_t n = 0;
        for (size_t at = 0; at + 8 <= text.size(); at += size_t(9 + round), ++n) std::memcpy(text.data() + at, "abcdefgh", 8);
        fake::late = round % 6;
        const int64_t count = call();
        CHECK(fake::late == 5 ? count == AC_EHIP : count == n);
        fake::join();
        if (count < 0) continue;
        for (int64_t i = 0; i < n; ++i) CHECK(off[size_t(i)] == i * (9 + round) && pid[size_t(i)] == 0);
    }
    ac_free(a);
    return 0;
}
""")
