// HIP kernels (gfx950) of the failure-less Aho-Corasick matcher.
//
// The method (paper, Section II; Fig. 3 "N", Fig. 5): every byte offset o of
// the text starts a walk of the Goto trie at the root, follows T[o], T[o+1],
// ... while transitions exist, and reports every keyword whose state it
// enters.  No failure links are used.  Two kernels compute it:
//
// filtered_kernel (default).  A wave owns a 1-4 KiB chunk of text per step:
//   each lane holds 16 contiguous bytes per 1 KiB segment in VGPRs (one
//   coalesced 16-byte load; the halo comes from the next lane), and tests them
//   against a hashed filter in LDS: at stride 1 the first K = min(3, shortest
//   keyword) bytes of every offset, at strides 2 and 4 every second or fourth
//   window against the keywords' windows.  What is not in the filter cannot
//   start a keyword (its walk dies without reaching a final state), so only
//   the rare candidates are queued (wave ballot + prefix count into a per-wave
//   LDS queue), looked up in an exact table, 64 at a time, and walked through
//   the transition table in global memory (L2-resident rows; dense rows for
//   shallow states, compact child lists for deep ones) or compared with the
//   one keyword their window belongs to.
//
// direct_kernel (plain PFAC).  A block stages its text tile plus a halo of
//   (longest keyword - 1) bytes in LDS and walks every offset from the root
//   through the dense table, itself in LDS when it fits.
//
// The filtered kernel stages matches in LDS, and one atomic per block reserves
// their output slots; the direct kernel reserves a slot per match.  The count is exact even when
// the output buffer is too small (only `cap` entries are written).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstdio>
#include <mutex>

#include "filtered.hpp"

namespace pfac {

using namespace dev;

namespace {

// ---------------------------------------------------------------------------
struct DirectLaunch {
    int64_t tile;          // offsets per block
    int32_t table_bytes;   // dense table bytes staged in LDS (0 = global)
    int32_t halo;          // longest keyword - 1
};

template <bool TABLE_LDS>
__global__ __launch_bounds__(1024) void direct_kernel(const DevAut A, const ScanArgs S, const DirectLaunch L) {
    extern __shared__ __align__(16) uint8_t smem[];
    uint8_t *scls = smem;
    int32_t *stab = reinterpret_cast<int32_t *>(smem + 256);
    uint8_t *stext = smem + 256 + (TABLE_LDS ? L.table_bytes : 0);
    if (threadIdx.x < 64) reinterpret_cast<uint32_t *>(scls)[threadIdx.x] =
        reinterpret_cast<const uint32_t *>(A.cls)[threadIdx.x];
    if (TABLE_LDS) {
        const uint4 *src = reinterpret_cast<const uint4 *>(A.dense);
        uint4 *dst = reinterpret_cast<uint4 *>(stab);
        for (int i = threadIdx.x; i < L.table_bytes / 16; i += blockDim.x) dst[i] = src[i];
    }
    const int64_t t0 = int64_t(blockIdx.x) * L.tile;
    const int64_t t1 = lmin(t0 + L.tile, S.n);
    const int64_t h1 = lmin(t1 + L.halo, S.n);
    for (int64_t i = threadIdx.x; i < h1 - t0; i += blockDim.x) stext[i] = S.text[t0 + i];
    __syncthreads();
    for (int64_t o = t0 + threadIdx.x; o < t1; o += blockDim.x) {
        int32_t s = 0;
        for (int64_t j = o; j < h1; ++j) {
            const uint32_t b = stext[j - t0];
            int32_t e;
            if (TABLE_LDS) e = stab[s * A.C + scls[b]];
            else e = step_global(A, scls, s, b);
            if (e == 0) break;
            s = e & 0x7fffffff;
            if (e < 0) emit(A, S, o, 0, s);
        }
    }
}

// Clears a count, the scratch's words (if given) and the per-text counts.
__global__ void zero_kernel(unsigned long long *count, unsigned long long *words, int64_t *per_text, int32_t n_texts) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i == 0) *count = 0ull;
    if (i == 0 && words) words[0] = words[kScanCount] = 0ull;
    if (per_text && i < n_texts) per_text[i] = 0;
}

// Achievable-bandwidth probe: every lane streams 16-byte words and folds them
// into one value, written once per wave so the loads cannot be dropped.  The
// loads are non-temporal, as the scan's stream loads are.
__global__ __launch_bounds__(256) void probe_read_kernel(const uint8_t *buf, int64_t n16, uint32_t *out) {
    uint32_t acc = 0;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride) {
        const u32x4 v = __builtin_nontemporal_load((const global_u32x4 *)(buf + i * 16));
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    for (int d = 32; d >= 1; d >>= 1) acc ^= __shfl_xor(acc, d);
    if (lane_id() == 0 && acc == 0x9E3779B9u) *out = acc;   // practically never taken
}

// strides 2 and 4 exist for K = 3 only; `win`: with the stride's window table
FilteredFn pick_filtered(int K, int kind, int segs, int stride, bool win) {
    if (win) return stride == 4 ? pick_filtered_s4w(kind, segs) : pick_filtered_s2w(kind, segs);
    if (stride == 4) return pick_filtered_s4(kind, segs);
    if (stride == 2) return pick_filtered_s2(kind, segs);
    if (K == 1) return pick_filtered_s1k1(kind, segs);
    if (K == 2) return pick_filtered_s1k2(kind, segs);
    return pick_filtered_s1k3(kind, segs);
}

int64_t filtered_lds(const FilterGeom &g) {
    const int64_t pt_slots = g.bytes > (64 << 10) ? 0 : 8192;
    return g.bytes + int64_t(kMaxWaves) * kQueueCap * 4 + pt_slots * 8 + int64_t(kMaxWaves) * kLdsHits * 8;
}

// Launch geometry of the filtered policy for a text of n bytes at `addr`.
struct FilteredGeom {
    FilterLaunch F;
    int64_t grid, waves;
};

FilteredGeom filtered_geom(const ac_automaton *a, const uint8_t *text, int64_t n, const ac_launch &cfg) {
    FilteredGeom G{};
    FilterLaunch &F = G.F;
    const uintptr_t addr = reinterpret_cast<uintptr_t>(text);
    F.base = reinterpret_cast<const uint8_t *>(addr & ~uintptr_t(15));
    F.mis = int64_t(addr & 15);
    F.V = F.mis + n;
    const int64_t CH = int64_t(cfg.segs) * kSegBytes;
    F.n_chunks = (F.V + CH - 1) / CH;
    F.c_hi = F.V >= 16 ? (F.V - 16) / CH : 0;
    F.filter = a->dfilter[stride_set(cfg.stride) * kNumFilterKinds + cfg.filter - 1];
    if (cfg.stride > 1) {
        const int ws = window_set(cfg.stride);
        F.win_keys = a->dwin_keys[ws];
        F.win_entries = reinterpret_cast<const int4 *>(a->dwin_entries[ws]);
        F.win_nb = a->host.win[ws].bits - 2;
    }
    const int waves = cfg.block / kWave;
    const int64_t want = (F.n_chunks + waves - 1) / waves;
    const int64_t cap = int64_t(a->cu_count) * cfg.grid_per_cu;
    G.grid = std::max<int64_t>(1, std::min(want, cap));
    G.waves = G.grid * waves;
    return G;
}

// Launch through hipExtLaunchKernel when start/stop events are wanted (they
// are then taken from the kernel's own dispatch packet), else hipLaunchKernel.
hipError_t launch_timed(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream,
                        hipEvent_t start, hipEvent_t stop) {
    if (start || stop) return hipExtLaunchKernel(fn, grid, block, args, lds, stream, start, stop, 0);
    return hipLaunchKernel(fn, grid, block, args, lds, stream);
}

std::mutex g_attr_mu;

void allow_lds(const void *fn, int64_t bytes) {
    // Raise the dynamic-LDS limit of a kernel once (160 KiB per CU on gfx950).
    std::lock_guard<std::mutex> lk(g_attr_mu);
    (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

}  // namespace

void resolve_launch(const ac_automaton *a, int64_t len, bool batch, ac_launch &cfg) {
    const Plan &P = a->host;
    if (cfg.policy == AC_POLICY_AUTO) cfg.policy = AC_POLICY_FILTERED;
    if (batch) cfg.policy = AC_POLICY_FILTERED;
    if (cfg.policy == AC_POLICY_FILTERED) {
        // Sampling stride and map, chosen by the number of keys the map must
        // hold and the text's length.  A stride of s divides the probes by s
        // but holds s windows per keyword.  A positive costs one lookup in the
        // exact window table (keywords of s + 4 bytes), so the longest stride
        // wins until the map lets too many through.  Measured on MI355X (kernel
        // us; stride/map/segments, maps by their AC_FILTER number):
        //   1 GiB     1000 printable keywords (4000 windows at stride 4)
        //             4/6/2 166, 2/6/4 170; 5000 byte keywords (20000)
        //             4/6/2 158, 2/6/4 163; 20000 (80000) 4/6/2 213,
        //             2/6/4 184; 50000 (200000) 4/6/2 421, 2/6/4 277
        //   256 MiB   5000 46.9 and 49.5, 20000 58.8 and 55.2 (57.4 both when a
        //             third share prefixes), 50000 113 and 77
        //   200 MiB   20000 47.2 and 46.4, with shared prefixes 46.0 and 48.0
        //   64 MiB    5000 18.4 and 21.6 (2/6/2), 20000 22.0 and 23.4, 50000
        //             34.5 and 27.8
        //   4 MiB     50000 keywords 4/6/2 9.8, 2/6/2 9.9, stride 1 11.8;
        //             5000 4/4/2 8.6, 4/6/2 8.8, 2/4/1 9.6; 1000 4/4/2 10.2,
        //             4/6/2 10.3, 2/4/1 11.6
        //   64 KiB    50000 keywords 4/6/1 7.2, stride 1 8.3
        // So stride 4 up to kPair4Keys windows, up to kPair4MidKeys on texts
        // short enough that fixed costs weigh as much as the stream, and up to
        // kPair4SmallKeys on small ones, which see few positives in all; else
        // stride 2 up to kPair2Keys, with the 4-byte-window map.  The window
        // tables exist where these rules choose their stride.  Without one
        // (windows on many paths) a positive costs a prefix lookup for each of
        // its offsets, and stride 4 is left to texts of 16 MiB and more and sets
        // of up to kPair4PrefixKeys windows (32 MiB of prose-like words, 2000 of
        // them, 4500 windows: 4/6/2 294, 2/6/2 284, stride 1 464).  Small texts
        // take the 64 KiB bit map while its keys are few: less to stage, and
        // room for the window keys beside it.
        const bool auto_filter = cfg.filter < AC_FILTER_BYTES17 || cfg.filter > AC_FILTER_PAIR20;
        const bool auto_stride = cfg.stride != 1 && cfg.stride != 2 && cfg.stride != 4;
        const bool small_text = len < (int64_t(16) << 20);
        if (auto_stride) {
            const int32_t most4 = P.win[window_set(4)].bits == 0 ? (small_text ? 0 : kPair4PrefixKeys)
                                  : small_text                   ? kPair4SmallKeys
                                  : len < (int64_t(256) << 20)   ? kPair4MidKeys
                                                                 : kPair4Keys;
            if (auto_filter && P.pair4 && P.n_quads4 <= most4) {
                cfg.stride = 4;
                cfg.filter = small_text && P.n_quads4 <= kPair4Keys ? AC_FILTER_BITS19 : AC_FILTER_PAIR20;
            } else if (P.sampled && (P.n_windows2 <= kStride2Keys ||
                                     (auto_filter && !small_text && P.pair2 && P.n_quads2 <= kPair2Keys))) {
                cfg.stride = 2;
                if (auto_filter && !small_text && P.pair2 && P.n_quads2 <= kPair2Keys) cfg.filter = AC_FILTER_PAIR20;
            } else {
                cfg.stride = 1;
            }
        }
        if (cfg.stride == 4 && !P.sampled4) cfg.stride = P.sampled ? 2 : 1;
        if (cfg.stride == 2 && !P.sampled) cfg.stride = 1;
        // the 4-byte-window map needs its stride's windows
        if (cfg.filter == AC_FILTER_PAIR20 && !((cfg.stride == 4 && P.pair4) || (cfg.stride == 2 && P.pair2)))
            cfg.filter = AC_FILTER_AUTO;
        if (cfg.filter < AC_FILTER_BYTES17 || cfg.filter > AC_FILTER_PAIR20) {
            // keys in the filter: prefixes (stride 1) or windows (strides 2, 4)
            const int64_t keys = cfg.stride == 4 ? P.n_windows4 : cfg.stride == 2 ? P.n_windows2 : P.n_prefixes;
            // A few prefixes at stride 1 keep the 64 KiB byte map, with the
            // prefix table in LDS beside it, up to 128 MiB (200 keywords of 2
            // to 8 bytes, 64 MiB: 33.1 us against 35.6 with the 128 KiB map;
            // 64 keywords of 4 to 12 bytes: 64 MiB 26.8 and 28.0, 256 MiB
            // 112.0 and 107.1).
            if (small_text || (cfg.stride == 1 && keys <= 1500 && len < (int64_t(128) << 20)))
                cfg.filter = keys > 1500 ? AC_FILTER_BITS19 : AC_FILTER_BYTES16;
            else if (keys <= 1500) cfg.filter = AC_FILTER_BYTES17;
            else if (keys <= 8192) cfg.filter = AC_FILTER_BITS20;
            else if (cfg.stride == 2 || keys > 20000) cfg.filter = AC_FILTER_DUAL19;
            else cfg.filter = AC_FILTER_BITS20;
        }
        FilterGeom g = filter_geom(cfg.filter);
        if (filtered_lds(g) > a->lds_per_block) {
            // the 128 KiB maps need a 160 KiB LDS; fall back to the 64 KiB ones
            if (cfg.filter == AC_FILTER_BYTES17) cfg.filter = AC_FILTER_BYTES16;
            if (cfg.filter == AC_FILTER_BITS20 || cfg.filter == AC_FILTER_DUAL19 || cfg.filter == AC_FILTER_PAIR20)
                cfg.filter = AC_FILTER_BITS19;
            g = filter_geom(cfg.filter);
        }
        if (cfg.block != 256 && cfg.block != 512 && cfg.block != 1024) cfg.block = 1024;
        // One segment per wave step for the shortest texts, which spreads
        // them over more waves, two from 3 MiB on: 1000 keywords, 4/4 (us): 512
        // KiB 8.8 with one, 9.6 with two, 2 MiB 9.7 and 9.5, 3 MiB 10.6 and
        // 9.8, 4 MiB 11.5 and 10.2; 50000 keywords, 2 MiB 8.9 and 9.5; 200 short
        // keywords at stride 1, 1 MiB 10.2 and 11.6, 2 MiB 10.6 and 11.4, 3 MiB
        // 11.4 and 11.6, 4 MiB 12.3 and 11.9.  Without a window table two only
        // from 8 MiB, where every wave has a step with either: many candidates
        // keep a wave busy and fill its records, so half of the waves cannot be
        // left idle (calls, 63 keywords of 4 to 6 letters of ACGT, 4 MiB 73 and
        // 507, 6 MiB 515 and 730, 8 MiB 956 and 953; 500 short words in prose, 4
        // MiB 47 and 66, 6 MiB 66 both).  Four for the 4-byte-window map at
        // stride 2 on texts of 256 MiB and more, where they halve the per-step
        // work of a filter-bound loop (20000 byte keywords: 256 MiB 55.2 with
        // four, 57.0 with two, 1 GiB 184 and 193; 50000: 192 MiB 60.4 and 60.2,
        // 256 MiB 77.4 both, 1 GiB 277 and 285); with the 4-byte-window map at
        // stride 4 four are slower (1000 keywords, 1 GiB: 171 and 166).
        if (cfg.segs != 1 && cfg.segs != 2 && cfg.segs != 4) {
            const bool win = cfg.stride > 1 && P.win[window_set(cfg.stride)].bits > 0;
            cfg.segs = len < (int64_t(win ? 3 : 8) << 20) ? 1 : 2;
            if (cfg.filter == AC_FILTER_PAIR20 && cfg.stride == 2 && len >= (int64_t(256) << 20)) cfg.segs = 4;
        }
        const int64_t fit = std::max<int64_t>(1, a->lds_per_cu / filtered_lds(g));
        if (cfg.grid_per_cu <= 0 || cfg.grid_per_cu > fit) cfg.grid_per_cu = int32_t(fit);
    } else {
        if (cfg.block != 256 && cfg.block != 512 && cfg.block != 1024) cfg.block = 256;
        const int64_t table_bytes = int64_t(P.S_dense) * P.C * 4;
        const bool fits = P.S_dense == P.S && table_bytes + 256 + 8192 + P.max_len + 64 <= a->lds_per_block;
        if (cfg.table_in_lds == 1 && !fits) cfg.table_in_lds = 2;
        if (cfg.table_in_lds != 1 && cfg.table_in_lds != 2) cfg.table_in_lds = fits ? 1 : 2;
    }
}

int launch_probe_read(const uint8_t *buf, int64_t n, uint32_t *out, hipStream_t stream, std::string &err) {
    if (n <= 0) return AC_OK;
    int dev = 0, cus = 1;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t n16 = n / 16;
    const int64_t grid = std::max<int64_t>(1, std::min<int64_t>((n16 + 255) / 256, int64_t(cus) * 8));
    probe_read_kernel<<<unsigned(grid), 256, 0, stream>>>(buf, n16, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { err = std::string("probe launch: ") + hipGetErrorString(e); return AC_EHIP; }
    return AC_OK;
}

int launch_zero(unsigned long long *count, unsigned long long *words, int64_t *per_text, int32_t n_texts,
                hipStream_t stream, std::string &err) {
    const int32_t threads = 256;
    const int32_t blocks = std::max<int32_t>(1, (std::max<int32_t>(n_texts, 1) + threads - 1) / threads);
    zero_kernel<<<blocks, threads, 0, stream>>>(count, words, per_text, n_texts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { err = std::string("zero_kernel launch: ") + hipGetErrorString(e); return AC_EHIP; }
    return AC_OK;
}

int64_t scan_regions(const ac_automaton *a, const uint8_t *text, int64_t n, const ac_launch &cfg) {
    if (cfg.policy != AC_POLICY_FILTERED || n <= 0) return 0;
    return filtered_geom(a, text, n, cfg).waves;
}

int64_t widest_scan_regions(int cu_count, int64_t lds_per_cu) {
    // a filtered launch has at most (LDS per CU / the smallest filter's LDS)
    // blocks per CU, each of at most kMaxWaves waves
    return int64_t(cu_count) * std::max<int64_t>(1, lds_per_cu / filtered_lds(filter_geom(AC_FILTER_BITS19))) *
           kMaxWaves;
}

int launch_scan(const ac_automaton *a, const ScanArgs &S, const ac_launch &cfg, const HitScratch &hs,
                hipStream_t stream, std::string &err, const KernelTiming *timing) {
    const KernelTiming none;
    const KernelTiming &T = timing ? *timing : none;
    if (S.n <= 0) return AC_OK;
    const Plan &P = a->host;
    hipError_t e = hipSuccess;
    if (cfg.policy == AC_POLICY_FILTERED) {
        FilteredGeom G = filtered_geom(a, S.text, S.n, cfg);
        FilterLaunch &F = G.F;
        if (!hs.hits || hs.regions < G.waves || hs.cap < kDrain) {
            err = "scan scratch too small for the launch";
            return AC_EINVAL;
        }
        F.hits = hs.hits;
        F.hit_cap = hs.cap;
        // queue entries hold (slot << 12 | position): a block's slots must fit 20 bits
        if (F.n_chunks / G.grid + 2 * (cfg.block / kWave) >= (int64_t(1) << 20)) {
            err = "text too large for one launch";
            return AC_EINVAL;
        }
        const bool win = F.win_keys != nullptr;
        FilteredFn fn = pick_filtered(P.K, cfg.filter, cfg.segs, cfg.stride, win);
        if (!fn) { err = "no kernel for this filter and stride"; return AC_EINVAL; }
        KArgs KA{a->dev, S, F};
        void *fargs[] = {&KA};
        e = launch_timed(reinterpret_cast<const void *>(fn), dim3(unsigned(G.grid)), dim3(unsigned(cfg.block)), fargs, 0,
                         stream, T.scan0, T.scan1);
        if (e != hipSuccess) { err = std::string("scan launch: ") + hipGetErrorString(e); return AC_EHIP; }
    } else if (cfg.policy == AC_POLICY_DIRECT) {
        if (S.text_off) { err = "direct policy does not scan batches"; return AC_ENOTSUP; }
        DirectLaunch L;
        L.tile = 8192;
        L.halo = P.max_len - 1;
        const bool lds_table = cfg.table_in_lds == 1;
        L.table_bytes = lds_table ? int32_t((int64_t(P.S_dense) * P.C * 4 + 15) / 16 * 16) : 0;
        const int64_t lds = 256 + L.table_bytes + L.tile + L.halo + 16;
        const int64_t grid = (S.n + L.tile - 1) / L.tile;
        if (lds > a->lds_per_block) { err = "direct policy: tile and table exceed LDS"; return AC_ENOTSUP; }
        auto fn = lds_table ? direct_kernel<true> : direct_kernel<false>;
        allow_lds(reinterpret_cast<const void *>(fn), lds);
        DevAut A = a->dev;
        ScanArgs SA = S;
        void *dargs[] = {&A, &SA, &L};
        e = launch_timed(reinterpret_cast<const void *>(fn), dim3(unsigned(grid)), dim3(unsigned(cfg.block)), dargs,
                         size_t(lds), stream, T.scan0, T.scan1);
    } else {
        err = "unknown policy";
        return AC_EINVAL;
    }
    if (e != hipSuccess) { err = std::string("scan launch: ") + hipGetErrorString(e); return AC_EHIP; }
    return AC_OK;
}

}  // namespace pfac
