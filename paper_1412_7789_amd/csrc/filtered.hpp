// Device side of the filtered scan: helpers, the candidate filter, the
// walk and the streaming kernel (templates), shared by the kernel library's
// translation units.  Each filtered_*.hip file instantiates the kernels of
// one sampling stride (and, at stride 1, one prefix length), so they compile
// in parallel; kernels.hip holds the other kernels and the launch code.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "pfac_internal.hpp"

namespace pfac {
namespace dev {

constexpr int kQueueCap = 256;   // per-wave candidate queue (dwords, two per entry)
// Hit records a wave keeps in LDS before it spills further ones to its
// global region.  Global stores in the streaming loop stall it (a later wait
// for the next chunk's loads also waits for them, and the data registers a
// store reads cannot be reused until it is done), so records stay on chip.
constexpr int kLdsHits = 128;
constexpr int kDrain = 64;       // candidates taken per drain (1 per lane; 128 and 192 measured slower)
// A queue holds fewer than kDrain entries before a round and gains at most
// one per lane in it, so its last dwords are never used by the queue: the last
// one of the first wave's queue holds the block's slot counter.
static_assert(2 * (2 * kDrain - 1) < kQueueCap, "queue room");
constexpr int kMaxWaves = 16;    // waves per block at most (1024 threads)
// (queue entry, keyword id) pairs a wave's queue holds as its match stage,
// after its count and before the slot counter
constexpr int kWaveStageCap = (kQueueCap - 4) / 2;

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }

__device__ __forceinline__ int64_t lmin(int64_t a, int64_t b) { return a < b ? a : b; }

__device__ __forceinline__ unsigned lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

__device__ __forceinline__ unsigned rank_in(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi(unsigned(mask >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(mask), 0u));
}

__device__ __forceinline__ unsigned long long readlane64(unsigned long long v, int lane) {
    unsigned lo = __builtin_amdgcn_readlane(unsigned(v), lane);
    unsigned hi = __builtin_amdgcn_readlane(unsigned(v >> 32), lane);
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// Third descriptor word of a raw (untyped, unswizzled) buffer on gfx9-family GPUs.
constexpr int kBufferFlags = 0x00020000;

// Loads through an explicit global-address-space pointer: pointers taken out
// of a by-value struct otherwise lower to flat loads, which also occupy the
// LDS counter and would serialise with the filter lookups.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) u32x4 global_u32x4;
typedef const __attribute__((address_space(1))) uint32_t global_u32;

__device__ __forceinline__ u32x4 gload16(const uint8_t *p) { return *(global_u32x4 *)(p); }
__device__ __forceinline__ uint32_t gload4(const uint8_t *p) { return *(global_u32 *)(p); }
__device__ __forceinline__ uint32_t gload1(const uint8_t *p) {
    return *(const __attribute__((address_space(1))) uint8_t *)(p);
}
__device__ __forceinline__ void gstore16(uint4 *p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    u32x4 v;
    v.x = a;
    v.y = b;
    v.z = c;
    v.w = d;
    *(__attribute__((address_space(1))) u32x4 *)(p) = v;
}

__device__ __forceinline__ void gstore8(uint2 *p, uint32_t a, uint32_t b) {
    u32x2 v;
    v.x = a;
    v.y = b;
    *(__attribute__((address_space(1))) u32x2 *)(p) = v;
}
__device__ __forceinline__ uint2 gload8(const uint2 *p) {
    const u32x2 v = *(const __attribute__((address_space(1))) u32x2 *)(p);
    return make_uint2(v.x, v.y);
}

// Orders LDS traffic between lanes of one wave (queue producer -> consumer).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One match into slot idx of the caller's arrays, written through to the
// device so that it is in place without a cache writeback (report_count).
template <typename T>
__device__ __forceinline__ void write_through(T *p, T v) {
    __hip_atomic_store((__attribute__((address_space(1))) T *)(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_out(const ScanArgs &S, unsigned long long idx, int64_t off, int32_t tid,
                                        int32_t pid) {
    if (idx >= static_cast<unsigned long long>(S.cap)) return;
    const bool near = idx < static_cast<unsigned long long>(S.near_cap);
    write_through((near ? S.near_off : S.out_off) + idx, off);
    write_through((near ? S.near_pid : S.out_pid) + idx, pid);
    if (S.out_tid) write_through(S.out_tid + idx, tid);
}

// Reports every keyword id of final state s at `off` (relative to its text).
// Called from divergent code: the lanes calling it together share one atomic
// per round; lanes with more ids loop more rounds.
__device__ __forceinline__ void emit(const DevAut &A, const ScanArgs &S, int64_t off, int32_t tid, int32_t s) {
    const int32_t k0 = A.out_off[s], k1 = A.out_off[s + 1];
    for (int32_t k = k0; k < k1; ++k) {
        const unsigned long long act = __ballot(1);
        const unsigned rank = rank_in(act);
        const int leader = __ffsll(static_cast<long long>(act)) - 1;
        unsigned long long base = 0;
        if (rank == 0) base = atomicAdd(S.count, static_cast<unsigned long long>(__popcll(act)));
        base = readlane64(base, leader);
        const unsigned long long idx = base + rank - S.count_base;
        put_out(S, idx, off, tid, A.out_pid[k]);
        if (S.per_text) atomicAdd(reinterpret_cast<unsigned long long *>(S.per_text + tid), 1ull);
    }
}

// Block-level staging of matches in LDS: one global atomic per block instead
// of one per match.  Matches beyond the stage's capacity go straight out
// through emit().
constexpr int kStageCap = 3072;   // 48 KiB: fits, with the walk's bookkeeping, in the smallest filter's LDS
struct MatchStage {
    int64_t off[kStageCap];
    int32_t pid[kStageCap];
    int32_t tid[kStageCap];
    int32_t n;
    unsigned long long base;
};

// One more match of text tid: in the block's LDS counters when it has them,
// else in global memory.  A counter that wraps hands its 2^32 on.
__device__ __forceinline__ void count_text(const ScanArgs &S, uint32_t *lcnt, int32_t tid) {
    if (!S.per_text) return;
    unsigned long long more = 1ull;
    if (lcnt) {
        if (atomicAdd(&lcnt[tid], 1u) != ~0u) return;
        more = 1ull << 32;
    }
    atomicAdd(reinterpret_cast<unsigned long long *>(S.per_text + tid), more);
}

// A place in the block's stage for one match, kStageCap or more when it is full.
// A full stage's count is left alone: states may have any number of ids.
__device__ __forceinline__ int32_t stage_place(MatchStage *st) {
    if (__hip_atomic_load(&st->n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= kStageCap) return kStageCap;
    return atomicAdd(&st->n, 1);
}

__device__ __forceinline__ void emit_staged(const DevAut &A, const ScanArgs &S, MatchStage *st, uint32_t *lcnt,
                                            int64_t off, int32_t tid, int32_t s) {
    const int32_t k0 = A.out_off[s], k1 = A.out_off[s + 1];
    for (int32_t k = k0; k < k1; ++k) {
        const int32_t i = stage_place(st);
        if (i < kStageCap) {
            st->off[i] = off;
            st->pid[i] = A.out_pid[k];
            st->tid[i] = tid;
        } else {
            // stage full: this id goes out directly (one atomic)
            const unsigned long long idx = atomicAdd(S.count, 1ull) - S.count_base;
            put_out(S, idx, off, tid, A.out_pid[k]);
        }
        count_text(S, lcnt, tid);
    }
}

// One keyword id `pid` found at `off` (the caller knows it is the state's only one).
__device__ __forceinline__ void emit_one(const ScanArgs &S, MatchStage *st, uint32_t *lcnt, int64_t off, int32_t tid,
                                         int32_t pid) {
    int32_t i = kStageCap;
    if (st) i = stage_place(st);
    if (i < kStageCap) {
        st->off[i] = off;
        st->pid[i] = pid;
        st->tid[i] = tid;
    } else {
        const unsigned long long idx = atomicAdd(S.count, 1ull) - S.count_base;
        put_out(S, idx, off, tid, pid);
    }
    count_text(S, lcnt, tid);
}

// Called by every thread of the block: writes the staged matches out with one
// atomic, and empties the stage.
__device__ __forceinline__ void write_stage(const ScanArgs &S, MatchStage *st) {
    __syncthreads();
    const int32_t n = imin(st->n, kStageCap);
    __syncthreads();
    if (threadIdx.x == 0) {
        st->base = n ? atomicAdd(S.count, static_cast<unsigned long long>(n)) - S.count_base : 0ull;
        st->n = 0;
    }
    __syncthreads();
    for (int32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long idx = st->base + unsigned(i);
        put_out(S, idx, st->off[i], st->tid[i], st->pid[i]);
    }
}

// Called by every thread of the block once all its walks are done.
__device__ __forceinline__ void flush_stage(const ScanArgs &S, MatchStage *st, const uint32_t *lcnt) {
    __syncthreads();
    const int32_t n = imin(st->n, kStageCap);
    if (lcnt)
        for (int32_t i = threadIdx.x; i < S.n_texts; i += blockDim.x)
            if (const uint32_t c = lcnt[i])
                atomicAdd(reinterpret_cast<unsigned long long *>(S.per_text + i), static_cast<unsigned long long>(c));
    if (threadIdx.x == 0) st->base = n ? atomicAdd(S.count, static_cast<unsigned long long>(n)) - S.count_base : 0ull;
    __syncthreads();
    for (int32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long idx = st->base + unsigned(i);
        put_out(S, idx, st->off[i], st->tid[i], st->pid[i]);
    }
}

// One Goto transition out of state s on byte b; returns next | final bit, or 0.
__device__ __forceinline__ int32_t step_global(const DevAut &A, const uint8_t *cls, int32_t s, uint32_t b) {
    if (s < A.S_dense) return A.dense[static_cast<int64_t>(s) * A.C + cls[b]];
    const int32_t r = s - A.S_dense;
    const int32_t fc = A.node[2 * r];
    int32_t lo = 0, hi = A.node[2 * r + 1] & 0x7fffffff;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (A.label[fc + mid] < b) lo = mid + 1;
        else hi = mid;
    }
    if (lo < (A.node[2 * r + 1] & 0x7fffffff) && A.label[fc + lo] == b) {
        const int32_t t = fc + lo;
        return t | (A.node[2 * (t - A.S_dense) + 1] & kFinalBit);
    }
    return 0;
}

// 24 x 24-bit product, low 32 bits, unsigned (__umul24 itself returns int,
// whose right shift would sign-extend).
__device__ __forceinline__ uint32_t hash24(uint32_t x, uint32_t mul) {
    return static_cast<uint32_t>(__umul24(x, mul));
}

// Exact prefix lookup for the K-byte prefix x: returns {key, value} of its
// slot -- key = x | next byte << 24, value = state at depth K | has-next bit
// 30 | final bit 31 -- or value 0 when no keyword starts with x.  The table
// holds buckets of four {key, value} slots and x lies in one of its two
// buckets, so both are read at once and no further probing is needed.
constexpr uint32_t kHasNext = 0x40000000u;
constexpr uint32_t kStateMask = 0x3fffffffu;

template <typename LoadBucket>
__device__ __forceinline__ uint2 prefix_state(LoadBucket load, int bits, uint32_t x, uint32_t mul) {
    const int nb = bits - 2;
    const uint32_t b1 = hash24(x, mul) >> (32 - nb);
    uint32_t b2 = hash24(x, kPrefixMul2) >> (32 - nb);
    if (b2 == b1) b2 = b1 ^ 1u;
    u32x4 q[4];
    load(b1, q[0], q[1]);
    load(b2, q[2], q[3]);
    // all four loads go out before the first compare: left alone, the
    // scheduler started comparing the first bucket first, so the second
    // bucket's loads waited for the first's (two round trips, not one)
    __builtin_amdgcn_sched_barrier(0);
    uint2 r = make_uint2(0u, 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (q[i].y != 0u && (q[i].x & 0xFFFFFFu) == x) r = make_uint2(q[i].x, q[i].y);
        if (q[i].w != 0u && (q[i].z & 0xFFFFFFu) == x) r = make_uint2(q[i].z, q[i].w);
    }
    return r;
}

// Text of a candidate offset: [start, end) of the text holding o and its id.
// A batch's text starts come from `loff` when the block has copied them to
// LDS (as offsets from the first text, all below 2^32), else from global
// memory.
__device__ __forceinline__ void locate_text(const ScanArgs &S, const uint32_t *loff, int64_t o, int64_t &tstart,
                                            int64_t &end, int32_t &tid) {
    tstart = 0;
    end = S.n;
    tid = 0;
    if (!S.text_off) return;
    int32_t lo = 0, hi = S.n_texts;   // largest t with start(t) <= o, in [lo, hi)
    if (loff) {
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (int64_t(loff[mid]) <= o) lo = mid;
            else hi = mid;
        }
        tstart = loff[lo];
        end = lmin(int64_t(loff[lo + 1]), S.n);
    } else {
        const int64_t base0 = S.text_off[0];
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (S.text_off[mid] - base0 <= o) lo = mid;
            else hi = mid;
        }
        tstart = S.text_off[lo] - base0;
        end = lmin(S.text_off[lo + 1] - base0, S.n);
    }
    tid = lo;
}

// 16 bytes from p, of any alignment, assembled from five aligned dword loads.
// Every dword address is clamped to at most `last` (the aligned dword holding
// the last readable byte), so no load leaves the buffer; bytes taken from a
// clamped dword are garbage and must be masked by the caller.
__device__ __forceinline__ u32x4 load16_clamped(const uint8_t *p, uintptr_t last) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p) & ~uintptr_t(3);
    const uint32_t sh = uint32_t(reinterpret_cast<uintptr_t>(p) & 3u);
    uint32_t w[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const uintptr_t ai = a + 4u * uintptr_t(i);
        w[i] = gload4(reinterpret_cast<const uint8_t *>(ai < last ? ai : last));
    }
    u32x4 r;
    r.x = __builtin_amdgcn_alignbyte(w[1], w[0], sh);
    r.y = __builtin_amdgcn_alignbyte(w[2], w[1], sh);
    r.z = __builtin_amdgcn_alignbyte(w[3], w[2], sh);
    r.w = __builtin_amdgcn_alignbyte(w[4], w[3], sh);
    return r;
}

// 16 bytes from p, of any alignment, in one load: global memory is accessed
// in the GPU's unaligned access mode, which ROCm enables.  [p, p + 16) must
// be readable.
__device__ __forceinline__ u32x4 load16_any(const uint8_t *p) {
    u32x4 r;
    __builtin_memcpy(&r, (const __attribute__((address_space(1))) uint8_t *)(p), 16);
    return r;
}

// XOR of the first n (0..16) bytes of a and b, 0 when they agree.
__device__ __forceinline__ uint32_t diff16(u32x4 a, u32x4 b, int n) {
    uint32_t d = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = n - 4 * i;    // bytes of word i that count
        const uint32_t keep = m >= 4 ? 0xFFFFFFFFu : (m <= 0 ? 0u : (1u << (8 * m)) - 1u);
        d |= (a[i] ^ b[i]) & keep;
    }
    return d;
}

// Whether text t[0 .. n) equals keyword bytes k[0 .. n) (text[0 .. text_n) is
// the scanned buffer, which holds t[0 .. n)).  The first 32 bytes of both are
// loaded in one round trip, as 16-byte loads of any alignment; longer tails take
// more.  Text bytes within 16 of the buffer's end come from clamped dword loads
// instead.  Keyword bytes may be read up to 32 bytes past a keyword's compared
// part: the keyword section is followed by at least 256 bytes of the same
// allocation.
__device__ __forceinline__ bool equal_bytes(const uint8_t *t, const uint8_t *k, int n, const uint8_t *text,
                                            int64_t text_n) {
    const uintptr_t tend = reinterpret_cast<uintptr_t>(text) + uintptr_t(text_n);
    const uintptr_t tlast = (tend - 1u) & ~uintptr_t(3);
    auto text16 = [&](const uint8_t *p) __attribute__((always_inline)) {
        return reinterpret_cast<uintptr_t>(p) + 16u <= tend ? load16_any(p) : load16_clamped(p, tlast);
    };
    const u32x4 k0 = load16_any(k), k1 = load16_any(k + 16);
    const u32x4 t0 = text16(t), t1 = text16(t + 16);
    uint32_t d = diff16(t0, k0, n) | diff16(t1, k1, n - 16);
    for (int i = 32; d == 0 && i < n; i += 16) d = diff16(text16(t + i), load16_any(k + i), n - i);
    return d == 0;
}

// Position of byte b among the first n (1 .. 16) bytes of v, which are
// distinct, or -1.  Per word, the lowest flag of the zero-byte test marks the
// first byte equal to b exactly (a false flag can only sit above a true one).
__device__ __forceinline__ int find_byte16(u32x4 v, int n, uint32_t b) {
    const uint32_t rep = b * 0x01010101u;
    int at = 16;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
        const uint32_t x = v[i] ^ rep;
        const uint32_t z = (x - 0x01010101u) & ~x & 0x80808080u;
        if (z) at = 4 * i + int(__builtin_ctz(z) >> 3);
    }
    return at < n ? at : -1;
}

// The walk from offset o (relative to the scanned buffer) below a state s of
// depth d0 whose path is known to match.  Each step
// reads the state's 16-byte walk record (tail info): whether a keyword ends
// there, and either a forced path (a unary chain to a leaf with no keyword
// ending in between, whose leaf keyword is then compared with the text
// directly), a unary chain to a deeper state that ends a keyword or
// branches (compared the same way, then the walk goes on from there), or
// the state's children.  A dense state's next state comes from its
// transition row, with the byte's class loaded beside the record; a compact
// state's children are consecutive states with sorted edge labels, found
// among up to 16 labels read in one load.  The walk never compares or steps
// past `end` (the end of o's text).  The 32 text bytes after depth d0
// are loaded at the start, beside the first record, and serve the
// first compare and the first transitions.  Every keyword starting at o and
// ending at s or below is reported, through ids(state) for all keyword ids of
// a final state or one(pid) for a single id.
template <typename Ids, typename One>
__device__ __forceinline__ void walk_below(const DevAut &A, const ScanArgs &S, int64_t o, int64_t end, int32_t s,
                                           int d0, Ids &&ids, One &&one) {
    if (o + d0 > end) return;         // the path ran into the next text of a batch
    // The 32 text bytes after the path, loaded beside the first walk
    // record: most walks compare them with a forced path's keyword and read
    // no other text.
    const uintptr_t tend = reinterpret_cast<uintptr_t>(S.text) + uintptr_t(S.n);
    const uintptr_t tlast = (tend - 1u) & ~uintptr_t(3);
    auto text16 = [&](int64_t j) __attribute__((always_inline)) {   // 16 bytes from text byte j < S.n
        const uint8_t *p = S.text + j;
        return reinterpret_cast<uintptr_t>(p) + 16u <= tend ? load16_any(p) : load16_clamped(p, tlast);
    };
    u32x4 t0 = {0u, 0u, 0u, 0u}, t1 = t0;
    if (o + d0 < end) {
        t0 = text16(o + d0);
        if (o + d0 + 16 < S.n) t1 = text16(o + d0 + 16);
    }
    auto byte_at = [&](int64_t j) -> uint32_t {   // text byte j (o + d0 <= j < end)
        const int64_t r = j - o - d0;
        if (r < 32) {
            const u32x4 t = r < 16 ? t0 : t1;
            const int q = int(r & 15);
            const uint32_t w = q < 4 ? t.x : q < 8 ? t.y : q < 12 ? t.z : t.w;
            return (w >> (8 * (q & 3))) & 0xFFu;
        }
        return gload1(S.text + j);
    };
    // whether text bytes o + dd .. o + dd + z equal keyword bytes kw[0 .. z):
    // from the preloaded bytes while the walk is still at its first state
    auto same = [&](int64_t dd, const uint8_t *kw, int32_t z) -> bool {
        if (dd == d0 && z <= 32) {
            const u32x4 k0 = load16_any(kw), k1 = load16_any(kw + 16);
            return (diff16(t0, k0, z) | diff16(t1, k1, z - 16)) == 0u;
        }
        return equal_bytes(S.text + o + dd, kw, z, S.text, S.n);
    };
    int64_t d = d0;
    while (true) {
        const int4 ti = A.tailinfo[s];
        const bool has_byte = o + d < end;
        const uint32_t b = has_byte ? byte_at(o + d) : 0u;
        const bool dense = s < A.S_dense;
        const uint32_t c = dense && has_byte ? uint32_t(A.cls[b]) : 0u;
        if (ti.w < 0) ids(s);          // a keyword ends at s
        if (ti.x >= 0) {
            // forced path: bytes d .. d + ti.z of the text against the keyword
            const int64_t L = d + ti.z;
            if (o + L > end) return;
            if (!same(d, A.kw_bytes + ti.y, ti.z)) return;
            const int32_t only = ti.w & 0x7fffffff;
            if (only > 0) one(only - 1);
            else ids(ti.x);
            return;
        }
        if (ti.x == -3) {
            // a unary chain of ti.z bytes (no keyword ends inside it) to
            // state ti.w: compared in one pass, like a forced path
            if (o + d + ti.z > end) return;
            if (!same(d, A.kw_bytes + ti.y, ti.z)) return;
            s = ti.w & 0x7fffffff;
            d += ti.z;
            continue;
        }
        if (ti.x == -2 || !has_byte) return;   // a leaf, or the text ends
        if (dense) {
            const int32_t e2 = A.dense[static_cast<int64_t>(s) * A.C + c];
            if (e2 == 0) return;
            s = e2 & 0x7fffffff;
        } else {
            const int32_t fc = ti.y, nc = ti.z;
            int i;
            if (nc <= 16) {
                i = find_byte16(load16_any(A.label + fc), nc, b);
            } else {
                int32_t lo = 0, hi = nc;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (A.label[fc + mid] < b) lo = mid + 1;
                    else hi = mid;
                }
                i = lo < nc && A.label[fc + lo] == b ? lo : -1;
            }
            if (i < 0) return;
            s = fc + i;
        }
        ++d;
    }
}

// Slot of the 4-byte window x in the exact window table (2^nb buckets of four
// keys), or -1.  Both buckets, 16 bytes each, are read at once.
template <typename LoadBucket>
__device__ __forceinline__ int window_slot(LoadBucket load, int nb, uint32_t x) {
    uint32_t b1, b2;
    window_buckets(x, nb, b1, b2);
    const u32x4 q1 = load(b1), q2 = load(b2);
    int at = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (q1[i] == x) at = int(4 * b1) + i;
        if (q2[i] == x) at = int(4 * b2) + i;
    }
    return at;
}

// Everything the window at offset w (found in `slot` of the window table)
// belongs to, inside the text [tstart, end) that holds w: each of its entries
// fixes the offset o = w - position that the window's path starts from and the
// bytes to compare there, either a whole keyword or the path down to a state
// from which a walk goes on.  ids(o, state) and one(o, pid) report.
template <typename Ids, typename One>
__device__ __forceinline__ void walk_window(const DevAut &A, const ScanArgs &S, const int4 *entries, int slot,
                                            int64_t w, int64_t tstart, int64_t end, Ids &&ids, One &&one) {
    while (true) {
        const int4 e = entries[slot];
        const int64_t o = w - (e.w & 7);
        if (o >= tstart && o + e.y <= end && equal_bytes(S.text + o, A.kw_bytes + e.x, e.y, S.text, S.n)) {
            if (uint32_t(e.w) & kWinGeneral)
                walk_below(A, S, o, end, e.z, e.y, [&](int32_t st) { ids(o, st); },
                           [&](int32_t pid) { one(o, pid); });
            else
                one(o, e.z);
        }
        const uint32_t next = uint32_t(e.w) >> 4;
        if (next == 0) return;
        slot = int(next) - 1;
    }
}

struct FilterLaunch {
    const uint8_t *base;     // text pointer rounded down to 16 bytes
    int64_t mis;             // text - base
    int64_t V;               // mis + n: end of the text in `base` coordinates
    int64_t n_chunks;        // ceil(V / chunk bytes)
    int64_t c_hi;            // chunks from c_hi on (two at most) reach past the text's last 16 bytes
    const uint8_t *filter;   // the filter map this launch stages in LDS
    int32_t hit_cap;         // 16-byte entries per wave region
    uint4 *hits;             // [waves * hit_cap]: two records in each, {slot << 12 | position,
                             //  window-table slot or prefix-table value}
    const uint32_t *win_keys;   // exact window table (4 << win_nb keys)
    const int4 *win_entries;
    int32_t win_nb;             // log2(buckets)
};

// The filtered kernel's one argument.
struct KArgs {
    DevAut A;
    ScanArgs S;
    FilterLaunch F;
};
typedef const __attribute__((address_space(4))) KArgs *KArgsPtr;

// Slot -> chunk of one block (see filtered_kernel).
struct SlotMap {
    int64_t bfirst;    // the block's first chunk
    int64_t nw;        // waves in the grid
    uint32_t wmask;    // waves per block - 1 (a power of two minus one)
    int32_t wlog;      // log2(waves per block)
    __device__ __forceinline__ int64_t chunk(uint32_t slot) const {
        return bfirst + int64_t(slot & wmask) + int64_t(slot >> wlog) * nw;
    }
};

template <int SEGS>
struct ChunkRegs {
    uint32_t d[SEGS][4];
    uint32_t tail;   // first dword after the chunk (halo of the last lane)
};

// One chunk: one coalesced 16-byte load per lane and segment, as buffer
// loads from a descriptor based at the chunk (uniform, in SGPRs) with
// per-lane offsets that never change, so issuing the next chunk's loads
// needs no address register that an earlier load might still be writing.
// The loads are non-temporal: the stream passes through the caches without
// pushing out the tables and records that drains and walks read (1 GiB,
// 1000 keywords: 0.178 ms instead of 0.191; the 4096-text batch, whose
// block-wide walk follows the stream closely, 1% slower; a uniform branch
// that kept the default policy for batches cost more than either).
//
// The first and the last chunks need no other path: the 16-byte granules that
// hold the text's ends are read whole (a granule never straddles a page), and
// the descriptor of a last chunk ends with the text's last dword, past which
// loads return 0.  Offsets that do not lie in the text are dropped where they
// are looked up.  (A path of its own for them, byte loads and walks by one
// wave, took 1.3 to 3.5 us at the end of every scan; kernel without it and with
// report_count's one store: 1 KiB 8.2 -> 5.9 us, 1 MiB 12.4 -> 10.6, paper
// lines 671 KB 14.0 -> 11.5, 64 MiB at stride 1 46.2 -> 41.8.)
template <int SEGS>
__device__ __forceinline__ void load_chunk(const FilterLaunch &F, int64_t c, unsigned lane, ChunkRegs<SEGS> &R) {
    constexpr int64_t CH = int64_t(SEGS) * kSegBytes;
    constexpr int kNonTemporal = 2;     // cache-policy operand of the buffer loads: nt
    const int records = c < F.c_hi ? int(CH + 16) : int(((F.V + 3) & ~int64_t(3)) - c * CH);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(F.base + c * CH), short(0), records, kBufferFlags);
#pragma unroll
    for (int j = 0; j < SEGS; ++j) {
        const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, int(lane * 16u + uint32_t(j) * kSegBytes), 0,
                                                              kNonTemporal);
        R.d[j][0] = q.x; R.d[j][1] = q.y; R.d[j][2] = q.z; R.d[j][3] = q.w;
    }
    R.tail = __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(CH), 0, 0);
}

// Segment j of a chunk alone.  The segment's offset is part of the vector
// offset, as in load_chunk: the scalar one takes no part in the check against
// `records`, which is what ends a last chunk's loads at the text's end.
template <int SEGS>
__device__ __forceinline__ void load_segment(const FilterLaunch &F, int64_t c, int j, unsigned lane, ChunkRegs<1> &R) {
    constexpr int64_t CH = int64_t(SEGS) * kSegBytes;
    const int records = c < F.c_hi ? int(CH + 16) : int(((F.V + 3) & ~int64_t(3)) - c * CH);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(F.base + c * CH), short(0), records, kBufferFlags);
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, int(lane * 16u) + j * kSegBytes, 0, 0);
    R.d[0][0] = q.x; R.d[0][1] = q.y; R.d[0][2] = q.z; R.d[0][3] = q.w;
    R.tail = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (j + 1) * kSegBytes, 0, 0);
}

// Candidate mask of the N segments from J0 on: bit 16 i + s is set when offset
// s of the lane's 16 bytes in segment J0 + i may start a keyword.  d4[i]
// receives the dword after the lane's 16 bytes.
//
// Stride 1: the K bytes at offset s hash to a set filter entry.
// Stride 2 and 4: only the 3-byte windows starting at s = STRIDE, 2 STRIDE,
// ..., 16 are tested (s = 16 is the next lane's first bytes), against the
// keywords' windows at positions 1 .. STRIDE; a keyword starting at o has its
// window at position s - o tested for the one sampled s in o + 1 .. o +
// STRIDE, so a positive makes the STRIDE offsets s - STRIDE .. s - 1
// candidates.  Windows at s = 4, 8, 12, 16 are whole registers (the hash
// reads 24 bits), so stride 4 extracts no bytes and stride 2 half as many.
// A bit map is tested without shifting the looked-up bit into place: the
// hash is p = x * mul + c with c = -b mod 32 for destination bit b, so
// rotating the word right by p (mod 32) moves the key's bit (x * mul) mod 32
// to b.  Adding c may carry into the word index; the host sets each key's
// bit in both words that can result.
// PAIR (strides 2 and 4): the 4-byte windows' map, tested as in filter_windows.
template <int K, bool BITMAP, int SEGS, int FLOG2, int STRIDE, bool DUAL, bool PAIR, int J0, int N>
__device__ __forceinline__ uint32_t filter_offsets(const ChunkRegs<SEGS> &R, unsigned lane, const uint8_t *sfilt,
                                                   uint32_t mul, uint32_t (&d4)[N]) {
    constexpr uint32_t kmask = K >= 3 ? 0xFFFFFFu : ((1u << (8 * K)) - 1u);
    // byte map: 2^FLOG2 entries; bit map: 2^(FLOG2-2) words of 32 bits
    constexpr int shift = BITMAP ? 32 - (FLOG2 - 2) : 32 - FLOG2;
    const uint32_t *fm = reinterpret_cast<const uint32_t *>(sfilt);
    static_assert(N <= 2, "one mask word");
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int j = J0 + i;
        const uint32_t from_next_lane = __builtin_amdgcn_ds_bpermute(int((lane + 1) * 4), int(R.d[j][0]));
        const uint32_t from_next_seg = (j + 1 < SEGS) ? __builtin_amdgcn_readlane(R.d[(j + 1) % SEGS][0], 0)
                                                      : R.tail;
        d4[i] = lane == 63 ? from_next_seg : from_next_lane;
        const uint32_t d[5] = {R.d[j][0], R.d[j][1], R.d[j][2], R.d[j][3], d4[i]};
        uint32_t mj = 0;
        if (STRIDE == 1) {
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const int w = s >> 2, r = s & 3;
                uint32_t x = r == 0 ? d[w] : __builtin_amdgcn_alignbyte(d[w + 1], d[w], uint32_t(r));
                if (K < 3) x &= kmask;
                const uint32_t p = hash24(x, mul);
                uint32_t v;
                if (DUAL) {
                    const uint32_t p2 = hash24(x, kFilterMul2);
                    v = __builtin_amdgcn_ubfe(fm[p >> (shift + 1)], p, 1u) &
                        __builtin_amdgcn_ubfe(fm[(1u << (FLOG2 - 3)) + (p2 >> (shift + 1))], p2, 1u);
                } else if (BITMAP) {
                    v = __builtin_amdgcn_ubfe(fm[p >> shift], p, 1u);
                } else {
                    v = sfilt[p >> shift];
                }
                mj |= v << s;
            }
        } else {
#pragma unroll
            for (int s = STRIDE; s <= 16; s += STRIDE) {
                const int w = s >> 2, r = s & 3;
                const uint32_t x = r == 0 ? d[w] : __builtin_amdgcn_alignbyte(d[w + 1], d[w], uint32_t(r));
                const int b = s - STRIDE;                 // destination bit
                const uint32_t c = uint32_t(32 - b) & 31u;
                const uint32_t p = hash24(x, mul) + c;
                if (PAIR) {
                    const uint32_t p1 = hash24(x, mul);
                    const uint32_t w1 = fm[p1 >> shift];
                    uint32_t v = (w1 >> (p1 & 31u)) & (w1 >> ((x >> 24) & 31u));
                    if (STRIDE == 2) v &= w1 >> ((x >> 16) & 31u);
                    mj |= (v & 1u) << b;
                } else if (BITMAP) {
                    uint32_t v;
                    if (DUAL) {
                        // two maps of 2^(FLOG2 - 3) words, independent hashes: both bits must be set
                        const uint32_t p2 = hash24(x, kFilterMul2) + c;
                        const uint32_t w1 = fm[p >> (shift + 1)];
                        const uint32_t w2 = fm[(1u << (FLOG2 - 3)) + (p2 >> (shift + 1))];
                        v = __builtin_amdgcn_alignbit(w1, w1, p) & __builtin_amdgcn_alignbit(w2, w2, p2);
                    } else {
                        const uint32_t w1 = fm[p >> shift];
                        v = __builtin_amdgcn_alignbit(w1, w1, p);
                    }
                    mj = (v & (1u << b)) | (mj & ~(1u << b));
                } else {
                    mj |= uint32_t(sfilt[p >> shift]) << b;
                }
            }
            // a positive at bit b covers the offsets b .. b + STRIDE - 1
            if (STRIDE == 2) mj |= mj << 1;
            if (STRIDE == 4) mj = __umul24(mj, 15u);
        }
        m |= mj << (16 * i);
    }
    return m;
}

// Positive windows of the N segments from J0 on, for the strides with the
// window table: bit i (16 / STRIDE) + t is set when the window starting at
// STRIDE (t + 1) of the lane's 16 bytes in segment J0 + i may lie at keyword
// positions 1 .. STRIDE.  d4[i] receives the dword after the lane's 16 bytes.
// PAIR: the window's first three bytes pick the word, and the bits (x * mul)
// mod 32 and (byte 3) mod 32 of that word must both be set; at stride 2 also
// bit (byte 2) mod 32.
// Bound by VALU issue, so the bits are moved as little as possible: each test
// shifts the word right so that its bit becomes bit 0 (a shift amount taken
// from a byte of x is an operand select, not an instruction), and one
// alignbit per window shifts the result into the mask: 8 instructions per
// window at stride 2 with the window's extraction apart, 7 at stride 4, where
// masking each result and shifting it into place took 10 and 8.
template <bool BITMAP, int SEGS, int FLOG2, int STRIDE, bool DUAL, bool PAIR, int J0, int N>
__device__ __forceinline__ uint32_t filter_windows(const ChunkRegs<SEGS> &R, unsigned lane, const uint8_t *sfilt,
                                                   uint32_t mul, uint32_t (&d4)[N]) {
    constexpr int shift = BITMAP ? 32 - (FLOG2 - 2) : 32 - FLOG2;
    constexpr int kWin = 16 / STRIDE;
    static_assert(N * kWin <= 32, "one mask word");
    const uint32_t *fm = reinterpret_cast<const uint32_t *>(sfilt);
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int j = J0 + i;
        const uint32_t from_next_lane = __builtin_amdgcn_ds_bpermute(int((lane + 1) * 4), int(R.d[j][0]));
        const uint32_t from_next_seg = (j + 1 < SEGS) ? __builtin_amdgcn_readlane(R.d[(j + 1) % SEGS][0], 0)
                                                      : R.tail;
        d4[i] = lane == 63 ? from_next_seg : from_next_lane;
        const uint32_t d[5] = {R.d[j][0], R.d[j][1], R.d[j][2], R.d[j][3], d4[i]};
#pragma unroll
        for (int s = STRIDE; s <= 16; s += STRIDE) {
            const int w = s >> 2, r = s & 3;
            const uint32_t x = r == 0 ? d[w] : __builtin_amdgcn_alignbyte(d[w + 1], d[w], uint32_t(r));
            const uint32_t p = hash24(x, mul);
            uint32_t v;
            if (PAIR) {
                const uint32_t w1 = fm[p >> shift];
                v = (w1 >> (p & 31u)) & (w1 >> ((x >> 24) & 31u));
                if (STRIDE == 2) v &= w1 >> ((x >> 16) & 31u);
            } else if (DUAL) {
                const uint32_t p2 = hash24(x, kFilterMul2);
                v = (fm[p >> (shift + 1)] >> (p & 31u)) &
                    (fm[(1u << (FLOG2 - 3)) + (p2 >> (shift + 1))] >> (p2 & 31u));
            } else if (BITMAP) {
                v = fm[p >> shift] >> (p & 31u);
            } else {
                v = sfilt[p >> shift];
            }
            acc = __builtin_amdgcn_alignbit(v, acc, 1u);
        }
    }
    return acc >> (32 - N * kWin);
}

// All ones when bit i of b is set, else 0; and the choice between two values
// by such a mask.
__device__ __forceinline__ uint32_t bit_mask(int b, int i) { return uint32_t(int32_t(uint32_t(b) << (31 - i)) >> 31); }
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

// A condition every lane of the wave agrees on, marked as such for the
// compiler, so that branching on it needs no exec-mask bookkeeping.  The
// ballot keeps the lane mask in scalar registers (a readfirstlane would first
// write it to a VGPR, whose reuse could wait for a load still in flight).
__device__ __forceinline__ bool uniform(bool c) { return __builtin_amdgcn_ballot_w64(c) != 0; }
// A value every lane holds, moved to scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v)));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(v) >> 32));
    return int64_t((uint64_t(hi) << 32) | lo);
}

// The kernel's argument block, read where it lies.  The empty asm hides the
// pointer's origin from the compiler, so the fields read through it are
// loaded here and not all at the kernel's entry, from where they would stay
// live (and spill) across the streaming loop.
__device__ __forceinline__ const KArgs *kernel_args() {
    KArgsPtr p = (KArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (const KArgs *)p;   // still known to be constant memory: read with scalar loads
}

// Exact prefix lookup through the LDS copy of the prefix table when it has
// one, else through global memory.
__device__ __forceinline__ uint2 probe_prefix(bool in_lds, const uint32_t *sptab, const uint32_t *gptab, int bits,
                                              uint32_t x, uint32_t mul) {
    if (in_lds)
        return prefix_state([&](uint32_t b, u32x4 &lo, u32x4 &hi) {
            lo = reinterpret_cast<const u32x4 *>(sptab)[2 * b];
            hi = reinterpret_cast<const u32x4 *>(sptab)[2 * b + 1];
        }, bits, x, mul);
    return prefix_state([&](uint32_t b, u32x4 &lo, u32x4 &hi) {
        lo = gload16(reinterpret_cast<const uint8_t *>(gptab + 8 * b));
        hi = gload16(reinterpret_cast<const uint8_t *>(gptab + 8 * b + 4));
    }, bits, x, mul);
}

// Exact window lookup through the LDS copy of the window keys when there is
// one, else through global memory.
__device__ __forceinline__ int find_window(bool in_lds, const uint32_t *skeys, const uint32_t *gkeys, int nb,
                                           uint32_t x) {
    if (in_lds) return window_slot([&](uint32_t b) { return reinterpret_cast<const u32x4 *>(skeys)[b]; }, nb, x);
    return window_slot([&](uint32_t b) { return gload16(reinterpret_cast<const uint8_t *>(gkeys + 4 * b)); }, nb, x);
}

// Called by every thread at the scan's end: the last block to finish hands the
// count to the host (or stores it in the caller's device word), once every
// block's matches are stored.  For device arrays no fence is needed.  Matches
// are written through to the device (put_out), each wave waits until its own
// have arrived, and the block's barrier collects its waves before the block
// counts itself done.  Atomics on one address are performed in one place, and
// every add to the count has returned its value by then, so the last block's
// access sees them all.  A release fence per block, which writes the XCD's
// whole L2 back, and the last block's acquire cost more (kernel): 1 MiB 10.9 ->
// 9.8 us, paper lines 671 KB 11.9 -> 10.9, 64 MiB at stride 1 40.0 -> 34.8, the
// 4096-text batch 57.5 -> 53.5, 1 GiB 173 -> 168.5.  The count and its tag go
// out in one store; the host takes them only when they belong together, so
// nothing orders them either (a fence between two stores waited for the host
// link).
//
// The host reads pinned match arrays when the count arrives, before the kernel's
// end, so there each block releases its matches to the system first (calls with
// host arrays of 16 KiB to 1 MiB, 4 to 65,000 matches: within 0.4 us of none).
// That does not order what arrives at the host: it takes each entry only once
// it is there.
__device__ __forceinline__ void report_count(const ScanArgs &S) {
    if (S.host_count) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (S.near_cap > 0) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    if (gridDim.x > 1) {
        if (atomicAdd(S.done, 1ull) != gridDim.x - 1) return;
        atomicExch(S.done, 0ull);    // for the next scan
    }
    if (S.dev_count) {
        *S.dev_count = atomicExch(S.count, 0ull);
        return;
    }
    const unsigned long long c = atomicAdd(S.count, 0ull);
    const unsigned long long tag = report_tag(c, S.host_seq);
    gstore16(reinterpret_cast<uint4 *>(S.host_count), uint32_t(c), uint32_t(c >> 32), uint32_t(tag), uint32_t(tag >> 32));
    __threadfence_system();
}

// Sum of v over lanes 0 .. lane - 1 (exclusive prefix), for the first 16
// lanes; v must be 0 in the others.
__device__ __forceinline__ int prefix16(int v, unsigned lane) {
    int s = v;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const int up = __shfl_up(s, unsigned(d));
        if (int(lane) >= d) s += up;
    }
    return s - v;
}

// Streaming kernel of the filtered policy.
//
// Work is dealt out in slots: slot i of block b is chunk b W
// + (i mod W) + (i div W) nw (W waves per block, nw waves in the grid, so a
// step of the grid still reads one contiguous stretch of text).  Each wave
// starts with slots `wave` and `wave + W` and takes every further slot from
// a counter in LDS, one slot ahead of need.  Waves of one block progress at
// very different rates (the SIMDs favour older waves), and with a fixed
// share per wave the block would wait for its slowest one.
//
// Candidates wait in a per-wave LDS queue; a drain takes kDrain of them at
// once.  The chunk loop has no walk, atomic in global memory, call or other
// dependent global access apart from drains.
//
// WIN (strides 2 and 4, with the stride's window table): a queue entry is a positive window and its four bytes, taken from the registers
// that were filtered.  A drain looks the bytes up in the exact window table
// (two 16-byte loads per lane) and keeps {position, table slot} of those that
// are a keyword's window.  It reads no text, and a positive is one entry
// where the offsets it stands for were STRIDE of them, each with a 16-byte
// text read (often from memory again: the stream is non-temporal) and a
// 64-byte prefix lookup.  The table's entry gives the walk the offset and,
// mostly, the one keyword to compare.  Measured on MI355X against prefix
// drains (kernel): 50000 keywords, 64 MiB 53.5 -> 30.5 us; 4096 texts, 267 MB,
// 72.9 -> 63.5; paper lines, 671 KB, 17.9 -> 14.0; 20000 keywords, 1 GiB,
// stride 2, 216 -> 217, and 197 with filter_windows' shorter tests; 1000
// keywords, 1 GiB, 173 -> 171 (bound by the stream), 220.8 -> 199.6 per call
// between other work.
//
// Otherwise an entry is a candidate offset and the four bytes from it on, and
// a drain looks the prefix up in the exact prefix table, in LDS beside a 64 KiB
// map.  (Drains that read each offset's text: 200 keywords of 2 to 8 bytes, 64
// MiB, 1.5 million candidates, 35.3 us, now 35.0; two keywords, 1 MiB, 10.0 ->
// 9.5.)
//
// Kept hits go to the wave's hit records (LDS, then its region).  A wave
// whose region has no room for another drain leaves the loop and goes on in
// a slow mode: it scans the rest of its slots one chunk at a time and walks
// every hit as soon as a table confirms it.  Finally each wave (one text) or the
// whole block (a batch) walks the stored hits.
template <int K, bool BITMAP, int SEGS, int FLOG2, int STRIDE, bool DUAL, bool PAIR, bool WIN>
__global__ __launch_bounds__(1024) void filtered_kernel(const KArgs) {
    __shared__ __align__(16) uint8_t sfilt[1 << FLOG2];
    __shared__ __align__(16) uint32_t squeue[kMaxWaves * kQueueCap];
    // Beside a 64 KiB filter, a copy of the prefix table (8192 slots) fits
    // too; beside a 128 KiB one only the queues and the hit records do.
    constexpr int PT_SLOTS = FLOG2 >= 17 ? 0 : 8192;
    constexpr int kHitBytes = kMaxWaves * kLdsHits * 8;
    __shared__ __align__(16) uint32_t sxtra[(2 * PT_SLOTS * 4 + kHitBytes) / 4];
    uint32_t *const sptab = sxtra;                                        // [2 * PT_SLOTS]
    uint2 *const shits = reinterpret_cast<uint2 *>(sxtra + 2 * PT_SLOTS);  // [waves * kLdsHits]
    constexpr int64_t CH = int64_t(SEGS) * kSegBytes;
    const int waves_per_block = int(blockDim.x) / kWave;
    const int wlog = __builtin_ctz(unsigned(waves_per_block));   // W is a power of two
    const unsigned lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
    uint32_t *q = squeue + wave * kQueueCap;
    const int64_t w = int64_t(blockIdx.x) * waves_per_block + wave;
    const int64_t nw = int64_t(gridDim.x) * waves_per_block;
    uint32_t &snext = squeue[kQueueCap - 1];              // next slot to hand out
    int hcount = 0;                    // hits stored in this wave's region
    int qlen = 0;

    // Where the streaming loop stopped: every slot from `cur` on is left to
    // the slow mode (none if cur_ok is false), of cur what `rest` holds of its
    // group of segments rest_g and the groups after it, and lane 0's `ahead`
    // holds the slot after nxt (taken when nxt is a chunk of the text).
    bool slow = false;
    bool cur_ok = false;
    uint32_t cur = 0, nxt = 0, ahead = 0;
    unsigned rest = 0;
    int rest_g = 0;

    // A queue entry is a candidate's position {slot << 12 | byte of the chunk}
    // and its four bytes, from the registers that were filtered: the positive
    // window's (its position the first offset it stands for), or those from a
    // candidate offset on (the prefix and at least one byte after it).
    constexpr int kBits = WIN ? 16 / STRIDE : 16;    // candidates per segment and lane
    constexpr int kBitsLog = __builtin_ctz(unsigned(kBits));
    uint2 *wq = reinterpret_cast<uint2 *>(q);
    // Queues the candidates m (those of N segments from J0 on), one per lane
    // and round; false, leaving the rest in m, if `drain` refuses to run.
    // Bound by VALU issue: a round costs some 30 instructions however few of
    // its lanes have a candidate, and there are as many as the fullest lane
    // has bits.  So both segments of a group share the rounds, which costs 6
    // more instructions to pick a lane's registers; kernel, a loop per segment
    // -> this: 20000 keywords, 1 GiB, 193 -> 182 us; 200 short keywords, 64
    // MiB, 35.1 -> 33.1; 50000 keywords, 64 MiB, 27.4 -> 26.5.  Four segments
    // at once need three times the picks: 1 GiB 203.
    auto queue_mask = [&](unsigned &m, const auto &R, const auto &d4, auto j0, uint32_t at0,
                          auto &&drain) __attribute__((always_inline)) {
        constexpr int J0 = decltype(j0)::value;
        constexpr int N = int(sizeof(d4) / 4);
        while (true) {
            if (qlen >= kDrain && !drain(kDrain)) return false;
            const unsigned long long act = __ballot(m != 0);
            if (act == 0) return true;
            if (m) {
                const int t = __builtin_ctz(m);
                // of two segments' registers, the one's that bit t lies in
                const uint32_t c1 = N == 2 ? bit_mask(t, kBitsLog) : 0u;
                auto reg = [&](int k) __attribute__((always_inline)) -> uint32_t {
                    const uint32_t r0 = k < 4 ? R.d[J0][k] : d4[0];
                    return N == 2 ? pick(c1, k < 4 ? R.d[J0 + N - 1][k] : d4[N - 1], r0) : r0;
                };
                const int b = WIN ? (t * STRIDE) & 15 : t & 15;
                // the four bytes, picked without branches
                const uint32_t c2 = bit_mask(b, 2), c3 = bit_mask(b, 3);
                const uint32_t w2 = reg(2), w3 = reg(3), w1 = reg(1);
                const uint32_t hi = pick(c3, pick(c2, reg(4), w3), pick(c2, w2, w1));
                uint32_t x;
                if (WIN && STRIDE == 4) {
                    x = hi;
                } else {
                    const uint32_t lo = pick(c3, pick(c2, w3, w2), pick(c2, w1, reg(0)));
                    if (WIN) x = pick(bit_mask(b, 1), hi, __builtin_amdgcn_alignbyte(hi, lo, 2u));
                    else x = __builtin_amdgcn_alignbyte(hi, lo, uint32_t(b) & 3u);
                }
                const uint32_t at = at0 + uint32_t(J0 * kSegBytes + int(lane) * 16 + b);
                wq[qlen + int(rank_in(act))] = make_uint2(N == 2 ? at + (c1 & kSegBytes) : at, x);
                m &= m - 1;
            }
            qlen += __popcll(act);
        }
    };
    // Filters the segments of R from J0 on.
    auto filter = [&](const auto &R, auto j0, uint32_t mul, auto &d4) __attribute__((always_inline)) -> unsigned {
        constexpr int J0 = decltype(j0)::value;
        constexpr int N = int(sizeof(d4) / 4);
        constexpr int NS = int(sizeof(R.d) / 16);
        if constexpr (WIN) return filter_windows<BITMAP, NS, FLOG2, STRIDE, DUAL, PAIR, J0, N>(R, lane, sfilt, mul, d4);
        else return filter_offsets<K, BITMAP, NS, FLOG2, STRIDE, DUAL, PAIR, J0, N>(R, lane, sfilt, mul, d4);
    };
    // Filters and queues the chunk held in R (slot k) in groups of at most two
    // segments (more at once spill registers).  On a refusal `rest` holds what
    // is left of group rest_g; the groups after it are left whole.
    auto push = [&](const ChunkRegs<SEGS> &R, uint32_t mul, uint32_t k, auto &&drain) __attribute__((always_inline)) {
        constexpr int kGroup = SEGS < 2 ? 1 : 2;
        auto group = [&](auto g) __attribute__((always_inline)) {
            constexpr int G = decltype(g)::value;
            uint32_t d4[kGroup];
            const std::integral_constant<int, G * kGroup> j0{};
            unsigned m = filter(R, j0, mul, d4);
            if (queue_mask(m, R, d4, j0, k << 12, drain)) return true;
            rest = m;
            rest_g = G;
            return false;
        };
        if (!group(std::integral_constant<int, 0>{})) return false;
        if constexpr (SEGS == 4)
            if (!group(std::integral_constant<int, 1>{})) return false;
        return true;
    };
    // The newest `take` queue entries, one per lane (lanes past `take` repeat
    // the first one).
    auto pop = [&](int take) __attribute__((always_inline)) {
        wave_sync();
        const uint2 e = wq[qlen - take + (int(lane) < take ? int(lane) : 0)];
        wave_sync();
        qlen -= take;
        return e;
    };
    // What the tables know of a queue entry's bytes: the window table's slot,
    // or the prefix table's value; kNoHit when no keyword has them.
    constexpr uint32_t kNoHit = WIN ? ~0u : 0u;
    auto look_up = [&](uint32_t y, bool in_lds, const FilterLaunch &F, const uint32_t *gptab, int bits,
                       uint32_t mul) __attribute__((always_inline)) -> uint32_t {
        if constexpr (WIN) return uint32_t(find_window(in_lds, sptab, F.win_keys, F.win_nb, y));
        const uint2 kv = probe_prefix(in_lds, sptab, gptab, bits, K >= 3 ? y & 0xFFFFFFu : y & ((1u << (8 * K)) - 1u), mul);
        // a non-final prefix state whose only child's byte differs from the
        // text's next byte ends the walk at the prefix
        if ((kv.y & kHasNext) && !(kv.y >> 31) && (kv.x >> 24) != ((y >> (8 * K)) & 0xFFu)) return kNoHit;
        return kv.y;
    };

    // ---- set-up and streaming: the fields they read, and no others ----
    {
        const KArgs *P1 = kernel_args();
        const FilterLaunch F = P1->F;
        const uint32_t *gptab = P1->A.ptab;
        const int ptab_bits = P1->A.ptab_bits;
        const uint32_t mul = P1->A.hash_mul;
        const bool pt_lds = FLOG2 < 17 && (WIN ? F.win_nb <= 12 : ptab_bits <= 13);
        // Tables to LDS, two loads in flight per thread.  Every block reads
        // the same lines, so the blocks of one XCD (blockIdx mod 8) start at
        // different ones (n16 is a power of two).
        auto stage = [&](const uint4 *src, uint4 *dst, int n16) __attribute__((always_inline)) {
            const int rot = (int(blockIdx.x >> 3) * 1024) & (n16 - 1);
            for (int i0 = int(threadIdx.x); i0 < n16; i0 += 2 * int(blockDim.x)) {
                const int i1 = i0 + int(blockDim.x);
                const uint4 v0 = src[(i0 + rot) & (n16 - 1)];
                uint4 v1;
                if (i1 < n16) v1 = src[(i1 + rot) & (n16 - 1)];
                dst[(i0 + rot) & (n16 - 1)] = v0;
                if (i1 < n16) dst[(i1 + rot) & (n16 - 1)] = v1;
            }
        };
        stage(reinterpret_cast<const uint4 *>(F.filter), reinterpret_cast<uint4 *>(sfilt), (1 << FLOG2) / 16);
        if (pt_lds) {
            if (WIN) stage(reinterpret_cast<const uint4 *>(F.win_keys), reinterpret_cast<uint4 *>(sptab), 1 << F.win_nb);
            else stage(reinterpret_cast<const uint4 *>(gptab), reinterpret_cast<uint4 *>(sptab), (2 << ptab_bits) / 4);
        }
        SlotMap M;
        M.bfirst = int64_t(blockIdx.x) * waves_per_block;
        M.nw = nw;
        M.wmask = uint32_t(waves_per_block - 1);
        M.wlog = wlog;
        if (threadIdx.x == 0) snext = uint32_t(2 * waves_per_block);
        __syncthreads();

        // Streaming-loop drain of the newest `take` entries.  Refuses when
        // the region might not hold its hits.
        uint2 *hits = reinterpret_cast<uint2 *>(F.hits + w * F.hit_cap);
        uint2 *lhits = shits + wave * kLdsHits;
        auto drain = [&](int take) __attribute__((always_inline)) {
            if (hcount + kDrain > kLdsHits + 2 * F.hit_cap) return false;
            const uint2 e = pop(take);
            uint32_t v = kNoHit;
            if (int(lane) < take) v = look_up(e.y, pt_lds, F, gptab, ptab_bits, mul);
            const unsigned long long hit = __ballot(v != kNoHit);
            if (hit == 0) return true;
            if (v != kNoHit) {
                const int at = hcount + int(rank_in(hit));
                if (at < kLdsHits) lhits[at] = make_uint2(e.x, v);
                else gstore8(hits + (at - kLdsHits), e.x, v);
            }
            hcount += __popcll(hit);
            return true;
        };

        // The chunks, two register sets in turn so that the next chunk's
        // loads are in flight while this one is filtered.  The next chunk's
        // loads are issued unconditionally (the last step reloads its own
        // chunk): with a fixed number of loads between a chunk's loads and
        // its first use, the compiler waits for that chunk only.
        ChunkRegs<SEGS> ra, rb;
        const int64_t n_chunks = uniform64(F.n_chunks);
        cur = uint32_t(wave);
        nxt = uint32_t(wave + waves_per_block);
        cur_ok = uniform(M.chunk(cur) < n_chunks);
        if (cur_ok) load_chunk<SEGS>(F, M.chunk(cur), lane, ra);
        // One half step: issue the next chunk's loads into `into` (or reload
        // the current one), take the slot after nxt from the block's counter
        // (lane 0), filter and queue the current chunk held in `regs`, then
        // move on.  The counter's divergent branch joins right after the
        // atomic, so the loop's back edge merges only uniform conditions.
        // Returns false when the loop must end (slow mode, or no slot left).
        auto half = [&](ChunkRegs<SEGS> &regs, ChunkRegs<SEGS> &into) __attribute__((always_inline)) {
            const bool nxt_ok = uniform(M.chunk(nxt) < n_chunks);
            load_chunk<SEGS>(F, M.chunk(nxt_ok ? nxt : cur), lane, into);
            if (lane == 0 && nxt_ok) ahead = atomicAdd(&snext, 1u);
            if (!uniform(push(regs, mul, cur, drain))) { slow = true; return false; }
            // slots held by a wave only grow, and so do their chunks: once
            // one is past the end, so is every later one
            cur = nxt;
            cur_ok = nxt_ok;
            nxt = __builtin_amdgcn_readfirstlane(ahead);
            return cur_ok;
        };
        while (cur_ok) {
            if (!half(ra, rb)) break;
            if (!half(rb, ra)) break;
        }
        while (!slow && qlen > 0)
            if (!drain(imin(qlen, kDrain))) slow = true;
    }

    // ---- slow mode, partial chunks, walks and output ----
    const KArgs *P2 = kernel_args();
    const DevAut A = P2->A;
    const ScanArgs S = P2->S;
    const FilterLaunch F = P2->F;
    SlotMap M;
    M.bfirst = int64_t(blockIdx.x) * waves_per_block;
    M.nw = nw;
    M.wmask = uint32_t(waves_per_block - 1);
    M.wlog = wlog;
    const bool pt_lds = FLOG2 < 17 && (WIN ? F.win_nb <= 12 : A.ptab_bits <= 13);
    const uint32_t mul = A.hash_mul;
    const uint2 *hits = reinterpret_cast<const uint2 *>(F.hits + w * F.hit_cap);
    auto offset_of = [&](uint32_t ent) __attribute__((always_inline)) {
        return M.chunk(ent >> 12) * CH + int64_t(ent & 4095u) - F.mis;
    };
    // Walks a hit {position, look_up's value}; text(at, start, end, id) gives
    // the text holding its window or offset, ids(o, id, start, state) and
    // one(o, id, start, keyword) report.
    auto walk_hit = [&](uint2 rec, auto &&text, auto &&ids, auto &&one) __attribute__((always_inline)) {
        const int64_t at = offset_of(rec.x) + (WIN ? STRIDE : 0);
        int64_t tstart, end;
        int32_t tid;
        text(at, tstart, end, tid);
        auto ids2 = [&](int64_t o, int32_t st) __attribute__((always_inline)) { ids(o, tid, tstart, st); };
        auto one2 = [&](int64_t o, int32_t pid) __attribute__((always_inline)) { one(o, tid, tstart, pid); };
        if constexpr (WIN)
            walk_window(A, S, F.win_entries, int(rec.y), at, tstart, end, ids2, one2);
        else if (at >= tstart)     // not before the text's first byte
            walk_below(A, S, at, end, int32_t(rec.y & kStateMask), K, [&](int32_t st) { ids2(at, st); },
                       [&](int32_t pid) { one2(at, pid); });
    };

    if (slow) {
        // A drain that walks what it confirms right here.
        auto drain_walk = [&](int take) __attribute__((always_inline)) {
            const uint2 e = pop(take);
            if (int(lane) >= take) return;
            const uint32_t v = look_up(e.y, pt_lds, F, A.ptab, A.ptab_bits, mul);
            if (v == kNoHit) return;
            walk_hit(make_uint2(e.x, v),
                     [&](int64_t at, int64_t &ts, int64_t &te, int32_t &id) { locate_text(S, nullptr, at, ts, te, id); },
                     [&](int64_t o, int32_t id, int64_t ts, int32_t st) { emit(A, S, o - ts, id, st); },
                     [&](int64_t o, int32_t id, int64_t ts, int32_t pid) {
                         emit_one(S, nullptr, nullptr, o - ts, id, pid);
                     });
        };
        // What is left of the wave's slots: cur first, with what its queueing
        // left (its text is read again), then its successors, one segment at a
        // time, since a segment's registers stay live while the walks of a
        // full queue run.  A queue is drained when it is full and at the very
        // end, so that a wave's matches share their atomics (18 keywords of 3
        // letters, 128 MiB of ACGT, 37.8 million matches: 7129 us a call; drained
        // at every segment's end 8734).
        auto full = [](int) __attribute__((always_inline)) { return false; };
        uint32_t sl = cur;
        bool ok = cur_ok, first = true;
        while (ok || qlen > 0) {
            for (int j = 0; j < SEGS; ++j) {
                const std::integral_constant<int, 0> j0{};
                bool queued = !ok;        // nothing (more) to queue
                ChunkRegs<1> r1;
                uint32_t d4[1];
                unsigned m = 0;
                if (ok) {
                    load_segment<SEGS>(F, M.chunk(sl), j, lane, r1);
                    m = filter(r1, j0, mul, d4);
                    if (first) {
                        const int g = SEGS < 2 ? j : j / 2;
                        if (g < rest_g) m = 0;
                        if (g == rest_g) m &= rest >> (SEGS < 2 ? 0 : kBits * (j & 1));
                    }
                }
                while (true) {
                    if (!queued) queued = queue_mask(m, r1, d4, j0, (sl << 12) + uint32_t(j * kSegBytes), full);
                    while (qlen >= kDrain || (!ok && qlen > 0)) drain_walk(imin(qlen, kDrain));
                    if (queued) break;
                }
            }
            first = false;
            if (ok) {
                sl = nxt;
                ok = M.chunk(sl) < F.n_chunks;
                if (ok) {
                    // the slot after it: taken by the streaming loop, or now
                    nxt = __builtin_amdgcn_readfirstlane(ahead);
                    uint32_t t = 0;
                    if (lane == 0 && M.chunk(nxt) < F.n_chunks) t = atomicAdd(&snext, 1u);
                    ahead = t;
                }
            }
        }
    }

    const int64_t r0 = int64_t(blockIdx.x) * waves_per_block;
    if (!S.text_off) {
        // One text: the wave walks its own stored hits as soon as its
        // streaming is done, while the block's other waves still stream.
        // Its (now empty) queue holds the matches: q[0] counts them, then
        // (queue entry, keyword id) pairs; the block stores them after its
        // barrier with one global atomic.  Matches beyond the stage's room go
        // out directly.
        wave_sync();
        if (lane == 0) q[0] = 0u;
        // the hit records were stored by other lanes of this wave
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        wave_sync();
        // stages one match (queue entry with the match's position, keyword id)
        auto stage_one = [&](uint32_t ent, int64_t o, int32_t pid) __attribute__((always_inline)) {
            const uint32_t at = atomicAdd(&q[0], 1u);
            if (at < uint32_t(kWaveStageCap)) {
                q[2 + 2 * at] = ent;
                q[3 + 2 * at] = uint32_t(pid);
            } else {
                emit_one(S, nullptr, nullptr, o, 0, pid);
            }
        };
        // Writes the staged matches out with one atomic, when there may be no room
        // for one of each of the next `left` records.  Called by the whole wave.
        // (A match past the stage's room takes an atomic with the lanes that
        // reach theirs in the same step, few of them where windows lie at
        // different positions: 1.28 million matches in 128 MiB of log lines, 850
        // us a call without this, 211 with it.  More would not pay: atomics on
        // one address pass at about 85 M/s.)
        auto flush = [&](int left) __attribute__((always_inline)) {
            wave_sync();
            const int n = imin(__builtin_amdgcn_readfirstlane(int(q[0])), kWaveStageCap);
            if (left <= 0 || n + imin(left, kWave) <= kWaveStageCap) return;
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(S.count, static_cast<unsigned long long>(n)) - S.count_base;
            base = readlane64(base, 0);
            for (int i = int(lane); i < n; i += kWave)
                put_out(S, base + unsigned(i), offset_of(q[2 + 2 * i]), 0, int32_t(q[3 + 2 * i]));
            wave_sync();
            if (lane == 0) q[0] = 0u;
            wave_sync();
        };
        for (int i0 = 0; i0 < hcount; i0 += kWave, flush(hcount - i0)) {
            const int i = i0 + int(lane);
            if (i >= hcount) continue;
            uint2 rec;
            if (i < kLdsHits) rec = shits[wave * kLdsHits + i];
            else rec = gload8(hits + (i - kLdsHits));
            // a match at a window's o = first .. first + STRIDE - 1 has the
            // entry's position moved by as much (it stays below 4096)
            const int64_t first = offset_of(rec.x);
            auto put = [&](int64_t o, int32_t, int64_t, int32_t pid) __attribute__((always_inline)) {
                stage_one(rec.x + uint32_t(o - first), o, pid);
            };
            walk_hit(rec, [&](int64_t, int64_t &ts, int64_t &te, int32_t &id) { ts = 0; te = S.n; id = 0; },
                     [&](int64_t o, int32_t, int64_t, int32_t st) {
                         for (int32_t k = A.out_off[st], k1 = A.out_off[st + 1]; k < k1; ++k) put(o, 0, 0, A.out_pid[k]);
                     },
                     put);
        }
        __syncthreads();
        // every wave's matches are staged: one atomic reserves the block's
        // output range, and each wave stores its own from where the waves
        // before it end (each adds the counts up for itself)
        const int staged = int(lane) < waves_per_block ? imin(int(squeue[int(lane) * kQueueCap]), kWaveStageCap) : 0;
        const int before = prefix16(staged, lane);
        const int total = __builtin_amdgcn_readlane(before + staged, kMaxWaves - 1);
        unsigned long long *wbase = reinterpret_cast<unsigned long long *>(sfilt);   // the filter is done with
        if (total > 0) {
            if (threadIdx.x == 0) *wbase = atomicAdd(S.count, static_cast<unsigned long long>(total)) - S.count_base;
            __syncthreads();
            const int mine = __builtin_amdgcn_readlane(staged, wave);
            const unsigned long long base = *wbase + unsigned(__builtin_amdgcn_readlane(before, wave));
            for (int i = int(lane); i < mine; i += kWave) {
                const unsigned long long idx = base + unsigned(i);
                put_out(S, idx, offset_of(q[2 + 2 * i]), 0, int32_t(q[3 + 2 * i]));
            }
        }
    } else {
        // A batch: the block walks the hits its waves stored, spread over all
        // its threads (one flat index over the waves' regions), once every
        // wave is done.  The filter and queues are then free, so their LDS
        // holds the match stage (one global atomic per block) and the
        // batch's text starts for the walks' text lookups.
        // Each wave leaves its hit count in its own (empty) queue; after the
        // barrier the stage and the prefix sums of the counts go where the
        // filter was.
        if (lane == 0) q[0] = uint32_t(hcount);
        // The text starts go to LDS after the barrier; a batch of up to
        // kPreTexts starts per thread reads them now, into registers, while
        // the block's slowest waves still stream.
        constexpr int kPreTexts = 8;
        const bool pre_ok = S.n_texts < kPreTexts * int(blockDim.x) && S.n < (int64_t(1) << 32);
        int64_t pre[kPreTexts];
        int64_t pre_base = 0;
        if (pre_ok) {
            pre_base = S.text_off[0];
#pragma unroll
            for (int k = 0; k < kPreTexts; ++k) {
                const int i = int(threadIdx.x) + k * int(blockDim.x);
                pre[k] = i <= S.n_texts ? S.text_off[i] : 0;
            }
        }
        __syncthreads();
        static_assert((sizeof(MatchStage) + 15) / 16 * 16 + (2 * kMaxWaves + 1) * 4 <= (1u << FLOG2),
                      "the walk's stage must fit where the filter was");
        MatchStage *st = reinterpret_cast<MatchStage *>(sfilt);
        int32_t *wfirst = reinterpret_cast<int32_t *>(sfilt + (sizeof(MatchStage) + 15) / 16 * 16);   // [kMaxWaves]
        // each wave adds the counts up for itself; the first leaves the sums
        // for the flat index's search
        const int whits = int(lane) < waves_per_block ? int(squeue[int(lane) * kQueueCap]) : 0;
        const int wbefore = prefix16(whits, lane);
        const int32_t total = __builtin_amdgcn_readlane(wbefore + whits, kMaxWaves - 1);
        if (wave == 0 && lane < kMaxWaves) wfirst[lane] = int(lane) < waves_per_block ? wbefore : 0x7fffffff;
        if (threadIdx.x == 0) st->n = 0;
        __syncthreads();
        // The text starts (as offsets from the first text) are copied to LDS
        // when they fit, beside the stage or where the prefix table was.
        constexpr int kStageEnd = ((sizeof(MatchStage) + 15) / 16 * 16 + (2 * kMaxWaves + 1) * 4 + 15) / 16 * 16;
        constexpr int kLdsTexts = FLOG2 >= 17 ? ((1 << FLOG2) - kStageEnd) / 4 : 2 * PT_SLOTS;
        static_assert(kLdsTexts >= 4096, "room for the text starts of a batch of 4096 texts");
        uint32_t *lds_off = FLOG2 >= 17 ? reinterpret_cast<uint32_t *>(sfilt + kStageEnd) : sptab;
        const uint32_t *loff = nullptr;
        // Per-text counts are added up in LDS behind the starts, when both
        // fit: the matches of a long text meet in every block, and atomics on
        // one address pass at about 85 M/s.
        uint32_t *lcnt = nullptr;
        if (S.per_text && total > 0 && 2 * int64_t(S.n_texts) + 1 <= kLdsTexts) {
            lcnt = lds_off + S.n_texts + 1;
            for (int i = int(threadIdx.x); i < S.n_texts; i += int(blockDim.x)) lcnt[i] = 0u;
        }
        if (total > 0 && S.n_texts < kLdsTexts && S.n < (int64_t(1) << 32)) {
            if (pre_ok) {
#pragma unroll
                for (int k = 0; k < kPreTexts; ++k) {
                    const int i = int(threadIdx.x) + k * int(blockDim.x);
                    if (i <= S.n_texts) lds_off[i] = uint32_t(pre[k] - pre_base);
                }
            } else {
                const int64_t base0 = S.text_off[0];
                for (int i = int(threadIdx.x); i <= S.n_texts; i += int(blockDim.x))
                    lds_off[i] = uint32_t(S.text_off[i] - base0);
            }
            loff = lds_off;
        }
        __syncthreads();
        // With more hits than the stage has room for, it is written out whenever
        // there may be no room for another of each thread (the log lines above
        // as a batch of 32 texts: 540 -> 147 us).
        for (int32_t i0 = 0; i0 < total; i0 += int32_t(blockDim.x)) {
            if (total > kStageCap) {
                __syncthreads();
                if (st->n > kStageCap - int32_t(blockDim.x)) write_stage(S, st);
                __syncthreads();
            }
            const int32_t i = i0 + int32_t(threadIdx.x);
            if (i >= total) continue;
            int j = 0;                               // wave (region) of flat index i
#pragma unroll
            for (int h = kMaxWaves / 2; h >= 1; h >>= 1)
                if (wfirst[j + h] <= i) j += h;
            const int k = i - wfirst[j];
            const uint2 rec = k < kLdsHits ? shits[j * kLdsHits + k]
                                           : reinterpret_cast<const uint2 *>(F.hits + (r0 + j) * F.hit_cap)[k - kLdsHits];
            walk_hit(rec,
                     [&](int64_t at, int64_t &ts, int64_t &te, int32_t &id) { locate_text(S, loff, at, ts, te, id); },
                     [&](int64_t o, int32_t id, int64_t ts, int32_t s2) { emit_staged(A, S, st, lcnt, o - ts, id, s2); },
                     [&](int64_t o, int32_t id, int64_t ts, int32_t pid) { emit_one(S, st, lcnt, o - ts, id, pid); });
        }
        flush_stage(S, st, lcnt);
    }

    if (S.host_count || S.dev_count) report_count(S);
}


using FilteredFn = void (*)(const KArgs);

template <int K, bool BM, int FLOG2, int STRIDE, bool DUAL, bool PAIR, bool WIN>
FilteredFn pick_segs(int segs) {
    switch (segs) {
        case 1: return filtered_kernel<K, BM, 1, FLOG2, STRIDE, DUAL, PAIR, WIN>;
        case 2: return filtered_kernel<K, BM, 2, FLOG2, STRIDE, DUAL, PAIR, WIN>;
        default: return filtered_kernel<K, BM, 4, FLOG2, STRIDE, DUAL, PAIR, WIN>;
    }
}

template <int K, int STRIDE, bool WIN>
FilteredFn pick_filter(int kind, int segs) {
    switch (kind) {
        case AC_FILTER_BYTES17: return pick_segs<K, false, 17, STRIDE, false, false, WIN>(segs);
        case AC_FILTER_BITS20: return pick_segs<K, true, 17, STRIDE, false, false, WIN>(segs);
        case AC_FILTER_BYTES16: return pick_segs<K, false, 16, STRIDE, false, false, WIN>(segs);
        case AC_FILTER_DUAL19: return pick_segs<K, true, 17, STRIDE, true, false, WIN>(segs);
        case AC_FILTER_PAIR20:
            // strides 2 and 4 only
            if constexpr (STRIDE > 1) return pick_segs<K, true, 17, STRIDE, false, true, WIN>(segs);
            else return nullptr;
        default: return pick_segs<K, true, 16, STRIDE, false, false, WIN>(segs);
    }
}

}  // namespace dev

// The filtered kernel of each stride (and prefix length), by filter kind and
// segments per chunk; nullptr for a combination that does not exist.
dev::FilteredFn pick_filtered_s1k1(int kind, int segs);
dev::FilteredFn pick_filtered_s1k2(int kind, int segs);
dev::FilteredFn pick_filtered_s1k3(int kind, int segs);
dev::FilteredFn pick_filtered_s2(int kind, int segs);
dev::FilteredFn pick_filtered_s4(int kind, int segs);
// strides 2 and 4 with the window table
dev::FilteredFn pick_filtered_s2w(int kind, int segs);
dev::FilteredFn pick_filtered_s4w(int kind, int segs);

}  // namespace pfac
