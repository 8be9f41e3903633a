// attn_split.h -- combining the split partial results of a unit (the work
// partition is described in attn_common.h).
//
// For a row with partials (o_s, lse_s), lse in log2 units:
//   M = max_s lse_s,  w_s = 2^(lse_s - M),  out = sum_s w_s o_s / sum_s w_s,
// and a split that saw no visible key (lse = -inf) has weight 0.  Partials
// are visited in worker order, so the result is deterministic.  (The sums
// are kept relative to the running maximum and rescaled when it grows, which
// gives the same value up to rounding.)
//
// Lane layout of a combining wavefront: lane (row, part) = 16 * row + part
// owns dims VE * part .. VE * part + VE - 1 (VE = D / 16) of row `row` of a
// group of 4 rows.  Partials are loaded kMergeBatch at a time (4 in the
// streaming kernels' own combine, whose registers are shared with the page
// pipeline), all loads issued before any is consumed.
#pragma once

#include "attn_common.h"

namespace tsattn {

constexpr int kMergeBatch = 8;

// Loads and stores coherent across the whole device (the L2 caches of all
// XCDs), so that the worker combining a unit sees the partials the others
// wrote in the same launch.  Scalar ones are relaxed atomics at agent scope;
// the 16-byte ones are buffer loads and stores over the partial area with the
// device-scope cache policy (the host combines in the kernel only while that
// area is below 2 GiB, so byte offsets fit the buffer's 32-bit offsets).  On
// gfx950 both are plain memory operations with that policy bit, and a store
// is visible device-wide once the issuing wavefront's vector memory counter
// has drained.
constexpr int kDeviceScope = 16;   // cache policy of buffer operations: sc1

__device__ __forceinline__ float ld_coherent(const float *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coherent(float *p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ block_rsrc_t partial_rsrc(const AttnParams &p) {
    return block_rsrc(p.ws_o, p.ws_o_bytes);
}
// The log-sum-exp area behind it: one float per row of D.
template <int D>
__device__ __forceinline__ block_rsrc_t lse_rsrc(const AttnParams &p) {
    return block_rsrc(p.ws_lse, p.ws_o_bytes / D);
}
// A row past both areas (which hold less than 2^31 and 2^31 / D bytes): loads
// from it return zeros and touch no memory.
template <int D>
constexpr uint32_t kNoRow = (1u << 31) / (D * sizeof(float));
// Partial-area elements elem .. elem + 3 (elem a multiple of 4).
__device__ __forceinline__ void st_partial16(const AttnParams &p, size_t elem, f32x4_t v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), partial_rsrc(p),
                                           (int)(elem * sizeof(float)), 0, kDeviceScope);
}
// Partial-area element elem.
__device__ __forceinline__ void st_partial4(const AttnParams &p, size_t elem, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), partial_rsrc(p), (int)(elem * sizeof(float)), 0,
                                          kDeviceScope);
}
__device__ __forceinline__ f32x4_t ld_partial16(const AttnParams &p, size_t elem) {
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                           partial_rsrc(p), (int)(elem * sizeof(float)), 0, kDeviceScope));
}
// Waits until every vector memory operation this wavefront issued is
// complete.  The wait itself is not a memory operation to the compiler, so
// compiler-only fences on both sides keep every memory access written before
// it above it and every one written after it below it (they emit no
// instruction; no cache is written back or invalidated).
__device__ __forceinline__ void wait_vmem() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0); expcnt, lgkmcnt left at their maximum
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Running log-sum-exp combination of partials for one lane's VE dims.
template <int VE>
struct Acc {
    float acc[VE];
    float den, M;
    __device__ void init() {
#pragma unroll
        for (int e = 0; e < VE; e++)
            acc[e] = 0.0f;
        den = 0.0f;
        M = -INFINITY;
    }
    // Adds a batch of up to kB partials (n valid) given their rows.  What is
    // not valid is not read and counts as zeros: another partial's values in
    // its place may be infinite, and a weight of 0 would make them NaN.
    // kCoherent: read them with device-coherent loads (partials written by
    // other workers of the same launch), else with plain vector loads.
    template <int D, bool kCoherent, int kB>
    __device__ void add_batch(const AttnParams &p, const size_t *rows, int n, int part) {
        float l[kB];
        float4 v[kB][VE / 4];
#pragma unroll
        for (int k = 0; k < kB; k++) {
            l[k] = -INFINITY;
#pragma unroll
            for (int e = 0; e < VE / 4; e++)
                v[k][e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k >= n)
                continue;
            const float *src = p.ws_o + rows[k] * D + VE * part;
            if constexpr (kCoherent) {
                l[k] = ld_coherent(p.ws_lse + rows[k]);
#pragma unroll
                for (int e = 0; e < VE / 4; e++) {
                    const f32x4_t t = ld_partial16(p, rows[k] * D + VE * part + 4 * e);
                    v[k][e] = make_float4(t[0], t[1], t[2], t[3]);
                }
            } else {
                l[k] = p.ws_lse[rows[k]];
#pragma unroll
                for (int e = 0; e < VE / 4; e++)
                    v[k][e] = *reinterpret_cast<const float4 *>(src + 4 * e);
            }
        }
        add_loaded<kB>(l, v);
    }
    // Adds the partials at rows at[0 .. kB - 1] of the partial area, with
    // device-coherent loads; the first n are rows, the others kNoRow<D>.
    template <int D, int kB>
    __device__ void add_at(const AttnParams &p, const uint32_t *at, int n, int part) {
        float l[kB];
        float4 v[kB][VE / 4];
#pragma unroll
        for (int k = 0; k < kB; k++) {
            l[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                lse_rsrc<D>(p), (int)(at[k] * (uint32_t)sizeof(float)), 0, kDeviceScope));
#pragma unroll
            for (int e = 0; e < VE / 4; e++) {
                const f32x4_t t = ld_partial16(p, (size_t)(at[k] * (uint32_t)D + (uint32_t)(VE * part + 4 * e)));
                v[k][e] = make_float4(t[0], t[1], t[2], t[3]);
            }
        }
#pragma unroll
        for (int k = 0; k < kB; k++)
            l[k] = k < n ? l[k] : -INFINITY;
        add_loaded<kB>(l, v);
    }
    // Adds kB partials held in registers (those with l = -inf count nothing;
    // their values are zero or finite, so a weight of 0 does).
    template <int kB>
    __device__ void add_loaded(const float (&l)[kB], const float4 (&v)[kB][VE / 4]) {
        float Mb = M;
#pragma unroll
        for (int k = 0; k < kB; k++)
            Mb = fmaxf(Mb, l[k]);
        if (Mb == -INFINITY)
            return;
        rescale(Mb);
        add_weighted<kB>(l, v);
    }
    // The same with M at least their maximum already.
    template <int kB>
    __device__ void add_weighted(const float (&l)[kB], const float4 (&v)[kB][VE / 4]) {
#pragma unroll
        for (int k = 0; k < kB; k++) {
            const float wt = l[k] == -INFINITY ? 0.0f : fast_exp2(l[k] - M);
            den += wt;
#pragma unroll
            for (int e = 0; e < VE / 4; e++) {
                acc[4 * e + 0] += wt * v[k][e].x;
                acc[4 * e + 1] += wt * v[k][e].y;
                acc[4 * e + 2] += wt * v[k][e].z;
                acc[4 * e + 3] += wt * v[k][e].w;
            }
        }
    }
    __device__ void rescale(float Mnew) {
        const float a = M == -INFINITY ? 0.0f : fast_exp2(M - Mnew);
        den *= a;
#pragma unroll
        for (int e = 0; e < VE; e++)
            acc[e] *= a;
        M = Mnew;
    }
};

// Adds to `a` the partials k = k0, k0 + kstep, ... of row rr of the unit,
// kB at a time.
template <int D, bool kCoherent, int kB = kMergeBatch>
__device__ void gather_partials(const AttnParams &p, const UnitSplit &u, size_t rr, int part,
                                int k0, int kstep, Acc<D / 16> &a) {
    const size_t R = p.rows_per_unit;
    for (int kb = k0; kb < u.nparts; kb += kstep * kB) {
        size_t rows[kB];
        int n = 0;
#pragma unroll
        for (int k = 0; k < kB; k++) {
            const int kk = kb + kstep * k;
            rows[k] = (size_t)u.slot(kk < u.nparts ? kk : kb) * R + rr;
            n += kk < u.nparts;
        }
        a.template add_batch<D, kCoherent, kB>(p, rows, n, part);
    }
}

// Normalises and writes row r (of the unit's rows_per_unit) as bf16.
template <int D>
__device__ __forceinline__ void write_merged(const AttnParams &p, int b, int g, int r, int part,
                                             const Acc<D / 16> &a) {
    constexpr int VE = D / 16;
    const float inv = a.den > 0.0f ? 1.0f / a.den : 0.0f;
    const int i = r / p.G;
    uint16_t *dst = p.out + (((size_t)b * p.Qmax + i) * p.Hq + (size_t)g * p.G + r % p.G) * D + VE * part;
    uint32_t w2[VE / 2];
#pragma unroll
    for (int e = 0; e < VE / 2; e++)
        w2[e] = pack_bf16x2(a.acc[2 * e] * inv, a.acc[2 * e + 1] * inv);
    if constexpr (VE == 8)
        *reinterpret_cast<uint4 *>(dst) = make_uint4(w2[0], w2[1], w2[2], w2[3]);
    else
        *reinterpret_cast<uint2 *>(dst) = make_uint2(w2[0], w2[1]);
}

// Combines all pieces of unit (b, g) and writes its rows (4 per pass and
// wavefront, from row `first`, `step` apart; rows of draft positions >= q_len
// are skipped).  Called by the worker that counted the last arrival on the
// unit, which then sets the counter back to zero for the next call.
template <int D>
__device__ void combine_unit(const AttnParams &p, int b, int g, const UnitSplit &u, int lane, int first = 0,
                             int step = 4) {
    const int part = lane & 15;
    const int R = p.rows_per_unit;
    const int Q = ld_meta(p.q_lens, b);
    for (int r0 = first; r0 < R; r0 += step) {
        const int r = r0 + (lane >> 4);
        const bool row_ok = r < R && r / p.G < Q;
        Acc<D / 16> a;
        a.init();
        gather_partials<D, true, 4>(p, u, row_ok ? r : 0, part, 0, 1, a);
        if (row_ok)
            write_merged<D>(p, b, g, r, part, a);
    }
    // every arrival has been counted: leave the counter zero for the next call
    __hip_atomic_store(unit_counter(p, b * p.Hkv + g), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// kCombineLast: counts this wavefront's arrival on the unit of a piece whose
// partial it has just written with device-coherent stores; the last arriver
// combines the unit.  The stores are complete once the vector memory counter
// has drained, so no cache-wide fence is needed, and the last arriver's loads
// are issued after its count returned.  The counters are zero between calls
// (the workspace is zero-filled before its first use, and each call leaves
// them zero).
template <int D>
__device__ void arrive_and_combine(const AttnParams &p, const Segment &s, int64_t ptot, int lane) {
    wait_vmem();
    int old = 0;
    if (lane == 0)
        old = atomicAdd(unit_counter(p, s.b * p.Hkv + s.g), 1);
    old = first_lane_int(old);
    const UnitSplit u = unit_split(ptot, s.us, s.np, p.W);
    if (old == u.nparts - 1)
        combine_unit<D>(p, s.b, s.g, u, lane);
}

// kCombineInLaunch: a worker has split pieces in at most two units (the first
// and the last segment of its range) and counts its arrivals on them once,
// after its whole range: every piece of a split unit ends near the end of
// the launch anyway, and a drain of the stores between segments would stall
// the worker for a memory round trip.
struct Arrivals {
    int u0, u1;   // units of the pending arrivals, -1 for none
    __device__ __forceinline__ void init() { u0 = u1 = -1; }
    __device__ __forceinline__ void add(const AttnParams &p, const Segment &s) {
        if (!s.whole && p.combine == kCombineInLaunch) {
            const int u = s.b * p.Hkv + s.g;
            if (u0 < 0)
                u0 = u;
            else
                u1 = u;
        }
    }
    // The same for a group of wavefronts, which writes at most two partials:
    // of the unit its range starts in and of the one it ends in.
    __device__ __forceinline__ void add_unit(const AttnParams &p, int u) {
        if (p.combine != kCombineKernel) {
            if (u0 < 0)
                u0 = u;
            else
                u1 = u;
        }
    }
    // kCombineLast for a workgroup of kGroupWaves wavefronts: the arrivals of
    // both units are counted at once, and the workgroup that counted a unit's
    // last one combines it.  `last`: two ints of LDS.
    template <int D>
    __device__ __forceinline__ void combine_last(const AttnParams &p, const int *s_pre, int64_t ptot, int *last) {
        if (u0 < 0)
            return;
        wait_vmem();
        __syncthreads();   // every wavefront's stores are complete
        if (threadIdx.x < 2) {
            const int unit = threadIdx.x ? u1 : u0;
            int mine = 0;
            if (unit >= 0) {
                const int old = atomicAdd(unit_counter(p, unit), 1);
                mine = old == split_of(p, s_pre, unit, ptot).nparts - 1;
            }
            last[threadIdx.x] = mine;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (!first_lane_int(last[k]))
                continue;
            const int unit = k ? u1 : u0;
            combine_unit<D>(p, unit / p.Hkv, unit % p.Hkv, split_of(p, s_pre, unit, ptot),
                            (int)(threadIdx.x & (kWave - 1)), 4 * (int)(threadIdx.x / kWave), 4 * kGroupWaves);
        }
    }
    __device__ static UnitSplit split_of(const AttnParams &p, const int *s_pre, int unit, int64_t ptot) {
        const int b = unit / p.Hkv, g = unit % p.Hkv;
        const int np = s_pre[b + 1] - s_pre[b];
        return unit_split(ptot, (int64_t)p.Hkv * s_pre[b] + (int64_t)g * np, np, p.W);
    }
    // kCombineInLaunch: called by every thread of the workgroup, at the end of
    // its work; the first wavefront counts.
    template <int D, bool kBlock>
    __device__ __forceinline__ void flush(const AttnParams &p, const int *s_pre, int64_t ptot);
};

// Sums of waves 1 .. kWaves - 1 of a workgroup added into wave 0's `a` (the
// same lanes of each wave hold the same rows and dims), through LDS at
// `comb` (3 * (VE + 2) * 64 floats).  Every thread of the workgroup calls it.
template <int VE, int kWaves>
__device__ void combine_waves(Acc<VE> &a, float *comb, int wave, int lane) {
    float(*c)[VE + 2][64] = reinterpret_cast<float(*)[VE + 2][64]>(comb);
    if (wave > 0) {
#pragma unroll
        for (int e = 0; e < VE; e++)
            c[wave - 1][e][lane] = a.acc[e];
        c[wave - 1][VE][lane] = a.den;
        c[wave - 1][VE + 1][lane] = a.M;
    }
    __syncthreads();
    if (wave != 0)
        return;
    float Mall = a.M;
#pragma unroll
    for (int w = 0; w < kWaves - 1; w++)
        Mall = fmaxf(Mall, c[w][VE + 1][lane]);
    if (Mall == -INFINITY)
        return;   // no partial saw a visible key: the sums stay zero
    a.rescale(Mall);
#pragma unroll
    for (int w = 0; w < kWaves - 1; w++) {
        const float Mw = c[w][VE + 1][lane];
        const float f = Mw == -INFINITY ? 0.0f : fast_exp2(Mw - Mall);
        a.den += f * c[w][VE][lane];
#pragma unroll
        for (int e = 0; e < VE; e++)
            a.acc[e] += f * c[w][e][lane];
    }
}

// ---------------------------------------------------------------------------
// Merge wavefronts in the streaming launch (kCombineInLaunch).
//
// The grid holds the W workers and then the merge workgroups, one wavefront
// per row of each unit (single-wavefront kernels: workgroup W + m is row
// m % R of unit m / R; group and team kernels: wave w of workgroup W + m is
// row 4 (m % ceil(R / 4)) + w of unit m / ceil(R / 4)).  A merge wavefront
// waits until every worker with a piece of its unit has counted its arrival,
// then its four 16-lane groups read pieces k, k + 4, ... (k = lane / 16)
// with device-coherent loads, so up to 4 * kMergeBatch pieces cost one
// memory round trip; the groups' sums meet through cross-lane exchanges and
// group 0 writes the row.  The host takes this mode for units with many
// pieces (a few long sequences), where the merge kernel's launch after the
// whole grid was a large share of a short call.
//
// Forward progress: the dispatcher starts the workgroups of each XCD in
// increasing order, so the merge workgroups of an XCD start after the workers
// of that XCD, and workers never wait.  But the workers of the other XCDs need
// not have started: another call, on another stream, may hold the slots they
// need with merge workgroups of its own.  The host therefore takes this mode
// only while the merge workgroups fill at most half of the slots of every XCD.
// Of two overlapping calls at least one then finds room for its workers beside
// the other's merge workgroups on every XCD, finishes, and frees the other.
// Three calls and more can fill an XCD between them.  So the wait is bounded
// (p.merge_polls polls): a merge wavefront that has waited that long leaves,
// which frees its slot, and the worker that arrives last on the unit merges
// the unit's rows in its place.  Nothing in a launch thus depends on the order
// or the place in which its workgroups start.
//
// Counter protocol: the unit's word counts arrivals of workers (low 32 bits),
// merge wavefronts that are through with the unit (16 bits) and those of them
// that left without the partials (16 bits), all in single 64-bit atomic
// additions.  Each of the nparts workers and of the merge wavefronts with a
// valid row adds exactly once:
//   * a merge wavefront that saw all arrivals reads the partials, then adds
//     kMergeDone;
//   * one that gives up adds kMergeDone + kMergeLeft.  If that finds all
//     arrivals counted, it merges its row after all; if not, the worker whose
//     arrival is the last finds kMergeLeft counted and merges every row of the
//     unit (rows that other wavefronts merge too get the same values twice);
//   * whoever adds last, by the counts, sets the word back to zero for the
//     next call.
// The host spaces the words of the units apart (cnt_shift, at least 9 in this
// mode): with all of them on one line, every worker's arrival and every merge
// wavefront's poll queued on that line, which made the block-draft call 38 %
// slower.
typedef unsigned long long unit_word_t;
constexpr unit_word_t kMergeDone = 1ull << 32, kMergeLeft = 1ull << 48;
__device__ __forceinline__ uint32_t word_arrived(unit_word_t w) { return (uint32_t)w; }
__device__ __forceinline__ int word_done(unit_word_t w) { return (int)((w >> 32) & 0xffff); }
__device__ __forceinline__ int word_left(unit_word_t w) { return (int)(w >> 48); }
__device__ __forceinline__ unit_word_t *unit_word(const AttnParams &p, int unit) {
    return reinterpret_cast<unit_word_t *>(unit_counter(p, unit));
}
__device__ __forceinline__ void clear_word(unit_word_t *w) {
    __hip_atomic_store(w, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until `target` workers have arrived; false if `polls` polls saw less.
__device__ __forceinline__ bool wait_arrivals(const unit_word_t *w, int target, int polls) {
    const int *c = reinterpret_cast<const int *>(w);   // the low half
    for (int i = 0; i < polls; i++) {
        const int v = first_lane_int(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (v >= target) {
            __atomic_signal_fence(__ATOMIC_SEQ_CST);   // later loads stay after the poll
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

// Sums of the four 16-lane groups (same part, different pieces) combined;
// every group gets the total.
template <int VE>
__device__ __forceinline__ void combine_lane_groups(Acc<VE> &a) {
    const auto add = [](float x, float y) { return x + y; };
    const float Mall = max_across_lane_groups(a.M);
    const float f = a.M == -INFINITY ? 0.0f : fast_exp2(a.M - Mall);
    a.den = across_lane_groups(a.den * f, add);
#pragma unroll
    for (int e = 0; e < VE; e++)
        a.acc[e] = across_lane_groups(a.acc[e] * f, add);
    a.M = Mall;
}

// Draft rows of unit (b, .) with i < q_len: the merge wavefronts that count.
__device__ __forceinline__ int valid_rows(const AttnParams &p, int b) {
    return min(p.rows_per_unit, ld_meta(p.q_lens, b) * p.G);
}

// Combines and writes row r of unit `unit` (one wavefront).
template <int D>
__device__ void merge_in_launch(const AttnParams &p, const int *s_pre, int unit, int r) {
    const int b = unit / p.Hkv, g = unit % p.Hkv;
    const int np = s_pre[b + 1] - s_pre[b];
    if (np == 0)
        return;
    const int nvalid = valid_rows(p, b);
    if (r >= nvalid)
        return;
    const int64_t ptot = (int64_t)p.Hkv * s_pre[p.B];
    const int64_t us = (int64_t)p.Hkv * s_pre[b] + (int64_t)g * np;
    const UnitSplit u = unit_split(ptot, us, np, p.W);
    if (u.wlo == u.whi)
        return;   // one worker saw the whole unit and wrote `out`
    const int lane = threadIdx.x & 63;
    unit_word_t *word = unit_word(p, unit);
    // Up to 4 * kMergeBatch pieces: where they lie is worked out before the
    // wait, so that only the loads follow it.
    constexpr int VE = D / 16;
    uint32_t at[kMergeBatch];
#pragma unroll
    for (int k = 0; k < kMergeBatch; k++) {
        const int kk = (lane >> 4) + 4 * k;
        at[k] = kk < u.nparts ? (uint32_t)u.slot(kk) * (uint32_t)p.rows_per_unit + (uint32_t)r : kNoRow<D>;
    }
    const int nmine = (u.nparts - (lane >> 4) + 3) >> 2;   // this lane group's pieces
    const bool seen = wait_arrivals(word, u.nparts, p.merge_polls);
    unit_word_t old = 0;
    if (__builtin_expect(!seen, 0)) {
        if (lane == 0)
            old = atomicAdd(word, kMergeDone + kMergeLeft);
        if (first_lane_int((int)word_arrived(old)) != u.nparts)
            return;   // the last worker to arrive merges the row
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
    }
    Acc<VE> a;
    a.init();
    if (u.nparts <= 4 * kMergeBatch) {
        // 16 pieces and fewer take half of the loads (wavefront-uniform)
        if (u.nparts <= 2 * kMergeBatch)
            a.template add_at<D, kMergeBatch / 2>(p, at, nmine, lane & 15);
        else
            a.template add_at<D, kMergeBatch>(p, at, nmine, lane & 15);
    } else {
        gather_partials<D, true>(p, u, r, lane & 15, lane >> 4, 4, a);
    }
    combine_lane_groups(a);
    if (lane < 16)
        write_merged<D>(p, b, g, r, lane, a);
    if (lane == 0) {
        if (seen)
            old = atomicAdd(word, kMergeDone);
        if (word_done(old) == nvalid - 1)   // all workers have arrived
            clear_word(word);
    }
}

// The rows of a unit whose merge wavefronts left, by the wavefront that
// counted the last arrival: the sums of merge_in_launch in its order (so the
// same values), but small rather than fast code, since it runs only when a
// call was held up.
template <int D>
__device__ void merge_rows(const AttnParams &p, const UnitSplit &u, int b, int g, int nvalid, int lane) {
    constexpr int VE = D / 16;
    const int part = lane & 15;
#pragma unroll 1
    for (int r = 0; r < nvalid; r++) {
        Acc<VE> a;
        a.init();
#pragma unroll 1
        for (int kb = lane >> 4; kb < u.nparts; kb += 4 * kMergeBatch) {
            const int ke = min(kb + 4 * kMergeBatch, u.nparts);
            float Mb = a.M;
#pragma unroll 1
            for (int k = kb; k < ke; k += 4)
                Mb = fmaxf(Mb, ld_coherent(p.ws_lse + (size_t)u.slot(k) * p.rows_per_unit + r));
            if (Mb == -INFINITY)
                continue;
            a.rescale(Mb);
#pragma unroll 1
            for (int k = kb; k < ke; k += 4) {
                const size_t row = (size_t)u.slot(k) * p.rows_per_unit + r;
                float l[1] = {ld_coherent(p.ws_lse + row)};
                float4 v[1][VE / 4];
#pragma unroll
                for (int e = 0; e < VE / 4; e++) {
                    const f32x4_t t = ld_partial16(p, row * D + VE * part + 4 * e);
                    v[0][e] = make_float4(t[0], t[1], t[2], t[3]);
                }
                a.template add_weighted<1>(l, v);
            }
        }
        combine_lane_groups(a);
        if (lane < 16)
            write_merged<D>(p, b, g, r, lane, a);
    }
}

// The first wavefront counts the workgroup's arrivals, lane 0 on the unit its
// range starts in, lane 1 on the one it ends in.  What it has to do for merge
// wavefronts that left is decided by the counts found.
template <int D, bool kBlock>
__device__ __forceinline__ void Arrivals::flush(const AttnParams &p, const int *s_pre, int64_t ptot) {
    if (u0 < 0)
        return;
    wait_vmem();
    if constexpr (kBlock) {
        __syncthreads();   // every wavefront's stores are complete
        if (threadIdx.x >= kWave)
            return;
    }
    const int lane = threadIdx.x;
    unit_word_t old = 0;
    if (lane < 2 && (lane ? u1 : u0) >= 0)
        old = atomicAdd(unit_word(p, lane ? u1 : u0), 1ull);
    // no merge wavefront is through with the unit: none has left, and others
    // will add after this one
    if (__builtin_expect(!__any(word_done(old) != 0), 1))
        return;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll 1
    for (int k = 0; k < 2; k++) {
        const int unit = k ? u1 : u0;
        const int arrived = __builtin_amdgcn_readlane((int)word_arrived(old), k);
        const int through = __builtin_amdgcn_readlane((int)(old >> 32), k);
        if (unit < 0 || through == 0)
            continue;
        const int b = unit / p.Hkv, g = unit % p.Hkv;
        const UnitSplit u = split_of(p, s_pre, unit, ptot);
        if (arrived != u.nparts - 1)
            continue;
        const int nvalid = valid_rows(p, b);
        if (word_left((unit_word_t)(uint32_t)through << 32))
            merge_rows<D>(p, u, b, g, nvalid, lane);
        if (lane == 0 && (through & 0xffff) == nvalid)
            clear_word(unit_word(p, unit));
    }
}

}  // namespace tsattn
