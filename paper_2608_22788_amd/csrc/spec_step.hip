// spec_step.hip -- the two steps around the verify attention in one
// speculative decoding step (paper Sec. 3.4: drafts are verified by the
// target model, losslessly, following the speculative sampling of Leviathan
// et al.):
//
//   * KV append: the step's 1 + gamma new tokens' key and value rows are
//     written into the paged pool before the attention reads them (the
//     attention's context length counts them).  One thread per 16-byte piece
//     of a row; HBM-bound and tiny.
//
//   * acceptance: per sequence, walk the drafts while u_i * q_i(d_i) <=
//     p_i(d_i); at the first rejection k draw the next token from the
//     leftover mass max(0, p_k - q_k), after full acceptance from the bonus
//     row p_gamma, by inverse CDF with the caller's uniform.  The rule is
//     stated over real numbers and is evaluated here without rounding: the
//     test u q <= p on float64 products (exact for float32 factors), and the
//     weights and their running sums as integers in units of 2^-149, the
//     smallest float32, held in three 64-bit words (Fx below).  So the result
//     does not depend on the order of the sums, and the parallel evaluation
//     gives exactly the sequential one.  The sampling row is a full
//     vocabulary of fp32 probabilities per sequence, so the work is a
//     streaming read of one or two rows:
//       - accept_blocks_kernel: every 1,024-element block of every sequence's
//         sampling row is summed by one wavefront (exact float64
//         accumulators, then a wavefront scan), so the whole chip shares the
//         read even for a handful of sequences.  A block of 512 elements
//         makes the walk and the cross-lane sum, which every wavefront pays,
//         5 % of the call dearer (128 sequences x 151,936 tokens: 31.9
//         against 30.3 us), and 8 sequences gain nothing;
//       - accept_pick_kernel: one wavefront per sequence scans the block sums
//         (lane runs of consecutive blocks, a wavefront scan of the run
//         totals), finds the block where the cumulative mass first exceeds
//         floor(u * total), then the lane run of 16 elements inside it and
//         the element.
//     The first kernel repeats the acceptance walk in every wavefront (two
//     dependent loads); the second reads its result.
//     Measured (151,936 tokens, 3 drafts, per call): 128 sequences 30.3 us
//     against 89 us with the weights added one by one as 192-bit integers
//     (block sums 86 -> 24 us; reading two rows of every sequence takes
//     22 us); 8 sequences 11.3 us of kernel time against 17.4 us, a chain of
//     memory latencies.
//   Readings: probabilities are clamped to [0, 1] and uniforms to
//   [0, 1 - 2^-24], NaN read as 0; a draft id outside [0, V) is rejected; if
//   the leftover mass is zero the next token is drawn from p_k itself; a
//   sampling row without mass gives token -1.
#include <hip/hip_runtime.h>

#include <climits>

#include "ts_attn.h"
#include "ts_internal.h"
#include "wave_scan.h"

namespace tsattn {

namespace {

constexpr int kWave = 64;
constexpr int kQuads = 4;          // groups of 4 elements per lane of a block
constexpr int kBlk = kWave * 4 * kQuads;   // vocabulary elements per block
constexpr int kWsBlk = 256;        // elements per block sum in the workspace size
constexpr int kPickThreads = 64;   // pick workgroup: one wavefront

struct AppendParams {
    const uint16_t *k_new, *v_new;   // [B][Qmax][Hkv][D]
    uint16_t *k_pages, *v_pages;     // [num_pages][Hkv][16][D]
    const int32_t *page_table, *ctx_lens, *q_lens;
    int64_t num_pages;
    int B, Qmax, Hkv, D, max_pages;
};

__global__ __launch_bounds__(256) void kv_append_kernel(AppendParams p) {
    const int chunks = p.D / 8;   // 16-byte pieces per row
    const int64_t total = (int64_t)p.B * p.Qmax * p.Hkv * chunks;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= total)
        return;
    const int c = (int)(id % chunks);
    int64_t r = id / chunks;
    const int g = (int)(r % p.Hkv);
    r /= p.Hkv;
    const int i = (int)(r % p.Qmax);
    const int b = (int)(r / p.Qmax);
    const int Q = p.q_lens[b];
    if (i >= Q)
        return;
    const int t = p.ctx_lens[b] - Q + i;
    if (t < 0 || t >= p.max_pages * 16)
        return;   // violated precondition: write nothing rather than out of bounds
    const int page = p.page_table[(size_t)b * p.max_pages + t / 16];
    if (page < 0 || page >= p.num_pages)
        return;
    const size_t src = (((size_t)b * p.Qmax + i) * p.Hkv + g) * p.D + 8 * c;
    const size_t dst = (((size_t)page * p.Hkv + g) * 16 + t % 16) * p.D + 8 * c;
    *reinterpret_cast<uint4 *>(p.k_pages + dst) = *reinterpret_cast<const uint4 *>(p.k_new + src);
    *reinterpret_cast<uint4 *>(p.v_pages + dst) = *reinterpret_cast<const uint4 *>(p.v_new + src);
}

struct AcceptParams {
    const float *p;          // [B][G+1][V]
    const float *q;          // [B][G][V]
    const int32_t *draft;    // [B][G]
    const int32_t *num_draft;
    const float *u_accept;   // [B][G]
    const float *u_sample;   // [B]
    int32_t *n_accepted, *next_token;
    uint64_t *bsum;          // [B][2][nblk][3] exact block sums of the sampling row
    int32_t *walk;           // [B] drafts accepted, as the block-sum kernel found them
    int B, V, G, nblk;
};

// ---- exact fixed point --------------------------------------------------------
// A float32 in [0, 1] is an integer number of units of 2^-149 (the smallest
// positive subnormal), below 2^150 of them; a row of at most 2^31 such
// weights sums to below 2^181.  Fx holds such integers in three 64-bit words,
// so every sum and comparison below is exact and independent of order.
struct Fx {
    uint64_t w0, w1, w2;
};

__device__ __forceinline__ Fx fx_zero() { return Fx{0, 0, 0}; }

__device__ __forceinline__ Fx fx_add(Fx a, Fx b) {
    Fx r;
    r.w0 = a.w0 + b.w0;
    const uint64_t c0 = r.w0 < a.w0;
    const uint64_t t = a.w1 + b.w1;
    uint64_t c1 = t < a.w1;
    r.w1 = t + c0;
    c1 += r.w1 < t;
    r.w2 = a.w2 + b.w2 + c1;
    return r;
}

__device__ __forceinline__ bool fx_gt(Fx a, Fx b) {
    if (a.w2 != b.w2)
        return a.w2 > b.w2;
    if (a.w1 != b.w1)
        return a.w1 > b.w1;
    return a.w0 > b.w0;
}

__device__ __forceinline__ bool fx_is_zero(Fx a) { return (a.w0 | a.w1 | a.w2) == 0; }

// a - b for a > b.
__device__ __forceinline__ Fx fx_sub(Fx a, Fx b) {
    Fx r;
    r.w0 = a.w0 - b.w0;
    const uint64_t b0 = a.w0 < b.w0;
    const uint64_t t = a.w1 - b.w1;
    uint64_t b1 = a.w1 < b.w1;
    r.w1 = t - b0;
    b1 += t < b0;
    r.w2 = a.w2 - b.w2 - b1;
    return r;
}

// A clamped probability in units of 2^-149: significand M (with the implicit
// bit for normal numbers) shifted left by (biased exponent - 1), at most 126.
__device__ __forceinline__ Fx fx_of_prob(float x) {
    const uint32_t bits = __float_as_uint(x);
    const uint32_t e = bits >> 23, f = bits & 0x7fffffu;
    const uint64_t M = e ? (uint64_t)(f | 0x800000u) : (uint64_t)f;
    const uint32_t sh = e ? e - 1 : 0;
    const uint32_t off = sh & 63;
    const uint64_t lo = M << off;
    const uint64_t hi = off ? M >> (64 - off) : 0;
    return sh < 64 ? Fx{lo, hi, 0} : Fx{0, lo, hi};
}

// A uniform clamped to [0, 1 - 2^-24] (NaN and negatives read as 0).
__device__ __forceinline__ float clamp_uniform(float u) {
    return u > 0.0f ? fminf(u, 0x1.fffffep-1f) : 0.0f;
}

// floor(u * Z) for a clamped uniform u: u = m 2^-s with m < 2^24 and
// s >= 24, so m Z < 2^205 takes four words before the shift.
__device__ __forceinline__ Fx fx_floor_mul(Fx Z, float u) {
    const uint32_t bits = __float_as_uint(u);
    const uint32_t e = bits >> 23, f = bits & 0x7fffffu;
    const uint64_t m = e ? (uint64_t)(f | 0x800000u) : (uint64_t)f;
    const uint32_t s = e ? 150 - e : 149;
    uint64_t r[4];
    const uint64_t lo0 = m * Z.w0, hi0 = __umul64hi(m, Z.w0);
    const uint64_t lo1 = m * Z.w1, hi1 = __umul64hi(m, Z.w1);
    const uint64_t lo2 = m * Z.w2, hi2 = __umul64hi(m, Z.w2);
    r[0] = lo0;
    r[1] = lo1 + hi0;
    const uint64_t c1 = r[1] < lo1;
    const uint64_t t = lo2 + hi1;
    uint64_t c2 = t < lo2;
    r[2] = t + c1;
    c2 += r[2] < t;
    r[3] = hi2 + c2;
    const uint32_t ws = s >> 6, bs = s & 63;
    uint64_t out[3];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        // words i + ws and i + ws + 1 of r (zero past the top), selected
        // without dynamic indexing
        uint64_t a = 0, b = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            a = (uint32_t)(i + (int)ws) == (uint32_t)j ? r[j] : a;
            b = (uint32_t)(i + (int)ws + 1) == (uint32_t)j ? r[j] : b;
        }
        out[i] = (a >> bs) | (bs ? b << (64 - bs) : 0);
    }
    return Fx{out[0], out[1], out[2]};
}

__device__ __forceinline__ Fx fx_shfl(Fx a, int lane) {
    return Fx{__shfl(a.w0, lane, kWave), __shfl(a.w1, lane, kWave), __shfl(a.w2, lane, kWave)};
}

template <int CTRL, int kRows>
__device__ __forceinline__ Fx lane_move(Fx x) {
    return Fx{tsattn::lane_move<CTRL, kRows>(x.w0), tsattn::lane_move<CTRL, kRows>(x.w1),
              tsattn::lane_move<CTRL, kRows>(x.w2)};
}
__device__ __forceinline__ Fx fx_incl_scan(Fx x) {
    return wave_incl_scan(x, [](Fx a, Fx b) { return fx_add(a, b); });
}

// ---- exact sums in float64 ------------------------------------------------------
// Adding every weight as an Fx costs about 60 instructions per element, which
// made the streaming kernel bound by the vector ALU (128 sequences x 151,936
// tokens: 86 us, 1.8 TB/s).  The weights are therefore summed in four float64
// accumulators, each of which only ever holds multiples of a power of two and
// stays below 2^53 of them, so that every addition is exact: multiples of
// 2^-40 (sums up to 2^10), 2^-81, 2^-122 and 2^-149.  Adding and subtracting
// 1.5 * 2^(52 - k) rounds a value to a multiple of 2^-k, and what is left over
// (at most half of that) is exact and goes to the next accumulator.  Only
// weights with bits below 2^-81 reach the last two, on a branch the whole
// wavefront skips otherwise.  About 20 instructions per element, and v_add_f64
// issues at the rate of v_add_f32.
constexpr int kBinA = 40, kBinB = 81, kBinC = 122, kBinD = 149;
struct Bins {
    double a, b, c, d;
};
__device__ __forceinline__ Bins bins_zero() { return Bins{0.0, 0.0, 0.0, 0.0}; }

template <int K>
__device__ __forceinline__ double to_multiple(double x) {
    constexpr double c = K == kBinA ? 0x1.8p12 : K == kBinB ? 0x1.8p-29 : 0x1.8p-70;   // 1.5 * 2^(52 - K)
    return (x + c) - c;
}

__device__ __forceinline__ uint32_t high_word(double x) {
    return (uint32_t)((uint64_t)__double_as_longlong(x) >> 32);
}

// Adds the weights of four elements (clamped probabilities): w_j =
// max(0, p_j - q_j) (kResid), else p_j.  p - min(p, q) is that weight; in
// float64 it may round, and err is then the exact rest (p >= q).
template <bool kResid>
__device__ __forceinline__ void bins_add4(Bins &s, const float pe[4], const float qe[4]) {
    double rest[4], err[4];
    uint32_t small = 0;   // a nonzero value of this size has a nonzero high word
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const double p = pe[j];
        double w = p;
        err[j] = 0.0;
        if constexpr (kResid) {
            // values in [0, 1] order as their bits do
            const double q = __uint_as_float(min(__float_as_uint(pe[j]), __float_as_uint(qe[j])));
            w = p - q;
            err[j] = (p - w) - q;
            small |= high_word(err[j]);
        }
        const double ha = to_multiple<kBinA>(w);
        const double lo = w - ha;
        const double hb = to_multiple<kBinB>(lo);
        s.a += ha;
        s.b += hb;
        rest[j] = lo - hb;
        small |= high_word(rest[j]);
    }
    if (__any(small != 0)) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const double eb = to_multiple<kBinB>(err[j]);
            s.b += eb;
            const double er = err[j] - eb;
            const double c0 = to_multiple<kBinC>(rest[j]), c1 = to_multiple<kBinC>(er);
            s.c += c0 + c1;
            s.d += (rest[j] - c0) + (er - c1);
        }
    }
}

// x (a multiple of 2^-K, negative or not) in units of 2^-149, modulo 2^192.
template <int K>
__device__ __forceinline__ Fx fx_of_bin(double x) {
    constexpr int sh = kBinD - K;   // 109, 68, 27, 0
    int64_t n;
    if constexpr (K == kBinA || K == kBinB) {
        // x is below a third of this constant, so the sum keeps its exponent
        // and counts the units in its significand
        constexpr double c = K == kBinA ? 0x1.8p12 : 0x1.8p-29;
        n = __double_as_longlong(x + c) - __double_as_longlong(c);
    } else {
        n = (int64_t)(K == kBinC ? x * 0x1p122 : (x * 0x1p75) * 0x1p74);
    }
    constexpr int o = sh & 63;
    const uint64_t lo = (uint64_t)n << o, hi = o ? (uint64_t)(n >> ((64 - o) & 63)) : (uint64_t)(n >> 63);
    const uint64_t sign = (uint64_t)(n >> 63);
    return sh < 64 ? Fx{lo, hi, sign} : Fx{0, lo, hi};
}
__device__ __forceinline__ Fx fx_of_bins(const Bins &s) {
    Fx r = fx_add(fx_of_bin<kBinA>(s.a), fx_of_bin<kBinB>(s.b));
    if (__any(s.c != 0.0 || s.d != 0.0))
        r = fx_add(r, fx_add(fx_of_bin<kBinC>(s.c), fx_of_bin<kBinD>(s.d)));
    return r;
}

// The sum over the wavefront, in lane 63 (the other lanes hold partial sums).
__device__ __forceinline__ Fx bins_wave_sum(Bins s) {
    s.a = wave_incl_scan(s.a);
    s.b = wave_incl_scan(s.b);
    if (__any(s.c != 0.0 || s.d != 0.0)) {
        s.c = wave_incl_scan(s.c);
        s.d = wave_incl_scan(s.d);
    }
    return fx_of_bins(s);
}

// Read-only for the launch: through the constant address space, so that a
// wavefront-uniform read is a scalar load.
typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;
__device__ __forceinline__ int clamp_gamma(const AcceptParams &a, int b) {
    const int g = ((const_i32_ptr)a.num_draft)[b];
    return g < 0 ? 0 : (g > a.G ? a.G : g);
}

// A probability clamped to [0, 1] (NaN and negatives read as 0).
__device__ __forceinline__ float clamp_prob(float x) {
    return __uint_as_float(x > 0.0f ? min(__float_as_uint(x), 0x3f800000u) : 0u);
}

// Drafts accepted before the first rejection (gamma if none).  The test
// u q <= p is exact: the product of two float32 values is exact in float64.
// Every lane of the calling wavefront tests one draft (i = c + lane for
// c = 0, 64, ...), so a walk costs two dependent loads per 64 drafts (the
// drafts and uniforms do not wait for the draft count); the first failing
// draft is the lowest set bit of the ballot.
__device__ int accept_walk(const AcceptParams &a, int b, int gamma) {
    const int lane = threadIdx.x & (kWave - 1);
    for (int c = 0; c < a.G; c += kWave) {
        const int i = c + lane;
        int d = 0;
        float u = 0.0f;
        if (i < a.G) {
            d = a.draft[(size_t)b * a.G + i];
            u = clamp_uniform(a.u_accept[(size_t)b * a.G + i]);
        }
        bool bad = false;
        if (i < gamma) {
            if (d < 0 || d >= a.V) {
                bad = true;
            } else {
                const float p = clamp_prob(a.p[((size_t)b * (a.G + 1) + i) * a.V + d]);
                const float q = clamp_prob(a.q[((size_t)b * a.G + i) * a.V + d]);
                bad = !((double)u * (double)q <= (double)p);
            }
        }
        const unsigned long long m = __ballot(bad);
        if (m)
            return c + __ffsll((long long)m) - 1;
        if (c + kWave >= gamma)
            break;
    }
    return gamma;
}

// A lane's elements of a block: of the target row p_k and, at a rejection, of
// the draft row q_k (else zero), clamped.
struct Row {
    float p[kQuads][4], q[kQuads][4];
};

// Elements e0 + step * i + j (i < kQuads, j < 4) of the block at `src`, where
// `n` >= 1 elements of the row are left (zero past them; only the row's last
// block is not whole).  A row starts on a 16-byte boundary only if V is a
// multiple of 4; the loads ask for no more than the 4 bytes that every row
// has.  kStream: the elements are read once, so the lines need not stay in
// the caches (7 % of the call at 128 sequences x 151,936 tokens).
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
template <bool kStream>
__device__ __forceinline__ void load_block(const float *src, int n, int e0, int step, float x[kQuads][4]) {
    if (n >= kBlk) {   // wavefront-uniform
#pragma unroll
        for (int i = 0; i < kQuads; i++) {
            const f4_any *at = reinterpret_cast<const f4_any *>(src + e0 + step * i);
            const f4_any v = kStream ? __builtin_nontemporal_load(at) : *at;
#pragma unroll
            for (int j = 0; j < 4; j++)
                x[i][j] = v[j];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kQuads; i++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int e = e0 + step * i + j;
                const float v = src[min(e, n - 1)];
                x[i][j] = e < n ? v : 0.0f;
            }
    }
}
template <bool kResid, bool kStream>
__device__ __forceinline__ void load_rows(const AcceptParams &a, int b, int k, int blk, int e0, int step, Row &r) {
    const int first = blk * kBlk, n = a.V - first;
    load_block<kStream>(a.p + ((size_t)b * (a.G + 1) + k) * a.V + first, n, e0, step, r.p);
    if constexpr (kResid)
        load_block<kStream>(a.q + ((size_t)b * a.G + k) * a.V + first, n, e0, step, r.q);
#pragma unroll
    for (int i = 0; i < kQuads; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            r.p[i][j] = clamp_prob(r.p[i][j]);
            r.q[i][j] = kResid ? clamp_prob(r.q[i][j]) : 0.0f;
        }
}

template <bool kResid>
__device__ __forceinline__ Bins sum_rows(const Row &r) {
    Bins s = bins_zero();
#pragma unroll
    for (int i = 0; i < kQuads; i++)
        bins_add4<kResid>(s, r.p[i], r.q[i]);
    return s;
}

__device__ __forceinline__ void store_fx(uint64_t *p, Fx x) {
    p[0] = x.w0;
    p[1] = x.w1;
    p[2] = x.w2;
}
__device__ __forceinline__ Fx load_fx(const uint64_t *p) { return Fx{p[0], p[1], p[2]}; }

// Block sums j0 .. j0 + kPickChunk - 1 of a row (zero from `hi` on), every
// load issued before any is used.
constexpr int kPickChunk = 4096 / kBlk;
__device__ __forceinline__ void load_chunk(const uint64_t *bs, int j0, int hi, Fx v[kPickChunk]) {
#pragma unroll
    for (int c = 0; c < kPickChunk; c++) {
        const int j = j0 + c;
        v[c] = j < hi ? load_fx(bs + 3 * (size_t)j) : fx_zero();
    }
}

// One wavefront per (sequence, block): the block's exact sum of sampling
// weights.  If a rejection's leftover mass is zero in the whole row, the pick
// samples the target row, so a block without leftover mass stores the target
// row's sum as well (when the row has any leftover mass nobody reads it).
template <bool kResid>
__device__ __forceinline__ void block_sum(const AcceptParams &a, int b, int k, int blk, int lane) {
    Row r;
    load_rows<kResid, true>(a, b, k, blk, 4 * lane, 4 * kWave, r);
    const Fx s = bins_wave_sum(sum_rows<kResid>(r));
    uint64_t *dst = a.bsum + ((size_t)b * 2 * a.nblk + blk) * 3;
    if (lane == kWave - 1)
        store_fx(dst, s);
    if constexpr (kResid) {
        if (__ballot(fx_is_zero(s)) >> (kWave - 1)) {
            const Fx sp = bins_wave_sum(sum_rows<false>(r));
            if (lane == kWave - 1)
                store_fx(dst + (size_t)a.nblk * 3, sp);
        }
    }
}

__global__ __launch_bounds__(256) void accept_blocks_kernel(AcceptParams a) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave));
    const int lane = threadIdx.x % kWave;
    if (wave >= a.B * a.nblk)
        return;
    const int b = wave / a.nblk, blk = wave % a.nblk;
    const int gamma = clamp_gamma(a, b);
    const int k = __builtin_amdgcn_readfirstlane(accept_walk(a, b, gamma));
    if (blk == 0 && lane == 0)
        a.walk[b] = k;   // read by the pick kernel, so it need not walk again
    if (k < gamma)
        block_sum<true>(a, b, k, blk, lane);
    else
        block_sum<false>(a, b, k, blk, lane);
}

// One wavefront per sequence: the total, the target T = floor(u Z), the block
// whose cumulative mass first exceeds T, the lane's run of elements inside it
// and the element.  Since the cumulative weights are integers, C_v > u Z
// exactly when C_v > T, and u < 1 makes T < Z, so the element exists and
// carries weight.
__global__ __launch_bounds__(kPickThreads) void accept_pick_kernel(AcceptParams a) {
    const int b = blockIdx.x;
    const int lane = threadIdx.x;
    const int gamma = clamp_gamma(a, b);
    const float u = clamp_uniform(a.u_sample[b]);
    const int k = __builtin_amdgcn_readfirstlane(a.walk[b]);
    const bool rejected = k < gamma;
    const int per = (a.nblk + kWave - 1) / kWave;   // consecutive blocks per lane
    const int lo = min(lane * per, a.nblk), hi = min(lo + per, a.nblk);
    // with at most kPickChunk blocks per lane (vocabularies up to 262,144),
    // v keeps the lane's block sums for the owner's search below
    const bool one_chunk = per <= kPickChunk;

    int pass = 0;
    Fx run, incl, Z;
    Fx v[kPickChunk];
    const uint64_t *bs = nullptr;
    for (;; pass++) {
        bs = a.bsum + ((size_t)b * 2 + pass) * a.nblk * 3;
        run = fx_zero();
        for (int j0 = lo; j0 < hi; j0 += kPickChunk) {
            load_chunk(bs, j0, hi, v);
#pragma unroll
            for (int c = 0; c < kPickChunk; c++)
                run = fx_add(run, v[c]);
        }
        incl = fx_incl_scan(run);
        Z = fx_shfl(incl, kWave - 1);
        // leftover mass zero: sample p_k itself (its sums are in pass 1)
        if (pass == 0 && rejected && fx_is_zero(Z))
            continue;
        break;
    }
    if (fx_is_zero(Z)) {
        if (lane == 0) {
            a.n_accepted[b] = k;
            a.next_token[b] = -1;   // a sampling row with no mass
        }
        return;
    }
    const Fx T = fx_floor_mul(Z, u);

    // the first lane whose run ends above T owns the block
    const unsigned long long own = __ballot(fx_gt(incl, T));
    const int owner = __ffsll((long long)own) - 1;   // exists: incl of lane 63 = Z > T
    int blk = 0;
    Fx base = fx_zero();
    if (lane == owner) {
        Fx acc = fx_sub(incl, run);   // mass before this lane's run (incl >= run)
        bool found = false;
        for (int j0 = lo; j0 < hi && !found; j0 += kPickChunk) {
            if (!one_chunk)
                load_chunk(bs, j0, hi, v);
#pragma unroll
            for (int c = 0; c < kPickChunk; c++) {
                const Fx next = fx_add(acc, v[c]);
                if (!found && fx_gt(next, T)) {   // blocks past hi add zero
                    blk = j0 + c;
                    found = true;
                }
                if (!found)
                    acc = next;
            }
        }
        base = acc;
    }
    blk = __builtin_amdgcn_readfirstlane(__shfl(blk, owner, kWave));
    base = fx_shfl(base, owner);

    // the lane inside that block: each lane sums its run of 4 * kQuads elements
    Row r;
    Fx lane_sum;
    if (rejected && pass == 0) {
        load_rows<true, false>(a, b, k, blk, 4 * kQuads * lane, 4, r);
        lane_sum = fx_of_bins(sum_rows<true>(r));
    } else {
        load_rows<false, false>(a, b, k, blk, 4 * kQuads * lane, 4, r);
        lane_sum = fx_of_bins(sum_rows<false>(r));
    }
    const Fx lincl = fx_add(base, fx_incl_scan(lane_sum));
    const unsigned long long hit = __ballot(fx_gt(lincl, T));
    const int first = __ffsll((long long)hit) - 1;   // exists: the block's total exceeds T
    const Fx before = fx_shfl(fx_sub(lincl, lane_sum), first);

    // the element inside that run: lane m takes element m of it
    float pm = 0.0f, qm = 0.0f;
#pragma unroll
    for (int m = 0; m < 4 * kQuads; m++) {
        const float pf = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(r.p[m / 4][m % 4]), first));
        const float qf = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(r.q[m / 4][m % 4]), first));
        pm = lane == m ? pf : pm;
        qm = lane == m ? qf : qm;
    }
    const Fx w = pm > qm ? fx_sub(fx_of_prob(pm), fx_of_prob(qm)) : fx_zero();
    const Fx eincl = fx_add(before, fx_incl_scan(w));
    const unsigned long long at = __ballot(fx_gt(eincl, T));
    if (lane == 0) {
        a.n_accepted[b] = k;
        a.next_token[b] = blk * kBlk + 4 * kQuads * first + __ffsll((long long)at) - 1;
    }
}

}  // namespace

// Workspace of the acceptance: the block sums, then (256-byte aligned) the
// per-sequence walk results.  It holds two sums for every 256 elements; the
// kernels use that for blocks of kBlk.
static_assert(kBlk >= kWsBlk, "the block sums must fit the workspace");
static size_t walk_offset(size_t num_seqs, size_t nblk) {
    return (num_seqs * 2 * nblk * 3 * sizeof(uint64_t) + 255) & ~(size_t)255;
}

}  // namespace tsattn

using namespace tsattn;

extern "C" {

int ts_kv_append(const ts_attn_shape *s, const void *k_new, const void *v_new, void *k_pages, void *v_pages,
                 const int32_t *page_table, const int32_t *ctx_lens, const int32_t *q_lens, void *stream) {
    clear_error();
    if (!s)
        return fail(TS_ERR_NULL, "shape is NULL");
    if (!k_new || !v_new || !k_pages || !v_pages || !page_table || !ctx_lens || !q_lens)
        return fail(TS_ERR_NULL, "a pointer is NULL");
    if (s->num_seqs < 1 || s->num_kv_heads < 1 || s->max_q_len < 1 || s->max_pages_per_seq < 1 ||
        s->num_pages < 1 || s->page_size != 16 || (s->head_dim != 64 && s->head_dim != 128))
        return fail(TS_ERR_SHAPE, "unsupported shape for the KV append");
    if (((uintptr_t)k_new | (uintptr_t)v_new | (uintptr_t)k_pages | (uintptr_t)v_pages) & 15)
        return fail(TS_ERR_ARG, "misaligned pointer (16 B needed)");
    int st = check_device();
    if (st)
        return st;
    AppendParams p;
    p.k_new = static_cast<const uint16_t *>(k_new);
    p.v_new = static_cast<const uint16_t *>(v_new);
    p.k_pages = static_cast<uint16_t *>(k_pages);
    p.v_pages = static_cast<uint16_t *>(v_pages);
    p.page_table = page_table;
    p.ctx_lens = ctx_lens;
    p.q_lens = q_lens;
    p.num_pages = s->num_pages;
    p.B = s->num_seqs;
    p.Qmax = s->max_q_len;
    p.Hkv = s->num_kv_heads;
    p.D = s->head_dim;
    p.max_pages = s->max_pages_per_seq;
    const int64_t total = (int64_t)p.B * p.Qmax * p.Hkv * (p.D / 8);
    if ((total + 255) / 256 > INT32_MAX)
        return fail(TS_ERR_SHAPE, "KV append of %lld rows is too large for one launch",
                    (long long)((int64_t)p.B * p.Qmax * p.Hkv));
    const unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(kv_append_kernel, dim3(blocks), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), p);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? TS_OK : hip_fail(e, "KV append launch");
}

size_t ts_spec_accept_workspace_size(int32_t num_seqs, int32_t vocab) {
    clear_error();
    if (num_seqs < 1 || vocab < 1) {
        fail(TS_ERR_ARG, "num_seqs and vocab must be positive");
        return 0;
    }
    const size_t nblk = ((size_t)vocab + kWsBlk - 1) / kWsBlk;
    return walk_offset(num_seqs, nblk) + (((size_t)num_seqs * sizeof(int32_t) + 255) & ~(size_t)255);
}

int ts_spec_accept(int32_t num_seqs, int32_t vocab, int32_t max_draft, const float *p_target,
                   const float *q_draft, const int32_t *draft_tokens, const int32_t *num_draft,
                   const float *u_accept, const float *u_sample, int32_t *num_accepted, int32_t *next_token,
                   void *workspace, size_t workspace_bytes, void *stream) {
    clear_error();
    if (num_seqs < 1 || vocab < 1 || max_draft < 0)
        return fail(TS_ERR_ARG, "num_seqs, vocab must be positive and max_draft >= 0");
    if (!p_target || !num_draft || !u_sample || !num_accepted || !next_token || !workspace ||
        (max_draft > 0 && (!q_draft || !draft_tokens || !u_accept)))
        return fail(TS_ERR_NULL, "a pointer is NULL");
    const size_t need = ts_spec_accept_workspace_size(num_seqs, vocab);
    if (workspace_bytes < need)
        return fail(TS_ERR_WORKSPACE, "workspace has %zu bytes, needs %zu", workspace_bytes, need);
    if ((((uintptr_t)p_target | (uintptr_t)q_draft) & 15) || ((uintptr_t)workspace & 255))
        return fail(TS_ERR_ARG, "misaligned pointer (probabilities 16 B, workspace 256 B)");
    int st = check_device();
    if (st)
        return st;
    AcceptParams a;
    a.p = p_target;
    a.q = q_draft;
    a.draft = draft_tokens;
    a.num_draft = num_draft;
    a.u_accept = u_accept;
    a.u_sample = u_sample;
    a.n_accepted = num_accepted;
    a.next_token = next_token;
    a.bsum = static_cast<uint64_t *>(workspace);
    a.walk = reinterpret_cast<int32_t *>(static_cast<char *>(workspace) +
                                         walk_offset(num_seqs, ((size_t)vocab + kWsBlk - 1) / kWsBlk));
    a.B = num_seqs;
    a.V = vocab;
    a.G = max_draft;
    a.nblk = (int)(((int64_t)vocab + kBlk - 1) / kBlk);
    hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
    const int64_t waves = (int64_t)a.B * a.nblk;
    if (((int64_t)a.B * (((int64_t)vocab + kWsBlk - 1) / kWsBlk) + 3) / 4 > INT32_MAX)
        return fail(TS_ERR_ARG, "num_seqs x vocab is too large for one launch");
    const unsigned blocks = (unsigned)((waves + 3) / 4);
    hipLaunchKernelGGL(accept_blocks_kernel, dim3(blocks), dim3(256), 0, hs, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "acceptance block-sum launch");
    hipLaunchKernelGGL(accept_pick_kernel, dim3(a.B), dim3(kPickThreads), 0, hs, a);
    e = hipGetLastError();
    return e == hipSuccess ? TS_OK : hip_fail(e, "acceptance pick launch");
}

}  // extern "C"
