// Device code of the MoE dispatch / combine path for gfx950 (wave64).
//
// The path itself (route, plan, pack, regather, combine and the mirrored return path)
// is bandwidth or latency bound: no dense contraction, so no MFMA.  The row movers
// move rows of 16-byte vectors straight through registers with several loads in
// flight per lane; the planning kernels are integer work on wavefront bit masks.
// The two optional stages around it, the gate projection and the expert layer, are
// dense contractions and run on the matrix cores; they follow further down.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace monta {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kWave = 64;
// Chosen by measurement on MI355X (128 and 512 threads, 2 and 8 vectors in flight were slower or equal).
constexpr int kMoverThreads = 256;   // threads per workgroup of the row movers
constexpr int kVecInFlight = 4;      // 16-byte loads issued by a lane before its first store

// meta[] slots (int32)
enum { META_R = 0, META_ALIVE = 1, META_C = 2, META_FINAL_ROWS = 4, META_SLOTS = 16 };

struct PlanPtrs {
    int32_t *meta, *counts, *kept, *offsets, *n, *stage_off, *unit_base, *send_rows, *unit_rows;
    int32_t *pos_final, *pos_stage, *row_map, *block_counts, *block_base, *local_rank, *kept_prefix;
};

// n / d for 0 <= n < 2^16 and d < 2^15, by a multiplication: an integer division takes about 40 instructions
struct FastDiv {
    uint32_t d, m;
};
inline FastDiv fast_div(int d) { return {(uint32_t)d, d > 1 ? (uint32_t)((1ull << 32) / (uint32_t)d + 1) : 0u}; }
__device__ __forceinline__ int operator/(int n, FastDiv f) { return f.m ? (int)__umulhi((uint32_t)n, f.m) : n; }

struct Shape {
    int32_t T, E, k, ep, tp, S, U, Tu;
    int32_t TB;        // tokens per route workgroup
    int32_t bpu;       // route workgroups per unit
    int32_t num_blocks;
    int32_t C;         // per-expert capacity
    int32_t renorm;
    int32_t vpr;       // 16-byte vectors per activation row
    int32_t lpr;       // lanes cooperating on one row in the movers (power of two <= kMoverThreads)
    int32_t max_rows;  // rows STAGE / FINAL hold; every row index read from a table is checked against it
    int32_t cache;     // CachePolicy bits: which streams of the movers use non-temporal accesses
    int32_t padded;    // 1: FINAL is [E][C][H] (expert e at row e*C), 0: compact
    int32_t lazy;      // 1: the single pass requests a token's row only when it knows that one of its choices is kept
    int32_t rl;        // lanes that share one token in the route kernel (1, 2, 4 or 8)
    FastDiv by_E, by_k, by_k1, by_Tu, by_ep;       // for the pairs of a route workgroup (by_k1: k - 1) and for small problems
    int32_t fast_plan; // 1: every workgroup reduces the histogram table; 0: block_scan_kernel scans it first
};

// A set bit makes that stream non-temporal (streaming, no reuse expected); a clear bit leaves
// it cacheable, which pays when the consumer kernel finds the data still in the memory-side cache.
enum CachePolicy {
    NT_PACK_LD = 1, NT_PACK_ST = 2, NT_REG_LD = 4, NT_REG_ST = 8, NT_COMB_LD = 16, NT_COMB_ST = 32
};

// ------------------------------------------------------------------ helpers

// Inclusive sum over the wave by DPP moves: shifts inside the rows of 16 lanes, then the rows' totals.  All 64 lanes take part.
// (Six shuffles through the LDS instead took about 600 clocks, and a plan needs several scans in a row.)
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);        // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);        // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);        // row_bcast:31 into rows 2 and 3
    return v;
}
// the sum over the wave, from its inclusive scan
__device__ __forceinline__ int wave_total(int scan) { return __builtin_amdgcn_readlane(scan, kWave - 1); }
template <typename T> int wave_inclusive_scan(T) = delete;        // wider values do not fit the 32-bit moves
template <typename T> T wave_total(T) = delete;

template <bool NT>
__device__ __forceinline__ u32x4 ld16(const u32x4 *p)
{
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NT>
__device__ __forceinline__ void st16(u32x4 *p, u32x4 v)
{
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Calls f(integral_constant<bool, load_nt>, integral_constant<bool, store_nt>) for the two policy bits:
// the four variants stay separate loops, so the compiler cannot fold the access kinds together.
template <typename F>
__device__ __forceinline__ void with_policy(bool ntl, bool nts, F f)
{
    if (ntl) {
        if (nts) f(std::true_type{}, std::true_type{});
        else f(std::true_type{}, std::false_type{});
    } else {
        if (nts) f(std::false_type{}, std::true_type{});
        else f(std::false_type{}, std::false_type{});
    }
}

// The same for the three streams of the single-pass dispatch.
template <typename F>
__device__ __forceinline__ void with_policy3(bool ntl, bool nts, bool ntf, F f)
{
    with_policy(ntl, nts, [&](auto l, auto st) {
        if (ntf) f(l, st, std::true_type{});
        else f(l, st, std::false_type{});
    });
}

// ------------------------------------------------------------ route + plan

// One workgroup routes TB consecutive tokens of ONE unit; s.rl lanes share a token (1 for few experts).
//  1. lane `sub` of a token's L lanes keeps its logits in registers, every L-th four of them, as unsigned keys of
//     the same order; the loads of a wave cover whole lines and nothing goes through the LDS;
//  2. k selections per token, ties to the lower index (route_select);
//  3. gates in fp64 from the winners' logits, one rounding to fp32;
//  4. every selection ORs its token's bit into mask[expert][wave] in LDS; popcounts of those masks give the workgroup's expert
//     histogram and each pair's stable rank inside the workgroup (bit order is token order).
// No atomics decide a position: the result is deterministic.
//
// The lanes of a token (L of them, s.rl = 1, 2, 4 or 8, for small problems up to 16, neighbours in the wave) agree through DPP moves:
// quads by permutation, the two quads of eight lanes by the half-row mirror, the two eights by the row mirror, whose lanes hold
// the same value by then.
template <int MASK>
__device__ __forceinline__ int xor_lanes(int v)
{
    static_assert(MASK == 1 || MASK == 2 || MASK == 4 || MASK == 8, "xor_lanes: lanes of one token");
    constexpr int kCtrl = MASK == 1 ? 0xb1 : MASK == 2 ? 0x4e : MASK == 4 ? 0x141 : 0x140;
    return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xf, 0xf, false);
}
// combine(xor_lanes<1>), then <2> and so on, over the L lanes of a token
template <int L, typename F>
__device__ __forceinline__ void over_token_lanes(F combine)
{
    if constexpr (L > 1) combine(std::integral_constant<int, 1>{});
    if constexpr (L > 2) combine(std::integral_constant<int, 2>{});
    if constexpr (L > 4) combine(std::integral_constant<int, 4>{});
    if constexpr (L > 8) combine(std::integral_constant<int, 8>{});
}

__device__ __forceinline__ void keep_larger_first(uint32_t &a, uint32_t &b)
{
    const uint32_t hi = max(a, b), lo = min(a, b);
    a = hi;
    b = lo;
}
// 4 or 8 keys in descending order (5 and 19 exchanges)
template <int K>
__device__ __forceinline__ void sort_keys(uint32_t *v)
{
    static_assert(K == 4 || K == 8, "sort_keys: lists of 4 or 8");
    auto cx = [&](int a, int b) { keep_larger_first(v[a], v[b]); };
    if constexpr (K == 4) {
        cx(0, 1), cx(2, 3), cx(0, 2), cx(1, 3), cx(1, 2);
    } else {
        cx(0, 1), cx(2, 3), cx(4, 5), cx(6, 7), cx(0, 2), cx(1, 3), cx(4, 6), cx(5, 7), cx(1, 2), cx(5, 6);
        cx(0, 4), cx(1, 5), cx(2, 6), cx(3, 7), cx(2, 4), cx(3, 5), cx(1, 2), cx(3, 4), cx(5, 6);
    }
}
// a: the K largest of two descending lists of K, in descending order; other(i) is element i of the second
template <int K, typename F>
__device__ __forceinline__ void merge_keys(uint32_t *a, F other)
{
    uint32_t b[K];
#pragma unroll
    for (int i = 0; i < K; ++i) b[i] = other(K - 1 - i);
#pragma unroll
    for (int i = 0; i < K; ++i) a[i] = max(a[i], b[i]);          // larger half, bitonic
#pragma unroll
    for (int d = K / 2; d >= 1; d /= 2)
#pragma unroll
        for (int i = 0; i < K; ++i)
            if ((i & d) == 0) keep_larger_first(a[i], a[i + d]);
}
// the K largest of a token's keys (NE in each of its L lanes), in descending order, in every lane of the token
template <int K, int L, int NE>
__device__ __forceinline__ void largest_keys(const uint32_t (&key)[NE], uint32_t (&top)[K])
{
#pragma unroll
    for (int i = 0; i < K; ++i) top[i] = key[i];
    sort_keys<K>(top);
#pragma unroll
    for (int q = K; q < NE; q += K) {
        uint32_t next[K];
#pragma unroll
        for (int i = 0; i < K; ++i) next[i] = key[q + i];
        sort_keys<K>(next);
        merge_keys<K>(top, [&](int i) { return next[i]; });
    }
    over_token_lanes<L>([&](auto mask) {
        uint32_t mine[K];
#pragma unroll
        for (int i = 0; i < K; ++i) mine[i] = top[i];
        merge_keys<K>(top, [&](int i) { return (uint32_t)xor_lanes<decltype(mask)::value>((int)mine[i]); });
    });
}

// key[q] by the bits of q: registers have no address
template <int N>
__device__ __forceinline__ uint32_t pick_key(const uint32_t (&key)[N], int q)
{
    if constexpr (N == 1) {
        return key[0];
    } else {
        uint32_t half[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const uint32_t even = key[2 * i], odd = key[2 * i + 1];     // values: a choice of places would be an address
            half[i] = q & 1 ? odd : even;
        }
        return pick_key<N / 2>(half, q >> 1);
    }
}

// Steps 1, 2 and the masks of 4: the choices of `nt` tokens whose logits start at src.  Choice j of token tok and its logit go to
// s_sel and s_top[tok * k + j]; bit tok % 64 of s_mask[e * expert_step + tok / 64 * word_step] (cleared by the caller) is
// set where token tok chose e.  s_den: sums of all exponentials, if it is not null.  All threads of the workgroup; ends without a
// barrier.  Nothing goes to memory here: choices and gates may be stored in the logits' own memory, and until the caller's barrier
// waves still read theirs, those of the sums a second time.
// Up to two choices, or more than eight, are found one after the other: the largest key of the token, its lowest place, and that key is
// cleared, about 4.5 instructions per key and choice.  Three to eight: the largest keys in order, from sorting networks over the
// lane's keys and then over the token's lanes, about 11 instructions per key for eight; then each lane looks up the few of its keys
// that are among them, and the number of larger ones is their place.  Equal keys among the chosen ones (seen by that some place would
// be taken twice, or too many keys qualify) are dealt with choice by choice, for the whole wave.
// What bounds it is instructions.  Measured on MI355X, routing and plan, logits through the LDS and choice after choice, now: 32768 tokens,
// 256 experts, top-8 35.7 -> 28.1 us (the kernel 22.3 -> 14.6), with logits of 8 bits, full of ties, 36.6 -> 32.7, all equal 30.1 -> 26.8;
// 65536 tokens, 64 experts, top-8 28.0 -> 23.9; 16384 tokens, 255 experts, top-2, renorm = 0 25.6 -> 23.9.
template <int L, int NE>
__device__ __forceinline__ void route_select(const float *__restrict__ src, int nt, int E, int k, int *s_sel, float *s_top,
                                             unsigned long long *s_mask, int expert_step, int word_step, double *s_den)
{
    static_assert(NE == 8 || NE == 16 || NE == 32, "route_select: keys of a lane");
    constexpr int kShift = L == 1 ? 2 : L == 2 ? 3 : L == 4 ? 4 : L == 8 ? 5 : 6;         // experts of all lanes' fours: 1 << kShift
    const int tid = threadIdx.x, tok = tid / L, sub = tid % L;      // token handled by this lane, and which of its L lanes it is
    const unsigned long long tbit = 1ull << (tok & 63);
    unsigned long long *const mask = s_mask + (tok >> 6) * word_step;
    int *const sel = s_sel + tok * k;
    float *const top_logit = s_top + tok * k;
    auto expert = [&](int q) { return ((q >> 2) << kShift) + sub * 4 + (q & 3); };        // of the lane's key q
    const int rest = E - sub * 4;
    auto exists = [&](int q) { return ((q >> 2) << kShift) + (q & 3) < rest; };           // (a constant against one register)

    // A lane's four logits from key q on are one load, which on this hardware has to be aligned to its elements only.  Where rows are not
    // whole fours, one that reaches past the row's end is read from the row's last four and shifted.  What no expert has is never
    // looked at.  Offsets of 32 bits from the workgroup's first logit (at most 1024 tokens of 256): one register per load on its way.
    const uint32_t row = tok < nt ? (uint32_t)(tok * E) : 0u;
    auto at = [&](int e) { return reinterpret_cast<const unsigned char *>(src) + (size_t)((row + (uint32_t)e) * 4u); };
    auto last_four = [&](int q) { return min(expert(q), E - 4); };
    auto load_four = [&](int q) { return *reinterpret_cast<const f32x4_any *>(at(last_four(q))); };
    auto shifted = [&](int q, f32x4 x) {
        const int past = expert(q) - last_four(q);
        const float y0 = past & 1 ? x[1] : x[0], y1 = past & 1 ? x[2] : x[1], y2 = past & 1 ? x[3] : x[2];
        return f32x4{past & 2 ? y2 : y0, past & 2 ? x[3] : y1, y2, x[3]};
    };
    auto load_few = [&](int i) { return *reinterpret_cast<const float *>(at(min(expert(i), E - 1))); };        // fewer than four experts
    float v[NE];
    if (E >= 4) {
        f32x4 x[NE / 4];
#pragma unroll
        for (int q = 0; q < NE; q += 4) x[q / 4] = load_four(q);
        if (E & 3) {
#pragma unroll
            for (int q = 0; q < NE; q += 4) x[q / 4] = shifted(q, x[q / 4]);
        }
#pragma unroll
        for (int q = 0; q < NE; ++q) v[q] = x[q / 4][q % 4];
    } else {
#pragma unroll
        for (int q = 0; q < NE; ++q) v[q] = q < 4 ? load_few(q) : 0.f;
    }
    __syncthreads();                                                // the masks are cleared
    if (tok >= nt) return;
    // Unsigned keys of the same order (zeros of both signs alike, NaN as -infinity); 0: taken, or no element.
    uint32_t key[NE];
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const uint32_t u = __float_as_uint((v[q] != v[q] ? -INFINITY : v[q]) + 0.f);
        key[q] = exists(q) ? u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u) : 0u;
    }
    auto pick = [&](int q) { return pick_key<NE>(key, q); };
    auto logit = [](uint32_t x) { return __uint_as_float(x & 0x80000000u ? x ^ 0x80000000u : ~x); };
    // called by one lane per choice
    auto choose = [&](int j, int e, uint32_t x) {
        sel[j] = e;
        top_logit[j] = logit(x);
        atomicOr(&mask[e * expert_step], tbit);
    };
    auto largest = [&] {                                            // of the token
        uint32_t most = key[0];
#pragma unroll
        for (int q = 1; q < NE; ++q) most = max(most, key[q]);
        over_token_lanes<L>([&](auto m) { most = max(most, (uint32_t)xor_lanes<decltype(m)::value>((int)most)); });
        return most;
    };
    if (s_den) {
        // softmax over all E: the token's lanes each sum their experts, read again four at a time, then add up across the lanes
        const double first = (double)logit(largest());
        double part = 0.0;
        auto add = [&](int q, f32x4 x) {
#pragma unroll
            for (int i = 0; i < 4; ++i) part += exp((double)(exists(q + i) && x[i] == x[i] ? x[i] : -INFINITY) - first);
        };
        if (E >= 4) {
            f32x4 next = load_four(0);
#pragma unroll 1
            for (int q = 0; q < NE && exists(q); q += 4) {
                const f32x4 x = E & 3 ? shifted(q, next) : next;
                next = load_four(q + 4);
                add(q, x);
            }
        } else {
            add(0, f32x4{load_few(0), load_few(1), load_few(2), load_few(3)});
        }
        for (int mk = 1; mk < L; mk <<= 1) part += __shfl_xor(part, mk, kWave);
        if (sub == 0) s_den[tok] = part;
    }
    auto lowest = [&](int at) {                                     // of the token's lanes' places; E only if k > E, then any in range
        over_token_lanes<L>([&](auto m) { at = min(at, xor_lanes<decltype(m)::value>(at)); });
        return min(at, E - 1);
    };
    auto one_by_one = [&] {
        for (int j = 0; j < k; ++j) {
            const uint32_t most = largest();
            int at = -1;
#pragma unroll
            for (int q = NE - 1; q >= 0; --q) at = key[q] == most ? q : at;
            const int best = lowest(at >= 0 ? expert(at) : E);
            const int mine = ((best >> 2) & (L - 1)) == sub ? ((best >> kShift) << 2) + (best & 3) : -1;
#pragma unroll
            for (int q = 0; q < NE; ++q) key[q] = mine == q ? 0u : key[q];
            if (sub == 0) choose(j, best, most);
        }
    };
    auto by_networks = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        uint32_t top[K];
        largest_keys<K, L, NE>(key, top);
        uint32_t least = top[0];                                    // the smallest that is chosen
        bool equal = false;
#pragma unroll
        for (int j = 1; j < K; ++j)
            if (j < k) {
                least = top[j];
                equal |= top[j] == top[j - 1];
            }
        uint32_t chosen = 0;                                        // bit q: key q is among them
#pragma unroll
        for (int q = NE - 1; q >= 0; --q) chosen = chosen + chosen + (key[q] >= least ? 1u : 0u);
        int count = __popc(chosen);
        over_token_lanes<L>([&](auto m) { count += xor_lanes<decltype(m)::value>(count); });
        if (__any(equal || count != k)) {
            int at = 0;
            uint32_t last = 0;
#pragma unroll 1
            for (int j = 0; j < k; ++j) {
                uint32_t want = top[0], same = 0;
#pragma unroll
                for (int i = 1; i < K; ++i) want = j == i ? top[i] : want;
#pragma unroll
                for (int q = NE - 1; q >= 0; --q) same = same + same + (key[q] == want ? 1u : 0u);
                if (want == last) {                                 // past the place of the one before
                    const int four = (at >> kShift) << 2, its_sub = (at >> 2) & (L - 1);
                    const int from = four + (sub < its_sub ? 4 : sub == its_sub ? (at & 3) + 1 : 0);
                    same = from < 32 ? same & (~0u << from) : 0u;
                }
                at = lowest(same ? expert(__builtin_ctz(same)) : E);
                last = want;
                if (sub == 0) choose(j, at, want);
            }
            return;
        }
        // Neighbouring tokens begin at different keys: all lanes at the same one would queue for one mask (496 tokens on 8 experts, top-8 12.8 us,
        // now 10.5).
        const int turn = tok & (NE - 1);
        if constexpr (NE == 32) chosen = __builtin_rotateright32(chosen, turn);
        else chosen = (chosen | chosen << NE) >> turn & ((1u << NE) - 1u);
        while (chosen) {
            const int q = (__builtin_ctz(chosen) + turn) & (NE - 1);
            chosen &= chosen - 1;
            const uint32_t x = pick(q);
            int j = 0;
#pragma unroll
            for (int i = 0; i < K; ++i) j += top[i] > x ? 1 : 0;
            choose(j, expert(q), x);
        }
    };
    if (k <= 2 || k > 8) one_by_one();
    else if (k <= 4) by_networks(std::integral_constant<int, 4>{});
    else by_networks(std::integral_constant<int, 8>{});
}

// Step 3 for tokens [0, nt), by threads tid of nthr, in two parts with a barrier between: w_j = exp(l_j - l_0) in fp64 (w_0 = 1
// needs no call), one (token, choice) pair per lane so that every lane has an exp to do, not only one per token; then the
// denominator, summed in j order (or taken from s_den, the sums over all experts, if that is not null), one division, one rounding
// to fp32: store(pair, gate).
__device__ __forceinline__ void route_weights(int nt, int k, const float *s_top, double *s_w, FastDiv by_k1, int tid, int nthr)
{
    for (int tk = tid; tk < nt; tk += nthr) s_w[tk * k] = 1.0;
    for (int idx = tid; idx < nt * (k - 1); idx += nthr) {               // only the choices j >= 1 need an exp
        const int tk = idx / by_k1, j = 1 + idx - tk * (k - 1);
        s_w[tk * k + j] = exp((double)s_top[tk * k + j] - (double)s_top[tk * k]);
    }
}
template <typename F>
__device__ __forceinline__ void route_gates(int nt, int k, const double *s_w, const double *s_den, FastDiv by_k, int tid, int nthr, F store)
{
    for (int idx = tid; idx < nt * k; idx += nthr) {
        const int tk = idx / by_k;
        double denom = 0.0;
        if (!s_den) {
            const double *wt = s_w + tk * k;
            for (int j = 0; j < k; ++j) denom += wt[j];
        } else {
            denom = s_den[tk];
        }
        store(idx, (float)(s_w[idx] / denom));
    }
}

// Dynamic LDS of route_plan_kernel (byte offsets): [TB][k] choices, their logits, bit masks [E][words of 64 tokens], [TB][k] weights,
// [TB] softmax denominators (renorm = 0).
struct RouteLds {
    int top, mask, w, den, bytes;
};
__host__ __device__ inline RouteLds route_lds(int TB, int E, int k)
{
    const int NW = TB > kWave ? TB / kWave : 1;
    RouteLds l;
    l.top = TB * k * 4;
    l.mask = (l.top + TB * k * 4 + 7) & ~7;
    l.w = l.mask + E * NW * 8;
    l.den = l.w + TB * k * 8;
    l.bytes = l.den + TB * 8;
    return l;
}

template <int L, int NE>
__global__ __launch_bounds__(1024) void route_plan_kernel(const float *__restrict__ logits,
                                                         int32_t *__restrict__ topk_idx,
                                                         float *__restrict__ gates, PlanPtrs p, Shape s)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int E = s.E, k = s.k, TB = s.TB;
    const int NW = TB > kWave ? TB / kWave : 1;
    const RouteLds lds = route_lds(TB, E, k);
    int *s_sel = reinterpret_cast<int *>(smem);
    float *s_top = reinterpret_cast<float *>(smem + lds.top);
    unsigned long long *s_mask = reinterpret_cast<unsigned long long *>(smem + lds.mask);
    double *s_w = reinterpret_cast<double *>(smem + lds.w), *s_den = reinterpret_cast<double *>(smem + lds.den);

    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    const int u = b / s.bpu, ib = b - u * s.bpu;
    const int t_begin = u * s.Tu + ib * TB;
    int nt = s.Tu - ib * TB;
    if (nt > TB) nt = TB;

    for (int i = tid; i < E * NW; i += blockDim.x) s_mask[i] = 0ull;
    route_select<L, NE>(logits + (size_t)t_begin * E, nt, E, k, s_sel, s_top, s_mask, NW, 1, s.renorm ? nullptr : s_den);
    __syncthreads();                                               // no logit is read any more: their memory may be stored to
    route_weights(nt, k, s_top, s_w, s.by_k1, tid, blockDim.x);
    __syncthreads();
    route_gates(nt, k, s_w, s.renorm ? nullptr : s_den, s.by_k, tid, blockDim.x,
                [&](int idx, float g) { gates[(size_t)t_begin * k + idx] = g; });
    const int npairs = nt * k;

    for (int e = tid; e < E; e += blockDim.x) {
        int c = 0;
        for (int w = 0; w < NW; ++w) c += __popcll(s_mask[e * NW + w]);
        p.block_counts[(size_t)b * E + e] = c;
    }
    for (int idx = tid; idx < npairs; idx += blockDim.x) {      // one pair per lane again
        const int tk = idx / s.by_k;
        const int e = s_sel[idx];
        topk_idx[(size_t)t_begin * k + idx] = e;
        const int word = tk >> 6;
        int r = 0;
        for (int w = 0; w < word; ++w) r += __popcll(s_mask[e * NW + w]);
        r += __popcll(s_mask[e * NW + word] & ((1ull << (tk & 63)) - 1ull));
        p.local_rank[(size_t)t_begin * k + idx] = r;    // rank inside the workgroup; the positions kernels finish it
    }

    if (b == 0 && tid == 0) p.meta[META_ALIVE] = s.T;  // the kernel that finishes the positions takes the tokens without a kept pair off
}

// Exclusive scans of the route workgroups' histograms, per expert, in workgroup (= token) order, for tables that are too
// large for every workgroup of the next kernel to reduce: block_base[b][e] = pairs of e in workgroups before b, and
// counts[e].  A chain of latencies (the table sits in the L2), so a workgroup takes only 16 experts, half a line of a row, and 64
// runs of rows at a time, one (expert, run) per thread: up to 1024 rows are one batch of loads, kept for the second walk, and
// the 64 runs of an expert are one scan over a wave.  A table of 512 x 256 takes 4.3 us; 64 experts a workgroup, 16 runs walked
// twice took 7.4 us, a scan by the last route workgroup to finish, expert by expert, 270.
constexpr int kScanExperts = 16;
__global__ __launch_bounds__(kScanExperts * kWave) void block_scan_kernel(PlanPtrs p, Shape s)
{
    constexpr int LD = 16;
    __shared__ int s_sum[kScanExperts][kWave + 1];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int col = threadIdx.x % kScanExperts, part = threadIdx.x / kScanExperts;
    const int E = s.E, nb = s.num_blocks, e0 = blockIdx.x * kScanExperts, e = e0 + col;
    const bool on = e < E;
    const int run = (nb + kWave - 1) / kWave;
    const int lo = min(part * run, nb), hi = min(lo + run, nb);
    auto load = [&](int b0, int (&c)[LD]) {
#pragma unroll
        for (int q = 0; q < LD; ++q) c[q] = on && b0 + q < hi ? p.block_counts[(size_t)(b0 + q) * E + e] : 0;
    };
    int first[LD], sum = 0;
    load(lo, first);
#pragma unroll
    for (int q = 0; q < LD; ++q) sum += first[q];
    for (int b0 = lo + LD; b0 < hi; b0 += LD) {
        int c[LD];
        load(b0, c);
#pragma unroll
        for (int q = 0; q < LD; ++q) sum += c[q];
    }
    s_sum[col][part] = sum;
    __syncthreads();
    const int mine = s_sum[wave][lane], incl = wave_inclusive_scan(mine);       // a wave scans the runs of one expert
    s_sum[wave][lane] = incl - mine;
    if (lane == kWave - 1 && e0 + wave < E) p.counts[e0 + wave] = incl;
    __syncthreads();
    int before = s_sum[col][part];
    auto store = [&](int b0, const int (&c)[LD]) {
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            if (on && b0 + q < hi) p.block_base[(size_t)(b0 + q) * E + e] = before;
            before += c[q];
        }
    };
    store(lo, first);
    for (int b0 = lo + LD; b0 < hi; b0 += LD) {
        int c[LD];
        load(b0, c);
        store(b0, c);
    }
}

// Shared-memory result of rebuilding the scans for one route workgroup b (see block_plan).
struct BlockPlan {
    int before[256];   // P[u][e]: pairs of expert e in units before b's unit
    int unit[256];     // pairs of e in b's unit
    int pre[256];      // pairs of e in b's unit, in workgroups before b
    int total[256];    // counts[e]
    int off[256];      // offsets[e]: first FINAL row of expert e
    int kpre[256];     // exclusive scan of the kept counts (= off when the layout is compact)
    int stage[256];    // stage_off[u][e]: first STAGE row of block (u, e)
    int alive[256];    // per token of the workgroup: has a kept pair (plan_positions_block)
    int sums[256 / kWave][3];      // of each wave's experts: kept counts, the unit's rows, the rows of the units before
    int R, unit_row0;
};
static_assert(kMoverThreads == 256, "block_plan: four waves scan 256 experts");

// One lane's share of the histogram-table reduction of block_plan: the counters of expert e in blocks bl, bl + bstep,
// ..., LD loads requested before any is added up.
struct BlockSums {
    int total, before, unit, pre;
};
template <int LD>
__device__ __forceinline__ BlockSums sum_blocks(const int32_t *__restrict__ block_counts, int E, int e, int bl, int bstep,
                                                int nblk, int b, int first, int last)
{
    BlockSums a = {0, 0, 0, 0};
    for (int bb0 = bl; bb0 < nblk; bb0 += bstep * LD) {
        int cnt[LD];
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            const int bb = bb0 + q * bstep;
            cnt[q] = bb < nblk ? block_counts[(size_t)bb * E + e] : 0;
        }
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            const int bb = bb0 + q * bstep;
            const int c = cnt[q];
            a.total += c;
            if (bb < first) a.before += c;
            else if (bb < last) {
                a.unit += c;
                if (bb < b) a.pre += c;
            }
        }
    }
    return a;
}

// With a small table every workgroup that calls this re-reads the whole [num_blocks][E] histogram table (a few KiB,
// L2 resident) and reduces it to four sums per expert; with a large one (s.fast_plan = 0) block_scan_kernel has left the
// scans, and the sums are four rows of them.  Two wave scans over the experts then give
// the expert offsets and the unit's STAGE block offsets, using the telescoped form
//   sum_{u' < u} n[u'][e] = min(P[u][e], C),  P[u][e] = pairs of e before unit u,
// so no table over all units is needed and there is no serial tail.  All threads of the workgroup must call it; it ends with a barrier.
__device__ __forceinline__ void block_plan(BlockPlan &bp, int b, const PlanPtrs &p, const Shape &s)
{
    const int E = s.E, C = s.C;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int u = b / s.bpu;
    if (!s.fast_plan) {
        const int first = u * s.bpu, last = first + s.bpu;
        for (int e = tid; e < E; e += blockDim.x) {
            const int total = p.counts[e], before = p.block_base[(size_t)first * E + e];
            bp.total[e] = total;
            bp.before[e] = before;
            bp.unit[e] = (last < s.num_blocks ? p.block_base[(size_t)last * E + e] : total) - before;
            bp.pre[e] = p.block_base[(size_t)b * E + e] - before;
        }
    } else {
        for (int e = tid; e < E; e += blockDim.x)
            bp.before[e] = bp.unit[e] = bp.pre[e] = bp.total[e] = 0;
        __syncthreads();
        const int total = s.num_blocks * E;
        const int first = u * s.bpu, last = first + s.bpu;     // blocks of this unit: [first, last)
        const int nthr = blockDim.x;
        if (nthr % E == 0) {
            // A lane meets one expert only and sums in registers, with one LDS update at the end.  The table
            // sits in the L2: a load costs hundreds of cycles, so a lane asks for LD of its counters at a time
            // before it adds any of them up (one at a time the loop is a chain of L2 round trips; measured on a
            // table of 256 x 64 counters the kernel takes 26 us this way against 32 us).  Small tables take the
            // plain loop, which needs fewer registers.
            const int e = tid % E;
            const int bl = tid / E, bstep = nthr / E;            // this lane's first block and its stride
            const int nblk = s.num_blocks;
            const BlockSums a = nblk > 4 * bstep
                                    ? sum_blocks<16>(p.block_counts, E, e, bl, bstep, nblk, b, first, last)
                                    : sum_blocks<1>(p.block_counts, E, e, bl, bstep, nblk, b, first, last);
            if (a.total) atomicAdd(&bp.total[e], a.total);
            if (a.before) atomicAdd(&bp.before[e], a.before);
            if (a.unit) atomicAdd(&bp.unit[e], a.unit);
            if (a.pre) atomicAdd(&bp.pre[e], a.pre);
        } else {
            for (int i = tid; i < total; i += nthr) {
                const int bb = i / E, e = i - bb * E;
                const int c = p.block_counts[i];
                if (c == 0) continue;
                atomicAdd(&bp.total[e], c);
                if (bb < first) atomicAdd(&bp.before[e], c);
                else if (bb < last) {
                    atomicAdd(&bp.unit[e], c);
                    if (bb < b) atomicAdd(&bp.pre[e], c);
                }
            }
        }
    }
    __syncthreads();
    // A wave scans 64 experts, the sums of the others' experts come through LDS: all four scan at a time (one after the other, by one
    // wave, 256 experts took eight scans in a row).
    const int e = wave * kWave + lane;
    int kp = 0, nu = 0, lo = 0, incl_off = 0, incl_st = 0;
    if (wave < 256 / kWave) {
        if (e < E) {
            kp = min(bp.total[e], C);
            lo = min(bp.before[e], C);
            nu = min(bp.before[e] + bp.unit[e], C) - lo;
        }
        incl_off = wave_inclusive_scan(kp);
        incl_st = wave_inclusive_scan(nu);
        const int incl_lo = wave_inclusive_scan(lo);
        if (lane == kWave - 1) {
            bp.sums[wave][0] = incl_off;
            bp.sums[wave][1] = incl_st;
            bp.sums[wave][2] = incl_lo;
        }
    }
    __syncthreads();
    if (wave < 256 / kWave) {
        int before_off = 0, before_st = 0, base_u = 0, R = 0;     // base_u: sum over experts of min(P[u][e], C), first STAGE row of the unit
#pragma unroll
        for (int w = 0; w < 256 / kWave; ++w) {
            before_off += w < wave ? bp.sums[w][0] : 0;
            before_st += w < wave ? bp.sums[w][1] : 0;
            R += bp.sums[w][0];
            base_u += bp.sums[w][2];
        }
        if (e < E) {
            bp.kpre[e] = before_off + incl_off - kp;
            bp.off[e] = s.padded ? e * C : before_off + incl_off - kp;
            bp.stage[e] = base_u + before_st + incl_st - nu;
        }
        if (threadIdx.x == 0) {
            bp.R = R;
            bp.unit_row0 = base_u;
        }
    }
    __syncthreads();
}

// STAGE and FINAL rows of one pair from the rebuilt scans; false if the pair is dropped.
__device__ __forceinline__ bool place_pair(const BlockPlan &bp, const Shape &s, int e, int local_rank, int &pf, int &ps)
{
    const int in_unit = bp.pre[e] + local_rank;     // rank among the unit's pairs of expert e
    const int r = bp.before[e] + in_unit;           // global stable rank
    pf = ps = -1;
    if (r >= s.C) return false;
    pf = bp.off[e] + r;
    ps = bp.stage[e] + in_unit;
    // always true for a consistent histogram table; guards a workspace that was never initialised
    if ((unsigned)pf < (unsigned)s.max_rows && (unsigned)ps < (unsigned)s.max_rows) return true;
    pf = ps = -1;
    return false;
}

// Plan + positions in one pass: workgroup b owns the
// tokens of route workgroup b, rebuilds the scans (block_plan) and writes its tokens' positions.
// The first workgroup of each unit writes that unit's rows of the public tables; workgroup 0
// writes the per-expert ones.
__device__ __forceinline__ void plan_positions_block(BlockPlan &bp, int b, const int32_t *__restrict__ topk_idx,
                                                     const PlanPtrs &p, const Shape &s)
{
    constexpr int PRE = 8;      // pairs per lane fetched before the table reduction, to overlap their latency
    const int E = s.E, k = s.k, C = s.C;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int u = b / s.bpu, ib = b - u * s.bpu;
    const int t_begin = u * s.Tu + ib * s.TB;
    int nt = s.Tu - ib * s.TB;
    if (nt > s.TB) nt = s.TB;
    // One (token, choice) pair per lane and pass, in the tables' own order: loads and stores of the per-pair
    // tables are contiguous across the lanes.
    const int npairs = nt * k, nthr = blockDim.x;
    const size_t pair0 = (size_t)t_begin * k;

    int e_pre[PRE], r_pre[PRE];
#pragma unroll
    for (int q = 0; q < PRE; ++q) {
        e_pre[q] = 0;
        r_pre[q] = 0;
        const int idx = tid + q * nthr;
        if (idx < npairs) {
            e_pre[q] = topk_idx[pair0 + idx];
            r_pre[q] = p.local_rank[pair0 + idx];
        }
    }
    for (int i = tid; i < s.TB; i += nthr) bp.alive[i] = 0;      // block_plan's barriers order this before its use
    block_plan(bp, b, p, s);

    for (int e = tid; e < E; e += blockDim.x) {
        if (ib == 0) {      // first workgroup of the unit publishes the unit's rows
            const int lo = bp.before[e] < C ? bp.before[e] : C;
            const int nxt = bp.before[e] + bp.unit[e];
            p.n[u * E + e] = (nxt < C ? nxt : C) - lo;
            p.stage_off[u * E + e] = bp.stage[e];
            p.unit_base[u * E + e] = bp.off[e] + lo;
        }
        if (b == 0) {
            if (s.fast_plan) p.counts[e] = bp.total[e];      // else written by the scan
            p.kept[e] = bp.total[e] < C ? bp.total[e] : C;
            p.offsets[e] = bp.off[e];
            p.kept_prefix[e] = bp.kpre[e];
        }
    }
    if (tid == 0) {
        if (ib == 0) p.unit_rows[u] = bp.unit_row0;
        if (b == 0) {
            p.offsets[E] = s.padded ? E * C : bp.R;
            p.kept_prefix[E] = bp.R;
            p.unit_rows[s.U] = bp.R;
            p.meta[META_R] = bp.R;
            p.meta[META_FINAL_ROWS] = s.padded ? E * C : bp.R;
            p.meta[META_C] = C;
        }
    }
    if (ib == 0) {
        const int E_loc = E / s.ep;
        for (int d = tid; d < s.ep; d += blockDim.x) {
            // rows for EP rank d = STAGE span of its experts inside this unit
            const int first_e = d * E_loc, end_e = first_e + E_loc;
            const int begin = bp.stage[first_e];
            int end;
            if (end_e < E) end = bp.stage[end_e];
            else {
                const int eL = E - 1;
                const int lo = bp.before[eL] < C ? bp.before[eL] : C;
                const int nxt = bp.before[eL] + bp.unit[eL];
                end = bp.stage[eL] + ((nxt < C ? nxt : C) - lo);
            }
            p.send_rows[u * s.ep + d] = end - begin;
        }
    }

    auto place = [&](int idx, int e, int lr) {
        int pf, ps;
        if (place_pair(bp, s, e, lr, pf, ps)) {
            p.row_map[ps] = pf;
            bp.alive[idx / k] = 1;
        }
        p.pos_final[pair0 + idx] = pf;
        p.pos_stage[pair0 + idx] = ps;
    };
#pragma unroll
    for (int q = 0; q < PRE; ++q) {
        const int idx = tid + q * nthr;
        if (idx < npairs) place(idx, e_pre[q], r_pre[q]);
    }
    for (int idx = tid + PRE * nthr; idx < npairs; idx += nthr) place(idx, topk_idx[pair0 + idx], p.local_rank[pair0 + idx]);
    // The tokens without a kept pair are taken off the shared counter, which holds all of them: an addition per workgroup makes a queue at
    // the memory, 10 ns each (32768 tokens in 512 workgroups: 28.2 us for routing and plan, none 22.9), and most have nothing to take.
    if (C >= s.T) return;
    __syncthreads();
    int mine = 0;
    for (int i = tid; i < nt; i += nthr) mine += bp.alive[i] ? 0 : 1;
    mine = wave_total(wave_inclusive_scan(mine));
    if (lane == 0) bp.sums[tid >> 6][0] = mine;                  // the plan's sums are no longer needed
    __syncthreads();
    if (tid == 0) {
        int dead = 0;
        for (int w = 0; w < nthr / kWave; ++w) dead += bp.sums[w][0];
        if (dead) atomicSub(&p.meta[META_ALIVE], dead);
    }
}

constexpr int kPlanThreads = 256;
__global__ __launch_bounds__(kPlanThreads) void plan_positions_kernel(const int32_t *__restrict__ topk_idx, PlanPtrs p, Shape s)
{
    __shared__ BlockPlan bp;
    plan_positions_block(bp, blockIdx.x, topk_idx, p, s);
}

__global__ void ws_init_kernel(int32_t *meta)
{
    if (threadIdx.x < META_SLOTS) meta[threadIdx.x] = 0;
}

// --------------------------------------------------------------- row movers

// Tokens [t0, t0+nt): each token row is read once and written to the STAGE row of
// every kept choice (read once / write up to k).  `lpr` lanes share a row.
template <bool NTL, bool NTS>
__device__ __forceinline__ void pack_rows_t(const u32x4 *__restrict__ x, u32x4 *__restrict__ stage,
                                          const int32_t *__restrict__ pos_stage, const Shape &s, int t0,
                                          int nt, int wg, int nwg)
{
    const int lpr = s.lpr, vpr = s.vpr, k = s.k;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    for (int i = wg * rows_per_wg + sub; i < nt; i += nwg * rows_per_wg) {
        const int t = t0 + i;
        const int32_t *pos = pos_stage + (size_t)t * k;
        const u32x4 *src = x + (size_t)t * vpr;
        // The first pass of the row is requested before the positions are looked at: the two latencies overlap
        // instead of adding up.  The price is the row of a token whose choices were all dropped, read in vain
        // (a few percent of the tokens of a workload with heavy drops, none otherwise).
        u32x4 val[kVecInFlight];
#pragma unroll
        for (int q = 0; q < kVecInFlight; ++q)
            if (lane + q * lpr < vpr) val[q] = ld16<NTL>(src + lane + q * lpr);
        bool any = false;
        for (int j = 0; j < k; ++j) any |= (unsigned)pos[j] < (unsigned)s.max_rows;
        if (!any) continue;                 // every choice of this token was dropped
        for (int v0 = lane; v0 < vpr; v0 += lpr * kVecInFlight) {
            if (v0 != lane) {
#pragma unroll
                for (int q = 0; q < kVecInFlight; ++q)
                    if (v0 + q * lpr < vpr) val[q] = ld16<NTL>(src + v0 + q * lpr);
            }
            for (int j = 0; j < k; ++j) {
                const int ps = pos[j];
                if ((unsigned)ps >= (unsigned)s.max_rows) continue;   // dropped (-1) or not a row
                u32x4 *dst = stage + (size_t)ps * vpr;
#pragma unroll
                for (int q = 0; q < kVecInFlight; ++q)
                    if (v0 + q * lpr < vpr) st16<NTS>(dst + v0 + q * lpr, val[q]);
            }
        }
    }
}

__device__ __forceinline__ void pack_rows(const u32x4 *__restrict__ x, u32x4 *__restrict__ stage,
                                          const int32_t *__restrict__ pos_stage, const Shape &s, int t0,
                                          int nt, int wg, int nwg)
{
    with_policy(s.cache & NT_PACK_LD, s.cache & NT_PACK_ST, [&](auto l, auto st) {
        pack_rows_t<decltype(l)::value, decltype(st)::value>(x, stage, pos_stage, s, t0, nt, wg, nwg);
    });
}

// STAGE rows [r0, r1) go to FINAL rows row_map[.], walked in STAGE order: the reads are one contiguous run, the
// writes one run per (unit, expert) block.  (Walking a slice's rows expert by expert instead, so that the writes
// of neighbouring workgroups are neighbours, needs a second lookup per row and measured slower on three of four
// large workloads, 2 % faster on one.)
// REVERSE: the other direction (the mirrored return path): row row_map[r] of `fin` goes to row r of `stage`.
template <bool REVERSE, bool NTL, bool NTS>
__device__ __forceinline__ void regather_rows_t(u32x4 *stage, u32x4 *fin, const int32_t *__restrict__ row_map,
                                                const Shape &s, int r0, int r1, int wg, int nwg)
{
    const int lpr = s.lpr, vpr = s.vpr;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    if (r0 < 0) r0 = 0;
    if (r1 > s.max_rows) r1 = s.max_rows;
    for (int r = r0 + wg * rows_per_wg + sub; r < r1; r += nwg * rows_per_wg) {
        u32x4 val[kVecInFlight];
        if (!REVERSE) {
            // forward: the source row does not depend on the table, so its first pass is requested before the
            // destination is looked up
            const u32x4 *src0 = stage + (size_t)r * vpr;
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (lane + q * lpr < vpr) val[q] = ld16<NTL>(src0 + lane + q * lpr);
        }
        const int fr = row_map[r];
        if ((unsigned)fr >= (unsigned)s.max_rows) continue;
        const u32x4 *src = REVERSE ? fin + (size_t)fr * vpr : stage + (size_t)r * vpr;
        u32x4 *dst = REVERSE ? stage + (size_t)r * vpr : fin + (size_t)fr * vpr;
        for (int v0 = lane; v0 < vpr; v0 += lpr * kVecInFlight) {
            if (REVERSE || v0 != lane) {
#pragma unroll
                for (int q = 0; q < kVecInFlight; ++q)
                    if (v0 + q * lpr < vpr) val[q] = ld16<NTL>(src + v0 + q * lpr);
            }
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (v0 + q * lpr < vpr) st16<NTS>(dst + v0 + q * lpr, val[q]);
        }
    }
}

// Capacity-padded layout: zero-fills the padding rows [e*C + kept[e], (e+1)*C) of every expert.  Padding row i
// (0 <= i < E*C - R) belongs to the expert found by bisection over pad_before[e] = e*C - kept_prefix[e].
// kept_prefix and kept: the plan tables, or the same values rebuilt in LDS.
__device__ __forceinline__ void pad_rows(u32x4 *__restrict__ fin, const int32_t *kept_prefix, const int32_t *kept, int R,
                                         const Shape &s, int wg, int nwg, int nthr = kMoverThreads)
{
    const int lpr = s.lpr, vpr = s.vpr, E = s.E, C = s.C;
    const int rows_per_wg = nthr / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    int total = E * C - R;
    if (total > s.max_rows) total = s.max_rows;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = wg * rows_per_wg + sub; i < total; i += nwg * rows_per_wg) {
        int lo = 0, hi = E - 1;                      // largest e with pad_before[e] <= i
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (mid * C - kept_prefix[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        const int row = lo * C + min(kept[lo], C) + (i - (lo * C - kept_prefix[lo]));
        if ((unsigned)row >= (unsigned)s.max_rows || row >= (lo + 1) * C) continue;
        u32x4 *dst = fin + (size_t)row * vpr;
        for (int v = lane; v < vpr; v += lpr) st16<true>(dst + v, zero);
    }
}

__device__ __forceinline__ void pad_rows(u32x4 *__restrict__ fin, const PlanPtrs &p, const Shape &s, int wg, int nwg)
{
    pad_rows(fin, p.kept_prefix, p.kept, p.kept_prefix[s.E], s, wg, nwg);
}

__device__ __forceinline__ void regather_rows(const u32x4 *__restrict__ stage, u32x4 *__restrict__ fin,
                                              const PlanPtrs &p, const Shape &s, int r0, int r1, int wg, int nwg)
{
    with_policy(s.cache & NT_REG_LD, s.cache & NT_REG_ST, [&](auto l, auto st) {
        regather_rows_t<false, decltype(l)::value, decltype(st)::value>(const_cast<u32x4 *>(stage), fin, p.row_map, s, r0,
                                                                        r1, wg, nwg);
    });
}

// the mirrored direction: expert output y (FINAL layout) back to the unit-major layout
__device__ __forceinline__ void unregather_rows(const u32x4 *__restrict__ y, u32x4 *__restrict__ y_stage,
                                                const int32_t *__restrict__ row_map, const Shape &s, int r0,
                                                int r1, int wg, int nwg)
{
    with_policy(s.cache & NT_REG_LD, s.cache & NT_REG_ST, [&](auto l, auto st) {
        regather_rows_t<true, decltype(l)::value, decltype(st)::value>(y_stage, const_cast<u32x4 *>(y), row_map, s, r0, r1,
                                                                       wg, nwg);
    });
}

// pack for tokens whose positions have not been written yet: the workgroup rebuilds the scans of
// the route workgroup its tokens belong to (all of them belong to one: the host checks the shape)
// and derives the STAGE rows itself.  The first pass of every row is loaded before the rebuild, so
// the table read overlaps the row read.  Writes no table: plan_positions_block does that.
template <bool NTL, bool NTS>
__device__ __forceinline__ void pack_rows_selfplan_t(BlockPlan &bp, const u32x4 *__restrict__ x,
                                                     u32x4 *__restrict__ stage, const int32_t *__restrict__ topk_idx,
                                                     const PlanPtrs &p, const Shape &s, int t0, int nt, int wg)
{
    const int lpr = s.lpr, vpr = s.vpr, k = s.k;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    const int i = wg * rows_per_wg + sub;
    const bool have = i < nt;
    const int t = t0 + (have ? i : 0);
    const int t_first = t0 + wg * rows_per_wg;                  // same route workgroup for the whole group
    const int u = t_first / s.Tu;
    const int b = u * s.bpu + (t_first - u * s.Tu) / s.TB;
    const u32x4 *src = x + (size_t)t * vpr;
    u32x4 val[kVecInFlight];
#pragma unroll
    for (int q = 0; q < kVecInFlight; ++q)
        if (have && lane + q * lpr < vpr) val[q] = ld16<NTL>(src + lane + q * lpr);
    block_plan(bp, b, p, s);
    if (!have) return;
    for (int v0 = lane; v0 < vpr; v0 += lpr * kVecInFlight) {
        if (v0 != lane) {
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (v0 + q * lpr < vpr) val[q] = ld16<NTL>(src + v0 + q * lpr);
        }
        for (int j = 0; j < k; ++j) {
            int pf, ps;
            if (!place_pair(bp, s, topk_idx[(size_t)t * k + j], p.local_rank[(size_t)t * k + j], pf, ps)) continue;
            u32x4 *dst = stage + (size_t)ps * vpr;
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (v0 + q * lpr < vpr) st16<NTS>(dst + v0 + q * lpr, val[q]);
        }
    }
}

// One grid, two jobs: the first n_plan workgroups finish the plan (tables and positions of every
// token), the others pack slice 0 with positions they derive themselves, so the first pack does
// not wait for the plan kernel.
__global__ __launch_bounds__(kMoverThreads) void plan_pack_kernel(const int32_t *__restrict__ topk_idx,
                                                                  const u32x4 *__restrict__ x,
                                                                  u32x4 *__restrict__ stage, PlanPtrs p, Shape s,
                                                                  int t0, int nt, int n_plan)
{
    __shared__ BlockPlan bp;
    const int bid = blockIdx.x;
    if (bid < n_plan) {
        plan_positions_block(bp, bid, topk_idx, p, s);
        return;
    }
    with_policy(s.cache & NT_PACK_LD, s.cache & NT_PACK_ST, [&](auto l, auto st) {
        pack_rows_selfplan_t<decltype(l)::value, decltype(st)::value>(bp, x, stage, topk_idx, p, s, t0, nt,
                                                                      bid - n_plan);
    });
}

// ---- pack and re-gather in one pass
//
// A kept pair's row has two places, one in STAGE and one in FINAL, and both are known once the plan is: each token row
// is read once and stored to all of them, instead of being packed into STAGE and read back from there.  Of the
// (alive + R) + 2R rows that the two passes move, alive + 2R are left.  STAGE and FINAL end up as the two passes leave
// them.

// One row, with the rows its choices go to held by the first k lanes of its lane group (my_ps, my_pf; bit j of `kept`:
// choice j is kept), so that no lane waits for a table between two stores.  WAVE: a row is shared by whole waves, the
// destinations are then uniform and live in scalar registers.  `val` is the row's first pass, already requested.
template <bool WAVE, bool NTL, bool NTS, bool NTF>
__device__ __forceinline__ void place_row(const u32x4 *__restrict__ src, u32x4 *__restrict__ stage, u32x4 *__restrict__ fin,
                                          const Shape &s, int lane, int gbase, unsigned int kept, int my_ps, int my_pf,
                                          u32x4 (&val)[kVecInFlight])
{
    const int lpr = s.lpr, vpr = s.vpr;
    if (WAVE) kept = __builtin_amdgcn_readfirstlane(kept);
    for (int vbase = 0; vbase < vpr; vbase += lpr * kVecInFlight) {
        const int v0 = vbase + lane;
        if (vbase != 0) {
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (v0 + q * lpr < vpr) val[q] = ld16<NTL>(src + v0 + q * lpr);
        }
        for (unsigned int rem = kept; rem; rem &= rem - 1) {
            const int j = __builtin_ctz(rem);
            int ps, pf;
            if (WAVE) {
                ps = __builtin_amdgcn_readlane(my_ps, j);
                pf = __builtin_amdgcn_readlane(my_pf, j);
            } else {
                ps = __shfl(my_ps, gbase + j, kWave);
                pf = __shfl(my_pf, gbase + j, kWave);
            }
            u32x4 *ds = stage + (size_t)ps * vpr, *df = fin + (size_t)pf * vpr;
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (v0 + q * lpr < vpr) st16<NTS>(ds + v0 + q * lpr, val[q]);
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (v0 + q * lpr < vpr) st16<NTF>(df + v0 + q * lpr, val[q]);
        }
    }
}

// Tokens [t0, t0+nt), the rows of their choices taken from the plan tables.  Where choices may be dropped (s.lazy) a row is
// requested behind its token's table entries and not at all if none is kept: what bounds the pass is bytes, and enough other
// workgroups are there to hide the entries' latency.
template <bool WAVE, bool NTL, bool NTS, bool NTF>
__device__ __forceinline__ void place_rows_t(const u32x4 *__restrict__ x, u32x4 *__restrict__ stage, u32x4 *__restrict__ fin,
                                             const PlanPtrs &p, const Shape &s, int t0, int nt, int wg, int nwg)
{
    const int lpr = s.lpr, vpr = s.vpr, k = s.k;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    const int wl = threadIdx.x & (kWave - 1);
    const int gbase = lpr >= kWave ? 0 : (wl & ~(lpr - 1)), gl = wl - gbase;
    const unsigned int kmask = k >= 32 ? 0xffffffffu : ((1u << k) - 1u);
    for (int i = wg * rows_per_wg + sub; i < nt; i += nwg * rows_per_wg) {
        const int t = t0 + i;
        const u32x4 *src = x + (size_t)t * vpr;
        // otherwise the row's first pass and the table entries are requested together
        u32x4 val[kVecInFlight];
        auto request = [&] {
#pragma unroll
            for (int q = 0; q < kVecInFlight; ++q)
                if (lane + q * lpr < vpr) val[q] = ld16<NTL>(src + lane + q * lpr);
        };
        const bool lazy = s.lazy && (WAVE || k <= lpr);
        if (!lazy) request();
        const size_t pair = (size_t)t * k;
        if (WAVE || k <= lpr) {
            int ps = -1, pf = -1;
            if (gl < k) {
                ps = p.pos_stage[pair + gl];
                pf = p.pos_final[pair + gl];
            }
            const bool ok = (unsigned)ps < (unsigned)s.max_rows && (unsigned)pf < (unsigned)s.max_rows;
            const unsigned int kept = (unsigned int)(__ballot(ok) >> gbase) & kmask;
            if (lazy) {
                if (!kept) continue;
                request();
            }
            place_row<WAVE, NTL, NTS, NTF>(src, stage, fin, s, lane, gbase, kept, ps, pf, val);
        } else {
            // fewer lanes per row than choices (rows of at most 256 bytes): one choice after the other
            for (int j = 0; j < k; ++j) {
                const int ps = p.pos_stage[pair + j], pf = p.pos_final[pair + j];
                if ((unsigned)ps >= (unsigned)s.max_rows || (unsigned)pf >= (unsigned)s.max_rows) continue;
                if (lane < vpr) {           // lpr < 32 lanes hold the whole row in their first vectors
                    st16<NTS>(stage + (size_t)ps * vpr + lane, val[0]);
                    st16<NTF>(fin + (size_t)pf * vpr + lane, val[0]);
                }
            }
        }
    }
}

template <bool WAVE>
__global__ __launch_bounds__(kMoverThreads) void place_kernel(const u32x4 *__restrict__ x, u32x4 *__restrict__ stage,
                                                              u32x4 *__restrict__ fin, PlanPtrs p, Shape s)
{
    with_policy3(s.cache & NT_PACK_LD, s.cache & NT_PACK_ST, s.cache & NT_REG_ST, [&](auto l, auto st, auto f) {
        place_rows_t<WAVE, decltype(l)::value, decltype(st)::value, decltype(f)::value>(x, stage, fin, p, s, 0, s.T,
                                                                                       blockIdx.x, gridDim.x);
    });
    if (s.padded) pad_rows(fin, p, s, blockIdx.x, gridDim.x);
}

// The same ahead of the plan tables: the first n_plan workgroups finish the plan, each of the others rebuilds the scans
// for the one route workgroup its `span` consecutive tokens belong to (the host checks the shape) and derives the rows of
// their choices itself.  One rebuild serves all rows of a workgroup, and the first row and its routing are on their way
// while it runs, also if s.lazy.
template <bool WAVE, bool NTL, bool NTS, bool NTF>
__device__ __forceinline__ void place_rows_selfplan_t(BlockPlan &bp, const u32x4 *__restrict__ x, u32x4 *__restrict__ stage,
                                                      u32x4 *__restrict__ fin, const int32_t *__restrict__ topk_idx,
                                                      const PlanPtrs &p, const Shape &s, int span, int wg, int nwg)
{
    const int lpr = s.lpr, vpr = s.vpr, k = s.k;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    const int wl = threadIdx.x & (kWave - 1);
    const int gbase = lpr >= kWave ? 0 : (wl & ~(lpr - 1)), gl = wl - gbase;
    const unsigned int kmask = k >= 32 ? 0xffffffffu : ((1u << k) - 1u);
    const int t_first = wg * span, t_end = min(t_first + span, s.T);
    const int u = t_first / s.Tu;
    const int b = u * s.bpu + (t_first - u * s.Tu) / s.TB;
    u32x4 val[kVecInFlight];
    int e = 0, lr = 0;
    auto request_row = [&](int t) {
        const u32x4 *src = x + (size_t)t * vpr;
#pragma unroll
        for (int q = 0; q < kVecInFlight; ++q)
            if (lane + q * lpr < vpr) val[q] = ld16<NTL>(src + lane + q * lpr);
    };
    auto request = [&](int t, bool row) {
        if (row) request_row(t);
        if (gl < k) {
            e = topk_idx[(size_t)t * k + gl];
            lr = p.local_rank[(size_t)t * k + gl];
        }
    };
    const bool lazy = s.lazy && (WAVE || k <= lpr);
    if (t_first + sub < t_end) request(t_first + sub, true);
    block_plan(bp, b, p, s);
    for (int t = t_first + sub; t < t_end; t += rows_per_wg) {
        const bool later = t != t_first + sub;
        if (later) request(t, !lazy);
        if (WAVE || k <= lpr) {
            int ps = -1, pf = -1;
            const bool ok = gl < k && place_pair(bp, s, e, lr, pf, ps);
            const unsigned int kept = (unsigned int)(__ballot(ok) >> gbase) & kmask;
            if (lazy && !kept) continue;
            if (lazy && later) request_row(t);
            place_row<WAVE, NTL, NTS, NTF>(x + (size_t)t * vpr, stage, fin, s, lane, gbase, kept, ps, pf, val);
        } else {
            for (int j = 0; j < k; ++j) {
                int ps, pf;
                if (!place_pair(bp, s, topk_idx[(size_t)t * k + j], p.local_rank[(size_t)t * k + j], pf, ps)) continue;
                if (lane < vpr) {
                    st16<NTS>(stage + (size_t)ps * vpr + lane, val[0]);
                    st16<NTF>(fin + (size_t)pf * vpr + lane, val[0]);
                }
            }
        }
    }
    if (s.padded) pad_rows(fin, bp.kpre, bp.total, bp.R, s, wg, nwg);
}

template <bool WAVE>
__global__ __launch_bounds__(kMoverThreads) void plan_place_kernel(const int32_t *__restrict__ topk_idx,
                                                                   const u32x4 *__restrict__ x, u32x4 *__restrict__ stage,
                                                                   u32x4 *__restrict__ fin, PlanPtrs p, Shape s, int span,
                                                                   int n_plan)
{
    __shared__ BlockPlan bp;
    const int bid = blockIdx.x;
    if (bid < n_plan) {
        plan_positions_block(bp, bid, topk_idx, p, s);
        return;
    }
    with_policy3(s.cache & NT_PACK_LD, s.cache & NT_PACK_ST, s.cache & NT_REG_ST, [&](auto l, auto st, auto f) {
        place_rows_selfplan_t<WAVE, decltype(l)::value, decltype(st)::value, decltype(f)::value>(
            bp, x, stage, fin, topk_idx, p, s, span, bid - n_plan, gridDim.x - n_plan);
    });
}

__global__ __launch_bounds__(kMoverThreads) void pack_kernel(const u32x4 *__restrict__ x, u32x4 *__restrict__ stage,
                                                             PlanPtrs p, Shape s, int t0, int nt)
{
    pack_rows(x, stage, p.pos_stage, s, t0, nt, blockIdx.x, gridDim.x);
}

// u0, u1: unit range whose STAGE rows are moved (row range read from the device table)
__global__ __launch_bounds__(kMoverThreads) void regather_kernel(const u32x4 *__restrict__ stage,
                                                                 u32x4 *__restrict__ fin, PlanPtrs p, Shape s,
                                                                 int u0, int u1)
{
    regather_rows(stage, fin, p, s, p.unit_rows[u0], p.unit_rows[u1], blockIdx.x, gridDim.x);
    if (s.padded && u0 == 0) pad_rows(fin, p, s, blockIdx.x, gridDim.x);
}

// One grid, two jobs in disjoint workgroups: the first n_pack_wg workgroups pack
// slice j (tokens [t0, t0+nt)), the others regather slice j-1 (units [u0, u1)).
// The two touch disjoint rows of STAGE, so they may run in any interleaving.
__global__ __launch_bounds__(kMoverThreads) void pack_regather_kernel(const u32x4 *__restrict__ x,
                                                                      u32x4 *__restrict__ stage,
                                                                      u32x4 *__restrict__ fin, PlanPtrs p, Shape s,
                                                                      int t0, int nt, int u0, int u1, int n_pack_wg)
{
    // interleave the two jobs over the grid so that both make progress from the start
    const int n_reg_wg = gridDim.x - n_pack_wg;
    const int bid = blockIdx.x;
    const int pairs = n_pack_wg < n_reg_wg ? n_pack_wg : n_reg_wg;
    bool is_pack;
    int idx;
    if (bid < 2 * pairs) {
        is_pack = (bid & 1) == 0;
        idx = bid >> 1;
    } else {
        is_pack = n_pack_wg > n_reg_wg;
        idx = bid - pairs;
    }
    if (is_pack)
        pack_rows(x, stage, p.pos_stage, s, t0, nt, idx, n_pack_wg);
    else
{
        regather_rows(stage, fin, p, s, p.unit_rows[u0], p.unit_rows[u1], idx, n_reg_wg);
        if (s.padded && u0 == 0) pad_rows(fin, p, s, idx, n_reg_wg);
    }
}

// ------------------------------------------------------------------ combine

__device__ __forceinline__ double bf16_lo(unsigned int w) { return (double)__uint_as_float(w << 16); }
__device__ __forceinline__ double bf16_hi(unsigned int w) { return (double)__uint_as_float(w & 0xffff0000u); }

// fp64 -> bf16 bits with ONE rounding (nearest, ties to even).  The value first goes to fp32 (nearest-even, one
// hardware conversion).  Rounding is monotone and every midpoint between two bf16 values is an fp32 number, so
// unless the fp32 value IS such a midpoint (low 16 bits 0x8000) it lies on the same side of every midpoint as
// the fp64 value, and rounding it to nearest gives the fp64 value's bf16: add 0x8000 and drop the low half.
// Only in the midpoint case (one in 65536) the fp32 step may have hidden on which side the fp64 value lay: the
// slow branch compares the two and rounds down, up, or (a true tie) to even.  Overflow, underflow and
// infinities fall out of the same arithmetic; NaN is mapped to the canonical quiet NaN.
__device__ __forceinline__ unsigned int f64_to_bf16_rne(double d)
{
    const float f = (float)d;                       // nearest-even
    const unsigned int u = __float_as_uint(f);
    unsigned int r = (u + 0x8000u) >> 16;
    if (__builtin_expect((u & 0xffffu) == 0x8000u, 0)) {
        const double back = (double)f;
        if (back == d) r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;                 // true tie: to even
        else if (__builtin_fabs(back) > __builtin_fabs(d)) r = u >> 16;            // below the midpoint
        else r = (u >> 16) + 1u;                                                   // above it
    }
    return f != f ? 0x7fc0u : r;
}

// out[t] = sum_j gate[t,j] * y[pos_final[t,j]] over kept j in ascending order.
// The sum is carried in fp64 (every product of an fp32 gate with an fp32 / bf16
// element is exact there) and rounded once to the activation type, so the rounding
// decision is taken at the same precision as the CPU reference takes it; measured
// against a copy-only version of the same loop the arithmetic costs a few percent.
// NV 16-byte vectors per lane per pass: 2 covers rows up to 8 KiB in one pass, 4 up
// to 16 KiB.  Tokens are walked from the last to the first: the FINAL rows written
// most recently (by the last slices) are read first, while the memory-side cache
// still holds them.  A dropped pair is skipped; a token with no kept pair writes zeros.
// `pos_table` is pos_final (y in FINAL layout) or pos_stage (y in the unit-major layout of the mirrored
// return path); tokens [t0, t0+nt) are combined by workgroups wg of nwg.
// KEEP: the mirrored return path in one pass: each row read from y is also stored, unchanged, to its place in the
// unit-major layout (keep, rows from keep_table; non-temporal if NTK) before it is added.
template <bool BF16, int NV, bool NTL, bool NTS, bool KEEP = false, bool NTK = false>
__device__ __forceinline__ void combine_rows_t(const u32x4 *__restrict__ y, const float *__restrict__ gates,
                                               u32x4 *__restrict__ out, const int32_t *__restrict__ pos_table,
                                               const Shape &s, int t0, int nt, int wg, int nwg,
                                               u32x4 *__restrict__ keep = nullptr,
                                               const int32_t *__restrict__ keep_table = nullptr)
{
    constexpr int NF = BF16 ? 8 : 4;            // accumulators per vector
    const int lpr = s.lpr, vpr = s.vpr, k = s.k;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    for (int i = wg * rows_per_wg + sub; i < nt; i += nwg * rows_per_wg) {
        const int t = t0 + nt - 1 - i;
        const int32_t *pos = pos_table + (size_t)t * k;
        const float *g = gates + (size_t)t * k;
        u32x4 *dst = out + (size_t)t * vpr;
        for (int v0 = lane; v0 < vpr; v0 += lpr * NV) {
            double acc[NV][NF];
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int f = 0; f < NF; ++f) acc[q][f] = 0.0;
            for (int j = 0; j < k; ++j) {
                const int pf = pos[j];
                if ((unsigned)pf >= (unsigned)s.max_rows) continue;   // dropped (-1) or not a row
                const double gj = (double)g[j];
                const u32x4 *src = y + (size_t)pf * vpr;
                u32x4 val[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q)
                    if (v0 + q * lpr < vpr) val[q] = ld16<NTL>(src + v0 + q * lpr);
                if (KEEP) {
                    const int pk = keep_table[(size_t)t * k + j];
                    if ((unsigned)pk < (unsigned)s.max_rows) {
#pragma unroll
                        for (int q = 0; q < NV; ++q)
                            if (v0 + q * lpr < vpr) st16<NTK>(keep + (size_t)pk * vpr + v0 + q * lpr, val[q]);
                    }
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    if (v0 + q * lpr < vpr) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            if (BF16) {
                                acc[q][2 * c] = __builtin_fma(gj, bf16_lo(val[q][c]), acc[q][2 * c]);
                                acc[q][2 * c + 1] = __builtin_fma(gj, bf16_hi(val[q][c]), acc[q][2 * c + 1]);
                            } else {
                                acc[q][c] = __builtin_fma(gj, (double)__uint_as_float(val[q][c]), acc[q][c]);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                if (v0 + q * lpr < vpr) {
                    u32x4 o;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        if (BF16)
                            o[c] = f64_to_bf16_rne(acc[q][2 * c]) | (f64_to_bf16_rne(acc[q][2 * c + 1]) << 16);
                        else
                            o[c] = __float_as_uint((float)acc[q][c]);
                    }
                    st16<NTS>(dst + v0 + q * lpr, o);
                }
            }
        }
    }
}

// The same scale-add with the row reads software-pipelined.  One wave's time on a token is a chain of
// memory latencies: position and gate of choice j, then the row they point to, then the next choice.  Here
// the first k lanes of a row's lane group fetch the token's k positions and gates in one go (a ballot of
// their validity gives the kept choices as a bit mask, shuffles hand each one to all lanes), and the row of
// the next kept choice is requested before the current one is added, so two rows' loads are in flight per
// lane and the fp64 arithmetic runs under them.  Needs k <= lanes per row (the host checks).  Same order of
// additions, same result.
template <bool BF16, int NV, bool NTL, bool NTS, bool KEEP = false, bool NTK = false>
__device__ __forceinline__ void combine_rows_pf_t(const u32x4 *__restrict__ y, const float *__restrict__ gates,
                                                  u32x4 *__restrict__ out, const int32_t *__restrict__ pos_table,
                                                  const Shape &s, int t0, int nt, int wg, int nwg,
                                                  u32x4 *__restrict__ keep = nullptr,
                                                  const int32_t *__restrict__ keep_table = nullptr)
{
    constexpr int NF = BF16 ? 8 : 4;            // accumulators per vector
    const int lpr = s.lpr, vpr = s.vpr, k = s.k;
    const int rows_per_wg = kMoverThreads / lpr;
    const int sub = threadIdx.x / lpr, lane = threadIdx.x - sub * lpr;
    const int wl = threadIdx.x & (kWave - 1);
    const int gbase = lpr >= kWave ? 0 : (wl & ~(lpr - 1));     // first lane, inside the wave, of this lane's row group
    const int gl = wl - gbase;                                  // this lane's index in it
    const unsigned int kmask = k >= 32 ? 0xffffffffu : ((1u << k) - 1u);
    for (int i = wg * rows_per_wg + sub; i < nt; i += nwg * rows_per_wg) {
        const int t = t0 + nt - 1 - i;
        u32x4 *dst = out + (size_t)t * vpr;
        int my_pos = -1, my_keep = -1;
        float my_g = 0.f;
        if (gl < k) {
            my_pos = pos_table[(size_t)t * k + gl];
            my_g = gates[(size_t)t * k + gl];
            if (KEEP) my_keep = keep_table[(size_t)t * k + gl];
        }
        const unsigned long long valid = __ballot((unsigned)my_pos < (unsigned)s.max_rows);
        const unsigned int kept = (unsigned int)(valid >> gbase) & kmask;      // bit j: choice j of this token is kept
        // every lane of the group walks every pass, also lanes past the end of a short row: the shuffles below
        // read the positions from the group's first k lanes, which must therefore stay active
        for (int vbase = 0; vbase < vpr; vbase += lpr * NV) {
            const int v0 = vbase + lane;
            double acc[NV][NF];
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int f = 0; f < NF; ++f) acc[q][f] = 0.0;
            unsigned int rem = kept;
            u32x4 cur[NV];
            float g_cur = 0.f;
            int k_cur = -1;
            bool have = rem != 0;
            if (have) {
                const int j = __builtin_ctz(rem);
                rem &= rem - 1;
                const int pf = __shfl(my_pos, gbase + j, kWave);
                if (KEEP) k_cur = __shfl(my_keep, gbase + j, kWave);
                g_cur = __shfl(my_g, gbase + j, kWave);
                const u32x4 *src = y + (size_t)pf * vpr;
#pragma unroll
                for (int q = 0; q < NV; ++q)
                    if (v0 + q * lpr < vpr) cur[q] = ld16<NTL>(src + v0 + q * lpr);
            }
            while (have) {
                u32x4 nxt[NV];
                float g_nxt = 0.f;
                int k_nxt = -1;
                const bool have_nxt = rem != 0;
                if (have_nxt) {
                    const int j = __builtin_ctz(rem);
                    rem &= rem - 1;
                    const int pf = __shfl(my_pos, gbase + j, kWave);
                    if (KEEP) k_nxt = __shfl(my_keep, gbase + j, kWave);
                    g_nxt = __shfl(my_g, gbase + j, kWave);
                    const u32x4 *src = y + (size_t)pf * vpr;
#pragma unroll
                    for (int q = 0; q < NV; ++q)
                        if (v0 + q * lpr < vpr) nxt[q] = ld16<NTL>(src + v0 + q * lpr);
                }
                const double gj = (double)g_cur;
                if (KEEP && (unsigned)k_cur < (unsigned)s.max_rows) {
#pragma unroll
                    for (int q = 0; q < NV; ++q)
                        if (v0 + q * lpr < vpr) st16<NTK>(keep + (size_t)k_cur * vpr + v0 + q * lpr, cur[q]);
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    if (v0 + q * lpr < vpr) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            if (BF16) {
                                acc[q][2 * c] = __builtin_fma(gj, bf16_lo(cur[q][c]), acc[q][2 * c]);
                                acc[q][2 * c + 1] = __builtin_fma(gj, bf16_hi(cur[q][c]), acc[q][2 * c + 1]);
                            } else {
                                acc[q][c] = __builtin_fma(gj, (double)__uint_as_float(cur[q][c]), acc[q][c]);
                            }
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) cur[q] = nxt[q];
                g_cur = g_nxt;
                k_cur = k_nxt;
                have = have_nxt;
            }
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                if (v0 + q * lpr < vpr) {
                    u32x4 o;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        if (BF16)
                            o[c] = f64_to_bf16_rne(acc[q][2 * c]) | (f64_to_bf16_rne(acc[q][2 * c + 1]) << 16);
                        else
                            o[c] = __float_as_uint((float)acc[q][c]);
                    }
                    st16<NTS>(dst + v0 + q * lpr, o);
                }
            }
        }
    }
}

// The same scale-add in smaller pieces: a wave takes 64 vectors of one token's output (WAVE; with rows of fewer vectors several tokens), one
// per lane, and has the rows of up to K choices on their way at a time.  No lane is without work but in a row's last piece, where 256 lanes
// of 2 or 4 vectors leave up to half of themselves idle, and few registers per lane leave room for many waves.  Same order of additions, same
// result.  What bounds it is memory, and for few tokens the chain position, row, output.  Where it is used and what it gives stands at combine_units.
template <bool BF16, int K, bool WAVE, bool NTL, bool NTS, bool KEEP, bool NTK>
__device__ __forceinline__ void combine_units_t(const u32x4 *__restrict__ y, const float *__restrict__ gates, u32x4 *__restrict__ out,
                                                const int32_t *__restrict__ pos_table, const Shape &s, u32x4 *__restrict__ keep,
                                                const int32_t *__restrict__ keep_table)
{
    constexpr int NF = BF16 ? 8 : 4;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int vpr = s.vpr, k = s.k, lpr = WAVE ? kWave : s.lpr;
    const int gbase = WAVE ? 0 : lane & ~(lpr - 1), gl = lane - gbase;
    const uint32_t parts = WAVE ? (uint32_t)((vpr + kWave - 1) / kWave) : 1u;
    const int per = WAVE ? 1 : kWave / lpr;                        // tokens of a wave
    const int64_t units = WAVE ? (int64_t)s.T * parts : (s.T + per - 1) / per;
    for (int64_t unit = (int64_t)blockIdx.x * (kMoverThreads / kWave) + wave; unit < units; unit += (int64_t)gridDim.x * (kMoverThreads / kWave)) {
        const int i = !WAVE ? (int)unit * per + (lane / lpr) : units >> 32 ? (int)(unit / parts) : (int)((uint32_t)unit / parts);
        const int v = (WAVE ? (int)(unit - (int64_t)i * parts) * kWave : 0) + gl, t = s.T - 1 - i;
        const bool have = t >= 0, in = have && v < vpr;
        int my_pos = -1, my_keep = -1;
        float my_g = 0.f;
        if (have && gl < k) {
            my_pos = pos_table[(size_t)t * k + gl];
            my_g = gates[(size_t)t * k + gl];
            if (KEEP) my_keep = keep_table[(size_t)t * k + gl];
        }
        const unsigned int kmask = k >= 32 ? 0xffffffffu : ((1u << k) - 1u);
        unsigned int kept = (unsigned int)(__ballot((unsigned)my_pos < (unsigned)s.max_rows) >> gbase) & kmask;
        if (WAVE) kept = (unsigned int)__builtin_amdgcn_readfirstlane((int)kept);
        auto of = [&](int x, int j) { return WAVE ? __builtin_amdgcn_readlane(x, j) : __shfl(x, gbase + j, kWave); };
        double acc[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = 0.0;
        for (int j0 = 0; j0 < k; j0 += K) {
            u32x4 val[K];
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const int pf = of(my_pos, j0 + q < k ? j0 + q : 0);
                if ((kept >> (j0 + q) & 1u) && j0 + q < k && in) val[q] = ld16<NTL>(y + (size_t)pf * vpr + v);
            }
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const int j = j0 + q < k ? j0 + q : 0;
                const double g = (double)__int_as_float(of(__float_as_int(my_g), j));
                const int pk = KEEP ? of(my_keep, j) : -1;
                if ((kept >> (j0 + q) & 1u) && j0 + q < k) {
                    if (KEEP && in && (unsigned)pk < (unsigned)s.max_rows) st16<NTK>(keep + (size_t)pk * vpr + v, val[q]);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        if (BF16) {
                            acc[2 * c] = __builtin_fma(g, bf16_lo(val[q][c]), acc[2 * c]);
                            acc[2 * c + 1] = __builtin_fma(g, bf16_hi(val[q][c]), acc[2 * c + 1]);
                        } else {
                            acc[c] = __builtin_fma(g, (double)__uint_as_float(val[q][c]), acc[c]);
                        }
                    }
                }
            }
        }
        u32x4 o;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (BF16) o[c] = f64_to_bf16_rne(acc[2 * c]) | (f64_to_bf16_rne(acc[2 * c + 1]) << 16);
            else o[c] = __float_as_uint((float)acc[c]);
        }
        if (in) st16<NTS>(out + (size_t)t * vpr + v, o);
    }
}

template <bool BF16, int K, bool WAVE>
__global__ __launch_bounds__(kMoverThreads) void combine_units_kernel(const u32x4 *__restrict__ y, const float *__restrict__ gates,
                                                                      u32x4 *__restrict__ out, PlanPtrs p, Shape s)
{
    with_policy(s.cache & NT_COMB_LD, s.cache & NT_COMB_ST, [&](auto l, auto st) {
        combine_units_t<BF16, K, WAVE, decltype(l)::value, decltype(st)::value, false, false>(y, gates, out, p.pos_final, s, nullptr, nullptr);
    });
}

template <bool BF16, int NV>
__global__ __launch_bounds__(kMoverThreads) void combine_pf_kernel(const u32x4 *__restrict__ y,
                                                                   const float *__restrict__ gates,
                                                                   u32x4 *__restrict__ out, PlanPtrs p, Shape s)
{
    with_policy(s.cache & NT_COMB_LD, s.cache & NT_COMB_ST, [&](auto l, auto st) {
        combine_rows_pf_t<BF16, NV, decltype(l)::value, decltype(st)::value>(y, gates, out, p.pos_final, s, 0, s.T,
                                                                             blockIdx.x, gridDim.x);
    });
}

template <bool BF16, int NV>
__global__ __launch_bounds__(kMoverThreads) void combine_kernel(const u32x4 *__restrict__ y,
                                                                const float *__restrict__ gates,
                                                                u32x4 *__restrict__ out, PlanPtrs p, Shape s)
{
    with_policy(s.cache & NT_COMB_LD, s.cache & NT_COMB_ST, [&](auto l, auto st) {
        combine_rows_t<BF16, NV, decltype(l)::value, decltype(st)::value>(y, gates, out, p.pos_final, s, 0, s.T,
                                                                          blockIdx.x, gridDim.x);
    });
}

// ---- small problems: routing, plan and rows in one launch
//
// A step of a few hundred tokens is three launches that wait for each other, each a chain of latencies (routing 5 us, plan and rows
// 5, combine 4 for 64 tokens on 8 experts) with hardly any work in it.  Here every workgroup routes ALL tokens for itself, which
// takes no longer than routing some of them as long as one pass of its threads covers them, and so knows every row without waiting
// for another workgroup: the choices are bit masks per expert over the tokens, a pair's rank is a count of the bits before its
// token, and what the units before send is a count of the bits before their first token.  Three workgroups write the
// positions, the other plan tables, and the choices with the gates, the others each move threads / lanes-per-row rows.
// WHAT: tables and gates alone (three workgroups), the rows as well, or the whole step with identity experts, in which a token's output is
// added up from its row while that is in registers (the rows of its choices are copies of it) instead of being read back from FINAL.
// What bounds it: a chain of latencies (kernel arguments, logits, choices, scans, positions, stores; of 15000 clocks the sums of the
// outputs took 7000 when each choice was a product of its own).  Measured on MI355X: 64 tokens, 8 experts, top-2, 4096 elements 12.8 us
// of GPU time in three launches, 7.7 in one, now 6.4; where the lines lie stands at small_lanes.
enum SmallWhat { SMALL_ROUTE = 0, SMALL_PLACE = 1, SMALL_COMBINE = 2 };

// Dynamic LDS of the kernel (byte offsets; made on the host: in every workgroup it is a chain of a hundred scalar instructions).
// NW: words of 64 tokens.
struct SmallLds {
    int NW, sel, top, mask, w, den, gate, pre, total, off, kpre, base, stage, bytes;
};
inline SmallLds small_lds(int T, int E, int k, int U)
{
    SmallLds l;
    l.NW = (T + kWave - 1) / kWave;
    int64_t at = 0;
    auto take = [&](int64_t n) {
        const int64_t o = (at + 7) & ~(int64_t)7;
        at = o + n;
        return (int)o;
    };
    l.sel = take((int64_t)T * k * 4);
    l.top = take((int64_t)T * k * 4);
    l.mask = take((int64_t)E * l.NW * 8);
    l.w = take((int64_t)T * k * 8);
    l.den = take((int64_t)T * 8);
    l.gate = take((int64_t)T * k * 4);
    l.pre = take((int64_t)E * l.NW * 4);
    l.total = take((int64_t)E * 4);
    l.off = take((int64_t)E * 4);
    l.kpre = take((int64_t)E * 4);
    l.base = take(((int64_t)U + 1) * 4);
    l.stage = take((int64_t)U * E * 4);
    l.bytes = (int)at;
    return l;
}

template <int L, int NE>
__global__ __launch_bounds__(1024) void small_step_kernel(const float *__restrict__ logits, const u32x4 *__restrict__ x,
                                                          int32_t *__restrict__ topk_idx, float *__restrict__ gates,
                                                          u32x4 *__restrict__ stage, u32x4 *__restrict__ fin, u32x4 *__restrict__ out,
                                                          PlanPtrs p, Shape s, SmallLds lds, int what, int bf16)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned long long s_alive[16];
    const int T = s.T, E = s.E, k = s.k, U = s.U, Tu = s.Tu, C = s.C, vpr = s.vpr, lpr = s.lpr;
    int *s_sel = reinterpret_cast<int *>(smem + lds.sel);
    float *s_top = reinterpret_cast<float *>(smem + lds.top);
    unsigned long long *s_mask = reinterpret_cast<unsigned long long *>(smem + lds.mask);      // [word][expert]
    double *s_w = reinterpret_cast<double *>(smem + lds.w), *s_den = reinterpret_cast<double *>(smem + lds.den);
    float *s_gate = reinterpret_cast<float *>(smem + lds.gate);                                 // of this workgroup's rows
    int *s_pre = reinterpret_cast<int *>(smem + lds.pre), *s_total = reinterpret_cast<int *>(smem + lds.total);
    int *s_off = reinterpret_cast<int *>(smem + lds.off), *s_kpre = reinterpret_cast<int *>(smem + lds.kpre);
    int *s_base = reinterpret_cast<int *>(smem + lds.base), *s_stage = reinterpret_cast<int *>(smem + lds.stage);
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & (kWave - 1), wave = tid >> 6, nwaves = nthr >> 6;
    const int NW = lds.NW;
    enum { PAIRS = 0, TABLES = 1, GATES = 2, ROWS = 3 };           // what workgroups 0, 1, 2 and the others write
    const int role = blockIdx.x < ROWS ? (int)blockIdx.x : ROWS;
    const bool mover = role == ROWS;

    // the first pass of this thread's row is on its way while the tokens are routed
    const int lshift = __builtin_ctz(lpr), rows = nthr >> lshift, sub = tid >> lshift, rl = tid - (sub << lshift);
    const int t0 = mover ? ((int)blockIdx.x - ROWS) * rows : 0, t1 = mover ? min(t0 + rows, T) : T;
    const int t = t0 + sub;
    const bool have = mover && t < t1;
    const u32x4 *src = x + (size_t)(have ? t : 0) * vpr;
    u32x4 val[kVecInFlight];
#pragma unroll
    for (int q = 0; q < kVecInFlight; ++q)
        if (have && rl + q * lpr < vpr) val[q] = src[rl + q * lpr];

    for (int i = tid; i < E * NW; i += nthr) s_mask[i] = 0ull;
    if (tid < 16) s_alive[tid] = 0ull;
    const bool weighted = role == GATES || (mover && what == SMALL_COMBINE);
    double *den = s.renorm || !weighted ? nullptr : s_den;
    route_select<L, NE>(logits, T, E, k, s_sel, s_top, s_mask, 1, E, den);
    __syncthreads();
    // Gates of all tokens, or of this workgroup's own: by the last waves first, beside the scans, which are the first waves' work.
    const int rtid = nthr - 1 - tid;
    if (weighted) route_weights(t1 - t0, k, s_top + t0 * k, s_w + t0 * k, s.by_k1, rtid, nthr);
    for (int e = tid; e < E; e += nthr) {
        int c = 0;
        for (int w = 0; w < NW; ++w) {
            s_pre[w * E + e] = c;
            c += __popcll(s_mask[w * E + e]);
        }
        s_total[e] = c;
    }
    __syncthreads();
    if (weighted) {
        route_gates(t1 - t0, k, s_w + t0 * k, den ? den + t0 : nullptr, s.by_k, rtid, nthr, [&](int idx, float g) {
            if (mover) {
                s_gate[idx] = g;
            } else {
                gates[idx] = g;
                topk_idx[idx] = s_sel[idx];
            }
        });
        if (role == GATES) return;
    }
    // pairs of expert e among the tokens before token `pos`
    auto before = [&](int e, int pos) {
        const int w = pos >> 6;
        return w >= NW ? s_total[e] : s_pre[w * E + e] + __popcll(s_mask[w * E + e] & ((1ull << (pos & 63)) - 1ull));
    };
    // first rows: of the experts in FINAL (wave 0), of the blocks of the units that this workgroup needs in STAGE (wave 1 first);
    // the counters of all experts are read before the first scan
    constexpr int CH = 256 / kWave;
    if (wave == 0) {
        int kp[CH], carry = 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) kp[c] = c * kWave + lane < E ? min(s_total[c * kWave + lane], C) : 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (c * kWave >= E) break;
            const int e = c * kWave + lane, incl = wave_inclusive_scan(kp[c]);
            if (e < E) {
                s_kpre[e] = carry + incl - kp[c];
                s_off[e] = s.padded ? e * C : carry + incl - kp[c];
            }
            carry += wave_total(incl);
        }
        if (lane == 0) s_base[U] = carry;
    }
    const int u_end = (t1 - 1) / s.by_Tu;
    for (int u = t0 / s.by_Tu + (wave == 0 ? nwaves - 1 : wave - 1); u <= u_end; u += nwaves) {
        int lo[CH], nu[CH], sum = 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int e = c * kWave + lane;
            lo[c] = nu[c] = 0;
            if (c * kWave < E && e < E) {
                lo[c] = min(before(e, u * Tu), C);
                nu[c] = min(before(e, (u + 1) * Tu), C) - lo[c];
            }
            sum += lo[c];
        }
        int carry = wave_total(wave_inclusive_scan(sum));
        if (lane == 0) s_base[u] = carry;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (c * kWave >= E) break;
            const int e = c * kWave + lane, incl = wave_inclusive_scan(nu[c]);
            if (e < E) s_stage[u * E + e] = carry + incl - nu[c];
            carry += wave_total(incl);
        }
    }
    __syncthreads();
    // rows of choice j of token tok; false if it is dropped.  All earlier pairs of a kept one are kept.
    auto place = [&](int tok, int j, int &pf, int &ps) {
        const int e = s_sel[tok * k + j], u = tok / s.by_Tu;
        const int r = before(e, tok), first = s_off[e], block = s_stage[u * E + e] - before(e, u * Tu);
        const bool ok = r < C;
        pf = ok ? first + r : -1;
        ps = ok ? block + r : -1;
        return ok;
    };

    if (role == PAIRS) {
        for (int i = tid; i < T * k; i += nthr) {
            const int tok = i / s.by_k;
            int pf, ps;
            if (place(tok, i - tok * k, pf, ps)) {
                p.row_map[ps] = pf;
                atomicOr(&s_alive[tok >> 6], 1ull << (tok & 63));
            }
            p.pos_final[i] = pf;
            p.pos_stage[i] = ps;
        }
        __syncthreads();
        if (tid == 0) {
            int alive = 0;
            for (int w = 0; w < NW; ++w) alive += __popcll(s_alive[w]);
            p.meta[META_ALIVE] = alive;
        }
        return;
    }
    if (role == TABLES) {
        const int R = s_base[U], E_loc = E / s.ep;
        for (int i = tid; i < U * E; i += nthr) {
            const int u = i / s.by_E, e = i - u * E, lo = min(before(e, u * Tu), C);
            p.n[i] = min(before(e, (u + 1) * Tu), C) - lo;
            p.stage_off[i] = s_stage[i];
            p.unit_base[i] = s_off[e] + lo;
        }
        for (int e = tid; e < E; e += nthr) {
            p.counts[e] = s_total[e];
            p.kept[e] = min(s_total[e], C);
            p.offsets[e] = s_off[e];
            p.kept_prefix[e] = s_kpre[e];
        }
        for (int u = tid; u <= U; u += nthr) p.unit_rows[u] = s_base[u];
        for (int i = tid; i < U * s.ep; i += nthr) {        // rows for EP rank d = STAGE span of its experts inside the unit
            const int u = i / s.by_ep, d = i - u * s.ep;
            p.send_rows[i] = (d + 1 < s.ep ? s_stage[u * E + (d + 1) * E_loc] : s_base[u + 1]) - s_stage[u * E + d * E_loc];
        }
        if (tid == 0) {
            p.offsets[E] = s.padded ? E * C : R;
            p.kept_prefix[E] = R;
            p.meta[META_R] = R;
            p.meta[META_C] = C;
            p.meta[META_FINAL_ROWS] = s.padded ? E * C : R;
        }
        return;
    }

    // One 16-byte vector of the output: the gate-weighted sum over the kept choices, in order, of copies of the row's vector.
    // each(add): add(gate) for every kept choice
    auto combined_as = [&](auto bf, u32x4 v, auto each) {
        constexpr bool BF16 = decltype(bf)::value;
        constexpr int NF = BF16 ? 8 : 4;
        double val[NF], acc[NF];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (BF16) {
                val[2 * c] = bf16_lo(v[c]);
                val[2 * c + 1] = bf16_hi(v[c]);
            } else {
                val[c] = (double)__uint_as_float(v[c]);
            }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = 0.0;
        each([&](double g) {
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f] = __builtin_fma(g, val[f], acc[f]);
        });
        u32x4 o;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (BF16) o[c] = f64_to_bf16_rne(acc[2 * c]) | (f64_to_bf16_rne(acc[2 * c + 1]) << 16);
            else o[c] = __float_as_uint((float)acc[c]);
        }
        return o;
    };
    auto combined = [&](u32x4 v, auto each) {
        return bf16 ? combined_as(std::true_type{}, v, each) : combined_as(std::false_type{}, v, each);
    };
    const int gbase = lpr >= kWave ? 0 : (lane & ~(lpr - 1)), gl = lane - gbase;
    u32x4 *dst = out + (size_t)(have ? t : 0) * vpr;
    if (k <= lpr) {
        int ps = -1, pf = -1;
        float my_g = 0.f;
        const bool ok = have && gl < k && place(t, gl, pf, ps);
        if (ok && what == SMALL_COMBINE) my_g = s_gate[sub * k + gl];
        const unsigned int kmask = k >= 32 ? 0xffffffffu : ((1u << k) - 1u);
        const unsigned int kept = (unsigned int)(__ballot(ok) >> gbase) & kmask;
        // All rows being copies of one, the sum of products is the product with the sum of the gates, and to the last bit of 64 where no
        // addition of the combine's chain but its last one can round.  A product of a gate and a bf16 element has 32 bits, so that sums of
        // up to 32 of them are exact in 53 bits if the gates' exponents are at most 16 apart, and then so is the sum of the gates.  Of
        // two products, in fp32, too, only the last addition rounds, and their gates' sum is exact with exponents up to 28 apart.
        // Otherwise, and with a gate of zero, which an infinite activation would tell from no choice, product after product.  Rows that
        // whole waves share have their destinations in scalar registers.
        auto move = [&](auto whole_waves) {
            constexpr bool WAVE = decltype(whole_waves)::value;
            const unsigned int mine = WAVE ? (unsigned int)__builtin_amdgcn_readfirstlane((int)kept) : kept;
            auto of = [&](int v, int j) { return WAVE ? __builtin_amdgcn_readlane(v, j) : __shfl(v, gbase + j, kWave); };
            double gate_sum = 0.0;
            bool summed = bf16 || k <= 2;
            if (what == SMALL_COMBINE && summed) {
                uint32_t most = 0, least = ~0u;                    // gates are positive: their bits are in their order
                for (unsigned int rem = mine; rem; rem &= rem - 1) {
                    const int bits = of(__float_as_int(my_g), __builtin_ctz(rem));
                    most = max(most, (uint32_t)bits);
                    least = min(least, (uint32_t)bits);
                    gate_sum += (double)__int_as_float(bits);
                }
                summed = least != 0 && (int)(most >> 23) - (int)(least >> 23) <= (k <= 2 ? 28 : 16);
            }
            for (int vbase = 0; vbase < vpr; vbase += lpr * kVecInFlight) {
                const int v0 = vbase + rl;
                if (vbase != 0) {
#pragma unroll
                    for (int q = 0; q < kVecInFlight; ++q)
                        if (have && v0 + q * lpr < vpr) val[q] = src[v0 + q * lpr];
                }
                for (unsigned int rem = mine; rem; rem &= rem - 1) {
                    const int j = __builtin_ctz(rem);
                    u32x4 *ds = stage + (size_t)of(ps, j) * vpr, *df = fin + (size_t)of(pf, j) * vpr;
#pragma unroll
                    for (int q = 0; q < kVecInFlight; ++q)
                        if (v0 + q * lpr < vpr) {
                            st16<true>(ds + v0 + q * lpr, val[q]);
                            df[v0 + q * lpr] = val[q];
                        }
                }
                if (what == SMALL_COMBINE) {
#pragma unroll
                    for (int q = 0; q < kVecInFlight; ++q) {
                        if (vbase + q * lpr >= vpr) break;
                        const u32x4 o = combined(val[q], [&](auto add) {
                            if (summed) {
                                if (mine) add(gate_sum);
                            } else {
                                for (unsigned int rem = mine; rem; rem &= rem - 1) add((double)__int_as_float(of(__float_as_int(my_g), __builtin_ctz(rem))));
                            }
                        });
                        if (have && v0 + q * lpr < vpr) st16<true>(dst + v0 + q * lpr, o);
                    }
                }
            }
        };
        if (lpr >= kWave) move(std::true_type{});
        else move(std::false_type{});
    } else if (have) {
        // fewer lanes per row than choices: rows of at most 256 bytes, one vector per lane
        for (int j = 0; j < k; ++j) {
            int pf, ps;
            if (place(t, j, pf, ps) && rl < vpr) {
                st16<true>(stage + (size_t)ps * vpr + rl, val[0]);
                fin[(size_t)pf * vpr + rl] = val[0];
            }
        }
        if (what == SMALL_COMBINE && rl < vpr) {
            const u32x4 o = combined(val[0], [&](auto add) {
                for (int j = 0; j < k; ++j) {
                    int pf, ps;
                    if (place(t, j, pf, ps)) add((double)s_gate[sub * k + j]);
                }
            });
            st16<true>(dst + rl, o);
        }
    }
    if (s.padded) pad_rows(fin, s_kpre, s_total, s_base[U], s, (int)blockIdx.x - ROWS, (int)gridDim.x - ROWS, nthr);
}

// The gather as a pass of its own: the STAGE rows of units [u0, u1) (one contiguous range, read from the
// device table) copied unchanged into a second buffer.
__device__ __forceinline__ void allgather_rows(const u32x4 *__restrict__ stage, u32x4 *__restrict__ gathered,
                                               const PlanPtrs &p, const Shape &s, int u0, int u1, int wg, int nwg)
{
    int r0 = p.unit_rows[u0], r1 = p.unit_rows[u1];
    if (r0 < 0) r0 = 0;
    if (r1 > s.max_rows) r1 = s.max_rows;
    if (r1 <= r0) return;
    const size_t first = (size_t)r0 * s.vpr, nvec = (size_t)(r1 - r0) * s.vpr;
    const size_t stride = (size_t)nwg * kMoverThreads * kVecInFlight;
    for (size_t base = (size_t)wg * kMoverThreads * kVecInFlight + threadIdx.x; base < nvec; base += stride) {
        u32x4 val[kVecInFlight];
#pragma unroll
        for (int q = 0; q < kVecInFlight; ++q)
            if (base + (size_t)q * kMoverThreads < nvec) val[q] = ld16<true>(stage + first + base + (size_t)q * kMoverThreads);
#pragma unroll
        for (int q = 0; q < kVecInFlight; ++q)
            if (base + (size_t)q * kMoverThreads < nvec) st16<false>(gathered + first + base + (size_t)q * kMoverThreads, val[q]);
    }
}

__global__ __launch_bounds__(kMoverThreads) void allgather_kernel(const u32x4 *__restrict__ stage,
                                                                  u32x4 *__restrict__ gathered, PlanPtrs p, Shape s,
                                                                  int u0, int u1)
{
    allgather_rows(stage, gathered, p, s, u0, u1, blockIdx.x, gridDim.x);
}

// The paper's third transform (paragraph "AllGather and D2D copy Pipelining", Fig. 8): while the D2D copy
// places chunk j from the gathered buffer, the gather of chunk j+1 already runs.  One grid, two jobs in
// disjoint, interleaved workgroups: the first n_gather_wg gather units [gu0, gu1) (STAGE -> gathered), the
// others copy units [cu0, cu1) from `gathered` to their index offsets in FINAL.  The two ranges are different
// chunks, so the jobs touch disjoint rows of `gathered`.
__global__ __launch_bounds__(kMoverThreads) void allgather_regather_kernel(const u32x4 *__restrict__ stage,
                                                                           u32x4 *gathered, u32x4 *__restrict__ fin,
                                                                           PlanPtrs p, Shape s, int gu0, int gu1,
                                                                           int cu0, int cu1, int n_gather_wg)
{
    const int n_copy_wg = gridDim.x - n_gather_wg;
    const int bid = blockIdx.x;
    const int pairs = n_gather_wg < n_copy_wg ? n_gather_wg : n_copy_wg;
    bool is_gather;
    int idx;
    if (bid < 2 * pairs) {
        is_gather = (bid & 1) == 0;
        idx = bid >> 1;
    } else {
        is_gather = n_gather_wg > n_copy_wg;
        idx = bid - pairs;
    }
    if (is_gather) {
        allgather_rows(stage, gathered, p, s, gu0, gu1, idx, n_gather_wg);
    } else {
        regather_rows(gathered, fin, p, s, p.unit_rows[cu0], p.unit_rows[cu1], idx, n_copy_wg);
        if (s.padded && cu0 == 0) pad_rows(fin, p, s, idx, n_copy_wg);
    }
}

// ---- the second AllToAll, mirrored: y (FINAL layout) -> unit-major layout -> token order, slice by slice

__global__ __launch_bounds__(kMoverThreads) void unregather_kernel(const u32x4 *__restrict__ y,
                                                                   u32x4 *__restrict__ y_stage, PlanPtrs p, Shape s,
                                                                   int u0, int u1)
{
    unregather_rows(y, y_stage, p.row_map, s, p.unit_rows[u0], p.unit_rows[u1], blockIdx.x, gridDim.x);
}

// One grid, up to two jobs in disjoint, interleaved workgroups: the unit-major rows of units [u0, u1)
// are fetched back from y (skipped if u0 >= u1) while the tokens [t0, t0+nt) of the slice before are
// combined from rows fetched by the previous launch (skipped if nt == 0).
// PF: the software-pipelined scale-add (three or more choices per token), as in combine_pf_kernel.
template <bool BF16, int NV, bool PF = false>
__global__ __launch_bounds__(kMoverThreads) void unregather_combine_kernel(const u32x4 *__restrict__ y,
                                                                           u32x4 *y_stage,
                                                                           const float *__restrict__ gates,
                                                                           u32x4 *__restrict__ out, PlanPtrs p,
                                                                           Shape s, int u0, int u1, int t0, int nt,
                                                                           int n_unreg_wg)
{
    const int n_comb_wg = gridDim.x - n_unreg_wg;
    const int bid = blockIdx.x;
    const int pairs = n_unreg_wg < n_comb_wg ? n_unreg_wg : n_comb_wg;
    bool is_unreg;
    int idx;
    if (bid < 2 * pairs) {
        is_unreg = (bid & 1) == 0;
        idx = bid >> 1;
    } else {
        is_unreg = n_unreg_wg > n_comb_wg;
        idx = bid - pairs;
    }
    if (is_unreg) {
        if (u0 < u1) unregather_rows(y, y_stage, p.row_map, s, p.unit_rows[u0], p.unit_rows[u1], idx, n_unreg_wg);
    } else if (nt > 0) {
        with_policy(s.cache & NT_COMB_LD, s.cache & NT_COMB_ST, [&](auto l, auto st) {
            if (PF)
                combine_rows_pf_t<BF16, NV, decltype(l)::value, decltype(st)::value>(y_stage, gates, out, p.pos_stage, s,
                                                                                     t0, nt, idx, n_comb_wg);
            else
                combine_rows_t<BF16, NV, decltype(l)::value, decltype(st)::value>(y_stage, gates, out, p.pos_stage, s, t0,
                                                                                  nt, idx, n_comb_wg);
        });
    }
}

// The whole return path in one pass: for every token the rows of its kept choices are read from y once, stored to their
// places in the unit-major layout and added up, instead of being fetched into that layout and read back from there
// (2R + T rows instead of 3R + T).  Same rows, same order of additions.  PF as above.
template <bool BF16, int NV, bool PF>
__global__ __launch_bounds__(kMoverThreads) void return_kernel(const u32x4 *__restrict__ y, u32x4 *__restrict__ y_stage,
                                                               const float *__restrict__ gates, u32x4 *__restrict__ out,
                                                               PlanPtrs p, Shape s)
{
    with_policy3(s.cache & NT_REG_LD, s.cache & NT_COMB_ST, s.cache & NT_REG_ST, [&](auto l, auto st, auto kp) {
        constexpr bool NTL = decltype(l)::value, NTS = decltype(st)::value, NTK = decltype(kp)::value;
        if (PF)
            combine_rows_pf_t<BF16, NV, NTL, NTS, true, NTK>(y, gates, out, p.pos_final, s, 0, s.T, blockIdx.x, gridDim.x,
                                                             y_stage, p.pos_stage);
        else
            combine_rows_t<BF16, NV, NTL, NTS, true, NTK>(y, gates, out, p.pos_final, s, 0, s.T, blockIdx.x, gridDim.x,
                                                          y_stage, p.pos_stage);
    });
}

template <bool BF16, int K, bool WAVE>
__global__ __launch_bounds__(kMoverThreads) void return_units_kernel(const u32x4 *__restrict__ y, u32x4 *__restrict__ y_stage,
                                                                     const float *__restrict__ gates, u32x4 *__restrict__ out, PlanPtrs p,
                                                                     Shape s)
{
    with_policy3(s.cache & NT_REG_LD, s.cache & NT_COMB_ST, s.cache & NT_REG_ST, [&](auto l, auto st, auto kp) {
        combine_units_t<BF16, K, WAVE, decltype(l)::value, decltype(st)::value, true, decltype(kp)::value>(y, gates, out, p.pos_final, s, y_stage,
                                                                                                          p.pos_stage);
    });
}

// --------------------------------------------------------- gate projection
//
// logits[t][e] = sum_h x[t][h] * w[e][h]  (section "MoE": the gate is a linear layer ahead of softmax and TopK).
// The contraction is read-bound on x: every element of x is used E times, far below what the matrix cores
// need to be busy, so the kernel is laid out for the x stream and uses MFMA to keep the arithmetic off the
// critical path at large E.
//
// bf16: a workgroup of 8 waves owns 32*MT tokens and all experts.  The hidden axis is cut into steps of KS
// elements; a step's tile (the tokens' rows, then the experts' rows, KS*2 bytes each) is fetched with 16-byte
// loads whose lanes run along a row, so every load instruction covers whole cache lines, parked in registers
// while the previous tile is multiplied, and then laid into LDS with a 16-byte pad per row.  The 32x32x16 bf16
// MFMA wants, from lane l, row l%32 and the 8 k-values 8*(l/32)..+7 of A and the same of B (column l%32); those
// fragments are single 16-byte LDS reads.  The k-slices of a step are dealt round robin to the waves, each wave
// carries MT*NT accumulator tiles (element i of lane l = row (i/4)*8 + (l/32)*4 + i%4, column l%32), and the
// waves' partial tiles are added through LDS in a fixed order at the end, so results are reproducible.

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kGateThreads = 512;
constexpr int kGateWaves = kGateThreads / 64;

template <int MT, int NT, int KS>
struct GateTile {
    static constexpr int kTokens = 32 * MT;
    static constexpr int kPiecesPerRow = KS / 8;                 // 16-byte pieces of one row of a step
    static constexpr int kRowStride = KS * 2 + 16;               // bytes in LDS
    static constexpr int kLoads = (32 * (MT + NT) * kPiecesPerRow + kGateThreads - 1) / kGateThreads;
    static constexpr int kLoadsX = kTokens * kPiecesPerRow / kGateThreads;      // of them from rows of x, by every thread
    static_assert(kTokens * kPiecesPerRow % kGateThreads == 0, "gate: a load is of x or of the weights for all threads");
    static constexpr int kTiles = MT * NT;
    // partial tiles of several waves side by side in 64 KiB; waves sharing a slot add one after the other
    static constexpr int kSlots = kTiles > 16 ? 1 : (16 / kTiles) < kGateWaves ? (16 / kTiles) : kGateWaves;
    static constexpr int kRounds = kGateWaves / kSlots;
    static_assert(kSlots * kRounds == kGateWaves, "gate reduction: waves must fill the slots evenly");
    static_assert((KS & (KS - 1)) == 0 && KS >= 64, "gate: KS must be a power of two");
    // `reduce`: the kernel variant that adds the waves' partial tiles through LDS at the end
    static constexpr size_t lds_bytes(int E, bool reduce)
    {
        const size_t tile = (size_t)(kTokens + E) * kRowStride, red = reduce ? (size_t)kSlots * kTiles * 4096 : 0;
        return tile > red ? tile : red;
    }
};

// DEEP: two tiles in flight instead of one (not where the accumulators leave no registers for it).
// SPLIT (needs MT*NT = number of waves): instead of dealing the k-slices, every wave owns one 32x32 output tile
// and walks all k-slices of it: one accumulator tile per wave, which leaves registers for larger tiles in
// flight, and no reduction across waves at the end.
// STREAM: x is requested as streaming.
template <int MT, int NT, int KS, bool DEEP, bool SPLIT, bool STREAM>
__global__ __launch_bounds__(kGateThreads) void gate_bf16_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                                 float *__restrict__ logits, int64_t T, int H, int E)
{
    using G = GateTile<MT, NT, KS>;
    extern __shared__ __align__(16) unsigned char gate_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 31, g = lane >> 5;
    const int64_t t0 = (int64_t)blockIdx.x * G::kTokens;
    const int cpr = H / 8;                                        // 16-byte pieces per row in memory
    const int pieces = (G::kTokens + E) * G::kPiecesPerRow;       // pieces of one tile
    const int nsteps = (cpr + G::kPiecesPerRow - 1) / G::kPiecesPerRow;
    const u32x4 zero = {0u, 0u, 0u, 0u};

    // Two tiles are kept in flight.  Every load is issued unconditionally, from a clamped in-bounds address, and
    // what lies outside the matrices is replaced by zeros when the piece is laid into LDS: the number of loads
    // between a tile's issue and its use is then fixed, and the wait before the use lets the younger tile's
    // loads stay outstanding.
    auto piece_ok = [&](int p, int step, int &row, int &c) {
        row = p / G::kPiecesPerRow;
        c = step * G::kPiecesPerRow + p % G::kPiecesPerRow;
        return p < pieces && c < cpr && (row >= G::kTokens || t0 + row < T);
    };
    auto fetch = [&](u32x4(&pre)[G::kLoads], int step) {
#pragma unroll
        for (int q = 0; q < G::kLoads; ++q) {
            int row, c;
            const bool ok = piece_ok(tid + q * kGateThreads, step, row, c);
            const u32x4 *src = x;
            if (ok) src = (row < G::kTokens) ? x + (t0 + row) * cpr + c : w + (int64_t)(row - G::kTokens) * cpr + c;
            if (STREAM && q < G::kLoadsX) pre[q] = ld16<true>(src);      // (as a choice of two values both would be plain loads)
            else pre[q] = *src;
        }
    };
    auto stage = [&](const u32x4(&pre)[G::kLoads], int step) {
        __syncthreads();                                          // the previous tile has been read by every wave
#pragma unroll
        for (int q = 0; q < G::kLoads; ++q) {
            const int p = tid + q * kGateThreads;
            int row, c;
            const bool ok = piece_ok(p, step, row, c);
            if (p < pieces)
                *reinterpret_cast<u32x4 *>(gate_lds + (size_t)row * G::kRowStride + (p % G::kPiecesPerRow) * 16) =
                    ok ? pre[q] : zero;
        }
        __syncthreads();
    };

    // SPLIT: wave v owns column tile v % NT and the row tiles v / NT + i * (waves / NT)
    constexpr int kPerWave = G::kTiles / kGateWaves, kRowTileStep = kGateWaves / NT;
    static_assert(!SPLIT || (kGateWaves % NT == 0 && kPerWave >= 1 && kPerWave * kRowTileStep == MT),
                  "gate: the output tiles must divide evenly among the waves");
    constexpr int kAcc = SPLIT ? kPerWave : G::kTiles;
    f32x16 acc[kAcc];
#pragma unroll
    for (int i = 0; i < kAcc; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    auto multiply = [&]() {
        if constexpr (SPLIT) {
            const int n = (wave % NT) * 32 + m;
            const unsigned char *pa = gate_lds + (size_t)((wave / NT) * 32 + m) * G::kRowStride + g * 16;
            const unsigned char *pb = gate_lds + (size_t)(G::kTokens + (n < E ? n : 0)) * G::kRowStride + g * 16;
#pragma unroll 4
            for (int ks = 0; ks < KS / 16; ++ks) {
                bf16x8 b = *reinterpret_cast<const bf16x8 *>(pb + ks * 32);
                if (n >= E) b = __builtin_bit_cast(bf16x8, zero);
#pragma unroll
                for (int i = 0; i < kAcc; ++i) {
                    const bf16x8 a =
                        *reinterpret_cast<const bf16x8 *>(pa + (size_t)i * kRowTileStep * 32 * G::kRowStride + ks * 32);
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i], 0, 0, 0);
                }
            }
            return;
        }
        for (int ks = wave; ks < KS / 16; ks += kGateWaves) {
            const int off = ks * 32 + g * 16;
            bf16x8 a[MT], b[NT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                a[mt] = *reinterpret_cast<const bf16x8 *>(gate_lds + (size_t)(mt * 32 + m) * G::kRowStride + off);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int n = nt * 32 + m;
                b[nt] = __builtin_bit_cast(bf16x8, zero);
                if (n < E)
                    b[nt] = *reinterpret_cast<const bf16x8 *>(gate_lds + (size_t)(G::kTokens + n) * G::kRowStride + off);
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt * NT + nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mt], b[nt], acc[mt * NT + nt], 0, 0, 0);
        }
    };

    if constexpr (DEEP) {
        u32x4 pre0[G::kLoads], pre1[G::kLoads];
        fetch(pre0, 0);
        fetch(pre1, 1);                                           // past the last step: clamped loads, never used
        for (int step = 0; step < nsteps; step += 2) {
            stage(pre0, step);
            fetch(pre0, step + 2);
            multiply();
            if (step + 1 < nsteps) {
                stage(pre1, step + 1);
                fetch(pre1, step + 3);
                multiply();
            }
        }
    } else {
        u32x4 pre0[G::kLoads];
        fetch(pre0, 0);
        for (int step = 0; step < nsteps; ++step) {
            stage(pre0, step);
            fetch(pre0, step + 1);
            multiply();
        }
    }

    if constexpr (SPLIT) {
        // element j of this lane: row (j/4)*8 + g*4 + j%4, column m of the wave's own tile
        const int n = (wave % NT) * 32 + m;
#pragma unroll
        for (int i = 0; i < kAcc; ++i)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int64_t t = t0 + (wave / NT + i * kRowTileStep) * 32 + (j >> 2) * 8 + g * 4 + (j & 3);
                if (t < T && n < E) logits[t * E + n] = acc[i][j];
            }
        return;
    }
    // partial tiles -> LDS [slot][tile][row][col]
    float *red = reinterpret_cast<float *>(gate_lds);
    const int slot = wave % G::kSlots, round = wave / G::kSlots;
    __syncthreads();                                              // the last tile is no longer needed
    for (int r = 0; r < G::kRounds; ++r) {
        if (round == r) {
#pragma unroll
            for (int i = 0; i < G::kTiles; ++i)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int row = (j >> 2) * 8 + g * 4 + (j & 3);
                    float *q = red + ((slot * G::kTiles + i) * 32 + row) * 32 + m;
                    *q = (r == 0) ? acc[i % kAcc][j] : *q + acc[i % kAcc][j];
                }
        }
        __syncthreads();
    }
    const int64_t rows = (T - t0 < G::kTokens) ? (T - t0) : G::kTokens;
    for (int64_t idx = tid; idx < rows * E; idx += kGateThreads) {
        const int row = (int)(idx / E), n = (int)(idx % E);
        const int tile = (row >> 5) * NT + (n >> 5);
        float sum = 0.f;
#pragma unroll
        for (int sl = 0; sl < G::kSlots; ++sl) sum += red[((sl * G::kTiles + tile) * 32 + (row & 31)) * 32 + (n & 31)];
        logits[t0 * E + idx] = sum;
    }
}

// bf16, at most 8 experts, H <= 8192 and a multiple of 64*NCH: the shapes of the paper's layers.  A tile of 32
// consecutive rows walked in column steps touches memory in short strided runs, which the memory system serves
// well below its streaming rate; here a workgroup reads 8 whole consecutive rows at a time (NCH = 1; halves of
// them if NCH = 2), i.e. one contiguous run of up to 64 KiB.  The 32 MFMA rows are (quarter of the row chunk,
// token) pairs and the 32 columns (quarter, expert) pairs: row qk*8+tok holds x[tok][quarter qk], column qk'*8+e
// holds w[e][quarter qk'], so the diagonal blocks qk = qk' of the accumulator carry the four quarter sums of
// every (token, expert) logit, and the off-diagonal blocks, which would be idle columns anyway with so few
// experts, are ignored.  The weights never change, so a persistent workgroup keeps its B fragments in registers
// for the whole launch: wave v owns steps v, v+8, ... of each quarter.  The sums over chunks (in the accumulator) and
// over waves and quarters (through LDS, by 64 threads, one tile later) run in a fixed order: results are reproducible.
// (A variant with direct-to-LDS loads, three tile buffers and two tiles in flight measured the same within 3 % on
// MI355X and is not kept.)

constexpr int kGateSmallTokens = 8;          // rows of one tile
constexpr int kGateSmallExperts = 8;         // expert slots of one quarter

__host__ __device__ constexpr int gate_small_quarter_stride(int chunk) { return chunk / 2 + 128; }      // bytes
__host__ __device__ constexpr int gate_small_row_stride(int chunk) { return 4 * gate_small_quarter_stride(chunk) + 16; }
__host__ __device__ constexpr size_t gate_small_lds_bytes(int chunk, int threads)
{
    // the tile, then two buffers of partial sums [wave][quarter][token][expert]
    return (size_t)kGateSmallTokens * gate_small_row_stride(chunk) +
           2 * sizeof(float) * (threads / 64) * 4 * kGateSmallTokens * kGateSmallExperts;
}

// NCH chunks per row, THREADS per workgroup, MAXCHUNK = most elements of a row in LDS at a time
template <int NCH, int THREADS, int MAXCHUNK>
__global__ __launch_bounds__(THREADS) void gate_small_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                             float *__restrict__ logits, int64_t T, int H, int E,
                                                             int64_t ngroups)
{
    constexpr int kGateThreads = THREADS, kGateWaves = THREADS / 64;
    constexpr int kGateSmallSteps = MAXCHUNK / 64 / kGateWaves;     // MFMA steps of a chunk per wave, at most
    constexpr int kGateSmallLoads = kGateSmallTokens * MAXCHUNK / 8 / THREADS;
    constexpr int kRedFloats = kGateWaves * 4 * kGateSmallTokens * kGateSmallExperts;
    static_assert(kGateSmallSteps >= 1 && kGateSmallLoads >= 1, "gate_small_kernel: chunk too small for the workgroup");
    extern __shared__ __align__(16) unsigned char gate_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5;
    const int chunk = H / NCH;                       // elements, a multiple of 64
    const int ppr = chunk / 8, ppq = chunk / 32;     // 16-byte pieces per row chunk / per quarter
    const int cpr = H / 8;
    const int QS = gate_small_quarter_stride(chunk), RS = gate_small_row_stride(chunk);
    const int nsteps = chunk / 64;                   // MFMA steps per chunk: a quarter is nsteps*16 elements
    float *red = reinterpret_cast<float *>(gate_lds + (size_t)kGateSmallTokens * RS);
    const u32x4 zero = {0u, 0u, 0u, 0u};

    // This thread's pieces of a tile, fixed for the whole launch: piece p = tid + q*threads is row p / ppr, column
    // p % ppr.  One division per thread; the others follow by stepping (integer division is slow here).
    int piece_row[kGateSmallLoads], piece_col[kGateSmallLoads], piece_lds[kGateSmallLoads];
    {
        const int step_rows = kGateThreads / ppr, step_cols = kGateThreads % ppr;
        int row = tid / ppr, col = tid % ppr;
#pragma unroll
        for (int q = 0; q < kGateSmallLoads; ++q) {
            const bool in_tile = row < kGateSmallTokens;
            const int qk = (col >= ppq ? 1 : 0) + (col >= 2 * ppq ? 1 : 0) + (col >= 3 * ppq ? 1 : 0);
            piece_row[q] = in_tile ? row : -1;
            piece_col[q] = in_tile ? col : 0;
            piece_lds[q] = in_tile ? row * RS + qk * QS + (col - qk * ppq) * 16 : 0;
            row += step_rows;
            col += step_cols;
            if (col >= ppr) {
                col -= ppr;
                ++row;
            }
        }
    }
    // fragment address of this lane at step 0: row lane%8, quarter (lane%32)/8, k-values 8*(lane/32)..+7
    const unsigned char *frag = gate_lds + (size_t)(lane & 7) * RS + (size_t)((lane & 31) >> 3) * QS + g * 16;

    // Loads are issued unconditionally, from clamped addresses, all of a tile before the first use; what lies
    // outside the matrix becomes zeros when the tile is laid into LDS.
    auto fetch = [&](u32x4(&dst)[kGateSmallLoads], const u32x4 *base, int64_t first_row, int64_t row_limit, int c) {
        unsigned ok = 0;
#pragma unroll
        for (int q = 0; q < kGateSmallLoads; ++q) {
            const int64_t r = first_row + piece_row[q];
            const bool live = piece_row[q] >= 0 && r < row_limit;
            dst[q] = *(live ? base + r * cpr + c * ppr + piece_col[q] : base);
            ok |= (live ? 1u : 0u) << q;
        }
        return ok;
    };
    auto lay = [&](const u32x4(&src)[kGateSmallLoads], unsigned ok) {
        __syncthreads();                                          // the previous tile has been read by every wave
#pragma unroll
        for (int q = 0; q < kGateSmallLoads; ++q)
            if (piece_row[q] >= 0)
                *reinterpret_cast<u32x4 *>(gate_lds + piece_lds[q]) = ((ok >> q) & 1u) ? src[q] : zero;
        __syncthreads();
    };

    // weights -> LDS (same layout, expert rows) -> B fragments in registers, while the first tile of x is already
    // on its way
    u32x4 pre[kGateSmallLoads];
    int64_t grp = blockIdx.x;
    unsigned ok = 0;
    bf16x8 bfrag[NCH][kGateSmallSteps];
    {
        u32x4 wpre[kGateSmallLoads];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const unsigned wok = fetch(wpre, w, 0, E, c);
            if (c == NCH - 1) ok = fetch(pre, x, grp * kGateSmallTokens, T, 0);
            lay(wpre, wok);
#pragma unroll
            for (int i = 0; i < kGateSmallSteps; ++i) {
                const int st = wave + i * kGateWaves;
                bfrag[c][i] = __builtin_bit_cast(bf16x8, zero);
                if (st < nsteps) bfrag[c][i] = *reinterpret_cast<const bf16x8 *>(frag + st * 32);
            }
        }
    }

    f32x16 acc;
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.f;

    // The waves' partial sums of a group go to LDS, and 64 threads add them up and store the logits one tile
    // later, behind that tile's barriers: no barrier of its own, and the additions run beside the other waves'
    // MFMAs.  Two buffers, used alternately.
    const int qn = (lane & 31) >> 3;
    int64_t pending = -1;                           // group whose partial sums wait in red[parity]
    int parity = 0;
    auto finish = [&](int64_t done, int buf) {
        if (tid < kGateSmallTokens * kGateSmallExperts) {
            const float *src = red + buf * kRedFloats + tid;      // [wave][quarter][token][expert], tid = token*8 + expert
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < kGateWaves * 4; ++i) sum += src[i * kGateSmallTokens * kGateSmallExperts];
            const int64_t t = done * kGateSmallTokens + (tid >> 3);
            if ((tid & 7) < E && t < T) logits[t * E + (tid & 7)] = sum;
        }
    };

    for (; grp < ngroups; grp += gridDim.x) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            lay(pre, ok);
            // the next tile is in flight during the MFMAs
            ok = (c + 1 < NCH) ? fetch(pre, x, grp * kGateSmallTokens, T, c + 1)
                               : fetch(pre, x, (grp + gridDim.x) * kGateSmallTokens, T, 0);
            if (pending >= 0) {
                finish(pending, parity ^ 1);
                pending = -1;
            }
            // steps past the chunk's end multiply zeros (their B fragments are zero, A is made zero here)
            bf16x8 a[kGateSmallSteps];
#pragma unroll
            for (int i = 0; i < kGateSmallSteps; ++i) {
                const int st = wave + i * kGateWaves;
                a[i] = __builtin_bit_cast(bf16x8, zero);
                if (st < nsteps) a[i] = *reinterpret_cast<const bf16x8 *>(frag + st * 32);
            }
#pragma unroll
            for (int i = 0; i < kGateSmallSteps; ++i)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bfrag[c][i], acc, 0, 0, 0);
        }
        // accumulator element j of this lane: row (j/4)*8 + g*4 + j%4 = (quarter j/4, token g*4 + j%4), column
        // (quarter (lane%32)/8, expert lane%8): only the diagonal blocks, quarter j/4 = quarter of the column, count
        float *dst = red + parity * kRedFloats + ((wave * 4 + qn) * kGateSmallTokens + g * 4) * kGateSmallExperts + (lane & 7);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            dst[i * kGateSmallExperts] = qn == 0 ? acc[i] : qn == 1 ? acc[4 + i] : qn == 2 ? acc[8 + i] : acc[12 + i];
        pending = grp;
        parity ^= 1;
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = 0.f;
    }
    if (pending >= 0) {
        __syncthreads();
        finish(pending, parity ^ 1);
    }
}

// fp32 activations and at most four experts: one wave per token, fp32 fused multiply-adds in four chains per expert (one per
// element of a 16-byte piece) and a shuffle reduction.  Bound by the stream of x and, for few tokens, by a row's latency; a 16 x 16
// tile with a split hidden axis multiplies twelve or more empty experts and waits for their rows.  Measured on MI355X, such tiles and
// this: 512 x 7168, 2 experts 18.3 -> 5.9 us, 4096 x 7168, 3 experts 20.5 -> 17.9, 65536 x 512, 4 experts 44 -> 26; error against 64
// bits at 7168: 2.0e-7 -> 1.2e-7.
template <int NE>
__global__ __launch_bounds__(256) void gate_f32_few_kernel(const float4 *__restrict__ x, const float4 *__restrict__ w,
                                                           float *__restrict__ logits, int64_t T, int vpr)
{
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const float4 *xr = x + t * vpr;
    float acc[NE][4];
#pragma unroll
    for (int j = 0; j < NE; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = 0.f;
    for (int v = lane; v < vpr; v += 64) {
        const float4 xv = xr[v];
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const float4 wv = w[(int64_t)j * vpr + v];
            acc[j][0] = fmaf(xv.x, wv.x, acc[j][0]);
            acc[j][1] = fmaf(xv.y, wv.y, acc[j][1]);
            acc[j][2] = fmaf(xv.z, wv.z, acc[j][2]);
            acc[j][3] = fmaf(xv.w, wv.w, acc[j][3]);
        }
    }
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        float sum = (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0) logits[t * NE + j] = sum;
    }
}

// ------------------------------------------------------------ expert layer
//
// y[r][n] = sum_k x_final[r][k] * w[e][n][k] for the rows r of expert e's range in the expert-major buffer
// (section "Expert Parallel": the experts process the tokens grouped to them between Dispatch and Combine).  A
// grouped GEMM whose group sizes exist only on the device: the ranges come from the plan tables, the launch is
// sized for the worst case and surplus workgroups leave at once.
//
// bf16: a workgroup of 4 waves computes a 128 x 256 tile of y (rows x output features) of one expert; the hidden
// axis goes in steps of 64 elements through registers into LDS (rows padded by 16 bytes, as in the gate kernels).
// The waves form a 2 x 2 grid; a wave owns 64 x 128 = 2 x 4 MFMA tiles (128 accumulator registers), so every A
// fragment read from LDS feeds 4 MFMAs and every B fragment 2.  Workgroups are numbered so that those which run
// together on one XCD (hardware deals consecutive workgroups round robin to the 8 XCDs) are row tiles of the
// same few weight tiles: the weight tile then comes from that XCD's L2 after its first reader.

constexpr int kExpBK = 64;
constexpr int kExpRowStride = kExpBK * 2 + 16;                                  // bytes in LDS
constexpr int kXcds = 8;

// BM x BN: the workgroup's tile of y; its WM x WN waves each own (BM/WM) x (BN/WN).  One LDS buffer, two barriers
// per step.  In use: 128 x 256 with 2 x 2 waves, two workgroups per CU.  Measured and not faster on MI355X (all
// within 5 % of it): 256 x 256 with 8 waves, 256 x 128, two register sets of tiles in flight, two LDS buffers, and
// staggered starts along the hidden axis; the stores of y cost nothing measurable.
template <int BM, int BN, int WM, int WN>
struct ExpertTile {
    static constexpr int kThreads = 64 * WM * WN;
    static constexpr int kRowsPerPass = kThreads / 8;             // tile rows the threads cover with one load each
    static constexpr int kLoads = (BM + BN) / kRowsPerPass;       // 16-byte pieces per thread and step
    static constexpr int kLdsBytes = (BM + BN) * kExpRowStride;
    static constexpr int kMT = BM / WM / 32, kNT = BN / WN / 32;  // MFMA tiles of a wave
    static constexpr int kWgsPerCu = kThreads <= 256 ? 2 : 1;     // what the registers allow
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0 && kExpBK == 64 && BM % kRowsPerPass == 0 &&
                      BN % kRowsPerPass == 0, "expert kernel: tile shape");
};

struct ExpertArgs {
    const int32_t *lo;      // [E] first row of the expert's range
    const int32_t *hi_base; // [E] one past its last row is hi_base[e] + hi_len[e] ...
    const int32_t *hi_len;  // [E] ... or hi_base[e] alone if this is nullptr
    int16_t E;              // one word for three fields: an argument of its own is one more trip to memory in a chain of them
    int8_t spread;          // 1: the short tiles' walks along the hidden axis start at different steps (walk_start)
    int8_t deal;            // the short tiles' numbers go to the XCDs in blocks of 1 << deal
    int32_t H, N, max_rows;
    int64_t stream_from;    // first row of all experts' weights (expert * N + column) that is requested as streaming (kStreamLoad)
                            // where one workgroup reads it
};

// The expert whose tiles include logical tile number L, found without walking the experts one by one (a walk costs
// one dependent table read per expert before the workgroup can start): 64 experts at a time, one per lane, a wave
// scan of their tile counts, a ballot for the first lane whose running total passes L.  Every lane of every wave
// takes part and gets the same answer.  e == E: no such tile (a surplus workgroup).
struct ExpertTileHit {
    int e, lo, hi, tiles;     // expert, its row range [lo, hi), its row tiles
    uint32_t L;               // tile number inside the expert: at most the number asked for, which is below 2^31, as grids are
};

// WHOLE: only the whole tiles of a segment count (its ragged last tile is numbered elsewhere); `all` returns the
// number of tiles counted over all experts when L lies past them.
template <int BM, bool WHOLE = false>
__device__ __forceinline__ ExpertTileHit find_expert_tile(const ExpertArgs &a, int nct, int64_t L, int lane,
                                                          int64_t *all = nullptr)
{
    ExpertTileHit h;
    h.e = a.E;
    h.lo = h.hi = h.tiles = 0;
    h.L = 0;
    int64_t before = 0;                                            // tiles of the experts of earlier rounds
    for (int e0 = 0; e0 < a.E; e0 += kWave) {
        const int e = e0 + lane;
        int lo = 0, hi = 0, tiles = 0;
        if (e < a.E) {
            lo = a.lo[e];
            hi = a.hi_base[e] + (a.hi_len ? a.hi_len[e] : 0);
            tiles = hi > lo ? (int)(((int64_t)hi - lo + (WHOLE ? 0 : BM - 1)) / BM) : 0;
        }
        const int64_t cnt = (int64_t)tiles * nct;
        int64_t incl = cnt;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int64_t o = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += o;
        }
        // 64 bits, and by a shuffle: from a lane read the compiler knows the tile's number for uniform and divides it in scalar code,
        // four long chains of which cost every large tile's workgroup about 2 us (128 experts of 1024 x 480, 512 rows each 97 and 94).
        // The quotients themselves are of 32 bits: those of 64 cost short tiles up to 2 % (fp32, 8 of 512 x 2496, 105 rows 28.9 and 28.3)
        const int64_t total = __shfl(incl, kWave - 1, kWave);
        if (L < before + total) {
            // an expert without tiles repeats its predecessor's running total, so the first lane past L has tiles
            const unsigned long long past = __ballot(L < before + incl);
            const int src = __ffsll((long long)past) - 1;
            h.e = e0 + src;
            h.lo = __shfl(lo, src, kWave);
            h.hi = __shfl(hi, src, kWave);
            h.tiles = __shfl(tiles, src, kWave);
            h.L = (uint32_t)(L - before - (__shfl(incl, src, kWave) - __shfl(cnt, src, kWave)));
            return h;
        }
        before += total;
    }
    if (all) *all = before;
    return h;
}

__device__ __forceinline__ unsigned int f32_to_bf16_rne(float f)
{
    const unsigned int u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;       // finite inputs
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN, (64 * WM * WN <= 256 ? 2 : 1)) void expert_bf16_kernel(const u32x4 *__restrict__ x,
                                                                                      const u32x4 *__restrict__ w,
                                                                                      unsigned short *__restrict__ y,
                                                                                      ExpertArgs a)
{
    using G = ExpertTile<BM, BN, WM, WN>;
    extern __shared__ __align__(16) unsigned char exp_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 31, g = lane >> 5;
    const int cpr = a.H / 8;                                       // 16-byte pieces per row in memory
    const int nct = (a.N + BN - 1) / BN;                           // column tiles

    // logical tile numbers go out in blocks, XCD i taking kPerXcd consecutive numbers of each block (the workgroups
    // that run together on one XCD, which hardware fills round robin, then share operand tiles, and surplus numbers at
    // the end are spread over all XCDs); the numbering is (expert, column tile, row tile), row tile fastest
    constexpr int kPerXcd = 32 * G::kWgsPerCu;
    const int64_t jx = blockIdx.x / kXcds;
    int64_t L = (jx / kPerXcd) * (kPerXcd * kXcds) + (int64_t)(blockIdx.x % kXcds) * kPerXcd + jx % kPerXcd;
    const ExpertTileHit hit = find_expert_tile<BM>(a, nct, L, lane);
    const int e = hit.e;
    int row0 = 0, row_end = 0, ct = 0;
    if (e < a.E) {
        ct = (int)(hit.L / (uint32_t)hit.tiles);
        row0 = hit.lo + (int)(hit.L % (uint32_t)hit.tiles) * BM;
        row_end = hit.hi < a.max_rows ? hit.hi : a.max_rows;
    }
    if (e == a.E || row0 < 0 || row0 >= row_end) return;          // surplus workgroup (uniform for the workgroup)
    const int col0 = ct * BN;

    // This thread's pieces of a step's tile: piece q is row tid/8 + (threads/8)*q of the tile, 16-byte column tid%8;
    // tile rows 0..BM-1 are rows of x, the others rows of the weight tile.  Loads are issued unconditionally from
    // clamped in-bounds addresses; what lies outside becomes zeros when the tile is laid into LDS.
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const int r8 = tid >> 3, c_real = tid & 7;
    const int c0 = c_real < cpr ? c_real : 0;                     // rows shorter than a step: stay inside the row
    int grow[G::kLoads];                                           // row of x, or row of w, that piece q reads
    unsigned live = 0;
#pragma unroll
    for (int q = 0; q < G::kLoads; ++q) {
        bool ok;
        if (q < BM / G::kRowsPerPass) {
            const int r = row0 + r8 + q * G::kRowsPerPass;
            ok = r < row_end;
            grow[q] = ok ? r : row0;
        } else {
            const int n = col0 + r8 + (q - BM / G::kRowsPerPass) * G::kRowsPerPass;
            ok = n < a.N;
            grow[q] = e * a.N + (ok ? n : 0);
        }
        live |= (ok ? 1u : 0u) << q;
    }
    const int nsteps = (cpr + kExpBK / 8 - 1) / (kExpBK / 8);
    unsigned char *lay_at = exp_lds + r8 * kExpRowStride + c_real * 16;

    // steps past the end of the hidden axis are fetched from clamped addresses and never laid down
    auto fetch = [&](u32x4(&pre)[G::kLoads], int step) {
        const int c = step * (kExpBK / 8) + c_real < cpr ? step * (kExpBK / 8) + c0 : c0;
#pragma unroll
        for (int q = 0; q < G::kLoads; ++q) pre[q] = (q < BM / G::kRowsPerPass ? x : w)[(int64_t)grow[q] * cpr + c];
    };
    auto lay = [&](const u32x4(&pre)[G::kLoads], int step) {
        const bool col_ok = step * (kExpBK / 8) + c_real < cpr;
        __syncthreads();                                           // the previous tile has been read by every wave
#pragma unroll
        for (int q = 0; q < G::kLoads; ++q)
            *reinterpret_cast<u32x4 *>(lay_at + q * G::kRowsPerPass * kExpRowStride) =
                (((live >> q) & 1u) && col_ok) ? pre[q] : zero;
        __syncthreads();
    };

    f32x16 acc[G::kMT][G::kNT];
#pragma unroll
    for (int i = 0; i < G::kMT; ++i)
#pragma unroll
        for (int j = 0; j < G::kNT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int wm = wave / WN, wn = wave % WN;                      // the wave's place in the WM x WN grid
    const unsigned char *pa = exp_lds + (size_t)(wm * (BM / WM) + m) * kExpRowStride + g * 16;
    const unsigned char *pb = exp_lds + (size_t)(BM + wn * (BN / WN) + m) * kExpRowStride + g * 16;
    auto multiply = [&]() {
#pragma unroll
        for (int ks = 0; ks < kExpBK / 16; ++ks) {
            bf16x8 fa[G::kMT], fb[G::kNT];
#pragma unroll
            for (int i = 0; i < G::kMT; ++i)
                fa[i] = *reinterpret_cast<const bf16x8 *>(pa + (size_t)i * 32 * kExpRowStride + ks * 32);
#pragma unroll
            for (int j = 0; j < G::kNT; ++j)
                fb[j] = *reinterpret_cast<const bf16x8 *>(pb + (size_t)j * 32 * kExpRowStride + ks * 32);
#pragma unroll
            for (int i = 0; i < G::kMT; ++i)
#pragma unroll
                for (int j = 0; j < G::kNT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    };

    u32x4 pre[G::kLoads];
    fetch(pre, 0);
    for (int step = 0; step < nsteps; ++step) {
        lay(pre, step);
        fetch(pre, step + 1);                                      // in flight during the MFMAs
        multiply();
    }

    // accumulator element v of a lane: row (v/4)*8 + g*4 + v%4, column m of the 32 x 32 tile
#pragma unroll
    for (int i = 0; i < G::kMT; ++i)
#pragma unroll
        for (int j = 0; j < G::kNT; ++j) {
            const int n = col0 + wn * (BN / WN) + j * 32 + m;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = row0 + wm * (BM / WM) + i * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
                if (r < row_end && n < a.N) y[(int64_t)r * a.N + n] = (unsigned short)f32_to_bf16_rne(acc[i][j][v]);
            }
        }
}

// The same contraction with direct-to-LDS loads, for long segments: a 256 x 256 tile of y per workgroup of 4 waves, one
// per SIMD, each 128 x 128 = 8 x 8 tiles of the 16x16x32 MFMA (256 accumulator registers; the other 256 hold two sets of
// fragments).  What bounds such a kernel is the matrix pipe, provided that everything else fits beside it:
//  - LDS reads.  A wave tile of 128 x 128 reads a third less per flop than 128 x 64 (128 KiB per step of 64 elements
//    against 192), and the fragments of the next 32-element slice are read while the present one is multiplied, one read
//    per four MFMAs, so no MFMA waits for the LDS.
//  - Register moves.  Left to itself the compiler rotates the accumulators through copies (about one per MFMA); the MFMA
//    is therefore written with its accumulator tied in place, and the order of reads, loads and MFMAs is pinned.
//  - Loads.  A step's tile (256 rows of x, 256 of w, 128 bytes each) goes straight to LDS while the stage before it is
//    multiplied; a stage's buffer is free once its second slice has been read, so the loads of stage s+2 are issued under the
//    second slice of stage s and have until the end of the first slice of stage s+1.  That covers an L2 hit but no miss.
//    Where several row tiles share a weight tile (DEEP_W = false) each workgroup also touches, one stage ahead, one line per
//    row of its share of the tiles it shares with the other workgroups on its XCD (its own eighth of a weight tile, its quarter
//    of an x tile), so that misses are taken early.  Where a weight tile has one or two users it comes from memory whatever is
//    done; there the LDS holds a third stage of w instead, whose loads are issued a stage earlier (DEEP_W = true).  Measured,
//    third stage against touches: 64 experts, 7168 x 2048, 191 rows each 419 and 445 us, 256 rows 593 and 606, 384 rows 764 and
//    683; 8 experts, 4096 x 4096, 256 rows 114 and 119, 2048 rows 459 and 449.
// Rows are 128 bytes in LDS without padding; the 16-byte piece c of row r sits at position c ^ ((r / 2) % 8): a fragment
// read has 16 lanes (16 consecutive rows, one piece each) share the 64 banks, two rows fill them, so the pieces must
// differ among the even rows and among the odd rows.  The LDS position of a lane's data is fixed by the instruction, so
// the swizzle is applied on the global side.  Buffer descriptors end at the segment's last row and at the last output
// feature: rows past them arrive as zeros and cost no traffic.  Needs H to be a multiple of 64.
// The weight rows are the MFMA's A operand, so that a lane ends up with four consecutive features of a row: 8-byte stores.
// Measured on MI355X, random normal inputs, bursts of 300 launches: 16384 x 4096 x 4096 in one segment 477-495 us with the
// 8-wave kernel this one replaced (128 x 64 per wave, 32x32x16 MFMA, fragment reads scheduled by the compiler), 376-380
// now (1.45 PFLOP/s; without any loads 329, a library GEMM 348-356); two segments of 4096 x 8192 x 8192 958-981 -> 743
// (805 without the early touch); eight uneven segments of about 2048 rows (4.3 rounds of workgroups) 553 -> 448.  What
// bounds it now: the matrix pipe at the clock the chip holds under this load, and the last round of a launch.
constexpr int kBigBM = 256, kBigBN = 256, kBigThreads = 256;
constexpr int kShortRows = 64;                                    // ragged tiles up to this many rows run as short tiles
constexpr int kBigXBytes = kBigBM * 128, kBigWBytes = kBigBN * 128;       // one stage of x, of w
// two stages of x; of w three, which takes all of a CU's 160 KiB, or two and 512 bytes per wave for the early touches
constexpr int big_lds_bytes(bool deep_w) { return 2 * kBigXBytes + (deep_w ? 3 * kBigWBytes : 2 * kBigWBytes + 2048); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}
typedef __attribute__((address_space(3))) void lds_void;
// Cache bits of a buffer load: `nt`, no reuse expected.  On weights that only one workgroup reads and that would not stay in the
// memory-side cache until the next call it is worth 10-17 %, as the lines push nothing else out on their way.  Where it is not: on
// rows that are not whole lines (a line at the seam of two rows is fetched twice), on a tile with a second reader, on weights
// that the cache does hold; and in the register-staged tiles it changes nothing (64 experts of 7168 x 2048, 60 rows: 333 us with
// and without).  Three sets of weights in turn, plain and streamed: 64 experts of 7168 x 2048, 16 rows 311 and 277 us; but 16 of
// 8184 x 2048 112 and 127; 16 of 4096 x 1024 in 32 x 64 tiles, 40 rows 31 and 37; 8 of 2048 x 2048 12.7 and 14.8.
constexpr int kStreamLoad = 2;
constexpr uint32_t kOutOfRange = 0x80000000u;                      // a lane offset past every descriptor: no access

// Scalar offset of the 128 bytes that follow those at `at` in every row of a tile of `turn` / 128 steps: from the last step round to the
// first.  The range check of a buffer load compares the lane's offset with num_records - scalar offset in 32 bits, and the smallest
// descriptor is one row, whose last step may hold a single piece of 16 bytes: the scalar offset must stay below that, or the difference
// wraps and every lane offset counts as in range.  Steps past the end, whose lanes are out of range anyway, therefore go round, too.
__host__ __device__ constexpr uint32_t next_step(uint32_t at, uint32_t turn) { return at + 128u == turn ? 0u : at + 128u; }
constexpr bool step_offsets_stay_inside(int nsteps, int start, int past)
{
    const uint32_t turn = (uint32_t)nsteps * 128u, records = turn - 112u;
    uint32_t at = (uint32_t)start * 128u;
    for (int step = 0; step < nsteps + past; ++step, at = next_step(at, turn))
        if (at >= records || kOutOfRange < records - at) return false;
    return true;
}
static_assert(step_offsets_stay_inside(1, 0, 8) && step_offsets_stay_inside(2, 1, 8) && step_offsets_stay_inside(7, 5, 8),
              "a one-row tile must refuse the loads of the steps past its end");
constexpr int kBigMaxHidden = 1 << 20;                             // a tile's 256 rows end far below it

// four fp32 -> four bf16, nearest-even, as 8 bytes
__device__ __forceinline__ uint2 pack_bf16x4(f32x4 v)
{
    uint2 o;
    o.x = f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16);
    o.y = f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16);
    return o;
}

// Where tile number `tile` starts its walk along the hidden axis.  Rows that are a multiple of 4096 bytes apart begin on the same memory
// channels, so that workgroups which walk in step all wait for a few of them: 256 MiB of weights in rows of 8192 bytes, 64 rows a workgroup,
// read and nothing else, arrive in 52 us, at 14336 bytes a row in 39 (6.9 TB/s); with the starts spread over the row in 39 and 39.  The
// multiplier spreads consecutive tiles evenly over any number of steps.  Rows have to be whole steps.
__device__ __forceinline__ int walk_start(int tile, int nsteps)
{
    return (int)(((uint32_t)tile * 40503u & 0xffffu) * (uint32_t)nsteps >> 16);
}

// A tile of at most XR rows x WR output features: so little arithmetic per step that the step is as long as its loads take
// to arrive, so what counts is how many bytes are on their way.  Compact stages of XR + WR rows, NST of them, the loads of
// NST - 1 steps in flight.  Four waves, each all rows x WR / 4 columns.  Every wave issues the same number of loads per step,
// also past the end (out of range: no traffic), because the wait for a stage counts the younger loads.  The barrier is the
// bare instruction behind a wait for the LDS reads: the compiler's own barrier would wait for every outstanding load, the
// next stages' included.  A row is `cpr` pieces of 16 bytes, a step 8 of them; the pieces of the last step that lie past the end
// of the row are out of range, too, and multiply as zeros.  The walk begins at step `start` (0 unless rows are whole steps) and goes round.
template <int XR, int WR, int NST>
struct ShortTile {
    static constexpr int kStageBytes = (XR + WR) * 128, kLdsBytes = NST * kStageBytes;
    static constexpr int kCX = XR / 32, kCW = WR / 32, kLoads = kCX + kCW;       // 8-row chunks per wave and step
    static constexpr int kYounger = (NST - 2) * kLoads;                         // loads issued after those of the stage waited for
    static constexpr int kWait = 0x0f70 | (kYounger & 15) | ((kYounger >> 4) << 14);        // s_waitcnt vmcnt(kYounger)
    static_assert(XR % 32 == 0 && WR % 64 == 0 && NST >= 3 && kYounger < 64, "short tile: shape");
};

// F32: the activations and weights are fp32, 32 of them per step; a lane's 16 bytes are then four elements for four 16x16x4
// MFMAs, each of which takes the same element of the four pieces of half a step.
// T: unsigned short, y is rounded to bf16; float, the sums themselves are stored, rows of whole 16-byte vectors (VEC) or of any N
// columns.  Sums of the first kind are taken in two levels, 8 steps of the hidden axis at a time.  Those of the second, the
// logits, in three, the lowest of one step (fp32) or of one to four, and there in a chain of additions per half of a step (in fp32
// per element of a piece), so that neither short rows nor long ones cost precision; the middle one, on bf16 rows of up to 16 steps,
// in a chain per even and odd step of each half of the row.  Error against 64 bits with one chain and two levels, and now: 512
// elements 1.2e-7, 6.1e-8; 1536 1.3e-7, 7.4e-8; 8192 1.5e-7, 1.05e-7; fp32, 1000 2.9e-7, 9.6e-8, 8192 3.1e-7, 1.4e-7.
// ANY_START, of bf16 logits whose walk begins at an even step: added so that where it begins does not show (run_any_start).
// FINE, of fp32 sums: a chain per half of a step and levels of 4 steps, 1 to 3 % of the time; error against 64 bits at 1024 elements 2.9e-7,
// 1.6e-7, at 5788 3.0e-7, 1.9e-7.
// AUX_W: cache bits of the weights' loads.
template <int XR, int WR, int NST, bool F32, bool VEC, int AUX_W = 0, bool ANY_START = false, bool FINE = false, typename T>
__device__ __forceinline__ void expert_short_tile(__amdgpu_buffer_rsrc_t rx, __amdgpu_buffer_rsrc_t rw, T *__restrict__ y, int cpr,
                                                  int N, int64_t row0, int64_t row_end, int col0, unsigned char *lds, int start)
{
    using G = ShortTile<XR, WR, NST>;
    constexpr int RB = XR / 16, CB = WR / 64;                      // 16-row blocks, 16-column blocks of a wave
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));      // share nothing with the caller's other path, which has no register left to keep it in
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 15, g = lane >> 4;
    const int nsteps = (cpr + 7) / 8;
    const uint32_t rowb = (uint32_t)cpr * 16;
    const int lr = lane >> 3;
    // row of the lane in chunk c: 8 c + lane / 8, so (row / 2) % 8 = (4 c + lr / 2) % 8
    auto piece = [&](int c) { return (lane & 7) ^ ((4 * c + (lr >> 1)) & 7); };
    auto offset = [&](int c) { return (uint32_t)(c * 8 + lr) * rowb + piece(c) * 16; };
    uint32_t ox[G::kCX], ow[G::kCW];
#pragma unroll
    for (int q = 0; q < G::kCX; ++q) ox[q] = offset(wave * G::kCX + q);
#pragma unroll
    for (int q = 0; q < G::kCW; ++q) ow[q] = offset(wave * G::kCW + q);
    auto load = [&](unsigned char *base, uint32_t so, auto lane_offset) {
#pragma unroll
        for (int q = 0; q < G::kCW; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(base + (XR / 8 + wave * G::kCW + q) * 1024), 16,
                                                     lane_offset(wave * G::kCW + q, ow[q]), so, 0, AUX_W);
#pragma unroll
        for (int q = 0; q < G::kCX; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)(base + (wave * G::kCX + q) * 1024), 16,
                                                     lane_offset(wave * G::kCX + q, ox[q]), so, 0, 0);
    };
    uint32_t so = (uint32_t)start * 128u;                          // of the step that is requested next
    auto issue_whole = [&](int, int slot) {                        // the row holds all 8 pieces of the step
        load(lds + slot * G::kStageBytes, so, [&](int, uint32_t o) { return o; });
        so = next_step(so, (uint32_t)nsteps * 128u);
    };
    auto issue_any = [&](int step, int slot) {
        const int left = cpr - step * 8;                           // pieces of the row in this step; none past the end
        load(lds + slot * G::kStageBytes, so, [&](int c, uint32_t o) { return piece(c) < left ? o : kOutOfRange; });
        so = next_step(so, (uint32_t)nsteps * 128u);
    };
    constexpr bool kLevels = std::is_same<T, float>::value;
    constexpr bool kLogits = kLevels && !VEC;
    constexpr int kChains = kLogits && F32 ? 4 : kLogits || FINE ? 2 : 1;
    static_assert(!ANY_START || (kLogits && !F32), "short tile: a start that does not show is one of bf16 logits");
    static_assert(!FINE || (kLevels && !kLogits), "short tile: finer levels are those of fp32 sums");
    f32x4 acc[kChains][RB][CB];
#pragma unroll
    for (int c = 0; c < kChains; ++c)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) acc[c][i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    f32x4 total[kLevels ? RB : 1][kLevels ? CB : 1], part[kLogits ? RB : 1][kLogits ? CB : 1];
    if constexpr (kLevels) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) total[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    if constexpr (kLogits) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) part[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    // adds the chains of one result to `to` and clears them
    auto fold = [&](int i, int j, f32x4 &to) {
#pragma unroll
        for (int c = kChains / 2; c >= 1; c /= 2)
#pragma unroll
            for (int b = 0; b < c; ++b) acc[b][i][j] += acc[b + c][i][j];
        to += acc[0][i][j];
#pragma unroll
        for (int c = 0; c < kChains; ++c) acc[c][i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    };
    const unsigned char *px = lds + m * 128, *pw = lds + (XR + wave * (WR / 4) + m) * 128;
    const int nb = (int)((row_end - row0 + 15) / 16);              // 16-row blocks with rows of the segment

    // one 16-row block times the wave's columns: half a step, or, of fp32 elements, element v of its pieces
    auto multiply = [&](const f32x4(&fw)[CB], const f32x4 &fx, f32x4(&to)[CB], int v) {
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            if constexpr (F32) to[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[j][v], fx[v], to[j], 0, 0, 0);
            else to[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[j]), __builtin_bit_cast(bf16x8, fx), to[j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int q = 0; q < NST - 1; ++q) issue_any(q, q);
    int slot = 0;
    // step `step`, whose loads ahead are of whole steps or not: use(weights, rows) with the fragments of its first BLOCKS blocks of rows
    auto advance = [&](auto blocks, auto whole, int step, auto use) {
        constexpr int BLOCKS = decltype(blocks)::value;
        __builtin_amdgcn_s_waitcnt(G::kWait);                          // stage `step` has landed (loads finish in order)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);                            // lgkmcnt(0): this wave's reads of the previous stage
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int free_slot = slot == 0 ? NST - 1 : slot - 1;          // of stage step-1
        if constexpr (decltype(whole)::value) issue_whole(step + NST - 1, free_slot);
        else issue_any(step + NST - 1, free_slot);
        const int buf = slot * G::kStageBytes;
        // all fragments of the step first, so that the reads' latency is paid once
        f32x4 fw[2][CB], fx[2][BLOCKS];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int at = buf + ((4 * ks + g) ^ ((m >> 1) & 7)) * 16;
#pragma unroll
            for (int j = 0; j < CB; ++j) fw[ks][j] = *reinterpret_cast<const f32x4 *>(pw + at + j * 2048);
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i) fx[ks][i] = *reinterpret_cast<const f32x4 *>(px + at + i * 2048);
        }
        use(fw, fx);
        slot = slot == NST - 1 ? 0 : slot + 1;
    };
    // steps [from, to), added to the chains
    auto walk = [&](auto blocks, auto whole, int from, int to) {
        for (int step = from; step < to; ++step)
            advance(blocks, whole, step, [&](const auto &fw, const auto &fx) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int v = 0; v < (F32 ? 4 : 1); ++v)
#pragma unroll
                        for (int i = 0; i < decltype(blocks)::value; ++i)
                            multiply(fw[ks], fx[ks][i], acc[kChains == 1 ? 0 : kChains == 2 ? ks : v][i], v);
                if constexpr (kLogits && F32) {
#pragma unroll
                    for (int i = 0; i < decltype(blocks)::value; ++i)
#pragma unroll
                        for (int j = 0; j < CB; ++j) fold(i, j, part[i][j]);
                }
            });
    };
    // All steps of bf16 logits, a row of at most 16, with the sums of one step as the lowest level: added to the partial sums of the
    // even or of the odd steps, with no chain to clear, which took a quarter of a short row's time (8192 x 512, 128 experts 7.3 us, now
    // 6.5, 2500 x 512, 65 experts 5.5 and 4.8).  Two chains, as one came out less exact than the split tiles: 384 elements 6.3e-8 off
    // 64 bits, now 5.9e-8, split tiles 5.9e-8; 640 7.0e-8, 6.4e-8 and 6.4e-8; 1024 7.0e-8, 6.8e-8 and 6.9e-8.
    auto run_each = [&](auto blocks, int whole_to) {
        constexpr int BLOCKS = decltype(blocks)::value;
        f32x4 odd[BLOCKS][CB];
        auto add_to = [&](auto sums) {
            return [&, sums](const auto &fw, const auto &fx) {
#pragma unroll
                for (int i = 0; i < BLOCKS; ++i) {
                    f32x4 half[2][CB];
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int j = 0; j < CB; ++j)
                            half[ks][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[ks][j]), __builtin_bit_cast(bf16x8, fx[ks][i]),
                                                                                  (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < CB; ++j) sums[i][j] += half[0][j] + half[1][j];
                }
            };
        };
        auto walk_each = [&](auto whole, int from, int to) {          // `from` is an even step
            for (int step = from; step < to; step += 2) {
                advance(blocks, whole, step, add_to(&part[0]));
                if (step + 1 < to) advance(blocks, whole, step + 1, add_to(&odd[0]));
            }
        };
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) odd[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
        const int span = nsteps <= 6 ? 6 : ((nsteps + 1) / 2 + 1) & ~1;                  // an even number, two of them from 7 steps on
        for (int from = 0; from < nsteps; from += span) {
            const int end = min(from + span, nsteps), mid = max(min(whole_to, end) & ~1, from);
            walk_each(std::true_type{}, from, mid);
            walk_each(std::false_type{}, mid, end);
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
                for (int j = 0; j < CB; ++j) {
                    total[i][j] += part[i][j] + odd[i][j];
                    part[i][j] = odd[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    // All steps of logits whose tiles begin at different even steps: equal tokens have to have equal logits wherever they stand.  The sums of
    // two neighbouring steps, always the same two, are added up in 64 bits: 24-bit numbers, up to 64 of them (rows of 8192
    // elements) without any rounding where they are at most 2^23 apart, and what rounds beyond that is 2^-53 of the sum, to be seen in
    // the logit only beside the middle of two 32-bit numbers.  It takes fewer registers than three levels, no more time, and is more
    // exact: 2048 elements 7.6e-8 off 64 bits, now 5.6e-8, 4096 9.1e-8 and 5.6e-8, 8192 1.05e-7 and 5.6e-8.
    auto run_any_start = [&](auto blocks, int whole_to) {
        constexpr int BLOCKS = decltype(blocks)::value;
        double sums[BLOCKS][CB][4];
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) sums[i][j][v] = 0.0;
        auto two_steps = [&](auto whole, int step) {
            f32x4 half[2][BLOCKS][CB];
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
                for (int j = 0; j < CB; ++j) half[0][i][j] = half[1][i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
            auto add = [&](const auto &fw, const auto &fx) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < BLOCKS; ++i) multiply(fw[ks], fx[ks][i], half[ks][i], 0);
            };
            advance(blocks, whole, step, add);
            advance(blocks, whole, step + 1, add);
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
                for (int j = 0; j < CB; ++j) {
                    const f32x4 both = half[0][i][j] + half[1][i][j];
#pragma unroll
                    for (int v = 0; v < 4; ++v) sums[i][j][v] += (double)both[v];
                }
        };
        int step = 0;
        for (; step + 1 < whole_to; step += 2) two_steps(std::true_type{}, step);
        for (; step < nsteps; step += 2) two_steps(std::false_type{}, step);
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) total[i][j][v] = (float)sums[i][j][v];
    };
    // With at most half of the row blocks in use only those are multiplied.  One choice before the loop, as for the steps that are
    // not whole: with a condition per block inside it a step waits for one read after the other (2 rows each of 16 experts of 5120 x
    // 152, 48 workgroups: 21.8 us, now 16.4; 2 experts of 8192 x 64, 60 rows: 38 and 25).
    auto run = [&](auto blocks) {
        const int whole_to = cpr / 8 - (NST - 1);                      // up to here the step NST - 1 ahead is a whole one
        if constexpr (ANY_START) return run_any_start(blocks, whole_to);
        if constexpr (kLogits && !F32)
            if (nsteps <= 16) return run_each(blocks, whole_to);
        const int span = FINE ? 4 : kLevels ? 8 : nsteps, sub = !kLogits || F32 ? span : nsteps <= 32 ? 2 : 4;
        for (int from = 0; from < nsteps; from += span) {
            const int end = min(from + span, nsteps);
            for (int first = from; first < end; first += sub) {
                const int to = min(first + sub, end), mid = min(max(whole_to, first), to);
                walk(blocks, std::true_type{}, first, mid);
                walk(blocks, std::false_type{}, mid, to);
                if constexpr (kLogits && !F32) {
#pragma unroll
                    for (int i = 0; i < decltype(blocks)::value; ++i)
#pragma unroll
                        for (int j = 0; j < CB; ++j) fold(i, j, part[i][j]);
                }
            }
            if constexpr (kLevels) {
#pragma unroll
                for (int i = 0; i < decltype(blocks)::value; ++i)
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        if constexpr (kLogits) {
                            total[i][j] += part[i][j];
                            part[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
                        } else {
                            fold(i, j, total[i][j]);
                        }
                    }
            }
        }
    };
    if (2 * nb <= RB) run(std::integral_constant<int, RB / 2>{});
    else run(std::integral_constant<int, RB>{});
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int64_t r = row0 + i * 16 + m;
        if (r < row_end) {
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                const int n = col0 + wave * (WR / 4) + j * 16 + 4 * g;
                if constexpr (std::is_same<T, float>::value) {
                    if constexpr (VEC) {
                        if (n < N) *reinterpret_cast<f32x4 *>(y + r * N + n) = total[i][j];
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (n + v < N) y[r * N + n + v] = total[i][j][v];
                    }
                } else {
                    if (n < N) *reinterpret_cast<uint2 *>(y + r * N + n) = pack_bf16x4(acc[0][i][j]);
                }
            }
        }
    }
}

// Few rows per expert (a decoding step): every weight is read once for a handful of rows, and the layer lasts as long as
// the weights take to arrive from memory.  Two workgroups per CU, 128 KiB of loads in flight per CU.  Measured on MI355X,
// register-staged 128 x 256 tiles before, now (floor: the weights at 6.4 TB/s): 8 experts of 4096 x 4096, 16 rows each, one set of
// weights used again 138 -> 40 us, several in turn 48 (42); 64 of 7168 x 2048, 16 rows 314 -> 269 us (294; 311 before the streaming);
// 64 of 2048 x 2048 133 -> 98 us (84); rows that are not whole steps: 2 of 7464 x 1904, 16 rows 199 -> 33 us, 8 of 1032 x 4096,
// 16 rows 55 -> 15 us (11).  Streaming the weights straight into registers in the MFMA's layout (16 rows x 64 bytes per load) was
// measured too: 61, 434 and 121 us.
// fp32, any number of rows: the same tiles, where the barrier and the reads of a step cost less than its MFMAs (16 of 32 clocks
// each for a wave of the 32 x 64 tile).  A 64 x 64 tile with one step in flight through registers before, now: 2 experts of 4096 x
// 4096, 8 rows each 108 -> 49 us (21), 10 of 516 x 516, about 240 rows 30 -> 19 us, 8 of 1024 x 1024, 600 rows 113 -> 100 us
// (70 at the 143 TFLOP/s of a library GEMM); error against 64 bits at 8192 elements 1.6e-6 -> 3.1e-7 (two levels of sums).
template <int XR, int WR, int NST, bool F32, bool FINE>
__global__ __launch_bounds__(256, 2) void expert_short_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                              void *__restrict__ y, ExpertArgs a)
{
    using T = std::conditional_t<F32, float, unsigned short>;
    extern __shared__ __align__(16) unsigned char short_lds[];
    const int lane = threadIdx.x & 63;
    const int cpr = F32 ? a.H / 4 : a.H / 8, nct = (a.N + WR - 1) / WR;
    // numbers are dealt to the XCDs in blocks, row tiles fastest: row tiles of one weight tile meet in one L2
    const int64_t j = blockIdx.x / kXcds;
    const int64_t L = ((((j >> a.deal) * kXcds) + (int64_t)(blockIdx.x % kXcds)) << a.deal) + (j & ((1 << a.deal) - 1));
    const ExpertTileHit hit = find_expert_tile<XR>(a, nct, L, lane);
    const int e = __builtin_amdgcn_readfirstlane(hit.e);
    if (e >= a.E) return;                                          // surplus workgroup
    const int ct = __builtin_amdgcn_readfirstlane((int)(hit.L / (uint32_t)hit.tiles));
    const int row0 = __builtin_amdgcn_readfirstlane(hit.lo + (int)(hit.L % (uint32_t)hit.tiles) * XR);
    const int seg_end = __builtin_amdgcn_readfirstlane(hit.hi < a.max_rows ? hit.hi : a.max_rows);
    if (row0 < 0 || row0 >= seg_end) return;
    const int row_end = min(seg_end, row0 + XR), col0 = ct * WR;
    const uint32_t rowb = (uint32_t)cpr * 16;
    const auto rx = make_rsrc(x + (int64_t)row0 * cpr, (uint32_t)(row_end - row0) * rowb);
    const auto rw = make_rsrc(w + ((int64_t)e * a.N + col0) * cpr, (uint32_t)min(a.N - col0, WR) * rowb);
    // by the column tile, whichever the rows: a row's result does not depend on the launch that computes it
    const int start = a.spread ? walk_start(e * nct + ct, cpr / 8) : 0;
    if ((int64_t)e * a.N + col0 >= a.stream_from && __builtin_amdgcn_readfirstlane(hit.tiles) == 1)
        expert_short_tile<XR, WR, NST, F32, F32, kStreamLoad, false, FINE>(rx, rw, static_cast<T *>(y), cpr, a.N, row0, row_end, col0, short_lds, start);
    else
        expert_short_tile<XR, WR, NST, F32, F32, 0, false, FINE>(rx, rw, static_cast<T *>(y), cpr, a.N, row0, row_end, col0, short_lds, start);
}

// Layers of so few tiles that one tile's walk along the hidden axis is what takes the time, not the bytes: a tile of 16 XB rows x 16 CB
// features whose steps are dealt to the W waves of its workgroup.  Each wave has a ring of NST stages of its own and waits for nobody: no
// barrier until the waves' sums are added, through LDS and in a fixed order.  16 x 16 tiles, four waves: 48 KiB, three workgroups per CU.
// A walk of the 32 x 64 tiles takes 0.23 us a step with the loads of three steps in flight.  Measured on MI355X, those tiles and these, three
// sets of weights in turn, us: 2 experts of 4096 x 512, 8 rows 12.7 and 5.2; 2 of 8192 x 488, 23 rows 28.0 and 9.5; 8 of 2048 x
// 704, 19 rows 10.0 and 7.4; fp32, 8 of 8192 x 136, 2 rows 72 and 14, 4 of 4096 x 68, 258 rows 54 and 15.  Where the lines lie stands at
// launch_expert_few.  fp32 error against 64 bits at 1024 elements 2.9e-7, now 1.6e-7: shorter chains.
template <int XB, int CB, int W, int NST>
struct SplitTile {
    static constexpr int kStageBytes = (XB + CB) * 2048, kRingBytes = NST * kStageBytes, kLdsBytes = W * kRingBytes, kThreads = 64 * W;
    static constexpr int kLoads = 2 * (XB + CB), kYounger = (NST - 2) * kLoads;        // of one step; issued after those of the stage waited for
    static constexpr int kWait = 0x0f70 | (kYounger & 15) | ((kYounger >> 4) << 14);   // s_waitcnt vmcnt(kYounger)
    static_assert(NST >= 3 && kYounger < 64 && kLdsBytes <= 160 * 1024, "split tile: shape");
    static_assert(XB * CB * 1024 <= kRingBytes, "split tile: the waves' sums lie in the rings");
};

// T: unsigned short, y is rounded to bf16; float, the sums themselves are stored, rows of whole 16-byte vectors (VEC) or of any N columns.
template <int XB, int CB, int W, int NST, bool F32, bool VEC, typename T>
__device__ __forceinline__ void split_tile(__amdgpu_buffer_rsrc_t rx, __amdgpu_buffer_rsrc_t rw, T *__restrict__ y, int cpr, int N, int64_t row0,
                                           int64_t row_end, int col0, unsigned char *split_lds)
{
    using G = SplitTile<XB, CB, W, NST>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), m = lane & 15, g = lane >> 4, lr = lane >> 3;
    const uint32_t rowb = (uint32_t)cpr * 16;
    // Rows in LDS and their swizzle as in the short tiles.  Every wave issues the same loads per step, also past the end of its share
    // (out of range, at scalar offset 0: no traffic), because the wait for a stage counts the younger ones.
    const int nsteps = (cpr + 7) / 8, first = nsteps * wave / W, last = nsteps * (wave + 1) / W;
    unsigned char *const ring = split_lds + wave * G::kRingBytes;
    auto piece = [&](int q) { return (lane & 7) ^ ((4 * q + (lr >> 1)) & 7); };
    uint32_t off[2];                                               // chunks 16 rows apart have the same swizzle
#pragma unroll
    for (int q = 0; q < 2; ++q) off[q] = (uint32_t)(q * 8 + lr) * rowb + piece(q) * 16;
    auto issue = [&](int step, int slot) {
        const int left = step < last ? cpr - step * 8 : 0;         // pieces of the row in this step
        const uint32_t so = step < last ? (uint32_t)step * 128u : 0u;
        unsigned char *const base = ring + slot * G::kStageBytes;
        uint32_t o[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) o[q] = piece(q) < left ? off[q] : kOutOfRange;
#pragma unroll
        for (int q = 0; q < 2 * CB; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(base + (2 * XB + q) * 1024), 16, o[q & 1] + (uint32_t)(q >> 1) * 16 * rowb, so, 0, 0);
#pragma unroll
        for (int q = 0; q < 2 * XB; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)(base + q * 1024), 16, o[q & 1] + (uint32_t)(q >> 1) * 16 * rowb, so, 0, 0);
    };
    // Two chains per result, by half of the step, and two levels, 8 steps at a time; of logits 2 or 1, whose error must not be above that of
    // eight shares with one level (gate_split_kernel and now, against 64 bits: 1024 elements 6.9e-8, 6.9e-8, 2048 8.1e-8, 7.5e-8, 8192
    // 1.4e-7, 9.9e-8; with 8 steps at a time 2048 9.7e-8, with 2 at 512 6.3e-8 in place of 6.1e-8).
    const int span = !(std::is_same<T, float>::value && !VEC) ? 8 : nsteps <= 16 ? 1 : 2;
    f32x4 acc[2][XB][CB], total[XB][CB];
#pragma unroll
    for (int i = 0; i < XB; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[0][i][c] = acc[1][i][c] = total[i][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NST - 1; ++q) issue(first + q, q);
    int slot = 0;
    for (int from = first; from < last; from += span) {
        const int to = min(from + span, last);
        for (int step = from; step < to; ++step) {
            __builtin_amdgcn_s_waitcnt(G::kWait);                  // stage `step` has landed (loads finish in order)
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xc07f);                    // lgkmcnt(0): the reads of the slot that is filled next
            asm volatile("" ::: "memory");
            issue(step + NST - 1, slot == 0 ? NST - 1 : slot - 1);
            f32x4 fw[2][CB], fx[2][XB];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const unsigned char *at = ring + slot * G::kStageBytes + m * 128 + ((4 * ks + g) ^ ((m >> 1) & 7)) * 16;
#pragma unroll
                for (int i = 0; i < XB; ++i) fx[ks][i] = *reinterpret_cast<const f32x4 *>(at + i * 2048);
#pragma unroll
                for (int c = 0; c < CB; ++c) fw[ks][c] = *reinterpret_cast<const f32x4 *>(at + (XB + c) * 2048);
            }
#pragma unroll
            for (int v = 0; v < (F32 ? 4 : 1); ++v)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < XB; ++i)
#pragma unroll
                        for (int c = 0; c < CB; ++c) {
                            if constexpr (F32) acc[ks][i][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[ks][c][v], fx[ks][i][v], acc[ks][i][c], 0, 0, 0);
                            else acc[ks][i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw[ks][c]),
                                                                                         __builtin_bit_cast(bf16x8, fx[ks][i]), acc[ks][i][c], 0, 0, 0);
                        }
            slot = slot == NST - 1 ? 0 : slot + 1;
        }
#pragma unroll
        for (int i = 0; i < XB; ++i)
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                total[i][c] += acc[0][i][c] + acc[1][i][c];
                acc[0][i][c] = acc[1][i][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
    }
    __builtin_amdgcn_s_waitcnt(0x0070);                            // what is still on its way would overwrite the sums
    asm volatile("" ::: "memory");
    __syncthreads();
    f32x4 *red = reinterpret_cast<f32x4 *>(split_lds);             // [wave][row block][column block][lane]
#pragma unroll
    for (int i = 0; i < XB; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) red[((wave * XB + i) * CB + c) * kWave + lane] = total[i][c];
    __syncthreads();
    for (int b = wave; b < XB * CB; b += W) {
        f32x4 sum[W];
#pragma unroll
        for (int v = 0; v < W; ++v) sum[v] = red[(v * XB * CB + b) * kWave + lane];
#pragma unroll
        for (int d = W / 2; d >= 1; d /= 2)
#pragma unroll
            for (int v = 0; v < d; ++v) sum[v] += sum[v + d];
        const int64_t r = row0 + (b / CB) * 16 + m;
        const int n = col0 + (b % CB) * 16 + 4 * g;
        if (r < row_end && n < N) {
            if constexpr (!std::is_same<T, float>::value) {
                *reinterpret_cast<uint2 *>(y + r * N + n) = pack_bf16x4(sum[0]);
            } else if constexpr (VEC) {
                *reinterpret_cast<f32x4 *>(y + r * N + n) = sum[0];
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < N) y[r * N + n + v] = sum[0][v];
            }
        }
    }
}

template <int XB, int CB, int W, int NST, bool F32>
__global__ __launch_bounds__(64 * W) void expert_split_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w, void *__restrict__ y,
                                                              ExpertArgs a)
{
    constexpr int XR = 16 * XB, WR = 16 * CB;
    extern __shared__ __align__(16) unsigned char split_lds[];
    const int lane = threadIdx.x & 63;
    const int cpr = F32 ? a.H / 4 : a.H / 8, nct = (a.N + WR - 1) / WR;
    // tile numbers in blocks of 8 per XCD: so few of them, in blocks of 32, would leave XCDs without any
    const int64_t j = blockIdx.x / kXcds;
    const int64_t L = (j / 8) * (8 * kXcds) + (int64_t)(blockIdx.x % kXcds) * 8 + j % 8;
    const ExpertTileHit hit = find_expert_tile<XR>(a, nct, L, lane);
    const int e = __builtin_amdgcn_readfirstlane(hit.e);
    if (e >= a.E) return;                                          // surplus workgroup
    const int ct = __builtin_amdgcn_readfirstlane((int)(hit.L / (uint32_t)hit.tiles));
    const int row0 = __builtin_amdgcn_readfirstlane(hit.lo + (int)(hit.L % (uint32_t)hit.tiles) * XR);
    const int seg_end = __builtin_amdgcn_readfirstlane(hit.hi < a.max_rows ? hit.hi : a.max_rows);
    if (row0 < 0 || row0 >= seg_end) return;
    const int row_end = min(seg_end, row0 + XR), col0 = ct * WR;
    const uint32_t rowb = (uint32_t)cpr * 16;
    const auto rx = make_rsrc(x + (int64_t)row0 * cpr, (uint32_t)(row_end - row0) * rowb);
    const auto rw = make_rsrc(w + ((int64_t)e * a.N + col0) * cpr, (uint32_t)min(a.N - col0, WR) * rowb);

    using T = std::conditional_t<F32, float, unsigned short>;
    split_tile<XB, CB, W, NST, F32, F32>(rx, rw, static_cast<T *>(y), cpr, a.N, row0, row_end, col0, split_lds);
}

// TAIL: rows are not whole steps; the last step's pieces past the end of a row are out of range.
template <bool RAGGED_LAST, bool DEEP_W, bool TAIL>
__global__ __launch_bounds__(kBigThreads, 1) void expert_big_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                                    unsigned short *__restrict__ y, ExpertArgs a)
{
#if defined(__HIP_DEVICE_COMPILE__)         // the matrix instruction is written out: nothing for the host pass to parse
    constexpr int BM = kBigBM, BN = kBigBN, P = 8;                 // P: row tiles of a panel
    extern __shared__ __align__(16) unsigned char big_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cpr = a.H / 8, nsteps = (cpr + 7) / 8;
    const int nct = (a.N + BN - 1) / BN;

    // Tile of this workgroup.  Hardware deals consecutive workgroups round robin to the 8 XCDs, each with its own L2;
    // the 32 workgroups that run together on one XCD should share tiles of x and of the weights.  So logical tile
    // numbers are handed out in blocks of 256, XCD i taking numbers 32 i .. 32 i + 31 of each block, and inside an
    // expert the numbering is (panel of 8 row tiles, column tile, row tile in the panel), innermost fastest: an XCD
    // then works on 8 row tiles x 4 column tiles at a time (12 distinct operand tiles instead of 33).
    const int64_t j = blockIdx.x / kXcds;
    int64_t L = (j / 32) * (32 * kXcds) + (int64_t)(blockIdx.x % kXcds) * 32 + j % 32;
    // With RAGGED_LAST the whole tiles of all experts are numbered first and the ragged last tiles of the segments
    // after them, the one with the most rows first: a launch rarely fills its last round of workgroups, and this way
    // that round consists of the tiles that cost least.  The price: a ragged tile no longer shares its weight tile's
    // trip through the L2 with the other row tiles of its panel, so the host asks for it only when the ragged tiles are
    // few (at most one round of workgroups).
    int64_t whole = 0;
    const ExpertTileHit hit = RAGGED_LAST ? find_expert_tile<BM, true>(a, nct, L, lane, &whole)
                                          : find_expert_tile<BM, false>(a, nct, L, lane);
    constexpr int WST = DEEP_W ? 3 : 2;                            // stages of w
    int e = hit.e, row0 = 0, row_end = 0, ct = 0;
    int sharers = 1, share = 0;                                    // row tiles side by side on one weight tile; which of them
    int alone = 0;                                                 // 1: the tile holds all rows of its expert
    if (e < a.E) {
        const int tiles = hit.tiles, full = tiles / P;             // whole panels
        int rt;
        if (hit.L < (int64_t)full * P * nct) {
            const int p = (int)(hit.L / (uint32_t)(P * nct)), rem = (int)(hit.L % (uint32_t)(P * nct));
            ct = rem / P;
            share = rem % P;
            rt = p * P + share;
            sharers = P;
        } else {
            const int rem = (int)(hit.L - (int64_t)full * P * nct), pr = tiles - full * P;
            ct = rem / pr;
            share = rem % pr;
            rt = full * P + share;
            sharers = pr;
        }
        row0 = hit.lo + rt * BM;
        row_end = hit.hi < a.max_rows ? hit.hi : a.max_rows;
        alone = hit.hi - hit.lo <= BM;
    } else if (RAGGED_LAST) {
        // ragged tiles: position L / nct in the order (rows in the ragged tile, descending; expert, ascending).  The
        // tile buffers are not in use yet, so their first bytes serve as the scratch of the ranking (E <= 256).
        // Those of at most 64 rows, the last ones, are split into halves of 128 columns: they last as long as their weights
        // take to arrive, and twice the workgroups have twice the loads on their way.
        const int64_t Lr = L - whole;
        int *scr = reinterpret_cast<int *>(big_lds);
        int my_rem = 0;
        if (tid < a.E) {
            const int lo = a.lo[tid], hi = a.hi_base[tid] + (a.hi_len ? a.hi_len[tid] : 0);
            my_rem = hi > lo ? (int)(((int64_t)hi - lo) % BM) : 0;
            scr[tid] = my_rem;
        }
        if (tid == 0) scr[256] = -1;
        __syncthreads();
        int rank = 0, long_ones = 0;
        for (int o = 0; o < a.E; ++o) {
            const int ro = scr[o];
            long_ones += ro > kShortRows ? 1 : 0;
            rank += (ro > my_rem || (ro == my_rem && o < tid)) ? 1 : 0;
        }
        const int64_t halves = Lr - (int64_t)long_ones * nct;      // number among the half tiles
        if (my_rem > 0 && rank == (halves < 0 ? Lr / nct : long_ones + halves / (2 * nct))) scr[256] = tid;
        __syncthreads();
        const int eh = scr[256];
        __syncthreads();                                           // everyone has read it before the tiles stream in
        if (eh >= 0 && eh < a.E) {
            e = eh;
            const int lo = a.lo[e], hi = a.hi_base[e] + (a.hi_len ? a.hi_len[e] : 0);
            ct = (int)(halves < 0 ? Lr % nct : halves % (2 * nct));
            row0 = lo + (int)(((int64_t)hi - lo) / BM) * BM;
            row_end = hi < a.max_rows ? hi : a.max_rows;
            alone = row0 == lo;
        }
    }
    // the same for the whole workgroup: into scalar registers
    e = __builtin_amdgcn_readfirstlane(e);
    row0 = __builtin_amdgcn_readfirstlane(row0);
    row_end = __builtin_amdgcn_readfirstlane(row_end);
    sharers = __builtin_amdgcn_readfirstlane(sharers);
    share = __builtin_amdgcn_readfirstlane(share);
    ct = __builtin_amdgcn_readfirstlane(ct);
    // Streamed weights only in the form whose tiles mostly have one user and whose rows are whole lines.
    constexpr bool kMayStream = DEEP_W && !TAIL;
    if (e >= a.E || row0 < 0 || row0 >= row_end) return;          // surplus workgroup
    constexpr int kShortCols = RAGGED_LAST ? 128 : 256, kStages = RAGGED_LAST ? 5 : 3;
    static_assert(ShortTile<64, kShortCols, kStages>::kLdsBytes <= big_lds_bytes(DEEP_W), "short tile: stages must fit the kernel's LDS");
    const int xr = min(row_end - row0, BM);
    const int cols = xr <= kShortRows ? kShortCols : BN, col0 = ct * cols;
    if (col0 >= a.N) return;                                       // the second half of a last column tile may be empty
    const bool stream = kMayStream && (int64_t)e * a.N + col0 >= a.stream_from && __builtin_amdgcn_readfirstlane(alone);
    const uint32_t rowb = (uint32_t)cpr * 16;
    const int wr = min(a.N - col0, cols);
    // by the expert, in tiles of every kind: a row may be in a large tile of one launch and in a short one of another
    const int start = DEEP_W && !TAIL && a.spread ? walk_start(e, nsteps) : 0;
    const auto rx = make_rsrc(x + (int64_t)row0 * cpr, (uint32_t)xr * rowb);
    const auto rw = make_rsrc(w + ((int64_t)e * a.N + col0) * cpr, (uint32_t)wr * rowb);
    if (xr <= kShortRows) {                                        // tiles with little arithmetic
        if (kMayStream && stream)
            expert_short_tile<64, kShortCols, kStages, false, false, kMayStream ? kStreamLoad : 0>(rx, rw, y, cpr, a.N, row0, row_end, col0, big_lds, start);
        else
            expert_short_tile<64, kShortCols, kStages, false, false>(rx, rw, y, cpr, a.N, row0, row_end, col0, big_lds, start);
        return;
    }

    // A step's tile is chunks of 8 rows (1 KiB), 32 of w and, as far as there are rows, of x; a wave fetches 8 neighbouring chunks of w and
    // an equal share of those of x.
    const int lr = lane >> 3;
    auto first_offset = [&](int chunk) { return (uint32_t)(chunk * 8 + lr) * rowb + (((lane & 7) ^ ((chunk * 4 + (lr >> 1)) & 7)) * 16); };
    uint32_t off_w[2], off_x[2];                                  // chunks 16 rows apart have the same swizzle
#pragma unroll
    for (int q = 0; q < 2; ++q) off_w[q] = first_offset(wave * 8 + q);
    auto off = [&](const uint32_t(&first)[2], int q) {
        uint32_t rows = (uint32_t)(q >> 1) * (16 * rowb);
        asm volatile("" : "+s"(rows));                             // added at each use: eight offsets kept would be spilled
        return first[q & 1] + rows;
    };
    // Before the first loads of step `step`, at whatever is the last step: the lane offsets of the pieces past the end of a row go
    // out of range, for good (what is loaded after them is the last step again, into buffers that are not read any more).
    auto trim = [&](int step) {
        if constexpr (TAIL) {
            const int left = step >= nsteps - 1 ? cpr - (nsteps - 1) * 8 : 8;
            int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
            asm volatile("" : "+v"(l));                            // found again each time: kept, the pieces would be spilled
#pragma unroll
            for (int q = 0; q < 2; ++q)                            // rows 8 apart: pieces 4 apart, the wave's 64 rows make no difference
                off_w[q] |= ((l & 7) ^ ((4 * q + (l >> 4)) & 7)) >= left ? kOutOfRange : 0u;
        }
    };
    unsigned char *const w_lds = big_lds + 2 * kBigXBytes;
    auto issue_w = [&](int q, uint32_t so, int at) {              // `at`: byte offset of the stage among those of w (of x)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(w_lds + at + (wave * 8 + q) * 1024), 16, off(off_w, q), so, 0, 0);
    };
    auto stream_w = [&](int q, uint32_t so, int at) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(w_lds + at + (wave * 8 + q) * 1024), 16, off(off_w, q), so, 0, kStreamLoad);
    };

    // the early touches (not with the third stage of w)
    const uint32_t touch_w = lane * sharers / 64 == share ? (uint32_t)(wave * 64 + lane) * rowb : kOutOfRange;
    const uint32_t touch_x = lane < 16 ? (uint32_t)((ct & 3) * 64 + wave * 16 + lane) * rowb : kOutOfRange;

    // The waves form a 2 x 2 grid.  In a ragged tile the rows are split evenly between the two row halves: nb 16-row
    // blocks each, at least 4.  The loop is compiled for each count: only rows in use are requested, read and multiplied, all spread evenly
    // under the MFMAs (64 experts of 7168 x 2048, 160 and 224 rows: 384 and 548 us with one loop for all counts, 376 and 534).
    const int m = lane & 15, g = lane >> 4, wm = wave >> 1, wn = wave & 1;
    const int nb = max((xr + 31) / 32, 4);
    f32x4 acc[8][8];                                               // [16-row block of x][16 output features]
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int n = 0; n < 8; ++n) acc[i][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const unsigned char *pw = w_lds + (wn * 128 + m) * 128;
    const int k0 = (g ^ ((m >> 1) & 7)) * 16, k1 = ((4 + g) ^ ((m >> 1) & 7)) * 16;      // this lane's piece, slice 0 and 1
    bf16x8 fx[2][8], fw[2][8];
    // no instruction near it reads the accumulator: the next MFMA on the same one is a whole slice away, and the epilogue
    // waits first
    auto mma = [&](int set, int i, int n) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][n]) : "v"(fw[set][n]), "v"(fx[set][i]));
    };
    auto barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // All steps of a tile of NB row blocks per half
    auto run = [&](auto nbc, auto load_w) {
        constexpr int NB = decltype(nbc)::value;
        constexpr int XL = TAIL ? 8 : NB;                          // loads of x per wave and step (TAIL: of all 256 rows, one trim for both)
        constexpr int kYoungerStage = DEEP_W ? 8 : 2, kYoungerFirst = XL + 8 + (DEEP_W ? 8 : 0);
        constexpr int kWaitStage = 0x0070 | kYoungerStage, kWaitFirst = 0x0f70 | (kYoungerFirst & 15) | (kYoungerFirst >> 4 << 14);
        const unsigned char *px = big_lds + (wm * NB * 16 + m) * 128;
        if constexpr (XL < 8) {
#pragma unroll
            for (int q = 0; q < 2; ++q) off_x[q] = first_offset(wave * XL + q);
        }
        auto issue_x = [&](int q, uint32_t so, int at) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)(big_lds + at + (wave * XL + q) * 1024), 16, off(XL == 8 ? off_w : off_x, q), so, 0, 0);
        };
        auto touch = [&](uint32_t so) {
            if constexpr (!DEEP_W) {
                lds_void *sink = (lds_void *)(w_lds + 2 * kBigWBytes + wave * 512);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, sink, 4, touch_w, so, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, sink, 4, touch_x, so, 0, 0);
            }
        };
        auto read = [&](int set, int r, int xat, int wat, int ko) {
            if (r < 8) fw[set][r] = *reinterpret_cast<const bf16x8 *>(pw + wat + ko + r * 2048);
            else fx[set][r - 8] = *reinterpret_cast<const bf16x8 *>(px + xat + ko + (r - 8) * 2048);
        };
        // One slice: 8 NB MFMAs on fragment set `set`; spread between them the 8 + NB reads of the other set (stages at xat and wat, piece
        // offset ko) and, if LOADS, the loads of x at column `xso` and then the 8 of w at `wso`, into the stages at xto and wto.
        auto slice = [&](int set, int xat, int wat, int ko, bool loads, uint32_t xso, int xto, uint32_t wso, int wto, int trim_x, int trim_w) {
#pragma unroll
            for (int q = 0; q < 2 * NB; ++q) {
#pragma unroll
                for (int r = q * (8 + NB) / (2 * NB); r < (q + 1) * (8 + NB) / (2 * NB); ++r) read(set ^ 1, r, xat, wat, ko);
                mma(set, q / 2, (q & 1) * 4 + 0);
                mma(set, q / 2, (q & 1) * 4 + 1);
                if (loads) {
#pragma unroll
                    for (int l = q * (XL + 8) / (2 * NB); l < (q + 1) * (XL + 8) / (2 * NB); ++l) {
                        if (l == 0 && !DEEP_W) trim(trim_x);
                        if (l == XL && DEEP_W) trim(trim_w);
                        if (l < XL) issue_x(l, xso, xto);
                        else load_w(l - XL, wso, wto);
                    }
                }
                mma(set, q / 2, (q & 1) * 4 + 2);
                mma(set, q / 2, (q & 1) * 4 + 3);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // the columns of the steps that are requested next: from `start` round, past the end the last one again
        const uint32_t turn = (uint32_t)nsteps * 128u;
        auto column = [&](int step) {
            const uint32_t at = (uint32_t)(min(step, nsteps - 1) + start) * 128u;
            if constexpr (!DEEP_W || TAIL) return at;
            return at >= turn ? at - turn : at;
        };
        trim(0);
#pragma unroll
        for (int q = 0; q < XL + 8; ++q) {                        // x and w in turn, then the rest of w
            if (q < 2 * XL && !(q & 1)) issue_x(q / 2, column(0), 0);
            else load_w(q < 2 * XL ? q / 2 : q - XL, column(0), 0);
        }
        trim(1);
#pragma unroll
        for (int q = 0; q < XL + 8; ++q) {
            if (q < 2 * XL && !(q & 1)) issue_x(q / 2, column(1), kBigXBytes);
            else load_w(q < 2 * XL ? q / 2 : q - XL, column(1), kBigWBytes);
        }
        if constexpr (DEEP_W) {
            trim(2);
#pragma unroll
            for (int q = 0; q < 8; ++q) load_w(q, column(2), 2 * kBigWBytes);
        }
        __builtin_amdgcn_s_waitcnt(kWaitFirst);                    // stage 0
        touch(column(2));
        barrier();
#pragma unroll
        for (int r = 0; r < 8 + NB; ++r) read(0, r, 0, 0, k0);
        int xat = 0, wat = 0;                                      // where stage s is
        for (int s = 0; s < nsteps; ++s) {
            slice(0, xat, wat, k1, false, 0, 0, 0, 0, 0, 0);
            // lgkmcnt(0): this wave has read all of stage s; vmcnt: stage s+1 is in LDS, younger are only the 8 loads of w for stage
            // s+2 or the early touches
            __builtin_amdgcn_s_waitcnt(kWaitStage);
            barrier();
            // past the end the last stage is fetched again, into buffers that are not read any more
            const int wnext = wat == (WST - 1) * kBigWBytes ? 0 : wat + kBigWBytes;
            slice(1, xat ^ kBigXBytes, wnext, k0, true, column(s + 2), xat, column(s + WST), wat, min(s + 2, nsteps - 1), min(s + WST, nsteps - 1));
            touch(column(s + 3));
            xat ^= kBigXBytes;
            wat = wnext;
        }
    };
    auto run_nb = [&](auto load_w) {
        if (nb == 8) run(std::integral_constant<int, 8>{}, load_w);
        else if (nb == 7) run(std::integral_constant<int, 7>{}, load_w);
        else if (nb == 6) run(std::integral_constant<int, 6>{}, load_w);
        else if (nb == 5) run(std::integral_constant<int, 5>{}, load_w);
        else run(std::integral_constant<int, 4>{}, load_w);
    };
    if constexpr (kMayStream) {
        if (stream) run_nb(stream_w);
        else run_nb(issue_w);
    } else {
        run_nb(issue_w);
    }
    asm volatile("s_nop 15\n\ts_nop 15");                          // the last MFMAs' results
    __builtin_amdgcn_sched_barrier(0);

    // acc[i][n][v]: row 16 i + lane % 16 of the wave's rows, output feature 16 n + 4 (lane / 16) + v of its columns.  The lane is
    // asked for again: kept in a register through the loop it would be spilled.
    const int l2 = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = row0 + (wm * nb + i) * 16 + (l2 & 15);
        if (i < nb && r < row_end) {
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int c = col0 + wn * 128 + n * 16 + 4 * (l2 >> 4);
                if (c < a.N) *reinterpret_cast<uint2 *>(y + (int64_t)r * a.N + c) = pack_bf16x4(acc[i][n]);
            }
        }
    }
#else
    (void)x;
    (void)w;
    (void)y;
    (void)a;
#endif
}

// Gate projection of a few thousand tokens, of short rows, and in fp32 of many experts: the same tiles, tokens x experts, sums
// stored as they are.  Bound by the trips of x and of the weights through the L2: T E row (1 / XR + 1 / WR) bytes, in fp32 by the
// matrix rate.  Against 32-token workgroups with the k-slices dealt to 8 waves: 16384 x 7168, 256 experts 190 -> 91 us, 8192 x 4096,
// 256 experts 61 -> 37, 1024 x 7168, 256 experts 92 -> 35; rows that are not whole steps: 1024 x 8184, 256 experts 109 -> 29, 12000 x
// 520, 9 experts 12.5 -> 5.8.  Against persistent workgroups of whole rows: 65536 x 512, 8 experts 49 -> 13.  fp32 against tiles of
// 16 tokens x 64 experts with a split hidden axis: 8192 x 4096, 128 experts 171 -> 99, 32000 x 8192, 64 experts 694 -> 333.
// SPREAD: the row tiles' walks begin at different even steps; rows of whole pairs of steps.
template <int XR, int WR, int NST, bool F32, bool SPREAD>
__global__ __launch_bounds__(256, 2) void gate_short_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                            float *__restrict__ logits, int64_t T, int H, int E)
{
    extern __shared__ __align__(16) unsigned char gshort_lds[];
    const int nct = (E + WR - 1) / WR, cpr = F32 ? H / 4 : H / 8;
    const int64_t t0 = (int64_t)(blockIdx.x / nct) * XR;
    const int e0 = (int)(blockIdx.x % nct) * WR;
    const int64_t t1 = t0 + XR < T ? t0 + XR : T;
    const uint32_t rowb = (uint32_t)cpr * 16;
    expert_short_tile<XR, WR, NST, F32, false, 0, SPREAD>(make_rsrc(x + t0 * cpr, (uint32_t)(t1 - t0) * rowb),
                                                          make_rsrc(w + (int64_t)e0 * cpr, (uint32_t)min(E - e0, WR) * rowb), logits, cpr, E, t0,
                                                          t1, e0, gshort_lds, SPREAD ? walk_start((int)(blockIdx.x / nct), cpr / 8) & ~1 : 0);
}

// Gate projection of few tiles, bf16, rows of 456 elements (eight steps) and more: the expert layer's split tiles, tokens x experts.  Against
// waves that stream their shares straight into registers, 64 bytes of 16 rows a load (gate_split_kernel), and against 32 x 64 tiles: 16 x
// 7168, 64 experts 15.5 -> 5.6 us, 300 x 7168, 256 experts 21.8 -> 9.9, 512 x 7168, 64 experts 15.9 -> 7.8, 1024 x 8192, 256 experts 28.6 -> 20.1.
template <int XB, int CB, int W, int NST>
__global__ __launch_bounds__(64 * W) void gate_ring_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w, float *__restrict__ logits,
                                                           int64_t T, int cpr, int E)
{
    extern __shared__ __align__(16) unsigned char ring_lds[];
    const int nct = (E + 16 * CB - 1) / (16 * CB);
    const int64_t t0 = (int64_t)(blockIdx.x / nct) * (16 * XB), t1 = t0 + 16 * XB < T ? t0 + 16 * XB : T;
    const int e0 = (int)(blockIdx.x % nct) * (16 * CB);
    const uint32_t rowb = (uint32_t)cpr * 16;
    split_tile<XB, CB, W, NST, false, false>(make_rsrc(x + t0 * cpr, (uint32_t)(t1 - t0) * rowb), make_rsrc(w + (int64_t)e0 * cpr, (uint32_t)min(E - e0, 16 * CB) * rowb),
                                             logits, cpr, E, t0, t1, e0, ring_lds);
}

// Gate projection with the hidden axis split over the 8 waves of a workgroup: 16 tokens x 16 NB experts each.  For fp32
// activations (16x16x4 fp32 MFMA) and for so few bf16 tokens that a tile's walk along the whole hidden axis is what takes the
// time, where gate_ring_kernel is not taken (rows below 456 elements or beyond 2^20, activations of more than 96 MiB).  A wave streams its
// share straight into registers, D steps of 128 bytes per row ahead; lane l holds 16 bytes of row l % 16, at the same place of x and of
// w, so which element of the hidden axis meets which MFMA does not matter.  The waves'
// sums are added through LDS in a fixed order.  Rows past the end repeat the last one and are not stored.  Steps past a
// wave's share multiply zeros: an MFMA takes no notice of a lane mask, so it may not stand under a condition that the
// compiler cannot prove uniform.
// Measured, fp32, a wave per token and eight experts at a time before: 8192 x 4096, 8 / 64 experts 48 / 325 -> 26 / 75.
template <bool BF16, int NB>
__global__ __launch_bounds__(512) void gate_split_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                         float *__restrict__ logits, int64_t T, int64_t cpr, int E)
{
    constexpr int D = NB == 1 ? 4 : NB == 2 ? 3 : 2, W = 8;
    __shared__ f32x4 red[W][NB][kWave];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), m = lane & 15, g = lane >> 4;
    const int nct = (E + 16 * NB - 1) / (16 * NB);
    const int64_t t0 = (int64_t)(blockIdx.x / nct) * 16;
    const int e0 = (int)(blockIdx.x % nct) * 16 * NB;
    const u32x4 *px = x + (t0 + m < T ? t0 + m : T - 1) * cpr + g;
    const u32x4 *pw[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) pw[n] = w + (int64_t)(e0 + n * 16 + m < E ? e0 + n * 16 + m : E - 1) * cpr + g;

    // C independent sums per result (by half of the step and, in fp32, by element of a piece): no MFMA waits for the one
    // before it, and the chains of additions stay short
    constexpr int C = BF16 ? 2 : 8;
    f32x4 acc[NB][C];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[n][c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int n, int h, u32x4 fw, u32x4 fx) {
        if constexpr (BF16) {
            acc[n][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fw), __builtin_bit_cast(bf16x8, fx),
                                                                acc[n][h], 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[n][4 * h + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(fw[i]), __uint_as_float(fx[i]),
                                                                         acc[n][4 * h + i], 0, 0, 0);
        }
    };
    // whole steps: 8 pieces of 16 bytes per row, pieces g and 4 + g for this lane; steps past the wave's share multiply zeros
    const int nsteps = (int)(cpr / 8), first = (int)((int64_t)nsteps * wave / W), last = (int)((int64_t)nsteps * (wave + 1) / W);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    u32x4 fx[D][2], fw[D][NB][2];
    auto fetch = [&](int d, int step) {
        const int64_t c = (int64_t)min(step, nsteps - 1) * 8;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            fx[d][h] = px[c + 4 * h];
#pragma unroll
            for (int n = 0; n < NB; ++n) fw[d][n][h] = pw[n][c + 4 * h];
        }
    };
    if (first < last) {
#pragma unroll
        for (int d = 0; d < D; ++d) fetch(d, first + d);
        for (int s = first; s < last; s += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        mma(n, h, s + d < last ? fw[d][n][h] : zero, s + d < last ? fx[d][h] : zero);
                fetch(d, s + d + D);
            }
        }
    }
    if (wave == W - 1 && cpr % 8) {                                // the rest of the row: what lies past it counts as zero
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t c = (int64_t)nsteps * 8 + 4 * h;
            const bool in = c + g < cpr;
            const u32x4 vx = in ? px[c] : zero;
#pragma unroll
            for (int n = 0; n < NB; ++n) mma(n, h, in ? pw[n][c] : zero, vx);
        }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
#pragma unroll
        for (int d = C / 2; d >= 1; d /= 2)
#pragma unroll
            for (int c = 0; c < d; ++c) acc[n][c] += acc[n][c + d];
        red[wave][n][lane] = acc[n][0];
    }
    __syncthreads();
    for (int n = wave; n < NB; n += W) {
        f32x4 sum[W];
#pragma unroll
        for (int v = 0; v < W; ++v) sum[v] = red[v][n][lane];
#pragma unroll
        for (int d = W / 2; d >= 1; d /= 2)
#pragma unroll
            for (int v = 0; v < d; ++v) sum[v] += sum[v + d];
        if (t0 + m < T) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int e = e0 + n * 16 + 4 * g + v;
                if (e < E) logits[(t0 + m) * E + e] = sum[0][v];
            }
        }
    }
}

// fp32 rows of more than kBigMaxHidden elements, whose tiles do not fit the 31-bit offsets of the direct loads: a 64 x 64 tile of y
// per workgroup of 4 waves (each 32 x 32, one accumulator of the 32x32x2 fp32 MFMA), 32 elements of the hidden axis per step through
// registers into LDS.  A lane takes four consecutive elements of its row with one LDS read: half g of the wave elements 8 p + 4 g ..
// + 3, element i of both halves in MFMA i.  Rows are padded by 16 bytes.  One step in flight: 108 us for 8 rows of 4096 x 4096, where
// the tiles above take 50.
constexpr int kF32Tile = 64, kF32Step = 32, kF32RowStride = kF32Step * 4 + 16;

__global__ __launch_bounds__(256) void expert_f32_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ w,
                                                         float *__restrict__ y, ExpertArgs a)
{
    __shared__ __align__(16) unsigned char f32_lds[2 * kF32Tile * kF32RowStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 31, g = lane >> 5;
    const int cpr = a.H / 4, nct = (a.N + kF32Tile - 1) / kF32Tile;
    const int64_t j = blockIdx.x / kXcds;
    const int64_t L = (j / 32) * (32 * kXcds) + (int64_t)(blockIdx.x % kXcds) * 32 + j % 32;
    const ExpertTileHit hit = find_expert_tile<kF32Tile>(a, nct, L, lane);
    if (hit.e >= a.E) return;                                      // surplus workgroup
    const int row0 = hit.lo + (int)(hit.L % (uint32_t)hit.tiles) * kF32Tile, col0 = (int)(hit.L / (uint32_t)hit.tiles) * kF32Tile;
    const int row_end = hit.hi < a.max_rows ? hit.hi : a.max_rows;
    if (row0 < 0 || row0 >= row_end) return;

    // piece q of this thread: row tid / 8 + 32 q of the step's tile (x rows, then weight rows), 16-byte column tid % 8.
    // Loads go out unconditionally from clamped addresses; what lies outside becomes zeros in LDS.
    const int pr = tid >> 3, pc = tid & 7;
    const u32x4 *src[4];
    bool live[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = pr + 32 * (q & 1);
        if (q < 2) {
            live[q] = row0 + r < row_end;
            src[q] = x + (int64_t)(live[q] ? row0 + r : row0) * cpr;
        } else {
            live[q] = col0 + r < a.N;
            src[q] = w + ((int64_t)hit.e * a.N + (live[q] ? col0 + r : col0)) * cpr;
        }
    }
    const int nsteps = (cpr + 7) / 8;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    u32x4 pre[4];
    auto fetch = [&](int step) {
        const int c = step * 8 + pc;
#pragma unroll
        for (int q = 0; q < 4; ++q) pre[q] = src[q][c < cpr ? c : 0];
    };
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const int wm = wave >> 1, wn = wave & 1;
    const bool rows = row0 + wm * 32 < row_end;                    // does this wave's half of the tile hold rows
    const unsigned char *pa = f32_lds + (wm * 32 + m) * kF32RowStride + g * 16;
    const unsigned char *pb = f32_lds + (kF32Tile + wn * 32 + m) * kF32RowStride + g * 16;
    fetch(0);
    for (int step = 0; step < nsteps; ++step) {
        const bool col_ok = step * 8 + pc < cpr;
        __syncthreads();                                           // the previous tile has been read by every wave
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<u32x4 *>(f32_lds + (pr + 32 * q) * kF32RowStride + pc * 16) = live[q] && col_ok ? pre[q] : zero;
        __syncthreads();
        fetch(step + 1);                                           // in flight during the MFMAs; past the end never used
        if (rows) {
#pragma unroll
            for (int p = 0; p < kF32Step / 8; ++p) {
                const f32x4 fa = *reinterpret_cast<const f32x4 *>(pa + p * 32), fb = *reinterpret_cast<const f32x4 *>(pb + p * 32);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[i], acc, 0, 0, 0);
            }
        }
    }
    // element v: row (v / 4) * 8 + g * 4 + v % 4, column m
    const int n = col0 + wn * 32 + m;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = row0 + wm * 32 + (v >> 2) * 8 + g * 4 + (v & 3);
        if (r < row_end && n < a.N) y[(int64_t)r * a.N + n] = acc[v];
    }
}

// ------------------------------------------------------------- plain copy

__global__ __launch_bounds__(kMoverThreads) void copy_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst,
                                                             size_t nvec)
{
    const size_t stride = (size_t)gridDim.x * kMoverThreads * kVecInFlight;
    for (size_t base = (size_t)blockIdx.x * kMoverThreads * kVecInFlight + threadIdx.x; base < nvec; base += stride) {
        u32x4 val[kVecInFlight];
#pragma unroll
        for (int q = 0; q < kVecInFlight; ++q)
            if (base + (size_t)q * kMoverThreads < nvec) val[q] = ld16<true>(src + base + (size_t)q * kMoverThreads);
#pragma unroll
        for (int q = 0; q < kVecInFlight; ++q)
            if (base + (size_t)q * kMoverThreads < nvec) st16<true>(dst + base + (size_t)q * kMoverThreads, val[q]);
    }
}

}  // namespace monta
