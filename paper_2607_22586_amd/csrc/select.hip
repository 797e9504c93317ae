// tau-sets, votes, anchor score and budgeted selection (Sec. 3.2.2 Eqs. 9-10,
// Sec. 3.2.3 Eq. 11, Algorithm 1) on gfx950.
//
// tau_cut   one workgroup per (b, c, group): a mass-weighted radix select on
//           the fp32 bit patterns of the group masses (non-negative floats
//           order like their bits; 11/11/9-bit digits below the sign bit)
//           finds the cut mass theta and, among keys whose mass equals theta,
//           the last admitted index, such that
//           {mass > theta} u {mass == theta, index <= tcut} is the shortest
//           (mass desc, index asc) prefix whose mass reaches tau * total.
//           Masses are summed as integers in units of 2^-S (converted from
//           the float bits exactly), so every decision is independent of
//           summation order.  The register-resident variant (T <= 65536)
//           and the sweep beyond stop their passes early once the crossing
//           bucket holds one key, and end by writing the group's membership
//           plane: one bit per key, 32 keys a word.
// vote      vote = #groups whose set holds the key, counted from the planes'
//           words; score = vote + lambda*anchor (fp64), or the total mass; and
//           per head the counts of the scores' first digits for the top-k.
// topk      one workgroup per (b, c): the bucket of the vote kernel's counts
//           that holds the (C-1)-th largest score key over [0, T-1) (or the
//           C-th over [0, T)), a radix select among that bucket's keys (11-bit
//           digits, stopping early once a bucket is taken whole), then an
//           index-ordered compaction writes the kept tokens in ascending
//           order and appends token T-1.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace mmskv {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kTauThreads = 512;                 // register-resident tau cut

// floor(m * 2^S) for the finite, non-negative float with bit pattern `bits`,
// computed exactly from the significand and exponent (the product m * 2^S
// stays below 2^63 for every mass the score pass can produce).
__device__ __forceinline__ uint64_t fixed_of(uint32_t bits, int S) {
    const uint32_t e = (bits >> 23) & 0xFFu;
    const uint64_t man = static_cast<uint64_t>((bits & 0x7FFFFFu) | (e != 0 ? 0x800000u : 0u));
    // value = man * 2^(e - 150) (normal) or man * 2^-149 (subnormal)
    const int sh = (e != 0 ? static_cast<int>(e) : 1) - 150 + S;
    if (sh >= 0) return man << sh;
    if (sh <= -24) return 0ull;
    return man >> (-sh);
}

// The fixed-point value floor(m * 2^S) of a non-negative float m = man *
// 2^(e' - 150) (e' = max(e, 1), man with the implicit bit when e > 0) is
// man << sh for sh = e' - 150 + S >= 0 and man >> -sh otherwise.  Every key
// in one bucket of the tau-cut passes has the same exponent (the first digit
// holds the exponent bits, the later passes keep them in the prefix), so a
// bucket can sum mant_part(bits) = man >> max(-sh, 0) (under 2^24) and take
// the common factor 2^max(sh, 0) once: bucket_fixed(sum, e) is then exactly
// the sum of fixed_of over the bucket.
__device__ __forceinline__ int fixed_shift(uint32_t e, int S) {
    return (e != 0 ? static_cast<int>(e) : 1) - 150 + S;
}
__device__ __forceinline__ uint32_t mant_part(uint32_t bits, int S) {
    const uint32_t e = bits >> 23;           // sign bit is 0
    const uint32_t man = (bits & 0x7FFFFFu) | (e != 0 ? 0x800000u : 0u);
    const int rs = -fixed_shift(e, S);
    return rs <= 0 ? man : (rs >= 24 ? 0u : man >> rs);
}
__device__ __forceinline__ uint64_t bucket_fixed(uint64_t sum, uint32_t e, int S) {
    const int sh = fixed_shift(e, S);
    return sh > 0 ? sum << min(sh, 63) : sum;   // sh stays below 40 for any non-empty bucket
}

// Block-wide exclusive prefix count of `flag` over the NT threads in thread
// order; returns the prefix and writes the block total.
template <int NT = kSelThreads>
__device__ __forceinline__ uint32_t block_excl_count(bool flag, uint32_t* wtot, uint32_t& total) {
    constexpr int kW = NT / kWave;
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const uint64_t m = __ballot(flag);
    const uint32_t below = static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
    if (lane == 0) wtot[wave] = static_cast<uint32_t>(__popcll(m));
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int w = 0; w < kW; ++w) {
        const uint32_t x = wtot[w];
        before += (w < wave) ? x : 0u;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return before + below;
}

// Block-wide exclusive prefix sum of `v` over the NT threads in thread
// order; also returns the block total.
template <typename U, int NT = kSelThreads, bool kFence = true>
__device__ __forceinline__ U block_excl_scan(U v, U* wtot, U& total) {
    constexpr int kW = NT / kWave;
    const int lane = lane_id(), wave = static_cast<int>(threadIdx.x) / kWave;
    const U x = wave_incl_scan(v);
    if (lane == kWave - 1) wtot[wave] = x;
    __syncthreads();
    U before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
        const U t = wtot[w];
        before += (w < wave) ? t : U(0);
        tot += t;
    }
    // without kFence the caller puts a barrier before wtot is written again
    if (kFence) __syncthreads();
    total = tot;
    return before + x - v;
}

// Digits [0, 2048) visited in descending order, thread i of NT covering the
// 2048/NT digits below 2048 - (2048/NT)*i, bucket d holding val_of(d): finds
// the digit whose bucket takes the running total (from the top) to need =
// need_of(total of all buckets) (1 <= need <= total; no digit when need is
// 0).  Returns the total; writes, through shared memory, the digit, `need`
// minus the total of higher buckets, and the bucket's count cnt_of(digit).
template <typename U, int NT, typename ValOf, typename CntOf, typename NeedOf>
__device__ __forceinline__ U crossing_of(ValOf val_of, CntOf cnt_of, NeedOf need_of, U* wtot,
                                         uint32_t* s_digit, U* s_rem, uint32_t* s_cnt) {
    constexpr int kPer = 2048 / NT;
    const int top = 2047 - kPer * static_cast<int>(threadIdx.x);
    U v[kPer];
    U mine = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        v[k] = val_of(top - k);
        mine += v[k];
    }
    U total;
    U excl = block_excl_scan<U, NT, false>(mine, wtot, total);   // the barrier below guards wtot
    const U need = need_of(total);
    if (excl < need && need <= excl + mine) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (excl < need && need <= excl + v[k]) {
                *s_digit = top - k;
                *s_rem = need - excl;
                *s_cnt = cnt_of(top - k);
            }
            excl += v[k];
        }
    }
    __syncthreads();
    return total;
}

template <typename U, int NT = kSelThreads>
__device__ __forceinline__ void descending_crossing(const U* val, const uint32_t* cnt, U need, U* wtot,
                                                    uint32_t* s_digit, U* s_rem, uint32_t* s_cnt) {
    crossing_of<U, NT>([val](int d) { return val[d]; }, [cnt](int d) { return cnt[d]; }, [need](U) { return need; },
                       wtot, s_digit, s_rem, s_cnt);
}

// tau-cut digits: bits 30..20, 19..9, 8..0 of the (sign-free) mass bits.
__device__ __forceinline__ int tau_shift(int pass) { return pass == 0 ? 20 : pass == 1 ? 9 : 0; }
__device__ __forceinline__ uint32_t tau_mask(int pass) { return pass == 0 ? 0u : pass == 1 ? 0xFFF00000u : 0xFFFFFE00u; }
__device__ __forceinline__ uint32_t tau_digit(uint32_t bits, int pass) {
    return (bits >> tau_shift(pass)) & (pass == 2 ? 0x1FFu : 0x7FFu);
}
// bits fixed once pass `pass` has chosen its digit
__device__ __forceinline__ uint32_t tau_fixed(int pass) {
    return pass == 0 ? 0xFFF00000u : pass == 1 ? 0xFFFFFE00u : 0xFFFFFFFFu;
}

// tau-set membership of key t for cut (theta, tcut): mass above the cut, or
// equal to it at an index up to tcut
__device__ __forceinline__ bool in_tau_set(uint32_t bits, int t, uint32_t theta, int32_t tcut) {
    return bits > theta || (bits == theta && t <= tcut);
}

// First digit (0..2047) of a score key, monotone in the score and fine where
// the scores lie.  VOTE mode: the whole part (votes), then, in digit_sub
// steps, the fraction (lambda * anchor, mostly far below 1) by its octave and
// 2^digit_q steps an octave; scores of G + 1 or more (lambda * anchor above
// 1) take the last digit.  MASS mode: 32 steps an octave from 2^-39 to 2^25.
// A key with the top bit set (a score of -0 or below) is above all others as a
// number and takes the last digit.
// (The top bits of the fp64 score would put all votes from 8 to 31, equal
// steps of the score all keys of one vote, into one bucket.)
__device__ __forceinline__ uint32_t key_digit(const SelectArgs& a, uint64_t key) {
    const double score = __longlong_as_double(static_cast<long long>(key));
    if (key >> 63) return 2047u;
    if (a.mode == 0) {
        const double whole = floor(score);
        if (!(whole <= static_cast<double>(a.G))) return 2047u;
        const int bits = __float_as_int(static_cast<float>(score - whole));
        const int sub = (bits >> (23 - a.digit_q)) - ((127 << a.digit_q) - a.digit_sub);
        return static_cast<uint32_t>(static_cast<int>(whole) * a.digit_sub + min(max(sub, 0), a.digit_sub - 1)) & 2047u;
    }
    const int d = (__float_as_int(static_cast<float>(score)) >> 18) - ((127 - 39) << 5);
    return static_cast<uint32_t>(min(max(d, 0), 2047));
}

// Group g's share of clearing the first-digit histogram of head hc (the
// vote kernel fills it).
__device__ __forceinline__ void clear_hist0_share(const SelectArgs& a, int64_t hc, int g) {
    const int lo = static_cast<int>((2048L * g) / a.G), hi = static_cast<int>((2048L * (g + 1)) / a.G);
    for (int i = lo + static_cast<int>(threadIdx.x); i < hi; i += static_cast<int>(blockDim.x)) a.hist0[hc * 2048 + i] = 0u;
}

// Word w of group g's membership plane of head hc.
__device__ __forceinline__ uint32_t* plane_word(const SelectArgs& a, int64_t hc, int g, int w) {
    const int nw = (a.T + 31) / 32;
    return a.planes + (hc * a.G + g) * nw + w;
}

// ---------------------------------------------------------------- tau cut
// Sweep form for rows too long for registers (T > 65536): every pass reads
// the group's masses again (from L2 when they fit), kSweepBatch loads per
// thread in flight.
constexpr int kSweepBatch = 8;

// f(t, bits of m[t]) for every key t of a row, the same trip count on every
// thread; t >= T (bits 0) marks a lane without a key (t is unsigned).
template <typename F>
__device__ __forceinline__ void sweep_row(const uint32_t* m, int T, F f) {
    // (unsigned: a batch of steps of 1024 keys may pass 2^31 - 1 at the longest rows)
    constexpr uint32_t kStep = kSelThreads * kSweepBatch;
    static_assert(static_cast<uint64_t>(INT32_MAX) + 2 * kStep <= UINT32_MAX, "row indices of a batch");
    const uint32_t n = static_cast<uint32_t>(T);
    for (uint32_t base = 0; base < n; base += kStep) {
        uint32_t v[kSweepBatch];
#pragma unroll
        for (int k = 0; k < kSweepBatch; ++k) {
            const uint32_t t = base + k * kSelThreads + threadIdx.x;
            v[k] = t < n ? m[t] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kSweepBatch; ++k) {
            // (uniform: whole waves past the row have nothing to do)
            if (base + k * kSelThreads < n) f(base + k * kSelThreads + threadIdx.x, v[k]);
        }
    }
}

__global__ void __launch_bounds__(kSelThreads) tau_cut_kernel(SelectArgs a) {
    __shared__ uint32_t cnt[2048];
    __shared__ unsigned long long sum[2048];
    __shared__ unsigned long long wtot64[kSelWaves];
    __shared__ uint32_t wtot[kSelWaves];
    __shared__ uint32_t s_digit, s_cnt, s_theta;
    __shared__ unsigned long long s_rem;
    __shared__ int32_t s_tcut;

    const int g = blockIdx.x, c = blockIdx.y, b = blockIdx.z;
    const int64_t hc = static_cast<int64_t>(b) * a.Hkv + c;
    const int64_t hcg = hc * a.G + g;
    const uint32_t* m = reinterpret_cast<const uint32_t*>(a.group_mass) + hcg * a.T;
    const int tid = threadIdx.x;
    const int S = a.fix_shift;
    const uint32_t n = static_cast<uint32_t>(a.T);
    clear_hist0_share(a, hc, g);

    // every mass below the fixed-point resolution: empty set
    uint32_t theta = 0xFFFFFFFFu;
    int32_t tcut = -1;
    unsigned long long need = 0;
    uint32_t prefix = 0;
    bool found = true;
    for (int pass = 0; pass < 3; ++pass) {
        const uint32_t mask = tau_mask(pass);
        for (int i = tid; i < 2048; i += kSelThreads) { cnt[i] = 0; sum[i] = 0; }
        __syncthreads();
        sweep_row(m, a.T, [&](uint32_t t, uint32_t bits) {
            if (t < n && (bits & mask) == prefix) {
                const uint32_t dg = tau_digit(bits, pass);
                atomicAdd(&cnt[dg], 1u);
                atomicAdd(&sum[dg], static_cast<unsigned long long>(mant_part(bits, S)));
            }
        });
        __syncthreads();
        const uint32_t e_pre = prefix >> 23;
        const unsigned long long total = crossing_of<unsigned long long, kSelThreads>(
            [&](int d) {
                return static_cast<unsigned long long>(
                    bucket_fixed(sum[d], pass == 0 ? static_cast<uint32_t>(d) >> 3 : e_pre, S));
            },
            [&](int d) { return cnt[d]; },
            [&](unsigned long long tot) {
                if (pass == 0) {
                    need = static_cast<unsigned long long>(ceil(a.tau * static_cast<double>(tot)));
                    if (need < 1) need = 1;
                    if (need > tot) need = tot;
                }
                return need;
            },
            wtot64, &s_digit, &s_rem, &s_cnt);
        if (pass == 0 && total == 0) {
            found = false;
            break;
        }
        prefix |= s_digit << tau_shift(pass);
        need = s_rem;
        if (pass < 2 && s_cnt == 1u) {
            // one key left in the crossing bucket: its mass is theta
            const uint32_t fixed = tau_fixed(pass);
            sweep_row(m, a.T, [&](uint32_t t, uint32_t bits) {
                if (t < n && (bits & fixed) == prefix) s_theta = bits;
            });
            __syncthreads();
            prefix = s_theta;
            break;
        }
    }
    if (found) {
        // keys with mass == theta each carry f_theta; the first k_eq by index
        // enter the set (all of them when k_eq covers the bucket)
        theta = prefix;
        const uint64_t f_theta = fixed_of(prefix, S);
        const uint64_t k_eq = f_theta == 0 ? 1 : (need + f_theta - 1) / f_theta;
        if (k_eq >= s_cnt) {
            tcut = a.T;
        } else {
            if (tid == 0) s_tcut = a.T - 1;
            __syncthreads();
            uint64_t seen = 0;
            for (int base = 0; base < a.T; base += kSelThreads) {
                const int t = base + tid;
                const bool eq = t < a.T && m[t] == prefix;
                uint32_t tot;
                const uint32_t before = block_excl_count(eq, wtot, tot);
                if (eq && seen + before + 1 == k_eq) s_tcut = t;
                seen += tot;
                if (seen >= k_eq) break;
            }
            __syncthreads();
            tcut = s_tcut;
        }
    }
    if (tid == 0) {
        a.theta[hcg] = theta;
        a.tcut[hcg] = tcut;
    }
    // membership plane: each wave's 64 consecutive keys are two words
    const int lane = lane_id();
    sweep_row(m, a.T, [&](uint32_t t, uint32_t bits) {
        const uint64_t mb = __ballot(t < n && in_tau_set(bits, static_cast<int>(t), theta, tcut));
        const uint32_t w = t / kWave * (kWave / 32) + lane;
        if (lane < 2 && 32 * w < n) *plane_word(a, hc, g, static_cast<int>(w)) = static_cast<uint32_t>(mb >> (32 * lane));
    });
}

// ---------------------------------------------------------------- vote + score
// One workgroup per 1024 keys of one head.  The membership words of 32
// groups at a time (a 128-byte line of each group's plane) are staged in LDS,
// one row per 32-key word; the 32 lanes that share a word read its row by
// broadcast, 4 groups a read, and each counts its own key's bit.  (One ballot
// per bit position and group word took 7.7 us a call for 16 heads of 16384
// keys, this 5.1: launch, load latency and the count histogram.)
constexpr int kVoteThreads = 256;
constexpr int kVoteWords = 32;                          // words per workgroup
constexpr int kVoteKeys = 32 * kVoteWords / kVoteThreads;   // keys per thread
constexpr int kVoteRow = 36;                            // words per LDS row (32 groups, 16-byte aligned)

__global__ void __launch_bounds__(kVoteThreads) vote_score_kernel(SelectArgs a) {
    __shared__ uint32_t lh[2048];            // this workgroup's first-digit counts
    __shared__ __align__(16) uint32_t pw[kVoteWords * kVoteRow];
    const int c = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int64_t hc = static_cast<int64_t>(b) * a.Hkv + c;
    const int nw = (a.T + 31) / 32;
    const int pool = a.keep_last ? a.T - 1 : a.T;
    const int w0 = static_cast<int>(blockIdx.x) * kVoteWords;
    const bool vote_mode = a.mode == 0;
    // key k of this thread: 32 w0 + 256 k + tid
    const int t0 = 32 * w0 + tid;
    float val[kVoteKeys];
    const float* src = vote_mode ? a.anchor : a.mass;
#pragma unroll
    for (int k = 0; k < kVoteKeys; ++k) {
        const int t = t0 + k * kVoteThreads;
        val[k] = t < a.T ? src[hc * a.T + t] : 0.f;
    }
    for (int i = tid; i < 2048; i += kVoteThreads) lh[i] = 0u;
    uint32_t vote[kVoteKeys] = {};
    if (vote_mode) {
        for (int g0 = 0; g0 < a.G; g0 += 32) {
            const int w = w0 + (tid & 31);
            uint32_t x[32 * kVoteWords / kVoteThreads];
#pragma unroll
            for (int k = 0; k < 32 * kVoteWords / kVoteThreads; ++k) {
                const int g = g0 + (tid >> 5) + k * (kVoteThreads / 32);
                x[k] = (w < nw && g < a.G) ? *plane_word(a, hc, g, w) : 0u;
            }
            if (g0 > 0) __syncthreads();
#pragma unroll
            for (int k = 0; k < 32 * kVoteWords / kVoteThreads; ++k)
                pw[(tid & 31) * kVoteRow + (tid >> 5) + k * (kVoteThreads / 32)] = x[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kVoteKeys; ++k) {
                const u32x4* row = reinterpret_cast<const u32x4*>(pw + ((k * kVoteThreads + tid) >> 5) * kVoteRow);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const u32x4 v = row[q];
#pragma unroll
                    for (int e = 0; e < 4; ++e) vote[k] += (v[e] >> (tid & 31)) & 1u;
                }
            }
        }
    } else {
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kVoteKeys; ++k) {
        const int t = t0 + k * kVoteThreads;
        if (t >= a.T) continue;
        double score = static_cast<double>(val[k]);
        if (vote_mode) {
            score = static_cast<double>(vote[k]) + a.lambda * score;
            if (a.votes != nullptr) a.votes[hc * a.T + t] = static_cast<uint8_t>(vote[k]);
        }
        const uint64_t key = static_cast<uint64_t>(__double_as_longlong(score));
        const uint32_t dg = key_digit(a, key);
        a.keys[hc * a.T + t] = key;
        a.digits[hc * a.digit_stride + t] = static_cast<uint16_t>(dg + 1u);
        if (t < pool) atomicAdd(&lh[dg], 1u);
    }
    __syncthreads();
    for (int i = tid; i < 2048; i += kVoteThreads)
        if (lh[i] != 0u) atomicAdd(&a.hist0[hc * 2048 + i], lh[i]);
}

// Clears the first-digit histograms where no tau cut runs before the vote
// kernel (MASS mode).
__global__ void __launch_bounds__(256) clear_hist0_kernel(SelectArgs a) {
    const int64_t n = static_cast<int64_t>(a.B) * a.Hkv * 2048;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * 256)
        a.hist0[i] = 0u;
}

// ---------------------------------------------------------------- top-k
// Budgeted selection of one (b, c).  Thread i owns keys i*kpt .. i*kpt + kpt
// - 1 through their first digits (16 bits each, kept in registers up to
// T = 32768: KPT > 0; read again from L2 by a rolled loop beyond, KPT = 0,
// where unrolled code of 64 keys a thread waits for its own instructions).  The vote
// kernel's counts name the digit bucket that holds the threshold; keys in
// higher buckets are selected, lower ones are not, and only the bucket's own
// keys (a few hundred of 16384 in the benchmark's layers) are read as 64-bit
// scores, from a list of them, and searched by radix, 11 bits at a time over
// the bits in which they differ.  A bucket too large for the list (1024 keys, a
// key a thread; 4096 beyond T = 32768) is searched in place: each thread's own
// keys in registers up to T = 32768, beyond that consecutive keys by consecutive
// threads, eight loads of a thread in flight, in every pass.
// Such buckets are those of peaked scores (most keys below the digits' range)
// or nearly equal ones: 4 heads, peaked votes of 16384 keys 81.6 us a selection
// with every key read by itself in each pass, 29.4 so; masses within 1% of
// 16384 / 32768 / 100000 keys 56 / 102 / 258 and 18.6 / 27.4 / 123.  A list
// limit of 128 keys costs 4 to 10 us at 16384 and 32768 keys.
// Bound by its chain of barriers (one workgroup per head):
// with all 64-bit keys in registers and their top bits as the first digit it
// took 15.4 us a call for 16 heads of 16384 keys, and in sweeps 75 us for 4 of
// 40000; this form takes 9.0 and 11.0 (8.3 and 11.8 within a layer).
constexpr int kTopkMaxKpt = 512;         // keys per thread (T = 524288) up to which selection bits fit in LDS
// Bucket sizes up to here: every key ranked against all others (beyond, the
// 64-bit comparisons cost more than radix passes: 4 us at 200 keys).
constexpr uint32_t kTopkRank = 128;
// MASS mode, bucket sizes up to here: the bits that all keys of the bucket
// share are taken from its digit; beyond, where a pass over equal keys would
// cost more than finding that they are, from the keys (4 heads, masses within
// 1% / all equal: 12.8 / 21.0 us and 13.3 / 12.8 at 4096 keys, 17.5 / 43.4 and
// 18.6 / 17.9 at 16384).
constexpr uint32_t kTopkKnown = 4096;

template <int KPT>
__global__ void __launch_bounds__(kSelThreads) topk_kernel(SelectArgs a) {
    static_assert(KPT % 8 == 0, "whole 16-byte pieces of digits");
    static_assert(KPT <= 32, "one word of selection bits a thread");
    constexpr int kWords = KPT > 0 ? 1 : kTopkMaxKpt / 32;   // words of selection bits per thread
    constexpr int kOwn = KPT > 0 ? 1 : 4;                    // listed keys per thread
    constexpr uint32_t kList = kOwn * kSelThreads;
    __shared__ uint32_t cnt[2][2048];                    // radix pass p counts into cnt[p % 2]
    __shared__ int32_t list[kList];                      // the bucket's keys (indices), in any order
    __shared__ uint32_t picked[kWords][kSelThreads];
    __shared__ uint32_t wtot[kSelWaves];
    __shared__ unsigned long long s_ones, s_zeros;
    __shared__ uint32_t same_bits[kWords];
    __shared__ uint32_t s_digit, s_cnt, s_rem, n_list;

    const int c = blockIdx.x, b = blockIdx.y;
    const int64_t hc = static_cast<int64_t>(b) * a.Hkv + c;
    const int tid = threadIdx.x;
    int32_t* out = a.idx + hc * a.c_max;
    int budget = a.budget;
    if (a.budgets != nullptr) budget = min(max(a.budgets[hc], 1), a.c_max);

    if (a.T <= budget) {
        for (int j = tid; j < a.c_max; j += kSelThreads) out[j] = (j < a.T) ? j : -1;
        if (tid == 0) a.counts[hc] = a.T;
        return;
    }
    const int pool = a.keep_last ? a.T - 1 : a.T;
    const uint32_t want = static_cast<uint32_t>(a.keep_last ? budget - 1 : budget);
    const uint64_t* key = a.keys + hc * a.T;
    const int kpt = KPT > 0 ? KPT : a.kpt;
    const int64_t t0 = static_cast<int64_t>(tid) * kpt;
    const int own = static_cast<int>(min(max(static_cast<int64_t>(pool) - t0, static_cast<int64_t>(0)),
                                         static_cast<int64_t>(kpt)));
    // digits as stored (digit + 1); 0 where there is no pool key
    const uint16_t* dig = a.digits + hc * a.digit_stride + t0;
    uint32_t pk[KPT > 0 ? KPT / 2 : 1];
#pragma unroll
    for (int q = 0; q < KPT / 8; ++q) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(dig + 8 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[4 * q + e] = x[e];
    }
    auto clip = [&](uint32_t w, int j) {                 // digits j and j + 1
        return j + 1 < own ? w : (j < own ? w & 0xFFFFu : 0u);
    };
#pragma unroll
    for (int q = 0; q < KPT / 2; ++q) pk[q] = clip(pk[q], 2 * q);
    // f(j, stored digit, key) for this thread's keys, ascending, from memory,
    // eight digits and keys fetched at once.  (Keys past the pool, up to seven,
    // are whatever follows in the workspace; their digit is 0.)
    const uint64_t* own_key = key + min(t0, static_cast<int64_t>(pool));
    auto each_mem = [&](auto&& f) {
#pragma nounroll
        for (int j0 = 0; j0 < own; j0 += 8) {
            const u32x4 x = *reinterpret_cast<const u32x4*>(dig + j0);
            uint64_t k[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) k[e] = own_key[j0 + e];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t w = clip(x[e / 2], j0 + (e & ~1));
                f(j0 + e, (e & 1) ? w >> 16 : w & 0xFFFFu, k[e]);
            }
        }
    };

    const uint32_t* h0 = a.hist0 + hc * 2048;
    for (int i = tid; i < 2048; i += kSelThreads) {
        cnt[0][i] = h0[i];
        cnt[1][i] = 0;
    }
    const int n_words = KPT > 0 ? 1 : min((kpt + 31) / 32, kWords);
    for (int w = 0; w < n_words; ++w) picked[w][tid] = 0;
    auto owner_of = [&](int32_t t) { return KPT > 0 ? t / (KPT > 0 ? KPT : 1) : t / kpt; };
    // sets the selection bit of key t with its owner
    auto pick = [&](int32_t t) {
        const int own_by = owner_of(t), j = t - own_by * kpt;
        atomicOr(&picked[j / 32][own_by], 1u << (j % 32));
    };
    if (tid == 0) {
        n_list = 0;
        s_ones = s_zeros = 0;
        s_digit = 0xFFFFu;
        s_cnt = s_rem = 0;
    }
    __syncthreads();
    uint32_t dg = 0x10000u, n_in = 0, need = 0;          // stored digit of the bucket; above all when want is 0
    if (want > 0) {
        descending_crossing<uint32_t>(cnt[0], cnt[0], want, wtot, &s_digit, &s_rem, &s_cnt);
        for (int i = tid; i < 2048; i += kSelThreads) cnt[0][i] = 0;   // every read of it is done
        dg = s_digit + 1u;
        n_in = s_cnt;
        need = s_rem;
    }
    const bool listed = (KPT > 0 || kpt <= kTopkMaxKpt) && n_in <= kList;

    // the keys above the bucket as bits, and the bucket's keys as bits (KPT >
    // 0) and as a list: each wave takes its place in it with one atomic a word
    uint32_t n_sel = 0, in_bits = 0;
    {
        uint32_t above = 0;
        auto eight = [&](int j0, const u32x4& x) {       // digits j0 .. j0 + 7
            uint32_t gt = 0, eq = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t d = (e & 1) ? x[e / 2] >> 16 : x[e / 2] & 0xFFFFu;
                gt |= (d > dg ? 1u : 0u) << e;
                eq |= (d == dg ? 1u : 0u) << e;
            }
            above |= gt << (j0 & 31);
            in_bits |= eq << (j0 & 31);
            n_sel += static_cast<uint32_t>(__popc(gt));
        };
        auto word_done = [&](int w) {                    // the whole wave
            picked[w][tid] = above;
            if (__ballot(in_bits != 0u) == 0) return;
            const uint32_t n = static_cast<uint32_t>(__popc(in_bits)), incl = wave_incl_scan(n);
            uint32_t base = 0;
            if (lane_id() == kWave - 1) base = atomicAdd(&n_list, incl);
            base = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(base), kWave - 1));
            uint32_t at = base + incl - n;
            for (uint32_t m = in_bits; m != 0; m &= m - 1, ++at)
                if (at < kList) list[at] = static_cast<int32_t>(t0) + 32 * w + __ffs(static_cast<int>(m)) - 1;
        };
        if constexpr (KPT > 0) {
#pragma unroll
            for (int q = 0; q < KPT / 8; ++q) eight(8 * q, u32x4{pk[4 * q], pk[4 * q + 1], pk[4 * q + 2], pk[4 * q + 3]});
            if (listed) word_done(0);
            else picked[0][tid] = above;
        } else {
            const int lim = __ballot(own > 0) != 0 ? kpt : 0;    // (whole waves)
#pragma unroll 2
            for (int j0 = 0; j0 < lim; j0 += 8) {
                u32x4 x = *reinterpret_cast<const u32x4*>(dig + j0);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = clip(x[e], j0 + 2 * e);
                eight(j0, x);
                if (listed && ((j0 & 31) == 24 || j0 + 8 >= lim)) {
                    word_done(j0 / 32);
                    above = in_bits = 0;
                }
            }
        }
    }
    __syncthreads();
    if (listed && n_in <= kTopkRank) {
        // a small bucket: each key's rank (score desc, index asc) among the
        // others by comparison, 8 threads a key, without radix passes
        uint64_t* lk = reinterpret_cast<uint64_t*>(cnt[1]);          // [kTopkRank]; not counted into yet
        const int n = static_cast<int>(min(n_in, n_list));
        if (tid < n) lk[tid] = key[list[tid]];
        __syncthreads();
        const int me = tid >> 3;
        if (me < n) {
            const uint64_t mk = lk[me];
            const int32_t mt = list[me];
            uint32_t rank = 0;
#pragma unroll 4
            for (int i = tid & 7; i < n; i += 8) {
                const uint64_t k = lk[i];
                rank += (k > mk || (k == mk && list[i] < mt)) ? 1u : 0u;
            }
#pragma unroll
            for (int o = 1; o < 8; o <<= 1) rank += static_cast<uint32_t>(__shfl_xor(static_cast<int>(rank), o, kWave));
            if ((tid & 7) == 0 && rank < need) pick(mt);
        }
        n_in = need = 0;                                 // nothing left to search
    }
    // the bucket's keys of this thread's share of the list, or, of a bucket too
    // large for it, its own ones (all of its keys up to T = 32768)
    uint64_t ck[kOwn];
    int32_t ct[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const uint32_t at = static_cast<uint32_t>(tid + i * kSelThreads);
        const bool in = listed && at < min(n_in, n_list);
        ct[i] = in ? list[at] : -1;
        ck[i] = in ? key[ct[i]] : 0ull;
    }
    uint64_t kv[KPT > 0 ? KPT : 1];
    if (!listed) {
#pragma unroll
        for (int j = 0; j < KPT; ++j) kv[j] = own_key[j];
    }
    // f(key) for those
    auto in_bucket = [&](auto&& f) {
        if (listed) {
#pragma unroll
            for (int i = 0; i < kOwn; ++i)
                if (ct[i] >= 0) f(ck[i]);
        } else if constexpr (KPT > 0) {
#pragma unroll
            for (int j = 0; j < KPT; ++j)
                if ((in_bits >> j) & 1u) f(kv[j]);
        } else {
            // (in any order: consecutive keys to consecutive threads)
            const uint16_t* all = a.digits + hc * a.digit_stride;
#pragma nounroll
            for (int64_t t1 = tid; t1 < pool; t1 += 8 * kSelThreads) {
                uint32_t d[8];
                uint64_t k[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int64_t t = min(t1 + e * kSelThreads, static_cast<int64_t>(pool) - 1);
                    d[e] = all[t];
                    k[e] = key[t];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (d[e] == dg && t1 + e * kSelThreads < pool) f(k[e]);
            }
        }
    };
    // threshold: {key > theta} plus the first k_eq keys (by index) equal to
    // it, or the whole bucket.  Keys compare as unsigned numbers, which gives
    // every bit pattern a place (a score of -0 or below has the top bit set)
    const bool whole = need >= n_in;
    uint64_t theta = 0;
    uint32_t k_eq = 0;
    if (!whole) {
        // the bits in which they differ: set in one and clear in another
        // (reduced within the wave first: the compiler turns a per-lane atomic
        // of varying values into a loop over the lanes)
        uint64_t ones = 0, diff = 0;
        if (a.mode != 0 && dg > 1u && dg < 2048u && n_in <= kTopkKnown) {
            // a float mass between the two end digits: the digit is its
            // exponent and upper 5 fraction bits, and the double's lower 29
            // are zero (any value with these bits will do)
            const uint32_t f = (dg - 1u + ((127u - 39u) << 5)) << 18;
            ones = static_cast<uint64_t>(__double_as_longlong(static_cast<double>(__uint_as_float(f))));
            diff = ((1ull << 18) - 1ull) << 29;
        } else {
            uint64_t zeros = 0;
            in_bucket([&](uint64_t k) {
                ones |= k;
                zeros |= ~k;
            });
            ones = wave_or_u64(ones);
            zeros = wave_or_u64(zeros);
            if (lane_id() == 0) {
                atomicOr(&s_ones, static_cast<unsigned long long>(ones));
                atomicOr(&s_zeros, static_cast<unsigned long long>(zeros));
            }
            __syncthreads();
            ones = s_ones;
            diff = ones & s_zeros;
        }
        if (diff == 0) {                                 // all equal: the first `need` by index
            theta = ones;
            k_eq = need;
        } else {
            const int top = 63 - __clzll(static_cast<long long>(diff)), low = __ffsll(static_cast<long long>(diff)) - 1;
            uint64_t mask = top == 63 ? 0ull : ~0ull << (top + 1);
            uint64_t prefix = ones & mask;
            int shift = max(top - 10, 0);
            for (int pass = 0;; ++pass) {
                uint32_t* pc = cnt[pass & 1];
                in_bucket([&](uint64_t kv) {
                    if ((kv & mask) == prefix) atomicAdd(&pc[static_cast<uint32_t>(kv >> shift) & 2047u], 1u);
                });
                __syncthreads();
                descending_crossing<uint32_t>(pc, pc, need, wtot, &s_digit, &s_rem, &s_cnt);
                // cleared for pass + 2, two barriers away
                for (int i = tid; i < 2048; i += kSelThreads) pc[i] = 0;
                prefix |= static_cast<uint64_t>(s_digit) << shift;
                mask |= 0x7FFull << shift;
                need = s_rem;
                if (s_cnt == need) {
                    // the rest is taken whole: every key >= its lower bound
                    // (> 0: the bucket is not taken whole)
                    theta = prefix - 1;
                    break;
                }
                if (shift <= low) {                      // every bit below is the same in all of them
                    theta = prefix | (ones & ((1ull << shift) - 1ull));
                    k_eq = need;
                    break;
                }
                shift = max(shift - 11, 0);
            }
        }
    }

    uint32_t sel_total, pos;
    if (listed) {
        // the selected ones of the list, as bits of their owners
        bool take[kOwn];
#pragma unroll
        for (int i = 0; i < kOwn; ++i) take[i] = ct[i] >= 0 && (whole || ck[i] > theta);
        if (k_eq > 0) {
            // equal keys by index, in time that does not grow with their
            // number: counted per owner (the count buffers are all zero after
            // the barrier), one scan over the owners, and the one owner that
            // takes some but not all of its own sets them as bits.  (Each
            // equal key counting the ones before it took 285 us for 4096.)
            uint32_t *same = cnt[0], *taken = cnt[1];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kOwn; ++i)
                if (ct[i] >= 0 && ck[i] == theta) atomicAdd(&same[owner_of(ct[i])], 1u);
            if (tid < kWords) same_bits[tid] = 0;
            __syncthreads();
            uint32_t eq_total;
            const uint32_t mine = same[tid], before = block_excl_scan<uint32_t>(mine, wtot, eq_total);
            taken[tid] = before < k_eq ? min(mine, k_eq - before) : 0u;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kOwn; ++i) {
                if (ct[i] < 0 || ck[i] != theta) continue;
                const int o = owner_of(ct[i]), j = ct[i] - o * kpt;
                take[i] = taken[o] == same[o];
                if (!take[i] && taken[o] > 0) atomicOr(&same_bits[j / 32], 1u << (j % 32));
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kOwn; ++i) {
                if (ct[i] < 0 || ck[i] != theta) continue;
                const int o = owner_of(ct[i]), j = ct[i] - o * kpt;
                if (taken[o] == 0 || taken[o] == same[o]) continue;
                uint32_t below = static_cast<uint32_t>(__popc(same_bits[j / 32] & ((1u << (j % 32)) - 1u)));
                for (int w = 0; w < j / 32; ++w) below += static_cast<uint32_t>(__popc(same_bits[w]));
                take[i] = below < taken[o];
            }
        }
#pragma unroll
        for (int i = 0; i < kOwn; ++i)
            if (take[i]) pick(ct[i]);
        __syncthreads();
    } else if constexpr (KPT > 0) {
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            gt |= (whole || kv[j] > theta ? 1u : 0u) << j;
            eq |= (kv[j] == theta ? 1u : 0u) << j;
        }
        if (k_eq > 0) {
            // the first k_eq equal keys by index
            eq &= in_bits;
            uint32_t eq_total;
            const uint32_t n_eq = static_cast<uint32_t>(__popc(eq));
            const uint32_t before = block_excl_scan<uint32_t>(n_eq, wtot, eq_total);
            for (uint32_t n = before < k_eq ? min(n_eq, k_eq - before) : 0u; n > 0; --n, eq &= eq - 1) gt |= eq & (0u - eq);
        }
        picked[0][tid] |= gt & in_bits;
    }
    if (KPT > 0 || listed) {
        n_sel = 0;
        for (int w = 0; w < n_words; ++w) n_sel += static_cast<uint32_t>(__popc(picked[w][tid]));
        pos = block_excl_scan<uint32_t>(n_sel, wtot, sel_total);
        for (int w = 0; w < n_words; ++w) {
            for (uint32_t m = picked[w][tid]; m != 0; m &= m - 1) {
                if (pos < want) out[pos] = static_cast<int32_t>(t0) + 32 * w + __ffs(static_cast<int>(m)) - 1;
                ++pos;
            }
        }
    } else {
        uint32_t n_eq = 0;
        each_mem([&](int, uint32_t d, uint64_t k) {
            if (d != dg) return;
            n_sel += whole || k > theta ? 1u : 0u;
            n_eq += k == theta ? 1u : 0u;
        });
        if (k_eq > 0) {
            // this thread's share of the k_eq equal keys, by index
            uint32_t eq_total;
            const uint32_t before = block_excl_scan<uint32_t>(n_eq, wtot, eq_total);
            k_eq = before < k_eq ? min(n_eq, k_eq - before) : 0u;
            n_sel += k_eq;
        }
        pos = block_excl_scan<uint32_t>(n_sel, wtot, sel_total);
        if (n_sel > 0) {
            each_mem([&](int j, uint32_t d, uint64_t k) {
                bool take = d > dg;
                if (d == dg) {
                    take = whole || k > theta;
                    if (k == theta && k_eq > 0) {
                        take = true;
                        --k_eq;
                    }
                }
                if (take) {
                    if (pos < want) out[pos] = static_cast<int32_t>(t0) + j;
                    ++pos;
                }
            });
        }
    }
    uint32_t written = min(sel_total, want);
    if (a.keep_last) {
        if (tid == 0) out[written] = a.T - 1;
        written += 1;
    }
    for (int j = static_cast<int>(written) + tid; j < a.c_max; j += kSelThreads) out[j] = -1;
    if (tid == 0) a.counts[hc] = static_cast<int32_t>(written);
}

// ------------------------------------------- register-resident tau cut
// The tau cut of one (b, c, group) for T <= NT * KPT, where the row of one
// workgroup fits in registers and is read from memory once; same result as
// tau_cut_kernel.  NT threads (512 up to T = 16384, so two workgroups share a
// CU and a launch of 512 workgroups is resident at once; 1024 up to T = 65536)
// of at most 128 VGPRs.  Thread i holds keys 4 NT q + 4 i + e (q < KPT / 4, e <
// 4), so every load is one contiguous 16-byte piece per lane; the index-ordered
// steps (ties, the plane) go through the chunks q of 4 NT keys in order.
template <int KPT, int NT>
__global__ void __launch_bounds__(NT) tau_cut_reg_kernel(SelectArgs a) {
    static_assert(KPT % 4 == 0, "whole 4-key pieces per thread");
    // one 64-bit LDS atomic per key carries its count (from bit kCntBit) and
    // its mantissa part (< 2^24): the row's sum stays below 2^kCntBit and its
    // count below 2^(64 - kCntBit)
    constexpr int kCntBit = 44;
    static_assert(static_cast<int64_t>(KPT) * NT < (1 << 20), "packed sum and count");
    constexpr unsigned long long kSumMask = (1ull << kCntBit) - 1;
    constexpr int kQ = KPT / 4;
    constexpr int kChunk = 4 * NT;
    constexpr int kW = NT / kWave;
    __shared__ unsigned long long sum[2048];
    __shared__ unsigned long long wtot64[kW];
    __shared__ uint32_t wtot[kW];
    __shared__ uint32_t s_digit, s_cnt;
    __shared__ unsigned long long s_rem;
    __shared__ int32_t s_tcut;
    __shared__ uint32_t s_theta;

    const int g = blockIdx.x, c = blockIdx.y, b = blockIdx.z;
    const int64_t hc = static_cast<int64_t>(b) * a.Hkv + c;
    const int64_t hcg = hc * a.G + g;
    const uint32_t* m = reinterpret_cast<const uint32_t*>(a.group_mass) + hcg * a.T;
    const int tid = threadIdx.x, lane = lane_id();
    const int S = a.fix_shift;
    clear_hist0_share(a, hc, g);
    auto key_of = [&](int q, int e) { return kChunk * q + 4 * tid + e; };

    // masses (bits), held for all passes (their fixed-point values are
    // recomputed where needed).  Keys past T read as mass 0, which no step
    // below counts: a mass of 0 adds nothing to a sum, and the cut is never 0
    // (a bucket whose sum is 0 is never the crossing one).
    uint32_t mb[KPT];
    if ((a.T & 3) == 0 && (reinterpret_cast<uintptr_t>(m) & 15u) == 0) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            u32x4 x = {0u, 0u, 0u, 0u};
            if (key_of(q, 0) < a.T) x = *reinterpret_cast<const u32x4*>(m + key_of(q, 0));
            mb[4 * q] = x[0]; mb[4 * q + 1] = x[1]; mb[4 * q + 2] = x[2]; mb[4 * q + 3] = x[3];
        }
    } else {
#pragma unroll
        for (int q = 0; q < kQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) mb[4 * q + e] = key_of(q, e) < a.T ? m[key_of(q, e)] : 0u;
    }
    // every mass below the fixed-point resolution: empty set
    uint32_t theta = 0xFFFFFFFFu;
    int32_t tcut = -1;
    unsigned long long need = 0;
    uint32_t prefix = 0;
    bool found = true;
    {
#pragma nounroll
        for (int pass = 0; pass < 3; ++pass) {
            const uint32_t mask = tau_mask(pass);
            for (int i = tid; i < 2048; i += NT) sum[i] = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                // opaque inside the pass loop, so the per-key values are not
                // hoisted out of it and kept live
                asm volatile("" : "+v"(mb[j]));
                if (mb[j] != 0u && (mb[j] & mask) == prefix) {
                    const uint32_t dg = tau_digit(mb[j], pass);
                    atomicAdd(&sum[dg], (1ull << kCntBit) | mant_part(mb[j], S));
                }
            }
            __syncthreads();
            // bucket d's exponent: the digit's top 8 bits in the first pass,
            // the prefix's in the later ones
            const uint32_t e_pre = prefix >> 23;
            const unsigned long long total = crossing_of<unsigned long long, NT>(
                [&](int d) {
                    return static_cast<unsigned long long>(
                        bucket_fixed(sum[d] & kSumMask, pass == 0 ? static_cast<uint32_t>(d) >> 3 : e_pre, S));
                },
                [&](int d) { return static_cast<uint32_t>(sum[d] >> kCntBit); },
                [&](unsigned long long tot) {
                    if (pass == 0) {
                        // the shortest prefix reaching tau * total (at least one key)
                        need = static_cast<unsigned long long>(ceil(a.tau * static_cast<double>(tot)));
                        if (need < 1) need = 1;
                        if (need > tot) need = tot;
                    }
                    return need;
                },
                wtot64, &s_digit, &s_rem, &s_cnt);
            if (pass == 0 && total == 0) {
                found = false;
                break;
            }
            prefix |= s_digit << tau_shift(pass);
            need = s_rem;
            if (pass < 2 && s_cnt == 1u) {
                // one key left in the crossing bucket: its mass is theta, and the
                // remaining passes would only spell out its low bits
#pragma unroll
                for (int j = 0; j < KPT; ++j)
                    if ((mb[j] & tau_fixed(pass)) == prefix) s_theta = mb[j];
                __syncthreads();
                prefix = s_theta;
                break;
            }
        }
    }
    if (found) {
        theta = prefix;
        const uint64_t f_theta = fixed_of(prefix, S);
        const uint64_t k_eq = f_theta == 0 ? 1 : (need + f_theta - 1) / f_theta;
        if (k_eq >= s_cnt) {
            tcut = a.T;
        } else {
            // the k_eq-th key (by index) whose mass equals theta, chunk by chunk
            if (tid == 0) s_tcut = a.T - 1;
            uint64_t seen = 0;
#pragma nounroll
            for (int q = 0; q < kQ; ++q) {
                uint32_t n_eq = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) n_eq += mb[4 * q + e] == prefix ? 1u : 0u;
                uint32_t tot;
                const uint32_t before = block_excl_scan<uint32_t, NT>(n_eq, wtot, tot);
                if (seen + before < k_eq && k_eq <= seen + before + n_eq) {
                    uint64_t at = seen + before;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (mb[4 * q + e] == prefix && ++at == k_eq) s_tcut = key_of(q, e);
                }
                seen += tot;
                if (seen >= k_eq) break;
            }
            __syncthreads();
            tcut = s_tcut;
        }
    }
    if (tid == 0) {
        a.theta[hcg] = theta;
        a.tcut[hcg] = tcut;
    }
    // membership plane: each lane's 4 bits, merged over the 8 lanes of a word
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        uint32_t word = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = key_of(q, e);
            word |= in_tau_set(mb[4 * q + e], t, theta, tcut) ? 1u << (4 * (lane & 7) + e) : 0u;
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) word |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(word), o, kWave));
        if ((lane & 7) == 0 && key_of(q, 0) < a.T) *plane_word(a, hc, g, key_of(q, 0) / 32) = word;
    }
}

}  // namespace

int select_kpt(int T) {
    // a power of two while the digits stay in registers, whole 16-byte pieces
    // beyond
    const int per = static_cast<int>((static_cast<int64_t>(T) + kSelThreads - 1) / kSelThreads);
    return per <= 8 ? 8 : per <= 16 ? 16 : per <= 32 ? 32 : (per + 7) / 8 * 8;
}

hipError_t launch_select(const SelectArgs& a, int stages, hipStream_t s) {
    if (a.kpt != select_kpt(a.T) || a.digit_stride != select_digit_stride(a.T)) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    if (stages & kSelectTau) {
        if (a.mode == 0) {
            // register-resident tau cut while a row fits in 32 masses per
            // thread of 512 (two workgroups on a CU), then 32 and 64 of 1024;
            // the sweep kernel beyond (T > 65536)
            dim3 g1(a.G, a.Hkv, a.B);
            const int tper = (a.T + kTauThreads - 1) / kTauThreads;
            const int tkpt = tper <= 8 ? 8 : tper <= 16 ? 16 : tper <= 32 ? 32 : tper <= 64 ? 64 : tper <= 128 ? 128 : 0;
            switch (tkpt) {
                case 8: hipLaunchKernelGGL((tau_cut_reg_kernel<8, kTauThreads>), g1, dim3(kTauThreads), 0, s, a); break;
                case 16: hipLaunchKernelGGL((tau_cut_reg_kernel<16, kTauThreads>), g1, dim3(kTauThreads), 0, s, a); break;
                case 32: hipLaunchKernelGGL((tau_cut_reg_kernel<32, kTauThreads>), g1, dim3(kTauThreads), 0, s, a); break;
                case 64: hipLaunchKernelGGL((tau_cut_reg_kernel<32, kSelThreads>), g1, dim3(kSelThreads), 0, s, a); break;
                case 128: hipLaunchKernelGGL((tau_cut_reg_kernel<64, kSelThreads>), g1, dim3(kSelThreads), 0, s, a); break;
                default: hipLaunchKernelGGL(tau_cut_kernel, g1, dim3(kSelThreads), 0, s, a); break;
            }
        } else {
            const int64_t n = static_cast<int64_t>(a.B) * a.Hkv * 2048;
            const int64_t blocks = (n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024;
            hipLaunchKernelGGL(clear_hist0_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (stages & kSelectVote) {
        const int nw = (a.T + 31) / 32;
        dim3 g2((nw + kVoteWords - 1) / kVoteWords, a.Hkv, a.B);
        hipLaunchKernelGGL(vote_score_kernel, g2, dim3(kVoteThreads), 0, s, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (stages & kSelectPick) {
        dim3 g3(a.Hkv, a.B);
        switch (a.kpt) {
            case 8: hipLaunchKernelGGL(topk_kernel<8>, g3, dim3(kSelThreads), 0, s, a); break;
            case 16: hipLaunchKernelGGL(topk_kernel<16>, g3, dim3(kSelThreads), 0, s, a); break;
            case 32: hipLaunchKernelGGL(topk_kernel<32>, g3, dim3(kSelThreads), 0, s, a); break;
            default: hipLaunchKernelGGL(topk_kernel<0>, g3, dim3(kSelThreads), 0, s, a); break;
        }
        e = hipGetLastError();
    }
    return e;
}

}  // namespace mmskv
