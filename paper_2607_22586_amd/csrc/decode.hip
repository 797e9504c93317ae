// Decode-time check on gfx950: the attention-mass coverage of Fig. 1b (the
// share of a decoding query's softmax mass over all prompt keys that falls
// on the keys kept after prefilling) and decode attention over the fixed
// compacted cache (Sec. 3.1's prefill-only protocol).
//
// Coverage: one workgroup of 4 waves per (b, c, block of 256 keys), each wave
// holding 64 keys in registers.  The Gh * n_dec decode queries of KV head c,
// scaled like the anchor query (log2(e)/sqrt(d), rounded to fp32, then to
// bf16), are staged in LDS and streamed past the keys in 32-row tiles with
// v_mfma_f32_32x32x16_bf16 in the K * Q^T layout (lane = query row, its 32
// values = its keys), so a row's block statistics are in-lane sums.  Per
// (row, block) the kernel writes (m, sum of 2^(s - m) over all keys, the same
// over the kept keys).  The keys are read once: the pass is bound by HBM
// reads of K and by the exps.
//
// Compacted attention: one workgroup of 4 waves per (b, c, 32 decode rows, 32
// output dims) on the matrix cores: S = K' Q^T, then O = P V', for a bf16
// cache with P split into two bf16 parts, for an fp32 cache in fp32 products
// (v_mfma_f32_32x32x2_f32).  It also merges the coverage partials of its rows.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace mmskv {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kDecWaves = 4;
constexpr int kDecKeys = 64 * kDecWaves;   // keys per workgroup
constexpr int kDecMaxRows = 256;           // Gh * n_dec, padded to 32
constexpr int kDecMaxCompact = 2048;       // rows of the compacted cache (c_max)

__device__ __forceinline__ floatx16 mfma_32x32x16(bf16x8 a, bf16x8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

__device__ __forceinline__ float pair_max2(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float pair_sum2(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Eight bf16 queries times the scale, rounded to fp32, then to bf16.  The
// scale comes as scale_hi + scale_lo with 16 significant bits in scale_hi, so
// that v * scale_hi is exact in fp32 and the fused multiply-add rounds the
// product once: for every bf16 value and both head sizes the same bits as the
// fp64 product rounded to fp32 and to bf16 (all 65536 values compared), at two
// instructions instead of the fp64 conversions.
__device__ __forceinline__ u32x4 scaled_queries(const DecodeArgs& a, const u32x4& raw) {
    u32x4 v;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float x0 = __uint_as_float(raw[w] << 16), x1 = __uint_as_float(raw[w] & 0xFFFF0000u);
        v[w] = pack_bf16(fmaf(x0, a.scale_lo, x0 * a.scale_hi), fmaf(x1, a.scale_lo, x1 * a.scale_hi));
    }
    return v;
}

// The decode queries of KV head (b, c): Gh * n_dec consecutive rows of D (row
// r = head c * Gh + r / n_dec, query r % n_dec).
template <int D>
__device__ __forceinline__ const uint16_t* head_queries(const DecodeArgs& a, int b, int c) {
    return a.q_dec + (static_cast<int64_t>(b) * a.Hq + static_cast<int64_t>(c) * a.Gh) * a.n_dec * D;
}

// LDS slot of 16-byte chunk ch of query row r: rows without padding, the
// chunks of a row permuted by its index, so that the reads of one chunk of
// 16 (8 at d = 64) consecutive rows fall in different banks.
template <int D>
__device__ __forceinline__ int query_slot(int r, int ch) {
    return r * (D / 8) + (ch ^ (r & (D / 8 - 1)));
}

// One wave's 64 keys of the coverage pass, all of them < T if FULL; the (max,
// sum all, sum kept) of every row go to pm / pa / pk[row].
template <int D, bool FULL>
__device__ __forceinline__ void cover_wave(const DecodeArgs& a, int key_base, int key0, const u32x4* qs,
                                           const uint32_t* kept, float* pm, float* pa, float* pk,
                                           const bf16x8 (&kf)[2][D / 16]) {
    constexpr int KC = D / 16;                 // 16-element k steps
    const int lane = lane_id();
    // value i of sub-tile s of this lane is key key0 + 32 s + 8 (i / 4) + 4 (lane / 32) + i % 4;
    // bit 16 s + i of valid / keep: that key is below T / kept
    uint32_t valid = 0xFFFFFFFFu, keep = 0u;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int t = key0 + 32 * s + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
            const int tl = t - key_base;
            const bool ok = FULL || t < a.T;
            if (!FULL && !ok) valid &= ~(1u << (16 * s + i));
            if (ok && ((kept[tl >> 5] >> (tl & 31)) & 1u)) keep |= 1u << (16 * s + i);
        }
    // most 32-key sub-tiles hold no kept key: their kept sums are skipped
    const bool kept0 = __ballot((keep & 0xFFFFu) != 0u) != 0, kept1 = __ballot((keep >> 16) != 0u) != 0;
    // the kept sum as one fused multiply-add per value with a 0 / 1 factor
    auto kmul = [&](int j) { return static_cast<float>((keep >> j) & 1u); };
#pragma unroll 1
    for (int r0 = 0; r0 < a.rows_pad; r0 += 32) {
        // opaque per row tile, so that the 0 / 1 factors are formed where
        // they are used instead of being kept in 32 registers
        asm volatile("" : "+v"(keep));
        // (the slots of the row's chunks likewise)
        int swz = lane & (D / 8 - 1);
        asm volatile("" : "+v"(swz));
        const u32x4* qrow = qs + (r0 + (lane & 31)) * (D / 8);
        floatx16 acc[2];
        auto logits = [&]() {
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const bf16x8 q = __builtin_bit_cast(bf16x8, qrow[(2 * kc + (lane >> 5)) ^ swz]);
#pragma unroll
                for (int s = 0; s < 2; ++s) acc[s] = mfma_32x32x16(kf[s][kc], q, kc == 0 ? zero16() : acc[s]);
                // (two fragments in registers at a time: four workgroups need the rest)
                if (kc % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
        };
        logits();
        // sums of 2^s relative to 0 while every lane's sum is in
        // [2^-60, lane_sum_limit(T, 32)) (as in the row log-sum-exp pass),
        // else relative to the exact per-column maximum
        float mx = 0.f, la = -0.f, lk = -0.f;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float e = (FULL || ((valid >> (16 * s + i)) & 1u)) ? fast_exp2(acc[s][i]) : 0.f;
                acc[s][i] = e;
                la += e;
            }
        if (kept0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) lk = fmaf(acc[0][i], kmul(i), lk);
        }
        if (kept1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) lk = fmaf(acc[1][i], kmul(16 + i), lk);
        }
        const bool in_range = (la >= 0x1p-60f || (!FULL && valid == 0u)) && la < a.lane_sum_hi;
        if (__ballot(!in_range) != 0) {
            // the logits again (the exps above replaced them) for the exact form
            logits();
            mx = -INFINITY;
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (FULL || ((valid >> (16 * s + i)) & 1u)) mx = fmaxf(mx, acc[s][i]);
            mx = pair_max2(mx);
            la = 0.f;
            lk = 0.f;
            if (mx != -INFINITY) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float e = (FULL || ((valid >> (16 * s + i)) & 1u)) ? fast_exp2(acc[s][i] - mx) : 0.f;
                        la += e;
                        lk = fmaf(e, kmul(16 * s + i), lk);
                    }
            }
        }
        la = pair_sum2(la);
        lk = pair_sum2(lk);
        if (lane < 32) {
            const bool any = la > 0.f;
            pm[r0 + lane] = any ? mx : -INFINITY;
            pa[r0 + lane] = any ? la : 0.f;
            pk[r0 + lane] = any ? lk : 0.f;
        }
    }
}

// A bf16 cache keeps four workgroups on a CU (128 registers; at d = 128 and
// 128 rows 38 KiB of LDS): the 1024 blocks of 4 x 4 KV heads of 16384 keys are
// then all resident at once, so that one round of key loads is in flight from
// the start.
template <int D, bool F32>
__global__ void __launch_bounds__(64 * kDecWaves, F32 ? 2 : 4) decode_cover_kernel(DecodeArgs a) {
    constexpr int KC = D / 16;                 // 16-element k steps
    constexpr int CH = D / 8;                  // 16-byte chunks of a query row
    // [rows_pad * CH] queries, then the waves' (max, sum all, sum kept) rows
    extern __shared__ u32x4 qs[];
    __shared__ uint32_t kept[kDecKeys / 32];
    float* part = reinterpret_cast<float*>(qs + a.rows_pad * CH);   // [3][kDecWaves][rows_pad]

    const int kb = blockIdx.x, bc = blockIdx.y;
    const int b = bc / a.Hkv, c = bc - b * a.Hkv;
    // (the wave in a scalar register, with what is formed from it)
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int key_base = kb * kDecKeys;
    constexpr int kThreads = 64 * kDecWaves;

    // The head's queries (L2-resident) and half of the block's keys (HBM) are
    // fetched before the first wait, the kept indices and the other half once the queries have left their registers (all at once they
    // would not fit in 128).  Indices are clamped instead of branched on, so
    // nothing serialises the loads.
    // (query chunks in rounds of kQPer per thread: one round up to 128 rows at d = 128)
    constexpr int kQPer = 8;
    const int nq = a.rows * CH, nq_pad = a.rows_pad * CH;
    const u32x4* qsrc = reinterpret_cast<const u32x4*>(head_queries<D>(a, b, c));
    u32x4 qv[kQPer];
#pragma unroll
    for (int j = 0; j < kQPer; ++j) qv[j] = qsrc[min(tid + kThreads * j, nq - 1)];
    constexpr int kIdxPer = kDecMaxCompact / kThreads;
    const int n_kept = min(max(a.counts[bc], 0), a.c_max);
    const int32_t* ids = a.idx + static_cast<int64_t>(bc) * a.c_max;

    // kf[s][kc] = key key0 + 32 s + lane % 32, dims 16 kc + 8 (lane / 32) ..
    // A key past T reads key T - 1 instead (unconditional loads, issued
    // together); its values are masked out of every sum.
    const int key0 = key_base + 64 * wave;
    bf16x8 kf[2][KC];
    auto load_sub = [&](int s) {
        const int t = min(key0 + 32 * s + (lane & 31), a.T - 1);
        const int64_t off = static_cast<int64_t>(b) * a.ksb + static_cast<int64_t>(c) * a.ksh +
                            static_cast<int64_t>(t) * a.kst + 8 * (lane >> 5);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            if constexpr (F32) kf[s][kc] = load_f32_as_bf16x8(static_cast<const float*>(a.k) + off + 16 * kc);
            else kf[s][kc] = load_bf16x8(static_cast<const uint16_t*>(a.k) + off + 16 * kc);
        }
    };
    load_sub(0);

    // scaled queries to LDS (rows past Gh * n_dec zero), kept flags cleared;
    // then the kept flags of this block's keys (idx is any list of in-range
    // indices)
    for (int i0 = 0; i0 < nq_pad; i0 += kThreads * kQPer) {
        if (i0 > 0) {
#pragma unroll
            for (int j = 0; j < kQPer; ++j) qv[j] = qsrc[min(i0 + tid + kThreads * j, nq - 1)];
        }
#pragma unroll
        for (int j = 0; j < kQPer; ++j) {
            const int i = i0 + tid + kThreads * j;
            if (i < nq_pad) {
                const int r = i / CH, ch = i - r * CH;
                qs[query_slot<D>(r, ch)] = i < nq ? scaled_queries(a, qv[j]) : u32x4{0u, 0u, 0u, 0u};
            }
        }
    }
    if (tid < kDecKeys / 32) kept[tid] = 0u;
    __syncthreads();
    int32_t iv[kIdxPer];
#pragma unroll
    for (int j = 0; j < kIdxPer; ++j) iv[j] = ids[min(tid + kThreads * j, a.c_max - 1)];
    load_sub(1);
#pragma unroll
    for (int j = 0; j < kIdxPer; ++j) {
        const int t = iv[j] - key_base;
        if (tid + kThreads * j < n_kept && t >= 0 && t < kDecKeys && t + key_base < a.T)
            atomicOr(&kept[t >> 5], 1u << (t & 31));
    }
    __syncthreads();
    float* pm = part + wave * a.rows_pad;
    float* pa = pm + kDecWaves * a.rows_pad;
    float* pk = pa + kDecWaves * a.rows_pad;
    // (key0 is the same in every lane: the MFMAs and lane swaps run in whole waves)
    if (key_base + kDecKeys <= a.T) {
        cover_wave<D, true>(a, key_base, key0, qs, kept, pm, pa, pk, kf);
    } else if (key0 < a.T) {
        cover_wave<D, false>(a, key_base, key0, qs, kept, pm, pa, pk, kf);
    } else {
        for (int r = lane; r < a.rows_pad; r += kWave) pm[r] = -INFINITY, pa[r] = 0.f, pk[r] = 0.f;
    }
    __syncthreads();
    // merge the 4 waves: one thread per row
    for (int r = tid; r < a.rows_pad; r += 64 * kDecWaves) {
        const float* q = part + r;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kDecWaves; ++w) M = fmaxf(M, q[w * a.rows_pad]);
        float sa = 0.f, sk = 0.f;
        if (M != -INFINITY) {
#pragma unroll
            for (int w = 0; w < kDecWaves; ++w) {
                const float f = fast_exp2(q[w * a.rows_pad] - M);
                sa += q[(kDecWaves + w) * a.rows_pad] * f;
                sk += q[(2 * kDecWaves + w) * a.rows_pad] * f;
            }
        }
        a.part[(static_cast<int64_t>(bc) * a.n_kb + kb) * a.rows_pad + r] = make_float4(M, sa, sk, 0.f);
    }
}

// decode attention over a compacted cache on the matrix cores: one workgroup
// of 4 waves per (b, c, 32 decode rows of KV head c, 32 output dims), walking
// the counts[b, c] cached keys in chunks of 256, 64 per wave.  Per chunk, wave w:
//   S = K'_w Q^T (keys as MFMA rows, so lane l % 32 is decode row l % 32 and
//   its 32 values are the wave's keys); the chunk's row maxima merged over
//   the waves through LDS into the running maximum M; p = 2^(s - M), the
//   earlier partial output and sum rescaled by 2^(M_old - M);
//   O_w += P V'_w, with P as the MFMA's A operand straight from the S
//   registers and V' read in the same key order, each lane its own dim of its
//   keys, straight from memory.  bf16 cache: 16-key steps (value i of step kk
//   holds key 16 kk + 8 (j / 4) + 4 (l / 32) + j % 4, j = i - 8 kk), P split
//   into two bf16 parts p = hi + lo so that the weights keep ~16 bits.  fp32
//   cache: 2-key fp32 steps, step i holding the keys of value i of the two
//   half-waves.
// At the end the waves' partial outputs and sums are added through LDS and
// divided.  fp32 accumulation throughout.
// What bounds it is the chain of latencies of one workgroup (loads, S, the
// maxima, P V', the merge), not a rate: every part of the output dims forms S
// anew, which is cheap, and has its own share of V' and of the coverage merge,
// so that four times as many CUs work on it (16 heads of 256 bf16 keys and 112
// rows: 10.4 us with one workgroup per 32 rows, 7.8 us so; 4 heads of 409 fp32
// keys and 28 rows: 37.9 us with a wave per query on the VALU, 13.9 us so).
template <int D, bool F32>
__global__ void __launch_bounds__(64 * kDecWaves) decode_attend_kernel(DecodeArgs a) {
    constexpr int KC = D / 16;                     // 16-dim k steps of S
    constexpr int NT = D / 32;                     // 32-dim output tiles
    constexpr int kCovRows = 32 / NT;              // rows whose coverage this workgroup merges
    constexpr int kCovGroups = 64 * kDecWaves / kCovRows;
    __shared__ __align__(16) float ob[kDecWaves][32 * 32];
    __shared__ float mx_w[kDecWaves][32];
    __shared__ float l_w[kDecWaves][32];
    __shared__ __align__(16) float fac_s[32];
    __shared__ float4 cov_w[kDecWaves][kCovRows];
    const int tile = static_cast<int>(blockIdx.x) / NT, td = static_cast<int>(blockIdx.x) % NT, bc = blockIdx.y;
    const int b = bc / a.Hkv, c = bc - b * a.Hkv;
    const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
    const int h = lane >> 5, l32 = lane & 31;
    const int n = min(max(a.counts[bc], 0), a.c_max);
    using Elem = std::conditional_t<F32, float, uint16_t>;
    const Elem* kc_base = static_cast<const Elem*>(a.k_out) + static_cast<int64_t>(bc) * a.c_max * D + 8 * h;
    const Elem* vc_base = static_cast<const Elem*>(a.v_out) + static_cast<int64_t>(bc) * a.c_max * D + 32 * td + l32;

    // coverage of kCovRows rows, the merge of the coverage kernel's per-key-
    // block partials (m, sum all, sum kept): thread t takes row t % kCovRows
    // and key blocks t / kCovRows + kCovGroups j; its first partials are
    // fetched here, with the other loads, and merged at the end
    constexpr int kCovPer = 2;
    const int cr = tid % kCovRows, cg = tid / kCovRows;
    const float4* pp = a.part + static_cast<int64_t>(bc) * a.n_kb * a.rows_pad + 32 * tile + kCovRows * td + cr;
    float4 pv[kCovPer];
#pragma unroll
    for (int j = 0; j < kCovPer; ++j)
        pv[j] = pp[static_cast<int64_t>(min(cg + kCovGroups * j, a.n_kb - 1)) * a.rows_pad];
    // query fragments: decode row 32 tile + l32 (zero past the last row), dims 16 kc + 8 h ..
    bf16x8 qf[KC];
    {
        const int row = 32 * tile + l32;
        const uint16_t* qrow = head_queries<D>(a, b, c) + static_cast<int64_t>(min(row, a.rows - 1)) * D + 8 * h;
        u32x4 raw[KC];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) raw[kc] = *reinterpret_cast<const u32x4*>(qrow + 16 * kc);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            const u32x4 q = scaled_queries(a, raw[kc]);
            qf[kc] = __builtin_bit_cast(bf16x8, row < a.rows ? q : u32x4{0u, 0u, 0u, 0u});
        }
    }
    floatx16 o = zero16();
    float M = -INFINITY, lsum = 0.f;               // running maximum and partial sum of row l32

    for (int k0 = 0; k0 < n; k0 += 64 * kDecWaves) {
        const int kw = k0 + 64 * wave;             // the wave's first key (same in every lane)
        // the wave's K' fragments (keys kw + 32 s + l32 as rows, dims 16 kc +
        // 8 h) and V' values (value i of sub-tile s: key kw + 32 s + 8 (i / 4) +
        // 4 h + i % 4, dim 32 td + l32), all loads issued together; a key at or
        // past n reads row n - 1 instead (its weight is 0)
        bf16x8 kf[2][KC];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const Elem* kr = kc_base + static_cast<int64_t>(min(kw + 32 * s2 + l32, n - 1)) * D;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                if constexpr (F32) kf[s2][kc] = load_f32_as_bf16x8(kr + 16 * kc);
                else kf[s2][kc] = load_bf16x8(kr + 16 * kc);
            }
        }
        Elem vv[2][16];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                vv[s2][i] = vc_base[static_cast<int64_t>(min(kw + 32 * s2 + 8 * (i >> 2) + 4 * h + (i & 3), n - 1)) * D];
        floatx16 sv[2];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) sv[s2] = mfma_32x32x16(kf[s2][kc], qf[kc], kc == 0 ? zero16() : sv[s2]);
        // keys past n drop out; the wave's row maxima
        float mloc = -INFINITY;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int key = kw + 32 * s2 + 8 * (i >> 2) + 4 * h + (i & 3);
                if (key >= n) sv[s2][i] = -INFINITY;
                mloc = fmaxf(mloc, sv[s2][i]);
            }
        mloc = pair_max2(mloc);
        if (lane < 32) mx_w[wave][lane] = mloc;
        __syncthreads();
        float mc = mx_w[0][l32];
#pragma unroll
        for (int w = 1; w < kDecWaves; ++w) mc = fmaxf(mc, mx_w[w][l32]);
        const float Mn = fmaxf(M, mc);             // finite: key k0 < n is in this chunk
        const float fac = M == -INFINITY ? 0.f : fast_exp2(M - Mn);
        M = Mn;
        if (wave == 0 && lane < 32) fac_s[lane] = fac;
        float ps = 0.f;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float p = fast_exp2(sv[s2][i] - Mn);
                sv[s2][i] = p;
                ps += p;
            }
        lsum = lsum * fac + ps;
        __syncthreads();
        if (k0 > 0) {
            // rows 8 m4 + 4 h + j of the output values
#pragma unroll
            for (int m4 = 0; m4 < 4; ++m4) {
                const float4 f = *reinterpret_cast<const float4*>(fac_s + 8 * m4 + 4 * h);
                o[4 * m4 + 0] *= f.x;
                o[4 * m4 + 1] *= f.y;
                o[4 * m4 + 2] *= f.z;
                o[4 * m4 + 3] *= f.w;
            }
        }
        // O += P V'
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            if constexpr (F32) {
#pragma unroll
                for (int i = 0; i < 16; ++i) o = __builtin_amdgcn_mfma_f32_32x32x2f32(sv[s2][i], vv[s2][i], o, 0, 0, 0);
            } else {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    u32x4 hi, lo, vw;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const int i = 8 * kk + 2 * w;
                        const float p0 = sv[s2][i], p1 = sv[s2][i + 1];
                        const uint32_t hb = pack_bf16(p0, p1);
                        hi[w] = hb;
                        lo[w] = pack_bf16(p0 - __uint_as_float(hb << 16), p1 - __uint_as_float(hb & 0xFFFF0000u));
                        vw[w] = static_cast<uint32_t>(vv[s2][i]) | (static_cast<uint32_t>(vv[s2][i + 1]) << 16);
                    }
                    const bf16x8 vf = __builtin_bit_cast(bf16x8, vw);
                    o = mfma_32x32x16(__builtin_bit_cast(bf16x8, hi), vf, o);
                    o = mfma_32x32x16(__builtin_bit_cast(bf16x8, lo), vf, o);
                }
            }
        }
    }
    // coverage partials merged in the thread, over the lanes of the same row,
    // then over the waves through LDS
    float m = -INFINITY, sa = 0.f, sk = 0.f;
    auto merge = [&](float vm, float va, float vk) {
        if (vm == -INFINITY) return;
        const float mn = fmaxf(m, vm);
        const float fo = m == -INFINITY ? 0.f : exp2f(m - mn), fv = exp2f(vm - mn);
        sa = sa * fo + va * fv;
        sk = sk * fo + vk * fv;
        m = mn;
    };
    for (int kb0 = 0; kb0 < a.n_kb; kb0 += kCovGroups * kCovPer) {
        if (kb0 > 0) {
#pragma unroll
            for (int j = 0; j < kCovPer; ++j)
                pv[j] = pp[static_cast<int64_t>(min(kb0 + cg + kCovGroups * j, a.n_kb - 1)) * a.rows_pad];
        }
#pragma unroll
        for (int j = 0; j < kCovPer; ++j)
            if (kb0 + cg + kCovGroups * j < a.n_kb) merge(pv[j].x, pv[j].y, pv[j].z);
    }
#pragma unroll
    for (int x = kCovRows; x < kWave; x <<= 1) {
        const float om = __shfl_xor(m, x), oa = __shfl_xor(sa, x), ok = __shfl_xor(sk, x);
        merge(om, oa, ok);
    }
    if (lane < kCovRows) cov_w[wave][lane] = make_float4(m, sa, sk, 0.f);
    // the waves' partial outputs and sums
    const float L = pair_sum2(lsum);
#pragma unroll
    for (int i = 0; i < 16; ++i) ob[wave][(8 * (i >> 2) + 4 * h + (i & 3)) * 32 + l32] = o[i];
    if (lane < 32) l_w[wave][lane] = L;
    __syncthreads();
    // element (row r of the head, 0) of [B, Hq, n_dec] arrays: consecutive rows
    const int64_t row0 = (static_cast<int64_t>(b) * a.Hq + static_cast<int64_t>(c) * a.Gh) * a.n_dec;
    // thread tid: row tid / 8, dims 32 td + 4 (tid % 8) ..
    const int r = tid >> 3, row = 32 * tile + r;
    if (row < a.rows) {
        float tot = 0.f;
        float4 acc4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < kDecWaves; ++w) {
            tot += l_w[w][r];
            const float4 v = *reinterpret_cast<const float4*>(&ob[w][r * 32 + 4 * (tid & 7)]);
            acc4.x += v.x; acc4.y += v.y; acc4.z += v.z; acc4.w += v.w;
        }
        const float inv = tot > 0.f ? 1.f / tot : 0.f;
        *reinterpret_cast<float4*>(a.out + (row0 + row) * D + 32 * td + 4 * (tid & 7)) =
            make_float4(acc4.x * inv, acc4.y * inv, acc4.z * inv, acc4.w * inv);
    }
    // coverage = (kept sums) / (all sums), both rescaled to the row's largest
    // block maximum
    if (tid < kCovRows) {
        m = -INFINITY;
        sa = 0.f;
        sk = 0.f;
#pragma unroll
        for (int w = 0; w < kDecWaves; ++w) merge(cov_w[w][tid].x, cov_w[w][tid].y, cov_w[w][tid].z);
        const int crow = 32 * tile + kCovRows * td + tid;
        if (crow < a.rows) a.coverage[row0 + crow] = sk / sa;
    }
}

template <int D, bool F32>
hipError_t decode_impl(const DecodeArgs& a, hipStream_t s) {
    // queries of 256 rows at most (64 KiB at d = 128), and the waves' rows
    const size_t lds = static_cast<size_t>(a.rows_pad) * (D / 8) * 16 + 3 * kDecWaves * sizeof(float) * a.rows_pad;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_cover_kernel<D, F32>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_cover_kernel<D, F32>), dim3(a.n_kb, a.B * a.Hkv), dim3(64 * kDecWaves), lds, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_attend_kernel<D, F32>), dim3(a.rows_pad / 32 * (D / 32), a.B * a.Hkv),
                       dim3(64 * kDecWaves), 0, s, a);
    return hipGetLastError();
}

}  // namespace

int decode_rows_pad(int Gh, int n_dec) { return (Gh * n_dec + 31) / 32 * 32; }
int decode_max_rows() { return kDecMaxRows; }
int decode_max_compact() { return kDecMaxCompact; }
int decode_key_blocks(int T) { return (T + kDecKeys - 1) / kDecKeys; }

hipError_t launch_decode_check(const DecodeArgs& a, hipStream_t s) {
    if (a.d == 64) return a.k_dtype == 1 ? decode_impl<64, false>(a, s) : decode_impl<64, true>(a, s);
    return a.k_dtype == 1 ? decode_impl<128, false>(a, s) : decode_impl<128, true>(a, s);
}

}  // namespace mmskv
