// Hidden-state form of the proxies (Sec. 3.2.1 Eqs. 4-6 as written, and
// Algorithm 1): statistics of a layer's prefill hidden states, variance-
// expanded samples of them, and their projection by every head's query
// weights, on gfx950.
//
// hidden_stats   per (batch row, feature): S = sum h and SS = sum h^2 over
//                chunks of tokens (token order inside a chunk, one thread
//                per 8 features, fp64), then the chunk sums in eight parts of
//                chunk order;
//                mean = S/T, std = sqrt((SS - S*mean)/(T - ddof)).
// hidden_proxies x = mu + (gamma*sigma) z per (batch row, sample, feature),
//                z from the counter-based generator with the head field set
//                to 0xFFFFFFFF (one set of samples per layer, shared by all
//                heads), fp64 -> fp32 -> bf16.
// project        q[b, h, i, :] = W_Q^(h) H~[b, i, :]: a bf16 GEMM of the
//                (B*P) x D samples against the (Hq*d) x D weights (both with
//                the reduction dimension contiguous) with fp32 accumulation.
//                Full tiles (of four sizes, by the matrix): four waves on
//                v_mfma_f32_16x16x32_bf16.  Otherwise 128x128 tiles of four
//                64x64 waves on v_mfma_f32_32x32x16_bf16.  The epilogue goes
//                through LDS so that the rotary pairs (e, e + d/2) of a head
//                meet in one thread; both multiply by the query scale
//                log2(e)/sqrt(d) in fp64 and round to bf16.
#pragma clang fp contract(off)

#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "normal.hpp"

namespace mmskv {
namespace {

constexpr int kStatThreads = 64;           // one wave per workgroup (no shared state)

// fp32 value times the query scale, in fp64, rounded back to fp32.
__device__ __forceinline__ float scaled(float v, double scale) {
    const double y = static_cast<double>(v) * scale;
    return static_cast<float>(y);
}
constexpr int kStatVec = 8;                 // features per thread (one 16-byte bf16 load)
constexpr int kStatFlight = 8;              // tokens per group of loads in flight
constexpr int kStatWaves = 4 * kPlanCus;    // waves of the chunk sums below which chunks are halved

// Running sums of one token's kStatVec features.  The square of a bf16 or fp32
// value is exact in fp64, so the fused multiply-add rounds exactly like a
// separate product and sum.
__device__ __forceinline__ void accum_token(const double (&v)[kStatVec], double (&s)[kStatVec],
                                       double (&ss)[kStatVec]) {
#pragma unroll
    for (int e = 0; e < kStatVec; ++e) {
        s[e] = s[e] + v[e];
        ss[e] = fma(v[e], v[e], ss[e]);
    }
}

__device__ __forceinline__ void unpack_bf16x8(const u32x4& r, double (&v)[kStatVec]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[2 * q] = static_cast<double>(__uint_as_float(r[q] << 16));
        v[2 * q + 1] = static_cast<double>(__uint_as_float(r[q] & 0xFFFF0000u));
    }
}

__device__ __forceinline__ void unpack_f32x8(const float4 (&r)[2], double (&v)[kStatVec]) {
    v[0] = r[0].x; v[1] = r[0].y; v[2] = r[0].z; v[3] = r[0].w;
    v[4] = r[1].x; v[5] = r[1].y; v[6] = r[1].z; v[7] = r[1].w;
}

// Chunk sums: grid (n_chunks, ceil(D / (8*64)), B); thread j owns features
// [8j, 8j+8) of the block and sums them over the chunk's tokens in token
// order.  The raw loads of the next group of tokens (kStatFlight of bf16 rows,
// half as many of fp32 rows) are issued before the current ones are summed
// (two register sets used in turn), so up to two groups of loads are in flight
// per thread.
__global__ void __launch_bounds__(kStatThreads) hidden_stats_partial_kernel(HiddenArgs a) {
    const int c = blockIdx.x, b = blockIdx.z;
    const int j0 = (static_cast<int>(blockIdx.y) * kStatThreads + static_cast<int>(threadIdx.x)) * kStatVec;
    if (j0 >= a.D) return;
    const int t0 = c * a.chunk, t1 = min(t0 + a.chunk, a.T);
    double s[kStatVec], ss[kStatVec];
#pragma unroll
    for (int e = 0; e < kStatVec; ++e) { s[e] = 0.0; ss[e] = 0.0; }
    const int64_t base = static_cast<int64_t>(b) * a.sb + j0;
    // tokens [t0, t1) in groups of F, load(t, raw) and unpack(raw, values) per token
    auto sweep = [&](auto& ra, auto& rb, auto load, auto unpack) {
        constexpr int F = sizeof(ra) / sizeof(ra[0]);
        auto fetch = [&](int t, auto& r) {
#pragma unroll
            for (int u = 0; u < F; ++u)
                if (t + u < t1) load(t + u, r[u]);
        };
        auto sum = [&](int t, auto& r) {
#pragma unroll
            for (int u = 0; u < F; ++u) {
                if (t + u < t1) {
                    double v[kStatVec];
                    unpack(r[u], v);
                    accum_token(v, s, ss);
                }
            }
        };
        // two register sets, A for tokens [t, t+F), B for [t+F, t+2F)
        fetch(t0, ra);
        for (int t = t0; t < t1; t += 2 * F) {
            if (t + F < t1) fetch(t + F, rb);
            sum(t, ra);
            if (t + 2 * F < t1) fetch(t + 2 * F, ra);
            if (t + F < t1) sum(t + F, rb);
        }
    };
    if (a.dtype == 1) {
        const uint16_t* h = static_cast<const uint16_t*>(a.hidden) + base;
        u32x4 ra[kStatFlight], rb[kStatFlight];
        sweep(ra, rb, [&](int t, u32x4& r) { r = *reinterpret_cast<const u32x4*>(h + static_cast<int64_t>(t) * a.st); },
              [](const u32x4& r, double (&v)[kStatVec]) { unpack_bf16x8(r, v); });
    } else {
        const float* h = static_cast<const float*>(a.hidden) + base;
        float4 ra[kStatFlight / 2][2], rb[kStatFlight / 2][2];
        sweep(ra, rb,
              [&](int t, float4 (&r)[2]) {
                  const float4* p = reinterpret_cast<const float4*>(h + static_cast<int64_t>(t) * a.st);
                  r[0] = p[0];
                  r[1] = p[1];
              },
              [](const float4 (&r)[2], double (&v)[kStatVec]) { unpack_f32x8(r, v); });
    }
    double2* out = a.partial + (static_cast<int64_t>(b) * a.n_chunks + c) * a.D + j0;
#pragma unroll
    for (int e = 0; e < kStatVec; ++e) out[e] = make_double2(s[e], ss[e]);
}

// Chunk sums -> mean, std: grid (ceil(D/32), B); thread (feature, eighth e of
// the chunks) adds its chunks in order, kFinalBatch of them fetched at once
// (their latencies overlap), then one thread per feature the eighths in order.
constexpr int kFinalFeatures = 32, kFinalParts = 8;
__global__ void __launch_bounds__(kFinalFeatures * kFinalParts) hidden_stats_final_kernel(HiddenArgs a) {
    __shared__ double2 part[kFinalParts][kFinalFeatures];
    const int f = static_cast<int>(threadIdx.x) % kFinalFeatures, e = static_cast<int>(threadIdx.x) / kFinalFeatures;
    const int j = static_cast<int>(blockIdx.x) * kFinalFeatures + f, b = blockIdx.y;
    double S = 0.0, SS = 0.0;
    if (j < a.D) {
        const double2* p = a.partial + static_cast<int64_t>(b) * a.n_chunks * a.D + j;
        const int c0 = static_cast<int>(static_cast<int64_t>(a.n_chunks) * e / kFinalParts);
        const int c1 = static_cast<int>(static_cast<int64_t>(a.n_chunks) * (e + 1) / kFinalParts);
        constexpr int kFinalBatch = 8;
        for (int c = c0; c < c1; c += kFinalBatch) {
            double2 v[kFinalBatch];
#pragma unroll
            for (int u = 0; u < kFinalBatch; ++u)
                if (c + u < c1) v[u] = p[static_cast<int64_t>(c + u) * a.D];
#pragma unroll
            for (int u = 0; u < kFinalBatch; ++u) {
                if (c + u < c1) {
                    S = S + v[u].x;
                    SS = SS + v[u].y;
                }
            }
        }
    }
    part[e][f] = make_double2(S, SS);
    __syncthreads();
    if (e > 0 || j >= a.D) return;
#pragma unroll
    for (int q = 1; q < kFinalParts; ++q) {
        S = S + part[q][f].x;
        SS = SS + part[q][f].y;
    }
    const double mean = S / static_cast<double>(a.T);
    const double sm = S * mean;
    double var = (SS - sm) / static_cast<double>(a.T - a.ddof);
    if (var < 0.0) var = 0.0;
    a.stats[(static_cast<int64_t>(b) * 2) * a.D + j] = mean;
    a.stats[(static_cast<int64_t>(b) * 2 + 1) * a.D + j] = sqrt(var);
}

// Samples: one thread per (sample i, feature quad jq); grid (ceil(P*D/4 / 256), B).
__global__ void __launch_bounds__(256) hidden_proxies_kernel(HiddenArgs a) {
    const int b = blockIdx.y;
    const int quads = a.D / 4;
    const int64_t item0 = static_cast<int64_t>(blockIdx.x) * 256;
    if (item0 + threadIdx.x >= static_cast<int64_t>(a.P) * quads) return;
    // (the 64-bit division once per workgroup, in scalars)
    const int i0 = static_cast<int>(item0 / quads);
    const uint32_t r = static_cast<uint32_t>(item0 - static_cast<int64_t>(i0) * quads) + threadIdx.x;
    const int i = i0 + static_cast<int>(r / static_cast<uint32_t>(quads)), jq = static_cast<int>(r % static_cast<uint32_t>(quads));
    const double* mu = a.stats + (static_cast<int64_t>(b) * 2) * a.D;
    const double* sg = a.stats + (static_cast<int64_t>(b) * 2 + 1) * a.D;
    double z[4];
    normal_quad(a.key0, a.key1, b, a.layer, -1, i, jq, z);
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = 4 * jq + e;
        const double gs = a.gamma * sg[j];
        const double t = gs * z[e];
        const double x = mu[j] + t;
        o[e] = static_cast<float>(x);
    }
    const uint2 pk = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
    *reinterpret_cast<uint2*>(a.hp + (static_cast<int64_t>(b) * a.P + i) * a.D + 4 * jq) = pk;
}

// ------------------------------------------------------------ projection GEMM
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kBM = 128, kBN = 128, kBK = 64;
constexpr int kGemmThreads = 256;
constexpr int kRowChunks = kBK / 8;            // 16-byte chunks per tile row
constexpr int kRowSlots = kRowChunks + 1;      // padded row (one spare chunk)
constexpr int kTileSlots = kBM * kRowSlots;    // per operand tile
constexpr int kLoads = kBM * kRowChunks / kGemmThreads;   // chunks per thread per operand

__device__ __forceinline__ floatx16 mfma32(bf16x8 a, bf16x8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Rows r of A (M x K) and of W (N x K) in 16-byte chunks; rows past the
// matrix and k past D read as zero.
struct GemmStage {
    u32x4 a[kLoads], w[kLoads];
};

__device__ __forceinline__ void gemm_fetch(const ProjectArgs& p, int m0, int n0, int k0, GemmStage& st) {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int c = static_cast<int>(threadIdx.x) + q * kGemmThreads;
        const int r = c / kRowChunks, kc = c % kRowChunks;
        const int k = k0 + 8 * kc;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        st.a[q] = (m0 + r < p.M && k < p.K)
                      ? *reinterpret_cast<const u32x4*>(p.a + static_cast<int64_t>(m0 + r) * p.K + k) : zero;
        st.w[q] = (n0 + r < p.N && k < p.K)
                      ? *reinterpret_cast<const u32x4*>(p.w + static_cast<int64_t>(n0 + r) * p.K + k) : zero;
    }
}

__device__ __forceinline__ void gemm_store(const GemmStage& st, u32x4* la, u32x4* lw) {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int c = static_cast<int>(threadIdx.x) + q * kGemmThreads;
        const int r = c / kRowChunks, kc = c % kRowChunks;
        la[r * kRowSlots + kc] = st.a[q];
        lw[r * kRowSlots + kc] = st.w[q];
    }
}

// Rotary pair (x0, x1), scaled.
__device__ __forceinline__ void rotate_pair(float x0, float x1, float c, float s, double scale, float& lo, float& hi) {
    const float a0 = x0 * c, a1 = x1 * s, b0 = x1 * c, b1 = x0 * s;
    lo = scaled(a0 - a1, scale);
    hi = scaled(b0 + b1, scale);
}

// Epilogue of a 128 x 128 output tile: the fp32 accumulators (wave (wm, wn)
// holds rows wm*64.., columns wn*64..) through LDS, then the rotary pairs,
// the softmax scale and the bf16 rounding, to the proxies' layout.
__device__ __forceinline__ void project_epilogue(const ProjectArgs& p, const floatx16 (&acc)[2][2], u32x4* lds,
                                                 int m0, int n0, int wm, int wn, int lane) {
    constexpr int kLd = kBN + 4;
    float* tile = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int r = wm * 64 + 32 * x + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
                const int cc = wn * 64 + 32 * y + (lane & 31);
                tile[r * kLd + cc] = acc[x][y][i];
            }
    __syncthreads();
    const int d = p.d, half = d / 2;
    const bool rope = p.cos != nullptr;
    // each thread: one row, 8 consecutive output columns (one head's
    // lower half when rotary pairs are formed)
    const int groups = rope ? kBN / 16 : kBN / 8;     // 8-column groups per row
    for (int g = static_cast<int>(threadIdx.x); g < kBM * groups; g += kGemmThreads) {
        const int r = g / groups, cg = g % groups;
        const int m = m0 + r;
        if (m >= p.M) continue;
        const int bb = m / p.P, i = m % p.P;
        int col;
        if (rope) {
            const int c8 = cg * 8;                     // lower-half column index inside the tile's heads
            col = (c8 / half) * d + (c8 % half);
        } else {
            col = cg * 8;
        }
        const int n = n0 + col;
        if (n >= p.N) continue;
        const int h = n / d, e = n % d;
        uint16_t* out = p.out + ((static_cast<int64_t>(bb) * p.Hq + h) * p.P + i) * d;
        u32x4 lo, hi;
        if (!rope) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                lo[q] = pack_bf16(scaled(tile[r * kLd + col + 2 * q], p.scale), scaled(tile[r * kLd + col + 2 * q + 1], p.scale));
            *reinterpret_cast<u32x4*>(out + e) = lo;
        } else {
            float lx[8], hx[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                rotate_pair(tile[r * kLd + col + q], tile[r * kLd + col + half + q], p.cos[e + q], p.sin[e + q], p.scale,
                            lx[q], hx[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                lo[q] = pack_bf16(lx[2 * q], lx[2 * q + 1]);
                hi[q] = pack_bf16(hx[2 * q], hx[2 * q + 1]);
            }
            *reinterpret_cast<u32x4*>(out + e) = lo;
            *reinterpret_cast<u32x4*>(out + e + half) = hi;
        }
    }
}

// Any shape (ragged tiles): register-staged loads, two LDS stages.
__global__ void __launch_bounds__(kGemmThreads) project_kernel(ProjectArgs p) {
    // two stages of (A tile, W tile); the fp32 output tile reuses the space
    __shared__ u32x4 lds[2 * 2 * kTileSlots];
    const int m0 = static_cast<int>(blockIdx.x) * kBM, n0 = static_cast<int>(blockIdx.y) * kBN;
    const int wave = static_cast<int>(threadIdx.x) / kWave, lane = lane_id();
    const int wm = wave >> 1, wn = wave & 1;           // 64 x 64 quadrant of the wave
    const int n_k = (p.K + kBK - 1) / kBK;

    floatx16 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[x][y][i] = 0.f;

    // k steps: LDS holds steps ks (being multiplied) and ks+1 (written during
    // step ks); two register stages hold the global loads of steps ks+1 and
    // ks+2, so every load has two steps of MFMA work to arrive in
    GemmStage s0, s1;
    gemm_fetch(p, m0, n0, 0, s0);
    gemm_store(s0, lds, lds + kTileSlots);
    if (1 < n_k) gemm_fetch(p, m0, n0, kBK, s1);
    if (2 < n_k) gemm_fetch(p, m0, n0, 2 * kBK, s0);
    __syncthreads();
    // step ks; `nx` holds the loads of step ks+1 and is refilled with ks+3
    auto step = [&](int ks, GemmStage& nx) {
        const int cur = ks & 1;
        const u32x4* la = lds + cur * 2 * kTileSlots;
        const u32x4* lw = la + kTileSlots;
#pragma unroll
        for (int kc = 0; kc < kBK / 16; ++kc) {
            bf16x8 fa[2], fw[2];
            const int chunk = 2 * kc + (lane >> 5);
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                fa[x] = __builtin_bit_cast(bf16x8, la[(wm * 64 + 32 * x + (lane & 31)) * kRowSlots + chunk]);
                fw[x] = __builtin_bit_cast(bf16x8, lw[(wn * 64 + 32 * x + (lane & 31)) * kRowSlots + chunk]);
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) acc[x][y] = mfma32(fa[x], fw[y], acc[x][y]);
        }
        if (ks + 1 < n_k) {
            u32x4* na = lds + (cur ^ 1) * 2 * kTileSlots;
            gemm_store(nx, na, na + kTileSlots);
            if (ks + 3 < n_k) gemm_fetch(p, m0, n0, (ks + 3) * kBK, nx);
        }
        __syncthreads();
    };
    int ks = 0;
    for (; ks < n_k; ks += 2) {
        step(ks, s1);
        if (ks + 1 < n_k) step(ks + 1, s0);
    }

    project_epilogue(p, acc, lds, m0, n0, wm, wn, lane);
}

// Full TM x TN output tiles (TM = 32 AX, TN = 32 AY), four waves of 16 AX x
// 16 AY on v_mfma_f32_16x16x32_bf16.  A k step is 64 wide and lands in one of
// NS LDS stages by direct loads: each wave issues AX + AY of the step's loads
// of 8 rows x 128 bytes, from a uniform base advanced per step plus
// loop-invariant 32-bit lane offsets (chunk c of row r at slot c ^ (r & 7)).
// A step runs its two 32-wide halves back to back: the A fragments of the
// next half are read before a half's MFMAs, and each W fragment is refilled
// right after the MFMAs that last read it.  The barrier sits between the
// halves: by then every wave has its own loads of the next stage and its
// reads of the current one complete, so after it the next stage can be read
// and the loads NS steps ahead overwrite the current stage.
// ROPE: columns [0, TN/2) of a tile are the lower columns of TN/2 rotary pairs
// and the rest their partners, so that a pair meets in one row of the tile.
constexpr int kWK = 64;
constexpr int kWRow = kWK * 2;                      // bytes per staged row
template <int AX, int AY, int NS>
struct WideTile {
    static constexpr int kM = 32 * AX, kN = 32 * AY;
    static constexpr int kTileA = kM * kWRow;       // the A rows of a stage
    static constexpr int kStage = (kM + kN) * kWRow;
    // loads per wave and stage: the four waves issue the 8-row groups in
    // turn, the A tile's 4 AX groups being loads j < AX of every wave
    static constexpr int kLoads = AX + AY;
    static constexpr int kLd = kN + 4;              // epilogue row pitch (floats)
    static constexpr int kLds = NS * kStage > kM * kLd * 4 ? NS * kStage : kM * kLd * 4;
};
typedef float floatx4 __attribute__((ext_vector_type(4)));
template <int N>
struct Tag {
    static constexpr int value = N;
};

__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 16 bytes per lane from memory to LDS (dst + 16 * lane)
__device__ __forceinline__ void load16_to_lds(const char* src, char* dst) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// s_waitcnt with vmcnt = N and the other counters not waited on
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// s_waitcnt vmcnt(N) lgkmcnt(0)
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
    static_assert(N < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

template <int AX, int AY, int NS, bool ROPE>
__global__ void __launch_bounds__(kGemmThreads) project_wide_kernel(ProjectArgs p) {
    using T = WideTile<AX, AY, NS>;
    static_assert(NS >= 2 && NS <= 4, "the waits count up to two later stages");
    __shared__ u32x4 lds[T::kLds / 16];
    char* base = reinterpret_cast<char*>(lds);
    const int half = p.d / 2;
    const int nN = p.N / T::kN;
    const int m0 = static_cast<int>(blockIdx.x) / nN * T::kM, n0 = static_cast<int>(blockIdx.x) % nN * T::kN;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave), lane = lane_id();
    const int wm = wave >> 1, wn = wave & 1;
    const int n_k = p.K / kWK;                      // at least NS (checked by the host)
    floatx4 acc[AX][AY];
#pragma unroll
    for (int x = 0; x < AX; ++x)
#pragma unroll
        for (int y = 0; y < AY; ++y) acc[x][y] = floatx4{0.f, 0.f, 0.f, 0.f};

    // load j of a stage: rows 8 (wave + 4 j) .. + 7 of the A tile (j < AX) or
    // of the W tile (j >= AX, less 4 AX groups); lane -> row + (lane >> 3),
    // slot lane & 7; offsets from the tile's first row (m0, w0)
    const int w0 = ROPE ? n0 / 2 / half * p.d + n0 / 2 % half : n0;
    uint32_t voff[T::kLoads];
#pragma unroll
    for (int j = 0; j < T::kLoads; ++j) {
        const int g = wave + 4 * j - (j < AX ? 0 : 4 * AX);
        const int r = 8 * g + (lane >> 3);
        int row = r;
        if (ROPE && j >= AX) {
            // rotary pair n0 / 2 + r % (TN / 2): its lower column, or its upper one
            const int hi = r >= T::kN / 2 ? 1 : 0, pr = n0 / 2 + r - hi * (T::kN / 2);
            row = pr / half * p.d + pr % half + hi * half - w0;
        }
        voff[j] = static_cast<uint32_t>(row * p.K * 2 + 16 * ((lane & 7) ^ (r & 7)));
    }
    const char* a0 = reinterpret_cast<const char*>(p.a + static_cast<int64_t>(m0) * p.K);
    const char* wr0 = reinterpret_cast<const char*>(p.w + static_cast<int64_t>(w0) * p.K);
    auto loads = [&](int k0, char* stage) {
        const char* ab = a0 + 2 * k0;
        const char* wb = wr0 + 2 * k0;
#pragma unroll
        for (int j = 0; j < T::kLoads; ++j) {
            const int g = wave + 4 * j - (j < AX ? 0 : 4 * AX);
            char* dst = stage + (j < AX ? 0 : T::kTileA) + 8 * g * kWRow;
            load16_to_lds((j < AX ? ab : wb) + voff[j], dst);
        }
    };
    // fragment rows wm*16*AX + 16x + (lane & 15) and wn*16*AY + 16y + (lane & 15)
    // (both = lane & 7 mod 8), 16-byte chunk 4 h + (lane >> 4) of half h
    const int rA = wm * 16 * AX + (lane & 15), rW = wn * 16 * AY + (lane & 15);
    const int oA0 = rA * kWRow + 16 * ((lane >> 4) ^ (lane & 7));
    const int oA1 = rA * kWRow + 16 * ((4 + (lane >> 4)) ^ (lane & 7));
    const int oW0 = T::kTileA + rW * kWRow + 16 * ((lane >> 4) ^ (lane & 7));
    const int oW1 = T::kTileA + rW * kWRow + 16 * ((4 + (lane >> 4)) ^ (lane & 7));
    auto rd = [&](const char* q) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(q)); };
    bf16x8 fa0[AX], fa1[AX], fw[AY];

#pragma unroll
    for (int st = 0; st < NS; ++st) loads(st * kWK, base + st * T::kStage);
    wait_vm<(NS - 1) * T::kLoads>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int x = 0; x < AX; ++x) fa0[x] = rd(base + oA0 + x * 16 * kWRow);
#pragma unroll
    for (int y = 0; y < AY; ++y) fw[y] = rd(base + oW0 + y * 16 * kWRow);

    // step ks on stage st (half 0's fragments already in fa0 / fw); nst is
    // the next stage; the loads of step ks + NS go to st.  LATER: stages in
    // flight after stage ks + 1 (min(NS - 2, n_k - 2 - ks)); -1: the last step
    auto step = [&](int ks, char* st, const char* nst, auto later_tag) {
        constexpr int kLater = decltype(later_tag)::value;
        constexpr bool kLast = kLater < 0;
#pragma unroll
        for (int x = 0; x < AX; ++x) fa1[x] = rd(st + oA1 + x * 16 * kWRow);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < AY; ++y) {
#pragma unroll
            for (int x = 0; x < AX; ++x) acc[x][y] = mfma16(fa0[x], fw[y], acc[x][y]);
            fw[y] = rd(st + oW1 + y * 16 * kWRow);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!kLast) {
            wait_vm_lgkm0<(kLast ? 0 : kLater) * T::kLoads>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (ks + NS < n_k) loads((ks + NS) * kWK, st);
#pragma unroll
            for (int x = 0; x < AX; ++x) fa0[x] = rd(nst + oA0 + x * 16 * kWRow);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < AY; ++y) {
#pragma unroll
            for (int x = 0; x < AX; ++x) acc[x][y] = mfma16(fa1[x], fw[y], acc[x][y]);
            if constexpr (!kLast) fw[y] = rd(nst + oW0 + y * 16 * kWRow);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int ks = 0;
    if constexpr (NS == 2) {
        for (; ks + 2 < n_k; ks += 2) {
            step(ks, base, base + T::kStage, Tag<0>{});
            step(ks + 1, base + T::kStage, base, Tag<0>{});
        }
        if (ks + 1 < n_k) {
            step(ks, base, base + T::kStage, Tag<0>{});
            ++ks;
        }
        step(ks, base + (ks & 1) * T::kStage, nullptr, Tag<-1>{});
    } else {
        int s0 = 0, s1 = 1;                         // stages of steps ks and ks + 1
        auto next = [&]() {
            ++ks;
            s0 = s1;
            s1 = s1 + 1 == NS ? 0 : s1 + 1;
        };
        for (; ks + NS <= n_k; next()) step(ks, base + s0 * T::kStage, base + s1 * T::kStage, Tag<NS - 2>{});
        if constexpr (NS == 4) {
            step(ks, base + s0 * T::kStage, base + s1 * T::kStage, Tag<1>{});
            next();
        }
        step(ks, base + s0 * T::kStage, base + s1 * T::kStage, Tag<0>{});
        next();
        step(ks, base + s0 * T::kStage, nullptr, Tag<-1>{});
    }

    // epilogue: the fp32 tile through LDS (every wave's stage reads are done),
    // then 8 consecutive columns of one row per thread and group: the query
    // scale in fp64, bf16, one 16-byte store into the proxies' layout
    asm volatile("" ::: "memory");
    __syncthreads();
    float* tile = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int x = 0; x < AX; ++x)
#pragma unroll
        for (int y = 0; y < AY; ++y)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                tile[(wm * 16 * AX + 16 * x + 4 * (lane >> 4) + i) * T::kLd + wn * 16 * AY + 16 * y + (lane & 15)] = acc[x][y][i];
    __syncthreads();
    if constexpr (ROPE) {
        // columns c .. c + 7 of a row with their partners TN / 2 columns on:
        // the same head's lower and upper half
        constexpr int kPairs = T::kN / 16;
        for (int g = static_cast<int>(threadIdx.x); g < T::kM * kPairs; g += kGemmThreads) {
            const int r = g / kPairs, c = 8 * (g % kPairs);
            const int m = m0 + r, pr = n0 / 2 + c;
            const int bb = m / p.P, i = m % p.P, h = pr / half, e = pr % half;
            const float* src = tile + r * T::kLd + c;
            float lx[8], hx[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                rotate_pair(src[q], src[T::kN / 2 + q], p.cos[e + q], p.sin[e + q], p.scale, lx[q], hx[q]);
            u32x4 lo, hi;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                lo[q] = pack_bf16(lx[2 * q], lx[2 * q + 1]);
                hi[q] = pack_bf16(hx[2 * q], hx[2 * q + 1]);
            }
            uint16_t* out = p.out + ((static_cast<int64_t>(bb) * p.Hq + h) * p.P + i) * p.d + e;
            *reinterpret_cast<u32x4*>(out) = lo;
            *reinterpret_cast<u32x4*>(out + half) = hi;
        }
        return;
    }
    constexpr int kGroups = T::kN / 8;
    for (int g = static_cast<int>(threadIdx.x); g < T::kM * kGroups; g += kGemmThreads) {
        const int r = g / kGroups, c = 8 * (g % kGroups);
        const int m = m0 + r, n = n0 + c;
        const int bb = m / p.P, i = m % p.P, h = n / p.d, e = n % p.d;
        const float* src = tile + r * T::kLd + c;
        u32x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = pack_bf16(scaled(src[2 * q], p.scale), scaled(src[2 * q + 1], p.scale));
        *reinterpret_cast<u32x4*>(p.out + ((static_cast<int64_t>(bb) * p.Hq + h) * p.P + i) * p.d + e) = v;
    }
}

template <int AX, int AY, int NS>
hipError_t launch_wide(const ProjectArgs& p, hipStream_t s) {
    using T = WideTile<AX, AY, NS>;
    const dim3 g((p.M / T::kM) * (p.N / T::kN));
    if (p.cos == nullptr) hipLaunchKernelGGL((project_wide_kernel<AX, AY, NS, false>), g, dim3(kGemmThreads), 0, s, p);
    else hipLaunchKernelGGL((project_wide_kernel<AX, AY, NS, true>), g, dim3(kGemmThreads), 0, s, p);
    return hipGetLastError();
}

// Tile sizes and the measured time of one k step of a round of workgroups
// (one per CU), in units of 10 ns: the loads, their wait and the barrier do not
// shrink with the tile, so a tile is only worth its size while the grid fills
// the CUs.  The two stages of a 128 x 128 tile leave a CU room for two
// workgroups, which wait at different times: slower while each has a CU to
// itself, and the fastest form of a grid of more (pair: the time of a round
// with two on each CU).
struct WideForm {
    int m, n, stages, cost, pair;
};
constexpr WideForm kWide[] = {{128, 224, 3, 104, 0}, {128, 128, 3, 68, 0}, {64, 128, 4, 44, 0}, {64, 64, 3, 33, 0},
                              {128, 128, 2, 85, 103}};

}  // namespace

// Tokens per chunk: 256, and fewer (a chunk has its own wave per 512 features)
// while the chunks leave most CUs without a wave, down to 32, below which the
// partials cost what the shorter chains gain.
int hidden_chunk(int B, int T, int D) {
    const int64_t waves = static_cast<int64_t>(B) * ((D + kStatThreads * kStatVec - 1) / (kStatThreads * kStatVec));
    int chunk = 256;
    while (chunk > 32 && waves * ((T + chunk - 1) / chunk) < kStatWaves) chunk /= 2;
    return chunk;
}

// Chunks of 256 tokens, or at most twice as many as leave less than
// kStatWaves waves (a halving doubles them), a wave being at most 512 features.
size_t hidden_partials_bound(int B, int T, int D) {
    const size_t BD = static_cast<size_t>(B) * D, t = static_cast<size_t>(T);
    const size_t whole = BD * ((t + 255) / 256), most = BD * ((t + 31) / 32);
    const size_t halved = 2 * static_cast<size_t>(kStatWaves) * kStatThreads * kStatVec;
    const size_t few = most < halved ? most : halved;
    return whole > few ? whole : few;
}

hipError_t launch_hidden_stats(const HiddenArgs& a, hipStream_t s) {
    dim3 g1(a.n_chunks, (a.D + kStatThreads * kStatVec - 1) / (kStatThreads * kStatVec), a.B);
    hipLaunchKernelGGL(hidden_stats_partial_kernel, g1, dim3(kStatThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 g2((a.D + kFinalFeatures - 1) / kFinalFeatures, a.B);
    hipLaunchKernelGGL(hidden_stats_final_kernel, g2, dim3(kFinalFeatures * kFinalParts), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_hidden_proxies(const HiddenArgs& a, hipStream_t s) {
    const int64_t items = static_cast<int64_t>(a.P) * (a.D / 4);
    dim3 g(static_cast<unsigned>((items + 255) / 256), a.B);
    hipLaunchKernelGGL(hidden_proxies_kernel, g, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_project(const ProjectArgs& p, hipStream_t s) {
    // the tile size with the smallest modelled time, among those that divide
    // the matrix and whose stages a reduction of K fills.  Measured (us), the
    // 128 x 128 and (2048 x 3584) 128 x 224 tiles in two stages that these
    // replace against the choice made here, M x N with K = N: 512 x 3584 47 ->
    // 25, 1024 x 3584 49 -> 37, 512 x 2048 24 -> 10.6, 1024 x 2048 25.6 -> 14.9,
    // 2048 x 2048 27.5 -> 22.5; 2048 x 3584 with rotary tables 68 -> 57.
    // 128 x 128 tiles in two stages, two workgroups on a CU, against the best of
    // the other forms, the weights from another buffer each time: 2048 x 3584
    // 57.4 and 59.1, 4096 x 3584 112 and 117, 2048 x 4096 67 and 84, 2048 x 8192
    // (K = N) 268 and 324, 1024 x 4096 (256 tiles, one a CU) 57 and 42.
    int best = -1;
    int64_t best_cost = 0;
    if (p.K % kWK == 0 && p.K <= (1 << 20)) {          // (lane offsets within 32 bits)
        for (int i = 0; i < 5; ++i) {
            const WideForm& f = kWide[i];
            if (p.M % f.m != 0 || p.N % f.n != 0 || p.K < f.stages * kWK) continue;
            const int64_t tiles = static_cast<int64_t>(p.M / f.m) * (p.N / f.n);
            int64_t cost = (tiles + kPlanCus - 1) / kPlanCus * f.cost;
            if (f.pair > 0) {
                const int64_t rest = tiles % (2 * kPlanCus);
                cost = tiles / (2 * kPlanCus) * f.pair + (rest > kPlanCus ? f.pair : rest > 0 ? f.cost : 0);
            }
            if (best < 0 || cost < best_cost) {
                best = i;
                best_cost = cost;
            }
        }
    }
    switch (best) {
        case 0: return launch_wide<4, 7, 3>(p, s);
        case 1: return launch_wide<4, 4, 3>(p, s);
        case 2: return launch_wide<2, 4, 4>(p, s);
        case 3: return launch_wide<2, 2, 3>(p, s);
        case 4: return launch_wide<4, 4, 2>(p, s);
        default: break;
    }
    dim3 g((p.M + kBM - 1) / kBM, (p.N + kBN - 1) / kBN);
    hipLaunchKernelGGL(project_kernel, g, dim3(kGemmThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace mmskv
