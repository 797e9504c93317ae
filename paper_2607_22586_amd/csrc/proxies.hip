// Variance-expanded query proxies (Sec. 3.2.1 Eqs. 4-5; Appendix A.4 Eq. 15)
// and the anchor query of Sec. 3.2.3 Eq. 11, on gfx950.
//
// Every floating-point step here is rounded on its own (no fused
// multiply-add), so the proxies are a fixed function of the inputs: window
// statistics summed in window order (fp64), Philox4x32-10 words, Box-Muller
// with series-evaluated ln / sin / cos (fp32, widened to fp64), the proxy
// formula and the softmax scale log2(e)/sqrt(d) that the queries carry
// (fp64; Sec. 3.2.2 Eq. 7, so the score products are base-2 logits), then
// fp64 -> fp32 -> bf16.  The anchor query is returned unscaled.
#pragma clang fp contract(off)

#include "common.hpp"
#include "kernels.hpp"
#include "normal.hpp"

namespace mmskv {
namespace {

constexpr int kProxyThreads = 256;
constexpr int kBlockDims = 16;      // dimensions (of every proxy of a head) per workgroup
constexpr int kWinChunk = 64;       // window rows staged in LDS at a time
constexpr int kStatBatch = 16;      // staged rows read per LDS round trip

__device__ __forceinline__ double load_q(const ProxyArgs& a, int64_t off) {
    if (a.q_dtype == 0) return static_cast<double>(static_cast<const float*>(a.q)[off]);
    const uint32_t bits = static_cast<uint32_t>(static_cast<const uint16_t*>(a.q)[off]) << 16;
    return static_cast<double>(__uint_as_float(bits));
}

__device__ __forceinline__ uint16_t to_bf16(double x) {
    return static_cast<uint16_t>(f32_to_bf16_bits(static_cast<float>(x)));
}

__global__ void __launch_bounds__(kProxyThreads) build_proxies_kernel(ProxyArgs a) {
    extern __shared__ double smem[];
    const int d = a.d, half = d / 2;
    double* mu = smem;            // [d]  (this block's dims only)
    double* gs = smem + d;        // [d]  gamma * sigma
    float* win = reinterpret_cast<float*>(smem + 2 * d);   // [kWinChunk][kBlockDims] staged window values
    const int h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int64_t qbase = static_cast<int64_t>(b) * a.qsb + static_cast<int64_t>(h) * a.qsh;

    // Workgroup x, part y of it, owns quads [x*qpb, (x+1)*qpb) of the part's
    // proxies of the head (with rotary placement also their partner quads d/8
    // further on), so it needs the statistics of kBlockDims = 16 dimensions
    // only.
    const bool rope = a.cos_f != nullptr;
    const int qsh = rope ? 1 : 2, qpb = 1 << qsh;
    static_assert(kBlockDims / 8 == 2 && kBlockDims / 4 == 4, "quads per workgroup");
    const int n_blocks = d / kBlockDims;
    const int part = static_cast<int>(blockIdx.x) / n_blocks, q0 = (static_cast<int>(blockIdx.x) % n_blocks) * qpb;
    const int parts = static_cast<int>(gridDim.x) / n_blocks;
    auto dim_of = [&](int slot) {
        return rope ? (slot < kBlockDims / 2 ? 4 * q0 + slot : half + 4 * q0 + slot - kBlockDims / 2) : 4 * q0 + slot;
    };
    // stage window rows [w0, w0 + n) of the block's dims in LDS (exact in fp32)
    auto stage = [&](int w0, int n) {
        for (int e = tid; e < n * kBlockDims; e += kProxyThreads) {
            const int w = e / kBlockDims, slot = e % kBlockDims;
            win[e] = static_cast<float>(load_q(a, qbase + static_cast<int64_t>(w0 + w) * a.qst + dim_of(slot)));
        }
    };
    // the draws of proxy i, quad jq, and with rotary placement of its partner
    // quad (the draws are fp32 values: keeping them as fp32 and widening later
    // is exact)
    auto draw = [&](int item, float (&z1)[4], float (&z2)[4]) {
        const int i = item >> qsh, jq = q0 + (item & (qpb - 1));
        double z[4];
        normal_quad(a.key0, a.key1, b, a.layer, h, i, jq, z);
#pragma unroll
        for (int e = 0; e < 4; ++e) z1[e] = static_cast<float>(z[e]);
        if (rope) normal_quad(a.key0, a.key1, b, a.layer, h, i, jq + d / 8, z);
#pragma unroll
        for (int e = 0; e < 4; ++e) z2[e] = rope ? static_cast<float>(z[e]) : 0.f;
    };
    const int n_items = static_cast<int>(static_cast<int64_t>(a.P) * (part + 1) / parts) << qsh;
    const int first = (static_cast<int>(static_cast<int64_t>(a.P) * part / parts) << qsh) + tid;
    // A window of up to kWinChunk rows is fetched by one round of loads (each
    // thread's at once), and this thread's first kPreItems items are drawn
    // before the statistics are published: every wave draws while the
    // statistics lanes run their serial sums.
    constexpr int kPreItems = 4;
    constexpr int kStagePer = kWinChunk * kBlockDims / kProxyThreads;
    const bool one_chunk = a.W <= kWinChunk;
    float zp[kPreItems][4], zp2[kPreItems][4];
    // element e of the window chunk: thread e % 256, load e / 256
    auto row_of = [&](int k) { return (tid + k * kProxyThreads) / kBlockDims; };
    if (one_chunk) {
        float sv[kStagePer];
        auto fetch = [&](auto* q) {
            const int64_t col = qbase + dim_of(tid % kBlockDims);
#pragma unroll
            for (int k = 0; k < kStagePer; ++k) {
                const auto x = q[col + static_cast<int64_t>(min(row_of(k), a.W - 1)) * a.qst];
                if constexpr (sizeof(x) == 4) sv[k] = x;
                else sv[k] = __uint_as_float(static_cast<uint32_t>(x) << 16);
            }
        };
        if (a.q_dtype == 0) fetch(static_cast<const float*>(a.q));
        else fetch(static_cast<const uint16_t*>(a.q));
#pragma unroll
        for (int k = 0; k < kStagePer; ++k)
            if (row_of(k) < a.W) win[tid + k * kProxyThreads] = sv[k];
        __syncthreads();
    }
    // mean, then (population or sample) variance, summed in window order;
    // thread `slot` < kBlockDims owns one dimension.  f(value) for the n
    // staged rows, kStatBatch of them per LDS round trip
    const bool owner = tid < kBlockDims;
    auto each_row = [&](int n, auto&& f) {
        int w = 0;
        for (; w + kStatBatch <= n; w += kStatBatch) {
            float v[kStatBatch];
#pragma unroll
            for (int k = 0; k < kStatBatch; ++k) v[k] = win[(w + k) * kBlockDims + tid];
#pragma unroll
            for (int k = 0; k < kStatBatch; ++k) f(static_cast<double>(v[k]));
        }
        for (; w < n; ++w) f(static_cast<double>(win[w * kBlockDims + tid]));
    };
    double acc = 0.0;
    for (int w0 = 0; w0 < a.W; w0 += kWinChunk) {
        const int n = min(kWinChunk, a.W - w0);
        if (!one_chunk) {
            __syncthreads();
            stage(w0, n);
            __syncthreads();
        }
        if (owner) each_row(n, [&](double v) { acc = acc + v; });
    }
    const double m = acc / static_cast<double>(a.W);
    double sq = 0.0;
    for (int w0 = 0; w0 < a.W; w0 += kWinChunk) {
        const int n = min(kWinChunk, a.W - w0);
        if (!one_chunk) {
            __syncthreads();
            stage(w0, n);
            __syncthreads();
        }
        if (owner) {
            each_row(n, [&](double v) {
                const double diff = v - m;
                const double dd = diff * diff;
                sq = sq + dd;
            });
        }
    }
    if (owner) {
        const int j = dim_of(tid);
        const double sg = sqrt(sq / static_cast<double>(a.W - a.ddof));
        mu[j] = m;
        gs[j] = a.gamma * sg;
        if (a.stats != nullptr && part == 0) {
            double* st = a.stats + (static_cast<int64_t>(b) * a.Hq + h) * 2 * d;
            st[j] = m;
            st[d + j] = sg;
        }
    }
    if (one_chunk) {
#pragma unroll
        for (int k = 0; k < kPreItems; ++k)
            if (first + k * kProxyThreads < n_items) draw(first + k * kProxyThreads, zp[k], zp2[k]);
    }
    __syncthreads();

    uint16_t* out_head = a.proxies + (static_cast<int64_t>(b) * a.Hq + h) * a.P * d;
    // proxy i, quad jq from its draws z (and z2, the partner quad's, with rotary placement)
    auto emit = [&](int i, int jq, const double (&z)[4], const double (&z2)[4]) {
        uint16_t* row = out_head + static_cast<int64_t>(i) * d;
        double x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 4 * jq + e;
            const double t = gs[j] * z[e];
            x[e] = mu[j] + t;
        }
        if (!rope) {
            double sx[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) sx[e] = x[e] * a.scale;
            uint2 pk;
            pk.x = pack_bf16(static_cast<float>(sx[0]), static_cast<float>(sx[1]));
            pk.y = pack_bf16(static_cast<float>(sx[2]), static_cast<float>(sx[3]));
            *reinterpret_cast<uint2*>(row + 4 * jq) = pk;
        } else {
            // partner dims j + d/2 come from quad jq + d/8
            const int jq2 = jq + d / 8;
            double y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 4 * jq2 + e;
                const double t = gs[j] * z2[e];
                y[e] = mu[j] + t;
            }
            float lo[4], hi[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 4 * jq + e;
                const double c = static_cast<double>(a.cos_f[j]), s = static_cast<double>(a.sin_f[j]);
                const double a0 = x[e] * c, a1 = y[e] * s;
                const double b0 = y[e] * c, b1 = x[e] * s;
                const double rl = a0 - a1, rh = b0 + b1;
                lo[e] = static_cast<float>(rl * a.scale);
                hi[e] = static_cast<float>(rh * a.scale);
            }
            const uint2 pl = make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]));
            const uint2 ph = make_uint2(pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3]));
            *reinterpret_cast<uint2*>(row + 4 * jq) = pl;
            *reinterpret_cast<uint2*>(row + half + 4 * jq) = ph;
        }
    };
    int item = first;
    if (one_chunk) {
#pragma unroll
        for (int k = 0; k < kPreItems; ++k, item += kProxyThreads) {
            if (item < n_items) {
                double z[4], z2[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    z[e] = static_cast<double>(zp[k][e]);
                    z2[e] = static_cast<double>(zp2[k][e]);
                }
                emit(item >> qsh, q0 + (item & (qpb - 1)), z, z2);
            }
        }
    }
    for (; item < n_items; item += kProxyThreads) {
        float z1[4], zr[4];
        draw(item, z1, zr);
        double z[4], z2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            z[e] = static_cast<double>(z1[e]);
            z2[e] = static_cast<double>(zr[e]);
        }
        emit(item >> qsh, q0 + (item & (qpb - 1)), z, z2);
    }

    // anchor query: window row W-1, all dims, by workgroup 0
    if (blockIdx.x == 0) {
        uint16_t* ql = a.q_last + (static_cast<int64_t>(b) * a.Hq + h) * d;
        const int64_t lrow = qbase + static_cast<int64_t>(a.W - 1) * a.qst;
        const bool rope_l = a.cos_l != nullptr;
        for (int j = tid; j < d; j += kProxyThreads) {
            double v = load_q(a, lrow + j);
            if (rope_l) {
                if (j < half) {
                    const double c = static_cast<double>(a.cos_l[j]), s = static_cast<double>(a.sin_l[j]);
                    const double a0 = v * c, a1 = load_q(a, lrow + j + half) * s;
                    v = a0 - a1;
                } else {
                    const int jj = j - half;
                    const double c = static_cast<double>(a.cos_l[jj]), s = static_cast<double>(a.sin_l[jj]);
                    const double b0 = v * c, b1 = load_q(a, lrow + jj) * s;
                    v = b0 + b1;
                }
            }
            ql[j] = to_bf16(v);
        }
    }
}

}  // namespace

hipError_t launch_build_proxies(const ProxyArgs& a, hipStream_t s) {
    // Few heads leave CUs without a workgroup (4 heads of 64: 16), and one wave a
    // SIMD has nothing to hide the window's loads and the serial sums behind:
    // a head's proxies are then shared by several workgroups, which each form
    // the statistics anew.  More than two workgroups per CU cost more than they
    // gain.  Measured (us), window loads one at a time and one part / one round
    // of loads and one part / the parts chosen here: 4 heads of 64, W = 16 9.4 /
    // 8.7 / 4.2, 28 heads of 128, W = 32 12.3 / 10.2 / 9.1 (1024 workgroups 10.7,
    // 2048 15.5); 4 x 28 heads, W = 64 25.3 / 20.8, one part either way.
    const int blocks = a.d / kBlockDims;
    const int64_t n = static_cast<int64_t>(blocks) * a.Hq * a.B;
    int parts = 1;
    while (n * parts < 2 * kPlanCus && a.P / (2 * parts) >= 32) parts *= 2;
    dim3 grid(blocks * parts, a.Hq, a.B);
    const size_t lds = 2 * static_cast<size_t>(a.d) * sizeof(double) +
                       static_cast<size_t>(kWinChunk) * kBlockDims * sizeof(float);
    hipLaunchKernelGGL(build_proxies_kernel, grid, dim3(kProxyThreads), lds, s, a);
    return hipGetLastError();
}

}  // namespace mmskv
