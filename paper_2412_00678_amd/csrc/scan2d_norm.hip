// The normalisation in front of a 2DMamba block (Sec. 3.3 lists "normalization, projection, and convolution" in front of
// the scan) on channel-major maps, over the channels of each position:
//     layer norm: out = (x - mean_c x) / sqrt(var_c x + eps) * gamma[c] + beta[c]      (biased variance)
//     RMS norm:   out = x / sqrt(mean_c x^2 + eps) * gamma[c] (+ beta[c])
// Bound: HBM (one read, one write per element).  The mean is taken first and the variance as the mean of squared
// deviations (no cancellation).
// scan2d_norm_kernel, up to 512 channels: a workgroup owns 64 positions, E consecutive ones per thread, and its PARTS rows of
// threads take every PARTS-th channel (any alignment, any H*W of at least 4).  A thread keeps its C / PARTS channels x E
// positions in registers as they were loaded, all loads in flight at once, so the tensor is read once; the sums over the
// parts meet in LDS and are added in the order of the parts.  Eight parts of two positions in bf16 (the order of sums of
// the other kernel, so both round alike), sixteen of four in fp32 (registers).
// scan2d_norm_any_kernel, any shape: 32 groups of E consecutive positions per workgroup, the channels split eight ways,
// three passes over the tile (the second and third from L2).
#include "scan2d_block.hpp"

#include "scan2d_contract.hpp"

namespace scan2d {
namespace {

struct NormArgs {
    const void* in; const float* gamma; const float* beta; void* out;
    int C, Bt, rms;
    float eps;
    long long P, groups;            // positions per map, groups of E positions per map
};

// E: consecutive positions of a thread, PARTS: threads that share a position's channels, CPT: channels per thread (PARTS CPT >= C)
template <typename T, int E, int PARTS, int CPT>
__global__ __launch_bounds__(64 / E * PARTS) void scan2d_norm_kernel(const NormArgs p) {
    constexpr int XW = words_of<T, E>(), LANES = 64 / E, TH = LANES * PARTS;
    __shared__ float red[2][PARTS][64];
    __shared__ float gb[2][PARTS * CPT];
    const int tid = threadIdx.x, n = tid % LANES, part = tid / LANES;
    const uint32_t P = (uint32_t)p.P, tiles = (P + 63u) / 64u;
    const int b = (int)(blockIdx.x / tiles), C = p.C;
    const LanePos<E> pos((blockIdx.x % tiles) * 64u, n, P);
    const T* src = static_cast<const T*>(p.in) + (size_t)b * C * P + pos.s;
    uint32_t raw[CPT][XW];
#pragma unroll
    for (int k = 0; k < CPT; ++k) load_words_any<XW>(src + (size_t)min(part + PARTS * k, C - 1) * P, raw[k]);
    for (int c = tid; c < PARTS * CPT; c += TH) {          // behind the first barrier
        gb[0][c] = p.gamma[min(c, C - 1)];
        gb[1][c] = p.beta ? p.beta[min(c, C - 1)] : 0.0f;
    }
    const float invC = 1.0f / (float)C;
    auto total = [&](int buf, float* v) {                 // sum over the parts in their order, every thread gets it
#pragma unroll
        for (int t = 0; t < E; ++t) red[buf][part][E * n + t] = v[t];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < E; ++t) v[t] = red[buf][0][E * n + t];
#pragma unroll
        for (int w = 1; w < PARTS; ++w)
#pragma unroll
            for (int t = 0; t < E; ++t) v[t] += red[buf][w][E * n + t];
    };
    float mean[E], v[E], rstd[E];
#pragma unroll
    for (int t = 0; t < E; ++t) mean[t] = v[t] = 0.0f;
    if (!p.rms) {
#pragma unroll
        for (int k = 0; k < CPT; ++k)
            if (part + PARTS * k < C) {
#pragma unroll
                for (int t = 0; t < E; ++t) mean[t] += get_elem<T, E>(raw[k], t);
            }
        total(0, mean);
#pragma unroll
        for (int t = 0; t < E; ++t) mean[t] *= invC;
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k)
        if (part + PARTS * k < C) {
#pragma unroll
            for (int t = 0; t < E; ++t) {
                const float e = get_elem<T, E>(raw[k], t) - mean[t];
                v[t] = fmaf(e, e, v[t]);
            }
        }
    total(1, v);
#pragma unroll
    for (int t = 0; t < E; ++t) rstd[t] = 1.0f / sqrtf(v[t] * invC + p.eps);
    T* dst = static_cast<T*>(p.out) + (size_t)b * C * P;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = part + PARTS * k;
        if (c < C) {
            const float gm = gb[0][c], bt = gb[1][c];
            float o[E];
#pragma unroll
            for (int t = 0; t < E; ++t) o[t] = fmaf((get_elem<T, E>(raw[k], t) - mean[t]) * rstd[t], gm, bt);
            pos.store(dst + (size_t)c * P, o);
        }
    }
}

constexpr int kNormGroups = 32, kNormSplit = 8, kNormDeep = 8;   // position groups and channel parts per workgroup, loads in flight
static_assert(kNormGroups * kNormSplit == 256, "one thread per (position group, channel part)");
template <typename T, int E>
__global__ __launch_bounds__(256) void scan2d_norm_any_kernel(const NormArgs p) {
    constexpr int EB = Elem<T>::kBytes;
    __shared__ float red[kNormSplit][kNormGroups][E];
    const int tid = threadIdx.x, q = tid % kNormGroups, cq = tid / kNormGroups;
    const long long per_item = (p.groups + kNormGroups - 1) / kNormGroups; // workgroups per batch item
    const int b = (int)(blockIdx.x / per_item);
    const long long grp = (blockIdx.x % per_item) * kNormGroups + q;
    const bool live = grp < p.groups;
    const long long pos = min(grp, p.groups - 1) * E;
    const int C = p.C;
    const T* src = static_cast<const T*>(p.in) + (size_t)b * C * p.P + pos;
    T* dst = static_cast<T*>(p.out) + (size_t)b * C * p.P + pos;

    auto load = [&](int c, float* v) {
        const T* a = src + (size_t)c * p.P;
        if constexpr (E == 4 && EB == 2) {
            const uint2 r = *reinterpret_cast<const uint2*>(a);
            v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xffff0000u);
            v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xffff0000u);
        } else if constexpr (E == 4) {
            const float4 r = *reinterpret_cast<const float4*>(a);
            v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
        } else {
            const uint32_t bits = elem_bits(a);
            v[0] = EB == 4 ? __uint_as_float(bits) : __uint_as_float(bits << 16);
        }
    };
    // sum over all channels of f(x) per position: this thread's channels kNormDeep loads deep, then the partial sums
    auto channel_sum = [&](auto f, float* total) {
        float acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.0f;
        for (int c0 = cq; c0 < C; c0 += kNormSplit * kNormDeep) {
            float v[kNormDeep][E];
#pragma unroll
            for (int u = 0; u < kNormDeep; ++u) load(min(c0 + kNormSplit * u, C - 1), v[u]);
#pragma unroll
            for (int u = 0; u < kNormDeep; ++u)
                if (c0 + kNormSplit * u < C) {
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[e] += f(v[u][e], e);
                }
        }
        __syncthreads();                                   // the previous sums have been read
#pragma unroll
        for (int e = 0; e < E; ++e) red[cq][q][e] = acc[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float t2 = 0.0f;
#pragma unroll
            for (int s = 0; s < kNormSplit; ++s) t2 += red[s][q][e];
            total[e] = t2;
        }
    };

    float mean[E], rstd[E], t[E];
#pragma unroll
    for (int e = 0; e < E; ++e) mean[e] = 0.0f;
    const float invC = 1.0f / (float)C;
    if (!p.rms) {
        channel_sum([](float x, int) { return x; }, t);
#pragma unroll
        for (int e = 0; e < E; ++e) mean[e] = t[e] * invC;
    }
    channel_sum([&](float x, int e) { const float d = x - mean[e]; return d * d; }, t);
#pragma unroll
    for (int e = 0; e < E; ++e) rstd[e] = 1.0f / sqrtf(t[e] * invC + p.eps);

    for (int c0 = cq; c0 < C; c0 += kNormSplit * kNormDeep) {
        float v[kNormDeep][E];
#pragma unroll
        for (int u = 0; u < kNormDeep; ++u) load(min(c0 + kNormSplit * u, C - 1), v[u]);
#pragma unroll
        for (int u = 0; u < kNormDeep; ++u) {
            const int c = c0 + kNormSplit * u;
            if (c < C && live) {
                const float gm = p.gamma[c], bt = p.beta ? p.beta[c] : 0.0f;
                float o[E];
#pragma unroll
                for (int e = 0; e < E; ++e) o[e] = fmaf((v[u][e] - mean[e]) * rstd[e], gm, bt);
                T* d = dst + (size_t)c * p.P;
                if constexpr (E == 4 && EB == 2) {
                    uint2 r;
                    r.x = pack_bf16x2(o[0], o[1]); r.y = pack_bf16x2(o[2], o[3]);
                    *reinterpret_cast<uint2*>(d) = r;
                } else if constexpr (E == 4) {
                    *reinterpret_cast<float4*>(d) = make_float4(o[0], o[1], o[2], o[3]);
                } else {
                    store_elem(d, o[0]);
                }
            }
        }
    }
}

int launch_norm(const scan2d_desc* d, int kind, float eps, const void* in, const float* gamma, const float* beta, void* out, hipStream_t stream) {
    if ((kind != 0 && kind != 1) || !(eps >= 0.0f)) return SCAN2D_ERR_BAD_SHAPE;
    NormArgs a;
    a.in = in; a.gamma = gamma; a.beta = beta; a.out = out;
    a.C = d->Dc; a.Bt = d->Bt; a.rms = kind; a.eps = eps;
    a.P = (long long)d->H * d->W;
    const bool bf16 = d->dtype == SCAN2D_BF16;
    (void)hipGetLastError();
    if (a.P >= 4 && a.P < (1LL << 31) && a.C <= 512) {
        const long long blocks = (a.P + 63) / 64 * d->Bt;
        if (!launch_fits(blocks, 256)) return SCAN2D_ERR_BAD_SHAPE;
        using Kernel = void (*)(const NormArgs);
        Kernel k;
        if (a.C <= 64) k = bf16 ? scan2d_norm_kernel<bf16_t, 2, 8, 8> : scan2d_norm_kernel<float, 4, 16, 4>;
        else if (a.C <= 128) k = bf16 ? scan2d_norm_kernel<bf16_t, 2, 8, 16> : scan2d_norm_kernel<float, 4, 16, 8>;
        else if (a.C <= 256) k = bf16 ? scan2d_norm_kernel<bf16_t, 2, 8, 32> : scan2d_norm_kernel<float, 4, 16, 16>;
        else k = bf16 ? scan2d_norm_kernel<bf16_t, 2, 8, 64> : scan2d_norm_kernel<float, 4, 16, 32>;
        hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, stream, a);
        return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
    }
    const bool vec = a.P % 4 == 0;
    a.groups = vec ? a.P / 4 : a.P;
    const long long blocks = (a.groups + kNormGroups - 1) / kNormGroups * d->Bt;
    if (!launch_fits(blocks, 256)) return SCAN2D_ERR_BAD_SHAPE;
    if (bf16) {
        if (vec) hipLaunchKernelGGL((scan2d_norm_any_kernel<bf16_t, 4>), dim3((unsigned)blocks), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((scan2d_norm_any_kernel<bf16_t, 1>), dim3((unsigned)blocks), dim3(256), 0, stream, a);
    } else {
        if (vec) hipLaunchKernelGGL((scan2d_norm_any_kernel<float, 4>), dim3((unsigned)blocks), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((scan2d_norm_any_kernel<float, 1>), dim3((unsigned)blocks), dim3(256), 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace

int block_norm_launch(const scan2d_desc* d, int kind, float eps, const void* in, const float* gamma, const float* beta, void* out,
                      hipStream_t stream) {
    const size_t each = (size_t)d->Dc * d->H * d->W * (d->dtype == SCAN2D_BF16 ? 2 : 4);
    return by_items(*d, [&](const scan2d_desc& q, size_t b) { return launch_norm(&q, kind, eps, item_at(in, b, each), gamma, beta, item_at(out, b, each), stream); });
}

}  // namespace scan2d
