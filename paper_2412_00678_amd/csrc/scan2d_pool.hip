// The aggregator behind the last 2DMamba block (Supp. A "Aggregator": attention pooling with two linear layers):
//     s_k = sum_d w[d] * tanh(sum_m V[d,m] * h[m,k]),   a_k = softmax of s over the bag,   z = sum_k a_k h_k.
// Three kernels, no workspace (attn holds the scores in between):
//   scan2d_pool_scores_kernel  : the scores.  V . h is a dense contraction (D x M x positions), so it runs on the matrix
//                                cores (scan2d_contract.hpp); tanh, the product with w and the sum over the D hidden
//                                units are its epilogue.  scan2d_pool_scores_any_kernel: maps of fewer than 4
//                                positions or 4 GB of weights.
//   scan2d_pool_softmax_kernel : per batch item, max and sum of exp over the bag in a fixed order, then the weights.
//   scan2d_pool_sum_kernel     : z[b][m], one workgroup per channel, fixed order.
#include "scan2d_block.hpp"

#include <algorithm>

#include "scan2d_contract.hpp"

namespace scan2d {
namespace {

constexpr int kPoolRows = 128;       // most hidden units

struct PoolArgs {
    const void* h; const void* V; const float* w; const uint8_t* mask;
    float* attn; float* z;
    int M, D, Bt, tiles;             // channels, hidden units, batch items, tiles of 64 positions per batch item
    long long P;                     // positions per map
};

__device__ __forceinline__ float fast_tanh(float v) {          // 1 - 2 / (1 + e^(2v)); saturates to +-1, keeps NaN
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(v * (2.0f * kLog2e)));
}

// A workgroup of four wavefronts per tile of 64 positions; wavefront v takes hidden units 32 v .. 32 v + 31, the parts of
// a score meet in LDS and are added in wavefront order.
template <typename T, bool TAIL, bool WIDE = false>
__global__ __launch_bounds__(256) void scan2d_pool_scores_kernel(const PoolArgs p) {
    __shared__ float part[4][64];
    const int tid = threadIdx.x, l = tid & 63, g = l >> 4, n = l & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), d0 = 32 * wv;
    const int b = blockIdx.x / p.tiles;
    const uint32_t p0 = (uint32_t)(blockIdx.x % p.tiles) * 64u, P = (uint32_t)p.P;
    const LanePos pos(p0, n, P);
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (d0 < p.D) {
        f32x4 acc[2][4];
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[ot][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        contract<T, 2, 2, TAIL, WIDE>(static_cast<const T*>(p.h) + (size_t)b * p.M * P, P, pos.s, static_cast<const T*>(p.V), p.M, p.D, d0, 0, p.M, acc);
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int d = d0 + 16 * ot + 4 * g + i;
                const float wd = p.w[min(d, p.D - 1)];
#pragma unroll
                for (int t = 0; t < 4; ++t) s[t] = d < p.D ? fmaf(wd, fast_tanh(acc[ot][t][i]), s[t]) : s[t];
            }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        s[t] += __shfl_xor(s[t], 16);
        s[t] += __shfl_xor(s[t], 32);
    }
    if (g == 0) *reinterpret_cast<float4*>(&part[wv][4 * n]) = make_float4(s[0], s[1], s[2], s[3]);
    __syncthreads();
    if (tid < 16) {
        float4 v = *reinterpret_cast<const float4*>(&part[0][4 * n]);
#pragma unroll
        for (int q = 1; q < 4; ++q) {
            const float4 a = *reinterpret_cast<const float4*>(&part[q][4 * n]);
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        }
        const float o[4] = {v.x, v.y, v.z, v.w};
        pos.store(p.attn + (size_t)b * P, o);
    }
}

// Any map: one wavefront per position, lane d and d + 64.
template <typename T>
__global__ __launch_bounds__(64) void scan2d_pool_scores_any_kernel(const PoolArgs p) {
    const long long b = blockIdx.x / p.P, pos = blockIdx.x % p.P;
    const T* h = static_cast<const T*>(p.h) + (size_t)b * p.M * p.P + pos;
    float s = 0.0f;
    for (int d = threadIdx.x; d < p.D; d += 64) {
        const T* v = static_cast<const T*>(p.V) + (size_t)d * p.M;
        float acc = 0.0f;
        for (int m = 0; m < p.M; ++m) acc = fmaf(widen_bits<T>(elem_bits(v + m)), widen_bits<T>(elem_bits(h + (size_t)m * p.P)), acc);
        s = fmaf(p.w[d], fast_tanh(acc), s);
    }
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) s += __shfl_xor(s, step);
    if (threadIdx.x == 0) p.attn[(size_t)b * p.P + pos] = s;
}

constexpr int kSoftThreads = 1024;
// Sum or maximum over the workgroup in a fixed order; every thread gets the result.
template <bool MAX>
__device__ __forceinline__ float block_reduce(float v, float* red) {
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const float o = __shfl_xor(v, step);
        v = MAX ? fmaxf(v, o) : v + o;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int w = 1; w < kSoftThreads / 64; ++w) r = MAX ? fmaxf(r, red[w]) : r + red[w];
    __syncthreads();
    return r;
}

// One workgroup per batch item, in place: scores -> attention weights.  Positions under the mask are not members of
// the bag: they are skipped by the maximum and the sum and get weight 0; an empty bag gets all zeros.
// Maps of 4 to 16384 NV / 4 positions: a thread keeps its NV groups of 4 positions in registers (scores outside the bag
// as -infinity), so the scores are read once and written once, all loads in flight together.  The one compute unit of a
// batch item moves 8 bytes per position: 65536 positions took 14 us in three passes.
template <int NV>
__global__ __launch_bounds__(kSoftThreads) void scan2d_pool_softmax_kernel(const PoolArgs p) {
    __shared__ float red[kSoftThreads / 64];
    const int b = blockIdx.x, tid = threadIdx.x;
    const uint32_t P = (uint32_t)p.P;
    float* a = p.attn + (size_t)b * P;
    const uint8_t* mk = p.mask ? p.mask + (size_t)b * P : nullptr;
    float sv[NV][4];
    float mx = -INFINITY;
    bool members = false;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t q = 4u * (uint32_t)(tid + k * kSoftThreads), s = min(q, P - 4u);
        load4<float>(a + s, sv[k]);
        uint32_t m = 0u;
        if (mk) load_words_any<1>(mk + s, &m);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool member = s + e >= q && ((m >> (8 * e)) & 0xffu) == 0u;         // else not this thread's, or not in the bag
            if (!member) sv[k][e] = -INFINITY;
            members |= member;
        }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sv[k][e]);
    mx = block_reduce<true>(mx, red);
    float sum = members && mx == -INFINITY ? NAN : 0.0f;  // every score of the bag is -infinity: no weights exist
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = sv[k][e];
            sv[k][e] = x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((x - mx) * kLog2e);
            sum += sv[k][e];
        }
    sum = block_reduce<false>(sum, red);
    const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;     // a NaN score makes the sum NaN: the weights then are NaN too
    const bool bad = sum != sum;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t q = 4u * (uint32_t)(tid + k * kSoftThreads);
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = sv[k][e] * inv;
        if (bad) {                                        // members only; the mask again
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (q + e < P && mk && mk[q + e] != 0) ? 0.0f : sum;
        }
        if (q + 4u <= P) store4<float>(a + q, o);
        else if (q < P) {
            const uint32_t s = P - 4u;
#pragma unroll
            for (int e = 1; e < 4; ++e)
                if (s + e >= q) a[s + e] = bad ? ((mk && mk[s + e] != 0) ? 0.0f : sum) : o[e];
        }
    }
}

// The same for any map, in three passes: every thread walks its positions four loads deep (VEC: four aligned groups of 4
// positions), in an order fixed by the shape.
template <bool VEC>
__global__ __launch_bounds__(kSoftThreads) void scan2d_pool_softmax_any_kernel(const PoolArgs p) {
    __shared__ float red[kSoftThreads / 64];
    constexpr int E = VEC ? 4 : 1;                        // positions per load
    const int b = blockIdx.x, tid = threadIdx.x;
    const long long P = p.P, PV = P / E;
    float* a = p.attn + (size_t)b * P;
    const uint8_t* mk = p.mask ? p.mask + (size_t)b * P : nullptr;
    // pass(f): f(position, score, member) over this thread's positions
    auto walk = [&](auto f) {
        for (long long base = 0; base < PV; base += 4 * kSoftThreads) {
            float sv[4][E];
            uint32_t mv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long idx = min(base + u * kSoftThreads + tid, PV - 1);
                if constexpr (VEC) {
                    const float4 t = *reinterpret_cast<const float4*>(a + 4 * idx);
                    sv[u][0] = t.x; sv[u][1] = t.y; sv[u][2] = t.z; sv[u][3] = t.w;
                    mv[u] = mk ? *reinterpret_cast<const uint32_t*>(mk + 4 * idx) : 0u;
                } else {
                    sv[u][0] = a[idx];
                    mv[u] = mk ? (uint32_t)mk[idx] : 0u;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long idx = base + u * kSoftThreads + tid;
                if (idx < PV) {
#pragma unroll
                    for (int e = 0; e < E; ++e) f(E * idx + e, sv[u][e], ((mv[u] >> (8 * e)) & 0xffu) == 0u);
                }
            }
        }
    };
    float mx = -INFINITY;
    walk([&](long long, float s, bool member) { mx = member ? fmaxf(mx, s) : mx; });
    mx = block_reduce<true>(mx, red);
    float sum = 0.0f;
    walk([&](long long, float s, bool member) { sum += member ? __builtin_amdgcn_exp2f((s - mx) * kLog2e) : 0.0f; });
    sum = block_reduce<false>(sum, red);
    const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;     // a NaN score makes the sum NaN: the weights then are NaN too
    const bool bad = sum != sum;
    walk([&](long long k, float s, bool member) {
        const float e = __builtin_amdgcn_exp2f((s - mx) * kLog2e);
        a[k] = member ? (bad ? sum : e * inv) : 0.0f;
    });
}

// z[b][m] = sum over the bag of a_k * h[m][k]: grid (M, Bt), fixed order (strided partial sums of groups of 4 positions,
// any alignment, four loads deep, then over the workgroup).  Maps of fewer than 4 positions: one position per thread.
template <typename T>
__global__ __launch_bounds__(kSoftThreads) void scan2d_pool_sum_kernel(const PoolArgs p) {
    __shared__ float red[kSoftThreads / 64];
    const int m = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const long long P = p.P;
    const T* hr = static_cast<const T*>(p.h) + ((size_t)b * p.M + m) * P;
    const float* a = p.attn + (size_t)b * P;
    float acc = 0.0f;
    if (P >= 4) {
        for (long long base = 0; base < P; base += 16 * kSoftThreads) {
            float av[4][4], hv[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long s = min(base + 4 * (u * kSoftThreads + tid), P - 4);
                load4<float>(a + s, av[u]);
                load4<T>(hr + s, hv[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long q = base + 4 * (u * kSoftThreads + tid), s = min(q, P - 4);
#pragma unroll
                for (int e = 0; e < 4; ++e)                // weight 0: outside the bag, never read into the sum
                    acc += (s + e >= q && av[u][e] != 0.0f) ? av[u][e] * hv[u][e] : 0.0f;
            }
        }
    } else if (tid < P) {
        acc = a[tid] != 0.0f ? a[tid] * widen_bits<T>(elem_bits(hr + tid)) : 0.0f;
    }
    acc = block_reduce<false>(acc, red);
    if (tid == 0) p.z[(size_t)b * p.M + m] = acc;
}

int launch_pool(const scan2d_desc* d, int D, const void* h, const void* V, const float* w, const uint8_t* mask, float* attn, float* z, hipStream_t stream) {
    PoolArgs a;
    a.h = h; a.V = V; a.w = w; a.mask = mask; a.attn = attn; a.z = z;
    a.M = d->Dc; a.D = D; a.Bt = d->Bt;
    a.P = (long long)d->H * d->W;
    const long long tiles = (a.P + 63) / 64;
    const bool bf16 = d->dtype == SCAN2D_BF16, fits = contract_fits(a.P, D, a.M, bf16 ? 2 : 4);
    if (!launch_fits((fits ? tiles : a.P) * d->Bt, fits ? 256 : 64)) return SCAN2D_ERR_BAD_SHAPE;
    a.tiles = (int)tiles;
    (void)hipGetLastError();
    const dim3 g1((unsigned)((fits ? tiles : a.P) * d->Bt)), g2((unsigned)d->Bt), g3((unsigned)d->Dc, (unsigned)d->Bt);
    using Kernel = void (*)(const PoolArgs);
    Kernel scores, soft;
    if (fits && !contract_narrow(a.P, bf16 ? 2 : 4)) scores = bf16 ? scan2d_pool_scores_kernel<bf16_t, true, true> : scan2d_pool_scores_kernel<float, true, true>;
    else if (fits && bf16) scores = a.M % 32 == 0 ? scan2d_pool_scores_kernel<bf16_t, false> : scan2d_pool_scores_kernel<bf16_t, true>;
    else if (fits) scores = a.M % 16 == 0 ? scan2d_pool_scores_kernel<float, false> : scan2d_pool_scores_kernel<float, true>;
    else scores = bf16 ? scan2d_pool_scores_any_kernel<bf16_t> : scan2d_pool_scores_any_kernel<float>;
    if (a.P < 4) soft = scan2d_pool_softmax_any_kernel<false>;
    else if (a.P <= 4 * kSoftThreads) soft = scan2d_pool_softmax_kernel<1>;
    else if (a.P <= 16 * kSoftThreads) soft = scan2d_pool_softmax_kernel<4>;
    else if (a.P <= 64 * kSoftThreads) soft = scan2d_pool_softmax_kernel<16>;
    else soft = a.P % 4 == 0 ? scan2d_pool_softmax_any_kernel<true> : scan2d_pool_softmax_any_kernel<false>;
    hipLaunchKernelGGL(scores, g1, dim3(fits ? 256 : 64), 0, stream, a);
    hipLaunchKernelGGL(soft, g2, dim3(kSoftThreads), 0, stream, a);
    if (bf16) hipLaunchKernelGGL(scan2d_pool_sum_kernel<bf16_t>, g3, dim3(kSoftThreads), 0, stream, a);
    else hipLaunchKernelGGL(scan2d_pool_sum_kernel<float>, g3, dim3(kSoftThreads), 0, stream, a);
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace

int block_attn_pool_launch(const scan2d_desc* d, int D, const void* h, const void* V, const float* w, const uint8_t* mask,
                           float* attn, float* z, hipStream_t stream) {
    if (D < 1 || D > kPoolRows || d->Bt > 65535) return SCAN2D_ERR_BAD_SHAPE;
    const size_t P = (size_t)d->H * d->W, each = P * d->Dc * (d->dtype == SCAN2D_BF16 ? 2 : 4);
    return by_items(*d, [&](const scan2d_desc& q, size_t b) {
        return launch_pool(&q, D, item_at(h, b, each), V, w, item_at(mask, b, P), item_at(attn, b, 4 * P), item_at(z, b, 4 * (size_t)d->Dc), stream);
    });
}

}  // namespace scan2d
