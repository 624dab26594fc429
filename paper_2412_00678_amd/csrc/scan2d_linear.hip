// The linear layers of a 2DMamba block (Fig. 2: the projections into and out of the block's inner width; the design of
// the original block, Sec. 3.2) on channel-major maps:
//     out[b,o,p] = bias[o] + sum_c Wt[o,c] * in[b,c,p] (+ residual[b,o,p]),   p = position of the map,
// a GEMM with the positions as its wide dimension, on the matrix cores (fp32 accumulation, one rounding after bias and
// residual).
//
// scan2d_linear_kernel: a wavefront owns 64 positions x 16 NOT output channels (scan2d_contract.hpp); no LDS, no barrier.
// The four wavefronts of a workgroup, and the workgroups that follow it on the same XCD, take the other output channels
// of the same positions, so `in` comes from HBM once and from L1 / L2 afterwards.  Bound: HBM for bf16 (the products of
// 128 -> 256 channels are 4.3 GFLOP beside 50 MB), the fp32 matrix rate for fp32.
// scan2d_linear_any_kernel: one thread per output, for maps of fewer than 4 positions or beyond 2^25.
#include "scan2d_block.hpp"

#include <algorithm>

#include "scan2d_contract.hpp"

namespace scan2d {
namespace {

struct LinArgs {
    const void* in; const void* Wt; const float* bias; const void* res; void* out;
    int Cin, Cout, Bt, ogroups;     // ogroups: wavefronts per tile of positions
    long long ptiles, P, waves;     // tiles of 64 positions per batch item, positions per map, wavefronts with work
};

template <typename T, int NOT, int DEPTH>
__global__ __launch_bounds__(256) void scan2d_linear_kernel(const LinArgs p) {
    const long long per = gridDim.x / kXcds;               // the grid is a multiple of 8: workgroups of one XCD follow each other
    const long long wg = (long long)(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    const long long wave = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= p.waves) return;
    const int og = (int)(wave % p.ogroups);
    const long long rest = wave / p.ogroups;
    const int b = (int)(rest / p.ptiles);
    const uint32_t p0 = (uint32_t)(rest % p.ptiles) * 64u, P = (uint32_t)p.P;
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15, o0 = og * 16 * NOT;
    const LanePos pos(p0, n, P);

    f32x4 acc[NOT][4];
#pragma unroll
    for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[ot][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    contract<T, NOT, DEPTH>(static_cast<const T*>(p.in) + (size_t)b * p.Cin * P, P, pos.s, static_cast<const T*>(p.Wt), p.Cin, p.Cout, o0,
                            0, p.Cin, acc);

    const T* res = static_cast<const T*>(p.res);
    T* out = static_cast<T*>(p.out);
#pragma unroll
    for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = o0 + 16 * ot + 4 * g + i;
            if (o >= p.Cout || !pos.any) continue;
            const float bv = p.bias ? p.bias[o] : 0.0f;
            const size_t row = ((size_t)b * p.Cout + o) * P;
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = acc[ot][t][i] + bv;
            if (res) {
                float rv[4];
                load4<T>(res + row + pos.s, rv);
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] += rv[t];
            }
            pos.store(out + row, v);
        }
}

// Any shape: one thread per output, channels in ascending order.
template <typename T>
__global__ __launch_bounds__(256) void scan2d_linear_any_kernel(const LinArgs p) {
    const long long P = p.P;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)p.Bt * p.Cout * P) return;
    const long long pos = idx % P;
    const int o = (int)((idx / P) % p.Cout), b = (int)(idx / (P * p.Cout));
    const T* in = static_cast<const T*>(p.in) + (size_t)b * p.Cin * P + pos;
    const T* w = static_cast<const T*>(p.Wt) + (size_t)o * p.Cin;
    float acc = 0.0f;
    for (int c = 0; c < p.Cin; ++c) acc = fmaf(widen_bits<T>(elem_bits(w + c)), widen_bits<T>(elem_bits(in + (size_t)c * P)), acc);
    if (p.bias) acc += p.bias[o];
    if (p.res) acc += widen_bits<T>(elem_bits(static_cast<const T*>(p.res) + idx));
    store_elem(static_cast<T*>(p.out) + idx, acc);
}

template <typename T, int NOT, int DEPTH>
int launch(LinArgs a, hipStream_t stream) {
    a.ogroups = (a.Cout + 16 * NOT - 1) / (16 * NOT);
    a.waves = a.ptiles * a.Bt * a.ogroups;
    const long long grid = ((a.waves + 3) / 4 + kXcds - 1) / kXcds * kXcds;
    if (grid > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    hipLaunchKernelGGL((scan2d_linear_kernel<T, NOT, DEPTH>), dim3((unsigned)grid), dim3(256), 0, stream, a);
    return SCAN2D_OK;
}

// Output channels per wavefront: 64 (each load of `in` then serves 16 products) where that leaves every SIMD two
// wavefronts, fewer where it does not: a small map is bound by the latency of its few steps, not by the loads.
template <typename T>
int launch_sized(const LinArgs& a, hipStream_t stream) {
    const long long tiles = a.ptiles * a.Bt, o16 = (a.Cout + 15) / 16;
    if (o16 >= 4 && tiles * ((o16 + 3) / 4) >= 2048) return launch<T, 4, 2>(a, stream);
    if (o16 >= 2 && tiles * ((o16 + 1) / 2) >= 2048) return launch<T, 2, 2>(a, stream);
    return launch<T, 1, 4>(a, stream);
}

}  // namespace

int block_linear_launch(const scan2d_desc* d, int Cout, const void* in, const void* Wt, const float* bias, const void* residual,
                        void* out, hipStream_t stream) {
    if (Cout < 1) return SCAN2D_ERR_BAD_SHAPE;
    LinArgs a;
    a.in = in; a.Wt = Wt; a.bias = bias; a.res = residual; a.out = out;
    a.Cin = d->Dc; a.Cout = Cout; a.Bt = d->Bt;
    a.P = (long long)d->H * d->W;
    a.ptiles = (a.P + 63) / 64;
    const bool bf16 = d->dtype == SCAN2D_BF16;
    (void)hipGetLastError();
    int rc = SCAN2D_OK;
    if (contract_fits(a.P, Cout, a.Cin, bf16 ? 2 : 4)) {
        rc = bf16 ? launch_sized<bf16_t>(a, stream) : launch_sized<float>(a, stream);
    } else {
        const long long blocks = ((long long)d->Bt * Cout * a.P + 255) / 256;
        if (blocks > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
        if (bf16) hipLaunchKernelGGL(scan2d_linear_any_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL(scan2d_linear_any_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    }
    if (rc != SCAN2D_OK) return rc;
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace scan2d
