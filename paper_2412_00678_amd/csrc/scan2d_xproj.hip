// The projections in front of the scan (2DMamba Eq. 3: step, B and C are linear functions of x):
//     low = Wx . x per position,  Bm / Cm = rows R.. of low,  delta_raw = Wdt . low[:R]
// written in the storage type the scan kernels read; low is not rounded before the second product.
//
// scan2d_xproj_kernel: a workgroup of four wavefronts owns 64 positions.
//   1. The wavefronts split the channels of x and each contracts its part for all rows of Wx (scan2d_contract.hpp: x goes
//      straight from global memory into the MFMA operands), so x is read once and a map of few tiles still has four
//      wavefronts per tile to cover the latency of the contraction.
//   2. The four partial sums of a row meet in LDS and are added in wavefront order.  Rows R.. are rounded and leave as
//      Bm / Cm, rows 0..R-1 stay in LDS as fp32.  Wx beyond 48 rows: in groups of 48.
//   3. delta_raw on v_mfma_f32_16x16x4_f32: rows are 16 channels, columns the same position groups, the contraction
//      index r = KR g + s for lane group g and MFMA s; the wavefronts take every fourth block of 16 channels.
// Bound: HBM (read x, write delta_raw).
// scan2d_xproj_any_kernel: one workgroup per position, for maps of fewer than 4 positions or beyond 2^25.
#include "scan2d_block.hpp"

#include "scan2d_contract.hpp"

namespace scan2d {
namespace {

struct XprojArgs {
    const void* x; const void* Wx; const float* Wdt;
    void* delta_raw; void* Bm; void* Cm;
    int Dc, N, R, tiles;         // tiles of 64 positions per batch item
    long long P;                 // positions per map
};

constexpr int kRowBlocks = 3;    // MFMA row blocks of Wx per pass

// KR: low-rank rows per lane group, 4 KR >= R
template <typename T, int KR, bool TAIL>
__global__ __launch_bounds__(256, 2) void scan2d_xproj_kernel(const XprojArgs p) {
    __shared__ float part[4][kRowBlocks * 16][64];
    __shared__ float low[4 * KR][64];
    const int tid = threadIdx.x, l = tid & 63, g = l >> 4, n = l & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Dc = p.Dc, N = p.N, R = p.R, M = R + 2 * N;
    const int b = blockIdx.x / p.tiles;
    const uint32_t p0 = (uint32_t)(blockIdx.x % p.tiles) * 64u, P = (uint32_t)p.P;
    const T* x = static_cast<const T*>(p.x) + (size_t)b * Dc * P;
    const LanePos pos(p0, n, P);

    auto weights = [&](int c0, float* a) {                 // row c0 + n of Wdt, columns KR g ..
        const float* row = p.Wdt + (size_t)min(c0 + n, Dc - 1) * R;
#pragma unroll
        for (int s = 0; s < KR; ++s) {
            const float v = row[min(KR * g + s, R - 1)];
            a[s] = KR * g + s < R ? v : 0.0f;
        }
    };
    float a[KR];
    weights(16 * wv, a);                                   // requested in front of everything else

    constexpr int KS = contract_step<T>();
    const int span = ((Dc + KS - 1) / KS + 3) / 4 * KS;    // channels of a wavefront: whole steps
    const int cbeg = min(wv * span, Dc), cend = min(cbeg + span, Dc);
    for (int m0 = 0; m0 < M; m0 += kRowBlocks * 16) {
        f32x4 acc[kRowBlocks][4];
#pragma unroll
        for (int mb = 0; mb < kRowBlocks; ++mb)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[mb][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        contract<T, kRowBlocks, 2, TAIL>(x, P, pos.s, static_cast<const T*>(p.Wx), Dc, M, m0, cbeg, cend, acc);
        if (m0 > 0) __syncthreads();                       // the sums of the previous rows have been read
#pragma unroll
        for (int mb = 0; mb < kRowBlocks; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<float4*>(&part[wv][16 * mb + 4 * g + i][4 * n]) = make_float4(acc[mb][0][i], acc[mb][1][i], acc[mb][2][i], acc[mb][3][i]);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kRowBlocks; ++it) {          // 16 rows x 16 groups of 4 positions
            const int row = 16 * it + (tid >> 4), m = m0 + row;
            float4 v = *reinterpret_cast<const float4*>(&part[0][row][4 * n]);
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const float4 t = *reinterpret_cast<const float4*>(&part[w][row][4 * n]);
                v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
            }
            if (m < R) *reinterpret_cast<float4*>(&low[m][4 * n]) = v;
            else if (m < M) {
                const float o[4] = {v.x, v.y, v.z, v.w};
                const int k = m - R;
                T* dst = static_cast<T*>(k < N ? p.Bm : p.Cm) + ((size_t)b * N + (k < N ? k : k - N)) * P;
                pos.store(dst, o);
            }
        }
    }
    __syncthreads();

    float bl[KR][4];                                       // low[KR g + s] of this lane's positions
#pragma unroll
    for (int s = 0; s < KR; ++s) {
        const int r = KR * g + s;
        const float4 v = *reinterpret_cast<const float4*>(&low[r][4 * n]);
        bl[s][0] = r < R ? v.x : 0.0f; bl[s][1] = r < R ? v.y : 0.0f; bl[s][2] = r < R ? v.z : 0.0f; bl[s][3] = r < R ? v.w : 0.0f;
    }
    for (int c0 = 16 * wv; c0 < Dc; c0 += 64) {
        float next[KR];
        weights(c0 + 64, next);
        f32x4 d[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < KR; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) d[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], bl[s][t], d[t], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + 4 * g + i;
            const float o[4] = {d[0][i], d[1][i], d[2][i], d[3][i]};
            if (c < Dc) pos.store(static_cast<T*>(p.delta_raw) + ((size_t)b * Dc + c) * P, o);
        }
#pragma unroll
        for (int s = 0; s < KR; ++s) a[s] = next[s];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void scan2d_xproj_any_kernel(const XprojArgs p) {
    __shared__ float low[64];
    const int tid = threadIdx.x, Dc = p.Dc, N = p.N, R = p.R;
    const long long b = blockIdx.x / p.P, pos = blockIdx.x % p.P;
    const T* x = static_cast<const T*>(p.x) + (size_t)b * Dc * p.P + pos;
    if (tid < R + 2 * N) {                                 // at most 64 + 2 * 64 rows
        const T* w = static_cast<const T*>(p.Wx) + (size_t)tid * Dc;
        float acc = 0.0f;
        for (int c = 0; c < Dc; ++c) acc = fmaf(widen_bits<T>(elem_bits(w + c)), widen_bits<T>(elem_bits(x + (size_t)c * p.P)), acc);
        if (tid < R) low[tid] = acc;
        else {
            const int k = tid - R;
            store_elem(static_cast<T*>(k < N ? p.Bm : p.Cm) + ((size_t)b * N + (k < N ? k : k - N)) * p.P + pos, acc);
        }
    }
    __syncthreads();
    for (int c = tid; c < Dc; c += 256) {
        float acc = 0.0f;
        for (int r = 0; r < R; ++r) acc = fmaf(p.Wdt[(size_t)c * R + r], low[r], acc);
        store_elem(static_cast<T*>(p.delta_raw) + ((size_t)b * Dc + c) * p.P + pos, acc);
    }
}

template <typename T, bool TAIL>
void launch(const XprojArgs& a, int Bt, hipStream_t stream) {
    const dim3 grid((unsigned)(a.tiles * Bt));
    if (a.R <= 8) hipLaunchKernelGGL((scan2d_xproj_kernel<T, 2, TAIL>), grid, dim3(256), 0, stream, a);
    else if (a.R <= 16) hipLaunchKernelGGL((scan2d_xproj_kernel<T, 4, TAIL>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((scan2d_xproj_kernel<T, 16, TAIL>), grid, dim3(256), 0, stream, a);
}
template <typename T>
void launch(const XprojArgs& a, int Bt, hipStream_t stream) {
    if (a.Dc % contract_step<T>() == 0) launch<T, false>(a, Bt, stream);
    else launch<T, true>(a, Bt, stream);
}

}  // namespace

int block_xproj_launch(const scan2d_desc* d, int R, const void* x, const void* Wx, const float* Wdt, void* delta_raw, void* Bm,
                       void* Cm, hipStream_t stream) {
    if (R < 1 || R > 64) return SCAN2D_ERR_BAD_SHAPE;
    const bool bf16 = d->dtype == SCAN2D_BF16;
    XprojArgs a;
    a.x = x; a.Wx = Wx; a.Wdt = Wdt; a.delta_raw = delta_raw; a.Bm = Bm; a.Cm = Cm;
    a.Dc = d->Dc; a.N = d->N; a.R = R;
    a.P = (long long)d->H * d->W;
    const long long tiles = (a.P + 63) / 64;
    const bool fits = contract_fits(a.P, R + 2 * d->N, d->Dc, bf16 ? 2 : 4);
    if ((fits ? tiles : a.P) * d->Bt > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    a.tiles = (int)tiles;
    (void)hipGetLastError();
    if (fits) {
        if (bf16) launch<bf16_t>(a, d->Bt, stream);
        else launch<float>(a, d->Bt, stream);
    } else {
        const dim3 grid((unsigned)(a.P * d->Bt));
        if (bf16) hipLaunchKernelGGL(scan2d_xproj_any_kernel<bf16_t>, grid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL(scan2d_xproj_any_kernel<float>, grid, dim3(256), 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace scan2d
