// The projections in front of the scan (2DMamba Eq. 3: step, B and C are linear functions of x):
//     low = Wx . x per position,  Bm / Cm = rows R.. of low,  delta_raw = Wdt . low[:R]
// written in the storage type the scan kernels read; low is not rounded before the second product.
//
// scan2d_xproj_kernel: a workgroup of four wavefronts owns 64 positions.
//   1. The contraction over the channels (x goes straight from global memory into the MFMA operands).  fp32: the wavefronts
//      split the channels, each contracts its part for all rows of Wx (scan2d_contract.hpp) and the four partial sums meet
//      in LDS in wavefront order.  bf16: the wavefronts split the rows of Wx, each contracts all channels for 16 of them,
//      in one chain of v_mfma_f32_16x16x16_bf16: rounded to bf16, a sum in another order would come out one unit apart now
//      and then, and the scan, the layers behind it and a peaked softmax enlarge that.
//   2. Rows R.. are rounded and leave as Bm / Cm, rows 0..R-1 stay in LDS as fp32.  Wx beyond 48 rows: in groups of 48.
//   3. delta_raw on v_mfma_f32_16x16x4_f32: rows are 16 channels, columns the same position groups, the contraction
//      index r = 4 s + g for lane group g and MFMA s; the wavefronts take every fourth block of 16 channels.
// scan2d_xproj_wave_kernel, bf16 from kWaveTiles tiles on: each wavefront does all of this for 64 positions of its own.
// Bound: HBM (read x, write delta_raw).  256 channels, R = 8, N = 16, bf16: 256x256 22.5 us (3.2 TB/s; split rows 28.4),
// 181x181 15.7 us (a wavefront each: 22.9), 57x83 10.9 us; 512 channels, R = 16, fp32: 128x200 37.0 us.
// scan2d_xproj_any_kernel: one workgroup per position, for maps of fewer than 4 positions or 4 GB of weights.
#include "scan2d_block.hpp"

#include "scan2d_contract.hpp"

namespace scan2d {
namespace {

struct XprojArgs {
    const void* x; const void* Wx; const float* Wdt;
    void* delta_raw; void* Bm; void* Cm;
    int Dc, N, R, tiles, Bt;         // tiles of 64 positions per batch item
    long long P;                 // positions per map
};

// Tiles of 64 positions from which every SIMD has a wavefront of its own to work on: below, a tile is shared by four.
constexpr long long kWaveTiles = 1024;
constexpr int kRowBlocks = 3;    // MFMA row blocks of Wx per pass

typedef short short4v __attribute__((ext_vector_type(4)));

// bf16: NB blocks of 16 rows of Wx . x from row m0, for 64 positions, as one chain of v_mfma_f32_16x16x16_bf16 per block over
// all channels, 16 a step, kDeep steps in flight (no load in a branch: past the last step it is requested again and not
// used).
template <int NB>
__device__ __forceinline__ void chain_bf16(const XprojArgs& p, const bf16_t* x, uint32_t s, int m0, f32x4 (&acc)[NB][4]) {
    constexpr int kDeep = 4;
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15;
    const int Dc = p.Dc, steps = Dc / 16;
    const uint32_t P = (uint32_t)p.P, boff = ((uint32_t)(4 * g) * P + s) * 2u;
    const bf16_t* Wx = static_cast<const bf16_t*>(p.Wx);
    uint32_t arow[NB], braw[kDeep][4][2], araw[kDeep][NB][2];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
        arow[mb] = (uint32_t)min(m0 + 16 * mb + n, p.R + 2 * p.N - 1) * (uint32_t)Dc + 4u * g;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[mb][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    auto load = [&](int buf, int k) {
        const bf16_t* xk = x + (size_t)(16 * k) * P;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) load_words_at<2>(Wx + 16 * k, arow[mb] * 2u, araw[buf][mb]);
#pragma unroll
        for (int e = 0; e < 4; ++e) load_words_at<2>(xk + (size_t)e * P, boff, braw[buf][e]);
    };
    auto products = [&](int buf) {
        short4v bv[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t sel = t % 2 ? 0x07060302u : 0x05040100u;
            const u32x2_t v = {__builtin_amdgcn_perm(braw[buf][1][t / 2], braw[buf][0][t / 2], sel),
                               __builtin_amdgcn_perm(braw[buf][3][t / 2], braw[buf][2][t / 2], sel)};
            bv[t] = __builtin_bit_cast(short4v, v);
        }
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) {
            const u32x2_t av = {araw[buf][mb][0], araw[buf][mb][1]};
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[mb][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, av), bv[t], acc[mb][t], 0, 0, 0);
        }
    };
    if (steps > 0) {
#pragma unroll
        for (int d = 0; d < kDeep; ++d) load(d, min(d, steps - 1));
        int k = 0;
        for (; k + kDeep < steps; k += kDeep) {
#pragma unroll
            for (int d = 0; d < kDeep; ++d) {
                products(d);
                load(d, min(k + d + kDeep, steps - 1));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < kDeep; ++d)
            if (k + d < steps) products(d);
    }
    if (16 * steps < Dc) {                                 // the last channels: element by element, zero past the end on both operands
        const int c = 16 * steps + 4 * g;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            load_words_any<2>(x + (size_t)min(c + e, Dc - 1) * P + s, braw[0][e]);
            if (c + e >= Dc) braw[0][e][0] = braw[0][e][1] = 0u;
        }
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) {
            uint32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = elem_bits(Wx + arow[mb] - 4 * g + min(c + e, Dc - 1));
                if (c + e >= Dc) v[e] = 0u;
            }
            araw[0][mb][0] = v[0] | (v[1] << 16);
            araw[0][mb][1] = v[2] | (v[3] << 16);
        }
        products(0);
    }
}

// KR MFMA of delta_raw = Wdt . low[:R]: their operands (contraction index r = 4 s + g) and the rows they give.
template <int KR>
__device__ __forceinline__ void step_weights(const XprojArgs& p, int c0, float* a) {      // row c0 + n of Wdt
    const int g = (threadIdx.x & 63) >> 4, n = threadIdx.x & 15, R = p.R;
    const float* row = p.Wdt + (size_t)min(c0 + n, p.Dc - 1) * R;
#pragma unroll
    for (int s = 0; s < KR; ++s) {
        const float v = row[min(4 * s + g, R - 1)];
        a[s] = 4 * s + g < R ? v : 0.0f;
    }
}
template <int KR>
__device__ __forceinline__ void step_inputs(const float (*low)[64], int R, float (*bl)[4]) {
    const int g = (threadIdx.x & 63) >> 4, n = threadIdx.x & 15;
#pragma unroll
    for (int s = 0; s < KR; ++s) {
        const int r = 4 * s + g;
        const float4 v = *reinterpret_cast<const float4*>(&low[r][4 * n]);
        bl[s][0] = r < R ? v.x : 0.0f; bl[s][1] = r < R ? v.y : 0.0f; bl[s][2] = r < R ? v.z : 0.0f; bl[s][3] = r < R ? v.w : 0.0f;
    }
}
template <typename T, int KR>
__device__ __forceinline__ void step_rows(const XprojArgs& p, int b, const LanePos<4>& pos, int c0, const float* a, const float (*bl)[4]) {
    const int g = (threadIdx.x & 63) >> 4;
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
        if (c < p.Dc) pos.store(static_cast<T*>(p.delta_raw) + ((size_t)b * p.Dc + c) * (size_t)p.P, o);
    }
}
template <int KR> constexpr int step_ahead() { return KR <= 4 ? 4 : 1; }      // blocks of 16 rows whose weights are in flight

// KR: low-rank rows per lane group, 4 KR >= R.  TAIL, WIDE: of contract(), fp32 only
template <typename T, int KR, bool TAIL, bool WIDE>
__global__ __launch_bounds__(256, 2) void scan2d_xproj_kernel(const XprojArgs p) {
    constexpr bool CHAIN = Elem<T>::kBytes == 2;
    __shared__ float part[CHAIN ? 1 : 4][kRowBlocks * 16][64];
    __shared__ float low[4 * KR][64];
    const int tid = threadIdx.x, l = tid & 63, g = l >> 4, n = l & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Dc = p.Dc, N = p.N, R = p.R, M = R + 2 * N;
    const int b = blockIdx.x / p.tiles;
    const uint32_t p0 = (uint32_t)(blockIdx.x % p.tiles) * 64u, P = (uint32_t)p.P;
    const T* x = static_cast<const T*>(p.x) + (size_t)b * Dc * P;
    const LanePos pos(p0, n, P);

    constexpr int AHEAD = step_ahead<KR>();
    float a[AHEAD][KR];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) step_weights<KR>(p, 16 * wv + 64 * u, a[u]);      // requested in front of everything else

    constexpr int KS = contract_step<T>();
    const int span = ((Dc + KS - 1) / KS + 3) / 4 * KS;    // channels of a wavefront: whole steps
    const int cbeg = min(wv * span, Dc), cend = min(cbeg + span, Dc);
    for (int m0 = 0; m0 < M; m0 += kRowBlocks * 16) {
        if constexpr (CHAIN) {
            f32x4 acc[1][4];
            if (wv < kRowBlocks) chain_bf16<1>(p, x, pos.s, m0 + 16 * wv, acc);
            if (m0 > 0) __syncthreads();                   // the sums of the previous rows have been read
            if (wv < kRowBlocks) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *reinterpret_cast<float4*>(&part[0][16 * wv + 4 * g + i][4 * n]) = make_float4(acc[0][0][i], acc[0][1][i], acc[0][2][i], acc[0][3][i]);
            }
        } else {
            f32x4 acc[kRowBlocks][4];
#pragma unroll
            for (int mb = 0; mb < kRowBlocks; ++mb)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[mb][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            contract<T, kRowBlocks, 2, TAIL, WIDE>(x, P, pos.s, static_cast<const T*>(p.Wx), Dc, M, m0, cbeg, cend, acc);
            if (m0 > 0) __syncthreads();                   // the sums of the previous rows have been read
#pragma unroll
            for (int mb = 0; mb < kRowBlocks; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *reinterpret_cast<float4*>(&part[wv][16 * mb + 4 * g + i][4 * n]) = make_float4(acc[mb][0][i], acc[mb][1][i], acc[mb][2][i], acc[mb][3][i]);
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kRowBlocks; ++it) {          // 16 rows x 16 groups of 4 positions
            const int row = 16 * it + (tid >> 4), m = m0 + row;
            float4 v = *reinterpret_cast<const float4*>(&part[0][row][4 * n]);
#pragma unroll
            for (int w = 1; w < (CHAIN ? 1 : 4); ++w) {
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

    float bl[KR][4];
    step_inputs<KR>(low, R, bl);
    for (int c0 = 16 * wv; c0 < Dc; c0 += 64 * AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            step_rows<T, KR>(p, b, pos, c0 + 64 * u, a[u], bl);
            step_weights<KR>(p, c0 + 64 * (u + AHEAD), a[u]);
        }
}

// The same for bf16 and many positions: a wavefront owns 64 positions from the first product to the last, so nothing waits for
// another wavefront and x passes the caches once.
template <int KR>
__global__ __launch_bounds__(256, 2) void scan2d_xproj_wave_kernel(const XprojArgs p) {
    using T = bf16_t;
    __shared__ float lowL[4][4 * KR][64];
    const int g = (threadIdx.x & 63) >> 4, n = threadIdx.x & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = p.N, R = p.R, M = R + 2 * N;
    const long long tile = (long long)blockIdx.x * 4 + wv;
    if (tile >= (long long)p.tiles * p.Bt) return;
    const int b = (int)(tile / p.tiles);
    const uint32_t P = (uint32_t)p.P;
    const LanePos pos((uint32_t)(tile % p.tiles) * 64u, n, P);
    const T* x = static_cast<const T*>(p.x) + (size_t)b * p.Dc * P;
    float (*low)[64] = lowL[wv];
    for (int m0 = 0; m0 < M; m0 += kRowBlocks * 16) {
        f32x4 acc[kRowBlocks][4];
        chain_bf16<kRowBlocks>(p, x, pos.s, m0, acc);
#pragma unroll
        for (int mb = 0; mb < kRowBlocks; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = m0 + 16 * mb + 4 * g + i;
                const float v[4] = {acc[mb][0][i], acc[mb][1][i], acc[mb][2][i], acc[mb][3][i]};
                if (m < R) *reinterpret_cast<float4*>(&low[m][4 * n]) = make_float4(v[0], v[1], v[2], v[3]);
                else if (m < M) {
                    const int k = m - R;
                    pos.store(static_cast<T*>(k < N ? p.Bm : p.Cm) + ((size_t)b * N + (k < N ? k : k - N)) * P, v);
                }
            }
    }
    __builtin_amdgcn_wave_barrier();                       // LDS accesses of a wavefront stay in order
    constexpr int AHEAD = step_ahead<KR>();
    float a[AHEAD][KR], bl[KR][4];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) step_weights<KR>(p, 16 * u, a[u]);
    step_inputs<KR>(low, R, bl);
    for (int c0 = 0; c0 < p.Dc; c0 += 16 * AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            step_rows<T, KR>(p, b, pos, c0 + 16 * u, a[u], bl);
            step_weights<KR>(p, c0 + 16 * (u + AHEAD), a[u]);
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

template <typename T, bool TAIL, bool WIDE = false>
void launch(const XprojArgs& a, int Bt, hipStream_t stream) {
    const dim3 grid((unsigned)(a.tiles * Bt));
    if (a.R <= 8) hipLaunchKernelGGL((scan2d_xproj_kernel<T, 2, TAIL, WIDE>), grid, dim3(256), 0, stream, a);
    else if (a.R <= 16) hipLaunchKernelGGL((scan2d_xproj_kernel<T, 4, TAIL, WIDE>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((scan2d_xproj_kernel<T, 16, TAIL, WIDE>), grid, dim3(256), 0, stream, a);
}

int launch_xproj(const scan2d_desc* d, int R, const void* x, const void* Wx, const float* Wdt, void* delta_raw, void* Bm, void* Cm, hipStream_t stream) {
    if (R < 1 || R > 64) return SCAN2D_ERR_BAD_SHAPE;
    const bool bf16 = d->dtype == SCAN2D_BF16;
    XprojArgs a;
    a.x = x; a.Wx = Wx; a.Wdt = Wdt; a.delta_raw = delta_raw; a.Bm = Bm; a.Cm = Cm;
    a.Dc = d->Dc; a.N = d->N; a.R = R;
    a.P = (long long)d->H * d->W;
    const long long tiles = (a.P + 63) / 64;
    const bool fits = contract_fits(a.P, R + 2 * d->N, d->Dc, bf16 ? 2 : 4);
    const bool wave = fits && bf16 && tiles * d->Bt >= kWaveTiles;
    if (!launch_fits(wave ? (tiles * d->Bt + 3) / 4 : (fits ? tiles : a.P) * d->Bt, 256)) return SCAN2D_ERR_BAD_SHAPE;
    a.tiles = (int)tiles; a.Bt = d->Bt;
    (void)hipGetLastError();
    if (fits) {
        if (wave) {
            const dim3 grid((unsigned)((tiles * d->Bt + 3) / 4));
            if (R <= 8) hipLaunchKernelGGL(scan2d_xproj_wave_kernel<2>, grid, dim3(256), 0, stream, a);
            else if (R <= 16) hipLaunchKernelGGL(scan2d_xproj_wave_kernel<4>, grid, dim3(256), 0, stream, a);
            else hipLaunchKernelGGL(scan2d_xproj_wave_kernel<16>, grid, dim3(256), 0, stream, a);
        } else if (bf16) launch<bf16_t, false>(a, d->Bt, stream);      // 13 rows of positions within 32-bit offsets: any map
        else if (!contract_narrow(a.P, 4)) launch<float, true, true>(a, d->Bt, stream);
        else if (a.Dc % contract_step<float>() == 0) launch<float, false>(a, d->Bt, stream);
        else launch<float, true>(a, d->Bt, stream);
    } else {
        const dim3 grid((unsigned)(a.P * d->Bt));
        if (bf16) hipLaunchKernelGGL(scan2d_xproj_any_kernel<bf16_t>, grid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL(scan2d_xproj_any_kernel<float>, grid, dim3(256), 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace

int block_xproj_launch(const scan2d_desc* d, int R, const void* x, const void* Wx, const float* Wdt, void* delta_raw, void* Bm,
                       void* Cm, hipStream_t stream) {
    const size_t row = (size_t)d->H * d->W * (d->dtype == SCAN2D_BF16 ? 2 : 4);
    return by_items(*d, [&](const scan2d_desc& q, size_t b) {
        return launch_xproj(&q, R, item_at(x, b, row * d->Dc), Wx, Wdt, item_at(delta_raw, b, row * d->Dc), item_at(Bm, b, row * d->N), item_at(Cm, b, row * d->N), stream);
    });
}

}  // namespace scan2d
