// The convolution in front of the scan inside a 2DMamba block (Sec. 3.2, Fig. 2):
//     x = SiLU(depth-wise correlation of u with a KH x KW filter + bias)
// written in the storage type that the projections and the scan read.
#include "scan2d_block.hpp"

#include <algorithm>

#include "scan2d_contract.hpp"

namespace scan2d {
namespace {

// ------------------------------------------------------------------------------------ convolution + SiLU
// Any filter, narrow maps: one thread per 4 consecutive outputs of a row.  Per filter row it reads the KW + 3 inputs its outputs need, element
// by element (any width, any alignment; L1 serves the overlap between neighbours), zero outside the map.
template <typename T>
__global__ __launch_bounds__(256) void scan2d_block_conv_silu_kernel(const T* __restrict__ u, const float* __restrict__ w,
                                                                     const float* __restrict__ bias, T* __restrict__ x,
                                                                     long long maps, int Dc, int H, int W, int KH, int KW, int PH, int PW) {
    const int J4 = (W + 3) / 4;
    const long long total = maps * H * J4;
    const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
    if (id >= total) return;
    const int jq = (int)(id % J4);
    const long long t = id / J4;
    const int i = (int)(t % H);
    const long long map = t / H;
    const int c = (int)(map % Dc);
    const int j0 = jq * 4;
    const T* um = u + (size_t)map * H * W;
    const float* wc = w + (size_t)c * KH * KW;
    const float b = bias != nullptr ? bias[c] : 0.0f;
    float acc[4] = {b, b, b, b};
    for (int p = 0; p < KH; ++p) {
        const int ii = i + p - PH;
        if (ii < 0 || ii >= H) continue;
        const T* row = um + (size_t)ii * W;
        float win[10];                                   // KW + 3 <= 10 inputs
#pragma unroll
        for (int e = 0; e < 10; ++e) {
            const int jj = j0 - PW + e;
            win[e] = (e < KW + 3 && jj >= 0 && jj < W) ? widen_bits<T>(elem_bits(row + jj)) : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 7; ++q) {
            if (q < KW) {
                const float wv = wc[p * KW + q];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = fmaf(wv, win[e + q], acc[e]);
            }
        }
    }
    T* out = x + (size_t)map * H * W + (size_t)i * W + j0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (j0 + e < W) store_elem(out + e, acc[e] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-acc[e] * kLog2e)));
}

// The centred 3x3 filter on maps of at least 8 columns: a lane owns 8 consecutive columns and walks down RS rows with the
// three input rows of its window in registers as fp32; per row it loads its 8 elements (any alignment) and the two beside
// them, two rows ahead of their use.  At the right edge the group of 8 moves back and overlaps its neighbour; only the
// columns it owns are stored.  Nothing passes through LDS.  Bound: HBM (one read, one write per element; about 16
// instructions per output, half of what 16-column LDS tiles took).
template <typename T, int RS>
__global__ __launch_bounds__(256) void scan2d_block_conv3_silu_kernel(const T* __restrict__ u, const float* __restrict__ w,
                                                                      const float* __restrict__ bias, T* __restrict__ x,
                                                                      long long lanes, int Dc, int H, int W, int groups, int strips) {
    constexpr int XW = words_of<T, 8>();
    const long long id = min((long long)blockIdx.x * 256 + threadIdx.x, lanes - 1);
    const bool live = (long long)blockIdx.x * 256 + threadIdx.x < lanes;
    const int cg = (int)(id % groups);
    const long long rest = id / groups;
    const int i0 = (int)(rest % strips) * RS;
    const long long map = rest / strips;
    const int c = (int)(map % Dc);
    const int col = 8 * cg, s = min(col, W - 8);          // first column owned, first column read
    const bool left = s > 0, right = s + 8 < W;
    const T* um = u + (size_t)map * H * W + s;
    float wt[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wt[k] = w[(size_t)c * 9 + k];
    const float b = bias != nullptr ? bias[c] : 0.0f;

    uint32_t raw[2][XW], rawl[2], rawr[2];
    auto request = [&](int buf, int i) {
        const T* row = um + (size_t)min(max(i, 0), H - 1) * W;
        load_words_any<XW>(row, raw[buf]);
        rawl[buf] = elem_bits(row - (left ? 1 : 0));
        rawr[buf] = elem_bits(row + (right ? 8 : 7));
    };
    float win[3][10];
    auto unpack = [&](int buf, int i, float* v) {
        const bool in = i >= 0 && i < H;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j + 1] = in ? get_elem<T, 8>(raw[buf], j) : 0.0f;
        v[0] = in && left ? widen_bits<T>(rawl[buf]) : 0.0f;
        v[9] = in && right ? widen_bits<T>(rawr[buf]) : 0.0f;
    };
    request(0, i0 - 1);
    request(1, i0);
    unpack(0, i0 - 1, win[0]);
    request(0, i0 + 1);
    unpack(1, i0, win[1]);
    request(1, i0 + 2);
    T* const om = x + (size_t)map * H * W + s;
#pragma unroll
    for (int r = 0; r < RS; ++r) {
        const int i = i0 + r;
        unpack(r & 1, i + 1, win[(r + 2) % 3]);
        if (r + 2 < RS) request(r & 1, i + 3);
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float acc = b;
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q) acc = fmaf(wt[3 * p + q], win[(r + p) % 3][j + q], acc);
            o[j] = acc * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-acc * kLog2e));
        }
        if (i < H && live) {
            T* out = om + (size_t)i * W;
            if (s == col) {
                uint32_t d[XW];
                if constexpr (Elem<T>::kBytes == 2) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) d[j] = pack_bf16x2(o[2 * j], o[2 * j + 1]);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) d[j] = __float_as_uint(o[j]);
                }
                store_words_any<XW>(out, d);
            } else {
#pragma unroll
                for (int j = 1; j < 8; ++j)
                    if (s + j >= col) store_elem(out + j, o[j]);
            }
        }
    }
}

// Any other filter on wide maps (W >= 32): one workgroup per tile of 32 rows x 64 columns.  The tile and its halo go to LDS as fp32 through
// aligned vector loads (zero outside the map), the channel's filter goes there too, then every thread forms 4 consecutive
// outputs in each of two rows from LDS.
constexpr int kConvTH = 32, kConvTW = 64, kConvHalo = 8, kConvCols = kConvTW + 2 * kConvHalo;   // 80 columns per tile row
// LDS row pitch: odd, so that the four rows a wavefront reads (lanes: 16 groups of 4 columns x 4 rows) fall on different banks
constexpr int kConvPitch = kConvCols + 1;
template <typename T>
__global__ __launch_bounds__(256) void scan2d_block_conv_silu_tile_kernel(const T* __restrict__ u, const float* __restrict__ w,
                                                                          const float* __restrict__ bias, T* __restrict__ x,
                                                                          int Dc, int H, int W, int KH, int KW, int PH, int PW,
                                                                          int tiles_w, int tiles_h) {
    constexpr int EB = Elem<T>::kBytes;
    __shared__ __align__(16) float tile[(kConvTH + 6) * kConvPitch];
    __shared__ float wts[52];
    const int tid = threadIdx.x;
    const int tw = blockIdx.x % tiles_w;
    const int th = (blockIdx.x / tiles_w) % tiles_h;
    const long long map = blockIdx.x / (tiles_w * tiles_h);
    const int c = (int)(map % Dc);
    const int i0 = th * kConvTH, j0 = tw * kConvTW;
    const T* um = u + (size_t)map * H * W;
    const int rows = min(kConvTH, H - i0) + KH - 1;
    const bool vec_ok = (W % 4) == 0;                     // rows and maps then start on vector boundaries
    if (tid < KH * KW) wts[tid] = w[(size_t)c * KH * KW + tid];
    if (tid == 63) wts[49] = bias != nullptr ? bias[c] : 0.0f;
    for (int idx = tid; idx < rows * (kConvCols / 4); idx += 256) {
        const int r = idx / (kConvCols / 4), q = idx % (kConvCols / 4);
        const int ii = i0 + r - PH, jj = j0 - kConvHalo + 4 * q;
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (ii >= 0 && ii < H && jj + 3 >= 0 && jj < W) {
            const T* src = um + (size_t)ii * W + jj;
            if (vec_ok && jj >= 0 && jj + 3 < W) {
                if constexpr (EB == 2) {
                    const uint2 t = *reinterpret_cast<const uint2*>(src);
                    v = make_float4(__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16),
                                    __uint_as_float(t.y & 0xffff0000u));
                } else {
                    v = *reinterpret_cast<const float4*>(src);
                }
            } else {
                if (jj >= 0 && jj < W) v.x = widen_bits<T>(elem_bits(src));
                if (jj + 1 >= 0 && jj + 1 < W) v.y = widen_bits<T>(elem_bits(src + 1));
                if (jj + 2 >= 0 && jj + 2 < W) v.z = widen_bits<T>(elem_bits(src + 2));
                if (jj + 3 >= 0 && jj + 3 < W) v.w = widen_bits<T>(elem_bits(src + 3));
            }
        }
        float* dst = tile + r * kConvPitch + 4 * q;
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
    }
    __syncthreads();
    const int jq = tid % 16, j = j0 + 4 * jq;
    if (j >= W) return;
    const float b = wts[49];
    constexpr int KHM = 7, KWM = 7;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int r = tid / 16 + 16 * half;               // output row inside the tile
        const int i = i0 + r;
        if (i >= H) continue;
        float acc[4] = {b, b, b, b};
#pragma unroll
        for (int pp = 0; pp < KHM; ++pp) {
            if (pp < KH) {
                const float* row = tile + (r + pp) * kConvPitch + kConvHalo + 4 * jq - PW;
                float win[KWM + 3];
#pragma unroll
                for (int e = 0; e < KWM + 3; ++e) win[e] = e < KW + 3 ? row[e] : 0.0f;
#pragma unroll
                for (int q = 0; q < KWM; ++q) {
                    if (q < KW) {
                        const float wv = wts[pp * KW + q];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[e] = fmaf(wv, win[e + q], acc[e]);
                    }
                }
            }
        }
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[e] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-acc[e] * kLog2e));   // SiLU: v_exp, v_rcp
        T* out = x + (size_t)map * H * W + (size_t)i * W + j;
        if (vec_ok && j + 3 < W) {
            if constexpr (EB == 2) {
                uint2 t;
                t.x = pack_bf16x2(o[0], o[1]);
                t.y = pack_bf16x2(o[2], o[3]);
                *reinterpret_cast<uint2*>(out) = t;
            } else {
                *reinterpret_cast<float4*>(out) = make_float4(o[0], o[1], o[2], o[3]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < W) store_elem(out + e, o[e]);
        }
    }
}

}  // namespace

int block_conv_silu_launch(const scan2d_desc* d, const scan2d_conv_shape* cs, const void* u, const float* w, const float* bias,
                           void* x, hipStream_t stream) {
    if (cs->KH < 1 || cs->KH > 7 || cs->KW < 1 || cs->KW > 7 || cs->PH < 0 || cs->PH >= cs->KH || cs->PW < 0 || cs->PW >= cs->KW)
        return SCAN2D_ERR_BAD_SHAPE;
    const long long maps = (long long)d->Bt * d->Dc;
    (void)hipGetLastError();
    if (cs->KH == 3 && cs->KW == 3 && cs->PH == 1 && cs->PW == 1 && d->W >= 8) {
        // strips of 8 rows re-read a quarter of the rows (from L2); strips of 4 where those would leave SIMDs idle
        const int groups = (d->W + 7) / 8;
        const bool tall = maps * ((d->H + 7) / 8) * groups >= 64LL * 2048;
        const int strips = tall ? (d->H + 7) / 8 : (d->H + 3) / 4;
        const long long lanes = maps * strips * groups, wgs = (lanes + 255) / 256;
        if (wgs > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
        if (d->dtype == SCAN2D_BF16) {
            auto kernel = tall ? scan2d_block_conv3_silu_kernel<bf16_t, 8> : scan2d_block_conv3_silu_kernel<bf16_t, 4>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(256), 0, stream, static_cast<const bf16_t*>(u), w, bias,
                               static_cast<bf16_t*>(x), lanes, d->Dc, d->H, d->W, groups, strips);
        } else {
            auto kernel = tall ? scan2d_block_conv3_silu_kernel<float, 8> : scan2d_block_conv3_silu_kernel<float, 4>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(256), 0, stream, static_cast<const float*>(u), w, bias,
                               static_cast<float*>(x), lanes, d->Dc, d->H, d->W, groups, strips);
        }
        return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
    }
    if (d->W >= 32) {                                     // tiles of 32 x 64 outputs staged through LDS
        const int tiles_w = (d->W + kConvTW - 1) / kConvTW, tiles_h = (d->H + kConvTH - 1) / kConvTH;
        const long long wgs = maps * tiles_w * tiles_h;
        if (wgs > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
        if (d->dtype == SCAN2D_BF16)
            hipLaunchKernelGGL(scan2d_block_conv_silu_tile_kernel<bf16_t>, dim3((unsigned)wgs), dim3(256), 0, stream, static_cast<const bf16_t*>(u), w,
                               bias, static_cast<bf16_t*>(x), d->Dc, d->H, d->W, cs->KH, cs->KW, cs->PH, cs->PW, tiles_w, tiles_h);
        else
            hipLaunchKernelGGL(scan2d_block_conv_silu_tile_kernel<float>, dim3((unsigned)wgs), dim3(256), 0, stream, static_cast<const float*>(u), w,
                               bias, static_cast<float*>(x), d->Dc, d->H, d->W, cs->KH, cs->KW, cs->PH, cs->PW, tiles_w, tiles_h);
        return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
    }
    const long long total = maps * d->H * ((d->W + 3) / 4);
    const long long blocks = (total + 255) / 256;
    if (blocks > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    if (d->dtype == SCAN2D_BF16)
        hipLaunchKernelGGL(scan2d_block_conv_silu_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, stream,
                           static_cast<const bf16_t*>(u), w, bias, static_cast<bf16_t*>(x), maps, d->Dc, d->H, d->W, cs->KH, cs->KW, cs->PH, cs->PW);
    else
        hipLaunchKernelGGL(scan2d_block_conv_silu_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream,
                           static_cast<const float*>(u), w, bias, static_cast<float*>(x), maps, d->Dc, d->H, d->W, cs->KH, cs->KW, cs->PH, cs->PW);
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace scan2d
