// Forward 2D selective scan for maps of at most 16 x 16 positions and 16 states when there are few of them (2DMamba
// Sec. 4.3 times 14 x 14 grids: the last stage of a hierarchical backbone).  Such a call is bound by the chain of
// dependent steps, not by work: a kernel that walks the rows one after the other pays H times the latency of a row
// step.  Here a workgroup of 256 threads owns a map and takes both recurrences as parallel scans:
//   1. thread (i, j) = (DPP row, lane) holds cell (i, j); Eq. 5 is a 16-lane DPP scan along j for all rows at once;
//   2. the row results pass through LDS, transposed, and thread (j, i) now holds cell (i, j); Eq. 6 is the same DPP
//      scan along i for all columns at once (the rows of a column are independent of the other columns), and the sum over
//      the states of C * h goes back through LDS;
//   3. thread (i, j) adds Dskip * x, applies the gate (GATE) and stores the cell.
// Two scans of four DPP steps instead of H row steps.  Every global access is made in the first layout (a wavefront
// touches four row segments per instruction; the same cells column-wise would touch sixteen cache lines); Cm and the step
// reach the second layout through LDS together with the row results, and the decay is recomputed there.  Cells past H or W
// lie to the right of / below every real cell, and both scans only run rightwards / downwards, so whatever they hold (valid
// memory is read: addresses are clamped) reaches no output.
// With more maps than the chip holds workgroups a workgroup takes several channels of a batch item one after the other:
// Bm stays in registers, Cm in LDS, and a channel's x, step and z are requested one channel ahead.
#include "../../include/scan2d.h"
#include "scan2d_fwd.hpp"
#include "scan2d_variants.hpp"

namespace scan2d {
namespace {

constexpr int kTile = 16, kTilePitch = 17, kTileStates = 16;

__device__ __forceinline__ float tile_widen(float, uint32_t bits) { return __uint_as_float(bits); }
__device__ __forceinline__ float tile_widen(bf16_t, uint32_t bits) { return __uint_as_float(bits << 16); }

// ONE: one channel per workgroup, no gate: the second layout stores its cells itself (x reaches it through the plane that the
// sums would come back in), which saves the third step and its barrier (1024 maps of 14x14 fp32: 7.3 against 7.5 us).
template <typename T, bool SP, bool GATE, bool ONE>
__global__ __launch_bounds__(256) void scan2d_fwd_tile16_kernel(const FwdArgs p) {
    static_assert(!GATE || (SP && !ONE), "the gate goes with the softplus step, and z stays in the first layout");
    // [value][column][row], value = row result of Eq. 5 per state, Cm per state, the step, the sum over the states
    __shared__ float tr[(2 * kTileStates + 2) * kTile * kTilePitch];
    const int tid = threadIdx.x;
    const int r = tid >> 4, q = tid & 15;                  // DPP row and lane: (i, j) in steps 1 and 3, (j, i) in step 2
    const int H = p.H, W = p.W, N = p.N;
    const size_t HW = (size_t)H * W;
    const int per = ONE ? 1 : p.MPW, groups = (p.Dc + per - 1) / per;      // of `per` channels per batch item
    const int b = (int)(blockIdx.x / groups), c0 = (int)(blockIdx.x % groups) * per, nch = ONE ? 1 : min(per, p.Dc - c0);
    const size_t map0 = (size_t)b * p.Dc + c0;
    const T* xm = reinterpret_cast<const T*>(p.x);
    const T* dm = reinterpret_cast<const T*>(p.delta);
    const T* zm = reinterpret_cast<const T*>(p.z);         // GATE only
    const uint8_t* mm = p.mask ? p.mask + (size_t)b * HW : nullptr;
    const T* Bb = reinterpret_cast<const T*>(p.Bm) + (size_t)b * N * HW;
    const T* Cb = reinterpret_cast<const T*>(p.Cm) + (size_t)b * N * HW;
    const uint32_t o1 = (uint32_t)(min(r, H - 1) * W + min(q, W - 1));   // this thread's cell, clamped into the map
    const bool live = r < H && q < W;

    // ---- everything this thread reads for the first channel, requested at once
    uint32_t rB[kTileStates], rC[kTileStates], rx, rd, rz = 0u;
    auto request = [&](int ch) {
        const size_t o = (map0 + ch) * HW + o1;
        rx = elem_bits(xm + o);
        rd = elem_bits(dm + o);
        if constexpr (GATE) rz = elem_bits(zm + o);
    };
    request(0);
    const bool background = mm != nullptr && mm[o1] != 0;
#pragma unroll
    for (int n = 0; n < kTileStates; ++n) {
        const size_t so = (size_t)min(n, N - 1) * HW;     // states past N re-read the last one and are not summed
        rB[n] = elem_bits(Bb + so + o1);
        rC[n] = elem_bits(Cb + so + o1);
    }
    float* const put = tr + q * kTilePitch + r;            // steps 1 and 3: [.][q][r]
    float* const get = tr + r * kTilePitch + q;            // step 2:        [.][r][q], the cell (q, r)
    constexpr int PLANE = kTile * kTilePitch;

    for (int ch = 0; ch < nch; ++ch) {
        const int c = c0 + ch;
        float Ap[kTileStates];
#pragma unroll
        for (int n = 0; n < kTileStates; ++n) Ap[n] = p.A[(size_t)c * N + min(n, N - 1)] * kLog2e;
        const float dsk = p.Dskip != nullptr ? p.Dskip[c] : 0.0f;
        const float dbias = (SP && p.delta_bias != nullptr) ? p.delta_bias[c] : 0.0f;

        // ---- step 1: Eq. 5 along the lanes of every row
        const float xe = background ? 0.0f : tile_widen(T{}, rx), zv = tile_widen(T{}, rz);
        {
            float dl = tile_widen(T{}, rd);
            if constexpr (SP) dl = softplus_f32(dl + dbias);
            if (ch + 1 < nch) request(ch + 1);             // uniform
            const float dxe = dl * xe;
            put[2 * kTileStates * PLANE] = dl;
            if constexpr (ONE) put[(2 * kTileStates + 1) * PLANE] = xe;
#pragma unroll
            for (int n0 = 0; n0 < kTileStates; n0 += 4) {
                if (n0 < N) {                              // uniform
                    float P[4], Hh[4], cin[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        P[t] = __builtin_amdgcn_exp2f(dl * Ap[n0 + t]);
                        Hh[t] = dxe * tile_widen(T{}, rB[n0 + t]);
                        if (ch == 0) put[(kTileStates + n0 + t) * PLANE] = tile_widen(T{}, rC[n0 + t]);
                    }
                    group_scan<16, 4>(P, Hh, cin);
#pragma unroll
                    for (int t = 0; t < 4; ++t) put[(n0 + t) * PLANE] = Hh[t];
                }
            }
        }
        __syncthreads();

        // ---- step 2: Eq. 6 along the lanes of every column, then the sum over the states
        {
            const float dl = get[2 * kTileStates * PLANE];
            float yacc = 0.0f;
#pragma unroll
            for (int n0 = 0; n0 < kTileStates; n0 += 4) {
                if (n0 < N) {
                    float P[4], Hh[4], cin[4], Cv[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        P[t] = __builtin_amdgcn_exp2f(dl * Ap[n0 + t]);
                        Hh[t] = get[(n0 + t) * PLANE];
                        Cv[t] = get[(kTileStates + n0 + t) * PLANE];
                    }
                    group_scan<16, 4>(P, Hh, cin);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (n0 + t < N) yacc = fmaf(Cv[t], Hh[t], yacc);
                }
            }
            if constexpr (ONE) {
                const float v = fmaf(dsk, get[(2 * kTileStates + 1) * PLANE], yacc);      // as in step 3
                if (q < H && r < W) store_elem(reinterpret_cast<T*>(p.y) + map0 * HW + (size_t)q * W + r, v);
                return;
            }
            get[(2 * kTileStates + 1) * PLANE] = yacc;
        }
        __syncthreads();                                   // also: step 2 has read what the next channel's step 1 overwrites

        // ---- step 3: skip term, gate, store
        if (live) {
            const float v = fmaf(dsk, xe, put[(2 * kTileStates + 1) * PLANE]);
            const size_t o = (map0 + ch) * HW + o1;
            if (!GATE || p.y != nullptr) store_elem(reinterpret_cast<T*>(p.y) + o, v);
            if constexpr (GATE) store_elem(reinterpret_cast<T*>(p.y_gated) + o, v * (zv * logistic_f32(zv)));
        }
    }
}

}  // namespace

namespace {
template <typename T>
FwdKernel tile16_kernel(bool sp, bool gate, bool one) {
    if (gate) return scan2d_fwd_tile16_kernel<T, true, true, false>;
    if (one) return sp ? scan2d_fwd_tile16_kernel<T, true, false, true> : scan2d_fwd_tile16_kernel<T, false, false, true>;
    return sp ? scan2d_fwd_tile16_kernel<T, true, false, false> : scan2d_fwd_tile16_kernel<T, false, false, false>;
}
}  // namespace

FwdKernel fwd_tile16_kernel(int dtype, bool sp, bool gate, bool one) {
    return dtype == SCAN2D_BF16 ? tile16_kernel<bf16_t>(sp, gate, one) : tile16_kernel<float>(sp, gate, one);
}

}  // namespace scan2d
