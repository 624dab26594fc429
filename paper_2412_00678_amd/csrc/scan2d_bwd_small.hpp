// Backward 2D selective scan for small maps (W <= 16, H <= 16, N <= 16): the 14x14 grids of
// the last stage of a hierarchical backbone (2DMamba Sec. 4.3), the four scans of Supp. B.
//
// A map has WPM wavefronts (ceil(N / 4): 1, 2 or 4); each of their DPP rows owns one state, lane l of a row owns column
// l, and the whole map fits the registers: Bm and Cm of all rows are loaded once, together, and kept for the GS channels
// that a workgroup handles one after the other; the forward sweep leaves h[i-1,j] and hhor[i,j-1] of every row in
// registers, the reverse sweep walks back up.  No checkpoints and no bands.
//   - The row recurrences of different rows do not depend on each other: four rows are scanned together (one interleaved
//     DPP scan of four recurrences), only the column recurrences go row by row.
//   - What depends on the position alone (step, step * x, dy) is produced once per channel by the map's threads, loaded one
//     channel ahead, and read from LDS; the thread that produces a cell also adds up its sums over the states and
//     stores ddelta and dx: ddelta = sum(t A) + x * sum(q B), dx = step * sum(q B) + Dskip * dy.  A wavefront's four
//     states are added with v_permlane32_swap / v_permlane16_swap (both sums of two rows in one register), the
//     wavefronts' parts in LDS.
//   - dBm, dCm accumulate in registers over the channels of a workgroup.
// Bound: vector issue (about 40 instructions per position, channel and state).  14x14 fp32, 8 x 128 channels: the form
// it replaces (one wavefront per map, four states per lane, loads two rows ahead) took 26 us, its partial sums of
// every channel another 37.
#pragma once

#include "scan2d_bwd_shared.hpp"   // group_sum_last, halves_sum, row_pairs_sum
#include "scan2d_fwd_small.hpp"    // raw_to_float

namespace scan2d {

// SP: delta is the raw projection, the step its softplus; GATE: as in scan2d_bwd_shared_kernel.
template <typename T, int WPM, bool SP, bool GATE>
__global__ __launch_bounds__(256) void scan2d_bwd_small_kernel(const BwdArgs p) {
    static_assert(!GATE || SP, "the gate goes with the softplus step");
    constexpr int HM = 16, JPW = 4 / WPM, TMJ = 64 * WPM, CPT = 256 / TMJ;    // rows at most, maps per workgroup, threads and cells per thread
    __shared__ float pos[JPW][3][256];                    // step, step * x, dy of cell 16 i + j
    __shared__ float part[4][HM / 2][64];                 // [wavefront][row pair]: ddelta of both rows, then dx of both
    __shared__ float red[2][2][4];                        // [channel parity][dDskip, bias gradient][wavefront]
    const int tid = threadIdx.x, lane = tid & 63, l = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jl = wave / WPM, tm = tid - jl * TMJ, n = (wave % WPM) * 4 + g;
    const long long job = (long long)blockIdx.x * JPW + jl;
    const bool live = job < (long long)p.Bt * p.CG;
    const int b = live ? (int)(job / p.CG) : 0, cg = live ? (int)(job % p.CG) : 0;
    const int c_first = cg * p.GS, nch = live ? min(p.GS, p.Dc - c_first) : 0;
    const int H = p.H, W = p.W, N = p.N;
    const size_t HW = (size_t)H * W;
    const bool state = n < N;
    const uint8_t* mm = p.mask ? p.mask + (size_t)b * HW : nullptr;

    // ---- the cells this thread produces and stores
    uint32_t cell[CPT];
    bool in[CPT];
#pragma unroll
    for (int v = 0; v < CPT; ++v) {
        const int id = tm + v * TMJ, i = id >> 4, j = id & 15;
        in[v] = i < H && j < W;
        cell[v] = in[v] ? (uint32_t)(i * W + j) : 0u;
    }
    uint32_t rx[CPT], rd[CPT], ry[CPT], rm[CPT], rz[GATE ? CPT : 1], rs[GATE ? CPT : 1];
    auto request = [&](int ch) {
        const size_t o = ((size_t)b * p.Dc + c_first + min(ch, max(nch - 1, 0))) * HW;
#pragma unroll
        for (int v = 0; v < CPT; ++v) {
            rx[v] = elem_bits(reinterpret_cast<const T*>(p.x) + o + cell[v]);
            rd[v] = elem_bits(reinterpret_cast<const T*>(p.delta) + o + cell[v]);
            ry[v] = elem_bits(reinterpret_cast<const T*>(p.dy) + o + cell[v]);
            if constexpr (GATE) {
                rz[v] = elem_bits(reinterpret_cast<const T*>(p.z) + o + cell[v]);
                rs[v] = elem_bits(reinterpret_cast<const T*>(p.y_scan) + o + cell[v]);
            }
        }
    };
    request(0);
#pragma unroll
    for (int v = 0; v < CPT; ++v) rm[v] = mm != nullptr ? (uint32_t)mm[cell[v]] : 0u;

    // ---- Bm, Cm of this lane's state and column, all rows
    float Bv[HM], Cv[HM];
    {
        const size_t o = ((size_t)b * N + min(n, N - 1)) * HW + (size_t)min(l, W - 1);
        uint32_t rB[HM], rC[HM];
#pragma unroll
        for (int i = 0; i < HM; ++i) {
            rB[i] = elem_bits(reinterpret_cast<const T*>(p.Bm) + o + (size_t)min(i, H - 1) * W);
            rC[i] = elem_bits(reinterpret_cast<const T*>(p.Cm) + o + (size_t)min(i, H - 1) * W);
        }
#pragma unroll
        for (int i = 0; i < HM; ++i) {                    // a state that does not exist contributes nothing
            Bv[i] = state ? raw_to_float(T{}, rB[i]) : 0.0f;
            Cv[i] = state ? raw_to_float(T{}, rC[i]) : 0.0f;
        }
    }
    float dBacc[HM], dCacc[HM];
#pragma unroll
    for (int i = 0; i < HM; ++i) { dBacc[i] = 0.0f; dCacc[i] = 0.0f; }

    for (int ch = 0; ch < p.GS; ++ch) {
        const bool act = ch < nch;
        const int c = c_first + (act ? ch : 0);
        const size_t map = (size_t)b * p.Dc + c;
        const float An = state ? p.A[(size_t)c * N + n] : 0.0f, Ap = An * kLog2e;
        const float dsk = p.Dskip != nullptr ? p.Dskip[c] : 0.0f;
        const float bias = (SP && p.delta_bias != nullptr) ? p.delta_bias[c] : 0.0f;

        float dl_[CPT], xe_[CPT], dy_[CPT], lg_[SP ? CPT : 1];
#pragma unroll
        for (int v = 0; v < CPT; ++v) {
            const bool ok = in[v] && act;
            float dl = raw_to_float(T{}, rd[v]);
            if constexpr (SP) {
                lg_[v] = logistic_f32(dl + bias);         // kept: formed from the step, it would have the step's absolute error
                dl = softplus_f32(dl + bias);
            }
            dl_[v] = ok ? dl : 0.0f;
            xe_[v] = ok && rm[v] == 0u ? raw_to_float(T{}, rx[v]) : 0.0f;        // select: nothing under the mask leaks
            float dyv = ok ? raw_to_float(T{}, ry[v]) : 0.0f;
            if constexpr (GATE) {
                const float zv = raw_to_float(T{}, rz[v]), sg = logistic_f32(zv);
                if (ok) store_elem(reinterpret_cast<T*>(p.dz) + map * HW + cell[v], dyv * raw_to_float(T{}, rs[v]) * (sg * fmaf(zv, 1.0f - sg, 1.0f)));
                dyv *= zv * sg;
                dyv = ok ? dyv : 0.0f;
            }
            dy_[v] = dyv;
            pos[jl][0][tm + v * TMJ] = dl_[v];
            pos[jl][1][tm + v * TMJ] = dl_[v] * xe_[v];
            pos[jl][2][tm + v * TMJ] = dyv;
        }
        request(ch + 1);
        __syncthreads();

        // ---- scans 1 and 2, top to bottom, four rows at a time
        float hprev[HM], hhl[HM], h = 0.0f;
#pragma unroll
        for (int q = 0; q < HM / 4; ++q) {
            if (4 * q < H) {                              // uniform; rows past H have step 0 and x 0 and change nothing
                float a[4], P[4], U[4], cin[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * q + e;
                    a[e] = __builtin_amdgcn_exp2f(pos[jl][0][16 * i + l] * Ap);
                    P[e] = a[e];
                    U[e] = pos[jl][1][16 * i + l] * Bv[i];
                }
                group_scan<16, 4>(P, U, cin);             // U = hhor[i,j], cin = hhor[i,j-1]
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    hhl[4 * q + e] = cin[e];
                    hprev[4 * q + e] = h;
                    h = fmaf(a[e], h, U[e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) { hprev[4 * q + e] = h; hhl[4 * q + e] = 0.0f; }
            }
        }
        // ---- scans 3 and 4, bottom to top
        float ga = 0.0f, dAb = 0.0f;
#pragma unroll
        for (int q = HM / 4 - 1; q >= 0; --q) {
            if (4 * q < H) {
                float dl[4], dxe[4], a[4], g3[4], gag[4], P[4], Q[4], qin[4], ar[4], t[4], s1[4], s2[4];
#pragma unroll
                for (int e = 3; e >= 0; --e) {
                    const int i = 4 * q + e;
                    dl[e] = pos[jl][0][16 * i + l];
                    dxe[e] = pos[jl][1][16 * i + l];
                    const float dyv = pos[jl][2][16 * i + l];
                    a[e] = __builtin_amdgcn_exp2f(dl[e] * Ap);
                    dCacc[i] = fmaf(dyv, i + 1 < HM ? hprev[i + 1 < HM ? i + 1 : i] : h, dCacc[i]);
                    g3[e] = fmaf(dyv, Cv[i], ga);         // scan 3: g[i,j]
                    ga = a[e] * g3[e];
                    gag[e] = ga;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    ar[e] = from_right<16>(a[e]);         // a[i,j+1]
                    P[e] = ar[e];
                    Q[e] = g3[e];
                }
                group_scan_left<16, 4>(P, Q, qin);        // qin = q[i,j+1]
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * q + e;
                    const float qv = fmaf(ar[e], qin[e], g3[e]);                   // scan 4: q[i,j]
                    t[e] = fmaf(a[e] * qv, hhl[i], gag[e] * hprev[i]);             // gradient of the decay, times the decay
                    dBacc[i] = fmaf(qv, dxe[e], dBacc[i]);
                    s1[e] = t[e] * An;
                    s2[e] = qv * Bv[i];
                }
                if (4 * q + 3 >= H) {                     // rows past H add nothing to dA (0 * infinity would be NaN); once per map
#pragma unroll
                    for (int e = 1; e < 4; ++e)
                        if (4 * q + e >= H) asm volatile("v_mov_b32 %0, 0" : "=v"(t[e]));
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) dAb = fmaf(t[e], dl[e], dAb);
#pragma unroll
                for (int e = 0; e < 4; e += 2)
                    part[wave][2 * q + e / 2][lane] = row_pairs_sum(halves_sum(s1[e], s2[e]), halves_sum(s1[e + 1], s2[e + 1]));
            }
        }
        {
            const float tot = row_sum16(l < W ? dAb : 0.0f);
            if (l == 0 && state && act) p.pA[map * N + n] = tot;
        }
        __syncthreads();

        // ---- the sums over the states of this thread's cells
        float dDb = 0.0f, dBb = 0.0f;
#pragma unroll
        for (int v = 0; v < CPT; ++v) {
            const int id = tm + v * TMJ, i = id >> 4, j = id & 15;
            float S1 = 0.0f, S2 = 0.0f;
#pragma unroll
            for (int w = 0; w < WPM; ++w) {
                S1 += part[jl * WPM + w][i / 2][16 * (i & 1) + j];
                S2 += part[jl * WPM + w][i / 2][32 + 16 * (i & 1) + j];
            }
            if (in[v] && act) {
                float dd = fmaf(xe_[v], S2, S1);
                if constexpr (SP) { dd *= lg_[v]; dBb += dd; }
                store_elem(reinterpret_cast<T*>(p.ddelta) + map * HW + cell[v], dd);
                store_elem(reinterpret_cast<T*>(p.dx) + map * HW + cell[v], rm[v] != 0u ? 0.0f : fmaf(dsk, dy_[v], dl_[v] * S2));
            }
            dDb = fmaf(dy_[v], xe_[v], dDb);
        }
        dDb = group_sum_last<64>(dDb);
        if constexpr (SP) dBb = group_sum_last<64>(dBb);
        if (lane == 63) { red[ch & 1][0][wave] = dDb; red[ch & 1][1][wave] = dBb; }
        __syncthreads();                                  // also: the parts have been read
        if (act && tm == 0) {
            float sD = 0.0f, sB = 0.0f;
#pragma unroll
            for (int w = 0; w < WPM; ++w) { sD += red[ch & 1][0][jl * WPM + w]; sB += red[ch & 1][1][jl * WPM + w]; }
            if (p.pD != nullptr) p.pD[map] = sD;
            if (SP && p.pBias != nullptr) p.pBias[map] = sB;
        }
    }
    if (live && state && l < W) {
        const size_t o = (((size_t)b * p.CG + cg) * N + n) * HW + l;
#pragma unroll
        for (int i = 0; i < HM; ++i)
            if (i < H) {
                p.pB[o + (size_t)i * W] = dBacc[i];
                p.pC[o + (size_t)i * W] = dCacc[i];
            }
    }
}

}  // namespace scan2d
