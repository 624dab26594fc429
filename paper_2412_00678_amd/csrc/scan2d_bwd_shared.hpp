// Backward main sweep, the form whose lane groups share the per-position work of a map through LDS
// (2DMamba Supp. B: two forward scans rebuild the states, a reverse column scan and a reverse row scan carry
// the gradients).  Same banded organisation as scan2d_bwd_main_kernel (scan2d_bwd_kernels.hpp): bands of RB
// rows walked bottom-up, per band and channel the states h[i-1,j] are rebuilt into registers from the band's
// checkpoint, then the band's rows are walked upwards with g (reverse column recurrence, an FMA on a register
// that persists from row to row) and q (reverse row recurrence: serial over the lane's columns plus a leftward
// lane-group scan); dBm/dCm accumulate in registers over the GS channels of a workgroup; a*g of every channel
// waits in LDS between two bands.
//
// A (band, channel) has two barriers:
//   produce   the job's threads form what depends on the position and the channel only (step, step * x, dy), a few cells
//             each, loaded one (band, channel) ahead, and leave it in LDS as fp32;
//   sweep     the lane groups rebuild the states of the band's rows and walk back up.  Bm and Cm of the band stay in
//             registers for all channels (BCR; the widest fp32 tilings read them per row), the checkpoint of the next
//             channel is requested one channel ahead.  Per row and column two sums over the states are needed: of (gradient
//             of the decay) * a * A and of (gradient of u) * B.  A wavefront adds its own states with
//             v_permlane32_swap / v_permlane16_swap, so that one value per column, tensor and WAVEFRONT goes to LDS;
//   finish    the thread that produced a cell adds the wavefronts' parts in a fixed order, applies the factors that
//             depend on the position (ddelta = first sum + x * second sum, dx = step * second sum + Dskip * dy, +0
//             under the mask; softplus: the logistic factor kept from produce) and stores.
// What it replaced had a barrier and 2 NG LDS reads per column in every row: 128x192 fp32 waited 43 % of the time.
// The row-scan states hhor[i,j-1] are not kept from the rebuild to the reverse sweep but formed again there from the
// column states, which are kept anyway (RECOMP): Eq. 6 read backwards, hhor[i,j] = h[i,j] - a[i,j] * h[i-1,j].  The column
// panels keep them: they have registers to spare (the fullest instantiation uses 252 of 256), and beside a column whose state
// has overflowed to infinity the difference is NaN (211x397 bf16 training 2950 us with the difference, 2934 without).
// dA is summed over the lane group once per (band, channel) (DPP) and accumulated by one lane in LDS; dDskip and the bias
// gradient are accumulated by the producing threads and summed per wavefront: all in a fixed order, so results are
// bit-reproducible.
// MP instantiations - column panels (maps wider than LG*K columns, one launch per panel, right to left): p.cb is the
// panel's first column; the row-scan state entering from the left panel (p.hc_in, left by the checkpoint sweeps) starts
// lane 0's rebuilt row recurrence, a*q entering from the right panel (p.qc_in) joins the last lane's reverse recurrence,
// a*q of the panel's first column goes to p.qc_out, and dA / dDskip / the bias gradient add to what the panels to the
// right have left (p.accum).
#pragma once

#include "scan2d_bwd_kernels.hpp"

namespace scan2d {

// Column of a panel -> float index in an LDS row stored chunk-wise: [K/4 chunks][LG][4], then [LG][K%4].
template <int LG, int K>
__device__ __forceinline__ int lds_colk(int c) {
    constexpr int K4 = (K / 4) * 4;
    const int j = c % K, l = c / K;
    return j < K4 ? (j / 4) * (LG * 4) + l * 4 + (j % 4) : (K4 / 4) * (LG * 4) + l * (K - K4) + (j - K4);
}
// The K values of lane l from such a row (128-bit loads, one 64-bit load for K % 4 == 2).
template <int LG, int K>
__device__ __forceinline__ void lds_read_k(const float* row, int l, float* out) {
    static_assert(K % 4 == 0 || K % 4 == 2, "columns per lane: even");
#pragma unroll
    for (int c4 = 0; c4 < K / 4; ++c4) {
        const float4 v = *reinterpret_cast<const float4*>(row + c4 * (LG * 4) + l * 4);
        out[4 * c4] = v.x; out[4 * c4 + 1] = v.y; out[4 * c4 + 2] = v.z; out[4 * c4 + 3] = v.w;
    }
    if constexpr (K % 4 == 2) {
        const float2 v = *reinterpret_cast<const float2*>(row + (K / 4) * (LG * 4) + l * 2);
        out[K - 2] = v.x; out[K - 1] = v.y;
    }
}
template <int LG, int K>
__device__ __forceinline__ void lds_write_k(float* row, int l, const float* v) {
#pragma unroll
    for (int c4 = 0; c4 < K / 4; ++c4)
        *reinterpret_cast<float4*>(row + c4 * (LG * 4) + l * 4) = make_float4(v[4 * c4], v[4 * c4 + 1], v[4 * c4 + 2], v[4 * c4 + 3]);
    if constexpr (K % 4 == 2) *reinterpret_cast<float2*>(row + (K / 4) * (LG * 4) + l * 2) = make_float2(v[K - 2], v[K - 1]);
}

// Sum over the LG lanes of a lane group; the group's last lane holds the total (LG = 16, 32 or 64).
template <int LG>
__device__ __forceinline__ float group_sum_last(float v) {
    asm volatile("s_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 : "+v"(v));
    if constexpr (LG >= 32)
        asm volatile("v_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\ts_nop 1\n\t" : "+v"(v));
    if constexpr (LG == 64)
        asm volatile("v_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\ts_nop 1\n\t" : "+v"(v));
    return v;
}

// Leftward scan of S recurrences over a lane group of any width (see group_scan_left); half-wave groups: inside the two
// DPP rows as for 16-lane groups, then the even row takes the value at the first lane of the odd row.
template <int LG, int S>
__device__ __forceinline__ void group_scan_left_any(float* P, float* Q, float* C) {
    if constexpr (LG == 32) {
        if constexpr (S == 4) {
            asm volatile("s_nop 1\n\t"
                         SCAN2D_S4_STEP(SCAN2D_SHL(1)) SCAN2D_S4_STEP(SCAN2D_SHL(2))
                         SCAN2D_S4_STEP(SCAN2D_SHL(4)) SCAN2D_S4_STEP(SCAN2D_SHL(8))
                         : "+v"(Q[0]), "+v"(Q[1]), "+v"(Q[2]), "+v"(Q[3]), "+v"(P[0]), "+v"(P[1]), "+v"(P[2]), "+v"(P[3]));
        } else if constexpr (S == 1) {
            asm volatile("s_nop 1\n\t"
                         SCAN2D_S1_STEP(SCAN2D_SHL(1)) SCAN2D_S1_STEP(SCAN2D_SHL(2))
                         SCAN2D_S1_STEP(SCAN2D_SHL(4)) SCAN2D_S1_STEP(SCAN2D_SHL(8))
                         : "+v"(Q[0]), "+v"(P[0]));
        } else {
            asm volatile("s_nop 1\n\t"
                         SCAN2D_S2_STEP(SCAN2D_SHL(1)) SCAN2D_S2_STEP(SCAN2D_SHL(2))
                         SCAN2D_S2_STEP(SCAN2D_SHL(4)) SCAN2D_S2_STEP(SCAN2D_SHL(8))
                         : "+v"(Q[0]), "+v"(Q[1]), "+v"(P[0]), "+v"(P[1]));
        }
#pragma unroll
        for (int t = 0; t < S; ++t) {
            float f;
            asm volatile("s_nop 1\n\tv_mov_b32_dpp %0, %1 row_newbcast:0 row_mask:0xf bank_mask:0xf" : "=&v"(f) : "v"(Q[t]));
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(f), __float_as_uint(f), false, false);
            const bool even = (threadIdx.x & 16u) == 0u;
            Q[t] = even ? fmaf(P[t], __uint_as_float(r[1]), Q[t]) : Q[t];
            C[t] = from_right<64>(Q[t]);
            C[t] = (threadIdx.x & 31u) == 31u ? 0.0f : C[t];
        }
    } else {
        group_scan_left<LG, S>(P, Q, C);
    }
}

// Value held by the lane to the right inside the lane group (0 for the group's last lane).
template <int LG>
__device__ __forceinline__ float from_right_any(float v) {
    if constexpr (LG == 32) {
        const float r = from_right<64>(v);
        return (threadIdx.x & 31u) == 31u ? 0.0f : r;
    } else {
        return from_right<LG>(v);
    }
}

// Value held by the lane to the left inside the lane group (0 for the group's first lane).
template <int LG>
__device__ __forceinline__ float from_left_any(float v) {
    float r;
    if constexpr (LG == 16) {
        asm volatile("s_nop 1\n\tv_mov_b32_dpp %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0" : "=&v"(r) : "v"(v));
    } else {
        asm volatile("s_nop 1\n\tv_mov_b32_dpp %0, %1 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0" : "=&v"(r) : "v"(v));
        if constexpr (LG == 32) r = (threadIdx.x & 31u) == 0u ? 0.0f : r;
    }
    return r;
}

template <typename P>
__device__ __forceinline__ P* at_byte(P* base, uint32_t bytes) {
    using B = std::conditional_t<std::is_const_v<P>, const char, char>;
    return reinterpret_cast<P*>(reinterpret_cast<B*>(base) + bytes);      // (through an integer the loads would become flat ones)
}
// lanes 0..31: a summed over the wavefront's halves, lanes 32..63: b
__device__ __forceinline__ float halves_sum(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// even DPP rows: a summed over the row pair, odd rows: b
__device__ __forceinline__ float row_pairs_sum(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The LDS rows of a wavefront's two sums over its states: kTensor floats per tensor, column c = l * K + j at at(c).
// Narrow groups: [j][LG] with the pitch that spreads a reader's consecutive columns over the banks; wave-wide groups:
// chunks of 4 columns per lane.
template <int LG, int K>
struct PartRow {
    static constexpr int kPitch = LG == 64 ? LG : LG + 1;
    static constexpr int kTensor = LG == 64 ? LG * K : kPitch * K + (LG == 16 ? 16 : 0);
    static constexpr int kRow = 2 * kTensor;
    static __device__ __forceinline__ int at(int c) {
        if constexpr (LG == 64) return lds_colk<LG, K>(c);
        else return (c % K) * kPitch + c / K;
    }
    // columns j and j + 1 (j even)
    static __device__ __forceinline__ void put2(float* row, int lane, int j, const float* s1, const float* s2) {
        if constexpr (LG == 32) {
            float* dst = row + (lane >> 5) * kTensor + (lane & 31);
            dst[j * kPitch] = halves_sum(s1[j], s2[j]);
            dst[(j + 1) * kPitch] = halves_sum(s1[j + 1], s2[j + 1]);
        } else {
            float* dst = row + (lane >> 5) * kTensor + ((lane >> 4) & 1) * kPitch + (lane & 15);
            dst[j * kPitch] = row_pairs_sum(halves_sum(s1[j], s2[j]), halves_sum(s1[j + 1], s2[j + 1]));
        }
    }
    static __device__ __forceinline__ void put(float* row, int lane, const float* s1, const float* s2) {
        if constexpr (LG == 64) {
            lds_write_k<LG, K>(row, lane, s1);
            lds_write_k<LG, K>(row + kTensor, lane, s2);
        } else {
#pragma unroll
            for (int j = K - 2; j >= 0; j -= 2) put2(row, lane, j, s1, s2);
        }
    }
};

// Bm and Cm of a band kept in registers: up to 32 of them.  Beyond, two rows at a time, each requested one row ahead
// (128x192 fp32: 1855 us for the sweep when a row requested its own, 1494 us one row ahead).
template <typename T, int K, int NW, int RB>
constexpr bool bwd_bc_in_registers() { return 2 * RB * NW * words_of<T, (K + 3) / 4 * 4>() <= 32; }

// Rows of a band whose decays stay in LDS from the rebuild to the reverse sweep (the others' are formed again).  The
// widest tilings run one wavefront per SIMD and have LDS for two rows beside eight channels; with all four rows there are
// four channels per workgroup and twice the partial sums (128x192 fp32: +160 us in their reduction).  Narrow tilings share
// the LDS with a second workgroup and gain 1 %.
template <int K, int NW>
constexpr int bwd_decay_rows() { return K * NW >= 12 ? 2 : 0; }

// Rows of a band whose row scans run together (the column recurrence alone ties the rows of a map to each other).  A lone
// scan is a chain of dependent lane movements with wait states between them; four of them side by side need none.  Where
// all rows of a band are scanned together their decays also stay in registers from the rebuild to the reverse sweep.  Only
// where that leaves two wavefronts per SIMD, i.e. up to 16 cells per lane (56x56 bf16 with step and gate, 6144 maps: 722
// instructions per band and channel became 631, the sweep 528 -> 501 us).
template <int K, int NW, int RB, bool MP>
constexpr int bwd_rows_per_scan() { return !MP && K * NW * RB <= 16 ? RB : 1; }

// Dynamic LDS layout (floats), TH = workgroup threads, SLOTS = TH / LG, JPW = SLOTS / NG, GS channels:
//   part [RB][WAVES][PartRow::kRow]    the wavefronts' sums over their states of the current (band, channel)
//   pp   [JPW][RB][3][PANEL]           the per-position values of the current (band, channel): step, step * x, dy
//   aL   [ALR][NW*K/4][TH][4]          the decays of the band's first ALR rows in the current channel, each thread its own
//   gaL  [GS][TH][NW*K]               a[i+1,j]*g[i+1,j] of every channel, kept between bands
//   dAL  [GS][SLOTS][NW]              dA of every channel, accumulated over the bands
//   dDL  [GS][WAVES][2]               dDskip and (SP) the bias gradient of every channel per wavefront, likewise
template <int LG, int K, int NW, int NG, int WAVES, int RB>
constexpr size_t bwd_shared_lds_fixed() {                  // floats that do not depend on GS
    constexpr size_t TH = WAVES * 64, JPW = TH / LG / NG;
    return (size_t)RB * WAVES * PartRow<LG, K>::kRow + JPW * RB * 3 * LG * K + (size_t)bwd_decay_rows<K, NW>() * TH * NW * K;
}
template <int LG, int K, int NW, int WAVES>
constexpr size_t bwd_shared_lds_per_channel() { return (size_t)WAVES * 64 * NW * K + (size_t)WAVES * 64 / LG * NW + 2 * WAVES; }

// CF: columns first (v = a * v[i-1,j] + u, then h = a * h[i,j-1] + v).  The checkpoints then hold v, the band
// arrays hold v[i-1,j] (in `hprev`) and h[i,j-1] (in `hhl`), the reverse row scan q runs on dy * Cm alone and the
// reverse column recurrence on its result (gv = q + a[i+1,j] * gv[i+1,j], kept in `ga` as a * gv); the gradient of u
// is gv, that of the decay gv * v[i-1,j] + q * h[i,j-1]: the same instructions in the other order.
// GATE: the backward of the block's output gate y = y_scan * SiLU(z) where the cells are produced: the thread that
// produces a cell also loads z and y_scan there, stores dz = dy * y_scan * s (1 + z (1 - s)), s the logistic function of
// z, and hands dy * SiLU(z), unrounded, to the sweeps in place of dy.
template <typename T, int LG, int K, int NW, int NG, int WAVES, int RB, bool FAST, bool SP, bool CF = false, bool MP = false, bool GATE = false>
__global__ __launch_bounds__(WAVES * 64, WAVES / 4) void scan2d_bwd_shared_kernel(const BwdArgs p) {
    static_assert(!MP || !CF, "column panels: rows first only");
    static_assert(!GATE || SP, "the gate goes with the softplus step");
    constexpr bool RECOMP = !CF && !MP;
    const int cb = MP ? p.cb : 0;                         // first column of this launch's panel
    constexpr int THREADS = WAVES * 64, SLOTS = THREADS / LG, JPW = SLOTS / NG, PANEL = LG * K, TMJ = NG * LG;
    static_assert(SLOTS % NG == 0 && JPW >= 1 && TMJ % 64 == 0, "whole jobs per workgroup, whole wavefronts per job");
    constexpr int WPJ = TMJ / 64;                         // wavefronts of a job
    constexpr int CELLS = RB * PANEL, CT = (CELLS + TMJ - 1) / TMJ;     // cells of a band per producing thread
    using Part = PartRow<LG, K>;
    constexpr int XW = words_of<T, (K + 3) / 4 * 4>();
    static_assert(bwd_decay_rows<K, NW>() == 0 || K % 4 == 0, "decays move in pieces of four");
    constexpr bool BCR = bwd_bc_in_registers<T, K, NW, RB>();
    constexpr int ALR = bwd_decay_rows<K, NW>();
    constexpr int RS = bwd_rows_per_scan<K, NW, RB, MP>();
    constexpr bool AREG = RS == RB;
    static_assert(RB % RS == 0 && (!AREG || ALR == 0), "whole scans per band, decays in one place");
    static_assert(RS == 1 || BCR, "rows scanned together have their Bm and Cm at hand");
    // SP: p.delta is the raw projection.  The softplus is applied where the cells are produced and the chain rule where
    // ddelta is summed, so ddelta receives the gradient of the raw projection directly.
    constexpr int PP_ROW = 3 * PANEL, PP_JOB = RB * PP_ROW;
    extern __shared__ float lds[];
    const int GS = p.GS;
    float* const part = lds;
    float* const pp = part + RB * WAVES * Part::kRow;
    float* const gaL = lds + bwd_shared_lds_fixed<LG, K, NW, NG, WAVES, RB>();
    float* const aL = gaL - ALR * THREADS * NW * K;
    float* const dAL = gaL + (size_t)GS * THREADS * NW * K;
    float* const dDL = dAL + (size_t)GS * SLOTS * NW;

    const int tid = threadIdx.x, slot = tid / LG, l = tid % LG, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int job_slot = wave / WPJ;
    const int sg = slot - job_slot * NG;
    const int tm = tid - job_slot * TMJ;                  // thread index inside the job
    const long long groups = (long long)p.Bt * p.CG * p.S;
    const long long job = (long long)blockIdx.x * JPW + job_slot;
    const bool live = job < groups;
    const int seg = live ? (int)(job % p.S) : 0;          // row segment: bands [band0, band0 + seg_bands), the last one's may lie past H
    const int b = live ? (int)(job / p.S / p.CG) : 0, cg = live ? (int)(job / p.S % p.CG) : 0;
    const int band0 = seg * p.seg_bands;
    const int c_first = cg * GS;
    const int nch = live ? min(GS, p.Dc - c_first) : 0;

    const int H = p.H, W = p.W, N = p.N;
    const size_t HW = (size_t)H * W;
    const int n0 = sg * NW;
    const int col0 = cb + l * K;                         // first column of this lane in the map
    const bool inside = col0 < W;
    const uint32_t lcol = inside ? (uint32_t)col0 : (uint32_t)cb;
    const TailRows<T> tl(p.tail, W);
    const bool lastm = b == p.Bt - 1;
    bool lastB[NW];
#pragma unroll
    for (int s = 0; s < NW; ++s) lastB[s] = lastm && (n0 + s == N - 1);
    const int nv = FAST ? (inside ? K : 0) : max(0, min(K, W - col0));   // cells of this lane inside the map
    const uint8_t* mm = p.mask ? p.mask + (size_t)b * HW : nullptr;
    // Addresses are a wave-uniform base (scalar registers) plus one 32-bit byte offset per lane: as 64-bit pointers per row
    // and tensor the compiler keeps them all in vector registers across the band loop.
    constexpr uint32_t EB = Elem<T>::kBytes;
    const T* const Bb = reinterpret_cast<const T*>(p.Bm) + (size_t)b * N * HW;
    const T* const Cb = reinterpret_cast<const T*>(p.Cm) + (size_t)b * N * HW;
    uint32_t soff[NW];                                    // state plane and column of this lane
#pragma unroll
    for (int s = 0; s < NW; ++s) soff[s] = ((uint32_t)(n0 + s) * (uint32_t)HW + lcol) * EB;
    float* const ppj = pp + job_slot * PP_JOB;
    const float* const partj = part + (size_t)job_slot * WPJ * Part::kRow;

    const uint32_t part_row = p.part_chunked ? (uint32_t)PANEL : (uint32_t)W;      // floats of a row of the partial sums
    const size_t part_job = ((size_t)b * p.CG + cg) * N * H * part_row;
    for (int ch = 0; ch < GS; ++ch) {
        const int seg_rows = p.seg_bands * RB;
        const bool below = seg + 1 < p.S && ch < nch;      // g below the map is 0
        const float* gk = (ch < seg_rows ? p.pB : p.pC) + part_job + (size_t)(seg * seg_rows + ch % seg_rows) * part_row;
#pragma unroll
        for (int s = 0; s < NW; ++s)
#pragma unroll
            for (int j = 0; j < K; ++j)
                gaL[((size_t)ch * THREADS + tid) * (NW * K) + s * K + j] = below && j < nv ? gk[(size_t)(n0 + s) * H * part_row + col0 + j] : 0.0f;
        if (l == LG - 1) {
#pragma unroll
            for (int s = 0; s < NW; ++s) dAL[((size_t)ch * SLOTS + slot) * NW + s] = 0.0f;
        }
        if ((lane & 31) == 31) dDL[(ch * WAVES + wave) * 2 + (lane >> 5)] = 0.0f;
    }
    // gaL entries are private to a thread, dAL entries to the last lane of a lane group, dDL entries to lanes 31 and 63 of
    // a wavefront: no barrier needed for them until the final sums

    // ---- the cells this thread produces: index inside the band -> (row, column), fixed for the whole kernel
    int cell_r[CT], cell_c[CT];
    bool cell_ok[CT];
#pragma unroll
    for (int v = 0; v < CT; ++v) {
        const int id = tm + v * TMJ;
        cell_r[v] = id / PANEL;
        cell_c[v] = id - cell_r[v] * PANEL;
        cell_ok[v] = id < CELLS && live;
        if (!cell_ok[v]) { cell_r[v] = 0; cell_c[v] = 0; }
        cell_ok[v] = cell_ok[v] && cb + cell_c[v] < W;
    }
    // Every access below runs unconditionally, in straight-line code: what does not exist is addressed past the end of its
    // buffer descriptor (loads then return 0, stores are dropped).  With loads and stores in branches the compiler has to
    // wait for ALL outstanding accesses wherever it needs one, the partial sums' stores of the previous band among them
    // (a panel sweep of 211x397 bf16 spent two thirds of its time there).
    constexpr uint32_t kNowhere = 0x80000000u;            // past every descriptor (at most 2^31 - 1 bytes)
    uint32_t rawx[CT], rawd[CT], rawy[CT], rawm[CT], rawz[GATE ? CT : 1], raws[GATE ? CT : 1];
    float ckn[NW][K], An_next[NW];                        // of the next (band, channel): checkpoint, A
    float hcn[MP ? RB : 1][NW], qcn[MP ? RB : 1][NW];     // and the carries from the neighbouring panels (lane 0, last lane; else 0)
    auto map_of = [&](int ch) { return (size_t)b * p.Dc + c_first + min(ch, max(nch - 1, 0)); };
    const uint32_t ck_row = p.ck_chunked ? (uint32_t)PANEL : (uint32_t)W;
    const uint32_t ck_lane = p.ck_chunked ? (uint32_t)l * 16u : lcol * 4u, ck_step = p.ck_chunked ? LG * 16u : 16u;
    const rsrc_t rs_m = make_rsrc(mm, mm != nullptr ? HW : 0);
    // Loads of (band, channel): clamped to a valid element; what lies outside the map is zeroed where the cell is produced.
    auto request = [&](int band, int ch) {
        const size_t map = map_of(ch);
        const T* xm = reinterpret_cast<const T*>(p.x) + map * HW;
        const T* dm = reinterpret_cast<const T*>(p.delta) + map * HW;
        const T* dym = reinterpret_cast<const T*>(p.dy) + map * HW;
        const T* zm = reinterpret_cast<const T*>(p.z) + map * HW;          // GATE only
        const T* ysm = reinterpret_cast<const T*>(p.y_scan) + map * HW;    // GATE only
#pragma unroll
        for (int v = 0; v < CT; ++v) {
            const uint32_t o = (uint32_t)min(band * RB + cell_r[v], H - 1) * (uint32_t)W + (uint32_t)min(cb + cell_c[v], W - 1);
            if constexpr (GATE) { rawz[v] = elem_bits(at_byte(zm, o * EB)); raws[v] = elem_bits(at_byte(ysm, o * EB)); }
            rawx[v] = elem_bits(at_byte(xm, o * EB));
            rawd[v] = elem_bits(at_byte(dm, o * EB));
            rawy[v] = elem_bits(at_byte(dym, o * EB));
        }
        // the checkpoint (band 0 starts from zero and reads what band 1 reads); past the row end: the next row, or what lies
        // behind the checkpoints (workspace: the next region; a caller's buffer: the spare bytes of bwd_saved_bytes)
        const float* ck = p.ck + (map * p.nb + min(max(band, 1), p.nb - 1)) * N * ck_row;
        const float* Am = p.A + (map - (size_t)b * p.Dc) * N;
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            const float* src = at_byte(ck, (uint32_t)(n0 + s) * ck_row * 4u + ck_lane);
#pragma unroll
            for (int j4 = 0; j4 < K / 4; ++j4) load_f32s<4>(at_byte(src, j4 * ck_step), &ckn[s][4 * j4]);
            if constexpr (K % 4 == 2) load_f32s<2>(src + K - 2, &ckn[s][K - 2]);
            An_next[s] = *at_byte(Am, (uint32_t)(n0 + s) * 4u);
        }
        if constexpr (MP) {
            const size_t rows = (size_t)N * H;
            const rsrc_t rh = make_rsrc(p.hc_in + map * rows, p.hc_in != nullptr ? rows * 4 : 0);
            const rsrc_t rq = make_rsrc(p.qc_in + map * rows, p.qc_in != nullptr ? rows * 4 : 0);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const uint32_t o = band * RB + r < H ? ((uint32_t)(n0 + s) * H + band * RB + r) * 4u : kNowhere;
                    hcn[r][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rh, l == 0 ? o : kNowhere, 0, 0));
                    qcn[r][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rq, l == LG - 1 ? o : kNowhere, 0, 0));
                }
        }
    };
    auto widen = [](uint32_t bits, auto tag) -> float {
        using E = decltype(tag);
        if constexpr (Elem<E>::kBytes == 4) return __uint_as_float(bits);
        else return __uint_as_float(bits << 16);
    };
    auto put_elem_at = [&](rsrc_t rs, uint32_t elem, bool ok, float v, auto tag) {      // one element, or nothing
        using E = decltype(tag);
        const uint32_t o = ok ? elem * (uint32_t)Elem<E>::kBytes : kNowhere;
        if constexpr (Elem<E>::kBytes == 4) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, o, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b16((uint16_t)f32_to_bf16_bits(v), rs, o, 0, 0);
    };
    auto put_row = [&](uint32_t* r, const T* rowp, uint32_t off, bool last, const T* tail_row) {
        const T* q = at_byte(rowp, off);
        if constexpr (!FAST) q = last ? tail_row + lcol : q;
        load_words_any<words_of<T, K>()>(q, r);
    };
    // Bm / Cm: of all rows of a band (BCR), or of the row at hand and the one after it
    constexpr int BR = BCR ? RB : 2;                      // rows held: all, or the current and the next one
    uint32_t bB[BR][NW][XW], bC[BR][NW][XW];
    auto load_B = [&](int k, int i) {
#pragma unroll
        for (int s = 0; s < NW; ++s) put_row(bB[k][s], Bb + (size_t)min(i, H - 1) * W, soff[s], lastB[s] && i >= H - 1, tl.B);
    };
    auto load_C = [&](int k, int i) {
#pragma unroll
        for (int s = 0; s < NW; ++s) put_row(bC[k][s], Cb + (size_t)min(i, H - 1) * W, soff[s], lastB[s] && i >= H - 1, tl.C);
    };
    auto load_band = [&](int band) {
        if constexpr (BCR) {
#pragma unroll
            for (int r = 0; r < RB; ++r) { load_B(r, band * RB + r); load_C(r, band * RB + r); }
        } else {
            load_B(0, band * RB);
        }
#pragma unroll
        for (int v = 0; v < CT; ++v)
            rawm[v] = __builtin_amdgcn_raw_buffer_load_b8(rs_m, (uint32_t)min(band * RB + cell_r[v], H - 1) * (uint32_t)W + (uint32_t)min(cb + cell_c[v], W - 1), 0, 0);
    };

    float dBacc[RB][NW][K], dCacc[RB][NW][K];
    // The partial sums of a band over this workgroup's channels (past the last band: nothing).
    const size_t part_bytes = (size_t)N * H * part_row * 4;
    const rsrc_t rs_B = make_rsrc(p.pB + part_job, part_bytes);
    const rsrc_t rs_C = make_rsrc(p.pC + part_job, part_bytes);
    auto store_band = [&](int band) {
        const uint32_t lane_at = p.part_chunked ? (uint32_t)l * 16u : (uint32_t)col0 * 4u, step = p.part_chunked ? LG * 16u : 16u;
        const bool whole = live && (p.part_chunked || nv == K);      // chunked: every lane stores; the reduction drops the columns past W
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = band * RB + r;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const uint32_t o = (((uint32_t)(n0 + s) * H + i) * part_row) * 4u + lane_at;
                const uint32_t ow = whole && i < H ? o : kNowhere;
#pragma unroll
                for (int j = 0; j + 4 <= K; j += 4) {
                    const u32x4_t vB = {__float_as_uint(dBacc[r][s][j]), __float_as_uint(dBacc[r][s][j + 1]), __float_as_uint(dBacc[r][s][j + 2]), __float_as_uint(dBacc[r][s][j + 3])};
                    const u32x4_t vC = {__float_as_uint(dCacc[r][s][j]), __float_as_uint(dCacc[r][s][j + 1]), __float_as_uint(dCacc[r][s][j + 2]), __float_as_uint(dCacc[r][s][j + 3])};
                    __builtin_amdgcn_raw_buffer_store_b128(vB, rs_B, ow, (j / 4) * step, 0);
                    __builtin_amdgcn_raw_buffer_store_b128(vC, rs_C, ow, (j / 4) * step, 0);
                }
                if constexpr (K % 4 == 2) {
                    const u32x2_t vB = {__float_as_uint(dBacc[r][s][K - 2]), __float_as_uint(dBacc[r][s][K - 1])};
                    const u32x2_t vC = {__float_as_uint(dCacc[r][s][K - 2]), __float_as_uint(dCacc[r][s][K - 1])};
                    __builtin_amdgcn_raw_buffer_store_b64(vB, rs_B, ow, (K - 2) * 4, 0);
                    __builtin_amdgcn_raw_buffer_store_b64(vC, rs_C, ow, (K - 2) * 4, 0);
                }
                if constexpr (!FAST) {                     // the lane across the row end
#pragma unroll
                    for (int j = 0; j + 1 < K; ++j) {
                        const uint32_t oe = live && !p.part_chunked && nv < K && j < nv && i < H ? o + 4u * j : kNowhere;
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dBacc[r][s][j]), rs_B, oe, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dCacc[r][s][j]), rs_C, oe, 0, 0);
                    }
                }
            }
        }
    };

    // One (band, channel).
    auto sweep = [&](int band, int ch) {
        const int r0 = band * RB;
        const bool act = ch < nch;
        const size_t map = map_of(ch);                     // idle iterations re-read a valid channel
        const int c = (int)(map - (size_t)b * p.Dc);
        const float dbc = (SP && p.delta_bias != nullptr) ? p.delta_bias[c] : 0.0f;
        float An[NW], Ap[NW], hcv[MP ? RB : 1][NW], qcv[MP ? RB : 1][NW];
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            An[s] = An_next[s];
            Ap[s] = An[s] * kLog2e;
            if constexpr (MP) {
#pragma unroll
                for (int r = 0; r < RB; ++r) { hcv[r][s] = hcn[r][s]; qcv[r][s] = qcn[r][s]; }
            }
        }
        const float dsk = p.Dskip != nullptr ? p.Dskip[c] : 0.0f;

        // ---- produce the per-position values of this (band, channel)
        // dlog (SP): d softplus(t) / dt of the raw projection, the logistic function.  It is kept from here: formed from the step,
        // log(1 + e^t), it would have the absolute error of 1 + e^t (steps around softplus(-4): 3e-5 of the factor against 3e-7).
        float xe[CT], dlog[SP ? CT : 1], dDb = 0.0f, dBb = 0.0f;       // dBb (SP): sum of the ddelta_raw this thread stores
#pragma unroll
        for (int v = 0; v < CT; ++v) {
            const bool in = cell_ok[v] && act && r0 + cell_r[v] < H;
            const bool m = rawm[v] != 0u;
            float dl = widen(rawd[v], T{});
            if constexpr (SP) { dlog[v] = logistic_f32(dl + dbc); dl = softplus_f32(dl + dbc); }
            dl = in ? dl : 0.0f;
            xe[v] = (in && !m) ? widen(rawx[v], T{}) : 0.0f;         // select: nothing under the mask leaks
            float dyv = in ? widen(rawy[v], T{}) : 0.0f;
            if constexpr (GATE) {
                const float zv = widen(rawz[v], T{}), sgm = logistic_f32(zv);
                put_elem_at(make_rsrc(reinterpret_cast<T*>(p.dz) + map * HW, HW * EB), (uint32_t)(r0 + cell_r[v]) * (uint32_t)W + (uint32_t)(cb + cell_c[v]), in,
                            dyv * widen(raws[v], T{}) * (sgm * fmaf(zv, 1.0f - sgm, 1.0f)), T{});
                dyv = in ? dyv * (zv * sgm) : 0.0f;
            }
            if (v + 1 < CT || CELLS % TMJ == 0 || tm + v * TMJ < CELLS) {
                float* row = ppj + cell_r[v] * PP_ROW + lds_colk<LG, K>(cell_c[v]);
                row[0] = dl;
                row[PANEL] = dl * xe[v];
                row[2 * PANEL] = dyv;
            }
            dDb = fmaf(dyv, xe[v], dDb);
        }
        float hcur[NW][K];                                 // the band's checkpoint
#pragma unroll
        for (int s = 0; s < NW; ++s)
#pragma unroll
            for (int j = 0; j < K; ++j) hcur[s][j] = band > 0 && j < nv ? ckn[s][j] : 0.0f;
        request(ch + 1 < GS ? band : max(band - 1, 0), ch + 1 < GS ? ch + 1 : 0);      // of the next (band, channel)
        __syncthreads();
        if constexpr (BCR && EB == 2) {                    // keep them packed: the compiler would widen them once, outside the channel loop
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int s = 0; s < NW; ++s)
#pragma unroll
                    for (int w = 0; w < XW; ++w) asm volatile("" : "+v"(bB[r][s][w]), "+v"(bC[r][s][w]));
        }

        // ---- scans 1 and 2: rebuild h[i-1,j] (CF: v[i-1,j] and h[i,j-1]) for the rows of the band.  Rows past H have step 0
        // and x 0: they change nothing.  A row recurrence runs twice over the lane's columns: first for the lane's own
        // (decay product, state) pair that the lanes scan, then from the state that enters the lane - as many
        // multiply-adds as adding the carry to stored partial results, without the arrays that hold them
        float hprev[RB][NW][K], hhl[RECOMP ? 1 : RB][NW][K];
        float ak[AREG ? RB : 1][NW][K], Prow[RB][NW];      // decays (AREG) and per lane their product over its columns
        // Rows scanned one by one (AHEAD): the next row's values are read from LDS in front of the current row's work.  One
        // wavefront per SIMD has nothing else to put beside that latency, eight times per band and channel.  Columns first (ONCE) has
        // no registers for that: every row's values are read in one place, and scan 4 runs on q itself (16 items of 96 channels of
        // 21x146 bf16: 844 us the other way, and 800 bytes of scratch per lane; 599).
        constexpr bool ONCE = CF && RS == 1, AHEAD = RS == 1 && !ONCE;
        float dlq[AHEAD ? 2 : 1][K], dxq[AHEAD ? 2 : 1][K];
        if constexpr (AHEAD) {
            lds_read_k<LG, K>(ppj, l, dlq[0]);
            lds_read_k<LG, K>(ppj + PANEL, l, dxq[0]);
        }
#pragma unroll
        for (int rb = 0; rb < RB; rb += RS) {
            float a[RS][NW][K], u[RS][NW][K], P[RS * NW], Hh[RS * NW], cin[RS * NW];
#pragma unroll
            for (int r = rb; r < rb + RS; ++r) {
                if constexpr (!BCR) {                      // row 0 is there: from the band's first request, then from the row sweep
                    if (r + 1 < RB) load_B((r + 1) % BR, r0 + r + 1);
                    else load_C(r % BR, r0 + r);
                }
                float (&dl)[K] = dlq[AHEAD ? r % 2 : 0], (&dxe)[K] = dxq[AHEAD ? r % 2 : 0];
                const int rr = AHEAD ? r + 1 : r;          // the row read here
                if (rr < RB) {
                    lds_read_k<LG, K>(ppj + rr * PP_ROW, l, dlq[AHEAD ? rr % 2 : 0]);
                    lds_read_k<LG, K>(ppj + rr * PP_ROW + PANEL, l, dxq[AHEAD ? rr % 2 : 0]);
                    if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const uint32_t* Br = bB[r % BR][s];
                    const int q = (r - rb) * NW + s;
                    float (&ar)[K] = a[r - rb][s], (&ur)[K] = u[r - rb][s];
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        ar[j] = __builtin_amdgcn_exp2f(dl[j] * Ap[s]);
                        if (r < ALR && j % 4 == 3) *reinterpret_cast<float4*>(aL + ((r * NW * K + s * K + j - 3) / 4 * THREADS + tid) * 4) = make_float4(ar[j - 3], ar[j - 2], ar[j - 1], ar[j]);
                        if constexpr (AREG) ak[r][s][j] = ar[j];
                        ur[j] = dxe[j] * get_elem<T, K>(Br, j);
                        if constexpr (CF) {
                            hprev[r][s][j] = hcur[s][j];                               // v[i-1,j]
                            ur[j] = hcur[s][j] = fmaf(ar[j], hcur[s][j], ur[j]);
                        }
                        P[q] = j == 0 ? ar[0] : P[q] * ar[j];
                        Hh[q] = j == 0 ? ur[0] : fmaf(ar[j], Hh[q], ur[j]);
                    }
                    Prow[r][s] = P[q];
                    if constexpr (MP) Hh[q] = fmaf(P[q], hcv[r][s], Hh[q]);            // state entering from the panel to the left
                }
            }
            group_scan<LG, RS * NW>(P, Hh, cin);
#pragma unroll
            for (int r = rb; r < rb + RS; ++r) {
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const float (&ar)[K] = a[r - rb][s], (&ur)[K] = u[r - rb][s];
                    float left = cin[(r - rb) * NW + s];   // hhor[i, j-1] (CF: h[i, j-1])
                    if constexpr (MP) left += hcv[r][s];   // one of them is 0
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        if constexpr (!RECOMP) hhl[r][s][j] = left;
                        if (!CF || j + 1 < K) left = fmaf(ar[j], left, ur[j]);
                        if constexpr (!CF) {
                            hprev[r][s][j] = hcur[s][j];
                            hcur[s][j] = fmaf(ar[j], hcur[s][j], left);
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);             // steps stay apart: merged, their temporaries would not fit the registers
        }

        // the compiler would keep step, step * x and the decays of all rows from here to the reverse sweep (3 RB NW K registers)
        asm volatile("" ::: "memory");
        // ---- scans 3 and 4, bottom row of the band first
        float ga[NW][K], dAb[NW];
        const int rows = H - r0;                           // of this band inside the map
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            dAb[s] = 0.0f;
#pragma unroll
            for (int j = 0; j < K; ++j) ga[s][j] = gaL[((size_t)ch * THREADS + tid) * (NW * K) + s * K + j];
        }
        // what a row's first half needs (AHEAD: read one row ahead): dy and, where the decays are formed again, the step
        float dln[K], dyn[K], dxn[K];                      // dxn (ONCE): step * x
        const auto first_half = [&](int r) {
            if constexpr (!AREG) {
                if (r >= ALR || ONCE) lds_read_k<LG, K>(ppj + r * PP_ROW, l, dln);
            }
            lds_read_k<LG, K>(ppj + r * PP_ROW + 2 * PANEL, l, dyn);
            if constexpr (ONCE) lds_read_k<LG, K>(ppj + r * PP_ROW + PANEL, l, dxn);
        };
        if constexpr (AHEAD) first_half(RB - 1);
#pragma unroll
        for (int rt = RB - 1; rt >= 0; rt -= RS) {         // RS rows per scan, the topmost rt - RS + 1
            float edge[NW];                                // ONCE: the decay of the lane to the right
            float a[RS][NW][K], g[RS][NW][K], gr[RS][NW][K], P[RS * NW], Q[RS * NW], qin[RS * NW];     // gr: a * g (CF: of this row's q)
#pragma unroll
            for (int d = 0; d < RS; ++d) {
                const int r = rt - d;
                if constexpr (!BCR) {
                    if (r > 0) { load_B((r - 1) % BR, r0 + r - 1); load_C((r - 1) % BR, r0 + r - 1); }
                }
                const float* prow = ppj + r * PP_ROW;
                float dxr[K];
                if constexpr (!AHEAD) first_half(r);
                if constexpr (CF && !ONCE) lds_read_k<LG, K>(prow + PANEL, l, dxr);
                const float (&dxe)[K] = ONCE ? dxn : dxr;
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const uint32_t* Cr = bC[r % BR][s];
                    float (&ar)[K] = a[d][s];
                    if (r < ALR) {
#pragma unroll
                        for (int j = 0; j < K; j += 4) {
                            const float4 v = *reinterpret_cast<const float4*>(aL + ((r * NW * K + s * K + j) / 4 * THREADS + tid) * 4);
                            ar[j] = v.x; ar[j + 1] = v.y; ar[j + 2] = v.z; ar[j + 3] = v.w;
                        }
                    }
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        if constexpr (AREG) ar[j] = ak[r][s][j];
                        else if (r >= ALR) ar[j] = __builtin_amdgcn_exp2f(dln[j] * Ap[s]);
                        float hv;
                        if constexpr (CF) {            // v[i,j], then h[i,j]
                            hv = fmaf(ar[j], hprev[r][s][j], dxe[j] * get_elem<T, K>(bB[r % BR][s], j));
                            hv = fmaf(ar[j], hhl[r][s][j], hv);
                        } else {                       // h[i,j] is what the row below started from
                            hv = r == RB - 1 ? hcur[s][j] : hprev[r + 1 < RB ? r + 1 : r][s][j];
                        }
                        dCacc[r][s][j] = fmaf(dyn[j], hv, dCacc[r][s][j]);
                        const float Cv = get_elem<T, K>(Cr, j);
                        if constexpr (CF) {
                            g[d][s][j] = dyn[j] * Cv;
                        } else {
                            g[d][s][j] = fmaf(dyn[j], Cv, ga[s][j]);                                // scan 3
                            ga[s][j] = ar[j] * g[d][s][j];
                        }
                        if constexpr (!ONCE) gr[d][s][j] = CF ? ar[j] * g[d][s][j] : ga[s][j];
                    }
                    // scan 4: q[j] = g[j] + a[j+1] * q[j+1], run on aq[j] = a[j] * q[j] = a[j] * g[j] + a[j] * aq[j+1]: a * g is
                    // there, and the lane's decay product is the one of the rebuild
                    const int k = d * NW + s;
                    if constexpr (ONCE) {
                        P[k] = edge[s] = from_right_any<LG>(ar[0]);
                        Q[k] = g[d][s][K - 1];
#pragma unroll
                        for (int j = K - 2; j >= 0; --j) {
                            Q[k] = fmaf(ar[j + 1], Q[k], g[d][s][j]);
                            P[k] *= ar[j + 1];
                        }
                        continue;
                    }
                    P[k] = Prow[r][s];
                    Q[k] = MP ? fmaf(ar[K - 1], qcv[r][s], gr[d][s][K - 1]) : gr[d][s][K - 1];      // MP: a*q entering from the right panel (last lane)
#pragma unroll
                    for (int j = K - 2; j >= 0; --j) Q[k] = fmaf(ar[j], Q[k], gr[d][s][j]);
                }
            }
            if constexpr (AHEAD) {
                if (rt > 0) first_half(rt - 1);
            }
            group_scan_left_any<LG, RS * NW>(P, Q, qin);
#pragma unroll
            for (int d = 0; d < RS; ++d) {
                const int r = rt - d;
                float dlr[K], dxr[K], s1[K], s2[K];
                if constexpr (!ONCE) {
                    lds_read_k<LG, K>(ppj + r * PP_ROW, l, dlr);
                    lds_read_k<LG, K>(ppj + r * PP_ROW + PANEL, l, dxr);
                }
                const float (&dl)[K] = ONCE ? dln : dlr, (&dxe)[K] = ONCE ? dxn : dxr;
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const float (&ar)[K] = a[d][s];
                    float aq = qin[d * NW + s], qr = aq, first = 0.0f;     // qr (ONCE): q to the right; first: hhor[i,j-1] of the lane's first column
                    if constexpr (MP) aq += qcv[r][s];             // one of them is 0
                    const auto hh = [&](int j) {                   // hhor[i,j]
                        const float hv = r == RB - 1 ? hcur[s][j] : hprev[r + 1 < RB ? r + 1 : r][s][j];
                        return fmaf(-ar[j], hprev[r][s][j], hv);
                    };
                    if constexpr (RECOMP) first = from_left_any<LG>(hh(K - 1));
#pragma unroll
                    for (int j = K - 1; j >= 0; --j) {
                        float q;
                        if constexpr (ONCE) {
                            q = qr = fmaf(j == K - 1 ? edge[s] : ar[j + 1], qr, g[d][s][j]);
                            aq = ar[j] * q;
                        } else {
                            q = g[d][s][j] + aq;
                            aq = CF ? ar[j] * q : fmaf(ar[j], aq, gr[d][s][j]);
                        }
                        if constexpr (MP) {
                            if (j == 0) put_elem_at(make_rsrc(p.qc_out + map * N * H, p.qc_out != nullptr ? (size_t)N * H * 4 : 0), (uint32_t)(n0 + s) * H + r0 + r,
                                                    l == 0 && act && r0 + r < H, aq, float{});
                        }
                        float left;                                // hhor[i,j-1] (CF: h[i,j-1])
                        if constexpr (RECOMP) left = j == 0 ? first : hh(j - 1);
                        else left = hhl[r][s][j];
                        float du = q, gv = CF ? 0.0f : gr[d][s][j];     // gradient of u; gv: a * (what the column recurrence adds)
                        if constexpr (CF) {
                            du = q + ga[s][j];
                            gv = ga[s][j] = ar[j] * du;
                        }
                        const float t = fmaf(aq, left, gv * hprev[r][s][j]);       // gradient of the decay, times the decay
                        dAb[s] = fmaf(t, dl[j], dAb[s]);
                        s1[j] = s == 0 ? t * An[s] : fmaf(t, An[s], s1[j]);
                        const float Bv = get_elem<T, K>(bB[r % BR][s], j);
                        s2[j] = s == 0 ? du * Bv : fmaf(du, Bv, s2[j]);
                        dBacc[r][s][j] = fmaf(du, dxe[j], dBacc[r][s][j]);
                    }
                }
                Part::put(part + (size_t)(r * WAVES + wave) * Part::kRow, lane, s1, s2);
                // rows past H come first and add nothing to dA (0 * infinity would be NaN)
#pragma unroll
                for (int s = 0; s < NW; ++s) dAb[s] = r < rows ? dAb[s] : 0.0f;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = 0; s < NW; ++s) {
#pragma unroll
            for (int j = 0; j < K; ++j) gaL[((size_t)ch * THREADS + tid) * (NW * K) + s * K + j] = ga[s][j];
            const float tot = group_sum_last<LG>(inside ? dAb[s] : 0.0f);
            if (l == LG - 1) dAL[((size_t)ch * SLOTS + slot) * NW + s] += tot;
        }
        __syncthreads();

        // ---- finish: the sums over the states of this thread's cells
#pragma unroll
        for (int v = 0; v < CT; ++v) {
            const bool in = cell_ok[v] && act && r0 + cell_r[v] < H;
            const float* src = partj + (size_t)cell_r[v] * WAVES * Part::kRow + Part::at(cell_c[v]);
            float sA = src[0], sB = src[Part::kTensor];
#pragma unroll
            for (int w = 1; w < WPJ; ++w) { sA += src[w * Part::kRow]; sB += src[w * Part::kRow + Part::kTensor]; }
            const float* cell = ppj + cell_r[v] * PP_ROW + lds_colk<LG, K>(cell_c[v]);     // written by this thread
            const float dl = cell[0], dyv = cell[2 * PANEL];
            const uint32_t o = (uint32_t)(r0 + cell_r[v]) * (uint32_t)W + (uint32_t)(cb + cell_c[v]);
            float dd = fmaf(xe[v], sB, sA);
            if constexpr (SP) { dd = in ? dd * dlog[v] : 0.0f; dBb += dd; }
            put_elem_at(make_rsrc(reinterpret_cast<T*>(p.ddelta) + map * HW, HW * EB), o, in, dd, T{});
            // skip term; exactly +0 under the mask
            put_elem_at(make_rsrc(reinterpret_cast<T*>(p.dx) + map * HW, HW * EB), o, in, rawm[v] != 0u ? 0.0f : fmaf(dsk, dyv, dl * sB), T{});
        }
        {
            const float tot = group_sum_last<32>(halves_sum(dDb, dBb));   // lane 31: dDskip, lane 63: the bias gradient
            if ((lane & 31) == 31) dDL[(ch * WAVES + wave) * 2 + (lane >> 5)] += tot;
        }
    };

    request(band0 + p.seg_bands - 1, 0);
    load_band(band0 + p.seg_bands - 1);
    for (int k = p.seg_bands - 1; k >= 0; --k) {
        const int band = band0 + k;
        store_band(k + 1 < p.seg_bands ? band + 1 : p.nb); // of the band below (first: rows past H, nothing is stored)
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int s = 0; s < NW; ++s)
#pragma unroll
                for (int j = 0; j < K; ++j) { dBacc[r][s][j] = 0.0f; dCacc[r][s][j] = 0.0f; }
        // The first channel is a copy of its own: behind it are a known number of accesses, which lets its waits leave the
        // stores above in flight.  (One channel per workgroup: there is no other.)
        sweep(band, 0);
        for (int ch = 1; ch < GS; ++ch) sweep(band, ch);
        load_band(max(band - 1, 0));
    }
    store_band(band0);

    // dA[b,c,n]: already summed over the lane group; dDskip[b,c] and the bias gradient: the sums over the job's wavefronts,
    // in index order
    __syncthreads();
    if (l == LG - 1) {
        for (int ch = 0; ch < nch; ++ch) {
#pragma unroll
            for (int s = 0; s < NW; ++s)
            {
                float* dst = p.pA + ((size_t)b * p.Dc + c_first + ch) * p.sum_map + seg * p.sum_seg + n0 + s;
                const float v = dAL[((size_t)ch * SLOTS + slot) * NW + s];
                *dst = (MP && p.accum) ? *dst + v : v;             // panels are launched one after the other
            }
        }
    }
    if (tm < 2) {
        float* const base = tm == 0 ? p.pD : (SP ? p.pBias : nullptr);
        if (base != nullptr) {
            for (int ch = 0; ch < nch; ++ch) {
                float acc = 0.0f;
                for (int w = 0; w < WPJ; ++w) acc += dDL[(ch * WAVES + job_slot * WPJ + w) * 2 + tm];
                float* dst = base + ((size_t)b * p.Dc + c_first + ch) * p.sum_map1 + seg * p.sum_seg;
                *dst = (MP && p.accum) ? *dst + acc : acc;
            }
        }
    }
}

}  // namespace scan2d
