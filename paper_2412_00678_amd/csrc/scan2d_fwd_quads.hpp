// Forward 2D selective scan for many maps (2DMamba Eq. 3, Eq. 5, Eq. 6, y = C h + D x): eight channels of one batch item per
// workgroup, states and channels along the lanes, columns along the time.
//
// The forms with columns along the lanes (scan2d_fwd.hpp, scan2d_fwd_shared.hpp) pay for the row recurrence with a scan across the
// lanes (decay products, log-step lane movements, a carry multiply-add) and widen Bm and Cm for every map.  Here a lane walks the
// columns of its block one after the other, so that Eq. 5 is one multiply-add like Eq. 6:
//   * lane = channel (bits 0-1) x state group (bits 2-3, four states each, N = 16) x column block (bits 4-5); a block is K
//     consecutive columns and the column state h of its columns and states stays in K * 4 registers;
//   * block g works on row t - g at step t: the row state at its first column is what block g - 1 ended with one step ago and comes
//     through LDS, one 16-byte word per lane, between wavefronts too (one barrier per step);
//   * Bm and Cm of a position belong to all channels: each lane of a quad holds a quarter of the block's columns, widened, and the
//     other three read them with a quad broadcast (DPP) inside the multiply and the multiply-add; of the two quads of channels in a
//     workgroup one fetches Bm and one Cm, a step ahead, and they exchange them through LDS;
//   * what depends on the position and the channel only (widening, softplus, mask, step * x, skip, gate) is done once, for the four
//     rows that a block passes in four steps, two columns per lane with neighbouring columns in neighbouring lanes; the products go to
//     LDS (private to the wavefront), the sums over the states come back in their place, and the lane that prepared a pair also
//     stores its results.
// Per (position, channel, state): two multiplies, an exponential and three multiply-adds, and 2.3 to 3.3 instructions of everything else
// (6144 maps of 56x56 bf16: 9.3, where the shared-producer form needs 14.5).
// What bounds it: with three wavefronts per SIMD vector issue (56x56 bf16 134 -> 111 us, the vector ALU at 78 % of the time; 28x28 67 ->
// 38); in fp32 and with the gate the L2, which holds the lines that a block has begun until its neighbours have passed (56x56 bf16 gated
// 161 -> 150; streaming hints on the stores make that 166, on the loads too 190); with one wavefront per SIMD the chain of a step, LDS,
// seven columns one after the other and the barrier: 0.9 us where the instructions take 0.45.  x, the step and z by
// elements instead of pairs: 6 % more; a first form in which every quad fetched Bm and Cm for itself, by unaligned loads: 215 us.
// The backward pass's checkpoints do not come from here: a block's 28-byte pieces of their rows took longer to write than the
// shared-producer form takes for all (saving forward of 56x56 bf16 297 us against 210), and in an order of this kernel's own
// (185 us) the main sweep lost 20 to 37 us on gathering them.
//
// Blocks are K or K - 1 columns wide, the narrow ones first, so that K columns from a block's first are always inside the row and no
// access is guarded; the last of a narrow block's K columns is its right neighbour's: its results are dropped.  Rows above and below
// the map (a block waits for its first row, or has passed the last) run on the nearest row's values: above, the column state is
// cleared after each such step; below, nothing is stored.
#pragma once

#include "scan2d_fwd.hpp"

namespace scan2d {

// the value that lane `l` (0..3, known at compile time once unrolled) of each quad of lanes holds
__device__ __forceinline__ float quad_bcast(float v, int l) {
    const int b = __float_as_int(v);
    int r;
    switch (l) {
        case 0: r = __builtin_amdgcn_mov_dpp(b, 0x00, 0xf, 0xf, true); break;
        case 1: r = __builtin_amdgcn_mov_dpp(b, 0x55, 0xf, 0xf, true); break;
        case 2: r = __builtin_amdgcn_mov_dpp(b, 0xaa, 0xf, 0xf, true); break;
        default: r = __builtin_amdgcn_mov_dpp(b, 0xff, 0xf, 0xf, true); break;
    }
    return __int_as_float(r);
}
// sum over four states of cv[s] (held by lane `l` of each quad) * h[s], plus the same sum of the lane eight further round the row of 16.
// The compiler folds a lane movement into a multiplication but not into a multiply-add.  The leading wait states stand for the
// instructions that may have written cv[] just before, which a DPP source must not follow closer.
#define SCAN2D_QUAD_DOT(Q)                                                                              \
    asm("s_nop 1\n\tv_mul_f32_dpp %0, %1, %5 quad_perm:" Q " row_mask:0xf bank_mask:0xf\n\t"            \
        "v_fmac_f32_dpp %0, %2, %6 quad_perm:" Q " row_mask:0xf bank_mask:0xf\n\t"                      \
        "v_fmac_f32_dpp %0, %3, %7 quad_perm:" Q " row_mask:0xf bank_mask:0xf\n\t"                      \
        "v_fmac_f32_dpp %0, %4, %8 quad_perm:" Q " row_mask:0xf bank_mask:0xf\n\t"                      \
        "s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf"                      \
        : "=&v"(y) : "v"(c0), "v"(c1), "v"(c2), "v"(c3), "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]))
__device__ __forceinline__ float quad_dot(float c0, float c1, float c2, float c3, const float* h, int l) {
    float y;
    switch (l) {
        case 0: SCAN2D_QUAD_DOT("[0,0,0,0]"); break;
        case 1: SCAN2D_QUAD_DOT("[1,1,1,1]"); break;
        case 2: SCAN2D_QUAD_DOT("[2,2,2,2]"); break;
        default: SCAN2D_QUAD_DOT("[3,3,3,3]"); break;
    }
    return y;
}
// Orders the LDS accesses of a wavefront's lanes among each other (no instruction: a wavefront's LDS accesses run in order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of a wavefront (floats): [4 rows][(K+1)/2 pairs of columns][16 (block, channel)] x (step, step * x) of both columns, replaced
// by the sums over half of the state groups (both columns of one half, both of the other); 4 floats more per pair and 16 per row keep
// neighbouring columns and rows in different banks.  Of two wavefronts with the same columns: [quad_sets steps][Bm, Cm]
// [ceil(K/4) columns][64 lanes] x 4 states.  Of a quad of channels:
// [2 steps] the row states at the blocks' right edges, a word per lane, one zero block in front.
constexpr int kQuadPair = 68;
template <int K> constexpr int quad_row() { return (K + 1) / 2 * kQuadPair + 16; }
template <int K> constexpr int quad_bc() { return (K + 3) / 4 * 256; }
// Steps of Bm and Cm in LDS: three where a step's are read into registers one step ahead.  From 13 columns on there are no registers
// for that, and with two a compute unit holds four workgroups of two wavefronts instead of three.
template <int K> constexpr bool quad_bc_ahead() { return K <= 12; }
template <int K> constexpr int quad_sets() { return quad_bc_ahead<K>() ? 3 : 2; }
constexpr int quad_carry(int cols) { return cols * 64 + 16; }
template <int K> constexpr size_t quad_lds_bytes(int cols) {
    return ((size_t)2 * 8 * quad_carry(cols) + (size_t)cols * (2 * 4 * quad_row<K>() + 2 * quad_sets<K>() * quad_bc<K>())) * sizeof(float);
}

// wavefronts per SIMD that the registers leave room for.  One instantiation does not fit: 16 columns, bf16, with the step and the gate, spills five
// registers (24 bytes of scratch per lane); it is still the faster one where it is chosen (8192 maps of 64x64: 213 us, K = 8 on two columns of
// wavefronts 228, the other forms 242).
template <int K> constexpr int quad_waves() { return K <= 4 ? 4 : (K <= 8 ? 3 : 2); }

// GATE: as in scan2d_fwd_shared.hpp.
template <typename T, int K, bool SP, bool GATE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(quad_waves<K>()))) void scan2d_fwd_quads_kernel(const FwdArgs p) {
    constexpr int N = 16, NS = 4;                          // states, states per lane
    constexpr int KQ = (K + 3) / 4;                        // columns of Bm and Cm that a lane of a quad holds
    constexpr uint32_t EB = (uint32_t)Elem<T>::kBytes;
    constexpr int BW = EB == 4 ? KQ : (KQ + 2) / 2;        // dwords that hold them, bf16 from the dword boundary below
    constexpr int PR = quad_row<K>(), BC = quad_bc<K>();
    constexpr int K2 = (K + 1) / 2;
    constexpr int SLOTS = K <= 8 ? 16 : 32, NI = SLOTS / 4;                     // pairs of columns that a lane prepares per batch
    constexpr int RV = SLOTS / 16;                                              // ... and the different rows among them
    constexpr int PW = 2;                                                       // dwords per pair (bf16: from the dword boundary below)
    constexpr bool AHEAD = K < 6 || (!GATE && K <= 8);     // a row's values read from LDS one step ahead, and Bm and Cm, where
    constexpr bool BC_AHEAD = quad_bc_ahead<K>();          // there are registers for them
    constexpr int SETS = quad_sets<K>();

    // consecutive workgroups go to the eight XCDs in turn: each XCD takes a contiguous range, so that the channels of a batch item
    // find its Bm and Cm in one L2
    const int wg = (int)(blockIdx.x & 7u) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    if (wg >= p.quad_wgs) return;                            // uniform over the workgroup
    const int b = wg / p.quad_groups;

    extern __shared__ float smem[];
    const int cols = p.quad_cols;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wc = wave >> 1, quad = wave & 1;             // place along the columns; quad of channels, and which of Bm, Cm it fetches
    const int c0 = (wg - b * p.quad_groups) * 8 + quad * 4;        // may be past the last channel (Dc % 8 <= 4): nothing is stored then
    const int lane = threadIdx.x & 63;
    const int ch = lane & 3, sg = (lane >> 2) & 3, blk = lane >> 4;
    const int cstride = quad_carry(cols);
    float4* const carry = reinterpret_cast<float4*>(smem) + quad * 2 * cstride;                 // [2][cols * 64 + 16]
    float4* const bc = reinterpret_cast<float4*>(smem + 16 * cstride + wc * 2 * SETS * BC);     // [SETS][2][KQ][64]
    float* const pp = smem + 16 * cstride + cols * 2 * SETS * BC + wave * 4 * PR;

    const int H = p.H, W = p.W;
    const size_t HW = (size_t)H * W;
    const int narrow = 4 * cols * K - W;                   // the first `narrow` blocks have K - 1 columns
    const int g = wc * 4 + blk;
    const int col0 = g * K - min(g, narrow);
    const bool full = g >= narrow;
    const int c = min(c0 + ch, p.Dc - 1);

    // the quad's first map, from the dword boundary below
    const size_t cb = ((size_t)b * p.Dc + min(c0, p.Dc - 1)) * HW * EB, base = cb & ~(size_t)3, left = (((size_t)p.maps * HW * EB + 3) & ~(size_t)3) - base;
    const uint32_t odd = (uint32_t)(cb - base);
    const rsrc_t rsx = make_rsrc(static_cast<const unsigned char*>(p.x) + base, left),
                 rsd = make_rsrc(static_cast<const unsigned char*>(p.delta) + base, left),
                 rsz = make_rsrc(static_cast<const unsigned char*>(GATE ? p.z : p.x) + base, left);
    const rsrc_t rsy = make_rsrc(static_cast<unsigned char*>(p.y) + base, left),
                 rsg = make_rsrc(static_cast<unsigned char*>(GATE ? p.y_gated : p.y) + base, left);
    const size_t bs = (size_t)b * N * HW * EB, sleft = (((size_t)p.maps / p.Dc - b) * N * HW * EB + 3) & ~(size_t)3;
    const rsrc_t rss = make_rsrc(static_cast<const unsigned char*>(quad == 0 ? p.Bm : p.Cm) + bs, sleft);
    const bool has_mask = p.mask != nullptr, want_y = !GATE || p.y != nullptr;
    const rsrc_t rsm = make_rsrc(p.mask + (has_mask ? (size_t)b * HW : 0), HW);

    float Ap[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) Ap[s] = p.A[(size_t)c * N + sg * NS + s] * kLog2e;
    const auto row_of = [&](int i) { return (uint32_t)min(max(i, 0), H - 1); };

    // ---- the pairs of columns that this lane prepares in a batch of four steps, one batch ahead: pair e is the wavefront's pair
    // `slot`, in step irow[e % RV] of the batch, of channel e_ch(e)
    const int slot = min(lane & (SLOTS - 1), 4 * K2 - 1), iblk = slot / K2, ij = (slot - iblk * K2) * 2, ig = wc * 4 + iblk;
    const int icol = ig * K - min(ig, narrow) + ij;
    const int iend = (lane & (SLOTS - 1)) < 4 * K2 ? (ig < narrow ? K - 1 : K) - ij : 0;     // how many of the two are the block's
    constexpr int RPI = 64 / SLOTS;                        // rows per pair index
    const auto e_ch = [](int e) { return e * RPI / 4; };
    const auto e_plane = [&](int e) { return (uint32_t)(min(c0 + e_ch(e), p.Dc - 1) - min(c0, p.Dc - 1)) * (uint32_t)HW * EB; };
    // neighbouring lanes take the blocks of one map row, which are in different steps of the batch: the four rows of a batch are seven
    // runs of neighbouring columns instead of sixteen (a sixth fewer cache accesses in all, bf16)
    int irow[RV];
    float* icell[RV];
#pragma unroll
    for (int v = 0; v < RV; ++v) {
        irow[v] = (v * RPI + lane / SLOTS + iblk) & 3;
        icell[v] = pp + irow[v] * PR + ij / 2 * kQuadPair + iblk * 16;
    }
    // bf16, whole blocks of even width: every pair is a dword in memory (6144 maps of 64x64, gated, two 16-bit stores 182 us, one dword 173)
    const bool dwords = EB == 2 && K % 2 == 0 && narrow == 0;
    float dsk[4], dbias[4];                                // uniform
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int ck = min(c0 + k, p.Dc - 1);
        const auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
        dsk[k] = uniform(p.Dskip != nullptr ? p.Dskip[ck] : 0.0f);
        dbias[k] = uniform(SP && p.delta_bias != nullptr ? p.delta_bias[ck] : 0.0f);
    }
    const auto cell_of = [&](int batch, int v) { return row_of(4 * batch + irow[v] - iblk) * (uint32_t)W + (uint32_t)icol; };
    // bf16: the two dwords from the boundary below the pair, the pair itself by a shift of 0 or 16 bits (a shift count is taken modulo
    // 32); where channels begin on odd boundaries the low bits differ from channel to channel
    const auto load = [&](rsrc_t rs, uint32_t cell, int e, uint32_t* r) {
        if constexpr (EB == 4) buffer_load_words<PW>(rs, cell * 4u + odd, e_plane(e), r);
        else buffer_load_words<PW>(rs, (cell * 2u + odd + e_plane(e)) & ~3u, 0u, r);
    };
    const auto widen = [&](const uint32_t* r, uint32_t cell, int e, float* v) {
        if constexpr (EB == 4) { v[0] = __uint_as_float(r[0]); v[1] = __uint_as_float(r[1]); }
        else {
            const uint32_t w = __builtin_amdgcn_alignbit(r[1], r[0], (cell * 2u + odd + e_plane(e)) << 3);
            v[0] = __uint_as_float(w << 16); v[1] = __uint_as_float(w & 0xffff0000u);
        }
    };
    uint32_t rx[NI][PW], rd[NI][PW], rz[GATE ? NI : 1][PW], rm[RV][2];
    const auto request = [&](int batch) {
#pragma unroll
        for (int v = 0; v < RV; ++v) {
            const uint32_t cell = cell_of(batch, v);
            rm[v][0] = has_mask ? (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rsm, cell, 0, 0) : 0u;
            rm[v][1] = has_mask ? (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rsm, cell + 1u, 0, 0) : 0u;
        }
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            load(rsx, cell_of(batch, e % RV), e, rx[e]);
            load(rsd, cell_of(batch, e % RV), e, rd[e]);
        }
    };
    const auto request_z = [&](int batch) {                // z is needed where the batch's results are stored
#pragma unroll
        for (int e = 0; e < NI; ++e) load(rsz, cell_of(batch, e % RV), e, rz[e]);
    };
    float sk[NI][2];
    const auto produce = [&](int batch) {
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            float dl[2], xe[2];
            widen(rd[e], cell_of(batch, e % RV), e, dl);
            widen(rx[e], cell_of(batch, e % RV), e, xe);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if constexpr (SP) dl[k] = softplus_f32(dl[k] + dbias[e_ch(e)]);
                xe[k] = rm[e % RV][k] != 0u ? 0.0f : xe[k];                        // select: nothing under the mask leaks
                sk[e][k] = dsk[e_ch(e)] * xe[k];
            }
            *reinterpret_cast<float4*>(icell[e % RV] + e_ch(e) * 4) = make_float4(dl[0], dl[0] * xe[0], dl[1], dl[1] * xe[1]);
        }
    };

    // ---- Bm or Cm of a step: requested three steps ahead, widened and handed over two steps ahead, read one step ahead (without
    // BC_AHEAD: two, one, none)
    uint32_t slane[NS], raw[NS][BW], sh[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) slane[s] = ((uint32_t)(sg * NS + s) * (uint32_t)HW + (uint32_t)(col0 + min(ch * KQ, K - KQ))) * EB;
    const auto request_bc = [&](int t, uint32_t (&rs_raw)[NS][BW], uint32_t (&rs_sh)[NS]) {
        const uint32_t ro = row_of(t - blk) * ((uint32_t)W * EB);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint32_t off = slane[s] + ro;
            if constexpr (EB == 2) rs_sh[s] = off << 3;    // the shift by 0 or 16 bits in its lowest five bits
            buffer_load_words<BW>(rss, EB == 2 ? off & ~3u : off, 0, rs_raw[s]);
        }
    };
    const auto hand_over = [&](int set, const uint32_t (&rs_raw)[NS][BW], const uint32_t (&rs_sh)[NS]) {
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            float v[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if constexpr (EB == 4) v[s] = __uint_as_float(rs_raw[s][q]);
                else {
                    const uint32_t w = __builtin_amdgcn_alignbit(q / 2 + 1 < BW ? rs_raw[s][q / 2 + 1] : 0u, rs_raw[s][q / 2], rs_sh[s]);
                    v[s] = q & 1 ? __uint_as_float(w & 0xffff0000u) : __uint_as_float(w << 16);
                }
            }
            bc[((set * 2 + quad) * KQ + q) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        }
    };

    float h[K][NS];
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int s = 0; s < NS; ++s) h[j][s] = 0.0f;

    if (wc == 0 && lane < 32) carry[(lane >> 4) * cstride + (lane & 15)] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int batches = (H + 6) / 4;                       // the last block of a wavefront starts three steps late
    {
        uint32_t raw0[NS][BW], sh0[NS], raw1[NS][BW], sh1[NS];
        request(0);
        request_bc(0, raw0, sh0);
        if constexpr (BC_AHEAD) request_bc(1, raw1, sh1);
        request_bc(SETS - 1, raw, sh);
        produce(0);
        request(min(1, batches - 1));
        hand_over(0, raw0, sh0);
        if constexpr (BC_AHEAD) hand_over(1, raw1, sh1);
    }
    __syncthreads();

    float uB[2][KQ][NS], uC[2][KQ][NS];
    const auto take_bc = [&](int set, int to) {
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const float4 vb = bc[(set * 2 * KQ + q) * 64 + lane], vc = bc[((set * 2 + 1) * KQ + q) * 64 + lane];
            uB[to][q][0] = vb.x; uB[to][q][1] = vb.y; uB[to][q][2] = vb.z; uB[to][q][3] = vb.w;
            uC[to][q][0] = vc.x; uC[to][q][1] = vc.y; uC[to][q][2] = vc.z; uC[to][q][3] = vc.w;
        }
    };
    float4 v4[2][(K + 1) / 2];
    const auto take_row = [&](int r, int to) {
#pragma unroll
        for (int j2 = 0; j2 < (K + 1) / 2; ++j2) v4[to][j2] = *reinterpret_cast<const float4*>(pp + r * PR + (blk * 4 + ch) * 4 + j2 * kQuadPair);
    };
    if constexpr (BC_AHEAD) take_bc(0, 0);
    int set1 = 1, set2 = 2;                                // the LDS sets of the next step and of the one after it

    for (int round = 0; round < batches + cols - 1; ++round) {
        const int batch = round - wc;                      // a wavefront's four blocks are one batch ahead of the next one's
        if ((unsigned)batch >= (unsigned)batches) {
#pragma unroll 1
            for (int r = 0; r < 4; ++r) __syncthreads();
            continue;
        }
        if constexpr (GATE) request_z(batch);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = 4 * batch + r;
            const float4 cin = carry[(r & 1) * cstride + wc * 64 + lane];
            float hh[NS] = {cin.x, cin.y, cin.z, cin.w};
            float* const mine = pp + r * PR + (blk * 4 + ch) * 4 + (sg & 1) * 2;
            const int at = r & 1;
            if (!AHEAD || r == 0) take_row(r, at);
            if (AHEAD && r < 3) take_row(r + 1, at ^ 1);
            if constexpr (BC_AHEAD) take_bc(set1, at ^ 1); else take_bc(at, at);
            float y0 = 0.0f, hn[NS];
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const int ql = min(j / KQ, 3), qe = j - min(ql * KQ, K - KQ);       // the quad's lane that holds column j, and where
                const float dl = j & 1 ? v4[at][j / 2].z : v4[at][j / 2].x, dx = j & 1 ? v4[at][j / 2].w : v4[at][j / 2].y;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const float a = __builtin_amdgcn_exp2f(dl * Ap[s]);
                    hh[s] = fmaf(a, hh[s], dx * quad_bcast(uB[at][qe][s], ql));         // Eq. 5
                    fma_inplace(h[j][s], a, hh[s]);                                 // Eq. 6
                }
                const float y = quad_dot(uC[at][qe][0], uC[at][qe][1], uC[at][qe][2], uC[at][qe][3], h[j], ql);
                if (j == K - 2) {
#pragma unroll
                    for (int s = 0; s < NS; ++s) hn[s] = hh[s];
                }
                // state groups two apart hold the same sum and write it to the same place
                if ((j & 1) != 0 || j == K - 1) *reinterpret_cast<float2*>(mine + j / 2 * kQuadPair) = make_float2(j & 1 ? y0 : y, j & 1 ? y : 0.0f);
                y0 = y;
            }
            // a narrow block ends one column earlier
            carry[((r & 1) ^ 1) * cstride + wc * 64 + lane + 16] =
                make_float4(full ? hh[0] : hn[0], full ? hh[1] : hn[1], full ? hh[2] : hn[2], full ? hh[3] : hn[3]);
            hand_over(BC_AHEAD ? set2 : at ^ 1, raw, sh);
            request_bc(t + SETS, raw, sh);
            const int set0 = 3 - set1 - set2;
            set1 = set2;
            set2 = set0;
            if (t < 3) {                                   // blocks that have not reached the map's first row yet
#pragma unroll
                for (int j = 0; j < K; ++j)
#pragma unroll
                    for (int s = 0; s < NS; ++s) h[j][s] = t < blk ? 0.0f : h[j][s];
            }
            __syncthreads();
        }
        // the pairs that this lane prepared: sum over the states, skip, gate, one rounding
        float4 part[NI];
#pragma unroll
        for (int e = 0; e < NI; ++e) part[e] = *reinterpret_cast<const float4*>(icell[e % RV] + e_ch(e) * 4);
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            const uint32_t cell = cell_of(batch, e % RV);
            const bool here = (unsigned)(4 * batch + irow[e % RV] - iblk) < (unsigned)H && c0 + e_ch(e) < p.Dc;
            float out[2];
            {
#pragma clang fp contract(off)                             // as in scan2d_fwd_shared.hpp: the same bits with and without the gate
                out[0] = (part[e].x + part[e].z) + sk[e][0];
                out[1] = (part[e].y + part[e].w) + sk[e][1];
            }
            // what does not exist is addressed past the end of the buffer
            const uint32_t none = 0x80000000u, at = cell * EB + odd;
            const auto store = [&](rsrc_t rs, const float* val) {
                if constexpr (EB == 4) {
                    const u32x2_t both = {__float_as_uint(val[0]), __float_as_uint(val[1])};
                    __builtin_amdgcn_raw_buffer_store_b64(both, rs, (here && iend > 1) ? at : none, e_plane(e), 0);
                    __builtin_amdgcn_raw_buffer_store_b32(both.x, rs, (here && iend == 1) ? at : none, e_plane(e), 0);
                } else {
                    const uint32_t both = pack_bf16x2(val[0], val[1]);
                    if (dwords) {
                        __builtin_amdgcn_raw_buffer_store_b32(both, rs, (here && iend > 0) ? at : none, e_plane(e), 0);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b16((short)both, rs, (here && iend > 0) ? at : none, e_plane(e), 0);
                        __builtin_amdgcn_raw_buffer_store_b16((short)(both >> 16), rs, (here && iend > 1) ? at + 2u : none, e_plane(e), 0);
                    }
                }
            };
            if (want_y) store(rsy, out);
            if constexpr (GATE) {
                float zv[2];
                widen(rz[e], cell, e, zv);
#pragma unroll
                for (int k = 0; k < 2; ++k) out[k] *= zv[k] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-zv[k] * kLog2e));   // SiLU(z)
                store(rsg, out);
            }
        }
        wave_lds_fence();
        produce(min(batch + 1, batches - 1));
        request(min(batch + 2, batches - 1));
        wave_lds_fence();
    }
}

template <typename T>
inline FwdKernel lookup_fwd_quads_kernel(int K, bool sp, bool gate) {
#define SCAN2D_X(k) \
    if (K == k) return gate ? scan2d_fwd_quads_kernel<T, k, true, true> : sp ? scan2d_fwd_quads_kernel<T, k, true, false> : scan2d_fwd_quads_kernel<T, k, false, false>;
    SCAN2D_FWD_QUADS_COLUMNS(SCAN2D_X)
#undef SCAN2D_X
    return nullptr;
}

}  // namespace scan2d
