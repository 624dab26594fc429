// The linear layers of a 2DMamba block (Fig. 2: the projections into and out of the block's inner width; the design of
// the original block, Sec. 3.2) on channel-major maps:
//     out[b,o,p] = bias[o] + sum_c Wt[o,c] * in[b,c,p] (+ residual[b,o,p]),   p = position of the map,
// a GEMM with the positions as its wide dimension, on the matrix cores (fp32 accumulation, one rounding after bias and
// residual).
//
// scan2d_linear_kernel: a wavefront owns 64 positions x 16 NOT output channels (scan2d_contract.hpp); no LDS, no barrier.
// The four wavefronts of a workgroup, and the workgroups that follow it on the same XCD, take the other output channels
// of the same positions, so `in` comes from HBM once and from L1 / L2 afterwards.  Bound: HBM for bf16 (the products of
// 128 -> 256 channels are 4.3 GFLOP beside 50 MB), the matrix rate for fp32.
// scan2d_linear_resident_kernel (bf16), scan2d_linear_split_kernel and scan2d_linear_stream_kernel (fp32): large maps.
// scan2d_linear_any_kernel: one thread per output, for maps of fewer than 4 positions or 4 GB of weights.
#include "scan2d_block.hpp"

#include <algorithm>

#include "scan2d_contract.hpp"

namespace scan2d {
bool allow_large_lds(const void* kernel, size_t bytes);   // scan2d_api.hip
namespace {

struct LinArgs {
    const void* in; const void* Wt; const float* bias; const void* res; void* out;
    int Cin, Cout, Bt, ogroups;     // ogroups: wavefronts per tile of positions
    long long ptiles, P, waves;     // tiles of 64 positions per batch item, positions per map, wavefronts (pieces) with work
};

template <typename T, int NOT, int DEPTH, bool TAIL, bool WIDE = false>
__global__ __launch_bounds__(256) void scan2d_linear_kernel(const LinArgs p) {
    const long long per = gridDim.x / kXcds;               // the grid is a multiple of 8: workgroups of one XCD follow each other
    const long long wg = (long long)(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pairs = (p.ogroups + 1) / 2;                 // the workgroup: 2 tiles of positions x 2 groups of output channels
    const int og = (int)(wg % pairs) * 2 + (wv & 1);
    const long long tile = wg / pairs * 2 + (wv >> 1);
    if (og >= p.ogroups || tile >= p.ptiles * p.Bt) return;
    const int b = (int)(tile / p.ptiles);
    const uint32_t p0 = (uint32_t)(tile % p.ptiles) * 64u, P = (uint32_t)p.P;
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15, o0 = og * 16 * NOT;
    const LanePos pos(p0, n, P);

    f32x4 acc[NOT][4];
#pragma unroll
    for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[ot][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    contract<T, NOT, DEPTH, TAIL, WIDE>(static_cast<const T*>(p.in) + (size_t)b * p.Cin * P, P, pos.s, static_cast<const T*>(p.Wt), p.Cin, p.Cout, o0,
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

// bf16, large maps, at most 32 KT input channels in whole steps of 32: a wavefront reads its 64 positions x all channels
// once, holds them as MFMA operands (16 KT registers) and walks over the output channels, whose rows of Wt it reads from
// L1 / L2 one block ahead.  With `in` shared by the four wavefronts of a workgroup (above) only 16 KB per compute unit
// were in flight, two steps deep, and 128 -> 256 channels at 65536 positions took 23 us; here every wavefront has 16 or
// 32 KB of its own in flight before its first product.
template <int KT>
__global__ __launch_bounds__(256) void scan2d_linear_resident_kernel(const LinArgs p, int oblocks) {
    const long long per = gridDim.x / kXcds;
    const long long wg = (long long)(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    const long long wave = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= p.waves) return;
    const int og = (int)(wave % p.ogroups);                // blocks of 16 output channels og * oblocks ..
    const long long rest = wave / p.ogroups;
    const int b = (int)(rest / p.ptiles);
    const uint32_t p0 = (uint32_t)(rest % p.ptiles) * 64u, P = (uint32_t)p.P;
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15;
    const int Cin = p.Cin, steps = Cin / 32;
    const LanePos pos(p0, n, P);
    const char* in = reinterpret_cast<const char*>(static_cast<const bf16_t*>(p.in) + (size_t)b * Cin * P);
    const uint32_t boff = ((uint32_t)(8 * g) * P + pos.s) * 2u;

    bf16x8 bv[KT][4];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const char* base = in + (size_t)min(k, steps - 1) * 64u * P;
        uint32_t raw[8][2];
#pragma unroll
        for (int e = 0; e < 8; ++e) load_words_any<2>(base + (size_t)e * P * 2u + boff, raw[e]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            u32x4_t v;
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2)
                v[e2] = __builtin_amdgcn_perm(raw[2 * e2 + 1][t / 2], raw[2 * e2][t / 2], t % 2 ? 0x07060302u : 0x05040100u);
            bv[k][t] = __builtin_bit_cast(bf16x8, v);
        }
    }
    const char* Wt = static_cast<const char*>(p.Wt);
    u32x4_t av[2][KT];
    const int o16 = (p.Cout + 15) / 16, ob = og * oblocks, oe = min(ob + oblocks, o16);
    auto load_a = [&](int buf, int blk) {
        const uint32_t off = ((uint32_t)min(16 * min(blk, oe - 1) + n, p.Cout - 1) * (uint32_t)Cin + (uint32_t)(8 * g)) * 2u;
#pragma unroll
        for (int k = 0; k < KT; ++k) av[buf][k] = *reinterpret_cast<const u32x4_a1*>(Wt + off + (uint32_t)(64 * min(k, steps - 1)));
    };
    const bf16_t* res = static_cast<const bf16_t*>(p.res);
    bf16_t* out = static_cast<bf16_t*>(p.out);
    auto block = [&](int buf, int blk) {
        uint32_t rr[4][2];
        float bias[4];
        size_t row[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = min(16 * blk + 4 * g + i, p.Cout - 1);
            row[i] = ((size_t)b * p.Cout + o) * P;
            bias[i] = p.bias ? p.bias[o] : 0.0f;
            if (res) load_words_any<2>(res + row[i] + pos.s, rr[i]);
        }
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < KT; ++k)
            if (k < steps) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[buf][k]), bv[k][t], acc[t], 0, 0, 0);
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = acc[t][i] + bias[i];
            if (res) {
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] += get_elem<bf16_t, 4>(rr[i], t);
            }
            if (16 * blk + 4 * g + i < p.Cout) pos.store(out + row[i], v);
        }
    };
    load_a(0, ob);
    for (int blk = ob; blk < oe; blk += 2) {
        load_a(1, blk + 1);
        block(0, blk);
        if (blk + 1 < oe) {
            load_a(0, blk + 2);
            block(1, blk + 1);
        }
    }
}

// fp32, enough work for every SIMD, input channels in whole steps of 16: the products bound the layer (157 TFLOP/s on
// v_mfma_f32_16x16x4_f32), and the matrix pipe of a SIMD is best kept busy by ONE wavefront: a loop of 64 products and 8
// loads ran at 134 TFLOP/s with one wavefront per SIMD, 120 with two and 113 with three (their streams alternate on the
// pipe and leave gaps).  So the launch is one workgroup per compute unit; its wavefronts walk over (tile of positions,
// 16 NOT output channels), DEPTH steps of loads ahead of the products, across the end of one piece of work into the next.
// No load in a branch (the residual is a template flag, a missing bias reads Wt and is not used): the compiler's wait
// counts would become "everything" at the head of the loop.
template <int NOT, int DEPTH, bool RES>
__global__ __launch_bounds__(256, 1) void scan2d_linear_stream_kernel(const LinArgs p) {
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ptiles = (uint32_t)p.ptiles, ogroups = (uint32_t)p.ogroups;
    const uint32_t items = (uint32_t)p.waves, stride = gridDim.x * 4;        // below 2^31 (checked on the host)
    const uint32_t first = ((blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds) * 4 + wv;
    if (first >= items) return;
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15;
    const int Cin = p.Cin, steps = Cin / 16;
    const uint32_t P = (uint32_t)p.P;

    struct Piece { const char* in; uint32_t boff, p0; int b, o0; uint32_t aoff[NOT]; };
    auto piece = [&](uint32_t item) {
        Piece w;
        const uint32_t tile = item / ogroups;
        w.o0 = (int)(item - tile * ogroups) * 16 * NOT;
        w.b = (int)(tile / ptiles);
        w.p0 = (tile - (uint32_t)w.b * ptiles) * 64u;
        w.in = reinterpret_cast<const char*>(static_cast<const float*>(p.in) + (size_t)w.b * Cin * P);
        w.boff = ((uint32_t)(4 * g) * P + LanePos(w.p0, n, P).s) * 4u;
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot) w.aoff[ot] = ((uint32_t)min(w.o0 + 16 * ot + n, p.Cout - 1) * (uint32_t)Cin + (uint32_t)(4 * g)) * 4u;
        return w;
    };
    uint32_t braw[DEPTH][4][4], araw[DEPTH][NOT][4];
    auto load = [&](int buf, const Piece& w, int k) {
        const char* bb = w.in + (size_t)k * 64u * P;
#pragma unroll
        for (int e = 0; e < 4; ++e) load_words_any<4>(bb + (size_t)e * P * 4u + w.boff, braw[buf][e]);
        const char* aa = static_cast<const char*>(p.Wt) + (size_t)k * 64u;
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot) load_words_any<4>(aa + w.aoff[ot], araw[buf][ot]);
    };
    f32x4 acc[NOT][4];
    auto products = [&](int buf) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[ot][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(araw[buf][ot][e]), __uint_as_float(braw[buf][e][t]),
                                                                      acc[ot][t], 0, 0, 0);
    };
    const float* res = static_cast<const float*>(p.res);
    const float* bsrc = p.bias ? p.bias : static_cast<const float*>(p.Wt);   // Wt has Cout rows: at least as many elements
    float* out = static_cast<float*>(p.out);

    Piece cur = piece(first);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d, cur, d);       // steps is a multiple of DEPTH
    for (uint32_t item = first; item < items; item += stride) {
        const Piece next = piece(min(item + stride, items - 1));
        const LanePos pos(cur.p0, n, P);
        float add[RES ? NOT : 1][4][4], bias[NOT][4];                // residual and bias, requested in front of the products
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int o = min(cur.o0 + 16 * ot + 4 * g + i, p.Cout - 1);
                if constexpr (RES) load4<float>(res + ((size_t)cur.b * p.Cout + o) * P + pos.s, add[ot][i]);
                bias[ot][i] = bsrc[o];
            }
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[ot][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int k = 0; k < steps - DEPTH; k += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                products(d);
                load(d, cur, k + d + DEPTH);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            products(d);
            load(d, next, d);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int o = cur.o0 + 16 * ot + 4 * g + i;
                float v[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    v[t] = acc[ot][t][i] + (p.bias ? bias[ot][i] : 0.0f);
                    if constexpr (RES) v[t] += add[ot][i][t];
                }
                if (o < p.Cout) pos.store(out + ((size_t)cur.b * p.Cout + o) * P, v);
            }
        cur = next;
    }
}

// fp32 as sums of bf16: x = x1 + x2 + x3 with x1 = bf16(x), x2 = bf16(x - x1) and x3 the rest, which has at most 8 bits, so the
// sum is x itself.  Of a product's nine terms all but x3 w3 are formed, on v_mfma_f32_16x16x32_bf16 (16 times the fp32
// matrix rate); it is below 2^-33 of the product.  (Six terms take 43 us where eight take 51, but a sum of one large product is then
// up to 1.1e-7 off, not 6.0e-8 as by fp32 products.)
struct Split { uint32_t part[3]; };                        // of two values, packed
__device__ __forceinline__ Split split_bf16(float a, float b) {
    Split s;
    s.part[0] = pack_bf16x2(a, b);
    a -= __uint_as_float(s.part[0] << 16);
    b -= __uint_as_float(s.part[0] & 0xffff0000u);
    s.part[1] = pack_bf16x2(a, b);
    a -= __uint_as_float(s.part[1] << 16);
    b -= __uint_as_float(s.part[1] & 0xffff0000u);
    s.part[2] = pack_bf16x2(a, b);
    return s;
}

// Largest / smallest magnitude so far (fmaxf and fminf would first quiet each value: one more instruction apiece).
__device__ __forceinline__ void max3_abs(float& m, uint32_t a, uint32_t b) { asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b)); }
__device__ __forceinline__ void min3_abs(float& m, float a, float b) { asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b)); }

// fp32, enough work for every SIMD, input channels in whole steps of 64: the layer as bf16 products (split_bf16).  A workgroup
// (one per compute unit) splits its 16 NOT rows of Wt once and keeps them in LDS as MFMA operands; its 8 wavefronts walk over
// pieces of 32 positions, whose channels they split on the way: a step of 32 channels is split beside the products of the
// step before it (4 vector slots per product pass), its loads a step earlier still, across the end of one piece into the next.
// The largest terms have accumulators of their own: theirs is the rounding that counts, once per 32 channels.
// Outside of bf16's range an output is formed again from fp32 products, each by its own row of Wt and its own position alone:
//   * not finite: an infinity or NaN among its operands, a value that rounds to infinity in bf16, a sum that overflowed;
//   * too small beside its operands: the parts of a value are exact down to 2^-133 (products and sums keep what is subnormal), so
//     up to 2^-134 of each input and of each weight may be lost, and of the output up to 768 * 2^-134 * (X + W), X and W the largest
//     magnitudes of its position and its row.  Where |output| >= 2^-96 (X + W), or X or W is 0, that is below 2^-28 of it.
// A piece is tested as a whole first, by the smallest output of a position and the largest weight of the slice.
// Bound: the matrix pipe (half its time in use) and the clock under it: 256 -> 512 channels at 24576 positions take 47 to 50 us, with
// all operands zero 41 us (scan2d_linear_stream_kernel 55 and 53 us).  Error against 64 bits, 2-norm: 0.9e-7 (2.9e-7).
constexpr int kSplitWaves = 8;
constexpr float kMost = 3.402823466e38f, kSmall = 0x1p-96f;
template <int NOT, bool RES>
__global__ __launch_bounds__(kSplitWaves * 64, 2) void scan2d_linear_split_kernel(const LinArgs p) {
    extern __shared__ u32x4_t wl[];                        // [steps][NOT][3][64 lanes], then bias and largest weights
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t slices = (uint32_t)p.ogroups, groups = gridDim.x / slices;
    const uint32_t wg = (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    const uint32_t slice = wg % slices, group = wg / slices;
    if (group >= groups) return;                           // the grid is a multiple of 8, not of the slices
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15;
    const int Cin = p.Cin, steps = Cin / 32, o0 = (int)slice * 16 * NOT;
    const uint32_t P = (uint32_t)p.P, ptiles = (uint32_t)p.ptiles, items = (uint32_t)p.waves, stride = groups * kSplitWaves;

    float* const bl = reinterpret_cast<float*>(wl + steps * NOT * 3 * 64);   // bias and largest weight of the 16 NOT output channels
    float* const wmax = bl + 16 * NOT;
    if (threadIdx.x < 16 * NOT) {
        bl[threadIdx.x] = p.bias != nullptr ? p.bias[min(o0 + (int)threadIdx.x, p.Cout - 1)] : 0.0f;
        wmax[threadIdx.x] = 0.0f;
    }
    __syncthreads();
    // four fragments' loads at a time (past the last one it is loaded again)
    for (int f0 = wv; f0 < steps * NOT; f0 += 4 * kSplitWaves) {
        uint32_t r[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int f = min(f0 + u * kSplitWaves, steps * NOT - 1), k = f / NOT, ot = f - k * NOT;
            load_words_any<8>(static_cast<const float*>(p.Wt) + (size_t)min(o0 + 16 * ot + n, p.Cout - 1) * Cin + 32 * k + 8 * g, r[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int f = f0 + u * kSplitWaves;
            if (f >= steps * NOT) break;
            Split s[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = split_bf16(__uint_as_float(r[u][2 * e]), __uint_as_float(r[u][2 * e + 1]));
#pragma unroll
            for (int q = 0; q < 3; ++q) wl[(f * 3 + q) * 64 + l] = u32x4_t{s[0].part[q], s[1].part[q], s[2].part[q], s[3].part[q]};
            uint32_t most = 0u;                            // magnitudes compare like their bits
#pragma unroll
            for (int e = 0; e < 8; ++e) most = max(most, r[u][e] & 0x7fffffffu);
            atomicMax(reinterpret_cast<uint32_t*>(wmax) + 16 * (f % NOT) + n, most);
        }
    }
    __syncthreads();
    float wmost = 0.0f;
#pragma unroll
    for (int o = 0; o < 16 * NOT; ++o) wmost = fmaxf(wmost, wmax[o]);

    struct Piece { const char* in; uint32_t boff, p0; int b; };
    auto piece = [&](uint32_t item) {
        Piece w;
        w.b = (int)(item / ptiles);
        w.p0 = (item - (uint32_t)w.b * ptiles) * 32u;
        w.in = reinterpret_cast<const char*>(static_cast<const float*>(p.in) + (size_t)w.b * Cin * P);
        w.boff = ((uint32_t)(8 * g) * P + LanePos<2>(w.p0, n, P).s) * 4u;
        return w;
    };
    uint32_t raw[2][8][2];
    u32x4_t x[2][2][3];
    f32x4 acc[NOT][2], low[NOT][2];                        // sums of x1 w1; of the other terms
    const uint32_t first = group + groups * wv;            // the last round's pieces spread over the groups, then over the SIMDs
    if (first >= items) return;
    Piece cur = piece(first), next = cur;
    auto load = [&](int buf, int k) {                      // step k of this piece, or of the next one behind its end (steps >= 4)
        const bool over = k >= steps;
        const char* bb = (over ? next.in : cur.in) + (size_t)(over ? k - steps : k) * 128u * P;
        const uint32_t off = over ? next.boff : cur.boff;
#pragma unroll
        for (int e = 0; e < 8; ++e) load_words_at<2>(bb + (size_t)e * P * 4u, off, raw[buf][e]);
    };
    float xmax[2] = {0.0f, 0.0f};                          // largest magnitude split of the lane's two positions
    auto split_pair = [&](int buf, int pair) {             // two channels of one of them
        const int t = pair / 4, e = pair % 4;
        max3_abs(xmax[t], raw[buf][2 * e][t], raw[buf][2 * e + 1][t]);
        const Split s = split_bf16(__uint_as_float(raw[buf][2 * e][t]), __uint_as_float(raw[buf][2 * e + 1][t]));
#pragma unroll
        for (int q = 0; q < 3; ++q) x[buf][t][q][e] = s.part[q];
    };
    u32x4_t wr[2][3];                                      // a block of 16 output channels ahead
    auto load_w = [&](int buf, int block) {
#pragma unroll
        for (int q = 0; q < 3; ++q) wr[buf][q] = wl[(block * 3 + q) * 64 + l];
    };
    // The products of step k beside the split of the step behind it, in pieces that the scheduler may not merge: left to
    // itself it puts chains of dependent products together and the operands' reads in front of their use.
    auto step = [&](int buf, int k) {
        int pair = 0;
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot) {
            const int at = (buf * NOT + ot) & 1;
            load_w(at ^ 1, ot + 1 < NOT ? k * NOT + ot + 1 : (k + 1 < steps ? (k + 1) * NOT : 0));
            const auto term = [&](f32x4 (&to)[2], int wq, int xq) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    to[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[at][wq]), __builtin_bit_cast(bf16x8, x[buf][t][xq]), to[t], 0, 0, 0);
            };
#pragma unroll
            for (int part = 0; part < 4; ++part) {
                if (part == 0) { term(low[ot], 2, 1); term(acc[ot], 0, 0); }
                else if (part == 1) { term(low[ot], 1, 2); term(low[ot], 2, 0); }
                else if (part == 2) { term(low[ot], 0, 2); term(low[ot], 1, 1); }
                else { term(low[ot], 1, 0); term(low[ot], 0, 1); }
#pragma unroll
                for (; pair < ((ot * 4 + part + 1) * 8 + 4 * NOT - 1) / (4 * NOT); ++pair) split_pair(buf ^ 1, pair);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    const float* res = static_cast<const float*>(p.res);
    float* out = static_cast<float*>(p.out);

    load(0, 0);
    load(1, 1);
    load_w(0, 0);
#pragma unroll
    for (int pair = 0; pair < 8; ++pair) split_pair(0, pair);
    load(0, 2);
    for (uint32_t item = first; item < items; item += stride) {
        next = piece(min(item + stride, items - 1));
        const LanePos<2> pos(cur.p0, n, P);
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[ot][t] = low[ot][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        float xm[2] = {0.0f, 0.0f};
        for (int k = 0; k < steps; k += 2) {
            step(0, k);
            load(1, k + 3);
            if (k + 2 == steps) {                          // what follows belongs to the next piece
                xm[0] = xmax[0]; xm[1] = xmax[1];
                xmax[0] = xmax[1] = 0.0f;
            }
            step(1, k + 1);
            load(0, k + 4);
        }
        uint32_t add[RES ? NOT : 1][4][2];
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[ot][t] += low[ot][t];
        if constexpr (RES) {                               // into the registers of `low`
#pragma unroll
            for (int ot = 0; ot < NOT; ++ot) {
                const int r0 = min(o0 + 16 * ot, p.Cout - 1);      // uniform; the lane's rows follow it
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    load_words_at<2>(res + ((size_t)cur.b * p.Cout + r0) * P, ((uint32_t)min(4 * g + i, p.Cout - 1 - r0) * P + pos.s) * 4u, add[ot][i]);
            }
        }
        bool again = false;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            xm[t] = fmaxf(xm[t], __shfl_xor(xm[t], 16));   // the four lanes of a position hold 8 channels of every 32 each
            xm[t] = fmaxf(xm[t], __shfl_xor(xm[t], 32));
            float size = 0.0f, least = kMost;
#pragma unroll
            for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    size += fabsf(acc[ot][t][i]);
                    size += fabsf(acc[ot][t][i + 1]);
                    min3_abs(least, acc[ot][t][i], acc[ot][t][i + 1]);
                }
            again |= !((size <= kMost) & ((xm[t] == 0.0f) | (least >= fmaf(kSmall, xm[t], kSmall * wmost))));
        }
        if (__any(again)) {
            uint32_t redo = 0u;                            // a bit per output of the lane
#pragma unroll
            for (int ot = 0; ot < NOT; ++ot) {
                const f32x4 wm = *reinterpret_cast<const f32x4*>(wmax + 16 * ot + 4 * g);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float v = fabsf(acc[ot][t][i]);
                        const bool good = (v <= kMost) & ((xm[t] == 0.0f) | (wm[i] == 0.0f) | (v >= fmaf(kSmall, xm[t], kSmall * wm[i])));
                        redo |= good ? 0u : 1u << (8 * ot + 4 * t + i);
                    }
            }
            if (__any(redo != 0u)) {
#pragma unroll
                for (int ot = 0; ot < NOT; ++ot) {
                    f32x4 full[2] = {};
                    uint32_t row = (uint32_t)min(o0 + 16 * ot + n, p.Cout - 1);
                    asm volatile("" : "+v"(row));          // the address is formed here: from in front of the loops it would hold registers there
                    for (int c = 0; c < Cin; c += 4) {
                        const float* in = static_cast<const float*>(p.in) + ((size_t)cur.b * Cin + c + g) * P + pos.s;
                        const float w = static_cast<const float*>(p.Wt)[(size_t)row * Cin + c + g];
#pragma unroll
                        for (int t = 0; t < 2; ++t) full[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, in[t], full[t], 0, 0, 0);
                    }
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[ot][t][i] = (redo >> (8 * ot + 4 * t + i) & 1u) != 0u ? full[t][i] : acc[ot][t][i];
                }
                load_w(0, 0);                              // again: its registers were needed here
            }
        }
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot) {
            const f32x4 bias = *reinterpret_cast<const f32x4*>(bl + 16 * ot + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int o = o0 + 16 * ot + 4 * g + i;
                float v[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    v[t] = p.bias != nullptr ? acc[ot][t][i] + bias[i] : acc[ot][t][i];
                    if constexpr (RES) v[t] += __uint_as_float(add[ot][i][t]);
                }
                if (o < p.Cout) pos.store(out + ((size_t)cur.b * p.Cout + o) * P, v);
            }
        }
        cur = next;
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

template <typename T, int NOT, int DEPTH, bool WIDE = false>
int launch(LinArgs a, hipStream_t stream) {
    a.ogroups = (a.Cout + 16 * NOT - 1) / (16 * NOT);
    const long long wgs = (a.ptiles * a.Bt + 1) / 2 * ((a.ogroups + 1) / 2), grid = (wgs + kXcds - 1) / kXcds * kXcds;
    if (!launch_fits(grid, 256)) return SCAN2D_ERR_BAD_SHAPE;
    auto kernel = a.Cin % contract_step<T>() == 0 ? scan2d_linear_kernel<T, NOT, DEPTH, false, WIDE> : scan2d_linear_kernel<T, NOT, DEPTH, true, WIDE>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, stream, a);
    return SCAN2D_OK;
}

// Output channels per wavefront: 64 (each load of `in` then serves 16 products) where that leaves every SIMD two
// wavefronts, fewer where it does not: a small map is bound by the latency of its few steps, not by the loads.
template <typename T>
int launch_sized(const LinArgs& a, hipStream_t stream) {
    const long long tiles = a.ptiles * a.Bt, o16 = (a.Cout + 15) / 16;
    if (!contract_narrow(a.P, Elem<T>::kBytes)) return launch<T, 4, 2, true>(a, stream);     // more than 82 million positions
    if constexpr (Elem<T>::kBytes == 2) {
        if (tiles >= 512 && o16 >= 4 && a.Cin % 32 == 0 && a.Cin <= 256) {
            LinArgs r = a;                                 // two wavefronts per tile until there are four per SIMD
            r.ogroups = tiles < 4096 ? 2 : 1;
            const int oblocks = (int)((o16 + r.ogroups - 1) / r.ogroups);
            r.waves = tiles * r.ogroups;
            const long long grid = ((r.waves + 3) / 4 + kXcds - 1) / kXcds * kXcds;
            if (!launch_fits(grid, 256)) return SCAN2D_ERR_BAD_SHAPE;
            if (a.Cin <= 128) hipLaunchKernelGGL(scan2d_linear_resident_kernel<4>, dim3((unsigned)grid), dim3(256), 0, stream, r, oblocks);
            else hipLaunchKernelGGL(scan2d_linear_resident_kernel<8>, dim3((unsigned)grid), dim3(256), 0, stream, r, oblocks);
            return SCAN2D_OK;
        }
    }
    if constexpr (Elem<T>::kBytes == 4) {
        // 16 NOT output channels per piece: the fewest rounds of 1024 wavefronts, counted in their products
        const auto cost = [&](long long n) { return (tiles * ((o16 + n - 1) / n) + 1023) / 1024 * n; };
        const bool stream_form = a.Cin % 64 == 0 && tiles * o16 >= 2048 && tiles * o16 < (1LL << 30);
        // bf16 products where an estimate of both forms in us says so, fitted to 344 shapes (128 to 768 -> 32 to 1024 channels, 800 to
        // 40000 positions; mean error 3 to 4 %, and the chip's power moves the bf16 side by as much again: hence the 5 %).  By bf16
        // and by fp32 products, us: 256 -> 512 channels at 25527 positions 50.8 and 64.0, at 8192 19.9 and 21.7, 384 -> 192 at 12000 19.9
        // and 28.6; fp32 products win where a round or two of wavefronts is all there is: 384 -> 256 at 3200 11.1 and 9.8, 512 -> 128 at
        // 8000 14.0 and 12.3.  LDS holds 32 rows of Wt up to 768 channels.
        const long long pieces = (a.P + 31) / 32 * a.Bt;
        if (a.Cin % 64 == 0 && a.Cin >= 128 && a.Cin <= 768 && 25 * a.P * 4 < (1LL << 32) && pieces < (1LL << 30) && o16 <= 512 && tiles * o16 < (1LL << 30)) {
            const double m = (double)(stream_form ? std::min(cost(2), cost(4)) : cost(1));
            const double fp32_us = 2.7 + 0.75 * m + a.Cin * (0.0147 * m + 0.0014);
            // 16 n output channels per workgroup, as many as its LDS holds: the fewest rounds of SIMDs, in products and the work of
            // splitting the inputs
            const auto rounds = [&](long long n) {
                const long long slices = (o16 + n - 1) / n, groups = 256 / slices;
                return a.Cin / 32 * n * 3072 > 150 * 1024 || groups < 1 ? 1LL << 40 : (pieces + groups * 4 - 1) / (groups * 4);
            };
            int n = 2;
            for (int k = 3; k <= 4; ++k)
                if (rounds(k) * (256 * k + 150) <= rounds(n) * (256 * n + 150)) n = k;
            if (2.6 + 0.97 * n + a.Cin * ((double)rounds(n) * (0.0053 * n + 0.0043) + 0.0018) < 0.95 * fp32_us) {
                LinArgs r = a;
                r.ogroups = (int)((o16 + n - 1) / n);
                r.ptiles = (a.P + 31) / 32;
                r.waves = pieces;
                using Kernel = void (*)(const LinArgs);
                const Kernel k = n == 4 ? (a.res ? scan2d_linear_split_kernel<4, true> : scan2d_linear_split_kernel<4, false>)
                               : n == 3 ? (a.res ? scan2d_linear_split_kernel<3, true> : scan2d_linear_split_kernel<3, false>)
                                        : (a.res ? scan2d_linear_split_kernel<2, true> : scan2d_linear_split_kernel<2, false>);
                const size_t lds = (size_t)a.Cin / 32 * n * 3072 + (size_t)n * 128;
                if (lds > 65536 && !allow_large_lds(reinterpret_cast<const void*>(k), lds)) return SCAN2D_ERR_LAUNCH_FAILED;
                hipLaunchKernelGGL(k, dim3(256), dim3(kSplitWaves * 64), lds, stream, r);
                return SCAN2D_OK;
            }
        }
        if (stream_form) {
            LinArgs r = a;
            const bool four = cost(4) <= cost(2);
            r.ogroups = (int)((o16 + (four ? 3 : 1)) / (four ? 4 : 2));
            r.waves = tiles * r.ogroups;
            using Kernel = void (*)(const LinArgs);
            Kernel k;
            if (four) k = a.res ? scan2d_linear_stream_kernel<4, 2, true> : scan2d_linear_stream_kernel<4, 2, false>;
            else k = a.res ? scan2d_linear_stream_kernel<2, 4, true> : scan2d_linear_stream_kernel<2, 4, false>;
            hipLaunchKernelGGL(k, dim3(256), dim3(256), 0, stream, r);
            return SCAN2D_OK;
        }
    }
    if (o16 >= 4 && tiles * ((o16 + 3) / 4) >= 2048) return launch<T, 4, 2>(a, stream);
    if (o16 >= 2 && tiles * ((o16 + 1) / 2) >= 2048) return launch<T, 2, 2>(a, stream);
    return launch<T, 1, 4>(a, stream);
}

int launch_linear(const scan2d_desc* d, int Cout, const void* in, const void* Wt, const float* bias, const void* residual, void* out, hipStream_t stream) {
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
        if (!launch_fits(blocks, 256)) return SCAN2D_ERR_BAD_SHAPE;
        if (bf16) hipLaunchKernelGGL(scan2d_linear_any_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL(scan2d_linear_any_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    }
    if (rc != SCAN2D_OK) return rc;
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace

int block_linear_launch(const scan2d_desc* d, int Cout, const void* in, const void* Wt, const float* bias, const void* residual,
                        void* out, hipStream_t stream) {
    const size_t row = (size_t)d->H * d->W * (d->dtype == SCAN2D_BF16 ? 2 : 4), each = row * Cout;
    return by_items(*d, [&](const scan2d_desc& q, size_t b) {
        return launch_linear(&q, Cout, item_at(in, b, row * d->Dc), Wt, bias, item_at(residual, b, each), item_at(out, b, each), stream);
    });
}

}  // namespace scan2d
