// Contraction over the channels of a channel-major map on the matrix cores, without LDS: what the linear layers, the
// projections of step, B and C and the aggregator's scores have in common.
//     acc[o][p] = sum over c in [cbeg, cend) of W[o][c] * in[c][p]
// for NOT * 16 rows of W and 64 positions per wavefront.
//
// Which position a column of an MFMA tile stands for is free, and so is the order of the contraction index, as long as
// both operands agree.  Column n (= lane % 16) of tile t is position 4 n + t of the wavefront's 64, so
//   - a lane reads 4 consecutive positions of a channel with one load (8 or 16 bytes; 16 lanes cover 128 or 256
//     contiguous bytes of the channel's row), and they are its operands of the four tiles.  fp32 needs nothing more; for
//     bf16, whose operand packs 8 channels of one position, 16 v_perm_b32 per 8 channels x 4 positions reorder them in
//     registers.  `in` therefore never passes through LDS;
//   - the accumulators of a lane are, for row 16 ot + 4 g + i (g = lane / 16), those 4 consecutive positions: results
//     leave as the same row segments.
// W is row-major in the contraction index: a lane reads 8 (bf16) or 4 (fp32) consecutive channels of its row.  The
// loads take any alignment (H*W and the channel count may be odd).
// bf16: v_mfma_f32_16x16x32_bf16, 32 channels per step; fp32: v_mfma_f32_16x16x4_f32, 16 channels per step (four MFMA,
// lane group g supplies channels 4 g .. 4 g + 3 in turn).  fp32 accumulation.
#pragma once

#include "scan2d_common.hpp"

namespace scan2d {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kXcds = 8;

template <typename T>
__device__ __forceinline__ float widen_bits(uint32_t bits) {
    if constexpr (Elem<T>::kBytes == 4) return __uint_as_float(bits);
    else return __uint_as_float(bits << 16);
}

// WORDS dwords at a wave-uniform base plus a 32-bit byte offset per lane.  Both are opaque to the compiler: seen through,
// they are merged into a 64-bit pointer per load, kept in two vector registers wherever a loop around the
// loads lets it (48 pointers in the projection kernel).
template <int WORDS>
__device__ __forceinline__ void load_words_at(const void* base, uint32_t off, uint32_t* r) {
    static_assert(WORDS == 1 || WORDS == 2 || WORDS == 4, "one load");
    uint64_t b = reinterpret_cast<uint64_t>(base);
    asm volatile("" : "+s"(b), "+v"(off));
    typedef const __attribute__((address_space(1))) char* Global;
    const Global q = reinterpret_cast<Global>(b) + off;
    if constexpr (WORDS == 1) {
        typedef uint32_t W __attribute__((aligned(2), may_alias));
        r[0] = *reinterpret_cast<const __attribute__((address_space(1))) W*>(q);
    } else {
        typedef uint32_t V __attribute__((ext_vector_type(WORDS)));
        typedef V W __attribute__((aligned(2), may_alias));
        const V v = *reinterpret_cast<const __attribute__((address_space(1))) W*>(q);
#pragma unroll
        for (int w = 0; w < WORDS; ++w) r[w] = v[w];
    }
}

// 4 consecutive elements as fp32 / from fp32, any alignment.
template <typename T>
__device__ __forceinline__ void load4(const T* p, float* v) {
    uint32_t r[words_of<T, 4>()];
    load_words_any<words_of<T, 4>()>(p, r);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = get_elem<T, 4>(r, j);
}
template <typename T>
__device__ __forceinline__ void store4(T* p, const float* v) {
    uint32_t r[words_of<T, 4>()];
    if constexpr (Elem<T>::kBytes == 2) { r[0] = pack_bf16x2(v[0], v[1]); r[1] = pack_bf16x2(v[2], v[3]); }
    else {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = __float_as_uint(v[j]);
    }
    store_words_any<words_of<T, 4>()>(p, r);
}

// The positions of a lane.  Loads always take 4 positions that exist: at the end of the map the group moves back and
// overlaps its neighbour, and only the positions from `p` on belong to this lane.  Maps have at least 4 positions.
template <int E = 4>
struct LanePos {
    uint32_t s, p;                        // first position read, first position owned (p >= s)
    bool whole, any;                      // all E are owned; at least one is
    __device__ __forceinline__ LanePos(uint32_t tile0, int n, uint32_t P) {
        p = tile0 + (uint32_t)(E * n);
        s = min(p, P - (uint32_t)E);
        whole = p == s;
        any = p < P;
    }
    // v[t] belongs to position s + t of `row`
    template <typename T> __device__ __forceinline__ void store(T* row, const float* v) const {
        if (whole) {
            if constexpr (E == 4) store4<T>(row + s, v);
            else if constexpr (Elem<T>::kBytes == 2) {
                const uint32_t w = pack_bf16x2(v[0], v[1]);
                store_words_any<1>(row + s, &w);
            } else {
                row[s] = v[0]; row[s + 1] = v[1];
            }
        } else if (any) {
#pragma unroll
            for (int t = 1; t < E; ++t)
                if (s + t >= p) store_elem(row + s + t, v[t]);
        }
    }
};

template <typename T> constexpr int contract_step() { return Elem<T>::kBytes == 2 ? 32 : 16; }     // channels per step

// `in`: the batch item's map, wave-uniform; s: first position this lane reads; W: row 0, wave-uniform, ldw channels per
// row; this lane supplies rows min(o0 + 16 ot + n, rows - 1).  DEPTH steps are in flight ahead of the products.
// TAIL: the channels are not whole steps (a flag, because the element-wise loads of the last ones take many registers).
// 32-bit byte offsets per lane: the whole of W stays below 2^32 bytes, and so do the rows of positions between a lane's
// address and the uniform base (contract_narrow; checked on the host).  WIDE: maps where the latter does not hold.
template <typename T, int NOT, int DEPTH, bool TAIL, bool WIDE = false>
__device__ __forceinline__ void contract(const T* __restrict__ in, uint32_t P, uint32_t s, const T* __restrict__ W, int ldw, int rows,
                                         int o0, int cbeg, int cend, f32x4 (&acc)[NOT][4]) {
    constexpr int EB = Elem<T>::kBytes, KS = contract_step<T>(), KL = KS / 4;        // channels per lane and step
    constexpr int BW = words_of<T, 4>();                                            // dwords of 4 positions
    const int l = threadIdx.x & 63, g = l >> 4, n = l & 15;
    const std::conditional_t<WIDE, uint64_t, uint32_t> boff = ((std::conditional_t<WIDE, uint64_t, uint32_t>)(KL * g) * P + s) * EB;
    uint32_t aoff[NOT];
#pragma unroll
    for (int ot = 0; ot < NOT; ++ot) aoff[ot] = ((uint32_t)min(o0 + 16 * ot + n, rows - 1) * (uint32_t)ldw + (uint32_t)(KL * g)) * EB;
    uint32_t braw[DEPTH][KL][BW], araw[DEPTH][NOT][4];
    auto load = [&](int buf, int c0) {
        const char* bb = reinterpret_cast<const char*>(in + (size_t)c0 * P);
#pragma unroll
        for (int e = 0; e < KL; ++e) {
            if constexpr (WIDE) load_words_any<BW>(bb + (size_t)e * P * EB + boff, braw[buf][e]);
            else load_words_at<BW>(bb + (size_t)e * P * EB, boff, braw[buf][e]);
        }
        const char* aa = reinterpret_cast<const char*>(W + c0);
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot) load_words_at<4>(aa, aoff[ot], araw[buf][ot]);
    };
    auto products = [&](int buf) {
        if constexpr (EB == 2) {
            bf16x8 b[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u32x4_t v;
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2)
                    v[e2] = __builtin_amdgcn_perm(braw[buf][2 * e2 + 1][t / 2], braw[buf][2 * e2][t / 2], t % 2 ? 0x07060302u : 0x05040100u);
                b[t] = __builtin_bit_cast(bf16x8, v);
            }
#pragma unroll
            for (int ot = 0; ot < NOT; ++ot) {
                const u32x4_t av = {araw[buf][ot][0], araw[buf][ot][1], araw[buf][ot][2], araw[buf][ot][3]};
                const bf16x8 a = __builtin_bit_cast(bf16x8, av);
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[ot][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[t], acc[ot][t], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int e = 0; e < KL; ++e)
#pragma unroll
                for (int ot = 0; ot < NOT; ++ot)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        acc[ot][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(araw[buf][ot][e]), __uint_as_float(braw[buf][e][t]),
                                                                          acc[ot][t], 0, 0, 0);
        }
    };
    const int steps = max(0, cend - cbeg) / KS;
    if (steps > 0) {                      // no load in a branch: past the last step it is requested again and not used
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load(d, cbeg + min(d, steps - 1) * KS);
        int k = 0;
        for (; k + DEPTH < steps; k += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                products(d);
                load(d, cbeg + min(k + d + DEPTH, steps - 1) * KS);
                __builtin_amdgcn_sched_barrier(0);         // the compiler would gather the products of all buffers in front of the loads
            }
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (k + d < steps) products(d);
    }
    const int c0 = cbeg + steps * KS;
    if (TAIL && c0 < cend) {                      // the last channels: element by element, zero past the end on both operands
        const int cl = c0 + KL * g;
#pragma unroll
        for (int e = 0; e < KL; ++e) {
            load_words_any<BW>(reinterpret_cast<const char*>(in + (size_t)min(cl + e, cend - 1) * P + s), braw[0][e]);
            if (cl + e >= cend) {
#pragma unroll
                for (int w = 0; w < BW; ++w) braw[0][e][w] = 0u;
            }
        }
#pragma unroll
        for (int ot = 0; ot < NOT; ++ot) {
            const T* row = W + (size_t)min(o0 + 16 * ot + n, rows - 1) * ldw;
            uint32_t v[KL];
#pragma unroll
            for (int e = 0; e < KL; ++e) {
                v[e] = elem_bits(row + min(cl + e, cend - 1));
                if (cl + e >= cend) v[e] = 0u;
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) araw[0][ot][w] = EB == 2 ? (v[(2 * w) % KL] | (v[(2 * w + 1) % KL] << 16)) : v[w % KL];
        }
        products(0);
    }
}

// Whether contract() takes the call: at least one group of positions, W within 32-bit offsets.  (Maps have fewer than 2^27
// positions.)
inline bool contract_fits(long long P, long long wrows, long long ldw, int elem_bytes) {
    return P >= 4 && P < (1LL << 27) && wrows * ldw * elem_bytes < (1LL << 32) - 64;
}
// Whether 32-bit lane offsets reach the positions too: lane group 3 stands 24 (bf16) or 12 (fp32) rows behind the uniform
// base and reads one row on.  85.9 and 82.6 million positions; beyond, the lanes carry 64-bit offsets (WIDE).
inline bool contract_narrow(long long P, int elem_bytes) { return (elem_bytes == 2 ? 25 : 13) * P * elem_bytes < (1LL << 32) - 64; }

}  // namespace scan2d
