// Host side of the backward pass: variant choice, workspace layout, launches.
#include "scan2d_bwd.hpp"

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "scan2d_bwd_variants.hpp"
#include "scan2d_memo.hpp"
#include "scan2d_tuning.hpp"

namespace scan2d {
namespace {

// ------------------------------------------------------------------------------ final sums
// What is left to add up behind the sweeps, in one launch: workgroups below `groups_wgs` form dBm / dCm (sums of the
// partials over the channel groups), the ones behind them dA, dA_v, dDskip and the bias gradient (sums over the batch
// items).
struct SumArgs {
    const float* pB; const float* pC; float* dBm; float* dCm;
    int Bt, CG;
    unsigned groups_wgs;              // 0: one channel group, nothing to add
    size_t per_item;                  // elements of a partial of one batch item
    // partials whose rows are LG*K floats in the lane order of the main sweep, [K/4][LG][4] (K = 0: plain rows): element q
    // of a row is column (q / 4 % LG) * K + (q / (4 * LG)) * 4 + q % 4
    int W, LG, K;
    // sums over batch items, [Bt][n] -> [n], or with S > 1 over batch items and row segments: element e = c * per + k of n is
    // the sum over items b and segments s of src[(b * n / per + c) * map + s * seg + k]
    int S, seg;
    struct Batch { const float* src; float* dst; int n, per; long long map; } batch[4];
};

// S threads per element split the channel groups (thread s: groups s, s + S, ...), 8 loads of each tensor in flight, and
// meet in LDS; the order is fixed.  Bound: HBM for large maps.  S > 1 where one thread per element would leave most of the
// chip's memory path idle: 8 batch items of 14x14 maps and 128 channels took 37 us with S = 1.
template <int S>
__global__ __launch_bounds__(S == 1 ? 256 : 64 * S) void scan2d_bwd_sums_kernel(const SumArgs p) {
    constexpr int THREADS = S == 1 ? 256 : 64 * S, E = THREADS / S;
    __shared__ float sh[S == 1 ? 1 : 2][S][E];
    const int tid = threadIdx.x;
    if (blockIdx.x >= p.groups_wgs) {
        long long e = (long long)(blockIdx.x - p.groups_wgs) * THREADS + tid;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const SumArgs::Batch& t = p.batch[k];
            if (t.dst == nullptr) continue;
            if (e >= 0 && e < t.n) {
                float acc = 0.0f;
                if (p.S == 1) {
                    for (int b = 0; b < p.Bt; b += 8) {    // in order; past the last item it is loaded again
                        float v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) v[u] = t.src[(size_t)min(b + u, p.Bt - 1) * t.n + e];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (b + u < p.Bt) acc += v[u];
                    }
                } else {
                    const int c = (int)e / t.per, k = (int)e - c * t.per, channels = t.n / t.per;
                    // one chain of loads of an item's segments each: requested eight at a time, added in the same order (32 batch
                    // items of 8 segments, one channel of 91x26 fp32: the whole backward 145 -> 121 us)
                    const long long total = (long long)p.Bt * p.S;
                    int b = 0, s = 0;                      // of the next load; past the last one it is loaded again
                    for (long long i = 0; i < total; i += 8) {
                        float v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            v[u] = t.src[((size_t)b * channels + c) * t.map + s * p.seg + k];
                            if (s + 1 < p.S) ++s;
                            else if (b + 1 < p.Bt) { ++b; s = 0; }
                        }
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (i + u < total) acc += v[u];
                    }
                }
                t.dst[e] = acc;
            }
            e -= t.n;
        }
        return;
    }
    const size_t per = p.per_item, total = (size_t)p.Bt * per;
    const int s = tid / E, CG = p.CG;
    for (size_t base = (size_t)blockIdx.x * E; base < total; base += (size_t)p.groups_wgs * E) {
        const size_t e = min(base + tid % E, total - 1);
        const size_t b = e / per, r = e - b * per;
        const float* sB = p.pB + b * CG * per + r;
        const float* sC = p.pC + b * CG * per + r;
        float aB = 0.0f, aC = 0.0f;
        int g = s;
        for (; g + 7 * S < CG; g += 8 * S) {
            float vB[8], vC[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { vB[u] = sB[(size_t)(g + u * S) * per]; vC[u] = sC[(size_t)(g + u * S) * per]; }
#pragma unroll
            for (int u = 0; u < 8; ++u) { aB += vB[u]; aC += vC[u]; }
        }
        for (; g < CG; g += S) { aB += sB[(size_t)g * per]; aC += sC[(size_t)g * per]; }
        if constexpr (S > 1) {
            sh[0][s][tid % E] = aB;
            sh[1][s][tid % E] = aC;
            __syncthreads();
            if (s == 0) {
#pragma unroll
                for (int k = 1; k < S; ++k) { aB += sh[0][k][tid]; aC += sh[1][k][tid]; }
            }
            __syncthreads();
            if (s != 0) continue;
        }
        if (base + tid % E >= total) continue;
        size_t o = e;
        if (p.K > 0) {
            const size_t panel = (size_t)p.LG * p.K, row = e / panel;
            const int q = (int)(e - row * panel);
            const int col = (q / 4 % p.LG) * p.K + (q / (4 * p.LG)) * 4 + q % 4;
            if (col >= p.W) continue;
            o = row * p.W + col;
        }
        p.dBm[o] = aB;
        p.dCm[o] = aC;
    }
}

// Softplus step, banded form: the step is computed once per position here, as fp32 whatever the storage
// type, instead of by each of a map's lane groups in both sweeps (16-fold in the main sweep for N = 16: a
// fifth of its run time); the SP instantiations of the sweeps read it.  One workgroup per 1024 positions of
// a map (`chunks` per map).
template <typename T>
__global__ __launch_bounds__(256) void scan2d_bwd_step_kernel(const T* __restrict__ raw, const float* __restrict__ bias,
                                                              float* __restrict__ step, size_t HW, int Dc, unsigned chunks) {
    const size_t map = blockIdx.x / chunks;
    const float b = bias != nullptr ? bias[map % Dc] : 0.0f;
    const T* src = raw + map * HW;
    float* dst = step + map * HW;
    const size_t e0 = ((size_t)(blockIdx.x % chunks) * 256 + threadIdx.x) * 4;
    if (e0 + 4 <= HW && (Elem<T>::kBytes == 4 || (HW & 1) == 0)) {      // four elements at once (rows of a map stay 4-byte aligned)
        uint32_t r[words_of<T, 4>()], o[4];
        load_words<words_of<T, 4>()>(reinterpret_cast<const uint32_t*>(src + e0), r);
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = __float_as_uint(softplus_f32(get_elem<T, 4>(r, j) + b));
        store_words<4>(reinterpret_cast<uint32_t*>(dst + e0), o);
        return;
    }
    for (size_t e = e0; e < e0 + 4 && e < HW; ++e) {
        float t;
        if constexpr (Elem<T>::kBytes == 4) t = __uint_as_float(elem_bits(src + e));
        else t = __uint_as_float(elem_bits(src + e) << 16);
        dst[e] = softplus_f32(t + b);
    }
}

// The matching chain rule: `dstep` (fp32, the gradient of the step as the main sweep left it in the workspace)
// becomes the gradient of the raw projection, ddelta_raw = dstep / (1 + exp(-(raw + bias))), rounded once to
// the storage type; its sum over the map's positions, taken from the stored values, goes to pbias (null: no
// bias) in a fixed order (strided partial sums per thread, then a tree over the workgroup).
// Bound: HBM.  A workgroup per map, because the sum is one per map, with 4 elements per load.  A slide's few hundred maps
// are a workgroup per compute unit, so each brings 16 wavefronts (211x397 bf16, 256 maps: 4 wavefronts and single elements
// 161 us, this 68); maps of a few elements per thread would wait for the barriers of its sum, so below 8192 elements it is 4
// (us with 4 and 16 wavefronts: 4096 maps of 20x20 6.7 and 16.7, of 56x56 19.2 and 26.8, 1024 of 80x80 11.6 and 12.7, of
// 100x100 23.5 and 22.5, 256 of 100x100 6.4 and 5.5).  Any alignment: maps of odd size start on odd elements.
constexpr int kChainThreads = 1024;                        // the most
inline int chain_threads(size_t HW) { return HW >= 8192 ? kChainThreads : 256; }      // a power of two, for the tree
template <typename T>
__global__ __launch_bounds__(kChainThreads) void scan2d_bwd_chain_kernel(const float* __restrict__ dstep, const T* __restrict__ raw,
                                                                         const float* __restrict__ bias, T* __restrict__ ddelta_raw,
                                                                         float* __restrict__ pbias, size_t HW, int Dc) {
    __shared__ float sh[kChainThreads];
    const size_t map = blockIdx.x;
    const float b = bias != nullptr ? bias[map % Dc] : 0.0f;
    const float* dd = dstep + map * HW;
    const T* src = raw + map * HW;
    T* dst = ddelta_raw + map * HW;
    float acc = 0.0f;
    auto stored = [](uint32_t bits) { return Elem<T>::kBytes == 4 ? __uint_as_float(bits) : __uint_as_float(bits << 16); };
    const size_t groups = HW / 4;
    const unsigned step = blockDim.x;
#pragma unroll 2
    for (size_t g = threadIdx.x; g < groups; g += step) {
        constexpr int XW = words_of<T, 4>();
        uint32_t r[XW], q[4], o[XW] = {};
        load_words_any<XW>(src + 4 * g, r);
        load_words_any<4>(dd + 4 * g, q);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bits = to_elem_bits<T>(__uint_as_float(q[j]) * logistic_f32(get_elem<T, 4>(r, j) + b));
            put_elem<T, 4>(o, j, bits);
            acc += stored(bits);
        }
        store_words_any<XW>(dst + 4 * g, o);
    }
    const size_t e = 4 * groups + threadIdx.x;             // the last HW % 4 elements
    if (e < HW) {
        const uint32_t bits = to_elem_bits<T>(dd[e] * logistic_f32(stored(elem_bits(src + e)) + b));
        store_elem(dst + e, stored(bits));
        acc += stored(bits);
    }
    if (pbias == nullptr) return;                        // uniform over the grid
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = (int)step / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) pbias[map] = sh[0];
}

// Row segments of the main sweep: what the reverse column recurrence g (a*g, the value the row above adds to) holds at the
// first row of every segment but the topmost one (left where BwdArgs says).  The recurrence of a column needs no
// other column, so a lane takes one column and all 16 states of a map (the sweep's tilings have no other number) and walks
// up the rows; same operations in the same order as the sweep, so the segments change no bit of it.  The step and (gated)
// dy * SiLU(z) are formed as in the sweep.
// Bound: vector issue (9 instructions per position, channel and state) and, with few maps, the loads of one row, which are
// requested two rows ahead (256 maps of 211x397 bf16: 125 us).
enum { kGcPlain = 0, kGcSoftplus = 1, kGcGated = 2 };
struct GcarryArgs {
    const void* delta; const float* delta_bias; const float* A; const void* Cm; const void* dy; const void* z;
    float* pB; float* pC;
    int Dc, H, W, seg_rows, GS, CG, part_row;
    unsigned waves, cols;                                  // wavefronts in all; 64-column pieces of a map
};
constexpr int kGcStates = 16;
template <typename T, int FORM>
__global__ __launch_bounds__(256) void scan2d_bwd_gcarry_kernel(const GcarryArgs p) {
    const unsigned id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    if (id >= p.waves) return;
    constexpr int N = kGcStates;
    const unsigned cb = id % p.cols;
    const size_t map = id / p.cols, b = map / p.Dc;
    const int c = (int)(map - b * p.Dc), H = p.H, W = p.W;
    const size_t HW = (size_t)H * W;
    const int col = (int)cb * 64 + (int)(threadIdx.x & 63u);
    const uint32_t lcol = (uint32_t)min(col, W - 1);
    const T* dym = static_cast<const T*>(p.dy) + map * HW;
    const T* dm = static_cast<const T*>(p.delta) + map * HW;
    const T* zm = static_cast<const T*>(p.z) + (FORM == kGcGated ? map * HW : 0);
    const T* Cb = static_cast<const T*>(p.Cm) + b * N * HW;
    const float bias = FORM != kGcPlain && p.delta_bias != nullptr ? p.delta_bias[c] : 0.0f;
    float Ap[N], ga[N];
#pragma unroll
    for (int s = 0; s < N; ++s) {
        Ap[s] = p.A[(size_t)c * N + s] * kLog2e;
        ga[s] = 0.0f;
    }
    auto widen = [](uint32_t bits, auto tag) -> float { return Elem<decltype(tag)>::kBytes == 4 ? __uint_as_float(bits) : __uint_as_float(bits << 16); };
    uint32_t rdy[2], rd[2], rz[2], rC[2][N];
    auto request = [&](int k, int i) {
        const uint32_t o = (uint32_t)max(i, 0) * (uint32_t)W + lcol;
        rdy[k] = elem_bits(dym + o);
        rd[k] = elem_bits(dm + o);
        if constexpr (FORM == kGcGated) rz[k] = elem_bits(zm + o);
#pragma unroll
        for (int s = 0; s < N; ++s) rC[k][s] = elem_bits(Cb + (size_t)s * HW + o);
    };
    const int first = p.seg_rows;                          // the topmost row that is needed
    request(0, H - 1);
    request(1, H - 2);
    int to_store = (H - 1) % p.seg_rows;                   // rows until the next segment's first row
    int seg = (H - 1) / p.seg_rows;
    for (int i = H - 1; i >= first; i -= 2) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (i - k < first) break;
            float step = widen(rd[k], T{});
            if constexpr (FORM != kGcPlain) step = softplus_f32(step + bias);
            float dyv = widen(rdy[k], T{});
            if constexpr (FORM == kGcGated) {
                const float zv = widen(rz[k], T{});
                dyv = dyv * (zv * logistic_f32(zv));
            }
#pragma unroll
            for (int s = 0; s < N; ++s) {
                const float a = __builtin_amdgcn_exp2f(step * Ap[s]);
                ga[s] = a * fmaf(dyv, widen(rC[k][s], T{}), ga[s]);
            }
            request(k, i - k - 2);
            if (to_store == 0) {
                const int ch = c % p.GS;                   // of its job, which reads it for segment seg - 1
                float* dst = (ch < p.seg_rows ? p.pB : p.pC) + (b * p.CG + c / p.GS) * N * H * p.part_row + (size_t)((seg - 1) * p.seg_rows + ch % p.seg_rows) * p.part_row;
                if (col < W) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        dst[(size_t)s * H * p.part_row + col] = ga[s];
                }
                to_store = p.seg_rows;
                --seg;
            }
            --to_store;
        }
    }
}
using GcarryKernel = void (*)(const GcarryArgs);
template <typename T>
GcarryKernel gcarry_kernel(int form) {
    return form == kGcGated ? scan2d_bwd_gcarry_kernel<T, kGcGated>
         : form == kGcSoftplus ? scan2d_bwd_gcarry_kernel<T, kGcSoftplus> : scan2d_bwd_gcarry_kernel<T, kGcPlain>;
}

// Padded copies of the rows behind which the input tensors end (layout: TailRows in scan2d_bwd_kernels.hpp):
// the last row of the last map of x, delta and dy, of the last state plane of Bm and Cm, and of the last
// batch item's mask, each followed by 16 zeros.  The instantiations for widths that are not a multiple of
// the columns per lane read these rows from here, because their last lane reads past the end of a row.
template <typename T>
__global__ __launch_bounds__(256) void scan2d_bwd_tail_kernel(const T* __restrict__ x, const T* __restrict__ delta, const T* __restrict__ dy,
                                                              const T* __restrict__ Bm, const T* __restrict__ Cm,
                                                              const uint8_t* __restrict__ mask, T* __restrict__ tail,
                                                              size_t last_map_row, size_t last_plane_row, size_t last_mask_row, int W) {
    const int ts = W + 16;
    uint8_t* tm = reinterpret_cast<uint8_t*>(tail + 5 * (size_t)ts);
    for (int j = threadIdx.x; j < ts; j += 256) {
        const bool in = j < W;
        T zero;
        if constexpr (Elem<T>::kBytes == 4) zero = 0.0f; else zero.bits = 0;
        tail[j] = in ? x[last_map_row + j] : zero;
        tail[ts + j] = in ? delta[last_map_row + j] : zero;
        tail[2 * (size_t)ts + j] = in ? dy[last_map_row + j] : zero;
        tail[3 * (size_t)ts + j] = in ? Bm[last_plane_row + j] : zero;
        tail[4 * (size_t)ts + j] = in ? Cm[last_plane_row + j] : zero;
        tm[j] = (in && mask != nullptr) ? mask[last_mask_row + j] : (uint8_t)0;
    }
}

struct BwdPlan {
    bool small = false;                                    // one to four wavefronts per map, no bands (scan2d_bwd_small.hpp)
    int LG = 0, K = 0, NW = 0, waves = 0, RB = 0;
    int NG = 0, GS = 0, CG = 0, nb = 0;
    int S = 1, seg_bands = 0;                              // row segments of the main sweep (scan2d_bwd_shared.hpp only), bands of each
    BwdKernels k;
    size_t lds_bytes = 0;
    int panels = 1;                                        // column panels of LG*K columns, one launch of each sweep per panel
    size_t off_hc = 0, off_qc = 0;                         // carries between panels: [panels-1][maps][N][H] and [2][maps][N][H]
    bool shared = false;                                   // main sweep of scan2d_bwd_shared.hpp
    int ck_LG = 0, ck_waves = 0;                           // lane tiling of the checkpoint sweep
    bool step_outside = false;                             // softplus step written by a kernel of its own (plain main sweep)
    bool step_for_ckpt = false;                            // the same for the checkpoint sweep alone (more than two column panels)
    size_t off_step = 0;                                   // the step [maps][H][W] fp32 (either of them), 256 spare bytes behind it
    bool fast = true;                                      // W is a multiple of the columns per lane
    size_t off_tail = 0;                                   // padded copies of the tensors' last rows (TailRows)
    size_t off_ck = 0, off_pB = 0, off_pC = 0, off_pA = 0, off_pD = 0, off_pb = 0, total = 0;   // pb: bias-gradient partials
    bool av = false;                                       // independent decay of the column recurrence
    bool ck_chunked = false;                               // checkpoint rows in the lane order of the two shared-producer sweeps
    bool part_chunked = false;                             // rows of the dBm / dCm partials in the lane order of the main sweep
    size_t off_pAv = 0;                                    // partial sums of dA_v over batch items
};

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

// Tilings whose shared-producer main sweep is the default.  Whole backward, us, plain -> shared: (16,4) 56x56 bf16, 6144
// maps 1417 -> 719; (16,8) 128x128 bf16, 1024 maps 1407 -> 787; (16,12) 128x192 fp32, 2048 maps 3730 -> 2047; (64,4) on 8
// waves, 256 maps of 256x256 bf16 2646 -> 1456, fp32 2484 -> 1579.  The other shared tilings run by the tuning override
// only: (64,4) on 16 waves takes 1501 and 1695 on the last two (plain 2191 and 2014), (32,6) 2496 on the third.
bool shared_by_default(int LG, int K, int NW) { return LG == 16 || (LG == 32 && K == 4) || (LG == 64 && K == 4 && NW == 2); }

}  // namespace
bool allow_large_lds(const void* kernel, size_t bytes);   // scan2d_api.hip
namespace {

bool rank_plan(const scan2d_desc* d, BwdPlan* out, bool sp, bool av) {
    BwdPlan pl;
    pl.av = av;
    const int W = d->W, N = d->N;
    // columns first inside the kernels: only the banded form with the shared-producer main sweep has such
    // instantiations; no plan otherwise (the caller then runs columns first through transposes)
    const bool cf = (d->flags & SCAN2D_FLAG_COLUMNS_FIRST) != 0;
    if (cf && av) return false;
    const TuneValues tb = av ? TuneValues() : tune_get(kTuneBwd);
    if (W <= 16 && d->H <= 16 && N <= 16 && tb.n == 0 && !av && !cf) {
        // small maps: the whole map stays in registers
        pl.small = true;
        const int wpm = N <= 4 ? 1 : (N <= 8 ? 2 : 4);
        pl.LG = 16; pl.K = 1; pl.NW = wpm; pl.waves = 4; pl.RB = d->H;       // NW: states per DPP row over a map's wavefronts
        pl.NG = 4 * wpm; pl.nb = 1; pl.lds_bytes = 0;
        // channels per workgroup: as few partial sums as leave every SIMD two wavefronts
        const long long wgs1 = ((long long)d->Bt * d->Dc * wpm + 3) / 4;
        pl.GS = (int)std::max(1LL, std::min({wgs1 / 512, 8LL, (long long)d->Dc}));
        pl.CG = (d->Dc + pl.GS - 1) / pl.GS;
        pl.k.main = d->dtype == SCAN2D_BF16 ? bwd_small_kernel_bf16(wpm, sp, false) : bwd_small_kernel_f32(wpm, sp, false);
        if (sp) pl.k.main_gate = d->dtype == SCAN2D_BF16 ? bwd_small_kernel_bf16(wpm, true, true) : bwd_small_kernel_f32(wpm, true, true);
        if (pl.k.main == nullptr) return false;
        const size_t maps = (size_t)d->Bt * d->Dc;
        const size_t parts = (size_t)d->Bt * pl.CG * N * d->H * W;
        size_t o = 0;
        pl.off_ck = o;
        pl.off_pB = o; o += pl.CG > 1 ? align_up(parts * sizeof(float)) : 0;
        pl.off_pC = o; o += pl.CG > 1 ? align_up(parts * sizeof(float)) : 0;
        pl.off_pA = o; o += d->Bt > 1 ? align_up(maps * N * sizeof(float)) : 0;
        pl.off_pD = o; o += d->Bt > 1 ? align_up(maps * sizeof(float)) : 0;
        pl.off_pb = o; o += align_up(maps * sizeof(float));
        pl.total = o;
        *out = pl;
        return true;
    }
    int LG, K;
    if (W <= 64) { LG = 16; K = 4; }
    // half-wave groups of 4 columns: two wavefronts per SIMD and all rows of a band in one scan, where 8 columns per lane leave
    // one wavefront per SIMD (us, (16,8) and (32,4): 2048 maps of 128x128 bf16 1271 and 1176, fp32 1415 and 1220; 1024 of 100x100
    // bf16 593 and 507; 256 of 57x83 160 and 145; with 8 and 16 maps there is no difference, 8 of 200x127 242 and 253)
    else if (W <= 128 && N == 16 && !cf && !av && (long long)d->Bt * d->Dc >= 32 && (double)N * d->H * 128.0 * 4.0 < 2147483648.0) { LG = 32; K = 4; }
    else if (W <= 128) { LG = 16; K = 8; }
    else if (W <= 192 && N <= 16) { LG = 16; K = 12; }         // 12 columns x 4 states per lane would not fit the registers
    else if (W <= 256) { LG = 64; K = 4; }
    else if (W <= 512) { LG = 64; K = 8; }
    else if (W <= 1024) { LG = 64; K = 16; }
    else { LG = 64; K = 4; }
    // maps wider than the widest tiling (and, beyond 16 states, wider than 256 columns: the band arrays of four
    // states per lane and 16 waves fill the LDS) are swept in panels of 256 columns
    // (faster than the 8- and 16-column tilings from 257 columns on; 256 maps, us: 300x300 fp32 3070 against 4709, 400x400
    // bf16 4315 against 6657, 512x512 bf16 5757 against 9535, 600x600 bf16 11180 against 26660)
    if (W > 256 || av) { LG = 64; K = 4; pl.panels = (W + 255) / 256; }
    int force_waves = 0, force_gs = 0, force_seg = 0, want_shared = -1;
    if (tb.n >= 1) {                                             // tuning aid: LG,K[,WAVES[,GS[,shared[,segments]]]]
        const int eLG = tb.v[0], eK = tb.v[1], eW = tb.v[2], eG = tb.v[3];
        const int got = tb.n;
        if (got >= 2 && (eLG == 16 || eLG == 32 || eLG == 64) && eLG * eK >= W && W <= 1024 && (N <= 16 || W <= 256)) {
            LG = eLG; K = eK; pl.panels = 1;                     // a single-panel tiling forced on a map it covers
        }
        if (got >= 3) force_waves = eW;
        if (got >= 4) force_gs = eG;
        if (got >= 5) want_shared = tb.v[4];
        if (got >= 6) force_seg = tb.v[5];
    }
    // states per lane and waves per workgroup: 16 lane groups of one DPP row with one state each;
    // wavefront-wide lane groups: 16 of them with one state each for 4 columns per lane (four waves
    // per SIMD: measured 20-30 % faster than 8 groups of two states), 8 with two states each for 8
    // columns; four states per lane beyond N = 16
    int waves, NW;
    if (LG == 16) { waves = 4; NW = N <= 16 ? 1 : 4; }
    else if (LG == 32) { waves = 8; NW = 1; }
    else if (N <= 16 && K == 16) { waves = 4; NW = 4; }     // widest maps: LDS bounds the workgroup size
    // (one panel of 16 states: two states per lane on 8 waves with the shared-producer main sweep, 256 maps of 256x256 bf16
    // 1456 us, against 2191 on 16 waves of one state that each repeat the per-position work)
    else if (N == 16 && K == 4 && !av && want_shared != 0 && force_waves != 16) { waves = 8; NW = 2; }
    else if (N <= 16 && K == 4 && force_waves != 8) { waves = 16; NW = 1; }
    else if (N <= 16) { waves = 8; NW = 2; }
    else { waves = 16; NW = 4; }
    const int slots = waves * 64 / LG;
    if ((N + NW - 1) / NW > slots) return false;
    const bool fast = (W % K) == 0;                          // otherwise: the instantiations that treat the row end
    pl.fast = fast;
    // the main sweep that shares the per-position work through LDS, where it exists for this tiling (N = NG * NW)
    // (its kernels take column panels too; their 32-bit offsets span one item's state planes)
    if (want_shared != 0 && N % NW == 0 && !av && (double)N * d->H * std::max(W, LG * K) * 4.0 < 2147483648.0) {
        BwdKernels ks;
        if (cf) ks = d->dtype == SCAN2D_BF16 ? bwd_shared_kernels_bf16_cf(LG, K, NW, N / NW, waves, W, sp)
                                             : bwd_shared_kernels_f32_cf(LG, K, NW, N / NW, waves, W, sp);
        else ks = d->dtype == SCAN2D_BF16 ? bwd_shared_kernels_bf16(LG, K, NW, N / NW, waves, W, sp)
                                          : bwd_shared_kernels_f32(LG, K, NW, N / NW, waves, W, sp);
        if (pl.panels > 1) { ks.main = ks.main_panels; ks.main_gate = ks.main_panels_gate; }      // column panels: the instantiations that take them, if any
        if (ks.main != nullptr && (want_shared == 1 || shared_by_default(LG, K, NW))) pl.k = ks;
    }
    if (cf && pl.k.main == nullptr) return false;
    if (av) {
        if (sp) return false;
        pl.k = d->dtype == SCAN2D_BF16 ? bwd_kernels_av_bf16(NW, fast) : bwd_kernels_av_f32(NW, fast);
    }
    if (pl.k.main == nullptr)
        pl.k = d->dtype == SCAN2D_BF16 ? bwd_kernels_bf16(LG, K, NW, waves, fast, sp) : bwd_kernels_f32(LG, K, NW, waves, fast, sp);
    if (pl.k.main == nullptr) return false;
    pl.shared = pl.k.shared;
    // the shared-producer sweeps apply the softplus and its chain rule themselves (their checkpoint sweep, the shared-producer
    // forward kernel, computes the step from the raw projection too; the plain checkpoint sweep of many panels reads it)
    pl.step_outside = sp && !pl.shared;
    pl.step_for_ckpt = sp && pl.shared && pl.panels > 1 && pl.k.ckpt_wide == nullptr;
    pl.fast = fast && pl.k.ckpt_fast;                        // false: the padded copies of the tensors' last rows are needed
    pl.ck_LG = pl.k.ckpt_LG; pl.ck_waves = pl.k.ckpt_waves;
    pl.LG = LG; pl.K = K; pl.NW = NW; pl.waves = waves; pl.RB = pl.k.RB;
    pl.NG = (N + NW - 1) / NW;
    pl.nb = (d->H + pl.RB - 1) / pl.RB;
    // Channels a workgroup handles one after the other (bounded by the 160 KB of LDS) and row segments per map, by an
    // estimate of the whole call in us:
    //   * rounds of resident workgroups (the runtime's occupancy figure for the kernel's registers and this much LDS, one per
    //     CU if it cannot be asked) times (band, channel) steps of a workgroup.
    //     The plain sweep repeats the per-position work in every lane group and takes about twice as long per step (with the
    //     shared sweep's figure it got too many channels: 256 maps of 84x1174 fp32, N = 12, one and two channels 3704 and 4541);
    //   * the dBm / dCm partials, one per channel group, written here and read by the reduction;
    //   * with segments, the pass in front of the sweep that forms what enters each from below.
    // More channels mean fewer partials, more segments keep the chip busy all the same: one slide of 256 channels of 211x397
    // bf16 has 256 maps, one for each CU, and without segments a partial per channel (us, one segment and now: the two panels'
    // sweeps 1648 and 1041, the partials' sum 526 and 93, the pass in front 125; the whole training step 2931 and 1975).
    // More than 8 channels: 6144 maps of 56x56 bf16 take 12 instead of 6, partials' sum 104 -> 42 us.
    // The constants are a fit to whole calls.  Checked for the shared sweep (0.12, 5.0, the partials' rates, the pass) on 1788 plans of 64
    // shapes of 16 states, 20 to 400 a side: the one taken is 1.9 % slower than the best in the geometric mean, 15 % at most (32 items
    // of 64 channels of 32x32: 16 channels in 4 segments 155 us, 4 in one 135).  For the plain sweep (0.28) on 486 plans of 70 shapes of 4 to
    // 64 states: 0.3 %, 9 % at most, with 0.25; 4 x 192 maps of 47x47, 8 states, then took two channels and 243 us where one takes 200.
    const size_t T = (size_t)waves * 64;
    size_t fixed = 4 * T * K, per = T * ((size_t)NW * K + NW + 1);
    if (pl.shared) { fixed = pl.k.lds_fixed; per = pl.k.lds_per_channel; }
    const int gs_lds = (int)std::max<size_t>(1, (40960 - std::min<size_t>(fixed, 40960)) / per);
    const int JPW = slots / pl.NG;
    const int gs_max = av ? 1 : std::min({gs_lds, 16, d->Dc});   // av: one channel per workgroup (its dA_v partial stays in registers)
    const size_t maps = (size_t)d->Bt * d->Dc;
    const bool tight = (size_t)LG * K * 15 <= (size_t)W * 16;
    auto layout = [&](BwdPlan& q) {
        size_t o = 0;
        // the shared-producer forward kernel writes the checkpoints and the shared-producer main sweep reads them with the same
        // lane tiling: rows of LG*K floats in lane order, so that both move whole 16-byte x LG pieces per instruction
        // (only where the padding of the rows to LG*K columns costs less than 7 %)
        q.ck_chunked = tight && q.shared && q.panels == 1 && q.k.ckpt_fwd != nullptr && N == q.k.cf_NG * q.k.cf_NW && q.k.cf_LG == LG &&
                       q.k.cf_K == K && K % 4 == 0;
        q.off_ck = o; o += align_up(maps * q.nb * N * (q.ck_chunked ? (size_t)LG * K : (size_t)W) * sizeof(float));
        q.part_chunked = tight && q.shared && q.panels == 1 && q.CG > 1 && K % 4 == 0;
        const size_t part_row = q.part_chunked ? (size_t)LG * K : (size_t)W;
        q.off_pB = o; o += q.CG > 1 ? align_up((size_t)d->Bt * q.CG * N * d->H * part_row * sizeof(float)) : 0;
        q.off_pC = o; o += q.CG > 1 ? align_up((size_t)d->Bt * q.CG * N * d->H * part_row * sizeof(float)) : 0;
        q.off_pA = o; o += d->Bt > 1 ? align_up(maps * N * sizeof(float)) : 0;
        q.off_pD = o; o += d->Bt > 1 ? align_up(maps * sizeof(float)) : 0;
        q.off_pb = o; o += align_up(maps * sizeof(float));
        q.off_step = o; o += q.step_outside || q.step_for_ckpt ? align_up(maps * (size_t)d->H * W * sizeof(float)) + 256 : 0;
        q.off_tail = o; o += align_up((size_t)(W + 16) * (5 * (d->dtype == SCAN2D_BF16 ? 2 : 4) + 1));
        if (av) { q.off_pAv = o; o += d->Bt > 1 ? align_up(maps * N * sizeof(float)) : 0; }
        if (q.panels > 1) {
            const size_t one = align_up(maps * N * (size_t)d->H * sizeof(float));
            q.off_hc = o; o += (size_t)(q.panels - 1) * one;
            q.off_qc = o; o += 2 * one;
        }
        q.total = o;
    };
    auto set = [&](int gs, int segments) {
        BwdPlan q = pl;
        q.GS = gs;
        q.CG = (d->Dc + gs - 1) / gs;
        q.seg_bands = (q.nb + segments - 1) / segments;
        q.S = (q.nb + q.seg_bands - 1) / q.seg_bands;
        q.lds_bytes = (fixed + (size_t)gs * per) * sizeof(float);
        layout(q);
        return q;
    };
    // The segments' sums over the map, N + 2 floats each, lie in the checkpoints' row of a map's first band, which has at least
    // N * W floats: 18 of 16 * W, so that maps below 17 columns take fewer than 15 segments (a single column none).
    const int held = std::min(15, d->N * std::min(W, 17) / (d->N + 2));
    const double units = (double)pl.RB * K * NW, cells = (double)d->N * d->H * W;      // of a step per lane; of a map
    double best_us = -1.0, fit_us = -1.0;
    long long plain_path = -1;
    BwdPlan best, fit, plain;                                  // the best; the best within the scratch array; the shortest without segments
    for (int g = 1; g <= gs_max; ++g) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(pl.k.main), (int)T,
                                                         (fixed + (size_t)g * per) * sizeof(float)) != hipSuccess || per_cu < 1) {
            (void)hipGetLastError();
            per_cu = 1;
        }
        // What enters the segments lies in their own rows of the partial sums.  (The pass in front counts its wavefronts in 32 bits.)
        const bool segs = pl.shared && !cf && N == kGcStates && (double)maps * ((W + 63) / 64) < 1073741824.0;
        const int most = segs ? std::max(1, std::min(held, pl.nb / 2)) : 1;
        int last = 0;
        for (int segments = 1; segments <= most; ++segments) {
            const BwdPlan q = set(g, segments);
            if (q.S == last || (q.S > 1 && g > 2 * q.seg_bands * q.RB)) continue;
            last = q.S;
            const double wgs = std::ceil((double)d->Bt * q.CG * q.S / JPW);
            const double resident = 256.0 * per_cu, rounds = std::ceil(wgs / resident);
            const double wps = std::min((double)per_cu, std::ceil(wgs / 256.0)) * waves / 4.0;
            double us = rounds * pl.panels * (5.0 + g * q.seg_bands * units * (pl.shared ? 0.12 : 0.28) * (0.5 + 0.5 * std::max(1.0, wps)));
            if (q.CG > 1) us += 2.0 * d->Bt * q.CG * cells * 4.0 * (1.0 / 4.0e6 + 1.0 / 5.0e6);
            if (q.S > 1) {
                const double up = 1.0 - 1.0 / q.S;
                us += 6.0 + std::max((double)maps * cells * up / 2.2e6, d->H * up * 0.3);
            }
            const auto better = [&](double than, const BwdPlan& p) {
                return than < 0.0 || us < than * (1.0 - 1e-9) || (us <= than * (1.0 + 1e-9) && q.S == p.S);
            };
            if (better(best_us, best)) { best_us = us; best = q; }
            if (q.total <= SCAN2D_STATIC_SCRATCH_BYTES && better(fit_us, fit)) { fit_us = us; fit = q; }
            if (q.S == 1 && g <= 8 && (plain_path < 0 || (long long)rounds * g <= plain_path)) { plain_path = (long long)rounds * g; plain = q; }
        }
    }
    // scan2d_bwd_static_scratch takes what fits its array with the fewest rounds of workgroups and up to 8 channels each;
    // such a shape has to fit it with the plan chosen here too
    if (best.total > SCAN2D_STATIC_SCRATCH_BYTES && plain.total <= SCAN2D_STATIC_SCRATCH_BYTES) best = fit;
    if (force_gs >= 1 && force_gs <= gs_lds && force_gs <= d->Dc) best = set(force_gs, 1);
    if (force_seg >= 1 && pl.shared && !cf && N == kGcStates && maps < 1000000) {
        const BwdPlan q = set(best.GS, std::max(1, std::min({force_seg, best.nb, held})));
        if (q.S == 1 || q.GS <= 2 * q.seg_bands * q.RB) best = q;      // ignored where the segments' rows do not hold what enters them
    }
    if (best.lds_bytes > 160 * 1024) return false;
    *out = best;
    return true;
}

bool make_plan(const scan2d_desc* d, BwdPlan* out, bool sp = false, bool av = false) {
    thread_local PlanMemo<BwdPlan> memo;
    return memo.get(*d, (sp ? 1u : 0u) | (av ? 2u : 0u), out, [&](BwdPlan* p) { return rank_plan(d, p, sp, av) ? 0 : 1; }) == 0;
}

// Workgroups of the small-map kernel: pl.NG lane groups (DPP rows) per map, 16 per workgroup.
long long small_wgs(const scan2d_desc* d, const BwdPlan& pl) { return ((long long)d->Bt * pl.CG * pl.NG + 15) / 16; }

}  // namespace

size_t bwd_workspace_bytes(const scan2d_desc* d, bool softplus, bool av) {
    BwdPlan pl;
    return make_plan(d, &pl, softplus, av) ? pl.total : 0;
}

// Everything bwd_launch could refuse, without enqueuing anything: the plan and the grid sizes of its launches.
int bwd_check(const scan2d_desc* d, bool softplus, bool av) {
    BwdPlan pl;
    if (!make_plan(d, &pl, softplus, av)) return SCAN2D_ERR_BAD_SHAPE;
    const long long maps = (long long)d->Bt * d->Dc;
    if (pl.small) return small_wgs(d, pl) > 2147483647LL ? SCAN2D_ERR_BAD_SHAPE : SCAN2D_OK;
    const int MPW = (pl.waves * 64 / pl.LG) / pl.NG;
    const int ck_NG = (d->N + pl.k.ckpt_NW - 1) / pl.k.ckpt_NW;
    const int MPW1 = (pl.ck_waves * 64 / pl.ck_LG) / ck_NG;
    const long long wg1 = (maps + MPW1 - 1) / MPW1, wg2 = ((long long)d->Bt * pl.CG * pl.S + MPW - 1) / MPW;
    if (wg1 > 2147483647LL || wg2 > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    const long long chunks = ((long long)d->H * d->W + 1023) / 1024;
    if ((pl.step_outside || pl.step_for_ckpt) && chunks * maps > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    return SCAN2D_OK;
}

namespace {
bool saving_plan(const scan2d_desc* d, BwdPlan* pl) {
    if (d->flags != 0u || !make_plan(d, pl)) return false;
    return !pl->small && pl->panels == 1 && pl->nb > 1 && pl->k.train_fwd != nullptr && d->N == pl->k.cf_NG * pl->k.cf_NW;
}
}  // namespace

size_t bwd_saved_bytes(const scan2d_desc* d) {
    BwdPlan pl;
    if (!saving_plan(d, &pl)) return 0;
    const size_t rows = align_up((size_t)d->Bt * d->Dc * pl.nb * d->N * (pl.ck_chunked ? (size_t)pl.LG * pl.K : (size_t)d->W) * sizeof(float));
    // rows by column: the lane across the row end reads all of its K columns, behind the last row up to 4 (K - 1) bytes
    return rows + (!pl.ck_chunked && d->W % pl.K != 0 ? 256 : 0);
}

int fwd_saving_launch(const scan2d_desc* d, const void* x, const void* delta, const float* A, const void* Bm, const void* Cm,
                      const float* Dskip, const uint8_t* mask, void* y, float* saved, hipStream_t stream) {
    BwdPlan pl;
    if (!saving_plan(d, &pl)) return SCAN2D_ERR_BAD_SHAPE;
    const long long maps = (long long)d->Bt * d->Dc;
    FwdArgs f;
    f.x = x; f.delta = delta; f.A = A; f.Bm = Bm; f.Cm = Cm; f.Dskip = Dskip; f.mask = mask; f.y = y;
    f.delta_bias = nullptr; f.carry = nullptr;
    f.ck = saved; f.nb = pl.nb; f.ck_chunked = pl.ck_chunked ? 1 : 0;
    f.maps = maps; f.Dc = d->Dc; f.H = d->H; f.W = d->W; f.N = d->N;
    const int slots = pl.k.cf_waves * 64 / pl.k.cf_LG;
    f.NG = pl.k.cf_NG; f.MPW = slots / pl.k.cf_NG; f.panels = 1; f.RPB = pl.k.cf_RPB;
    const long long wgf = (maps + f.MPW - 1) / f.MPW;
    if (wgf > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    const size_t panel = (size_t)pl.k.cf_LG * pl.k.cf_K;
    const size_t lds = (2 * (size_t)f.MPW * f.RPB * 2 * panel + 2 * (size_t)f.RPB * slots * panel) * sizeof(float);
    if (lds > 160 * 1024) return SCAN2D_ERR_BAD_SHAPE;
    (void)hipGetLastError();
    if (lds > 65536 && !allow_large_lds(reinterpret_cast<const void*>(pl.k.train_fwd), lds)) return SCAN2D_ERR_LAUNCH_FAILED;
    hipLaunchKernelGGL(pl.k.train_fwd, dim3((unsigned)wgf), dim3(pl.k.cf_waves * 64), lds, stream, f);
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

bool bwd_describe(const scan2d_desc* d, char* text, size_t text_bytes) {
    BwdPlan pl;
    if (!make_plan(d, &pl)) return false;
    long long wgs;
    if (pl.small) wgs = small_wgs(d, pl);
    else {
        const int per_wg = (pl.waves * 64 / pl.LG) / pl.NG;
        wgs = ((long long)d->Bt * pl.CG * pl.S + per_wg - 1) / per_wg;
    }
    std::snprintf(text, text_bytes, "%sbwd form=%s LG=%d K=%d NW=%d waves=%d RB=%d GS=%d CG=%d bands=%d panels=%d segments=%d wgs=%lld lds=%zu workspace=%zu",
                  (d->flags & SCAN2D_FLAG_COLUMNS_FIRST) != 0 ? "columns-first(in-kernel) " : "",
                  pl.small ? "small" : (pl.shared ? "banded-shared" : "banded"), pl.LG, pl.K, pl.NW, pl.waves, pl.RB, pl.GS, pl.CG, pl.nb,
                  pl.panels, pl.S, wgs, pl.lds_bytes, pl.total);
    return true;
}

bool bwd_gate_in_sweep(const scan2d_desc* d) {
    BwdPlan pl;
    return d->flags == 0u && make_plan(d, &pl, true, false) && (pl.small || pl.shared) &&
           pl.k.main_gate != nullptr;
}

namespace {
// The sums behind the sweeps (scan2d_bwd_sums_kernel): channel groups, if there are several, and batch items, if there
// are several.
void launch_sums(const scan2d_desc* d, const BwdPlan& pl, const BwdArgs& a, float* dBm, float* dCm, float* dA, float* dA_v, float* dDskip,
                 float* dbias, const float* pbias, hipStream_t stream) {
    SumArgs s;
    s.pB = a.pB; s.pC = a.pC; s.dBm = dBm; s.dCm = dCm; s.Bt = d->Bt; s.CG = pl.CG; s.W = d->W;
    s.LG = pl.part_chunked ? pl.LG : 0;
    s.K = pl.part_chunked ? pl.K : 0;
    s.per_item = (size_t)d->N * d->H * (pl.part_chunked ? (size_t)pl.LG * pl.K : (size_t)d->W);
    const size_t total = (size_t)d->Bt * s.per_item;
    // threads per element: until about 400000 threads read, with at least two groups each
    int S = total >= 400000 || pl.CG < 8 ? 1 : (total >= 100000 || pl.CG < 32 ? 4 : 16);
    const unsigned E = S == 1 ? 256 : 64, threads = S == 1 ? 256 : 64 * S;
    s.groups_wgs = pl.CG > 1 ? (unsigned)std::min<size_t>((total + E - 1) / E, 16384) : 0;
    size_t n = 0;
    for (auto& t : s.batch) t = {nullptr, nullptr, 0, 1, 0};
    s.S = pl.S; s.seg = a.sum_seg;
    if (d->Bt > 1 || pl.S > 1) {
        s.batch[0] = {a.pA, dA, d->Dc * d->N, d->N, a.sum_map};
        if (dDskip != nullptr) s.batch[1] = {a.pD, dDskip, d->Dc, 1, a.sum_map1};
        if (dbias != nullptr) s.batch[2] = {pbias, dbias, d->Dc, 1, a.sum_map1};      // (plain sweeps: one segment, summed by the chain kernel)
        if (dA_v != nullptr) s.batch[3] = {a.pAv, dA_v, d->Dc * d->N, d->N, a.sum_map};
    }
    for (const auto& t : s.batch) n += (size_t)t.n;
    const unsigned wgs = s.groups_wgs + (unsigned)((n + threads - 1) / threads);
    if (wgs == 0) return;
    if (S == 1) hipLaunchKernelGGL(scan2d_bwd_sums_kernel<1>, dim3(wgs), dim3(threads), 0, stream, s);
    else if (S == 4) hipLaunchKernelGGL(scan2d_bwd_sums_kernel<4>, dim3(wgs), dim3(threads), 0, stream, s);
    else hipLaunchKernelGGL(scan2d_bwd_sums_kernel<16>, dim3(wgs), dim3(threads), 0, stream, s);
}
}  // namespace

int bwd_launch(const scan2d_desc* d, const void* x, const void* delta, const float* delta_bias, bool softplus,
               const float* A, const void* Bm,
               const void* Cm, const float* Dskip, const uint8_t* mask, const void* dy, void* dx,
               void* ddelta, float* ddelta_bias, float* dA, float* dBm, float* dCm, float* dDskip, void* workspace,
               size_t workspace_bytes, hipStream_t stream, const float* A_v, float* dA_v, const float* saved,
               const void* z, const void* y_scan, void* dz) {
    BwdPlan pl;
    if (!make_plan(d, &pl, softplus, A_v != nullptr)) return SCAN2D_ERR_BAD_SHAPE;
    if (z != nullptr) {                                        // the output gate's backward inside the main sweep
        if (!softplus || y_scan == nullptr || dz == nullptr || pl.k.main_gate == nullptr || !(pl.small || pl.shared))
            return SCAN2D_ERR_BAD_SHAPE;
        pl.k.main = pl.k.main_gate;
    }
    if (pl.total > 0 && (workspace == nullptr || workspace_bytes < pl.total)) return SCAN2D_ERR_WORKSPACE_SMALL;
    char* ws = static_cast<char*>(workspace);
    BwdArgs a;
    a.x = x; a.delta = delta; a.A = A; a.Bm = Bm; a.Cm = Cm; a.Dskip = Dskip; a.mask = mask; a.dy = dy;
    a.dx = dx; a.ddelta = ddelta; a.delta_bias = delta_bias;
    a.z = z; a.y_scan = y_scan; a.dz = dz;
    if (pl.step_outside) a.delta = ws + pl.off_step;
    a.tail = pl.small ? nullptr : ws + pl.off_tail;
    a.ck = saved != nullptr ? const_cast<float*>(saved) : reinterpret_cast<float*>(ws + pl.off_ck);
    a.pB = pl.CG > 1 ? reinterpret_cast<float*>(ws + pl.off_pB) : dBm;   // one group: the partial is the result
    a.pC = pl.CG > 1 ? reinterpret_cast<float*>(ws + pl.off_pC) : dCm;
    a.pA = d->Bt > 1 ? reinterpret_cast<float*>(ws + pl.off_pA) : dA;
    a.pD = dDskip == nullptr ? nullptr : (d->Bt > 1 ? reinterpret_cast<float*>(ws + pl.off_pD) : dDskip);
    a.sum_map = d->N; a.sum_map1 = 1; a.sum_seg = 0;
    if (pl.S > 1) {                                            // N, 1 and 1 floats per segment in the checkpoint row of band 0
        float* row = reinterpret_cast<float*>(ws + pl.off_ck);
        a.sum_map = a.sum_map1 = (long long)pl.nb * d->N * (pl.ck_chunked ? pl.LG * pl.K : d->W);
        a.sum_seg = d->N + 2;
        a.pA = row;
        a.pD = dDskip != nullptr ? row + d->N : nullptr;
    }
    a.Bt = d->Bt; a.Dc = d->Dc; a.H = d->H; a.W = d->W; a.N = d->N;
    a.NG = pl.NG; a.GS = pl.GS; a.CG = pl.CG; a.nb = pl.nb;
    a.S = pl.S; a.seg_bands = pl.seg_bands;
    a.A_v = A_v;
    a.ck_chunked = pl.ck_chunked ? 1 : 0;
    a.part_chunked = pl.part_chunked ? 1 : 0;
    a.pAv = A_v == nullptr ? nullptr : (d->Bt > 1 ? reinterpret_cast<float*>(ws + pl.off_pAv) : dA_v);
    // the sweeps that apply the softplus themselves also add up ddelta_raw per map
    float* const pbias = softplus && ddelta_bias != nullptr ? (pl.S > 1 ? a.pA + d->N + 1 : (d->Bt > 1 ? reinterpret_cast<float*>(ws + pl.off_pb) : ddelta_bias)) : nullptr;
    if (!pl.step_outside) a.pBias = pbias;

    const long long maps = (long long)d->Bt * d->Dc;
    if (pl.small) {
        const long long wgs = small_wgs(d, pl);
        if (wgs > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
        (void)hipGetLastError();
        hipLaunchKernelGGL(pl.k.main, dim3((unsigned)wgs), dim3(256), 0, stream, a);
        launch_sums(d, pl, a, dBm, dCm, dA, nullptr, dDskip, softplus ? ddelta_bias : nullptr, pbias, stream);
        return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
    }
    const int MPW = (pl.waves * 64 / pl.LG) / pl.NG;
    BwdArgs ac = a;                                            // the checkpoint sweep may hold more states per lane
    if (pl.step_for_ckpt) ac.delta = ws + pl.off_step;
    ac.NG = (d->N + pl.k.ckpt_NW - 1) / pl.k.ckpt_NW;
    const int MPW1 = (pl.ck_waves * 64 / pl.ck_LG) / ac.NG;
    const long long wg1 = (maps + MPW1 - 1) / MPW1;
    const long long jobs = (long long)d->Bt * pl.CG * pl.S;
    const long long wg2 = (jobs + MPW - 1) / MPW;
    if (wg1 > 2147483647LL || wg2 > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
    (void)hipGetLastError();
    const size_t HW = (size_t)d->H * d->W;
    if (!pl.fast) {
        const size_t r1 = ((size_t)maps - 1) * HW + (size_t)(d->H - 1) * d->W;
        const size_t r2 = ((size_t)d->Bt * d->N - 1) * HW + (size_t)(d->H - 1) * d->W;
        const size_t r3 = ((size_t)d->Bt - 1) * HW + (size_t)(d->H - 1) * d->W;
        if (d->dtype == SCAN2D_BF16)
            hipLaunchKernelGGL(scan2d_bwd_tail_kernel<bf16_t>, dim3(1), dim3(256), 0, stream, static_cast<const bf16_t*>(x),
                               static_cast<const bf16_t*>(delta), static_cast<const bf16_t*>(dy), static_cast<const bf16_t*>(Bm),
                               static_cast<const bf16_t*>(Cm), mask, reinterpret_cast<bf16_t*>(ws + pl.off_tail), r1, r2, r3, d->W);
        else
            hipLaunchKernelGGL(scan2d_bwd_tail_kernel<float>, dim3(1), dim3(256), 0, stream, static_cast<const float*>(x),
                               static_cast<const float*>(delta), static_cast<const float*>(dy), static_cast<const float*>(Bm),
                               static_cast<const float*>(Cm), mask, reinterpret_cast<float*>(ws + pl.off_tail), r1, r2, r3, d->W);
    }
    if (pl.step_outside || pl.step_for_ckpt) {
        const unsigned chunks = (unsigned)((HW + 1023) / 1024);
        if ((long long)chunks * maps > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
        float* step = reinterpret_cast<float*>(ws + pl.off_step);
        if (d->dtype == SCAN2D_BF16)
            hipLaunchKernelGGL(scan2d_bwd_step_kernel<bf16_t>, dim3((unsigned)(chunks * maps)), dim3(256), 0, stream,
                               static_cast<const bf16_t*>(delta), delta_bias, step, HW, d->Dc, chunks);
        else
            hipLaunchKernelGGL(scan2d_bwd_step_kernel<float>, dim3((unsigned)(chunks * maps)), dim3(256), 0, stream,
                               static_cast<const float*>(delta), delta_bias, step, HW, d->Dc, chunks);
    }
    if (pl.S > 1) {
        GcarryArgs g;
        g.delta = a.delta; g.delta_bias = delta_bias; g.A = A; g.Cm = Cm; g.dy = dy; g.z = z;
        g.pB = a.pB; g.pC = a.pC; g.GS = pl.GS; g.CG = pl.CG; g.part_row = pl.part_chunked ? pl.LG * pl.K : d->W;
        g.Dc = d->Dc; g.H = d->H; g.W = d->W; g.seg_rows = pl.seg_bands * pl.RB;
        g.cols = (unsigned)((d->W + 63) / 64);
        g.waves = (unsigned)((unsigned long long)maps * g.cols);           // rank_plan: fits
        const int form = z != nullptr ? kGcGated : (softplus ? kGcSoftplus : kGcPlain);
        hipLaunchKernelGGL(d->dtype == SCAN2D_BF16 ? gcarry_kernel<bf16_t>(form) : gcarry_kernel<float>(form), dim3((g.waves + 3) / 4), dim3(256),
                           0, stream, g);
    }
    if (pl.lds_bytes > 65536 && !allow_large_lds(reinterpret_cast<const void*>(pl.k.main), pl.lds_bytes)) return SCAN2D_ERR_LAUNCH_FAILED;
    // the checkpoint sweep by the shared-producer forward kernel (checkpoint mode): it computes the softplus step itself from
    // the raw projection, with the same function as the step kernel above
    auto ckpt_args = [&](int NG, int LG, int waves, int RPB) {
        FwdArgs f;
        f.x = x; f.delta = delta; f.A = A; f.Bm = Bm; f.Cm = Cm; f.Dskip = nullptr; f.mask = mask; f.y = nullptr;
        f.delta_bias = delta_bias; f.carry = nullptr;
        f.ck = a.ck; f.nb = pl.nb; f.ck_chunked = pl.ck_chunked ? 1 : 0;
        f.maps = maps; f.Dc = d->Dc; f.H = d->H; f.W = d->W; f.N = d->N;
        f.NG = NG; f.MPW = (waves * 64 / LG) / NG; f.panels = 1; f.RPB = RPB;
        return f;
    };
    if (pl.panels > 1) {
        // wide maps: checkpoint sweeps left to right (row-end states handed on), main sweeps right to left (a*q handed on)
        const size_t one = align_up((size_t)maps * d->N * d->H * sizeof(float));
        const int PW = pl.LG * pl.K;
        if (pl.k.ckpt_wide != nullptr && d->N == kWideNG * kWideNW) {
            // two panels: one sweep over whole rows (211x397 bf16, 256 maps: 340 us against 2 x 320)
            FwdArgs f = ckpt_args(kWideNG, kWideLG, kWideWaves, kWideRPB);
            f.hc = reinterpret_cast<float*>(ws + pl.off_hc);
            f.hc_panel = one / sizeof(float);
            const size_t lds_f = 2 * (size_t)f.MPW * f.RPB * 2 * kWideLG * kWideK * sizeof(float);         // the per-position buffers only
            hipLaunchKernelGGL(pl.k.ckpt_wide, dim3((unsigned)((maps + f.MPW - 1) / f.MPW)), dim3(kWideWaves * 64), lds_f, stream, f);
        } else {
            for (int q = 0; q < pl.panels; ++q) {
                BwdArgs c = ac;
                c.cb = q * PW;
                c.hc_in = q > 0 ? reinterpret_cast<const float*>(ws + pl.off_hc + (size_t)(q - 1) * one) : nullptr;
                c.hc_out = q + 1 < pl.panels ? reinterpret_cast<float*>(ws + pl.off_hc + (size_t)q * one) : nullptr;
                hipLaunchKernelGGL(pl.k.ckpt, dim3((unsigned)wg1), dim3(pl.ck_waves * 64), 0, stream, c);
            }
        }
        for (int q = pl.panels - 1; q >= 0; --q) {
            BwdArgs m = a;
            m.cb = q * PW;
            m.hc_in = q > 0 ? reinterpret_cast<const float*>(ws + pl.off_hc + (size_t)(q - 1) * one) : nullptr;
            m.qc_in = q + 1 < pl.panels ? reinterpret_cast<const float*>(ws + pl.off_qc + (size_t)((q + 1) & 1) * one) : nullptr;
            m.qc_out = q > 0 ? reinterpret_cast<float*>(ws + pl.off_qc + (size_t)(q & 1) * one) : nullptr;
            m.accum = q + 1 < pl.panels ? 1 : 0;
            hipLaunchKernelGGL(pl.k.main, dim3((unsigned)wg2), dim3(pl.waves * 64), pl.lds_bytes, stream, m);
        }
    } else {
        if (saved != nullptr) {
            // the forward pass of the training step has left the checkpoints
        } else if (pl.nb > 1 && pl.k.ckpt_fwd != nullptr && d->N == pl.k.cf_NG * pl.k.cf_NW) {
            const FwdArgs f = ckpt_args(pl.k.cf_NG, pl.k.cf_LG, pl.k.cf_waves, pl.k.cf_RPB);
            const long long wgf = (maps + f.MPW - 1) / f.MPW;
            if (wgf > 2147483647LL) return SCAN2D_ERR_BAD_SHAPE;
            const size_t lds_f = 2 * (size_t)f.MPW * f.RPB * 2 * pl.k.cf_LG * pl.k.cf_K * sizeof(float);   // the per-position buffers only
            hipLaunchKernelGGL(pl.k.ckpt_fwd, dim3((unsigned)wgf), dim3(pl.k.cf_waves * 64), lds_f, stream, f);
        } else if (pl.nb > 1) {
            hipLaunchKernelGGL(pl.k.ckpt, dim3((unsigned)wg1), dim3(pl.ck_waves * 64), 0, stream, ac);
        }
        hipLaunchKernelGGL(pl.k.main, dim3((unsigned)wg2), dim3(pl.waves * 64), pl.lds_bytes, stream, a);
    }
    if (pl.step_outside) {
        const float* dstep = reinterpret_cast<const float*>(ws + pl.off_step);
        if (d->dtype == SCAN2D_BF16)
            hipLaunchKernelGGL(scan2d_bwd_chain_kernel<bf16_t>, dim3((unsigned)maps), dim3(chain_threads(HW)), 0, stream, dstep,
                               static_cast<const bf16_t*>(delta), delta_bias, static_cast<bf16_t*>(ddelta), pbias, HW, d->Dc);
        else
            hipLaunchKernelGGL(scan2d_bwd_chain_kernel<float>, dim3((unsigned)maps), dim3(chain_threads(HW)), 0, stream, dstep,
                               static_cast<const float*>(delta), delta_bias, static_cast<float*>(ddelta), pbias, HW, d->Dc);
    }
    launch_sums(d, pl, a, dBm, dCm, dA, dA_v, dDskip, softplus ? ddelta_bias : nullptr, pbias, stream);
    return hipGetLastError() == hipSuccess ? SCAN2D_OK : SCAN2D_ERR_LAUNCH_FAILED;
}

}  // namespace scan2d
