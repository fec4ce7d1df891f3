// Convolutions whose input tile stays in LDS while the weights stream past it: 3x3 filters at stride 1 or 2 and any padding with
// any multiple of 32 input channels, and strided (2) or padded 1x1 filters (ResNet stages 2-4, downsampling layers, small
// batches).  Which calls it gets beyond one round of blocks: conv_route() in gemm.hip.  Linear layers of up to 544 channels are served as well where a call is one short round of blocks (up to 1024 channels such calls are k_chunk's, which it tells from the choice here).
//
// What bounded these calls in the tiled implicit-GEMM kernel (k_mixed) was not matrix work: a K-step there is 64 channels of
// one filter tap, whose activations are fetched (and, for 4-bit groups, bit-lowered) again for each of the nine taps through
// the 64 B/clk path into LDS, behind a block barrier per K-step (about 700 cycles whatever the tile height).  Here
//   * a block owns a run of consecutive output pixels (of the flattened [B][Ho][Wo], so it may begin inside an image row and
//     end in another image) and up to 256 output columns.  The input rows under those pixels, all channels, with the padding
//     as zeros, go to LDS once, through registers, where the 4-bit channels are lowered on the way (Section 4.1): once per
//     activation and block instead of once per tap;
//   * after the one barrier that publishes them the waves run on their own: a wave owns 32 output columns (and, with WK > 1,
//     every WK-th 32-channel unit of the reduction), so every weight fragment is needed by one wave only (per row group) and
//     goes from global memory straight into MFMA operand registers, one whole filter (nine taps of a unit) ahead of its use;
//     activation fragments are nine shifted reads of the LDS image;
//   * the sums of the waves that share an output fragment meet in LDS (the image is dead by then).
// Same int8 MFMA, int32 sums and epilogue arithmetic as the other kernels: bit-identical outputs.
//
// Measured (graph replays, int8 out, us in the tiled kernel and here): 3x3 256 -> 256 @14x14, batch 64, r = 0 / 0.5 / 1: 19.9 / 22.9 /
// 24.9 and 10.7 / 10.5 / 10.3 (1.4 POP/s; the K loop takes 9.9 thousand cycles of which the matrix instructions are 9.2, before it
// 6.5 thousand of set-up and copying); batch 1: 17.4 and 4.9; 512 -> 512 @7x7, batch 128: 40 and 19.5, batch 1: 27.3 and 5.6;
// stride 2, 96 -> 160 @57x43, batch 5: 14.9 and 7.2; 1x1 stride 2, 256 -> 512 @56x56, batch 128: 40.8 and 33.7.
//
// LDS image: a pixel is C + 16 bytes, an odd number of 16-byte pieces, so that the 32 lanes of a fragment read fall into
// different banks without a permutation; the pixels of an image row are ordered by column modulo the stride first, so that
// the lanes of a strided fragment read neighbouring pixels as well.
#include <algorithm>

#include "flexiq_internal.h"
#include "flexiq_test.h"
#include "stream_common.h"

namespace flexiq {
namespace halo {

using namespace resident;

// n / d for the small indices of this kernel: exact while n * d < 2^32 (checked in choose()), m = ceil(2^32 / d)
struct Div {
    uint32_t m, d;
};
__device__ __forceinline__ int quot(int n, Div v) { return v.d == 1 ? n : (int)__umulhi((uint32_t)n, v.m); }

struct Params {
    const int8_t *X;        // int8 NHWC [B][H][W][C], stored channel order
    const int8_t *W8;       // [taps * CUp][2][Npad][16], and the position-expanded 4-bit copy w4x_delta bytes further
    const int32_t *ashift;  // [G + 1]
    const float *cs;        // [2][Npad]
    int32_t *acc;
    float *y;
    int8_t *q;
    float r_out;
    int32_t M, N, Npad;
    int32_t w4x_delta;
    int32_t units, CUp;     // C / 32, and rounded up to even (units per tap of the weight tiles)
    int32_t units4;         // leading units computed at 4 bits
    int32_t n_low;          // ... whose activations the kernel lowers (0: they arrive lowered)
    int32_t gs_shift;
    int32_t B, H, W, C, Ho, Wo;
    int32_t st;             // LDS pixels between neighbouring output pixels (the stride; 1 for 1x1 filters)
    int32_t window;         // bytes a block may read from its first image on (linear calls: rows beyond M lie outside)
    int32_t step, pad;      // input pixels between neighbouring LDS pixels (1; the stride for 1x1 filters), padding
    int32_t VH;             // LDS rows per image: (Ho - 1) * st + R
    int32_t Wv, Wh, rowpx;  // LDS pixels of an image row; per column phase, ceil(Wv / st); allotted per row, st * Wh
    int32_t ppc, cpr;       // LDS pixels a wave copies at a time (even when st is 2), such runs per row
    int32_t pxb;            // bytes per LDS pixel, C + 16
    Div dWo, dHo, dVH, dCpr, dPiece, dBand, dTail;   // divisors Wo, Ho, VH, cpr, C / 16, 8 * ncb, tiles % 8
    int32_t ncb, tiles;     // column blocks, pixel tiles
    int32_t wn_log2, wmn_log2, wk;   // waves of a block: log2 of its 32-column groups, of those times its pixel groups; shares of the reduction
    // LOWER builds: the layer that reads the int8 output (its positions, 4-bit prefix and log2 of its group size)
    const int32_t *next_ashift;
    int32_t next_K4, next_gs_log2;
};

constexpr int kMaxCols = 256;                 // output columns per block, at most
constexpr int kTabBytes = 3 * kMaxCols * 4;   // multipliers, addends, the consumer's lowering table

// FR: fragments of 32 pixels per wave.  TAPS: 9 or 1.  QONLY / LOWER: as in store_fragment.
template <int FR, int TAPS, bool QONLY, bool LOWER>
__global__ __launch_bounds__(1024) void k_halo(const Params p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char *const img = lds + kTabBytes;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    // (all three counts are powers of two)
    const int wn = wave & ((1 << p.wn_log2) - 1), wmn = wave & ((1 << p.wmn_log2) - 1), wm = wmn >> p.wn_log2, wk = wave >> p.wmn_log2;
    // the column blocks of a pixel tile sit 8 blocks apart: on one XCD, whose L2 then fetches the activations once; the last
    // few tiles, fewer than XCDs, are dealt out over all of them
    int tile, cb;
    {
        const int g = quot(blockIdx.x, p.dBand), r = (int)blockIdx.x - g * (int)p.dBand.d;
        cb = r >> 3;
        tile = 8 * g + (r & 7);
        if (8 * g + 8 > p.tiles) {
            cb = quot(r, p.dTail);
            tile = 8 * g + r - cb * (int)p.dTail.d;
        }
    }
    const int P = (32 * FR) << (p.wmn_log2 - p.wn_log2);
    const int m0 = tile * P;
    const int n_blk = cb * 32 << p.wn_log2;

    // ---- the tile's LDS rows: row v of the flattened, padded images; the tile begins at row v0
    auto lds_row = [&](int m, int &ox) {
        const int j = quot(m, p.dWo), b = quot(j, p.dHo);
        ox = m - j * p.Wo;
        return b * p.VH + (j - b * p.Ho) * p.st;
    };
    int ox_unused;
    const int v0 = lds_row(m0, ox_unused);
    const int m_last = min(m0 + P, p.M) - 1;
    const int nrows = lds_row(m_last, ox_unused) - v0 + (TAPS == 9 ? 3 : 1);
    const int ppp = p.C >> 4;                       // 16-byte pieces per pixel

    // ---- weights: this wave's columns n_blk + 32 wn + fr, k-half fh of every unit
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W8, 0, 2 * p.w4x_delta, kRsrcFlags);
    const int wlane = (fh * p.Npad + n_blk + 32 * wn + fr) * 16;   // (columns of a block are < Npad: checked by the launcher)
    const int ustride = 32 * p.Npad, tstride = p.CUp * ustride;
    constexpr int G = TAPS == 9 ? 9 : 8;            // steps whose weights travel together
    auto unit_off = [&](int c) { return c * ustride + (c < p.units4 ? p.w4x_delta : 0); };
    v4i w[G];
    // step t of the group that begins at unit c: tap t of unit c (3x3), or unit c + t * WK (1x1; there() = there is such a unit)
    auto there = [&](int c, int t) { return TAPS == 9 || c + t * p.wk < p.units; };
    auto wload = [&](int c, int t) {
        const int soff = TAPS == 9 ? unit_off(c) + t * tstride : unit_off(c + t * p.wk);
        return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, wlane, soff, 0));
    };
    int c = wk;                                     // (wk < units: checked by the launcher)

    // ---- scales and biases travel with the first operands
    float cs_t = 0.f, bi_t = 0.f;
    if (tid < 32 << p.wn_log2) {
        cs_t = p.cs[n_blk + tid];
        bi_t = p.cs[p.Npad + n_blk + tid];
    }

    // ---- activations into LDS, through registers.  A wave takes a run of `ppc` neighbouring LDS pixels of one row at a time,
    // a lane always the same 16-byte piece (so the same channel group) of the same pixel of a run.  Where the runs begin is
    // worked out for 64 of them at once, one per lane, and handed round by v_readlane (measured: with the full index
    // arithmetic per lane and piece this phase took 7 to 9 thousand cycles, all of it instruction issue; as scalar work per
    // run 5 to 6 thousand).
    const int lpx = quot(lane, p.dPiece), lpc = lane - lpx * ppp;
    const bool lane_on = lpx < p.ppc;
    const bool lane_low = (lpc >> 1) < p.n_low;
    const int sa = p.ashift[lane_low ? (lpc >> 1) >> p.gs_shift : 0];   // (used once the activations are on their way)
    const int lane_src = lpx * (p.step * p.C) + 16 * lpc, lane_ix = lane_on ? lpx * p.step : -0x40000000;
    const int lane_dst = (p.st == 2 ? (lpx & 1) * p.Wh + (lpx >> 1) : lpx) * p.pxb + 16 * lpc, lane_px = lane_on ? lpx : 0x40000000;
    constexpr int UB = 8;   // runs in flight per wave
    constexpr int kFar = 0x40000000;   // an offset beyond the window below: reads as zero
    const int runs = nrows * p.cpr, nw = (int)(blockDim.x >> 6);
    const int b0 = quot(v0, p.dVH);
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.X + (int64_t)b0 * p.H * p.W * p.C), 0, p.window, kRsrcFlags);
    const int mine = (runs - wave + nw - 1) / nw;   // this wave's runs: wave, wave + nw, ...
    int run_src = 0, run_ix = 0, run_px = 0, run_dst = 0;
    auto runs_of = [&](int i) {   // of this wave's runs i + lane
        const int j = wave + (i + lane) * nw;
        const int row = quot(j, p.dCpr), px0 = (j - row * p.cpr) * p.ppc;
        const int v = v0 + row, b = quot(v, p.dVH);
        const int iy = (v - b * p.VH) * p.step - p.pad, ix0 = px0 * p.step - p.pad;
        run_src = (((b - b0) * p.H + iy) * p.W + ix0) * p.C;   // (below 0 when a run begins in the padding: its lanes add to it)
        run_ix = b < p.B && (unsigned)iy < (unsigned)p.H ? ix0 : -0x40000000;   // (a row outside the image: no lane is in it)
        run_px = px0;
        run_dst = (row * p.rowpx + (p.st == 2 ? px0 >> 1 : px0)) * p.pxb;
    };
    bool first = true;
    for (int i0 = 0; i0 < mine || first; i0 += UB) {
        if ((i0 & 63) == 0) runs_of(i0);
        v4i x[UB];
        int dst[UB];
#pragma unroll
        for (int k = 0; k < UB; ++k) {
            if (i0 + k < mine) {
                const int at = (i0 & 63) + k;
                const bool in = (unsigned)(__builtin_amdgcn_readlane(run_ix, at) + lane_ix) < (unsigned)p.W;
                const int voff = in ? __builtin_amdgcn_readlane(run_src, at) + lane_src : kFar;
                x[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, voff, 0, 0));
                dst[k] = __builtin_amdgcn_readlane(run_px, at) + lane_px < p.Wv ? __builtin_amdgcn_readlane(run_dst, at) + lane_dst : -1;
            }
        }
        if (first) {   // the first weights follow the first activations
#pragma unroll
            for (int t = 0; t < G; ++t)
                if (there(c, t)) w[t] = wload(c, t);
            first = false;
        }
        // (channels read at 8 bits: nothing is clamped or cleared)
        const short lo = lane_low ? (short)((-(8 << sa)) << 8) : (short)0x8000, hi = lane_low ? (short)((((8 << sa) - 1) << 8) | 0xFF) : (short)0x7FFF;
        const v2s lo2 = {lo, lo}, hi2 = {hi, hi};
        const uint32_t mask = lane_low ? 0x01010101u * ((0xFFu << sa) & 0xFFu) : 0xFFFFFFFFu;
#pragma unroll
        for (int k = 0; k < UB; ++k) {
            if (i0 + k < mine) {
                if (p.n_low > 0) {
                    x[k].x = (int)lower4((uint32_t)x[k].x, lo2, hi2, mask);
                    x[k].y = (int)lower4((uint32_t)x[k].y, lo2, hi2, mask);
                    x[k].z = (int)lower4((uint32_t)x[k].z, lo2, hi2, mask);
                    x[k].w = (int)lower4((uint32_t)x[k].w, lo2, hi2, mask);
                }
                if (dst[k] >= 0) *reinterpret_cast<v4i *>(img + dst[k]) = x[k];
            }
        }
    }

    // ---- scales and biases (pre-multiplied for the int8 output when it is the only scaled one)
    const bool pre_scaled = QONLY || (p.q != nullptr && p.y == nullptr);
    float *const tab = reinterpret_cast<float *>(lds);
    if (tid < 32 << p.wn_log2) {   // (a block has at least that many threads)
        tab[tid] = pre_scaled ? cs_t * p.r_out : cs_t;
        tab[kMaxCols + tid] = pre_scaled ? bi_t * p.r_out + 128.0f : bi_t;
    }
    if constexpr (LOWER) fill_lower_table(lds + 2 * kMaxCols * 4, 8 << p.wn_log2, n_blk, p.next_ashift, p.next_K4, p.next_gs_log2, tid, (int)blockDim.x);

    // ---- this wave's pixels
    int base[FR];   // LDS offset of the lane's pixel under the first tap, k-half folded in
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        int m = m0 + 32 * (wm * FR + f) + fr;
        if (m > m_last) m = m0;   // (lanes beyond the tile compute its first pixel again and store nothing)
        int ox;
        const int v = lds_row(m, ox) - v0;
        base[f] = (v * p.rowpx + ox) * p.pxb + 16 * fh;
    }
    int toff[TAPS];
#pragma unroll
    for (int t = 0; t < TAPS; ++t) {
        const int r = t / 3, s = t % 3;
        toff[t] = TAPS == 1 ? 0 : (r * p.rowpx + (p.st == 1 ? s : (s & 1) * p.Wh + (s >> 1))) * p.pxb;
    }
    v16i acc[FR];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[f][e] = 0;
    __syncthreads();

    // ---- the reduction.  Activation fragments are read one step ahead, weights one group ahead; the scheduling fences keep
    // that order (left alone, the compiler hoists every read and spills).
    v4i x[2][FR];
    auto xload = [&](int k, int off) {
#pragma unroll
        for (int f = 0; f < FR; ++f) x[k][f] = *reinterpret_cast<const v4i *>(img + base[f] + off);
    };
    auto xoff = [&](int cc, int t) { return TAPS == 9 ? 32 * cc + toff[TAPS == 9 ? t : 0] : 32 * min(cc + t * p.wk, p.units - 1); };
    const int cstep = TAPS == 9 ? p.wk : G * p.wk;
    xload(0, xoff(c, 0));
    auto group = [&](auto more_c, auto guard_c) {
        constexpr bool MORE = decltype(more_c)::value, GUARD = decltype(guard_c)::value;
        const int cn = c + cstep;
#pragma unroll
        for (int t = 0; t < G; ++t) {
            const int k = t & 1;
            if (t + 1 < G) xload(k ^ 1, xoff(c, t + 1));
            else if (MORE) xload(k ^ 1, xoff(cn, 0));
            __builtin_amdgcn_sched_barrier(0);
            if (!GUARD || there(c, t)) {
#pragma unroll
                for (int f = 0; f < FR; ++f) acc[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[t], x[k][f], acc[f], 0, 0, 0);
            }
            if (MORE && there(cn, t)) w[t] = wload(cn, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (MORE && (G & 1)) {
#pragma unroll
            for (int f = 0; f < FR; ++f) x[0][f] = x[1][f];
        }
        c = cn;
    };
    using T = std::integral_constant<bool, true>;
    using F = std::integral_constant<bool, false>;
    while (c + cstep < p.units) group(T{}, F{});
    group(F{}, std::integral_constant<bool, TAPS == 1>{});

    // ---- the sums of the waves that share a fragment meet in LDS: share f % WK of them finishes fragment f
    const int64_t mrow = m0 + 32 * (wm * FR) + fr;
    if (p.wk > 1) {
        __syncthreads();   // every wave is past the image
        v4i *const red = reinterpret_cast<v4i *>(img);   // [fragment][WK - 1][quad][lane]
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            const int own = f & (p.wk - 1);
            if (own != wk) {
                v4i *const to = red + (((wmn * FR + f) * (p.wk - 1)) + (wk < own ? wk : wk - 1)) * 256 + lane;
#pragma unroll
                for (int g = 0; g < 4; ++g) to[64 * g] = (v4i){acc[f][4 * g], acc[f][4 * g + 1], acc[f][4 * g + 2], acc[f][4 * g + 3]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            if ((f & (p.wk - 1)) == wk) {
                for (int k = 0; k < p.wk - 1; ++k) {
                    const v4i *const from = red + (((wmn * FR + f) * (p.wk - 1)) + k) * 256 + lane;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const v4i s = from[64 * g];
                        acc[f][4 * g] += s.x; acc[f][4 * g + 1] += s.y; acc[f][4 * g + 2] += s.z; acc[f][4 * g + 3] += s.w;
                    }
                }
            }
        }
    }

    const bool q_rows = p.q != nullptr && (p.N & 15) == 0;
    const FragOut fo = {p.acc, p.y, p.q, p.r_out, p.N};
    int lim = p.N - n_blk - 4 * fh;
    asm volatile("" : "+v"(lim));
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        if ((f & (p.wk - 1)) == wk) store_fragment<QONLY, kMaxCols, LOWER>(acc[f], fo, lds, wn, n_blk, mrow + 32 * f, mrow + 32 * f < p.M, lim, fh, pre_scaled, q_rows);
        __builtin_amdgcn_sched_barrier(0);   // (one fragment at a time: interleaved, their temporaries spill)
    }
}

struct DeviceState {
    bool ready = false;
    int num_cu = 0;
};
static DeviceState g_dev[64];
static int g_force = -1;   // test hook: >= 1: take this kernel with plan g_force - 1 whenever the call qualifies, 0 = never, -1 = automatic
static int g_last = 0;

typedef void (*Fn)(const Params);
template <int FR, int TAPS> static Fn pick(bool q_only, bool lowering)
{
    return lowering ? k_halo<FR, TAPS, true, true> : (q_only ? k_halo<FR, TAPS, true, false> : k_halo<FR, TAPS, false, false>);
}
static Fn kernel(int fr, int taps, bool q_only, bool lowering)
{
    if (taps == 9) return fr == 1 ? pick<1, 9>(q_only, lowering) : pick<2, 9>(q_only, lowering);
    return fr == 1 ? pick<1, 1>(q_only, lowering) : pick<2, 1>(q_only, lowering);
}

// Shapes of a block: fragments per wave, waves along pixels, columns and the reduction.  These are what is left of 38 that were
// measured on 317 layers of every size (3x3 and 1x1, stride 1 and 2, 64 to 512 channels, 16 pixels to 400 thousand): the best
// of these is within 1 % of the best of all (geometric mean); four fragments per wave (159 registers, one block per compute
// unit) never won by more than 2 %.
struct Plan {
    int fr, wm, wn, wk;
};
constexpr Plan kPlans[] = {{2, 1, 8, 1}, {2, 1, 4, 2}, {1, 1, 4, 2}, {1, 1, 2, 4}, {1, 1, 1, 8}, {2, 2, 4, 1}, {2, 4, 2, 1},
                           {2, 2, 8, 1}, {2, 2, 2, 1}, {2, 1, 4, 1}, {1, 1, 4, 1}, {1, 1, 2, 2}, {1, 2, 2, 2}};
constexpr int kNumPlans = sizeof(kPlans) / sizeof(kPlans[0]);

}  // namespace halo

int prepare_halo_kernels(int device)
{
    using namespace halo;
    if (device < 0 || device >= 64) return FLEXIQ_EINVAL;
    if (g_dev[device].ready) return FLEXIQ_OK;
    hipDeviceProp_t prop;
    FLEXIQ_HIP(hipGetDeviceProperties(&prop, device));
    g_dev[device].num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    for (int taps : {1, 9})
        for (int fr : {1, 2})
            for (int k = 0; k < 3; ++k)
                FLEXIQ_HIP(hipFuncSetAttribute((const void *)kernel(fr, taps, k > 0, k > 1), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    g_dev[device].ready = true;
    return FLEXIQ_OK;
}

namespace halo {

// What the choice of a block shape depends on: the sizes of a call and of its layer.
struct Sizes {
    int32_t B, H, W, stride, pad;
    int32_t N, Npad, C, R, S;
    int32_t out_bytes;   // per output element
    int32_t num_cu;
    bool linear;         // rows of a linear call: B = H = 1, W rows
};

// The block shape for a call (`only` >= 0: that one or none).  Host arithmetic only.
static HaloChoice choose(const Sizes &s, int only)
{
    HaloChoice c;
    const int taps = s.R * s.S;
    if (!((s.R == 3 && s.S == 3) || taps == 1) || s.stride > 2) return c;
    const int Ho = (s.H + 2 * s.pad - s.R) / s.stride + 1, Wo = (s.W + 2 * s.pad - s.S) / s.stride + 1;
    const int64_t M = (int64_t)s.B * Ho * Wo;
    const int st = taps == 1 ? 1 : s.stride;
    const int64_t VH = (int64_t)(Ho - 1) * st + s.R;
    const int Wv = (Wo - 1) * st + s.S, rowpx = st * ((Wv + st - 1) / st), pxb = s.C + 16;
    int ppc = 64 / (s.C / 16);
    if (st == 2) ppc &= ~1;
    if (ppc < 1) return c;   // (more than 1024 channels; 512 for strided filters)
    if (M > 0x7fffffff - 512) return c;   // (row indices are 32-bit: a tile may begin at the last row; such calls are refused further on)
    // the kernel's divisions: index times divisor below 2^32
    if (!s.linear && (M * std::max(Wo, Ho) >= (1ll << 31) || (s.B + 1ll) * VH * VH >= (1ll << 31) || s.W > 4096)) return c;
    if ((int64_t)s.H * s.W * s.C * (256 / ((int64_t)Ho * Wo) + 2) >= (1 << 30)) return c;   // the images under a tile: one 1 GiB window
    auto image_rows = [&](int P) {   // LDS rows under P consecutive output pixels, wherever they begin
        const int64_t nr = std::min<int64_t>((P + Wo - 2) / Wo + 1, (int64_t)s.B * Ho);
        const int64_t cross = std::min<int64_t>((nr - 1 + Ho - 1) / Ho, s.B - 1);
        return (nr - 1) * st + cross * (s.R - st) + s.R;
    };
    const int units = s.C / kUnit;
    for (int i = 0; i < kNumPlans; ++i) {
        const Plan &pl = kPlans[i];
        if (only >= 0 && only != i) continue;
        if (pl.wk > units) continue;
        const int P = 32 * pl.fr * pl.wm, BN = 32 * pl.wn;
        const int64_t ncb = (s.N + BN - 1) / BN, tiles = (M + P - 1) / P;
        if (ncb * BN > s.Npad) continue;
        const int64_t red = (int64_t)(pl.wk - 1) * pl.wm * pl.wn * pl.fr * 4096;
        const int64_t rows = s.linear ? 1 : image_rows(P), lds = kTabBytes + std::max(rows * (s.linear ? P : rowpx) * pxb, red);
        const int64_t cpr = s.linear ? (P + ppc - 1) / ppc : (Wv + ppc - 1) / ppc;
        if (lds > 160 * 1024 || tiles * ncb > 0x3fffffff) continue;
        if (tiles * ncb * 8 * ncb >= (1ll << 32)) continue;   // (the division of the block index)
        // Modelled cycles of the busiest compute unit: per block the matrix instructions (or, for blocks of few pixels, the
        // weight bytes), a price per wave (dispatch, set-up, epilogue) and per output byte; per round of co-resident blocks the
        // copy of the input tile (per run of a wave) and a constant.  Fitted to 200 convolutions and 220 linear calls; the
        // shape it picks is within 0.7 % resp. 1.5 % of the best (geometric mean; at worst 17 %), and 3 us + cost * 0.59 ns
        // is the time of the call within about 10 %.
        const int waves = pl.wm * pl.wn * pl.wk;
        const int64_t blocks = tiles * ncb, per_cu = (blocks + s.num_cu - 1) / s.num_cu;
        const int64_t fits = std::max<int64_t>(1, std::min<int64_t>({160 * 1024 / lds, 16 / waves, 8})), conc = std::min(fits, per_cu);
        const double mfma = (double)taps * ((units + pl.wk - 1) / pl.wk) * waves * pl.fr * 8.0;
        const double weights = (double)taps * units * 32.0 * BN * pl.wm;
        const double body = std::max(mfma, 0.27 * mfma + 0.007 * weights) + 190.0 * waves + 0.1 * P * BN * s.out_bytes;
        const double round = 200.0 + 370.0 * (double)(rows * cpr) / waves + (pl.wk > 1 ? 300.0 : 0.0);
        const double cost = (double)per_cu * body + (double)((per_cu + conc - 1) / conc) * round;
        if (c.shape < 0 || cost < c.cost) {
            c.shape = i;
            c.tiles = tiles;
            c.ncb = ncb;
            c.lds = lds;
            c.cost = cost;
            // The time of the call, for the choice between kernels (gemm.hip, which says how well it is met): the parts of the same
            // sum at their own rates, and where several blocks share a compute unit its last round counts by half.
            const double even = conc == 1 ? (double)per_cu : std::max((double)conc, 0.5 * (per_cu + (double)blocks / s.num_cu));
            const double rounds = conc == 1 ? (double)per_cu : std::max(1.0, 0.5 * ((per_cu + conc - 1) / conc + (double)blocks / s.num_cu / conc));
            c.one_round = per_cu <= conc;
            c.crowded = taps != 1 && st == 2 && P == 32 && fits == 1 && ncb > 1 && per_cu > 2;
            c.us = 3.3 + 1e-3 * (even * (0.78 * std::max(mfma, 0.27 * mfma + 0.007 * weights) + 0.57 * 190.0 * waves + 0.42 * 0.1 * P * BN * s.out_bytes) +
                                 (taps == 1 ? 0.65 : 0.48) * rounds * 370.0 * (double)(rows * cpr) / waves);
        }
    }
    return c;
}

}  // namespace halo

// The shape of a call that qualifies: a 3x3 filter or a 1x1 filter that is not a plain linear call, stride 1 or 2; plain outputs or
// int8 output lowered for a consumer; an input tile that fits LDS.
static HaloChoice choice_any(const flexiq_layer *L, int B, int H, int W, int stride, int pad, bool linear, const flexiq_out *out, const LowerArgs *lower)
{
    using namespace halo;
    g_last = 0;
    if (g_force == 0 || (g_force < 0 && conv3_forced())) return HaloChoice();   // (the 3x3 kernel's hook, in any forced state, keeps this one out of its comparisons)
    if (out->scan_for || out->x4 || out->x6) return HaloChoice();
    const bool q_only = out->q && !out->acc && !out->y && (L->N & 15) == 0;
    const bool lowering = lower && lower->ashift;   // (null positions: the consumer has no 4-bit channels at its ratio)
    if (lowering && !q_only) return HaloChoice();   // (the lowering build writes int8 only)
    const DeviceState &ds = g_dev[L->device];
    if (!ds.ready) return HaloChoice();
    const Sizes sizes = {B, H, W, stride, pad, L->N, L->Npad, L->C, L->R, L->S, (out->q ? 1 : 0) + (out->y ? 4 : 0) + (out->acc ? 4 : 0), ds.num_cu, linear};
    return choose(sizes, g_force > 0 ? g_force - 1 : -1);
}

static int launch_any(const flexiq_layer *L, const int8_t *X, int B, int H, int W, int stride, int pad, bool linear, const flexiq_out *out, void *stream_,
                      const HaloChoice &c, const LowerArgs *lower)
{
    using namespace halo;
    const bool q_only = out->q && !out->acc && !out->y && (L->N & 15) == 0, lowering = lower && lower->ashift;
    const Plan &pl = kPlans[c.shape];
    const int P = 32 * pl.fr * pl.wm, taps = L->R * L->S, units = L->C / kUnit;
    const int Ho = (H + 2 * pad - L->R) / stride + 1, Wo = (W + 2 * pad - L->S) / stride + 1;
    const int64_t M = (int64_t)B * Ho * Wo;
    Params p = {};
    p.st = taps == 1 ? 1 : stride;
    p.step = taps == 1 ? stride : 1;
    p.VH = (Ho - 1) * p.st + L->R;
    p.Wv = (Wo - 1) * p.st + L->S;
    p.Wh = (p.Wv + p.st - 1) / p.st;
    p.rowpx = p.st * p.Wh;
    p.window = 0x40000000;
    p.pxb = L->C + 16;
    p.ppc = 64 / (L->C / 16);
    if (p.st == 2) p.ppc &= ~1;
    p.cpr = (p.Wv + p.ppc - 1) / p.ppc;
    p.X = X; p.W8 = L->d_w8; p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift; p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad;
    p.w4x_delta = L->U * 32 * L->Npad;
    p.units = units; p.CUp = (units + 1) & ~1;
    p.units4 = L->max_4bit_ch / kUnit;
    p.n_low = L->x_prelowered ? 0 : p.units4;
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.B = B; p.H = H; p.W = W; p.C = L->C; p.Ho = Ho; p.Wo = Wo;
    if (linear) {   // one image whose rows are the tiles
        p.Ho = p.H = p.VH = (int)((M + P - 1) / P);
        p.Wo = p.W = p.Wv = p.Wh = p.rowpx = P;
        p.cpr = (P + p.ppc - 1) / p.ppc;
        p.window = (int)(M * L->C);
    }
    p.pad = pad;
    auto div = [](int d) { return Div{d == 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d), (uint32_t)d}; };
    p.dWo = div(p.Wo); p.dHo = div(p.Ho); p.dVH = div(p.VH); p.dCpr = div(p.cpr); p.dPiece = div(L->C / 16);
    p.ncb = (int)c.ncb;
    p.tiles = (int)c.tiles;
    p.wn_log2 = __builtin_ctz(pl.wn); p.wmn_log2 = __builtin_ctz(pl.wm * pl.wn); p.wk = pl.wk;
    p.dBand = div(8 * p.ncb); p.dTail = div(p.tiles % 8 ? p.tiles % 8 : 1);
    if (lowering) { p.next_ashift = lower->ashift; p.next_K4 = lower->K4; p.next_gs_log2 = lower->gs_log2; }
    FLEXIQ_HIP(launch_kernel(kernel(pl.fr, taps, q_only, lowering), dim3((unsigned)(p.tiles * p.ncb)), dim3(64 * pl.wm * pl.wn * pl.wk), (size_t)c.lds, stream_, p));
    g_last = 1 + c.shape;
    return FLEXIQ_OK;
}

HaloChoice halo_choice(const flexiq_layer *L, int B, int H, int W, int stride, int pad, const flexiq_out *out, const LowerArgs *lower)
{
    return choice_any(L, B, H, W, stride, pad, false, out, lower);
}

int launch_halo(const flexiq_layer *L, const int8_t *X, int B, int H, int W, int stride, int pad, const flexiq_out *out, void *stream_,
                const HaloChoice &c, const LowerArgs *lower)
{
    return launch_any(L, X, B, H, W, stride, pad, false, out, stream_, c, lower);
}

bool halo_forced() { return halo::g_force >= 0; }

// The same for a linear call of M rows of at most 1024 channels (the rows of a tile are all there is to its image): shape < 0 also
// where the tiled kernel is ahead.
HaloChoice halo_rows_choice(const flexiq_layer *L, int64_t M, const flexiq_out *out, const LowerArgs *lower)
{
    halo::g_last = 0;
    if (M > (1 << 20) || M * L->C >= (1 << 30)) return HaloChoice();   // (row indices times the tile's rows, and the window of the input)
    if (halo::g_force < 0) {
        if (L->N & (out->q ? 15 : 3)) return HaloChoice();   // (ragged output rows leave element by element here)
        if (few_rows_forced() || stream_forced()) return HaloChoice();   // (those hooks compare with the tiled kernel)
    }
    const HaloChoice c = choice_any(L, 1, 1, (int)M, 1, 0, true, out, lower);
    // Linear calls of more than one short round stay with the tiled kernel: its blocks keep several tiles' loads in flight, where
    // a block here copies, multiplies and stores one after the other (us there and here: 1576 x 768 -> 3072 10.2 and 11.2; 6304 x
    // 768 -> 3072 22.7 and 26.1; below the line, 1576 x 1024 -> 1024 8.7 and 7.2; 177 x 448 -> 1856 6.4 and 4.9; 1234 x 704 -> 128 7.2
    // and 5.4: 11 % on average over 131 such calls, the worst 5 % behind).
    return halo::g_force < 0 && c.cost > 10000.0 ? HaloChoice() : c;
}

int launch_halo_rows(const flexiq_layer *L, const int8_t *X, int64_t M, const flexiq_out *out, void *stream_, const HaloChoice &c, const LowerArgs *lower)
{
    return launch_any(L, X, 1, 1, (int)M, 1, 0, true, out, stream_, c, lower);
}

}  // namespace flexiq

extern "C" int flexiq_debug_force_halo(int mode)
{
    if (mode < -1 || mode > flexiq::halo::kNumPlans) return FLEXIQ_EINVAL;
    flexiq::halo::g_force = mode;
    return flexiq::halo::g_last;
}

extern "C" int flexiq_debug_halo_plan(const int64_t *call, int64_t *plan)
{
    using namespace flexiq::halo;
    if (!call || !plan) return FLEXIQ_EINVAL;
    const int64_t N = call[5], C = call[6], R = call[7];
    for (int i = 0; i < 10; ++i)
        if (call[i] < (i == 4 || i == 8 ? 0 : 1) || call[i] > 0x7fffffff) return FLEXIQ_EINVAL;
    if (C % flexiq::kUnit || C > (1 << 20) || N > (1 << 24) || call[1] > (1 << 20) || call[2] > (1 << 20) || call[4] > (1 << 10) || std::min(call[1], call[2]) + 2 * call[4] < R)
        return FLEXIQ_EINVAL;
    const Sizes sizes = {(int32_t)call[0], (int32_t)call[1], (int32_t)call[2], (int32_t)call[3], (int32_t)call[4], (int32_t)N, (int32_t)((N + 255) & ~255ll),
                         (int32_t)C, (int32_t)R, (int32_t)R, (int32_t)call[8], (int32_t)call[9], false};
    const flexiq::HaloChoice c = choose(sizes, g_force > 0 ? g_force - 1 : -1);
    if (c.shape < 0) return 0;
    plan[0] = 32 * kPlans[c.shape].fr * kPlans[c.shape].wm;
    plan[1] = 32 * kPlans[c.shape].wn;
    plan[2] = c.tiles;
    plan[3] = c.ncb;
    plan[4] = c.lds;
    return 1 + c.shape;
}
