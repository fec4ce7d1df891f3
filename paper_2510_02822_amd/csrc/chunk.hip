// Linear layers of a long reduction on calls of a few hundred to some thousand rows (the second layer of an MLP, mostly): a block owns
// 32 FR rows and 256, 128 or 64 columns and walks the reduction in chunks of 128, 256 or 512 channels.
//
// What bounded these calls in the tiled kernel (k_mixed) was a block barrier, and the waits around it, per K-step of 64 channels and the
// instructions beside its matrix instructions: 700 to 1000 cycles per K-step of a 128 x 128 tile that holds 256 cycles of matrix work.  Here
//   * the eight waves of a block are WN = 8 / WK groups of 32 columns times WK shares of the reduction: a weight fragment is needed by one
//     wave only and goes from global memory straight into the registers of the matrix instruction, eight units of 32 channels ahead;
//   * activations go to LDS through registers, whole runs of a row to neighbouring lanes, the 4-bit channels lowered on the way (Section
//     4.1; once per activation and block): a ring of three chunks, the loads two further chunks ahead;
//   * a wave has four units of every chunk, so there is one barrier per 4 FR matrix instructions of a wave, and it waits for nothing but
//     the wave's own LDS writes: the chunk it publishes is not read before the next one is used up;
//   * the sums of the WK shares meet in LDS.
// Same int8 MFMA, int32 sums and epilogue arithmetic as the other kernels: bit-identical outputs.
#include <algorithm>
#include <cmath>

#include "flexiq_internal.h"
#include "flexiq_test.h"
#include "stream_common.h"

namespace flexiq {
namespace chunk {

using namespace resident;

// n / d for block indices: exact while n * d < 2^32 (checked in choose()), m = ceil(2^32 / d)
struct Div {
    uint32_t m, d;
};
__device__ __forceinline__ int quot(int n, Div v) { return v.d == 1 ? n : (int)__umulhi((uint32_t)n, v.m); }

struct Params {
    const int8_t *X;        // int8 [M][C], stored channel order
    const int8_t *W8;       // [U][2][Npad][16], and the position-expanded 4-bit copy w4x_delta bytes further
    const int32_t *ashift;  // [G + 1]
    const float *cs;        // [2][Npad]
    int32_t *acc;
    float *y;
    int8_t *q;
    float r_out;
    int32_t M, N, Npad, C;
    int32_t w4x_delta;
    int32_t units;          // C / 32
    int32_t units4;         // leading units computed at 4 bits
    int32_t n_low;          // ... whose activations the kernel lowers (0: they arrive lowered)
    int32_t gs_shift;
    int32_t chunks;         // ceil(units / (4 WK))
    int32_t ncb, tiles;     // column blocks, row tiles
    Div dBand, dTail;       // divisors 8 * ncb, tiles % 8
    // LOWER builds: the layer that reads the int8 output (its positions, 4-bit prefix and log2 of its group size)
    const int32_t *next_ashift;
    int32_t next_K4, next_gs_log2;
};

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kMaxCols = 256;                 // output columns per block, at most
constexpr int kTabBytes = 3 * kMaxCols * 4;   // multipliers, addends, the consumer's lowering table
constexpr int kPosBytes = (kMaxGroups + 1) * 4;
constexpr int kUnits = 4;                     // units of a chunk per wave
constexpr int kSlots = 3;                     // chunks in LDS
constexpr int kFar = 0x40000000;              // an offset beyond every window: reads as zero

constexpr int pitch(int wk) { return 32 * kUnits * wk + 16; }   // bytes of a row in LDS (an odd number of 16-byte pieces: the lanes of a read fall into different banks)
constexpr int slot_bytes(int fr, int wk) { return 32 * fr * pitch(wk); }
constexpr int lds_bytes(int fr, int wk)
{
    return kTabBytes + kPosBytes + std::max(kSlots * slot_bytes(fr, wk), (wk - 1) * (kWaves / wk) * fr * 4096);
}

// FR: fragments of 32 rows.  WK: shares of the reduction.  QONLY / LOWER: as in store_fragment.
template <int FR, int WK, bool QONLY, bool LOWER>
__global__ __launch_bounds__(kThreads) void k_chunk(const Params p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int WN = kWaves / WK, P = 32 * FR, PITCH = pitch(WK), SLOT = slot_bytes(FR, WK);
    constexpr int LPR = 8 * WK;                      // 16-byte pieces of a chunk per row: so many lanes load a row
    constexpr int NP = (P * LPR + kThreads - 1) / kThreads;   // pieces of a chunk per thread
    constexpr int RSTEP = kThreads / LPR;            // rows between a thread's pieces
    unsigned char *const img = lds + kTabBytes + kPosBytes;
    int *const pos = reinterpret_cast<int *>(lds + kTabBytes);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    const int wn = wave % WN, wk = wave / WN;
    // the column blocks of a row tile sit 8 blocks apart: on one XCD, whose L2 then fetches the activations once; the last
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
    const int m0 = tile * P, n_blk = cb * 32 * WN;

    // ---- activations: this thread's 16-byte piece of rows xr, xr + RSTEP, ... of a chunk.  The window is what is left of the tile's
    // rows (rows beyond M read as zero); pieces beyond the last channel are sent beyond it.
    const int xr = tid / LPR, xp = tid % LPR;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)(p.X + (int64_t)m0 * p.C), 0, std::min(p.M - m0, P) * p.C, kRsrcFlags);
    const int xoff = xr * p.C + 16 * xp;
    unsigned char *const put = img + xr * PITCH + 16 * xp;
    auto xload = [&](v4i (&st)[NP], int ch) {
        const int at = (4 * WK * ch + (xp >> 1)) < p.units ? xoff + 128 * WK * ch : kFar;
#pragma unroll
        for (int k = 0; k < NP; ++k) st[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, at + k * RSTEP * p.C, 0, 0));
    };
    // ---- weights: this wave's columns n_blk + 32 wn + fr, k-half fh of unit 4 WK chunk + WK t + wk
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W8, 0, 2 * p.w4x_delta, kRsrcFlags);
    const int wlane = (fh * p.Npad + n_blk + 32 * wn + fr) * 16;
    auto wload = [&](int ch, int t) {
        const int u = std::min((kUnits * ch + t) * WK + wk, p.units - 1);
        return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, wlane, u * 32 * p.Npad + (u < p.units4 ? p.w4x_delta : 0), 0));
    };

    v4i st[2][NP], w[2][kUnits];
    {
        // ---- positions and scales, then the first four chunks of activations and two of weights are on their way at once (the fences: in this
        // order, which the waits of the loop count on)
        const int groups = p.n_low > 0 ? ((p.n_low - 1) >> p.gs_shift) + 1 : 0;   // (at most kMaxGroups)
        int sa_t = 0;
        if (tid < groups) sa_t = p.ashift[tid];
        float cs_t = 0.f, bi_t = 0.f;
        if (tid < 32 * WN) {
            cs_t = p.cs[n_blk + tid];
            bi_t = p.cs[p.Npad + n_blk + tid];
        }
        __builtin_amdgcn_sched_barrier(0);
        v4i t0[NP], t1[NP];
        xload(t0, 0);
        xload(t1, 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < kUnits; ++t) w[0][t] = wload(0, t);
        __builtin_amdgcn_sched_barrier(0);
        xload(st[0], 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < kUnits; ++t) w[1][t] = wload(1, t);
        __builtin_amdgcn_sched_barrier(0);
        xload(st[1], 3);
        __builtin_amdgcn_sched_barrier(0);
        if (tid < groups) pos[tid] = sa_t;
        const bool pre_scaled = QONLY || (p.q != nullptr && p.y == nullptr);
        float *const tab = reinterpret_cast<float *>(lds);
        if (tid < 32 * WN) {
            tab[tid] = pre_scaled ? cs_t * p.r_out : cs_t;
            tab[kMaxCols + tid] = pre_scaled ? bi_t * p.r_out + 128.0f : bi_t;
        }
        if constexpr (LOWER) fill_lower_table(lds + 2 * kMaxCols * 4, 8 * WN, n_blk, p.next_ashift, p.next_K4, p.next_gs_log2, tid, kThreads);
        __syncthreads();   // (the positions are read by every thread)
        auto first = [&](v4i (&x)[NP], int ch) {
            const int u = 4 * WK * ch + (xp >> 1);
            if (4 * WK * ch < p.n_low) {
                const bool low = u < p.n_low;
                const int sa = pos[low ? u >> p.gs_shift : 0];
                const short lo = low ? (short)((-(8 << sa)) << 8) : (short)0x8000, hi = low ? (short)((((8 << sa) - 1) << 8) | 0xFF) : (short)0x7FFF;
                const v2s lo2 = {lo, lo}, hi2 = {hi, hi};
                const uint32_t mask = low ? 0x01010101u * ((0xFFu << sa) & 0xFFu) : 0xFFFFFFFFu;
#pragma unroll
                for (int k = 0; k < NP; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[k][i] = (int)lower4((uint32_t)x[k][i], lo2, hi2, mask);
            }
#pragma unroll
            for (int k = 0; k < NP; ++k)
                if (NP * RSTEP <= P || k + 1 < NP || xr + k * RSTEP < P) *reinterpret_cast<v4i *>(put + ch * SLOT + k * RSTEP * PITCH) = x[k];
        };
        first(t0, 0);
        if (p.chunks > 1) first(t1, 1);
    }

    v16i acc[FR];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[f][e] = 0;
    __builtin_amdgcn_s_waitcnt(0xc07f);   // this wave's LDS writes
    block_barrier();

    // ---- the reduction.  Position j = FR t + f of a chunk: unit t times fragment f.  Activation fragments are read XA positions ahead, across
    // the end of the chunk; the scheduling fences keep that order (left alone, the compiler hoists every read and spills).
    constexpr int XA = FR == 1 ? 2 : 4, J = kUnits * FR;
    const unsigned char *const get = img + fr * PITCH + 32 * wk + 16 * fh;
    v4i x[XA];
    auto read = [&](int slot, int j) {
        return *reinterpret_cast<const v4i *>(get + slot + (j % FR) * 32 * PITCH + (j / FR) * 32 * WK);
    };
    int here = 0;   // slot of the chunk
    auto next_slot = [&](int s) { return s == (kSlots - 1) * SLOT ? 0 : s + SLOT; };
#pragma unroll
    for (int j = 0; j < XA; ++j) x[j] = read(0, j);
    // chunk ch, with buffer B of weights and of activations in flight (those of chunk ch + 2, which go to LDS here)
    auto body = [&](auto b_c, int ch) {
        constexpr int B = decltype(b_c)::value;
        const int after = next_slot(here), free_ = next_slot(after);
        const int u = 4 * WK * (ch + 2) + (xp >> 1);
        const bool lowers = 4 * WK * (ch + 2) < p.n_low;
        const bool low = u < p.n_low;
        const int sa = pos[lowers && low ? u >> p.gs_shift : 0];
        const short lo = low ? (short)((-(8 << sa)) << 8) : (short)0x8000, hi = low ? (short)((((8 << sa) - 1) << 8) | 0xFF) : (short)0x7FFF;
        const v2s lo2 = {lo, lo}, hi2 = {hi, hi};
        const uint32_t mask = low ? 0x01010101u * ((0xFFu << sa) & 0xFFu) : 0xFFFFFFFFu;
#pragma unroll
        for (int t = 0; t < kUnits; ++t) {
            const bool there = (kUnits * ch + t) * WK + wk < p.units;
            if (there) {
#pragma unroll
                for (int f = 0; f < FR; ++f) {
                    const int j = FR * t + f;
                    acc[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[B][t], x[j % XA], acc[f], 0, 0, 0);
                    x[j % XA] = j + XA < J ? read(here, j + XA) : read(after, j + XA - J);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            w[B][t] = wload(ch + 2, t);
            // a quarter of the pieces of chunk ch + 2
#pragma unroll
            for (int k = t * NP / kUnits; k < (t + 1) * NP / kUnits; ++k) {
                if (lowers) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) st[B][k][i] = (int)lower4((uint32_t)st[B][k][i], lo2, hi2, mask);
                }
                if (NP * RSTEP <= P || k + 1 < NP || xr + k * RSTEP < P) *reinterpret_cast<v4i *>(put + free_ + k * RSTEP * PITCH) = st[B][k];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        xload(st[B], ch + 4);
        here = after;
        __builtin_amdgcn_s_waitcnt(0xc07f);
        block_barrier();
    };
    for (int ch = 0; ch < p.chunks; ch += 2) {
        body(std::integral_constant<int, 0>{}, ch);
        body(std::integral_constant<int, 1>{}, ch + 1);
    }

    // ---- the sums of the waves that share a fragment meet in LDS: share f % WK of them finishes fragment f
    const int64_t mrow = m0 + fr;
    if constexpr (WK > 1) {
        v4i *const red = reinterpret_cast<v4i *>(img);   // [fragment][WK - 1][quad][lane]; (every wave is past its last read: barrier above)
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            const int own = f % WK;
            if (own != wk) {
                v4i *const to = red + (((wn * FR + f) * (WK - 1)) + (wk < own ? wk : wk - 1)) * 256 + lane;
#pragma unroll
                for (int g = 0; g < 4; ++g) to[64 * g] = (v4i){acc[f][4 * g], acc[f][4 * g + 1], acc[f][4 * g + 2], acc[f][4 * g + 3]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            if (f % WK == wk) {
#pragma unroll
                for (int k = 0; k < WK - 1; ++k) {
                    const v4i *const from = red + (((wn * FR + f) * (WK - 1)) + k) * 256 + lane;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const v4i s = from[64 * g];
                        acc[f][4 * g] += s.x; acc[f][4 * g + 1] += s.y; acc[f][4 * g + 2] += s.z; acc[f][4 * g + 3] += s.w;
                    }
                }
            }
        }
    }

    const bool pre_scaled = QONLY || (p.q != nullptr && p.y == nullptr), q_rows = p.q != nullptr && (p.N & 15) == 0;
    const FragOut fo = {p.acc, p.y, p.q, p.r_out, p.N};
    int lim = p.N - n_blk - 4 * fh;
    asm volatile("" : "+v"(lim));
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        if (f % WK == wk) store_fragment<QONLY, kMaxCols, LOWER>(acc[f], fo, lds, wn, n_blk, mrow + 32 * f, mrow + 32 * f < p.M, lim, fh, pre_scaled, q_rows);
        __builtin_amdgcn_sched_barrier(0);   // (one fragment at a time: interleaved, their temporaries spill)
    }
}

static int g_force = -1;   // test hook: >= 1: take this kernel with shape g_force - 1 whenever the call qualifies, 0 = never, -1 = automatic
static int g_last = 0;

typedef void (*Fn)(const Params);
template <int FR, int WK> static Fn pick(int out)
{
    return out == 2 ? k_chunk<FR, WK, true, true> : (out == 1 ? k_chunk<FR, WK, true, false> : k_chunk<FR, WK, false, false>);
}
// Block shapes, and what a chunk costs in each (ns; measured, see choose()): with all channels at 8 bits, more per share of 4-bit channels that
// the block lowers, and both for two blocks that share a compute unit (0: registers or LDS do not allow it).
struct Shape {
    int fr, wk;
    Fn (*fn)(int);
    int step, low, step2, low2;
};
constexpr Shape kShapes[] = {{2, 1, pick<2, 1>, 366, 75, 768, 21}, {3, 1, pick<3, 1>, 566, 100, 0, 0}, {4, 1, pick<4, 1>, 699, 65, 0, 0},
                             {5, 1, pick<5, 1>, 893, 131, 0, 0}, {6, 1, pick<6, 1>, 1020, 123, 0, 0}, {7, 1, pick<7, 1>, 1165, 121, 0, 0},
                             {8, 1, pick<8, 1>, 1249, 144, 0, 0}, {1, 2, pick<1, 2>, 300, 87, 685, 0}, {2, 2, pick<2, 2>, 476, 145, 991, 73},
                             {3, 2, pick<3, 2>, 728, 200, 0, 0}, {4, 2, pick<4, 2>, 927, 218, 0, 0}, {5, 2, pick<5, 2>, 1155, 267, 0, 0},
                             {1, 4, pick<1, 4>, 379, 205, 837, 123}, {2, 4, pick<2, 4>, 767, 290, 0, 0}, {3, 4, pick<3, 4>, 1158, 433, 0, 0}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

struct DeviceState {
    bool ready = false;
    int num_cu = 0;
    bool two[kNumShapes] = {};   // two blocks share a compute unit, whatever the outputs
};
static DeviceState g_dev[64];

}  // namespace chunk

int prepare_chunk_kernels(int device)
{
    using namespace chunk;
    if (device < 0 || device >= 64) return FLEXIQ_EINVAL;
    if (g_dev[device].ready) return FLEXIQ_OK;
    hipDeviceProp_t prop;
    FLEXIQ_HIP(hipGetDeviceProperties(&prop, device));
    g_dev[device].num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    for (int i = 0; i < kNumShapes; ++i) {
        const Shape &s = kShapes[i];
        g_dev[device].two[i] = s.step2 > 0;   // (measured; and what was compiled still fits)
        for (int out = 0; out < 3; ++out) {
            int resident = 0;
            FLEXIQ_HIP(hipFuncSetAttribute((const void *)s.fn(out), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(s.fr, s.wk)));
            FLEXIQ_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, (const void *)s.fn(out), kThreads, lds_bytes(s.fr, s.wk)));
            if (resident < 2) g_dev[device].two[i] = false;
        }
    }
    g_dev[device].ready = true;
    return FLEXIQ_OK;
}

// The block shape for a call of M rows, by the least modelled time: 0.6 us and per round of blocks 4.2 us, 32 fs per output byte, and the longer of the
// chunks and the weights' way from the last-level cache (the fourth root of the sum of their fourth powers).  A block reads the weights of its columns once, straight
// into registers, and shares them with no block but those of its XCD that work on the same columns of other row tiles: the weights cross once per row tile,
// up to eight times (XCDs), at 7.1 to 7.4 TB/s at most.  (Up to 1280 channels they are on their way before a block's other trips to memory end: counted,
// they made 560 such calls 2 % slower, up to 1.38 times; not counted.)  Fitted to 58900 times (7700 calls of 1344 to 8192 channels, 64 to 16384 columns, 65 to 64000
// rows, every shape whose blocks are one round), 6.8 % off (root mean square; 15.8 % without the weights, which took 2.7 times the modelled time where they are
// the most: 157 x 4992 -> 12144 34.7 us in the tiled kernel, 44.7 here, modelled at 18).
struct Choice {
    int shape = -1;
    double us = 0;
    double weights = 0;      // the weights' share of it
    bool one_round = false;  // every block is resident from the start
};
static Choice choose(const flexiq_layer *L, int64_t M, int out_bytes, const chunk::DeviceState &ds, int only)
{
    using namespace chunk;
    Choice c;
    const int num_cu = ds.num_cu;
    const int units = L->C / kUnit;
    const double low = L->x_prelowered ? 0.0 : (double)L->max_4bit_ch / L->C;
    for (int i = 0; i < kNumShapes; ++i) {
        if (only >= 0 && only != i) continue;
        const Shape &s = kShapes[i];
        const int P = 32 * s.fr, BN = 32 * kWaves / s.wk;
        const int64_t ncb = (L->N + BN - 1) / BN, tiles = (M + P - 1) / P, blocks = ncb * tiles;
        if (blocks * 8 * ncb >= (1ll << 32) || blocks > 0x3fffffff) continue;   // (the division of the block index)
        const bool two = ds.two[i] && blocks > num_cu;
        const int64_t side = two ? 2 : 1, rounds = (blocks + side * num_cu - 1) / (side * num_cu);
        const double chunks = 1e-3 * ((units + kUnits * s.wk - 1) / (kUnits * s.wk)) * (two ? s.step2 + low * s.low2 : s.step + low * s.low);
        const double weights = L->C > 1280 ? (double)std::min<int64_t>(tiles, 8) * (double)(ncb * BN) * L->C / 7.4e6 : 0.0;
        const double c2 = chunks * chunks, w2 = weights / rounds * (weights / rounds);
        const double us = 0.6 + (double)rounds * (4.2 + std::sqrt(std::sqrt(c2 * c2 + w2 * w2)) + 32e-6 * (double)(side * P * BN) * out_bytes);
        if (c.shape < 0 || us < c.us) {
            c.shape = i;
            c.us = us;
            c.weights = weights / us;
            c.one_round = rounds == 1;
        }
    }
    return c;
}

// Launches k_chunk when the call qualifies: plain outputs or int8 rows lowered for a consumer.  It is offered what the kernels for few rows and few
// tiles leave, and takes calls of more than 1280 channels (up to there k_wreg is level) whose blocks are all resident at once.
// Times here over times in the tiled kernel on 1800 such calls of 544 to 8192 channels, 64 to 16384 columns and 65 to 40000 rows, geometric mean 0.79, 3 % of
// them more than 3 % behind (the worst 1.27, 826 x 4704 -> 8048 at r = 0.5).  Not, by 7700 calls timed in every shape:
//   * tiles of 192 rows and more by 256 columns whose activations need no lowering, int8 out: there the tiled kernel keeps its matrix cores busy as well (0.99
//     to 1.04; 12608 x 4096 -> 1024 level to 2 % behind; fp32 out 0.90 to 0.96, with lowering 0.78 to 1.03);
//   * 128 rows and more per tile where a layer has at most 128 columns: the block computes up to four times as many (1.00 to 1.24 by shape, up to 1.48; smaller
//     tiles 0.68 to 0.91);
//   * 128 rows and more per tile, or two blocks on a compute unit, where the weights take more than 0.4 of the time, unless at least three channels in ten are at 4
//     bits: both kernels then wait for the same weights (0.93 to 1.02, up to 1.72: 450 x 2176 -> 8096 15.0 us there, 24.2 here; smaller tiles 0.77 to 0.93);
//   * two rounds and more: 0.80 to 1.07, up to 1.20 at r = 0 with int8 out; fp32 out with lowering 0.62 to 1 (the tiled kernel's blocks walk several tiles without a
//     new prologue).
// Of 576 to 1024 channels it takes what k_halo would where a block has at most seven fragments of rows times shares and a compute unit to itself: 635 calls
// 0.90 (the worst 1.04; larger ones 1.04 to 1.14; 512 and 544 channels 0.95, up to 1.13, fp32 out 1.01, up to 1.28), and at most five of them where a layer has at most
// 64 columns, of the 128 that such a block computes (96 rows in two shares 1.04 to 1.09: 22799 x 768 -> 64 at r = 1 7.4 us there, 8.0 here; fewer rows 0.90 to 1.01).
int launch_chunk(const flexiq_layer *L, const int8_t *X, int64_t M, const flexiq_out *out, void *stream_, bool halo, int *taken, const LowerArgs *lower)
{
    using namespace chunk;
    *taken = 0;
    g_last = 0;
    if (g_force == 0) return FLEXIQ_OK;
    if (g_force < 0 && (few_rows_forced() || stream_forced() || halo_forced())) return FLEXIQ_OK;   // (those hooks compare with the tiled kernel)
    if (out->scan_for || out->x4 || out->x6) return FLEXIQ_OK;
    const bool q_only = out->q && !out->acc && !out->y && (L->N & 15) == 0;
    const bool lowering = lower && lower->ashift;   // (null positions: the consumer has no 4-bit channels at its ratio)
    if (lowering && !q_only) return FLEXIQ_OK;      // (the lowering build writes int8 only)
    const DeviceState &ds = g_dev[L->device];
    if (!ds.ready) return FLEXIQ_OK;
    if (g_force < 0 && L->C <= 1280 && (L->C < 576 || !halo)) return FLEXIQ_OK;
    if (M > (1 << 24) || (int64_t)32 * 8 * L->C >= kFar) return FLEXIQ_OK;   // (row indices and the window of a tile)
    const Choice c = choose(L, M, (out->q ? 1 : 0) + (out->y ? 4 : 0) + (out->acc ? 4 : 0), ds, g_force > 0 ? g_force - 1 : -1);
    if (c.shape < 0 || (g_force < 0 && !c.one_round)) return FLEXIQ_OK;
    const Shape &s = kShapes[c.shape];
    const int P = 32 * s.fr, BN = 32 * kWaves / s.wk;
    const int64_t blocks = ((M + P - 1) / P) * ((L->N + BN - 1) / BN);
    if (g_force < 0) {   // (as said above)
        const int low = L->x_prelowered ? 0 : L->max_4bit_ch;
        if (s.fr >= 6 && s.wk == 1 && !out->y && low == 0) return FLEXIQ_OK;
        if (s.fr >= 4 && L->N <= 128) return FLEXIQ_OK;
        if (L->C <= 1280 && (s.fr * s.wk >= (L->N <= 64 ? 6 : 8) || blocks > ds.num_cu)) return FLEXIQ_OK;
        if (c.weights > 0.4 && ((s.fr >= 4 && 10 * low < 3 * L->C) || blocks > ds.num_cu)) return FLEXIQ_OK;
    }
    Params p = {};
    p.units = L->C / kUnit;
    p.X = X; p.W8 = L->d_w8; p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift; p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad; p.C = L->C;
    p.w4x_delta = L->U * 32 * L->Npad;
    p.units4 = L->max_4bit_ch / kUnit;
    p.n_low = L->x_prelowered ? 0 : p.units4;
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.chunks = (p.units + kUnits * s.wk - 1) / (kUnits * s.wk);
    p.ncb = (L->N + BN - 1) / BN;
    p.tiles = (int)((M + P - 1) / P);
    auto div = [](int d) { return Div{d == 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d), (uint32_t)d}; };
    p.dBand = div(8 * p.ncb); p.dTail = div(p.tiles % 8 ? p.tiles % 8 : 1);
    if (lowering) { p.next_ashift = lower->ashift; p.next_K4 = lower->K4; p.next_gs_log2 = lower->gs_log2; }
    FLEXIQ_HIP(launch_kernel(s.fn(lowering ? 2 : (q_only ? 1 : 0)), dim3((unsigned)(p.tiles * p.ncb)), dim3(kThreads), lds_bytes(s.fr, s.wk), stream_, p));
    *taken = g_last = 1 + c.shape;
    return FLEXIQ_OK;
}

}  // namespace flexiq

extern "C" int flexiq_debug_force_chunk(int mode)
{
    if (mode < -1 || mode > flexiq::chunk::kNumShapes) return FLEXIQ_EINVAL;
    flexiq::chunk::g_force = mode;
    return flexiq::chunk::g_last;
}
