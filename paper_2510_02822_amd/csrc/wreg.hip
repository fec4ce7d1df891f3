// Linear layers (and 1x1 convolutions with stride 1) of 288 to 1280 channels with the weights of a block resident in registers.
//
// What bounded these calls in the tiled kernel (k_mixed) was everything around its K loop: with 9 to 40 K-steps per tile a block
// spends a third of its time in the prologue of its tiles and in an epilogue that nothing overlaps, and every K-step brings weights
// and activations into LDS behind a block barrier.  The registers of a compute unit hold 512 KB, more than the weights of 256
// columns: here a block of eight waves keeps them for good, a wave 32 columns of every unit (up to 160 of its 256 registers per
// lane), and only activations move: tiles of 32 rows, whole rows, through a ring of LDS slots, copied up to three tiles ahead.
// A fragment of them is read by each wave once and used by one matrix instruction (128 B/clk of the compute unit's LDS).
//   * One barrier per tile, which the two waves of a SIMD reach half a tile apart, so that one's epilogue runs beside the other's
//     matrix instructions (in step, both SIMD pipes took turns: 2420 cycles per tile of 24 units instead of 1920; 1536 are matrix
//     instructions).  The first fragments of a tile are read before the barrier that ends the one before.
//   * 4-bit channels are lowered in LDS, in place, by the wave that copied them, between matrix instructions (one tile of 24 units at
//     r = 1: 2570 cycles; with the pieces read and written one after the other 3340).
//   * The copies of a tile are spread over half a tile's matrix instructions: in one burst behind the barrier they held up the output
//     stores (2060 cycles).
//   * Each XCD serves few column blocks and many row groups, so that its L2 fetches few of the weights before the first tile can
//     begin: bands of eight column blocks; with all column blocks on every XCD 6304 x 768 -> 3072 took 18.5 us instead of 16.9.
// What bounds it now: on many tiles the clock.  12608 x 1024 -> 4096 takes 33.1 us on zeros and 40.9 on activations (r = 0.5: 39.0 and 44.1) in the same
// number of cycles; matrix instructions alone, no LDS reads, copies or epilogue, take 36 us on activations.  Not on few: 6304 x 768 -> 3072, four tiles per
// block, takes 14.3 and 14.8, 3 us of it the weights' way into registers and the rest launch, tiles and last stores.
//
// Measured (graph replays, us in the tiled kernel and here): 6304 x 768 -> 3072, int8 out, r = 0 / 0.5 / 1: 21.7 / 22.5 / 24.2 and 17.8 /
// 19.1 / 20.8, fp32 out (r = 0.5) 42.3 and 25.0; 12608 x 1024 -> 4096: 62 / 67 / 68 and 46 / 51 / 53, input lowered by its producer 63 and 45, fp32
// out (r = 0.5) 128 and 59; 12608 x 1216 -> 4864 at r = 0 / 1: 80 / 80 and 63 / 75; 1576 x 768 -> 3072 9.6 and 8.2.
#include <algorithm>

#include "flexiq_internal.h"
#include "flexiq_test.h"
#include "stream_common.h"

namespace flexiq {
namespace wreg {

using namespace resident;

struct Params {
    const int8_t *X;        // int8 [M][C], stored channel order
    const int8_t *W8;       // [CUp][2][Npad][16], and the position-expanded 4-bit copy w4x_delta bytes further
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
    int32_t ncb, groups;    // column blocks, row groups: the grid is their product
    int32_t band;           // column blocks that share a band of the grid
    int32_t per_group, extra;     // row tiles of a group, and how many groups take one more
    const int32_t *next_ashift;   // LOWER builds: the layer that reads the int8 output
    int32_t next_K4, next_gs_log2;
};

constexpr int kWaves = 8, kCols = 32 * kWaves, kRows = 32;
constexpr int kTabBytes = 3 * kCols * 4;   // multipliers, addends, the consumer's lowering table
constexpr int stage_bytes(int nu) { return nu * 1024; }
constexpr int slots(int nu) { return stage_bytes(nu) * 4 + kTabBytes <= 160 * 1024 ? 4 : 3; }

template <int N> __device__ __forceinline__ void wait_vm()   // at most N vector-memory operations outstanding
{
    static_assert(N <= 63, "the counter has six bits");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}
template <int N> __device__ __forceinline__ void wait_lds()   // ... LDS operations
{
    static_assert(N <= 15, "the counter has four bits");
    __builtin_amdgcn_s_waitcnt(0xc07f | (N << 8));
}

// The outputs of a call: any of them; int8 rows and nothing else, N a multiple of 16; those lowered for a consumer; fp32 rows and
// nothing else, N a multiple of 4.
enum Out { kAny, kCodes, kLowered, kFloats, kFloatsAtOnce };
constexpr int kOuts = 5;

// NU: units held in registers (C / 32 rounded up to a multiple of eight); EXACT: C = 32 NU.  LOWIN: the kernel lowers the 4-bit
// channels of its input.
template <int NU, Out OUT, bool LOWIN, bool EXACT>
__global__ __launch_bounds__(64 * kWaves, 2) void k_wreg(const Params p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr bool QONLY = OUT == kCodes || OUT == kLowered, LOWER = OUT == kLowered;
    constexpr int S = slots(NU), STAGE = stage_bytes(NU), NCP = NU / kWaves;
    unsigned char *const ring = lds + kTabBytes;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;

    // the blocks of an XCD take neighbouring entries of the grid [band of columns][row group][column block of the band]
    int cb, g;
    {
        const int nb = (int)gridDim.x, x = (int)blockIdx.x & 7, i = (int)blockIdx.x >> 3;
        int lin = x * (nb >> 3) + min(x, nb & 7) + i;
        const int b = lin / (p.band * p.groups);
        lin -= b * p.band * p.groups;
        const int width = min(p.band, p.ncb - b * p.band);
        g = lin / width;
        cb = b * p.band + lin - g * width;
    }
    const int n_blk = cb * kCols;
    const int t0 = g * p.per_group + min(g, p.extra), nt = p.per_group + (g < p.extra ? 1 : 0);   // (nt >= 1)

    // ---- copies of a row tile: 64-byte chunks of 16 rows per instruction; this wave's are wave / 2 + 4 k, its half of the rows wave % 2
    const int crow = 16 * (wave & 1) + (lane >> 2);
    const int cpc = (lane & 3) ^ swizzle(crow, 4);   // logical piece of the chunk
    const int chunk0 = wave >> 1;
    const int voff = crow * p.C + 64 * chunk0 + 16 * cpc;
    const bool whole = EXACT || chunk0 + 4 * (NCP - 1) < ((p.units + 1) >> 1);   // the wave copies NCP chunks of a tile (else NCP - 1)
    const int tile_bytes = kRows * p.C;
    const int8_t *next_x = p.X + (int64_t)t0 * tile_bytes;   // the next tile to ask for, what is left of X there, and its slot
    int left = (int)((int64_t)p.M * p.C - (int64_t)t0 * tile_bytes), asked = 0, next_slot = 0;   // (M * C < 2^31)
    // (rows beyond M, and tiles beyond the block's, read as zeros: the copies in flight are the same in every round)
    auto copy = [&](int j) {
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)next_x, 0, asked < nt ? left : 0, kRsrcFlags);
        if (j < NCP - 1 || whole) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(ring + next_slot + 1024 * (wave + kWaves * j)), 16, voff + 256 * j, 0, 0, 0);
    };
    auto copied = [&]() {
        ++asked;
        next_x += tile_bytes;
        left -= tile_bytes;
        next_slot = next_slot == (S - 1) * STAGE ? 0 : next_slot + STAGE;
    };
    auto issue = [&]() {
#pragma unroll
        for (int j = 0; j < NCP; ++j) copy(j);
        copied();
    };
    // positions of this lane's pieces of a tile, scales and biases: on their way before everything else
    int sa[NCP];
    if constexpr (LOWIN) {
#pragma unroll
        for (int j = 0; j < NCP; ++j) {
            const int u = 2 * (chunk0 + 4 * j) + (cpc >> 1);
            sa[j] = p.ashift[u < p.n_low ? u >> p.gs_shift : 0];
        }
    }
    float cs_t = 0.f, bi_t = 0.f;
    if (tid < kCols) {
        cs_t = p.cs[n_blk + tid];
        bi_t = p.cs[p.Npad + n_blk + tid];
    }
    issue();
    __builtin_amdgcn_sched_barrier(0);   // (in this order: the waits below count on it)
    // ---- weights: columns n_blk + 32 wave + fr, k-half fh of every unit
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W8, 0, 2 * p.w4x_delta, kRsrcFlags);
    const int wlane = (fh * p.Npad + n_blk + 32 * wave + fr) * 16;
    v4i w[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {   // (units the layer does not have: the last one again, not used)
        const int v = EXACT || u <= NU - 8 ? u : min(u, p.units - 1);
        w[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, wlane, v * 32 * p.Npad + (v < p.units4 ? p.w4x_delta : 0), 0));
    }
    __builtin_amdgcn_sched_barrier(0);   // (likewise)
#pragma unroll
    for (int k = 1; k < S - 1; ++k) issue();

    // (channels that stay as they are: nothing is clamped or cleared)
    uint32_t low_lo[NCP], low_mask[NCP];
    if constexpr (LOWIN) {
#pragma unroll
        for (int j = 0; j < NCP; ++j) {
            const bool low = 2 * (chunk0 + 4 * j) + (cpc >> 1) < p.n_low;
            low_lo[j] = low ? ((0xfffff800u << sa[j]) & 0xffffu) * 0x10001u : 0x80008000u;
            low_mask[j] = low ? 0x01010101u * ((0xffu << sa[j]) & 0xffu) : 0xffffffffu;
        }
    }
    const bool pre_scaled = QONLY || (p.q != nullptr && p.y == nullptr);
    float *const tab = reinterpret_cast<float *>(lds);
    if (tid < kCols) {
        tab[tid] = pre_scaled ? cs_t * p.r_out : cs_t;
        tab[kCols + tid] = pre_scaled ? bi_t * p.r_out + 128.0f : bi_t;
    }
    if constexpr (LOWER) fill_lower_table(lds + 2 * kCols * 4, kCols / 4, n_blk, p.next_ashift, p.next_K4, p.next_gs_log2, tid, 64 * kWaves);

    // ---- bit-lowering (Section 4.1) of the pieces that this lane copied, in place.  Every wave lowers its own copies of a tile
    // between the landing of those copies and the barrier that publishes the tile.
    unsigned char *const own = ring + 1024 * wave + 16 * lane;
    v4i piece[NCP];
    auto lower_read = [&](int slot) {
#pragma unroll
        for (int j = 0; j < NCP; ++j) piece[j] = *reinterpret_cast<const v4i *>(own + slot + 1024 * kWaves * j);
#pragma unroll
        for (int j = 0; j < NCP; ++j) asm volatile("" : "+v"(piece[j]));
    };
    auto lower_write = [&](int slot, int j) {
        if (2 * (chunk0 + 4 * j) >= p.n_low) return;
        const v2s lo2 = __builtin_bit_cast(v2s, low_lo[j]), hi2 = ~lo2;
        const uint32_t mask = low_mask[j];
        v4i b = piece[j];
        b.x = (int)lower4((uint32_t)b.x, lo2, hi2, mask);
        b.y = (int)lower4((uint32_t)b.y, lo2, hi2, mask);
        b.z = (int)lower4((uint32_t)b.z, lo2, hi2, mask);
        b.w = (int)lower4((uint32_t)b.w, lo2, hi2, mask);
        *reinterpret_cast<v4i *>(own + slot + 1024 * kWaves * j) = b;
    };
    auto lower_tile = [&](int slot) {
        lower_read(slot);
#pragma unroll
        for (int j = 0; j < NCP; ++j) lower_write(slot, j);
    };
    // this wave's copies have landed, but for those of the last S - 3 tiles asked for (one count for all waves: the compiler then
    // knows behind the first wait that the weights have landed, and does not wait for everything in front of the loop)
    auto wait_tile = [&]() { wait_vm<(S - 3) * (EXACT ? NCP : NCP - 1)>(); };

    wait_vm<NU + (S - 2) * (NCP - 1)>();   // the first tile is there, weights and later tiles are on their way
    if constexpr (LOWIN) lower_tile(0);

    const bool q_rows = p.q != nullptr && (p.N & 15) == 0;
    const FragOut fo = {p.acc, p.y, p.q, p.r_out, p.N};
    const int xe = fr * 64 + ((fh ^ swizzle(fr, 4)) << 4), xo = fr * 64 + (((2 + fh) ^ swizzle(fr, 4)) << 4);
    // The sums of a tile leave between the matrix instructions of the next one: fp32 rows, whose stores then spread over the tile (r = 0.5 / 1:
    // 6304 x 768 -> 3072 27.0 / 27.5 -> 24.3 / 24.4 us, 12608 x 1024 -> 4096 62.5 / 62.9 -> 53.2 / 55.4), and codes of short layers without lowering (12608 x 512 ->
    // 2048 at r = 0 17.2 -> 16.2).  Other codes leave at once: beside the lowering they held up the matrix instructions (12608 x 1024 -> 4096 at
    // r = 1 50.1 -> 52.7), and without it nothing was gained.
    // (That does not pay where memory itself takes the stores, fp32 rows that do not fit the last-level cache, for all numbers of units: launch_wreg.)
    constexpr bool FLOATS = OUT == kFloats || OUT == kFloatsAtOnce;
    constexpr bool INTER = NU <= 32 && (OUT == kFloats || (!FLOATS && OUT != kAny && NU == 16 && !LOWIN));
    constexpr bool REGTAB = OUT != kAny && NU <= (INTER && LOWIN ? 24 : 32);   // the epilogue's constants stay in registers
    constexpr int D = NU <= 32 ? 4 : 2;          // units that activation fragments are read ahead
    // the pieces to lower leave one after the other from the third unit of a half on
    constexpr int PSTEP = 2, LASTP = 2 + PSTEP * (NCP - 1);
    static_assert(LASTP < NU / 2 && NU % D == 0, "all of a half's pieces");

    // The two waves of a SIMD run half a tile apart, so that one's epilogue goes beside the other's matrix instructions: there is
    // one barrier per tile, which waves 0-3 reach in the middle of tile i and waves 4-7 (LATE) at the end of tile i - 1.  Behind it
    // tile i + 1 is in place, and nobody reads tile i - 1 any more: its slot takes tile i + S - 1.
    auto walk = [&](auto late_c) {
        constexpr bool LATE = decltype(late_c)::value;
        if constexpr (LOWIN && LATE) {
            if (nt > 1) {
                wait_tile();
                lower_tile(STAGE);
            }
        }
        wait_lds<0>();
        block_barrier();
        v4i mul[4], add[4];
        if constexpr (REGTAB) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = 32 * wave + 8 * i + 4 * fh;
                mul[i] = *reinterpret_cast<const v4i *>(lds + 4 * c);
                add[i] = *reinterpret_cast<const v4i *>(lds + 4 * (kCols + c));
                asm volatile("" : "+v"(mul[i]), "+v"(add[i]));
            }
        }
        v4i x[D];
        const unsigned char *se = ring + xe, *so = ring + xo;
        auto xload = [&](int u) { x[u % D] = *reinterpret_cast<const v4i *>((u & 1 ? so : se) + (u >> 1) * 2048); };
#pragma unroll
        for (int u = 0; u < D; ++u) xload(u);
        auto sync = [&]() {   // (LDS reads may be in flight: their slot is not written before the barrier after this one)
            wait_tile();
            block_barrier();
        };
        const int lim_lane = p.N - n_blk - 4 * fh;
        // ---- epilogue of tile t0 + i: value e of the lane's sixteen (register 4 k + j: column 8 k + 4 fh + j of the wave's), then the rest.
        // (What is computed here is pinned in its place: as pure data flow the optimiser moves it past the branches, to its use.)
        uint32_t qrow[4];
        v4i yq, lt;
        auto value = [&](const v16i &acc, int i, int e) {
            const int k = e >> 2, j = e & 3, c = 32 * wave + 8 * k + 4 * fh;
            if (j == 0) {
                if constexpr (!REGTAB) {
                    mul[k] = *reinterpret_cast<const v4i *>(lds + 4 * c);
                    add[k] = *reinterpret_cast<const v4i *>(lds + 4 * (kCols + c));
                    asm volatile("" : "+v"(mul[k]), "+v"(add[k]));
                }
                if constexpr (LOWER) {
                    lt = *reinterpret_cast<const v4i *>(lds + 4 * (2 * kCols + c));
                    asm volatile("" : "+v"(lt));
                }
            }
            float v = __builtin_fmaf((float)acc[e], __int_as_float(mul[k][j]), __int_as_float(add[k][j]));
            if constexpr (FLOATS) {
                yq[j] = __float_as_int(v);
                asm volatile("" : "+v"(yq));
                const uint32_t at = (uint32_t)(fr * p.N + n_blk + c) * 4u;
                if (j == 3 && fr < p.M - (t0 + i) * kRows && c - 4 * fh < lim_lane)
                    *reinterpret_cast<v4i *>(reinterpret_cast<unsigned char *>(p.y + (int64_t)(t0 + i) * kRows * p.N) + at) = yq;
            } else {
                if constexpr (LOWER) v = __builtin_amdgcn_fmed3f(v, __int_as_float(lt.x), __int_as_float(lt.y));
                qrow[k] = __builtin_amdgcn_cvt_pk_u8_f32(v, j, j == 0 ? 0 : qrow[k]);
                if (j == 3) {
                    qrow[k] ^= 0x80808080u;
                    if constexpr (LOWER) qrow[k] &= (uint32_t)lt.z;
                }
                asm volatile("" : "+v"(qrow[k]));
            }
        };
        auto finish = [&](int i) {
            if constexpr (!FLOATS) {
                const FragOut at = {nullptr, nullptr, p.q + (int64_t)(t0 + i) * kRows * p.N, 0.0f, p.N};   // (its rows from this tile on)
                store_codes(at, qrow, wave, n_blk, fr, fr < p.M - (t0 + i) * kRows, lim_lane, fh);
            }
        };
        float *y_lane = p.y + ((int64_t)t0 * kRows + fr) * p.N + n_blk + 32 * wave + 4 * fh;
        int8_t *q_tile = p.q + (int64_t)t0 * kRows * p.N;
        auto leave = [&](const v16i &acc, int i) {   // all of a tile's sums at once
            if constexpr (INTER) {
#pragma unroll
                for (int e = 0; e < 16; ++e) value(acc, i, e);
                finish(i);
                return;
            }
            int lim = p.N - n_blk - 4 * fh;
            asm volatile("" : "+v"(lim));
            const int64_t m = (int64_t)(t0 + i) * kRows + fr;
            if constexpr (FLOATS) {
                if (m < p.M) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int c = 32 * wave + 8 * k + 4 * fh;
                        v4i mu, ad;
                        if constexpr (REGTAB) {
                            mu = mul[k];
                            ad = add[k];
                        } else {
                            mu = *reinterpret_cast<const v4i *>(lds + 4 * c);
                            ad = *reinterpret_cast<const v4i *>(lds + 4 * (kCols + c));
                            asm volatile("" : "+v"(mu), "+v"(ad));
                        }
                        v4i v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = __float_as_int(__builtin_fmaf((float)acc[4 * k + e], __int_as_float(mu[e]), __int_as_float(ad[e])));
                        if (c - 4 * fh < lim) *reinterpret_cast<v4i *>(y_lane + 8 * k) = v;
                    }
                }
                y_lane += kRows * (int64_t)p.N;
            } else if constexpr (REGTAB) {
                v4i lt[4];
                if constexpr (LOWER) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) lt[k] = *reinterpret_cast<const v4i *>(lds + 4 * (2 * kCols) + 4 * (32 * wave + 8 * k + 4 * fh));
                }
                uint32_t qrow[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    uint32_t qw = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float v = __builtin_fmaf((float)acc[4 * k + e], __int_as_float(mul[k][e]), __int_as_float(add[k][e]));
                        if constexpr (LOWER) v = __builtin_amdgcn_fmed3f(v, __int_as_float(lt[k].x), __int_as_float(lt[k].y));
                        qw = __builtin_amdgcn_cvt_pk_u8_f32(v, e, qw);
                    }
                    qrow[k] = qw ^ 0x80808080u;
                    if constexpr (LOWER) qrow[k] &= (uint32_t)lt[k].z;
                }
                FragOut at = fo;   // (its rows from this tile on)
                at.q = q_tile;
                q_tile += kRows * p.N;
                store_codes(at, qrow, wave, n_blk, fr, m < p.M, lim, fh);
            } else {
                store_fragment<QONLY, kCols, LOWER>(acc, fo, lds, wave, n_blk, m, m < p.M, lim, fh, pre_scaled, q_rows);
            }
        };
        int after = STAGE;   // slot of the next tile
        // half of a tile's units, from U0 on; LOW: the wave lowers its part of the tile in `low_slot`
        // meanwhile; COPY: it asks for a tile (in one go the copies of all waves would hold up each other and the stores); PREV: the sums of the
        // tile before leave
        auto half = [&](auto begin, auto low, int low_slot, auto copy_c, auto prev_c, int i, v16i &acc, const v16i &prev) {
            constexpr int U0 = decltype(begin)::value;
            constexpr bool LOW = decltype(low)::value, COPY = decltype(copy_c)::value, PREV = INTER && decltype(prev_c)::value;
            if constexpr (LOW) lower_read(low_slot);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = U0; u < U0 + NU / 2; ++u) {
                if (EXACT || u <= NU - 8 || u < p.units) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[u], x[u % D], INTER && u == 0 ? v16i{} : acc, 0, 0, 0);
                if constexpr (INTER) asm volatile("" : "+v"(acc));
                if (u + D == NU) {   // the next tile's fragments (beyond the last tile: whatever the slot holds, not used)
                    se = ring + xe + after;
                    so = ring + xo + after;
                }
                xload((u + D) % NU);
                if constexpr (COPY) {
                    if ((u - U0) % 3 == 1 && (u - U0) / 3 < NCP) copy((u - U0) / 3);
                }
                if constexpr (LOW) {
                    const int k = u - U0 - 2;
                    if (k >= 0 && k % PSTEP == 0 && k / PSTEP < NCP) lower_write(low_slot, k / PSTEP);
                }
                if constexpr (PREV) {
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (e * (NU - 4) / 16 + 2 == u) value(prev, i - 1, e);
                    if (u == NU - 1) finish(i - 1);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (COPY) copied();
            if constexpr (LOW) wait_lds<NU / 2 - 1 - LASTP>();   // (the fragment reads behind the last piece may be in flight)
        };
        using L = std::integral_constant<bool, LOWIN>;
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        using H0 = std::integral_constant<int, 0>;
        using H1 = std::integral_constant<int, NU / 2>;
        auto tile = [&](int i, auto first, v16i &acc, const v16i &prev) {
            // (in the last rounds the barriers and, behind them, copies of nothing go on, and a slot that nobody reads is lowered
            // again; but a block of two tiles or one does not put them behind its weights)
            constexpr bool FIRST = decltype(first)::value;
            using P = std::integral_constant<bool, !FIRST>;
            if constexpr (!INTER) {
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 0;
            }
            if (!LATE) {
                if (LOWIN && (!FIRST || nt > 1)) {
                    wait_tile();
                    half(H0{}, L{}, after, F{}, P{}, i, acc, prev);
                } else {
                    half(H0{}, F{}, 0, F{}, P{}, i, acc, prev);
                }
                sync();
                if (!FIRST || nt > 2) half(H1{}, F{}, 0, T{}, P{}, i, acc, prev);
                else half(H1{}, F{}, 0, F{}, P{}, i, acc, prev);
            } else {
                if (!FIRST || nt > 2) half(H0{}, F{}, 0, T{}, P{}, i, acc, prev);
                else half(H0{}, F{}, 0, F{}, P{}, i, acc, prev);
                if (LOWIN && (!FIRST || nt > 2)) {
                    wait_tile();
                    half(H1{}, L{}, after == (S - 1) * STAGE ? 0 : after + STAGE, F{}, P{}, i, acc, prev);
                } else {
                    half(H1{}, F{}, 0, F{}, P{}, i, acc, prev);
                }
                if (i + 1 < nt) sync();
            }
            after = after == (S - 1) * STAGE ? 0 : after + STAGE;
            if constexpr (!INTER) leave(acc, i);
            __builtin_amdgcn_sched_barrier(0);
        };
        if (LATE) sync();
        v16i sum0, sum1;
        tile(0, T{}, sum0, sum0);   // (waits for each weight at its first use: a copy of the code that the loop need not carry)
        if constexpr (INTER) {
            int i = 1;
            for (; i + 1 < nt; i += 2) {
                tile(i, F{}, sum1, sum0);
                tile(i + 1, F{}, sum0, sum1);
            }
            if (i < nt) {
                tile(i, F{}, sum1, sum0);
                leave(sum1, nt - 1);
            } else {
                leave(sum0, nt - 1);
            }
        } else {
            for (int i = 1; i < nt; ++i) tile(i, F{}, sum0, sum0);
        }
        wait_vm<0>();   // nothing of this wave's copies is in flight when the block's LDS is released
    };
    if (wave >= kWaves / 2) walk(std::integral_constant<bool, true>{});
    else walk(std::integral_constant<bool, false>{});
}

struct DeviceState {
    bool ready = false;
    int num_cu = 0;
};
static DeviceState g_dev[64];
static int g_force = -1;   // test hook: 1 = whenever the call qualifies, 0 = never, -1 = automatic
static int g_last = 0;

typedef void (*Fn)(const Params);
template <int NU, bool LOWIN, bool EXACT> static Fn pick(int out)
{
    switch (out) {
    case kCodes: return k_wreg<NU, kCodes, LOWIN, EXACT>;
    case kLowered: return k_wreg<NU, kLowered, LOWIN, EXACT>;
    case kFloats: return k_wreg<NU, kFloats, LOWIN, EXACT>;
    case kFloatsAtOnce: return k_wreg<NU, NU <= 32 ? kFloatsAtOnce : kFloats, LOWIN, EXACT>;
    default: return k_wreg<NU, kAny, LOWIN, EXACT>;
    }
}
template <int NU> static Fn pick(int out, bool lowin, bool exact)
{
    return lowin ? (exact ? pick<NU, true, true>(out) : pick<NU, true, false>(out)) : (exact ? pick<NU, false, true>(out) : pick<NU, false, false>(out));
}
static Fn kernel(int nu, int out, bool lowin, bool exact)
{
    switch (nu) {
    case 16: return pick<16>(out, lowin, exact);
    case 24: return pick<24>(out, lowin, exact);
    case 32: return pick<32>(out, lowin, exact);
    default: return pick<40>(out, lowin, exact);
    }
}

}  // namespace wreg

int prepare_wreg_kernels(int device)
{
    using namespace wreg;
    if (device < 0 || device >= 64) return FLEXIQ_EINVAL;
    if (g_dev[device].ready) return FLEXIQ_OK;
    hipDeviceProp_t prop;
    FLEXIQ_HIP(hipGetDeviceProperties(&prop, device));
    g_dev[device].num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    for (int nu = 16; nu <= 40; nu += 8)
        for (int k = 0; k < 4 * kOuts; ++k)
            FLEXIQ_HIP(hipFuncSetAttribute((const void *)kernel(nu, k >> 2, (k & 1) != 0, (k & 2) != 0), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    g_dev[device].ready = true;
    return FLEXIQ_OK;
}

// Launches k_wreg when the call qualifies: plain outputs or int8 rows lowered for a consumer, 288 to 1280 channels (below, the
// weights fit LDS: k_stream; above, they do not fit the registers of 256-column blocks).  It is offered what the kernels for
// few rows and for one short round of blocks leave (where those qualify they are ahead: blocks of one or two tiles pay for the weights alone;
// 3262 x 512 -> 576 at r = 0.5, fp32: 9.1 us against 7.0 in k_halo).  Of that it takes all but the calls that give its blocks several
// tiles and leave too much of the grid unused, in a last round of few tiles or in columns beyond N: the tiled kernel has smaller tiles to
// fill the chip with.  Measured on 10800 calls (200 to 400 thousand rows) by the used share of the grid; time here over time there, geometric
// means.  Rows of whole quads, share below 0.2 / 0.3 / 0.4 / 0.5 / 0.6 / 1: 1.33 / 1.15 / 1.05 / 0.96 / 0.87 / 0.80, hardly changed by how many tiles a block
// walks; int32 sums alone, which the tiled kernel stores in an epilogue of their own: 1.05 to 1.2 up to 0.55.  Rows that leave element by element (N
// not a multiple of 4), whose stores a block hides behind its other tiles: with two or three tiles 1.00 to 1.11 up to 0.6 for one output and
// 1.03 to 1.24 up to 0.8 for more, with more tiles 1.05 to 1.46 below 0.2 and 0.85 to 1.0 beyond.  With one tile per block it is ahead whatever
// the share (0.78, 0.83 and 0.93).
int launch_wreg(const flexiq_layer *L, const int8_t *X, int64_t M, const flexiq_out *out, void *stream_, int *taken, const LowerArgs *lower)
{
    using namespace wreg;
    *taken = 0;
    g_last = 0;
    if (g_force == 0 || L->C <= 256 || L->C > 1280) return FLEXIQ_OK;
    if (g_force < 0 && (few_rows_forced() || stream_forced() || halo_forced())) return FLEXIQ_OK;   // (those hooks compare with the tiled kernel)
    if (out->scan_for || out->x4 || out->x6) return FLEXIQ_OK;
    const bool q_only = out->q && !out->acc && !out->y && (L->N & 15) == 0;
    const bool lowering = lower && lower->ashift;   // (null positions: the consumer has no 4-bit channels at its ratio)
    if (lowering && !q_only) return FLEXIQ_OK;
    const DeviceState &ds = g_dev[L->device];
    if (!ds.ready) return FLEXIQ_OK;
    Params p = {};
    p.units = L->C / kUnit;
    const int nu = (p.units + 7) & ~7;
    const int64_t tiles = (M + kRows - 1) / kRows;
    if (M * L->C >= (1ll << 31)) return FLEXIQ_OK;   // (what is left of X is a 32-bit window)
    p.X = X; p.W8 = L->d_w8; p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift; p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad; p.C = L->C;
    p.w4x_delta = L->U * 32 * L->Npad;
    p.units4 = L->max_4bit_ch / kUnit;
    p.n_low = L->x_prelowered ? 0 : p.units4;
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.ncb = (L->N + kCols - 1) / kCols;
    p.band = std::min(p.ncb, 8);
    p.groups = (int)std::max<int64_t>(1, std::min<int64_t>(tiles, ds.num_cu / p.ncb));
    p.per_group = (int)(tiles / p.groups);
    p.extra = (int)(tiles % p.groups);
    {
        const int per_block = p.per_group + (p.extra > 0 ? 1 : 0), outputs = (out->acc ? 1 : 0) + (out->y ? 1 : 0) + (out->q ? 1 : 0);
        const double used = (double)M * L->N / ((double)ds.num_cu * per_block * kRows * kCols);
        const double least = (L->N & 3) ? (per_block > 3 ? 0.25 : outputs == 1 ? 0.6 : 0.8) : (out->acc && outputs == 1 ? 0.55 : 0.4);
        if (g_force < 0 && per_block > 1 && used < least) return FLEXIQ_OK;
    }
    if (lowering) { p.next_ashift = lower->ashift; p.next_K4 = lower->K4; p.next_gs_log2 = lower->gs_log2; }
    Out kind = lowering ? kLowered : (q_only ? kCodes : (out->y && !out->q && !out->acc && (L->N & 3) == 0 ? kFloats : kAny));
    // fp32 rows beyond the last-level cache (256 MB): spread over the next tile, time over that of rows that leave at once, 3152 x 36864 (465 MB) / 51200 (646 MB) at
    // r = 0: 320 channels 0.90 / 0.93, 384 1.04 / 1.11, 512 1.18 / 1.16, 640 1.05 / 1.14, 768 1.33 / 1.38, 896 0.89 / 0.92, 1024 1.12 / 1.11, 448, 576, 704, 832
    // and 960 0.81 to 0.92; 12608 x 5120 (258 MB) 512 1.00, 768 1.20, 1024 1.10; 12608 x 4096 (207 MB) 0.92 to 1.04.
    if (kind == kFloats) {
        const double bytes = 4.0 * (double)M * L->N;
        if (p.units == nu && nu > 16 ? bytes > 240e6 : (p.units & 3) == 0 && nu < 32 && bytes > 400e6) kind = kFloatsAtOnce;
    }
    const size_t lds = kTabBytes + (size_t)slots(nu) * stage_bytes(nu);
    FLEXIQ_HIP(launch_kernel(kernel(nu, kind, p.n_low > 0, p.units == nu), dim3((unsigned)(p.ncb * p.groups)), dim3(64 * kWaves), lds, stream_, p));
    *taken = 1;
    g_last = kind == kFloatsAtOnce ? 2 : 1;
    return FLEXIQ_OK;
}

}  // namespace flexiq

extern "C" int flexiq_debug_force_wreg(int mode)
{
    if (mode < -1 || mode > 1) return FLEXIQ_EINVAL;
    flexiq::wreg::g_force = mode;
    return flexiq::wreg::g_last;
}
