// Linear layers of up to 1280 channels with all of them on the FP6 matrix path (fp6_kernel.h has the number format, the layouts and why
// the sums are exact), the weights of a block resident in registers as in wreg.hip.
//
// What bounded these calls in the tiled FP6 kernel: an FP6 K-step of 64 channels is 512 matrix cycles of a 256 x 256 tile, shorter than
// the way of its 24 KB of operands from memory into LDS, every block pays for a prologue and an epilogue beside which nothing runs, and
// packing the consumer's FP6 codes took a third of the call.  Here a block of eight waves keeps the weights of 256 columns in registers,
// a wave 32 columns of every K-step (six registers a lane and step), and tiles of 32 rows stream past through a ring of LDS slots.
//   * The sums of a tile leave between the matrix instructions of the next one.  What is computed there is pinned in its place with empty
//     asm: as pure data flow the optimiser moves it past the branches to its use, behind the last matrix instruction (2000 cycles per
//     tile of 16 K-steps instead of 1500; 1090 are matrix instructions).
//   * One barrier per tile, in its middle: behind it the next tile is in place and nobody reads the one before, whose slot takes a new
//     one, copied over the other half.
//   * A tile in LDS is the two 16-byte planes of every K-step, then the 8-byte tails of every K-step.  The sums stay fp32 (exact
//     integers) into the epilogue, which saves its conversion.
//   * A consumer's FP6 codes: five operations make a code of a sum (scale, clamp, round, to the consumer's position, floor), one instruction
//     packs the sixteen of a lane.
// What bounds it now: reads of LDS (24 bytes a lane per 32 matrix cycles, 1020 + 190 cycles per tile of 16 K-steps with the copies) beside
// the matrix instructions, the clock (12608 x 1024 -> 4096 28.1 us on activations and 24.3 on zeros, in the same number of cycles), and about 8 us of weight
// loads, launch and last stores.  Four waves of
// 64 columns, which read half as much, were no faster (0.86 us): one wave per SIMD issues an instruction in four to five cycles.  A form with
// int8 K-steps behind the FP6 ones (a branch per step) needs more registers than there are from 13 K-steps on: 0.4 to 0.97 times the
// tiled kernel's speed.
//
// Measured (graph replays, us in the tiled kernel's build without int8 operands and here, r = 1; int8 codes / fp32 / FP6 codes for a consumer): 12608 x 1024 ->
// 4096 54.0 / 79.3 / 77.2 and 31.9 / 54.5 / 35.6; 12608 x 384 -> 1536 15.0 / 26.1 / 23.9 and 12.1 / 19.7 / 13.1; 400 x 512 -> 512 6.2 / 7.5 / 7.9 and 5.3 / 5.9 /
// 5.4; two tiles per block, 3000 x 1024 -> 1024, 8.4 / 11.1 / 10.2 and 8.3 / 12.5 / 8.7.
#include <algorithm>

#include "flexiq_internal.h"
#include "flexiq_test.h"
#include "stream_common.h"

namespace flexiq {
namespace wreg6 {

using namespace resident;

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v6u __attribute__((ext_vector_type(6)));

struct Params {
    const uint8_t *X6;      // FP6 activations [ceil(M / 64)][S][3][64][16]
    const uint8_t *W6;      // [S][3][Npad][16]
    const uint8_t *W6S;     // [ceil(S / 4)][Npad][2][4]
    const int32_t *ashift;  // [G + 1]
    const float *cs;        // [2][Npad]
    int32_t *acc;
    float *y;
    int8_t *q;
    float r_out;
    int32_t M, N, Npad;
    int32_t S;              // K-steps of 64 channels
    int32_t gs_shift, G;
    int32_t ncb, groups;    // column blocks, row groups: the grid is their product
    int32_t band;           // column blocks that share a band of the grid
    int32_t per_group, extra;     // row tiles of a group, and how many groups take one more
    // the layer that reads the int8 output (kChain)
    uint8_t *nx6;                 // its FP6 activations; null: it gets int8 rows only
    const int32_t *next_ashift;
    int32_t next_K4, next_K6, next_gs_log2, next_S;
};

constexpr int kWaves = 8, kCols = 32 * kWaves, kRows = 32;
constexpr int kTabBytes = 2 * kCols * 4;   // multipliers, addends
// copies of a wave per tile, 1 KB each; every wave has as many (what a layer does not have reads as zeros)
constexpr int copies(int ns) { return (3 * ns / 2 + kWaves - 1) / kWaves; }
constexpr int stage_bytes(int ns) { return 1024 * kWaves * copies(ns); }
constexpr int slots(int ns)
{
    const int n = (160 * 1024 - kTabBytes) / stage_bytes(ns);
    return n < 6 ? n : 6;
}

template <int N> __device__ __forceinline__ void wait_vm()   // at most N vector-memory operations outstanding (the counter has six bits)
{
    constexpr int n = N < 63 ? N : 63;
    __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | ((n >> 4) << 14));
}

// The outputs of a call: any of them; int8 rows and nothing else, N a multiple of 16; those for a consumer (lowered int8 and FP6
// codes); fp32 rows and nothing else, N a multiple of 4.
enum Out { kAny, kCodes, kChain, kFloats };

// NS: K-steps held in registers (C / 64 rounded up to a multiple of four).
template <int NS, Out OUT>
__global__ __launch_bounds__(64 * kWaves, 2) void k_wreg6(const Params p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NCP = copies(NS), STAGE = stage_bytes(NS), S = slots(NS);
    constexpr int D = NS >= 8 ? 4 : 2;   // K-steps that activation fragments are read ahead
    constexpr bool REGTAB = OUT != kAny && NS <= 16;   // the epilogue's constants stay in registers
    static_assert(NS % D == 0 && 2 * D <= NS && S >= 3, "the ring of fragments, read ahead behind the barrier that publishes the next tile; the ring of tiles");
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

    // ---- copies of a row tile.  The per-lane offset carries the whole address inside a tile: the range check of the descriptor then
    // turns what the layer does not have into zeros (kNone is beyond every window).
    constexpr int kNone = 0x7ffffff0;
    int voff[NCP];
#pragma unroll
    for (int j = 0; j < NCP; ++j) {   // 1 KB pieces: planes 0 and 1 of K-step id, then plane 2 of two K-steps
        const int id = wave + kWaves * j, step = id < NS ? id : 2 * (id - NS) + fh;
        voff[j] = step < p.S ? step * 3072 + (id < NS ? 1024 * fh : 2048) + 16 * fr : kNone;
    }
    int asked = 0, next_slot = 0;
    const int block_bytes = p.S * 3072;   // of 64 rows of X6
    const uint8_t *next_x6 = p.X6 + (int64_t)(t0 >> 1) * block_bytes + 512 * (t0 & 1);
    auto copy = [&](int j) {
        const int odd = (t0 + asked) & 1;
        const __amdgpu_buffer_rsrc_t r6 = __builtin_amdgcn_make_buffer_rsrc((void *)next_x6, 0, asked < nt ? block_bytes - 512 * odd : 0, kRsrcFlags);
        const int from = voff[j];   // (an argument of dependent type: the host pass would refuse the size of the copy and drop the kernel)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r6, (lds_ptr_t)(ring + next_slot + 1024 * (wave + kWaves * j)), 16, from, 0, 0, 0);
    };
    auto copied = [&]() {
        next_x6 += (t0 + asked) & 1 ? block_bytes - 512 : 512;
        ++asked;
        next_slot = next_slot == (S - 1) * STAGE ? 0 : next_slot + STAGE;
    };
    auto issue = [&]() {
#pragma unroll
        for (int j = 0; j < NCP; ++j) copy(j);
        copied();
    };
    float cs_t = 0.f, bi_t = 0.f;
    if (tid < kCols) {
        cs_t = p.cs[n_blk + tid];
        bi_t = p.cs[p.Npad + n_blk + tid];
    }
    // block scales 2^(position + 3) as E8M0 bytes: of this lane's column and unit, and of the activations of its unit (four steps a word)
    const int col = n_blk + 32 * wave + fr;
    const int words = (p.S + 3) >> 2;
    int ws[NS / 4], as[NS / 4];
#pragma unroll
    for (int k = 0; k < NS / 4; ++k) {
        ws[k] = k < words ? *reinterpret_cast<const int *>(p.W6S + (((int64_t)k * p.Npad + col) * 2 + fh) * 4) : 0;
        as[k] = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) as[k] |= (130 + p.ashift[min((2 * (4 * k + i) + fh) >> p.gs_shift, p.G)]) << (8 * i);
    }
    issue();
    __builtin_amdgcn_sched_barrier(0);   // (in this order: the waits below count on it)
    // ---- weights of the wave's 32 columns
    v8i w[NS];
    {
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W6, 0, p.S * 3 * p.Npad * 16, kRsrcFlags);
        const int head = (fh * p.Npad + col) * 16, tail = (2 * p.Npad + col) * 16 + 8 * (fh ^ ((col >> 4) & 1));
#pragma unroll
        for (int k = 0; k < NS; ++k) {   // (K-steps the layer does not have: the last one again, not used)
            const int at = (k <= NS - 4 ? k : min(k, p.S - 1)) * 3 * p.Npad * 16;
            const v4i h = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, head, at, 0));
            const v2i t = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rw, tail, at, 0));
            w[k] = (v8i){h.x, h.y, h.z, h.w, t.x, t.y, 0, 0};
        }
    }
    __builtin_amdgcn_sched_barrier(0);   // (likewise)
#pragma unroll
    for (int k = 1; k < S - 1; ++k) issue();

    constexpr bool QONLY = OUT == kCodes || OUT == kChain;
    const bool pre_scaled = QONLY || (p.q != nullptr && p.y == nullptr);
    float *const tab = reinterpret_cast<float *>(lds);
    if (tid < kCols) {
        tab[tid] = pre_scaled ? cs_t * p.r_out : cs_t;
        tab[kCols + tid] = pre_scaled ? bi_t * p.r_out + 128.0f : bi_t;
    }
    // what the consumer does with this wave's columns, one of its units: position, clamp bounds of the offset code, mask
    bool to6 = false;
    float lo = 0.0f, hi = 255.0f, step_inv = 1.0f, step_add = -128.0f;
    uint32_t mask = 0xffffffffu;
    if constexpr (OUT == kChain) {
        const int n = n_blk + 32 * wave;
        if (n < p.next_K4) {
            const int s = p.next_ashift[n >> p.next_gs_log2];
            lo = (float)(128 - (8 << s));
            hi = (float)(127 + (8 << s));
            mask = 0x01010101u * ((0xffu << s) & 0xffu);
            // (both exact in fp32, and so is what they make of a whole number of 0 .. 255)
            step_inv = __int_as_float((127 - s) << 23);
            step_add = -128.0f * step_inv;
        }
        to6 = p.nx6 != nullptr && n < p.next_K6;
    }

    // this wave's copies have landed, but for those of the last S - 3 tiles asked for
    auto wait_tile = [&]() { wait_vm<(S - 3) * NCP>(); };
    wait_vm<2 * NS + (S - 2) * NCP>();   // the first tile is there, weights and later tiles are on their way

    const bool q_rows = p.q != nullptr && (p.N & 15) == 0;
    // fragment addresses inside a tile: 16 bytes and 8 bytes of a K-step (the tail of unit h of row r in half h ^ ((r >> 4) & 1))
    const int xa = 512 * fh + 16 * fr, xb = NS * 1024 + 16 * fr + 8 * (fh ^ (fr >> 4));
    const int lim = p.N - n_blk - 4 * fh;

    // SIX: the wave's columns leave as FP6 codes
    auto walk = [&](auto six_c) {
        constexpr bool SIX = decltype(six_c)::value;
        __builtin_amdgcn_s_waitcnt(0xc07f);
        block_barrier();
        v4i mul[4], add[4];   // the epilogue's constants of a quad of columns
        auto fetch = [&](int k) {
            const int c = 32 * wave + 8 * k + 4 * fh;
            mul[k] = *reinterpret_cast<const v4i *>(lds + 4 * c);
            add[k] = *reinterpret_cast<const v4i *>(lds + 4 * (kCols + c));
            asm volatile("" : "+v"(mul[k]), "+v"(add[k]));
        };
        if constexpr (REGTAB) {
#pragma unroll
            for (int k = 0; k < 4; ++k) fetch(k);
        }
        v8i x[D];
        const unsigned char *slot = ring;
        auto xload = [&](int k) {
            const v4i a = *reinterpret_cast<const v4i *>(slot + xa + 1024 * k);
            const v2i b = *reinterpret_cast<const v2i *>(slot + xb + 512 * k);
            x[k % D] = (v8i){a.x, a.y, a.z, a.w, b.x, b.y, 0, 0};
        };
#pragma unroll
        for (int k = 0; k < D; ++k) xload(k);

        auto mult = [&](int k, v16f &acc) {   // (the first K-step starts from zero)
            const v16f c = k == 0 ? v16f{} : acc;
            const v8i b = x[k % D];
            // (the byte of a scale word is an immediate)
            switch (k & 3) {
            case 0: acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[k], b, c, 2, 2, 0, ws[k >> 2], 0, as[k >> 2]); break;
            case 1: acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[k], b, c, 2, 2, 1, ws[k >> 2], 1, as[k >> 2]); break;
            case 2: acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[k], b, c, 2, 2, 2, ws[k >> 2], 2, as[k >> 2]); break;
            default: acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w[k], b, c, 2, 2, 3, ws[k >> 2], 3, as[k >> 2]); break;
            }
        };

        // ---- epilogue of tile t0 + i: value e of the lane's sixteen (register 4 g + j: column 8 g + 4 fh + j of the wave's), then the rest
        uint32_t qrow[4];
        v4i yq;
        v16f even = {}, odd = {};
        // (what is computed here and there is pinned in its place: as pure data flow the optimiser moves it past the branches, to its use)
        auto value = [&](const v16f &acc, int i, int e) {
            const int k = e >> 2, j = e & 3;
            if constexpr (!REGTAB) {
                if (j == 0) fetch(k);
            }
            const float v = __builtin_fmaf(acc[e], __int_as_float(mul[k][j]), __int_as_float(add[k][j]));
            if constexpr (OUT == kFloats) {
                yq[j] = __float_as_int(v);
                asm volatile("" : "+v"(yq));
                const uint32_t at = (uint32_t)(fr * p.N + n_blk + 32 * wave + 4 * fh + 8 * k) * 4u;
                if (j == 3 && fr < p.M - (t0 + i) * kRows && 32 * wave + 8 * k < lim)
                    *reinterpret_cast<v4i *>(reinterpret_cast<unsigned char *>(p.y + (int64_t)(t0 + i) * kRows * p.N) + at) = yq;
            } else if constexpr (SIX) {
                // element 2 i + h of a fragment's sixteen in entry i of half h: the conversion takes its elements from the two in turn
                const float c = __builtin_rintf(__builtin_amdgcn_fmed3f(v, lo, hi));
                float f = __builtin_floorf(__builtin_fmaf(c, step_inv, step_add));   // (never -0)
                asm volatile("" : "+v"(f));
                if (e & 1) odd[e >> 1] = f;
                else even[e >> 1] = f;
            } else {
                qrow[k] = __builtin_amdgcn_cvt_pk_u8_f32(OUT == kChain ? __builtin_amdgcn_fmed3f(v, lo, hi) : v, j, j == 0 ? 0 : qrow[k]);
                asm volatile("" : "+v"(qrow[k]));
            }
        };
        auto finish = [&](const v16f &acc, int i) {
            const int64_t m0 = (int64_t)(t0 + i) * kRows;
            const bool row_ok = fr < p.M - (t0 + i) * kRows;
            if constexpr (OUT == kAny) {
                const FragOut fo = {p.acc, p.y, p.q, p.r_out, p.N};
                int left_n = lim;
                asm volatile("" : "+v"(left_n));
                v16i whole;
#pragma unroll
                for (int e = 0; e < 16; ++e) whole[e] = (int)acc[e];
                store_fragment<false, kCols>(whole, fo, lds, wave, n_blk, m0 + fr, row_ok, left_n, fh, pre_scaled, q_rows);
            } else if constexpr (SIX) {
                const v6u d = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(even, odd, 8.0f);
                const int unit = (n_blk >> 5) + wave;
                uint8_t *const block = p.nx6 + ((int64_t)((t0 + i) >> 1) * p.next_S + (unit >> 1)) * 3072 + 512 * ((t0 + i) & 1);
                // lanes 0..31: elements 0..15 of the unit, 32..63: the other half, whose first dword belongs to the first 16 bytes
                const auto sw = __builtin_amdgcn_permlane32_swap(d[0], d[0], false, false);
                const int hh = unit & 1;
                // (non-temporal: 34.9 -> 32.6 us on 12608 x 1024 -> 4096; int8 rows that way 31.1 -> 30.7, but 26.3 -> 31.3 on zeros)
                if (row_ok) {
                    if (fh == 0) __builtin_nontemporal_store((v4i){(int)d[0], (int)d[1], (int)d[2], (int)sw[1]}, reinterpret_cast<v4i *>(block + 1024 * hh + (uint32_t)(16 * fr)));
                    else __builtin_nontemporal_store((v2i){(int)d[1], (int)d[2]}, reinterpret_cast<v2i *>(block + 2048 + (uint32_t)(16 * fr + 8 * (hh ^ (fr >> 4)))));
                }
            } else if constexpr (QONLY) {
                const FragOut at = {nullptr, nullptr, p.q + m0 * p.N, 0.0f, p.N};   // (its rows from this tile on)
#pragma unroll
                for (int k = 0; k < 4; ++k) qrow[k] = (qrow[k] ^ 0x80808080u) & (OUT == kChain ? mask : 0xffffffffu);
                store_codes(at, qrow, wave, n_blk, fr, row_ok, lim, fh);
            }
        };

        int after = STAGE;   // slot of the next tile
        // half of a tile's K-steps, from K0 on; COPY: the wave asks for a tile meanwhile (in one go the copies of all waves would hold up
        // each other and the stores)
        auto half = [&](auto begin, auto copy_c, auto first, int i, v16f &acc, const v16f &prev) {
            constexpr int K0 = decltype(begin)::value;
            constexpr bool COPY = decltype(copy_c)::value, FIRST = decltype(first)::value;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = K0; k < K0 + NS / 2; ++k) {
                if (k <= NS - 4 || k < p.S) mult(k, acc);
                asm volatile("" : "+v"(acc));
                if (k + D == NS) slot = ring + after;   // the next tile's fragments (beyond the last tile: whatever the slot holds, not used)
                xload((k + D) % NS);
                if constexpr (COPY) {
#pragma unroll
                    for (int j = 0; j < NCP; ++j)
                        if (j * (NS / 2) / NCP == k - K0) copy(j);
                }
                if constexpr (!FIRST) {
                    if constexpr (OUT != kAny) {
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            if (e * (NS - 2) / 16 + 1 == k) value(prev, i - 1, e);
                    }
                    if (k == NS - 1) finish(prev, i - 1);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (COPY) copied();
        };
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        using H0 = std::integral_constant<int, 0>;
        using H1 = std::integral_constant<int, NS / 2>;
        auto tile = [&](int i, auto first, v16f &acc, const v16f &prev) {
            half(H0{}, F{}, first, i, acc, prev);
            wait_tile();   // (LDS reads may be in flight: their slot is not written before the barrier after this one)
            block_barrier();
            // (in the last rounds copies of nothing go on; but a block of two tiles or one does not put them behind its weights)
            if (!decltype(first)::value || nt > 2) half(H1{}, T{}, first, i, acc, prev);
            else half(H1{}, F{}, first, i, acc, prev);
            after = after == (S - 1) * STAGE ? 0 : after + STAGE;
        };
        auto last = [&](const v16f &acc) {
            if constexpr (OUT != kAny) {
#pragma unroll
                for (int e = 0; e < 16; ++e) value(acc, nt - 1, e);
            }
            finish(acc, nt - 1);
        };
        v16f sum0, sum1;
        tile(0, T{}, sum0, sum0);   // (waits for each weight at its first use: a copy of the code that the loop need not carry)
        int i = 1;
        for (; i + 1 < nt; i += 2) {
            tile(i, F{}, sum1, sum0);
            tile(i + 1, F{}, sum0, sum1);
        }
        if (i < nt) {
            tile(i, F{}, sum1, sum0);
            last(sum1);
        } else {
            last(sum0);
        }
        wait_vm<0>();   // nothing of this wave's copies is in flight when the block's LDS is released
    };
    if constexpr (OUT == kChain) {
        if (to6) walk(std::integral_constant<bool, true>{});
        else walk(std::integral_constant<bool, false>{});
    } else {
        walk(std::integral_constant<bool, false>{});
    }
}

struct DeviceState {
    bool ready = false;
    int num_cu = 0;
};
static DeviceState g_dev[64];
static int g_force = -1;   // test hook: 1 = whenever the call qualifies, 0 = never, -1 = automatic
static int g_last = 0;

typedef void (*Fn)(const Params);
template <int NS> static Fn pick(int out)
{
    switch (out) {
    case kCodes: return k_wreg6<NS, kCodes>;
    case kChain: return k_wreg6<NS, kChain>;
    case kFloats: return k_wreg6<NS, kFloats>;
    default: return k_wreg6<NS, kAny>;
    }
}
static Fn kernel(int ns, int out)
{
    switch (ns) {
    case 4: return pick<4>(out);
    case 8: return pick<8>(out);
    case 12: return pick<12>(out);
    case 16: return pick<16>(out);
    default: return pick<20>(out);
    }
}

// Whether the call is faster here than in the tiled kernel (its build without int8 operands).  Measured on 46800 calls (96 to 25200 rows of 256 to 1280
// channels, 64 to 65536 columns, on 256 compute units), time here over time there, geometric means of a class by its outputs:
//   * what leaves for a consumer 0.70 (FP6 codes) and 0.75 (lowered rows), never above 0.97; one tile per block 0.81 to 0.87, never above 1.06.
//   * two tiles: 0.97 to 1.00 from a used share of the grid of 0.7 on (N not a multiple of 4: 0.8); below that 0.98 for fp32 rows, 1.01 to 1.05 for the
//     others, 1.06 to 1.12 if N is not a multiple of 4.
//   * three to seven: 0.88 to 0.98; N not a multiple of 4 0.92 to 0.95 with fewer rows in a block than in one there and 0.99 to 1.05 with as many; 1.00 to
//     1.08 with more than 224 column blocks, which all bring their weights for few rows.
//   * eight and more: 0.60 to 1.00 while a block has less than 1.3 times the rows of one there.  Beyond (129 column blocks and more leave a part of the
//     chip idle) 1.07 to 1.21 if N is not a multiple of 4, 1.04 to 1.11 for int8 rows that are not whole 16-byte pieces, 0.64 to 0.97 else.
//   * fp32 rows of whole 256 bytes that do not fit the last-level cache (256 MB) leave in pieces of 32 bytes, which memory takes worse than that kernel's:
//     1.18, up to 1.5; sums alone of less than 512 channels 1.11; int8 rows 0.88, but 1.06 with 1.3 times the rows and more.
// By these lines 0.845 of the tiled kernel's time over all calls (0.850 without them), and of the 4300 that are left to it 450 would have been more than 5 % faster here.
static bool ahead(const flexiq_layer *L, int64_t M, const flexiq_out *out, const Params &p, int num_cu, int64_t tiled_rows)
{
    const int outputs = (out->acc ? 1 : 0) + (out->y ? 1 : 0) + (out->q ? 1 : 0), per_block = p.per_group + (p.extra > 0 ? 1 : 0);
    const bool quads = (L->N & 3) == 0, floats = out->y && outputs == 1 && quads, codes = out->q && outputs == 1;
    const int64_t elements = M * L->N, kCache = 1ll << 28;
    if (per_block == 1) return true;
    if ((L->N & 63) == 0 && 4 * elements > kCache && (floats || (out->acc && outputs == 1 && L->C < 512))) return false;
    if (per_block == 2) return floats || (double)elements >= (quads ? 0.7 : 0.8) * num_cu * 2 * kRows * kCols;
    const double rows = (double)per_block * kRows / (double)tiled_rows;
    if (per_block < 8) return 8 * p.ncb <= 7 * num_cu && (quads || rows < 0.95);
    if (rows < 1.3) return true;
    return quads && (!codes || ((L->N & 15) == 0 && elements <= kCache));
}

}  // namespace wreg6

int prepare_wreg6_kernels(int device)
{
    using namespace wreg6;
    if (device < 0 || device >= 64) return FLEXIQ_EINVAL;
    if (g_dev[device].ready) return FLEXIQ_OK;
    hipDeviceProp_t prop;
    FLEXIQ_HIP(hipGetDeviceProperties(&prop, device));
    g_dev[device].num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    for (int ns = 4; ns <= 20; ns += 4)
        for (int k = 0; k < 4; ++k)
            FLEXIQ_HIP(hipFuncSetAttribute((const void *)kernel(ns, k), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    g_dev[device].ready = true;
    return FLEXIQ_OK;
}

// Launches k_wreg6 when the call qualifies: every channel on the FP6 path, 256 to 1280 of them (with fewer the tiled kernel is as fast:
// 6304 x 128 -> 512 5.6 us there, 5.9 here), outputs of any kind, those for a consumer with int8 rows alone and N a multiple of 16.  It is
// offered what the kernels for few rows and few tiles leave, and takes 96 rows and more (below, up to 1.2 times the tiled kernel's 5 to 6 us)
// where it is ahead.
int launch_wreg6(const flexiq_layer *L, const uint8_t *X6, int64_t M, const flexiq_out *out, void *stream, int K6, int64_t tiled_rows, int *taken,
                 const LowerArgs *lower)
{
    using namespace wreg6;
    *taken = 0;
    g_last = 0;
    if (g_force == 0 || K6 != L->C || L->C > 1280 || (g_force < 0 && (L->C < 256 || M < 96))) return FLEXIQ_OK;
    const bool q_only = out->q && !out->acc && !out->y && (L->N & 15) == 0;
    const bool chain = lower && lower->ashift;
    if (chain && !q_only) return FLEXIQ_OK;
    const DeviceState &ds = g_dev[L->device];
    if (!ds.ready) return FLEXIQ_OK;
    Params p = {};
    p.S = L->C / 64;
    const int ns = (p.S + 3) & ~3;
    const int64_t tiles = (M + kRows - 1) / kRows;
    p.X6 = X6; p.W6 = L->d_w6; p.W6S = L->d_w6s;
    p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift;
    p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad;
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.G = L->G;
    p.ncb = (L->N + kCols - 1) / kCols;
    p.band = std::min(p.ncb, 8);
    p.groups = (int)std::max<int64_t>(1, std::min<int64_t>(tiles, ds.num_cu / p.ncb));
    p.per_group = (int)(tiles / p.groups);
    p.extra = (int)(tiles % p.groups);
    if (g_force < 0 && !chain && !ahead(L, M, out, p, ds.num_cu, tiled_rows)) return FLEXIQ_OK;
    if (chain) {
        p.next_ashift = lower->ashift; p.next_K4 = lower->K4; p.next_gs_log2 = lower->gs_log2;
        p.nx6 = lower->x6; p.next_K6 = lower->x6 ? lower->K6 : 0; p.next_S = lower->S;
    }
    const Out kind = chain ? kChain : (q_only ? kCodes : (out->y && !out->q && !out->acc && (L->N & 3) == 0 ? kFloats : kAny));
    const size_t lds = kTabBytes + (size_t)slots(ns) * stage_bytes(ns);
    FLEXIQ_HIP(launch_kernel(kernel(ns, kind), dim3((unsigned)(p.ncb * p.groups)), dim3(64 * kWaves), lds, stream, p));
    *taken = 1;
    g_last = 1;
    return FLEXIQ_OK;
}

}  // namespace flexiq

extern "C" int flexiq_debug_force_wreg6(int mode)
{
    if (mode < -1 || mode > 1) return FLEXIQ_EINVAL;
    flexiq::wreg6::g_force = mode;
    return flexiq::wreg6::g_last;
}
