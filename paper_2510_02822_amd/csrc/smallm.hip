// Few-row calls of the mixed GEMM (at most 64 activation rows): the regime in which the call is a stream of the
// weight matrix and little else, i.e. the one place where the integer path on gfx950 moves fewer bytes as the
// low-bit ratio rises (Section 7: 4-bit groups move half the weight bytes).
//
// The tiled kernel launches one block per 64 x 64 output tile here: 16 to 64 blocks on 256 compute units, each
// walking the whole reduction alone.  The two kernels below give a block a few output columns and split the reduction
// over its waves, which meet in LDS.  Weights never go through LDS: the packed weight layouts hold 16-channel pieces of
// a weight row contiguously, which is both the MFMA fragment order and what a dot-product lane wants, so a lane loads
//   * 8-bit units: 16 bytes from the 8-bit tiles;
//   * 4-bit units: 16 bytes from the position-expanded copy, or 8 bytes of packed 4-bit codes (half the bytes) plus one
//     position byte.
// k_few_rows (3 .. 64 rows) feeds the matrix cores as the tiled kernel does: 4-bit units from the position-expanded int8 copy
// (16 bytes per lane like 8-bit units), their activations bit-lowered (same int8 MFMA, same int32 sums); up to 16 rows against
// weights of 40 MiB and more from the packed codes (P4 builds).
// k_few_rows_dot (1 .. 4 rows) multiplies on the vector ALU, 4-bit units as the packed 4-bit codes (Section 7's shifted
// accumulation): the kernel for calls that are bound by weight bytes.
// Both give the tiled kernel's results bit for bit.
#include <algorithm>

#include "flexiq_internal.h"

namespace flexiq {
namespace smallm {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef short v2s __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kRsrcFlags = 0x00020000;

// What lowers the four int8 lanes of a dword at position s: clamp(v, -(8 << s), (8 << s) - 1) with the low s bits cleared, the bit-lowered
// value L(v, s) put back at its position (Section 4.1); or what leaves them as they are (no select per dword: it is the vector ALU that
// bounds the lowering).
struct Lowering {
    v2s lo, hi;      // the bounds in the upper byte of both 16-bit halves
    uint32_t mask;
    __device__ __forceinline__ Lowering(int s, bool low = true)
    {
        const short l = low ? (short)((-(8 << s)) << 8) : (short)0x8000, h = low ? (short)((((8 << s) - 1) << 8) | 0xFF) : (short)0x7FFF;
        lo = (v2s){l, l};
        hi = (v2s){h, h};
        mask = low ? 0x01010101u * ((0xFFu << s) & 0xFFu) : 0xFFFFFFFFu;
    }
    __device__ __forceinline__ uint32_t operator()(uint32_t d) const
    {
        v2s o = __builtin_bit_cast(v2s, d);   // odd bytes sit on top of the 16-bit halves
        v2s e = o << (short)8;                // even bytes moved up
        o = __builtin_elementwise_min(__builtin_elementwise_max(o, lo), hi);
        e = __builtin_elementwise_min(__builtin_elementwise_max(e, lo), hi);
        const uint32_t r = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, o), __builtin_bit_cast(uint32_t, e), 0x07030501u);
        return r & mask;
    }
};
__device__ __forceinline__ uint32_t lower4(uint32_t d, int s) { return Lowering(s)(d); }

// Eight packed activation codes (a dword: channels 0 .. 3 in the low halves of its bytes, 4 .. 7 in the high halves) put back at position s as int8
// values, code << s: hi = the dword with the wanted halves on top.
__device__ __forceinline__ uint32_t expand4(uint32_t hi, int s)
{
    v2s o = __builtin_bit_cast(v2s, hi);
    v2s e = o << (short)8;
    o = o >> (short)(4 - s);   // (sign-extends; what comes from the other half of the byte is cleared below)
    e = e >> (short)(4 - s);
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, o), __builtin_bit_cast(uint32_t, e), 0x07030501u) & (0x01010101u * ((0xFFu << s) & 0xFFu));
}

// A wave's K-steps ks, ks + stride, ...: `left` of them, D in flight, each slot loaded again as soon as it is used up.  BEGUN: the first D are on their way.
// EXACT: D steps have a path of their own, on which the compiler knows how many loads are in flight; behind loads that depend on `left` the first step waits for all
// of them, and the steps' ways through LDS follow one by one.  r = 0, us with loads in operand order, without that path and with it: 3 x 3520 -> 128 3.25 / 3.53 /
// 3.48, 4 x 864 -> 10912 3.26 / 3.6 / 3.46, 4 x 3936 -> 480 3.5 / 3.75 / 3.6.  (Elsewhere it costs more: FP6 builds of few rows up to 1.07 times slower with
// it, those of a tile per block spill.  Tried: one step's way through LDS ahead of the multiplication: no gain; loads masked to the rows there are: few rows 1.01, tiles of FP6 calls
// of few rows 0.95, of others 1.01.)
template <int D, bool BEGUN, bool EXACT, class Load, class Use>
__device__ __forceinline__ void wave_steps(const Load &load, const Use &use, int ks, int left, int stride)
{
    if (EXACT && !BEGUN && left == D) {
#pragma unroll
        for (int k = 0; k < D; ++k) load(k, ks + k * stride);
#pragma unroll
        for (int k = 0; k < D; ++k) use(k, ks + k * stride);
        return;
    }
    if constexpr (!BEGUN) {
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (k < left) load(k, ks + k * stride);
    }
    for (; left >= 2 * D; left -= D, ks += stride * D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            use(k, ks + k * stride);
            load(k, ks + (k + D) * stride);
        }
    }
#pragma unroll
    for (int k = 0; k < 2 * D - 1; ++k)
        if (k < left) {
            use(k % D, ks + k * stride);
            if (k + D < left) load(k % D, ks + (k + D) * stride);
        }
}

// ---- A block owns 16 output columns and the whole reduction.
//
// Splitting the reduction across blocks makes the slices meet in memory (store, ticket, re-read: three dependent trips;
// built and measured: ViT-L fc2 with 16 rows took 11 us that way, 4.7 us this way).  Here the slices of a column tile are
// the waves of one block (up to sixteen), which meet in LDS: every wave takes the K-steps (64 channels) wave,
// wave + waves, ... of the block's 16 columns, issues the loads of up to four of them at once
// (weight fragments straight into MFMA operand registers: 16 bytes per lane), multiplies with `v_mfma_i32_16x16x64_i8` (lane: weight row
// n0 + lane % 16 resp. activation row 16 f + lane % 16, channels 16 (lane / 16) ... of the K-step) and leaves its
// accumulators in LDS; waves 0 .. MF-1 add them up and run the epilogue of one 16-row fragment each.  One trip to memory
// for the operands and one for the outputs; nothing to zero, nothing to hand in.
// What bounds it, where the weights do not come from memory, is the rate at which a compute unit pulls its operands: a wave load in operand order
// touches sixteen rows of activations with neighbouring lanes, 15 B/clk per compute unit, and every block reads all rows.  They are loaded four lanes to
// a row instead (46 B/clk) and cross the wave's lanes through LDS, and the K-steps in flight are a ring, each slot loaded again as soon as it is used up.
// int8 out, r = 0 / 0.5 / 1, before and now: 16384 x 4096 weights, 16 rows 14.5 / 13.6 / 15.1 and 12.6 / 11.7 / 12.1 us, 8 rows 12.7 / 13.1 / 14.1 and 12.7 / 11.5 / 11.7;
// 1024 x 4096, 16 rows 4.4 / 4.6 / 4.8 and 3.65 / 4.1 / 4.7, 32 rows 6.3 / 6.5 / 6.8 and 4.4 / 5.05 / 6.05.
struct RowsParams {
    const int8_t *X;        // int8 [M][C], stored channel order
    const int8_t *W8;       // [U][2][Npad][16]
    int32_t w4x_delta;      // bytes from the 8-bit tiles to the position-expanded copy of every 4-bit group (same layout)
    const uint8_t *W4;      // [U][Npad][16] packed 4-bit codes                  (k_few_rows_dot)
    const uint8_t *wshift;  // [G + 1][Npad] weight positions                    (k_few_rows_dot)
    const int32_t *ashift;  // [G + 1]
    const float *cs;        // [2][Npad]: x_scale * w_scale, then bias
    int32_t *acc;
    float *y;
    int8_t *q;
    float r_out;
    int32_t M, N, Npad, C;
    int32_t units;          // C / 32
    int32_t units4;         // leading units computed at 4 bits
    int32_t x_pre;          // activations of those units arrive lowered
    int32_t gs_shift;
    int32_t steps;          // K-steps of 64 channels (the last one may hold a single unit)
    // FP6 builds of k_few_rows (the variant of the 4-bit phase on the f8f6f4 matrix path, fp6_kernel.h): the leading s6 K-steps
    // come as FP6 codes, 24 bytes per (row, 32-channel unit), in the layouts of that kernel
    const uint8_t *X6;      // activations [ceil(M/64)][C/64][3][64][16]
    const uint8_t *W6;      // weights [C/64][3][Npad][16]
    const uint8_t *W6S;     // weight block scales [ceil(C/256)][Npad][2][4] (E8M0 bytes of four consecutive K-steps)
    int32_t s6;             // K-steps on the FP6 path (K6 / 64)
    int32_t s4;             // P4 builds of k_few_rows: leading K-steps from packed codes
    // optional: the layer that reads the int8 output (flexiq_out.lower_for): its positions, 4-bit prefix, log2 of its group size;
    // the codes of its 4-bit channels then leave clamped and masked at its positions (Section 4.1 applied at the producer)
    const int32_t *next_ashift;
    int32_t next_K4, next_gs_log2;
    uint8_t *nx6;           // optional (k_tile_splitk, FP6 calls): the consumer's FP6 activation buffer; its leading next_K6 channels
    int32_t next_K6, next_S;   //   leave as FP6 codes as well (next_S = its C / 64)
    const uint8_t *X4;      // optional (k_few_rows_dot, k_tile_splitk): packed activation codes [M][C / 2] of the leading pieces_p pieces of a row
    int32_t pieces_p;       // 16-channel pieces whose codes come from X4 (a multiple of 4: whole K-steps)
    uint8_t *nx4;           // optional (k_tile_splitk): the consumer's packed activation buffer [M][N / 2]; its leading next_K4P channels
    int32_t next_K4P;       //   leave as codes there instead of in q (a multiple of 64)
};

constexpr int kRowCols = 16;   // output columns per block

// MF: 16-row fragments of activations (M <= 16 MF).  COOP (MF = 1, at most 8 rows, activations not lowered yet): the 4-bit
// channels of the rows are lowered once per block into LDS instead of per lane in fragment layout.  FP6: the leading s6
// K-steps run on the FP6 matrix path first (`v_mfma_scale_f32_16x16x128_f8f6f4`: two K-steps per instruction, a lane holds
// the 32 codes of one unit and its block scale; exact integer sums in fp32, see fp6_kernel.h), every other K-step as usual
// with activations that arrive lowered.
// P4 (MF = 1, groups of 64): the leading s4 K-steps, the 4-bit groups, read the packed codes, half the bytes.  What made their
// expansion cost more than it saved was the sign and the position of every code; here a code stays where it is in the upper
// half of its byte, code * 16 as an int8 value, two operations per four codes (`and`, or `shift` and `and`), and the position
// of a column, one per group, is applied to the group's four sums of a lane, exactly: sum >> (4 - position).
// (Groups of 32, two matrix instructions per K-step, half of each masked: on 67 MB of weights 2 % faster with 16 rows and 4 to 6 % with 5, slower below. Not kept.)
template <int MF, bool COOP, bool FP6 = false, bool P4 = false>
__global__ __launch_bounds__(1024) void k_few_rows(const RowsParams p)
{
    static_assert(!P4 || (MF == 1 && !FP6 && !COOP), "packed codes: up to 16 rows, lowered by every wave");
    static_assert(!COOP || MF == 1, "the cooperative pass is for calls of a few rows");
    static_assert(!(COOP && FP6), "FP6 calls bring lowered activations");
    extern __shared__ __align__(16) unsigned char lds[];   // [waves][MF][64 lanes] accumulator quads, then (COOP) the lowered rows
    v4i *const red = reinterpret_cast<v4i *>(lds);
    const int xl_stride = 32 * p.units4 + 16;   // (+16: rows start in different banks)
    unsigned char *const xl = lds + (blockDim.x >> 6) * MF * 1024;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)(blockDim.x >> 6);
    const int c = lane & 15, qd = lane >> 4;   // row of the fragment (weight row / activation row), 16-channel quarter of the K-step
    const int n0 = blockIdx.x * kRowCols;
    const int n = n0 + c;                      // < Npad: the weight tiles are padded

    // the epilogue's scales and biases travel with the first operands (waves 0 .. MF-1: fragment `wave`, rows 16 wave + c,
    // output channels n0 + 4 qd + i)
    float cs4[4] = {0.f, 0.f, 0.f, 0.f}, bi4[4] = {0.f, 0.f, 0.f, 0.f};
    if (wave < MF) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            cs4[i] = p.cs[n0 + 4 * qd + i];
            bi4[i] = p.cs[p.Npad + n0 + 4 * qd + i];
        }
    }
    // ... and so does the consumer's position of these four columns (flexiq_out.lower_for; 4: no 4-bit channels of a consumer)
    const int sn_pre = wave < MF && p.next_ashift != nullptr && n0 + 4 * qd < p.next_K4 ? p.next_ashift[(n0 + 4 * qd) >> p.next_gs_log2] : 4;

    v4i acc[MF];
#pragma unroll
    for (int f = 0; f < MF; ++f) acc[f] = (v4i){0, 0, 0, 0};

    int ks0 = wave;
    if constexpr (FP6) {
        // chunks of two FP6 K-steps (128 channels), dealt to the waves in turn; the int8 K-steps after them continue the deal
        const int chunks = (p.s6 + 1) >> 1, S = p.C >> 6;
        v4f accf[MF];
#pragma unroll
        for (int f = 0; f < MF; ++f) accf[f] = (v4f){0.f, 0.f, 0.f, 0.f};
        constexpr int U6 = 2;   // chunks in flight
        for (int c0 = wave; c0 < chunks; c0 += nw * U6) {
            v4i wlo[U6], xlo[U6][MF];
            v2i whi[U6], xhi[U6][MF];
            int wsc[U6], asc[U6];
#pragma unroll
            for (int k = 0; k < U6; ++k) {
                const int ks = 2 * (c0 + k * nw) + (qd >> 1), h = qd & 1;   // this lane's K-step and unit
                const bool ok = ks < p.s6;
                wlo[k] = (v4i){0, 0, 0, 0};
                whi[k] = (v2i){0, 0};
                wsc[k] = asc[k] = 127;
                if (ok) {
                    // the first 16 code bytes of unit h in plane h, the last 8 of both units in plane 2 (unit h in half h ^ ((row / 16) % 2))
                    wlo[k] = *reinterpret_cast<const v4i *>(p.W6 + (((int64_t)ks * 3 + h) * p.Npad + n) * 16);
                    whi[k] = *reinterpret_cast<const v2i *>(p.W6 + (((int64_t)ks * 3 + 2) * p.Npad + n) * 16 + 8 * (h ^ ((n >> 4) & 1)));
                    wsc[k] = p.W6S[((int64_t)(ks >> 2) * p.Npad + n) * 8 + 4 * h + (ks & 3)];
                    asc[k] = 130 + p.ashift[(2 * ks + h) >> p.gs_shift];   // 2^(position + 3): the codes are k / 8
                }
#pragma unroll
                for (int f = 0; f < MF; ++f) {
                    const int m = 16 * f + c, blk = m >> 6, r = m & 63;
                    xlo[k][f] = (v4i){0, 0, 0, 0};
                    xhi[k][f] = (v2i){0, 0};
                    if (ok && m < p.M) {
                        xlo[k][f] = *reinterpret_cast<const v4i *>(p.X6 + ((((int64_t)blk * S + ks) * 3 + h) * 64 + r) * 16);
                        xhi[k][f] = *reinterpret_cast<const v2i *>(p.X6 + ((((int64_t)blk * S + ks) * 3 + 2) * 64 + r) * 16 + 8 * (h ^ ((r >> 4) & 1)));
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < U6; ++k)
#pragma unroll
                for (int f = 0; f < MF; ++f)
                    accf[f] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        (v8i){wlo[k].x, wlo[k].y, wlo[k].z, wlo[k].w, whi[k].x, whi[k].y, 0, 0},
                        (v8i){xlo[k][f].x, xlo[k][f].y, xlo[k][f].z, xlo[k][f].w, xhi[k][f].x, xhi[k][f].y, 0, 0}, accf[f], 2, 2, 0, wsc[k], 0, asc[k]);
        }
#pragma unroll
        for (int f = 0; f < MF; ++f)
            acc[f] = (v4i){(int)accf[f].x, (int)accf[f].y, (int)accf[f].z, (int)accf[f].w};   // exact integers below 2^24
        ks0 = p.s6 + (wave + nw - chunks % nw) % nw;
    }
    // ---- activations of a K-step: loaded four lanes to a row (neighbouring lanes on neighbouring pieces; rows beyond M read as zero), they cross
    // the wave's lanes through its own part of LDS (no barrier: LDS serves a wave's accesses in order).  The pad unit of an odd unit count
    // has zero weights.
    unsigned char *const mine = lds + wave * MF * 1024;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)p.X, 0, p.M * p.C, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W8, 0, 2 * p.w4x_delta, kRsrcFlags);
    const int xr = lane >> 2, xp = lane & 3;   // row of a fragment and 16-byte piece of the K-step that this lane loads
    const int xoff = xr * p.C + 16 * xp;
    unsigned char *const put = mine + xr * 64 + 16 * (xp ^ (xr >> 2));
    const unsigned char *const get = mine + c * 64 + 16 * (qd ^ (c >> 2));
    const unsigned char *const own = xl + min(c, p.M - 1) * xl_stride + 16 * qd;   // (COOP: rows beyond M are computed from the last one and not stored)
    const int woff = (qd * p.Npad + n) * 16;
    auto load_x = [&](v4i &x, int f, int ks) { x = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, xoff + 16 * f * p.C + 64 * ks, 0, 0)); };
    auto cross = [&](const v4i (&x)[MF], v4i (&b)[MF]) {
#pragma unroll
        for (int f = 0; f < MF; ++f) *reinterpret_cast<v4i *>(put + 1024 * f) = x[f];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int f = 0; f < MF; ++f) b[f] = *reinterpret_cast<const v4i *>(get + 1024 * f);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // weight fragments.  4-bit units come from the position-expanded copy (code << w_shift as int8, 16 bytes per lane like an 8-bit unit):
    // measured against the packed codes expanded in registers (8 bytes and a position byte per lane, 22 vector-ALU operations per 16 codes)
    // it is faster at every size (ViT-L fc2, 16 rows, r = 1: 5.2 against 6.1 us; 16384 x 4096 weights, 8 rows: 16.1 against 18.7 us): what the
    // packed codes save in bytes that expansion costs in instructions.  One and two rows, where bytes decide, go to k_few_rows_dot;
    // the P4 builds have a cheaper expansion.
    constexpr int UN = MF <= 3 ? 4 : 3;   // K-steps in flight per wave, each slot loaded again as soon as it is used up
    v4i w8[UN], x[UN][MF];
    int sa0[UN], sa1[UN];
    auto load8 = [&](int k, int ks) {
        if (!COOP && !FP6 && !p.x_pre) {   // (scalar, and ahead of its use; the table has an entry for the pad unit)
            sa0[k] = p.ashift[2 * ks >> p.gs_shift];
            sa1[k] = p.ashift[(2 * ks + 1) >> p.gs_shift];
        }
        w8[k] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, woff + (2 * ks + (qd >> 1) < p.units4 ? p.w4x_delta : 0), ks * 64 * p.Npad, 0));
        if (!COOP || 2 * ks + 1 >= p.units4) {   // (COOP: a K-step all of 4-bit units is in LDS, lowered)
#pragma unroll
            for (int f = 0; f < MF; ++f) load_x(x[k][f], f, ks);
        }
    };
    auto use8 = [&](int k, int ks) {
        if (!COOP && !FP6 && !p.x_pre && 2 * ks < p.units4) {
            const Lowering lower(xp >> 1 ? sa1[k] : sa0[k], 2 * ks + (xp >> 1) < p.units4);   // (... or a unit read at 8 bits)
#pragma unroll
            for (int f = 0; f < MF; ++f)
#pragma unroll
                for (int i = 0; i < 4; ++i) x[k][f][i] = (int)lower((uint32_t)x[k][f][i]);
        }
        v4i b[MF];
        if (COOP && 2 * ks + 1 < p.units4) {
            b[0] = *reinterpret_cast<const v4i *>(own + 64 * ks);
        } else {
            cross(x[k], b);
            if (COOP && 2 * ks < p.units4 && qd < 2) b[0] = *reinterpret_cast<const v4i *>(own + 64 * ks);
        }
#pragma unroll
        for (int f = 0; f < MF; ++f) acc[f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w8[k], b[f], acc[f], 0, 0, 0);
    };
    // packed K-steps wave, wave + nw, ... of the leading s4
    constexpr int U4 = 4;   // (eight in flight: more code to fetch, slower at every size)
    v2i w4[P4 ? U4 : 1];
    uint32_t ws4[P4 ? U4 : 1];
    v4i x4[P4 ? U4 : 1][MF];
    int sa4[P4 ? U4 : 1];
    auto load4 = [&](int k, int ks) {
        const int u = 2 * ks + (qd >> 1), h = qd & 1;
        w4[k] = *reinterpret_cast<const v2i *>(p.W4 + ((int64_t)u * p.Npad + n) * 16 + 8 * h);
        ws4[k] = *reinterpret_cast<const uint32_t *>(p.wshift + (int64_t)ks * p.Npad + n0 + 4 * qd);   // (the K-step is a group)
        if (!p.x_pre) sa4[k] = p.ashift[ks];
        load_x(x4[k][0], 0, ks);
    };
    auto use4 = [&](int k, int ks) {
        if (!p.x_pre) {
#pragma unroll
            for (int i = 0; i < 4; ++i) x4[k][0][i] = (int)lower4((uint32_t)x4[k][0][i], sa4[k]);
        }
        v4i b[MF];
        cross(x4[k], b);
        const v4i a = {(w4[k].x << 4) & (int)0xf0f0f0f0, w4[k].x & (int)0xf0f0f0f0, (w4[k].y << 4) & (int)0xf0f0f0f0, w4[k].y & (int)0xf0f0f0f0};
        const v4i t = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b[0], (v4i){0, 0, 0, 0}, 0, 0, 0);
        const uint32_t down = 0x04040404u - ws4[k];   // (positions are 0 .. 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][i] += t[i] >> ((down >> (8 * i)) & 31u);
    };
    auto count = [&](int first, int end) { return first < end ? (end - first + nw - 1) / nw : 0; };
    int left4 = 0;
    if constexpr (P4) {
        left4 = count(wave, p.s4);
#pragma unroll
        for (int k = 0; k < U4; ++k)
            if (k < left4) load4(k, wave + k * nw);
        ks0 = p.s4 + (wave + nw - p.s4 % nw) % nw;   // (the deal goes on with the other K-steps)
    }
    const int left8 = count(ks0, p.steps);
    if constexpr (P4) wave_steps<U4, true, false>(load4, use4, wave, left4, nw);
    if constexpr (COOP) {
#pragma unroll
        for (int k = 0; k < UN; ++k)
            if (k < left8) load8(k, ks0 + k * nw);   // (a wave beyond the last K-step loads nothing)
        // few rows: in the fragment layout most lanes would hold no row, and lowering there would cost every wave the full
        // instruction count for a handful of values.  The block lowers the 4-bit channels of its rows once, every lane a
        // 16-byte piece, into LDS, while the first weight fragments are on their way.
        const int per_row = 2 * p.units4;   // pieces per row
        for (int i = tid; i < p.M * per_row; i += (int)blockDim.x) {
            const int m = i / per_row, j = i - m * per_row;
            const v4i v = *reinterpret_cast<const v4i *>(p.X + (int64_t)m * p.C + 16 * j);
            const int s_ = p.ashift[(j >> 1) >> p.gs_shift];
            *reinterpret_cast<v4i *>(xl + m * xl_stride + 16 * j) =
                (v4i){(int)lower4((uint32_t)v.x, s_), (int)lower4((uint32_t)v.y, s_), (int)lower4((uint32_t)v.z, s_), (int)lower4((uint32_t)v.w, s_)};
        }
        __syncthreads();
    }
    wave_steps<UN, COOP, !FP6 && !P4>(load8, use8, ks0, left8, nw);

    // ---- the waves' sums meet in LDS
#pragma unroll
    for (int f = 0; f < MF; ++f) red[(wave * MF + f) * 64 + lane] = acc[f];
    __syncthreads();
    if (wave >= MF) return;
    v4i s = {0, 0, 0, 0};
    for (int w = 0; w < nw; ++w) s += red[(w * MF + wave) * 64 + lane];

    // ---- epilogue.  Lane: row m = 16 wave + c; accumulator register i: output channel n0 + 4 qd + i
    const int m = 16 * wave + c;
    if (m >= p.M) return;
    const int nn0 = n0 + 4 * qd;
    if (nn0 >= p.N) return;
    const int64_t o = (int64_t)m * p.N + nn0;
    float yv[4];
    uint32_t qw = 0;
    // the consumer's position for these four columns (one channel group of the consumer: nn0 is a multiple of four)
    const bool lower = p.next_ashift != nullptr && nn0 < p.next_K4;
    const int sn = sn_pre;
    const float lo = 128.0f - (float)(8 << sn), hi = 127.0f + (float)(8 << sn);   // (position 4: the whole int8 range)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        yv[i] = __builtin_fmaf((float)s[i], cs4[i], bi4[i]);
        // offset form, as in the tiled kernel: round to nearest-even, saturate to 0..255, flip the top bit; for a consumer's
        // 4-bit channel the offset code is clamped first (integer bounds: the same as clamping the rounded code)
        qw = __builtin_amdgcn_cvt_pk_u8_f32(
            __builtin_amdgcn_fmed3f(__builtin_fmaf((float)s[i], cs4[i] * p.r_out, bi4[i] * p.r_out + 128.0f), lo, hi), i, qw);
    }
    qw ^= 0x80808080u;
    if (lower) qw &= 0x01010101u * ((0xFFu << sn) & 0xFFu);
    if ((p.N & 3) == 0) {   // four whole columns, aligned rows
        if (p.acc) *reinterpret_cast<v4i *>(p.acc + o) = s;
        if (p.y) *reinterpret_cast<float4 *>(p.y + o) = make_float4(yv[0], yv[1], yv[2], yv[3]);
        if (p.q) *reinterpret_cast<uint32_t *>(p.q + o) = qw;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (nn0 + i >= p.N) continue;
            if (p.acc) p.acc[o + i] = s[i];
            if (p.y) p.y[o + i] = yv[i];
            if (p.q) p.q[o + i] = (int8_t)(qw >> (8 * i));
        }
    }
}

// ---- Calls of at most four rows: matrix-vector products on the vector ALU's integer dot instructions.
//
// With so few rows the matrix cores have nothing to reuse a weight fragment for, and their 16-column fragments tie the
// block count to N / 16.  Here a lane multiplies a 16-channel piece of one weight row with the same piece of every
// activation row: 8-bit units with `v_dot4_i32_i8` (four per piece and row), 4-bit units with `v_dot8_i32_i4` on the packed
// codes as they are stored (two per piece and row; the sum of code products is put at its position afterwards,
// sum << (activation position + weight position): Section 7's shifted accumulation, one `v_lshl_add_u32`).  This is the one
// place on this chip where 4-bit groups cost fewer bytes AND fewer operations than 8-bit ones: nothing is expanded.
// The activation codes of the 4-bit channels are produced once per block (clamp at the group's position, Section 4.1,
// then two codes per byte in the order of the packed weights) and kept in LDS.  A block owns 8 output columns (a
// wave load covers 8 columns x 8 pieces: 128-byte runs of the weight tiles) and the whole reduction; lanes of a
// column meet by cross-lane adds, waves in LDS.
constexpr int kVecCols = 8;

// MR: activation rows (1 .. 4).  CG: groups of 8 columns per block (1 or 4; a lane then holds a piece of CG weight rows per
// activation piece: more bytes in flight per wave, activation pieces and the block's set-up shared by more columns; for
// layers with enough columns to still give every compute unit several blocks).
template <int MR, int CG>
__global__ __launch_bounds__(512) void k_few_rows_dot(const RowsParams p)
{
    // LDS: [waves][MR][8 CG] wave sums, then [MR][units4][16] packed activation codes, then [MR][C] the activation rows
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int BC = kVecCols * CG;   // columns per block
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)(blockDim.x >> 6);
    int *const red = reinterpret_cast<int *>(lds);
    unsigned char *const xl = lds + nw * MR * BC * 4;
    const int xl_stride = 16 * p.units4;
    unsigned char *const xr = xl + MR * xl_stride;   // (8-bit channels only are read from here)
    const int col = lane & 7, sub = lane >> 3;   // column of a group, piece of the wave load
    const int n0 = blockIdx.x * BC;
    const int n = n0 + col;                      // + 8 c for column group c; < Npad (checked by the launcher)
    const int pieces = 2 * p.units;              // 16-channel pieces of the reduction
    const int groups = (pieces + 7) >> 3;        // wave loads of 8 pieces

    // the epilogue's scale and bias travel with the first operands (thread BC m + j: row m, column n0 + j)
    float cs_e = 0.f, bi_e = 0.f;
    if (tid < MR * BC) {
        cs_e = p.cs[n0 + tid % BC];
        bi_e = p.cs[p.Npad + n0 + tid % BC];
    }
    // ... and so does the consumer's position of that column (flexiq_out.lower_for; 4: no 4-bit channel of a consumer)
    const int sn_e = tid < MR * BC && p.next_ashift != nullptr && n0 + tid % BC < p.next_K4 ? p.next_ashift[(n0 + tid % BC) >> p.next_gs_log2] : 4;
    constexpr int UN = CG == 4 ? 2 : 4;   // wave loads in flight per wave and column group
    v4i w8[UN][CG];
    v2i w4[UN][CG];
    int sh[UN][CG], sa[UN];
    bool low[UN], valid[UN];
    auto issue = [&](int g0) {
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            const int j = 8 * (g0 + k * nw) + sub;   // this lane's piece: unit j / 2, half j % 2
            const int u = j >> 1;
            valid[k] = g0 + k * nw < groups && j < pieces;
            low[k] = valid[k] && u < p.units4;
            sa[k] = 0;
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                w8[k][c] = (v4i){0, 0, 0, 0};
                w4[k][c] = (v2i){0, 0};
                sh[k][c] = 0;
            }
            if (low[k]) {
#pragma unroll
                for (int c = 0; c < CG; ++c) {
                    w4[k][c] = *reinterpret_cast<const v2i *>(p.W4 + ((int64_t)u * p.Npad + n + 8 * c) * 16 + 8 * (j & 1));
                    sh[k][c] = p.wshift[(int64_t)(u >> p.gs_shift) * p.Npad + n + 8 * c];
                }
                sa[k] = p.ashift[u >> p.gs_shift];
            } else if (valid[k]) {
#pragma unroll
                for (int c = 0; c < CG; ++c) w8[k][c] = *reinterpret_cast<const v4i *>(p.W8 + ((int64_t)j * p.Npad + n + 8 * c) * 16);
            }
        }
    };
    int g0 = wave;
    issue(g0);   // (a wave beyond the last piece loads nothing)

    // ---- the activation rows go to LDS once per block (the eight columns of a wave load read the same pieces: a broadcast
    // there, a trip through the vector memory path per lane otherwise); every thread one 16-channel piece of one row at a
    // time: 8-bit channels as they are, 4-bit channels as codes
    {
        const int per_row = 2 * p.units4, all_per_row = 2 * p.units;
        for (int i = tid; i < p.M * (all_per_row - per_row); i += (int)blockDim.x) {
            const int m = i / (all_per_row - per_row), j = per_row + i - m * (all_per_row - per_row);
            *reinterpret_cast<v4i *>(xr + m * p.C + 16 * j) = *reinterpret_cast<const v4i *>(p.X + (int64_t)m * p.C + 16 * j);
        }
        for (int i = tid; i < p.M * per_row; i += (int)blockDim.x) {
            const int m = i / per_row, j = i - m * per_row;
            if (j < p.pieces_p) {   // the producer has made the codes (same layout: flexiq_lower_packed4, flexiq_out.x4)
                *reinterpret_cast<v2i *>(xl + m * xl_stride + 8 * j) = *reinterpret_cast<const v2i *>(p.X4 + (int64_t)m * (p.C >> 1) + 8 * j);
                continue;
            }
            const v4i v = *reinterpret_cast<const v4i *>(p.X + (int64_t)m * p.C + 16 * j);
            const int s_ = p.ashift[(j >> 1) >> p.gs_shift];
            // lowered bytes are code << s with the low s bits clear, so a dword-wide shift right leaves the code's two's
            // complement nibble at the bottom of every byte; dword e of a piece: channels 8 e .. 8 e + 3 in the low
            // halves of its bytes, 8 e + 4 .. 8 e + 7 in the high halves (the order of the packed weight codes)
            const uint32_t a = (lower4((uint32_t)v.x, s_) >> s_) & 0x0F0F0F0Fu, b = (lower4((uint32_t)v.y, s_) >> s_) & 0x0F0F0F0Fu;
            const uint32_t c = (lower4((uint32_t)v.z, s_) >> s_) & 0x0F0F0F0Fu, d = (lower4((uint32_t)v.w, s_) >> s_) & 0x0F0F0F0Fu;
            *reinterpret_cast<v2i *>(xl + m * xl_stride + 8 * j) = (v2i){(int)(a | (b << 4)), (int)(c | (d << 4))};
        }
        __syncthreads();
    }

    int acc[MR][CG];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int c = 0; c < CG; ++c) acc[m][c] = 0;
    for (;;) {
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            const int j = 8 * (g0 + k * nw) + sub;
            if (low[k]) {
#pragma unroll
                for (int m = 0; m < MR; ++m) {
                    const v2i xc = m < p.M ? *reinterpret_cast<const v2i *>(xl + m * xl_stride + 8 * j) : (v2i){0, 0};
#pragma unroll
                    for (int c = 0; c < CG; ++c) {
                        int t = __builtin_amdgcn_sdot8(w4[k][c].x, xc.x, 0, false);
                        t = __builtin_amdgcn_sdot8(w4[k][c].y, xc.y, t, false);
                        acc[m][c] += (int)((uint32_t)t << (sh[k][c] + sa[k]));
                    }
                }
            } else if (valid[k]) {
#pragma unroll
                for (int m = 0; m < MR; ++m) {
                    const v4i xv = m < p.M ? *reinterpret_cast<const v4i *>(xr + m * p.C + 16 * j) : (v4i){0, 0, 0, 0};
#pragma unroll
                    for (int c = 0; c < CG; ++c) {
                        int t = __builtin_amdgcn_sdot4(w8[k][c].x, xv.x, acc[m][c], false);
                        t = __builtin_amdgcn_sdot4(w8[k][c].y, xv.y, t, false);
                        t = __builtin_amdgcn_sdot4(w8[k][c].z, xv.z, t, false);
                        acc[m][c] = __builtin_amdgcn_sdot4(w8[k][c].w, xv.w, t, false);
                    }
                }
            }
        }
        g0 += nw * UN;
        if (g0 >= groups) break;
        issue(g0);
    }

    // ---- the eight lanes of a column, then the waves
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            int a = acc[m][c];
            a += __shfl_xor(a, 8);
            a += __shfl_xor(a, 16);
            a += __shfl_xor(a, 32);
            if (sub == 0) red[(wave * MR + m) * BC + 8 * c + col] = a;
        }
    __syncthreads();
    if (tid >= MR * BC) return;
    const int m = tid / BC, jn = tid % BC, nn = n0 + jn;
    if (m >= p.M || nn >= p.N) return;
    int v = 0;
    for (int w = 0; w < nw; ++w) v += red[(w * MR + m) * BC + jn];
    const float c = cs_e, b = bi_e;
    const int64_t o = (int64_t)m * p.N + nn;
    if (p.acc) p.acc[o] = v;
    if (p.y) p.y[o] = __builtin_fmaf((float)v, c, b);
    if (p.q) {
        // offset form, as in the tiled kernel: round to nearest-even, saturate to 0..255, flip the top bit
        // (for a 4-bit channel of the consumer named by lower_for: clamped and masked at its position, as in k_few_rows)
        const bool lower = p.next_ashift != nullptr && nn < p.next_K4;
        const int sn = sn_e;
        const float t = __builtin_amdgcn_fmed3f(__builtin_fmaf((float)v, c * p.r_out, b * p.r_out + 128.0f), 128.0f - (float)(8 << sn),
                                                127.0f + (float)(8 << sn));
        uint32_t code = __builtin_amdgcn_cvt_pk_u8_f32(t, 0, 0u) ^ 0x80u;
        if (lower) code &= (0xFFu << sn) & 0xFFu;
        p.q[o] = (int8_t)code;
    }
}

// ---- Calls of 65 rows to about a thousand on layers with few output tiles: a 64 x 64 tile per block, the reduction split
// over its waves.
//
// The tiled kernel gives such a call a handful of 64 x 64 blocks that each walk the whole reduction, one barrier per
// K-step: bound by the latency of a step (ViT-L fc2 with 197 rows: 64 steps, 14.6 us at r = 0 and 22.1 us at r = 1 for
// 0.3 us of matrix work).  Here the eight waves of a block take the K-steps wave, wave + 8, ... of the tile on their own
// (every byte of the tile's weights and activations is loaded by exactly one lane of the block), sixteen v_mfma_i32_16x16x64_i8
// per K-step and wave, no barrier until the waves' sums meet in LDS.  4-bit units come from the position-expanded weight copy and
// their activations are lowered in registers.
// What bounds it is the rate at which a compute unit pulls its operands, and that depends on which lane loads what: a wave load whose
// neighbouring lanes read neighbouring 16-byte pieces (64 or more bytes of a row) delivers 46 B/clk per compute unit, one in the order of the MFMA operand
// (neighbouring lanes on sixteen different rows) 15 (128 KB per block, 256 blocks: 2850 and 8560 cycles).  The packed weights lie in operand
// order; activation rows do not.  They are loaded four lanes to a row and cross the wave's lanes through its own part of LDS (no barrier:
// LDS serves a wave's accesses in order).  The sums are finished four lanes to a row as well, so the stores are whole 64-byte runs of fp32.
// int8 out, r = 0 / 0.5 / 1, loaded in operand order and now: 197 x 4096 -> 1024 7.4 / 7.7 / 8.1 and 5.5 / 6.1 / 7.0 us; 512 x 3072 -> 768 7.3 / 7.6 / 7.9
// and 5.7 / 6.0 / 6.7; 1024 x 4096 -> 1024 13.9 / 14.2 / 14.6 and 11.5 / 12.3 / 14.1; 40 x 832 -> 192 3.75 / 3.9 / 4.1 and 3.1 / 3.3 / 3.4.  (Tried: masking
// alone where no byte of a wave reaches the clamp: no gain, a wave of 1024 and more activations nearly always holds one.)
// FR x FC: 16 x 16 fragments of the tile (rows x columns), NW: waves.  A smaller tile means more blocks, i.e. more compute
// units pulling operands, at more operand bytes per multiply.
// FP6: the leading s6 K-steps run first on `v_mfma_scale_f32_16x16x128_f8f6f4`, as in the FP6 build of k_few_rows (chunks of
// two K-steps dealt to the waves in turn; a lane holds the 32 codes of one unit and its block scale), every other K-step as
// usual with activations that arrive lowered.
// XP: the leading K-steps of activations are read from packed codes.
template <int FR, int FC, int NW, int UN, bool FP6 = false, bool XP = false>
__global__ __launch_bounds__(64 * NW) void k_tile_splitk(const RowsParams p)
{
    constexpr int kTileRows = 16 * FR, kTileCols = 16 * FC, kTileWaves = NW, NF = FR * FC;
    constexpr int E = (NF + NW - 1) / NW;   // fragments a wave finishes: wave, wave + NW, ...
    constexpr int kStage = NF > FR ? NF : FR;   // KB of LDS per wave: its sums, and before that the activations that cross its lanes
    extern __shared__ __align__(16) unsigned char lds[];   // [waves][fragments][64 lanes] accumulator quads
    v4i *const red = reinterpret_cast<v4i *>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, qd = lane >> 4;
    const int n0 = blockIdx.x * kTileCols;      // columns n0 + 16 g + c < Npad: the weight tiles are padded
    const int m0 = blockIdx.y * kTileRows;

    // the epilogue's scales and biases travel with the first operands
    // (fragment id = FC f + g: rows m0 + 16 f + er, columns n0 + 16 g + 4 eq + i: four neighbouring lanes finish 16 columns of a row)
    const int er = lane >> 2, eq = lane & 3;
    float cs4[E][4], bi4[E][4];
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int nn = n0 + 16 * ((wave + NW * e) % FC) + 4 * eq + i;   // < Npad
            cs4[e][i] = p.cs[nn];
            bi4[e][i] = p.cs[p.Npad + nn];
        }
    // ... and so does the consumer's position of the lane's four columns (flexiq_out.lower_for): those of its FP6 prefix leave
    // clamped in q and as FP6 codes in its activation buffer, its other 4-bit channels clamped and masked in q
    int sn_e[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int nn0 = n0 + 16 * ((wave + NW * e) % FC) + 4 * eq;
        const bool to6 = FP6 && p.nx6 != nullptr && nn0 < p.next_K6;
        sn_e[e] = p.next_ashift != nullptr && (to6 || nn0 < p.next_K4) ? p.next_ashift[nn0 >> p.next_gs_log2] : 4;
    }

    v4i acc[FR][FC];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int g = 0; g < FC; ++g) acc[f][g] = (v4i){0, 0, 0, 0};

    int first = wave;
    if constexpr (FP6) {
        const int chunks = (p.s6 + 1) >> 1, S = p.C >> 6;
        v4f accf[FR][FC];
#pragma unroll
        for (int f = 0; f < FR; ++f)
#pragma unroll
            for (int g = 0; g < FC; ++g) accf[f][g] = (v4f){0.f, 0.f, 0.f, 0.f};
        constexpr int U6 = UN >= 4 ? 2 : 1;   // chunks in flight
        for (int c0 = wave; c0 < chunks; c0 += NW * U6) {
            v4i wlo[U6][FC], xlo[U6][FR];
            v2i whi[U6][FC], xhi[U6][FR];
            int wsc[U6][FC], asc[U6];
#pragma unroll
            for (int k = 0; k < U6; ++k) {
                const int ks = 2 * (c0 + k * NW) + (qd >> 1), h = qd & 1;   // this lane's K-step and unit
                const bool ok = ks < p.s6;
                asc[k] = ok ? 130 + p.ashift[(2 * ks + h) >> p.gs_shift] : 127;   // 2^(position + 3): the codes are k / 8
#pragma unroll
                for (int g = 0; g < FC; ++g) {
                    const int n = n0 + 16 * g + c;
                    wlo[k][g] = (v4i){0, 0, 0, 0};
                    whi[k][g] = (v2i){0, 0};
                    wsc[k][g] = 127;
                    if (ok) {
                        wlo[k][g] = *reinterpret_cast<const v4i *>(p.W6 + (((int64_t)ks * 3 + h) * p.Npad + n) * 16);
                        whi[k][g] = *reinterpret_cast<const v2i *>(p.W6 + (((int64_t)ks * 3 + 2) * p.Npad + n) * 16 + 8 * (h ^ ((n >> 4) & 1)));
                        wsc[k][g] = p.W6S[((int64_t)(ks >> 2) * p.Npad + n) * 8 + 4 * h + (ks & 3)];
                    }
                }
#pragma unroll
                for (int f = 0; f < FR; ++f) {
                    const int m = m0 + 16 * f + c, blk = m >> 6, r = m & 63;
                    xlo[k][f] = (v4i){0, 0, 0, 0};
                    xhi[k][f] = (v2i){0, 0};
                    if (ok && m < p.M) {
                        xlo[k][f] = *reinterpret_cast<const v4i *>(p.X6 + ((((int64_t)blk * S + ks) * 3 + h) * 64 + r) * 16);
                        xhi[k][f] = *reinterpret_cast<const v2i *>(p.X6 + ((((int64_t)blk * S + ks) * 3 + 2) * 64 + r) * 16 + 8 * (h ^ ((r >> 4) & 1)));
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < U6; ++k)
#pragma unroll
                for (int f = 0; f < FR; ++f)
#pragma unroll
                    for (int g = 0; g < FC; ++g)
                        accf[f][g] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                            (v8i){wlo[k][g].x, wlo[k][g].y, wlo[k][g].z, wlo[k][g].w, whi[k][g].x, whi[k][g].y, 0, 0},
                            (v8i){xlo[k][f].x, xlo[k][f].y, xlo[k][f].z, xlo[k][f].w, xhi[k][f].x, xhi[k][f].y, 0, 0}, accf[f][g], 2, 2, 0,
                            wsc[k][g], 0, asc[k]);
        }
#pragma unroll
        for (int f = 0; f < FR; ++f)
#pragma unroll
            for (int g = 0; g < FC; ++g)
                acc[f][g] = (v4i){(int)accf[f][g].x, (int)accf[f][g].y, (int)accf[f][g].z, (int)accf[f][g].w};   // exact integers below 2^24
        first = p.s6 + (wave + NW - chunks % NW) % NW;   // the int8 K-steps continue the deal
    }
    // ---- the int8 K-steps first, first + NW, ...: UN of them in flight per wave, each slot loaded again as soon as it is used up
    if (first < p.steps) {
        unsigned char *const mine = lds + wave * kStage * 1024;
        const int rows = min(p.M - m0, kTileRows);
        // (rows beyond M and channels beyond the last row read as zero; the pad unit of an odd unit count has zero weights)
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)(p.X + (int64_t)m0 * p.C), 0, rows * p.C, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W8, 0, 2 * p.w4x_delta, kRsrcFlags);
        const int xr = lane >> 2, xp = lane & 3;   // row of a fragment and 16-byte piece of the K-step that this lane loads
        const int xoff = xr * p.C + 16 * xp;
        unsigned char *const put = mine + xr * 64 + 16 * (xp ^ (xr >> 2));
        const unsigned char *const get = mine + c * 64 + 16 * (qd ^ (c >> 2));
        const int woff = (qd * p.Npad + n0 + c) * 16;
        v4i w8[UN][FC], x[UN][FR];
        int sa0[UN], sa1[UN];
        auto load = [&](int k, int ks) {
            if constexpr (!FP6) {   // (scalar, and ahead of its use: a vector load would wait for all of the operands in flight; the table has an entry for the pad unit)
                sa0[k] = p.ashift[2 * ks >> p.gs_shift];
                sa1[k] = p.ashift[(2 * ks + 1) >> p.gs_shift];
            }
            const int wo = woff + (2 * ks + (qd >> 1) < p.units4 ? p.w4x_delta : 0);
#pragma unroll
            for (int f = 0; f < FR; ++f) x[k][f] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, xoff + 16 * f * p.C + 64 * ks, 0, 0));
#pragma unroll
            for (int g = 0; g < FC; ++g) w8[k][g] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, wo + 256 * g, ks * 64 * p.Npad, 0));
        };
        auto multiply = [&](int k, const v4i (&v)[FR]) {
#pragma unroll
            for (int f = 0; f < FR; ++f) *reinterpret_cast<v4i *>(put + 1024 * f) = v[f];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            v4i b[FR];
#pragma unroll
            for (int f = 0; f < FR; ++f) b[f] = *reinterpret_cast<const v4i *>(get + 1024 * f);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int f = 0; f < FR; ++f)
#pragma unroll
                for (int g = 0; g < FC; ++g) acc[f][g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w8[k][g], b[f], acc[f][g], 0, 0, 0);
        };
        auto use = [&](int k, int ks) {
            if (!FP6 && !p.x_pre && 2 * ks < p.units4) {   // (lowered before it crosses the lanes: fewer registers live)
                const Lowering lower(xp >> 1 ? sa1[k] : sa0[k], 2 * ks + (xp >> 1) < p.units4);   // (... or a unit read at 8 bits)
#pragma unroll
                for (int f = 0; f < FR; ++f)
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[k][f][i] = (int)lower((uint32_t)x[k][f][i]);
            }
            multiply(k, x[k]);
        };
        auto count = [&](int first, int end) { return first < end ? (end - first + NW - 1) / NW : 0; };
        if constexpr (XP) {
            // the K-steps of packed codes first, 8 bytes per lane and fragment
            const int s4 = p.pieces_p >> 2;
            const __amdgpu_buffer_rsrc_t rx4 = __builtin_amdgcn_make_buffer_rsrc((void *)(p.X4 + (int64_t)m0 * (p.C >> 1)), 0, rows * (p.C >> 1), kRsrcFlags);
            v2i x4[UN][FR];
            auto load4 = [&](int k, int ks) {
                sa0[k] = p.ashift[2 * ks >> p.gs_shift];
                sa1[k] = p.ashift[(2 * ks + 1) >> p.gs_shift];
#pragma unroll
                for (int f = 0; f < FR; ++f) x4[k][f] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rx4, (xoff >> 1) + 8 * f * p.C + 32 * ks, 0, 0));
#pragma unroll
                for (int g = 0; g < FC; ++g) w8[k][g] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, woff + p.w4x_delta + 256 * g, ks * 64 * p.Npad, 0));
            };
            auto use4 = [&](int k, int) {
                const int sa = xp >> 1 ? sa1[k] : sa0[k];
                v4i e[FR];
#pragma unroll
                for (int f = 0; f < FR; ++f) {
                    const uint32_t lo = (uint32_t)x4[k][f].x, hi = (uint32_t)x4[k][f].y;
                    e[f] = (v4i){(int)expand4(lo << 4, sa), (int)expand4(lo, sa), (int)expand4(hi << 4, sa), (int)expand4(hi, sa)};
                }
                multiply(k, e);
            };
            wave_steps<UN, false, false>(load4, use4, wave, count(wave, s4), NW);
            first = s4 + (wave + NW - s4 % NW) % NW;   // (the deal goes on with the other K-steps)
        }
        wave_steps<UN, false, false>(load, use, first, count(first, p.steps), NW);
    }

    // ---- the waves' sums meet in LDS; wave w adds up and finishes fragments w, w + NW, ...
    const int slot = 16 * qd + (c ^ (4 * qd));   // (the quads of a row are read by four neighbouring lanes below: no bank twice in either pattern)
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int g = 0; g < FC; ++g) red[(wave * NF + FC * f + g) * 64 + slot] = acc[f][g];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int id = wave + NW * e, f = id / FC, g = id % FC;
        if (id >= NF) break;
        v4i s = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < kTileWaves; ++w) s += red[(w * NF + id) * 64 + 16 * eq + (er ^ (4 * eq))];
        const int m = m0 + 16 * f + er, nn0 = n0 + 16 * g + 4 * eq;
        if (m >= p.M || nn0 >= p.N) continue;
        const int64_t o = (int64_t)m * p.N + nn0;
        float yv[4];
        uint32_t qw = 0;
        const bool to6 = FP6 && p.nx6 != nullptr && nn0 < p.next_K6;
        const bool lower = p.next_ashift != nullptr && !to6 && nn0 < p.next_K4;
        const int sn = sn_e[e];
        const float lo = 128.0f - (float)(8 << sn), hi = 127.0f + (float)(8 << sn);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            yv[i] = __builtin_fmaf((float)s[i], cs4[e][i], bi4[e][i]);
            qw = __builtin_amdgcn_cvt_pk_u8_f32(
                __builtin_amdgcn_fmed3f(__builtin_fmaf((float)s[i], cs4[e][i] * p.r_out, bi4[e][i] * p.r_out + 128.0f), lo, hi), i, qw);
        }
        if (to6) {
            // four codes (offset form u = code + 128, clamped above): floor(code / 2^sn) + 8 = (u >> sn) - ((128 >> sn) - 8), 0 .. 15 per
            // byte; E2M3 pattern of L / 8: sign << 5 | |L|.  Element 16 a + 4 b + i of a unit is its channel 8 b + 4 a + i (the order of the
            // packed FP6 weights), so the 24 bits are bytes 3 j .. 3 j + 2 of the unit's 24 with j = 4 a + b:
            // the first 16 bytes of a unit lie in plane (unit % 2) of the consumer's K-step, the last 8 in plane 2
            const uint32_t cb = ((qw >> sn) & (0x01010101u * (0xFFu >> sn))) - 0x01010101u * (uint32_t)((128 >> sn) - 8);
            const uint32_t neg = (~cb >> 3) & 0x01010101u;
            const uint32_t mag = ((cb & 0x07070707u) ^ (neg * 7u)) + neg;
            const uint32_t c6 = mag | (neg << 5);
            const uint32_t w24 = (c6 & 0x3Fu) | ((c6 >> 2) & 0xFC0u) | ((c6 >> 4) & 0x3F000u) | ((c6 >> 6) & 0xFC0000u);
            const int u = nn0 >> 5, hh = u & 1, rr = m & 63, j = 4 * ((nn0 >> 2) & 1) + ((nn0 & 31) >> 3);
            uint8_t *const blk = p.nx6 + ((int64_t)(m >> 6) * p.next_S + (u >> 1)) * 3072;
            // (one 2-byte and one 1-byte store: the even one of 3 j and 3 j + 1 starts the pair, which never straddles bytes 15 | 16)
            auto at = [&](int byte) { return byte < 16 ? blk + hh * 1024 + rr * 16 + byte : blk + 2048 + rr * 16 + 8 * (hh ^ ((rr >> 4) & 1)) + byte - 16; };
            if (j & 1) {
                *at(3 * j) = (uint8_t)w24;
                *reinterpret_cast<uint16_t *>(at(3 * j + 1)) = (uint16_t)(w24 >> 8);
            } else {
                *reinterpret_cast<uint16_t *>(at(3 * j)) = (uint16_t)w24;
                *at(3 * j + 2) = (uint8_t)(w24 >> 16);
            }
        }
        qw ^= 0x80808080u;
        if (lower) qw &= 0x01010101u * ((0xFFu << sn) & 0xFFu);
        const bool to4 = !FP6 && p.nx4 != nullptr && nn0 < p.next_K4P;
        if (to4) {
            // channels 8 e .. 8 e + 3 of the consumer lie in the low halves of a dword's bytes, 8 e + 4 .. 8 e + 7, the neighbouring lane's, in the high ones
            const uint32_t codes = (qw >> sn) & 0x0F0F0F0Fu, next = (uint32_t)__shfl_xor((int)codes, 1);
            if (!(eq & 1)) *reinterpret_cast<uint32_t *>(p.nx4 + (int64_t)m * (p.N >> 1) + (nn0 >> 1)) = codes | (next << 4);
        }
        if ((p.N & 3) == 0) {
            if (p.acc) *reinterpret_cast<v4i *>(p.acc + o) = s;
            if (p.y) *reinterpret_cast<float4 *>(p.y + o) = make_float4(yv[0], yv[1], yv[2], yv[3]);
            if (p.q && !to4) *reinterpret_cast<uint32_t *>(p.q + o) = qw;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (nn0 + i >= p.N) continue;
                if (p.acc) p.acc[o + i] = s[i];
                if (p.y) p.y[o + i] = yv[i];
                if (p.q) p.q[o + i] = (int8_t)(qw >> (8 * i));
            }
        }
    }
}

static int g_force_tile_splitk = -1;   // test hook: 1 = take k_tile_splitk whenever the call qualifies, 0 = never, -1 = automatic
static int g_last_tile_splitk = 0;
static bool g_tile_splitk_ready[64] = {};
// up to here the few-row kernels measure faster (r = 0 / 1, us there and on a tile per block: 4096 -> 1024 channels, 32 rows 4.4 / 5.9 and 4.9 / 6.3, 33 rows 5.2 / 7.0 and 4.95 / 6.4; 3072 ->
// 768, 32 rows 4.2 / 5.1 and 4.5 / 5.5, 33 rows 4.8 / 6.1 and 4.55 / 5.6)
constexpr int kTileMinRows = 32;

static int g_force_cg = 0;      // test hook: column groups per block of k_few_rows_dot (0 = automatic)
static int g_force_rows = -1;   // test hook: 1 / 2 = take k_few_rows / k_few_rows_dot whenever the call qualifies (3: k_few_rows with packed weight codes), 0 = never, -1 = automatic
static int g_last_rows = 0;
static bool g_last_codes = false;   // ... and whether that was a build that reads packed weight codes

}  // namespace smallm

bool few_rows_last_packed() { return smallm::g_last_codes; }
bool few_rows_forced() { return smallm::g_force_rows >= 0 || smallm::g_force_tile_splitk >= 0; }

// Launches k_few_rows (*taken = 1) or k_few_rows_dot (*taken = 2) for a linear call with at most 64 rows; *taken = 0: the call
// was left to the other kernels.
int launch_few_rows(const flexiq_layer *L, const int8_t *X, int64_t M, const flexiq_out *out, void *stream, int num_cu, int *taken,
                    const uint8_t *X4, const LowerArgs *lower)
{
    using namespace smallm;
    *taken = 0;
    g_last_rows = 0;
    g_last_codes = false;
    if (g_force_rows == 0 || M < 1 || M > 64) return FLEXIQ_OK;
    if (out->scan_for || out->x4 || out->x6) return FLEXIQ_OK;
    if (out->lower_for && !lower) return FLEXIQ_OK;   // (the caller has checked the consumer; null positions: nothing to lower)
    if ((reinterpret_cast<uintptr_t>(X) & 15u) || (L->C & 15)) return FLEXIQ_OK;   // 16-byte activation pieces
    // Every block reads all activation rows: with more than 16 rows that traffic (blocks x M x C bytes through the compute
    // units' 64 B/clk path) decides, and beyond about one block per compute unit the kernels with taller tiles win (r = 0 / 1, us here and in the kernel taken,
    // kept in cache: 16384 x 4096 weights, 17 rows 14.0 / 16.8 and 13.5 / 13.4, 32 rows 16.0 / 18.4 and 13.9 / 13.9, 64 rows 25.3 / 29.0 and 14.1 / 15.0; 8192 x 2048, 17 rows
    // 5.2 / 6.8 and 5.3 / 6.0, 32 rows 5.25 / 7.0 and 5.3 / 6.0).
    if (g_force_rows < 0 && M > 16 && (L->N + kRowCols - 1) / kRowCols > num_cu) return FLEXIQ_OK;
    RowsParams p = {};
    p.X = X; p.W8 = L->d_w8; p.W4 = L->d_w4; p.wshift = L->d_wshift;
    p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift;
    p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad; p.C = L->C;
    p.units = L->C / kUnit;
    p.units4 = L->max_4bit_ch / kUnit;
    p.x_pre = L->x_prelowered ? 1 : 0;
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.steps = (p.units + 1) / 2;
    p.w4x_delta = L->U * 32 * L->Npad;
    if (lower && lower->ashift) { p.next_ashift = lower->ashift; p.next_K4 = lower->K4; p.next_gs_log2 = lower->gs_log2; }
    // packed activation codes of the leading whole K-steps of 4-bit channels (the caller has checked alignment): the dot-product
    // kernel takes them as they are; the matrix-core kernel has no use for them and leaves such a call to the tiled kernel (from 17 rows on
    // k_tile_splitk has been asked before)
    p.X4 = X4 && !L->x_prelowered ? X4 : nullptr;
    p.pieces_p = p.X4 ? (L->max_4bit_ch / 64) * 4 : 0;
    // One or two rows: the dot-product kernel.  Three or four rows: where the layer has columns enough for four column groups per
    // block and at least half of the channels run at 4 bits (us here and on the matrix-core kernel with expanded weights, r = 0.5 / 1, from HBM: 16384 x 4096 weights, three rows
    // 14.8 / 11.9 and 15.6 / 15.8, four 15.6 / 12.9 and 16.1 / 16.2; 8192 x 8192, four rows 16.3 / 15.1 and 15.4 / 16.8; from six rows on it is bound by its vector-ALU work, 22
    // us; at ViT-L sizes the matrix-core kernel is ahead from three rows on).  The line is older than the loads of whole rows there: with packed weight codes that
    // kernel takes 13.9 / 12.6 us on the first of them, and on layers of short rows it is ahead, 16384 x 1024, four rows, 6.3 / 6.4 against 7.7 / 7.0.
    const int ncg = (L->N + kVecCols - 1) / kVecCols;
    const bool wide = ncg >= 4 * num_cu && (ncg + 3) / 4 * 4 * kVecCols <= L->Npad;
    if (g_force_rows == 2 || (g_force_rows < 0 && (M <= 2 || (M <= 4 && wide && 2 * L->max_4bit_ch >= L->C)))) {
        const int groups = (2 * p.units + 7) / 8;
        const int nw = groups >= 32 ? 8 : 4;   // (eight waves for shorter reductions measured slower: 3.6 against 3.4 us on 4096 x 1024)
        // column groups per block: four where the layer still gives every compute unit several blocks (measured on 16384 x 4096
        // and 8192 x 8192 weights, one row, r = 0 / 1: 12.0 / 7.9 us and 12.0 / 9.3 us against 12.1 / 14.4 and 12.9 / 13.1 us with one
        // group; ViT-L sizes are faster with one); the last block's columns must stay inside the padded weight tiles
        int cg = g_force_cg > 0 ? g_force_cg : (wide ? 4 : 1);
        if (((ncg + cg - 1) / cg) * cg * kVecCols > L->Npad) cg = 1;
        const size_t lds = (size_t)nw * M * kVecCols * cg * 4 + (size_t)M * 16 * p.units4 + (size_t)M * L->C;
        if (M <= 4 && lds <= 64 * 1024) {
            void (*fn)(const RowsParams) = nullptr;
            switch ((int)M) {
            case 1: fn = cg == 4 ? k_few_rows_dot<1, 4> : k_few_rows_dot<1, 1>; break;
            case 2: fn = cg == 4 ? k_few_rows_dot<2, 4> : k_few_rows_dot<2, 1>; break;
            case 3: fn = cg == 4 ? k_few_rows_dot<3, 4> : k_few_rows_dot<3, 1>; break;
            default: fn = cg == 4 ? k_few_rows_dot<4, 4> : k_few_rows_dot<4, 1>; break;
            }
            FLEXIQ_HIP(launch_kernel(fn, dim3((unsigned)((ncg + cg - 1) / cg)), dim3(64 * nw), lds, stream, p));
            *taken = 2;
            g_last_rows = 2;
            return FLEXIQ_OK;
        }
        if (g_force_rows == 2) return FLEXIQ_OK;
    }
    if (X4) return FLEXIQ_OK;
    const int mf = (int)((M + 15) / 16);
    const unsigned blocks = (unsigned)((L->N + kRowCols - 1) / kRowCols);
    // waves per block: as many as there are K-steps to split while the layer gives a compute unit a block or so (the call is one
    // trip to memory: widest wins); with several blocks per compute unit four waves that each stream batch after batch, so that
    // one block's meeting in LDS and epilogue hide behind the others' loads (16384 x 4096 weights, 8 rows: 13.4 against 17.2 us)
    const int nw = (int)blocks >= 2 * num_cu ? 4 : (p.steps >= 12 ? 16 : (p.steps >= 6 ? 8 : 4));
    size_t lds = (size_t)nw * mf * 64 * 16;
    // Packed codes where the weight bytes decide: up to eight rows from 40 MiB of 8-bit weights on, more from above 41 MiB and half of the channels
    // at 4 bits on.  The expanded copies and the codes, us, r = 0.5 / 1, from HBM and (kept in cache): 8192 x 5120 (40 MiB), 8 rows 12.5 / 13.9 (11.1 / 12.5) and
    // 12.6 / 10.5 (9.8 / 8.8), 12 rows 11.6 / 12.1 (9.9 / 10.6) and 12.75 / 10.4 (9.85 / 8.7); 11008 x 4096 (43 MiB), 12 rows 12.65 / 13.4 (10.1 / 10.9) and 11.4 / 10.0 (9.5 / 9.4);
    // 8192 x 4096 (32 MiB), 8 rows 10.6 / 11.7 (7.4 / 8.6) and 10.1 / 8.95 (7.2 / 7.7), 5 rows 10.2 / 10.6 (6.9 / 7.4) and 10.3 / 9.0 (7.2 / 7.7); 4096 x 4096, 8 rows 6.7 / 6.9 (4.5 / 4.8) and
    // 6.15 / 5.5 (5.0 / 5.15).
    p.s4 = p.units4 / 2;
    const bool p4 = mf == 1 && L->group_size == 64 && p.s4 > 0 && (g_force_rows == 3 || (g_force_rows < 0 && (M <= 8 ? (int64_t)L->N * L->C >= (40 << 20)
                                                                                                                     : (int64_t)L->N * L->C > (41 << 20) && 2 * L->max_4bit_ch >= L->C)));
    // few rows whose 4-bit channels the kernel lowers: once per block, through LDS (4096 x 4096, 4 rows, r = 0.5 / 1: 3.85 / 4.0 us, by every wave 4.25 / 4.8; the
    // packed codes leave every wave the time: 16384 x 4096, 8 rows 12.65 / 13.2 with a block's pass and 11.45 / 11.65 without)
    const size_t rows_bytes = (size_t)M * (32 * (size_t)p.units4 + 16);
    const bool coop = !p4 && M <= 8 && !p.x_pre && p.units4 > 0 && lds + rows_bytes <= 64 * 1024;
    if (coop) lds += rows_bytes;
    void (*fn)(const RowsParams) =
        mf == 1 ? (p4 ? k_few_rows<1, false, false, true> : (coop ? k_few_rows<1, true> : k_few_rows<1, false>))
                : (mf == 2 ? k_few_rows<2, false> : (mf == 3 ? k_few_rows<3, false> : k_few_rows<4, false>));
    FLEXIQ_HIP(launch_kernel(fn, dim3(blocks), dim3(64 * nw), lds, stream, p));
    *taken = 1;
    g_last_rows = 1;
    g_last_codes = p4;
    return FLEXIQ_OK;
}

// The FP6 variant of a linear call with at most 64 rows (flexiq_mixed_gemm_fp6): k_few_rows with the leading K6 channels on the
// FP6 matrix path; *taken = 0: the call was left to the tiled FP6 kernel.
int launch_few_rows_fp6(const flexiq_layer *L, const int8_t *X, const uint8_t *X6, int64_t M, const flexiq_out *out, void *stream, int K6,
                        int num_cu, int *taken)
{
    using namespace smallm;
    *taken = 0;
    if (g_force_rows == 0 || M < 1 || M > 64) return FLEXIQ_OK;
    if (out->lower_for || out->scan_for || out->x4 || out->x6) return FLEXIQ_OK;
    if (g_force_rows < 0 && M > 16 && (L->N + kRowCols - 1) / kRowCols > num_cu) return FLEXIQ_OK;   // (as in launch_few_rows)
    RowsParams p = {};
    p.X = X; p.W8 = L->d_w8; p.X6 = X6; p.W6 = L->d_w6; p.W6S = L->d_w6s;
    p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift;
    p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad; p.C = L->C;
    p.units = L->C / kUnit;
    p.units4 = L->max_4bit_ch / kUnit;
    p.x_pre = 1;   // the 4-bit channels beyond the FP6 ones arrive lowered
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.steps = (p.units + 1) / 2;
    p.w4x_delta = L->U * 32 * L->Npad;
    p.s6 = K6 / 64;
    const int mf = (int)((M + 15) / 16);
    const unsigned blocks = (unsigned)((L->N + kRowCols - 1) / kRowCols);
    const int items = (p.s6 + 1) / 2 + (p.steps - p.s6);   // FP6 chunks and int8 K-steps to deal out
    const int nw = (int)blocks >= 2 * num_cu ? 4 : (items >= 12 ? 16 : (items >= 6 ? 8 : 4));
    const size_t lds = (size_t)nw * mf * 64 * 16;
    void (*fn)(const RowsParams) = mf == 1 ? k_few_rows<1, false, true> : (mf == 2 ? k_few_rows<2, false, true> : (mf == 3 ? k_few_rows<3, false, true> : k_few_rows<4, false, true>));
    FLEXIQ_HIP(launch_kernel(fn, dim3(blocks), dim3(64 * nw), lds, stream, p));
    *taken = 1;
    g_last_rows = 3;
    g_last_codes = false;
    return FLEXIQ_OK;
}

// Once per device, when the first layer is packed on it: the dynamic-LDS limit of every build of k_tile_splitk, so that a
// launch is only a launch (and safe under stream capture).
int prepare_tile_splitk_kernels(int device)
{
    using namespace smallm;
    if (device < 0 || device >= 64) return FLEXIQ_EINVAL;
    if (g_tile_splitk_ready[device]) return FLEXIQ_OK;
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<4, 4, 8, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<2, 4, 16, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<2, 2, 16, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<4, 4, 8, 2, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<2, 4, 8, 4, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<2, 2, 16, 4, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<4, 4, 8, 2, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<2, 4, 16, 2, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
    FLEXIQ_HIP(hipFuncSetAttribute((const void *)k_tile_splitk<2, 2, 16, 4, false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    g_tile_splitk_ready[device] = true;
    return FLEXIQ_OK;
}

static int launch_tile_any(const flexiq_layer *L, const int8_t *X, const uint8_t *X6, int K6, const uint8_t *X4, int64_t M, const flexiq_out *out,
                           void *stream, int num_cu, int *taken, const LowerArgs *lower)
{
    using namespace smallm;
    *taken = 0;
    g_last_tile_splitk = 0;
    // FP6 calls that lower for a consumer have no few-row kernel to go to: this one takes them at any row count
    const bool only_here = (X6 && out->lower_for) || (out->x4 && !X4);
    // Calls that read or write packed codes have the tiled kernel alone else, whose few blocks each walk the reduction with a barrier per K-step: they
    // come here from 17 rows on, producers at any row count, and with shorter reductions.  us there and here, r = 0.5 / 1, reading: 100 x 384 -> 1536 5.8 / 6.2
    // and 4.0 / 4.0; 20 x 832 -> 576 8.45 / 7.7 and 4.1 / 4.1; 200 x 3072 -> 768 14.9 / 16.8 and 5.5 / 5.8; 200 x 2880 -> 2784 15.7 / 16.2 and 8.6 / 8.9; writing: 6 x 768 ->
    // 3072 7.1 / 7.8 and 4.0 / 4.15, 1000 x 1024 -> 1024 8.4 / 9.1 and 6.4 / 7.0.  Beyond one tile per compute unit it is behind: 1000 x 768 -> 3072 10.2 there, 11.7 here.  (Readers of 3 to 16 rows stay in the
    // tiled kernel: not measured here.)
    const bool packed = X4 || out->x4;
    if (g_force_tile_splitk == 0 || M < 1 || (M <= 16 && !only_here) || M > 0x7fffffff / 2) return FLEXIQ_OK;
    // (calls of at most 64 rows: the few-row hook, in any forced state, keeps this kernel out of its comparisons)
    if (M <= 64 && (g_force_rows >= 0 || (g_force_tile_splitk < 0 && M <= kTileMinRows && !only_here && !packed))) return FLEXIQ_OK;
    if (out->scan_for || (out->lower_for && !lower) || (out->x4 && !(lower && lower->x4 == out->x4 && (L->N & 31) == 0))) return FLEXIQ_OK;
    if (out->x6 && !(X6 && lower && lower->x6 == out->x6 && (L->N & 63) == 0 && (lower->K6 & 63) == 0)) return FLEXIQ_OK;   // FP6 output: FP6 calls only
    if ((reinterpret_cast<uintptr_t>(X) & 15u) || (L->C & 15) || L->device < 0 || L->device >= 64) return FLEXIQ_OK;
    const int steps = (L->C / kUnit + 1) / 2;
    auto tiles_of = [&](int tr, int tc) { return ((M + tr - 1) / tr) * (int64_t)((L->N + tc - 1) / tc); };
    // Where it measures faster than the tiled kernel: at most about one 64 x 64 tile per compute unit and a reduction of at
    // least 12 K-steps for the waves to split.  The tile shrinks while the blocks would leave half the compute units idle.
    if (g_force_tile_splitk < 0 && (tiles_of(64, 64) > (int64_t)num_cu || steps < (packed ? 6 : 12))) return FLEXIQ_OK;
    int shape = g_force_tile_splitk >= 2 ? g_force_tile_splitk - 2 : tiles_of(64, 64) * 2 > num_cu ? 0 : tiles_of(32, 64) * 2 > num_cu ? 1 : 2;
    if (shape > 2) return FLEXIQ_EINVAL;
    const int tr = shape == 0 ? 64 : 32, tc = shape == 2 ? 32 : 64;
    if (tiles_of(tr, tc) > 0x7fffffff || (M + tr - 1) / tr > 65535) return FLEXIQ_OK;
    const size_t lds = shape == 2 ? 64 * 1024 : 128 * 1024;   // waves x fragments x 1 KB
    if (!g_tile_splitk_ready[L->device]) return FLEXIQ_OK;   // (set up when the first layer is packed on the device)
    RowsParams p = {};
    p.X = X; p.W8 = L->d_w8;
    p.ashift = L->dynamic ? L->d_ashift_dyn : L->d_ashift;
    p.cs = L->d_cs;
    p.acc = out->acc; p.y = out->y; p.q = out->q;
    p.r_out = out->q ? 1.0f / out->out_scale : 1.0f;
    p.M = (int)M; p.N = L->N; p.Npad = L->Npad; p.C = L->C;
    p.units = L->C / kUnit;
    p.units4 = L->max_4bit_ch / kUnit;
    p.x_pre = L->x_prelowered || X6 ? 1 : 0;   // (FP6 calls: the 4-bit channels beyond the FP6 ones arrive lowered)
    p.gs_shift = L->group_size == 64 ? 1 : 0;
    p.steps = steps;
    p.w4x_delta = L->U * 32 * L->Npad;
    if (lower && lower->ashift) {
        p.next_ashift = lower->ashift; p.next_K4 = lower->K4; p.next_gs_log2 = lower->gs_log2;
        if (out->x4) { p.nx4 = lower->x4; p.next_K4P = lower->K4P; }
        if (X6 && lower->x6) { p.nx6 = lower->x6; p.next_K6 = lower->K6; p.next_S = lower->S; }
    }
    const dim3 grid((unsigned)((L->N + tc - 1) / tc), (unsigned)((M + tr - 1) / tr));
    hipError_t err;
    if (X6) {
        p.X6 = X6; p.W6 = L->d_w6; p.W6S = L->d_w6s;
        p.s6 = K6 / 64;
        if (shape == 0) err = launch_kernel(k_tile_splitk<4, 4, 8, 2, true>, grid, dim3(512), lds, stream, p);
        else if (shape == 1) err = launch_kernel(k_tile_splitk<2, 4, 8, 4, true>, grid, dim3(512), lds / 2, stream, p);   // (eight waves: registers)
        // (one row fragment where the call has no more; the second is a load, a way through LDS and two multiplications of nothing in every step of the chain.  r = 0.25 / 0.5 / 1,
        // two fragments and one: 2 x 4992 -> 3904 5.75 / 5.7 / 5.5 and 5.0 / 5.25 / 5.4 us, 8 x 1088 -> 64 3.2 / 3.25 / 3.4 and 2.95 / 3.0 / 3.2)
        else if (M <= 16) err = launch_kernel(k_tile_splitk<1, 2, 16, 4, true>, grid, dim3(1024), lds / 2, stream, p);
        else err = launch_kernel(k_tile_splitk<2, 2, 16, 4, true>, grid, dim3(1024), lds, stream, p);
    } else if (X4) {
        p.X4 = X4;
        p.pieces_p = (L->max_4bit_ch / 64) * 4;
        if (shape == 0) err = launch_kernel(k_tile_splitk<4, 4, 8, 2, false, true>, grid, dim3(512), lds, stream, p);
        else if (shape == 1) err = launch_kernel(k_tile_splitk<2, 4, 16, 2, false, true>, grid, dim3(1024), lds, stream, p);
        else err = launch_kernel(k_tile_splitk<2, 2, 16, 4, false, true>, grid, dim3(1024), lds, stream, p);
    } else if (shape == 0) err = launch_kernel(k_tile_splitk<4, 4, 8, 2>, grid, dim3(512), lds, stream, p);
    else if (shape == 1) err = launch_kernel(k_tile_splitk<2, 4, 16, 2>, grid, dim3(1024), lds, stream, p);
    else err = launch_kernel(k_tile_splitk<2, 2, 16, 4>, grid, dim3(1024), lds, stream, p);
    FLEXIQ_HIP(err);
    *taken = 1 + shape;
    g_last_tile_splitk = 1 + shape;
    g_last_rows = 0;
    return FLEXIQ_OK;
}

// Launches k_tile_splitk for a linear call of more than 32 rows (packed codes: fewer) whose output tiles leave most compute units idle on a long
// reduction; *taken = 0: the call was left to the other kernels, else 1 / 2 / 3: tiles of 64 x 64 / 32 x 64 / 32 x 32.
int launch_tile_splitk(const flexiq_layer *L, const int8_t *X, int64_t M, const flexiq_out *out, void *stream, int num_cu, int *taken,
                       const LowerArgs *lower, const uint8_t *X4)
{
    return launch_tile_any(L, X, nullptr, 0, X4, M, out, stream, num_cu, taken, lower);
}

// The same for the FP6 variant of the 4-bit phase: X holds the lowered activations, X6 the FP6 codes of the leading K6 channels.
int launch_tile_splitk_fp6(const flexiq_layer *L, const int8_t *X, const uint8_t *X6, int64_t M, const flexiq_out *out, void *stream, int K6,
                           int num_cu, int *taken, const LowerArgs *lower)
{
    *taken = 0;
    if (!X6 || K6 < 0 || (K6 & 63)) return FLEXIQ_OK;
    return launch_tile_any(L, X, X6, K6, nullptr, M, out, stream, num_cu, taken, lower);
}

}  // namespace flexiq

extern "C" int flexiq_debug_force_few_rows(int mode)
{
    // (mode 14: the dot-product kernel with 4 column groups per block where rows and padding allow)
    if (mode == 14) {
        flexiq::smallm::g_force_cg = 4;
        mode = 2;
    } else {
        flexiq::smallm::g_force_cg = 0;
    }
    if (mode < -1 || mode > 3) return FLEXIQ_EINVAL;
    flexiq::smallm::g_force_rows = mode;
    return flexiq::smallm::g_last_rows;
}

extern "C" int flexiq_debug_force_tile_splitk(int mode)
{
    if (mode < -1 || mode > 4) return FLEXIQ_EINVAL;
    flexiq::smallm::g_force_tile_splitk = mode;
    return flexiq::smallm::g_last_tile_splitk;
}
