// Matmul for a few rows (2 <= n <= 64: batched decode, short prompts) as ONE barrier-free stream over the weights:
//   out[i,r] = epilogue(sum_c x[i,c] * W(r,c)),  W packed 4-bit (groups of 32, 64 or 128), native 3-bit or plain fp16.
//
// With a few rows the contraction is bound by the one pass over the weights, and what a kernel loses is everything that is
// not that stream: row tiles that do not divide over the CUs, staging of x behind barriers, partial tiles and finishing
// launches.  Mapping for gfx950:
//   - One workgroup of eight wavefronts per CU (two per SIMD, up to 256 registers).  A wavefront owns a SLICE OF THE
//     COLUMNS (UW units of 256, fp16: 128) for good: its share of x sits in registers as ready MFMA operands, read once, and it
//     streams its slice of row tile after row tile (16 weight rows) of the workgroup's range.  Nothing is shared inside the loop:
//     no LDS staging, no barrier, the only memory operations in flight are weights and scales.
//   - Little in flight: one row tile (8 KB per CU and unit, 16 in two tiles of one unit; fp16 16 KB per unit, half a tile from six units on).  A bare read of 235 MB in this pattern takes 39.4 us with 64 KB per CU and 42.5
//     with 128 (lines of 128, 256 or 512 bytes per row and load: the same; neighbouring tiles dealt out over the CUs: slower), and the
//     kernels gain more than that (us, two or three tiles / one: 4 bits, 16 rows 22016 x 4096 18.2 / 16.5, 57344 x 8192 60.5 / 56.6, 8192 x
//     28672 39.7 / 35.3; 3 bits, 8 rows 22016 x 4096 21.3 / 18.7; fp16, 8 rows of 8192 x 8192 four units / two 35.6 / 31.3).
//   - v_mfma_f32_16x16x32_f16 with the weights as the A operand (4-bit sums, below: B) straight from global memory.  A load takes whole
//     128-byte lines: 8 rows x 8 lanes, rows 0..7 and 8..15 of a tile by two loads; exchanging the two registers between the lanes
//     l and l ^ 8 (one DPP move each) leaves lane l with row l % 16 and pieces 2 q and 2 q + 1 of the row's line, q = l / 16: the
//     A layout, with the columns of a unit dealt to the quarters in pairs of sub-groups.  Because every line is touched by one
//     instruction only, the loads carry the non-temporal hint (27648 x 5120 in fp16, two rows: 55 -> 50 us; loads of 16 rows x
//     64 bytes got slower with it).  3-bit rows are 96 bytes per unit: no hint there.
//   - A 16-byte piece is one sub-group of 32 columns and gives four MFMA steps, one per word; scales come as one load per lane
//     and four units and are dealt to the quarters with v_permlane swaps.
//   - 4-bit scales meet the fp32 sums of their groups, not the codes (all groups at up to 16 rows, 64 and 128 up to 32): permlane swaps put columns
//     of one group into all quarters of an MFMA, whose result has x rows in registers and the weight row in the lane, so one scale per lane
//     does for a group; the codes go in as 64 + u, and what that adds leaves with three small MFMAs of the scales per four units.  Nothing is
//     rounded before the result (2.07e-4 off the 64-bit one at 4096 x 5120, the rounding of the result itself; scaled codes 2.78e-4), and a
//     word costs 9 (128) to 13 (32) vector operations instead of 18: 16 rows, groups of 128 / 32, 5120 x 5120 14.6 / 13.2 -> 11.6 / 12.2 us, 15360 x
//     5120 20.9 / 19.4 -> 15.6 / 16.4, 22016 x 4096 18.1 / 18.4 -> 15.1 / 16.6, 57344 x 8192 57 / 59 -> 53 / 57 (little in flight included).  Beyond,
//     groups of 32 would need more operations for the sums of 32 x rows than for the codes.
//   - The order of k inside an MFMA is free as long as A and B agree: x is put into the order the decode yields.  What x
//     costs is its bytes (256 workgroups x n rows from the L2s, 13 TB/s), not the pattern: fetching it in 64-byte pieces per row
//     and transposing in registers took the same time.
//   - The wavefronts' partial tiles meet in LDS once per batch of row tiles (every tile of the launch on most shapes); then
//     all threads add the eight shares in a fixed order and apply the epilogue: fp16 store, rotary + KV append, residual add,
//     SwiGLU.  A row tile is 8 + 8 rows so that both members of a rotation pair / a gate and its up value meet in one tile.
//   - Rows longer than eight slices hold (or that would leave CUs idle) are also cut along k over kg workgroups; these write
//     fp32 partial rows that the finishing pass of the split-K kernel adds in order.
//   - Loads are buffer loads: rows past the matrix, x rows past n, dead units and tiles past the range are out of range and
//     return 0 without traffic, so the schedule of requests is the same everywhere and the compiler's wait counts stay exact.
#pragma once

#include <algorithm>
#include <atomic>

#include "relax_common.h"

namespace relax {

namespace fewrow {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));

enum { F_Q4G32 = 0, F_Q4G64 = 1, F_Q4G128 = 2, F_Q3 = 3, F_F16 = 4 };

constexpr int kWaves = 8, kThreads = kWaves * 64;
// 4-bit: whether a group's scale meets the fp32 sum of its products (exact), or its codes (one rounding per weight; three units of 32 x rows leave
// no registers for sums, and in two k ranges instead a 13B layer of 17 rows with groups of 64 took 123 us, so 120; nor do six of 16: in two
// or three ranges 57344 x 12288 with groups of 32 took 88 us at 12 rows, so 83, 4096 x 11008 at two rows 12.8, so 11.6)
constexpr bool scale_sums(int fmt, int nb, int uw) { return fmt == F_Q4G64 || fmt == F_Q4G128 ? nb <= 2 && uw * nb < 6 : fmt == F_Q4G32 && nb == 1 && uw < 6; }
constexpr int unit_columns(bool f16) { return f16 ? 128 : 256; }      // a row's share of a unit: 128 bytes, 96 (3-bit) or 2 x 128 (fp16)
constexpr int kTileRows = 16;
constexpr uint32_t kNowhere = 0x80000000u;                // an offset past every buffer (they are at most 2^31 - 1 bytes)
constexpr size_t kLdsBytes = 160 * 1024, kShareBytes = 152 * 1024;        // the CU's; of the wavefronts' shares where there are no offsets
// Offsets of 4-bit codes, per wavefront and block of x rows: three parts of 16 rows for four units a pack, or, where row tiles need the space, for the
// units that there are (and a place for what the lanes of the others write)
constexpr bool dense_offsets(int fmt, int uw, bool wait) { return wait || (fmt == F_Q4G32 && uw == 5); }
constexpr size_t offset_bytes(int fmt, int nb, int uw, bool wait)
{
    const int units = dense_offsets(fmt, uw, wait) ? nb * uw * 3 + 1 : nb * ((uw + 3) / 4) * 12;
    return scale_sums(fmt, nb, uw) ? (size_t)kWaves * units * (fmt == F_Q4G32 ? 256 : fmt == F_Q4G64 ? 128 : 64) : 0;
}

// One block of x rows with scales on sums: whether there is a form of the kernel (WAIT) that takes the shares of a batch of tiles together inside the
// loop, so that as many row tiles fit a workgroup (kMostTiles) as without offsets.  A second wave of workgroups instead, with x and the first data
// once more, cost 8 to 20 % (16 rows, groups of 32: 77824 x 4096 46 us, so 41, 36864 x 14336 83, so 68); the other launches keep the form
// without, which is 0.2 us (three units: 1.2) faster on 5120 x 5120.  Five units leave no registers for it.
constexpr bool sums_wait(int fmt, int nb, int uw) { return scale_sums(fmt, nb, uw) && nb == 1 && uw <= 4; }
constexpr int kMostTiles = (int)(kShareBytes / (kWaves * 1024));

struct Args {
    const uint16_t *x;       // [n,k] fp16
    const void *w;           // packed words or fp16 values
    const uint16_t *s;       // scales
    uint32_t x_bytes, w_bytes, s_bytes;
    int32_t n, m, k;
    int32_t kg, rg;          // workgroups along k, row ranges
    int32_t tiles, batch;    // row tiles of the matrix; tiles whose wavefronts' shares fit LDS together
    int32_t epi;             // Epilogue, or kPartial
    int32_t delta;           // the second eight rows of a tile start delta rows after the first eight
    int32_t ropeshift;       // EPI_ROPE_KV: log2(head_dim / 16)
    uint16_t *out_f16;
    float *out_f32;          // x1, or the partial rows [kg][n][m]
    const void *resid;
    uint16_t *kc, *vc;       // EPI_ROPE_KV: cache and rotary table; out_f16 is the qkv buffer [n,m] (q part written)
    const float *rope;
    int32_t h, g, d, cap, rope_once;
    SeqTable st;
};
constexpr int kPartial = 100;

__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, a) + __builtin_bit_cast(half2_t, b));
}
__device__ __forceinline__ uint32_t pk_mul(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, a) * __builtin_bit_cast(half2_t, b));
}
__device__ __forceinline__ uint32_t pk_fma(uint32_t a, uint32_t b, uint32_t c)
{
    half2_t r = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b), __builtin_bit_cast(half2_t, c));
    return __builtin_bit_cast(uint32_t, r);
}
// one packed 4-bit word -> its 8 codes u (0..15) as fp16 64 + u in the order [e0 e4 e1 e5 e2 e6 e3 e7]: a nibble at bits 4..7 of fp16
// 64 counts ones.  (Without the shift of the first pair, at the bottom of 1024, the fp32 sums of 1024 + u were 2.2e-5 off, where the matvec kernels
// are 1.1e-5 off and 64 + u is below 2e-6.)
__device__ __forceinline__ half8_t raw_q4(uint32_t w)
{
    const uint32_t mask = 0x00F000F0u, base = 0x54005400u;
    return __builtin_bit_cast(half8_t, u32x4_t{and_or3(w << 4, mask, base), and_or3(w, mask, base), and_or3(w >> 4, mask, base), and_or3(w >> 8, mask, base)});
}
constexpr uint32_t kOffset = 0x54805480u;                              // the codes mean u - 8: 72 is in every one too many
// its codes less 8, in the same order: 1024 + u - 1032, 64 + u - 72 (two shifts less than raw_q4)
__device__ __forceinline__ u32x4_t decode_q4(uint32_t w)
{
    const uint32_t w8 = w >> 8, kNeg1032 = 0xE408E408u, kNeg72 = 0xD480D480u;
    return u32x4_t{pk_add(and_or3(w, 0x000F000Fu, 0x64006400u), kNeg1032), pk_add(and_or3(w, 0x00F000F0u, 0x54005400u), kNeg72),
                   pk_add(and_or3(w8, 0x000F000Fu, 0x64006400u), kNeg1032), pk_add(and_or3(w8, 0x00F000F0u, 0x54005400u), kNeg72)};
}
// packet j (columns 8j .. 8j+7) of a 3-bit group from its three words -> its codes less 4 as fp16: pairs (1024 + f u) with f = 1, 8
// or 64 by class, one packed fma removes weight and offset exactly ((1024 + f u) / f - (1024 / f + 4) = u - 4).
// QUARTER: a quarter of that, as exact (all constants are fp16 values)
template <bool QUARTER>
__device__ __forceinline__ u32x4_t decode_q3(const u32x3_t &w, int j)
{
    const uint32_t base = 0x64006400u;
    u32x4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int p = 4 * j + i, cls = q3n_class(p);
        uint32_t pair;
        if (p == 15) {
            pair = and_or3(w[0] >> 15, 0x00010001u, base);
            pair = and_or3(w[1] >> 14, 0x00020002u, pair);
            pair = and_or3(w[2] >> 13, 0x00040004u, pair);
        } else {
            const uint32_t v = p % 5 >= 3 ? w[p / 5] >> 9 : w[p / 5];
            pair = and_or3(v, cls == 0 ? 0x00070007u : cls == 1 ? 0x00380038u : 0x01C001C0u, base);
        }
        if (QUARTER) r[i] = cls == 0 ? pk_fma(pair, 0x34003400u, 0xDC04DC04u) : cls == 1 ? pk_fma(pair, 0x28002800u, 0xD020D020u) : pk_fma(pair, 0x1C001C00u, 0xC500C500u);
        else r[i] = cls == 0 ? pk_add(pair, 0xE404E404u) : cls == 1 ? pk_fma(pair, 0x30003000u, 0xD820D820u) : pk_fma(pair, 0x24002400u, 0xCD00CD00u);
    }
    return r;
}
__device__ __forceinline__ half8_t scaled(const u32x4_t &v, uint32_t s2)
{
    return __builtin_bit_cast(half8_t, u32x4_t{pk_mul(v[0], s2), pk_mul(v[1], s2), pk_mul(v[2], s2), pk_mul(v[3], s2)});
}

// a b + c rounded to fp16 once: what the compiler makes of the stand-alone rotary kernel's expression, whose bits the epilogue repeats
__device__ __forceinline__ uint16_t fma_f16(float a, float b, float c)
{
    uint32_t r = 0;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3" : "+v"(r) : "v"(a), "v"(b), "v"(c));
    return (uint16_t)r;
}

// orders LDS only: requests in flight stay in flight across it
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// a: rows 0..7 in lanes with bit 3 clear and set, b: rows 8..15 -> a: piece 2 q of row l % 16, b: piece 2 q + 1
__device__ __forceinline__ void rows_to_lanes(uint32_t &a, uint32_t &b)
{
    const uint32_t a0 = a;
    a = __builtin_amdgcn_update_dpp(a, b, 0x128, 0xF, 0xC, false);      // row_ror:8, upper eight lanes of each row of 16
    b = __builtin_amdgcn_update_dpp(b, a0, 0x128, 0xF, 0x3, false);     // ... lower eight
}

// A wavefront's share of the launch: units u0 .. u0 + nu - 1 of the row tiles t0 .. t0 + nt - 1.  Neighbouring workgroups (they go to different
// XCDs) take different k ranges of the same rows.
struct Share {
    int kgi, nu, u0, nt, t0;
    template <typename A>
    __device__ __forceinline__ Share(const A &a, int wave, int unit_cols)
    {
        const int rgi = blockIdx.x / a.kg;
        kgi = blockIdx.x - rgi * a.kg;
        const int units = a.k / unit_cols, slices = a.kg * kWaves, slice = kgi * kWaves + wave;
        const int ubase = units / slices, urem = units - ubase * slices;
        nu = ubase + (slice < urem), u0 = slice * ubase + min(slice, urem);
        const int tbase = a.tiles / a.rg, trem = a.tiles - tbase * a.rg;
        nt = tbase + (rgi < trem), t0 = rgi * tbase + min(rgi, trem);
    }
};
// first matrix row of a tile's first half
template <typename A>
__device__ __forceinline__ int tile_first_row(const A &a, int t)
{
    if (a.epi == EPI_SWIGLU) return t * 8;
    if (a.epi == EPI_ROPE_KV) return ((t >> a.ropeshift) * a.d) + (t & ((1 << a.ropeshift) - 1)) * 8;
    return t * 16;
}

// The kernel's arguments, its one parameter, read again from where they were passed.  What the compiler holds in scalar registers over the loop for the code behind it, it spills: 45 moves in front
// of the first data, 80 (with redo_rows 280) behind the loop.  Without them a launch takes 0.5 to 1 us less (us: 4 rows, groups of 32, 4096 x
// 4096 7.1 -> 6.3, 22016 x 4096 16.2 -> 14.9, 57344 x 8192 53.9 -> 53.2; 32 rows, groups of 128, 12288 x 4096 15.9 -> 14.9).
__device__ __forceinline__ const Args &args_again()
{
    const __attribute__((address_space(4))) Args *p = (const __attribute__((address_space(4))) Args *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const Args *)p;
}

// Rows of x with an infinity or a NaN where 4-bit scales meet sums: the sums of 64 + u lose an infinity to the offset (inf - inf), where its product
// with a code less 8 is infinite.  The wavefront that holds one computes its shares of these rows (bits of `odd`) once more from codes less 8,
// in plain fp32 (40 us per row and tile at most), for the `count` tiles from `first` of its range on, whose shares are in red; the rows beside them
// keep their bits, the calls without pay 0.1 us for the look.
template <int FMT, int NB>
__device__ __forceinline__ void redo_rows(float4_t *red, uint32_t odd, int first, int count)
{
    constexpr int SG = FMT == F_Q4G64 ? 64 : FMT == F_Q4G128 ? 128 : 32, kUnit = unit_columns(false);
    const Args &a = args_again();
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r16 = lane & 15, qd = lane >> 4;
    const int k = a.k;
    const Share sh(a, wave, kUnit);
#pragma unroll 1
    for (int it = 0; it < count * NB; ++it) {
        const int bt = it / NB, nb = it - bt * NB;
        // (rows past the matrix: the last one's results, which nobody reads)
        const size_t row = min(tile_first_row(a, sh.t0 + first + bt) + (r16 & 7) + (r16 >> 3) * a.delta, a.m - 1);
        float *dst = (float *)&red[((bt * kWaves + wave) * NB + nb) * 64];
#pragma unroll 1
        for (uint32_t todo = odd >> (nb * 16 % 32) & 0xFFFFu; todo; todo &= todo - 1) {
            const int i = __builtin_ctz(todo);
            float sum = 0.0f;
#pragma unroll 1
            for (int c = sh.u0 * kUnit + qd * 8; c < (sh.u0 + sh.nu) * kUnit; c += 32) {
                const uint32_t w = ((const uint32_t *)a.w)[row * (k / 8) + c / 8];
                const half8_t xv = *(const half8_t *)(a.x + (size_t)(nb * 16 + i) * k + c);
                float part = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) part = fmaf((float)((int)(w >> (4 * e) & 15u) - 8), (float)xv[e], part);
                sum = fmaf(part, h2f(a.s[row * (k / SG) + c / SG]), sum);
            }
            sum += __shfl_xor(sum, 16, kWave);
            sum += __shfl_xor(sum, 32, kWave);
            if (qd == 0) dst[(16 * (r16 >> 2) + (i ^ (r16 >> 2))) * 4 + (r16 & 3)] = sum;
        }
    }
}

// UW units per wavefront, NB blocks of 16 x rows; in flight per wavefront: T row tiles (D == UW), or D units (T == 1, D < UW).
// WAIT: the shares of a full batch of tiles are taken together inside the loop (sums_wait).
template <int FMT, int NB, int UW, int T, int D, bool WAIT>
__global__ __launch_bounds__(kThreads) void fewrow_kernel(Args args)
{
    const Args &a = args;
    constexpr bool Q3 = FMT == F_Q3, F16 = FMT == F_F16;
    static_assert(D == UW || (T == 1 && UW % D == 0), "ring of units");
    constexpr int NL = F16 ? 2 : 1;                       // lines of a row per unit
    constexpr int ST = F16 ? 4 : 8;                       // MFMA steps per unit
    constexpr int kUnit = unit_columns(F16);
    constexpr int kUnitBytes = Q3 ? 96 : F16 ? 256 : 128; // of one row
    constexpr int kPiece = Q3 ? 12 : 16;                  // bytes per lane and load
    constexpr int SP = F16 ? 0 : (UW + 3) / 4;            // scale loads per tile (four units each)
    constexpr int SG = FMT == F_Q4G64 ? 64 : FMT == F_Q4G128 ? 128 : 32;
    constexpr int SW = 128 / SG;                          // words of scales per unit and row: 4, 2 or 1
    constexpr int kNt = Q3 ? 0 : 2;                       // non-temporal
    // 3-bit weights at up to 16 rows are exact for every finite scale: a scale is split into its upper eight significant bits and the
    // rest, both products with a quarter of a code (at most 1, so that nothing leaves fp16) fit its eleven bits, and the second
    // goes through MFMAs of its own (scaled by 2^8, which its largest value, 224 x 2^8, still bears).  Below 16 rows
    // the 3-bit matvec kernels, which multiply by the scale in fp32, served these calls; with one rounding per weight the appended V
    // of a 7B layer was 3.20e-4 off the 64-bit result instead of 2.95e-4 (the split costs 4 us of 62).  Elsewhere the products are
    // rounded once, as in the split-K kernel and the tiled GEMM.
    constexpr bool EXACT = NB == 1 && Q3;
    constexpr bool SUMS = scale_sums(FMT, NB, UW);
    constexpr int GU = SUMS ? 256 / SG : 1;               // groups of a unit: one, two or four MFMA steps each
    constexpr int GS = ST / GU;
    extern __shared__ __align__(16) float4_t red[];       // [tile of the batch][wavefront][NB][64]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, qd = lane >> 4;
    const Share sh(a, wave, kUnit);
    const int kgi = sh.kgi, nu = sh.nu, u0 = sh.u0, nt = sh.nt, t0 = sh.t0;      // nu: UW or UW - 1
    auto tile_row = [&](int t) { return tile_first_row(a, t); };

    // ---- x of the wavefront's columns, in the order the decode yields ----
    // step s of a packed unit: word s % 4 of piece 2 q + s / 4; of an fp16 unit: piece 2 q + s % 2 of line s / 2
    // of a 4-bit unit: what set_to_steps makes of the sets of pieces 0..3 and 4..7
    auto x_step = [](int s) {
        return F16 || (SUMS && SG == 64) ? (s >> 1) * 128 + (s & 1) * 16 : !SUMS ? s * 16 : SG == 128 ? (s >> 2) * 256 + (s & 3) * 16 : s * 64;
    };
    u32x4_t X[UW][ST][NB];
    {
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x), 0, a.x_bytes, 0x00020000);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const uint32_t row = (uint32_t)(16 * nb + r16);
            const uint32_t xq = F16 ? qd * 32 : !SUMS ? qd * 128 : SG == 32 ? qd * 16 : SG == 64 ? (qd & 1) * 64 + (qd >> 1) * 32 : qd * 64;
            const uint32_t xo = row < (uint32_t)a.n ? row * (uint32_t)a.k * 2 + (uint32_t)(u0 * kUnit) * 2 + xq : kNowhere;
            const uint32_t xo_last = nu < UW ? kNowhere : xo + (UW - 1) * kUnit * 2;
#pragma unroll
            for (int u = 0; u < UW; ++u)
#pragma unroll
                for (int s = 0; s < ST; ++s)
                    X[u][s][nb] = __builtin_amdgcn_raw_buffer_load_b128(xr, (u == UW - 1 ? xo_last : xo + u * kUnit * 2) + x_step(s), 0, 0);
        }
    }

    struct Tile {
        u32x4_t w[Q3 ? 1 : D][NL][2];                     // unit u of the tile is in entry u % D; rows 0..7, rows 8..15
        u32x3_t w3[Q3 ? D : 1][2];
        u32x4_t s[SP ? SP : 1];
    };
    const uint32_t wpitch = F16 ? (uint32_t)a.k * 2 : Q3 ? (uint32_t)(a.k / 32) * 12 : (uint32_t)a.k / 2;
    const uint32_t spitch = (uint32_t)(a.k / SG) * 2;
    const uint32_t piece = SUMS ? (uint32_t)((lane >> 3) & 1) * 4 + qd : (uint32_t)(lane >> 3);
    const uint32_t wo0 = (uint32_t)(lane & 7) * wpitch + (uint32_t)u0 * kUnitBytes + piece * kPiece, wo1 = wo0 + (uint32_t)a.delta * wpitch;
    const uint32_t wo0_last = nu < UW ? kNowhere : wo0 + (UW - 1) * kUnitBytes, wo1_last = nu < UW ? kNowhere : wo1 + (UW - 1) * kUnitBytes;
    // scale load of pack p: quarter q brings the scales of unit 4 p + q
    const uint32_t so = ((r16 & 7) + (r16 >> 3) * (uint32_t)a.delta) * spitch + (uint32_t)(u0 + qd) * (SW * 4);
    const uint32_t so_last = SUMS && (SP - 1) * 4 + qd >= nu ? kNowhere : so + (SP - 1) * (4 * SW * 4);      // 0 for units that are not the wavefront's
    struct Where {                                        // the rest of the matrix from one row tile on; empty for a tile past the range
        __amdgpu_buffer_rsrc_t w, s;
    };
    auto where = [&](int t) {
        const bool live = t < nt;
        const uint32_t row = live ? (uint32_t)tile_row(t0 + t) : 0u;
        Where at;
        at.w = __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<void *>(a.w) + row * wpitch, 0, live ? a.w_bytes - row * wpitch : 0, 0x00020000);
        if (SP) at.s = __builtin_amdgcn_make_buffer_rsrc((char *)const_cast<uint16_t *>(a.s) + row * spitch, 0, live ? a.s_bytes - row * spitch : 0, 0x00020000);
        return at;
    };
    auto load_unit = [&](Tile &b, const Where &at, int u) {
#pragma unroll
        for (int l = 0; l < NL; ++l)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t o = (u == UW - 1 ? (i ? wo1_last : wo0_last) : (i ? wo1 : wo0) + u * kUnitBytes) + l * 128;
                if (Q3) b.w3[Q3 ? u % D : 0][i] = __builtin_amdgcn_raw_buffer_load_b96(at.w, o, 0, kNt);
                else b.w[Q3 ? 0 : u % D][l][i] = __builtin_amdgcn_raw_buffer_load_b128(at.w, o, 0, kNt);
            }
    };
    auto load_scales = [&](Tile &b, const Where &at, int p) {
        const uint32_t o = p == SP - 1 ? so_last : so + p * (4 * SW * 4);
        if (SW == 4) {
            b.s[p] = __builtin_amdgcn_raw_buffer_load_b128(at.s, o, 0, 0);
        } else if (SW == 2) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(at.s, o, 0, 0);
            b.s[p][0] = v[0], b.s[p][1] = v[1];
        } else {
            b.s[p][0] = __builtin_amdgcn_raw_buffer_load_b32(at.s, o, 0, 0);
        }
    };
    // rows of 16 lanes r0..r3: v[0] of all four -> one word per unit of the pack
    auto swap16 = [](uint32_t va, uint32_t vb, uint32_t &ra, uint32_t &rb) {
        const auto r = __builtin_amdgcn_permlane16_swap(va, vb, false, false);
        ra = r[0], rb = r[1];
    };
    // 4 x 4 transpose over words and quarters: word q of what quarter i holds -> r[i]
    auto transpose4 = [&](const uint32_t (&v)[4], uint32_t (&r)[4]) {
        const auto p02 = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false), p13 = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
        swap16(p02[0], p13[0], r[0], r[1]);
        swap16(p02[1], p13[1], r[2], r[3]);
    };
    // scales on codes: the scale pairs of units 4 p .. 4 p + 3 for this lane's sub-groups 2 q and 2 q + 1
    const uint32_t sel = (SW == 2 ? qd & 1 : qd >> 1) ? 0x03020302u : 0x01000100u;
    auto unpack_scales = [&](const u32x4_t v, uint32_t (*s2)[2]) {
        uint32_t c4[4];
        if (SW == 4) {
            const uint32_t vv[4] = {v[0], v[1], v[2], v[3]};
            transpose4(vv, c4);
        } else {                                          // two words: quarters 0, 1 need word 0 of a unit, quarters 2, 3 word 1; or one for all
            const auto r = __builtin_amdgcn_permlane32_swap(v[0], SW == 2 ? v[1] : v[0], false, false);
            swap16(r[0], r[0], c4[0], c4[1]);             // units 4 p, 4 p + 1 in the even and odd rows of 16 lanes
            swap16(r[1], r[1], c4[2], c4[3]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s2[i][0] = __builtin_amdgcn_perm(c4[i], c4[i], SW == 4 ? 0x01000100u : sel);
            s2[i][1] = __builtin_amdgcn_perm(c4[i], c4[i], SW == 4 ? 0x03020302u : sel);
        }
    };
    // 4-bit: the scales of units 4 p + 2 half and the next, as loaded by the quarters, for all quarters
    auto spread_scales = [&](const u32x4_t v, int half, uint32_t (*su)[SW]) {
#pragma unroll
        for (int i = 0; i < SW; ++i) {
            const auto r = __builtin_amdgcn_permlane32_swap(v[i], v[i], false, false);
            swap16(r[half], r[half], su[0][i], su[1][i]);
        }
    };
    // 4-bit, pieces 0..3 (or 4..7) of a unit, piece q in quarter q -> one word per MFMA step, such that the quarters of a step hold columns of
    // one group: groups of 32 are four quarters of a piece, groups of 64 two halves of two pieces, groups of 128 the four pieces as they are
    auto set_to_steps = [&](const u32x4_t v, uint32_t (&r)[4]) {
        if (SG == 32) {
            const uint32_t vv[4] = {v[0], v[1], v[2], v[3]};
            transpose4(vv, r);
        } else if (SG == 64) {
            const auto p02 = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false), p13 = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
            r[0] = p02[0], r[1] = p13[0], r[2] = p02[1], r[3] = p13[1];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = v[j];
        }
    };

    Tile buf[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const Where at = where(i);
#pragma unroll
        for (int p = 0; p < SP; ++p) load_scales(buf[i], at, p);
#pragma unroll
        for (int u = 0; u < D; ++u) load_unit(buf[i], at, u);
    }
    if (!F16 && !Q3) {                                    // [x0 x1 | x2 x3 | x4 x5 | x6 x7] -> [x0 x4 | x1 x5 | x2 x6 | x3 x7]
#pragma unroll
        for (int u = 0; u < UW; ++u)
#pragma unroll
            for (int s = 0; s < ST; ++s)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const u32x4_t v = X[u][s][nb];
                    X[u][s][nb] = u32x4_t{__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                                          __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u)};
                }
    }

    // 4-bit: what the offsets of the codes add to a group's sum for x row r16, negated, in the lanes that load the scales of the group's unit, as three fp16
    // parts (2^-13 or less of it, so that no x overflows; the next part scaled by 2^11).  The contraction over the groups with the
    // scales as they are loaded takes the offsets out of a tile: three MFMAs per four units.
    constexpr float kDown = SG == 32 ? 0x1p-13f : SG == 64 ? 0x1p-14f : 0x1p-15f;
    // They wait in LDS (a slot of each wavefront's own): the registers are x's.
    typedef _Float16 part_t __attribute__((ext_vector_type(GU > 1 ? GU : 2)));
    part_t *const off = reinterpret_cast<part_t *>(red + (size_t)a.batch * (kWaves * NB * 64)) + wave * (int)(offset_bytes(FMT, NB, UW, WAIT) / (kWaves * sizeof(part_t)));
    constexpr bool DENSE = dense_offsets(FMT, UW, WAIT);
    auto part_at = [&](int l, int nb, int p, int i) {     // part i of lane l's unit of pack p (a unit that the pack does not have: another's, times scales of 0)
        const int unit = 4 * p + 3 < UW ? 4 * p + (l >> 4) : 4 * p + 1 == UW ? 4 * p : min(4 * p + (l >> 4), UW - 1);
        return DENSE ? ((nb * UW + unit) * 3 + i) * 16 + (l & 15) : ((nb * SP + p) * 3 + i) * 64 + l;
    };
    uint32_t odd = 0;                                     // bits of the x rows whose sums are not finite in the wavefront's columns (see redo_rows)
    static_assert(!SUMS || NB <= 2, "a bit per row");
    if constexpr (SUMS) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float nan = 0.0f;
#pragma unroll
            for (int p = 0; p < SP; ++p) {
                // rows of a constant matrix: those of quarter u % 4 hold what unit u's columns count, so that a lane gets its own units' sums
                float o[GU];
#pragma unroll
                for (int j = 0; j < GU; ++j) {
                    float4_t d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int u = 4 * p; u < UW && u < 4 * p + 4; ++u) {
                        const uint32_t c1 = (r16 >> 2) == (u & 3) ? kOffset : 0u;
                        const u32x4_t c = {c1, c1, c1, c1};
#pragma unroll
                        for (int s = j * GS; s < (j + 1) * GS; ++s)
                            d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, c), __builtin_bit_cast(half8_t, X[u][s][nb]), d, 0, 0, 0);
                    }
                    o[j] = d[0];
                    nan = fmaf(o[j], 0.0f, nan);
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    part_t part;
#pragma unroll
                    for (int j = 0; j < GU; ++j) {
                        const float v = o[j] * (i == 0 ? -kDown : 1.0f);
                        part[j] = (_Float16)v;
                        o[j] = (v - (float)part[j]) * 0x1p11f;
                    }
                    off[!DENSE || 4 * p + 3 < UW || 4 * p + qd < UW ? part_at(lane, nb, p, i) : NB * UW * 3 * 16 + r16] = part;
                }
            }
            const uint64_t lanes = __ballot(nan != nan);
            odd |= ((uint32_t)(lanes | lanes >> 16 | lanes >> 32 | lanes >> 48) & 0xFFFFu) << (nb * 16 % 32);
        }
    }

    // one row tile: its MFMAs, unit by unit, each unit's registers re-requested for tile t + T as soon as it is consumed
    auto consume = [&](Tile &b, int t, int at_batch) {
        float4_t acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        float4_t rest = {0.0f, 0.0f, 0.0f, 0.0f};
        const Where next = where(t + T), cur = D < UW ? where(t) : next;
        uint32_t s2[SUMS ? 1 : 4][2], su[2][SW];
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            float4_t d[2][NB];                            // 4-bit: sums of two groups
            auto apply_scale = [&](int grp) {
                const float sc = (float)__builtin_bit_cast(half2_t, su[u % 2][grp / 2])[grp % 2];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[nb][e] = fmaf(d[grp % 2][nb][e], sc, acc[nb][e]);
            };
            if (SP && u % 4 == 0) {
                if constexpr (SUMS) {
                    const u32x4_t v = b.s[SP ? u / 4 : 0];
                    int l = lane;
                    asm volatile("" : "+v"(l));           // read per tile: as loop invariants the parts, or their addresses, would be kept in registers, or spilled
                    const half8_t sv = __builtin_bit_cast(half8_t, u32x4_t{v[0], SW >= 2 ? v[1] : 0u, SW == 4 ? v[2] : 0u, SW == 4 ? v[3] : 0u});
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        float4_t d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                        for (int i = 2; i >= 0; --i) {
                            const part_t part = off[part_at(l, nb, u / 4, i)];
                            half8_t pf;
#pragma unroll
                            for (int j = 0; j < 8; ++j) pf[j] = j < GU ? part[j < GU ? j : 0] : (_Float16)0.0f;
                            d = __builtin_amdgcn_mfma_f32_16x16x32_f16(pf, sv, d, 0, 0, 0) * (i > 0 ? 0x1p-11f : 1.0f / kDown);
                        }
                        acc[nb] += d;
                    }
                } else {
                    unpack_scales(b.s[SP ? u / 4 : 0], s2);
                    load_scales(b, next, u / 4);
                }
            }
            if (SUMS && u % 2 == 0) {
                spread_scales(b.s[SP ? u / 4 : 0], u % 4 / 2, su);
                if (u % 4 == 2 || u + 2 >= UW) load_scales(b, next, u / 4);
            }
            if (u < UW - 1 || nu == UW) {                 // wavefront-uniform, no memory operation inside
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    if (Q3) {
#pragma unroll
                        for (int e = 0; e < 3; ++e) {
                            uint32_t lo = b.w3[Q3 ? u % D : 0][0][e], hi = b.w3[Q3 ? u % D : 0][1][e];
                            rows_to_lanes(lo, hi);
                            b.w3[Q3 ? u % D : 0][0][e] = lo, b.w3[Q3 ? u % D : 0][1][e] = hi;
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            uint32_t lo = b.w[Q3 ? 0 : u % D][l][0][e], hi = b.w[Q3 ? 0 : u % D][l][1][e];
                            rows_to_lanes(lo, hi);
                            b.w[Q3 ? 0 : u % D][l][0][e] = lo, b.w[Q3 ? 0 : u % D][l][1][e] = hi;
                        }
                    }
                }
                if constexpr (SUMS) {
                    // x rows times weight rows: lane l holds weight row l % 16 of a group's sum and meets it with that row's scale in fp32, while the
                    // next group's first MFMA runs (left to itself the compiler waits for every MFMA: 8 of 18 slots per step)
                    uint32_t word[4];
#pragma unroll
                    for (int s = 0; s < ST; ++s) {
                        if (s % 4 == 0) set_to_steps(b.w[u % D][0][s / 4], word);
                        const half8_t wf = raw_q4(word[s % 4]);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            d[s / GS % 2][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, X[u][s][nb]), wf,
                                                                                       s % GS == 0 ? float4_t{0.0f, 0.0f, 0.0f, 0.0f} : d[s / GS % 2][nb], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (s >= GS && s % GS == 0) apply_scale(s / GS - 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    apply_scale(GU - 1);
                }
#pragma unroll
                for (int s = 0; s < (SUMS ? 0 : ST); ++s) {
                    half8_t af;
                    if (F16) {
                        af = __builtin_bit_cast(half8_t, b.w[Q3 ? 0 : u % D][F16 ? s >> 1 : 0][s & 1]);
                    } else {
                        const uint32_t sc = s2[SUMS ? 0 : u % 4][(s >> 2) & 1];
                        const u32x4_t codes = Q3 ? decode_q3<EXACT>(b.w3[Q3 ? u % D : 0][(s >> 2) & 1], s & 3) : decode_q4(b.w[Q3 ? 0 : u % D][0][(s >> 2) & 1][s & 3]);
                        if (EXACT) {
                            const uint32_t upper = sc & 0xFFF8FFF8u;
                            const half8_t low = scaled(codes, pk_mul(pk_add(sc, upper ^ 0x80008000u), 0x5C005C00u));
                            rest = __builtin_amdgcn_mfma_f32_16x16x32_f16(low, __builtin_bit_cast(half8_t, X[u][s][0]), rest, 0, 0, 0);
                            af = scaled(codes, upper);
                        } else {
                            af = scaled(codes, sc);
                        }
                    }
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af, __builtin_bit_cast(half8_t, X[u][s][nb]), acc[nb], 0, 0, 0);
                    if (UW * NB >= 6 && !F16) __builtin_amdgcn_sched_barrier(0);       // x takes 192 registers: one step's decode at a time
                }
            }
            if (u + D < UW) load_unit(b, cur, u + D);
            else load_unit(b, next, u + D - UW);
            __builtin_amdgcn_sched_barrier(0);            // keeps decodes of later units (and their registers) out of this one
        }
        if (EXACT) acc[0] = (acc[0] + rest * 0x1p-8f) * 4.0f;
        if constexpr (SUMS) {
            // lane l holds x rows 4 (l / 16) .. + 3 of weight row l % 16: into the layout that finish reads (float4 lane & 15 of row group
            // l / 16 there is one x row's four weight rows), its lanes permuted so that the four stores meet no bank twice
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float *dst = (float *)&red[((at_batch * kWaves + wave) * NB + nb) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[(16 * (r16 >> 2) + ((4 * qd + e) ^ (r16 >> 2))) * 4 + (r16 & 3)] = acc[nb][e];
            }
        } else {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) red[((at_batch * kWaves + wave) * NB + nb) * 64 + lane] = acc[nb];
        }
    };
    const int at_lane = SUMS ? lane ^ qd : lane;

    // ---- the wavefronts' shares of `count` tiles from t0 + first on: sum in order, epilogue ----
    // value layout of a tile block: lane l holds x row l % 16 of the block and tile rows 4 (l / 16) .. + 3; tile rows 0..7 are the
    // first half of the tile, 8..15 the second, so lane l and lane l ^ 32 hold the two members of a pair
    // WAIT: the sums of the tiles before `first`, behind the offsets
    float4_t *const sums = (float4_t *)((char *)(red + (size_t)a.batch * (kWaves * NB * 64)) + offset_bytes(FMT, NB, UW, WAIT));
    auto finish = [&](int first, int count) {
        const Args &a = SUMS ? args_again() : args;
        for (int it = (WAIT ? -first : 0) + wave; it < count * NB; it += kWaves) {
            const int bt = NB == 1 ? it : it / NB, nb = NB == 1 ? 0 : it - bt * NB, t = t0 + first + bt;
            const int i = nb * 16 + r16, half = lane >> 5;
            if (nb * 16 >= a.n) continue;
            float4_t v;
            if (WAIT && it < 0) {
                v = sums[(first + it) * 64 + lane];
            } else {
                v = red[(bt * kWaves * NB + nb) * 64 + at_lane];
#pragma unroll
                for (int w = 1; w < kWaves; ++w) v += red[((bt * kWaves + w) * NB + nb) * 64 + at_lane];
            }
            const int row = tile_row(t) + (qd & 1) * 4 + half * a.delta;       // matrix row of v[0]
            if (a.epi == EPI_SWIGLU) {
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float2 p = pair_xor32(v[e]);                         // gate, up
                    o[e] = p.x / (1.0f + __expf(-p.x)) * p.y;
                }
                if (half == 0 && i < a.n && row < a.delta)
                    *(uint2 *)(a.out_f16 + (size_t)i * a.delta + row) = make_uint2(f2h(o[0]) | ((uint32_t)f2h(o[1]) << 16), f2h(o[2]) | ((uint32_t)f2h(o[3]) << 16));
                continue;
            }
            if (a.epi == EPI_ROPE_KV) {
                // the fp16 rounding of the plain epilogue comes first (rope_once: does not); then both members of each rotation pair in either lane
                const uint32_t h01 = f2h(v[0]) | ((uint32_t)f2h(v[1]) << 16), h23 = f2h(v[2]) | ((uint32_t)f2h(v[3]) << 16);
                const auto p01 = __builtin_amdgcn_permlane32_swap(h01, h01, false, false), p23 = __builtin_amdgcn_permlane32_swap(h23, h23, false, false);
                const uint32_t ab[4] = {p01[0], p23[0], p01[1], p23[1]};
                float pa[4], pb[4];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    pa[2 * e] = h2f((uint16_t)(ab[e] & 0xFFFFu)), pa[2 * e + 1] = h2f((uint16_t)(ab[e] >> 16));
                    pb[2 * e] = h2f((uint16_t)(ab[2 + e] & 0xFFFFu)), pb[2 * e + 1] = h2f((uint16_t)(ab[2 + e] >> 16));
                }
                if (a.rope_once) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float2 p = pair_xor32(v[e]);
                        pa[e] = p.x, pb[e] = p.y;
                    }
                }
                if (i >= a.n) continue;
                const RowInfo ri = row_info(a.st, i);
                const int j = t >> a.ropeshift, tt = (t & ((1 << a.ropeshift) - 1)) * 8 + (qd & 1) * 4, hd2 = a.d >> 1;
                uint16_t o[4];
                if (j < a.h + a.g) {
                    const float *cs = a.rope + ((size_t)ri.pos * hd2 + tt) * 2;
                    const float4_t c01 = *(const float4_t *)cs, c23 = *(const float4_t *)(cs + 4);
                    const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = fma_f16(pa[e], half ? si[e] : co[e], pb[e] * (half ? co[e] : -si[e]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = f2h(v[e]);
                }
                const uint2 packed = make_uint2(o[0] | ((uint32_t)o[1] << 16), o[2] | ((uint32_t)o[3] << 16));
                const int e0 = tt + half * hd2;
                if (j < a.h) {
                    *(uint2 *)(a.out_f16 + (size_t)i * a.m + j * a.d + e0) = packed;
                } else {
                    const size_t tok = ((size_t)ri.slot * a.cap + ri.pos) * (size_t)(a.g * a.d);
                    if (j < a.h + a.g) *(uint2 *)(a.kc + tok + (size_t)(j - a.h) * a.d + e0) = packed;
                    else *(uint2 *)(a.vc + tok + (size_t)(j - a.h - a.g) * a.d + e0) = packed;
                }
                continue;
            }
            if (i >= a.n || row >= a.m) continue;                              // m % 4 == 0 is checked by the launcher
            const size_t at = (size_t)i * a.m + row;
            if (a.epi == kPartial) {
                *(float4_t *)(a.out_f32 + ((size_t)kgi * a.n + i) * a.m + row) = v;
                continue;
            }
            if (a.epi == EPI_RESID_F32) {
                const uint2 xx = *(const uint2 *)((const uint16_t *)a.resid + at);
                *(float4_t *)(a.out_f32 + at) = float4_t{h2f((uint16_t)(xx.x & 0xFFFFu)) + v.x, h2f((uint16_t)(xx.x >> 16)) + v.y,
                                                         h2f((uint16_t)(xx.y & 0xFFFFu)) + v.z, h2f((uint16_t)(xx.y >> 16)) + v.w};
                continue;
            }
            if (a.epi == EPI_RESID_F16) v += *(const float4_t *)((const float *)a.resid + at);
            *(uint2 *)(a.out_f16 + at) = make_uint2(f2h(v.x) | ((uint32_t)f2h(v.y) << 16), f2h(v.z) | ((uint32_t)f2h(v.w) << 16));
        }
    };

    // the same for partial rows inside the loop, in few registers (x and the requested weights stay where they are)
    auto flush = [&](int first, int count) {
        for (int it = wave; it < count * NB; it += kWaves) {
            const int bt = it / NB, nb = it - bt * NB, i = nb * 16 + r16, row = (t0 + first + bt) * 16 + qd * 4;
            if (i >= a.n || row >= a.m) continue;
            float4_t v = red[(bt * kWaves * NB + nb) * 64 + at_lane];
#pragma unroll 1
            for (int w = 1; w < kWaves; ++w) v += red[((bt * kWaves + w) * NB + nb) * 64 + at_lane];
            *(float4_t *)(a.out_f32 + ((size_t)kgi * a.n + i) * a.m + row) = v;
        }
    };

    int first = 0, filled = 0;                            // tiles first .. first + filled - 1 of the range sit in LDS
    for (int t = 0;; t += T) {
        bool done = false;
#pragma unroll
        for (int u = 0; u < T; ++u) {
            consume(buf[u], t + u, filled);
            ++filled;
            if (t + u + 1 >= nt) {
                done = true;
                break;
            }
            if (WAIT && filled == a.batch) {              // more tiles than LDS holds shares of
                if constexpr (SUMS)
                    if (odd) redo_rows<FMT, NB>(red, odd, first, filled);
                lds_barrier();
                for (int it = wave; it < filled; it += kWaves) {
                    float4_t v = red[it * kWaves * 64 + at_lane];
#pragma unroll 1
                    for (int w = 1; w < kWaves; ++w) v += red[(it * kWaves + w) * 64 + at_lane];
                    sums[(first + it) * 64 + lane] = v;
                }
                lds_barrier();
                first += filled, filled = 0;
            }
            if (NB > 1 && filled == a.batch) {            // (partial rows only: the launcher sees to it)
                if constexpr (SUMS)
                    if (odd) redo_rows<FMT, NB>(red, odd, first, filled);
                lds_barrier();
                flush(first, filled);
                lds_barrier();
                first += filled, filled = 0;
            }
        }
        if (done) break;
    }
    if constexpr (SUMS)
        if (odd) redo_rows<FMT, NB>(red, odd, first, filled);
    lds_barrier();
    finish(first, filled);
}

// ---- host side ------------------------------------------------------------------------------------------------------
struct Plan {
    int kg, rg, uw, tiles;
};

// row tiles in flight (packed formats: 8 registers and 1 KB per unit), and units of a tile: the whole tile but where registers are short
template <int FMT, int NB, int UW>
constexpr int tiles_in_flight()
{
    return UW == 1 ? 2 : 1;
}
template <int FMT, int NB, int UW>
constexpr int units_in_flight()
{
    if (FMT == F_F16) return UW >= 6 ? 2 : UW % 2 == 0 && UW * NB >= 6 ? UW / 2 : UW;
    return UW == 6 ? 2 : UW;
}

template <int FMT, int NB, int UW, bool WAIT = false>
hipError_t launch_one(const Args &a, size_t lds_bytes, bool wait, hipStream_t stream)
{
    if constexpr (sums_wait(FMT, NB, UW) && !WAIT)
        if (wait) return launch_one<FMT, NB, UW, true>(a, lds_bytes, wait, stream);
    constexpr int T = tiles_in_flight<FMT, NB, UW>(), D = units_in_flight<FMT, NB, UW>();
    static std::atomic<bool> attr_done{false};            // setting the attribute twice is harmless; the flag only has to be a defined read
    if (!attr_done.load()) {
        if (hipFuncSetAttribute((const void *)fewrow_kernel<FMT, NB, UW, T, D, WAIT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes) != hipSuccess)
            return hipErrorInvalidValue;
        attr_done.store(true);
    }
    hipLaunchKernelGGL((fewrow_kernel<FMT, NB, UW, T, D, WAIT>), dim3(a.kg * a.rg), dim3(kThreads), lds_bytes, stream, a);
    return hipGetLastError();
}

template <int FMT, int NB, int... UWS>
hipError_t launch_uw(int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream)
{
    hipError_t e = hipErrorInvalidValue;
    (void)((uw == UWS ? (e = launch_one<FMT, NB, UWS>(a, lds_bytes, wait, stream), true) : false) || ...);
    return e;
}

// units per wavefront the kernels are built for (registers: 32 NB per unit of x, fp16 16 NB; 8 resp. 16 per unit of weights in
// flight): {16 x rows, 32, 64}
template <int FMT>
hipError_t launch_nb(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream)
{
    if constexpr (FMT == F_F16) {
        if (nb == 1) return launch_uw<FMT, 1, 1, 2, 3, 4, 5, 6, 8>(uw, a, lds_bytes, wait, stream);
        return launch_uw<FMT, 2, 1, 2, 3, 4>(uw, a, lds_bytes, wait, stream);
    } else {
        if (nb == 1) return launch_uw<FMT, 1, 1, 2, 3, 4, 5, 6>(uw, a, lds_bytes, wait, stream);
        if (nb == 2) return launch_uw<FMT, 2, 1, 2, 3>(uw, a, lds_bytes, wait, stream);
        return launch_uw<FMT, 4, 1>(uw, a, lds_bytes, wait, stream);
    }
}

}  // namespace fewrow

}  // namespace relax
