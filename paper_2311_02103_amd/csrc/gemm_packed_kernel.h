// Tiled MFMA GEMM on packed 4-bit weights: out[i,r] = sum_c x[i,c] * (u(r,c) - 8) * s[r, c / group].  One source file per tile includes this.
//
// At large n the contraction is dense (Relax, Sec. 5.1: library-grade GEMM for batch sizes other than 1; Sec. 4.2: the decode stays
// fused into the matmul).  What bounds it on gfx950 is, in this order, the power the chip may draw, the issue slots of a wavefront and the
// bandwidth of the LDS and of the L2s, and the form follows from these (22016 x 4096 at n = 2048: 382 -> 320 us, 0.97 -> 1.15 PFLOP/s;
// 12288 x 4096 218 -> 185, 4096 x 11008 197 -> 163, 4096 x 4096 80 -> 67, 8192 x 28672 at 511 rows 267 -> 234, against eight wavefronts of
// 32 x 32 x 16 MFMAs with decoded weights in the LDS; both sides on one card, cards differ by 5 %):
//   - v_mfma_f32_16x16x32_f16, not 32x32x16: under the power limit a bare loop on 4-bit weights and normal x reaches 2010 TFLOP/s with
//     the one and 1630 with the other (both 2440 on zeros).
//   - One wavefront per SIMD with a tile of 64 x 256 (weight rows x rows of x; 256 accumulation registers), four of them along the weight rows:
//     no weight is decoded twice, and a block of 64 columns costs a wavefront 128 MFMAs and 290 other instructions, where an MFMA leaves
//     three issue slots.  (As eight wavefronts of 64 x 128 every weight was decoded twice and the vector instructions alone filled the issue
//     port: 343 us.)  Hence everything else is dealt out evenly behind the MFMAs, by hand.
//   - Weights go to LDS as they are, packed: 8 KB per 64 columns of 256 rows instead of 32 KB of decoded fp16, and are decoded in registers a
//     k step ahead of their MFMAs.  The decode merges nibbles into the mantissa of fp16 1024.0, removes the offset exactly (1024 + u - 1032,
//     (1024 + 16 u) / 16 - 72) and multiplies by the group scale: 13 packed-fp16 operations per 8 weights.
//   - Weights are fetched in ROUNDS of 256 columns, whole 128-byte lines of eight lanes each; a quarter of the next round per k block.
//     Fetched 32 bytes of a row per block, and their scales two bytes at a time, they touch a line per row each, and by the
//     next block the x tile has flushed the L1: 792 lines per block and 256 x 256 tile (256 of them x), 10.7 TB/s over the chip, and 541 lines at
//     13.4 TB/s, all that the L2s give, per 128 x 256 tile.  Now 400 and 325.
//   - A block's x fragments are read in four phases of half a k step, each under the MFMAs of the phase before, so that the four wavefronts'
//     reads (16 bytes per lane, 128 bytes a cycle) never queue.  One barrier per block, in front of the last phase.
//   - For the gate/up matrix a tile is half gate rows, half the matching up rows and a wavefront owns matching fragments of both, so SwiGLU is
//     an element-wise epilogue on the accumulators.
//   - n, m need not be multiples of the tile: rows are clamped on load and masked on store.  k must be a multiple of 128.
#pragma once

#include <type_traits>
#include <utility>

#include "gemm_tile.h"

namespace relax {

namespace packed {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef uint32_t uint4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int BK = kTileK;
constexpr int kXPitch = 2 * BK;          // bytes of a row of the x tile: 64 columns of a block, swizzled
constexpr int kWPitch = 128 + 16;        // ... and of the weight tile: 256 columns of a round

// The vector operations of the main loop, in asm so that they stay in the issue slots behind the MFMAs where they are written: left to the
// compiler they gather in front of their uses, four or five in a slot that holds three.
//
// Pair p (0..3) of a packed word (8 codes, elements 0..7): elements p and p + 4, so that the four pairs of a word are the packet
// [e0 e4 e1 e5 e2 e6 e3 e7] (pairs 2 and 3: of the word shifted by 8).  Merged into the mantissas of fp16 1024 (1024 + u, odd pairs
// 1024 + 16 u), then the offset and the 16 removed, exactly, then times the group's scale (in the lower half of s).
// (mask from a scalar register, bits from a vector register: the encoding takes no literal and only one scalar source)
__device__ __forceinline__ uint32_t q4_merge(uint32_t w, int p)
{
    uint32_t r;
    asm volatile("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(p % 2 == 0 ? 0x000F000Fu : 0x00F000F0u), "v"(0x64006400u));
    return r;
}
__device__ __forceinline__ uint32_t q4_offset(uint32_t v, int p)
{
    uint32_t r;
    if (p % 2 == 0) asm volatile("v_pk_add_f16 %0, %1, %2" : "=v"(r) : "v"(v), "s"(0xE408E408u));                              // - 1032
    else asm volatile("v_pk_fma_f16 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(0x2C002C00u), "v"(0xD480D480u));                   // / 16 - 72
    return r;
}
__device__ __forceinline__ uint32_t q4_scale(uint32_t v, uint32_t s)
{
    uint32_t r;
    asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel_hi:[1,0]" : "=v"(r) : "v"(v), "v"(s));
    return r;
}
__device__ __forceinline__ uint32_t shift8(uint32_t w)
{
    uint32_t r;
    asm volatile("v_lshrrev_b32 %0, 8, %1" : "=v"(r) : "v"(w));
    return r;
}
__device__ __forceinline__ uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    uint32_t r;
    asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(r) : "v"(hi), "v"(lo), "s"(sel));
    return r;
}

// fp16(a x + c), x fp16, rounded once: what the compiler makes of the sums of products in rope_append_kernel, whose second product it rounds.  Left
// to contract here, it fuses the other product of the second sum, and results differ in the last place now and then.
__device__ __forceinline__ uint16_t fma_to_half(float a, uint16_t x, float c)
{
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[0,1,0]" : "=v"(r) : "v"(a), "v"((uint32_t)x), "v"(c));
    return (uint16_t)r;
}

// eight bytes at the alignment of a scale
struct __attribute__((packed, aligned(2))) Load8 { uint32_t lo, hi; };

// acc += A B on v_mfma_f32_16x16x32_f16, in place in the accumulation registers.  The builtin leaves result and addend free to differ,
// and with an accumulator in every register of that half of the file the allocator moved them about (1000 moves per 256 MFMAs).  What the
// compiler would see to for a builtin: an operand must not be written by a vector operation in the two issue slots before (the decode of a k step ends
// two MFMAs before it; the build checks the distances in the listing), and the accumulators must not be read before the pipe has drained, nor multiplied into right behind their
// initialisation (settle: in front of the first MFMA and behind the last one).
__device__ __forceinline__ void mfma(float4_t &acc, const uint4_t &a, const half8_t &b)
{
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// one wait for all fragments of a phase, not one per MFMA
__device__ __forceinline__ void arrived(half8_t (&b)[2]) { asm volatile("" ::"v"(b[0]), "v"(b[1])); }
__device__ __forceinline__ void arrived(half8_t (&b)[4]) { asm volatile("" ::"v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3])); }
__device__ __forceinline__ void arrived(half8_t (&b)[6]) { asm volatile("" ::"v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5])); }
__device__ __forceinline__ void arrived(half8_t (&b)[8])
{
    asm volatile("" ::"v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]), "v"(b[6]), "v"(b[7]));
}
template <int MF, int NF>
__device__ __forceinline__ void settle(float4_t (&acc)[MF][NF])
{
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int j = 0; j < NF; ++j) asm volatile("" : "+a"(acc[f][j]));       // every write is in front of the wait, every read behind it
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int j = 0; j < NF; ++j) asm volatile("" : "+a"(acc[f][j]));
}

template <int I>
using Int = std::integral_constant<int, I>;
// f(Int<0>), f(Int<1>), ... in order: indexes known to the compiler whatever the length
template <typename Fn, int... I>
__device__ __forceinline__ void each(Fn &&f, std::integer_sequence<int, I...>)
{
    (f(Int<I>{}), ...);
}

// One-dimensional grid of tiles_m * tiles_n * splits workgroups of four wavefronts along the weight rows, each with MF fragments of 16 weight
// rows and NF fragments of 16 x rows.
constexpr int WM = 4;
template <int EPI, int MF, int NF>
__global__ __launch_bounds__(WM * 64) void gemm_packed_kernel(GemmArgs a)
{
    constexpr int T = WM * 64, BM = 16 * MF * WM, BN = 16 * NF;
    constexpr int KW = 2 * BM / T;                        // pieces of codes a thread stages per k block, pieces of scales per round
    constexpr int kRows = T / 8;                          // weight rows of T pieces of codes
    static_assert(KW >= 1 && KW <= 2 && KW * T == 2 * BM, "staging roles");
    constexpr int XP = BN * 8 / T;                        // 16-byte packets of x a thread stages per block
    constexpr int NH = NF / 2;                            // x fragments of a phase: half of a k step's
    constexpr int PH = MF * NH;                           // MFMAs of a phase, four phases a block
    static_assert(2 * PH - PH / 2 - 3 > 0 && NF % 2 == 0 && XP >= 1 && 3 * PH / XP >= 5, "staging roles");
    // k blocks between a load and its way to LDS.  A block of the 64-column tile is shorter than the way to memory, so a launch that leaves most of
    // the chip idle, as every call without a workspace at few rows does, waited for each of its loads: 4096 x 4096 at 65 rows 40.6 -> 26.3 us,
    // 2048 x 5632 at 17 rows 54.7 -> 33.7.  Wider tiles gain nothing, or lose on a full chip what they gain on long rows (128 columns: 5120 x 5120 at
    // 640 rows 44.9 against 46.4 us, 4096 x 11008 at 129 rows 101 against 84).
    constexpr int AHEAD = BN == 64 ? 2 : 1;
    // two buffers each of the x tile of a block, of the codes of a round and of its scales, one for every sub-group of 32 columns
    constexpr uint32_t kXBuf = BN * kXPitch, kWBuf = BM * kWPitch, kSBuf = BM * 16;
    constexpr uint32_t kWs = 2 * kXBuf, kSs = kWs + 2 * kWBuf;
    __shared__ __align__(16) char lds[kSs + 2 * kSBuf];

    const int tid = threadIdx.x, lane = tid & 63, wm = tid >> 6;
    const int row16 = lane & 15, quarter = lane >> 4;
    // Workgroups are handed to the 8 XCDs round-robin by linear id, and each XCD has its own L2.  Renumber them so
    // that an XCD owns a contiguous run of tiles: the x tiles a workgroup streams are then fetched into one L2 instead of eight.
    const int nb = gridDim.x, xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int tile = xcd * (nb >> 3) + min(xcd, nb & 7) + idx;
    // Inside an XCD's run the x-row tile changes fastest within a PAIR of x-row tiles: a round of 32 workgroups then is 16
    // weight-row tiles x 2 x-row tiles, and an XCD streams half of the weight matrix instead of all of it (requests of the L2s
    // to the fabric on the 7B gate/up shape at n = 2048: 324 MB; the kernel before this one 304 MB, without the pairs 456; neither operand
    // fits a 4 MB L2).
    const int per_split = a.tiles_m * a.tiles_n, split = tile / per_split, t2 = tile - split * per_split;
    const int pair = t2 / (2 * a.tiles_m), r2 = t2 - pair * 2 * a.tiles_m;
    const bool whole = 2 * pair + 1 < a.tiles_n;          // the last pair of an odd count is a single tile
    const int tile_m = whole ? r2 >> 1 : r2, tile_n = whole ? 2 * pair + (r2 & 1) : 2 * pair;
    const int n0 = tile_n * BN;
    const int F = a.m >> 1;
    const int ldm = a.ldm > 0 ? a.ldm : a.m;
    const int kb0 = split * a.kb_per_split;               // this workgroup's k range: blocks kb0 .. kb0 + nkb - 1, an even number
    const int nkb = min(a.kb_per_split, a.k / BK - kb0);

    // ---- staging roles.  Rows of the weight tile: matrix rows from row0 on, or (EPI_SWIGLU) half of them gate rows from row0 on and
    // half the matching up rows F + row0 ..; clamped to the matrix.  A thread stages piece tid % 8 of row tid / 8 of each quarter.  Offsets
    // are counted from the tile's first row (the matrix may hold more bytes than 32 bits count). ----
    const int row0 = EPI == EPI_SWIGLU ? tile_m * (BM / 2) : tile_m * BM;
    const int last_row = min((EPI == EPI_SWIGLU ? F : a.m) - row0, EPI == EPI_SWIGLU ? BM / 2 : BM) - 1;
    const uint32_t row_bytes = (uint32_t)a.k >> 1;
    const uint32_t piece16 = (tid & 7) * 16, woff0 = (uint32_t)(tid >> 3) * row_bytes, last_off = (uint32_t)last_row * row_bytes;
    const char *const wbase = (const char *)a.q + (size_t)row0 * row_bytes;
    const int nsc = scales_per_row(a.k, a.gshift);
    const int sub0 = kb0 * (BK / 32);                     // first sub-group of this workgroup's k range
    auto load_w = [&](int u, int h) {                     // share h of quarter u & 3 of round u >> 2; clamped to the row: a short last round re-reads the row's end (never consumed)
        const uint32_t col = min((uint32_t)sub0 * 16 + (uint32_t)(u >> 2) * 128 + piece16, row_bytes - 16);
        int first = ((u & 3) * KW + h) * kRows;
        const char *base = wbase;
        if (EPI == EPI_SWIGLU && first >= BM / 2) base += (size_t)F * row_bytes, first -= BM / 2;
        return *(const uint4 *)(base + (min(woff0 + (uint32_t)first * row_bytes, last_off) + col));
    };
    // LDS addresses; those of the weights move to the other buffer from round to round
    uint32_t wst = kWs + (tid >> 3) * kWPitch + piece16;
    int wst_step = kWBuf;
    auto store_w = [&](const uint4 &v, int u, int h) { *(uint4 *)(lds + wst + ((u & 3) * KW + h) * (kRows * kWPitch)) = v; };
    // Scales of a round: eight bytes of a row per thread, from the scale of sub-group 4 (tid % 2) on, stored once per sub-group (a wider
    // group's scale twice or four times).  Where eight bytes would pass the end of the matrix they are read further in front and shifted into place.
    uint32_t sat0[KW];
#pragma unroll
    for (int h = 0; h < KW; ++h) {
        const int srow = (tid + h * T) >> 1;
        sat0[h] = (uint32_t)(EPI == EPI_SWIGLU && srow >= BM / 2 ? F + min(srow - BM / 2, last_row) : min(srow, last_row)) * nsc +
                  ((sub0 + 4 * (tid & 1)) >> a.gshift);
    }
    const uint16_t *const sbase = a.s + (size_t)row0 * nsc;
    const uint32_t last_s = (uint32_t)min((int64_t)(a.m - row0) * nsc - 4, (int64_t)1 << 30);
    const uint32_t sel_lo = a.gshift == 0 ? 0x03020100u : 0x01000100u, sel_hi = a.gshift == 0 ? 0x07060504u : a.gshift == 1 ? 0x03020302u : 0x01000100u;
    auto load_s = [&](int round, int h) {
        const uint32_t from = min(sat0[h] + ((8 * round) >> a.gshift), last_s);
        const Load8 v = *(const Load8 *)((const char *)sbase + 2 * from);
        return ((uint64_t)v.hi << 32) | v.lo;
    };
    const uint32_t sst = kSs + tid * 8;
    auto store_s = [&](uint64_t v, int round, int h) {    // (the shift belongs here: next to the load it would wait for it)
        const uint32_t at = sat0[h] + ((8 * round) >> a.gshift);
        v >>= 16 * min(at - min(at, last_s), 3u);
        const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
        *(uint2 *)(lds + sst + (round & 1) * kSBuf + h * T * 8) = make_uint2(__builtin_amdgcn_perm(hi, lo, sel_lo), __builtin_amdgcn_perm(hi, lo, sel_hi));
    };
    uint32_t xoff[XP];
    const char *const xbase = (const char *)(a.x + (size_t)n0 * a.k + (size_t)kb0 * BK);
#pragma unroll
    for (int p = 0; p < XP; ++p) {
        const int pk = tid + p * T;
        xoff[p] = (uint32_t)min(pk >> 3, a.n - 1 - n0) * (uint32_t)(2 * a.k) + (pk & 7) * 16;
    }
    auto load_x = [&](int kb, int p) {
        asm volatile("" : "+v"(xoff[p]));                 // keeps the address a scalar base and this offset: no 64-bit pointer per packet
        return *(const uint4_t *)(xbase + (size_t)min(kb, nkb - 1) * (2 * BK) + xoff[p]);
    };
    // Packet c of row r sits at slot (c / 2 + 4 (c % 2)) ^ ((r / 2) % 8): packets 2 q and 2 q + 1 are what quarter q of the lanes reads, for one k
    // step each, and the sixteen lanes that a 16-byte read serves at a time (rows 0..3 and 12..15 of one quarter, 4..11 of its neighbour) hit distinct banks.
    const uint32_t xst = (tid >> 3) * kXPitch + ((((tid & 7) >> 1) + 4 * (tid & 1)) ^ ((tid >> 4) & 7)) * 16;
    // [x0 x1 | x2 x3 | x4 x5 | x6 x7] -> [x0 x4 | x1 x5 | x2 x6 | x3 x7], a word at a time
    auto pack_x = [](uint4_t &o, const uint4_t &v, int i) {
        o[i] = byte_perm(v[2 + i / 2], v[i / 2], i % 2 == 0 ? 0x05040100u : 0x07060302u);
    };
    auto store_x = [&](const uint4_t &o, int buf, int p) { *(uint4_t *)(lds + xst + buf * kXBuf + p * (T / 8) * kXPitch) = o; };
    // LDS-only workgroup barrier: the global loads of later k blocks stay in flight across it
    auto lds_barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    // ---- MFMA roles.  Quarter q of the lanes holds columns 16 q .. 16 q + 15 of a block: eight for each of its two k steps ----
    // Fragment f: rows (wm MF + f) 16 .. of the tile.  EPI_SWIGLU: half of the fragments in the gate half, half in the up half.  EPI_ROPE_KV:
    // half of them in the lower half of a head of 128 rows, half in its upper half, so that a lane holds both values of a rotation.
    constexpr int W2 = MF / 2 * 16;                       // rows of a wavefront in either half
    const int wrow = EPI == EPI_SWIGLU ? wm * W2 : EPI == EPI_ROPE_KV ? wm * W2 / 64 * 128 + wm * W2 % 64 : wm * MF * 16;
    const int arow = wrow + row16;
    auto frag_row = [](int f) {
        return EPI == EPI_SWIGLU ? f / (MF / 2) * (BM / 2) + f % (MF / 2) * 16 : EPI == EPI_ROPE_KV ? f / (MF / 2) * 64 + f % (MF / 2) * 16 : f * 16;
    };
    uint32_t wrd = kWs + arow * kWPitch + quarter * 8, srd = kSs + arow * 16 + (quarter >> 1) * 2;
    int wrd_step = kWBuf, srd_step = kSBuf;
    uint32_t xrd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) xrd[ks] = row16 * kXPitch + ((quarter + 4 * ks) ^ (row16 >> 1)) * 16;

    float4_t acc[MF][NF];
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[f][j] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // Registers of the pipeline: codes and scales of a block, the weight fragments of two k steps, the x fragments of two phases, and what
    // is on its way to LDS.
    uint32_t raw[MF][2], sc[MF];
    uint4_t af[2][MF];
    half8_t bf[2][NH];
    uint4_t xr[AHEAD][XP];
    uint4 wr[AHEAD][KW];
    uint64_t sr[KW];

    auto read_raw = [&](int j, int f) {                   // block j of the round that wrd and srd stand at
        const uint2 v = *(const uint2 *)(lds + wrd + frag_row(f) * kWPitch + j * 32);
        raw[f][0] = v.x, raw[f][1] = v.y;
        sc[f] = *(const uint16_t *)(lds + srd + frag_row(f) * 16 + j * 4);
    };
    // one of the three operations that decode pair d % 4 of fragment d / 4
    auto decode = [&](int ks, int d, int stage) {
        const int f = d / 4, p = d % 4;
        uint32_t v = af[ks][f][p];
        if (stage == 0 && p == 2) raw[f][ks] = shift8(raw[f][ks]);
        if (stage == 0) v = q4_merge(raw[f][ks], p);
        else if (stage == 1) v = q4_offset(v, p);
        else v = q4_scale(v, sc[f]);
        af[ks][f][p] = v;
    };
    auto read_b = [&](int set, int buf, int ks, int i) { bf[set][i] = *(const half8_t *)(lds + xrd[ks] + buf * kXBuf + (set * NH + i) * 16 * kXPitch); };

    // Block kb = 4 r + j: MFMAs on x buffer j & 1, while x of block kb + 1 and the quarter of the weights that is five ahead go to LDS and
    // their successors are requested.  A phase is half of the x fragments of a k step against all weight fragments; the next phase's are read
    // under it, evenly, as are all other steps: behind an MFMA a wavefront has three issue slots until the pipe takes the next.
    auto block = [&](auto jc, int r) {
        constexpr int j = decltype(jc)::value, buf = j & 1, set = (j + 1) % AHEAD;
        const int kb = 4 * r + j;
        uint4_t packed = {};
        each([&](auto slot) {
            constexpr int at = decltype(slot)::value, phase = at / PH, ks = phase / 2, h = phase % 2, f = at % PH / NH, i = at % NH;
            if (at == 3 * PH) lds_barrier();              // in front of the last phase, which reads the first x fragments of the next block
            if (at % PH == 0) arrived(bf[h]);
            mfma(acc[f][h * NH + i], af[ks][f], bf[h][i]);

            // (all in the first three quarters of the phase, so that they are there when it ends)
            each([&](auto ic) {
                constexpr int i2 = decltype(ic)::value;
                if constexpr (at % PH == i2 * 3 * MF / 4) read_b(h ^ 1, phase == 3 ? buf ^ 1 : buf, phase == 3 ? 0 : (phase + 1) / 2, i2);
            }, std::make_integer_sequence<int, NH>{});
            if (phase == 2 && at % PH < MF) {             // the second k step's fragments are decoded: the codes of the next block
                if (at % PH == 0 && j == 3) wrd += wrd_step, wrd_step = -wrd_step, srd += srd_step, srd_step = -srd_step;
                read_raw((j + 1) & 3, at % PH);
            }
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                if (at == PH / 2 + q) {
                    if (q == 0 && j == 3) wst += wst_step, wst_step = -wst_step;
                    store_w(wr[set][q], j + 1, q);
                    wr[set][q] = load_w(kb + 5 + AHEAD, q);
                }
                if (j == 0 && at == PH + 1 + q * PH / 2) sr[q] = load_s(r + 1, q);
                if (j == AHEAD && at == PH + 1 + q * PH / 2) store_s(sr[q], r + 1, q);
            }
#pragma unroll
            for (int p = 0; p < XP; ++p) {
                const int first = p * (3 * PH) / XP;
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    if (at == first + i4) pack_x(packed, xr[set][p], i4);
                if (at == first + 3) store_x(packed, buf ^ 1, p);
                if (at == first + 4) xr[set][p] = load_x(kb + 1 + AHEAD, p);
            }
            // k step 1 is decoded under k step 0; the next block's k step 0 under k step 1, from half a phase behind the reads of its codes on
            constexpr int D = 4 * MF, from = at < 2 * PH ? 0 : 2 * PH + PH / 2, span = at < 2 * PH ? 2 * PH - 3 : 2 * PH - PH / 2 - 3;
            each([&](auto sc) {                           // pair d: its operation `stage` at slot from + d span / D + stage
                constexpr int stage = 2 - decltype(sc)::value, pos = at - from - stage;
                constexpr int d0 = (pos * D + span - 1) / span, d1 = ((pos + 1) * D + span - 1) / span;
                if constexpr (pos >= 0 && d0 < D)
                    each([&](auto dc) { decode(at < 2 * PH ? 1 : 0, d0 + decltype(dc)::value, stage); }, std::make_integer_sequence<int, (d1 < D ? d1 : D) - d0>{});
            }, std::make_integer_sequence<int, 3>{});
            __builtin_amdgcn_sched_barrier(0);
        }, std::make_integer_sequence<int, 4 * PH>{});
#pragma unroll
        for (int f = 0; f < MF; ++f) asm volatile("" : "+v"(af[0][f]));      // decoded here, not where they are used
    };

    // ---- prologue: round 0, a quarter of round 1 and block 0 in LDS, the next quarter and block 1 on their way ----
    {
        uint4 w0[5][KW];
        uint4_t x0[XP];
#pragma unroll
        for (int u = 0; u < 5; ++u)
#pragma unroll
            for (int h = 0; h < KW; ++h) w0[u][h] = load_w(u, h);
#pragma unroll
        for (int h = 0; h < KW; ++h) sr[h] = load_s(0, h);
#pragma unroll
        for (int p = 0; p < XP; ++p) x0[p] = load_x(0, p);
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            if (u == 4) wst += wst_step, wst_step = -wst_step;
#pragma unroll
            for (int h = 0; h < KW; ++h) store_w(w0[u][h], u, h);
        }
#pragma unroll
        for (int h = 0; h < KW; ++h) store_s(sr[h], 0, h), wr[1 % AHEAD][h] = load_w(5, h);
#pragma unroll
        for (int p = 0; p < XP; ++p) {
            uint4_t o;
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) pack_x(o, x0[p], i4);
            store_x(o, 0, p);
            xr[1 % AHEAD][p] = load_x(1, p);
        }
        if constexpr (AHEAD > 1) {
#pragma unroll
            for (int h = 0; h < KW; ++h) wr[0][h] = load_w(6, h);
#pragma unroll
            for (int p = 0; p < XP; ++p) xr[0][p] = load_x(2, p);
        }
    }
    lds_barrier();
#pragma unroll
    for (int f = 0; f < MF; ++f) read_raw(0, f);
#pragma unroll
    for (int i = 0; i < NH; ++i) read_b(0, 0, 0, i);
#pragma unroll
    for (int d = 0; d < 4 * MF; ++d)
#pragma unroll
        for (int stage = 0; stage < 3; ++stage) decode(0, d, stage);
    settle(acc);
    const int rounds = nkb >> 2;
    for (int r = 0; r < rounds; ++r) {
        block(Int<0>{}, r);
        block(Int<1>{}, r);
        block(Int<2>{}, r);
        block(Int<3>{}, r);
    }
    if (nkb & 2) {
        block(Int<0>{}, rounds);
        block(Int<1>{}, rounds);
    }

    settle(acc);

    // ---- epilogue.  acc[f][j][v]: tile row of fragment f + 4 (lane / 16) + v, x row n0 + 16 j + lane % 16 ----
    const int off = quarter * 4;
    if (a.partial) {
        // k split: the raw fp32 tile goes to partial[split][x row][weight row] (gate rows first, up rows from F on, as in the
        // matrix), and the finishing pass adds the splits in order and applies the epilogue
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int xrow = n0 + j * 16 + row16;
            if (xrow >= a.n) continue;
            float *dst = a.partial + ((size_t)split * a.n + xrow) * a.m;
#pragma unroll
            for (int f = 0; f < MF; ++f) {
                int row;                                         // matrix row of this granule of four
                bool ok;
                if (EPI == EPI_SWIGLU) {
                    const int g = row0 + (wm * (MF / 2) + f % (MF / 2)) * 16 + off;
                    row = (f / (MF / 2)) * F + g, ok = g < F;
                } else {
                    row = row0 + (wm * MF + f) * 16 + off, ok = row < a.m;
                }
                if (ok) *(float4 *)(dst + row) = make_float4(acc[f][j][0], acc[f][j][1], acc[f][j][2], acc[f][j][3]);
            }
        }
        return;
    }
    if constexpr (EPI == EPI_ROPE_KV) {
        // rotary embedding and KV append with the arithmetic of the kernel that does it alone (on values rounded to fp16): a layer call of the 7B
        // shape 275 -> 268 us with 300 prompt rows and 20 decode rows, 837.6 -> 834.9 at 2048 rows, where the pieces of 32 bytes that a
        // quarter of the lanes writes cost most of what the separate launch did.  Position and slot of the tile's x rows are looked up once, a thread per row.
        int2 *const rows = (int2 *)lds;
        __syncthreads();
        for (int t = tid; t < BN; t += T) {
            const RowInfo ri = row_info(a.seqs, min(n0 + t, a.n - 1));
            rows[t] = make_int2(ri.pos, ri.slot);
        }
        __syncthreads();
        const int head = (a.first_row + row0 + wrow) >> 7, t0 = (wrow & 127) + off;
        if (head >= a.h + 2 * a.g) return;
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int local = j * 16 + row16, xrow = n0 + local;
            if (xrow >= a.n) continue;
            const int2 at = rows[local];
            const size_t token = (size_t)at.y * a.kv_capacity + at.x;
            uint16_t *dst = head < a.h ? a.out_f16 + (size_t)xrow * ldm + (row0 + wrow) / 128 * 128
                                       : head < a.h + a.g ? a.kcache + (token * a.g + head - a.h) * 128 : a.vcache + (token * a.g + head - a.h - a.g) * 128;
#pragma unroll
            for (int f = 0; f < MF / 2; ++f) {
                const int t = t0 + f * 16;
                uint16_t lo[4], hi[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) lo[v] = f2h(acc[f][j][v]), hi[v] = f2h(acc[f + MF / 2][j][v]);
                if (head < a.h + a.g) {
                    const float4 cs[2] = {*(const float4 *)(a.rope + ((size_t)at.x * 64 + t) * 2), *(const float4 *)(a.rope + ((size_t)at.x * 64 + t + 2) * 2)};
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float x1 = h2f(hi[v]), co = v % 2 ? cs[v / 2].z : cs[v / 2].x, si = v % 2 ? cs[v / 2].w : cs[v / 2].y;
                        hi[v] = fma_to_half(si, lo[v], co * x1), lo[v] = fma_to_half(co, lo[v], -(si * x1));
                    }
                }
                *(uint2 *)(dst + t) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
                *(uint2 *)(dst + 64 + t) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int xrow = n0 + j * 16 + row16;
        if (xrow >= a.n) continue;
        if (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int f = 0; f < MF / 2; ++f) {
                const int g = row0 + (wm * (MF / 2) + f) * 16 + off;
                if (g < F) {                                     // F % 4 == 0 is checked by the launcher
                    uint16_t o[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float gte = acc[f][j][r], up = acc[f + MF / 2][j][r];
                        o[r] = f2h(gte / (1.0f + __expf(-gte)) * up);
                    }
                    *(uint2 *)(a.out_f16 + (size_t)xrow * F + g) = make_uint2(o[0] | ((uint32_t)o[1] << 16), o[2] | ((uint32_t)o[3] << 16));
                }
            }
        } else {
#pragma unroll
            for (int f = 0; f < MF; ++f) {
                const int r0 = row0 + (wm * MF + f) * 16 + off;
                if (r0 < a.m) {                                  // m % 4 == 0 is checked by the launcher
                    const size_t at = (size_t)xrow * ldm + r0;
                    float v[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[f][j][r];
                    if (EPI == EPI_RESID_F32) {
                        const uint2 xx = *(const uint2 *)((const uint16_t *)a.resid + at);
                        float4 o;
                        o.x = h2f((uint16_t)(xx.x & 0xFFFFu)) + v[0], o.y = h2f((uint16_t)(xx.x >> 16)) + v[1];
                        o.z = h2f((uint16_t)(xx.y & 0xFFFFu)) + v[2], o.w = h2f((uint16_t)(xx.y >> 16)) + v[3];
                        *(float4 *)(a.out_f32 + at) = o;
                    } else {
                        if (EPI == EPI_RESID_F16) {
                            const float4 rr = *(const float4 *)((const float *)a.resid + at);
                            v[0] += rr.x, v[1] += rr.y, v[2] += rr.z, v[3] += rr.w;
                        }
                        *(uint2 *)(a.out_f16 + at) = make_uint2(f2h(v[0]) | ((uint32_t)f2h(v[1]) << 16), f2h(v[2]) | ((uint32_t)f2h(v[3]) << 16));
                    }
                }
            }
        }
    }
}

// a launcher of gemm_tile.h for this tile
template <int MF, int NF>
hipError_t launch_packed(const GemmArgs &a_in, int splits, hipStream_t stream)
{
    GemmArgs a = a_in;
    const dim3 grid(gemm_tile_grid(a, 16 * MF * WM, 16 * NF, splits)), block(WM * 64);
    switch (a.epi) {
    case EPI_F16: hipLaunchKernelGGL((gemm_packed_kernel<EPI_F16, MF, NF>), grid, block, 0, stream, a); break;
    case EPI_ROPE_KV: hipLaunchKernelGGL((gemm_packed_kernel<EPI_ROPE_KV, MF, NF>), grid, block, 0, stream, a); break;
    case EPI_RESID_F32: hipLaunchKernelGGL((gemm_packed_kernel<EPI_RESID_F32, MF, NF>), grid, block, 0, stream, a); break;
    case EPI_RESID_F16: hipLaunchKernelGGL((gemm_packed_kernel<EPI_RESID_F16, MF, NF>), grid, block, 0, stream, a); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((gemm_packed_kernel<EPI_SWIGLU, MF, NF>), grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace packed

}  // namespace relax
