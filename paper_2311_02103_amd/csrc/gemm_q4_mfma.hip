// Tiled MFMA GEMM on native 3-bit and on plain fp16 weights for large n (prefill), out[i,r] = sum_c x[i,c] * W(r,c), and the tile plan of
// these and of the 4-bit kernel (gemm_packed_kernel.h).
//
//   - v_mfma_f32_32x32x16_f16, fp32 accumulate.  The 256-row tiles (weight rows x x-rows) run as eight wavefronts,
//     two per SIMD with up to 256 registers each, so that one wavefront's decode, LDS
//     traffic and waits run under the other's MFMAs; the narrower tiles and the fp16-weight variant run as four
//     wavefronts (2 x 2), one per SIMD (128 x 256 as eight wavefronts of 64 x 64 was measured 4 to 11 % slower than as
//     four of 64 x 128: twice the fragment reads per MFMA).
//   - Both operands go through LDS in 64-wide k blocks, double buffered with ONE LDS-only barrier per block
//     (global loads of the next block stay in flight across it).  3-bit weights are decoded on the way in,
//     once per workgroup: every thread loads its share of the codes and the group scale of one weight row, turns
//     them into fp16 values and writes them to LDS.  A quarter of a block's loads, decode and LDS writes is placed next to the
//     MFMAs of each of its four k steps.
//   - Rows are padded to 144 bytes: 16-byte reads and writes of consecutive rows hit distinct banks.  fp16 weights and their x tile keep
//     the packet order [e0 e4 e1 e5 e2 e6 e3 e7] (the order of k inside an MFMA is free as long as A and B agree); 3-bit ones the natural order.
//   - n, m need not be multiples of the tile: rows are clamped on load and masked on store (one binary for
//     every n: 17, 511, 2048 ...).  k must be a multiple of 128 (else the matvec path serves the call).
#include <atomic>
#include <iterator>

#include "gemm_tile.h"

namespace relax {

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int BK = 64;                  // k per main-loop step
constexpr int kPitch = BK + 8;          // LDS row pitch in halfs (144 bytes)

__device__ __forceinline__ uint32_t pk_mul(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, a) * __builtin_bit_cast(half2_t, b));
}
__device__ __forceinline__ uint32_t pk_fma(uint32_t a, uint32_t b, uint32_t c)
{
    half2_t r = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b), __builtin_bit_cast(half2_t, c));
    return __builtin_bit_cast(uint32_t, r);
}

// (w & mask) | bits as one VALU op (mask from a scalar register, bits from a vector register: the encoding
// takes no literal and only one scalar source)
__device__ __forceinline__ uint32_t and_or(uint32_t w, uint32_t mask, uint32_t bits)
{
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(mask), "v"(bits));
    return r;
}

// 3-bit weights in the native word layout (three words per group of 32 columns: word w, position j holds column 2(5w+j)
// in bits 3j.. and column 2(5w+j)+1 in bits 16+3j..; bit i of columns 30 / 31 is bit 15 / 31 of word i): the four fp16 pairs
// of packet t (columns 8t .. 8t+7 of the group, NATURAL order) times the group scale.  v_and_or_b32 merges a pair of codes
// into the mantissas of fp16 (1024, 1024) at weight 1, 8 or 64; one packed fma removes offset and weight exactly
// ((1024 + f u) / f - (1024 / f + 4) = u - 4), one packed multiply applies the scale.
__device__ __forceinline__ half8_t decode_q3_packet(uint32_t w0, uint32_t w1, uint32_t w2, int t, uint32_t s2)
{
    const uint32_t base = 0x64006400u;
    const uint32_t kOne = 0x3C003C00u, kEighth = 0x30003000u, k64th = 0x24002400u;          // 1, 1/8, 1/64
    const uint32_t kNeg1028 = 0xE404E404u, kNeg132 = 0xD820D820u, kNeg20 = 0xCD00CD00u;     // -(1024 / f + 4)
    uint32_t r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int p = 4 * t + q;                              // pair p = columns 2p, 2p + 1
        uint32_t pair;
        int cls;                                              // 0: weight 1, 1: weight 8, 2: weight 64
        if (p == 15) {
            uint32_t g = and_or(w0 >> 15, 0x00010001u, base);
            g = and_or(w1 >> 14, 0x00020002u, g);
            pair = and_or(w2 >> 13, 0x00040004u, g), cls = 0;
        } else {
            const uint32_t w = p / 5 == 0 ? w0 : p / 5 == 1 ? w1 : w2;
            const int j = p % 5;
            const uint32_t v = j >= 3 ? w >> 9 : w;
            cls = j >= 3 ? j - 3 : j;
            pair = and_or(v, cls == 0 ? 0x00070007u : cls == 1 ? 0x00380038u : 0x01C001C0u, base);
        }
        const uint32_t scaled = cls == 0 ? pk_fma(pair, kOne, kNeg1028) : cls == 1 ? pk_fma(pair, kEighth, kNeg132) : pk_fma(pair, k64th, kNeg20);
        r[q] = pk_mul(scaled, s2);
    }
    uint4 o = {r[0], r[1], r[2], r[3]};
    return __builtin_bit_cast(half8_t, o);
}

// One-dimensional grid of tiles_m * (x-row tiles) workgroups.  Wavefront w owns MF fragments of 32 weight rows (w % WM picks which)
// and NF fragments of 32 x-rows (w / WM picks which) of the workgroup tile of 32 MF WM weight rows x 32 NF WN x-rows.
// FP16W: plain fp16 weights (the fp16-weight configurations of the paper's LLM charts, Sec. 5.1): the staging copies 16-byte packets.
// Otherwise 3-bit weights in the native word layout (Sec. 5.3 of the paper deploys 3-bit models): a thread stages a whole group of 32
// columns (three words), the decode yields the columns in natural order, so the x tile is staged unpermuted.
// WM = 2: four wavefronts, one per SIMD, each with up to 512 registers.  WM = 4: eight wavefronts, two per SIMD with up to 256 registers each.
template <int NF, bool FP16W, int WM = 2>
__global__ __launch_bounds__(WM * 128) void gemm_mfma_kernel(GemmArgs a)
{
    constexpr bool Q3 = !FP16W;
    constexpr int MF = 2, WN = 2;
    constexpr int ST = 2;                                 // register stages; four were measured and gained nothing
    constexpr int kThreadsG = WM * WN * 64;
    constexpr int BM = 32 * MF * WM, BN = 32 * NF * WN;
    // packets of 8 columns a thread stages per k block: its share of the BM x 8 of the weight tile (every thread stages weights, so
    // the staging has no branch for the compiler's wait-count pass to merge across)
    constexpr int W = 4, TPR = 8 / W;                     // ... and threads per weight row
    static_assert(W * kThreadsG == BM * 8, "staging roles");
    constexpr int XP = BN * 8 / kThreadsG;                // 16-byte x packets a thread stages per k block
    constexpr int kABuf = BM * kPitch, kBBuf = BN * kPitch;
    extern __shared__ __align__(16) uint16_t lds[];       // A[2][BM][kPitch], B[2][BN][kPitch]
    uint16_t *const As = lds, *const Bs = lds + 2 * kABuf;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row32 = lane & 31, hf = lane >> 5;
    const int wm = wave % WM, wn = wave / WM;
    // Workgroups are handed to the 8 XCDs round-robin by linear id, and each XCD has its own L2.  Renumber them so
    // that an XCD owns a contiguous run of tiles: the x tiles a workgroup streams are then fetched into one L2 instead of eight.
    const int nb = gridDim.x, xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int tile = xcd * (nb >> 3) + min(xcd, nb & 7) + idx;
    // Inside an XCD's run the x-row tile changes fastest within a PAIR of x-row tiles: a round of 32 workgroups then is 16
    // weight-row tiles x 2 x-row tiles, and an XCD streams half of the weight matrix instead of all of it (requests of the L2s
    // to the fabric on the 7B gate/up shape at n = 2048: 304 MB against 456 MB; neither operand fits a 4 MB L2).
    const int per_split = a.tiles_m * a.tiles_n, split = tile / per_split, t2 = tile - split * per_split;
    const int pair = t2 / (2 * a.tiles_m), r2 = t2 - pair * 2 * a.tiles_m;
    const bool whole = 2 * pair + 1 < a.tiles_n;          // the last pair of an odd count is a single tile
    const int tile_m = whole ? r2 >> 1 : r2, tile_n = whole ? 2 * pair + (r2 & 1) : 2 * pair;
    const int n0 = tile_n * BN;

    // ---- staging roles ----
    const int arow = tid / TPR, apart = tid % TPR, acol0 = apart * W * 8;
    const int grow = min(tile_m * BM + arow, a.m - 1);
    const uint32_t *qsrc = FP16W ? nullptr : a.q + ((size_t)grow * (a.k >> 5) + apart) * 3;
    const uint16_t *ssrc = FP16W ? nullptr : a.s + (size_t)grow * scales_per_row(a.k, a.gshift);
    const uint16_t *hsrc = FP16W ? a.wh + (size_t)grow * a.k + acol0 : nullptr;
    const uint16_t *xsrc[XP];
#pragma unroll
    for (int p = 0; p < XP; ++p) {
        const int pk = tid + p * kThreadsG;
        xsrc[p] = a.x + (size_t)min(n0 + (pk >> 3), a.n - 1) * a.k + (pk & 7) * 8;
    }

    // Staged registers of one k block: packed codes + scales of this thread's weight row part, and its x packets.
    struct Stage {
        uint4 wq[FP16W ? W : 1];                          // 16-byte packets of fp16 weights, or the three words of a 3-bit group
        uint32_t wsc;
        uint4 xr[XP];
    };
    const int kb0 = split * a.kb_per_split;               // this workgroup's k range: blocks kb0 .. kb0 + nkb - 1
    const int nkb = min(a.kb_per_split, a.k / BK - kb0);
    // The loads of k block kb, in four shares: share `part` is issued next to k step `part` of the running block -- a
    // workgroup that issued all its loads in one burst at the top of a block filled the address queue of the texture unit and
    // stalled in front of its own MFMAs.  Loads return in order, so the order of issue is what the wait counts stand on:
    // weights first (the decode of share 0 needs them first), then per share the x packets.
    auto stage_load = [&](Stage &S, int kb, int part) {   // kb is clamped: the tail re-reads the last block (never consumed)
        kb = kb0 + min(kb, nkb - 1);
        if (FP16W) {
#pragma unroll
            for (int i = 0; i < W; ++i)
                if (i == part) S.wq[i] = *(const uint4 *)(hsrc + kb * BK + i * 8);
        } else {
            if (part == 0) {
                const uint32_t *g3 = qsrc + kb * (BK / 32) * 3;            // 4-byte aligned
                S.wq[0].x = g3[0], S.wq[0].y = g3[1], S.wq[0].z = g3[2];
            }
            if (part == 1) S.wsc = ssrc[(kb * (BK / 32) + apart) >> a.gshift];
        }
#pragma unroll
        for (int p = 0; p < XP; ++p)
            if (p * 4 / XP == part) S.xr[p] = *(const uint4 *)(xsrc[p] + kb * BK);
    };
    // a whole block's loads in the order the running loop issues them (prologue): the compiler's wait counts at the loop
    // head are the merge of this order and the loop's own, so the two must agree or every wait in the loop is pessimistic
    auto stage_load_all = [&](Stage &S, int kb) {
#pragma unroll
        for (int part = 0; part < 4; ++part) {
            stage_load(S, kb, part);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // quarter `part` (0..3) of the decode + LDS write of a staged block
    auto stage_store = [&](const Stage &S, int buf, int part) {
        uint16_t *ad = As + buf * kABuf + arow * kPitch + acol0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            if (i != part) continue;
            if (FP16W) {                                  // same packet order as the decode and the x tile
                const uint4 &h = S.wq[FP16W ? i : 0];
                uint4 o;
                o.x = __builtin_amdgcn_perm(h.z, h.x, 0x05040100u);
                o.y = __builtin_amdgcn_perm(h.z, h.x, 0x07060302u);
                o.z = __builtin_amdgcn_perm(h.w, h.y, 0x05040100u);
                o.w = __builtin_amdgcn_perm(h.w, h.y, 0x07060302u);
                *(uint4 *)(ad + i * 8) = o;
                continue;
            }
            const uint4 &wv = S.wq[0];
            *(half8_t *)(ad + i * 8) = decode_q3_packet(wv.x, wv.y, wv.z, i, S.wsc | (S.wsc << 16));
        }
        uint16_t *bd = Bs + buf * kBBuf;
#pragma unroll
        for (int p = 0; p < XP; ++p) {
            if (p * 4 / XP != part) continue;
            const int pk = tid + p * kThreadsG;
            // [x0 x1 | x2 x3 | x4 x5 | x6 x7] -> [x0 x4 | x1 x5 | x2 x6 | x3 x7]
            uint4 o = S.xr[p];                            // Q3: the decode yields natural order
            if (!Q3) {
                o.x = __builtin_amdgcn_perm(S.xr[p].z, S.xr[p].x, 0x05040100u);
                o.y = __builtin_amdgcn_perm(S.xr[p].z, S.xr[p].x, 0x07060302u);
                o.z = __builtin_amdgcn_perm(S.xr[p].w, S.xr[p].y, 0x05040100u);
                o.w = __builtin_amdgcn_perm(S.xr[p].w, S.xr[p].y, 0x07060302u);
            }
            *(uint4 *)(bd + (pk >> 3) * kPitch + (pk & 7) * 8) = o;
        }
    };
    // LDS-only workgroup barrier: the global loads of later k blocks stay in flight across it
    auto lds_barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    // ---- MFMA roles ----
    int afrag_off[MF];                                    // offset of this lane's fragment rows inside a weight tile
#pragma unroll
    for (int f = 0; f < MF; ++f) afrag_off[f] = ((wm * MF + f) * 32 + row32) * kPitch + hf * 8;
    const int bfrag_off = (wn * NF * 32 + row32) * kPitch + hf * 8;

    float16_t acc[MF][NF];
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[f][j][v] = 0.0f;

    // One k block: MFMAs on LDS buffer `buf` while the staged block S is decoded into the other buffer.  The
    // fragments of k step ks+1 are requested before the MFMAs of step ks are issued, and a quarter of the decode
    // is placed next to each step's MFMAs; the scheduling fences keep the compiler from undoing either.
    auto block = [&](int buf, const Stage &S, Stage &L, int kb_load) {
        const uint16_t *ab = As + buf * kABuf, *bb = Bs + buf * kBBuf + bfrag_off;
        half8_t af[2][MF], bf[2][NF];
#pragma unroll
        for (int f = 0; f < MF; ++f) af[0][f] = *(const half8_t *)(ab + afrag_off[f]);
#pragma unroll
        for (int j = 0; j < NF; ++j) bf[0][j] = *(const half8_t *)(bb + j * 32 * kPitch);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int cur = ks & 1, nxt = cur ^ 1;
            if (ks + 1 < BK / 16) {
#pragma unroll
                for (int f = 0; f < MF; ++f) af[nxt][f] = *(const half8_t *)(ab + afrag_off[f] + (ks + 1) * 16);
#pragma unroll
                for (int j = 0; j < NF; ++j) bf[nxt][j] = *(const half8_t *)(bb + j * 32 * kPitch + (ks + 1) * 16);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (WM * WN > 4) __builtin_amdgcn_s_setprio(1);      // two wavefronts per SIMD: the one that has its fragments issues its MFMAs first
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int f = 0; f < MF; ++f)
                    acc[f][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[cur][f], bf[cur][j], acc[f][j], 0, 0, 0);
            if (WM * WN > 4) __builtin_amdgcn_s_setprio(0);
            stage_load(L, kb_load, ks);
            stage_store(S, buf ^ 1, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Software pipeline over k blocks, ST register stages deep: the global loads of block kb+ST are issued during block kb
    // (a share next to each k step) into the stage whose block was decoded during block kb-1, and are consumed (decoded
    // into LDS) during block kb+ST-1, ST-1 blocks of MFMAs later (the k blocks of a workgroup are a multiple of ST).
    Stage S[ST];
    stage_load_all(S[0], 0);
#pragma unroll
    for (int part = 0; part < 4; ++part) stage_store(S[0], 0, part);
    lds_barrier();
#pragma unroll
    for (int d = 1; d < ST; ++d) stage_load_all(S[d], d);
    for (int kb = 0; kb < nkb; kb += ST) {
#pragma unroll
        for (int b = 0; b < ST; ++b) {
            // MFMAs on buffer b & 1 (block kb+b), block kb+b+1 decoded into the other buffer, loads of block kb+b+ST
            block(b & 1, S[(b + 1) % ST], S[b], kb + b + ST);
            lds_barrier();
        }
    }

    // ---- epilogue.  acc[f][j][v]: tile row of fragment f + 8 (v/4) + 4 (lane/32) + v%4, x row n0 + 32 (NF wn + j) + lane%32 ----
    // k split: the raw fp32 tile goes to partial[split][x row][weight row], and the finishing pass adds the splits in order and applies the epilogue
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int xrow = n0 + (wn * NF + j) * 32 + row32;
        if (xrow >= a.n) continue;
#pragma unroll
        for (int f = 0; f < MF; ++f)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int row = tile_m * BM + (wm * MF + f) * 32 + b * 8 + hf * 4;
                if (row >= a.m) continue;                        // m % 4 == 0 is checked by the launcher
                const float v0 = acc[f][j][b * 4], v1 = acc[f][j][b * 4 + 1], v2 = acc[f][j][b * 4 + 2], v3 = acc[f][j][b * 4 + 3];
                if (a.partial) *(float4 *)(a.partial + ((size_t)split * a.n + xrow) * a.m + row) = make_float4(v0, v1, v2, v3);
                else *(uint2 *)(a.out_f16 + (size_t)xrow * a.m + row) = make_uint2(f2h(v0) | ((uint32_t)f2h(v1) << 16), f2h(v2) | ((uint32_t)f2h(v3) << 16));
            }
    }
}

template <int NF, bool FP16W, int WM = 2>
hipError_t launch_tile(const GemmArgs &a_in, hipStream_t stream, int splits)
{
    constexpr int BM = 64 * WM, BN = 64 * NF, kThreadsG = WM * 128;
    GemmArgs a = a_in;
    if (a.epi != EPI_F16) return hipErrorInvalidValue;   // plain matmuls only: a split launch's epilogue is the finishing pass
    const dim3 grid(gemm_tile_grid(a, BM, BN, splits));
    const size_t lds = 2 * (size_t)(BM + BN) * kPitch * sizeof(uint16_t);    // up to 147456 bytes: one workgroup per CU
    static std::atomic<bool> attr_done{false};   // setting the attribute twice is harmless; the flag only has to be a defined read
    if (!attr_done.load()) {
        if (hipFuncSetAttribute((const void *)gemm_mfma_kernel<NF, FP16W, WM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return hipErrorInvalidValue;
        attr_done.store(true);
    }
    hipLaunchKernelGGL((gemm_mfma_kernel<NF, FP16W, WM>), grid, dim3(kThreadsG), lds, stream, a);
    return hipGetLastError();
}

}  // namespace

// Whether the MFMA path can serve this matrix (k in whole 128-blocks, 16-byte aligned rows, 4-row store granules).
bool gemm_mfma_eligible(const relax_qmat &w, const void *x, int epi)
{
    if (w.k % (2 * BK) != 0 || gshift_of(w.group) < 0) return false;
    if ((reinterpret_cast<uintptr_t>(w.q) & 15) != 0 || (reinterpret_cast<uintptr_t>(w.s) & 1) != 0) return false;
    if ((reinterpret_cast<uintptr_t>(x) & 15) != 0) return false;
    if (epi == EPI_SWIGLU) return w.m % 8 == 0;
    return w.m % 4 == 0;
}

// Tile and cut of a launch: the least estimated time over the tiles (weight rows x x-rows) and over k splits, of which there
// may be up to kSplitKMax of at least 8 k blocks each for up to kSplitKMaxN rows; the fp32 partial tiles of a split launch go to
// the caller's workspace (it has to hold them) and the finishing pass of the few-row kernel adds them in order and applies the
// epilogue: 0.6 us, 0.3 per split and the partial rows twice over at 5 TB/s.
// A k block of a wave of 256 workgroups takes longer the more of them there are (clock and fabric), and the two small tiles fit a
// CU twice, so a launch of 257 to 512 of them is still one round.  The figures are the ones whose choice is closest to the fastest launch:
// of 4-bit weights over 27 matrices from 768 x 256 to 57344 x 8192 at 65 to 2048 rows, every tile, every split up to 512 rows and two launches,
// with and without a workspace, 0.5 % off on average and 9 % at most (the figures before them, under which 256 x 128 tiles were held to matrices
// of one round at 640 rows and more, 1.0 %: 12288 x 4096 at 600 rows 64.3 against 70.2 us); of 3-bit and fp16 weights over 28 matrices 0.3 % and 0.1 %.
// With one figure per tile, taken on a full chip, 256 x 192 tiles were preferred to 144 of 256 x 256 or 480 of 128 x 128 (12288 x 4096 of 3-bit weights
// at 640 rows 97 against 86 us).  Fp16 weights have no tiles of 256 weight rows: their staging needs more registers than two wavefronts
// per SIMD leave, and as four wavefronts they lost to two of 128 rows on all but the longest rows (27648 x 5120 at 2048 rows 741 to 882
// against 667 us; 8192 x 28672 at 1200 877 against 943).
namespace {
struct TilePlan {
    int mf, nf, splits, kb_per_split;
    int m_big;               // > 0: the first m_big weight rows go through a launch of 256 x 256 tiles of their own (whole rounds of them)
    double us;               // estimated time less the launch
};
struct TileCost {
    int mf, nf;
    int per_cu;              // workgroups a CU holds
    double few[2], full[2];  // us per k block of a wave with few and with 256 workgroups; [1]: of the second workgroup of every CU, both together
};
constexpr TileCost kTiles[] = {{4, 4, 1, {1.376}, {1.729}}, {4, 3, 1, {0.803}, {1.377}}, {4, 2, 1, {0.716}, {1.029}}, {2, 4, 1, {0.569}, {1.076}},
                               {2, 3, 1, {0.563}, {0.841}}, {2, 2, 2, {0.418, 0.938}, {0.671, 1.142}}, {2, 1, 2, {0.296, 0.707}, {0.464, 0.707}}};
constexpr TileCost kTilesQ3[] = {{4, 4, 1, {1.67}, {1.85}}, {4, 3, 1, {1.25}, {1.50}}, {2, 4, 1, {0.90}, {1.08}}, {2, 3, 1, {0.74}, {0.88}},
                                 {2, 2, 2, {0.59, 1.04}, {0.70, 1.22}}, {2, 1, 2, {0.475, 0.78}, {0.515, 0.90}}};
constexpr TileCost kTilesF16[] = {{2, 4, 1, {0.985}, {1.13}}, {2, 3, 1, {0.85}, {0.96}}, {2, 2, 2, {0.70, 1.45}, {0.82, 1.60}}, {2, 1, 2, {0.58, 1.05}, {0.67, 1.43}}};
constexpr long kCUs = 256;

double tile_us(const TileCost &t, long workgroups, int k_blocks)
{
    const long slots = kCUs * t.per_cu, rest = workgroups % slots;
    double us = (double)(workgroups / slots) * t.full[t.per_cu - 1];
    if (rest > 0) {
        const int level = rest > kCUs;
        us += t.few[level] + (t.full[level] - t.few[level]) * (double)(rest - level * kCUs) / kCUs;
    }
    return us * k_blocks;
}

TilePlan tile_plan(int wmode, int m, int k, int n, int epi, size_t partial_floats)
{
    const long rows = epi == EPI_SWIGLU ? m / 2 : m;
    const long rdiv = epi == EPI_SWIGLU ? 2 : 1;
    auto blocks = [&](int mf, int nf) { return ((rows + 64 * mf / rdiv - 1) / (64 * mf / rdiv)) * (long)((n + 64 * nf - 1) / (64 * nf)); };
    const int nkb = k / BK;
    const int most = n <= kSplitKMaxN ? kSplitKMax : 1;
    TilePlan p = {2, 1, 1, nkb, 0, 0.0};
    double best_us = 0.0;
    const double finish0 = wmode == W_Q4 ? 0.58 : 1.6, finish1 = wmode == W_Q4 ? 0.27 : 0.4;
    const TileCost *const first = wmode == W_F16 ? std::begin(kTilesF16) : wmode == W_Q3 ? std::begin(kTilesQ3) : std::begin(kTiles);
    const TileCost *const last = wmode == W_F16 ? std::end(kTilesF16) : wmode == W_Q3 ? std::end(kTilesQ3) : std::end(kTiles);
    for (const TileCost *c = first; c != last; ++c) {
        const TileCost &t = *c;
        if (t.nf > 2 && n <= 128) continue;               // (one x tile is enough; the wide ones were not measured there)
        const long tiles = blocks(t.mf, t.nf);
        for (int s = 1; s <= most && (s == 1 || nkb / s >= 8); ++s) {
            const int per = s == 1 ? nkb : ((nkb + s - 1) / s + 1) & ~1, splits = (nkb + per - 1) / per;
            if (splits != s || (s > 1 && (size_t)s * n * m > partial_floats)) continue;
            const double us = tile_us(t, tiles * s, per) + (s > 1 ? finish0 + finish1 * s + (double)s * n * m * 8.0 / 5e6 : 0.0);
            if (best_us == 0.0 || us < best_us) best_us = us, p.mf = t.mf, p.nf = t.nf, p.splits = s, p.kb_per_split = per;
        }
    }
    // Or two launches (4-bit, plain rows): whole rounds of 256 x 256 tiles on the first weight rows, 128 x 256 tiles on the rest, and 3.3 us
    // for the second launch (7B QKV at n = 2048: 194 -> 185 us; 27648 x 5120 at n = 2048 491 against 515 in one launch).
    const long tn = (n + 255) / 256, rows_round = kCUs / std::min(tn, kCUs) * 256;      // weight rows of one round of wide tiles
    if (wmode == W_Q4 && epi != EPI_SWIGLU && n > 128 && tn <= kCUs)
        for (long big = rows_round; big < rows; big += rows_round) {
            const double us = (double)(big / rows_round) * kTiles[0].full[0] * nkb + tile_us(kTiles[3], (rows - big + 127) / 128 * tn, nkb) + 3.3;
            if (us < best_us) best_us = us, p = {2, 4, 1, nkb, (int)big, 0.0};
        }
    p.us = best_us;
    return p;
}

// Splits a workspace is sized for: a launch whose tiles of the best useful share (256 x 256, 128 x 256, 128 x 128 at 1, 0.9, 0.6 per
// MFMA) would leave more than half of the CUs idle, cut into about one workgroup per CU.  tile_plan takes what fits.
int sized_splits(int m, int k, int n, int epi)
{
    const long rows = epi == EPI_SWIGLU ? m / 2 : m, rdiv = epi == EPI_SWIGLU ? 2 : 1;
    auto blocks = [&](int mf, int nf) { return ((rows + 64 * mf / rdiv - 1) / (64 * mf / rdiv)) * (long)((n + 64 * nf - 1) / (64 * nf)); };
    auto score = [&](int mf, int nf, double tile_eff) {
        const double rounds = (double)((blocks(mf, nf) + kCUs - 1) / kCUs);
        return tile_eff * (double)rows * (double)n / (rounds * kCUs * (64.0 * mf / rdiv) * (64.0 * nf));
    };
    const double s44 = score(4, 4, 1.0), s24 = score(2, 4, 0.9), s22 = score(2, 2, 0.6);
    const long tiles = s44 >= s24 && s44 >= s22 ? blocks(4, 4) : s24 >= s22 ? blocks(2, 4) : blocks(2, 2);
    const int nkb = k / BK;
    if (tiles > kCUs / 2) return 1;
    const int splits = std::max(1, std::min(std::min(kSplitKMax, (int)(kCUs / tiles)), nkb / 8)), per = ((nkb + splits - 1) / splits + 1) & ~1;
    return (nkb + per - 1) / per;
}
}  // namespace

// fp32 elements of workspace a caller brings for the k-split form at any row count up to n (0: this matrix is not sized for it)
size_t gemm_splitk_partial_floats(int m, int k, int n, int epi)
{
    if (k % (2 * BK) != 0) return 0;
    size_t worst = 0;
    const int top = n < kSplitKMaxN ? n : kSplitKMaxN;
    for (int nn = 256; nn <= top + 127; nn += 128) {               // splits change with the tile counts only: the top of each bracket
        const int r = nn < top ? nn : top;
        if (r <= 128) continue;
        const int splits = sized_splits(m, k, r, epi);
        if (splits > 1) worst = std::max(worst, (size_t)splits * (size_t)r * (size_t)m);
    }
    return worst;
}

double gemm_tile_us(int m, int k, int n, int epi, size_t partial_floats) { return 5.1 + tile_plan(W_Q4, m, k, n, epi, partial_floats).us; }

void gemm_tile_plan(int wmode, int m, int k, int n, int epi, size_t partial_floats, relax_matmul_plan *plan)
{
    const TilePlan p = tile_plan(wmode, m, k, n, epi, partial_floats);
    plan->k_ranges = p.splits, plan->tile_rows = 64 * p.mf, plan->tile_cols = 64 * p.nf, plan->wide_rows = p.m_big;
}

// k splits the launch would make for n rows with this much workspace (1: one pass over k, no finishing pass)
int gemm_mfma_splits(const relax_qmat &w, int n, int epi, const float *partial, size_t partial_floats)
{
    return tile_plan(W_Q4, w.m, w.k, n, epi, partial && (reinterpret_cast<uintptr_t>(partial) & 15) == 0 ? partial_floats : 0).splits;
}

// out[n,m] = x[n,k] . w[m,k]^T with plain fp16 weights: the same tiles, no decode, one pass over k
bool gemm_f16_eligible(const void *x, const void *w, const void *out, int m, int k)
{
    return k % (2 * BK) == 0 && m % 4 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w)) & 15) == 0 &&
           (reinterpret_cast<uintptr_t>(out) & 7) == 0;
}

hipError_t launch_gemm_f16(const uint16_t *x, const uint16_t *w, int n, int m, int k, uint16_t *out, hipStream_t stream, float *partial, size_t partial_floats)
{
    GemmArgs a = {};
    a.x = x, a.wh = w, a.n = n, a.m = m, a.k = k, a.epi = EPI_F16, a.out_f16 = out, a.partial = partial;
    const TilePlan p = tile_plan(W_F16, m, k, n, EPI_F16, partial ? partial_floats : 0);
    a.kb_per_split = p.kb_per_split;
    if (p.nf == 4) return launch_tile<4, true>(a, stream, p.splits);
    if (p.nf == 3) return launch_tile<3, true>(a, stream, p.splits);
    if (p.nf == 2) return launch_tile<2, true>(a, stream, p.splits);
    return launch_tile<1, true>(a, stream, p.splits);
}

// out[n,m] = x[n,k] . w[m,k]^T with 3-bit weights in the native word layout (group 32): the same tiles, one pass over k
bool gemm_q3_eligible(const void *x, const relax_qmat &w, const void *out)
{
    return w.k % (2 * BK) == 0 && w.m % 4 == 0 && (w.group == 0 || w.group == 32) && (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
           (reinterpret_cast<uintptr_t>(w.q) & 3) == 0 && (reinterpret_cast<uintptr_t>(w.s) & 1) == 0 && (reinterpret_cast<uintptr_t>(out) & 7) == 0;
}

hipError_t launch_gemm_q3(const uint16_t *x, const relax_qmat &w, int n, uint16_t *out, hipStream_t stream, float *partial, size_t partial_floats)
{
    GemmArgs a = {};
    a.x = x, a.q = w.q, a.s = w.s, a.gshift = 0, a.n = n, a.m = w.m, a.k = w.k, a.epi = EPI_F16, a.out_f16 = out, a.partial = partial;
    const TilePlan p = tile_plan(W_Q3, w.m, w.k, n, EPI_F16, partial ? partial_floats : 0);
    a.kb_per_split = p.kb_per_split;
    if (p.mf == 4 && p.nf == 4) return launch_tile<4, false, 4>(a, stream, p.splits);
    if (p.mf == 4) return launch_tile<3, false, 4>(a, stream, p.splits);
    if (p.nf == 4) return launch_tile<4, false>(a, stream, p.splits);
    if (p.nf == 3) return launch_tile<3, false>(a, stream, p.splits);
    if (p.nf == 2) return launch_tile<2, false>(a, stream, p.splits);
    return launch_tile<1, false>(a, stream, p.splits);
}

// k splits of the two launches above with this much workspace: more than one leaves partial rows for launch_skinny_finish
int gemm_flat_splits(int wmode, int n, int m, int k, size_t partial_floats) { return k % (2 * BK) == 0 ? tile_plan(wmode, m, k, n, EPI_F16, partial_floats).splits : 1; }

// Whether the one-pass launch on this QKV matrix can rotate q and k and append k and v in its epilogue
bool gemm_rope_fuse_ok(const relax_layer_dims &dm, const relax_kv_cache &cache, const relax_qmat &w)
{
    return dm.head_dim == 128 && w.m == (dm.n_heads + 2 * dm.n_kv_heads) * 128 &&
           ((reinterpret_cast<uintptr_t>(cache.k) | reinterpret_cast<uintptr_t>(cache.v)) & 7) == 0 && (reinterpret_cast<uintptr_t>(cache.rope) & 15) == 0;
}

hipError_t launch_gemm_mfma(const uint16_t *x, const relax_qmat &w, int n, int epi, uint16_t *out_f16, float *out_f32, const void *resid,
                            hipStream_t stream, float *partial, size_t partial_floats, const SkinnyFuse *fuse)
{
    GemmArgs a = {};
    a.wh = nullptr;
    a.x = x, a.q = w.q, a.s = w.s, a.gshift = gshift_of(w.group), a.n = n, a.m = w.m, a.k = w.k, a.epi = epi;
    a.out_f16 = out_f16, a.out_f32 = out_f32, a.resid = resid;
    const TilePlan p = tile_plan(W_Q4, w.m, w.k, n, epi, partial && (reinterpret_cast<uintptr_t>(partial) & 15) == 0 ? partial_floats : 0);
    if (fuse && p.splits < 2) {                                   // one pass over k: the rotary step of a QKV matrix is an epilogue, a norm is not
        if (epi != EPI_F16 || !fuse->dm || !gemm_rope_fuse_ok(*fuse->dm, *fuse->cache, w)) return hipErrorInvalidValue;
        a.epi = EPI_ROPE_KV;
        a.h = fuse->dm->n_heads, a.g = fuse->dm->n_kv_heads, a.kv_capacity = fuse->dm->kv_capacity;
        a.kcache = fuse->cache->k, a.vcache = fuse->cache->v, a.rope = fuse->cache->rope, a.seqs = *fuse->st;
    }
    a.partial = p.splits > 1 ? partial : nullptr;
    a.kb_per_split = p.kb_per_split;
    hipError_t e;
    if (p.m_big > 0 && p.splits == 1 && epi != EPI_SWIGLU) {
        // rows [0, m_big) on wide tiles, rows [m_big, m) on the narrow ones: two launches on the same stream
        GemmArgs b = a;
        b.m = p.m_big, b.ldm = w.m;
        e = launch_packed_tile(b, 4, 4, 1, stream);
        if (e != hipSuccess) return e;
        GemmArgs c = a;
        const size_t skip = (size_t)p.m_big;
        c.q = a.q + skip * (size_t)(w.k / 8), c.s = a.s + skip * (size_t)scales_per_row(w.k, a.gshift);
        c.m = w.m - p.m_big, c.ldm = w.m, c.first_row = p.m_big;
        if (c.out_f16) c.out_f16 = a.out_f16 + skip;
        if (c.out_f32) c.out_f32 = a.out_f32 + skip;
        if (c.resid) c.resid = (epi == EPI_RESID_F32) ? (const void *)((const uint16_t *)a.resid + skip) : (const void *)((const float *)a.resid + skip);
        return launch_packed_tile(c, 2, 4, 1, stream);
    }
    e = launch_packed_tile(a, p.mf, p.nf, p.splits, stream);
    if (e != hipSuccess || p.splits < 2) return e;
    return launch_skinny_finish(partial, p.splits, n, w.m, epi, out_f16, out_f32, resid, stream, fuse);
}

}  // namespace relax
