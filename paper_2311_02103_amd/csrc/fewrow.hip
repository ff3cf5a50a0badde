// Host side of the streaming few-row matmul (fewrow_kernel.h): which calls it takes, how they are cut, the launch.
#include "fewrow_kernel.h"

namespace relax {

namespace fewrow {
hipError_t launch_q4g32(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream);
hipError_t launch_q4g64(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream);
hipError_t launch_q4g128(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream);
hipError_t launch_q3(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream);
hipError_t launch_f16(int nb, int uw, const Args &a, size_t lds_bytes, bool wait, hipStream_t stream);
}  // namespace fewrow

namespace {

using namespace fewrow;

bool uw_built(int fmt, int nb, int uw)                    // the instances of launch_nb
{
    if (fmt == F_F16) return uw >= 1 && (nb == 1 ? uw <= 6 || uw == 8 : nb == 2 && uw <= 4);
    return uw >= 1 && uw <= (nb == 1 ? 6 : nb == 2 ? 3 : 1);
}

// Row tiles whose shares the LDS of a workgroup holds at a time (wait: beside the sums of all its `per` tiles, 1 KB each)
int lds_tiles(int fmt, int nb, int uw, bool wait = false, int per = 0)
{
    const size_t room = (scale_sums(fmt, nb, uw) && nb == 1 ? kLdsBytes : kShareBytes) - offset_bytes(fmt, nb, uw, wait) - (wait ? (size_t)per * 1024 : 0);
    return (int)(room / ((size_t)kWaves * nb * 1024));
}

int blocks_of(int n) { return n <= 16 ? 1 : n <= 32 ? 2 : 4; }

int tiles_of(int m, int epi) { return epi == EPI_SWIGLU ? (m / 2 + 7) / 8 : (m + kTileRows - 1) / kTileRows; }

// The cut into kg k ranges; false: no instance of the kernel for it.
bool cut(int fmt, int nb, int m, int k, int epi, int kg, Plan &p)
{
    const bool f16 = fmt == F_F16;
    const int units = k / unit_columns(f16);
    p.kg = kg, p.uw = (units + kWaves * kg - 1) / (kWaves * kg);
    if (!uw_built(fmt, nb, p.uw)) return false;
    p.tiles = tiles_of(m, kg > 1 ? (int)EPI_F16 : epi);
    p.rg = std::min(p.tiles, 256 / kg);
    // a workgroup whose epilogue is not plain partial rows keeps all its tiles in LDS (one block of x rows: any): more workgroups if they don't fit
    const int most = std::max(lds_tiles(fmt, nb, p.uw), sums_wait(fmt, nb, p.uw) ? kMostTiles : 0);
    if (kg == 1 || nb == 1)
        while ((p.tiles + p.rg - 1) / p.rg > most) p.rg = std::min(p.tiles, p.rg + 256 / kg);
    return true;
}

// What a launch takes, in us, for blocks of 16, 32 and 64 rows of x: fitted to 22 matrices from 1024 x 4096 to 57344 x 8192 (groups of 32 beyond
// 16 rows: to 73) at 2 to 64 rows, weights cold, every k range the kernel is built for.  What the 4-bit figures choose is 0.3 % off the fastest k
// range on average for blocks of 16, 0.6 % for 32, 9 and 10 % at most; the estimates are within 4 % of the times on average (launches with scales on
// sums of before their arguments were read behind the loop, which takes 0.5 to 1 us off each).
//   launch                 the launch, the first data and the sums over the wavefronts
//   tb_per_s               the stream of the weights, or, where few row tiles or uneven slices leave it to the slowest workgroup,
//   unit, tile             ... per row tile of a workgroup: its longest slice's units, and the sums
//   x                      per MB of x a workgroup fetches from its L2: long rows and many rows of x want k ranges
//   finish, range, partial the finishing launch, per k range of it, and the partial rows at TB/s
//   full                   more where every wavefront holds four units of x or more and none has one to spare (8192 columns in one range)
//   round                  more per wave of workgroups behind the first, which begins with x and the first data again
struct Cost {
    double launch, tb_per_s, unit, tile, x, finish, range, partial, full, round;
};
constexpr Cost kCostQ4[3] = {{4.1, 6.2, 0.62, 0.31, 23, 2.0, 0.32, 7.9, 1.4, 6.6}, {4.6, 5.4, 0.79, 0.0, 32, 2.2, 0.57, 2.7, 0.0, 8.0}, {4.8, 3.1, 1.39, 0.05, 25, 2.6, 0.79, 38}};
// ... of six units, which have scales on codes, and of plain matmuls of up to 16 rows: fitted to the kernel with two and three row tiles in flight and
// scales on codes.  Plain matmuls keep these figures, and so the kernel and cut that the host tests pin with that kernel's times, although the
// stream has become faster: over 76 launches (19 matrices, 2 to 16 rows) what they choose is 3.6 % off the fastest on average, 22 % at
// most, where that is split-K or too few k ranges (us, split-K / stream: 8192 x 8192 at 4 rows 15.2 / 12.5, 15360 x 5120 at 16 rows 18.9 / 15.8, 10240 x
// 8192 at 8 rows 18.2 / 15.1).
constexpr Cost kCostQ4Alone = {4.2, 9.5, 0.65, 0.17, 35, 3.1, 0.33, 3.3, 3.4};
// ... groups of 64 and 128 (at 32 rows the arithmetic of a unit is what counts: the fit leaves the stream nothing)
constexpr Cost kCostQ4Coarse[2] = {{4.1, 6.8, 0.64, 0.06, 22, 1.9, 0.32, 2.7, 1.6, 6.9}, {4.8, 36, 0.49, 0.42, 27, 1.5, 0.34, 2.8, 9.3, 2.2}};
// 3-bit and fp16 matrices: the rates of the stream alone (what is estimated for them only picks the k ranges of a layer's matrices)
constexpr Cost kCostQ3[3] = {{5.8, 5.9, 0.46, 0.0, 25, 3.1, 0.0, 5.8}, {5.8, 5.35, 0.51, 0.0, 27, 3.4, 0.0, 5.3}, {5.8, 4.7, 0.58, 0.0, 31, 3.9, 0.0, 4.6}};
constexpr Cost kCostF16[2] = {{5.8, 5.9, 1.05, 0.0, 25, 3.1, 0.0, 5.8}, {5.8, 5.35, 1.17, 0.0, 27, 3.4, 0.0, 5.3}};
constexpr double kSumsWait = 2.0;                         // two ranges whose sums wait in LDS (34816 x 8192 at 8 rows, groups of 64, 37.1 us, one range without 35.4)
constexpr double kFolded = 2.5;                           // a finishing pass that is also a step of the layer saves that step's launch

int block_class(int n) { return n <= 16 ? 0 : n <= 32 ? 1 : 2; }

// The number of k ranges with the least estimated time (`folded`: the finishing pass is also the RMSNorm of the result; `exact`: scales on sums only).
int best_ranges(int fmt, int n, int m, int k, int epi, bool folded, bool alone, bool exact, size_t partial_floats, double *time_us)
{
    const bool f16 = fmt == F_F16, q4 = !f16 && fmt != F_Q3;
    const Cost &cost = alone && fmt == F_Q4G32 && n <= 16 ? kCostQ4Alone : (f16 ? kCostF16 : fmt == F_Q3 ? kCostQ3 : fmt == F_Q4G32 ? kCostQ4 : kCostQ4Coarse)[block_class(n)];
    const double bytes = (double)m * k * (f16 ? 2.0 : fmt == F_Q3 ? 0.4375 : fmt == F_Q4G32 ? 0.5625 : fmt == F_Q4G64 ? 0.53125 : 0.515625);
    double best_us = 0.0;
    int best = 0;
    for (int kg = 1; kg <= 16 && (kg == 1 || (size_t)kg * n * m <= partial_floats); ++kg) {
        Plan p;
        if (!cut(fmt, blocks_of(n), m, k, epi, kg, p) || (exact && !scale_sums(fmt, blocks_of(n), p.uw))) continue;
        const Cost &c = q4 && p.uw == 6 ? kCostQ4Alone : cost;
        const double per = (p.tiles + p.rg - 1) / p.rg, rounds = (p.rg * kg + 255) / 256;
        double us = std::max(bytes / (c.tb_per_s * 1e6), rounds * per * (p.uw * c.unit + c.tile)) + rounds * n * ((double)k / kg) * 2e-6 * c.x + (rounds - 1) * c.round;
        if (p.uw >= 4 && k / unit_columns(f16) == p.uw * kWaves * kg) us += c.full;
        if (kg > 1 && sums_wait(fmt, blocks_of(n), p.uw) && per > lds_tiles(fmt, blocks_of(n), p.uw)) us += kSumsWait;
        if (kg > 1) us += c.finish + kg * c.range + (double)kg * n * m * 8e-6 / c.partial - (folded ? kFolded : 0.0);
        us += c.launch;
        if (best == 0 || us < best_us) best = kg, best_us = us;
        if (p.uw == 1) break;
    }
    *time_us = best_us;
    return best;
}

// The same for the split-K few-row kernel (4-bit matrices): workgroups of 128 rows and `rounds` rounds of 256 columns, whole waves of 256
// of them (12288 x 12288 has 288: 34.8 us at 6 rows, the stream 23.6) or what the chip makes of all of them.
struct SplitCost {
    double launch, row, wave, chip, split, partial;
};
constexpr SplitCost kCostSplit[3] = {{7.0, 0.054, 0.81, 0.65, 0.2, 2.1}, {4.9, 0.09, 1.1, 0.48, 0.27, 4.3}, {5.1, 0.01, 1.7, 1.55, 0.6, 4.0}};
double split_us(int n, int m, int k)
{
    const SplitCost &c = kCostSplit[block_class(n)];
    int tiles_m, splits, rounds;
    gemm_skinny_cut(m, k, &tiles_m, &splits, &rounds);
    const int workgroups = tiles_m * splits;
    return c.launch + c.row * n + std::max((workgroups + 255) / 256 * rounds * c.wave, workgroups / 256.0 * rounds * c.chip) + splits * c.split +
           (double)splits * n * m * 8e-6 / c.partial;
}

// Groups of 64 and 128: its scale staging is made for groups of 32 (us at 6, 16 and 32 rows, groups of 32 / 64 / 128: 4096 x 4096 11.6 / 13.1 / 12.9,
// 12.0 / 13.5 / 13.4, 13.5 / 14.8 / 14.7; 5120 x 13824 16.5 / 19.5 / 18.9, 17.3 / 21.4 / 19.8, 19.5 / 22.0 / 21.8; 22016 x 4096 22.5 / 25.9 / 25.0, 23.4 /
// 26.2 / 26.0, 26.7 / 29.3 / 29.4; without the factor a 13B layer of 8 rows takes 79.3 us with groups of 64, so 77.2).
constexpr double kSplitCoarse = 1.1;

bool shape_ok(bool f16, int n, int m, int k, int epi)
{
    if (n < kFewRowMin || n > kFewRowMax || k < 1 || k % unit_columns(f16) != 0) return false;
    return epi == EPI_SWIGLU ? m % 8 == 0 : m % 4 == 0;
}

constexpr size_t kMaxBuffer = 0x7FFFFFFFu;                // offsets into a buffer stay below 2^31

hipError_t launch(int fmt, const uint16_t *x, const void *w, size_t w_bytes, const uint16_t *s, size_t s_bytes, int n, int m, int k, int epi, int k_ranges,
                  uint16_t *out_f16, float *out_f32, const void *resid, float *partial, hipStream_t stream, const SkinnyFuse *fuse)
{
    Plan p;
    const int nb = blocks_of(n);
    if (!cut(fmt, nb, m, k, epi, k_ranges, p)) return hipErrorInvalidValue;
    Args a = {};
    a.x = x, a.w = w, a.s = s, a.x_bytes = (uint32_t)((size_t)n * k * 2), a.w_bytes = (uint32_t)w_bytes, a.s_bytes = (uint32_t)s_bytes;
    a.n = n, a.m = m, a.k = k, a.kg = p.kg, a.rg = p.rg, a.tiles = p.tiles;
    a.out_f16 = out_f16, a.out_f32 = out_f32, a.resid = resid;
    a.delta = 8;
    const bool rope = epi == EPI_F16 && fuse;
    if (p.kg > 1) {
        a.epi = kPartial, a.out_f32 = partial;
    } else if (rope) {
        const relax_layer_dims &dm = *fuse->dm;
        a.epi = EPI_ROPE_KV, a.delta = dm.head_dim / 2, a.ropeshift = dm.head_dim == 128 ? 3 : 2;
        a.kc = fuse->cache->k, a.vc = fuse->cache->v, a.rope = fuse->cache->rope;
        a.h = dm.n_heads, a.g = dm.n_kv_heads, a.d = dm.head_dim, a.cap = dm.kv_capacity, a.rope_once = fuse->rope_once, a.st = *fuse->st;
    } else {
        a.epi = epi;
        if (epi == EPI_SWIGLU) a.delta = m / 2;
    }
    const int per = (p.tiles + p.rg - 1) / p.rg;
    const bool wait = sums_wait(fmt, nb, p.uw) && per > lds_tiles(fmt, nb, p.uw);
    a.batch = std::min(per, lds_tiles(fmt, nb, p.uw, wait, per));
    const size_t lds = (size_t)a.batch * kWaves * nb * 1024 + offset_bytes(fmt, nb, p.uw, wait) + (wait ? (size_t)per * 1024 : 0);
    hipError_t e;
    switch (fmt) {
    case F_Q4G32: e = launch_q4g32(nb, p.uw, a, lds, wait, stream); break;
    case F_Q4G64: e = launch_q4g64(nb, p.uw, a, lds, wait, stream); break;
    case F_Q4G128: e = launch_q4g128(nb, p.uw, a, lds, wait, stream); break;
    case F_Q3: e = launch_q3(nb, p.uw, a, lds, wait, stream); break;
    default: e = launch_f16(nb, p.uw, a, lds, wait, stream); break;
    }
    if (e != hipSuccess || p.kg == 1) return e;
    return launch_skinny_finish(partial, p.kg, n, m, epi, out_f16, out_f32, resid, stream, fuse);
}

}  // namespace

double gemm_skinny_us(int n, int m, int k, int gshift) { return split_us(n, m, k) * (gshift == 0 ? 1.0 : kSplitCoarse); }

int fewrow_ranges(int wmode, int gshift, int n, int m, int k, int epi, bool folded, bool alone, bool exact, size_t partial_floats)
{
    // From 33 rows on all groups are decoded alike (scales on codes) and one estimate serves them (us at 33 and 64 rows, groups of 32 / 128: 22016 x 4096
    // 29.5 / 29.6 and 32.9 / 34.7, 27648 x 5120 43 / 44 and 48 / 46, 57344 x 8192 95 / 96 and 97 / 98, 8192 x 28672 56 / 57 and 64 / 62).
    if (n > 32) gshift = 0;
    const int fmt = wmode == W_F16 ? F_F16 : wmode == W_Q3 ? F_Q3 : gshift == 0 ? F_Q4G32 : gshift == 1 ? F_Q4G64 : F_Q4G128;
    if (!shape_ok(fmt == F_F16, n, m, k, epi) || (n > 32 && fmt == F_F16)) return 0;
    const size_t row = wmode == W_F16 ? (size_t)k * 2 : wmode == W_Q3 ? (size_t)k / 32 * 12 : (size_t)k / 2;
    if ((size_t)m * row > kMaxBuffer) return 0;
    double us = 0.0;
    const int kr = best_ranges(fmt, n, m, k, epi, folded, alone, exact, partial_floats, &us);
    // A 4-bit matrix may also go through the split-K few-row kernel, whose workgroups own 128 rows and an eighth of k: an eighth of the
    // x traffic, a lower rate.  It is the better one where its workgroups fill the chip, rows are long and x has many of them (groups of 32, split-K /
    // stream, us: 4096 x 11008 at 32 rows 16.6 / 20.6, 8192 x 8192 18.6 / 23.0, 15360 x 5120 at 64 28.2 / 35.8), a tie at 16 rows of such
    // matrices (8192 x 8192 16.5 / 15.9), the stream on the others (at 16 rows 22016 x 4096 23.5 / 16.6, 57344 x 8192 81 / 58.5).
    // Up to kMatvecRows rows of a layer stay here: that kernel rounds the weights, which the matvec kernels do not.
    if (wmode == W_Q4 && kr > 0 && (alone || n > kMatvecRows) && gemm_skinny_partial_floats(m, k, n) > 0 && partial_floats >= gemm_skinny_partial_floats(m, k, n) &&
        gemm_skinny_us(n, m, k, gshift) - (folded ? kFolded : 0.0) < us)
        return 0;
    // ... and on matrices that fill the chip with tiles through the tiled GEMM (48 rows: 49152 x 2048 26.5 against 45.3 us, 57344 x 8192 87 against 99),
    // in a layer from 33 rows on wherever that is estimated faster (64 rows, stream / split-K / tiled: 22016 x 4096 33 / 39 / 30, 27648 x 5120 47 / 53
    // / 40, 4096 x 4096 16.8 / 17.4 / 15.2; a 7B layer on 64 rows of 300 tokens 157 -> 145 us, 13B 199 -> 180, 70B 244 -> 231)
    if (wmode == W_Q4 && (gemm_prefers_tiled(m, n) || (!alone && n > 32)) && gemm_tile_us(m, k, n, epi, partial_floats) < us) return 0;
    return kr;
}

// A matmul on its own (no epilogue, no workspace) on 3-bit or fp16 weights: whether the streaming kernel is at least as fast as the
// kernels that take the call otherwise.  What those cost at few rows is passes over the matrix, so they are ahead where one pass
// serves all rows, and on matrices so small that the launch is what counts (stream against the other kernel, us):
//   3-bit  2 rows of up to 8192 columns are one pass: 22016 x 4096 19.2 / 14.0, 8192 x 8192 16.5 / 12.1, 57344 x 8192 59 / 52; 12288
//          columns take two: 4096 x 11008 13.3 / 14.6.  3 and 4 rows of up to 2048 columns: 5632 x 2048 7.7 / 6.7; 4096 x 4096 8.0 / 10.2.
//          Up to 1024 rows of 4096 columns at 8 rows: 1024 x 1024 5.2 / 4.4, 1000 x 3584 7.4 / 6.3, 1408 x 256 at 5 4.7 / 5.3; 256 x
//          768 at 15 5.2 / 4.0.
//          From 17 rows on the other kernel is the tiled GEMM: 256 columns at 32 rows 5.7 / 5.3, at 64 7.1 / 5.7; 768 columns 6.3 / 9.1;
//          from 33 rows on it is ahead on tall matrices (32000 x 2048 28.8 / 24.1, 5632 x 2048 12.4 / 19.8).
//   fp16   2, 4 and 8 rows are one pass of the matvec kernel.  2 rows up to 190 MB: 8192 x 8192 32.6 / 28.7, 22016 x 4096 35.6 / 34.1;
//          28672 x 4096 41.5 / 43.3.  4 rows up to 72 MB, and on very long or very short rows: 5120 x 5120 17.2 / 15.7, 10240 x 8192
//          37.0 / 35.2, 32000 x 2048 28.2 / 26.8; 12288 x 4096 20.5 / 21.1.  8 rows up to 8 MB: 1024 x 1024 5.9 / 4.8, 1000 x 3584 8.9 / 7.2; 2048 x 2048 a tie.
bool fewrow_pays_alone(int wmode, int n, int m, int k)
{
    if (wmode == W_Q3) {
        if (n == 2) return k > 8192;
        if (n <= 4 && k <= 2048) return false;
        if (n <= 8) return m > 1024 || k > 4096;
        if (n <= 15) return m > 256 || k > 1024;
        return n == 16 || (k > 256 && (n <= 32 || m <= 16384));
    }
    if (wmode == W_F16) {
        const double mb = (double)m * k * 2e-6;
        if (n == 2) return mb > 190.0;
        if (n == 4) return mb > 72.0 && k > 2048 && k < 8192;
        if (n == 8) return mb > 8.0;
    }
    return true;
}

bool fewrow_fuse_ok(const relax_layer_dims &dm, const relax_kv_cache &cache)
{
    return ((reinterpret_cast<uintptr_t>(cache.k) | reinterpret_cast<uintptr_t>(cache.v)) & 7) == 0 && (reinterpret_cast<uintptr_t>(cache.rope) & 15) == 0 &&
           (dm.head_dim == 64 || dm.head_dim == 128);
}

hipError_t launch_fewrow_q4(const uint16_t *x, const relax_qmat &w, int n, int epi, int k_ranges, uint16_t *out_f16, float *out_f32, const void *resid, float *partial,
                            hipStream_t stream, const SkinnyFuse *fuse)
{
    const int gs = gshift_of(w.group);
    return launch(gs == 0 ? F_Q4G32 : gs == 1 ? F_Q4G64 : F_Q4G128, x, w.q, (size_t)w.m * w.k / 2, w.s, (size_t)w.m * scales_per_row(w.k, gs) * 2, n, w.m, w.k,
                  epi, k_ranges, out_f16, out_f32, resid, partial, stream, fuse);
}
hipError_t launch_fewrow_q3(const uint16_t *x, const relax_qmat &w, int n, int epi, int k_ranges, uint16_t *out_f16, float *out_f32, const void *resid, float *partial,
                            hipStream_t stream, const SkinnyFuse *fuse)
{
    return launch(F_Q3, x, w.q, (size_t)w.m * (w.k / 32) * 12, w.s, (size_t)w.m * (w.k / 32) * 2, n, w.m, w.k, epi, k_ranges, out_f16, out_f32, resid, partial,
                  stream, fuse);
}
hipError_t launch_fewrow_f16(const uint16_t *x, const uint16_t *w, int n, int m, int k, int epi, int k_ranges, uint16_t *out_f16, float *out_f32, const void *resid,
                             float *partial, hipStream_t stream, const SkinnyFuse *fuse)
{
    return launch(F_F16, x, w, (size_t)m * k * 2, nullptr, 0, n, m, k, epi, k_ranges, out_f16, out_f32, resid, partial, stream, fuse);
}

}  // namespace relax
