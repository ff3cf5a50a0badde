// What the two tiled GEMM kernels share: their arguments, and the launchers of one tile shape each (a launch covers the whole matrix,
// or the weight rows the arguments name).
#pragma once

#include "relax_common.h"

namespace relax {

constexpr int kTileK = 64;               // columns per k block of the main loops

struct GemmArgs {
    const uint16_t *x;       // [n,k] fp16
    const uint32_t *q;       // [m,k/8]; 3-bit weights: [m, 3 k / 32] words of the native layout
    const uint16_t *s;       // [m, k / (32 << gshift)]
    int32_t gshift;          // 32-column sub-group index >> gshift = scale index (quantisation group 32, 64 or 128)
    const uint16_t *wh;      // plain fp16 weights [m,k] instead of q, s
    int32_t n, m, k;
    int32_t ldm;             // row pitch of out / resid in elements; 0: m (a launch on a range of the weight rows brings the matrix's m here)
    int32_t epi;
    int32_t tiles_m;         // weight-row tiles of the launch (the grid is one-dimensional: tiles_m * x-row tiles * k splits)
    int32_t tiles_n;         // x-row tiles
    int32_t kb_per_split;    // k blocks (of kTileK columns) per k split, even; one split: all of them
    float *partial;          // more than one k split: [split][n][m] fp32 partial tiles, finished by the few-row kernel's finishing pass
    uint16_t *out_f16;       // EPI_F16: [n,m]; EPI_RESID_F16: [n,m]; EPI_SWIGLU: [n,m/2]
    float *out_f32;          // EPI_RESID_F32: [n,m]
    const void *resid;       // EPI_RESID_F32: fp16 [n,m]; EPI_RESID_F16: fp32 [n,m]
    // EPI_ROPE_KV (a QKV matrix, heads of 128): rotated q goes to out_f16, rotated k and v to the cache
    int32_t first_row;       // matrix row of the launch's row 0
    int32_t h, g, kv_capacity;
    uint16_t *kcache, *vcache;
    const float *rope;
    SeqTable seqs;
};

// Tile counts of a launch and its grid; splits < 2: one pass over k, no partial tiles.
inline int gemm_tile_grid(GemmArgs &a, int tile_rows, int tile_cols, int splits)
{
    const int rows = a.epi == EPI_SWIGLU ? a.m / 2 : a.m, per = a.epi == EPI_SWIGLU ? tile_rows / 2 : tile_rows;
    a.tiles_m = (rows + per - 1) / per;
    a.tiles_n = (a.n + tile_cols - 1) / tile_cols;
    if (splits < 2) a.partial = nullptr, a.kb_per_split = a.k / kTileK, splits = 1;
    return a.tiles_m * a.tiles_n * splits;
}

// 4-bit weights (gemm_packed_kernel.h): weight rows x rows of x of a tile
hipError_t launch_packed_256x256(const GemmArgs &a, int splits, hipStream_t stream);
hipError_t launch_packed_256x192(const GemmArgs &a, int splits, hipStream_t stream);
hipError_t launch_packed_256x128(const GemmArgs &a, int splits, hipStream_t stream);
hipError_t launch_packed_128x256(const GemmArgs &a, int splits, hipStream_t stream);
hipError_t launch_packed_128x192(const GemmArgs &a, int splits, hipStream_t stream);
hipError_t launch_packed_128x128(const GemmArgs &a, int splits, hipStream_t stream);
hipError_t launch_packed_128x64(const GemmArgs &a, int splits, hipStream_t stream);
inline hipError_t launch_packed_tile(const GemmArgs &a, int mf, int nf, int splits, hipStream_t stream)
{
    if (mf == 4 && nf == 2) return launch_packed_256x128(a, splits, stream);
    if (mf == 4) return nf == 4 ? launch_packed_256x256(a, splits, stream) : launch_packed_256x192(a, splits, stream);
    if (nf == 4) return launch_packed_128x256(a, splits, stream);
    if (nf == 3) return launch_packed_128x192(a, splits, stream);
    return nf == 2 ? launch_packed_128x128(a, splits, stream) : launch_packed_128x64(a, splits, stream);
}

}  // namespace relax
