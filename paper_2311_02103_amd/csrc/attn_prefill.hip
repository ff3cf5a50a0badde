// Causal attention for calls with many rows per sequence (prefill): the contraction is dense, so it runs on
// MFMA, tiled over the KV length with the running (max, sum) rescaling of an online softmax.  In the paper's
// terms this is the attention operator lowered to a hand-written library kernel whose q length n and KV length
// L are runtime values (Relax, Sec. 4.2 custom attention pattern, Sec. 4.5 cross-level library dispatch,
// Sec. 5.1 dynamic sequence length); scores, softmax and accumulation are fp32.
//
// Mapping for gfx950 (v_mfma_f32_32x32x16_f16, 64-wide wavefronts):
//   - Everything is computed transposed, S^T = K Q^T and O^T = V^T P^T, so that a query is a COLUMN of the MFMA
//     result: lane l of a wavefront then owns query (l % 32) in every accumulator register.  The row maximum and
//     row sum of the softmax become in-lane reductions plus one exchange with lane l ^ 32, the rescaling of O is a
//     per-lane scalar, and the probabilities a lane holds after S^T are exactly the eight k-values the B operand
//     of the second product wants from it -- P never goes through LDS or a shuffle.
//   - K tile in LDS as [t][d]: the A operand of K Q^T is a 16-byte row read.  V tile in LDS as [t][d] too; the A
//     operand of V^T P^T needs eight t-values of one d per lane, which the LDS transpose read of gfx950
//     (ds_read_b64_tr_b16) delivers from the untransposed tile: inside a block of 16 lanes, lane r supplies the
//     address of 4 halfs and lane L receives half (L % 4) of the rows supplied by lanes L/4 + 4j, j = 0..3.
//     With lane r pointing at V[t0 + r/4][d0 + 4 (r%4)], lane L receives V[t0 + 0..3][d0 + L].
//   - A workgroup is 128 queries of one (sequence, head) on 8 wavefronts (calls with few of them: 64 queries and 4 KV groups): 4 query
//     groups of 32 x 2 groups along the KV length (a wavefront takes every second 32-token sub-tile; the two states of a query group are merged
//     through LDS at the end).  The step count of the longest prefix sets the kernel time, and this halves it; fewer
//     queries per workgroup cost more than they give because every workgroup stages every K/V tile of its prefix.
//     A wavefront keeps its 32 queries' Q fragments in registers, O^T (32 x d fp32) in accumulators.  KV tiles of
//     64 tokens (one sub-tile per wavefront) are staged through registers into one of two LDS buffers, one barrier per
//     tile; the next tile's global loads are in flight during the MFMAs.  They are issued without a condition
//     (behind the last tile: the sequence's last row once more), 3 to 12 % faster than behind a branch.
//   - The query heads of a KV head get numbers that are equal modulo the number of KV heads: with 8 of them (or a multiple)
//     they go to the same XCD, and its K and V are fetched into one L2.
//   - Workgroups of the longest prefixes are first in dispatch order (causal work grows with the q position).
//   - Cache rows past a sequence's length are never read (loads are clamped to its last row); masked scores are
//     replaced, not multiplied, so stale cache contents cannot leak in.
#include "attn_device.h"

namespace relax {

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kTB = 32;              // tokens per KV tile

struct SeqInfo {
    int32_t q_start, q_len, kv_len, slot;
};

__device__ inline SeqInfo seq_info(const SeqTable &st, int b)
{
    SeqInfo s;
    if (st.dev) {
        s.q_start = st.dev[b], s.q_len = st.dev[st.B + b], s.kv_len = st.dev[2 * st.B + b], s.slot = st.dev[3 * st.B + b];
    } else {
        s.q_start = s.q_len = s.kv_len = s.slot = 0;
#pragma unroll
        for (int j = 0; j < kInlineSeqs; ++j)
            if (j == b) s.q_start = st.q_start[j], s.q_len = st.q_len[j], s.kv_len = st.kv_len[j], s.slot = st.slot[j];
    }
    return s;
}

// LDS-only workgroup barrier: outstanding global loads (the next KV tile) stay in flight across it
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A sequence with one row beside a prompt: the eight wavefronts stream its cache like the split kernel of the decode calls do, one workgroup per
// head, nothing staged; the states meet in LDS (float [wavefront][D + 2]).  As a 128-query tile with one live query it waited for
// every 64-token tile: a 7B call of a 300-row chunk on 1201 tokens beside 20 rows on 90 to 1173 took 72 us, now 49; its K and V alone are 37.
template <int D, int WAVES>
__device__ __forceinline__ void decode_row(const uint16_t *q, const uint16_t *kc, const uint16_t *vc, uint16_t *out, const SeqInfo &si, int h, int g, int kvh, int cap,
                                           float *sm)
{
    constexpr int LPT = D / 8, NL = D == 128 ? 4 : 2;         // heads of 64 have half the registers
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), e0 = (lane % LPT) * 8;
    const size_t base = ((size_t)si.slot * cap * g + kvh) * D;
    const char *ks = (const char *)(kc + base), *vs = (const char *)(vc + base);
    auto load_q = [&] { return *(const u32x4a_t *)(q + e0); };
    float m, l, acc[8];
    if (h == g) attend_tokens<D, WAVES, NL, true>(ks, vs, (uint32_t)g * D * 2, 0, si.kv_len, wave, lane, load_q, m, l, acc);
    else attend_tokens<D, WAVES, NL, false>(ks, vs, (uint32_t)g * D * 2, 0, si.kv_len, wave, lane, load_q, m, l, acc);
    if (lane < LPT) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sm[wave * (D + 2) + e0 + e] = acc[e];
        if (lane == 0) sm[wave * (D + 2) + D] = m, sm[wave * (D + 2) + D + 1] = l;
    }
    __syncthreads();
    if (tid < D) {
        float mm = -INFINITY, num = 0.0f, den = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mm = fmaxf(mm, sm[w * (D + 2) + D]);
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float *src = sm + w * (D + 2);
            const float sc = src[D] == -INFINITY ? 0.0f : __expf(src[D] - mm);     // a wavefront without a token
            num += src[tid] * sc;
            den += src[D + 1] * sc;
        }
        out[tid] = f2h(num / den);
    }
}

// grid: x = query head, y = q tile (reversed: longest prefix first), z = sequence
// MINW: wavefronts per SIMD the registers have to leave room for.  Heads of 64 fit two workgroups on a CU (4 per SIMD), which calls of
// many short sequences live on.
template <int D, int NWV, int KVS, int MINW>
__global__ __launch_bounds__(64 * NWV, MINW) void attn_prefill_kernel(const uint16_t *__restrict__ q, int q_stride,
                                                                 const uint16_t *__restrict__ kc, const uint16_t *__restrict__ vc,
                                                                 uint16_t *__restrict__ out, SeqTable st, int h, int g, int cap, int stream_rows)
{
    // NWV wavefronts = QW query groups x KVS groups along the KV length: wavefront (qw, kg) owns queries qw WQ .. + WQ of the
    // workgroup and every KVS-th 32-token sub-tile (the longest prefix is then KVS times fewer steps per wavefront);
    // the KVS states of a query group are merged through LDS at the end.
    static_assert(NWV % KVS == 0, "one sub-tile of a tile for every KV group");
    constexpr int QW = NWV / KVS;
    constexpr int kQB = QW * 32;             // queries per workgroup
    constexpr int kPThreads = 64 * NWV, WQ = 32;
    constexpr int KS = D / 16;       // k steps of K Q^T
    constexpr int DB = D / 32;       // 32-wide blocks of the head dimension in O^T
    static_assert(KS == 2 * DB, "both products of a sub-tile are KS MFMAs");
    constexpr int KP = D + 8;        // K tile pitch in halfs: 16-byte row reads of 32 rows hit distinct banks
    constexpr int VP = D + 32;       // V tile pitch in halfs: the 8-byte transpose reads of a 32-lane half hit distinct banks
    constexpr int TT = kTB * KVS;    // tokens staged per barrier
    constexpr int PK = TT * (D / 8) / kPThreads;    // 16-byte packets per thread and tile, for K and for V
    constexpr int kTileHalfs = TT * KP + TT * VP;
    constexpr int kMergeFloats = KVS > 1 ? (KVS / 2) * QW * 64 * (DB * 16 + 2) : 0;   // one merge round: half of the KV groups write
    static_assert(2 * kTileHalfs * 2 >= kMergeFloats * 4, "the states to merge fit the tiles");
    __shared__ __align__(16) unsigned char smem[2 * kTileHalfs * 2];         // two tiles [K rows | V rows]
    uint16_t *const tiles = reinterpret_cast<uint16_t *>(smem);

    const SeqInfo si = seq_info(st, blockIdx.z);
    const int qt = gridDim.y - 1 - blockIdx.y;
    const int rows = min(kQB, si.q_len - qt * kQB);
    if (rows <= 0) return;                                        // uniform for the workgroup
    // heads in an order that deals the KV heads out to the XCDs (workgroups go to them round-robin): the query heads of a KV head meet
    // in one L2
    const int kvh = blockIdx.x % g, head = kvh * (h / g) + blockIdx.x / g;
    if (si.q_len == 1 && stream_rows) {
        decode_row<D, NWV>(q + (size_t)si.q_start * q_stride + (size_t)head * D, kc, vc, out + ((size_t)si.q_start * h + head) * D, si, h, g, kvh, cap,
                           reinterpret_cast<float *>(smem));
        return;
    }
    const int past = si.kv_len - si.q_len;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, qw = wave % QW, kg = wave / QW;
    const int i32 = lane & 31, hf = lane >> 5;
    const int pos_block_max = past + qt * kQB + rows - 1;         // last token any query of the workgroup attends to
    const int wave_rows = min(WQ, rows - qw * WQ);              // <= 0: the wavefront only helps staging
    const int pos_wave_max = wave_rows > 0 ? past + qt * kQB + qw * WQ + wave_rows - 1 : -1;
    const int pos_wave_min = past + qt * kQB + qw * WQ;            // position of the wavefront's first query
    const float scale = 1.0f / sqrtf((float)D), c = scale * 1.44269504088896340736f, slack = 6.0f * sqrtf((float)D);

    // ---- Q fragments (B operand of K Q^T): lane owns query i32 of each 32-query sub-tile, 8 d-values per k step ----
    half8_t qf[KS];
    const int local = qw * WQ + i32, pos_q = past + qt * kQB + local;
    {
        const int row = si.q_start + qt * kQB + min(local, rows - 1);
        const uint16_t *src = q + (size_t)row * q_stride + (size_t)head * D + hf * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const half8_t *)(src + ks * 16);
    }

    float16_t O[DB];
    float m_run = -INFINITY, l_run = 0.0f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[db][v] = 0.0f;

    // ---- KV tile staging ----
    const size_t slot_base = (size_t)si.slot * cap;
    const int t_last = si.kv_len - 1;
    u32x4_t kreg[PK], vreg[PK];
    auto tile_load = [&](int t0) {
#pragma unroll
        for (int p = 0; p < PK; ++p) {
            const int pk = tid + p * kPThreads, r = pk / (D / 8), c = pk % (D / 8);
            const size_t at = ((slot_base + min(t0 + r, t_last)) * g + kvh) * D + c * 8;
            kreg[p] = *(const u32x4_t *)(kc + at);
            vreg[p] = *(const u32x4_t *)(vc + at);
        }
    };
    auto tile_store = [&](int b) {
        uint16_t *const Ks = tiles + b * kTileHalfs, *const Vs = Ks + TT * KP;
#pragma unroll
        for (int p = 0; p < PK; ++p) {
            const int pk = tid + p * kPThreads, r = pk / (D / 8), c = pk % (D / 8);
            *(u32x4_t *)(Ks + r * KP + c * 8) = kreg[p];
            *(u32x4_t *)(Vs + r * VP + c * 8) = vreg[p];
        }
    };

    // lane roles of the transpose read: lane r of a 16-lane block addresses V[.. + r/4][.. + 4 (r%4)]
    const int tr_row = hf * 4 + ((lane & 15) >> 2), tr_col = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;

    // The two products of a sub-tile are KS MFMAs each (KS = 2 DB), and an LDS read takes as long as three or four of them: the
    // operands of all products of a step are one stream of reads that runs PD MFMAs ahead of its use, across the softmax between
    // the products.  (With the reads one MFMA ahead the matrix pipe was busy 30 % of the time, the wavefronts waiting 41 %.)
    constexpr int PD = 4;
    half8_t ring[PD];
    auto read_k = [&](const uint16_t *Kb, int i) { return *(const half8_t *)(Kb + i32 * KP + hf * 8 + i * 16); };
    auto read_v = [&](const uint16_t *Vb, int i) {
        const uint16_t *vp = Vb + ((i / DB) * 16 + tr_row) * VP + (i % DB) * 32 + tr_col;
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t *)vp);
        const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t *)(vp + 8 * VP));
        return __builtin_bit_cast(half8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // S^T = K Q^T; next(i): operand i of whatever follows this product
    auto scores = [&](const uint16_t *Kb, float16_t &S, const auto &next) {
#pragma unroll
        for (int v = 0; v < 16; ++v) S[v] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            S = __builtin_amdgcn_mfma_f32_32x32x16_f16(ring[ks % PD], qf[ks], S, 0, 0, 0);
            ring[ks % PD] = ks + PD < KS ? read_k(Kb, ks + PD) : next(ks + PD - KS);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // O^T += V^T P^T
    auto accumulate = [&](const uint16_t *Vb, const half8_t *pf) {
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            O[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ring[i % PD], pf[i / DB], O[i % DB], 0, 0, 0);
            if (i + PD < KS) ring[i % PD] = read_v(Vb, i + PD);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto mask = [&](int t0, float16_t &S) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (t0 + 8 * (v >> 2) + 4 * hf + (v & 3) > pos_q) S[v] = -INFINITY;
    };
    // Online softmax of one sub-tile in two parts: the reference point, then the exponentials (P^T packed as the B operand of the
    // second product).  Everything stays in units of the raw scores, the softmax scale and log2(e) are one factor c of the
    // multiply-add in front of the exponential: exp(scale (s - m)) = exp2(c s - c m).  c m is rounded, so the largest exponent is
    // off zero by up to half a unit in the last place of c m: 2^-17 (5e-6 of a weight, the same for all weights of the row) up to
    // c m = kFar, but 16 and more from 2^28 on, past the fp16 range of P.  Beyond kFar the reference is subtracted from the scores
    // first, which is exact for the largest one (a subtraction more per score in all steps took 2 to 3 % at n = 4096).
    constexpr float kFar = 256.0f;
    auto reference = [&](const float16_t &S, float &cm, float &alpha) {
        float mx = fmaxf(S[0], S[1]);
#pragma unroll
        for (int v = 2; v < 16; ++v) mx = fmaxf(mx, S[v]);
        const float2 both = pair_xor32(mx);
        mx = fmaxf(both.x, both.y);
        // The reference point of the exponentials only has to stay within reach of the true maximum: it is moved (and O, l
        // rescaled) when the scaled maximum has grown by more than 6, so that most tiles skip the rescaling of the
        // 32 x d accumulator.  exp(6) stays far inside fp16 for P and fp32 for l.
        const bool move = mx > m_run + slack;                     // first tile: m_run = -inf -> always
        const float m_new = move ? mx : m_run;                    // finite from the first tile on: token 0 is visible
        // a KV group's first sub-tiles can be masked entirely for the earlier queries of the wavefront: no reference yet,
        // every weight is exp(-inf - 0) = 0 and the state stays empty
        cm = m_new == -INFINITY ? 0.0f : c * m_new;
        alpha = move ? __builtin_amdgcn_exp2f(c * (m_run - m_new)) : 1.0f;      // exp2(-inf) = 0 on the first tile
        l_run *= alpha;
        m_run = m_new;
        return move;
    };
    auto weights = [&](const float16_t &S, float cm, half8_t *pf) {
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(c, S[v], -cm)), p1 = __builtin_amdgcn_exp2f(fmaf(c, S[v + 1], -cm));
            l_run += p0;
            l_run += p1;
            const half2_t h = __builtin_convertvector(float2_t{p0, p1}, half2_t);
            pf[v >> 3][v & 7] = h.x, pf[v >> 3][(v & 7) + 1] = h.y;
        }
    };
    // rare: the reference has moved, or lies beyond kFar (then the scores become differences and cm 0)
    auto rescale = [&](bool move, float alpha, float16_t &S, float &cm) {
        const bool far = fabsf(cm) > kFar;
        if (__any(move || far)) {
            const float off = far ? m_run : 0.0f;
            cm = far ? 0.0f : cm;
#pragma unroll
            for (int v = 0; v < 16; ++v) S[v] -= off;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) O[db][v] *= alpha;
        }
    };
    tile_load(0);
    tile_store(0);
    lds_barrier();
    int buf = 0;
    for (int tb = 0; tb <= pos_block_max; tb += TT) {
        const bool more = tb + TT <= pos_block_max;               // uniform for the workgroup
        tile_load(tb + TT);
        const uint16_t *Kb = tiles + buf * kTileHalfs + kg * kTB * KP, *Vb = tiles + buf * kTileHalfs + TT * KP + kg * kTB * VP;
        const int t0 = tb + kg * kTB;                             // this wavefront's sub-tile
        if (t0 <= pos_wave_max) {                                 // wavefront-uniform, like every branch here
            float16_t S;
            half8_t p[2];
            float cm, alpha;
#pragma unroll
            for (int i = 0; i < PD; ++i) ring[i] = read_k(Kb, i);
            scores(Kb, S, [&](int i) { return read_v(Vb, i); });
            if (t0 + kTB - 1 > pos_wave_min) mask(t0, S);
            const bool move = reference(S, cm, alpha);            // writes alpha: a statement of its own, ahead of its use
            rescale(move, alpha, S, cm);
            weights(S, cm, p);
            accumulate(Vb, p);
        }
        buf ^= 1;
        if (more) tile_store(buf);
        lds_barrier();                                            // the next tile is there, and this one consumed
    }

    // ---- merge the KV groups of each query group: log2(KVS) rounds, the upper half of the groups hands its state to the lower half ----
    if (KVS > 1) {
        float *const mg = reinterpret_cast<float *>(smem);        // [writer wavefront][value][lane]: the tiles are consumed
        constexpr int kVals = DB * 16 + 2;
#pragma unroll
        for (int half = KVS / 2; half >= 1; half >>= 1) {
            if (kg >= half && kg < 2 * half) {
                float *dst = mg + ((size_t)((kg - half) * QW + qw) * kVals) * 64 + lane;
                dst[0] = m_run, dst[64] = l_run;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) dst[(2 + db * 16 + v) * 64] = O[db][v];
            }
            __syncthreads();
            if (kg < half) {
                const float *src = mg + ((size_t)(kg * QW + qw) * kVals) * 64 + lane;
                const float mb = src[0], lb = src[64];
                const float mn = fmaxf(m_run, mb);
                const float ca = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(c * (m_run - mn));
                const float cb = mb == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(c * (mb - mn));
                l_run = l_run * ca + lb * cb;
                m_run = mn;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) O[db][v] = O[db][v] * ca + src[(2 + db * 16 + v) * 64] * cb;
            }
            __syncthreads();
        }
        if (kg != 0) return;
    }

    // ---- normalise and store: lane holds query i32; register v of block db is d = 32 db + 8 (v/4) + 4 hf + v%4 ----
    const float l_tot = xor32_sum(l_run);
    if (local >= rows) return;
    const float inv = 1.0f / l_tot;
    uint16_t *dst = out + (size_t)(si.q_start + qt * kQB + local) * ((size_t)h * D) + (size_t)head * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int b4 = 0; b4 < 4; ++b4) {
            const int dd = db * 32 + b4 * 8 + hf * 4;
            const uint32_t w0 = f2h(O[db][b4 * 4] * inv) | ((uint32_t)f2h(O[db][b4 * 4 + 1] * inv) << 16);
            const uint32_t w1 = f2h(O[db][b4 * 4 + 2] * inv) | ((uint32_t)f2h(O[db][b4 * 4 + 3] * inv) << 16);
            *(uint2 *)(dst + dd) = make_uint2(w0, w1);
        }
}

template <int D, int NWV, int KVS, int MINW>
hipError_t launch_one(const uint16_t *q, int32_t q_stride, const relax_kv_cache &cache, const relax_layer_dims &dm, const SeqTable &st, uint16_t *out,
                      hipStream_t stream)
{
    const int queries = NWV / KVS * 32;
    const dim3 grid(dm.n_heads, (st.q_max + queries - 1) / queries, st.B);
    // attend_tokens: 32-bit byte offsets inside a slot of the cache, and the two steps of all wavefronts that it counts past the end
    const int stream_rows = ((size_t)dm.kv_capacity + 1024) * dm.n_kv_heads * D * 2 < ((size_t)1 << 31);
    hipLaunchKernelGGL((attn_prefill_kernel<D, NWV, KVS, MINW>), grid, dim3(64 * NWV), 0, stream, q, q_stride, cache.k, cache.v, out, st, dm.n_heads,
                       dm.n_kv_heads, dm.kv_capacity, stream_rows);
    return hipGetLastError();
}

}  // namespace

bool attn_prefill_supported(const relax_layer_dims &dm) { return dm.head_dim == 128 || dm.head_dim == 64; }

hipError_t launch_attention_prefill(const uint16_t *q, int32_t q_stride, const relax_kv_cache &cache, const relax_layer_dims &dm,
                                    const SeqTable &st, int32_t L_max, uint16_t *out, hipStream_t stream)
{
    // A call whose tiles of 64 queries leave no CU with two takes them, with 4 KV groups (tiles of 128 tokens, 152 KB; heads of 64: 86 KB): half the
    // steps of the longest prefix, and the CUs it takes stood idle (us, 128 queries x 2 groups / 64 x 4: 7B heads, 100 rows on 0, 500 and 1500
    // cached tokens 9.1 / 8.2, 17.2 / 14.4, 32.8 / 27.5; 511 rows 16.1 / 13.8, 25.4 / 21.9, 40.6 / 33.3; 32 / 8 heads of 64, 300 rows on 1500 27.0 /
    // 18.9).  One more tile per CU and the other form is the faster one (7B heads, 700 rows on 1500 42.7 / 56.1), as it is on short
    // prefixes of up to 64 queries, where both have one tile (7B heads, 64 rows with a total of 200, 400, 450, 640 and 1000 tokens 10.0 / 10.5, 13.0 /
    // 13.6, 13.9 / 13.8, 16.0 / 15.7, 21.6 / 20.1; 17 rows 8.9 / 9.2, 12.0 / 12.1, 13.0 / 12.5, 15.0 / 14.2, 20.6 / 18.8): from seven tiles of 64 tokens
    // on.  Heads of 64 gain earlier (32 / 8, 64 rows, 400 tokens 9.2 / 8.3).
    const long long tiles = (long long)dm.n_heads * st.B * ((st.q_max + 63) / 64);
    if (tiles <= 256 && (st.q_max > 64 || L_max >= (dm.head_dim == 64 ? 400 : 449))) {
        if (dm.head_dim == 128) return launch_one<128, 8, 4, 2>(q, q_stride, cache, dm, st, out, stream);
        if (dm.head_dim == 64) return launch_one<64, 8, 4, 2>(q, q_stride, cache, dm, st, out, stream);
    }
    // 8 wavefronts = 4 query groups of 32 x 2 KV groups, two tiles of 64 tokens in LDS (76 KB; heads of 64: 43 KB).  Measured, against one
    // tile of 64 tokens with the softmax in units of e and masks on every tile, and against two tiles of 128 tokens (152 KB, 86 KB):
    //   4096 rows, 32 / 8 heads of 128               181 us   214   188
    //   2048 rows, 32 / 32 heads of 128               55       64    57
    //   64 x 20 rows on 300 cached tokens, 32 / 32    96       97   105
    //   16 x 1 row on 100..2000 tokens beside 16     113      114   121
    //   64 x 20 rows, 32 / 8 heads of 64            16.9     18.2  25.8
    //   64 x 100 rows on 200 cached, 32 / 8, 64       43       50    68
    // Long tiles lose on cached prefixes (bursts of loads, part of the last tile empty) and, with heads of 64, the second workgroup of
    // a CU.  One buffer instead of two: the 64-row call on 2000 cached tokens 41.7 instead of 37.9 us.  With the loads of the next
    // tile left out 4096 rows took 178 us of 200 in an earlier form, without its stores too 162: matrix pipe and vector unit together
    // are busy 70 % of the time at two wavefronts per SIMD.  Ordering the exponentials of one sub-tile between the MFMAs of another
    // changed nothing.  Earlier forms at n = 2048: without the KV groups 82-84 us, 64 queries per wavefront 128 us, 64 queries per
    // workgroup 93-117 us.
    if (dm.head_dim == 128) return launch_one<128, 8, 2, 2>(q, q_stride, cache, dm, st, out, stream);
    if (dm.head_dim == 64) return launch_one<64, 8, 2, 4>(q, q_stride, cache, dm, st, out, stream);
    return hipErrorInvalidValue;
}

}  // namespace relax
