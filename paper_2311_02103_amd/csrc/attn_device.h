// Device functions of the attention kernels that stream a decode row's keys and values (attn_decode.hip, attn_prefill.hip).
#pragma once

#include "relax_common.h"

namespace relax {

typedef uint32_t u32x4a_t __attribute__((ext_vector_type(4)));
typedef _Float16 half2a_t __attribute__((ext_vector_type(2)));

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

template <bool NT>
__device__ __forceinline__ u32x4a_t row_load(const char *p)
{
    return NT ? stream_load((const u32x4a_t *)p) : *(const u32x4a_t *)p;
}

// One wavefront's share of tokens t_begin .. t_end - 1 of one query against one KV head: the softmax state (m, l) and the un-normalised
// accumulator of elements 8 (lane % (D / 8)) .. + 7, the same in all lanes of a group.  kslot, vslot: token 0 of the slot at the head;
// row_bytes: one token of the cache, all heads.  load_q is asked for the lane's eight query elements behind the first requests.  NT: the
// rows are read by this workgroup alone.  NL: K (and V) loads per step.
template <int D, int WAVES, int NL, bool NT, typename LoadQ>
__device__ __forceinline__ void attend_tokens(const char *kslot, const char *vslot, uint32_t row_bytes, int t_begin, int t_end, int wave, int lane,
                                              const LoadQ &load_q, float &m_out, float &l_out, float (&acc_out)[8])
{
    constexpr int LPT = D / 8;        // lanes that share one token (each owns 8 of its d elements)
    constexpr int TPW = kWave / LPT;  // tokens per load instruction of a wavefront
    constexpr int TS = NL * TPW;      // tokens per wavefront step
    const int sub = lane / LPT, e0 = (lane % LPT) * 8;
    const float inv_sqrt_d = 1.0f / sqrtf((float)D);

    // step s of this wavefront covers tokens t_begin + (WAVES s + wave) TS .. + TS - 1
    const int first = t_begin + wave * TS;
    const int ns = first < t_end ? (t_end - first + WAVES * TS - 1) / (WAVES * TS) : 0;
    // Addresses: a uniform base per (slot, head) plus a 32-bit byte offset per lane that K and V share (the launcher
    // checks that a slot of the cache stays under 2 GiB).  The offsets of a step are those of the step before plus a
    // constant, clamped to the last token of the split: two vector instructions per K / V pair instead of a 64-bit
    // multiply-add each, ahead of the first request as well as in the stream.
    const uint32_t last_off = (uint32_t)(t_end - 1) * row_bytes + (uint32_t)e0 * 2;
    const uint32_t step_bytes = WAVES * TS * row_bytes;
    uint32_t run[NL];                                          // offsets of the next step to request, not clamped
#pragma unroll
    for (int j = 0; j < NL; ++j) run[j] = (uint32_t)(first + sub + j * TPW) * row_bytes + (uint32_t)e0 * 2;

    struct Step {
        u32x4a_t k[NL], v[NL];
    };
    // requests step s; the calls come in the order s = 0, 1, 2, ..
    auto step_load = [&](Step &sp, int) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const uint32_t at = min(run[j], last_off);         // tokens past the end re-read the last one, masked below
            sp.k[j] = row_load<NT>(kslot + at);
            sp.v[j] = row_load<NT>(vslot + at);
            run[j] += step_bytes;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    Step sa, sb;
    step_load(sa, 0);
    step_load(sb, 1);
    const u32x4a_t qv = load_q();

    // locals: on the references the compiler pairs other products and sums into multiply-adds, and takes three registers more
    float acc[8], m = -INFINITY, l = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;

    auto consume = [&](const Step &sp, int s) {
        const int t0 = first + s * WAVES * TS + sub;
        float sc[NL];
        float mx = m;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            float dot = 0.0f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t kw = sp.k[j][w], qw = qv[w];    // element copies: a bit_cast applied to the subscript itself reads word 0
                dot = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2a_t, kw), __builtin_bit_cast(half2a_t, qw), dot, false);
            }
            dot += dpp_f<0xB1>(dot);                           // lane ^ 1
            dot += dpp_f<0x4E>(dot);                           // lane ^ 2
            if (LPT == 16) {
                dot += dpp_f<0x124>(dot);                      // rotate the row of 16 by 4, then by 8
                dot += dpp_f<0x128>(dot);
            } else {
                dot += dpp_f<0x141>(dot);                      // mirror within the half row of 8
            }
            sc[j] = (t0 + j * TPW < t_end) ? dot * inv_sqrt_d : -INFINITY;
            mx = fmaxf(mx, sc[j]);
        }
        const float mref = (mx == -INFINITY) ? 0.0f : mx;      // nothing valid yet: every weight below is exp(-inf) = 0
        const float ca = __expf(m - mref);
        float p[NL], psum = 0.0f;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            p[j] = __expf(sc[j] - mref);
            psum += p[j];
        }
        l = l * ca + psum;
        m = mx;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= ca;
#pragma unroll
        for (int j = 0; j < NL; ++j)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t vw = sp.v[j][w];
                const half2a_t vv = __builtin_bit_cast(half2a_t, vw);
                acc[2 * w] += p[j] * (float)vv.x;
                acc[2 * w + 1] += p[j] * (float)vv.y;
            }
    };

    const int nq = ns >> 1;
    int s = 0;
#pragma unroll 1
    for (; s + 2 < 2 * nq; s += 2) {
        consume(sa, s);
        step_load(sa, s + 2);
        consume(sb, s + 1);
        step_load(sb, s + 3);
    }
    if (nq > 0) {
        if (ns & 1) {
            consume(sa, s);
            step_load(sa, s + 2);
            consume(sb, s + 1);
            consume(sa, s + 2);
        } else {
            consume(sa, s);
            consume(sb, s + 1);
        }
    } else if (ns == 1) {
        consume(sa, 0);
    }

    // merge the TPW token groups of the wavefront (lanes that own the same 8 elements)
#pragma unroll
    for (int off = LPT; off < kWave; off <<= 1) {
        float mb = __shfl_xor(m, off, kWave), lb = __shfl_xor(l, off, kWave), accb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) accb[e] = __shfl_xor(acc[e], off, kWave);
        const float mn = fmaxf(m, mb), sa = m == -INFINITY ? 0.0f : __expf(m - mn), sb = mb == -INFINITY ? 0.0f : __expf(mb - mn);
        l = fmaf(l, sa, lb * sb);                              // multiply-adds written out: which product is rounded is not the compiler's choice
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(accb[e], sb, acc[e] * sa);
        m = mn;
    }
    m_out = m, l_out = l;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc_out[e] = acc[e];
}

}  // namespace relax
