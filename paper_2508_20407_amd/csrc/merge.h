// Exact merge of attention partials by their log-sum-exp statistics.
//
// A partial s of a query row is (O_s, m_s, l_s): O_s = sum_j 2^(x_j - m_s) V_j and
// l_s = sum_j 2^(x_j - m_s) over the keys j of that partition, with x_j the logit in base-2
// units.  Softmax attention over the union of the partitions (the single softmax of Section
// 3's formula) is
//     O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s,      M = max_s m_s.
// The history axis split into partitions uses this; so does the JOINT layer, where the window
// causal partial is one more partition.  The SUM layer normalises the history partitions and
// the window partial separately and adds the two outputs.
#pragma once
#include "common.h"

namespace tlin {

// SL threads ("slot lanes") share one (row, 4 columns) item: lane sl takes the partials
// sl, sl + SL, ..., and the SL running results are joined, inside a wave by exchanges, over the waves of
// a row through LDS.  With many partitions the kernel is bound by the latency of its loads, not by
// bytes: the partials of a row are spread over threads, and a thread requests the statistics and the
// values of four partials at once, before it has seen a maximum (85 partials of 12 rows of 36 columns:
// 10.4 -> 4.7 us; 16 partials of 2048 rows of 64: 6.7 -> 4.7 us).
template <int D, int SL>
__global__ __launch_bounds__(D / 4 * SL > 256 ? D / 4 * SL : 256) void merge_kernel(const MergeArgs a)
{
    constexpr int TPR = D / 4;                 // column groups per row, 4 columns each
    constexpr int NT = TPR * SL > 256 ? TPR * SL : 256;
    constexpr int RPB = NT / (TPR * SL);       // rows per block
    constexpr int SPW = 64 / TPR;              // slot lanes (or rows) side by side in a wave
    constexpr int NWR = SL / SPW;              // waves that share a row (0: a wave holds several rows)
    static_assert(NT <= 1024 && (SL == 1 || SL % SPW == 0), "a row takes whole waves, at most a block");
    __shared__ float red[NWR > 1 ? NT / 64 * TPR * 6 : 1];

    const int tid = threadIdx.x;
    const int cg = tid % TPR, sl = (tid / TPR) % SL, rb = tid / (TPR * SL);
    const int64_t grow = (int64_t)blockIdx.x * RPB + rb;          // flat row index over (b,h,row)
    const bool live = grow < a.total_rows;
    const int c4 = cg * 4;
    // Sliding schedule: the row belongs to chunk orow / W of its head, the partials of a chunk sit
    // in its own group of slots, and chunk 0 has no history partials.
    const int rows_per_head = a.nchunks ? a.seq_rows : a.W;
    const int bh = live ? (int)(grow / rows_per_head) : 0, orow = live ? (int)(grow % rows_per_head) : 0;
    const int chunk = a.nchunks ? orow / a.W : 0;
    const int row = orow - chunk * a.W;
    const int b = bh / a.H, hd = bh % a.H;
    const int64_t slot0 = ((int64_t)bh * (a.nchunks ? a.nchunks : 1) + chunk) * a.nparts;
    const int nhist = (a.nchunks && chunk == 0) ? 0 : a.nhist;
    const int64_t wslot = slot0 + a.nhist;             // the window partial's slot
    // columns beyond the tensors' head dimension are neither in the partials nor stored
    const int njoint = live && c4 < a.D ? nhist + ((a.has_window && a.joint) ? 1 : 0) : 0;
    // joint slots: the history partials, then (JOINT) the window partial
    auto slot_of = [&](int s) { return s < nhist ? slot0 + s : wslot; };

    // this lane's share of the joint partials, relative to its own maximum
    float M = -INFINITY, den = 0.f;
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    // takes in another share (M2, den2, num2); a share without partials, and an empty partition, hold -inf
    auto join = [&](float M2, float den2, f32x4 num2) __attribute__((always_inline)) {
        const float Mn = fmaxf(M, M2);
        const float w1 = M == -INFINITY ? 0.f : exp2f(M - Mn), w2 = M2 == -INFINITY ? 0.f : exp2f(M2 - Mn);
        den = w1 * den + w2 * den2;
        num = w1 * num + w2 * num2;
        M = Mn;
    };
    constexpr int NB = 4;                      // partials requested at once
    for (int s0 = sl; s0 < njoint; s0 += NB * SL) {
        float ms[NB], ls[NB];
        f32x4 os[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            ms[k] = -INFINITY;
            ls[k] = 0.f;
            os[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (s0 + k * SL < njoint) {
                const int64_t idx = slot_of(s0 + k * SL) * a.W + row;
                ms[k] = a.Mpart[idx];
                ls[k] = a.Lpart[idx];
                os[k] = *(const f32x4 *)(a.Opart + idx * D + c4);
            }
        }
        float Mn = M;
#pragma unroll
        for (int k = 0; k < NB; ++k) Mn = fmaxf(Mn, ms[k]);
        const float w0 = M == -INFINITY ? 0.f : exp2f(M - Mn);
        den *= w0;
        num *= w0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const float w = ms[k] == -INFINITY ? 0.f : exp2f(ms[k] - Mn);     // an empty partition holds -inf and zeros
            den += w * ls[k];
            num += w * os[k];
        }
        M = Mn;
    }
    if (SL > 1) {
#pragma unroll
        for (int off = TPR; off < 64; off *= 2) {
            const float M2 = __shfl_xor(M, off), d2 = __shfl_xor(den, off);
            f32x4 n2;
#pragma unroll
            for (int e = 0; e < 4; ++e) n2[e] = __shfl_xor(num[e], off);
            join(M2, d2, n2);
        }
        if (NWR > 1) {
            // wave w of the row leaves its share for the row's first wave
            const int wave = tid >> 6, lane = tid & 63;
            if (lane < TPR) {
                float *mine = red + (wave * TPR + lane) * 6;
                mine[0] = M; mine[1] = den; mine[2] = num[0]; mine[3] = num[1]; mine[4] = num[2]; mine[5] = num[3];
            }
            __syncthreads();
            if (sl != 0) return;
#pragma unroll
            for (int k = 1; k < NWR; ++k) {
                const float *o = red + ((wave + k) * TPR + cg) * 6;
                join(o[0], o[1], f32x4{o[2], o[3], o[4], o[5]});
            }
        } else if (sl != 0) {
            return;
        }
    }
    if (!live || c4 >= a.D) return;

    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    float lse2 = -INFINITY;
    if (njoint > 0) {
        o = num * (1.0f / den);
        lse2 = M + log2f(den);
    }
    if (a.has_window && !a.joint) {
        const int64_t idx = wslot * a.W + row;
        o += *(const f32x4 *)(a.Opart + idx * D + c4) * (1.0f / a.Lpart[idx]);
    }

    const int64_t off = (int64_t)b * a.o_sb + (int64_t)hd * a.o_sh + (int64_t)orow * a.o_sr + c4;
    if (a.out_bf16) {
        bf16x4 ob;
#pragma unroll
        for (int e = 0; e < 4; ++e) ob[e] = (__bf16)o[e];
        *(bf16x4 *)((__bf16 *)a.O + off) = ob;
    } else {
        *(f32x4 *)((float *)a.O + off) = o;
    }
    if (a.lse && c4 == 0) a.lse[grow] = lse2 * 0.6931471805599453f;
}

}  // namespace tlin
