// Row pass over a score block in memory, shared by the launch of its own (block_small.hip) and the one that it shares with the sorts of
// the step's row ids (sparse_adam.hip): loss statistics of a row of S and their finish; with C the row's coefficients, fp32 or two bf16
// pieces (C may be S itself: a thread overwrites what it has read).
#pragma once
#include "block_kernel.hpp"
#include "prep_kernels.h"
#include "row_finish.hpp"

struct KgeSmallRowsShared { float red[4][4], fb; };
// 256 threads (tid) and `sh` per row; a workgroup may hold several such groups, all of which pass the same barriers.  Rows past B get what
// kge_rowfinish_kernel gives them, groups past Bp do nothing.
__device__ __forceinline__ void kge_small_rows_body(const int b, const int tid, KgeSmallRowsShared &sh, const KgeSmallRowsArgs &a) {
    const int lane = tid & 63, wave = tid >> 6, N = a.N, loss = a.loss;
    const bool live = b < a.B;
    const int npad = (N + 31) / 32 * 32;
    auto put = [&](int n, float c) -> float {                   // returns what the contraction over the negatives sees of it
        uint32_t w = __float_as_uint(c);
        if (a.bf16) {
            const __bf16 x0 = (__bf16)c, x1 = (__bf16)(c - (float)x0);
            w = (uint32_t)__builtin_bit_cast(uint16_t, x0) | (uint32_t)__builtin_bit_cast(uint16_t, x1) << 16;
            c = (float)x0 + (float)x1;
        }
        a.C[(size_t)b * a.ldS + n] = w;
        return c;
    };
    if (!live && b < a.Bp) {
        if (tid == 0) { a.lossb[b] = 0.f; a.gpos[b] = 0.f; a.rowinfo[b].K = -INFINITY; }
        if (a.C && b < (a.B + 31) / 32 * 32) for (int n = tid; n < npad; n += 256) put(n, 0.f);
    }
    const float xscale = (loss == KGE_LOGSIGMOID ? a.adv_temp : 1.f) * KGE_LOG2E;
    const float *row = a.S + (size_t)(live ? b : 0) * a.ldS;
    constexpr int R = 8;                                        // scores that a thread keeps (2,048 negatives)
    float v[R];
#pragma unroll
    for (int j = 0; j < R; ++j) { const int n = tid + 256 * j; v[j] = live && n < N ? row[n] : -INFINITY; }
    const float fp = live ? a.pos[b] : 0.f;
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < R; ++j) m = fmaxf(m, v[j]);
    const int n_more = live ? N : 0;                            // (negatives past those)
    for (int n = tid + 256 * R; n < n_more; n += 256) m = fmaxf(m, row[n]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (lane == 0) sh.red[0][wave] = m;
    __syncthreads();
    const float s_max = fmaxf(fmaxf(sh.red[0][0], sh.red[0][1]), fmaxf(sh.red[0][2], sh.red[0][3]));
    m = s_max > -INFINITY ? s_max * xscale : -INFINITY;
    const float m_neg = m > -INFINITY ? -m : 0.f;               // (a row of nothing but -inf: every weight 0)
    // m is rounded, s xscale below is not: the largest score's own weight would be off by more than a factor of two beyond 2^24, and
    // nothing or infinite beyond 2^31; there its remainder is taken from every exponent (not without C: who makes the coefficients
    // elsewhere, from K, has the same rounding in K)
    const float rest = fmaf(s_max, xscale, m_neg), rem = a.C && fabsf(rest) > 1.f && fabsf(rest) < INFINITY ? rest : 0.f;
    auto weight = [&](float s) { return kge_exp2(fmaf(s, xscale, m_neg) - rem); };       // relative to the largest: at most about 1
    float l = 0.f, ac = 0.f;
    auto add = [&](float s) {
        const float e = weight(s);
        l += e;
        if (loss == KGE_LOGSIGMOID) {
            const float y = a.gamma + s, t = kge_exp2(-fabsf(y) * KGE_LOG2E);
            if (e > 0.f) ac = fmaf(e, fmaxf(y, 0.f) + KGE_LN2 * kge_log2(1.f + t), ac);
        }
    };
#pragma unroll
    for (int j = 0; j < R; ++j) if (live && tid + 256 * j < N) add(v[j]);
    for (int n = tid + 256 * R; n < n_more; n += 256) add(row[n]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { l += __shfl_xor(l, o); ac += __shfl_xor(ac, o); }
    if (lane == 0) { sh.red[1][wave] = l; sh.red[2][wave] = ac; }
    __syncthreads();
    if (live && tid == 0) {
        l = (sh.red[1][0] + sh.red[1][1]) + (sh.red[1][2] + sh.red[1][3]);
        ac = (sh.red[2][0] + sh.red[2][1]) + (sh.red[2][2] + sh.red[2][3]);
        const KgeRowFinish o = kge_rowfinish_merged(m, l, ac, N, loss, a.gamma, a.c_corr, a.scale, fp);
        a.lossb[b] = o.L; a.gpos[b] = o.gp; a.rowinfo[b].K = o.K;
        sh.fb = l > 0.f ? a.scale * o.share / l : 0.f;
    }
    if (!a.C) return;
    __syncthreads();
    const float f = sh.fb;                                         // dL / d(score) of a weight of 1 (log-sigmoid: times sigma(gamma + s))
    float csum = 0.f;
    auto coef = [&](int n, float s) {
        float w = weight(s) * f;
        if (loss == KGE_LOGSIGMOID) {
            const float y = a.gamma + s;
            const float t = kge_exp2(-fabsf(y) * KGE_LOG2E), rcp = __builtin_amdgcn_rcpf(1.f + t);
            w *= y >= 0.f ? rcp : t * rcp;
        }
        if (a.dist) w = s < 0.f ? w * __builtin_amdgcn_rcpf(-s) : 0.f;
        csum += put(n, w);
    };
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int n = tid + 256 * j;
        if (live && n < N) coef(n, v[j]); else if (live && n < npad) put(n, 0.f);
    }
    for (int n = tid + 256 * R; n < (live ? npad : 0); n += 256) { if (n < N) coef(n, row[n]); else put(n, 0.f); }
    if (a.dist) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) csum += __shfl_xor(csum, o);
        if (lane == 0) sh.red[3][wave] = csum;
        __syncthreads();
        for (int s = tid; s < (live ? a.q_splits : 0); s += 256)    // (the whole sum with the first split's partial rows)
            a.sumq[(size_t)s * a.Bp + b] = make_float4(s == 0 ? (sh.red[3][0] + sh.red[3][1]) + (sh.red[3][2] + sh.red[3][3]) : 0.f, 0.f, 0.f, 0.f);
    }
}
