// Both passes of kge_loss_bwd for small blocks (2-norm and bilinear scorers, all but TransH): the score block is written to memory.
//
// A micro-batch of a few hundred triples and negatives (Table 3 trains with B 256-640, N 256-1,536) leaves the chip idle: the
// block kernels own 128 rows per workgroup, so the streamed operand is cut into one or two tiles per workgroup, and what a pass
// takes is not its contractions but the fixed part of a workgroup, the split partials it writes (128 rows x d fp32 each, 20-30 MB
// for any batch) and the reads of dozens of partials per row in the chain rule.  While B x N fp32 scores stay in the L2 the job
// is better cut differently:
//   scores      S[b, n], one 32 x 32 tile per wave, operands straight from memory (both are contiguous along d)
//   rows        one workgroup per query: loss, gradient of the positive score and the coefficients C[b, n] = dL/dS[b, n] (distance
//               scorers: over the distance) from its row of S; once per pair - made from S and a row constant by every workgroup of
//               the gradients, the exponentials bound that launch (a third more time for the RotatE case below)
//   gradients   one launch for both operands: dQ = C T and dT = C^t Q; a workgroup makes 32 rows x 64 or 128 columns, its eight waves
//               share out the contraction index and add up through the LDS, so that there are no partials in memory
// (kge_loss_bwd, block kernels / here: RotatE fp32, B 448, N 1,088, d 256: 108 / 44 us; ComplEx bf16, B 640, N 1,536, d 400: 112 / 39 us.)
// What bounds each launch is its latency: start-up, two or three dependent loads and the matrix instructions of one wave.
// Arithmetic: bf16 operands with fp32 accumulation, or three bf16 pieces per fp32 value.  On bf16 tables the coefficients are
// finished when they are made, where the block kernels round the weight relative to a row reference (the dominating pairs are 1 and
// round to themselves) and apply the normaliser in fp32; so dQ takes every coefficient as TWO bf16 pieces, 17 significand bits, and its
// error stays below theirs.  dT takes the first piece alone, as their pass over the negatives does; the sum of a negative's
// coefficients (distance scorers) both, so that the rounding stays on the queries (rounded sums: dT's error 6-22 % larger).
#include "block_kernel.hpp"
#include "prep_kernels.h"
#include "small_rows.hpp"

namespace {

constexpr int SMALL_AHEAD = 2;         // matrix steps of the gradients in flight (3: the same time, 1-4 % slower for rows of 1,024 bytes)

struct SmallArgs {
    const void *Q, *T;                 // [Bp][dp] queries, [Np][dp] negatives (rows past B, N and columns past d are zero)
    const KgeRowInfo *rowinfo;         // [Bp]
    const float *tn;                   // [Np] squared norms of the negatives
    float *S; int64_t ldS;             // [Bp][ldS] scores (written for b < B, n < N only)
    const uint32_t *C;                 // [Bp][ldS] coefficients (zero behind the block up to a multiple of 32): fp32, or two bf16 pieces
                                       // (low half + high half) on bf16 tables
    int32_t B, N, Bp, Np, dp, dim;
    float *accq, *acct;                // [q_splits][Bp][dp], [t_splits][Np][dp] gradient rows (columns < dim rounded up to a tile)
    float4 *sumt;                      // [t_splits][Np] {sum of the coefficients of the column, 0, 0, 0}: distance scorers
    int32_t q_blocks, d_tiles;         // gradient launch: workgroups of the queries' part, column tiles
    int32_t q_splits, t_splits, q_steps, t_steps;   // ... splits of the contraction index, matrix steps of sixteen per split
};

// eight consecutive values of a row as one operand of a 16-deep matrix step: a bf16 fragment or three bf16 pieces
template <bool BF16> struct Frag;
template <> struct Frag<true> { uint4 v; };
template <> struct Frag<false> { KgeP3 v; };
template <bool BF16> __device__ __forceinline__ kge_f32x16 small_mma(kge_f32x16 acc, const Frag<BF16> &a, const Frag<BF16> &b) {
    if constexpr (BF16) return kge_mma16<true>(acc, a.v, b.v);
    else return kge_mma3(acc, a.v, b.v);
}

// ---- scores: workgroup = 64 queries x 64 negatives, wave = 32 x 32 ----
// The workgroup's 128 rows come into the LDS in NCH pieces of 256 bytes a row, all of them requested at once by asynchronous copies
// (four rows of a piece per instruction); the matrix steps of a piece run while the later ones are under way.  Operands taken straight
// from memory, 32 rows x 32 bytes per load instruction and every row by two waves, were bound by the lines that a load touches:
// ComplEx bf16 640 x 1,536 x 400 12.7 -> 7.4 us, TransE bf16 512 x 1,024 x 256 8.2 -> 5.6, RotatE fp32 448 x 1,088 x 256 12.8 -> 10.4 (12.2
// with one group of four waves).
// Piece: [64 queries, 64 negatives][256 bytes], 16-byte chunk c of row r at position c ^ kge_pl_swz(r).
constexpr int SMALL_PIECE = 128 * 256;
// fp32: two groups of four waves share a tile's steps (the three pieces of every value cost more than the matrix instructions), the
// second hands its sums over through the LDS.
constexpr int small_score_groups(bool bf16) { return bf16 ? 1 : 2; }
template <bool BF16, int KIND, int NCH>
__global__ __launch_bounds__(256 * small_score_groups(BF16)) void small_score_kernel(const SmallArgs a) {
    constexpr int ES = BF16 ? 2 : 4, STEP = 16 * ES, SPP = 256 / STEP;     // bytes of a matrix step of sixteen columns, steps per piece
    constexpr int G = small_score_groups(BF16), IPW = 32 / (4 * G);        // copies per wave and piece
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int lane = threadIdx.x & 63, wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave8 & 3, grp = wave8 >> 2;
    const int lr = lane & 31, g = lane >> 5;
    const int bw = blockIdx.y * 64, nw = blockIdx.x * 64;
    const int b0 = bw + (wave >> 1) * 32, n0 = nw + (wave & 1) * 32;
    // norms of the wave's rows: 32 of the queries, 32 of the negatives
    const uint32_t side = NCH * SMALL_PIECE + wave * 256;
    if constexpr (KIND == KGE_KIND_DIST)
        kge_async_copy4(g == 0 ? (const void *)&a.rowinfo[b0 + lr].qn : (const void *)(a.tn + n0 + lr), lds0 + side);
    const int steps = (a.dim + 15) / 16;                        // (dp is a multiple of 256 (bf16) or 128 columns, zero past d)
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int j = 0; j < IPW; ++j) {
            const int i = j * 4 * G + wave8;                    // rows 4 i .. + 3; i % 4 = wave
            const int chunk = (lane & 15) ^ ((lane >> 4) << 2) ^ wave;
            const char *src = (i < 16 ? (const char *)a.Q + (size_t)(bw + 4 * i) * a.dp * ES : (const char *)a.T + (size_t)(nw + 4 * i - 64) * a.dp * ES) + c * 256;
            // (columns that no step reads stay where they are; every row has some that one does)
            if (c * 256 + chunk * 16 < steps * STEP)
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + c * SMALL_PIECE + i * 1024),
                             "v"((lane >> 4) * a.dp * ES + chunk * 16), "s"(src) : "memory");
        }
    kge_f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    const char *pq = lds + ((wave >> 1) * 32 + lr) * 256, *pt = lds + (64 + (wave & 1) * 32 + lr) * 256;
    const int swz = kge_pl_swz(lr);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        // (piece c of this wave's copies is here when only those of the later pieces are in flight)
        if (c == NCH - 1) kge_wait_vmcnt<0>();
        else if (c == NCH - 2) kge_wait_vmcnt<IPW>();
        else if (c == NCH - 3) kge_wait_vmcnt<2 * IPW>();
        else kge_wait_vmcnt<3 * IPW>();
        __syncthreads();
#pragma unroll
        for (int v = 0; v < SPP / G; ++v) {
            const int u = v * G + grp;
            if (c * SPP + u >= steps) break;
            Frag<BF16> fq, ft;
            auto at = [&](const char *p, int e) { return *(const uint4 *)(p + c * SMALL_PIECE + ((u * ES + g * (ES / 2) + e) ^ swz) * 16); };
            if constexpr (BF16) { fq.v = at(pq, 0); ft.v = at(pt, 0); }
            else { fq.v = kge_split3(at(pq, 0), at(pq, 1)); ft.v = kge_split3(at(pt, 0), at(pt, 1)); }
            acc = small_mma<BF16>(acc, fq, ft);
        }
    }
    if constexpr (G == 2) {
        __syncthreads();                                        // (the pieces are done with)
        float4 *half = (float4 *)lds + wave * 256 + lane;
        if (grp == 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) half[i * 64] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
        }
        __syncthreads();
        if (grp == 1) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 h = half[i * 64];
            acc[4 * i] += h.x; acc[4 * i + 1] += h.y; acc[4 * i + 2] += h.z; acc[4 * i + 3] += h.w;
        }
    }
    if (b0 >= a.B || n0 >= a.N) return;
    // lane = negative n0 + lr; register i = query b0 + 8 (i / 4) + 4 g + i % 4
    const int n = n0 + lr;
    float sv[16];
    if constexpr (KIND == KGE_KIND_MULT) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sv[i] = acc[i];
    } else {
        // |q|^2 + |t|^2 - 2 q.t; entries where it cancels (below 1e-3 of the norms) by direct differences
        const float *norms = (const float *)(lds + side);
        const float tn = norms[32 + lr];
        float d2[16], thr[16];
        bool cancel = false;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float qn = norms[8 * (i >> 2) + 4 * g + (i & 3)];
            d2[i] = fmaf(-2.f, acc[i], qn + tn);
            thr[i] = 1e-3f * (qn + tn);
            cancel = cancel || d2[i] < thr[i];
        }
        if (__any(cancel)) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (d2[i] < thr[i])
                    d2[i] = kge_direct_d2<BF16, false>((const char *)a.Q + (size_t)(b0 + 8 * (i >> 2) + 4 * g + (i & 3)) * a.dp * ES,
                                                       (const char *)a.T + (size_t)n * a.dp * ES, nullptr, a.dp);
                asm volatile("" ::: "memory");                  // keeps the branch from being turned into selects
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float dd = fmaxf(d2[i], 0.f);
            sv[i] = dd > 0.f ? -dd * __builtin_amdgcn_rsqf(dd) : 0.f;
        }
    }
    if (n < a.N) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int b = b0 + 8 * (i >> 2) + 4 * g + (i & 3);
            if (b < a.B) a.S[(size_t)b * a.ldS + n] = sv[i];
        }
    }
}

__device__ __forceinline__ uint32_t small_low_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t small_high_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
// (p and bytes are the same in every lane)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t small_buffer(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, bytes, 0x00027000);
}

// ---- gradients: workgroup = 32 own rows x CT columns, eight waves share the split's part of the contraction index ----
// A lane's columns are CT / 32 neighbours (one load per streamed row), column h of every lane is block h of the matrix product.
template <bool BF16, int KIND, bool OWN_Q, int CT>
__device__ __forceinline__ void small_grad_body(const SmallArgs &a, int own_tile, int d_tile, int split, float *lds) {
    constexpr int NB = CT / 32;                                 // columns per lane, column blocks
    constexpr int ES = BF16 ? 2 : 4, XW = NB * ES / 4;          // 32-bit words of a lane's columns
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 31, g = lane >> 5;
    const int o = own_tile * 32 + lr;                           // own row of the lane's coefficients
    const int str_n = OWN_Q ? a.N : a.B;
    const int xrow = a.dp * ES;
    // (buffer loads: a scalar offset, streamed row 16 s + j of the step, and one of the lane that never changes; no vector instruction)
    const char *X = (const char *)(OWN_Q ? a.T : a.Q) + (size_t)d_tile * (CT * ES);
    const uint32_t x_lane = (uint32_t)(8 * g * xrow + NB * ES * lr);
    const int ldc = (int)a.ldS * 4;
    const char *Cq = (const char *)a.C + (OWN_Q ? (size_t)own_tile * 32 * ldc : (size_t)own_tile * 128);
    const uint32_t c_lane = OWN_Q ? (uint32_t)(lr * ldc + 32 * g) : (uint32_t)(8 * g * ldc + 4 * lr);
    const auto xbuf = small_buffer(X, (OWN_Q ? a.Np : a.Bp) * xrow - d_tile * (CT * ES));
    const auto cbuf = small_buffer(Cq, OWN_Q ? 32 * ldc : a.Bp * ldc - own_tile * 128);
    kge_f32x16 acc[NB];
#pragma unroll
    for (int h = 0; h < NB; ++h) for (int i = 0; i < 16; ++i) acc[h][i] = 0.f;
    float csum = 0.f;
    const int steps = (str_n + 15) / 16, per_split = OWN_Q ? a.q_steps : a.t_steps;
    const int s0 = split * per_split, s1 = min(steps, s0 + per_split), per = (s1 - s0 + 7) / 8;
    const int s_lo = s0 + wave * per, s_hi = min(s1, s_lo + per);
    // raw operands of a step: the lane's eight streamed rows (rows and columns behind the block: zero coefficients, zero rows)
    struct Raw { uint32_t c[8], x[8][XW]; };
    auto load = [&](int s, Raw &r) {
        if constexpr (OWN_Q) {                                  // (rows of C start 16-byte aligned)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(cbuf, c_lane + 16 * e, s * 64, 0));
                r.c[4 * e] = v.x; r.c[4 * e + 1] = v.y; r.c[4 * e + 2] = v.z; r.c[4 * e + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) r.c[j] = __builtin_amdgcn_raw_buffer_load_b32(cbuf, c_lane, (s * 16 + j) * ldc, 0);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = (s * 16 + j) * xrow;
            if constexpr (XW == 1) r.x[j][0] = __builtin_amdgcn_raw_buffer_load_b32(xbuf, x_lane, row, 0);
            else if constexpr (XW == 2) { const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(xbuf, x_lane, row, 0)); r.x[j][0] = v.x; r.x[j][1] = v.y; }
            else { const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xbuf, x_lane, row, 0)); r.x[j][0] = v.x; r.x[j][1] = v.y; r.x[j][2] = v.z; r.x[j][3] = v.w; }
        }
    };
    auto step = [&](Raw &r) {
        Frag<BF16> fc, fc2;                                     // fc2: the second pieces (dQ on bf16 tables)
        // (pinned here as they came: otherwise their packing moves to the request, and the wait for memory with it)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            asm volatile("" : "+v"(r.c[j]));
#pragma unroll
            for (int w = 0; w < XW; ++w) asm volatile("" : "+v"(r.x[j][w]));
        }
        if constexpr (BF16) {
            auto first = [&](int j) { return small_low_halves(r.c[j], r.c[j + 1]); };
            auto second = [&](int j) { return small_high_halves(r.c[j], r.c[j + 1]); };
            fc.v = make_uint4(first(0), first(2), first(4), first(6));
            if constexpr (OWN_Q) fc2.v = make_uint4(second(0), second(2), second(4), second(6));
        } else fc.v = kge_split3(make_uint4(r.c[0], r.c[1], r.c[2], r.c[3]), make_uint4(r.c[4], r.c[5], r.c[6], r.c[7]));
        if constexpr (!OWN_Q && KIND == KGE_KIND_DIST) {
#pragma unroll
            for (int j = 0; j < 8; ++j)                         // (both pieces: dT = sum c q - (sum c) t, and t is not part of the rounding)
                csum += BF16 ? __uint_as_float(r.c[j] << 16) + __uint_as_float(r.c[j] & 0xffff0000u) : __uint_as_float(r.c[j]);
        }
#pragma unroll
        for (int h = 0; h < NB; ++h) {
            Frag<BF16> f;
            if constexpr (BF16) {                               // column h of the eight streamed rows, two rows per word
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t x0 = r.x[2 * j][h >> 1], x1 = r.x[2 * j + 1][h >> 1];
                    w[j] = h & 1 ? small_high_halves(x0, x1) : small_low_halves(x0, x1);
                }
                f.v = make_uint4(w[0], w[1], w[2], w[3]);
            } else
                f.v = kge_split3(make_uint4(r.x[0][h], r.x[1][h], r.x[2][h], r.x[3][h]), make_uint4(r.x[4][h], r.x[5][h], r.x[6][h], r.x[7][h]));
            if constexpr (BF16 && OWN_Q) acc[h] = small_mma<BF16>(acc[h], fc2, f);
            acc[h] = small_mma<BF16>(acc[h], fc, f);
        }
    };
    // (the next AH - 1 steps are requested before this one is used; the scheduler is held to that order: left alone it moved every
    // request behind the step in front of it, and a wave waited for memory in every step)
    if (s_lo < s_hi) {
        constexpr int AH = SMALL_AHEAD;
        Raw r[AH];
#pragma unroll
        for (int u = 0; u < AH - 1; ++u) load(min(s_lo + u, s_hi - 1), r[u]);
        int s = s_lo;
        for (; s + AH <= s_hi; s += AH) {
#pragma unroll
            for (int u = 0; u < AH; ++u) {
                load(min(s + u + AH - 1, s_hi - 1), r[(u + AH - 1) % AH]);
                __builtin_amdgcn_sched_barrier(0);
                step(r[u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int u = 0; u < AH - 1; ++u) if (s + u < s_hi) step(r[u]);
    }
    // Register i of acc[h]: own row 8 (i / 4) + 4 g + i % 4, column NB lr + h.  The upper four waves hand theirs to the lower four,
    // those add up in wave order.
    float *mine = lds + (wave & 3) * 32 * CT;
    auto at = [&](int i) { return mine + (8 * (i >> 2) + 4 * g + (i & 3)) * CT + NB * lr; };
    float *csums = lds + 4 * 32 * CT;
    if constexpr (!OWN_Q && KIND == KGE_KIND_DIST) {
        csum += __shfl_xor(csum, 32);
        if (g == 0) csums[wave * 32 + lr] = csum;
    }
    if (wave >= 4) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int h = 0; h < NB; h += 2) *(float2 *)(at(i) + h) = make_float2(acc[h][i], acc[h + 1][i]);
    }
    __syncthreads();
    if (wave < 4) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int h = 0; h < NB; h += 2) {
                const float2 v = *(const float2 *)(at(i) + h);
                *(float2 *)(at(i) + h) = make_float2(acc[h][i] + v.x, acc[h + 1][i] + v.y);
            }
    }
    __syncthreads();
    float *out = (OWN_Q ? a.accq : a.acct) + (size_t)split * (OWN_Q ? a.Bp : a.Np) * a.dp;
#pragma unroll
    for (int e = 0; e < CT / 64; ++e) {
        const int i = (e * 512 + threadIdx.x) * 4;
        kge_f32x4 v = *(const kge_f32x4 *)(lds + i);
#pragma unroll
        for (int w = 1; w < 4; ++w) v += *(const kge_f32x4 *)(lds + w * 32 * CT + i);
        *(kge_f32x4 *)(out + (size_t)(own_tile * 32 + i / CT) * a.dp + d_tile * CT + i % CT) = v;
    }
    if constexpr (!OWN_Q && KIND == KGE_KIND_DIST)
        if (d_tile == 0 && threadIdx.x < 32) {
            float t = csums[threadIdx.x];
#pragma unroll
            for (int w = 1; w < 8; ++w) t += csums[w * 32 + threadIdx.x];
            a.sumt[(size_t)split * a.Np + own_tile * 32 + threadIdx.x] = make_float4(t, 0.f, 0.f, 0.f);
        }
}

template <bool BF16, int KIND, int CT>
__global__ __launch_bounds__(512) void small_grad_kernel(const SmallArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[4 * 32 * CT + 8 * 32];
    // (workgroups go to the eight dies in turn: the column tiles and splits of an own tile, which read the same rows of C or X, stay together)
    int blk = blockIdx.x;
    const bool q = blk < a.q_blocks;
    if (!q) blk -= a.q_blocks;
    const int splits = q ? a.q_splits : a.t_splits, inner = a.d_tiles * splits;
    const int kk = blk >> 3, own = (kk / inner) * 8 + (blk & 7), d_tile = kk % inner % a.d_tiles, split = kk % inner / a.d_tiles;
    if (own * 32 >= (q ? a.B : a.N)) return;
    if (q) small_grad_body<BF16, KIND, true, CT>(a, own, d_tile, split, lds);
    else small_grad_body<BF16, KIND, false, CT>(a, own, d_tile, split, lds);
}

// ---- rows: one workgroup per query (small_rows.hpp) ----
__global__ __launch_bounds__(256) void small_rows_kernel(const KgeSmallRowsArgs a) {
    __shared__ KgeSmallRowsShared sh;
    kge_small_rows_body((int)blockIdx.x, (int)threadIdx.x, sh, a);
}

}  // namespace

int kge_run_small_rows(const KgeSmallRowsArgs &a, hipStream_t st) {
    if (a.Bp == 0) return KGE_OK;
    hipLaunchKernelGGL(small_rows_kernel, dim3(a.Bp), dim3(256), 0, st, a);
    return kge_launch_status();
}

int kge_run_small_score(bool bf16, int kind, const void *Q, const void *T, const KgeRowInfo *rowinfo, const float *tn, int B, int N, int Bp,
                        int Np, int dp, int dim, float *S, int64_t ldS, hipStream_t st) {
    if (dp % 128 || Bp % 64 || Np % 64 || B < 1 || N < 1 || Bp / 64 > 65535) return KGE_E_INVALID_ARG;
    KgeProfScope prof(KGE_PROF_BLOCK_FWD, st);
    SmallArgs a{};
    a.Q = Q; a.T = T; a.rowinfo = rowinfo; a.tn = tn; a.S = S; a.ldS = ldS; a.B = B; a.N = N; a.Bp = Bp; a.Np = Np; a.dp = dp; a.dim = dim;
    const dim3 grid((N + 63) / 64, (B + 63) / 64);
    const int pieces = (dim * (bf16 ? 2 : 4) + 255) / 256;
    if (pieces > 4 || dp * (bf16 ? 2 : 4) < pieces * 256) return KGE_E_INVALID_ARG;
#define SMALL_SCORE3(BF, KD, NCH)                                                                                           \
    {                                                                                                                       \
        static KgeLdsLimit limit;                                                                                           \
        constexpr int bytes = NCH * SMALL_PIECE + 4 * 256;                                                                  \
        if (limit.set((const void *)small_score_kernel<BF, KD, NCH>, bytes) != KGE_OK) return KGE_E_HIP;                    \
        hipLaunchKernelGGL((small_score_kernel<BF, KD, NCH>), grid, dim3(256 * small_score_groups(BF)), bytes, st, a);                               \
        return kge_launch_status();                                                                                         \
    }
#define SMALL_SCORE(BF, KD)                                                                                                 \
    switch (pieces) {                                                                                                       \
    case 1: SMALL_SCORE3(BF, KD, 1) case 2: SMALL_SCORE3(BF, KD, 2) case 3: SMALL_SCORE3(BF, KD, 3) default: SMALL_SCORE3(BF, KD, 4)  \
    }
    if (bf16) { if (kind == KGE_KIND_DIST) SMALL_SCORE(true, KGE_KIND_DIST) else SMALL_SCORE(true, KGE_KIND_MULT) }
    else      { if (kind == KGE_KIND_DIST) SMALL_SCORE(false, KGE_KIND_DIST) else SMALL_SCORE(false, KGE_KIND_MULT) }
#undef SMALL_SCORE
#undef SMALL_SCORE3
}

// splits of the gradients' contraction index (str streamed rows): a wave of a workgroup's eight takes sixteen matrix steps at most
int kge_small_splits(int str) { return (str + 2047) / 2048; }

// columns of a workgroup of the gradients: 128 read the coefficients half as often as 64, if they fill the chip and few of them lie
// behind the row.  Calls, 128 / 64 columns, us: TransE bf16 512 x 1,024 x 256 (96 workgroups of 128 columns) 32.7 / 30.7, RotatE fp32
// 448 x 1,088 x 256 (96) 45.2 / 41.1, ComplEx bf16 640 x 1,536 x 400 (272) 44.7 / 43.0, 512 x 4,096 x 256 (288) 51.9 / 48.4;  TransE bf16
// 1,024 x 3,900 x 256 (308) 57.7 / 60.0, ComplEx 1,000 x 2,000 x 400 (380) 54.6 / 56.6, 1,500 x 2,500 x 512 (504) 85.4 / 89.6;  rows that
// 128 columns pad by a fifth or a third: DistMult 2,048 x 2,048 x 320 73.1 / 69.6, fp32 2,500 x 2,500 x 192 132.8 / 112.4
static int small_columns(int B, int N, int dim) {
    const int wide = (dim + 127) / 128, narrow = (dim + 63) / 64, tiles = (B + 31) / 32 + (N + 31) / 32;
    return tiles * wide <= 300 || 12 * wide > 7 * narrow ? 64 : 128;
}

int kge_run_small_grad(bool bf16, int kind, const void *Q, const void *T, const void *C, int64_t ldS, int B, int N, int Bp, int Np, int dp,
                       int dim, int q_splits, int t_splits, float *accq, float *acct, float4 *sumt, hipStream_t st) {
    if (dp % 128 || Bp % 32 || Np % 32 || ldS % 8 || B < 1 || N < 1 || q_splits != kge_small_splits(N) || t_splits != kge_small_splits(B))
        return KGE_E_INVALID_ARG;
    KgeProfScope prof(KGE_PROF_BLOCK_GRADT, st);
    SmallArgs a{};
    a.Q = Q; a.T = T; a.C = (const uint32_t *)C; a.ldS = ldS; a.B = B; a.N = N; a.Bp = Bp; a.Np = Np; a.dp = dp; a.dim = dim;
    a.accq = accq; a.acct = acct; a.sumt = sumt;
    const int ct = small_columns(B, N, dim);
    a.d_tiles = (dim + ct - 1) / ct;
    a.q_splits = q_splits; a.t_splits = t_splits;
    a.q_steps = ((N + 15) / 16 + q_splits - 1) / q_splits; a.t_steps = ((B + 15) / 16 + t_splits - 1) / t_splits;
    a.q_blocks = (B + 255) / 256 * 8 * a.d_tiles * q_splits;
    const dim3 grid(a.q_blocks + (N + 255) / 256 * 8 * a.d_tiles * t_splits);
#define SMALL_GRAD(BF, KD) do { if (ct == 128) hipLaunchKernelGGL((small_grad_kernel<BF, KD, 128>), grid, dim3(512), 0, st, a); \
                                else hipLaunchKernelGGL((small_grad_kernel<BF, KD, 64>), grid, dim3(512), 0, st, a); } while (0)
    if (bf16) { if (kind == KGE_KIND_DIST) SMALL_GRAD(true, KGE_KIND_DIST); else SMALL_GRAD(true, KGE_KIND_MULT); }
    else      { if (kind == KGE_KIND_DIST) SMALL_GRAD(false, KGE_KIND_DIST); else SMALL_GRAD(false, KGE_KIND_MULT); }
#undef SMALL_GRAD
    return kge_launch_status();
}
