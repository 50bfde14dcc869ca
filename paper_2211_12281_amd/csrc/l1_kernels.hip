// The distance scorers with the 1-norm (Table 2, p = 1): f = -sum_j |q_j - t_j| over the query q = h + r (TransE)
// or h o e^{ir} taken in R^d (RotatE).  There is no contraction form: every (query, negative, dimension) triple
// costs vector instructions, so the score block IS written to memory here (4 bytes per pair against 2 d vector
// operations) and the backward pass reads it back instead of recomputing it:
//   scores      S[b, n] = -sum_j |q_bj - t_nj|
//   row pass    per query the maximum and the sums of the loss weights over its row of S
//   gradients   dq[b, j] = -sum_n w(b, n) sign(q_bj - t_nj),   dt[n, j] = +sum_b w(b, n) sign(q_bj - t_nj)
// with w(b, n) = dL/dS[b, n] from S and the finished row constants; sign(0) = 0 (sub-gradient at the kink).
// The queries are read from an unrounded fp32 copy also when the tables are bf16 (a sign flips when rounding moves a
// difference across zero; the table rows themselves are exact).  The block kernels stage fp32 tiles in the LDS (row pitch 68 floats: the
// 16 lanes that read 16 different rows at one column offset hit 16 different 16-byte bank groups): the scores 64 x 64, 32 x 64 or 32 x 48
// with a 4 x 4, 2 x 4 or 2 x 3 register tile per thread, the gradients 32 streamed rows x 64 columns against an 8 x 4 register tile; they are bound by the vector pipe in large blocks and by the latency of a chunk (loads, barrier) in small ones, so the loads of
// the next chunk are issued before the present one is used (gradient passes 44 -> 24 us each at 512 x 1,280 x 384).  Small blocks take both
// gradients from one kernel (l1_grad_both_kernel).
#include "row_ops.hpp"

namespace {

constexpr int L1_TILE = 64;            // rows and columns of a staged tile
constexpr int L1_PITCH = 68;           // floats per LDS row
constexpr float L1_LOG2E = 1.4426950408889634f;
constexpr float L1_BIG = 0x1p100f;     // scale of the operands of the sign computation

typedef float l1_f32x4 __attribute__((ext_vector_type(4)));

// rows [r0, r0 + 64) x columns [c0, c0 + 64) of a row-major [rows][ld] array of the table type -> fp32 LDS tile, in two halves:
// the loads of the next tile are issued before this one is used
template <int R> struct L1TileR { uint32_t w[R / 16][4]; };      // R rows
using L1Tile = L1TileR<L1_TILE>;
template <bool BF16, int R>                                       // (rows: of the array; a tile may reach past them)
__device__ __forceinline__ void l1_fetch(const void *src, int64_t ld, int r0, int c0, L1TileR<R> &t, int rows = 0x7fffffff) {
#pragma unroll
    for (int k = 0; k < R / 16; ++k) {
        const int e = threadIdx.x + 256 * k, row = e >> 4, cq = e & 15;
        const int64_t off = (int64_t)min(r0 + row, rows - 1) * ld + c0 + 4 * cq;
        if constexpr (BF16) {
            const uint2 raw = *(const uint2 *)((const __bf16 *)src + off);
            t.w[k][0] = raw.x; t.w[k][1] = raw.y;
        } else {
            const uint4 raw = *(const uint4 *)((const float *)src + off);
            t.w[k][0] = raw.x; t.w[k][1] = raw.y; t.w[k][2] = raw.z; t.w[k][3] = raw.w;
        }
    }
}
template <bool BF16, int R>
__device__ __forceinline__ void l1_put(const L1TileR<R> &t, float *tile) {
#pragma unroll
    for (int k = 0; k < R / 16; ++k) {
        const int e = threadIdx.x + 256 * k, row = e >> 4, cq = e & 15;
        l1_f32x4 v;
        if constexpr (BF16)
            v = l1_f32x4{__uint_as_float(t.w[k][0] << 16), __uint_as_float(t.w[k][0] & 0xffff0000u),
                         __uint_as_float(t.w[k][1] << 16), __uint_as_float(t.w[k][1] & 0xffff0000u)};
        else v = l1_f32x4{__uint_as_float(t.w[k][0]), __uint_as_float(t.w[k][1]), __uint_as_float(t.w[k][2]), __uint_as_float(t.w[k][3])};
        *(l1_f32x4 *)(tile + row * L1_PITCH + 4 * cq) = v;
    }
}
template <bool BF16>
__device__ __forceinline__ void l1_stage(const void *src, int64_t ld, int r0, int c0, float *tile) {
    L1Tile t;
    l1_fetch<BF16>(src, ld, r0, c0, t);
    l1_put<BF16>(t, tile);
}

// S[b, n] = -sum_j |q_bj - t_nj|; workgroup = 16 QR queries x 16 KN negatives, thread = queries QR ty + i, negatives tx + 16 k
template <bool BF16, int QR, int KN>
__global__ __launch_bounds__(256) void l1_score_kernel(const float *Q, const void *T, int B, int N, int Np, int dp, int cols, float *S, int64_t ldS) {
    __shared__ __attribute__((aligned(16))) float qs[16 * QR * L1_PITCH], ts[16 * KN * L1_PITCH];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int n0 = blockIdx.x * 16 * KN, b0 = blockIdx.y * 16 * QR;
    float acc[QR][KN];
#pragma unroll
    for (int i = 0; i < QR; ++i)
        for (int k = 0; k < KN; ++k) acc[i][k] = 0.f;
    L1TileR<16 * QR> tq;
    L1TileR<16 * KN> tt;
    l1_fetch<false>(Q, dp, b0, 0, tq);
    l1_fetch<BF16>(T, dp, n0, 0, tt, Np);
    for (int j0 = 0; j0 < cols; j0 += L1_TILE) {
        __syncthreads();
        l1_put<false>(tq, qs);
        l1_put<BF16>(tt, ts);
        __syncthreads();
        if (j0 + L1_TILE < cols) {
            l1_fetch<false>(Q, dp, b0, j0 + L1_TILE, tq);
            l1_fetch<BF16>(T, dp, n0, j0 + L1_TILE, tt, Np);
        }
#pragma unroll 4
        for (int jq = 0; jq < 16; ++jq) {
            l1_f32x4 q4[QR], t4[KN];
#pragma unroll
            for (int i = 0; i < QR; ++i) q4[i] = *(const l1_f32x4 *)(qs + (QR * ty + i) * L1_PITCH + 4 * jq);
#pragma unroll
            for (int i = 0; i < KN; ++i) t4[i] = *(const l1_f32x4 *)(ts + (tx + 16 * i) * L1_PITCH + 4 * jq);
#pragma unroll
            for (int i = 0; i < QR; ++i)
#pragma unroll
                for (int k = 0; k < KN; ++k)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[i][k] += fabsf(q4[i][c] - t4[k][c]);
        }
    }
#pragma unroll
    for (int i = 0; i < QR; ++i) {
        const int b = b0 + QR * ty + i;
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            const int n = n0 + tx + 16 * k;
            if (b < B && n < N) S[(int64_t)b * ldS + n] = -acc[i][k];
        }
    }
}

__device__ __forceinline__ float l1_sigmoid(float y) {
    const float t = __builtin_amdgcn_exp2f(-fabsf(y) * L1_LOG2E), rcp = 1.f / (1.f + t);
    return y >= 0.f ? rcp : t * rcp;
}

// out[split][o, j] = -sum_s w(o, s) sign(own_oj - str_sj) over the split's rows of the streamed operand: with
// own = queries this is dq (s runs over the negatives), with own = negatives it is dt (s runs over the queries;
// the sign flips twice).  Workgroup = 128 own rows x 64 dimensions; thread = own rows 4 ty + i + 64 i',
// dimensions 4 tx + c (an 8 x 4 register tile: three 16-byte LDS reads feed 32 sign terms; 156 to 162 registers
// with the next chunk in flight, three waves per SIMD).  The queries
// are fp32, the negatives of the table type.  Both operands are scaled by 2^100 when they are loaded (exact), so that
// sign(own - str) = median(-1, (own - str) 2^100, 1) is one subtraction and one median: a non-zero difference of
// two floats whose magnitudes exceed 2^-76 is at least 2^-100, its scaled value at least 1; a zero difference
// stays zero (sub-gradient 0).  Three vector operations per (own row, streamed row, dimension).  The weights w come from the
// row pass, which leaves them in place of the scores.
constexpr int L1_GO = 128, L1_GD = 64, L1_GS = 32;   // own rows, dimensions, streamed rows per chunk of a gradient workgroup
constexpr int L1_WP = 132;                            // floats per LDS row of the weights (16 lanes x 16 bytes stay conflict-free)

struct L1GradPart { const void *own, *str; float *acc_part; int own_pad, own_tiles, col_tiles, chunks, cps; };

template <bool BF16, bool OWN_Q>
__device__ __forceinline__ void l1_grad_body(const L1GradPart &p, int blk, const float *W, int64_t ldW, int B, int N, int dp, float *ss, float *ws) {
    const void *own = p.own, *str = p.str;
    const int own_pad = p.own_pad, chunks = p.chunks, cps = p.cps;
    float *acc_part = p.acc_part;
    constexpr bool SBF = BF16 && OWN_Q, OBF = BF16 && !OWN_Q;   // table type of the streamed / own operand
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int rest = blk / p.own_tiles, split = rest / p.col_tiles;
    const int o0 = (blk - rest * p.own_tiles) * L1_GO, j0 = (rest - split * p.col_tiles) * L1_GD;
    float ov[8][4], acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t off = (int64_t)(o0 + 4 * ty + (i & 3) + 64 * (i >> 2)) * dp + j0 + 4 * tx;
        l1_f32x4 v;
        if constexpr (OBF) {
            const uint2 r = *(const uint2 *)((const __bf16 *)own + off);
            v = l1_f32x4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u), __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u)};
        } else v = *(const l1_f32x4 *)((const float *)own + off);
#pragma unroll
        for (int c = 0; c < 4; ++c) { ov[i][c] = v[c] * L1_BIG; acc[i][c] = 0.f; }
    }
    const int c_lo = split * cps, c_hi = min(chunks, (split + 1) * cps);
    // a chunk's rows and weights are requested before the chunk in front of it is used
    uint32_t raw[2][4];
    float wv[16];
    auto fetch = [&](int ch) {
        const int s0 = ch * L1_GS;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int e = threadIdx.x + 256 * k, row = e >> 4, cq = e & 15;
            const int64_t off = (int64_t)(s0 + row) * dp + j0 + 4 * cq;
            if constexpr (SBF) {
                const uint2 v = *(const uint2 *)((const __bf16 *)str + off);
                raw[k][0] = v.x; raw[k][1] = v.y;
            } else {
                const uint4 v = *(const uint4 *)((const float *)str + off);
                raw[k][0] = v.x; raw[k][1] = v.y; raw[k][2] = v.z; raw[k][3] = v.w;
            }
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int e = threadIdx.x + 256 * k;
            // consecutive threads take consecutive negatives: the reads of W are coalesced either way
            const int ol = OWN_Q ? e >> 5 : e & 127, sl = OWN_Q ? e & 31 : e >> 7;
            const int b = OWN_Q ? o0 + ol : s0 + sl, n = OWN_Q ? s0 + sl : o0 + ol;
            wv[k] = b < B && n < N ? W[(int64_t)b * ldW + n] : 0.f;
        }
    };
    if (c_lo < c_hi) fetch(c_lo);
    for (int ch = c_lo; ch < c_hi; ++ch) {
        __syncthreads();                                    // everyone is done with the previous chunk
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int e = threadIdx.x + 256 * k, row = e >> 4, cq = e & 15;
            l1_f32x4 v;
            if constexpr (SBF)
                v = l1_f32x4{__uint_as_float(raw[k][0] << 16), __uint_as_float(raw[k][0] & 0xffff0000u),
                             __uint_as_float(raw[k][1] << 16), __uint_as_float(raw[k][1] & 0xffff0000u)};
            else v = l1_f32x4{__uint_as_float(raw[k][0]), __uint_as_float(raw[k][1]), __uint_as_float(raw[k][2]), __uint_as_float(raw[k][3])};
            *(l1_f32x4 *)(ss + row * L1_PITCH + 4 * cq) = v * L1_BIG;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int e = threadIdx.x + 256 * k;
            const int ol = OWN_Q ? e >> 5 : e & 127, sl = OWN_Q ? e & 31 : e >> 7;
            ws[sl * L1_WP + ol] = wv[k];
        }
        if (ch + 1 < c_hi) fetch(ch + 1);
        __syncthreads();
#pragma unroll 4
        for (int sl = 0; sl < L1_GS; ++sl) {
            const l1_f32x4 w4[2] = { *(const l1_f32x4 *)(ws + sl * L1_WP + 4 * ty), *(const l1_f32x4 *)(ws + sl * L1_WP + 4 * ty + 64) };
            const l1_f32x4 t4 = *(const l1_f32x4 *)(ss + sl * L1_PITCH + 4 * tx);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[i][c] = fmaf(-w4[i >> 2][i & 3], __builtin_amdgcn_fmed3f(ov[i][c] - t4[c], -1.f, 1.f), acc[i][c]);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
        *(l1_f32x4 *)(acc_part + ((int64_t)split * own_pad + o0 + 4 * ty + (i & 3) + 64 * (i >> 2)) * dp + j0 + 4 * tx) =
            l1_f32x4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
}

// Both passes in ONE launch, the queries' workgroups first: they need nothing of one another, and each alone leaves a last round of
// workgroups that covers a part of the chip (512 x 1,280 x 384: 24.7 + 23.6 -> 44 us;  whole calls, us: TransE bf16 4,000 x 300 x 64 76 -> 60,
// fp32 512 x 1,280 x 128 57 -> 48, bf16 4,096 x 4,096 x 256 726 -> 686).
template <bool BF16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void l1_grad_kernel(
        const L1GradPart q, const L1GradPart t, const int q_blocks, const float *W, int64_t ldW, int B, int N, int dp) {
    __shared__ __attribute__((aligned(16))) float ss[L1_GS * L1_PITCH], ws[L1_GS * L1_WP];
    if ((int)blockIdx.x < q_blocks) l1_grad_body<BF16, true>(q, (int)blockIdx.x, W, ldW, B, N, dp, ss, ws);
    else l1_grad_body<BF16, false>(t, (int)blockIdx.x - q_blocks, W, ldW, B, N, dp, ss, ws);
}

// Both gradients from ONE sign per (query, negative, dimension): subtraction, median and a multiply-add for either side, four vector
// operations where the two passes above take six.  A lane is a dimension: a wave owns 16 negatives (16 values and 16 sums in registers)
// and the queries stream by in chunks of 32, whose weights lie in the LDS (a row's 16 in four reads that all lanes share) and whose values
// are requested eight queries ahead.  A query's sum over the wave's negatives goes to the LDS; at the end of the chunk the workgroup adds
// its four waves up into its group's partial row - one block of 64 negatives of the group after the other, so that there are no more
// partials than the passes above leave: [groups][Bp][dp] and, by splits of the queries, [splits][Np][dp].
// Bound by that chunk (weights and values in, sums out, two barriers, about 2,000 vector instructions per wave), not by the pipe: a step
// is faster where a workgroup has few of them (512 x 1,280 x 384 bf16: 43.7 -> 34 us).  32 negatives per wave halve the LDS sums per pair,
// but leave two waves per SIMD (call 67 -> 71 us), and weights by scalar loads wait for the line of a query's row at every step (71).
constexpr int L1_BQ = 32, L1_BW = 16, L1_BN = 4 * L1_BW;       // queries of a chunk, negatives of a wave and of a block
struct L1BothArgs { const float *Q; const void *T; const float *W; int64_t ldW; int B, N, Bp, Np, dp, col_tiles, groups, bpg, chunks, cps; float *accq, *acct; };

template <bool BF16>
__global__ __launch_bounds__(256) void l1_grad_both_kernel(const L1BothArgs a) {
    __shared__ __attribute__((aligned(16))) float red[4][L1_BQ][64], ws[L1_BQ][L1_BN];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = (int)blockIdx.x % a.col_tiles, rest = (int)blockIdx.x / a.col_tiles, group = rest % a.groups, split = rest / a.groups;
    const int j = col * 64 + lane;
    const int c_lo = split * a.cps, c_hi = min(a.chunks, c_lo + a.cps), blocks = (a.N + L1_BN - 1) / L1_BN, npad = (a.N + 31) / 32 * 32;
    constexpr int WL = L1_BQ * L1_BW / 256;                     // 16-byte pieces of a chunk's weights per thread
    for (int nb = group * a.bpg; nb < min(blocks, (group + 1) * a.bpg); ++nb) {
        const int n0 = (nb * 4 + wave) * L1_BW;
        const bool live = n0 < a.N;
        l1_f32x4 wn[WL];
        auto fetch_w = [&](int ch) {                         // (the weights end at the next multiple of 32 behind N)
#pragma unroll
            for (int k = 0; k < WL; ++k) {
                const int e = tid + 256 * k, row = e / L1_BW, n = nb * L1_BN + e % L1_BW * 4;
                wn[k] = n < npad ? *(const l1_f32x4 *)(a.W + (int64_t)(ch * L1_BQ + row) * a.ldW + n) : l1_f32x4{0.f, 0.f, 0.f, 0.f};
            }
        };
        if (c_lo < c_hi) fetch_w(c_lo);
        float ov[L1_BW], acc[L1_BW];
#pragma unroll
        for (int i = 0; i < L1_BW; ++i) {
            const int64_t off = (int64_t)(n0 + i) * a.dp + j;
            ov[i] = (BF16 ? (float)((const __bf16 *)a.T)[off] : ((const float *)a.T)[off]) * L1_BIG;
            acc[i] = 0.f;
        }
        for (int ch = c_lo; ch < c_hi; ++ch) {
            const int b0 = ch * L1_BQ;
            const float *qp = a.Q + (int64_t)b0 * a.dp + j;
#pragma unroll
            for (int k = 0; k < WL; ++k) { const int e = tid + 256 * k; *(l1_f32x4 *)&ws[e / L1_BW][e % L1_BW * 4] = wn[k]; }
            __syncthreads();
            if (ch + 1 < c_hi) fetch_w(ch + 1);
            if (live) {
                float qn[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) qn[u] = qp[(int64_t)u * a.dp];
#pragma unroll 1
                for (int b8 = 0; b8 < L1_BQ; b8 += 8) {
                    float qc[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) { qc[u] = qn[u] * L1_BIG; qn[u] = qp[(int64_t)min(b8 + 8 + u, L1_BQ - 1) * a.dp]; }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        float d[2] = {0.f, 0.f};
#pragma unroll
                        for (int i4 = 0; i4 < L1_BW / 4; ++i4) {
                            const l1_f32x4 w4 = *(const l1_f32x4 *)&ws[b8 + u][wave * L1_BW + 4 * i4];
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                const int i = 4 * i4 + c;
                                const float s = __builtin_amdgcn_fmed3f(qc[u] - ov[i], -1.f, 1.f);
                                acc[i] = fmaf(w4[c], s, acc[i]);
                                d[c & 1] = fmaf(-w4[c], s, d[c & 1]);
                            }
                        }
                        red[wave][b8 + u][lane] = d[0] + d[1];
                    }
                }
            } else {
                for (int bb = 0; bb < L1_BQ; ++bb) red[wave][bb][lane] = 0.f;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < L1_BQ * 64 / 256; ++k) {
                const int bb = k * 4 + (tid >> 6), b = b0 + bb;
                const float v = (red[0][bb][lane] + red[1][bb][lane]) + (red[2][bb][lane] + red[3][bb][lane]);
                if (b < a.B) {
                    float *p = a.accq + ((int64_t)group * a.Bp + b) * a.dp + j;
                    *p = nb == group * a.bpg ? v : *p + v;
                }
            }
            // (the next chunk's weights are written before, its sums behind a barrier)
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < L1_BW; ++i) if (n0 + i < a.N) a.acct[((int64_t)split * a.Np + n0 + i) * a.dp + j] = acc[i];
    }
}

// ---------------------------------------------------------------------------------------------
// TransH under the 1-norm (Table 2, p = 1): x_j = q'_j - t_j + A w^_j with q' = h_perp + r, A = w^ . t, and
//   f = -sum_j |x_j|,  u_j = sign(x_j),  P = u . w^
//   df/dq'_j = -u_j,   df/dt_j = u_j - P w^_j,   df/dw^_j = -(P t_j + A u_j)
// The hyperplane term sits inside the absolute values, so the score kernel walks the dimensions twice (first A,
// then the distance and P) and leaves A and P beside S for the two gradient kernels.  Queries and unit normals are
// unrounded fp32 rows.  Same tiling as above with 64 own rows per gradient workgroup (a 4 x 4 register tile; the
// pass over the queries carries two accumulators, dq' and dw^).
// ---------------------------------------------------------------------------------------------
// PN = 2 runs the same three kernels for the 2-norm (rows too wide for the matrix-core TransH kernels): the distance sums
// x_j^2, u = x / ||x|| (0 at distance 0), P = (x . w^) / ||x||; the gradient kernels fold 1 / ||x|| = -1 / S into the
// weight of the pair and use x itself where the 1-norm has sign(x).
template <bool BF16, int PN>
__global__ __launch_bounds__(256) void l1h_score_kernel(const float *Q, const float *W, const void *T, int B, int N, int dp,
                                                        float *S, float *A, float *P, int64_t ldS) {
    __shared__ __attribute__((aligned(16))) float qs[L1_TILE * L1_PITCH], ws[L1_TILE * L1_PITCH], ts[L1_TILE * L1_PITCH];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int n0 = blockIdx.x * L1_TILE, b0 = blockIdx.y * L1_TILE;
    float a[4][4], acc[4][4], pp[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        for (int k = 0; k < 4; ++k) a[i][k] = acc[i][k] = pp[i][k] = 0.f;
    for (int j0 = 0; j0 < dp; j0 += L1_TILE) {
        __syncthreads();
        l1_stage<false>(W, dp, b0, j0, ws);
        l1_stage<BF16>(T, dp, n0, j0, ts);
        __syncthreads();
#pragma unroll 4
        for (int jq = 0; jq < 16; ++jq) {
            l1_f32x4 w4[4], t4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w4[i] = *(const l1_f32x4 *)(ws + (4 * ty + i) * L1_PITCH + 4 * jq);
                t4[i] = *(const l1_f32x4 *)(ts + (tx + 16 * i) * L1_PITCH + 4 * jq);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < 4; ++c) a[i][k] = fmaf(w4[i][c], t4[k][c], a[i][k]);
        }
    }
    for (int j0 = 0; j0 < dp; j0 += L1_TILE) {
        __syncthreads();
        l1_stage<false>(Q, dp, b0, j0, qs);
        l1_stage<false>(W, dp, b0, j0, ws);
        l1_stage<BF16>(T, dp, n0, j0, ts);
        __syncthreads();
#pragma unroll 2
        for (int jq = 0; jq < 16; ++jq) {
            l1_f32x4 q4[4], w4[4], t4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                q4[i] = *(const l1_f32x4 *)(qs + (4 * ty + i) * L1_PITCH + 4 * jq);
                w4[i] = *(const l1_f32x4 *)(ws + (4 * ty + i) * L1_PITCH + 4 * jq);
                t4[i] = *(const l1_f32x4 *)(ts + (tx + 16 * i) * L1_PITCH + 4 * jq);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x = fmaf(a[i][k], w4[i][c], q4[i][c] - t4[k][c]);
                        if constexpr (PN == 1) {
                            acc[i][k] += fabsf(x);
                            pp[i][k] = fmaf(__builtin_amdgcn_fmed3f(x * L1_BIG, -1.f, 1.f), w4[i][c], pp[i][k]);
                        } else {
                            acc[i][k] = fmaf(x, x, acc[i][k]);
                            pp[i][k] = fmaf(x, w4[i][c], pp[i][k]);
                        }
                    }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = b0 + 4 * ty + i;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int n = n0 + tx + 16 * k;
            if (b < B && n < N) {
                const float dist = PN == 1 ? acc[i][k] : sqrtf(acc[i][k]);
                S[(int64_t)b * ldS + n] = -dist;
                if (A) { A[(int64_t)b * ldS + n] = a[i][k]; P[(int64_t)b * ldS + n] = PN == 1 ? pp[i][k] : (dist > 0.f ? pp[i][k] / dist : 0.f); }
            }
        }
    }
}

constexpr int L1H_GO = 64;             // own rows of a TransH gradient workgroup

// OWN_Q: own = 64 queries (q' and w^), streamed = negatives: acc_part = dq' = -sum_n w u,
//        acc_part2 = dw^ = -sum_n (w P) t_n + (w A) u.
// else:  own = 64 negatives, streamed = queries: acc_part = dt = sum_b w u - (w P) w^_b.
// u = sign(x) = median(-1, x 2^100, 1) (a non-zero x of magnitude at least 2^-100 scales to at least 1).
template <bool BF16, bool OWN_Q, int PN>
__global__ __launch_bounds__(256) void l1h_grad_kernel(const float *Q, const float *W, const void *T, const float *S,
                                                       const float *A, const float *P, int64_t ldS, const KgeRowInfo *rowinfo,
                                                       int B, int N, int own_pad, int dp, int chunks, int cps, int loss,
                                                       float gamma, float adv_temp, float *acc_part, float *acc_part2) {
    __shared__ __attribute__((aligned(16))) float s1[L1_GS * L1_PITCH], s2[L1_GS * L1_PITCH];
    __shared__ __attribute__((aligned(16))) float cw[L1_GS * L1_PITCH], ca[L1_GS * L1_PITCH], cp[L1_GS * L1_PITCH];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int o0 = blockIdx.x * L1H_GO, j0 = blockIdx.y * L1_GD, split = blockIdx.z;
    const float xscale = (loss == KGE_LOGSIGMOID ? adv_temp : 1.f) * L1_LOG2E;
    float o1[4][4], o2[4][4], acc1[4][4], acc2[4][4];      // own rows: (q', w^) or (t, -)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t off = (int64_t)(o0 + 4 * ty + i) * dp + j0 + 4 * tx + c;
            o1[i][c] = OWN_Q ? Q[off] : El<BF16>::ld(T, off);
            o2[i][c] = OWN_Q ? W[off] : 0.f;
            acc1[i][c] = acc2[i][c] = 0.f;
        }
    const int c_lo = split * cps, c_hi = min(chunks, (split + 1) * cps);
    for (int ch = c_lo; ch < c_hi; ++ch) {
        const int s0 = ch * L1_GS;
        __syncthreads();                                    // everyone is done with the previous chunk
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int e = threadIdx.x + 256 * k, row = e >> 4, cq = e & 15;
            const int64_t off = (int64_t)(s0 + row) * dp + j0 + 4 * cq;
            if constexpr (OWN_Q) {
                l1_f32x4 v;
                if constexpr (BF16) {
                    const uint2 raw = *(const uint2 *)((const __bf16 *)T + off);
                    v = l1_f32x4{__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xffff0000u),
                                 __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xffff0000u)};
                } else {
                    v = *(const l1_f32x4 *)((const float *)T + off);
                }
                *(l1_f32x4 *)(s1 + row * L1_PITCH + 4 * cq) = v;
            } else {
                *(l1_f32x4 *)(s1 + row * L1_PITCH + 4 * cq) = *(const l1_f32x4 *)(Q + off);
                *(l1_f32x4 *)(s2 + row * L1_PITCH + 4 * cq) = *(const l1_f32x4 *)(W + off);
            }
        }
#pragma unroll 4
        for (int k = 0; k < 8; ++k) {
            const int e = threadIdx.x + 256 * k;
            // consecutive threads take consecutive negatives: the reads of S, A and P are coalesced either way
            const int ol = OWN_Q ? e >> 5 : e & 63, sl = OWN_Q ? e & 31 : e >> 6;
            const int b = OWN_Q ? o0 + ol : s0 + sl, n = OWN_Q ? s0 + sl : o0 + ol;
            float w = 0.f, av = 0.f, pv = 0.f;
            if (b < B && n < N) {
                const float sc = S[(int64_t)b * ldS + n];
                w = __builtin_amdgcn_exp2f(fmaf(sc, xscale, rowinfo[b].K));
                if (loss == KGE_LOGSIGMOID) w *= l1_sigmoid(gamma + sc);
                av = A[(int64_t)b * ldS + n];
                pv = w * P[(int64_t)b * ldS + n];
                if constexpr (PN == 2) w = sc < 0.f ? -w / sc : 0.f;    // u = x / ||x||: the pair's 1 / ||x|| rides on its weight
            }
            cw[sl * L1_PITCH + ol] = w; ca[sl * L1_PITCH + ol] = av; cp[sl * L1_PITCH + ol] = pv;
        }
        __syncthreads();
#pragma unroll 2
        for (int sl = 0; sl < L1_GS; ++sl) {
            const l1_f32x4 w4 = *(const l1_f32x4 *)(cw + sl * L1_PITCH + 4 * ty);
            const l1_f32x4 a4 = *(const l1_f32x4 *)(ca + sl * L1_PITCH + 4 * ty);
            const l1_f32x4 p4 = *(const l1_f32x4 *)(cp + sl * L1_PITCH + 4 * ty);
            const l1_f32x4 r1 = *(const l1_f32x4 *)(s1 + sl * L1_PITCH + 4 * tx);
            if constexpr (OWN_Q) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float wa = w4[i] * a4[i];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x = fmaf(a4[i], o2[i][c], o1[i][c] - r1[c]);
                        const float u = PN == 1 ? __builtin_amdgcn_fmed3f(x * L1_BIG, -1.f, 1.f) : x;
                        acc1[i][c] = fmaf(-w4[i], u, acc1[i][c]);
                        acc2[i][c] = fmaf(-p4[i], r1[c], fmaf(-wa, u, acc2[i][c]));
                    }
                }
            } else {
                const l1_f32x4 r2 = *(const l1_f32x4 *)(s2 + sl * L1_PITCH + 4 * tx);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x = fmaf(a4[i], r2[c], r1[c] - o1[i][c]);
                        const float u = PN == 1 ? __builtin_amdgcn_fmed3f(x * L1_BIG, -1.f, 1.f) : x;
                        acc1[i][c] = fmaf(w4[i], u, fmaf(-p4[i], r2[c], acc1[i][c]));
                    }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t off = ((int64_t)split * own_pad + o0 + 4 * ty + i) * dp + j0 + 4 * tx;
        *(l1_f32x4 *)(acc_part + off) = l1_f32x4{acc1[i][0], acc1[i][1], acc1[i][2], acc1[i][3]};
        if constexpr (OWN_Q) *(l1_f32x4 *)(acc_part2 + off) = l1_f32x4{acc2[i][0], acc2[i][1], acc2[i][2], acc2[i][3]};
    }
}

}  // namespace

int kge_run_l1_score(bool bf16, const float *Q, const void *T, int B, int N, int Bp, int Np, int dp, int dim, float *S, int64_t ldS,
                     hipStream_t st) {
    if (Bp % L1_TILE || Np % L1_TILE || dp % L1_TILE) return KGE_E_INVALID_ARG;
    if (Bp == 0 || Np == 0) return KGE_OK;
    if (Bp / L1_TILE > 65535) return KGE_E_UNSUPPORTED;   // grid limit of the second dimension
    KgeProfScope prof(KGE_PROF_BLOCK_SCORE, st);
    // (rows past B and N and columns past the dimension are padding: no workgroup takes a tile of them alone)
    const int cols = (dim + L1_TILE - 1) / L1_TILE * L1_TILE;
    auto tiles = [&](int qr, int kn) { return (int64_t)((N + 16 * kn - 1) / (16 * kn)) * ((B + 16 * qr - 1) / (16 * qr)); };
    // 64 x 64 tiles feed eight operations from every LDS read; 32 queries per tile where the others would not fill the chip twice
    // (512 x 1,280 x 384: 22 us against 31), and there 48 negatives or 64, whichever leaves the fullest compute unit less to do
    // (512 x 1,280 x 384: 432 workgroups of 48, 18.7 us; 320 of 64, 21.5)
    const bool half = tiles(4, 4) < 512;
    auto load = [&](int kn) { return (tiles(2, kn) + 255) / 256 * kn; };
    const int kn = !half || load(4) <= load(3) ? 4 : 3;
    const dim3 grid((N + 16 * kn - 1) / (16 * kn), half ? (B + 31) / 32 : (B + 63) / 64);
#define L1_SCORE(BF, QR, KN) hipLaunchKernelGGL((l1_score_kernel<BF, QR, KN>), grid, dim3(256), 0, st, Q, T, B, N, Np, dp, cols, S, ldS)
    if (bf16) { if (!half) L1_SCORE(true, 4, 4); else if (kn == 4) L1_SCORE(true, 2, 4); else L1_SCORE(true, 2, 3); }
    else      { if (!half) L1_SCORE(false, 4, 4); else if (kn == 4) L1_SCORE(false, 2, 4); else L1_SCORE(false, 2, 3); }
#undef L1_SCORE
    return kge_launch_status();
}

// splits over the streamed rows: enough workgroups for about four per compute unit
int kge_l1_nsplit(int own_pad, int str_pad, int dp, bool transh) {
    const int base = (own_pad / (transh ? L1H_GO : L1_GO)) * (dp / L1_GD), chunks = str_pad / L1_GS;
    if (base == 0 || chunks == 0) return 0;
    int want = (1024 + base - 1) / base;
    if (want > chunks) want = chunks;
    const int cps = (chunks + want - 1) / want;
    return (chunks + cps - 1) / cps;
}

size_t kge_l1_most_part(int own_pad, int str_pad, int dp, bool transh) {
    const size_t go = transh ? L1H_GO : L1_GO, own = own_pad / go, split = own + 1023 / (dp / L1_GD), whole = own * (str_pad / L1_GS);
    return go * (split < whole ? split : whole);
}

int kge_run_l1_grad(bool bf16, const float *Q, const void *T, const float *W, int64_t ldW, int B, int N, int Bp, int Np, int dp, int dim,
                    int &nsplit_q, int &nsplit_t, float *accq, float *acct, hipStream_t st) {
    if (Bp % L1_GO || Np % L1_GO || Bp % L1_GS || Np % L1_GS || dp % L1_GD) return KGE_E_INVALID_ARG;
    if (nsplit_q <= 0 || nsplit_t <= 0 || nsplit_q != kge_l1_nsplit(Bp, Np, dp, false) || nsplit_t != kge_l1_nsplit(Np, Bp, dp, false))
        return KGE_E_INVALID_ARG;
    KgeProfScope prof(KGE_PROF_BLOCK_FWD, st);
    {
        L1BothArgs a{Q, T, W, ldW, B, N, Bp, Np, dp};
        const int blocks = (N + L1_BN - 1) / L1_BN;
        a.col_tiles = (dim + L1_GD - 1) / L1_GD; a.chunks = (B + L1_BQ - 1) / L1_BQ;
        const int most_g = nsplit_q < blocks ? nsplit_q : blocks, most_s = nsplit_t < a.chunks ? nsplit_t : a.chunks;
        a.bpg = (blocks + most_g - 1) / most_g; a.groups = (blocks + a.bpg - 1) / a.bpg;
        a.cps = (a.chunks + most_s - 1) / most_s;
        const int splits = (a.chunks + a.cps - 1) / a.cps;
        // A workgroup walks bpg blocks of negatives and, for each, cps chunks of queries: rounds that are bound by their latency, so long
        // walks pay only where the chip is full of them.  Whole calls against the two passes, us, by rounds (workgroups): up to 3, always
        // (243 to 1,392: 61.2 -> 59.6 to 117 -> 93; 270 and 300: 62.2 -> 61.4, 63.3 -> 63.6); 4 (165) 61 -> 70, (252) 67 -> 78, (368) 93 -> 98,
        // (462) 77.9 -> 76.1, (476) 78.3 -> 79.7, (576) 115 -> 110, (612) 127 -> 115, (1,029) 126 -> 107; 6 (192) 66 -> 90, (352) 78 -> 91, (492) 106 ->
        // 108, (567) 118.4 -> 117.9, (630) 118 -> 122, (704) 127 -> 118, (1,044) 186 -> 168; 8 (248) 83 -> 116, (464) 132 -> 136, (540) 121 -> 124,
        // (684) 156 -> 151, (686) 138 -> 146, (693) 165 -> 155, (800) 160 -> 152, (1,024) 199 -> 184; 32 1,000 x 4,000 x 384 287 -> 398, 2,048 x 4,096 x
        // 256 360 -> 422; 45 3,000 x 3,000 x 256 403 -> 552
        const int rounds = a.bpg * a.cps;
        const int64_t wgs = (int64_t)a.col_tiles * a.groups * splits;
        if (rounds <= 3 || (rounds <= 8 && wgs >= (rounds == 4 ? 512 : 690))) {
            a.accq = accq; a.acct = acct;
            nsplit_q = a.groups; nsplit_t = splits;
            if (wgs > 0x7fffffff) return KGE_E_UNSUPPORTED;
            if (bf16) hipLaunchKernelGGL(l1_grad_both_kernel<true>, dim3((unsigned)wgs), dim3(256), 0, st, a);
            else      hipLaunchKernelGGL(l1_grad_both_kernel<false>, dim3((unsigned)wgs), dim3(256), 0, st, a);
            return kge_launch_status();
        }
    }
    // (the split counts are those of the padded block, their work that of the rows and columns there are; a split past them writes zeros)
    auto part = [&](const void *own, const void *str, float *acc, int own_pad, int own_n, int str_n, int nsplit) {
        const int chunks = (str_n + L1_GS - 1) / L1_GS;
        return L1GradPart{own, str, acc, own_pad, (own_n + L1_GO - 1) / L1_GO, (dim + L1_GD - 1) / L1_GD, chunks, (chunks + nsplit - 1) / nsplit};
    };
    const L1GradPart q = part(Q, T, accq, Bp, B, N, nsplit_q), t = part(T, Q, acct, Np, N, B, nsplit_t);
    const int64_t qb = (int64_t)q.own_tiles * q.col_tiles * nsplit_q, tb = (int64_t)t.own_tiles * t.col_tiles * nsplit_t;
    if (qb + tb > 0x7fffffff) return KGE_E_UNSUPPORTED;
    if (bf16) hipLaunchKernelGGL(l1_grad_kernel<true>, dim3((unsigned)(qb + tb)), dim3(256), 0, st, q, t, (int)qb, W, ldW, B, N, dp);
    else      hipLaunchKernelGGL(l1_grad_kernel<false>, dim3((unsigned)(qb + tb)), dim3(256), 0, st, q, t, (int)qb, W, ldW, B, N, dp);
    return kge_launch_status();
}

// TransH: scores (and, with A and P given, the two per-pair scalars that the gradient kernels need)
int kge_run_l1h_score(bool bf16, const float *Q, const float *W, const void *T, int B, int N, int Bp, int Np, int dp, float *S,
                      float *A, float *P, int64_t ldS, hipStream_t st, int pn) {
    if (Bp % L1_TILE || Np % L1_TILE || dp % L1_TILE || (A == nullptr) != (P == nullptr)) return KGE_E_INVALID_ARG;
    if (Bp == 0 || Np == 0) return KGE_OK;
    if (Bp / L1_TILE > 65535) return KGE_E_UNSUPPORTED;
    KgeProfScope prof(KGE_PROF_BLOCK_SCORE, st);
    const dim3 grid(Np / L1_TILE, Bp / L1_TILE);
#define L1H_SCORE(BF, PN) hipLaunchKernelGGL((l1h_score_kernel<BF, PN>), grid, dim3(256), 0, st, Q, W, T, B, N, dp, S, A, P, ldS)
    if (bf16) { if (pn == 1) L1H_SCORE(true, 1); else L1H_SCORE(true, 2); }
    else      { if (pn == 1) L1H_SCORE(false, 1); else L1H_SCORE(false, 2); }
#undef L1H_SCORE
    return kge_launch_status();
}

int kge_run_l1h_grad(bool bf16, bool own_is_query, const float *Q, const float *W, const void *T, const float *S, const float *A,
                     const float *P, int64_t ldS, const KgeRowInfo *rowinfo, int B, int N, int own_pad, int str_pad, int dp,
                     int loss, float gamma, float adv_temp, int nsplit, float *acc_part, float *acc_part2, hipStream_t st, int pn) {
    if (own_pad % L1H_GO || str_pad % L1_GS || dp % L1_GD) return KGE_E_INVALID_ARG;
    if (nsplit <= 0 || nsplit != kge_l1_nsplit(own_pad, str_pad, dp, true)) return KGE_E_INVALID_ARG;
    KgeProfScope prof(own_is_query ? KGE_PROF_BLOCK_FWD : KGE_PROF_BLOCK_GRADT, st);
    const int chunks = str_pad / L1_GS, cps = (chunks + nsplit - 1) / nsplit;
    const dim3 grid(own_pad / L1H_GO, dp / L1_GD, nsplit);
    if (grid.z > 65535 || grid.y > 65535) return KGE_E_UNSUPPORTED;
#define L1H_GRAD(BF, OQ) do { if (pn == 1) hipLaunchKernelGGL((l1h_grad_kernel<BF, OQ, 1>), grid, dim3(256), 0, st, Q, W, T, S, A, P, ldS, rowinfo, B, N, \
                                                                  own_pad, dp, chunks, cps, loss, gamma, adv_temp, acc_part, acc_part2); \
                              else hipLaunchKernelGGL((l1h_grad_kernel<BF, OQ, 2>), grid, dim3(256), 0, st, Q, W, T, S, A, P, ldS, rowinfo, B, N, \
                                                      own_pad, dp, chunks, cps, loss, gamma, adv_temp, acc_part, acc_part2); } while (0)
    if (bf16) { if (own_is_query) L1H_GRAD(true, true); else L1H_GRAD(true, false); }
    else      { if (own_is_query) L1H_GRAD(false, true); else L1H_GRAD(false, false); }
#undef L1H_GRAD
    return kge_launch_status();
}
