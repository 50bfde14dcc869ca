// Feature-projection encoder (arXiv 2211.12281, Section 3.1 "Encoder", eq. (embedding)):
//     e = e_S + M_H e_F  for head entities,   e = e_S + M_T e_F  for tail entities,
// with dropout on the projection and the L3 regularisers of e, e_S and M e_F (Section 3.1
// "Regularisation").  The projection of the 2B + N gathered slots is the second dense contraction of
// the paper's cost model, (B + N) |e_F| d (Section 4.1), and so is its backward pass to M_H, M_T.
//
//   forward    P[slot, d]  = F[idx[slot], :] . M[d, :]^t     both operands contiguous along the contraction (enc_gemm_nt_kernel);
//                                                            the feature rows are gathered by the copies into the LDS
//   backward   G[d, f]     = sum over slots of dP[slot, d] F[idx[slot], f]     both operands contiguous ACROSS it
//                                                            (enc_gemm_tn_kernel): rows are copied into the LDS as they lie - the
//                                                            feature rows again straight from the table - and read transposed;
//                                                            split over the slots, partials summed in order
// (The backward contraction used to run on transposed copies of both operands: writing them took 39 us of gather, 9 us of zeroing their
// padding and the detour of the row kernel through the LDS, against 22 us for the contraction itself; 24,576 slots,
// 768 x 256, bf16: encode + encode_bwd 182 -> 94 us.)
#include "kge_internal.h"
#include "row_ops.hpp"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 enc_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float enc_f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float enc_f32x4;
typedef uint32_t enc_u32x4 __attribute__((ext_vector_type(4)));   // (arrays of HIP's uint4 struct end up in scratch memory)

namespace {

constexpr int ENC_TILE = 128;          // rows and columns of a workgroup's output tile; slot counts are padded to it

template <bool BF16>
__device__ __forceinline__ enc_f32x16 enc_mma16(enc_f32x16 acc, enc_u32x4 a, enc_u32x4 b) {
    if constexpr (BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(enc_bf16x8, a), __builtin_bit_cast(enc_bf16x8, b),
                                                       acc, 0, 0, 0);
    } else {
        const enc_f32x4 fa = __builtin_bit_cast(enc_f32x4, a), fb = __builtin_bit_cast(enc_f32x4, b);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[r], fb[r], acc, 0, 0, 0);
        return acc;
    }
}

// One contraction C[M, N] (fp32) = A[M, K] . B[N, K]^t, K counted in k-steps of 32 bytes of a row (16 bf16 or 8 fp32).
// A's row r is table row idx0[r] for r < n_idx0, idx1[r - n_idx0] beyond: the gather of the feature rows is part of the load.
struct EncGemm {
    const char *A; int64_t lda_b; const int32_t *idx0, *idx1; int n_idx0, m_valid;
    const char *B; int64_t ldb_b; int n_valid;
    float *C; int64_t ldc;
    int ksteps, tiles_m, tiles_n;                            // (tiles: of the launched kernel's size)
};
// A launch runs two contractions (heads against M_H, tails and negatives against M_T) so that the chip is filled
// once; work items enumerate (contraction, row tile, column tile), column tile fastest.
struct EncGemmPair { EncGemm g[2]; int wgs0, total; };

constexpr int ENC_NSTAGE = 4;                                // chunks resident in the LDS ring
constexpr int ENC_ROW_BYTES = 64;                            // a chunk is two k-steps: 64 bytes of every row
constexpr int ENC_HALF_BYTES = ENC_TILE * ENC_ROW_BYTES;     // one operand's rows of one chunk
constexpr int ENC_STAGE_BYTES = 2 * ENC_HALF_BYTES;
constexpr int ENC_LDS_BYTES = ENC_NSTAGE * ENC_STAGE_BYTES;  // 64 KB: two workgroups per compute unit
constexpr int ENC_LPW = 4;                                   // asynchronous copies per wave and chunk

__device__ __forceinline__ void enc_async_copy16(const void *g, uint32_t lds_addr) {
    // lane l of the wave writes its 16 bytes to LDS byte address lds_addr + 16 l; completion is tracked by vmcnt and
    // the compiler does not see the load, so the waits below are explicit
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(g) : "memory");
}
template <int N> __device__ __forceinline__ void enc_wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup = MT x NT outputs (128 x 128, or 64 on a side: enc_launch_pair), wave = a quarter of them (2 x 2 blocks of 32 x 32 at 128 x
// 128).  Both operands pass through the LDS
// in chunks of two k-steps (64 bytes of every row).  The chunks are copied global -> LDS asynchronously into a
// ring of ENC_NSTAGE stages, so that the rows of ENC_NSTAGE - 1 chunks (random table rows in the forward pass:
// pure latency) are in flight while one chunk is multiplied; no registers are tied up by the copies.  The ring
// takes 64 KB at 128 x 128 and the kernel at most 128 registers per lane, so two workgroups share a compute unit: one's
// prologue, barriers and write-out overlap the other's products.  A 64-byte LDS row keeps its four 16-byte pieces
// XOR-swizzled by (row / 2) % 4, so that the fragment reads of 8 consecutive rows fall into 8 different bank
// groups; a copy instruction fills 16 rows, lane l fetching piece (l % 4) ^ ((l / 8) % 4) of row l / 4 into slot
// l % 4.  Fragment of (row block, k-step): lane l reads piece 2 ks + l / 32 of row l % 32.  Rows beyond m_valid /
// n_valid are read from row 0 instead (valid memory); their outputs are never stored.  An odd last k-step goes
// through registers with zeros selected for the missing pieces.
// Workgroup ids are dealt round-robin to the 8 dies: id -> work item (id % 8) * ceil(total / 8) + id / 8, so that
// the tiles that share operand rows run on the same die and meet in its L2.
template <bool BF16, int MT, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MT == 128 ? 2 : 3, MT == 128 ? 2 : 3))) void enc_gemm_nt_kernel(const EncGemmPair pr) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int NI = MT / 64, NJ = NT / 64, RPW = MT / 4, BPW = NT / 4;    // row and column blocks of a wave; rows that it copies
    constexpr int A_BYTES = MT * ENC_ROW_BYTES, STAGE = A_BYTES + NT * ENC_ROW_BYTES, LPW = NI + NJ;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, g = lane >> 5;
    const int per = (pr.total + 7) >> 3;
    int w = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (w >= pr.total) return;
    const bool second = w >= pr.wgs0;
    const EncGemm &q = pr.g[second ? 1 : 0];
    w -= second ? pr.wgs0 : 0;
    const int m0 = w / q.tiles_n * MT, n0 = w % q.tiles_n * NT;
    const int nfull = q.ksteps >> 1, rem = q.ksteps & 1;
    // staging: copy j of wave v fills rows 16 NI v + 16 j .. + 15 of A's tile, 16 NJ v + 16 j .. + 15 of B's; this lane's row and piece
    const int srow = lane >> 2, piece = (lane & 3) ^ ((srow >> 1) & 3);
    const char *ga[NI], *gb[NJ];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int ra = m0 + RPW * wave + 16 * j + srow;
        int64_t src = 0;
        if (ra < q.m_valid) src = ra < q.n_idx0 ? (int64_t)q.idx0[ra] : (int64_t)q.idx1[ra - q.n_idx0];
        ga[j] = q.A + src * q.lda_b + piece * 16;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int rb = n0 + BPW * wave + 16 * j + srow;
        gb[j] = q.B + (int64_t)(rb < q.n_valid ? rb : 0) * q.ldb_b + piece * 16;
    }
    // the row indices must have arrived before the loop: a compiler-inserted wait inside it would drain the ring
#pragma unroll
    for (int j = 0; j < NI; ++j) asm volatile("" : "+v"(ga[j]));
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(gb[j]));
    auto issue = [&](int c) {                             // chunk min(c, nfull - 1) -> stage c % ENC_NSTAGE
        const int64_t off = (int64_t)min(c, nfull - 1) * ENC_ROW_BYTES;
        const uint32_t sb = lds0 + (uint32_t)(c & (ENC_NSTAGE - 1)) * STAGE;
#pragma unroll
        for (int j = 0; j < NI; ++j) enc_async_copy16(ga[j] + off, __builtin_amdgcn_readfirstlane(sb + (uint32_t)wave * (RPW * ENC_ROW_BYTES) + j * 1024));
#pragma unroll
        for (int j = 0; j < NJ; ++j) enc_async_copy16(gb[j] + off, __builtin_amdgcn_readfirstlane(sb + A_BYTES + (uint32_t)wave * (BPW * ENC_ROW_BYTES) + j * 1024));
    };
    enc_f32x16 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
        for (int j = 0; j < NJ; ++j)
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const int wm = (wave & 1) * (32 * NI), wn = (wave >> 1) * (32 * NJ);
    auto compute = [&](int stage) {
        const char *sa = lds + stage * STAGE, *sb = sa + A_BYTES;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            enc_u32x4 fa[NI], fb[NJ];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int rowa = wm + 32 * i + lr;
                fa[i] = *(const enc_u32x4 *)(sa + rowa * ENC_ROW_BYTES + (((2 * ks + g) ^ ((rowa >> 1) & 3)) * 16));
            }
#pragma unroll
            for (int i = 0; i < NJ; ++i) {
                const int rowb = wn + 32 * i + lr;
                fb[i] = *(const enc_u32x4 *)(sb + rowb * ENC_ROW_BYTES + (((2 * ks + g) ^ ((rowb >> 1) & 3)) * 16));
            }
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[i][j] = enc_mma16<BF16>(acc[i][j], fa[i], fb[j]);
        }
    };
    static_assert((ENC_NSTAGE & (ENC_NSTAGE - 1)) == 0 && (ENC_NSTAGE - 2) * LPW < 64, "ring size");
    if (nfull > 0) {
        for (int c = 0; c < ENC_NSTAGE - 1; ++c) issue(c);
        for (int c = 0; c < nfull; ++c) {
            // chunks up to c + ENC_NSTAGE - 2 are issued; all but the last ENC_NSTAGE - 2 of them must have landed
            enc_wait_vmcnt<(ENC_NSTAGE - 2) * LPW>();
            __syncthreads();                                // chunk c is complete; everyone is done with chunk c - 1
            issue(c + ENC_NSTAGE - 1);                      // ... whose stage is refilled (past the end: a harmless repeat)
            compute(c & (ENC_NSTAGE - 1));
        }
        enc_wait_vmcnt<0>();                                // no copy may be in flight when the LDS is reused or released
    }
    if (rem > 0) {
        __syncthreads();
        const enc_u32x4 zero = {0u, 0u, 0u, 0u};
        const bool in = (piece >> 1) < rem;
#pragma unroll
        for (int j = 0; j < NI; ++j)
            *(enc_u32x4 *)(lds + (RPW * wave + 16 * j) * ENC_ROW_BYTES + lane * 16) = in ? *(const enc_u32x4 *)(ga[j] + (int64_t)nfull * ENC_ROW_BYTES) : zero;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            *(enc_u32x4 *)(lds + A_BYTES + (BPW * wave + 16 * j) * ENC_ROW_BYTES + lane * 16) = in ? *(const enc_u32x4 *)(gb[j] + (int64_t)nfull * ENC_ROW_BYTES) : zero;
        __syncthreads();
        compute(0);
    }
    // accumulator layout: lane holds column lr of the B side; register e holds A-side row 8 (e/4) + 4 g + e%4
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int col = n0 + wn + 32 * j + lr;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = m0 + wm + 32 * i + 8 * (e >> 2) + 4 * g + (e & 3);
                if (row < q.m_valid && col < q.n_valid) q.C[(int64_t)row * q.ldc + col] = acc[i][j][e];
            }
        }
}

__device__ __forceinline__ void enc_philox_round(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
}
// dropout factors of elements (slot, column .. column + 3), column a multiple of four: counter (slot, column / 4, step, tag), word
// column % 4; kept when the word is >= thr = floor(p 2^32), then scaled by 1 / (1 - p).  (One generator block for four columns: with a
// block per element the row kernels were bound by its integer multiplications, 23 and 40 us where these take 13 and 20.)
__device__ __forceinline__ void enc_dropout4(uint32_t seed_lo, uint32_t seed_hi, uint32_t step, uint32_t tag, uint32_t slot, int col,
                                             uint32_t thr, float scale, float (&f)[4]) {
    if (thr == 0u) { f[0] = f[1] = f[2] = f[3] = 1.f; return; }
    uint32_t c[4] = { slot, (uint32_t)(col >> 2), step, tag };
    uint32_t k0 = seed_lo, k1 = seed_hi;
#pragma unroll
    for (int r = 0; r < 10; ++r) { enc_philox_round(c, k0, k1); k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
#pragma unroll
    for (int u = 0; u < 4; ++u) f[u] = c[u] >= thr ? scale : 0.f;
}

struct EncRowArgs {
    const void *ent_s; int64_t ent_ld; const int32_t *h, *t, *neg; int B, N, d;
    uint32_t seed_lo, seed_hi, step, tag, thr; float scale, reg_t, reg_s, reg_f;
    int wide;                                              // every row of every operand starts where four elements load and store at once
};
// four consecutive elements of a row
template <bool BF16> __device__ __forceinline__ void enc_ld4(const void *p, int64_t i, bool wide, float (&v)[4]) {
    if (wide) {
        if constexpr (BF16) {
            const uint2 r = *(const uint2 *)((const __bf16 *)p + i);
            v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xffff0000u);
            v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xffff0000u);
        } else { const enc_f32x4 r = *(const enc_f32x4 *)((const float *)p + i); v[0] = r[0]; v[1] = r[1]; v[2] = r[2]; v[3] = r[3]; }
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = El<BF16>::ld(p, i + u);
    }
}
template <bool BF16> __device__ __forceinline__ void enc_st4(void *p, int64_t i, bool wide, const float (&v)[4]) {
    if (wide) {
        if constexpr (BF16) {
            typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf4;
            const bf4 r = { (__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3] };
            *(uint2 *)((__bf16 *)p + i) = __builtin_bit_cast(uint2, r);
        } else *(enc_f32x4 *)((float *)p + i) = enc_f32x4{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) El<BF16>::st(p, i + u, v[u]);
    }
}
__device__ __forceinline__ int enc_slot_entity(const EncRowArgs &a, int i) {
    return i < a.B ? a.h[i] : (i < 2 * a.B ? a.t[i - a.B] : a.neg[i - 2 * a.B]);
}
__device__ __forceinline__ float enc_l3(float c3) { return cbrtf(kge_wave_sum(c3)); }

// forward rows: e = s + D o P, the three norms of the slot; one wave per slot, a lane holds columns 4 lane + 256 k .. + 3; regv: one
// sum per workgroup of four slots
constexpr int ENC_G4 = 2;                                  // groups of four columns per lane (d <= 512)
template <bool BF16>
__global__ __launch_bounds__(256) void enc_finish_kernel(EncRowArgs a, const float *P, void *e_out, double *regv) {
    __shared__ float part[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + wave;
    const bool reg = a.reg_t > 0.f || a.reg_s > 0.f || a.reg_f > 0.f, wide = a.wide != 0;
    float v = 0.f;
    if (i < 2 * a.B + a.N) {
        const int64_t soff = (int64_t)enc_slot_entity(a, i) * a.ent_ld, off = (int64_t)i * a.d;
        float ct = 0.f, cs = 0.f, cf = 0.f;
#pragma unroll
        for (int k = 0; k < ENC_G4; ++k) {
            const int j = 4 * lane + 256 * k;
            if (j >= a.d) continue;
            float p[4], s[4], D[4], e[4];
            enc_ld4<false>(P, off + j, wide, p);
            enc_ld4<BF16>(a.ent_s, soff + j, wide, s);
            enc_dropout4(a.seed_lo, a.seed_hi, a.step, a.tag, (uint32_t)i, j, a.thr, a.scale, D);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                e[u] = s[u] + D[u] * p[u];
                ct += fabsf(e[u]) * e[u] * e[u]; cs += fabsf(s[u]) * s[u] * s[u]; cf += fabsf(p[u]) * p[u] * p[u];
            }
            enc_st4<BF16>(e_out, off + j, wide, e);
        }
        if (reg) v = a.reg_t * enc_l3(ct) + a.reg_s * enc_l3(cs) + a.reg_f * enc_l3(cf);
    }
    if (!reg) return;
    if (lane == 0) part[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) regv[blockIdx.x] = ((double)part[0] + (double)part[1]) + ((double)part[2] + (double)part[3]);
}

// reg_out = sum of the workgroups' sums in a fixed order (one workgroup)
__global__ void enc_reg_reduce_kernel(const double *regv, int n, int on, float *reg_out) {
    __shared__ double sh[1024];
    double p[4] = {0, 0, 0, 0};
    if (on)
        for (int i0 = threadIdx.x; i0 < n; i0 += 4 * 1024)
#pragma unroll
            for (int u = 0; u < 4; ++u) { const int i = i0 + u * 1024; p[u] += i < n ? regv[i] : 0.0; }
    sh[threadIdx.x] = (p[0] + p[1]) + (p[2] + p[3]);
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *reg_out = (float)sh[0];
}

// backward rows, one wave per slot: de' = de + reg_t grad||e||, g_es = de' + reg_s grad||s||, dP = D o de' + reg_f grad||P||; dP in the
// table type, row by row (16 bytes per lane's group; the rows start 16-byte aligned).  Workgroup 0 also writes the zero bytes that the
// contraction reads where there is no element.
template <bool BF16>
__global__ __launch_bounds__(256) void enc_bwd_rows_kernel(EncRowArgs a, const float *P, const float *de, float *g_es, void *dP, uint32_t *zeros) {
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x < 64) zeros[threadIdx.x] = 0u;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= 2 * a.B + a.N) return;
    const bool wide = a.wide != 0;
    const int64_t soff = (int64_t)enc_slot_entity(a, i) * a.ent_ld, off = (int64_t)i * a.d;
    float pv[ENC_G4][4], sv[ENC_G4][4], ev[ENC_G4][4], dv[ENC_G4][4], Df[ENC_G4][4];
    float ct = 0.f, cs = 0.f, cf = 0.f;
#pragma unroll
    for (int k = 0; k < ENC_G4; ++k) {
        const int j = 4 * lane + 256 * k;
        if (j >= a.d) continue;
        enc_ld4<false>(P, off + j, wide, pv[k]);
        enc_ld4<BF16>(a.ent_s, soff + j, wide, sv[k]);
        enc_ld4<false>(de, off + j, wide, dv[k]);
        enc_dropout4(a.seed_lo, a.seed_hi, a.step, a.tag, (uint32_t)i, j, a.thr, a.scale, Df[k]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float e = sv[k][u] + Df[k][u] * pv[k][u];
            ev[k][u] = e;
            ct += fabsf(e) * e * e; cs += fabsf(sv[k][u]) * sv[k][u] * sv[k][u]; cf += fabsf(pv[k][u]) * pv[k][u] * pv[k][u];
        }
    }
    float ft = 0.f, fs = 0.f, ff = 0.f;
    if (a.reg_t > 0.f) { const float nrm = enc_l3(ct); ft = nrm > 0.f ? a.reg_t / (nrm * nrm) : 0.f; }
    if (a.reg_s > 0.f) { const float nrm = enc_l3(cs); fs = nrm > 0.f ? a.reg_s / (nrm * nrm) : 0.f; }
    if (a.reg_f > 0.f) { const float nrm = enc_l3(cf); ff = nrm > 0.f ? a.reg_f / (nrm * nrm) : 0.f; }
#pragma unroll
    for (int k = 0; k < ENC_G4; ++k) {
        const int j = 4 * lane + 256 * k;
        if (j >= a.d) continue;
        float gs[4], dp[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float dep = dv[k][u] + ft * fabsf(ev[k][u]) * ev[k][u];
            gs[u] = dep + fs * fabsf(sv[k][u]) * sv[k][u];
            dp[u] = Df[k][u] * dep + ff * fabsf(pv[k][u]) * pv[k][u];
        }
        enc_st4<false>(g_es, off + j, wide, gs);
        enc_st4<BF16>(dP, off + j, true, dp);
    }
}

// One section (heads against M_H, or tails and negatives against M_T) of the backward contraction, C[split][d, fd] (fp32) =
// sum over the split's slots of A[slot, d] F[id(slot), fd]; slot s of the section is entity ids0[s] (s < n0) or ids1[s - n0].
struct EncTn { const char *A; const int32_t *ids0, *ids1; int n0, slots; float *C; };
struct EncTnPair { EncTn g[2]; const char *feat; int64_t ldf_b; int d, fd, sps, tiles_m, tiles_n, wgs0, total; const void *zeros; };

// Workgroup = 128 x 128 outputs, wave = 64 x 64; both operands come into the LDS as rows of 128 columns, in chunks of 8 KB per operand
// (32 slots bf16, 16 fp32) through the same ring as above.  bf16: a fragment holds eight slots of one column, which the LDS transpose
// read (ds_read_b64_tr_b16) makes of four 8-byte pieces of four rows; the 16-byte pieces of a row are XOR-swizzled by 4 (row % 4) so that
// the four rows of a read lie in different quarters of the banks.  fp32: a lane reads single values (one slot, consecutive columns
// across the lanes), pieces swizzled by 8 (row % 2).  The ids of the split's slots are fetched into the LDS first: a load in the loop
// would wait for the copies in flight.  Columns past d or fd and slots past the section read zero bytes.
constexpr int ENC_MAX_SPS = 1024;                            // slots per split at most
constexpr int ENC_TN_WGS = 512;                              // (both calls, 24,576 slots x 768 x 256, the same slots again and again - new ones take 94: bf16 82 us, 384 workgroups 83, 256 86; fp32 242 / 265 / 292)
template <bool BF16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void enc_gemm_tn_kernel(const EncTnPair pr) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int ES = BF16 ? 2 : 4, RBY = 128 * ES, CH = ENC_HALF_BYTES / RBY, LPR = RBY / 16, RPI = 64 / LPR;   // row bytes, slots per chunk, lanes per row, rows per copy
    static_assert(CH == 8 * RPI, "eight copies per operand and chunk");
    int32_t *ids = (int32_t *)(lds + ENC_LDS_BYTES);         // [ENC_MAX_SPS]
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, g = lane >> 5;
    const int per = (pr.total + 7) >> 3;
    int w = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (w >= pr.total || ((int)blockIdx.x >> 3) >= per) return;
    const bool second = w >= pr.wgs0;
    const EncTn &q = pr.g[second ? 1 : 0];
    w -= second ? pr.wgs0 : 0;
    const int tn = w % pr.tiles_n; w /= pr.tiles_n;
    const int tm = w % pr.tiles_m, split = w / pr.tiles_m;
    const int m0 = tm * ENC_TILE, n0 = tn * ENC_TILE;
    const int s_lo = split * pr.sps, s_hi = min(q.slots, s_lo + pr.sps), nch = (s_hi - s_lo + CH - 1) / CH;
    for (int i = tid; i < nch * CH; i += 256) {
        const int sl = s_lo + i;
        ids[i] = sl < s_hi ? (sl < q.n0 ? q.ids0[sl] : q.ids1[sl - q.n0]) : -1;
    }
    __syncthreads();
    // copy j (j < 2) of wave v fills rows (2 v + j) RPI .. of a chunk; this lane's row of a copy and its piece of the row
    const int srow = lane / LPR;
    int piece[2];
    bool in_a[2], in_b[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = (2 * wave + j) * RPI + srow;
        piece[j] = (lane % LPR) ^ (BF16 ? (row & 3) << 2 : (row & 1) << 3);
        in_a[j] = m0 + piece[j] * (16 / ES) < pr.d;          // (d and fd are multiples of a piece)
        in_b[j] = n0 + piece[j] * (16 / ES) < pr.fd;
    }
    const char *fa = pr.feat + (int64_t)n0 * ES, *aa = q.A + (int64_t)m0 * ES;
    auto issue = [&](int c) {                                // chunk min(c, nch - 1) -> stage c % ENC_NSTAGE
        const int cc = min(c, nch - 1);
        const uint32_t sb = lds0 + (uint32_t)(c & (ENC_NSTAGE - 1)) * ENC_STAGE_BYTES + (uint32_t)wave * 2048;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = cc * CH + (2 * wave + j) * RPI + srow, id = ids[row];
            const void *pa = id >= 0 && in_a[j] ? (const void *)(aa + (int64_t)(s_lo + row) * pr.d * ES + piece[j] * 16) : pr.zeros;
            const void *pb = id >= 0 && in_b[j] ? (const void *)(fa + (int64_t)id * pr.ldf_b + piece[j] * 16) : pr.zeros;
            enc_async_copy16(pa, __builtin_amdgcn_readfirstlane(sb + j * 1024));
            enc_async_copy16(pb, __builtin_amdgcn_readfirstlane(sb + ENC_HALF_BYTES + j * 1024));
        }
    };
    enc_f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j)
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;
    auto compute = [&](int stage) {
        const char *sa = lds + stage * ENC_STAGE_BYTES, *sb = sa + ENC_HALF_BYTES;
        if constexpr (BF16) {
            typedef short i16x4 __attribute__((ext_vector_type(4)));
            const int i16 = lane & 15, q16 = (lane >> 4) & 1;
            // source lane i16 of a group of sixteen points at row 16 ks + 8 g + 4 hh + i16 / 4, columns .. + 16 q16 + 4 (i16 % 4) .. + 3 and
            // receives column .. + lane % 32 of the rows 16 ks + 8 g + 4 hh .. + 3
            auto frag = [&](const char *s, int c0, int ks) {
                const int pc = (c0 / 8 + 2 * q16 + ((i16 & 3) >> 1)) ^ ((i16 >> 2) << 2);
                const char *p = s + (16 * ks + 8 * g + (i16 >> 2)) * RBY + pc * 16 + (i16 & 1) * 8;
                const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3))) *)p));
                const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3))) *)(p + 4 * RBY)));
                return enc_u32x4{lo.x, lo.y, hi.x, hi.y};
            };
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                enc_u32x4 xa[2], xb[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) { xa[i] = frag(sa, wm + 32 * i, ks); xb[i] = frag(sb, wn + 32 * i, ks); }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = enc_mma16<true>(acc[i][j], xa[i], xb[j]);
            }
        } else {
            auto val = [&](const char *s, int c0, int kk) {  // slot 2 kk + g, column c0 + lane % 32
                return *(const float *)(s + (2 * kk + g) * RBY + ((((c0 + lr) >> 2) ^ (g << 3)) * 16) + (lr & 3) * 4);
            };
#pragma unroll
            for (int kk = 0; kk < CH / 2; ++kk) {
                float xa[2], xb[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) { xa[i] = val(sa, wm + 32 * i, kk); xb[i] = val(sb, wn + 32 * i, kk); }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[i], xb[j], acc[i][j], 0, 0, 0);
            }
        }
    };
    for (int c = 0; c < ENC_NSTAGE - 1; ++c) issue(c);
    for (int c = 0; c < nch; ++c) {
        enc_wait_vmcnt<(ENC_NSTAGE - 2) * ENC_LPW>();
        __syncthreads();                                     // chunk c is complete; everyone is done with chunk c - 1
        issue(c + ENC_NSTAGE - 1);                           // ... whose stage is refilled (past the end: a harmless repeat)
        compute(c & (ENC_NSTAGE - 1));
    }
    enc_wait_vmcnt<0>();                                     // no copy may be in flight when the LDS is released
    float *Cs = q.C + (int64_t)split * pr.d * pr.fd;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn + 32 * j + lr;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = m0 + wm + 32 * i + 8 * (e >> 2) + 4 * g + (e & 3);
                if (row < pr.d && col < pr.fd) Cs[(int64_t)row * pr.fd + col] = acc[i][j][e];
            }
        }
}

// out[e] = sum over the splits, in split order; both projections in one launch
__global__ void enc_split_reduce_kernel(const float *part, int nsplit_h, int nsplit_t, int64_t count, float *g_mh, float *g_mt) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * count) return;
    const bool tail = i >= count;
    i -= tail ? count : 0;
    const float *p = part + (tail ? (int64_t)nsplit_h * count : 0) + i;
    const int n = tail ? nsplit_t : nsplit_h;
    float s = 0.f;
    int k = 0;
    for (; k + 8 <= n; k += 8) {                             // eight loads in flight
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(k + u) * count];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < n; ++k) s += p[(int64_t)k * count];
    (tail ? g_mt : g_mh)[i] = s;
}

struct EncPlan { int n, es; int sps, nsplit_h, nsplit_t; int64_t most_splits; };   // most_splits: of any call that is no larger

EncPlan enc_plan(const kge_encoder_t &e, int64_t B, int64_t N) {
    EncPlan p{};
    p.n = (int)(2 * B + N);
    p.es = e.dtype == KGE_BF16 ? 2 : 4;
    // Slots per split of the backward contraction: as many splits as keep its 128 x 128 output tiles within ENC_TN_WGS workgroups (two per
    // compute unit: one more would be a second turn), but no more than one per 128 slots and no more partials than fit where the
    // transposed feature rows of the batch would have.
    const int64_t tiles = ((e.dim + ENC_TILE - 1) / ENC_TILE) * (int64_t)((e.feat_dim + ENC_TILE - 1) / ENC_TILE);
    auto splits = [&](int64_t sps) { return (B + sps - 1) / sps + (B + N + sps - 1) / sps; };
    const int64_t room = (B + 1023) / 1024 + (B + N + 1023) / 1024 + (2 * B + N) * p.es / (4 * (int64_t)e.dim);
    const int64_t most = ENC_TN_WGS / tiles < room ? ENC_TN_WGS / tiles : room;
    int64_t sps = 128;
    while (sps < ENC_MAX_SPS && splits(sps) > most) sps += 32;
    p.sps = (int)sps;
    p.nsplit_h = (int)((B + sps - 1) / sps); p.nsplit_t = (int)((B + N + sps - 1) / sps);
    // (sps jumps by 32, so the splits of a larger batch can be fewer; all of these bounds grow with the batch)
    const int64_t bound = most > splits(ENC_MAX_SPS) ? most : splits(ENC_MAX_SPS);
    p.most_splits = bound < splits(128) ? bound : splits(128);
    return p;
}

// x, y, z: addresses of the [slots][dim] arrays that the row kernel reads and writes
EncRowArgs enc_row_args(const kge_encoder_t &e, const int32_t *h, const int32_t *t, int64_t B, const int32_t *neg, int64_t N,
                        uint64_t seed, uint64_t step, uintptr_t x, uintptr_t y, uintptr_t z = 0) {
    EncRowArgs a{};
    a.ent_s = e.ent_s; a.ent_ld = e.ent_ld; a.h = h; a.t = t; a.neg = neg; a.B = (int)B; a.N = (int)N; a.d = e.dim;
    a.seed_lo = (uint32_t)seed; a.seed_hi = (uint32_t)(seed >> 32); a.step = (uint32_t)step; a.tag = e.dropout_tag;
    a.thr = e.dropout > 0.f ? (uint32_t)floor((double)e.dropout * 4294967296.0) : 0u;
    a.scale = e.dropout > 0.f ? (float)(1.0 / (1.0 - (double)e.dropout)) : 1.f;
    a.reg_t = e.reg_t; a.reg_s = e.reg_s; a.reg_f = e.reg_f;
    // (dim is a multiple of eight: a row of the [slots][dim] arrays is aligned if the array is)
    a.wide = (e.ent_ld % 4 == 0 && ((uintptr_t)e.ent_s & 15) == 0 && ((x | y | z) & 15) == 0) ? 1 : 0;
    return a;
}

EncGemm enc_gemm_desc(const void *A, int64_t lda_b, const int32_t *idx0, int n_idx0, const int32_t *idx1, int m_valid, const void *Bm,
                      int64_t ldb_b, int n_valid, float *C, int64_t ldc, int ksteps) {
    EncGemm q{};
    q.A = (const char *)A; q.lda_b = lda_b; q.idx0 = idx0; q.idx1 = idx1; q.n_idx0 = n_idx0; q.m_valid = m_valid;
    q.B = (const char *)Bm; q.ldb_b = ldb_b; q.n_valid = n_valid; q.C = C; q.ldc = ldc; q.ksteps = ksteps;
    return q;
}

template <bool BF16, int MT, int NT>
int enc_launch_nt(EncGemmPair pr, hipStream_t st) {
    constexpr int LDS = ENC_NSTAGE * (MT + NT) * ENC_ROW_BYTES;
    static KgeLdsLimit limit;                               // the ring of stages is larger than the default dynamic limit
    if (limit.set((const void *)enc_gemm_nt_kernel<BF16, MT, NT>, LDS) != KGE_OK) return KGE_E_HIP;
    for (EncGemm &g : pr.g) { g.tiles_m = (g.m_valid + MT - 1) / MT; g.tiles_n = (g.n_valid + NT - 1) / NT; }
    pr.wgs0 = pr.g[0].tiles_m * pr.g[0].tiles_n;
    pr.total = pr.wgs0 + pr.g[1].tiles_m * pr.g[1].tiles_n;
    if (pr.total == 0) return KGE_OK;
    hipLaunchKernelGGL((enc_gemm_nt_kernel<BF16, MT, NT>), dim3((pr.total + 7) / 8 * 8), dim3(256), LDS, st, pr);
    return KGE_OK;
}

// Tiles of 128 x 128 share most of what they read, smaller ones fill the chip where those are few.
// Whole encode + encode_bwd, us, on new slots in every pass (on the same slots again and again, their rows in the caches, small tiles look
// better than they are).  bf16 (bound by the rows' latency and bytes): 64 x 64 while two of them to a compute unit are about
// all there are.  128 x 128 / 64 x 64, by the number of small tiles: 251 57.9 / 52.8, 470 62.1 / 59.8, 511 52.8 / 50.0, 532 55.9 / 54.4, 536 57.3 / 56.4,
// 558 57.4 / 57.2 (d 128: 534 65.1 / 66.8), 568 58.0 / 58.6, 57.6 / 58.1, 596 58.4 / 59.3, 664 60.1 / 61.2, 760 61.6 / 63.0, 1,536 96.4 / 102.2.
// fp32 (bound by the matrix pipe of the fullest compute unit): 64 x 128, or 64 x 64 where that leaves it less to do.  128 x 128 / 64 x
// 128 / 64 x 64: 24,576 slots, d 256 255 / 235 / 237; 16,384 169 / 166 / 184; 8,192 125 / 101 / 99; 1,234, d 80 88 / 61 / 49.  From 512 large
// tiles, two of them on every unit, those: 16,384, d 400 288 / 302 / 300; 40,960, d 256 (640 tiles) 395 / 397 / 394.
int enc_launch_pair(bool bf16, const EncGemm &g0, const EncGemm &g1, hipStream_t st) {
    EncGemmPair pr{};
    pr.g[0] = g0; pr.g[1] = g1;
    auto tiles = [&](int mt, int nt) {
        int64_t n = 0;
        for (const EncGemm &g : pr.g) n += (int64_t)((g.m_valid + mt - 1) / mt) * ((g.n_valid + nt - 1) / nt);
        return n;
    };
    if (bf16) return tiles(64, 64) <= 560 ? enc_launch_nt<true, 64, 64>(pr, st) : enc_launch_nt<true, 128, 128>(pr, st);
    if (tiles(128, 128) >= 512) return enc_launch_nt<false, 128, 128>(pr, st);
    auto rounds = [&](int mt, int nt) { return (tiles(mt, nt) + 255) / 256 * mt * nt; };
    return rounds(64, 64) < rounds(64, 128) ? enc_launch_nt<false, 64, 64>(pr, st) : enc_launch_nt<false, 64, 128>(pr, st);
}

}  // namespace

int kge_validate_encoder(const kge_encoder_t *e) {
    if (!e || (e->dtype != KGE_F32 && e->dtype != KGE_BF16)) return KGE_E_INVALID_ARG;
    const int es = e->dtype == KGE_BF16 ? 2 : 4;
    if (e->dim <= 0 || e->dim > 512 || e->dim % (32 / es) != 0) return KGE_E_INVALID_ARG;
    if (e->feat_dim <= 0 || e->feat_dim > 1024 || e->feat_dim % (32 / es) != 0) return KGE_E_INVALID_ARG;
    if (e->n_ent <= 0 || e->n_ent >= (1ll << 31) || !e->ent_s || !e->feat || !e->m_h || !e->m_t) return KGE_E_INVALID_ARG;
    if (e->ent_ld < e->dim || e->feat_ld < e->feat_dim || e->m_ld < e->feat_dim) return KGE_E_INVALID_ARG;
    // fragments are 16-byte loads: rows of the features and of the projections must start 16-byte aligned
    if ((e->feat_ld * es) % 16 != 0 || (e->m_ld * es) % 16 != 0 || ((uintptr_t)e->feat & 15) || ((uintptr_t)e->m_h & 15) ||
        ((uintptr_t)e->m_t & 15)) return KGE_E_INVALID_ARG;
    if (!(e->dropout >= 0.f && e->dropout < 1.f) || !(e->reg_t >= 0.f) || !(e->reg_s >= 0.f) || !(e->reg_f >= 0.f))
        return KGE_E_INVALID_ARG;
    return KGE_OK;
}

size_t kge_encode_ws(const kge_encoder_t &e, int64_t B, int64_t N, bool bwd, bool most) {
    const EncPlan p = enc_plan(e, B, N);
    size_t off = 0;
    auto take = [&](size_t bytes) { off += (bytes + 255) / 256 * 256; };
    if (!bwd) take((size_t)(p.n + 3) / 4 * 8);                                    // regulariser sums of four slots each
    else {
        take(256);                                                                // zero bytes
        take((size_t)e.dim * p.n * p.es);                                         // dP
        take((size_t)(most ? p.most_splits : p.nsplit_h + p.nsplit_t) * e.dim * e.feat_dim * 4);         // split partials of both contractions
    }
    return off + 256;
}

int kge_run_encode(const kge_encoder_t &e, const int32_t *h, const int32_t *t, int64_t B, const int32_t *neg, int64_t N,
                   uint64_t seed, uint64_t step, void *e_out, float *proj_out, float *reg_out, void *ws, hipStream_t st) {
    const EncPlan p = enc_plan(e, B, N);
    const bool bf16 = e.dtype == KGE_BF16;
    double *regv = (double *)ws;
    const int ksteps = e.feat_dim * p.es / 32;
    {
        KgeProfScope prof(KGE_PROF_ENC_FWD, st);          // heads against M_H, tails and negatives against M_T: one launch
        const EncGemm gh = enc_gemm_desc(e.feat, e.feat_ld * p.es, h, (int)B, nullptr, (int)B, e.m_h, e.m_ld * p.es, e.dim, proj_out, e.dim, ksteps);
        const EncGemm gt = enc_gemm_desc(e.feat, e.feat_ld * p.es, t, (int)B, neg, (int)(B + N), e.m_t, e.m_ld * p.es, e.dim,
                                         proj_out + (size_t)B * e.dim, e.dim, ksteps);
        if (int rc = enc_launch_pair(bf16, gh, gt, st)) return rc;
    }
    const EncRowArgs a = enc_row_args(e, h, t, B, neg, N, seed, step, (uintptr_t)proj_out, (uintptr_t)e_out);
    const bool reg = e.reg_t > 0.f || e.reg_s > 0.f || e.reg_f > 0.f;
    if (p.n > 0) {
        if (bf16) hipLaunchKernelGGL(enc_finish_kernel<true>, dim3((p.n + 3) / 4), dim3(256), 0, st, a, proj_out, e_out, regv);
        else      hipLaunchKernelGGL(enc_finish_kernel<false>, dim3((p.n + 3) / 4), dim3(256), 0, st, a, proj_out, e_out, regv);
    }
    if (reg_out) hipLaunchKernelGGL(enc_reg_reduce_kernel, dim3(1), dim3(1024), 0, st, regv, (p.n + 3) / 4, reg ? 1 : 0, reg_out);
    return kge_launch_status();
}

int kge_run_encode_bwd(const kge_encoder_t &e, const int32_t *h, const int32_t *t, int64_t B, const int32_t *neg, int64_t N,
                       uint64_t seed, uint64_t step, const float *proj, const float *de, float *g_es, float *g_mh, float *g_mt,
                       void *ws, hipStream_t st) {
    const EncPlan p = enc_plan(e, B, N);
    const bool bf16 = e.dtype == KGE_BF16;
    char *b = (char *)ws; size_t off = 0;
    auto take = [&](size_t bytes) { void *q = b + off; off += (bytes + 255) / 256 * 256; return q; };
    uint32_t *zeros = (uint32_t *)take(256);
    char *dP = (char *)take((size_t)e.dim * p.n * p.es);
    float *part = (float *)take(1);
    const int64_t mcount = (int64_t)e.dim * e.feat_dim;
    const EncRowArgs a = enc_row_args(e, h, t, B, neg, N, seed, step, (uintptr_t)proj, (uintptr_t)de, (uintptr_t)g_es);
    if (p.n > 0) {
        if (bf16) hipLaunchKernelGGL(enc_bwd_rows_kernel<true>, dim3((p.n + 3) / 4), dim3(256), 0, st, a, proj, de, g_es, dP, zeros);
        else      hipLaunchKernelGGL(enc_bwd_rows_kernel<false>, dim3((p.n + 3) / 4), dim3(256), 0, st, a, proj, de, g_es, dP, zeros);
    }
    EncTnPair pr{};
    pr.g[0] = EncTn{dP, h, nullptr, (int)B, (int)B, part};
    pr.g[1] = EncTn{dP + (size_t)B * e.dim * p.es, t, neg, (int)B, (int)(B + N), part + (size_t)p.nsplit_h * mcount};
    pr.feat = (const char *)e.feat; pr.ldf_b = e.feat_ld * p.es; pr.d = e.dim; pr.fd = e.feat_dim; pr.sps = p.sps; pr.zeros = zeros;
    pr.tiles_m = (e.dim + ENC_TILE - 1) / ENC_TILE; pr.tiles_n = (e.feat_dim + ENC_TILE - 1) / ENC_TILE;
    pr.wgs0 = pr.tiles_m * pr.tiles_n * p.nsplit_h; pr.total = pr.wgs0 + pr.tiles_m * pr.tiles_n * p.nsplit_t;
    if (pr.total > 0) {
        KgeProfScope prof(KGE_PROF_ENC_BWD, st);
        constexpr int TN_LDS = ENC_LDS_BYTES + ENC_MAX_SPS * 4;
        static KgeLdsLimit lim_bf16, lim_f32;                // the ring of stages is larger than the default dynamic limit
        if (lim_bf16.set((const void *)enc_gemm_tn_kernel<true>, TN_LDS) != KGE_OK || lim_f32.set((const void *)enc_gemm_tn_kernel<false>, TN_LDS) != KGE_OK)
            return KGE_E_HIP;
        const int grid = (pr.total + 7) / 8 * 8;
        if (bf16) hipLaunchKernelGGL(enc_gemm_tn_kernel<true>, dim3(grid), dim3(256), TN_LDS, st, pr);
        else      hipLaunchKernelGGL(enc_gemm_tn_kernel<false>, dim3(grid), dim3(256), TN_LDS, st, pr);
    }
    hipLaunchKernelGGL(enc_split_reduce_kernel, dim3((unsigned)((2 * mcount + 255) / 256)), dim3(256), 0, st, part, p.nsplit_h, p.nsplit_t, mcount, g_mh, g_mt);
    return kge_launch_status();
}
