// The shared-negative block kernel (gfx950, wave64, MFMA 32x32).
//
// The micro-batch's queries Q [B, d] (built from h and r) meet ONE block of negative tails
// T [N, d] shared by all of them (arXiv 2211.12281, Section 4 "Training", eq. (negsamples)), so the
// B x N scores of Table 2 are a dense contraction Q T^t followed by an elementwise map; the loss of
// Section 3.1 needs row reductions of that block, and its backward pass two more contractions
// (G T and G^t Q).  The block itself never goes to memory: it is recomputed tile by tile.
//
// One template serves all passes.  A workgroup (4 waves) OWNS 128 rows of one operand, held in
// registers as MFMA B-fragments for the whole launch, and STREAMS the other operand through an LDS
// ring of 2-4 stages in tiles of 32 rows.  The ring is filled by asynchronous global->LDS copies
// (no registers, several tiles in flight); rows are stored unpadded with their 16-byte chunks
// XOR-swizzled so that the fragment reads of 8 consecutive rows hit 8 different bank groups.
// Workgroups that read the same rows share a die and its L2 (kge_place_plan).  Per tile and wave:
//   phase 1   acc[32 stream x 32 own] = X_tile . own^t          (contraction over d)
//   epilogue  score / loss weights / gradient coefficients, element by element
//   phase 2   out^t[d x 32 own] += Xt_tile[d x 32 stream] . coef[stream x own]
//             (contraction over the stream index; the coefficients go from the accumulator
//             registers straight into the B-operand, the transposed tile Xt supplies the A-fragments)
// In both phases an own row lives in ONE lane pair (l, l+32), so every per-row quantity (running
// maximum, sums, rescaling factors) is a per-lane scalar.
//
//   MODE_SCORE  own = negatives, stream = queries : writes the scores S[b, n]
//   MODE_FWD    own = queries,   stream = negatives: one pass gives the loss statistics of each row
//               (running max / sum of the softmax weights, weighted loss terms) AND the
//               unnormalised gradient of the queries, rescaled online when the running max moves
//   MODE_GRADT  own = negatives, stream = queries : gradient of the negatives, needs the per-row
//               constants that MODE_FWD's statistics produce
//
// Accumulator layout of v_mfma_f32_32x32x*: lane l holds column (l & 31) and, in register i,
// row 8*(i/4) + 4*(l/32) + (i%4).
#pragma once
#include "kge_internal.h"
#include <type_traits>

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 kge_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float kge_f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float kge_f32x4;
typedef uint32_t kge_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t kge_u32x2 __attribute__((ext_vector_type(2)));

constexpr float KGE_LOG2E = 1.4426950408889634f;
constexpr float KGE_LN2 = 0.6931471805599453f;
constexpr float KGE_TAU = 8.f;     // log2 headroom of the softmax weights over their reference exponent

template <bool BF16> struct KgeElem;
template <> struct KgeElem<true>  { using type = __bf16; static constexpr int size = 2; };
template <> struct KgeElem<false> { using type = float;  static constexpr int size = 4; };

// acc += A(16 bytes per lane) . B(16 bytes per lane): one 32x32x16 bf16 MFMA, or four 32x32x2 fp32
template <bool BF16>
__device__ __forceinline__ kge_f32x16 kge_mma16(kge_f32x16 acc, uint4 a, uint4 b) {
    if constexpr (BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(kge_bf16x8, a),
                                                       __builtin_bit_cast(kge_bf16x8, b), acc, 0, 0, 0);
    } else {
        kge_f32x4 fa = __builtin_bit_cast(kge_f32x4, a), fb = __builtin_bit_cast(kge_f32x4, b);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[0], fb[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[1], fb[1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[2], fb[2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[3], fb[3], acc, 0, 0, 0);
        return acc;
    }
}

__device__ __forceinline__ uint32_t kge_pack_bf16x2(float lo, float hi) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf2;
    bf2 v = { (__bf16)lo, (__bf16)hi };          // round-to-nearest-even, lo in bits 0..15
    return __builtin_bit_cast(uint32_t, v);
}

// fp32 operands on the bf16 matrix pipe, for the small blocks (block_small.hip), whose operands come straight from fp32 rows and
// coefficients: the fp32 MFMA of gfx950 runs at 1/16 of the bf16 rate, so every operand value is split into THREE bf16 pieces,
// x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1) (round to nearest; 8 significand bits each,
// |x1| <= 2^-9 |x|, |x2| <= 2^-18 |x|; the bf16 exponent range is that of fp32, so nothing is scaled), and the six products of total
// order <= 2 are accumulated in fp32: a.b = a0 b0 + a0 b1 + a1 b0 + a1 b1 + a0 b2 + a2 b0 + O(2^-26 |a| |b|).
// Eight values of a lane (two 16-byte fragments: slot j of lane half g of both operands is one contraction index,
// whatever its number) become three bf16 fragments.
struct KgeP3 { uint4 p[3]; };
__device__ __forceinline__ KgeP3 kge_split3(uint4 a, uint4 b) {
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t q[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x0 = __uint_as_float(w[2 * i]), x1 = __uint_as_float(w[2 * i + 1]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            const uint32_t pk = kge_pack_bf16x2(x0, x1);
            q[pl][i] = pk;
            if (pl < 2) { x0 -= __uint_as_float(pk << 16); x1 -= __uint_as_float(pk & 0xffff0000u); }
        }
    }
    KgeP3 r;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) r.p[pl] = make_uint4(q[pl][0], q[pl][1], q[pl][2], q[pl][3]);
    return r;
}
// acc += A . B over the sixteen contraction indices of two fragment pairs (smallest terms first)
__device__ __forceinline__ kge_f32x16 kge_mma3(kge_f32x16 acc, const KgeP3 &A, const KgeP3 &B) {
    auto mm = [](kge_f32x16 c, uint4 x, uint4 y) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(kge_bf16x8, x), __builtin_bit_cast(kge_bf16x8, y), c, 0, 0, 0);
    };
    acc = mm(acc, A.p[0], B.p[2]);
    acc = mm(acc, A.p[2], B.p[0]);
    acc = mm(acc, A.p[1], B.p[1]);
    acc = mm(acc, A.p[0], B.p[1]);
    acc = mm(acc, A.p[1], B.p[0]);
    acc = mm(acc, A.p[0], B.p[0]);
    return acc;
}

// Two fp16 pieces of a value scaled by a power of two (KgePlaneScale: rows; coefficients below): x = x0 + x1 to 2^-24 of x or to
// 2^-25 over the scale, whichever is larger, three products per pair, a0 b0 + a0 b1 + a1 b0 (a1 b1 <= 2^-24 |a| |b| is left out).
struct KgeP2 { uint4 p[2]; };
typedef _Float16 kge_f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ KgeP2 kge_split2(const float (&x)[8]) {
    kge_f16x8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) { h[i] = (_Float16)x[i]; l[i] = (_Float16)(x[i] - (float)h[i]); }
    KgeP2 r;
    r.p[0] = __builtin_bit_cast(uint4, h); r.p[1] = __builtin_bit_cast(uint4, l);
    return r;
}
__device__ __forceinline__ kge_f32x16 kge_mma2(kge_f32x16 acc, const KgeP2 &A, const KgeP2 &B) {
    auto mm = [](kge_f32x16 c, uint4 x, uint4 y) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(kge_f16x8, x), __builtin_bit_cast(kge_f16x8, y), c, 0, 0, 0);
    };
    acc = mm(acc, A.p[0], B.p[1]);
    acc = mm(acc, A.p[1], B.p[0]);
    return mm(acc, A.p[0], B.p[0]);
}

// Asynchronous global -> LDS copies: lane l of a wave-wide instruction writes its 16 (4) bytes to LDS
// byte address m0 + 16 l (4 l).  Completion is tracked by vmcnt; the compiler does not see these
// loads, so the waits are explicit.
__device__ __forceinline__ void kge_async_copy16(const void *g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(g) : "memory");
}
__device__ __forceinline__ void kge_async_copy4(const void *g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(g) : "memory");
}
template <int N> __device__ __forceinline__ void kge_wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ float kge_elem_to_float(float x) { return x; }
__device__ __forceinline__ float kge_elem_to_float(__bf16 x) { return (float)x; }
__device__ __forceinline__ float kge_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float kge_log2(float x) { return __builtin_amdgcn_logf(x); }

// Squared distance of one (query, tail) pair by direct differences; the fallback for block entries
// whose norm-expansion form cancels.  TransH: u = q - t + (w.t) w.
template <bool BF16, bool TRANSH>
__device__ __forceinline__ float kge_direct_d2_inline(const void *qv, const void *tv, const void *wv, int dp) {
    using E = typename KgeElem<BF16>::type;
    const E *q = (const E *)qv, *t = (const E *)tv, *w = (const E *)wv;
    float A = 0.f;
    if constexpr (TRANSH)
#pragma unroll 1
        for (int j = 0; j < dp; ++j) A += kge_elem_to_float(w[j]) * kge_elem_to_float(t[j]);
    float acc = 0.f;
#pragma unroll 1
    for (int j = 0; j < dp; ++j) {
        float x = kge_elem_to_float(q[j]) - kge_elem_to_float(t[j]);
        if constexpr (TRANSH) x += A * kge_elem_to_float(w[j]);
        acc += x * x;
    }
    return acc;
}
template <bool BF16, bool TRANSH>
__device__ __noinline__ float kge_direct_d2(const void *qv, const void *tv, const void *wv, int dp) {
    return kge_direct_d2_inline<BF16, TRANSH>(qv, tv, wv, dp);
}

template <bool BF16, int RB, int MODE, bool TRANSH, int KIND, int DSPLIT>
struct KgeBlockCfg {
    static constexpr bool OWN_ROW = MODE == KGE_MODE_FWD;
    static constexpr int OW = kge_block_ow(BF16, RB, TRANSH, MODE, KIND);   // 32-row own fragments per wave
    static constexpr int OWN_TILE = 128 * OW;              // own rows of a workgroup
    static constexpr int ES = KgeElem<BF16>::size;
    static constexpr int DP = RB / ES;                     // padded dim
    static constexpr int KS = RB / 32;                     // 32-byte k-steps of phase 1
    static constexpr int ST = KGE_STREAM_TILE;
    static constexpr int NB = DP / 32;                     // 32-column output blocks of phase 2
    static constexpr int NBH = NB / DSPLIT;                // ... handled by one z-slice
    // PL: the operands come as two fp16 planes; a tile is two planes of [ST rows][2 DP bytes], chunk c of row r at c ^ kge_pl_swz(r), and the
    // transposed fragments of phase 2 are LDS transpose reads of it (ds_read_b64_tr_b16)
    static constexpr bool PL = kge_block_planes(BF16, RB, MODE);
    static constexpr int PLANE = ST * DP * 2;
    // groups of fragments requested together: what the registers hold without scratch
    static constexpr int PL_CHUNK = TRANSH ? 4 : OWN_ROW && KIND == KGE_KIND_DIST ? 1 : 2;
    static constexpr int X_BYTES = PL ? 2 * PLANE : ST * RB;    // else [ST rows][RB bytes], chunk c of row r at c ^ (r & 7)
    static constexpr int XT_ROWB = ST * ES;                // one transposed row: ST stream entries (bf16: 64 bytes)
    static constexpr int XT_BYTES = DP * XT_ROWB;
    static constexpr bool HAS_X2 = TRANSH && !OWN_ROW;     // second streamed operand (normals)
    static constexpr bool HAS_XT = MODE != KGE_MODE_SCORE && !PL;
    static constexpr int NX = HAS_X2 ? 2 : 1;
    static constexpr int STAGE_BYTES = X_BYTES * NX + (HAS_XT ? XT_BYTES * NX : 0);
    static constexpr int SIDE_SLOT = OWN_ROW ? 4 * 256 : 4 * 1024;   // per-wave copies of the tile's side info
    // Workgroups per compute unit (= waves per SIMD): two where a workgroup's registers fit in 256, so that
    // the MFMA, LDS and vector phases of one workgroup run under those of the other.
    static constexpr int OCC = kge_block_occ(BF16, RB, TRANSH, MODE);
    // TransH queries as planes: q and w^ together would take 128 registers, and the compiler then reloads fifty of them from scratch in
    // every tile, so the wave's 32 rows of w^ stay in the LDS, laid out like a tile
    static constexpr bool WL = PL && TRANSH && OWN_ROW;
    static constexpr int WL_BYTES = WL ? 4 * X_BYTES : 0;
    static constexpr int LDS_MAX = 160 * 1024 / OCC - WL_BYTES;
    static constexpr int NSTAGE_RAW = (LDS_MAX - SIDE_SLOT) / (STAGE_BYTES + SIDE_SLOT);   // n stages + (n+1) side slots fit
    static constexpr int NSTAGE = NSTAGE_RAW > 4 ? 4 : NSTAGE_RAW;
    static constexpr int SIDE_SLOTS = NSTAGE + 1;
    static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES + SIDE_SLOTS * SIDE_SLOT + WL_BYTES;
    static constexpr int X_IPW = X_BYTES / 1024 / 4;       // 1 KB wave-wide copies per wave and tile
    static constexpr int XT_IPW = XT_BYTES / 1024 / 4;
    static constexpr int LPW = X_IPW * NX + (HAS_XT ? XT_IPW * NX : 0) + 1;
    static_assert(NSTAGE >= 2, "two stages must fit");
    static_assert(X_BYTES % 4096 == 0 && XT_BYTES % 4096 == 0, "tile copies must divide over four waves");
    static_assert((NSTAGE - 2) * LPW < 64, "vmcnt range");
    static_assert(BF16 || PL || MODE == KGE_MODE_SCORE, "fp32 rows are trained on planes (TransH of more than 512 bytes: on the vector pipe)");
    static_assert(OW == 1 || !TRANSH, "two own fragments per wave leave no registers for the TransH operands");
    static_assert(KS % 8 == 0, "phase 1 works in groups of four fragments, split in two halves");
};

// Position of the 16-byte chunks of a plane row of 256 or 512 bytes: sixteen consecutive rows at one chunk index (phase 1) fall into sixteen
// different bank groups, and so do four consecutive rows at four neighbouring chunks (the transpose reads of phase 2).
__device__ __forceinline__ constexpr int kge_pl_swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
typedef short kge_i16x4 __attribute__((ext_vector_type(4)));

template <bool BF16, int RB, int MODE, bool TRANSH, int KIND, int LOSS, int DSPLIT>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256),
                          amdgpu_waves_per_eu(kge_block_occ(BF16, RB, TRANSH, MODE), kge_block_occ(BF16, RB, TRANSH, MODE))))
void kge_block_kernel(const KgeBlockArgs a) {
    using C = KgeBlockCfg<BF16, RB, MODE, TRANSH, KIND, DSPLIT>;
    constexpr bool OWN_ROW = C::OWN_ROW;
    constexpr bool PHASE2 = MODE != KGE_MODE_SCORE;
    constexpr int OW = C::OW;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    char *side_ring = lds + C::NSTAGE * C::STAGE_BYTES;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, g = lane >> 5;
    int own_tile, split;
    if (!kge_place(a.own_tiles, a.nsplit, a.xcd_per, own_tile, split)) return;
    const int own_base = own_tile * C::OWN_TILE;
    const int dblk0 = blockIdx.y * C::NBH;
    const int oidx0 = own_base + wave * 32 * OW + lr;     // own row of fragment h: oidx0 + 32 h
    const int t0 = split * a.tiles_per_split;
    const int t1 = min(a.str_tiles, t0 + a.tiles_per_split);
    const int str_limit = OWN_ROW ? a.N : a.B;            // valid stream rows

    // ---- own operand fragments: 16 bytes per lane per 32-byte k-step --------------------------
    constexpr bool PL = C::PL;
    // One wave per SIMD on planes: the own operand and the gradient accumulators stay in the accumulator registers (matrix
    // instructions read them there), which leaves the vector registers for fragments requested ahead of their use.
    constexpr bool ALONE = PL && C::OCC == 1;
    const int64_t own_plane = (int64_t)a.own_pad * C::DP * 2, str_plane = (int64_t)a.str_tiles * C::ST * C::DP * 2;   // PL: bytes per plane
    uint4 own[OW][PL ? 1 : C::KS];
    uint4 ownw[(TRANSH && OWN_ROW && !PL) ? C::KS : 1];
    // the own operand as fp16 pieces, sixteen contraction indices per entry
    constexpr bool WL = C::WL;
    static_assert(!PL || (OW == 1 && DSPLIT == 1), "");
    KgeP2 own2p[PL ? C::KS / 2 : 1];
    int o_exp = 0;                                        // PL: exponent of 1 / scale of the own row
    float o_qn[OW], o_c[OW], o_wn[OW], o_tn[OW];          // own-side scalars
#pragma unroll
    for (int h = 0; h < OW; ++h) {
        const int oidx = oidx0 + 32 * h;
        if constexpr (PL) {
            const char *p = (const char *)a.own + (size_t)oidx * (C::DP * 2) + g * 16;
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                for (int k2 = 0; k2 < C::KS / 2; ++k2) own2p[k2].p[pl] = *(const uint4 *)(p + pl * own_plane + k2 * 32);
            o_exp = a.own_exp[oidx];
        } else {
            const char *p = (const char *)a.own + (size_t)oidx * RB + g * 16;
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) own[h][ks] = *(const uint4 *)(p + ks * 32);
            if constexpr (TRANSH && OWN_ROW) {
                const char *pw = (const char *)a.own2 + (size_t)oidx * RB + g * 16;
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) ownw[ks] = *(const uint4 *)(pw + ks * 32);
            }
        }
        o_qn[h] = 0.f; o_c[h] = 0.f; o_wn[h] = 1.f; o_tn[h] = 0.f;
        if constexpr (OWN_ROW) {
            KgeRowInfo ri = a.rowinfo[oidx];
            o_qn[h] = ri.qn; o_c[h] = ri.c; o_wn[h] = ri.wn;
        } else {
            o_tn[h] = a.tn[oidx];
        }
    }

    // ---- accumulators of the launch ------------------------------------------------------------
    kge_f32x16 acc2[OW][PHASE2 ? C::NBH : 1];
    kge_f32x16 acc2b[(PHASE2 && TRANSH && OWN_ROW) ? C::NBH : 1];
    if constexpr (PHASE2) {
#pragma unroll
        for (int b = 0; b < C::NBH; ++b) {
#pragma unroll
            for (int h = 0; h < OW; ++h)
                for (int i = 0; i < 16; ++i) acc2[h][b][i] = 0.f;
            if constexpr (TRANSH && OWN_ROW) for (int i = 0; i < 16; ++i) acc2b[b][i] = 0.f;
        }
    }
    float sum1[OW], sum2[OW], sum3[OW];                   // sums of the coefficients over the stream index
    float st_m[OW], st_l[OW], st_acc[OW];                 // FWD: running max (log2 domain) / sum / weighted loss
#pragma unroll
    for (int h = 0; h < OW; ++h) { sum1[h] = sum2[h] = sum3[h] = 0.f; st_m[h] = -INFINITY; st_l[h] = st_acc[h] = 0.f; }

    // ---- asynchronous staging of one stream tile --------------------------------------------------
    // X tile: instruction jj of this wave covers LDS bytes [(wave*X_IPW + jj) KB, +1 KB) of the tile; the
    // lane's 16 bytes are position (byte % RB)/16 of row byte/RB and must hold source chunk pos ^ (row & 7).
    // (PL: copy c = wave X_IPW + jj fills the RPC rows from RPC (c % CPP) on of plane c / CPP; the lane's offset differs in the swizzle only)
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    constexpr int RPC = PL ? 1024 / (C::DP * 2) : 1, CPP = PL ? C::PLANE / 1024 : 1;
    static_assert(!PL || RPC == 4 || RPC == 2, "");
    const int pl_row = RPC == 4 ? lane >> 4 : lane >> 5;
    const int pl_off = pl_row * (C::DP * 2) + (((lane & (64 / RPC - 1)) ^ (pl_row << 2)) * 16);
    auto pl_swz = [](int c) { return (RPC == 4 ? c & 3 : (c & 1) << 3 | ((c >> 1) & 3)) << 4; };       // rest of kge_pl_swz of the copy's rows
    int x_off[PL ? 1 : C::X_IPW];                          // source byte offset inside the tile
#pragma unroll
    for (int jj = 0; jj < (PL ? 0 : C::X_IPW); ++jj) {
        const int byte = (wave * C::X_IPW + jj) * 1024 + lane * 16;
        const int r = byte / RB, pos = (byte % RB) / 16;
        x_off[jj] = r * RB + ((pos ^ (r & 7)) * 16);
    }
    // Xt tile: rows of 64 bytes (dcol-major), two rows per 128-byte line, chunk slot ((row&1)*4 + c) ^ ((row>>1)&7) within the line.
    int64_t xt_off[C::HAS_XT ? C::XT_IPW : 1];             // source byte offset relative to the tile's first column
    if constexpr (C::HAS_XT) {
#pragma unroll
        for (int jj = 0; jj < C::XT_IPW; ++jj) {
            const int byte = (wave * C::XT_IPW + jj) * 1024 + lane * 16;
            const int line = byte >> 7, slot = (byte >> 4) & 7;
            const int sslot = slot ^ (line & 7), row = 2 * line + (sslot >> 2), c = sslot & 3;
            xt_off[jj] = (int64_t)row * a.strT_ld * C::ES + c * 16;
        }
    }
    const char *own_w = lds + C::NSTAGE * C::STAGE_BYTES + C::SIDE_SLOTS * C::SIDE_SLOT + wave * (WL ? C::X_BYTES : 0);
    if constexpr (WL) {                                    // (the wave's own copies: the wait for its first tile covers them)
        const uint32_t wl0 = lds0 + C::NSTAGE * C::STAGE_BYTES + C::SIDE_SLOTS * C::SIDE_SLOT + wave_u * C::X_BYTES;
        const int64_t woff = (int64_t)(own_base + wave_u * 32) * (C::DP * 2);
#pragma unroll
        for (int c = 0; c < C::X_BYTES / 1024; ++c) {
            const char *src = (const char *)a.own2 + (c / CPP) * own_plane + woff + (c % CPP) * 1024;
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(wl0 + c * 1024)),
                         "v"(pl_off ^ pl_swz(c)), "s"(src) : "memory");
        }
    }
    auto issue = [&](int tile, int slot) {
        tile = tile < t1 ? tile : t1 - 1;                  // past the end: a harmless repeat keeps vmcnt uniform
        const uint32_t sbase = lds0 + (slot % C::NSTAGE) * C::STAGE_BYTES;
        if constexpr (PL) {
            const int64_t toff = (int64_t)__builtin_amdgcn_readfirstlane(tile) * (C::ST * C::DP * 2);
#pragma unroll
            for (int op = 0; op < C::NX; ++op)
#pragma unroll
                for (int jj = 0; jj < C::X_IPW; ++jj) {
                    const int c = wave_u * C::X_IPW + jj;
                    const char *src = (const char *)(op ? a.str2 : a.str) + (c / CPP) * str_plane + toff + (c % CPP) * 1024;
                    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(sbase + op * C::X_BYTES + c * 1024)),
                                 "v"(pl_off ^ pl_swz(c)), "s"(src) : "memory");
                }
        } else {
            const char *src = (const char *)a.str + (size_t)tile * C::ST * RB;
#pragma unroll
            for (int jj = 0; jj < C::X_IPW; ++jj)
                kge_async_copy16(src + x_off[jj], __builtin_amdgcn_readfirstlane(sbase + (wave * C::X_IPW + jj) * 1024));
            if constexpr (C::HAS_X2) {
                const char *src2 = (const char *)a.str2 + (size_t)tile * C::ST * RB;
#pragma unroll
                for (int jj = 0; jj < C::X_IPW; ++jj)
                    kge_async_copy16(src2 + x_off[jj], __builtin_amdgcn_readfirstlane(sbase + C::X_BYTES + (wave * C::X_IPW + jj) * 1024));
            }
        }
        if constexpr (C::HAS_XT) {
            const char *srct = (const char *)a.strT + (size_t)tile * C::ST * C::ES;
#pragma unroll
            for (int jj = 0; jj < C::XT_IPW; ++jj)
                kge_async_copy16(srct + xt_off[jj], __builtin_amdgcn_readfirstlane(sbase + C::X_BYTES * C::NX + (wave * C::XT_IPW + jj) * 1024));
            if constexpr (C::HAS_X2) {
                const char *srct2 = (const char *)a.strT2 + (size_t)tile * C::ST * C::ES;
#pragma unroll
                for (int jj = 0; jj < C::XT_IPW; ++jj)
                    kge_async_copy16(srct2 + xt_off[jj], __builtin_amdgcn_readfirstlane(sbase + C::X_BYTES * C::NX + C::XT_BYTES + (wave * C::XT_IPW + jj) * 1024));
            }
        }
        // side info of the tile's 32 stream rows, one private copy per wave
        const uint32_t sside = lds0 + C::NSTAGE * C::STAGE_BYTES + (slot % C::SIDE_SLOTS) * C::SIDE_SLOT;
        // (PL: the second half of the copy are the rows' exponents)
        if constexpr (OWN_ROW)
            kge_async_copy4(PL && g ? (const void *)(a.str_exp + tile * C::ST + lr) : (const void *)(a.tn + tile * C::ST + lr), __builtin_amdgcn_readfirstlane(sside + wave * 256));
        else
            kge_async_copy16(PL && g ? (const void *)(a.str_exp + tile * C::ST + 4 * (lr & 7)) : (const void *)(a.rowinfo + tile * C::ST + lr),
                             __builtin_amdgcn_readfirstlane(sside + wave * 1024));
    };
    // fragment addresses inside a stage: chunk (2 ks + g) of row lr sits at position chunk ^ (lr & 7)
    int frag_off[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) frag_off[b] = lr * RB + 16 * (((2 * b) ^ (lr & 6)) | (g ^ (lr & 1)));
    // PL: chunk (2 k2 + g) of row lr of a plane; and the transpose reads: source lane i of a group of sixteen points at row
    // 16 j2 + 8 hh + 4 g + i / 4, columns 32 blk + 16 q16 + 4 (i % 4) .. + 3, and lane l receives column 32 blk + l % 32 of the rows
    // 16 j2 + 8 hh + 4 g .. + 3 - the streamed rows of its coefficients 8 j2 + 4 hh .. + 3
    // (rows of 512 bytes in a plane: the swizzle leaves the upper bit of the chunk alone, so the second half of the row is 256 bytes on)
    int pl_frag[8], pl_tr[2][4];
    if constexpr (PL) {
        const int i16 = lane & 15, q16 = (lane >> 4) & 1;
#pragma unroll
        for (int k2 = 0; k2 < 8; ++k2) pl_frag[k2] = lr * (C::DP * 2) + ((2 * k2 + g) ^ kge_pl_swz(lr)) * 16;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int row = 8 * hh + 4 * g + (i16 >> 2);
                pl_tr[hh][b] = row * (C::DP * 2) + ((4 * b + 2 * q16 + ((i16 & 3) >> 1)) ^ kge_pl_swz(row)) * 16 + (i16 & 1) * 8;
            }
    }

    constexpr int FILL = C::NSTAGE - (ALONE ? 2 : 1);      // tiles requested ahead of the loop
#pragma unroll
    for (int s2 = 0; s2 < FILL; ++s2) issue(t0 + s2, s2);
    // Pin the own operand as loaded before the loop.  Otherwise the compiler defers its waits for these
    // ordinary loads to their first uses inside the hot loop, and such a wait (which counts every memory
    // operation in flight) would also drain the asynchronous copies of the coming tiles on every iteration.
#pragma unroll
    for (int h = 0; h < OW; ++h) {
        if constexpr (PL) {
#pragma unroll
            for (int k2 = 0; k2 < C::KS / 2; ++k2)
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) {
                    uint4 &v = own2p[k2].p[pl];
                    if constexpr (ALONE) asm volatile("" : "+a"(v.x), "+a"(v.y), "+a"(v.z), "+a"(v.w));
                    else asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
                }
            asm volatile("" : "+v"(o_exp));
        } else {
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) {
                asm volatile("" : "+v"(own[h][ks].x), "+v"(own[h][ks].y), "+v"(own[h][ks].z), "+v"(own[h][ks].w));
                if constexpr (TRANSH && OWN_ROW)
                    asm volatile("" : "+v"(ownw[ks].x), "+v"(ownw[ks].y), "+v"(ownw[ks].z), "+v"(ownw[ks].w));
            }
        }
        asm volatile("" : "+v"(o_qn[h]), "+v"(o_c[h]), "+v"(o_wn[h]), "+v"(o_tn[h]));
    }

    // ---- state of the tile in work (set by the loops below, used by the pieces) -------------------
    int tile = t0;
    const char *base = lds, *side = side_ring;
    int sbase = 0;                                        // stream index of register i: sbase + 8*(i/4) + (i%4)
    bool tile_full = true;
    const float xscale = (LOSS == KGE_LOGSIGMOID ? a.adv_temp : 1.f) * KGE_LOG2E;
    auto set_tile = [&](int t) {
        tile = t;
        const int slot = t - t0;
        base = lds + (slot % C::NSTAGE) * C::STAGE_BYTES;
        side = side_ring + (slot % C::SIDE_SLOTS) * C::SIDE_SLOT + wave * (OWN_ROW ? 256 : 1024);
        sbase = t * C::ST + 4 * g;
        tile_full = t * C::ST + C::ST <= str_limit;
    };
    kge_f32x16 acc[OW], accw;                              // phase-1 accumulators: [stream, own]
    uint4 bf[OW][2], bf2[2];                               // bf16 B-operands of phase 2
    KgeP2 coef2p[2], coefw2p[2];                           // PL: the fp16 pieces of coefficients times c_scale
    float coef_a[16], coef2_a[16];                         // ALONE: coefficients of phase 2 (coef2: TransH's normals)
    // PL: what the own row's coefficients, and with them its accumulated gradient, are multiplied by (a power of two until its reference is
    // raised); 0: none yet, what has accumulated counts for nothing
    float c_scale = 0.f;

    // ---- phase 1: acc[h][stream, own] = X_tile . own^t; a fragment read from the LDS feeds all own fragments
    constexpr bool HASW = TRANSH && !OWN_ROW;
    constexpr int G1 = HASW ? 2 : 4, NG1 = C::KS / G1;      // fragments per group, groups
    uint4 av[PL ? 1 : C::KS], aw[HASW && !PL ? C::KS : 1];
    KgeP2 xp[PL ? C::KS / 2 : 1], xwp[HASW && PL ? C::KS / 2 : 1], owp[WL ? C::KS / 2 : 1];
    auto ld1 = [&](const char *stage, int grp) {
        if constexpr (PL) {
#pragma unroll
            for (int k = 0; k < G1 / 2; ++k) {
                const int k2 = grp * (G1 / 2) + k;
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) {
                    xp[k2].p[pl] = *(const uint4 *)(stage + pl_frag[k2 & 7] + (k2 >> 3) * 256 + pl * C::PLANE);
                    if constexpr (WL) owp[k2].p[pl] = *(const uint4 *)(own_w + pl_frag[k2 & 7] + (k2 >> 3) * 256 + pl * C::PLANE);
                    if constexpr (HASW) xwp[k2].p[pl] = *(const uint4 *)(stage + C::X_BYTES + pl_frag[k2 & 7] + (k2 >> 3) * 256 + pl * C::PLANE);
                }
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < (PL ? 0 : G1); ++k) {
            const int ks = grp * G1 + k;
            av[ks] = *(const uint4 *)(stage + frag_off[ks & 3] + 128 * (ks >> 2));
            if constexpr (HASW) aw[ks] = *(const uint4 *)(stage + C::X_BYTES + frag_off[ks & 3] + 128 * (ks >> 2));
        }
    };
    auto zero1 = [&]() {
#pragma unroll
        for (int h = 0; h < OW; ++h) for (int i = 0; i < 16; ++i) acc[h][i] = 0.f;
        for (int i = 0; i < 16; ++i) accw[i] = 0.f;
    };
    auto mma1 = [&](int grp) {
#pragma unroll
        for (int k = 0; k < G1; ++k) {
            const int ks = grp * G1 + k;
            if constexpr (PL) {
                if ((k & 1) == 0) {
                    acc[0] = kge_mma2(acc[0], xp[ks >> 1], own2p[ks >> 1]);
                    if constexpr (WL) accw = kge_mma2(accw, xp[ks >> 1], owp[ks >> 1]);
                    if constexpr (HASW) accw = kge_mma2(accw, xwp[ks >> 1], own2p[ks >> 1]);
                }
            } else {
#pragma unroll
                for (int h = 0; h < OW; ++h) acc[h] = kge_mma16<BF16>(acc[h], av[ks], own[h][ks]);
                if constexpr (TRANSH && OWN_ROW) accw = kge_mma16<BF16>(accw, av[ks], ownw[ks]);
                if constexpr (HASW) accw = kge_mma16<BF16>(accw, aw[ks], own[0][ks]);
            }
        }
    };
    // ---- phase 2: out^t[d, own] += Xt_tile[d, stream] . coef[stream, own] ---------------------------
    constexpr int G2 = BF16 ? (HASW ? 1 : 2) : 1;          // blocks per group
    constexpr int NG2 = PHASE2 ? C::NBH / G2 : 0;
    uint4 av2[PHASE2 && !PL ? C::NBH : 1][2], aw2[(PHASE2 && HASW && !PL) ? C::NBH : 1][2];   // (bf16: two 16-byte fragments per block)
    KgeP2 tp[PL ? C::NBH : 1][2], twp[PL && HASW ? C::NBH : 1][2];
    auto ld2 = [&](const char *stage, int grp) {
        if constexpr (PL) {
            auto frag = [&](const char *s, int blk, int j2, KgeP2 &x) {
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) {
                    const char *q = s + pl * C::PLANE + j2 * (16 * C::DP * 2) + (blk >> 2) * 256;
                    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((kge_i16x4 __attribute__((address_space(3))) *)(q + pl_tr[0][blk & 3])));
                    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((kge_i16x4 __attribute__((address_space(3))) *)(q + pl_tr[1][blk & 3])));
                    x.p[pl] = make_uint4(lo.x, lo.y, hi.x, hi.y);
                }
            };
#pragma unroll
            for (int bb = 0; bb < G2; ++bb)
#pragma unroll
                for (int j2 = 0; j2 < 2; ++j2) {
                    frag(stage, grp * G2 + bb, j2, tp[grp * G2 + bb][j2]);
                    if constexpr (HASW) frag(stage + C::X_BYTES, grp * G2 + bb, j2, twp[grp * G2 + bb][j2]);
                }
            return;
        }
        const char *xt = stage + C::X_BYTES * C::NX;
#pragma unroll
        for (int bb = 0; bb < (PL ? 0 : G2); ++bb) {
            const int blk = grp * G2 + bb;
            const int row = (dblk0 + blk) * 32 + lr;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                // The transposed operand keeps, inside every group of 16 stream entries, the 8 entries of
                // one lane half contiguous (the producer swaps bits 2 and 3 of the column), so the
                // A-fragment of (block, f) is ONE 16-byte chunk: chunk 2 f + g of row dcol, at its slot.
                const int sslot = (((row & 1) << 2) | (2 * f + g)) ^ ((row >> 1) & 7);
                const char *p = xt + (row >> 1) * 128 + sslot * 16;
                av2[blk][f] = *(const uint4 *)p;
                if constexpr (HASW) aw2[blk][f] = *(const uint4 *)(p + C::XT_BYTES);
            }
        }
    };
    auto mma2 = [&](int grp) {
#pragma unroll
        for (int bb = 0; bb < G2; ++bb) {
            const int blk = grp * G2 + bb;
            if constexpr (BF16) {
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
                    for (int h = 0; h < OW; ++h) acc2[h][blk] = kge_mma16<true>(acc2[h][blk], av2[blk][s2], bf[h][s2]);
                    if constexpr (TRANSH && OWN_ROW) acc2b[blk] = kge_mma16<true>(acc2b[blk], av2[blk][s2], bf2[s2]);
                    if constexpr (HASW) acc2[0][blk] = kge_mma16<true>(acc2[0][blk], aw2[blk][s2], bf2[s2]);
                }
            } else {
#pragma unroll
                for (int j2 = 0; j2 < 2; ++j2) {
                    acc2[0][blk] = kge_mma2(acc2[0][blk], tp[blk][j2], coef2p[j2]);
                    if constexpr (TRANSH && OWN_ROW) acc2b[blk] = kge_mma2(acc2b[blk], tp[blk][j2], coefw2p[j2]);
                    if constexpr (HASW) acc2[0][blk] = kge_mma2(acc2[0][blk], twp[blk][j2], coefw2p[j2]);
                }
            }
        }
    };
    // orders a region of the scheduler: a matrix instruction, then a share of its vector instructions
#define KGE_MIX(n, valu)                                                        \
    _Pragma("unroll") for (int mix_i = 0; mix_i < (n); ++mix_i) {               \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                      \
        __builtin_amdgcn_sched_group_barrier(0x002, (valu), 0);                 \
    }
    // ---- epilogue: scores / loss weights / gradient coefficients of the tile, element by element ----
    auto str_exp_of = [&](int sl) { return *(const int *)(side + (OWN_ROW ? 128 : 512) + sl * 4); };       // PL: exponent of 1 / scale of a streamed row
    // the first part of the scores of own fragment h against the tile: products (bilinear scorers) or squared distances by the norm
    // expansion |q|^2 + |t|^2 - 2 q.t (TransH: plus the terms of the projection), w.t, and whether any of the lane's entries cancels
    auto norms_of = [&](int h, int i, float &qn, float &cc, float &wn, float &tnv) {
        const int sl = 8 * (i >> 2) + 4 * g + (i & 3);
        if constexpr (OWN_ROW) { qn = o_qn[h]; cc = o_c[h]; wn = o_wn[h]; tnv = *(const float *)(side + sl * 4); }
        else { float4 ri = *(const float4 *)(side + sl * 16); qn = ri.x; cc = ri.y; wn = ri.w; tnv = o_tn[h]; }
    };
    // (the streamed rows of the entries 4 j .. 4 j + 3 are neighbours: one read each of their norms and exponents, four of their row info)
    struct Side4 { kge_f32x4 tn, ri[OWN_ROW ? 1 : 4]; kge_u32x4 e; };
    auto side4 = [&](int j, Side4 &x) {
        x.e = *(const kge_u32x4 *)(side + (OWN_ROW ? 128 : 512) + (8 * j + 4 * g) * 4);
        if constexpr (KIND == KGE_KIND_DIST) {
            if constexpr (OWN_ROW) x.tn = *(const kge_f32x4 *)(side + (8 * j + 4 * g) * 4);
            else {
#pragma unroll
                for (int u = 0; u < 4; ++u) x.ri[u] = *(const kge_f32x4 *)(side + (8 * j + 4 * g + u) * 16);
            }
        }
    };
    // squared distance of an entry by direct differences, from the unscaled rows
    auto again = [&](int h, int i) {
        const int oidx = oidx0 + 32 * h, sidx = tile * C::ST + 8 * (i >> 2) + 4 * g + (i & 3);
        const int b = OWN_ROW ? oidx : sidx, n = OWN_ROW ? sidx : oidx;
        const char *own = (const char *)(PL ? a.own32 : a.own), *str = (const char *)(PL ? a.str32 : a.str);
        const char *qb = (OWN_ROW ? own : str) + (size_t)b * RB, *tb = (OWN_ROW ? str : own) + (size_t)n * RB;
        const char *wb = !TRANSH ? nullptr : PL ? (const char *)a.w32 + (size_t)b * RB : (const char *)(OWN_ROW ? a.own2 : a.str2) + (size_t)b * RB;
        if constexpr (BF16) return kge_direct_d2<BF16, TRANSH>(qb, tb, wb, C::DP);
        else return kge_direct_d2_inline<BF16, TRANSH>(qb, tb, wb, C::DP);
    };
    // fp32: the entries below their line by a loop over them, in line - a call costs its caller-saved registers all through the kernel, where
    // the pieces leave none (bf16 tables have them, and lose 0.5-1.5 % by this form)
    auto again_of = [&](int h, float (&d2)[16], auto &&line) {
        uint32_t todo = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) todo |= d2[i] < line(i) ? 1u << i : 0u;
        while (todo) {
            const int i = __builtin_ctz(todo);
            todo &= todo - 1;
            const float v = again(h, i);
#pragma unroll
            for (int k = 0; k < 16; ++k) d2[k] = k == i ? v : d2[k];
        }
    };
    auto from_squares = [&](const float (&d2)[16], float (&sv)[16], float (&dv)[16]) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float dd = fmaxf(d2[i], 0.f);
            const float inv = dd > 0.f ? __builtin_amdgcn_rsqf(dd) : 0.f;
            dv[i] = inv;
            sv[i] = -dd * inv;                              // -sqrt(d2)
        }
    };
    // scores of own fragment h against the tile (SCORE mode stores them), 1/distance, w.t, in one piece: kernels of several waves per SIMD
    // (in the parts below, with the line of the cancellation recomputed, bf16 TransH takes 593 us a step of 8,192 x 4,096 for 527)
    auto scores = [&](int h, float (&sv)[16], float (&dv)[16], float (&Av)[16]) {
#pragma unroll
        for (int i = 0; i < 16; ++i) { dv[i] = 0.f; Av[i] = 0.f; }
        if constexpr (PL) {                                // (exact: powers of two)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int s_exp = str_exp_of(8 * (i >> 2) + 4 * g + (i & 3));
                acc[0][i] = ldexpf(acc[0][i], o_exp + s_exp);
                if constexpr (TRANSH) accw[i] = ldexpf(accw[i], (OWN_ROW ? s_exp : o_exp) + KGE_PLANE_UNIT_EXP);
            }
        }
        if constexpr (KIND == KGE_KIND_MULT) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sv[i] = acc[h][i];
        } else {
            // (squared distances and their cancellation: scores2)
            float d2[16], thr[16];
            bool cancel = false;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float qn, cc, wn, tnv;
                norms_of(h, i, qn, cc, wn, tnv);
                d2[i] = fmaf(-2.f, acc[h][i], qn + tnv);
                if constexpr (TRANSH) { const float A = accw[i]; Av[i] = A; d2[i] += A * (2.f * cc - A * (2.f - wn)); }
                thr[i] = 1e-3f * (qn + tnv);
                cancel = cancel || d2[i] < thr[i];
            }
            if (__any(cancel)) {
                if constexpr (BF16) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        if (d2[i] < thr[i]) d2[i] = again(h, i);
                        asm volatile("" ::: "memory");      // keeps the branch from being turned into selects
                    }
                } else again_of(h, d2, [&](int i) { return thr[i]; });
            }
            from_squares(d2, sv, dv);
        }
        if constexpr (MODE == KGE_MODE_SCORE) {
            const int oidx = oidx0 + 32 * h;
            if (oidx < a.N) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int b = sbase + 8 * (i >> 2) + (i & 3);
                    if (b < a.B) a.S_out[(size_t)b * a.N + oidx] = sv[i];
                }
            }
        }
    };
    int s_exps[16];                                        // ALONE: exponents of the streamed rows of the lane's entries
    auto scores4 = [&](int h, int j, const Side4 &x, float (&d2)[16], float (&Av)[16], bool &cancel) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = 4 * j + u;
            s_exps[i] = (int)x.e[u];
            acc[0][i] = ldexpf(acc[0][i], o_exp + s_exps[i]);           // (exact: powers of two)
            if constexpr (TRANSH) accw[i] = ldexpf(accw[i], (OWN_ROW ? s_exps[i] : o_exp) + KGE_PLANE_UNIT_EXP);
            Av[i] = 0.f;
            if constexpr (KIND == KGE_KIND_MULT) d2[i] = acc[h][i];
            else {
                const float qn = OWN_ROW ? o_qn[h] : x.ri[OWN_ROW ? 0 : u][0], cc = OWN_ROW ? o_c[h] : x.ri[OWN_ROW ? 0 : u][1];
                const float wn = OWN_ROW ? o_wn[h] : x.ri[OWN_ROW ? 0 : u][3], tnv = OWN_ROW ? x.tn[u] : o_tn[h];
                d2[i] = fmaf(-2.f, acc[h][i], qn + tnv);
                if constexpr (TRANSH) { const float A = accw[i]; Av[i] = A; d2[i] += A * (2.f * cc - A * (2.f - wn)); }
                cancel = cancel || d2[i] < 1e-3f * (qn + tnv);
            }
        }
    };
    auto scores1 = [&](int h, float (&d2)[16], float (&Av)[16], bool &cancel) {
        cancel = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) { Side4 x; side4(j, x); scores4(h, j, x, d2, Av, cancel); }
    };
    // ALONE: the scores themselves and 1/distance.  Distances whose expansion cancels (below 1e-3 of the norms) are
    // redone by direct differences in a rarely taken branch.  (The line with planes: above it their errors are 0.6 to 0.9 times those of
    // 24-bit operands with norms summed in 32 bits, negatives at 0.05 and 0.1 of its length from a query; four products are no
    // better.  A line of 4e-3 gives a tenth of the error at 0.05, but tables with a common part ten to thirty times their spread take 15 to
    // 100 times as long: TransE 8,192 x 4,096 x 128 at 0.05 7.0 ms instead of 0.2)
    auto scores2 = [&](int h, float (&d2)[16], bool cancel, float (&sv)[16], float (&dv)[16]) {
#pragma unroll
        for (int i = 0; i < 16; ++i) dv[i] = 0.f;
        if constexpr (KIND == KGE_KIND_MULT) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sv[i] = d2[i];
        } else {
            auto line = [&](int i) {
                float qn, cc, wn, tnv;
                norms_of(h, i, qn, cc, wn, tnv);
                return 1e-3f * (qn + tnv);
            };
            if (__any(cancel)) again_of(h, d2, line);
            from_squares(d2, sv, dv);
        }
    };
    // FWD: exponents of the softmax weights of own fragment h relative to its reference st_m (log2
    // domain; entries past the end of the stream operand get -inf: only the last tile has any, the
    // branch is wave-uniform), and their maximum over the tile.  Lanes l and l^32 hold the two halves
    // of the same own row and feed ONE contraction in phase 2, so they share the maximum.
    auto exponents = [&](int h, const float (&sv)[16], float (&x2)[16]) -> float {
        const float m_neg = st_m[h] > -INFINITY ? -st_m[h] : 0.f;
        float tm = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) x2[i] = fmaf(sv[i], xscale, m_neg);
        if (!tile_full) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (sbase + 8 * (i >> 2) + (i & 3) >= str_limit) x2[i] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) tm = fmaxf(tm, x2[i]);
        return fmaxf(tm, __shfl_xor(tm, 32));
    };
    // what an own row has accumulated times r.  (ALONE: in place.  As ordinary products the accumulators are vector registers here, and
    // the compiler carries them to and from the accumulator registers in every tile: 250 of 1,280 vector instructions.  It counts no
    // wait states for what inline asm reads and writes: settle() stands before the first call and behind the last.)
    // 20 wait states are due between a matrix instruction of sixteen passes and a read of what it wrote, two between a write and a
    // matrix instruction that reads it; the branch that rescales holds no matrix instruction.  (The last ones are most of an epilogue ago.)
    auto settle = [] {
        if constexpr (ALONE) { asm volatile("s_nop 15\n\ts_nop 7" ::: "memory"); __builtin_amdgcn_sched_barrier(0); }
    };
    auto rescale = [&](kge_f32x16 &x, float r) {
        if constexpr (ALONE) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float v = x[i], tmp;
                asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1" : "+a"(v), "=&v"(tmp) : "v"(r));
                x[i] = v;
            }
        } else {
            for (int i = 0; i < 16; ++i) x[i] *= r;
            asm volatile("" ::: "memory");
        }
    };
    // PL: the coefficients of phase 2 as its B-operand
    constexpr int NPC = TRANSH ? 4 : 2;
    auto make_piece = [&](int p) {
        const int j2 = TRANSH ? p >> 1 : p;
        const float *c = (TRANSH && (p & 1) ? coef2_a : coef_a) + 8 * j2;
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = c[i] * c_scale;
        if (TRANSH && (p & 1)) coefw2p[j2] = kge_split2(x); else coef2p[j2] = kge_split2(x);
    };
    float row_K[16], row_c[16];                            // ALONE, GRADT: constants of the streamed rows, requested ahead of their use
    // the coefficients of phase 2 for own fragment h, packed as its B-operand
    auto weights = [&](int h, const float (&sv)[16], const float (&dv)[16], const float (&Av)[16], const float (&x2)[16]) {
        float coef[16], coef2[16];
        if constexpr (MODE == KGE_MODE_FWD) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float e = kge_exp2(x2[i]);                             // masked entries: exp2(-inf) = 0
                st_l[h] += e;
                float u = e;
                if constexpr (LOSS == KGE_LOGSIGMOID) {
                    // weight * sigma(gamma + s) for the gradient, weight * softplus(gamma + s) for the loss
                    const float y = a.gamma + sv[i];
                    const float t = kge_exp2(-fabsf(y) * KGE_LOG2E);
                    const float rcp = __builtin_amdgcn_rcpf(1.f + t);
                    const float sig = y >= 0.f ? rcp : t * rcp;
                    const float softplus = fmaxf(y, 0.f) + KGE_LN2 * kge_log2(1.f + t);
                    if (e > 0.f) st_acc[h] = fmaf(e, softplus, st_acc[h]);
                    u = e * sig;
                }
                const float c1 = KIND == KGE_KIND_DIST ? u * dv[i] : u;
                coef[i] = c1;
                if constexpr (KIND == KGE_KIND_DIST) sum1[h] += c1;  // only the distance scorers' chain rule needs it
                if constexpr (TRANSH) { coef2[i] = c1 * Av[i]; sum2[h] += coef2[i]; sum3[h] += coef2[i] * Av[i]; }
            }
        }
        if constexpr (MODE == KGE_MODE_GRADT) {
            // gradient coefficient of every (query, negative) pair from the finished row constants
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int sl = 8 * (i >> 2) + 4 * g + (i & 3);
                const float K2 = ALONE ? row_K[i] : *(const float *)(side + sl * 16 + 8);       // -inf for padded queries
                float u = kge_exp2(fmaf(sv[i], xscale, K2));
                if constexpr (LOSS == KGE_LOGSIGMOID) {
                    const float y = a.gamma + sv[i];
                    const float t = kge_exp2(-fabsf(y) * KGE_LOG2E);
                    const float rcp = __builtin_amdgcn_rcpf(1.f + t);
                    u *= y >= 0.f ? rcp : t * rcp;
                }
                const float c1 = KIND == KGE_KIND_DIST ? u * dv[i] : u;
                coef[i] = c1;
                if constexpr (KIND == KGE_KIND_DIST) sum1[h] += c1;
                // (planes: the streamed rows are q and w^ themselves, not q - c w^ and w^)
                if constexpr (TRANSH && PL) coef2[i] = c1 * (Av[i] - (ALONE ? row_c[i] : *(const float *)(side + sl * 16 + 4)));
                else if constexpr (TRANSH) coef2[i] = c1 * Av[i];
            }
        }
        if constexpr (PHASE2) {
            if constexpr (BF16) {
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    bf[h][s2] = make_uint4(kge_pack_bf16x2(coef[8 * s2 + 0], coef[8 * s2 + 1]),
                                           kge_pack_bf16x2(coef[8 * s2 + 2], coef[8 * s2 + 3]),
                                           kge_pack_bf16x2(coef[8 * s2 + 4], coef[8 * s2 + 5]),
                                           kge_pack_bf16x2(coef[8 * s2 + 6], coef[8 * s2 + 7]));
                    if constexpr (TRANSH)
                        bf2[s2] = make_uint4(kge_pack_bf16x2(coef2[8 * s2 + 0], coef2[8 * s2 + 1]),
                                             kge_pack_bf16x2(coef2[8 * s2 + 2], coef2[8 * s2 + 3]),
                                             kge_pack_bf16x2(coef2[8 * s2 + 4], coef2[8 * s2 + 5]),
                                             kge_pack_bf16x2(coef2[8 * s2 + 6], coef2[8 * s2 + 7]));
                }
            } else {
                // coefficients of the scaled rows; their own scale keeps the own row's largest below 2^14.  It is lowered in a rarely taken
                // branch when a tile has larger ones (and what the row has accumulated with it), set by the first tile that has any:
                // to 2^6, so that what is 2^-30 of it is still more than the second piece's last bit.
                float cm = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int s_exp = ALONE ? s_exps[i] : str_exp_of(8 * (i >> 2) + 4 * g + (i & 3));
                    coef[i] = ldexpf(coef[i], s_exp);
                    cm = fmaxf(cm, fabsf(coef[i]));
                    if constexpr (TRANSH) { coef2[i] = ldexpf(coef2[i], OWN_ROW ? s_exp : KGE_PLANE_UNIT_EXP); cm = fmaxf(cm, fabsf(coef2[i])); }
                }
                cm = fmaxf(cm, __shfl_xor(cm, 32));        // (lanes l and l ^ 32 feed the same row)
                const bool trip = cm * c_scale > 16384.f || (c_scale == 0.f && cm > 0.f);
                if (__any(trip)) {
                    const int e = 133 + 127 - (int)((__float_as_uint(cm) >> 23) & 255u);
                    const float s_new = trip ? __uint_as_float((uint32_t)(e < 1 ? 1 : e > 254 ? 254 : e) << 23) : c_scale;
                    const float r = !trip ? 1.f : c_scale > 0.f ? s_new / c_scale : 0.f;
                    c_scale = s_new;
                    settle();
#pragma unroll
                    for (int b = 0; b < C::NBH; ++b) {
                        rescale(acc2[0][b], r);
                        if constexpr (TRANSH && OWN_ROW) rescale(acc2b[b], r);
                    }
                    settle();
                }
                if constexpr (ALONE) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) { coef_a[i] = coef[i]; if constexpr (TRANSH) coef2_a[i] = coef2[i]; }
                } else {
                    auto pieces = [&](const float *c) {
                        float x[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) x[i] = c[i] * c_scale;
                        return kge_split2(x);
                    };
#pragma unroll
                    for (int j2 = 0; j2 < 2; ++j2) {
                        coef2p[j2] = pieces(coef + 8 * j2);
                        if constexpr (TRANSH) coefw2p[j2] = pieces(coef2 + 8 * j2);
                    }
                }
            }
        }
    };
    // The FWD pass keeps all weights relative to a per-row reference exponent st_m that is only
    // raised (and what the row has accumulated rescaled) when a tile's maximum exceeds it by more than
    // KGE_TAU: weights stay below 2^KGE_TAU, and the rescaling is a rarely taken branch of the loop.
    auto of_scores = [&](int h, const float (&sv)[16], const float (&dv)[16], const float (&Av)[16]) {
        float x2[16];
        if constexpr (MODE == KGE_MODE_FWD) {
            const float tm = exponents(h, sv, x2);
            const bool have = st_m[h] > -INFINITY;
            const bool trip = tm > (have ? KGE_TAU : -INFINITY);   // without a reference, any finite entry sets one
            if (__any(trip)) {
                // the rows that tripped take the tile's maximum as their reference
                const float m_new = trip ? (have ? tm + st_m[h] : tm) : st_m[h];
                const float shift = trip ? -tm : 0.f;              // exponents relative to the new reference
                const float r = trip ? (have ? kge_exp2(-tm) : 0.f) : 1.f;   // nothing accumulated yet without one
                st_m[h] = m_new;
                st_l[h] *= r; st_acc[h] *= r; sum1[h] *= r; sum2[h] *= r; sum3[h] *= r;
                if constexpr (PL) {
                    // What has accumulated is worth 2^-tm of itself: the scale that it carries, which the coefficients of the new
                    // reference take, rises by as much (left where it was set for earlier rows, later ones that now outweigh them would
                    // have the last bits of it), until it ends at 2^126: then what there is counts for nothing and the next tile sets another.
                    // (With the accumulators rescaled here instead: TransH step 8,192 x 4,096 379 us for 369, ComplEx 4,096 x 4,096 x 256 194 / 185.)
                    const float s_new = c_scale * kge_exp2(tm);
                    if (trip) c_scale = s_new < 0x1p126f ? s_new : 0.f;
                } else {
#pragma unroll
                    for (int b = 0; b < C::NBH; ++b) {
                        // one block at a time: the accumulators live in AGPRs and pass through VGPRs here; the
                        // empty statements keep this rarely executed code from being turned into selects
                        for (int i = 0; i < 16; ++i) acc2[h][b][i] *= r;
                        asm volatile("" ::: "memory");
                        if constexpr (TRANSH) { for (int i = 0; i < 16; ++i) acc2b[b][i] *= r; asm volatile("" ::: "memory"); }
                    }
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) x2[i] += shift;       // masked entries stay at -inf
            }
        }
        weights(h, sv, dv, Av, x2);
    };
    auto epilogue2 = [&](int h, float (&d2)[16], const float (&Av)[16], bool cancel) {
        float sv[16], dv[16];
        scores2(h, d2, cancel, sv, dv);
        of_scores(h, sv, dv, Av);
    };
    auto epilogue = [&]() {
#pragma unroll
        for (int h = 0; h < OW; ++h) {
            float sv[16], dv[16], Av[16];
            scores(h, sv, dv, Av);
            of_scores(h, sv, dv, Av);
        }
    };

    if constexpr (ALONE) {
        // One wave per SIMD: what it issues beside the matrix instructions has to run under them.  A round takes tile t from its squared
        // distances to its coefficients; then the first contraction of tile t + 1 runs with their split into pieces, and the
        // second contraction of tile t with the first part of the epilogue of tile t + 1.  What bounds it is what a wave can issue: about 1,000
        // vector instructions, 96 matrix instructions and 350 others per tile and wave, one in four to five cycles (vector pipe 44 to 50 %,
        // matrix pipe 33 % busy).  us, the parts one after the other / here: TransH 8,192 x 4,096 x 128 step 367 / 338, TransE 4,096 x
        // 4,096 x 256 169 / 162, ComplEx 171 / 165, DistMult 2,048 x 8,192 x 200 142 / 140.  (With the fragments' order left to the
        // compiler, which reads them where they are used, 359, 170, 171; the first contraction of tile t + 1 under the distances and
        // weights of tile t instead: 336, 162, 169, 141.)
        static_assert(C::NSTAGE >= 4, "tiles t and t + 1 are read, one is in flight, one is being refilled");
        static_assert(NG1 % NPC == 0 && NG2 % 4 == 0, "");
        constexpr int AH1 = 2, AH2 = 2, P1_MFMAS = NG1 * G1 / 2 * (TRANSH ? 6 : 3), P2_MFMAS = NG2 * (TRANSH ? 12 : 6);
        auto land = [&]() {                                // the next tile has landed: NSTAGE - 3 younger ones may be in flight
            kge_wait_vmcnt<(C::NSTAGE - 3) * C::LPW>();
            __syncthreads();
        };
        float d2[16], Av[16];
        bool cancel;
        land();
        issue(t0 + C::NSTAGE - 2, C::NSTAGE - 2);
        set_tile(t0);
        zero1();
#pragma unroll
        for (int gq = 0; gq < NG1; ++gq) { ld1(base, gq); mma1(gq); }
        scores1(0, d2, Av, cancel);
        for (int t = t0;;) {
            if constexpr (MODE == KGE_MODE_GRADT) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float *ri = (const float *)(side + (8 * (i >> 2) + 4 * g + (i & 3)) * 16);
                    row_K[i] = ri[2];
                    if constexpr (TRANSH) row_c[i] = ri[1];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            epilogue2(0, d2, Av, cancel);
            __builtin_amdgcn_sched_barrier(0);
            land();
            issue(t + C::NSTAGE - 1, t - t0 + C::NSTAGE - 1);
            const char *stage = base;
            set_tile(t + 1);                               // (past the end: the last tile again, unused)
#pragma unroll
            for (int gq = 0; gq < AH1; ++gq) ld1(base, gq);
            __builtin_amdgcn_sched_barrier(0);
            zero1();
            Side4 sd[2];
            // (fragments are requested two groups ahead of their matrix instructions, the side information of four entries a group
            // ahead and before them: reads complete in order)
#pragma unroll
            for (int gq = 0; gq < NG1; ++gq) {
                if (gq + 1 == NG1) side4(0, sd[0]);
                if (gq + AH1 < NG1) ld1(base, gq + AH1);
                else if (gq + AH1 - NG1 < AH2) ld2(stage, gq + AH1 - NG1);
                __builtin_amdgcn_sched_barrier(0);
                mma1(gq);
#pragma unroll
                for (int p = 0; p < NPC; ++p) if (p * NG1 / NPC == gq) make_piece(p);
                KGE_MIX(P1_MFMAS / NG1, 6)
                __builtin_amdgcn_sched_barrier(0);
            }
            cancel = false;
#pragma unroll
            for (int gq = 0; gq < NG2; ++gq) {
                constexpr int every = NG2 / 4;             // groups per four entries
                const int j = gq / every;
                if (gq % every == 0 && j < 3) side4(j + 1, sd[(j + 1) & 1]);
                if (gq + AH2 < NG2) ld2(stage, gq + AH2);
                __builtin_amdgcn_sched_barrier(0);
                mma2(gq);
                if (gq % every == every - 1) scores4(0, j, sd[j & 1], d2, Av, cancel);
                KGE_MIX(P2_MFMAS / NG2, 6)
                __builtin_amdgcn_sched_barrier(0);
            }
            if (++t >= t1) break;
        }
    } else
    for (int t = t0; t < t1; ++t) {
        // tile t has landed when at most NSTAGE-2 younger tiles are still in flight; after the
        // barrier every wave has finished tile t-1, whose stage receives tile t + NSTAGE - 1
        kge_wait_vmcnt<(C::NSTAGE - 2) * C::LPW>();
        __syncthreads();
        issue(t + C::NSTAGE - 1, t - t0 + C::NSTAGE - 1);
        set_tile(t);
        // The fragments of a chunk are requested before its first MFMA (the whole phase where the registers
        // allow it).  Deeper software pipelining of the reads, enforced with scheduling barriers, was
        // measured and did not pay: inside a chunk the order is left to the compiler.
        zero1();
        constexpr int CH1 = OW > 1 ? 1 : PL ? C::PL_CHUNK : (NG1 > 4 ? 4 : NG1);   // groups per chunk: at most 64 (16) registers in flight
#pragma unroll
        for (int c0 = 0; c0 < NG1; c0 += CH1) {
#pragma unroll
            for (int gq = c0; gq < c0 + CH1; ++gq) ld1(base, gq);
#pragma unroll
            for (int gq = c0; gq < c0 + CH1; ++gq) mma1(gq);
        }
        epilogue();
        if constexpr (PHASE2) {
            constexpr int CH2 = OW > 1 ? 1 : PL ? C::PL_CHUNK : NG2;
#pragma unroll
            for (int c0 = 0; c0 < NG2; c0 += CH2) {
#pragma unroll
                for (int gq = c0; gq < c0 + CH2; ++gq) ld2(base, gq);
#pragma unroll
                for (int gq = c0; gq < c0 + CH2; ++gq) mma2(gq);
            }
        }
    }
    kge_wait_vmcnt<0>();                                  // no copy may be in flight when the LDS is released

    // ---- write-out ---------------------------------------------------------------------------------
    if constexpr (PHASE2) {
#pragma unroll
        for (int h = 0; h < OW; ++h) {
            const int oidx = oidx0 + 32 * h;
            // lanes l and l^32 hold the same own row over disjoint stream entries (same running max):
            // add their scalars.  The phase-2 accumulators already contain both halves.
            if constexpr (MODE == KGE_MODE_FWD) { st_l[h] += __shfl_xor(st_l[h], 32); st_acc[h] += __shfl_xor(st_acc[h], 32); }
            sum1[h] += __shfl_xor(sum1[h], 32); sum2[h] += __shfl_xor(sum2[h], 32); sum3[h] += __shfl_xor(sum3[h], 32);
            if (g == 0 && blockIdx.y == 0) {
                a.sum_part[(size_t)split * a.own_pad + oidx] = make_float4(sum1[h], sum2[h], sum3[h], 0.f);
                if constexpr (MODE == KGE_MODE_FWD)
                    a.stat_part[(size_t)split * a.own_pad + oidx] = make_float4(st_m[h], st_l[h], st_acc[h], 0.f);
            }
            if constexpr (PL) {
                const float inv = c_scale > 0.f ? 1.f / c_scale : 0.f;
#pragma unroll
                for (int blk = 0; blk < C::NBH; ++blk)
                    for (int i = 0; i < 16; ++i) {
                        acc2[h][blk][i] *= inv;
                        if constexpr (TRANSH && OWN_ROW) acc2b[blk][i] *= inv;
                    }
            }
#pragma unroll
            for (int blk = 0; blk < C::NBH; ++blk) {
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int dcol = (dblk0 + blk) * 32 + 8 * q4 + 4 * g;
                    const size_t o = ((size_t)split * a.own_pad + oidx) * C::DP + dcol;
                    *(float4 *)(a.acc_part + o) = make_float4(acc2[h][blk][4 * q4], acc2[h][blk][4 * q4 + 1], acc2[h][blk][4 * q4 + 2], acc2[h][blk][4 * q4 + 3]);
                    if constexpr (TRANSH && OWN_ROW)
                        *(float4 *)(a.acc_part2 + o) = make_float4(acc2b[blk][4 * q4], acc2b[blk][4 * q4 + 1], acc2b[blk][4 * q4 + 2], acc2b[blk][4 * q4 + 3]);
                }
            }
        }
    }
}

template <bool BF16, int RB, int MODE, bool TRANSH, int KIND, int LOSS, int DSPLIT>
int kge_block_launch(const KgeBlockArgs &a, int own_tiles, int nsplit, hipStream_t st) {
    using C = KgeBlockCfg<BF16, RB, MODE, TRANSH, KIND, DSPLIT>;
    auto kern = kge_block_kernel<BF16, RB, MODE, TRANSH, KIND, LOSS, DSPLIT>;
    static KgeLdsLimit lds_limit;
    if (lds_limit.set((const void *)kern, C::LDS_BYTES) != KGE_OK) return KGE_E_HIP;
    if ((int64_t)own_tiles * C::OWN_TILE != a.own_pad) return KGE_E_INVALID_ARG;   // the caller's geometry must match
    KgeBlockArgs b = a;
    b.own_tiles = own_tiles; b.nsplit = nsplit;
    constexpr int GRID_Y = MODE != KGE_MODE_SCORE ? DSPLIT : 1;
    const int groups = kge_place_plan(own_tiles, nsplit, C::OWN_TILE, (int64_t)C::ST * a.str_tiles, GRID_Y, &b.xcd_per);
    dim3 grid(8 * groups, GRID_Y);
    hipLaunchKernelGGL(kern, grid, dim3(256), C::LDS_BYTES, st, b);
    return kge_launch_status();
}
