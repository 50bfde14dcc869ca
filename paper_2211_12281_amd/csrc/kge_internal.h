// Internal declarations shared by the translation units of the gfx950 library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <mutex>
#include "../../include/kge.h"

#define KGE_HIP_TRY(expr)                                   \
    do {                                                    \
        hipError_t e__ = (expr);                            \
        if (e__ != hipSuccess) return KGE_E_HIP;            \
    } while (0)

static inline int kge_launch_status() {
    return hipGetLastError() == hipSuccess ? KGE_OK : KGE_E_HIP;
}

// RAII pair of HIP events around a kernel launch; a no-op unless kge_profile_enable(1) was called.
struct KgeProfScope {
    KgeProfScope(int slot, hipStream_t st);
    ~KgeProfScope();
    int slot_; hipStream_t st_; void *a_, *b_;
};

// Raises a kernel's dynamic LDS limit once per process; safe when several threads make the first launch together.
struct KgeLdsLimit {
    std::once_flag once;
    hipError_t err = hipSuccess;
    int set(const void *kern, int bytes) {
        std::call_once(once, [&] { err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
        return err == hipSuccess ? KGE_OK : KGE_E_HIP;
    }
};

// Kernel choices that only tests and benchmarks override (kge_debug_select); 0 = the library's own choice.
enum { KGE_KNOB_FWD_ONE_ROLE = 0, KGE_KNOB_GRADT_ONE_ROLE = 1, KGE_KNOB_SCORE_F32_MFMA = 2, KGE_KNOB_TWO_ROLE = 3,
       KGE_KNOB_GRADT_RECOMPUTE = 4, KGE_KNOB_BLOCK_PASSES = 5, KGE_KNOBS = 6 };
int kge_knob(int knob);

static inline int64_t kge_round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// ---------------------------------------------------------------------------------------------
// Tile geometry of the block kernels
// ---------------------------------------------------------------------------------------------
constexpr int KGE_STREAM_TILE = 32;   // rows streamed through LDS per iteration
constexpr int KGE_PAD = 256;          // B and N are padded to this in the workspace copies

constexpr float KGE_PLANE_UNIT_SCALE = 1024.f;      // scale of the planes of TransH's unit normals (all rows), score-only calls
// training calls: rows are scaled to a largest element in [2^(KGE_PLANE_TOP - 1), 2^KGE_PLANE_TOP), as near to the end of the fp16 range as
// they can be, unit normals by 2^-KGE_PLANE_UNIT_EXP: an element keeps 2^-24 of itself down to 2^-16 of the largest, and 2^-40 of the largest below
// (columns between 2^0 and 2^-24, the worst column's error against 64 bits: 1.2e-4, with a largest element of 2^11 2.8e-3)
constexpr int KGE_PLANE_TOP = 15, KGE_PLANE_UNIT_EXP = -15;

enum { KGE_MODE_SCORE = 0, KGE_MODE_FWD = 1, KGE_MODE_GRADT = 2 };
enum { KGE_KIND_MULT = 0, KGE_KIND_DIST = 1 };

// 32-row fragments of its operand that each of a workgroup's four waves owns (the workgroup owns
// 128 times this many rows).  Two where the registers allow it: every fragment read from the LDS then
// feeds two MFMAs, which halves the LDS traffic per flop.  Not with the TransH operands; not in the
// FWD pass, whose gradient accumulators for two fragments of 256 dimensions would take the whole
// accumulator file and more; not in the GRADT pass of the distance scorers, whose epilogue needs
// the registers.
constexpr int kge_block_ow(bool bf16, int rb, bool transh, int mode, int kind) {
    if (!bf16 || rb != 512 || transh || mode == KGE_MODE_FWD) return 1;
    return (mode == KGE_MODE_GRADT && kind == KGE_KIND_DIST) ? 1 : 2;
}

// Workgroups of a block-kernel pass that share a compute unit: the SCORE pass keeps no gradient
// accumulators and fits two, where two ring stages of its tiles fit in half of the LDS; so do the training passes on planes
// of 256 bytes a row with one operand.
constexpr int kge_block_occ(bool bf16, int rb, bool transh, int mode) {
    if (!bf16 && rb == 512 && !transh && mode != KGE_MODE_SCORE) return 2;
    return (mode == KGE_MODE_SCORE && !transh && KGE_STREAM_TILE * rb <= 32 * 1024) ? 2 : 1;
}

// The fp32 training passes read their operands as two fp16 planes [2][rows][dp] of rows scaled by a power of two of their own (kge_split2),
// which the gather writes beside the fp32 rows; there are no transposed copies.  The fp32 matrix instruction runs at 1/16 of the 16-bit
// rate; three products of pieces replace sixteen.  Calls in us, before / here.  Rows of 512 bytes (before: three bf16 pieces, six products):
// TransH 8,192 x 4,096 x 128 388 / 310, TransE 234 / 178, ComplEx 8,000 x 3,000 x 128 229 / 154, DistMult 4,096 x 4,096 x 96 110 / 93.  Rows of 1,024 bytes (fp32
// instructions over the queries, bf16 pieces made in registers over the negatives): TransE 4,096 x 4,096 x 256 366 / 214, DistMult 2,048 x
// 8,192 x 200 302 / 145, RotatE 8,192 x 2,000 x 256 384 / 228.
// Errors against 64 bits over 120 drawn calls on rows of up to 512 bytes: 0.97-1.00 times those of before (geometric mean of every gradient),
// half on rows of 1,024 bytes.  Beyond those ranges: rows at 0.05 and 0.1 of its length from a query 0.6-0.9 times, at 1e-5 (where the
// gradient is the difference of two rows' sums: 1e-2 of it either way) 1.05-1.2 times; a column that is 2^-20 of the others the same, one of
// 2^-24 1.2e-4 instead of 1.1e-5.
constexpr bool kge_block_planes(bool bf16, int rb, int mode) { (void)rb; return !bf16 && mode != KGE_MODE_SCORE; }

// Per-row side information of the queries: squared norm of q, c = w.q (TransH), the per-row
// constant K of the gradient coefficient exp2(x * log2e + K) (log2 domain), squared norm of the
// (rounded) TransH normal.
struct __attribute__((aligned(16))) KgeRowInfo { float qn, c, K, wn; };

// Placement of the workgroups (own tile, split) of the block kernels but block_gradp.hip on the 8 dies, to which workgroup ids go in turn: a
// die takes the splits congruent to xcd / per modulo 8 / per and the own tiles congruent to xcd % per modulo per (per 1,
// 2, 4 or 8), so its L2 fills with 1 / per of the own rows and per / 8 of the streamed ones.
__device__ __forceinline__ bool kge_place(int own_tiles, int nsplit, int per, int &own_tile, int &split) {
    const int lp = __builtin_ctz(per), xcd = blockIdx.x & 7, kk = blockIdx.x >> 3;
    const int own_per = (own_tiles + per - 1) >> lp, turn = kk / own_per;
    own_tile = ((kk - turn * own_per) << lp) + (xcd & (per - 1));
    split = (xcd >> lp) + (turn << (3 - lp));
    return own_tile < own_tiles && split < nsplit;
}
// Returns the workgroups per die (the grid is 8 times that, in x; y of them per id).  First the fewest workgroups on the
// fullest die, counted in turns of its 32 compute units; then the fewest rows into a die, the own ones weighed three times:
// a workgroup waits for its own rows before its first tile, while the streamed ones arrive under the products of the tile
// before.  Measured for per = 1 / 2 / 4 / 8, us of the whole call: fp32 scores DistMult 2,048 x 8,192 x 256 45.4 / 45.3 /
// 43.7 / 42.2, ComplEx 512 x 4,096 x 128 16.1 / 15.3 / 15.0 / 14.3, bf16 2,048 x 8,192 x 256 31.9 / 31.2 / 30.5 / 29.1;
// loss + gradients ComplEx 4,096 x 4,096 x 400 bf16 234.8 / 229.0 / 226.0 / 228.4 and RotatE x 256 fp32 243.3 / 241.8 /
// 241.8 / 244.0 (there the streamed operand is as large as a die's L2, 4 MB).  Weights 2 and 3 take the best or next to it in
// all of these; 1 gives DistMult fp32 1,024 x 8,192 x 128 86.8 for 86.0, 4 gives the d 400 block 229.0 for 226.8.
inline int kge_place_plan(int own_tiles, int nsplit, int own_rows, int64_t str_rows, int y, int32_t *per) {
    if (nsplit < 1) nsplit = 1;                            // nothing to stream: the workgroups find no split and end
    int64_t best_load = 0, best_rows = 0;
    int groups = 0;
    for (int p = 8; p >= 1; p >>= 1) {
        const int d = 8 / p;
        const int64_t own_die = (own_tiles + p - 1) / p, split_die = (nsplit + d - 1) / d;
        const int64_t load = (own_die * split_die * y + 31) / 32;
        const int64_t rows = 3 * own_die * own_rows + str_rows * split_die / nsplit;
        if (groups && (load > best_load || (load == best_load && rows >= best_rows))) continue;
        best_load = load; best_rows = rows; groups = (int)(own_die * split_die); *per = p;
    }
    return groups;
}

// Arguments of one block-kernel launch.  "own" is the operand a workgroup keeps in registers
// (queries when OWN_ROW, negatives otherwise); "str" is the operand streamed through LDS.
struct KgeBlockArgs {
    // (kge_block_planes: own, own2, str, str2 are fp16 planes [2][own_pad or 32 str_tiles][dp] of rows times 2^-own_exp, 2^-str_exp -
    // the normals times 2^-KGE_PLANE_UNIT_EXP -, own32, str32 and w32 the fp32 rows; there are no transposed copies)
    const int32_t *own_exp, *str_exp;
    const float *own32, *str32, *w32;
    const void *own, *own2;        // [own_pad][dp]; own2: TransH normals when OWN_ROW
    const void *str, *str2;        // [str_pad][dp]; str2: TransH normals when !OWN_ROW
    const void *strT, *strT2;      // [dp][strT_ld] transposed stream operand(s), GRAD only
    int64_t strT_ld;               // elements
    const KgeRowInfo *rowinfo;     // [Bp]
    const float *tn;               // [Np] squared norms of the negatives
    int32_t B, N;                  // true sizes (padding is masked)
    int32_t dp;                    // padded dim (elements) = RB / sizeof(elem)
    int32_t str_tiles;             // number of stream tiles in total
    int32_t tiles_per_split;       // stream tiles handled by one workgroup
    int32_t kind;                  // KGE_KIND_*
    int32_t loss;                  // kge_loss_t
    float gamma, adv_temp, c_corr; // c_corr: sampled-softmax correction c
    // outputs
    float *S_out;                  // SCORE: [B][N]
    float4 *stat_part;             // FWD: [nsplit][Bp] {running max (log2 domain), sum of weights, weighted loss, 0}
    float *acc_part, *acc_part2;   // FWD / GRADT: [nsplit][own_pad][dp]
    float4 *sum_part;              // FWD / GRADT: [nsplit][own_pad] {s1, s2, s3, 0}
    int32_t own_pad;
    int32_t own_tiles, nsplit;     // launch geometry (the grid is one-dimensional in (split, own tile))
    int32_t xcd_per;               // dies that share one split (kge_place_plan)
    const float *str_bias;         // FWD, kernel of block_sym.hip: [Np] 0 for a negative, -inf for a padding row (added to its scores)
    // the coefficients of the forward pass, kept for the pass over the negatives (block_sym.hip writes, block_gradp.hip reads):
    // one 4 KB record per (own tile of 128 queries, split, round of 64 negatives, wave), in the writer's register layout
    void *pstore;
    int32_t ps_nsplit, ps_rounds;  // splits and rounds per split of the forward pass that wrote them
    // block_sym.hip (forward pass that keeps its weights) and block_gradp.hip: the split partials of the gradient rows are
    // written as bf16 (round to nearest even), half the bytes that the finishing launch reads back.  acc_part then holds
    // [nsplit][own_pad][dp] bf16: the pass over the negatives in column order; the pass over the queries as dp/2 32-bit
    // words per row, word 64 (c / 128) + c % 64 = columns c (low half) and c + 64 (high half) for c % 128 < 64 - the
    // pairs that one lane of the chain-rule kernel holds.
    int32_t part_bf16;
};

// arguments of the rows' finish that also scales the query rows per forward split (row_finish.hpp)
struct KgeRowFinishQArgs {
    const float4 *stat_part; int nsplit, Bp, B, N, loss; float gamma, c_corr, scale; const float *pos;
    KgeRowInfo *rowinfo; float *lossb, *gpos; const uint16_t *Q; uint16_t *Qs;
};

// Row pass over a score block in memory (small_rows.hpp).  C null: statistics alone; bf16: coefficients as two bf16 pieces; dist: over the
// distance, their sums to sumq [q_splits][Bp]
struct KgeSmallRowsArgs {
    const float *S; int64_t ldS; int B, N, Bp; int loss; float gamma, adv_temp, c_corr, scale; const float *pos; KgeRowInfo *rowinfo;
    float *lossb, *gpos; uint32_t *C; int bf16, dist; float4 *sumq; int q_splits;
};


bool kge_fwd_pp_applies(bool bf16, int rb, bool transh, int dsplit);
bool kge_gradt_pp_applies(bool bf16, int rb, bool transh, int dsplit);
// the kernel of block_sym.hip serves both passes of the same configurations; it walks the stream in tiles of 64 rows
bool kge_sym_applies(bool bf16, int rb, bool transh, int dsplit);
// sampled softmax, bilinear scorers: the pass over the negatives without recomputing the scores (block_gradp.hip);
// kge_gradp_applies: the configurations whose forward pass keeps its weights for it
bool kge_gradp_applies(bool bf16, int rb, bool transh, int dsplit, int kind);
int kge_launch_gradp(const KgeBlockArgs &a, int own_tiles, int nsplit, hipStream_t st);
// launchers implemented in block_*.hip (one file per element type and pass to bound compile time)
int kge_launch_block(bool bf16, int rb, int mode, bool transh, int kind, int loss, int dsplit, const KgeBlockArgs &a,
                     int own_tiles, int nsplit, hipStream_t st);
