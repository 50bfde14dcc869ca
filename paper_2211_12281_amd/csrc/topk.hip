// Link prediction (arXiv 2211.12281, Section 3.2 "Inference"): every query is scored against a range of
// entity rows and the K best are kept.
//
//   1. prep      build the queries (Table 2), their norms and rounding residuals (and, for distance scorers with many query
//                tiles, the squared norms of the candidates; otherwise the scan makes those from its tiles)
//   2. scan      MFMA scoring of [128 or 256 queries] x [candidate tiles]; an accumulator entry that beats the
//                query's current threshold is appended to the query's candidate buffer (rare after warm-up);
//                the table is walked in growing chunks, thresholds are refreshed between chunks
//   3. compact   per query: keep the KP best buffered entries (KP > K), new threshold = the KP-th value
//   4. finish    survivors get the ranking key in fp64 with a sequential fused-multiply-add loop; sort by (key, index),
//                check with a rigorous rounding bound that no discarded candidate could belong to the top-K, write
//                the list and the rank of the held-out tail; queries that fail the check (or overflowed their
//                buffer) are re-ranked by an exhaustive fp64 scan
#include "row_ops.hpp"
#include "block_kernel.hpp"
#include "topk_bound.hpp"
#include "topk_sample.hpp"
#include <math.h>

namespace {

constexpr int TK_ST = 32;               // candidate rows per tile
constexpr int TK_HALF = 64;             // entries of one private append area

struct TopkArgs {
    const void *Qmat;                   // [Qp][dp] queries (table element type)
    const void *Wmat;                   // [Qp][dp] unit normals of the queries' relations (TransH), else nullptr
    const float *cq;                    // [Qp] w^ . q' of every query (TransH)
    const char *ent;                    // first candidate row
    int64_t ent_stride;                 // bytes between rows
    int32_t valid_bytes;                // d * sizeof(element)
    int64_t ncand;
    const float *tn;                    // [ncand rounded up to a tile] MINUS the squared norms of the candidates, or nullptr:
                                        // the scan makes them itself (kernels with FN)
    uint32_t *tmax;                     // largest squared norm of a candidate (kernels with FN)
    const float *thr;                   // [Qp] current threshold (local value units)
    const float *vt;                    // [Qp] value of the held-out tail (local units), +inf when absent
    const int32_t *true_t;              // [Q] entity ids, or nullptr
    uint2 *seg;                         // [Qp][nseg][2][TK_HALF] {value bits, candidate index}: private append
    int32_t *segcnt;                    // [Qp][nseg][2]           areas of each (query, split, lane half)
    int32_t nseg;
    uint32_t *rankcnt;                  // [Qp] candidates whose value beats the held-out tail's
    int32_t nq;                         // number of real queries (rows past it are padding)
    int32_t tile_lo, tile_hi;           // positions in the walk (topk_stride) whose tiles are scanned
    int32_t nsplit;                     // position tile_lo + i belongs to split i mod nsplit
    int32_t walk;                       // positions in all, as many as tiles or a few more: position p is tile p stride mod walk
    int32_t stride, start, step;        // start: tile of position tile_lo; step: nsplit stride mod walk
    double ratio;                       // stride / walk
    int32_t tiles, own_tiles;           // tiles of candidates, of queries
    TopkSample samp;                    // kernels with SAMPLE: the candidates of tile_hi tiles
    int32_t flush;                      // ... tiles behind one group of maxima, at most
    int32_t fold;                       // ... one maximum per lane and group instead of four
    const void *zeros;                  // 16 zero bytes (source of the padding columns)
};

// stages of the ring: two workgroups share a compute unit, but on bf16 rows over 512 bytes
constexpr int tk_stages(bool bf16, int rb) { return rb == 512 ? 4 : bf16 ? 3 : 2; }
// offset of the upper pieces in the sixteen bytes of four elements of row r: lanes that read eight bytes each of rows at one chunk index
// take different banks, sixteen of them of 32 (rows r and r ^ 4, whose chunks lie 128 bytes apart) and 32 of 64 (r and r + 16)
__device__ __forceinline__ int tk_flip(int r) { return (((r >> 2) ^ (r >> 4)) & 1) * 8; }
// the power of two that takes a row whose largest element is m to [2^14, 2^15) (zeros and subnormal numbers as the smallest normal one)
__device__ __forceinline__ int tk_plane_exp(float m) {
    const int e = (int)(__float_as_uint(m) >> 23);
    return 141 - (e > 1 ? e : 1);
}

// Asynchronous global -> LDS copies (gfx950): lane l of a wave-wide instruction writes its 16 (or 4)
// bytes to LDS byte address m0 + l*16 (l*4); the data never passes through registers, completion is
// tracked by vmcnt.  The compiler does not see these loads, so the waits are explicit.
__device__ __forceinline__ int tk_swz(int r) { return (((r >> 1) & 3) << 2) | (((r >> 3) & 1) << 1) | (r & 1); }
__device__ __forceinline__ void async_copy16(const void *g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(g) : "memory");
}
__device__ __forceinline__ void async_copy4(const void *g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(g) : "memory");
}
// u stride mod n for u, stride < n < 2^31 (ratio: stride / n): the quotient from doubles, off by one at most, in place of a 64-bit division
__device__ __forceinline__ uint32_t topk_place(uint32_t u, uint32_t stride, uint32_t n, double ratio) {
    int64_t r = (int64_t)((uint64_t)u * stride) - (int64_t)((uint64_t)(uint32_t)((double)u * ratio) * n);
    r += r < 0 ? (int64_t)n : 0;
    return (uint32_t)(r >= (int64_t)n ? r - (int64_t)n : r);
}
// (v > 0: bit order = value order; an old value that is read only costs an update more)
__device__ __forceinline__ void topk_raise(uint32_t *tmax, float v) {
    if (v > 0.f && __float_as_uint(v) > __hip_atomic_load(tmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(tmax, __float_as_uint(v));
}
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// "Local value": larger is better; DistMult: q.t; TransE: 2 q.t - |t|^2 (= -dist^2 + |q|^2); TransH (TH): with
// q' = h_perp + r, A = w^ . t and c = w^ . q', -|q' - t_perp|^2 + |q'|^2 + c^2 = 2 q'.t - |t|^2 + (A - c)^2: the
// wave's two row blocks hold q' and w^ of the SAME 32 queries, so both contractions share every fragment read and
// meet lane for lane in the accumulators.
//
// Candidate tiles (32 rows) stream through an LDS ring of NSTAGE stages filled by asynchronous copies,
// so several tiles are in flight per compute unit.  A row of RB bytes is stored unpadded with its
// 16-byte chunks XOR-swizzled by a bit permutation of (row mod 16) (tk_swz): the MFMA A-fragment reads of 16
// consecutive rows at one chunk index then fall into 16 different bank groups (an XOR with row mod 8 reaches half the
// LDS's rate: half of the LDS's active cycles were bank conflicts).  The MFMAs of tile t+1 are issued before the epilogue of tile t, so the
// matrix pipe works while the vector ALU filters.  What bounds it is what the two waves of a SIMD issue beside their MFMAs, and then
// the power that MFMAs on toggling operands draw (8,192 queries over 4M rows without hits: 1,390-1,420 TFLOP/s; 1,500 without the
// copies, 1,540 with neither copies nor epilogue).  So a tile costs the epilogue one maximum per accumulator: the held-out tail's
// count and the appends are behind one test of it, no accumulator is copied (two rounds per turn of the loop), no register is
// spilled (a reload waits for the copies in flight), and the copies of rows that do not fill RB bytes are as cheap as the others' (a
// lane mask each).  8,192 queries x 10M, d 256: 39.3 -> 35.8 ms; 539 x 4.7M, d 112 (padded): 3.55 -> 1.87 ms.
//
// FN: the squared norms of the candidates (distance scorers: part of the value; all: their maximum, which the safety check
// needs) come from the tiles in the LDS instead of a pass of their own over the table.  Every workgroup of a distance scan
// makes the norms of every tile (a wave those of eight rows), which pays while few query tiles share a candidate tile;
// the bilinear scan needs only the maximum and gives each candidate tile to one of the query tiles.
//
// fp32 rows (PL below): the fp32 MFMA runs at 1/16 of the 16-bit rate, so every element is taken as two fp16 pieces of the row scaled by
// a power of two of its own, and three products of pieces replace one of fp32 (a value's error is no larger: the pieces' 2^-23 is less
// than what the fp32 MFMAs' chain of sums adds; mean distance of held-out tails' ranks from 64 bits, 512 of 200,000, over five scorers, five
// kinds of tables and d 16 / 32 / 64 / 120 / 200 / 256: 0.285 0.320 0.307 0.301 0.317 0.317 before, 0.269 0.296 0.279 0.280 0.286 0.286 here, d
// 8 0.256 and 0.254; the tops alike).  The
// table is not rewritten: a tile's rows are split in the LDS, in place, by the walk that makes their norms - eight lanes per row, a
// chunk of four elements becomes eight bytes of upper and eight of lower pieces, so no lane waits for another's reads - between two
// barriers.  A tile is split, multiplied and filtered in one round while the other workgroup of the compute unit has the matrix pipe;
// rows of 1,024 bytes keep two stages of the ring so that there is another, where there are two query tiles or more (make_plan).  Bound by what the two waves of a SIMD issue (d 256, 6,774
// queries: vector pipe 38 %, matrix pipe 29 %, LDS 33 % of the cycles, a seventh of that bank conflicts, half of it before tk_flip: 2.20 -> 2.15 ms).
// Whole calls, fp32 MFMA / pieces: DistMult d 256, 6,774 x 92,000 3.95 / 2.03 ms, 128 x 1M 697 / 421 us; RotatE d 232, 391 x 963,002 2.35 /
// 0.99 ms; TransE d 128, 300 x 1M 1.03 / 0.56 ms; TransH d 56, 50 x 5.4M 2.67 / 0.91 ms; TransE d 128, 26 x 32,113 80 / 75 us.
//
// A split's tiles are dealt round-robin, so that neighbouring rows that all beat the threshold - a table sorted by type or
// community - are spread over the append areas of many splits.  Where these are few, the tiles are walked in strides of about 0.618 of
// the table (topk_stride), so that any stretch of the walk - a chunk, and in it the tiles of a split - holds rows from all over
// the table: one sorted by length or popularity, too, appends about as many rows per area as a shuffled one.  (In order of the ids the first chunk is the head of the table, and
// where that is the better part its rows beat a threshold that stands for all of it: 8,192 queries over 1M rows, d 128, lengths falling
// from 1.5 to 0.3 262 ms, here 4.4; 2M rows, d 256, as rank^-0.2 1,560 and 7.6; shuffled 4.35 and 8.26 / 4.27 and 8.22.)
//
// SAMPLE: no appends; a tile has a row of each of 32 parts of the table (topk_sample.hpp), and every lane leaves the maxima of its
// rows by groups.  The KP-th largest group maximum is a value that at least KP candidates reach: the threshold that the scan proper
// starts with.  Every group of maxima stands for all of the table - tiles from all over it, at changing places within their pieces, four of
// the eight groups of a split for every part - so that about as many rows beat the threshold whatever their order (0.9 to 1.7 times
// KP / sample of them over sorted, periodic, clustered and shuffled tables of 20,000 to 5.7M rows, and 2.5 over 8,000 sorted ones).
// (Rows at even distances see one phase of a table that repeats with a period of the distance, and give a sorted table's best rows to one
// group in eight.  Rows in strides of 0.618 of the table do neither, but take eight vector instructions a copy where these take two: a sample of
// 23 queries x 378,761, d 432 23.8 us, here 21.9; fp32, 6,759 x 85,599, d 144 190 and 173.)
template <bool BF16, int RB, int KIND, int OB, bool TH = false, bool FN = false, bool SAMPLE = false>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
void topk_scan_kernel(const TopkArgs a) {
    static_assert(!TH || (OB == 2 && KIND == KGE_KIND_DIST), "TransH: one block of queries, one of normals");
    constexpr bool PL = !BF16;                          // fp32 rows: two fp16 pieces of every element
    static_assert(!PL || FN, "the pieces' scales and the norms come from one walk over the tile");
    constexpr int NQ = TH ? 1 : OB;                     // blocks of 32 queries per wave
    constexpr int KS = RB / 32;
    constexpr int TILE_BYTES = TK_ST * RB;
    constexpr int NINST = TILE_BYTES / 1024;            // wave-wide 1 KB copies per tile
    constexpr int IPW = NINST / 4;                      // ... per wave
    constexpr bool SIDE = KIND == KGE_KIND_DIST && !FN; // the norms stream beside the tiles
    constexpr int LPW = IPW + (SIDE ? 1 : 0);
    constexpr int NSTAGE = tk_stages(BF16, RB);
    constexpr int SIDE_SLOTS = NSTAGE + 1;
    extern __shared__ __attribute__((aligned(256))) char lds[];
    char *side_base = lds + NSTAGE * TILE_BYTES;        // [SIDE_SLOTS][4 waves][64 floats]
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, g = lane >> 5;
    // Workgroups are handed to the 8 XCDs round-robin.  All query tiles that walk the same candidate
    // range are given ids with the same residue mod 8, so they share one XCD's L2 and the range is
    // fetched from HBM once.
    const int xcd = blockIdx.x & 7, kk = blockIdx.x >> 3;
    const int own_tile = kk % a.own_tiles, split = xcd + 8 * (kk / a.own_tiles);
    const int own_base = own_tile * (128 * NQ);
    const int npos = a.tile_hi - a.tile_lo;
    int nt = 0;                                         // tiles of this split
    if (split < a.nsplit) nt = (npos - split + a.nsplit - 1) / a.nsplit;
    // Every (query, split, lane half) owns a private append area, so appending needs no atomics: the
    // count lives in a register and is stored once at the end.  Two lanes (g = 0, 1) serve one query.
    if (nt <= 0) {
        if (split < a.nseg)
            for (int ob = 0; ob < NQ; ++ob)
                a.segcnt[((size_t)(own_base + (wave * NQ + ob) * 32 + lr) * a.nseg + split) * 2 + g] = 0;
        return;
    }

    uint4 own[OB][KS];                                  // (PL: 2 ks the upper pieces of step ks, 2 ks + 1 the lower)
    int own_e[PL ? OB : 1];
    // PL: a query row in pieces, scaled by the power of two that takes its largest element to [2^14, 2^15)
    auto split_own = [&](int ob, const char *p) {
        auto at = [&](int ks) { return p + 512 * (ks >> 3) + 32 * (ks & 7); };
        float m = 0.f;
        auto row_max = [&](const uint4 &v) {
            m = fmaxf(fmaxf(fmaxf(m, fabsf(__uint_as_float(v.x))), fmaxf(fabsf(__uint_as_float(v.y)), fabsf(__uint_as_float(v.z)))), fabsf(__uint_as_float(v.w)));
        };
#pragma unroll 4
        for (int ks = 0; ks < KS / 2; ++ks) { row_max(*(const uint4 *)at(ks)); row_max(*(const uint4 *)(at(ks) + 256)); }
        m = fmaxf(m, __shfl_xor(m, 32));
        const int e = tk_plane_exp(m);
        own_e[PL ? ob : 0] = -e;
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks) {
            if (ks % 2 == 0) __builtin_amdgcn_sched_barrier(0);                  // (a row of elements beside the pieces would spill)
            const uint4 a0 = *(const uint4 *)at(ks), a1 = *(const uint4 *)(at(ks) + 256);
            const float x[8] = { ldexpf(__uint_as_float(a0.x), e), ldexpf(__uint_as_float(a0.y), e), ldexpf(__uint_as_float(a0.z), e), ldexpf(__uint_as_float(a0.w), e),
                                 ldexpf(__uint_as_float(a1.x), e), ldexpf(__uint_as_float(a1.y), e), ldexpf(__uint_as_float(a1.z), e), ldexpf(__uint_as_float(a1.w), e) };
            const KgeP2 two = kge_split2(x);
            own[ob][2 * ks] = two.p[0]; own[ob][2 * ks + 1] = two.p[1];
        }
    };
    float thr[NQ], vt[NQ], low[NQ];
    int qid[NQ], myc[NQ];
    uint32_t above[NQ];
#pragma unroll
    for (int ob = 0; ob < NQ; ++ob) {
        qid[ob] = own_base + (wave * NQ + ob) * 32 + lr;
        myc[ob] = 0;
        const char *p = (const char *)a.Qmat + (size_t)qid[ob] * RB + g * 16;
        if constexpr (PL) split_own(ob, p);
        else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) own[ob][ks] = *(const uint4 *)(p + ks * 32);
        }
        thr[ob] = SAMPLE ? 0.f : a.thr[qid[ob]];
        vt[ob] = SAMPLE ? 0.f : a.vt[qid[ob]];
        low[ob] = fminf(thr[ob], vt[ob]);               // (vt is +inf where there is no held-out tail)
        above[ob] = 0;
    }
    float cq = 0.f;
    if constexpr (TH) {
        const char *p = (const char *)a.Wmat + (size_t)qid[0] * RB + g * 16;
        if constexpr (PL) split_own(1, p);
        else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) own[1][ks] = *(const uint4 *)(p + ks * 32);
        }
        cq = a.cq[qid[0]];
    }

    // ---- loader geometry of this lane: instruction jj covers LDS bytes [(wave*IPW+jj) KB, +1 KB) ----
    // A copy takes a wave-uniform base (the tile's first row, scalar registers) and ONE 32-bit offset per lane that does not
    // change from tile to tile (row in the tile x stride + source chunk), and its LDS address is scalar arithmetic on the
    // wave's number: no vector instruction per copy in the loop.  The table's last, ragged tile (and rows too far apart for the
    // offset) take per-lane 64-bit addresses, computed where they are needed; their padding columns read the 16 zero bytes.
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    auto ld_row_of = [&](int jj, int ln) { return ((wave_u * IPW + jj) * 1024 + ln * 16) / RB; };
    auto ld_col_of = [&](int jj, int ln) {
        const int byte = (wave_u * IPW + jj) * 1024 + ln * 16, r = byte / RB, pos = (byte % RB) / 16;
        return (pos ^ tk_swz(r)) * 16;                  // source chunk that belongs at this LDS position
    };
    uint32_t ld_off[IPW];
#pragma unroll
    for (int jj = 0; jj < IPW; ++jj) ld_off[jj] = (uint32_t)(ld_row_of(jj, lane) * a.ent_stride + ld_col_of(jj, lane));
    // (a lane number that the compiler cannot see through: what rare paths derive from it is computed there instead of in
    // front of the loop, where it would hold - and spill - registers; a reload waits for the asynchronous copies in flight)
    auto here = [&] { int ln = lane; asm volatile("" : "+v"(ln)); return ln; };
    // Rows shorter than RB: the lanes of the padding columns take no part in the copies (they may lie behind the table's end), and
    // what they would write is zeroed once, here.
    uint64_t ld_live[IPW];
#pragma unroll
    for (int jj = 0; jj < IPW; ++jj) ld_live[jj] = __ballot(ld_col_of(jj, lane) < a.valid_bytes);
    if (a.valid_bytes != RB) {
        for (int i = tid * 16; i < NSTAGE * TILE_BYTES; i += 256 * 16) *(uint4 *)(lds + i) = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    }
    const bool offsets32 = a.ent_stride < (1ll << 26);  // (uniform; 32 rows x stride fits the offset)
    // the tiles of the split's positions, one after the other (the copies run ahead of the epilogue); below 2^27, sums below 2^28
    auto along = [&](int tile) { return tile < a.walk ? tile : tile - a.walk; };
    int in_tile = 0, out_tile = 0;
    if constexpr (!SAMPLE)
        in_tile = out_tile = along(__builtin_amdgcn_readfirstlane((int)topk_place(split, a.stride, a.walk, a.ratio)) + a.start);
    // SAMPLE: the split's tiles are split + nsplit x, and of `groups` groups of maxima number v takes x = v, v + groups, ...: every group has
    // tiles from all over, and the splits, in step, are at about one place of every part of the table
    int in_x = 0, in_group = 0;
    const int groups = SAMPLE ? (nt + a.flush - 1) / a.flush : 0;
    const char *ld_ptr[SAMPLE ? IPW : 1];               // rows from all over the table: a pointer per copy
    if constexpr (SAMPLE) {
#pragma unroll
        for (int jj = 0; jj < IPW; ++jj) ld_ptr[jj] = a.ent + (int64_t)a.samp.first(ld_row_of(jj, lane)) * a.ent_stride + ld_col_of(jj, lane);
    }
    auto issue = [&](int k, int slot) {
        const bool on = k > 0 && k < nt;                // past the end: a harmless repeat keeps vmcnt uniform
        const int stage = slot % NSTAGE;
        const uint32_t lbase = lds0 + stage * TILE_BYTES + wave_u * (IPW * 1024);
        if constexpr (SAMPLE) {
            if (on && (in_x += groups) >= nt) in_x = ++in_group;
            const uint32_t place = a.samp.place((uint32_t)(split + a.nsplit * in_x));
            const int64_t at = place * a.ent_stride;
#pragma unroll
            for (int jj = 0; jj < IPW; ++jj)
                asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %2\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b64 exec, -1"
                             ::"s"(lbase + jj * 1024), "v"(ld_ptr[jj] + at), "s"(ld_live[jj]) : "memory");
            if constexpr (SIDE) async_copy4(a.tn + a.samp.first(lr) + place, lds0 + NSTAGE * TILE_BYTES + ((slot % SIDE_SLOTS) * 4 + wave_u) * 256);
            return;
        }
        if (on) in_tile = along(in_tile + a.step);               // (one behind the table repeats the last row, masked in the epilogue like those of the last tile)
        const int64_t tile = in_tile;
        if (offsets32 && tile * TK_ST + TK_ST <= a.ncand) {
            const char *tb = a.ent + tile * TK_ST * a.ent_stride;
#pragma unroll
            for (int jj = 0; jj < IPW; ++jj)
                // (the whole wave is here: all lanes are live again behind the copy)
                asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1"
                             ::"s"(lbase + jj * 1024), "v"(ld_off[jj]), "s"(tb), "s"(ld_live[jj]) : "memory");
        } else {
            const int ln = here();
#pragma unroll
            for (int jj = 0; jj < IPW; ++jj) {
                int64_t cand = tile * TK_ST + ld_row_of(jj, ln);
                cand = cand < a.ncand ? cand : a.ncand - 1; // rows past the end are masked in the epilogue
                const int col = ld_col_of(jj, ln);
                const char *gp = col < a.valid_bytes ? a.ent + cand * a.ent_stride + col : (const char *)a.zeros;
                async_copy16(gp, lbase + jj * 1024);
            }
        }
        if constexpr (SIDE) async_copy4(a.tn + (tile < a.tiles ? tile : a.tiles - 1) * TK_ST + lr, lds0 + NSTAGE * TILE_BYTES + ((slot % SIDE_SLOTS) * 4 + wave_u) * 256);
    };
    // ---- A-fragment addresses: chunk (2 ks + g) of row lr sits at position chunk ^ tk_swz(lr) ----------
    // (stages and rows are whole multiples of 256 bytes, so chunk 2 b + g of a row is chunk g's address with b's bits flipped: one
    // register instead of eight)
    const uint32_t frag0 = lds0 + lr * RB + 16 * (g ^ tk_swz(lr));
    auto mma_tile = [&](int slot, kge_f32x16 (&acc)[OB]) {
        const uint32_t frag = frag0 + (slot % NSTAGE) * TILE_BYTES;
        auto fragment = [&](int ks) {
            return *(const __attribute__((address_space(3))) kge_u32x4 *)(uintptr_t)((frag ^ (32 * (ks & 7))) + 256 * (ks >> 3));
        };
        // Rows of 512 bytes: the fragment of step ks + AH is requested before the MFMAs of step ks are issued, and the
        // scheduler is held to that order (left to itself the compiler reads each fragment right before its two MFMAs and
        // waits for it).  The kernels of 1,024-byte rows have no registers for fragments in flight: held to this order they
        // spill operands inside the loop, so they keep the compiler's.
        constexpr int AH = RB == 512 ? (TH ? 2 : 3) : 0;
        kge_u32x4 av[AH > 0 ? AH + 1 : KS];
        if constexpr (!PL) {
#pragma unroll
            for (int ks = 0; ks < (AH > 0 ? AH : KS); ++ks) av[ks] = fragment(ks);
        }
        if constexpr (SIDE) {
            // TransE: the accumulators start at -|t|^2 of their candidate row and the queries are stored
            // doubled, so the contraction itself yields 2 q.t - |t|^2
            const char *tside = side_base + ((slot % SIDE_SLOTS) * 4 + wave_u) * 256;
            // (rows 8 j + 4 g .. + 3 of the tile are registers 4 j .. 4 j + 3: one 16-byte read per j)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // (the side array holds -|t|^2: the accumulators are loaded, not computed)
                const kge_f32x4 tn4 = *(const kge_f32x4 *)(tside + (8 * j + 4 * g) * 4);
#pragma unroll
                for (int ob = 0; ob < NQ; ++ob)
                    for (int u = 0; u < 4; ++u) acc[ob][4 * j + u] = tn4[u];
            }
            if constexpr (TH) for (int i = 0; i < 16; ++i) acc[1][i] = 0.f;
        } else {
#pragma unroll
            for (int ob = 0; ob < OB; ++ob) for (int i = 0; i < 16; ++i) acc[ob][i] = 0.f;
        }
        if constexpr (PL) {
            // chunk c of a row (four elements) and chunk c + 16, 256 bytes on, make a step: the upper pieces of both are one operand, the
            // lower ones the other.
            constexpr int AP = OB == 2 ? 1 : 2;
            const uint32_t up = frag + tk_flip(lr), down = frag + 8 - tk_flip(lr);
            auto pieces = [&](uint32_t f, int ks) {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const uint32_t at = (f ^ (32 * (ks & 7))) + 512 * (ks >> 3);
                const u32x2 lo = *(const __attribute__((address_space(3))) u32x2 *)(uintptr_t)at;
                const u32x2 hi = *(const __attribute__((address_space(3))) u32x2 *)(uintptr_t)(at + 256);
                return make_uint4(lo.x, lo.y, hi.x, hi.y);
            };
            KgeP2 fv[AP + 1];
#pragma unroll
            for (int ks = 0; ks < AP; ++ks) { fv[ks].p[0] = pieces(up, ks); fv[ks].p[1] = pieces(down, ks); }
#pragma unroll
            for (int ks = 0; ks < KS / 2; ++ks) {
                if (ks + AP < KS / 2) { fv[(ks + AP) % (AP + 1)].p[0] = pieces(up, ks + AP); fv[(ks + AP) % (AP + 1)].p[1] = pieces(down, ks + AP); }
                __builtin_amdgcn_sched_barrier(0);
                const KgeP2 &f = fv[ks % (AP + 1)];
                auto mm = [](kge_f32x16 c, uint4 x, uint4 y) {
                    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(kge_f16x8, x), __builtin_bit_cast(kge_f16x8, y), c, 0, 0, 0);
                };
#pragma unroll
                for (int ob = 0; ob < OB; ++ob) acc[ob] = mm(acc[ob], f.p[0], own[ob][2 * ks + 1]);
#pragma unroll
                for (int ob = 0; ob < OB; ++ob) acc[ob] = mm(acc[ob], f.p[1], own[ob][2 * ks]);
#pragma unroll
                for (int ob = 0; ob < OB; ++ob) acc[ob] = mm(acc[ob], f.p[0], own[ob][2 * ks]);
                __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (AH == 0) {
#pragma unroll
                for (int ob = 0; ob < OB; ++ob) acc[ob] = kge_mma16<BF16>(acc[ob], __builtin_bit_cast(uint4, av[ks]), own[ob][ks]);
            } else {
                if (ks + AH < KS) av[(ks + AH) % (AH + 1)] = fragment(ks + AH);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ob = 0; ob < OB; ++ob) acc[ob] = kge_mma16<BF16>(acc[ob], __builtin_bit_cast(uint4, av[ks % (AH + 1)]), own[ob][ks]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // ---- norms of a tile from its LDS stage: eight lanes per row, 16 bytes per lane and 128-byte piece of the row (an odd row
    // starts one piece later, so that the two rows of sixteen lanes fall into different halves of the banks) ----
    float *nrm = (float *)side_base;                    // [2][32] minus the squared norms (even and odd slots)
    float nmax = 0.f;
    auto norm_tile = [&](int slot) {
        const int ln = KIND == KGE_KIND_MULT ? here() : lane;    // (bilinear: one tile in own_tiles)
        const int row = wave * 8 + (ln >> 3);
        const char *base = lds + (slot % NSTAGE) * TILE_BYTES + row * RB + (ln & 7) * 16;
        constexpr int NP = RB / 128;
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const kge_u32x4 v = *(const kge_u32x4 *)(base + ((i + row) % NP) * 128);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float x0 = __uint_as_float(v[k] << 16), x1 = __uint_as_float(v[k] & 0xffff0000u);
                sq = fmaf(x0, x0, sq); sq = fmaf(x1, x1, sq);
            }
        }
        sq += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(sq), 0xB1, 0xf, 0xf, true));    // lane ^ 1
        sq += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(sq), 0x4E, 0xf, 0xf, true));    // lane ^ 2
        sq += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(sq), 0x141, 0xf, 0xf, true));   // 7 - lane: the other four
        if constexpr (KIND == KGE_KIND_DIST) if ((ln & 7) == 0) nrm[(slot & 1) * 32 + row] = -sq;
        nmax = fmaxf(nmax, sq);
    };
    // ---- fp32 rows: the same lanes put two fp16 pieces of each element in its place, sixteen bytes of four elements -> eight of upper
    // and eight of lower pieces; the row is scaled by the power of two that takes its largest element to [2^14, 2^15) ----
    int *row_e = (int *)side_base + 64;                 // [2][32] the exponents that take the products back
    auto split_tile = [&](int slot) {
        const int row = wave * 8 + (lane >> 3);
        char *base = lds + (slot % NSTAGE) * TILE_BYTES + row * RB + (lane & 7) * 16;
        constexpr int NP = RB / 128;
        kge_f32x4 v[NP];
        float sq = 0.f, m = 0.f;
#pragma unroll
        for (int i = 0; i < NP; ++i) v[i] = *(const kge_f32x4 *)(base + ((i + row) % NP) * 128);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            m = fmaxf(fmaxf(m, fabsf(v[i][0])), fabsf(v[i][1])); m = fmaxf(fmaxf(m, fabsf(v[i][2])), fabsf(v[i][3]));
#pragma unroll
            for (int k = 0; k < 4; ++k) sq = fmaf(v[i][k], v[i][k], sq);
        }
        auto dpp = [](float x, auto c) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(c)::value, 0xf, 0xf, true)); };
        constexpr std::integral_constant<int, 0xB1> x1{}; constexpr std::integral_constant<int, 0x4E> x2{}; constexpr std::integral_constant<int, 0x141> x7{};
        m = fmaxf(m, dpp(m, x1)); sq += dpp(sq, x1);
        m = fmaxf(m, dpp(m, x2)); sq += dpp(sq, x2);
        m = fmaxf(m, dpp(m, x7)); sq += dpp(sq, x7);
        const int e = tk_plane_exp(m);
        const int up = tk_flip(row);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            // (two conversions per instruction and the remainder as a mixed multiply-add: six instructions for two elements)
            typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            uint2 hi, lo;
            auto pair = [&](float a, float b, uint32_t &h, uint32_t &l) {
                const f32x2 y = { ldexpf(a, e), ldexpf(b, e) };
                const f16x2 top = __builtin_convertvector(y, f16x2);
                const f32x2 rest = { __builtin_fmaf((float)top[0], -1.f, y[0]), __builtin_fmaf((float)top[1], -1.f, y[1]) };
                h = __builtin_bit_cast(uint32_t, top); l = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, f16x2));
            };
            pair(v[i][0], v[i][1], hi.x, lo.x); pair(v[i][2], v[i][3], hi.y, lo.y);
            char *at = base + ((i + row) % NP) * 128;
            *(uint2 *)(at + up) = hi; *(uint2 *)(at + 8 - up) = lo;
        }
        if ((lane & 7) == 0) { nrm[(slot & 1) * 32 + row] = -sq; row_e[(slot & 1) * 32 + row] = -e; }
        nmax = fmaxf(nmax, sq);
    };
    int turn = 0;                                       // bilinear: the query tile whose turn a candidate tile is
    auto norms_of = [&](int slot) {
        if constexpr (FN) {
            if constexpr (KIND == KGE_KIND_DIST) norm_tile(slot);
            else if constexpr (!SAMPLE) {
                if (turn == own_tile) norm_tile(slot);
                turn = turn + 1 == a.own_tiles ? 0 : turn + 1;
            }
        }
    };

#pragma unroll
    for (int s2 = 0; s2 < NSTAGE - 1; ++s2) issue(s2, s2);
    if constexpr (!PL) {
        wait_vmcnt<(NSTAGE - 2) * LPW>();
        __syncthreads();
        issue(NSTAGE - 1, NSTAGE - 1);
    }
    float best[SAMPLE ? NQ : 1][4];                     // running maxima of a group: tile k leaves those of its rows 8 j + 4 g .. + 3 in number j + k
    int out_x = 0, out_group = 0;                       // SAMPLE: as in_x, in_group
    if constexpr (SAMPLE) for (int ob = 0; ob < NQ; ++ob) for (int j = 0; j < 4; ++j) best[ob][j] = -INFINITY;
    // One round: start the MFMAs of the next tile, then the epilogue of this one, whose accumulators the other name holds (two
    // rounds per turn of the loop, so that no accumulator is copied).
    auto round = [&](int slot, kge_f32x16 (&acc)[OB], kge_f32x16 (&accn)[OB]) {
        const int64_t tile = out_tile;
        // ---- tile + 1: wait for its data, refill the stage that tile `tile` just vacated, start its MFMAs
        // (PL: this tile's own data, split, multiplied and filtered in one round: the other workgroup of the compute unit has the
        // pipe meanwhile, and there are no registers for a second set of accumulators)
        wait_vmcnt<(NSTAGE - 2) * LPW>();
        __syncthreads();
        if constexpr (PL) {
            issue(slot + NSTAGE - 1, slot + NSTAGE - 1);
            split_tile(slot);
            __syncthreads();
            mma_tile(slot, acc);
        } else {
            issue(slot + NSTAGE, slot + NSTAGE);
            if constexpr (FN) { if (slot + 1 < nt) norms_of(slot + 1); }
            mma_tile(slot + 1, accn);                   // (the last iteration recomputes a stale stage: unused)
        }
        // ---- epilogue of tile `tile`: cheap wave-level test first, counting and appending only on a hit ----
        const bool tile_full = tile * TK_ST + TK_ST <= a.ncand;
        if constexpr (PL) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                typedef int i32x4 __attribute__((ext_vector_type(4)));
                const i32x4 e4 = *(const i32x4 *)(row_e + (slot & 1) * 32 + 8 * j + 4 * g);
#pragma unroll
                for (int ob = 0; ob < OB; ++ob)
                    for (int u = 0; u < 4; ++u) acc[ob][4 * j + u] = ldexpf(acc[ob][4 * j + u], e4[u] + own_e[ob]);
            }
        }
        if constexpr (FN && KIND == KGE_KIND_DIST) {    // (this tile's norms were written before the barrier above)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const kge_f32x4 tn4 = *(const kge_f32x4 *)(nrm + (slot & 1) * 32 + 8 * j + 4 * g);
#pragma unroll
                for (int ob = 0; ob < NQ; ++ob)
                    for (int u = 0; u < 4; ++u) acc[ob][4 * j + u] += tn4[u];
            }
        }
        if constexpr (TH) {
#pragma unroll
            for (int i = 0; i < 16; ++i) { const float x = acc[1][i] - cq; acc[0][i] = fmaf(x, x, acc[0][i]); }
        }
        if constexpr (SAMPLE) {
#pragma unroll
            for (int ob = 0; ob < NQ; ++ob) {
                float m[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    m[j] = fmaxf(fmaxf(fmaxf(best[ob][(j + 3) & 3], acc[ob][4 * j]), fmaxf(acc[ob][4 * j + 1], acc[ob][4 * j + 2])), acc[ob][4 * j + 3]);
                for (int j = 0; j < 4; ++j) best[ob][j] = m[j];
            }
            if ((out_x += groups) >= nt) {
                out_x = ++out_group;
#pragma unroll
                for (int ob = 0; ob < NQ; ++ob) {
                    const size_t area = ((size_t)qid[ob] * a.nseg + split) * 2 + g;
                    auto put = [&](float x) {           // (the plan keeps a split's groups within an area)
                        if (myc[ob] >= TK_HALF) return;
                        a.seg[area * TK_HALF + myc[ob]] = make_uint2(__float_as_uint(x), (uint32_t)((split * 2 + g) * TK_HALF + myc[ob]));
                        ++myc[ob];
                    };
                    if (a.fold) put(fmaxf(fmaxf(best[ob][0], best[ob][1]), fmaxf(best[ob][2], best[ob][3])));
                    else for (int j = 0; j < 4; ++j) put(best[ob][j]);
                    for (int j = 0; j < 4; ++j) best[ob][j] = -INFINITY;
                }
            }
            return;
        }
        if (!tile_full) {
            const int gg = here() >> 5;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const bool out = tile * TK_ST + 8 * (i >> 2) + 4 * gg + (i & 3) >= a.ncand;
#pragma unroll
                for (int ob = 0; ob < NQ; ++ob) acc[ob][i] = out ? -INFINITY : acc[ob][i];
            }
        }
#pragma unroll
        for (int ob = 0; ob < NQ; ++ob) {
            const kge_f32x16 &v = acc[ob];              // the values are the accumulators themselves
            float mx = v[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, v[i]);
            if (__any(mx > low[ob])) {
                if (a.true_t && __any(mx > vt[ob])) {
                    // v > vt exactly when vt - v is negative: the sign bits are shifted into one word (one subtraction and
                    // one funnel shift per entry, no compare results through scalar registers) and counted at the end
                    uint32_t signs = 0;
#pragma unroll
                    for (int i = 0; i < 16; ++i) signs = __builtin_amdgcn_alignbit(signs, __float_as_uint(vt[ob] - v[i]), 31);
                    above[ob] += (uint32_t)__builtin_popcount(signs);
                }
                // (a held-out tail that ranks low brings nearly every tile here: the comparisons below cost two calls of 8,192 x 10M 81.0
                // ms, behind this test 72.6; with tails that rank high 33.7 -> 33.9 a call)
                if (!__any(mx > thr[ob])) continue;
                // A hit is nearly always the only one of its lane, and then it is the maximum: its place comes from a mask of the
                // comparisons, without sixteen branches that each wait for a compare result.
                uint32_t hits = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) hits |= v[i] > thr[ob] ? 1u << i : 0u;
                // (an entry's area is addressed here, on the rarely taken path, instead of living in registers)
                const int ln = here(), gg = ln >> 5, qq = own_base + (wave_u * NQ + ob) * 32 + (ln & 31);
                auto append = [&](int i, float x) {
                    const int64_t cand = tile * TK_ST + 8 * (i >> 2) + 4 * gg + (i & 3);
                    if (myc[ob] < TK_HALF)
                        a.seg[(((size_t)qq * a.nseg + split) * 2 + gg) * TK_HALF + myc[ob]] = make_uint2(__float_as_uint(x), (uint32_t)cand);
                    ++myc[ob];                          // counts past the area mark the overflow for the compaction
                };
                if (!__any((hits & (hits - 1)) != 0)) {
                    if (hits) append(__builtin_ctz(hits), mx);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) if (hits >> i & 1) append(i, v[i]);
                }
            }
        }
    };
    kge_f32x16 acc_a[OB], acc_b[OB];
    if constexpr (PL) {
        for (int k = 0; k < nt; ++k, out_tile = along(out_tile + a.step)) round(k, acc_a, acc_b);
    } else {
        norms_of(0);
        mma_tile(0, acc_a);
        for (int k = 0; k < nt; k += 2) {
            round(k, acc_a, acc_b);
            out_tile = along(out_tile + a.step);
            if (k + 1 < nt) round(k + 1, acc_b, acc_a);
            out_tile = along(out_tile + a.step);
        }
    }
    wait_vmcnt<0>();                                    // no copy may still be in flight when the LDS is released
#pragma unroll
    for (int ob = 0; ob < NQ; ++ob) a.segcnt[((size_t)qid[ob] * a.nseg + split) * 2 + g] = myc[ob];
    if constexpr (SAMPLE) return;
    if (a.true_t) {
#pragma unroll
        for (int ob = 0; ob < NQ; ++ob) if (above[ob] && qid[ob] < a.nq) atomicAdd(a.rankcnt + qid[ob], above[ob]);
    }
    if constexpr (FN) {
        // One update per workgroup, and only where the maximum grows: updates of one address follow each other at 11 ns.
        nmax = kge_wave_max(nmax);
        __syncthreads();                                // (the ring is no longer read)
        float *wmax = (float *)lds;
        if (lane == 0) wmax[wave] = nmax;
        __syncthreads();
        if (tid == 0) topk_raise(a.tmax, fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])));
    }
}

// ---------------------------------------------------------------------------------------------
// bitonic sorts in LDS (256 threads)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint64_t pack_value(uint32_t vbits, uint32_t idx) {
    // unsigned order of the float, then smaller index first: sort DESCENDING on the packed word
    const uint32_t ord = vbits ^ ((vbits >> 31) ? 0xFFFFFFFFu : 0x80000000u);
    return ((uint64_t)ord << 32) | (uint64_t)(0xFFFFFFFFu - idx);
}
__device__ __forceinline__ uint2 unpack_value(uint64_t w) {
    const uint32_t ord = (uint32_t)(w >> 32);
    const uint32_t vbits = ord ^ ((ord >> 31) ? 0x80000000u : 0xFFFFFFFFu);
    return make_uint2(vbits, 0xFFFFFFFFu - (uint32_t)w);
}

struct KeyIdx { double key; int idx; };
__device__ __forceinline__ bool worse(double ka, int ia, double kb, int ib) { return ka > kb || (ka == kb && ia > ib); }

__device__ void bitonic_asc_pair(double *key, int *idx, int P) {
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < P / 2; t += blockDim.x) {
                const int i = 2 * t - (t & (j - 1)), p = i + j;
                const bool asc = (i & k) == 0;
                const double kx = key[i], ky = key[p];
                const int ix = idx[i], iy = idx[p];
                if (worse(kx, ix, ky, iy) == asc) { key[i] = ky; key[p] = kx; idx[i] = iy; idx[p] = ix; }
            }
            __syncthreads();
        }
}

// Per query: merge the kept list with the fresh append areas, keep the KP best (in no particular order), refresh the threshold;
// without a list to keep (the maxima of a sample), the threshold alone.
// All of it is latency: a thread holds up to TK_MINE entries in registers (4,096 per query; the rest of a longer list is read again
// in every round), all loads of a list are in flight together, and the KP-th key is found by refining a range - a histogram of the
// keys in it over 1,024 bins, the bin that holds the KP-th, again with that bin - until the bin holds no more than a wave, which
// ranks it.  One round as a rule, six at most, since the keys (value, index) differ.
constexpr int TK_MINE = 16;
constexpr int TK_MAXAREAS = 1024;       // 2 nseg at most
constexpr int TK_BINS = 1024;
__global__ __launch_bounds__(256) void topk_compact_kernel(uint2 *keep, int32_t *keepcnt, const uint2 *seg, const int32_t *segcnt,
                                                           int nseg, int nsplit, int KP, float *thr, int32_t *flag, int Q) {
    __shared__ uint16_t place[TK_MINE * 256];               // the area (place in abase) of entry i
    __shared__ int hist[TK_BINS];
    __shared__ int abase[TK_MAXAREAS + 1];                  // start of every area's entries behind the kept list; area t + 256 j at 4 t + j
    __shared__ uint64_t few[64];
    __shared__ uint64_t found_lo, found_hi, cut_s;
    __shared__ uint32_t wlo[4], whi[4];
    __shared__ int wsum[4], total_s, over, few_n, found_need, found_count, out_n;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (q >= Q) return;
    const int kept = keep ? keepcnt[q] : 0;
    const int nareas = nsplit * 2;                          // <= 2 * nseg <= TK_MAXAREAS
    auto area_of = [](int p) { return (p >> 2) + 256 * (p & 3); };
    if (tid == 0) { over = 0; out_n = 0; few_n = 0; }
    __syncthreads();
    // counts (clamped to the area size) and their exclusive prefix sums behind the kept list: thread t takes the areas t + 256 j, a
    // shuffle scan inside every wave, the waves' sums through the LDS
    {
        int c[4], incl = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = tid + 256 * j < nareas ? segcnt[(size_t)q * nseg * 2 + tid + 256 * j] : 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (c[j] > TK_HALF) { over = 1; c[j] = TK_HALF; }
            incl += c[j];
        }
        const int own = incl;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o); if (lane >= o) incl += v; }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int start = kept + incl - own;
        for (int w = 0; w < wave; ++w) start += wsum[w];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            abase[4 * tid + j] = start;
            for (int e = 0; e < c[j]; ++e) if (start + e < TK_MINE * 256) place[start + e] = (uint16_t)(4 * tid + j);
            start += c[j];
        }
        if (tid == 255) { abase[TK_MAXAREAS] = start; total_s = start; }
    }
    __syncthreads();
    if (over && tid == 0) flag[q] = 1;                      // entries were dropped: exhaustive re-rank later
    const int total = total_s;
    const uint2 *areas = seg + (size_t)q * nseg * 2 * TK_HALF;
    uint64_t mine[TK_MINE];                                 // entries tid + 256 j
    {
        uint2 e[TK_MINE];
#pragma unroll
        for (int j = 0; j < TK_MINE; ++j) {
            e[j] = make_uint2(0u, 0u);
            if (j * 256 < total) {                          // (uniform)
                const int i = tid + j * 256;
                if (i < kept) e[j] = keep[(size_t)q * KP + i];
                else if (i < total) { const int p = place[i]; e[j] = areas[area_of(p) * TK_HALF + (i - abase[p])]; }
            }
        }
#pragma unroll
        for (int j = 0; j < TK_MINE; ++j) mine[j] = pack_value(e[j].x, e[j].y);
    }
    auto walk = [&](auto &&f) {                             // f(key) for every entry of the list
#pragma unroll
        for (int j = 0; j < TK_MINE; ++j) if (j * 256 < total && tid + j * 256 < total) f(mine[j]);
        for (int i = TK_MINE * 256 + tid; i < total; i += 256) {
            int p = 0;
            for (int step = TK_MAXAREAS / 2; step > 0; step >>= 1) if (abase[p + step] <= i) p += step;
            const uint2 e = areas[area_of(p) * TK_HALF + (i - abase[p])];
            f(pack_value(e.x, e.y));
        }
    };
    uint64_t cut = 0;                                       // keys >= cut stay
    if (total >= KP) {
        uint32_t mn = ~0u, mx = 0u;
        walk([&](uint64_t k) { const uint32_t v = (uint32_t)(k >> 32); mn = v < mn ? v : mn; mx = v > mx ? v : mx; });
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t x = __shfl_xor(mn, o), y = __shfl_xor(mx, o);
            mn = x < mn ? x : mn; mx = y > mx ? y : mx;
        }
        if (lane == 0) { wlo[wave] = mn; whi[wave] = mx; }
#pragma unroll
        for (int j = 0; j < TK_BINS / 256; ++j) hist[j * 256 + tid] = 0;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) { mn = wlo[w] < mn ? wlo[w] : mn; mx = whi[w] > mx ? whi[w] : mx; }
        uint64_t lo = (uint64_t)mn << 32, hi = (uint64_t)mx << 32 | 0xFFFFFFFFu;
        int need = KP, count = total;                       // taken from the top of [lo, hi]; entries in it
        while (count > 64 && hi > lo) {
            const uint64_t width = hi - lo;
            const int bits = width ? 64 - __clzll((long long)width) : 0, shift = bits > 10 ? bits - 10 : 0;
            walk([&](uint64_t k) { if (k >= lo && k <= hi) atomicAdd(&hist[(int)((k - lo) >> shift)], 1); });
            __syncthreads();
            // thread t holds four bins from the top; its first bin counts behind those of the threads before it
            const int b0 = TK_BINS - 1 - 4 * tid;
            int c[4], incl = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { c[j] = hist[b0 - j]; incl += c[j]; hist[b0 - j] = 0; }
            const int own = incl;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o); if (lane >= o) incl += v; }
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            int before = incl - own;
            for (int w = 0; w < wave; ++w) before += wsum[w];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (before < need && before + c[j] >= need) {      // (exactly one bin of all)
                    found_lo = lo + ((uint64_t)(b0 - j) << shift);
                    found_hi = found_lo + ((1ull << shift) - 1);
                    found_need = need - before;                    // taken from this bin
                    found_count = c[j];
                }
                before += c[j];
            }
            __syncthreads();
            lo = found_lo; hi = found_hi < hi ? found_hi : hi;
            need = found_need; count = found_count;
        }
        // (at most 64 entries left in [lo, hi]: a wave ranks them)
        walk([&](uint64_t k) { if (k >= lo && k <= hi) { const int i = atomicAdd(&few_n, 1); if (i < 64) few[i] = k; } });
        __syncthreads();
        if (wave == 0) {
            const uint64_t k = lane < count ? few[lane] : 0ull;
            int larger = 0;
            for (int i = 0; i < count; ++i) larger += few[i] > k;
            if (lane < count && larger == need - 1) cut_s = k;
        }
        __syncthreads();
        cut = cut_s;
        if (tid == 0) thr[q] = __uint_as_float(unpack_value(cut).x);
    }
    if (!keep) return;
    __syncthreads();                                        // (every entry of the kept list is in a register: its copy may be rewritten)
    walk([&](uint64_t k) { if (k >= cut) keep[(size_t)q * KP + atomicAdd(&out_n, 1)] = unpack_value(k); });
    if (tid == 0) keepcnt[q] = total < KP ? total : KP;
}

// ---------------------------------------------------------------------------------------------
// fp64 ranking key (smaller is better), defined on the exact query q (fp64 from the table values) and the tail row:
//   DistMult  q = h r,            key = -acc,  acc = fma(q_j, t_j, acc)
//   TransE    q = h + r,          key =  acc,  x = q_j - t_j, acc = fma(x, x, acc)
//   ComplEx   q = h * r (complex),  key = -acc,  acc = acc + (q_re t_re + q_im t_im) per complex coordinate
//   RotatE    q = h * e^{ir},       key =  acc,  acc = acc + (x_re^2 + x_im^2), x = q - t
//   TransH    u = w / max(|w|, 1e-12), q' = (h - (u.h) u) + r (both fp64, made once per query by the preparation
//             kernel), A = sum fma(u_j, t_j, .), key = acc, x = fma(A, u_j, q'_j - t_j), acc = fma(x, x, acc)
// every operation rounded on its own (no contraction), in this order: the same sequence of IEEE operations as
// the direct loops of Table 2 written in C give.  RotatE goes through cos / sin of the phase in fp64, whose last
// bit is the math library's.
// ---------------------------------------------------------------------------------------------
constexpr int TK_MAXD = 512;

__device__ __forceinline__ bool topk_mult(int scorer) { return scorer == KGE_DISTMULT || scorer == KGE_COMPLEX; }
__device__ __forceinline__ bool topk_cplx(int scorer) { return scorer == KGE_COMPLEX || scorer == KGE_ROTATE; }

// component j of the exact query (complex scorers: j < d/2 real parts, then imaginary parts)
template <bool BF16>
__device__ double query_f64(const KgeModelDev &m, int64_t hoff, int64_t roff, int j) {
    if (m.scorer == KGE_DISTMULT) return __dmul_rn((double)El<BF16>::ld(m.ent, hoff + j), (double)El<BF16>::ld(m.rel, roff + j));
    if (m.scorer == KGE_TRANSE) return __dadd_rn((double)El<BF16>::ld(m.ent, hoff + j), (double)El<BF16>::ld(m.rel, roff + j));
    const int c = m.dim >> 1, jr = j < c ? j : j - c;
    const double hre = (double)El<BF16>::ld(m.ent, hoff + jr), him = (double)El<BF16>::ld(m.ent, hoff + jr + c);
    double rre, rim;
    if (m.scorer == KGE_COMPLEX) { rre = (double)El<BF16>::ld(m.rel, roff + jr); rim = (double)El<BF16>::ld(m.rel, roff + jr + c); }
    else { const double ph = (double)El<BF16>::ld(m.rel, roff + jr); rre = cos(ph); rim = sin(ph); }
    return j < c ? __dsub_rn(__dmul_rn(hre, rre), __dmul_rn(him, rim)) : __dadd_rn(__dmul_rn(hre, rim), __dmul_rn(him, rre));
}

// one step of the key's accumulation: real scorers one column, complex scorers one complex coordinate
__device__ __forceinline__ double key_step(int scorer, double acc, double q0, double t0, double q1, double t1) {
    switch (scorer) {
    case KGE_DISTMULT: return fma(q0, t0, acc);
    case KGE_TRANSE: { const double x = __dsub_rn(q0, t0); return fma(x, x, acc); }
    case KGE_COMPLEX: return __dadd_rn(acc, __dadd_rn(__dmul_rn(q0, t0), __dmul_rn(q1, t1)));
    default: { const double xr = __dsub_rn(q0, t0), xi = __dsub_rn(q1, t1);
               return __dadd_rn(acc, __dadd_rn(__dmul_rn(xr, xr), __dmul_rn(xi, xi))); }
    }
}

// One walk over `steps` key steps of a row (whole 16-byte pieces: rows are, and so are their halves): the scorer is decided once
// per walk, since a branch per step costs as much as the step.  re(p) and im(p) are the pieces of the row behind step p 16 / ES
// (complex scorers: its real and imaginary parts), qv, qi and wv the query's components of these steps.  TransH walks twice: A = u . t,
// then the squared distance.
template <bool BF16, class Re, class Im>
__device__ __forceinline__ void key_walk(int scorer, bool second, int steps, const double *qv, const double *qi, const double *wv, Re &&re, Im &&im,
                                         double &A, double &acc) {
    constexpr int PER = BF16 ? 8 : 4;                   // columns of a piece
    auto elem = [](const kge_u32x4 &x, int e) -> double {
        if constexpr (BF16) return (double)__uint_as_float((e & 1) ? (x[e >> 1] & 0xffff0000u) : (x[e >> 1] << 16));
        else return (double)__uint_as_float(x[e]);
    };
    auto real = [&](auto &&step) {
        for (int p = 0; p * PER < steps; ++p) {
            const kge_u32x4 x = re(p);
#pragma unroll
            for (int e = 0; e < PER; ++e) step(qv[p * PER + e], elem(x, e), p * PER + e);
        }
    };
    auto complex_ = [&](auto &&step) {
        for (int p = 0; p * PER < steps; ++p) {
            const kge_u32x4 x = re(p), y = im(p);
#pragma unroll
            for (int e = 0; e < PER; ++e) step(qv[p * PER + e], elem(x, e), qi[p * PER + e], elem(y, e));
        }
    };
    switch (scorer) {
    case KGE_DISTMULT: real([&](double a, double t, int) { acc = key_step(KGE_DISTMULT, acc, a, t, 0.0, 0.0); }); break;
    case KGE_TRANSE: real([&](double a, double t, int) { acc = key_step(KGE_TRANSE, acc, a, t, 0.0, 0.0); }); break;
    case KGE_COMPLEX: complex_([&](double a, double t, double a2, double t2) { acc = key_step(KGE_COMPLEX, acc, a, t, a2, t2); }); break;
    case KGE_ROTATE: complex_([&](double a, double t, double a2, double t2) { acc = key_step(KGE_ROTATE, acc, a, t, a2, t2); }); break;
    default:
        if (!second) real([&](double, double t, int j) { A = fma(wv[j], t, A); });
        else real([&](double a, double t, int j) { const double z = fma(A, wv[j], __dsub_rn(a, t)); acc = fma(z, z, acc); });
    }
}

// key of one tail row against the exact query qv[0 .. d) (TransH: q', and the unit normal wv[0 .. d))
template <bool BF16>
__device__ double canonical_key(int scorer, int d, const double *qv, const double *wv, const void *ent, int64_t toff) {
    constexpr int ES = BF16 ? 2 : 4;
    const kge_u32x4 *row = (const kge_u32x4 *)((const char *)ent + toff * ES);
    const int half = d >> 1, imag = half * ES / 16;
    double A = 0.0, acc = 0.0;
    auto re = [&](int p) { return row[p]; };
    auto im = [&](int p) { return row[imag + p]; };
    key_walk<BF16>(scorer, false, topk_cplx(scorer) ? half : d, qv, qv + half, wv, re, im, A, acc);
    if (scorer == KGE_TRANSH) key_walk<BF16>(scorer, true, d, qv, qv + half, wv, re, im, A, acc);
    return topk_mult(scorer) ? -acc : acc;
}

template <bool BF16> constexpr int TK_ROW_STRIDE = 64 * (BF16 ? 2 : 4) + 16;
constexpr int TK_FINISH_LDS = 4096 + 1024 * 12 + 4 * 64 * TK_ROW_STRIDE<false>;    // the most that a call takes (K <= 256, rows <= 1,024 bytes)

struct QInfo { double qn; float eps_a, eps_b; float eps_w, c; };   // |q~|^2 (fp64), rounding-bound coefficients; TransH: |dw|, c

// Exhaustive fp64 re-rank of one query by its workgroup (lds: TK_EXACT_BYTES; qv, wv: its exact components).
constexpr int TK_CAPX = 2048;
constexpr int TK_EXACT_BYTES = TK_CAPX * 12;
template <bool BF16>
__device__ __forceinline__ void topk_exact(const KgeModelDev &m, int64_t cand_lo, int64_t ncand, int K, int32_t *out_idx, float *out_score,
                                           const int32_t *true_t, int tt, int64_t *out_rank, int q, const double *qv, const double *wv, char *lds) {
    double *key = (double *)lds;
    int *idx = (int *)(lds + TK_CAPX * 8);
    __shared__ int count;
    __shared__ double tau;
    __shared__ unsigned long long above;
    auto key_of = [&](int64_t toff) { return canonical_key<BF16>(m.scorer, m.dim, qv, wv, m.ent, toff); };
    if (threadIdx.x == 0) { count = 0; tau = INFINITY; above = 0ull; }
    for (int i = threadIdx.x; i < TK_CAPX; i += blockDim.x) { key[i] = INFINITY; idx[i] = 0x7FFFFFFF; }
    __syncthreads();
    double tkey = 0.0;
    if (true_t) { tkey = key_of((int64_t)tt * m.ent_ld); }
    unsigned long long mine = 0;
    for (int64_t c0 = 0; c0 < ncand; c0 += blockDim.x) {
        const int64_t c = c0 + threadIdx.x;
        if (c < ncand) {
            const double kc = key_of((cand_lo + c) * m.ent_ld);
            if (true_t && (kc < tkey || (kc == tkey && cand_lo + c < tt))) ++mine;
            if (kc <= tau) { const int s = atomicAdd(&count, 1); key[s] = kc; idx[s] = (int)c; }   // s < TK_CAPX by the compaction below
        }
        __syncthreads();
        // every thread reads the counter between two barriers, so that no wave can start the next round's appends before
        // a slower one has taken the same decision
        const bool compact = count > TK_CAPX - (int)blockDim.x;   // next round could overflow: compact to the K best
        __syncthreads();
        if (compact) {
            bitonic_asc_pair(key, idx, TK_CAPX);
            if (threadIdx.x == 0) { count = K; tau = key[K - 1]; }
            __syncthreads();
            for (int i = K + threadIdx.x; i < TK_CAPX; i += blockDim.x) { key[i] = INFINITY; idx[i] = 0x7FFFFFFF; }
            __syncthreads();
        }
    }
    bitonic_asc_pair(key, idx, TK_CAPX);
    const bool dm = topk_mult(m.scorer);
    for (int i = threadIdx.x; i < K; i += blockDim.x) {
        const bool ok = idx[i] != 0x7FFFFFFF;
        out_idx[(size_t)q * K + i] = ok ? (int32_t)(cand_lo + idx[i]) : -1;
        out_score[(size_t)q * K + i] = ok ? (dm ? (float)(-key[i]) : (float)(-sqrt(key[i]))) : -INFINITY;
    }
    if (true_t) {
        atomicAdd(&above, mine);
        __syncthreads();
        if (threadIdx.x == 0) out_rank[q] = 1 + (int64_t)above;
    }
}

// Re-scoring, final ordering, safety check and outputs: one query per workgroup.
//
// A wave re-scores 64 survivors at a time, lane = survivor, so that the 64 sequential fp64 chains run in lockstep.  The candidate
// rows arrive through the LDS in chunks of 64 columns (complex scorers: 32 real parts followed by the 32 imaginary parts of the same
// coordinates), 16 bytes per lane and load; the loads of the next chunk are in flight while a chunk is walked.  Rows are 16 bytes
// longer in the LDS than in memory: sixteen lanes' 16-byte pieces fall into different banks.  The key is the one of
// canonical_key, step by step, against the exact query, whose components are made once per workgroup.
template <bool BF16>
__global__ __launch_bounds__(256) void topk_finish_kernel(KgeModelDev m, const int32_t *h, const int32_t *r, int Q, int64_t cand_lo,
                                  int64_t ncand, const int32_t *cnt, const uint2 *buf, int KP, int KPP,
                                  const float *thr, const QInfo *qinfo, const float *tmax2,
                                  int K, int32_t *out_idx, float *out_score, const int32_t *true_t,
                                  const uint32_t *rankcnt, int64_t *out_rank, const int32_t *flag, const double *qx) {
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int PIECES = 64 * ES / 16;                // 16-byte pieces of a row's chunk
    constexpr int PER = 16 / ES;                        // columns of a piece
    constexpr int RPL = 64 / PIECES;                    // rows per wave-wide load
    constexpr int NL = 64 / RPL;                        // loads per chunk
    constexpr int STRIDE = TK_ROW_STRIDE<BF16>;         // bytes between rows in the LDS
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ int pos_s, flag_s;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (q >= Q) return;
    const int d = m.dim, half = d >> 1;
    const bool cplx = topk_cplx(m.scorer), th = m.scorer == KGE_TRANSH, dm = topk_mult(m.scorer);
    double *qv = (double *)lds, *wv = qv + d;                       // exact query; TransH: unit normal
    double *key = qv + (th ? 2 * d : d);
    int *idx = (int *)(key + KPP);
    char *rows = (char *)(idx + KPP);                   // [waves with survivors][64][STRIDE]
    const int n = cnt[q];
    const float theta = thr[q], tm2 = *tmax2;
    const QInfo qi = qinfo[q];
    const int64_t hoff = (int64_t)h[q] * m.ent_ld, roff = (int64_t)r[q] * m.rel_ld;
    const int tt = true_t ? true_t[q] : -1;
    if (tid == 0) { pos_s = -1; flag_s = flag[q]; }
    const int span = cplx ? 32 : 64, total = cplx ? half : d;       // key steps per chunk, in all
    const int nchunk = (total + span - 1) / span, walks = th ? 2 * nchunk : nchunk;    // (TransH: A = u . t first, then the distance)
    const int piece = lane % PIECES, lrow = lane / PIECES;
    char *mine = rows + wave * 64 * STRIDE;
    uint32_t own, cand[NL];
    kge_u32x4 v[NL];
    auto load = [&](int w) {
        const int at = (w < nchunk ? w : w - nchunk) * span + (cplx ? piece % (PIECES / 2) : piece) * PER;
        const int col = at + (cplx && piece >= PIECES / 2 ? half : 0);
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            v[u] = kge_u32x4{0u, 0u, 0u, 0u};
            if (at < total) v[u] = *(const kge_u32x4 *)((const char *)m.ent + ((cand_lo + cand[u]) * m.ent_ld + col) * ES);
        }
    };
    auto begin = [&](int s0) {
        own = buf[(size_t)q * KP + (s0 + lane < n ? s0 + lane : s0)].y;
#pragma unroll
        for (int u = 0; u < NL; ++u) cand[u] = __shfl(own, u * RPL + lrow);
        load(0);
    };
    if (wave * 64 < n) begin(wave * 64);
    for (int j = tid; j < d; j += 256) {                // (while the first rows are on their way)
        if (th) { qv[j] = qx[(size_t)q * 2 * d + j]; wv[j] = qx[(size_t)q * 2 * d + d + j]; }
        else qv[j] = query_f64<BF16>(m, hoff, roff, j);
    }
    for (int i = n + tid; i < KPP; i += 256) { key[i] = INFINITY; idx[i] = 0x7FFFFFFF; }
    __syncthreads();
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (int s0 = wave * 64; s0 < n; s0 += 256) {
        if (s0 > wave * 64) begin(s0);
        double acc = 0.0, A = 0.0;
        for (int w = 0; w < walks; ++w) {
#pragma unroll
            for (int u = 0; u < NL; ++u) *(kge_u32x4 *)(mine + (u * RPL + lrow) * STRIDE + piece * 16) = v[u];
            if (w + 1 < walks) load(w + 1);
            wave_fence();
            const int c0 = (w < nchunk ? w : w - nchunk) * span, steps = total - c0 < span ? total - c0 : span;
            const kge_u32x4 *row = (const kge_u32x4 *)(mine + lane * STRIDE);
            key_walk<BF16>(m.scorer, w >= nchunk, steps, qv + c0, qv + half + c0, wv + c0, [&](int p) { return row[p]; },
                           [&](int p) { return row[PIECES / 2 + p]; }, A, acc);
            wave_fence();
        }
        if (s0 + lane < n) { key[s0 + lane] = dm ? -acc : acc; idx[s0 + lane] = (int)own; }
    }
    __syncthreads();
    bitonic_asc_pair(key, idx, KPP);
    const int lim = K < n ? K : n;
    for (int i = tid; i < K; i += 256) {
        const bool ok = i < n;
        out_idx[(size_t)q * K + i] = ok ? (int32_t)(cand_lo + idx[i]) : -1;
        out_score[(size_t)q * K + i] = ok ? (dm ? (float)(-key[i]) : (float)(-sqrt(key[i]))) : -INFINITY;
        if (ok && true_t && cand_lo + idx[i] == tt) pos_s = i;      // (at most one)
    }
    if (tid == 0) {
        // Everything that was discarded has a matrix-core value <= theta (the KP-th best value, or the sample's).  Its
        // exact value is at most theta + eps; the list is safe if that stays strictly below the exact
        // value of the K-th entry.  eps bounds the rounding of the query to the table type and the
        // fp32 accumulation (units as topk_bound.hpp counts them):  DistMult (|dq| + units 2^-23 |q~|) Tmax;  TransE 2|dq|(|q~|+Tmax) +
        // |dq|^2 + units 2^-22 (|q~|+Tmax)^2, with Tmax the largest candidate norm; ComplEx and RotatE are the same two forms on
        // their own query (h * r, h * e^{ir}), whose fp32 evaluation error is part of dq.
        const bool cut = theta > -INFINITY && ncand > KP;
        // (the pieces of an infinite element make every sum a NaN, which is in no list)
        const bool no_sums = !BF16 && (qi.qn == INFINITY || (dm && tm2 == INFINITY));
        if (no_sums || (cut && K > n)) flag_s = 1;                   // (the sample's threshold, and not enough above it)
        else if (cut) {
            const double Tm = sqrt((double)tm2);
            double eps, exactK;
            if (dm) { eps = ((double)qi.eps_a + (double)qi.eps_b) * Tm; exactK = -key[K - 1]; }
            else if (m.scorer == KGE_TRANSH) {
                // value 2 q~.t - |t|^2 + (A~ - c)^2 against -key + |q~|^2 + c^2: the TransE terms for q~ (the
                // distance is taken to t_perp, no longer than t), then x = A - c: A~ is off by the rounding of the
                // normal to the table type (dw) and its fp32 accumulation, c (fp32 of u . q') by |dq| against u . q~.
                const double s = sqrt(qi.qn) + Tm, dq = qi.eps_a, dw = qi.eps_w, c = fabs((double)qi.c);
                const double wn = 1.0 + dw;                                            // |w~| <= |u| + |dw|
                const double dc = dq + 6e-8 * c;
                const double dx = (dw + (double)topk_product_units(m.dim, BF16) * 1.1920929e-07 * wn) * Tm + dc;
                const double xm = wn * Tm * 1.0001 + c;                                // |A~ - c| at most
                eps = 2.0 * dq * s + dq * dq + (double)qi.eps_b * s * s               // q~ for q', fp32 sums
                      + dx * (2.0 * xm + dx) + 4.8e-7 * (xm * xm + s * s)              // x~^2 for x^2, its fp32 evaluation
                      + dc * (2.0 * c + dc);                                           // c^2 for (u . q~)^2
                exactK = -key[K - 1] + qi.qn + (double)qi.c * (double)qi.c;
            } else {
                const double s = sqrt(qi.qn) + Tm;
                eps = 2.0 * qi.eps_a * s + (double)qi.eps_a * qi.eps_a + (double)qi.eps_b * s * s;
                exactK = -key[K - 1] + qi.qn;
            }
            eps = eps * 1.01 + 1e-30;
            if (!((double)theta + eps < exactK)) flag_s = 1;
        }
    }
    __syncthreads();
    if (flag_s) {                                       // (the same for every thread)
        topk_exact<BF16>(m, cand_lo, ncand, K, out_idx, out_score, true_t, tt, out_rank, q, qv, wv, rows);
        return;
    }
    if (tid == 0 && out_rank) {
        int64_t rank = 1 + (int64_t)rankcnt[q];
        if (pos_s >= 0) rank = pos_s + 1;                // exact: position in the fp64 ordering
        else if (tt >= cand_lo && tt < cand_lo + ncand && rank <= lim) rank = lim + 1;    // it is not in the exact list, so it ranks below it
        out_rank[q] = rank;
    }
}

// ---------------------------------------------------------------------------------------------
// preparation
// ---------------------------------------------------------------------------------------------
// (the launch of the queries also clears the running maximum of the norms and writes the zero bytes of padding columns)
__device__ __forceinline__ void topk_clear(uint32_t *tmax, uint32_t *zeros) {
    if (blockIdx.x == 0 && threadIdx.x < 64) { zeros[threadIdx.x] = 0u; if (threadIdx.x == 0) *tmax = 0u; }
}

// one wave per query: Q row in the table type, value of the held-out tail, rounding-bound coefficients
template <bool BF16>
__global__ void topk_prep_kernel(KgeModelDev m, const int32_t *h, const int32_t *r, const int32_t *true_t, int Q,
                                 int Qp, int dp, void *Qm, float *vt, QInfo *qinfo, float *thr, int32_t *cnt,
                                 int32_t *flag, uint32_t *rankcnt, uint32_t *tmax, uint32_t *zeros) {
    topk_clear(tmax, zeros);
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (q >= Qp) return;
    if (q >= Q) {
        for (int j = lane; j < dp; j += 64) El<BF16>::st(Qm, (int64_t)q * dp + j, 0.f);
        if (lane == 0) { vt[q] = INFINITY; thr[q] = INFINITY; cnt[q] = 0; flag[q] = 0; rankcnt[q] = 0; }
        return;
    }
    KgeRowCtx<BF16> cx;
    kge_build_query<BF16>(m, h[q], r[q], lane, cx);
    const int d = m.dim;
    const bool mult = topk_mult(m.scorer);
    const int64_t hoff = (int64_t)h[q] * m.ent_ld, roff = (int64_t)r[q] * m.rel_ld;
    double qn = 0.0, dq2 = 0.0;
    float vtl = 0.f, tnl = 0.f;
    const int64_t toff = true_t ? (int64_t)true_t[q] * m.ent_ld : 0;
#pragma unroll
    for (int k = 0; k < KGE_MAXJ; ++k) {
        const int j = lane + 64 * k;
        const float qr = El<BF16>::rnd(cx.q[k]);
        // (TransE: stored doubled - exact - so that the scan's contraction yields 2 q.t directly)
        if (j < dp) El<BF16>::st(Qm, (int64_t)q * dp + j, mult ? cx.q[k] : 2.f * cx.q[k]);
        if (j >= d) continue;
        const double dq = (double)qr - query_f64<BF16>(m, hoff, roff, j);     // against the exact query component
        qn += (double)qr * (double)qr; dq2 += dq * dq;
        if (true_t) { const float tv = El<BF16>::ld(m.ent, toff + j); vtl += qr * tv; tnl += tv * tv; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        qn += __shfl_xor(qn, o); dq2 += __shfl_xor(dq2, o); vtl += __shfl_xor(vtl, o); tnl += __shfl_xor(tnl, o);
    }
    if (lane == 0) {
        QInfo qi;
        qi.qn = qn;
        qi.eps_a = (float)(sqrt(dq2) * 1.0001);
        qi.eps_b = mult ? (float)(topk_product_units(d, BF16) * 1.1920929e-07 * sqrt(qn) * 1.0001)
                                            : (float)(topk_distance_units(d, BF16) * 2.3841858e-07);
        qi.eps_w = 0.f; qi.c = 0.f;
        qinfo[q] = qi;
        vt[q] = true_t ? (mult ? vtl : 2.f * vtl - tnl) : INFINITY;
        thr[q] = -INFINITY; cnt[q] = 0; flag[q] = 0; rankcnt[q] = 0;
    }
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// TransH, one wave per query: unit normal u and q' = (h - (u.h) u) + r in fp64 (kept for the re-scoring), their
// roundings to the table type (q~ stored doubled, like TransE's), c = u . q', the value of the held-out tail
// and the rounding-bound coefficients.
template <bool BF16>
__global__ void topk_prep_th_kernel(KgeModelDev m, const int32_t *h, const int32_t *r, const int32_t *true_t, int Q,
                                    int Qp, int dp, void *Qm, void *Wm, float *cq, double *qx, float *vt, QInfo *qinfo,
                                    float *thr, int32_t *cnt, int32_t *flag, uint32_t *rankcnt, uint32_t *tmax, uint32_t *zeros) {
    topk_clear(tmax, zeros);
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (q >= Qp) return;
    if (q >= Q) {
        for (int j = lane; j < dp; j += 64) { El<BF16>::st(Qm, (int64_t)q * dp + j, 0.f); El<BF16>::st(Wm, (int64_t)q * dp + j, 0.f); }
        if (lane == 0) { cq[q] = 0.f; vt[q] = INFINITY; thr[q] = INFINITY; cnt[q] = 0; flag[q] = 0; rankcnt[q] = 0; }
        return;
    }
    const int d = m.dim;
    const int64_t hoff = (int64_t)h[q] * m.ent_ld, roff = (int64_t)r[q] * m.rel_ld, woff = (int64_t)r[q] * m.relw_ld;
    double hv[KGE_MAXJ], rv[KGE_MAXJ], wv[KGE_MAXJ];
    double nn = 0.0;
#pragma unroll
    for (int k = 0; k < KGE_MAXJ; ++k) {
        const int j = lane + 64 * k;
        const bool ok = j < d;
        hv[k] = ok ? (double)El<BF16>::ld(m.ent, hoff + j) : 0.0;
        rv[k] = ok ? (double)El<BF16>::ld(m.rel, roff + j) : 0.0;
        wv[k] = ok ? (double)El<BF16>::ld(m.relw, woff + j) : 0.0;
        nn += wv[k] * wv[k];
    }
    nn = wave_sum_f64(nn);
    const double nrm = fmax(sqrt(nn), 1e-12);
    double wh = 0.0;
#pragma unroll
    for (int k = 0; k < KGE_MAXJ; ++k) { wv[k] = wv[k] / nrm; wh += wv[k] * hv[k]; }
    wh = wave_sum_f64(wh);
    double ce = 0.0, qn = 0.0, dq2 = 0.0, dw2 = 0.0;
    float qt = 0.f, tnl = 0.f, wt = 0.f;
    const int64_t toff = true_t ? (int64_t)true_t[q] * m.ent_ld : 0;
    double *qxq = qx + (size_t)q * 2 * d;
#pragma unroll
    for (int k = 0; k < KGE_MAXJ; ++k) {
        const int j = lane + 64 * k;
        const double qe = (hv[k] - wh * wv[k]) + rv[k];
        const float qr = El<BF16>::rnd((float)qe), wr = El<BF16>::rnd((float)wv[k]);
        if (j < dp) { El<BF16>::st(Qm, (int64_t)q * dp + j, 2.f * qr); El<BF16>::st(Wm, (int64_t)q * dp + j, wr); }
        if (j >= d) continue;
        qxq[j] = qe; qxq[d + j] = wv[k];
        ce += wv[k] * qe; qn += (double)qr * (double)qr;
        dq2 += ((double)qr - qe) * ((double)qr - qe); dw2 += ((double)wr - wv[k]) * ((double)wr - wv[k]);
        if (true_t) { const float tv = El<BF16>::ld(m.ent, toff + j); qt += qr * tv; tnl += tv * tv; wt += wr * tv; }
    }
    ce = wave_sum_f64(ce); qn = wave_sum_f64(qn); dq2 = wave_sum_f64(dq2); dw2 = wave_sum_f64(dw2);
    qt = kge_wave_sum(qt); tnl = kge_wave_sum(tnl); wt = kge_wave_sum(wt);
    if (lane == 0) {
        const float c = (float)ce;
        QInfo qi;
        qi.qn = qn;
        qi.eps_a = (float)(sqrt(dq2) * 1.0001);
        qi.eps_b = (float)(topk_distance_units(d, BF16) * 2.3841858e-07);
        qi.eps_w = (float)(sqrt(dw2) * 1.0001);
        qi.c = c;
        qinfo[q] = qi;
        cq[q] = c;
        vt[q] = true_t ? fmaf(wt - c, wt - c, 2.f * qt - tnl) : INFINITY;
        thr[q] = -INFINITY; cnt[q] = 0; flag[q] = 0; rankcnt[q] = 0;
    }
}

// squared norms of the candidate rows (stored negated: the scan starts its accumulators from them) and their maximum.  A lane
// reads 16 bytes (rows are multiples of 16 bytes and aligned to them), a wave 64 / LPR rows per step, four steps in flight.
__global__ __launch_bounds__(256) void topk_tnorm_kernel(const char *ent, int64_t stride, int d, int64_t ncand, int64_t npad, float *tn,
                                  uint32_t *tmax_bits) {
    __shared__ float wmax[4];
    const int lane = threadIdx.x & 63;
    const int64_t wid = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * 4;
    float mx = 0.f;
    const int chunks = d * 2 / 16;                                  // 16-byte chunks of a row
    const int lpr = chunks <= 1 ? 1 : 1 << (32 - __clz(chunks - 1)); // lanes per row
    const int rpw = 64 / lpr, sub = lane / lpr, li = lane % lpr;    // rows per wave step
    constexpr int U = 4;
    for (int64_t c0 = wid * rpw * U; c0 < npad; c0 += nw * rpw * U) {
        kge_u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = c0 + u * rpw + sub;
            v[u] = kge_u32x4{0u, 0u, 0u, 0u};
            if (c < ncand && li < chunks) v[u] = *(const kge_u32x4 *)(ent + c * stride + li * 16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float a0 = __uint_as_float(v[u][k] << 16), a1 = __uint_as_float(v[u][k] & 0xffff0000u);
                s += a0 * a0; s += a1 * a1;
            }
            for (int o = lpr >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o);
            const int64_t c = c0 + u * rpw + sub;
            if (li == 0 && c < npad) tn[c] = -s;
            mx = fmaxf(mx, s);
        }
    }
    mx = kge_wave_max(mx);
    if (lane == 0) wmax[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) topk_raise(tmax_bits, fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])));
}

__global__ void topk_fill_empty_kernel(int32_t *out_idx, float *out_score, int64_t n, int64_t *out_rank, int Q) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) { out_idx[i] = -1; out_score[i] = -INFINITY; }
    if (out_rank && i < Q) out_rank[i] = 1;
}

struct TopkPlan {
    bool bf16, th, fn; int es, rb, dp, ob, own, dim; int Qp; int KP, KPP, nseg; int64_t npad;
};

TopkPlan make_plan(const kge_model_t &m, int64_t Q, int64_t ncand, int K) {
    TopkPlan p{};
    p.bf16 = m.dtype == KGE_BF16; p.es = p.bf16 ? 2 : 4;
    p.rb = m.dim * p.es <= 512 ? 512 : 1024; p.dp = p.rb / p.es;
    p.th = m.scorer == KGE_TRANSH; p.dim = m.dim;
    // Two blocks of 32 queries per wave where the registers allow it (TransH: the second block holds the normals), so that an
    // LDS fragment feeds two MFMAs.  Up to 512 queries one block: the scan is then bound by the table's bytes and by a round's
    // latency, tiles of 128 queries pad less, and the registers have room for the norms (TransE, d 256, 2M candidates, one block
    // against two: 730 / 893 us for 256 queries, 1,059 / 1,218 for 512, 1,850 / 1,781 for 1,024).
    p.ob = p.rb == 512 && (p.th || Q > 512) ? 2 : 1; p.own = p.th ? 128 : 128 * p.ob;
    p.Qp = (int)kge_round_up(Q, p.own);
    p.KP = (int)kge_round_up(2 * K + 56, 64);
    p.KPP = 1; while (p.KPP < p.KP) p.KPP <<= 1;
    // Splits of the candidates, each with its append areas.  Two workgroups per compute unit, so that the copies of one run beside the
    // epilogue of the other: 512 splits for one query tile on rows of 512 bytes (TransH, 128 queries, 5M candidates: 979 us, 256 splits
    // 1,253), 256 for two (TransE, 256 queries, 1M: 456; 512 splits 525) and on wider rows: bf16, whose ring of stages leaves one workgroup
    // the LDS of a compute unit (d 512, 128 queries, 1M: 550 / 595), and fp32, where two would fit and 512 splits are faster on large tables
    // and slower on small ones (d 256, 256 / 512 splits: 128 queries x 4M 1,420 / 1,189, 1M 439 / 404, 300,000 193 / 194, 64 x 60,000
    // 111 / 119, 30 x 25,000 92 / 105), but whose areas would take twice the workspace; about four turns of the 256 compute units above.
    const int tiles = p.Qp > 0 ? p.Qp / p.own : 1;
    { int w = 1024 / tiles; p.nseg = w < 32 ? 32 : tiles == 1 && p.rb == 512 ? 512 : (w > 256 ? 256 : w); }
    // Norms inside the scan (FN) or in a pass of their own.  Bilinear: always inside (one query tile's turn per candidate tile:
    // 9.66 against 10.0 ms for 8,192 queries over 2M rows, 0.64 against 0.92 for 256).  Distance: every query tile makes them
    // again, so inside while there are few - up to 24 for TransH (1M rows, 8 / 16 tiles: 1.41 / 2.57 inside, 1.62 / 2.72 ms
    // outside), up to 4 for rows over 512 bytes (4 / 8 / 16 tiles: 1.55 / 2.62 / 4.94 against 1.87 / 2.52 / 4.43); with two
    // blocks of queries per wave never (the kernel spills 40 registers: 892 against 943 us for one tile, 1,477 against 1,244 for two).
    // fp32 rows: inside, by the walk that makes their pieces.
    p.fn = !p.bf16 || (m.scorer == KGE_DISTMULT || m.scorer == KGE_COMPLEX) || (p.th ? tiles <= 24 : p.rb == 1024 ? tiles <= 4 : p.ob == 1);
    p.npad = kge_round_up(ncand > 0 ? ncand : 1, TK_ST);
    return p;
}

// Size of the sample and growth of the chunks.  What is weighed (seconds, measured): scanning a row for all queries - 0.1 ns while
// the table's bytes bound it, 0.37 ps per query and 512 bytes beyond (fp32 rows 1.1 to 1.4: a factor of 3.5); a stage - threshold, launches and their latencies, 26 us +
// 5.4 ns per query; an append, 40 ps.  A sample of S rows costs S rows, a stage that multiplies what the threshold stands for by g
// costs itself and KP (g - 1) appends per query, so with ln(n / S) / ln(g) stages the best g depends on stage / appends alone (2.6 for 8,192
// queries, 12 for 128) and the best S is where a row more saves as much of a stage.  g keeps a query's expected appends within what
// a workgroup of the compaction holds in registers and 24 per area (of 64: an overflow would rank the query exhaustively).
struct TopkStages { int64_t sample; double growth; };
TopkStages topk_stages(const TopkPlan &p, int64_t Q, int64_t total_tiles) {
    const double width = (p.rb == 512 ? 1.0 : 2.0) * (p.th ? 2.0 : 1.0) * (p.bf16 ? 1.0 : 3.5);
    const double row = fmax(0.1e-9 * p.rb / 512, 0.37e-12 * (double)Q * width), stage = 26e-6 + 5.4e-9 * (double)Q;
    const double appends = 40e-12 * (double)Q * p.KP;
    const double most = fmin(3500.0, 24.0 * 2.0 * p.nseg) / (1.15 * p.KP);
    double g = fmin(2.1 + 0.5 * stage / appends, most);
    if (g < 1.5) g = 1.5;
    TopkStages s;
    s.sample = (int64_t)((stage + appends * (g - 1.0)) / log(g) / (1.2 * row) / TK_ST);
    if (s.sample > total_tiles / 2) s.sample = total_tiles / 2;
    if (s.sample < 128) s.sample = 128 < total_tiles - 1 ? 128 : total_tiles - 1;      // (whole tiles of candidates)
    const double all = (double)total_tiles / (double)s.sample;
    double stages = ceil(log(all) / log(g) - 0.25);
    if (stages < 1.0) stages = 1.0;
    s.growth = pow(all, 1.0 / stages);
    if (s.growth > most && most >= 1.5) s.growth = pow(all, 1.0 / (stages + 1.0));
    return s;
}

// A stride of the walk over n places that are visited at p stride mod n: coprime with n, about 0.618 n, so that the visits of any stretch
// of the walk lie at most a few times their mean distance apart, and with partial quotients of stride / n as small as a few tries find
// (a large one would bring every q-th visit, q small, back to the same neighbourhood).
int32_t topk_stride(int64_t n) {
    if (n < 3) return n == 2 ? 1 : 0;
    int64_t best = 1, best_q = INT64_MAX;
    int64_t s = (int64_t)((double)n * 0.6180339887498949);
    for (int tries = 0; tries < 8; ++s) {
        if (s >= n) break;
        int64_t a = n, b = s, most = 0;
        while (b) {                                           // Euclid; the first and the last quotients say nothing
            const int64_t q = a / b, r = a - q * b;
            if (r && q > most) most = q;
            a = b; b = r;
        }
        if (a != 1) continue;
        if (most < best_q) { best = s; best_q = most; }
        if (best_q <= 8) break;
        ++tries;
    }
    return (int32_t)best;
}

struct TopkWs {
    void *Qm; float *vt, *thr, *tn; QInfo *qinfo; int32_t *cnt, *flag; uint32_t *rankcnt, *tmax; uint2 *keep, *seg; int32_t *segcnt; uint32_t *zeros;
    void *Wm; float *cq; double *qx;                    // TransH only
};

// most: sizes that no smaller call exceeds (fewer queries can take more areas in all: 1,024 / tiles is rounded down)
size_t topk_carve(const TopkPlan &p, void *ws, TopkWs &w, bool most = false) {
    char *b = (char *)ws; size_t off = 0;
    auto take = [&](size_t bytes) { void *q = b ? b + off : nullptr; off += (bytes + 255) / 256 * 256; return q; };
    w.Qm = take((size_t)p.Qp * p.rb);
    w.vt = (float *)take((size_t)p.Qp * 4); w.thr = (float *)take((size_t)p.Qp * 4);
    w.qinfo = (QInfo *)take((size_t)p.Qp * sizeof(QInfo));
    w.cnt = (int32_t *)take((size_t)p.Qp * 4); w.flag = (int32_t *)take((size_t)p.Qp * 4);
    w.rankcnt = (uint32_t *)take((size_t)p.Qp * 4); w.tmax = (uint32_t *)take(256); w.zeros = (uint32_t *)take(256);
    w.tn = p.fn ? nullptr : (float *)take((size_t)p.npad * 4);
    w.keep = (uint2 *)take((size_t)p.Qp * p.KP * 8);
    size_t areas = (size_t)p.Qp * p.nseg * 2;
    if (most && p.Qp / p.own > 4 && areas < (size_t)p.own * 1024 * 2) areas = (size_t)p.own * 1024 * 2;
    w.seg = (uint2 *)take(areas * TK_HALF * 8);
    w.segcnt = (int32_t *)take(areas * 4);
    w.Wm = nullptr; w.cq = nullptr; w.qx = nullptr;
    if (p.th) {
        w.Wm = take((size_t)p.Qp * p.rb); w.cq = (float *)take((size_t)p.Qp * 4);
        w.qx = (double *)take((size_t)p.Qp * 2 * p.dim * 8);
    }
    return off + 256;
}

template <bool BF16, int RB, int KIND, int OB, bool TH, bool FN, bool SAMPLE>
int launch_scan(const TopkArgs &a, hipStream_t st) {
    constexpr int NSTAGE = tk_stages(BF16, RB);
    constexpr int LDS = NSTAGE * TK_ST * RB + (NSTAGE + 1) * 4 * 256;
    static KgeLdsLimit lds_limit;
    if (lds_limit.set((const void *)topk_scan_kernel<BF16, RB, KIND, OB, TH, FN, SAMPLE>, LDS) != KGE_OK) return KGE_E_HIP;
    hipLaunchKernelGGL((topk_scan_kernel<BF16, RB, KIND, OB, TH, FN, SAMPLE>), dim3(a.own_tiles * ((a.nsplit + 7) / 8 * 8)), dim3(256), LDS, st, a);
    return kge_launch_status();
}

template <bool BF16, bool SAMPLE>
int scan(const TopkPlan &p, int kind, const TopkArgs &a, hipStream_t st) {
    if (kind == KGE_KIND_MULT) {
        if (p.rb == 1024) return launch_scan<BF16, 1024, KGE_KIND_MULT, 1, false, true, SAMPLE>(a, st);
        return p.ob == 1 ? launch_scan<BF16, 512, KGE_KIND_MULT, 1, false, true, SAMPLE>(a, st)
                         : launch_scan<BF16, 512, KGE_KIND_MULT, 2, false, true, SAMPLE>(a, st);
    }
    if constexpr (BF16) if (!p.fn) {
        if (p.th) return launch_scan<true, 512, KGE_KIND_DIST, 2, true, false, SAMPLE>(a, st);
        if (p.rb == 1024) return launch_scan<true, 1024, KGE_KIND_DIST, 1, false, false, SAMPLE>(a, st);
        return launch_scan<true, 512, KGE_KIND_DIST, 2, false, false, SAMPLE>(a, st);
    }
    if (p.th) return launch_scan<BF16, 512, KGE_KIND_DIST, 2, true, true, SAMPLE>(a, st);
    if (p.rb == 1024) return launch_scan<BF16, 1024, KGE_KIND_DIST, 1, false, true, SAMPLE>(a, st);
    if constexpr (!BF16) if (p.ob == 2) return launch_scan<false, 512, KGE_KIND_DIST, 2, false, true, SAMPLE>(a, st);
    return launch_scan<BF16, 512, KGE_KIND_DIST, 1, false, true, SAMPLE>(a, st);
}

}  // namespace

size_t kge_topk_ws(const kge_model_t &model, int64_t Q, int64_t ncand, int K, bool most) {
    if (Q < 0 || ncand < 0 || K < 1 || K > 256) return 0;
    TopkPlan p = make_plan(model, Q, ncand, K);
    TopkWs w;
    return topk_carve(p, nullptr, w, most);
}

int kge_run_topk(const kge_model_t &model, const int32_t *h, const int32_t *r, int64_t Q, int64_t lo, int64_t hi,
                 int K, int32_t *out_idx, float *out_score, const int32_t *true_t, int64_t *out_rank, void *ws,
                 size_t ws_bytes, hipStream_t st) {
    (void)ws_bytes;
    const int64_t ncand = hi - lo;
    if (ncand == 0) {
        const int64_t n = Q * K;
        hipLaunchKernelGGL(topk_fill_empty_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, out_idx, out_score, n,
                           out_rank, (int)Q);
        return kge_launch_status();
    }
    const TopkPlan p = make_plan(model, Q, ncand, K);
    TopkWs w;
    topk_carve(p, ws, w);
    KgeModelDev md;
    md.scorer = model.scorer; md.bf16 = p.bf16; md.dim = model.dim; md.rel_dim = model.rel_dim; md.p1 = 0;
    md.ent = model.ent; md.rel = model.rel; md.relw = model.relw;
    md.ent_ld = model.ent_ld; md.rel_ld = model.rel_ld; md.relw_ld = model.relw_ld;
    const char *cand0 = (const char *)model.ent + lo * model.ent_ld * p.es;
    const int64_t stride = model.ent_ld * p.es;
    if (stride * TK_ST >= (1ll << 32)) return KGE_E_UNSUPPORTED;     // the scan advances its sources by a 32-bit step per tile
    const int kind = (model.scorer == KGE_DISTMULT || model.scorer == KGE_COMPLEX) ? KGE_KIND_MULT : KGE_KIND_DIST;

    if (p.th) {
        if (p.bf16) hipLaunchKernelGGL(topk_prep_th_kernel<true>, dim3((p.Qp + 3) / 4), dim3(256), 0, st, md, h, r, true_t, (int)Q, p.Qp, p.dp, w.Qm, w.Wm, w.cq, w.qx, w.vt, w.qinfo, w.thr, w.cnt, w.flag, w.rankcnt, w.tmax, w.zeros);
        else hipLaunchKernelGGL(topk_prep_th_kernel<false>, dim3((p.Qp + 3) / 4), dim3(256), 0, st, md, h, r, true_t, (int)Q, p.Qp, p.dp, w.Qm, w.Wm, w.cq, w.qx, w.vt, w.qinfo, w.thr, w.cnt, w.flag, w.rankcnt, w.tmax, w.zeros);
    }
    if (p.bf16) {
        if (!p.th) hipLaunchKernelGGL(topk_prep_kernel<true>, dim3((p.Qp + 3) / 4), dim3(256), 0, st, md, h, r, true_t, (int)Q, p.Qp, p.dp, w.Qm, w.vt, w.qinfo, w.thr, w.cnt, w.flag, w.rankcnt, w.tmax, w.zeros);
        if (!p.fn) hipLaunchKernelGGL(topk_tnorm_kernel, dim3((unsigned)(p.npad / 32 < 2048 ? p.npad / 32 : 2048)), dim3(256), 0, st, cand0, stride, model.dim, ncand, p.npad, w.tn, w.tmax);
    } else {
        if (!p.th) hipLaunchKernelGGL(topk_prep_kernel<false>, dim3((p.Qp + 3) / 4), dim3(256), 0, st, md, h, r, true_t, (int)Q, p.Qp, p.dp, w.Qm, w.vt, w.qinfo, w.thr, w.cnt, w.flag, w.rankcnt, w.tmax, w.zeros);
    }
    if (hipGetLastError() != hipSuccess) return KGE_E_HIP;

    TopkArgs base{};
    base.Qmat = w.Qm; base.Wmat = w.Wm; base.cq = w.cq; base.ent = cand0; base.ent_stride = stride; base.valid_bytes = model.dim * p.es;
    base.ncand = ncand; base.tn = w.tn; base.tmax = w.tmax; base.thr = w.thr; base.vt = w.vt; base.true_t = true_t;
    base.seg = w.seg; base.segcnt = w.segcnt; base.nseg = p.nseg; base.rankcnt = w.rankcnt; base.nq = (int)Q; base.zeros = w.zeros;
    const int own_tiles = p.Qp / p.own;
    const int64_t total_tiles = p.npad / TK_ST;
    // One chunk appends everything where it fits: at most 128 tiles and two per split, so that an area (one lane half: TK_ST / 2
    // candidates of a tile) takes 32 entries and a query 4,096.  Longer tables are sampled first (SAMPLE in the kernel); the scan then
    // goes by chunks between which the thresholds are refreshed: the first covers g times the rows of the sample, the next g times
    // that.
    constexpr int FIRST_TILES = 2;
    static_assert(FIRST_TILES * TK_ST / 2 <= TK_HALF, "the first chunk overflows no area");
    auto compact = [&](uint2 *keep, int nsplit) {
        const int areas_of = (nsplit + 7) / 8 * 8 < p.nseg ? (nsplit + 7) / 8 * 8 : p.nseg;
        hipLaunchKernelGGL(topk_compact_kernel, dim3((unsigned)Q), dim3(256), 0, st, keep, w.cnt, w.seg, w.segcnt, p.nseg, areas_of, p.KP,
                           w.thr, w.flag, (int)Q);
    };
    double reach = (double)total_tiles, growth = 1.0;
    int64_t walk = total_tiles, stride_t = 1;
    int most_splits = p.nseg;                                 // one split per private area
    if (total_tiles > (p.nseg * FIRST_TILES < 128 ? p.nseg * FIRST_TILES : 128)) {
        const TopkStages s = topk_stages(p, Q, total_tiles);
        growth = s.growth; reach = s.sample * s.growth;
        // In order of the ids where the areas have room for all rows of the table that beat the first threshold, about KP / sample of
        // them, wherever they lie (from 512 queries down as a rule: pages are walked one after the other, 128 queries x 5.7M 660 us against
        // 681 in strides); otherwise in strides, over a number of positions that has no small factor.  Neither is dealt to the splits in the
        // period of a table that repeats every 2^k tiles: the splits are odd in number, or the strides turn over an odd one.  (An odd number costs: 303
        // queries x 213,340, d 256 68.3 us of scan with 255 splits, 65.7 with 256; 67 to 69 with 256 dealt with a skew from turn to turn.)
        if ((double)p.KP * total_tiles <= 24.0 * 2.0 * p.nseg * s.sample) most_splits -= most_splits % 2 == 0;
        else {
            while (walk % 2 == 0 || walk % 3 == 0 || walk % 5 == 0 || walk % 7 == 0) ++walk;
            stride_t = topk_stride(walk);
        }
        TopkArgs c = base;
        c.tile_lo = 0; c.tile_hi = (int32_t)s.sample; c.own_tiles = own_tiles;
        c.nsplit = s.sample < p.nseg ? (int)s.sample : p.nseg;
        c.samp = topk_sample(ncand, s.sample);                // (TK_ST sample <= ncand)
        // about 1,000 to 2,500 groups of a query in all, at most 64 of a split and lane half
        c.fold = c.nsplit * 8 > 2500;
        const int64_t per = (s.sample + c.nsplit - 1) / c.nsplit, each = c.fold ? 2 : 8;      // tiles of a split; groups of a split and flush
        c.flush = (int)((per * c.nsplit * each + 2047) / 2048);
        const int64_t least = (per * each / 2 + TK_HALF - 1) / TK_HALF;
        if (c.flush < least) c.flush = (int)least;
        const int rc = p.bf16 ? scan<true, true>(p, kind, c, st) : scan<false, true>(p, kind, c, st);
        if (rc != KGE_OK) return rc;
        compact(nullptr, c.nsplit);
    }
    for (int64_t seen = 0; seen < walk; reach *= growth) {
        int64_t upto = (int64_t)(reach * 1.01);               // (no chunk of a few tiles at the end)
        if (upto >= total_tiles || upto <= seen) upto = walk;
        TopkArgs c = base;
        c.tile_lo = (int32_t)seen; c.tile_hi = (int32_t)upto; c.own_tiles = own_tiles;
        c.nsplit = upto - seen < most_splits ? (int)(upto - seen) : most_splits;
        c.walk = (int32_t)walk; c.tiles = (int32_t)total_tiles; c.stride = (int32_t)stride_t; c.ratio = (double)stride_t / (double)walk;
        c.start = (int32_t)(seen * stride_t % walk); c.step = (int32_t)(c.nsplit * stride_t % walk);
        int rc;
        {
            KgeProfScope prof(KGE_PROF_TOPK_SCAN, st);
            rc = p.bf16 ? scan<true, false>(p, kind, c, st) : scan<false, false>(p, kind, c, st);
        }
        if (rc != KGE_OK) return rc;
        seen = upto;
        compact(w.keep, c.nsplit);
    }
    const int groups = p.KP / 64 < 4 ? p.KP / 64 : 4, row_bytes = groups * 64 * (p.bf16 ? TK_ROW_STRIDE<true> : TK_ROW_STRIDE<false>);
    const int finish_lds = p.dim * (p.th ? 16 : 8) + p.KPP * 12 + (row_bytes > TK_EXACT_BYTES ? row_bytes : TK_EXACT_BYTES);
    auto finish = [&](auto kernel, KgeLdsLimit &limit) {
        if (limit.set((const void *)kernel, TK_FINISH_LDS) != KGE_OK) return (int)KGE_E_HIP;
        hipLaunchKernelGGL(kernel, dim3((unsigned)Q), dim3(256), finish_lds, st, md, h, r, (int)Q, lo, ncand, w.cnt, w.keep, p.KP, p.KPP, w.thr,
                           w.qinfo, (const float *)w.tmax, K, out_idx, out_score, true_t, w.rankcnt, out_rank, w.flag, w.qx);
        return kge_launch_status();
    };
    static KgeLdsLimit limit_bf16, limit_f32;
    return p.bf16 ? finish(topk_finish_kernel<true>, limit_bf16) : finish(topk_finish_kernel<false>, limit_f32);
}
