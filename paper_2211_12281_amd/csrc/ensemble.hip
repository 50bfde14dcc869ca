// Power-rank ensemble of M top-K lists per query (Section 3.2 "Inference", paragraph "Ensemble", eq. (ensemble)):
// s(t) = sum over the models, in model order, of -sgn(p) k^p where t is the k-th entry of the model's list and of
// -[p > 0] (K + 1)^p where the list does not hold t; the K_out entities with the largest s(t) are returned, ties
// to the smaller id.  An entity in no list has the smallest possible score, so only listed entities compete.
// The K + 1 possible terms come from the host as a kernel argument, so they are the host math library's powers.
//
// ens_top_kernel, one wave per query.  An entity that no list holds among its first r ranks scores at most M times the term of
// rank r + 1 (floating-point addition is monotone, so the sum of M such terms in model order bounds its sum as rounded), and r
// of the size of K_out leaves a few dozen entities that can win:
//   1. the entities of the first r ranks, rank by rank, go into a small hash table in the LDS (buckets of four slots, one 16-byte
//      read per probe) and are numbered as they come; a table that fills up ends the walk at a smaller r
//   2. every entry of every list is looked up; those found leave their rank in a byte of their own per (model, candidate)
//   3. a lane sums its candidates' terms in model order, in registers
//   4. the K_out best: a threshold on the high words of the sums by bisection with ballots, then ranks by counting
//   5. if the K_out-th best does not exceed the bound (or the table held too few) the query is left to ens_kernel, flagged in its
//      output; with r = K nothing is left out and there is nothing to check.
// What bounds it is instruction issue (vector and scalar about alike: 1,500 and 1,500 for a query of 16 lists of 100, half of the
// vector ones in the look-ups); no wave waits for another, and 32 queries share a compute unit.  16 lists of 100, ten winners of
// 8,192 queries: 94 us with ens_kernel -> 35 (p = 1: 204 -> 40; 100 winners 301 -> 177; 64 lists, 4,096 queries 613 -> 113).
// Look-ups whose loads and stores were predicated entry by entry took 51 us, a ring of 16 requests 39, of 8 35.4.
//
// ens_kernel, one workgroup of four waves per query, for what the other kernel can't hold (many winners, ranks beyond a byte) or
// could not prove:
//   1. the entries' entities go into a hash table in the LDS (linear probing); wave w takes the lists of models w, w + 4, ..,
//      so that an entity that a list holds twice is found inside one wave, and notes every entry's slot
//   2. one wave walks the models in order and adds every entry's term to its slot's fp64 sum: a wave's LDS accesses happen in
//      the order it issues them, so the sums are in model order without a barrier per model
//   3. the K_out winners: a lower bound of the K_out-th best from the best of every bin of slots, then the few entries that
//      reach it are ranked by counting
// What bounds it is the latency of the LDS chains of a query, so what counts is the number of workgroups on a compute unit (12
// bytes of LDS per slot: five at M K = 1,600).
#include "kge_internal.h"
#include <math.h>
#include <type_traits>

int kge_run_ensemble(const int32_t *lists, int M, int64_t Q, int K, double p, int K_out, int32_t *out_idx, float *out_score,
                     hipStream_t st);

namespace {

constexpr int ENS_CU_LDS = 163840;
constexpr int ENS_MAX_K = 256, ENS_MAX_M = 128, ENS_MAX_ENTRIES = 8192;    // the table and the sums of a query live in the LDS (123 KB at most)
struct EnsTerms { double rank[ENS_MAX_K]; double absent; };     // rank[k - 1] = -sgn(p) k^p


constexpr int32_t ENS_FLAG = -2;                                // first output of a query that is left to ens_flagged_kernel
constexpr double ENS_NONE = -INFINITY;                          // slot that is no candidate

__device__ __forceinline__ void ens_wave_fence() {              // orders the wave's LDS accesses for the compiler
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ bool ens_better(double sa, int ea, double sb, int eb) { return sa > sb || (sa == sb && ea < eb); }

__device__ __forceinline__ void ens_lds_add(double *p, double v) {
    __builtin_amdgcn_ds_atomic_fadd_f64((__attribute__((address_space(3))) double *)p, v);
}

// slots of a query's table: never fewer than its entries (a full table still ends every probe: each entity is in it)
static inline int ens_slots(int n) { int s = 256; while (s < n + n / 4 && s < ENS_MAX_ENTRIES) s <<= 1; return s; }

__device__ __forceinline__ void ens_query(const int64_t q, const int32_t *lists, int M, int64_t Q, int K, int slots, int shift, const EnsTerms &tm,
                                          int K_out, int32_t *out_idx, float *out_score) {
    extern __shared__ __attribute__((aligned(16))) char ens_lds[];
    double *sum = (double *)ens_lds;                            // [slots]
    int32_t *ent = (int32_t *)(ens_lds + (size_t)slots * 8);    // [slots] entity of the slot, -1: free
    uint16_t *slot_of = (uint16_t *)(ent + slots);              // [M K] slot of every entry, 0xffff: counts for nothing
    uint8_t *next = (uint8_t *)(slot_of + ((M * K + 1) & ~1));  // [slots], p > 0 only: first model not yet in the slot's sum
    volatile uint16_t *claim = (volatile uint16_t *)sum;        // [slots][4] while the table is built (one column per wave)
    __shared__ __attribute__((aligned(16))) char small[256 * 12];
    double *terms = (double *)small;                            // [256] term of rank k + 1, until the sums are done
    double *bin_s = (double *)small;                            // [256] then: the best entry of every bin of slots
    int *bin_e = (int *)(small + 256 * 8);
    __shared__ int part[4][64], ncand;
    __shared__ double thr_s;
    __shared__ int thr_e;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    terms[tid] = tm.rank[tid];
    const double absent = tm.absent;
    const bool dense = absent != 0.0;                           // absent models contribute
    for (int i = tid; i < slots / 4; i += 256) ((int4 *)ent)[i] = make_int4(-1, -1, -1, -1);
    if (tid == 0) { ncand = 0; thr_s = ENS_NONE; thr_e = 0x7fffffff; }
    __syncthreads();

    // ---- 1. table ----
    constexpr int CH = ENS_MAX_K / 64;                          // pieces of 64 ranks
    auto load = [&](int m, int32_t (&t)[CH]) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int k = c * 64 + lane;
            t[c] = (m < M && k < K) ? lists[((int64_t)m * Q + q) * K + k] : -1;
        }
    };
    int32_t cur[CH], nxt[CH];
    load(wave, cur);
    for (int m = wave; m < M; m += 4) {
        load(m + 4, nxt);                                       // (in flight while this list is entered)
        // (a free slot or the entity's own ends the probe; the first probes of all pieces are in flight together)
        int sl[CH], have[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            sl[c] = (int)(((uint32_t)cur[c] * 2654435761u) >> shift);
            have[c] = -1;
            if (c * 64 < K && cur[c] >= 0) have[c] = atomicCAS(ent + sl[c], -1, cur[c]);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
            while (have[c] != -1 && have[c] != cur[c]) {
                sl[c] = (sl[c] + 1) & (slots - 1);
                have[c] = atomicCAS(ent + sl[c], -1, cur[c]);
            }
        // first occurrence in the list: the smallest rank wins its slot's claim (this wave's column)
#pragma unroll
        for (int c = CH - 1; c >= 0; --c) if (c * 64 < K && cur[c] >= 0) claim[sl[c] * 4 + wave] = (uint16_t)(c * 64 + lane);
        for (;;) {
            ens_wave_fence();
            bool wrong = false;
#pragma unroll
            for (int c = CH - 1; c >= 0; --c)
                if (c * 64 < K && cur[c] >= 0 && claim[sl[c] * 4 + wave] > (uint16_t)(c * 64 + lane)) {
                    claim[sl[c] * 4 + wave] = (uint16_t)(c * 64 + lane);
                    wrong = true;
                }
            if (!__any(wrong)) break;                           // (a claim only ever falls: the loop ends)
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int k = c * 64 + lane;
            if (k < K) slot_of[m * K + k] = cur[c] >= 0 && claim[sl[c] * 4 + wave] == (uint16_t)k ? (uint16_t)sl[c] : (uint16_t)0xffff;
            cur[c] = nxt[c];
        }
    }
    __syncthreads();
    for (int i = tid; i < slots / 2; i += 256) ((double2 *)sum)[i] = make_double2(0.0, 0.0);
    if (dense) for (int i = tid; i < slots / 4; i += 256) ((uint32_t *)next)[i] = 0u;
    __syncthreads();

    // ---- 2. sums, model by model ----
    // (the slots of four models are read ahead; without absent terms the additions return nothing, so the wave waits for none)
    if (wave == 0) {
        constexpr int AHEAD = 4;
        double term[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) term[c] = terms[c * 64 + lane];
        for (int m0 = 0; m0 < M; m0 += AHEAD) {
            uint32_t at[AHEAD][CH];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const int k = c * 64 + lane;
                    at[i][c] = 0xffffu;
                    if (c * 64 < K && m0 + i < M && k < K) at[i][c] = slot_of[(m0 + i) * K + k];
                }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i)
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    if (c * 64 >= K) break;
                    if (at[i][c] != 0xffffu) {
                        double *p = sum + at[i][c];
                        if (dense) {
                            double s = *p;
                            for (int l = next[at[i][c]]; l < m0 + i; ++l) s += absent;
                            next[at[i][c]] = (uint8_t)(m0 + i + 1);
                            *p = s + term[c];
                        } else ens_lds_add(p, term[c]);
                    }
                    ens_wave_fence();
                }
        }
    }
    __syncthreads();

    // ---- 3. selection ----
    double bs = ENS_NONE; int be = 0x7fffffff;                  // best of the slots tid, tid + 256, ..
#pragma unroll 4
    for (int i = tid; i < slots; i += 256) {                    // (a free slot's sum is 0: read without a look at its entity)
        const int e = ent[i];
        double s = sum[i];
        if (dense && e >= 0) { for (int l = next[i]; l < M; ++l) s += absent; sum[i] = s; }
        if (e >= 0 && ens_better(s, e, bs, be)) { bs = s; be = e; }
    }
    bin_s[tid] = bs; bin_e[tid] = be;
    __syncthreads();
    // The K_out-th best of the bins' bests bounds the K_out-th best from below; its rank among the bins is found by counting.  Up
    // to 32 winners: 64 bins (of four threads' slots), every wave counting against sixteen of them; more: 256 bins.
    if (K_out <= 32) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const double s = bin_s[w * 64 + lane]; const int e = bin_e[w * 64 + lane];
            if (w == 0 || ens_better(s, e, bs, be)) { bs = s; be = e; }
        }
        int rank = 0;
        const int w0 = __builtin_amdgcn_readfirstlane(wave * 16);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const double s = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(bs), w0 + j), __builtin_amdgcn_readlane(__double2loint(bs), w0 + j));
            rank += ens_better(s, __builtin_amdgcn_readlane(be, w0 + j), bs, be) ? 1 : 0;
        }
        part[wave][lane] = rank;
        __syncthreads();
        if (wave == 0 && bs != ENS_NONE && part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane] == K_out - 1) { thr_s = bs; thr_e = be; }
    } else if (bs != ENS_NONE) {
        int rank = 0;
#pragma unroll 8
        for (int j = 0; j < 256; ++j) rank += ens_better(bin_s[j], bin_e[j], bs, be) ? 1 : 0;
        if (rank == K_out - 1) { thr_s = bs; thr_e = be; }
    }
    __syncthreads();
    uint16_t *cand = slot_of;                                   // (the entries' slots are done with; one candidate per entity at most)
    {
        const double ts = thr_s; const int te = thr_e;
#pragma unroll 4
        for (int i = tid; i < slots; i += 256) {
            const int e = ent[i];
            const double s = sum[i];
            if (e >= 0 && !ens_better(ts, te, s, e)) cand[atomicAdd(&ncand, 1)] = (uint16_t)i;
        }
    }
    __syncthreads();
    const int C = ncand;
    if (C <= 256) {                                             // (as a rule; then the candidates lie densely in the bins' arrays)
        if (tid < C) { bin_s[tid] = sum[cand[tid]]; bin_e[tid] = ent[cand[tid]]; }
        __syncthreads();
        if (tid < C) {
            const double s = bin_s[tid]; const int e = bin_e[tid];
            int rank = 0;
            for (int j = 0; j < C; ++j) rank += ens_better(bin_s[j], bin_e[j], s, e) ? 1 : 0;
            if (rank < K_out) { out_idx[q * K_out + rank] = e; out_score[q * K_out + rank] = (float)s; }
        }
    } else {
        for (int i = tid; i < C; i += 256) {
            const double s = sum[cand[i]]; const int e = ent[cand[i]];
            int rank = 0;
            for (int j = 0; j < C; ++j) rank += ens_better(sum[cand[j]], ent[cand[j]], s, e) ? 1 : 0;
            if (rank < K_out) { out_idx[q * K_out + rank] = e; out_score[q * K_out + rank] = (float)s; }
        }
    }
    for (int i = C + tid; i < K_out; i += 256) { out_idx[q * K_out + i] = -1; out_score[q * K_out + i] = -INFINITY; }
}

__global__ __launch_bounds__(256) void ens_kernel(const int32_t *lists, int M, int64_t Q, int K, int slots, int shift, EnsTerms tm,
                                                  int K_out, int32_t *out_idx, float *out_score) {
    ens_query(blockIdx.x, lists, M, Q, K, slots, shift, tm, K_out, out_idx, out_score);
}

// the queries that ens_top_kernel flagged: workgroup w looks after w, w + gridDim.x, ..
__global__ __launch_bounds__(256) void ens_flagged_kernel(const int32_t *lists, int M, int64_t Q, int K, int slots, int shift, EnsTerms tm,
                                                          int K_out, int32_t *out_idx, float *out_score) {
    __shared__ uint64_t todo[4];
    const int64_t G = gridDim.x;
    for (int64_t first = blockIdx.x; first < Q; first += 256 * G) {
        const int64_t mine = first + threadIdx.x * G;
        const uint64_t b = __ballot(mine < Q && out_idx[mine * K_out] == ENS_FLAG);
        if ((threadIdx.x & 63) == 0) todo[threadIdx.x >> 6] = b;
        __syncthreads();
        for (int w = 0; w < 4; ++w) {
            uint64_t left = todo[w];
            while (left) {
                const int i = w * 64 + __builtin_ctzll(left);
                left &= left - 1;
                ens_query(first + i * G, lists, M, Q, K, slots, shift, tm, K_out, out_idx, out_score);
                __syncthreads();
            }
        }
        __syncthreads();
    }
}

// ---- one wave per query ----
// CPL: candidates per lane.  LDS of a wave: the table, the candidates of its slots, the ranks by (candidate, model); at the end the
// winners from the start on and the candidates' entities in the last C words.  One candidate more than C takes the entries of the
// entities that came when the numbers were used up.
template <int CPL> struct EnsTop {
    static constexpr int C = 64 * CPL, LOG = CPL == 2 ? 7 : 8, BUCKETS = 1 << LOG;
    using Idx = typename std::conditional<(CPL <= 2), uint8_t, uint16_t>::type;
    static constexpr int TABLE = BUCKETS * 16 + BUCKETS * 4 * (int)sizeof(Idx);
    static __host__ __device__ int words(int M) { return M > 4 ? (M + 3) / 4 : 2; }        // of a candidate's ranks
    static __host__ __device__ int bytes(int M) { return TABLE + (C + 4) * words(M) * 4; }
    static_assert(C * 16 <= TABLE + C * 4 && C + 64 < BUCKETS * 4, "");
};
static __host__ __device__ inline int ens_term_bytes(int K) { return (K + 2) / 2 * 16; }

template <int CPL>
__global__ __launch_bounds__(256) void ens_top_kernel(const int32_t *lists, int M, int64_t Q, int K, int R, EnsTerms tm, int K_out,
                                                      int32_t *out_idx, float *out_score) {      // (one to four waves)
    using T = EnsTop<CPL>;
    using Idx = typename T::Idx;
    constexpr int C = T::C;
    extern __shared__ __attribute__((aligned(16))) char ens_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *terms = (double *)ens_lds;                          // [K + 1] term of rank k + 1; [K] of an absent model
    char *own = ens_lds + ens_term_bytes(K) + wave * T::bytes(M);
    int32_t *tab = (int32_t *)own;                              // [BUCKETS][4] entities, -2: free
    Idx *num = (Idx *)(own + T::BUCKETS * 16);                  // [BUCKETS][4] the slot's candidate
    uint32_t *rk = (uint32_t *)(own + T::TABLE);                // [C + 4][words] ranks, a byte per model, K: absent
    uint8_t *rkb = (uint8_t *)rk;
    const int words = T::words(M), pitch = words * 4;
    const bool dense = tm.absent != 0.0;                        // absent models contribute (p > 0)
    for (int i = tid; i <= K; i += blockDim.x) terms[i] = i == K ? tm.absent : tm.rank[i];
#pragma unroll
    for (int i = 0; i < T::BUCKETS / 64; ++i) ((int4 *)tab)[i * 64 + lane] = make_int4(-2, -2, -2, -2);
    {
        const int all = (int)((uint32_t)C * (sizeof(Idx) == 1 ? 0x01010101u : 0x00010001u));
#pragma unroll
        for (int i = 0; i < T::BUCKETS * (int)sizeof(Idx) / 64; ++i) ((int *)num)[i * 64 + lane] = all;
    }
    const int none = (int)((uint32_t)K * 0x01010101u);
    for (int i = lane; i < (C + 4) / 4 * words; i += 64) ((int4 *)rk)[i] = make_int4(none, none, none, none);
    __syncthreads();
    const int64_t q = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (q >= Q) return;                                         // (no barrier below)
    const int32_t *base = lists + q * K;
    const int64_t QK = Q * K;
    // (24 bits of the entity decide: a 24-bit product is one instruction, a 32-bit one takes four times as long)
    auto bucket = [&](int x) { return (int)(((uint32_t)x & 0xffffffu) * 0x9e3779u >> (32 - T::LOG)); };

    // The lists from the last entry to the first, in pieces of 64 lanes: 64 ranks of a list, or g whole short lists.  A lane's place
    // in a piece never changes, and every lane of every piece has an entry: the last pieces reach back over the one before, lanes
    // past g lists do what lane 0 does (an entry may be looked up twice).  The first RING pieces are requested before anything else.
    constexpr int RING = 4, U = 4;
    const int ch = (K + 63) / 64, g = K > 64 ? 1 : min(64 / K, M);
    const int sub = K > 64 || lane >= g * K ? 0 : lane / K, sk = K > 64 ? lane : lane >= g * K ? 0 : lane - sub * K;   // list and rank
    const int pieces = K > 64 ? M * ch : (M + g - 1) / g;
    const int32_t *at_lane = base + sub * QK + sk;
    int t[RING];
    int at_piece[RING];                                         // (first) list and first rank of the piece
    int am = M - g, ac = ch - 1;                                // next piece to request: (first) list, 64 ranks
    const int32_t *row = at_lane + am * QK;
    const int64_t down = g * QK;
    auto request = [&](int i, bool again) {
        const int rank = min(ac * 64, max(K - 64, 0));
        at_piece[i] = am << 8 | rank;
        t[i] = row[rank];
        if (again) return;
        const bool wrap = ac == 0;
        ac = wrap ? ch - 1 : ac - 1;
        if (wrap) {                                             // (a short first piece reaches back; past it the pieces stay there)
            row = am >= g ? row - down : row - am * QK;
            am = max(am - g, 0);
        }
    };
    // (the walk has to end with the last piece, the first ranks of list 0: what is missing to whole rings, the first piece makes up for)
    const int extra = -pieces & (RING - 1);
#pragma unroll
    for (int i = 0; i < RING; ++i) request(i, i < extra);

    // ---- 1. candidates: the entities of the first ranks, rank by rank ----
    // (64 / M ranks at a time, or 64 models of one; every lane has an entry here too, ranks past R do no harm)
    int n = 0, r = R, walked;
    {
        constexpr int DEEP = 4;
        const int per = M < 64 ? min(64 / M, K) : 1, mch = (M + 63) / 64;
        const int ik = M < 64 && lane < per * M ? lane / M : 0, im = M >= 64 ? lane : lane < per * M ? lane - ik * M : 0;
        walked = min((R + per - 1) / per * per, K);
        const int32_t *mine = base + im * QK + ik;
        int k0 = 0, mc = 0;                                     // next to request: (first) rank, 64 models
        int in[DEEP], low[DEEP];
        auto fetch = [&](int i) {
            low[i] = min(k0, K - per);
            in[i] = (mine + (mc > 0 ? (M - 64) * QK : 0) + low[i])[0];
            if (k0 >= R) low[i] = R;
            if (++mc >= mch) { mc = 0; k0 += per; }
        };
#pragma unroll
        for (int i = 0; i < DEEP; ++i) fetch(i);
        for (bool more = true; more;) {
#pragma unroll
            for (int i = 0; i < DEEP; ++i) {
                const int at_rank = low[i], x = in[i];
                if (at_rank >= R) { more = false; break; }
                fetch(i);
                int b = bucket(x), at = -1;
                bool act = x >= 0;
                while (act) {                                   // (at least a quarter of the slots stays free: every probe ends)
                    const int4 v = ((const int4 *)tab)[b];
                    if (v.x == x || v.y == x || v.z == x || v.w == x) break;
                    const int f = v.x < 0 ? 0 : v.y < 0 ? 1 : v.z < 0 ? 2 : v.w < 0 ? 3 : 4;
                    if (f == 4) { b = (b + 1) & (T::BUCKETS - 1); continue; }
                    const int old = atomicCAS(tab + b * 4 + f, -2, x);
                    if (old == -2) at = b * 4 + f;
                    act = old != -2 && old != x;
                }
                const uint64_t fresh = __ballot(at >= 0);
                if (at >= 0) {
                    const int c = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(fresh >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)fresh, 0));
                    num[at] = (Idx)(c < C ? c : C);
                }
                n += __popcll(fresh);
                if (n > C) { n = C; r = walked = at_rank; more = false; break; }         // (this rank is not whole)
            }
        }
    }
    // Models that do not agree: the proof fails as a rule where the table is full before five sixths of the R ranks, and for p > 0 where
    // the walked ranks name the same entities too seldom (less than 1.4 (1 - 1 / M) repeats per winner and further model; agreeing models:
    // 1.5 to 2.4).  Those queries leave here (8 lists of 50 at random from pools of 125, p = 1, 8,192 queries: 103 us without the second
    // test, 88 with it, 47 with ens_kernel alone; 16 of 100 from pools of 250, p = -1: 138 with a line at two thirds of R, 117).
    if (r < K && (n < K_out || 6 * r < 5 * R || (dense && 5 * M * (M * walked - n) < 7 * (M - 1) * (M - 1) * K_out))) {
        if (lane == 0) out_idx[q * K_out] = ENS_FLAG;
        return;
    }
    ens_wave_fence();

    // ---- 2. every entry, from the last to the first: the smaller of two ranks of one list is written later ----
    // (no branch depends on what is found: a free slot's candidate is number C, whose ranks are nobody's)
    {
        for (int done = 0; done < pieces; done += RING) {
#pragma unroll
            for (int h = 0; h < RING; h += U) {
                int x[U], k[U], at[U], b[U], s[U];
                int4 v[U];
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    x[i] = max(t[h + i], -1);
                    b[i] = bucket(x[i]);
                    v[i] = ((const int4 *)tab)[b[i]];
                    k[i] = (at_piece[h + i] & 255) + sk; at[i] = (at_piece[h + i] >> 8) + sub;
                }
#pragma unroll
                for (int i = 0; i < U; ++i) request(h + i, false);
                int full = 0;                                   // (not found in a full bucket: the entity may lie in the next)
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    s[i] = v[i].x == x[i] ? 0 : 3;
                    s[i] = v[i].y == x[i] ? 1 : s[i];
                    s[i] = v[i].z == x[i] ? 2 : s[i];
                    full |= s[i] == 3 && v[i].w != x[i] ? ~v[i].w : 0;
                }
                if (__any(full < 0)) {
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        while (s[i] == 3 && v[i].w != x[i] && v[i].w >= 0) {
                            b[i] = (b[i] + 1) & (T::BUCKETS - 1);
                            v[i] = ((const int4 *)tab)[b[i]];
                            s[i] = v[i].x == x[i] ? 0 : v[i].y == x[i] ? 1 : v[i].z == x[i] ? 2 : 3;
                        }
                }
                int c[U];
#pragma unroll
                for (int i = 0; i < U; ++i) c[i] = num[b[i] * 4 + s[i]];
                int seen[U];
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    at[i] += __umul24(c[i], pitch);
                    seen[i] = -1;
                    if (c[i] != C) {
                        rkb[at[i]] = (uint8_t)k[i];
                        ens_wave_fence();
                        seen[i] = rkb[at[i]];
                    }
                }
                bool wrong = false;
#pragma unroll
                for (int i = 0; i < U; ++i) wrong |= seen[i] > k[i];
                while (__any(wrong)) {                          // two of 64 entries name one entity: the smaller rank stays
                    wrong = false;
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        if (c[i] != C && rkb[at[i]] > k[i]) { rkb[at[i]] = (uint8_t)k[i]; wrong = true; }
                    ens_wave_fence();
                }
            }
        }
    }
    ens_wave_fence();

    // ---- 3. sums in model order ----
    double s[CPL], bound = 0.0;
#pragma unroll
    for (int i = 0; i < CPL; ++i) s[i] = 0.0;
    const double most = terms[r];
    for (int m4 = 0; m4 * 4 < M; ++m4) {
        uint32_t w[CPL];
#pragma unroll
        for (int i = 0; i < CPL; ++i) w[i] = rk[(i * 64 + lane) * words + m4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (m4 * 4 + j >= M) break;
            bound += most;
#pragma unroll
            for (int i = 0; i < CPL; ++i) s[i] += terms[(w[i] >> (8 * j)) & 255];
        }
    }

    // ---- 4. the K_out best ----
    uint32_t key[CPL];                                          // high word of the sum's bits in ascending order; 0: no candidate
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        const int h = __double2hiint(s[i]);
        key[i] = i * 64 + lane < n ? (uint32_t)(h < 0 ? ~h : h | (int)0x80000000) : 0u;
    }
    uint32_t thr = 0;                                           // the largest value that K_out keys reach, or one that just they reach
    for (int bit = 31; bit >= 0 && n > K_out; --bit) {
        const uint32_t x = thr | 1u << bit;
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < CPL; ++i) cnt += __popcll(__ballot(key[i] >= x));
        if (cnt >= K_out) thr = x;
        if (cnt == K_out) break;
    }
    thr = thr ? thr : 1u;
    int32_t *ent = (int32_t *)(own + T::bytes(M)) - (C + 1);    // (the ranks are done with)
#pragma unroll
    for (int i = 0; i < T::BUCKETS / 64; ++i) {
        const int4 v = ((const int4 *)tab)[i * 64 + lane];
        const int vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (vv[j] < 0) break;                               // (a bucket fills from its first slot on)
            ent[num[(i * 64 + lane) * 4 + j]] = vv[j];
        }
    }
    ens_wave_fence();
    double *sel = (double *)own;                                // [C] sum, entity (the table is done with)
    int W = 0;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        const uint64_t in = __ballot(key[i] >= thr);
        if (key[i] >= thr) {
            const int c = W + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0));
            sel[2 * c] = s[i];
            ((int *)sel)[4 * c + 2] = ent[i * 64 + lane];
        }
        W += __popcll(in);
    }
    ens_wave_fence();
    double x[CPL];
    int e[CPL], rank[CPL];
    bool proved = r == K;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        rank[i] = K_out;
        if (i * 64 >= W) continue;
        const int c = i * 64 + lane;
        x[i] = c < W ? sel[2 * c] : 0.0;
        e[i] = c < W ? ((const int *)sel)[4 * c + 2] : -1;
        if (c < W) rank[i] = 0;
#pragma unroll 2
        for (int j = 0; j < W; ++j) rank[i] += ens_better(sel[2 * j], ((const int *)sel)[4 * j + 2], x[i], e[i]) ? 1 : 0;
        proved |= __any(rank[i] == K_out - 1 && x[i] > bound);
    }
    if (!proved) {
        if (lane == 0) out_idx[q * K_out] = ENS_FLAG;
        return;
    }
#pragma unroll
    for (int i = 0; i < CPL; ++i)
        if (rank[i] < K_out) { out_idx[q * K_out + rank[i]] = e[i]; out_score[q * K_out + rank[i]] = (float)x[i]; }
    for (int c = W + lane; c < K_out; c += 64) { out_idx[q * K_out + c] = -1; out_score[q * K_out + c] = -INFINITY; }
}

// candidates per lane of ens_top_kernel, 0: ens_kernel alone.  (Models that agree roughly name 1.8 R entities in the first R ranks
// of four lists, 2.9 R in sixteen, 4.2 R in 64.)
static inline int ens_candidates(int M, int K, int R) {
    int log = 0;
    while (2 << log <= M) ++log;
    const int most = M < 4 ? M * R : R * (2 + log) / 2;
    return K > 255 || most > 512 ? 0 : most <= 128 ? 2 : most <= 256 ? 4 : 8;
}
// waves per workgroup: as many as share the compute unit's LDS best
static inline int ens_waves(int own, int K) {
    int best = 1, held = 0;
    for (int w = 1; w <= 4; ++w) {
        int h = ENS_CU_LDS / (ens_term_bytes(K) + w * own) * w;
        if (h > 32) h = 32;
        if (h >= held) { best = w; held = h; }
    }
    return best;
}

}  // namespace

int kge_run_ensemble(const int32_t *lists, int M, int64_t Q, int K, double p, int K_out, int32_t *out_idx, float *out_score,
                     hipStream_t st) {
    if (M < 1 || M > ENS_MAX_M || K < 1 || K > ENS_MAX_K || M * K > ENS_MAX_ENTRIES) return KGE_E_UNSUPPORTED;
    EnsTerms tm;
    const double sg = p > 0.0 ? -1.0 : 1.0;
    for (int k = 0; k < ENS_MAX_K; ++k) tm.rank[k] = k < K ? sg * pow((double)(k + 1), p) : 0.0;
    tm.absent = p > 0.0 ? -pow((double)(K + 1), p) : 0.0;
    const int slots = ens_slots(M * K);
    int shift = 32;
    for (int v = slots; v > 1; v >>= 1) --shift;
    const int lds = slots * (tm.absent != 0.0 ? 13 : 12) + (M * K + 1) / 2 * 4;
    static KgeLdsLimit lds_limit, flagged_limit;
    if (lds_limit.set((const void *)ens_kernel, ENS_MAX_ENTRIES * 15) != KGE_OK ||
        flagged_limit.set((const void *)ens_flagged_kernel, ENS_MAX_ENTRIES * 15) != KGE_OK) return KGE_E_HIP;
    // (models that agree roughly: ten winners of 10^2 queries needed the first 9 to 14 ranks for p < 0, 12 to 20 for p = 1)
    const int want = p > 0.0 ? (K_out * 5 + 1) / 2 : (K_out * 3 + 1) / 2, R = want < K ? want : K;
    const int per_cu = ENS_CU_LDS / (lds + 4096) < 1 ? 1 : ENS_CU_LDS / (lds + 4096) > 8 ? 8 : ENS_CU_LDS / (lds + 4096);
    // A wave per query costs a second, nearly empty launch (4.6 us, 3 us of the caller's time), has the longer chain for one query (64 lists
    // of 100: 42 us against 37), and what it can't prove is done twice.  So the line lies where agreeing models gain: queries that ens_kernel
    // holds all at once stay there, but for short lists taken whole (32 lists of 10: 14.9 / 14.3 us for 128 queries, 25.3 / 17.2 for
    // 2,048; 100 winners of 16 lists of 50: 40.1 / 36.6).  ens_kernel / here, us, ten winners, p = -1 and 1, agreeing models:  16 lists of
    // 100: 2,500 queries 33 / 27, 75 / 31, 8,192 queries 99 / 40, 209 / 47;  8 of 50: 2,500 queries 16 / 16, 20 / 19, 8,192 queries 39 / 24, 47 / 28.
    // Models that do not agree LOSE by it - nothing known before the launch tells them apart -: lists drawn at random from pools 2.5 times as
    // long, 8,192 queries: 16 of 100 100 / 117, 187 / 209;  8 of 50 40 / 26, 47 / 88;  16 of 200 302 / 320, 565 / 585;  64 of 100, 4,096
    // queries 622 / 638, 1,249 / 1,266.
    const int cpl = (R == K && K <= 64) || Q > 256 * per_cu ? ens_candidates(M, K, R) : 0;
    if (cpl == 0) {
        hipLaunchKernelGGL(ens_kernel, dim3((unsigned)Q), dim3(256), lds, st, lists, M, Q, K, slots, shift, tm, K_out, out_idx, out_score);
        return kge_launch_status();
    }
#define ENS_TOP(CPL)                                                                                                                     \
    {                                                                                                                                     \
        static KgeLdsLimit limit;                                                                                                         \
        if (limit.set((const void *)ens_top_kernel<CPL>, ENS_CU_LDS) != KGE_OK) return KGE_E_HIP;                                         \
        const int own = EnsTop<CPL>::bytes(M), waves = ens_waves(own, K);                                                                 \
        hipLaunchKernelGGL(ens_top_kernel<CPL>, dim3((unsigned)((Q + waves - 1) / waves)), dim3(64 * waves),                              \
                           ens_term_bytes(K) + waves * own, st, lists, M, Q, K, R, tm, K_out, out_idx, out_score);                        \
    }
    if (cpl == 2) ENS_TOP(2) else if (cpl == 4) ENS_TOP(4) else ENS_TOP(8)
#undef ENS_TOP
    if (kge_launch_status() != KGE_OK) return KGE_E_HIP;
    if (R == K && M * K <= 64 * cpl) return KGE_OK;             // (every list whole and every entity in the table: nothing is ever flagged)
    const int64_t most = 256 * (per_cu < 6 ? per_cu : 6);         // (its registers allow six)
    hipLaunchKernelGGL(ens_flagged_kernel, dim3((unsigned)(Q < most ? Q : most)), dim3(256), lds, st, lists, M, Q, K, slots, shift, tm, K_out,
                       out_idx, out_score);
    return kge_launch_status();
}
