// Power-rank ensemble of M top-K lists per query (Section 3.2 "Inference", paragraph "Ensemble", eq. (ensemble)):
// s(t) = sum over the models, in model order, of -sgn(p) k^p where t is the k-th entry of the model's list and of
// -[p > 0] (K + 1)^p where the list does not hold t; the K_out entities with the largest s(t) are returned, ties
// to the smaller id.  An entity in no list has the smallest possible score, so only listed entities compete.
// One workgroup of four waves per query:
//   1. the entries' entities go into a hash table in the LDS (linear probing); wave w takes the lists of models w, w + 4, ..,
//      so that an entity that a list holds twice is found inside one wave, and notes every entry's slot
//   2. one wave walks the models in order and adds every entry's term to its slot's fp64 sum: a wave's LDS accesses happen in
//      the order it issues them, so the sums are in model order without a barrier per model
//   3. the K_out winners: a lower bound of the K_out-th best from the best of every bin of slots, then the few entries that
//      reach it are ranked by counting
// The K + 1 possible terms come from the host as a kernel argument, so they are the host math library's powers.
// What bounds it is the latency of the LDS chains of a query, so what counts is the number of workgroups on a compute unit (12
// bytes of LDS per slot: five at M K = 1,600).  Sorting the M K keys in the LDS, one thread per run of equal entities and K_out
// workgroup-wide arg-max rounds took 1,106 us for 16 lists of 100 and 8,192 queries (66 sorting steps with a barrier each);
// this takes 94 us (one pass of the lists: 52 MB, 11 us at the copy rate).
#include "kge_internal.h"
#include <math.h>

int kge_run_ensemble(const int32_t *lists, int M, int64_t Q, int K, double p, int K_out, int32_t *out_idx, float *out_score,
                     hipStream_t st);

namespace {

constexpr int ENS_MAX_K = 256, ENS_MAX_M = 128, ENS_MAX_ENTRIES = 8192;    // the table and the sums of a query live in the LDS (123 KB at most)
struct EnsTerms { double rank[ENS_MAX_K]; double absent; };     // rank[k - 1] = -sgn(p) k^p


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

__global__ __launch_bounds__(256) void ens_kernel(const int32_t *lists, int M, int64_t Q, int K, int slots, int shift, EnsTerms tm,
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
    const int64_t q = blockIdx.x;
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
    static KgeLdsLimit lds_limit;
    if (lds_limit.set((const void *)ens_kernel, ENS_MAX_ENTRIES * 15) != KGE_OK) return KGE_E_HIP;
    hipLaunchKernelGGL(ens_kernel, dim3((unsigned)Q), dim3(256), lds, st, lists, M, Q, K, slots, shift, tm, K_out, out_idx, out_score);
    return kge_launch_status();
}
