// Stage 1 in one kernel: query-centroid scores S_cq = C . Q^T (Eq. 2), the centroid pruning map of
// Eq. 5, the nprobe best centroids of every query token (Section 4.1) and the table of surviving
// centroids that stage 2 consumes.
//
// Every later decision of the pipeline (which centroids are probed, which survive t_cs, which
// passages make the ndocs and ndocs/4 cuts) is a comparison of S_cq values or of sums of them,
// so they are computed the way the definition reads: each S[c][i] is the dot product accumulated
// in double over the dimensions in index order, rounded once to fp32.  A product of two fp32
// values is exact in double, so a chain of fused multiply-adds in that order gives the same bits
// as "multiply, then add" on any machine -- the scores carry no accumulation-order freedom.
//
// Two kernels compute the same bits.
//
// Matrix form (scq_mfma_kernel): the double-precision matrix instruction D = A(16x4) B(4x16) + C adds its four
// products to C one after the other, rounding after each, i.e. it IS the chain of fused multiply-adds over four
// consecutive dimensions; 32 of them in a row walk the 128 dimensions in index order.  A workgroup of four waves
// owns 128 centroid rows and the 64 token columns of two queries; centroid rows are staged in LDS 32 dimensions at
// a time with coalesced loads, next to the same 32 dimensions of the queries in operand order, and a wave holds a
// 32 x 64 block of double accumulators.  That the instruction reproduces the chain is checked once per process on
// the device (plaid_scq_matrix_form_ok): if it ever did not, the vector form below is used instead.
//
// Vector form (scq_fused_kernel): a workgroup of eight waves owns 64 centroid rows, staged once in LDS with coalesced
// loads; wave g computes query tokens 4g..4g+3 for all 64 rows (lane = centroid, four double
// accumulators).  The query, pre-converted to double and laid out [token group][dim][4], is
// uniform across a wave and is fetched through the scalar unit, so the inner loop is one
// v_fma_f64 per (dimension, token) whose only per-lane operand is the LDS-resident centroid row.
//
// Either way the tile of results then yields the row maxima (pruning bits) and, per query token, the maximum of the
// tile's column.  The probes come from those maxima: with T the nprobe-th largest tile maximum of a token, each of
// the nprobe best tiles holds a score >= T, so the nprobe-th best score is >= T and every centroid among the nprobe
// best lies in a tile whose maximum is >= T -- normally just nprobe tiles.  The tail kernel finds T, ranks the rows of
// those tiles from S_cq and builds the duplicate-free union of the probes, and next to that the survivor table.
// (Ranking inside the score kernel instead costs it a third of its running time: its waves' vector instructions
// queue behind other waves' matrix instructions.)
#include "plaid_internal.h"

#include <math.h>


#define SCQ_THREADS 512
#define SCQ_ROWS 64
#define SCQ_HALF 64      // dimensions staged at a time
#define SCQ_RSTRIDE 68   // floats per staged half row: 16-byte aligned, consecutive rows 4 banks apart
#define SCQ_SSTRIDE 33   // floats per row of the result tile (conflict-free column and row walks)
#define SCQ_GROUPS 8     // token groups = waves per workgroup
#define SCQ_TOK 4        // query tokens per wave
#define TAIL_THREADS 1024
#define TAIL_LANES 32     // lanes of the tail kernel that share one query token

// Vector form only (the matrix form does both inside its score kernel): clears the workspace region that must start
// at zero and lays out the queries, Qd[q][g][t][u] = (double) Q[q][4g + u][t].
__global__ __launch_bounds__(256) void stage1_prep_kernel(const float *__restrict__ Q, double *__restrict__ Qd, int nq,
                                                          uint32_t *__restrict__ zero, int64_t zero_words)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < zero_words; i += (int64_t)gridDim.x * blockDim.x)
        zero[i] = 0u;
    for (int q = blockIdx.x; q < nq; q += gridDim.x)
        for (int e = threadIdx.x; e < QLEN * DIM; e += blockDim.x) {
            const int u = e & 3, t = (e >> 2) & (DIM - 1), g = e >> 9;
            Qd[(int64_t)q * QLEN * DIM + e] = (double)Q[(int64_t)q * QLEN * DIM + (4 * g + u) * DIM + t];
        }
}

template <int NP>
__device__ __forceinline__ void scq_insert_key(uint64_t (&best)[NP], uint64_t key)
{
    if (key < best[NP - 1]) {
#pragma unroll
        for (int j = NP - 1; j >= 0; --j) {
            if (key < best[j]) {
                if (j + 1 < NP) best[j + 1] = best[j];
                best[j] = key;
            }
        }
    }
}

struct Stage1Out {          // per-query outputs of the tail (device pointers, leading dimension = query)
    int32_t *probed;        // [nq][32][nprobe] best first
    int32_t *uniq;          // [nq][uniq_stride] ascending distinct probed centroids (see probes_apart)
    int32_t *n_uniq;        // [nq]
    int uniq_stride;
    S2Meta *meta;           // [nq]
    int32_t *kept_ids;      // [nq][S2_MAX_KEPT]
    float *T;               // [nq][S2_MAX_KEPT + 1][32]
    const int64_t *ivf_offsets;  // [C + 1] inverted-list offsets: slots are numbered by list length (null: by id)
    int32_t *qcount;        // [4] / [3][qlist_stride]: the queries by number of surviving centroids (none, 1..31, 32..63; more:
    int32_t *qlist;         //   from the end of the last row), appended as their workgroups finish (null: not recorded).
    int qlist_stride;       //   Stage 2 takes its queries from these lists.
    int32_t *list_counts;   // stage 2's, to be cleared (null: none)
    bool need_hash;         // stage 2 will use the streaming form
    bool probes_apart;      // uniq holds every probe of the query, with duplicates and in no order
};

// Floats per query row in the probe kernel's LDS.  The survivor table is evaluated with a lane per query token: with rows
// of 128 floats the 32 tokens' reads fall into one bank group, and the table took 12 of the kernel's 31 us for one query.
#define TAIL_QSTRIDE (DIM + 4)
#define TX_STRIDE 33  // floats per row of the survivors' entries in LDS: walks along rows and along columns hit all banks
// Largest, smallest and `rank`-th largest (the smallest, when there are fewer) of column `tid` of the K rows, to colmm.
#define SCQ_BASE_FIRST 30  // survivors from which on the rank is (K + 6) / 9 = 4 .. 7
static_assert((S2_MAX_KEPT + 6) / 9 <= 7 && (SCQ_BASE_FIRST + 6) / 9 == 4, "the ranks are 3 .. 7");
template <int N>
__device__ __forceinline__ void scq_column_bounds(const float *Tx, int K, int rank, int tid, float *colmm /*[3][32]*/)
{
    float t[N], mn = INFINITY;
#pragma unroll
    for (int k = 0; k < N; ++k) t[k] = -INFINITY;
#pragma unroll 4
    for (int s = 0; s < K; ++s) {
        float v = Tx[s * TX_STRIDE + tid];
        mn = fminf(mn, v);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float a = fminf(t[k], v);
            t[k] = fmaxf(t[k], v);
            v = a;
        }
    }
    float base = t[2];
#pragma unroll
    for (int k = 3; k < N; ++k) base = rank > k ? t[k] : base;
    colmm[tid] = t[0];
    colmm[QLEN + tid] = mn;
    colmm[2 * QLEN + tid] = K >= 3 ? base : mn;
}

// What the survivor table keeps in LDS.
#define TAIL_AMB 2048  // ambiguous rows decided per round
struct SurvivorScratch {
    float Tx[S2_MAX_KEPT * TX_STRIDE];
    uint32_t trial[S2_NHASH * (S2_HASH / 32)];
    float colmm[3 * QLEN];
    int32_t ids[S2_MAX_KEPT + 1], rank[S2_MAX_KEPT + 1];
    int32_t misc[2];  // number of survivors, chosen hash trial
    float gain[S2_MAX_KEPT + 1];
    int32_t amb_n, amb_total;
    uint32_t amb_pass[TAIL_AMB / 32];
};
struct SurvivorRows {  // APPROX only: the re-evaluations' operands, written and read in 16-byte pieces
    alignas(16) float Qs[QLEN * TAIL_QSTRIDE];
    alignas(16) union {
        float row[(S2_MAX_KEPT + 1) * TAIL_QSTRIDE];  // (whole tiles of sixteen)
        int32_t amb[TAIL_AMB];
    };
    bool matrix;  // see tail_exact_rows
};

// The dot products of n rows with the 32 query rows, both in LDS TAIL_QSTRIDE floats apart, as the definition reads: put(row,
// token, value).  All threads of the workgroup call this; what it read may be written again after a barrier, rows n ..
// up to a multiple of sixteen are read and not used.  matrix: by the double-precision matrix instruction, which is the chain
// of fused multiply-adds (see the top of this file) -- a tile of 16 rows and 16 tokens per wave, 32 instructions one after
// the other; else a product per thread.  The conversions to double and the additions of 768 products, a thread each, take 19 us on one
// compute unit, the tiles 2.
typedef double scq_double4 __attribute__((ext_vector_type(4)));
template <typename Put>
__device__ __forceinline__ void tail_exact_rows(const float *row, int n, const float *Qs, bool matrix, Put put)
{
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    if (matrix) {  // uniform
        const int n_tiles = ((n + 15) >> 4) * (QLEN / 16);
        for (int t = __builtin_amdgcn_readfirstlane(tid >> 6); t < n_tiles; t += (int)blockDim.x >> 6) {
            const int r0 = 16 * (t / (QLEN / 16)), c0 = 16 * (t % (QLEN / 16));
            const float *a = row + (r0 + li) * TAIL_QSTRIDE + lg, *b = Qs + (c0 + li) * TAIL_QSTRIDE + lg;
            scq_double4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 16
            for (int s = 0; s < DIM / 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[4 * s], (double)b[4 * s], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r0 + 4 * r + lg < n) put(r0 + 4 * r + lg, c0 + li, (float)acc[r]);
        }
    } else {
        for (int e = tid; e < n * QLEN; e += (int)blockDim.x)
            put(e >> 5, e & 31, plaid_exact_dot_lds(row + (e >> 5) * TAIL_QSTRIDE, Qs + (e & 31) * TAIL_QSTRIDE));
    }
}

// The rows whose bit is set in the query's pruning words, in any order (the table sorts them), and with amb the number of
// those set there, to amb_total: FLY words of each per thread in flight, nearly all of them zero.  All threads call this;
// the counters are zero and published, a barrier has to follow.
template <int FLY>
__device__ __forceinline__ void stage1_list_survivors(const uint32_t *__restrict__ kb, const uint32_t *__restrict__ amb, int64_t keep_words,
                                                      SurvivorScratch &sh)
{
    const int tid = threadIdx.x, nthreads = blockDim.x;
    int open = 0;
    for (int64_t w0 = tid; w0 < keep_words; w0 += (int64_t)FLY * nthreads) {
        uint32_t v[FLY], a[FLY];
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            const int64_t w = w0 + (int64_t)u * nthreads;
            v[u] = w < keep_words ? kb[w] : 0u;
            a[u] = amb && w < keep_words ? amb[w] : 0u;
        }
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            open += __popc(a[u]);
            if (v[u]) {
                int pos = atomicAdd(&sh.misc[0], __popc(v[u]));
                for (uint32_t rest = v[u]; rest && pos < S2_MAX_KEPT; rest &= rest - 1)
                    sh.ids[pos++] = (int32_t)((w0 + (int64_t)u * nthreads) * 32 + __ffs(rest) - 1);
            }
        }
    }
    if (open) atomicAdd(&sh.amb_total, open);
}

// Survivor table of one query (runs in one workgroup, all of whose threads call it).  misc[0] = number K of centroids
// passing Eq. 5, ids = the first of them, in any order; when K <= S2_MAX_KEPT their ids are listed by decreasing length of
// their inverted lists (without lists, and among equals, ascending), their rows copied to T (slot s at T[s], s = 1..K), a
// collision-free hash shift is chosen for the streaming form's table, the gains and the base of the additive score bound are
// set, and bin_hi / bin_scale from bounds of any non-empty passage's pruned score.  col_max(colmm): the largest entry of each
// of the 32 columns to colmm[0 .. 31] (asked for when K is large; all threads call it, a barrier follows).
// APPROX (Sq comes from the split-fp16 kernel): the rows of T are re-evaluated in double from the centroids Cm and the query
// in x.Qs, which makes every stage-2 score that is built from T the exact one.  The rows are staged in LDS, so that the
// chains of additions wait for one round trip to memory and not for four.
template <bool APPROX, typename ColMax>
__device__ __forceinline__ void stage1_survivor_table(const float *__restrict__ Sq, int64_t C, ColMax col_max, S2Meta *meta_q,
                                      int32_t *__restrict__ kept_ids_q, float *__restrict__ Tq, SurvivorScratch &sh,
                                      SurvivorRows *x = nullptr, const float *__restrict__ Cm = nullptr,
                                      const int64_t *__restrict__ ivf_offsets = nullptr, int q = 0,
                                      int32_t *qcount = nullptr, int32_t *qlist = nullptr, int qlist_stride = 0, int32_t *list_counts = nullptr,
                                      bool need_hash = true /* the streaming form looks survivors up */)
{
    const int tid = threadIdx.x, nthreads = blockDim.x;
    int32_t *ids = sh.ids, *misc = sh.misc;
    uint32_t *trial = sh.trial;
    float *colmm = sh.colmm, *Tx = sh.Tx;
    int K = misc[0];
    if (list_counts && tid < S2_COPIES) list_counts[(int64_t)q * S2_COUNTS_QUERY + tid * S2_COUNT_STRIDE] = 0;
    if (C > (1ll << 26) - 2 && K <= S2_MAX_KEPT) K = S2_MAX_KEPT + 1;  // ids must fit the 26-bit field of a table entry
    // Slots in one order, whatever order the ids were found in: by decreasing inverted-list length, ties by id, so that a
    // query's gains are the same each time.  Stage 2 needs no particular order.
    if (K > 0 && K <= S2_MAX_KEPT) {
        int32_t my_id = 0;
        uint32_t *lens = trial;  // its first K words serve as the list lengths; the hash trials start from zeros
        for (int e = tid; need_hash && e < S2_NHASH * (S2_HASH / 32); e += nthreads)
            if (e >= K) trial[e] = 0u;
        if (tid < K) {
            my_id = ids[tid];
            // at most P < 2^31 entries (no lists: in the order of the ids)
            lens[tid] = ivf_offsets ? (uint32_t)(ivf_offsets[my_id + 1] - ivf_offsets[my_id]) : 0u;
        }
        if (APPROX)
            for (int e0 = tid; e0 < K * (DIM / 4); e0 += 2 * nthreads) {  // (two pieces in flight: all of them)
                float4 piece[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int e = e0 + u * nthreads;
                    piece[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (e < K * (DIM / 4)) piece[u] = *reinterpret_cast<const float4 *>(Cm + (int64_t)ids[e / (DIM / 4)] * DIM + 4 * (e % (DIM / 4)));
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int e = e0 + u * nthreads;
                    if (e < K * (DIM / 4)) *reinterpret_cast<float4 *>(x->row + e / (DIM / 4) * TAIL_QSTRIDE + 4 * (e % (DIM / 4))) = piece[u];
                }
            }
        __syncthreads();
        for (int e = tid; e < 16 * K; e += nthreads) {  // a slot's rank by counting, sixteen threads a slot (whole groups of them)
            const int s = e >> 4;
            const uint32_t my_len = lens[s];
            const int32_t id = ids[s];
            int rank = 0;
#pragma unroll
            for (int u0 = 0; u0 <= S2_MAX_KEPT; u0 += 16) {
                const int u = u0 + (e & 15);
                const uint32_t len = u < K ? lens[u] : 0u;
                const int32_t other = u < K ? ids[u] : 0x7FFFFFFF;
                rank += (len > my_len || (len == my_len && other < id)) ? 1 : 0;
            }
            rank += __shfl_xor(rank, 1);
            rank += __shfl_xor(rank, 2);
            rank += __shfl_xor(rank, 4);
            rank += __shfl_xor(rank, 8);
            if ((e & 15) == 0) sh.rank[s] = rank;
        }
        __syncthreads();
        if (tid < K) {
            ids[sh.rank[tid]] = my_id;
            lens[tid] = 0u;
        }
        __syncthreads();
    }
    // a hash h(c) = (c ^ (c >> sh)) & (S2_HASH - 1) that maps the survivors to distinct entries makes a lookup one
    // probe; thread t tries shift S2_SHIFT0 + t on a private bitmap.  No such shift (very rare): gather kernel.
    if (need_hash && K <= S2_MAX_KEPT) {  // (K = 0: any shift will do, no trial is looked at)
        bool ok = tid < S2_NHASH;
        if (ok) {
            const int sh = S2_SHIFT0 + tid;
            uint32_t *mine = trial + tid * (S2_HASH / 32);
            for (int s = 0; s < K; ++s) {
                const uint32_t c = (uint32_t)ids[s];
                const uint32_t h = (c ^ (c >> sh)) & (S2_HASH - 1);
                const uint32_t bit = 1u << (h & 31);
                if (mine[h >> 5] & bit) ok = false;
                mine[h >> 5] |= bit;
            }
        }
        if (ok) atomicMax(&misc[1], S2_NHASH - 1 - tid);  // smallest successful shift wins
        __syncthreads();
        if (misc[1] < 0) K = S2_MAX_KEPT + 1;
    }
    const int hash_shift = (need_hash && K <= S2_MAX_KEPT) ? S2_SHIFT0 + (S2_NHASH - 1 - misc[1]) : 0;
    if (K <= S2_MAX_KEPT) {
        auto put = [&](int slot, int tok, float v) {
            Tq[QLEN + slot * QLEN + tok] = v;
            Tx[slot * TX_STRIDE + tok] = v;
        };
        if (APPROX)  // (the staged rows lie in the order the ids were found in)
            tail_exact_rows(x->row, K, x->Qs, x->matrix, [&](int r, int tok, float v) { put(sh.rank[r], tok, v); });
        else
            for (int e = tid; e < K * QLEN; e += nthreads) put(e >> 5, e & 31, Sq[(int64_t)ids[e >> 5] * QLEN + (e & 31)]);
        if (tid < K) kept_ids_q[tid] = ids[tid];
        __syncthreads();
        // Per query token: bounds of the rows for the bins, and the base of the additive bound
        // score(bag) <= sum_i base_i + sum over the members of sum_i max(0, row_i - base_i): true for any base, and tight
        // for one that only a token's own centroid (and perhaps one more) exceeds.  That is the third largest entry of some
        // twenty-five rows, but every further row is one more that may exceed it by chance, so that the
        // rank grows with their number, by one in nine.  Passages whose bound reaches the ndocs-th best score, as a multiple of ndocs, with the
        // third / fifth / sixth largest entry (400 000 passages, 65536 centroids, ndocs 1024): 4.1 / 9.8 / 14 with 24..29
        // survivors, 15 / 4.2 / 6.6 with 42..47, 56 / 7.6 / 5.6 with 54..59.  Stage 2 of one query with 58 survivors took
        // 119 to 184 us with the third, 82 to 100 with this; 64 queries with 36 to 66 each 693 -> 356.
        if (tid < QLEN) {
            if (K < SCQ_BASE_FIRST) scq_column_bounds<3>(Tx, K, 3, tid, colmm);
            else scq_column_bounds<7>(Tx, K, (K + 6) / 9, tid, colmm);
        }
        __syncthreads();
        // the slots' gains, eight threads a slot
        float *gain = sh.gain;
        for (int e = tid; e < 8 * K; e += nthreads) {  // (whole groups of eight)
            const int s = e >> 3;
            float g = 0.f;
#pragma unroll
            for (int u = 0; u < QLEN / 8; ++u) {
                const int i = (e & 7) + 8 * u;
                g += fmaxf(Tx[s * TX_STRIDE + i] - colmm[2 * QLEN + i], 0.f);
            }
            g += __shfl_xor(g, 1);
            g += __shfl_xor(g, 2);
            g += __shfl_xor(g, 4);
            if ((e & 7) == 0) gain[s] = g;
        }
        __syncthreads();
        if (tid < 64 && K > 0) {  // one wave, lane = slot (the next one fills in the rest of the record)
            const float g = tid < K ? gain[tid] : 0.f;
            float base = tid < QLEN ? colmm[2 * QLEN + tid] : 0.f;
            float scale = tid < QLEN ? fmaxf(fabsf(colmm[tid]), fabsf(colmm[QLEN + tid])) : 0.f;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                base += __shfl_xor(base, d);
                scale += __shfl_xor(scale, d);
            }
            float total = g;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) total += __shfl_xor(total, d);
            // the rounding of these fp32 sums (at most 64 additions of values within `scale`) and of the scores themselves
            const float slack = 2e-5f * scale;
            const bool finite = total < INFINITY && scale < INFINITY;  // (false also when an entry is not a number)
            const float unit = finite ? total * (1.0f / S2_UB_TOTAL) : 0.f;
            int gq = 0;
            if (unit > 0.f && g > 0.f) gq = (int)ceilf(g / unit * 1.00002f);
            if (tid < K) reinterpret_cast<uint16_t *>(Tq)[tid] = (uint16_t)gq;
            if (tid == 0) {
                meta_q->ub_base = finite ? base + slack : INFINITY;  // infinity: nothing is ever pruned
                meta_q->ub_unit = unit;
            }
        }
    } else {
        // many survivors: the largest entry of each column bounds every row from above
        col_max(colmm);
        __syncthreads();
        if (tid < QLEN) colmm[QLEN + tid] = -colmm[tid] - 1.0f;
        __syncthreads();
    }
    if (tid >= 64 && tid < 128) {  // (one wave; the bounds need no particular order of summation)
        const int i = tid - 64;
        double u = i < QLEN ? (double)colmm[i] : 0.0, l = i < QLEN ? (double)colmm[QLEN + i] : 0.0;
#pragma unroll
        for (int d = 1; d < QLEN; d <<= 1) {
            u += __shfl_xor(u, d);
            l += __shfl_xor(l, d);
        }
        if (i == 0) {
            meta_q->K = K;
            meta_q->bin_hi = (float)u;
            const float range = (float)u - (float)l;
            meta_q->bin_scale = (K > 0 && range > 0.f && range < INFINITY) ? (float)SEL_BINS / range : 0.f;
            meta_q->hash_shift = hash_shift;
            if (qlist) {
                const int cls = K == 0 ? 0 : (K <= 31 ? 1 : (K <= S2_MAX_KEPT ? 2 : 3));
                const int at = atomicAdd(&qcount[cls], 1);
                // (always in range, when the counts start at zero)
                if (at < qlist_stride) qlist[cls < 3 ? (int64_t)cls * qlist_stride + at : 3ll * qlist_stride - 1 - at] = q;
            }
        }
    }
}

// Standalone form for the general top-nprobe path (nprobe > 8), where the probes come from the generic selection.
__global__ __launch_bounds__(512) void stage1_survivor_kernel(const float *__restrict__ S, int64_t C,
                                                              const uint32_t *__restrict__ keepbits, int64_t keep_words,
                                                              const int32_t *__restrict__ probed, int nprobe, Stage1Out o)
{
    __shared__ SurvivorScratch sh;
    __shared__ int32_t top1[QLEN];
    const int q = blockIdx.x;
    const float *Sq = S + (int64_t)q * C * QLEN;
    if (threadIdx.x < QLEN) top1[threadIdx.x] = probed[((int64_t)q * QLEN + threadIdx.x) * nprobe];
    if (threadIdx.x == 0) {
        sh.misc[0] = 0;
        sh.misc[1] = -1;
    }
    __syncthreads();
    stage1_list_survivors<8>(keepbits + (int64_t)q * keep_words, nullptr, keep_words, sh);
    __syncthreads();
    stage1_survivor_table<false>(Sq, C,
                                 [&](float *colmm) { if (threadIdx.x < QLEN) colmm[threadIdx.x] = Sq[(int64_t)top1[threadIdx.x] * QLEN + threadIdx.x]; },
                                 o.meta + q, o.kept_ids + (int64_t)q * S2_MAX_KEPT, o.T + (int64_t)q * (S2_MAX_KEPT + 1) * QLEN, sh,
                                 nullptr, nullptr, o.ivf_offsets, q, o.qcount, o.qlist, o.qlist_stride, o.list_counts, o.need_hash);
}

// tilemax: [q][tile][32] column maxima of each tile (null: scores and pruning bits only).
__global__ __launch_bounds__(SCQ_THREADS) void scq_fused_kernel(const float *__restrict__ Cm, int64_t C,
                                                                const double *__restrict__ Qd, float t_cs,
                                                                float *__restrict__ S, uint32_t *__restrict__ keepbits,
                                                                int64_t keep_words, float *__restrict__ tilemax)
{
    // one LDS arena: half of the centroid tile (64 dimensions) at a time during the contraction; afterwards the 64x32
    // result tile and the partial column maxima
    constexpr int ARENA_FLOATS = SCQ_ROWS * SCQ_RSTRIDE > SCQ_ROWS * SCQ_SSTRIDE + 8 * QLEN
                                     ? SCQ_ROWS * SCQ_RSTRIDE
                                     : SCQ_ROWS * SCQ_SSTRIDE + 8 * QLEN;
    __shared__ __align__(16) float arena[ARENA_FLOATS];
    float *tile = arena;                             // [64][SCQ_SSTRIDE]
    float *cm = arena + SCQ_ROWS * SCQ_SSTRIDE;      // [8][32]
    const int q = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int g = __builtin_amdgcn_readfirstlane(tid >> 6);  // token group of this wave (uniform -> scalar loads of Qd)
    const int64_t c0 = (int64_t)blockIdx.x * SCQ_ROWS;
    const int nrows = (int)(C - c0 < SCQ_ROWS ? C - c0 : SCQ_ROWS);

    // staging: a half tile is 64 rows x 64 dims = 1024 float4, two per thread; 256-byte row halves read contiguously.
    // The second half is requested before the first is multiplied, so only the first load's latency is exposed.
    const int r0 = tid >> 4, c4 = tid & 15;  // this thread stages rows r0 and r0 + 32, float4 column c4
    float4 pre[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int r = r0 + 32 * k;
        pre[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r < nrows) pre[k] = *reinterpret_cast<const float4 *>(Cm + (c0 + r) * DIM + 4 * c4);
    }
    const double *__restrict__ qd = Qd + ((int64_t)q * SCQ_GROUPS + g) * DIM * SCQ_TOK;
    const float4 *row = reinterpret_cast<const float4 *>(arena + lane * SCQ_RSTRIDE);
    double acc[SCQ_TOK] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int half = 0; half < DIM / SCQ_HALF; ++half) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
            *reinterpret_cast<float4 *>(arena + (r0 + 32 * k) * SCQ_RSTRIDE + 4 * c4) = pre[k];
        __syncthreads();
        if (half + 1 < DIM / SCQ_HALF) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int r = r0 + 32 * k;
                if (r < nrows) pre[k] = *reinterpret_cast<const float4 *>(Cm + (c0 + r) * DIM + SCQ_HALF * (half + 1) + 4 * c4);
            }
        }
        // the query operands of the next four dimensions are requested (scalar loads) before the current four are used
        const double *__restrict__ qh = qd + half * SCQ_HALF * SCQ_TOK;
        double qa[4 * SCQ_TOK], qb[4 * SCQ_TOK];
#pragma unroll
        for (int e = 0; e < 4 * SCQ_TOK; ++e) qa[e] = qh[e];
#pragma unroll 1
        for (int t8 = 0; t8 < SCQ_HALF / 8; ++t8) {
            {
#pragma unroll
                for (int e = 0; e < 4 * SCQ_TOK; ++e) qb[e] = qh[(8 * t8 + 4) * SCQ_TOK + e];
                const float4 a4 = row[2 * t8];
                const double a[4] = {(double)a4.x, (double)a4.y, (double)a4.z, (double)a4.w};
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < SCQ_TOK; ++i) acc[i] = fma(a[u], qa[u * SCQ_TOK + i], acc[i]);
            }
            {
                const int tn = t8 + 1 < SCQ_HALF / 8 ? 8 * t8 + 8 : 0;  // the last round re-reads the first operands (unused)
#pragma unroll
                for (int e = 0; e < 4 * SCQ_TOK; ++e) qa[e] = qh[tn * SCQ_TOK + e];
                const float4 a4 = row[2 * t8 + 1];
                const double a[4] = {(double)a4.x, (double)a4.y, (double)a4.z, (double)a4.w};
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < SCQ_TOK; ++i) acc[i] = fma(a[u], qb[u * SCQ_TOK + i], acc[i]);
            }
        }
        __syncthreads();  // every wave is done with this half: the arena is rewritten next
    }
    const float4 s4 = make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]);
    if (lane < nrows) *reinterpret_cast<float4 *>(S + ((int64_t)q * C + c0 + lane) * QLEN + SCQ_TOK * g) = s4;
    float *trow = tile + lane * SCQ_SSTRIDE + SCQ_TOK * g;
    trow[0] = s4.x;
    trow[1] = s4.y;
    trow[2] = s4.z;
    trow[3] = s4.w;
    __syncthreads();

    // Eq. 5: pruning bits of the 64 rows (wave 0)
    if (tid < 64) {
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < QLEN; ++i) m = fmaxf(m, tile[tid * SCQ_SSTRIDE + i]);
        const unsigned long long b = __ballot(tid < nrows && m >= t_cs);
        if (tid == 0) {
            uint32_t *kb = keepbits + (int64_t)q * keep_words + (c0 >> 5);
            kb[0] = (uint32_t)b;
            if ((c0 >> 5) + 1 < keep_words) kb[1] = (uint32_t)(b >> 32);
        }
    }
    if (!tilemax) return;  // uniform

    // column maxima of the tile: thread (i, p) takes rows 8p .. 8p+7 of column i
    if (tid < 256) {
        const int i = tid & 31, p = tid >> 5;
        float m = -INFINITY;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int rr = 8 * p + r;
            if (rr < nrows) m = fmaxf(m, tile[rr * SCQ_SSTRIDE + i]);
        }
        cm[p * QLEN + i] = m;
    }
    __syncthreads();
    if (tid < QLEN) {
        float m = cm[tid];
#pragma unroll
        for (int p = 1; p < 8; ++p) m = fmaxf(m, cm[p * QLEN + tid]);
        tilemax[((int64_t)q * gridDim.x + blockIdx.x) * QLEN + tid] = m;
    }
}


// ------------------------------------------------------------------ matrix form
// Four waves of 32 rows measured best: eight waves of 16 rows (more waves per SIMD to fill the matrix pipe while
// others are in their epilogue) lose more to the per-wave epilogue instructions than they gain (5.2 vs 4.95 ms per 512
// queries on C = 65536), 64 rows per wave halve the occupancy.
#define SM_THREADS 256
#define SM_RT 2                      // 16-row tiles per wave
#define SM_WAVES (SM_THREADS / 64)
#define SM_WROWS (16 * SM_RT)        // centroid rows per wave
#define SM_ROWS (SM_WAVES * SM_WROWS)  // centroid rows per workgroup
static_assert(SM_WROWS == 16 || SM_WROWS == 32, "pruning bits are assembled from 16- or 32-row pieces");
static_assert(SM_ROWS % (SM_THREADS / 8) == 0 && SM_THREADS >= QLEN, "tile shape");
#define SM_KC 32                     // dimensions staged at a time
#define SM_ASTRIDE 36                // floats per staged row chunk: the 64 operand reads of a step hit 64 banks
#define SM_MIN_WAVES 4               // waves per SIMD the register allocation leaves room for

// Operand and result layout of v_mfma_f64_16x16x4_f64 for lane = 16 g + i: A operand = A[i][g], B operand = B[g][i],
// result register r = D[4 r + g][i].
__device__ __forceinline__ scq_double4 scq_mma(double a, double b, scq_double4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also waits for every outstanding global store, and
// this kernel has 16 KB of score stores in flight per query when it reaches the barriers that guard the LDS tile.
__device__ __forceinline__ void scq_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// NQ = queries per workgroup (1 or 2).  Grid: x = query group, y = row block.
// tilemax: [q][32-row block][32] column maxima over the 32 rows a wave owns (null: scores and pruning bits only).
template <int NQ>
__global__ __launch_bounds__(SM_THREADS, SM_MIN_WAVES) void scq_mfma_kernel(const float *__restrict__ Cm, int64_t C,
                                                              const float *__restrict__ Q, int nq, float t_cs,
                                                              float *__restrict__ S, uint32_t *__restrict__ keepbits,
                                                              int64_t keep_words, float *__restrict__ tilemax,
                                                              uint32_t *__restrict__ zero, int64_t zero_words)
{
    constexpr int NT = 2 * NQ;  // 16-column tiles
    __shared__ __align__(16) float arena[SM_ROWS * SM_ASTRIDE];  // staged centroid chunk
    __shared__ __align__(16) float Bq[(SM_KC / 4) * NT * 64];    // the chunk's query operands: [step][column tile][lane]
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Outside the matrix loop a wave runs at raised priority: its few vector instructions (set-up, staging, epilogue)
    // would otherwise wait their turn behind the matrix instructions of every other wave on the SIMD, and the sooner a
    // wave is through them, the sooner it feeds the matrix pipe again.
    __builtin_amdgcn_s_setprio(3);
    // the workspace words that later kernels expect to be zero are cleared here, by the whole grid (no kernel of this
    // search has touched them yet, and every kernel of the previous one has finished)
    for (int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * SM_THREADS + tid; i < zero_words;
         i += (int64_t)gridDim.x * gridDim.y * SM_THREADS)
        zero[i] = 0u;
    const int q0 = blockIdx.x * NQ;
    const int64_t c0 = (int64_t)blockIdx.y * SM_ROWS;
    const int nrows = (int)(C - c0 < SM_ROWS ? C - c0 : SM_ROWS);

    // staging: a chunk is SM_ROWS rows x 32 dims = 8 float4 per row; thread -> rows tid/8 + SM_RPP k, float4 column tid%8
    constexpr int SM_RPP = SM_THREADS / 8;  // rows per staging pass
    const int r0 = tid >> 3, c4 = tid & 7;
    float4 pre[SM_ROWS / SM_RPP];
#pragma unroll
    for (int k = 0; k < SM_ROWS / SM_RPP; ++k) {
        const int r = r0 + SM_RPP * k;
        pre[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r < nrows) pre[k] = *reinterpret_cast<const float4 *>(Cm + (c0 + r) * DIM + 4 * c4);
    }
    // The queries' operands of a chunk, in operand order [step][column tile][lane]: 8 steps x 2 halves x 64 lanes per
    // query, four consecutive lanes per thread: 256 threads per query, thread bt of them (zeros for a query past the
    // end).  Lane 16 g + i of step s, half h holds Q[16 h + i][4 s + g], so a thread's four values are one column of
    // four consecutive query tokens.
    static_assert(SM_THREADS % 256 == 0, "query staging works in groups of 256 threads");
    constexpr int BQ_PASSES = (NQ * 256 + SM_THREADS - 1) / SM_THREADS;  // queries staged per thread
    const int bt = tid & 255;
    const int bdst = (((bt >> 5) * NT + ((bt >> 4) & 1)) * 64 + 4 * (bt & 15));  // + 2 qi column tiles
    const int bsrc = (16 * ((bt >> 4) & 1) + 4 * (bt & 3)) * DIM + 4 * (bt >> 5) + ((bt >> 2) & 3);  // + 32 ch
    float4 preb[BQ_PASSES];
#pragma unroll
    for (int k = 0; k < BQ_PASSES; ++k) {
        const int qi = (tid >> 8) + (SM_THREADS / 256) * k;
        preb[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (qi < NQ && q0 + qi < nq) {
            const float *src = Q + (int64_t)(q0 + qi) * QLEN * DIM + bsrc;
            preb[k] = make_float4(src[0], src[DIM], src[2 * DIM], src[3 * DIM]);
        }
    }
    scq_double4 acc[SM_RT][NT];
#pragma unroll
    for (int m = 0; m < SM_RT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = scq_double4{0.0, 0.0, 0.0, 0.0};
    const float *arow = arena + (wave * SM_WROWS + li) * SM_ASTRIDE + lg;  // + 16 m rows, + 4 j floats
    const float *bcol = Bq + lane;
#pragma unroll 1
    for (int ch = 0; ch < DIM / SM_KC; ++ch) {
#pragma unroll
        for (int k = 0; k < SM_ROWS / SM_RPP; ++k)
            *reinterpret_cast<float4 *>(arena + (r0 + SM_RPP * k) * SM_ASTRIDE + 4 * c4) = pre[k];
#pragma unroll
        for (int k = 0; k < BQ_PASSES; ++k) {
            const int qi = (tid >> 8) + (SM_THREADS / 256) * k;
            if (qi < NQ) *reinterpret_cast<float4 *>(Bq + bdst + 2 * qi * 64) = preb[k];
        }
        scq_lds_barrier();
        if (ch + 1 < DIM / SM_KC) {
#pragma unroll
            for (int k = 0; k < SM_ROWS / SM_RPP; ++k) {
                const int r = r0 + SM_RPP * k;
                if (r < nrows) pre[k] = *reinterpret_cast<const float4 *>(Cm + (c0 + r) * DIM + SM_KC * (ch + 1) + 4 * c4);
            }
#pragma unroll
            for (int k = 0; k < BQ_PASSES; ++k) {
                const int qi = (tid >> 8) + (SM_THREADS / 256) * k;
                if (qi < NQ && q0 + qi < nq) {
                    const float *src = Q + (int64_t)(q0 + qi) * QLEN * DIM + bsrc + SM_KC * (ch + 1);
                    preb[k] = make_float4(src[0], src[DIM], src[2 * DIM], src[3 * DIM]);
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int j = 0; j < SM_KC / 4; ++j) {
            double a[SM_RT], b[NT];
#pragma unroll
            for (int m = 0; m < SM_RT; ++m) a[m] = (double)arow[16 * m * SM_ASTRIDE + 4 * j];
#pragma unroll
            for (int t = 0; t < NT; ++t) b[t] = (double)bcol[(j * NT + t) * 64];
#pragma unroll
            for (int m = 0; m < SM_RT; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[m][t] = scq_mma(a[m], b[t], acc[m][t]);
        }
        __builtin_amdgcn_s_setprio(3);
        if (ch + 1 < DIM / SM_KC) scq_lds_barrier();  // every wave is done with this chunk: the arena is rewritten next
    }

    // Epilogue, straight from the accumulators (no LDS, no barrier: every vector instruction here queues behind the
    // matrix instructions of the other waves on the SIMD, so the fewer the better).  Lane 16 g + i holds rows 4 r + g of
    // columns i and 16 + i of each 16-row tile: a store instruction writes four 64-byte row halves, the two halves of
    // a row back to back.  Eq. 5: the comparison's lane mask holds, in its 16-bit field g, the columns of row 4 r + g, so
    // a row passes when its field is not zero -- scalar work on the mask, none per lane.
    const bool ragged = nrows < SM_ROWS;  // rows past the end of the table hold zeros: not stored, not in a maximum
    const int wrow0 = wave * SM_WROWS;
    const int wrows = nrows - wrow0 < 0 ? 0 : (nrows - wrow0 < SM_WROWS ? nrows - wrow0 : SM_WROWS);  // this wave's rows
    static_assert(SM_WROWS == 32, "one word of the pruning bitmap per wave");
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi) {
        const int q = q0 + qi;
        if (q >= nq) break;  // uniform
        uint32_t kbits = 0u;                     // uniform: bit = row within the wave's 32 rows
        float cm0 = -INFINITY, cm1 = -INFINITY;  // maxima of this lane's two columns (tokens li and 16 + li) over its rows
        float *srow = S + ((int64_t)q * C + c0 + wrow0 + lg) * QLEN + li;
#pragma unroll
        for (int m = 0; m < SM_RT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * m + 4 * r;  // + lg
                const float v0 = (float)acc[m][2 * qi][r], v1 = (float)acc[m][2 * qi + 1][r];
                if (!ragged || row + lg < wrows) {
                    srow[row * QLEN] = v0;
                    srow[row * QLEN + 16] = v1;
                    // med3(a, b, +inf) = max(a, b) for ordered operands, without the canonicalising copies of fmaxf
                    cm0 = __builtin_amdgcn_fmed3f(cm0, v0, INFINITY);
                    cm1 = __builtin_amdgcn_fmed3f(cm1, v1, INFINITY);
                }
                const unsigned long long pass = __ballot(v0 >= t_cs || v1 >= t_cs);
                const uint32_t lo = (uint32_t)pass, hi = (uint32_t)(pass >> 32);
                const uint32_t nib = ((lo & 0xFFFFu) ? 1u : 0u) | ((lo >> 16) ? 2u : 0u) | ((hi & 0xFFFFu) ? 4u : 0u) |
                                     ((hi >> 16) ? 8u : 0u);
                kbits |= nib << row;
            }
        if (tilemax) {  // uniform
            cm0 = __builtin_amdgcn_fmed3f(cm0, __shfl_xor(cm0, 16), INFINITY);
            cm1 = __builtin_amdgcn_fmed3f(cm1, __shfl_xor(cm1, 16), INFINITY);
            cm0 = __builtin_amdgcn_fmed3f(cm0, __shfl_xor(cm0, 32), INFINITY);
            cm1 = __builtin_amdgcn_fmed3f(cm1, __shfl_xor(cm1, 32), INFINITY);
            const int64_t blk = (int64_t)blockIdx.y * SM_WAVES + wave, n_blk = (C + SM_WROWS - 1) / SM_WROWS;
            if (lg == 0 && blk < n_blk) {  // a block with a row in range; rows past the end were left out above
                float *tmx = tilemax + ((int64_t)q * n_blk + blk) * QLEN + li;
                tmx[0] = cm0;
                tmx[16] = cm1;
            }
        }
        // rows past the end of the centroid table (a ragged last block) never pass
        if (wrows < SM_WROWS) kbits &= (1u << wrows) - 1u;
        const int64_t w0 = (c0 >> 5) + wave;  // one 32-bit word of the pruning bitmap per 32 rows
        if (lane == 0 && w0 < keep_words) keepbits[(int64_t)q * keep_words + w0] = kbits;
    }
}

// One wave: the matrix instruction chained over 128 dimensions against the chain of fused multiply-adds, on
// pseudo-random fp32 operands; mismatch[0] counts results whose bits differ.
__global__ __launch_bounds__(64) void scq_matrix_form_check_kernel(uint32_t seed, int32_t *__restrict__ mismatch)
{
    __shared__ float A[16][DIM], B[DIM][16];
    const int lane = threadIdx.x, li = lane & 15, lg = lane >> 4;
    uint32_t x = seed * 2654435761u + (uint32_t)lane * 40503u + 12345u;
    for (int e = lane; e < 16 * DIM; e += 64) {
        x = x * 1664525u + 1013904223u;
        (&A[0][0])[e] = (float)(int32_t)(x >> 8) * (1.0f / 8388608.0f) - 1.0f;
        x = x * 1664525u + 1013904223u;
        (&B[0][0])[e] = (float)(int32_t)(x >> 8) * (1.0f / 8388608.0f) - 1.0f;
    }
    __syncthreads();
    scq_double4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < DIM / 4; ++s) acc = scq_mma((double)A[li][4 * s + lg], (double)B[4 * s + lg][li], acc);
    int bad = 0;
    for (int r = 0; r < 4; ++r) {
        const int row = 4 * r + lg;
        double c = 0.0;
        for (int k = 0; k < DIM; ++k) c = fma((double)A[row][k], (double)B[k][li], c);
        bad += __double_as_longlong(c) != __double_as_longlong(acc[r]) ? 1 : 0;
    }
    if (bad) atomicAdd(mismatch, bad);
}

int plaid_scq_matrix_form_ok(hipStream_t st, int *ok)
{
    *ok = 0;
    int32_t *d = nullptr;
    hipError_t e = hipMalloc((void **)&d, sizeof(int32_t));
    if (e != hipSuccess) return (int)e;
    int32_t h = -1;
    e = hipMemsetAsync(d, 0, sizeof(int32_t), st);
    for (uint32_t seed = 1; e == hipSuccess && seed <= 64; ++seed)
        hipLaunchKernelGGL(scq_matrix_form_check_kernel, dim3(1), dim3(64), 0, st, seed, d);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&h, d, sizeof(int32_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(d);
    if (e != hipSuccess) return (int)e;
    *ok = h == 0 ? 1 : 0;
    return 0;
}

// Probes and survivors of a query, a workgroup each (blockIdx.y): the two share nothing but their inputs, and each is a
// chain of dependent steps of a microsecond, so that side by side they take half the time (one query of 400 000 passages,
// 65536 centroids: 40 us one after the other, with the tiles' maxima read twice over by one workgroup and the rows to
// re-evaluate fetched in four round trips; 19 now; 8.8 M passages, 262144 centroids 79 -> 27; 10 000, 1024 27 -> 12.5).
//
// Probes (rank order), from the column maxima of the score kernel's tiles, and their ascending duplicate-free union.  Where
// there are many tiles the split-fp16 kernel also reports the maxima of groups of 2^gs of them; otherwise a tile is its own group.  gmax is
// [group][token]: a thread reads four tokens of every 128th group (16-byte loads, consecutive threads at consecutive
// addresses, eight loads in flight) and keeps their largest values; its rows are one of 128 blocks.  Then 32 consecutive
// lanes share a token: the nprobe-th largest of the block maxima (nprobe rounds of "maximum over the 32 lanes, its first
// holder drops it"), and the groups whose maximum reaches it, listed in LDS; the same once more over the tiles of those
// groups gives T, the nprobe-th largest tile maximum, and the tiles whose maximum is >= T (normally nprobe of them; a tie
// group too long for a list makes the lanes walk all tiles instead).  Their rows with a score >= T are ranked by (score
// descending, id ascending).  tile_rows = centroid rows per tile.
//
// APPROX: S, its tile maxima and the pruning bits come from the split-fp16 kernel, every entry within eps =
// PLAID_SCQ16_EPS of the exact one.  The decisions stay those of the exact scores:
//   probes   at least nprobe entries are >= T (approximately), hence >= T - eps exactly, so the nprobe-th best exact
//            score is >= T - eps and every centroid among the nprobe best has an approximate score >= T - 2 eps.  The
//            tiles with maximum >= T - 2 eps are listed, and each of their rows with a score >= T - 2 eps (normally
//            just the nprobe best) is re-evaluated in double and ranked by its exact score;
//   pruning  a row whose approximate maximum lies within eps of t_cs was left open by the score kernel (ambbits): its
//            entries >= t_cs - eps are re-evaluated and the row's bit is set when one of them reaches t_cs;
//   table    the rows of the surviving centroids that stage 2 scores with are re-evaluated (stage1_survivor_table).
#define TAIL_FLY 8    // group maxima in flight per thread
#define TAIL_PARTS (TAIL_THREADS / (QLEN / 4))  // threads that share four tokens
#define TAIL_SEL 16   // listed groups, and listed tiles, per token
#define TAIL_XCAP 32  // listed rows per token: one per lane
// Rows staged at most for the re-evaluation of the probes, half of their dimensions at a time: 32 tokens with four each.  More of them
// (a near tie at nprobe 4, most queries from 5 on) are re-evaluated straight from memory, a lane each.  At 128 rows each wave has one
// tile; no step shows there.  Probe kernel, us, 65536 centroids, nprobe 2 / 3 / 4 / 5 / 6 / 8: one query 19.4 / 24.4 / 29.0 / 32.3 /
// 35.7 / 43.4, 32 queries 20.4 / 25.8 / 31.1 / 33.6 / 37.2 / 45.2, 512 81 / 107 / 125 / 142 / 157 / 190.
#define TAIL_ROWS 128
#define TAIL_HSTRIDE (DIM / 2 + 4)  // floats per staged half row
struct Stage1Exact {        // what the re-evaluations need (APPROX only)
    const float *Cm;        // [C][128] centroids
    const float *Q;         // [nq][32][128] queries
    const uint32_t *ambbits;  // [nq][keep_words]
    float t_cs, t_lo;       // threshold of Eq. 5 and the smallest approximate score that can still reach it
    float margin;           // 2 eps
    bool matrix;            // the double-precision matrix instruction gives the definition's bits
};
// The query's rows to LDS, TAIL_QSTRIDE floats apart.
__device__ __forceinline__ void tail_stage_query(const float *__restrict__ Q, int q, float *Qs)
{
    static_assert(TAIL_THREADS * 4 == QLEN * DIM, "one 16-byte load per thread stages the query");
    const int tid = threadIdx.x;
    *reinterpret_cast<float4 *>(Qs + (tid / (DIM / 4)) * TAIL_QSTRIDE + 4 * (tid % (DIM / 4))) =
        *reinterpret_cast<const float4 *>(Q + (int64_t)q * QLEN * DIM + 4 * tid);
}

template <bool APPROX>
struct ProbeScratch {
    float Qs[APPROX ? QLEN * TAIL_QSTRIDE : 4];
    union {
        float block[4 * TAIL_LANES][QLEN + 4];                // each thread's largest group maximum of its tokens
        float row[APPROX ? TAIL_ROWS * TAIL_HSTRIDE : 4];   // later: half of the dimensions of the rows to re-evaluate
    };
    union {
        int32_t sel_grp[QLEN][TAIL_SEL];   // listed groups
        float xscore[QLEN][TAIL_XCAP];     // later: exact scores of the listed rows
    };
    int32_t xc_id[QLEN][TAIL_XCAP];    // the listed rows
    int32_t xc_cnt[QLEN], xc_first[QLEN + 1];
    int16_t row_of[TAIL_ROWS];       // token and place among its listed rows of the rows that are staged
    int32_t sel_tile[QLEN][TAIL_SEL];  // listed tiles
    int32_t grp_cnt[QLEN], tile_cnt[QLEN];
    float Tsh[QLEN];
    int32_t wave_n[4];
    alignas(16) int32_t idl[256];    // probed ids
    int32_t sorted[256];
};

// Maximum over the 32 lanes of a token (every lane gets it): rotations within rows of sixteen lanes, then the other row's.
__device__ __forceinline__ float tail_max32(float m)
{
#define TAIL_ROR(n) __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(m), 0x120 + (n), 0xf, 0xf, false))
    m = fmaxf(m, TAIL_ROR(8));
    m = fmaxf(m, TAIL_ROR(4));
    m = fmaxf(m, TAIL_ROR(2));
    m = fmaxf(m, TAIL_ROR(1));
#undef TAIL_ROR
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// The nprobe-th largest of the values the 32 lanes of a token hold, four each (-infinity where there are fewer).
__device__ __forceinline__ float tail_nth_largest(float (&v)[4], int nprobe, int l)
{
    // each lane's in descending order, so that it drops the first
    auto order = [&](int a, int b) {
        const float x = v[a], y = v[b];
        v[a] = fmaxf(x, y);
        v[b] = fminf(x, y);
    };
    order(0, 1), order(2, 3), order(0, 2), order(1, 3), order(1, 2);
    float T = tail_max32(v[0]);
    for (int r = 1; r < nprobe; ++r) {  // uniform
        const unsigned long long who = __ballot(v[0] == T);
        const uint32_t half = (threadIdx.x & 32) ? (uint32_t)(who >> 32) : (uint32_t)who;  // this token's 32 lanes
        if (l == __ffs(half) - 1) v[0] = v[1], v[1] = v[2], v[2] = v[3], v[3] = -INFINITY;  // the first holder drops it
        T = tail_max32(v[0]);
    }
    return T;
}

// TOK query tokens from t0 on: all of them, or TAIL_TOKENS (APPROX only), by as many waves as they need; the others leave.  Then the
// probed ids are left as they are, token by token, in the place of their union.
#define TAIL_TOKENS 8
template <int NP, bool APPROX, int TOK>
__device__ __forceinline__ void tail_probes(ProbeScratch<APPROX> &sh, int q, int t0, const float *__restrict__ S, int64_t C,
                                            const float *__restrict__ tmq, int nblk, int tile_rows, const float *__restrict__ gmq,
                                            int ng, int gs, int nprobe, const Stage1Out o, const Stage1Exact x)
{
    static_assert(TAIL_LANES == 32, "32 lanes per query token");
    static_assert(TOK == QLEN || (APPROX && TOK == TAIL_TOKENS && 16 % TOK == 0), "whole waves, and one tile of sixteen tokens");
    constexpr int THREADS = TOK * TAIL_LANES, ROWS = TAIL_ROWS * TOK / QLEN;
    const int tid = threadIdx.x;
    if (TOK < QLEN && tid >= THREADS) return;  // whole waves
    const float *__restrict__ Sq = S + (int64_t)q * C * QLEN;
    const float margin = APPROX ? x.margin : 0.f;
    const int q16 = t0 & ~15;  // a part's sixteen tokens of a tile
    if constexpr (APPROX && TOK < QLEN) {
#pragma unroll
        for (int e = tid; e < 16 * (DIM / 4); e += THREADS)
            *reinterpret_cast<float4 *>(sh.Qs + (q16 + e / (DIM / 4)) * TAIL_QSTRIDE + 4 * (e % (DIM / 4))) =
                *reinterpret_cast<const float4 *>(x.Q + ((int64_t)q * QLEN + q16) * DIM + 4 * e);
    } else if (APPROX) {
        tail_stage_query(x.Q, q, sh.Qs);
    }
    // pass 1: the maxima of groups part, part + 128, ... of tokens 4 tk4 .. 4 tk4 + 3, one block of rows per thread
    const int tk4 = tid % (TOK / 4), part = tid / (TOK / 4);
    static_assert(THREADS / (TOK / 4) == TAIL_PARTS, "as many threads share four tokens");
    float4 g[TAIL_FLY];  // the first of them stay in registers
    auto load = [&](int b0) {
#pragma unroll
        for (int u = 0; u < TAIL_FLY; ++u) {
            const int b = b0 + TAIL_PARTS * u;
            g[u] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (b < ng) g[u] = *reinterpret_cast<const float4 *>(gmq + (int64_t)b * QLEN + t0 + 4 * tk4);
        }
    };
    float4 most = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    for (int b0 = part; b0 < ng; b0 += TAIL_PARTS * TAIL_FLY) {
        load(b0);
#pragma unroll
        for (int u = 0; u < TAIL_FLY; ++u)
            most = make_float4(fmaxf(most.x, g[u].x), fmaxf(most.y, g[u].y), fmaxf(most.z, g[u].z), fmaxf(most.w, g[u].w));
    }
    *reinterpret_cast<float4 *>(&sh.block[part][4 * tk4]) = most;
    __syncthreads();
    const int i = tid / TAIL_LANES, l = tid % TAIL_LANES;  // the token (of TOK) that this lane shares, its number among those that do
    const int tok = t0 + i;
    {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = sh.block[l + TAIL_LANES * u][i];
        static_assert(TAIL_PARTS == 4 * TAIL_LANES, "four blocks per lane");
        const float T0 = tail_nth_largest(v, nprobe, l);
        if (l == 0) {
            sh.Tsh[i] = T0;
            sh.grp_cnt[i] = 0;
            sh.tile_cnt[i] = 0;
            sh.xc_cnt[i] = 0;
        }
    }
    __syncthreads();
    {
        // pass 2, same thread -> (tokens, groups) map: list the groups that can hold one of the nprobe best
        const float T4[4] = {sh.Tsh[4 * tk4] - margin, sh.Tsh[4 * tk4 + 1] - margin, sh.Tsh[4 * tk4 + 2] - margin,
                             sh.Tsh[4 * tk4 + 3] - margin};
        for (int b0 = part; b0 < ng; b0 += TAIL_PARTS * TAIL_FLY) {
            if (ng > TAIL_PARTS * TAIL_FLY) load(b0);  // uniform
#pragma unroll
            for (int u = 0; u < TAIL_FLY; ++u) {
                const int b = b0 + TAIL_PARTS * u;
                const float e[4] = {g[u].x, g[u].y, g[u].z, g[u].w};
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (b < ng && e[c] >= T4[c]) {
                        const int pos = atomicAdd(&sh.grp_cnt[4 * tk4 + c], 1);
                        if (pos < TAIL_SEL) sh.sel_grp[4 * tk4 + c][pos] = b;
                    }
            }
        }
    }
    __syncthreads();
    float T;  // the nprobe-th largest tile maximum (or a smaller value that nprobe rows reach), less the margin
    {
        // tiles of the listed groups (of all, when too many groups tie): up to four per lane stay in registers
        const bool listed = sh.grp_cnt[i] <= TAIL_SEL;
        const int n_tiles = listed ? sh.grp_cnt[i] << gs : nblk;
        auto tile_of = [&](int it) { return listed ? (sh.sel_grp[i][it >> gs] << gs) + (it & ((1 << gs) - 1)) : it; };
        float v[4], kept[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int it = l + TAIL_LANES * u, t = it < n_tiles ? tile_of(it) : nblk;
            v[u] = kept[u] = t < nblk ? tmq[(int64_t)t * QLEN + tok] : -INFINITY;
        }
        for (int it = l + 4 * TAIL_LANES; it < n_tiles; it += TAIL_LANES) {  // more than that: a lane's share is one block
            const int t = tile_of(it);
            if (t < nblk) kept[0] = fmaxf(kept[0], tmq[(int64_t)t * QLEN + tok]);
        }
        T = tail_nth_largest(kept, nprobe, l) - margin;
        auto list = [&](float m, int t) {
            if (m >= T) {
                const int pos = atomicAdd(&sh.tile_cnt[i], 1);
                if (pos < TAIL_SEL) sh.sel_tile[i][pos] = t;
            }
        };
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int it = l + TAIL_LANES * u;
            if (it < n_tiles && tile_of(it) < nblk) list(v[u], tile_of(it));
        }
        for (int it = l + 4 * TAIL_LANES; it < n_tiles; it += TAIL_LANES) {
            const int t = tile_of(it);
            if (t < nblk) list(tmq[(int64_t)t * QLEN + tok], t);
        }
    }
    __syncthreads();
    {
        uint64_t best[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) best[j] = PLAID_KEY_MAX;
        const int n_sel = sh.tile_cnt[i];
        const bool listed = n_sel <= TAIL_SEL;
        // 32-row pieces of a tile (one with approximate scores, which spares the divisions below)
        static_assert(SM_WROWS == TAIL_LANES, "a row per lane");
        const int rows = APPROX ? TAIL_LANES : tile_rows, chunks = (rows + TAIL_LANES - 1) / TAIL_LANES;
        const int n_items = (listed ? n_sel : nblk) * chunks;
        // walk: every listed row with its score; what happens to a row is up to `visit`
        constexpr int FLY = NP <= 2 ? 4 : 8;  // score rows in flight per lane
        auto walk = [&](auto visit) {
            for (int it0 = 0; it0 < n_items; it0 += FLY) {
                float sv[FLY];
                int64_t cc[FLY];
                bool ok[FLY];
#pragma unroll
                for (int u = 0; u < FLY; ++u) {
                    const int it = it0 + u;
                    ok[u] = it < n_items;
                    const int k = ok[u] ? it / chunks : 0, r = (it % chunks) * TAIL_LANES + l;
                    const int t = listed ? sh.sel_tile[i][k] : k;
                    if (!listed && ok[u]) ok[u] = tmq[(int64_t)t * QLEN + tok] >= T;
                    cc[u] = (int64_t)t * rows + r;
                    ok[u] = ok[u] && r < rows && cc[u] < C;
                    sv[u] = ok[u] ? Sq[cc[u] * QLEN + tok] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < FLY; ++u)
                    if (ok[u]) visit(sv[u], cc[u]);
            }
        };
        // (listed with no tile at all: scores that are not numbers; sel_tile is not read then, n_items is zero)
        bool ranked = false;  // the keys of this token are in LDS, to be ranked by counting
        int n_x = 0;
        if (!APPROX) {
            walk([&](float sv, int64_t cc) { scq_insert_key<NP>(best, plaid_make_key(sv, (uint32_t)cc)); });
        } else {
            // Only a row that can be among the nprobe best (score >= T - 2 eps) is ranked, and by its exact score.  The
            // rows are listed first and re-evaluated all at once: staged in LDS, a thread each.  A token with more such rows
            // than lanes (many equal scores) re-evaluates them as it meets them.
            walk([&](float sv, int64_t cc) {
                if (sv >= T) {
                    const int pos = atomicAdd(&sh.xc_cnt[i], 1);
                    if (pos < TAIL_XCAP) sh.xc_id[i][pos] = (int32_t)cc;
                }
            });
            __syncthreads();
            n_x = sh.xc_cnt[i];
            if (tid < 64) {  // where each token's rows start in the list of all
                const int n = tid < TOK && sh.xc_cnt[tid & (TOK - 1)] <= TAIL_XCAP ? sh.xc_cnt[tid & (TOK - 1)] : 0;
                int incl = n;
#pragma unroll
                for (int d = 1; d < QLEN; d <<= 1) {
                    const int below = __shfl_up(incl, d);
                    incl += tid >= d ? below : 0;
                }
                if (tid < TOK) sh.xc_first[tid] = incl - n;
                if (tid == TOK - 1) sh.xc_first[QLEN] = incl;
            }
            __syncthreads();
            const int n_all = sh.xc_first[QLEN];  // uniform
            ranked = n_x <= TAIL_XCAP;
            if (x.matrix && n_all <= ROWS) {
                // a token's lanes fetch its rows, a 16-byte piece per lane, all of them before the first is used; the lower half
                // of the dimensions is staged and multiplied, then the upper half (see tail_exact_rows; a wave keeps its tiles'
                // sums in between)
                constexpr int PIECES = NP <= 2 ? 4 : 8;
                float4 piece[PIECES];
                const float *src = x.Cm + 4 * l;
                const int mine = ranked ? n_x : 0;
#pragma unroll
                for (int u = 0; u < PIECES; ++u) {
                    piece[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (u < mine) piece[u] = *reinterpret_cast<const float4 *>(src + (int64_t)sh.xc_id[i][u] * DIM);
                }
                if (ranked && l < n_x) sh.row_of[sh.xc_first[i] + l] = (int16_t)(i * TAIL_XCAP + l);
                // (tiles of 16 rows and 16 tokens: all the query's, or the one that a part's tokens lie in)
                constexpr int ACROSS = TOK == QLEN ? QLEN / 16 : 1, TILES = (ROWS / 16 * ACROSS + THREADS / 64 - 1) / (THREADS / 64);  // of a wave
                static_assert(TOK < QLEN || TILES * (THREADS / 64) == ROWS / 16 * ACROSS, "every wave has as many tiles");
                const int lane = tid & 63, li = lane & 15, lg = lane >> 4, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
                scq_double4 acc[TILES];
#pragma unroll
                for (int t = 0; t < TILES; ++t) acc[t] = scq_double4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
                for (int half = 0; half < 2; ++half) {
                    if (half) __syncthreads();  // the lower half is used
                    if (l / (TAIL_LANES / 2) == half) {
                        float *dst = sh.row + sh.xc_first[i] * TAIL_HSTRIDE + 4 * (l % (TAIL_LANES / 2));
#pragma unroll
                        for (int u = 0; u < PIECES; ++u)
                            if (u < mine) *reinterpret_cast<float4 *>(dst + u * TAIL_HSTRIDE) = piece[u];
                        for (int u = PIECES; u < mine; ++u)  // (near ties)
                            *reinterpret_cast<float4 *>(dst + u * TAIL_HSTRIDE) =
                                *reinterpret_cast<const float4 *>(src + (int64_t)sh.xc_id[i][u] * DIM);
                    }
                    __syncthreads();
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        const int at = wave + t * (THREADS / 64), r0 = 16 * (at / ACROSS), c0 = TOK == QLEN ? 16 * (at % ACROSS) : q16;
                        if (r0 < n_all) {  // uniform
                            const float *a = sh.row + (r0 + li) * TAIL_HSTRIDE + lg, *bq = sh.Qs + (c0 + li) * TAIL_QSTRIDE + half * (DIM / 2) + lg;
#pragma unroll 8
                            for (int k = 0; k < DIM / 8; ++k)
                                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[4 * k], (double)bq[4 * k], acc[t], 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    const int at = wave + t * (THREADS / 64), r0 = 16 * (at / ACROSS), c0 = (TOK == QLEN ? 16 * (at % ACROSS) : q16) - t0;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r0 + 4 * r + lg < n_all) {  // (the row's own token is the only one of interest)
                            const int of = sh.row_of[r0 + 4 * r + lg];
                            if (of / TAIL_XCAP == c0 + li) sh.xscore[c0 + li][of % TAIL_XCAP] = (float)acc[t][r];
                        }
                }
            } else if (ranked && l < n_x) {
                sh.xscore[i][l] = plaid_exact_dot(x.Cm + (int64_t)sh.xc_id[i][l] * DIM, sh.Qs + tok * TAIL_QSTRIDE);
            }
            if (!ranked)
                walk([&](float sv, int64_t cc) {
                    if (sv >= T) scq_insert_key<NP>(best, plaid_make_key(plaid_exact_dot(x.Cm + cc * DIM, sh.Qs + tok * TAIL_QSTRIDE), (uint32_t)cc));
                });
            __syncthreads();
        }
        // A list entry can only be missing when the scores are not numbers (a query holding NaN compares false against
        // every threshold): later kernels index the inverted lists with these ids, so such a slot gets centroid j
        // (nprobe <= C), never an id out of range.
        int32_t *probed_i = o.probed + ((int64_t)q * QLEN + tok) * nprobe;
        auto put = [&](int j, int32_t id) {
            probed_i[j] = id;
            if (TOK == QLEN) sh.idl[i * nprobe + j] = id;
            else o.uniq[(int64_t)q * o.uniq_stride + tok * nprobe + j] = id;
        };
        if (__any(!ranked)) {
            // shuffle tree over the 32 lanes of this token (lanes l and l ^ d exchange lists; both keep the merged list)
#pragma unroll
            for (int d = 1; d < TAIL_LANES; d <<= 1) {
                uint64_t other[NP];
#pragma unroll
                for (int j = 0; j < NP; ++j) other[j] = __shfl_xor(best[j], d);
#pragma unroll
                for (int j = 0; j < NP; ++j) scq_insert_key<NP>(best, other[j]);
            }
        }
        if (ranked) {
            // each key's rank by counting (keys are unique)
            if (l < n_x) {
                const uint64_t key = plaid_make_key(sh.xscore[i][l], (uint32_t)sh.xc_id[i][l]);
                int rank = 0;
                for (int j = 0; j < n_x; ++j) rank += plaid_make_key(sh.xscore[i][j], (uint32_t)sh.xc_id[i][j]) < key ? 1 : 0;
                if (rank < nprobe) put(rank, (int32_t)(key & 0xFFFFFFFFu));
            }
            if (l >= n_x && l < nprobe) put(l, l);
        } else if (l == 0) {
#pragma unroll
            for (int j = 0; j < NP; ++j)
                if (j < nprobe) put(j, best[j] == PLAID_KEY_MAX ? j : (int32_t)(best[j] & 0xFFFFFFFFu));
        }
    }
    if (TOK < QLEN) {
        if (t0 == 0 && tid == 0) o.n_uniq[q] = QLEN * nprobe;
        return;
    }
    __syncthreads();
    // ascending duplicate-free union of the n = 32 * nprobe (<= 256) probed ids: each id's place in sorted order by counting
    // (four lanes share the comparisons, four ids per read), then those that differ from the id before them
    {
        const int n = QLEN * nprobe;
        const int t = tid >> 2, part = tid & 3;
        const int32_t id = t < n ? sh.idl[t] : 0x7FFFFFFF;
        int place = 0;
        if (t < n)
#pragma unroll 2
            for (int u = 4 * part; u < n; u += 16) {
                const int4 v = *reinterpret_cast<const int4 *>(sh.idl + u);
                place += (v.x < id || (v.x == id && u < t) ? 1 : 0) + (v.y < id || (v.y == id && u + 1 < t) ? 1 : 0) +
                         (v.z < id || (v.z == id && u + 2 < t) ? 1 : 0) + (v.w < id || (v.w == id && u + 3 < t) ? 1 : 0);
            }
        place += __shfl_xor(place, 1);
        place += __shfl_xor(place, 2);
        if (part == 0 && t < n) sh.sorted[place] = id;
        __syncthreads();
        if (tid < 256) {  // four whole waves
            const bool first = tid < n && (tid == 0 || sh.sorted[tid] != sh.sorted[tid - 1]);
            const unsigned long long m = __ballot(first);
            if ((tid & 63) == 0) sh.wave_n[tid >> 6] = __popcll(m);
        }
        __syncthreads();
        if (tid < n) {
            const int32_t v = sh.sorted[tid];
            const bool first = tid == 0 || v != sh.sorted[tid - 1];
            const unsigned long long m = __ballot(first);
            int before = 0;
            for (int w = 0; w < (tid >> 6); ++w) before += sh.wave_n[w];
            if (first) o.uniq[(int64_t)q * o.uniq_stride + before + __popcll(m & ((1ull << (tid & 63)) - 1ull))] = v;
        }
        if (tid == 0) o.n_uniq[q] = sh.wave_n[0] + sh.wave_n[1] + sh.wave_n[2] + sh.wave_n[3];
    }
}

template <bool APPROX>
struct TableScratch {
    SurvivorScratch t;
    SurvivorRows x[APPROX ? 1 : 0];
};

template <bool APPROX>
__device__ __forceinline__ void tail_survivors(TableScratch<APPROX> &ts, int q, const float *__restrict__ S, int64_t C,
                                               uint32_t *__restrict__ kbq, int64_t keep_words, const float *__restrict__ gmq, int ng,
                                               const Stage1Out o, const Stage1Exact x)
{
    SurvivorScratch &sh = ts.t;
    const int tid = threadIdx.x;
    const float *__restrict__ Sq = S + (int64_t)q * C * QLEN;
    const uint32_t *abq = APPROX ? x.ambbits + (int64_t)q * keep_words : nullptr;
    if (tid == 0) {
        sh.misc[0] = 0;
        sh.misc[1] = -1;
        sh.amb_total = 0;
    }
    if (APPROX) tail_stage_query(x.Q, q, ts.x[0].Qs);
    if (APPROX && tid == 0) ts.x[0].matrix = x.matrix;
    __syncthreads();
    // (a thread's instructions take the time here, sixteen waves on one compute unit: no more words than it has)
    if (keep_words <= 2ll * TAIL_THREADS) stage1_list_survivors<2>(kbq, abq, keep_words, sh);
    else stage1_list_survivors<8>(kbq, abq, keep_words, sh);
    __syncthreads();
    if (APPROX) {
        // Eq. 5 for the rows the score kernel left open.  Rounds of at most TAIL_AMB rows: the rows of a range of bitmap
        // words are listed in LDS, then their 32 entries each are spread over the workgroup; a row that passes joins the
        // survivors, once, and its bit the pruning words that later kernels read.  (One round, a handful of rows, unless the
        // threshold sits where many row maxima do.)
        const int total = sh.amb_total;  // uniform
        // words taken per round: all of them when every open row fits the list (the usual case: one round), else as
        // many as always fit
        const int64_t round_words = total <= TAIL_AMB ? keep_words : TAIL_AMB / 32;
        for (int64_t w0 = 0; total > 0 && w0 < keep_words; w0 += round_words) {
            int32_t *amb_rows = ts.x[0].amb;
            __syncthreads();
            if (tid == 0) sh.amb_n = 0;
            if (tid < TAIL_AMB / 32) sh.amb_pass[tid] = 0u;
            __syncthreads();
            const int64_t w1 = w0 + round_words < keep_words ? w0 + round_words : keep_words;
            for (int64_t w = w0 + tid; w < w1; w += TAIL_THREADS) {
                uint32_t v = abq[w];
                while (v) {
                    const int b = __ffs(v) - 1;
                    v &= v - 1;
                    amb_rows[atomicAdd(&sh.amb_n, 1)] = (int32_t)(w * 32 + b);
                }
            }
            __syncthreads();
            const int n_amb = sh.amb_n;
            for (int p = tid; p < n_amb * QLEN; p += TAIL_THREADS) {
                const int32_t c = amb_rows[p >> 5];
                const int tok = p & 31;
                if (Sq[(int64_t)c * QLEN + tok] >= x.t_lo &&
                    plaid_exact_dot(x.Cm + (int64_t)c * DIM, ts.x[0].Qs + tok * TAIL_QSTRIDE) >= x.t_cs) {
                    const uint32_t bit = 1u << ((p >> 5) & 31);
                    if (!(atomicOr(&sh.amb_pass[p >> 10], bit) & bit)) {  // the first of the row's entries
                        atomicOr(&kbq[c >> 5], 1u << (c & 31));
                        const int pos = atomicAdd(&sh.misc[0], 1);
                        if (pos < S2_MAX_KEPT) sh.ids[pos] = c;
                    }
                }
            }
        }
        __syncthreads();
    }
    auto col_max = [&](float *colmm) {  // over the groups' maxima
        float m = -INFINITY;
        for (int64_t e = tid; e < (int64_t)ng * QLEN; e += TAIL_THREADS) m = fmaxf(m, gmq[e]);
        float *part = sh.Tx;  // [the waves' halves][32]
        part[tid] = m;
        __syncthreads();
        if (tid < QLEN) {
            for (int w = 1; w < TAIL_THREADS / QLEN; ++w) m = fmaxf(m, part[w * QLEN + tid]);
            colmm[tid] = m;
        }
    };
    static_assert(TAIL_THREADS <= S2_MAX_KEPT * TX_STRIDE, "the partial maxima take the place of the survivors' entries");
    stage1_survivor_table<APPROX>(Sq, C, col_max, o.meta + q, o.kept_ids + (int64_t)q * S2_MAX_KEPT,
                                  o.T + (int64_t)q * (S2_MAX_KEPT + 1) * QLEN, sh, APPROX ? ts.x : nullptr, x.Cm, o.ivf_offsets, q, o.qcount,
                                  o.qlist, o.qlist_stride, o.list_counts, o.need_hash);
}

template <int NP, bool APPROX>
__global__ __launch_bounds__(TAIL_THREADS) void stage1_tail_kernel(const float *__restrict__ S, int64_t C,
                                                                   uint32_t *__restrict__ keepbits, int64_t keep_words,
                                                                   const float *__restrict__ tilemax, int nblk, int tile_rows,
                                                                   const float *__restrict__ gmax, int ng, int gs,
                                                                   int nprobe, Stage1Out o, Stage1Exact x)
{
    __shared__ __align__(16) union {
        ProbeScratch<APPROX> p;
        TableScratch<APPROX> t;
    } sh;
    const int q = blockIdx.x;
    const float *gmq = gmax + (int64_t)q * ng * QLEN;
    if (blockIdx.y == 0)
        tail_probes<NP, APPROX, QLEN>(sh.p, q, 0, S, C, tilemax + (int64_t)q * nblk * QLEN, nblk, tile_rows, gmq, ng, gs, nprobe, o, x);
    else
        tail_survivors<APPROX>(sh.t, q, S, C, keepbits + (int64_t)q * keep_words, keep_words, gmq, ng, o, x);
}

// The same with a workgroup per TAIL_TOKENS query tokens (blockIdx.y; the last one: the survivors).
template <int NP>
__global__ __launch_bounds__(TAIL_THREADS) void stage1_parts_kernel(const float *__restrict__ S, int64_t C, uint32_t *__restrict__ keepbits,
                                                                    int64_t keep_words, const float *__restrict__ tilemax, int nblk,
                                                                    const float *__restrict__ gmax, int ng, int gs, int nprobe, Stage1Out o,
                                                                    Stage1Exact x)
{
    __shared__ __align__(16) union {
        ProbeScratch<true> p;
        TableScratch<true> t;
    } sh;
    const int q = blockIdx.x;
    const float *gmq = gmax + (int64_t)q * ng * QLEN;
    if (blockIdx.y < QLEN / TAIL_TOKENS)
        tail_probes<NP, true, TAIL_TOKENS>(sh.p, q, TAIL_TOKENS * (int)blockIdx.y, S, C, tilemax + (int64_t)q * nblk * QLEN, nblk, SM_WROWS,
                                           gmq, ng, gs, nprobe, o, x);
    else
        tail_survivors<true>(sh.t, q, S, C, keepbits + (int64_t)q * keep_words, keep_words, gmq, ng, o, x);
}

// np = capacity of the tail's lists (1, 2, 4 or 8 >= nprobe); np = 0: scores and pruning bits only (large nprobe).
static void launch_fused(hipStream_t st, int phases, int np, const float *centroids, int64_t C, const float *Q, const void *Qx,
                         int form, bool matrix_ok, const void *A16, int nq, float t_cs, float *S, uint32_t *keepbits, uint32_t *ambbits,
                         int64_t keep_words, float *tilemax, float *groupmax, int nprobe, const Stage1Out &o, uint32_t *zero,
                         int64_t zero_words, unsigned long long *score_clocks)
{
    const bool matrix_form = form == PLAID_SCQ_MATRIX;
    const int tile_rows = form == PLAID_SCQ_VECTOR ? SCQ_ROWS : SM_WROWS;  // rows per tile of column maxima
    const int grid_rows = matrix_form ? SM_ROWS : SCQ_ROWS;   // rows per workgroup (the two double-precision forms)
    const unsigned nblk = (unsigned)((C + grid_rows - 1) / grid_rows);
    const int n_tiles = (int)((C + tile_rows - 1) / tile_rows);
    float *tmx = np > 0 ? tilemax : nullptr;
    static_assert(SM_WROWS == 32, "the split-fp16 kernel emits column maxima per 32 rows, like the matrix form");
    // The split-fp16 kernel reports maxima of groups of eight tiles too, where there is room for them and a query has more tiles
    // than the probe kernel has loads for in one round.  They cost the score kernel 2 to 4 %, and save the probe kernel a round
    // of loads per 1024 tiles.  Scores and probes together, us, with / without: one query of 65536 centroids 38 / 42, of 262144
    // 77 / 95; 512 queries of 65536 1009 / 1006, of 131072 1899 / 1936; 256 of 262144 1871 / 1930.  Up to 1024 tiles they save
    // nothing: 512 queries of 16384 centroids 327 / 323, of 32768 565 / 553, one of 32768 31.6 / 31.7.
    const bool grouped = form == PLAID_SCQ_SPLIT16 && tmx && groupmax && n_tiles > TAIL_PARTS * TAIL_FLY;
    static_assert(PLAID_SCQ16_GROUP_ROWS == SM_WROWS << 3, "eight tiles per group");
    const bool takes = form == PLAID_SCQ_SPLIT16 && plaid_scq16_takes_queries(C, nq, zero_words);
    if (!(phases & PLAID_STAGE1_SCORES)) {
    } else if (form == PLAID_SCQ_SPLIT16) {
        plaid_launch_scq16(st, A16, C, Qx, nq, t_cs, S, keepbits, ambbits, keep_words, tmx, grouped ? groupmax : nullptr, score_clocks,
                           takes ? Q : nullptr, takes ? zero : nullptr, takes ? zero_words : 0);
    } else if (matrix_form) {
        if (nq == 1)
            hipLaunchKernelGGL(scq_mfma_kernel<1>, dim3(1, nblk), dim3(SM_THREADS), 0, st, centroids, C, Q, nq, t_cs, S, keepbits,
                               keep_words, tmx, zero, zero_words);
        else
            hipLaunchKernelGGL(scq_mfma_kernel<2>, dim3((unsigned)((nq + 1) / 2), nblk), dim3(SM_THREADS), 0, st, centroids, C, Q,
                               nq, t_cs, S, keepbits, keep_words, tmx, zero, zero_words);
    } else {
        hipLaunchKernelGGL(scq_fused_kernel, dim3(nblk, nq), dim3(SCQ_THREADS), 0, st, centroids, C, (const double *)Qx, t_cs, S,
                           keepbits, keep_words, tmx);
    }
    if (np > 0 && (phases & PLAID_STAGE1_PROBES)) {
        Stage1Exact x;
        x.Cm = centroids;
        x.Q = Q;
        x.ambbits = ambbits;
        x.t_cs = t_cs;
        x.t_lo = (t_cs > -INFINITY && t_cs < INFINITY) ? nextafterf(t_cs - PLAID_SCQ16_EPS, -INFINITY) : t_cs;
        x.margin = 2.0f * PLAID_SCQ16_EPS;
        x.matrix = matrix_ok;
        const int gs = grouped ? 3 : 0, ng = (n_tiles + (1 << gs) - 1) >> gs;
        const float *gmx = grouped ? groupmax : tilemax;
#define TAIL(NP_, AP_)                                                                                                     \
    hipLaunchKernelGGL((stage1_tail_kernel<NP_, AP_>), dim3(nq, 2), dim3(TAIL_THREADS), 0, st, S, C, keepbits, keep_words, \
                       tilemax, n_tiles, tile_rows, gmx, ng, gs, nprobe, o, x)
#define PARTS(NP_)                                                                                                              \
    hipLaunchKernelGGL(stage1_parts_kernel<NP_>, dim3(nq, QLEN / TAIL_TOKENS + 1), dim3(TAIL_THREADS), 0, st, S, C, keepbits, keep_words, \
                       tilemax, n_tiles, gmx, ng, gs, nprobe, o, x)
        if (form == PLAID_SCQ_SPLIT16 && o.probes_apart) {
            if (np == 1) PARTS(1);
            else if (np == 2) PARTS(2);
            else if (np == 4) PARTS(4);
            else PARTS(8);
        } else if (form == PLAID_SCQ_SPLIT16) {
            if (np == 1) TAIL(1, true);
            else if (np == 2) TAIL(2, true);
            else if (np == 4) TAIL(4, true);
            else TAIL(8, true);
        } else {
            if (np == 1) TAIL(1, false);
            else if (np == 2) TAIL(2, false);
            else if (np == 4) TAIL(4, false);
            else TAIL(8, false);
        }
#undef TAIL
#undef PARTS
    }
}

size_t plaid_stage1_tilemax_bytes(int64_t C, int nq, int nprobe)
{
    if (nprobe > PLAID_PROBE_FAST_MAX) return 256;
    const int rows = SM_WROWS < SCQ_ROWS ? SM_WROWS : SCQ_ROWS;  // sized for the smaller of the two tile heights
    return (size_t)nq * ((C + rows - 1) / rows) * QLEN * 4;
}

size_t plaid_stage1_groupmax_bytes(int64_t C, int nq)
{
    return (size_t)nq * ((C + PLAID_SCQ16_GROUP_ROWS - 1) / PLAID_SCQ16_GROUP_ROWS) * QLEN * 4;
}

void plaid_launch_stage1(hipStream_t st, int phases, const float *centroids, int64_t C, const float *Q, void *Qd, int form,
                         bool matrix_ok, const void *A16, int nq, float t_cs, int nprobe, float *S, uint32_t *keepbits, uint32_t *ambbits,
                         int64_t keep_words, float *tilemax, float *groupmax, uint32_t *zero, int64_t zero_words, int32_t *probed,
                         int32_t *uniq, int uniq_stride, int32_t *n_uniq, const Stage2Buffers &s2, void *probe_scratch,
                         size_t probe_scratch_bytes, unsigned long long *score_clocks)
{
    if ((phases & PLAID_STAGE1_PREP) && form == PLAID_SCQ_SPLIT16 && !plaid_scq16_takes_queries(C, nq, zero_words))
        plaid_launch_scq16_split_queries(st, Q, nq, Qd, zero, zero_words);
    if ((phases & PLAID_STAGE1_PREP) && form == PLAID_SCQ_VECTOR) {
        int64_t gz = (zero_words + 256 * 8 - 1) / (256 * 8);
        if (gz < nq) gz = nq;
        if (gz > 1024) gz = 1024;
        hipLaunchKernelGGL(stage1_prep_kernel, dim3((unsigned)gz), dim3(256), 0, st, Q, (double *)Qd, nq, zero, zero_words);
    }
    if (!(phases & (PLAID_STAGE1_SCORES | PLAID_STAGE1_PROBES))) return;
    Stage1Out o;
    o.probed = probed;
    o.uniq = uniq;
    o.n_uniq = n_uniq;
    o.uniq_stride = uniq_stride;
    o.meta = s2.meta;
    o.kept_ids = s2.kept_ids;
    o.T = s2.T;
    o.ivf_offsets = s2.ivf_offsets;
    o.qcount = s2.qcount;
    o.qlist = s2.qlist;
    o.qlist_stride = s2.qlist_stride;
    o.list_counts = s2.list_counts;
    o.need_hash = s2.need_hash;
    o.probes_apart = s2.probes_apart;
    const int np = nprobe == 1 ? 1 : (nprobe == 2 ? 2 : (nprobe <= 4 ? 4 : (nprobe <= PLAID_PROBE_FAST_MAX ? 8 : 0)));
    if (np > 0)
        launch_fused(st, phases, np, centroids, C, Q, Qd, form, matrix_ok, A16, nq, t_cs, S, keepbits, ambbits, keep_words, tilemax, groupmax, nprobe,
                     o, zero, zero_words, score_clocks);
    else {
        // large nprobe: scores and pruning bits here, probes through the generic selection, survivor table after it
        launch_fused(st, phases, 0, centroids, C, Q, Qd, form, matrix_ok, A16, nq, t_cs, S, keepbits, ambbits, keep_words, tilemax, groupmax, nprobe,
                     o, zero, zero_words, score_clocks);
        if (phases & PLAID_STAGE1_PROBES) {
            plaid_launch_top_nprobe_general(st, S, C, nq, nprobe, probed, uniq, uniq_stride, n_uniq, probe_scratch,
                                            probe_scratch_bytes);
            hipLaunchKernelGGL(stage1_survivor_kernel, dim3(nq), dim3(512), 0, st, S, C, keepbits, keep_words, probed, nprobe, o);
        }
    }
}
