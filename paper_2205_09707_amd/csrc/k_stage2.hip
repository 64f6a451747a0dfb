// Stage 2: centroid interaction with centroid pruning (Eq. 3-5) over every candidate passage.
//
// A passage's pruned score is sum_i max_j S_cq[code_j][i] over its tokens whose centroid passes Eq. 5, so it depends only on
// WHICH surviving centroids occur in the passage.  Few centroids survive t_cs (a small tail of high scores, Section 3.4), so
// the work splits in two: find every passage's set of surviving centroids, then take the column maxima of the rows the set
// names (rows staged in LDS) and sum the 32 maxima in double, in index order.  No matrix D~ is ever stacked
// (Section 4.5's padding-free idea), nothing is padded, and the order-independent max plus the fixed-order sum make a
// score a pure function of the passage.  There are two forms:
//
//   streaming   the candidates' token codes are read once, coalesced, straight from HBM (128-byte lines that no candidate
//               touches are skipped); each code is looked up in a small LDS table of the K surviving centroids and turned
//               into a slot number; one lane per passage folds its slots into a K-bit set and scores it.  Queries with
//               more than S2_MAX_KEPT survivors (very low thresholds) take one wave per passage instead, which fetches the
//               surviving rows from S_cq.  Output per query: the score word of candidate p at position p of its region
//               (slots of non-candidates are neither written nor read), the fine histogram of the scores' bins, counted in
//               LDS and added once per workgroup, and the bitmap of the candidates whose bag is empty (score -infinity;
//               they rank last, in passage-id order).  No atomics with a return value on this path.
//   inverted    candidates and sets follow from the inverted lists, and only passages whose score bound reaches the best
//               ndocs so far are scored (see there).  Output per query: the keys of the scored candidates as a LIST, a
//               wave's positions in which come from one returning atomic per round of up to 2048 passages, the coarse
//               histogram of their bins, the candidate words and the bitmap of the empty bags.  Queries with more than
//               S2_MAX_KEPT survivors are scored from their token codes and leave what the streaming form leaves.
//
// A query without any surviving centroid skips all of this: its candidates are exactly its empty-bag set.
#include "plaid_internal.h"

#include <math.h>

#define S2_THREADS 256
#define S2W_PASS 64      // passages per wave tile = 2 words of the candidate bitmap
#define S2_ITEMS 9       // 16-byte loads per lane and round, all in flight at once
#define S2W_CAP (64 * 4 * S2_ITEMS - 32)  // tokens a wave stages per round (one byte each), whatever their alignment
#define S2_LBWORDS ((S2_ITEMS + 3) / 4)   // words of the round's line bitmap (8 lines per item)
#define S2_TSTRIDE 36    // floats per staged S_cq row (16-byte aligned, rows spread over the banks)
static_assert(S2_LBWORDS <= 64, "one lane clears one word of the line bitmap");

// ------------------------------------------------------------------ gather form (K > S2_MAX_KEPT) of the streaming kernel
// Pruned score of the passage with tokens [t0, t1): uniform across the wave; `any` tells whether a token survived.
__device__ __forceinline__ float s2_gather_passage(const float *__restrict__ Sq, const uint32_t *__restrict__ kb,
                                                   int64_t t0, int64_t t1, const int32_t *__restrict__ codes, int lane,
                                                   bool &any)
{
    const int i = lane & 31, h = lane >> 5;
    float m = -INFINITY;
    any = false;
    for (int64_t base = t0; base < t1; base += 64) {
        const int cnt = t1 - base < 64 ? (int)(t1 - base) : 64;
        const int32_t code = lane < cnt ? codes[base + lane] : 0;
        bool hit = lane < cnt;
        if (hit) hit = (kb[code >> 5] >> (code & 31)) & 1u;
        unsigned long long mask = __ballot(hit);
        any = any || mask != 0;
        while (mask) {
            const int j0 = __ffsll((long long)mask) - 1;
            mask &= mask - 1;
            int j1 = j0;
            if (mask) {
                j1 = __ffsll((long long)mask) - 1;
                mask &= mask - 1;
            }
            const int c = __shfl(code, h ? j1 : j0);
            m = fmaxf(m, Sq[(int64_t)c * QLEN + i]);
        }
    }
    m = fmaxf(m, __shfl_xor(m, 32));
    return plaid_sum32_in_order(m);
}

// Body for one query over the bitmap words w_first + k * w_step < w_end (32 passages each), one wave per word at a
// time; cb[w - cb_first] is the candidate word w (global memory or LDS).
__device__ __forceinline__ void s2_gather_body(int q, const float *__restrict__ S, int64_t C,
                                               const uint32_t *__restrict__ keepbits, int64_t keep_words, const uint32_t *cb,
                                               int64_t cb_first, int64_t w_first, int64_t w_step, int64_t w_end,
                                               int64_t cand_words, int64_t P, const int64_t *__restrict__ doc_offsets,
                                               const int32_t *__restrict__ codes, float bin_hi, float bin_scale,
                                               uint32_t *__restrict__ keys_out, int32_t *lhist,
                                               uint32_t *__restrict__ emptybits)
{
    const int lane = threadIdx.x & 63;
    const float *Sq = S + (int64_t)q * C * QLEN;
    const uint32_t *kb = keepbits + (int64_t)q * keep_words;
    uint32_t *eb = emptybits + (int64_t)q * cand_words;
    for (int64_t w = w_first; w < w_end; w += w_step) {
        const uint32_t word = cb[w - cb_first];
        if (!word) {
            if (lane == 0) eb[w] = 0u;
            continue;
        }
        const int64_t p0 = w * 32;
        int64_t off = 0;
        if (lane <= 32 && p0 + lane <= P) off = doc_offsets[p0 + lane];
        float my = -INFINITY;
        bool my_empty = false;
        uint32_t rest = word;
        while (rest) {
            const int b = __ffs(rest) - 1;
            rest &= rest - 1;
            const int64_t t0 = __shfl(off, b), t1 = __shfl(off, b + 1);
            bool any;
            const float sc = s2_gather_passage(Sq, kb, t0, t1, codes, lane, any);
            if (lane == b) {
                my = sc;
                my_empty = !any;
            }
        }
        const bool cand = lane < 32 && ((word >> lane) & 1u);
        const bool live = cand && !my_empty;
        if (cand) keys_out[p0 + lane] = live ? plaid_score_to_ord(my) : PLAID_S2_NO_SCORE;
        if (live) atomicAdd(&lhist[plaid_s2_bin(my, bin_hi, bin_scale)], 1);
        const unsigned long long e64 = __ballot(cand && my_empty);
        if (lane == 0) eb[w] = (uint32_t)e64;
    }
}

// ------------------------------------------------------------------ streaming form (K <= S2_MAX_KEPT)
// Survivor table entry: (centroid id << 6) | slot, 0xFFFFFFFF = free.  The hash is collision-free on the survivors,
// so one probe decides: returns the slot (1..63) of a surviving centroid, 0 otherwise.
__device__ __forceinline__ uint32_t s2_lookup(const uint32_t *htab, uint32_t code, int hash_shift)
{
    const uint32_t e = htab[(code ^ (code >> hash_shift)) & (S2_HASH - 1)] ^ (code << 6);
    return e < 64u ? e : 0u;
}

// LDS traffic between the lanes of one wave needs no workgroup barrier: a wave's LDS operations complete in
// program order.  This only stops the compiler from moving accesses across the hand-over point.
__device__ __forceinline__ void s2_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Every value that steers control flow below is wave-uniform and is forced into scalar registers with
// readfirstlane, so that all cross-lane operations (__shfl, __ballot) run with the full wave active.
__device__ __forceinline__ int s2_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// First set bit of m at position >= from, 64 when there is none (all operands uniform).
__device__ __forceinline__ int s2_next_bit(unsigned long long m, int from)
{
    const unsigned long long rest = from < 64 ? (m >> from) << from : 0ull;
    return rest ? __ffsll((long long)rest) - 1 : 64;
}

// End of a workgroup: its LDS bin counts go to the query's histogram (all threads of the workgroup call this).
__device__ __forceinline__ void s2_flush_hist(const int32_t *lhist, int32_t *__restrict__ hist_q)
{
    __syncthreads();
    for (int e = threadIdx.x; e < SEL_BINS; e += blockDim.x) {
        const int32_t n = lhist[e];
        if (n) atomicAdd(&hist_q[e], n);
    }
}

// Pruned score of a bag whose surviving centroids are the slots in `members` (non-empty, bit 0 clear): column maxima
// of those rows of the staged table, summed over the query tokens in index order; eight query tokens at a time, so
// that few registers are live.  A bag with one survivor takes that row's precomputed sum (same additions, same order).
__device__ __forceinline__ float s2_score_members(uint64_t members, const float *Tl, const float *rowsum)
{
    if ((members & (members - 1)) == 0) return rowsum[__ffsll((long long)members) - 1];
    double d = 0.0;
#pragma unroll 1
    for (int g = 0; g < QLEN / 8; ++g) {
        float acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = -INFINITY;
        uint64_t rest = members;
        while (rest) {
            const int s = __ffsll((long long)rest) - 1;
            rest &= rest - 1;
            const float4 *row = reinterpret_cast<const float4 *>(Tl + s * S2_TSTRIDE + 8 * g);
            const float4 r0 = row[0], r1 = row[1];
            acc[0] = fmaxf(acc[0], r0.x);
            acc[1] = fmaxf(acc[1], r0.y);
            acc[2] = fmaxf(acc[2], r0.z);
            acc[3] = fmaxf(acc[3], r0.w);
            acc[4] = fmaxf(acc[4], r1.x);
            acc[5] = fmaxf(acc[5], r1.y);
            acc[6] = fmaxf(acc[6], r1.z);
            acc[7] = fmaxf(acc[7], r1.w);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) d += (double)acc[i];
    }
    return (float)d;
}

// The same score with slot s at row s - 1.  COLS query tokens at a time and two rows per step; the additions are the same
// and in the same order as in s2_score_members.
__device__ __forceinline__ int s2_first_bit(uint32_t v) { return __ffs((int)v) - 1; }
__device__ __forceinline__ int s2_first_bit(unsigned long long v) { return __ffsll((long long)v) - 1; }
// pairs (uniform): the lanes 2 j and 2 j + 1 share a bag and take half of the query tokens each, the odd lane continuing
// the even lane's sum (half the steps where at most 32 passages are to be scored); the score is then the odd lane's.
template <int COLS, typename SetT>
__device__ __forceinline__ float s2_score_rows(SetT rows, const float *Tl, const float *rowsum, bool pairs, int lane)
{
    double d = 0.0;
    const int g_first = pairs && (lane & 1) ? QLEN / 8 : 0, g_count = pairs ? QLEN / 8 : QLEN / 4;
#pragma unroll 1
    for (int g0 = 0; g0 < g_count; g0 += COLS / 4) {
        float acc[COLS];
#pragma unroll
        for (int i = 0; i < COLS; ++i) acc[i] = -INFINITY;
        SetT rest = rows;
        while (rest) {
            const int r0 = s2_first_bit(rest);
            rest &= rest - 1;
            int r1 = r0;  // (an odd member count folds its last row twice)
            if (rest) {
                r1 = s2_first_bit(rest);
                rest &= rest - 1;
            }
#pragma unroll
            for (int g = 0; g < COLS / 4; ++g) {
                const float4 a = *reinterpret_cast<const float4 *>(Tl + r0 * S2_TSTRIDE + 4 * (g_first + g0 + g));
                const float4 b = *reinterpret_cast<const float4 *>(Tl + r1 * S2_TSTRIDE + 4 * (g_first + g0 + g));
                acc[4 * g] = fmaxf(acc[4 * g], fmaxf(a.x, b.x));
                acc[4 * g + 1] = fmaxf(acc[4 * g + 1], fmaxf(a.y, b.y));
                acc[4 * g + 2] = fmaxf(acc[4 * g + 2], fmaxf(a.z, b.z));
                acc[4 * g + 3] = fmaxf(acc[4 * g + 3], fmaxf(a.w, b.w));
                if (g == COLS / 8 - 1) __builtin_amdgcn_sched_barrier(0);  // (all rows in flight at once would spill)
            }
        }
#pragma unroll 1
        for (int t = pairs ? 0 : 1; t < 2; ++t) {
#pragma unroll
            for (int i = 0; i < COLS; ++i) d += (double)acc[i];
            if (t == 0) d = __shfl_xor(d, 1);  // the odd lane goes on from the even lane's sum
        }
    }
    return (float)d;
}

// The query's survivor table in LDS: hash table, rows (slot 0 = -infinity) and single-survivor sums.  All threads of
// the workgroup call this; K <= S2_MAX_KEPT.
__device__ __forceinline__ void s2_stage_tables(int q, int K, int hsh, const int32_t *__restrict__ kept_ids,
                                                const float *__restrict__ T, uint32_t *htab, float *Tl, float *rowsum)
{
    const int tid = threadIdx.x;
    for (int e = tid; e < S2_HASH; e += blockDim.x) htab[e] = 0xFFFFFFFFu;
    const float *Tq = T + (int64_t)q * (S2_MAX_KEPT + 1) * QLEN;
    for (int e = tid; e < (K + 1) * QLEN; e += blockDim.x)
        Tl[(e >> 5) * S2_TSTRIDE + (e & 31)] = (e >> 5) ? Tq[e] : -INFINITY;
    __syncthreads();
    if (tid < K) {
        const uint32_t code = (uint32_t)kept_ids[(int64_t)q * S2_MAX_KEPT + tid];
        htab[(code ^ (code >> hsh)) & (S2_HASH - 1)] = (code << 6) | (uint32_t)(tid + 1);
        // one survivor in the bag: the maxima are its row, summed in the same order as in s2_score_members
        double d = 0.0;
        for (int i = 0; i < QLEN; ++i) d += (double)Tl[(tid + 1) * S2_TSTRIDE + i];
        rowsum[tid + 1] = (float)d;
    }
    __syncthreads();
}

// Persistent workgroups; wave w of the grid scores the 64-passage tiles w, w + W, w + 2W, ... (lane = passage).
__global__ __launch_bounds__(S2_THREADS) void s2_stream_kernel(
    const float *__restrict__ S, int64_t C, const uint32_t *__restrict__ keepbits, int64_t keep_words,
    const int32_t *__restrict__ codes, int64_t N, const int64_t *__restrict__ doc_offsets, int64_t P,
    const uint32_t *__restrict__ candbits, int64_t cand_words, const S2Meta *__restrict__ meta,
    const int32_t *__restrict__ kept_ids, const float *__restrict__ T, uint64_t *__restrict__ keys2, int64_t key_stride,
    int32_t *__restrict__ hist, uint32_t *__restrict__ emptybits)
{
    __shared__ __align__(16) uint8_t stage_all[S2_THREADS / 64][S2W_CAP + 64];
    __shared__ uint32_t linebits_all[S2_THREADS / 64][S2_LBWORDS];
    __shared__ uint32_t htab[S2_HASH];
    __shared__ __align__(16) float Tl[(S2_MAX_KEPT + 1) * S2_TSTRIDE];
    __shared__ int32_t lhist[SEL_BINS];
    __shared__ float rowsum[S2_MAX_KEPT + 1];  // score of a bag holding only slot s
    const int q = blockIdx.y;
    const int K = s2_uniform(meta[q].K);
    const float bin_hi = meta[q].bin_hi, bin_scale = meta[q].bin_scale;
    uint32_t *keys_out = reinterpret_cast<uint32_t *>(keys2 + (int64_t)q * key_stride);  // slot p: passage p's score word
    int32_t *hist_q = hist + (int64_t)q * SEL_BINS;
    const int tid = threadIdx.x, lane = tid & 63;
    if (K == 0) {
        // no centroid passes Eq. 5: every bag is empty whatever the codes are, so they are not read.  There is no valid
        // key and the histogram stays zero; the candidates themselves are the empty-bag set.
        const uint32_t *cb0 = candbits + (int64_t)q * cand_words;
        uint32_t *eb0 = emptybits + (int64_t)q * cand_words;
        for (int64_t w = (int64_t)blockIdx.x * S2_THREADS + tid; w < cand_words; w += (int64_t)gridDim.x * S2_THREADS)
            eb0[w] = cb0[w];
        return;
    }
    for (int e = tid; e < SEL_BINS; e += S2_THREADS) lhist[e] = 0;
    if (K > S2_MAX_KEPT) {  // too many survivors for slot sets (uniform for the whole workgroup): gather form
        __syncthreads();
        s2_gather_body(q, S, C, keepbits, keep_words, candbits + (int64_t)q * cand_words, 0,
                       (int64_t)blockIdx.x * 4 + (tid >> 6), (int64_t)gridDim.x * 4, cand_words, cand_words, P, doc_offsets, codes,
                       bin_hi, bin_scale, keys_out, lhist, emptybits);
        s2_flush_hist(lhist, hist_q);
        return;
    }
    const int hsh = s2_uniform(meta[q].hash_shift);
    const int wave = s2_uniform(tid >> 6);
    s2_stage_tables(q, K, hsh, kept_ids, T, htab, Tl, rowsum);

    uint8_t *stage = stage_all[wave];
    uint32_t *linebits = linebits_all[wave];
    const uint32_t *cb = candbits + (int64_t)q * cand_words;
    uint32_t *eb = emptybits + (int64_t)q * cand_words;
    const int ntiles = (int)((P + S2W_PASS - 1) / S2W_PASS);
    const int nwaves = (int)gridDim.x * (S2_THREADS / 64);

    // A tile's metadata (candidate words, passage offsets) is requested one tile ahead of its use.
    int tile = (int)blockIdx.x * (S2_THREADS / 64) + wave;
    uint32_t cword_n = 0u;
    int64_t olane_n = 0, oend_n = 0;
    auto request_meta = [&](int t) {
        if (t < ntiles) {  // uniform
            const int64_t p0n = (int64_t)t * S2W_PASS;
            const int tpn = (int)(P - p0n < S2W_PASS ? P - p0n : S2W_PASS);
            const int64_t win = (p0n >> 5) + (lane >> 5);
            cword_n = (lane < tpn && win < cand_words) ? cb[win] : 0u;
            olane_n = doc_offsets[p0n + (lane <= tpn ? lane : tpn)];
            oend_n = doc_offsets[p0n + tpn];
        }
    };
    request_meta(tile);
    for (; tile < ntiles; tile += nwaves) {
        const int64_t p0 = (int64_t)tile * S2W_PASS;
        const int tp = (int)(P - p0 < S2W_PASS ? P - p0 : S2W_PASS);
        const uint32_t cword = cword_n;
        const int64_t o_lane = olane_n, o_end = oend_n;
        request_meta(tile + nwaves);
        const bool cand = lane < tp && ((cword >> (lane & 31)) & 1u);
        const unsigned long long candm = __ballot(cand);
        if (candm == 0ull) {  // (uniform) no candidate here: only the empty-bag words are cleared
            const int64_t wi = (p0 >> 5) + (lane >> 5);
            if ((lane & 31) == 0 && wi < cand_words) eb[wi] = 0u;
            continue;
        }
        uint64_t set = 0;  // bit s = slot s occurs in my passage; bit 0 collects the pruned tokens

        // token range of my passage relative to the tile's first token
        const int64_t o0 = __shfl(o_lane, 0);
        int64_t r = o_lane - o0;
        const int my_lo = r > 0x7FFFFFFFll ? 0x7FFFFFFF : (int)r;
        int my_hi = __shfl_down(my_lo, 1);
        if (lane == 63) {  // lane 63 has no right neighbour: its end is the tile's end
            r = o_end - o0;
            my_hi = r > 0x7FFFFFFFll ? 0x7FFFFFFF : (int)r;
        }
        if (lane >= tp) my_hi = my_lo;

        // Rounds of consecutive whole passages that fit the staging buffer, each starting at a candidate; the passages
        // after the tile's last candidate are never staged.
        int ps = s2_uniform(__ffsll((long long)candm) - 1);
        const int plast = s2_uniform(63 - __clzll((long long)candm));
        while (ps <= plast) {  // ps, fit, pe are uniform; each round advances ps by at least one
            const int base = s2_uniform(__shfl(my_lo, ps));
            const int fit = s2_uniform(__popcll(__ballot(lane >= ps && lane <= plast && my_hi - base <= S2W_CAP)));
            if (fit == 0) {
                // a single passage longer than the staging buffer: its lane folds it straight from global memory
                if (lane == ps)
                    for (int64_t j = o0 + my_lo; j < o0 + my_hi; ++j) set |= 1ull << s2_lookup(htab, (uint32_t)codes[j], hsh);
                ps = s2_uniform(s2_next_bit(candm, ps + 1));
            } else {
                const int pe = ps + fit;
                const int end = s2_uniform(__shfl(my_hi, pe - 1));
                const int64_t g0 = o0 + base;   // first token of the round
                const int64_t a0 = g0 & ~31ll;  // start of its 128-byte line
                const int shift = (int)(g0 - a0);
                const int nchunk = (shift + (end - base) + 31) >> 5;  // 128-byte lines of the round, <= 8 * S2_ITEMS
                const bool mine = lane >= ps && lane < pe && cand;
                // lines of the round that hold a candidate's tokens; when every passage of the round is a candidate
                // that is all of them
                const unsigned long long round_mask = (pe < 64 ? (1ull << pe) : 0ull) - (1ull << ps);
                const bool dense = (candm & round_mask) == round_mask;  // uniform
                if (lane < S2_LBWORDS) linebits[lane] = dense ? 0xFFFFFFFFu : 0u;
                s2_wave_sync();
                if (!dense) {
                    if (mine && my_hi > my_lo) {
                        const int c0 = (my_lo - base + shift) >> 5, c1 = (my_hi - 1 - base + shift) >> 5;
                        for (int c = c0; c <= c1; ++c) atomicOr(&linebits[c >> 5], 1u << (c & 31));
                    }
                    s2_wave_sync();
                }
                // Stage one byte per token: the slot of its centroid (0 = pruned).  Item u of a lane is the 16 bytes at token
                // 4 * (64 u + lane), so item u of the wave covers lines 8u .. 8u+7, which is byte u of the line bitmap: a
                // uniform test skips the item when no candidate touches those lines.  All loads of the round are issued
                // before the first is used, so a round costs one memory latency.
                const int nitem = nchunk * 8;
                const int32_t *__restrict__ src = codes + a0;  // uniform base, 32-bit lane offsets
                uint32_t need[S2_LBWORDS];
    #pragma unroll
                for (int k = 0; k < S2_LBWORDS; ++k) need[k] = (uint32_t)s2_uniform((int)linebits[k]);
                int4 v[S2_ITEMS];
                uint32_t okm = 0u;
    #pragma unroll
                for (int u = 0; u < S2_ITEMS; ++u) {
                    v[u] = make_int4(-1, -1, -1, -1);
                    const uint32_t lines8 = (need[u >> 2] >> (8 * (u & 3))) & 0xFFu;  // uniform
                    if (lines8 != 0u) {
                        const int it = 64 * u + lane;
                        const bool ok = it < nitem && ((lines8 >> (lane >> 3)) & 1u) && a0 + 4ll * it + 3 < N;
                        if (ok) v[u] = *reinterpret_cast<const int4 *>(src + 4 * it);
                        okm |= ok ? 1u << u : 0u;
                    }
                }
                uint32_t hit = 0u;
    #pragma unroll
                for (int u = 0; u < S2_ITEMS; ++u) {
                    const uint32_t lines8 = (need[u >> 2] >> (8 * (u & 3))) & 0xFFu;  // uniform
                    if (lines8 != 0u) {
                        if ((okm >> u) & 1u) {
                            const uint32_t packed = s2_lookup(htab, (uint32_t)v[u].x, hsh) |
                                                    (s2_lookup(htab, (uint32_t)v[u].y, hsh) << 8) |
                                                    (s2_lookup(htab, (uint32_t)v[u].z, hsh) << 16) |
                                                    (s2_lookup(htab, (uint32_t)v[u].w, hsh) << 24);
                            *reinterpret_cast<uint32_t *>(stage + 4 * (64 * u + lane)) = packed;
                            hit |= packed;
                        }
                    }
                }
                // the one item that straddles the end of the code array (tokens past N belong to no passage)
                if (a0 + 4ll * nitem > N) {
                    const int64_t it = (N - a0) >> 2;
                    if (lane < 4 && it < nitem && a0 + 4 * it + lane < N) {
                        const uint32_t sl = s2_lookup(htab, (uint32_t)codes[a0 + 4 * it + lane], hsh);
                        stage[4 * it + lane] = (uint8_t)sl;
                        hit |= sl;
                    }
                }
                s2_wave_sync();
                const bool any_hit = __ballot(hit != 0u) != 0ull;  // uniform
                if (any_hit && mine && my_hi > my_lo) {
                    // four staged bytes at a time; most are zero (pruned tokens) and are skipped as a word
                    const int v0 = my_lo - base + shift, v1 = my_hi - base + shift;
                    const uint32_t *stage32 = reinterpret_cast<const uint32_t *>(stage);
                    for (int wd = v0 >> 2; wd <= (v1 - 1) >> 2; ++wd) {
                        uint32_t x = stage32[wd];
                        if (4 * wd < v0) x &= 0xFFFFFFFFu << (8 * (v0 - 4 * wd));       // bytes before the passage
                        if (4 * wd + 4 > v1) x &= 0xFFFFFFFFu >> (8 * (4 * wd + 4 - v1));  // bytes after it
                        if (x) {
                            set |= 1ull << (x & 0xFFu);
                            set |= 1ull << ((x >> 8) & 0xFFu);
                            set |= 1ull << ((x >> 16) & 0xFFu);
                            set |= 1ull << (x >> 24);
                        }
                    }
                }
                s2_wave_sync();
                ps = s2_uniform(s2_next_bit(candm, pe));
            }
        }

        // score: column maxima of the rows in the set, summed over the query tokens in index order; eight query tokens
        // at a time, so that few registers are live
        const uint64_t members = set & ~1ull;
        const bool empty = members == 0;
        float score = -INFINITY;
        if (cand && !empty) score = s2_score_members(members, Tl, rowsum);
        // emit: slot p of the key array belongs to candidate p; no counters, no ordering between waves
        const bool live = cand && !empty;
        if (cand) keys_out[p0 + lane] = live ? plaid_score_to_ord(score) : PLAID_S2_NO_SCORE;
        if (live) atomicAdd(&lhist[plaid_s2_bin(score, bin_hi, bin_scale)], 1);
        const unsigned long long eb64 = __ballot(cand && empty);
        if (lane == 0) {
            const int64_t w0 = p0 >> 5;
            if (w0 < cand_words) eb[w0] = (uint32_t)eb64;
            if (w0 + 1 < cand_words) eb[w0 + 1] = (uint32_t)(eb64 >> 32);
        }
    }
    s2_flush_hist(lhist, hist_q);
}


// ------------------------------------------------------------------ inverted form: candidates and bags from the inverted lists
// A passage contains centroid c exactly when it is in c's inverted list (Section 4.1 stores unique passage ids per
// centroid).  So the candidate set is the union of the probed centroids' lists, and the pruned bag of a passage
// (Eq. 5) is the set of surviving centroids whose lists contain it: both follow from the inverted lists of at most
// 32 nprobe + S2_MAX_KEPT centroids, far fewer bytes than the candidates' token codes whenever few centroids
// survive.  Where a list enters a range of 2^SHIFT passages comes from a table built once per index: table[c][r] =
// position in list c of its first entry with passage id >= r * 2^SHIFT.
#define IVR_EMPTY 0xFFFFFFFFu
#define IVR_LISTS 256  // lists per round of the wide union
#define IVR_DENSE_DIV 16  // a list with at least P / 16 entries also gets a bitmap over the passages

// table[c][r] for every non-empty (list, range) pair; the others keep IVR_EMPTY until ivr_fill_kernel.
__global__ __launch_bounds__(256) void ivr_mark_kernel(const int64_t *__restrict__ ivf_offsets,
                                                       const int32_t *__restrict__ ivf_pids, int64_t C, int64_t nr,
                                                       int shift, uint32_t *__restrict__ table)
{
    for (int64_t c = blockIdx.x; c < C; c += gridDim.x) {
        const int64_t s = ivf_offsets[c], t = ivf_offsets[c + 1];
        for (int64_t e = s + threadIdx.x; e < t; e += blockDim.x) {
            const int64_t r = (int64_t)(uint32_t)ivf_pids[e] >> shift;
            const bool first = e == s || ((int64_t)(uint32_t)ivf_pids[e - 1] >> shift) != r;
            if (first && r < nr) table[c * (nr + 1) + r] = (uint32_t)(e - s);
        }
    }
}
// A range a list has no entry in starts where the next one does; the last column is the list's length.
__global__ __launch_bounds__(256) void ivr_fill_kernel(const int64_t *__restrict__ ivf_offsets, int64_t C, int64_t nr,
                                                       uint32_t *__restrict__ table)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    uint32_t next = (uint32_t)(ivf_offsets[c + 1] - ivf_offsets[c]);
    uint32_t *row = table + c * (nr + 1);
    row[nr] = next;
    for (int64_t r = nr - 1; r >= 0; --r) {
        const uint32_t v = row[r];
        if (v == IVR_EMPTY || v > next) row[r] = next;  // (v > next only if a list is not ascending: keep the row monotone)
        else next = v;
    }
}

size_t plaid_ivf_range_table_bytes(int64_t C, int64_t P, int shift)
{
    const int64_t nr = (P + (1ll << shift) - 1) >> shift;
    return (size_t)C * (size_t)(nr + 1) * sizeof(uint32_t);
}
void plaid_launch_ivf_range_table(hipStream_t st, const int64_t *ivf_offsets, const int32_t *ivf_pids, int64_t C, int64_t P,
                                  int shift, uint32_t *table)
{
    const int64_t nr = (P + (1ll << shift) - 1) >> shift;
    plaid_launch_fill_u32(st, table, C * (nr + 1), IVR_EMPTY);
    hipLaunchKernelGGL(ivr_mark_kernel, dim3((unsigned)(C < 8192 ? C : 8192)), dim3(256), 0, st, ivf_offsets, ivf_pids, C, nr, shift, table);
    hipLaunchKernelGGL(ivr_fill_kernel, dim3((unsigned)((C + 255) / 256)), dim3(256), 0, st, ivf_offsets, C, nr, table);
}

// Dense lists.  The centroid of a frequent token occurs in a large share of the passages: its list is then longer than
// a bitmap over the passages (P / 8 bytes), and a query that probes it would read megabytes of passage ids to set
// nearly every candidate bit.  Lists with at least P / IVR_DENSE_DIV entries therefore also get such a bitmap at index
// creation: dense_id[c] = row of the bitmap, or -1.
__global__ __launch_bounds__(256) void ivr_dense_mark_kernel(const int64_t *__restrict__ ivf_offsets, int64_t C, int64_t P,
                                                             int32_t *__restrict__ dense_id, int32_t *__restrict__ counter)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    const int64_t len = ivf_offsets[c + 1] - ivf_offsets[c];
    dense_id[c] = (len > 0 && len * IVR_DENSE_DIV >= P) ? atomicAdd(counter, 1) : -1;
}
__global__ __launch_bounds__(256) void ivr_dense_fill_kernel(const int64_t *__restrict__ ivf_offsets,
                                                             const int32_t *__restrict__ ivf_pids, int64_t C, int64_t P,
                                                             const int32_t *__restrict__ dense_id, uint32_t *__restrict__ bits,
                                                             int64_t words)
{
    for (int64_t c = blockIdx.x; c < C; c += gridDim.x) {
        const int32_t d = dense_id[c];
        if (d < 0) continue;  // uniform
        uint32_t *row = bits + (int64_t)d * words;
        const int64_t s = ivf_offsets[c], t = ivf_offsets[c + 1];
        for (int64_t e = s + threadIdx.x; e < t; e += blockDim.x) {
            const uint32_t pid = (uint32_t)ivf_pids[e];
            if ((int64_t)pid < P) atomicOr(&row[pid >> 5], 1u << (pid & 31));
        }
    }
}
// total += entries x columns with an entry of the lists without a bitmap.  A workgroup per list, since the rows lie one after the other:
// one pass over the table when the index is made, 51 MB in 78 us, 4.4 GB in 1.4 ms (3.1 TB/s).
__global__ __launch_bounds__(256) void ivr_plane_share_kernel(const uint32_t *__restrict__ table, const int32_t *__restrict__ dense_id,
                                                              int64_t C, int64_t nr, double *__restrict__ total)
{
    __shared__ int32_t columns;
    double sum = 0.0;
    for (int64_t c = blockIdx.x; c < C; c += gridDim.x) {
        if (dense_id[c] >= 0) continue;  // uniform
        const uint32_t *row = table + c * (nr + 1);
        if (threadIdx.x == 0) columns = 0;
        __syncthreads();
        int n = 0;
        for (int64_t r = threadIdx.x; r < nr; r += 256) n += row[r + 1] > row[r] ? 1 : 0;
        if (n) atomicAdd(&columns, n);
        __syncthreads();
        sum += (double)row[nr] * columns;
        __syncthreads();
    }
    if (threadIdx.x == 0 && sum > 0.0) atomicAdd(total, sum);
}
void plaid_launch_ivf_plane_share(hipStream_t st, const uint32_t *table, const int32_t *dense_id, int64_t C, int64_t P, int shift,
                                  double *total)
{
    const int64_t nr = (P + (1ll << shift) - 1) >> shift;
    hipLaunchKernelGGL(ivr_plane_share_kernel, dim3((unsigned)(C < 4096 ? C : 4096)), dim3(256), 0, st, table, dense_id, C, nr, total);
}
void plaid_launch_ivf_dense_mark(hipStream_t st, const int64_t *ivf_offsets, int64_t C, int64_t P, int32_t *dense_id,
                                 int32_t *counter)
{
    hipLaunchKernelGGL(ivr_dense_mark_kernel, dim3((unsigned)((C + 255) / 256)), dim3(256), 0, st, ivf_offsets, C, P, dense_id,
                       counter);
}
void plaid_launch_ivf_dense_fill(hipStream_t st, const int64_t *ivf_offsets, const int32_t *ivf_pids, int64_t C, int64_t P,
                                 const int32_t *dense_id, uint32_t *bits, int64_t words)
{
    hipLaunchKernelGGL(ivr_dense_fill_kernel, dim3((unsigned)(C < 8192 ? C : 8192)), dim3(256), 0, st, ivf_offsets, ivf_pids, C,
                       P, dense_id, bits, words);
}

// Queries none of whose centroids passes Eq. 5: every bag is empty, so stage 2 only has to produce the candidate set,
// and a passage needs one bit instead of a set word.  A workgroup then covers 2^19 passages (64 KB of LDS bits): a wave
// walks one probed centroid's list at a time (512 entries per step, eight loads in flight), and the bits are written
// out once, as the candidate words and as the empty-bag words.  The fine-grained kernel below skips these queries.
#define UW_SHIFT 19
#define UW_WORDS (1 << (UW_SHIFT - 5))
#define UW_THREADS 1024
#define UW_LONG 4096  // entries from which on a list is walked by all waves together
#define IVR_WIDE_MIN_QUERIES 32
static_assert(UW_SHIFT >= 13, "a wide range is a whole number of table ranges");
__global__ __launch_bounds__(UW_THREADS) void s2_union_wide_kernel(
    const int32_t *__restrict__ uniq, const int32_t *__restrict__ n_uniq, int uniq_stride,
    const int64_t *__restrict__ ivf_offsets, const int32_t *__restrict__ ivf_pids, const uint32_t *__restrict__ table,
    int64_t nr, int shift, int64_t P, const S2Meta *__restrict__ meta, const int32_t *__restrict__ dense_id,
    const uint32_t *__restrict__ dense_bits, uint32_t *__restrict__ candbits, int64_t cand_words,
    uint32_t *__restrict__ emptybits)
{
    __shared__ uint32_t bits[UW_WORDS];
    __shared__ int64_t first[IVR_LISTS];
    __shared__ int32_t count[IVR_LISTS];
    __shared__ int32_t dense[IVR_LISTS];  // rows of the dense-list bitmaps probed in this round
    __shared__ int32_t n_dense;
    const int q = blockIdx.y;
    if (s2_uniform(meta[q].K) != 0) return;  // uniform
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = s2_uniform(tid >> 6);
    const int64_t fr0 = (int64_t)blockIdx.x << (UW_SHIFT - shift);  // table ranges [fr0, fr1)
    const int64_t fr1 = fr0 + (1ll << (UW_SHIFT - shift)) < nr ? fr0 + (1ll << (UW_SHIFT - shift)) : nr;
    const uint32_t p0 = (uint32_t)blockIdx.x << UW_SHIFT;
    for (int e = tid; e < UW_WORDS; e += UW_THREADS) bits[e] = 0u;
    const int nu = n_uniq[q];
    for (int u0 = 0; u0 < nu; u0 += IVR_LISTS) {
        const int nb = nu - u0 < IVR_LISTS ? nu - u0 : IVR_LISTS;
        __syncthreads();  // the bits are zero / the previous round's lists are done
        if (tid == 0) n_dense = 0;
        __syncthreads();
        if (tid < nb) {
            const int32_t c = uniq[(int64_t)q * uniq_stride + u0 + tid];
            const int32_t d = dense_id[c];
            if (d >= 0) {  // its bitmap is OR-ed in below
                dense[atomicAdd(&n_dense, 1)] = d;
                count[tid] = 0;
            } else {
                const uint32_t a = table[(int64_t)c * (nr + 1) + fr0], b = table[(int64_t)c * (nr + 1) + fr1];
                first[tid] = ivf_offsets[c] + a;
                count[tid] = b > a ? (int)(b - a) : 0;
            }
        }
        __syncthreads();
        // steps s0, s0 + stride, ... of list l (a step = 512 entries).  A lane takes eight consecutive entries and merges
        // the bits that fall into one word before it touches LDS: in the list of a centroid that occurs in nearly every
        // passage consecutive entries are consecutive passages, and one entry per lane would send 32 lanes to each word.
        auto walk = [&](int l, int s0, int stride) {
            const int n = s2_uniform(count[l]);
            const int32_t *__restrict__ src = ivf_pids + first[l];
            for (int e0 = s0 * 512; e0 < n; e0 += stride * 512) {
                uint32_t pid[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + 8 * lane + u;
                    pid[u] = e < n ? (uint32_t)src[e] : 0xFFFFFFFFu;
                }
                uint32_t cw = 0xFFFFFFFFu, acc = 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t loc = pid[u] - p0;
                    if (pid[u] != 0xFFFFFFFFu && loc < (1u << UW_SHIFT)) {
                        const uint32_t w = loc >> 5, bit = 1u << (loc & 31);
                        if (w != cw) {
                            if (acc) atomicOr(&bits[cw], acc);
                            cw = w;
                            acc = bit;
                        } else {
                            acc |= bit;
                        }
                    }
                }
                if (acc) atomicOr(&bits[cw], acc);
            }
        };
        // a wave takes whole lists of ordinary length; the lists of centroids that occur in most passages (hundreds
        // of thousands of entries) are shared by all waves
        for (int l = wave; l < nb; l += UW_THREADS / 64)
            if (count[l] <= UW_LONG) walk(l, 0, 1);
        for (int l = 0; l < nb; ++l)
            if (count[l] > UW_LONG) walk(l, wave, UW_THREADS / 64);
        const int nd = n_dense;
        if (nd > 0) {  // uniform
            __syncthreads();  // the walks' atomics are done: each word now has one owner thread
            const int64_t wf = (int64_t)p0 >> 5;
            const int64_t nwr = cand_words - wf < UW_WORDS ? cand_words - wf : UW_WORDS;
            for (int64_t w = tid; w < nwr; w += UW_THREADS) {
                uint32_t v = bits[w];
                for (int d = 0; d < nd; ++d) v |= dense_bits[(int64_t)dense[d] * cand_words + wf + w];
                bits[w] = v;
            }
        }
    }
    __syncthreads();
    const int64_t w_first = (int64_t)p0 >> 5;
    uint32_t *cbq = candbits + (int64_t)q * cand_words + w_first;
    uint32_t *ebq = emptybits + (int64_t)q * cand_words + w_first;
    const int64_t nw = cand_words - w_first < UW_WORDS ? cand_words - w_first : UW_WORDS;
    for (int64_t w = tid; w < nw; w += UW_THREADS) {
        uint32_t v = bits[w];
        const int64_t pbase = (int64_t)p0 + 32 * w;  // passages past the end never enter the lists; the mask is a guard
        if (pbase + 32 > P) v &= pbase < P ? (1u << (uint32_t)(P - pbase)) - 1u : 0u;
        cbq[w] = v;
        ebq[w] = v;
    }
}

// The range kernel.  A WAVE owns 2^len passages at a time (2048 unless the launch is small).  Every surviving slot has a
// bit plane over them: word w, bit b = the slot is in the bag of passage p0 + 32 w + b.  The planes of long lists are the
// index's bitmaps, those of the other lists are filled entry by entry in the wave's own LDS area.  With lane = 32 passages:
//   bound    every passage's additive bound (S2Meta::ub_base, gains) is summed bit-sliced: the gains are wave-uniform
//            whole numbers, a ten-bit ripple-carry addition of "gain where the plane's bit is set" serves 32 passages
//            per lane with three instructions per bit and slot.
//   prune    the coarse histogram of the scores computed so far (by every wave of the query) tells a bin that at least m
//            scores have reached or passed; a passage whose bound falls into a worse bin cannot be among the best m and
//            is not scored.  Which passages are skipped depends on timing, the best m do not.
//   score    the remaining passages, 64 at a time with lane = passage: the bag's slots are collected from the planes
//            and scored exactly (s2_score_rows), the key appended to the query's list, the bin counted.
// While the histogram does not prune yet (the first waves of a query), a wave scores the passages with the highest
// bounds of its range, some dozens, and looks again: a thousand such waves know the final threshold almost exactly.
//
// Why: of 400 000 candidates per query (65536 centroids, ndocs 1024) about one in thirty is scored.  Scoring all of them (a
// set word per passage built with LDS atomics, one lane per passage, sorted by bag size) took 3.5 ms per 512 queries, this
// 0.9; 150 queries of 8.8 M passages at 262144 centroids 25 ms, now 6.6.  What bounds it now: a wave's step of 2048
// passages takes 16 to 20 us with 12 to 16 waves per compute unit: the additions of the bounds and the chains of dependent
// loads and LDS accesses of the other parts.
#define IV_WAVES 4
#define IV_LISTS 256    // probed lists a workgroup classifies; beyond (nprobe > 8) s2_candidates_kernel walks them

// Makes the compiler forget what it has derived from v.  Addresses and lane masks computed from the lane number would
// otherwise be kept in registers across the range kernel's loops (25 registers past what four waves per SIMD leave).
__device__ __forceinline__ void s2_opaque(int &v) { asm volatile("" : "+v"(v)); }

// Inclusive prefix sum over the lanes: additions with data-parallel-primitive operands (shifts by 1, 2, 4, 8 within a row of
// sixteen lanes, then the last lane of a row added to the rows that follow), no LDS exchange.  All lanes active.
__device__ __forceinline__ int s2_wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Sum over the lanes, uniform.
__device__ __forceinline__ int s2_wave_sum(int v) { return __builtin_amdgcn_readlane(s2_wave_scan(v), 63); }

// Counts of coarse bins 2 lane and 2 lane + 1, read where the other compute units' additions arrive.
__device__ __forceinline__ int2 s2_coarse_load(const int32_t *coarse_q, int lane)
{
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(coarse_q) + lane, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    return make_int2((int)(uint32_t)v, (int)(uint32_t)(v >> 32));
}
// Probes found by several workgroups (Stage2Buffers::probes_apart) are a query's with duplicates.  Whether this thread is the first to
// bring c, by a table of S2_SEEN places, -1 at the start, of which the probes of a query (up to IV_LISTS) take at most half.
#define S2_SEEN (2 * IV_LISTS)
__device__ __forceinline__ bool s2_first_probe(int32_t *seen, int32_t c)
{
    static_assert(S2_SEEN == 512, "nine bits of the hash");
    for (uint32_t h = (uint32_t)c * 0x9E3779B1u >> 23;; h = (h + 1) & (S2_SEEN - 1)) {
        const int32_t was = atomicCAS(&seen[h], -1, c);
        if (was == -1) return true;
        if (was == c) return false;
    }
}
// The candidates among the passages of the bitmap words [w0, w0 + nw), nw <= 64, all in one column of the range table: the
// union of the nu probed lists, probe(e) the e-th's centroid or -1, into lcand[0 .. nw).  All 256 threads of a workgroup call this; thread t
// asks for probes t, t + 256, ...; a barrier ends it.
struct S2CandScratch {
    int64_t first[IV_LISTS];
    int32_t count[IV_LISTS];
};
template <typename F>
__device__ __forceinline__ void s2_block_candidates(F &&probe, int nu, const int64_t *__restrict__ ivf_offsets,
                                                    const int32_t *__restrict__ ivf_pids, const uint32_t *__restrict__ table,
                                                    int64_t nr, int shift, const int32_t *__restrict__ dense_id,
                                                    const uint32_t *__restrict__ dense_bits, int64_t cand_words, int64_t P,
                                                    int64_t w0, int nw, uint32_t *lcand /*[64]*/, S2CandScratch &cs,
                                                    int32_t *rows /*[IV_LISTS]*/, int32_t *counts /*[2]*/)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid & 15;
    const int64_t col = (w0 << 5) >> shift;
    const uint32_t p0 = (uint32_t)(w0 << 5), len = 32u * (uint32_t)nw;
    if (tid < 64) lcand[tid] = 0u;
    for (int u0 = 0; u0 < nu; u0 += IV_LISTS) {
        __syncthreads();  // the words are zero / the previous lists are done
        if (tid < 2) counts[tid] = 0;
        __syncthreads();
        const int32_t c = u0 + tid < nu ? probe(u0 + tid) : -1;
        if (c >= 0) {
            const int32_t d = dense_id[c];
            const uint32_t a = table[(int64_t)c * (nr + 1) + col], b = table[(int64_t)c * (nr + 1) + col + 1];
            if (d >= 0) {
                rows[atomicAdd(&counts[0], 1)] = d;
            } else if (b > a) {
                const int i = atomicAdd(&counts[1], 1);
                cs.first[i] = ivf_offsets[c] + a;
                cs.count[i] = (int)(b - a);
            }
        }
        __syncthreads();
        const int n_rows = counts[0], n_lists = counts[1];
        uint32_t v = 0u;
        if (lane < nw)
            for (int d0 = wave; d0 < n_rows; d0 += 4 * IV_WAVES) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (d0 + IV_WAVES * u < n_rows) v |= dense_bits[(int64_t)rows[d0 + IV_WAVES * u] * cand_words + w0 + lane];
            }
        if (v) atomicOr(&lcand[lane], v);
        // sixteen lanes per list, four lists each in flight
        for (int l0 = tid >> 4; l0 < n_lists; l0 += 4 * (64 * IV_WAVES / 16)) {
            int n[4];
            const int32_t *src[4];
            uint32_t pid[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = l0 + u * (64 * IV_WAVES / 16);
                n[u] = l < n_lists ? cs.count[l] : 0;
                src[u] = ivf_pids + (l < n_lists ? cs.first[l] : 0);
                pid[u] = sub < n[u] ? (uint32_t)src[u][sub] : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (pid[u] - p0 < len) atomicOr(&lcand[(pid[u] - p0) >> 5], 1u << (pid[u] & 31));
#pragma unroll
            for (int u = 0; u < 4; ++u)
                for (int x = 16 + sub; x < n[u]; x += 16) {
                    const uint32_t loc = (uint32_t)src[u][x] - p0;
                    if (loc < len) atomicOr(&lcand[loc >> 5], 1u << (loc & 31));
                }
        }
    }
    __syncthreads();
    if (tid == nw - 1 && P < ((w0 + nw) << 5)) lcand[tid] &= (1u << (uint32_t)(P & 31)) - 1u;  // (a guard: lists hold ids below P)
    __syncthreads();
}

// The candidate words of every query, 64 per workgroup, for launches whose probed lists are more than a workgroup of the range
// kernel classifies (nprobe > 8).  A wave of that kernel owns 2048 passages, and walked all of the lists for them alone, 64 to
// a round and the long ones entry by entry: stage 2 of one query of 400 000 passages took 35 / 129 / 219 us with nprobe 9 / 16 /
// 64 that way, 44 / 46 / 58 with the
// words given; 64 queries 539 / 621 / 981 and 203 / 231 / 408.
__global__ __launch_bounds__(64 * IV_WAVES) void s2_candidates_kernel(
    const int32_t *__restrict__ uniq, const int32_t *__restrict__ n_uniq, int uniq_stride, const int64_t *__restrict__ ivf_offsets,
    const int32_t *__restrict__ ivf_pids, const uint32_t *__restrict__ table, int64_t nr, int shift, int64_t P,
    const S2Meta *__restrict__ meta, const int32_t *__restrict__ dense_id, const uint32_t *__restrict__ dense_bits,
    uint32_t *__restrict__ candbits, int64_t cand_words, int skip_none /* s2_union_wide_kernel has done those without survivors */)
{
    __shared__ S2CandScratch cs;
    __shared__ uint32_t lcand[64];
    __shared__ int32_t rows[IV_LISTS], counts[2];
    const int q = blockIdx.y, tid = threadIdx.x;
    if (skip_none && s2_uniform(meta[q].K) == 0) return;  // uniform
    const int64_t w0 = (int64_t)blockIdx.x * 64;
    const int nw = cand_words - w0 < 64 ? (int)(cand_words - w0) : 64;
    const int32_t *uq = uniq + (int64_t)q * uniq_stride;
    s2_block_candidates([=](int e) { return uq[e]; }, n_uniq[q], ivf_offsets, ivf_pids, table, nr, shift, dense_id, dense_bits,
                        cand_words, P, w0, nw, lcand, cs, rows, counts);
    if (tid < nw) candbits[(int64_t)q * cand_words + w0 + tid] = lcand[tid];
}

// Queries with more than S2_MAX_KEPT surviving centroids (low thresholds, or none): no slot sets, no planes and no bound; every
// candidate is scored from its token codes.  Bound by the rows of S_cq it gathers, 128 bytes per surviving token.
// S2_GATHER_BLOCKS workgroups at the end of the 64-bit instance's grid share these queries (the probe kernel lists them
// from the end of the row of that instance's class; a launch without any loses nothing, they leave while the others
// work).  Their shares are even in bitmap words: eight queries at a time go to one XCD each, whose workgroups
// then gather from one query's S_cq, what is left over eight to all workgroups together.
// Per wave sixteen passages at a time: the codes and the pruning bits of eight of them in flight, the surviving ones listed
// in LDS, then eight rows per load instruction as in stage 3.  Bins are counted in LDS and added once per share.
// 400 000 passages, one query: 4.1 ms per search with four waves per 2048 passages fetching two rows at a time, 15.6 with one,
// 0.40 now; 64 queries 92, 117 and 16.
// One round of workgroups, as many per compute unit as run there together: shares are even, so what is missing to a round
// leaves units behind the others, and what exceeds it runs alone.  No pruning, 400 000 passages, ndocs 4096, 128 / 8 / 1 queries,
// us per search with 512, 768, 1024, 1280, 2048 workgroups where four run together: 48 800, 36 100, 27 000, 37 900, 28 400 /
// 3140, 2180, 1710, 2310, 1710 / 449, 360, 317, 401, 342 (768 where three do: 32 600 / 2090 / 402).
#define S2_UNIT_BLOCKS 4
#define S2_GATHER_BLOCKS (256 * S2_UNIT_BLOCKS)
#define S2_FITS_BLOCKS 768    // launches of up to this many workgroups run the 64-bit instance alone
#define S2_PLANES 26          // of a wave of the 64-bit instance, and of the one that is TALL
#define S2_TALL_PLANES 36
#define S2_TALL_UNIT_BLOCKS 3
#define S2_GATHER_STRIDE 68   // of a passage's list: eight lanes that read one column of eight lists hit all banks
struct S2GatherScratch {
    S2CandScratch cand;
    float part_max[IV_WAVES][8][QLEN];
    int32_t list[IV_WAVES][8][S2_GATHER_STRIDE];  // centroids of the surviving tokens; then the passage's column maxima
    int32_t hist[SEL_BINS];
};

template <int N>
__device__ __forceinline__ float4 s2_gather_rows(const float *__restrict__ Sq, const int32_t *list, int cnt, int r, int part, float4 m)
{
    float4 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int t = 8 * u + r;
        v[u] = *reinterpret_cast<const float4 *>(Sq + (int64_t)list[t < cnt ? t : cnt - 1] * QLEN + 4 * part);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) m = make_float4(fmaxf(m.x, v[u].x), fmaxf(m.y, v[u].y), fmaxf(m.z, v[u].z), fmaxf(m.w, v[u].w));
    return m;
}
__device__ __forceinline__ float4 s2_gather_list(const float *__restrict__ Sq, const int32_t *list, int cnt, int lane, float4 m)
{
    const int r = lane >> 3, part = lane & 7;
    switch ((cnt + 7) >> 3) {  // uniform
    case 0: return m;
    case 1: return s2_gather_rows<1>(Sq, list, cnt, r, part, m);
    case 2: return s2_gather_rows<2>(Sq, list, cnt, r, part, m);
    case 3: return s2_gather_rows<3>(Sq, list, cnt, r, part, m);
    case 4: return s2_gather_rows<4>(Sq, list, cnt, r, part, m);
    case 5: return s2_gather_rows<5>(Sq, list, cnt, r, part, m);
    case 6: return s2_gather_rows<6>(Sq, list, cnt, r, part, m);
    case 7: return s2_gather_rows<7>(Sq, list, cnt, r, part, m);
    default: return s2_gather_rows<8>(Sq, list, cnt, r, part, m);
    }
}
__device__ __forceinline__ int64_t s2_lane64(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)((uint64_t)hi << 32 | lo);
}

// Share j of nj of query q (all threads of the workgroup call this).
__device__ __forceinline__ void s2_gather_share(int q, int64_t j, int64_t nj, const int32_t *__restrict__ uniq, const int32_t *__restrict__ n_uniq,
                                int uniq_stride, const int64_t *__restrict__ ivf_offsets, const int32_t *__restrict__ ivf_pids,
                                const uint32_t *__restrict__ table, int64_t nr, int shift, const float *__restrict__ S, int64_t C,
                                const uint32_t *__restrict__ keepbits, int64_t keep_words, const int32_t *__restrict__ codes,
                                const int64_t *__restrict__ doc_offsets, int64_t P, float bin_hi, float bin_scale,
                                uint32_t *__restrict__ candbits, int64_t cand_words, uint64_t *__restrict__ keys2, int64_t key_stride,
                                int32_t *__restrict__ hist, uint32_t *__restrict__ emptybits,
                                const int32_t *__restrict__ dense_id, const uint32_t *__restrict__ dense_bits, S2GatherScratch &gs,
                                uint32_t *lcand, uint32_t *lempty, int32_t *rows, int32_t *counts, bool given, bool apart)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = s2_uniform(tid >> 6);
    const int64_t wa = cand_words * j / nj, wb = cand_words * (j + 1) / nj;
    if (wa == wb) return;  // uniform
    const float *Sq = S + (int64_t)q * C * QLEN;
    const uint32_t *kb = keepbits + (int64_t)q * keep_words;
    uint32_t *keys_out = reinterpret_cast<uint32_t *>(keys2 + (int64_t)q * key_stride);
    for (int e = tid; e < SEL_BINS; e += 64 * IV_WAVES) gs.hist[e] = 0;
    // This thread's probe, -1 where another thread has the same one: a list walked again costs what it did the first time.  us per search
    // of 31 queries of 200 000 passages, some 200 survivors and 19 to 29 distinct ones of 128 probes (means of eight sets of queries, whose
    // order alone makes 4 %): probes united beforehand 2229, every duplicate walked 2257, so 2220; nprobe 8 2239, 2286, 2232.
    const int nu = given ? 0 : n_uniq[q];
    int32_t mine = tid < nu ? uniq[(int64_t)q * uniq_stride + tid] : -1;
    if (apart && !given) {  // uniform
        static_assert(sizeof(gs.list) >= S2_SEEN * sizeof(int32_t), "the table takes the place of the lists");
        static_assert(S2_SEEN == 2 * 64 * IV_WAVES, "two places a thread");
        int32_t *seen = &gs.list[0][0][0];
        seen[tid] = seen[tid + 64 * IV_WAVES] = -1;
        __syncthreads();
        if (mine >= 0 && !s2_first_probe(seen, mine)) mine = -1;
    }
    for (int64_t w0 = wa; w0 < wb;) {
        const int64_t we = (w0 | 63) + 1 < wb ? (w0 | 63) + 1 : wb;  // within 2048 aligned passages: one column of the table
        const int nw = (int)(we - w0);
        uint32_t *cbq = candbits + (int64_t)q * cand_words + w0;
        if (given) {  // uniform: s2_candidates_kernel's
            if (tid < nw) lcand[tid] = cbq[tid];
        } else {
            s2_block_candidates([=](int) { return mine; }, nu, ivf_offsets, ivf_pids, table, nr, shift, dense_id, dense_bits, cand_words,
                                P, w0, nw, lcand, gs.cand, rows, counts);
            if (tid < nw) cbq[tid] = lcand[tid];
        }
        if (tid < 64) lempty[tid] = 0u;
        __syncthreads();
        for (int h = wave; h < 2 * nw; h += IV_WAVES) {
            uint32_t rest = (uint32_t)s2_uniform((int)((lcand[h >> 1] >> (16 * (h & 1))) & 0xFFFFu));
            const int64_t p0 = ((w0 + (h >> 1)) << 5) + 16 * (h & 1);
            int64_t off = 0;
            if (lane <= 16) off = doc_offsets[p0 + lane < P ? p0 + lane : P];
            uint32_t none = 0u;  // candidates without a surviving token
            while (rest) {
                // the first 64 codes of up to eight candidates; lane a: bit and number of surviving tokens of the a-th
                int32_t code[8];
                int my_bit = 0, my_cnt = 0, n = 0;
#pragma unroll
                for (int a = 0; a < 8; ++a) {
                    code[a] = -1;
                    if (rest) {
                        const int b = __ffs((int)rest) - 1;
                        rest &= rest - 1;
                        if (lane == a) my_bit = b;
                        const int64_t t0 = s2_lane64(off, b), t1 = s2_lane64(off, b + 1);
                        if (t0 + lane < t1) code[a] = codes[t0 + lane];
                        n = a + 1;
                    }
                }
                uint32_t kept[8];
#pragma unroll
                for (int a = 0; a < 8; ++a) kept[a] = code[a] >= 0 ? kb[code[a] >> 5] : 0u;
#pragma unroll
                for (int a = 0; a < 8; ++a) {
                    const bool hit = (kept[a] >> (code[a] & 31)) & 1u;
                    const unsigned long long mask = __ballot(hit);
                    if (hit) gs.list[wave][a][__popcll(mask & ((1ull << lane) - 1ull))] = code[a];
                    if (lane == a) my_cnt = __popcll(mask);
                }
                s2_wave_sync();
#pragma unroll 1
                for (int a = 0; a < n; ++a) {
                    int32_t *list = gs.list[wave][a];
                    const int b = __builtin_amdgcn_readlane(my_bit, a);
                    int cnt = __builtin_amdgcn_readlane(my_cnt, a);
                    float4 m = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
                    m = s2_gather_list(Sq, list, cnt, lane, m);
                    bool any = cnt > 0;
                    const int64_t t1 = s2_lane64(off, b + 1);
                    for (int64_t tb = s2_lane64(off, b) + 64; tb < t1; tb += 64) {  // a passage of more than 64 tokens
                        const int32_t c = tb + lane < t1 ? codes[tb + lane] : -1;
                        const bool hit = c >= 0 && ((kb[c >> 5] >> (c & 31)) & 1u);
                        const unsigned long long mask = __ballot(hit);
                        s2_wave_sync();
                        if (hit) list[__popcll(mask & ((1ull << lane) - 1ull))] = c;
                        s2_wave_sync();
                        cnt = __popcll(mask);
                        any = any || cnt > 0;
                        m = s2_gather_list(Sq, list, cnt, lane, m);
                    }
                    if (!any) none |= 1u << b;
                    *reinterpret_cast<float4 *>(&gs.part_max[wave][lane >> 3][4 * (lane & 7)]) = m;
                    s2_wave_sync();
                    if (lane < QLEN) {
                        float v = gs.part_max[wave][0][lane];
#pragma unroll
                        for (int r = 1; r < 8; ++r) v = fmaxf(v, gs.part_max[wave][r][lane]);
                        reinterpret_cast<float *>(list)[lane] = v;
                    }
                    s2_wave_sync();
                }
                if (lane < n) {  // lane a: the sum over the query tokens for the a-th, in double, in index order
                    const float4 *col = reinterpret_cast<const float4 *>(gs.list[wave][lane]);
                    double d = 0.0;
#pragma unroll
                    for (int i4 = 0; i4 < QLEN / 4; ++i4) {
                        const float4 v = col[i4];
                        d += (double)v.x;
                        d += (double)v.y;
                        d += (double)v.z;
                        d += (double)v.w;
                    }
                    const bool empty = (none >> my_bit) & 1u;
                    const float score = (float)d;
                    keys_out[p0 + my_bit] = empty ? PLAID_S2_NO_SCORE : plaid_score_to_ord(score);
                    if (!empty) atomicAdd(&gs.hist[plaid_s2_bin(score, bin_hi, bin_scale)], 1);
                }
                s2_wave_sync();  // the lists are written again for the next candidates
            }
            if (lane == 0 && none) atomicOr(&lempty[h >> 1], none << (16 * (h & 1)));
        }
        __syncthreads();
        if (tid < nw) emptybits[(int64_t)q * cand_words + w0 + tid] = lempty[tid];
        __syncthreads();  // the words are set up again for the next ones
        w0 = we;
    }
    s2_flush_hist(gs.hist, hist + (int64_t)q * SEL_BINS);
    __syncthreads();
}

// A += g where b's bits are set, for 32 passages per lane; A[k] bit p = bit k of the sum of passage p, g < 2^S2_UB_BITS.  A full
// adder is two three-input instructions (v_bitop3_b32: sum 0x96, carry 0xE8; src0, src1, src2 stand for 0xF0, 0xCC, 0xAA)
// once the gain's bit has been masked in; the compiler's own choice for the same expressions took five, and the additions
// were 2000 of the 3400 vector instructions per 2048 passages of a query with 38 survivors.  With that, the comparison
// and the reductions of a round in fewer instructions and rows that are addressed without arithmetic: batch of 150
// queries of 8.8 M passages 9.46 -> 8.66 ms, of 512 of 400 000 2.90 -> 2.74, of 256 of 200 000 561 -> 532 us (whole search).
__device__ __forceinline__ uint32_t s2_gain_bit(int g, int k) { return (uint32_t)(((int32_t)((uint32_t)g << (31 - k))) >> 31); }
__device__ __forceinline__ void s2_add_gain(uint32_t (&A)[S2_UB_BITS], uint32_t b, int g)
{
    const uint32_t g0 = s2_gain_bit(g, 0);
    uint32_t carry = __builtin_amdgcn_bitop3_b32(A[0], b, g0, 0x80);
    A[0] = __builtin_amdgcn_bitop3_b32(A[0], b, g0, 0x78);
#pragma unroll
    for (int k = 1; k < S2_UB_BITS; ++k) {
        const uint32_t x = b & s2_gain_bit(g, k), up = __builtin_amdgcn_bitop3_b32(A[k], x, carry, 0xE8);
        A[k] = __builtin_amdgcn_bitop3_b32(A[k], x, carry, 0x96);
        carry = up;
    }
}
// The passages whose sum is at least `least` (uniform): the carry of sum + ~least + 1, one instruction per bit.
__device__ __forceinline__ uint32_t s2_sum_reaches(const uint32_t (&A)[S2_UB_BITS], int least)
{
    uint32_t ge = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < S2_UB_BITS; ++k) ge = __builtin_amdgcn_bitop3_b32(A[k], s2_gain_bit(least, k), ge, 0xB2);
    return ge;
}

// SHIFT: log2 of the passages per range-table column.  SetT: word that holds a bag's slot set; the 32-bit instance serves
// the queries with at most 31 surviving centroids, the 64-bit instance the others (for small launches: all queries).
// PLAIN: no copies of the histogram and no candidate words given (large batches; the two cost the kernel 2 % there).
// ALL: a 64-bit instance that is launched alone and takes every query; only these lend areas.
// TALL: a 64-bit instance with more planes and fewer workgroups per compute unit (s2_tall_queries).
static_assert(IV_WAVES == 4, "a workgroup is a wave per SIMD");
template <int SHIFT, typename SetT, bool PLAIN, bool ALL, bool TALL>
__global__ __launch_bounds__(64 * IV_WAVES, TALL ? S2_TALL_UNIT_BLOCKS : S2_UNIT_BLOCKS) void s2_invert_kernel(
    const int32_t *__restrict__ uniq, const int32_t *__restrict__ n_uniq, int uniq_stride,
    const int64_t *__restrict__ ivf_offsets, const int32_t *__restrict__ ivf_pids, const uint32_t *__restrict__ table,
    int64_t nr, const float *__restrict__ S, int64_t C, const uint32_t *__restrict__ keepbits, int64_t keep_words,
    const int32_t *__restrict__ codes, const int64_t *__restrict__ doc_offsets, int64_t P, const S2Meta *__restrict__ meta,
    const int32_t *__restrict__ kept_ids, const float *__restrict__ T, uint32_t *__restrict__ candbits, int64_t cand_words,
    uint64_t *__restrict__ keys2, int64_t key_stride, int32_t *__restrict__ hist,
    int32_t *__restrict__ list_counts, uint32_t *__restrict__ emptybits, const int32_t *__restrict__ dense_id,
    const uint32_t *__restrict__ dense_bits, int mode, const int32_t *__restrict__ qcount, const int32_t *__restrict__ qlist, int qlist_stride,
    int nqx, int len_log, int steps, int32_t m, int first_batch, unsigned main_blocks, uint32_t tall)
{
    constexpr int KMAX = sizeof(SetT) == 4 ? 31 : S2_MAX_KEPT;
    // Planes of 64 words that fit a wave's area: what lets four workgroups share a compute unit.  Only lists with an entry in
    // the range's column need one: of the 20 to 32 lists without a bitmap that a query of 40 survivors has on 8.8 M passages,
    // five or more have none in 2048 passages.  Where there are more planes than fit, one wave takes the area of two, or of all
    // four, if the launch has workgroups to spare (mode bits 5 and 7), otherwise half or a quarter of the passages at a time.  (36
    // planes and three workgroups for all queries: 150 of 8.8 M passages 8.66 ms, this 7.2.)
    constexpr int FULL_PLANES = sizeof(SetT) == 4 ? 31 : (SHIFT == 11 ? (TALL ? S2_TALL_PLANES : S2_PLANES) : 24);
    static_assert(4 * FULL_PLANES >= KMAX, "every slot has a plane at a quarter of the length");
    constexpr int SLOTS = KMAX + 1;
    constexpr int MORE = ALL ? 6 : (SHIFT == 11 ? 2 : 4);  // loads in flight per lane of a long list (of a coarse column: four times as long)
    __shared__ __align__(16) uint32_t area_all[IV_WAVES][FULL_PLANES * 64];
    __shared__ __align__(16) float Tl[KMAX * S2_TSTRIDE];
    __shared__ float rowsum[SLOTS];
    __shared__ int32_t kid[SLOTS], drow[SLOTS];  // slot - 1 -> centroid, row of its list's bitmap or -1
    __shared__ int32_t plist[IV_LISTS];    // probed lists of no surviving centroid: bitmap rows from the front, centroids from the back
    __shared__ uint32_t probed_mask[2];    // bit s: slot s + 1 is also probed
    __shared__ int32_t n_front[2], n_sparse;  // [1]: of those from the back
    // per wave; while lists are applied: start (low 32 bits), start (high bits) << 21 | entries << 7 | plane, candidate words;
    // while passages are scored: 16-bit counts of the coarse bins, ranks of the words' first bits, selected words
    __shared__ uint32_t lstart_all[IV_WAVES][64];
    __shared__ uint32_t lcnt_all[IV_WAVES][64];
    __shared__ uint32_t lcand_all[IV_WAVES][64];
    static_assert(S2_COARSE == 128, "two 16-bit coarse counts per lane");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = s2_uniform(tid >> 6);
    uint32_t *lstart = lstart_all[wave];
    uint32_t *lcnt = lcnt_all[wave];
    uint32_t *lcand = lcand_all[wave];
    const bool given = !PLAIN && (mode & 16);  // s2_candidates_kernel has written the candidate words
    if constexpr (sizeof(SetT) == 8) {
        if (blockIdx.x >= main_blocks) {  // uniform: a workgroup of the gather form
            static_assert(sizeof(S2GatherScratch) <= sizeof(area_all), "the gather form's arrays take the place of the planes");
            S2GatherScratch &gs = *reinterpret_cast<S2GatherScratch *>(&area_all[0][0]);
            const int64_t g = blockIdx.x - main_blocks, ng = gridDim.x - main_blocks;
            const int n_more = mode & 4 ? (s2_uniform(meta[0].K) > S2_MAX_KEPT ? 1 : 0) : s2_uniform(qcount[3]);
            const int by_xcd = n_more & ~7;
            const int32_t *more = qlist + 3ll * qlist_stride - 1;  // the i-th is more[-i]
            for (int i = by_xcd ? (int)(blockIdx.x & 7) : 0; i < n_more;) {
                const bool own_xcd = i < by_xcd;
                const int q = mode & 4 ? 0 : s2_uniform(more[-i]);
                s2_gather_share(q, own_xcd ? g >> 3 : g, own_xcd ? ng >> 3 : ng, uniq, n_uniq, uniq_stride, ivf_offsets, ivf_pids,
                                table, nr, SHIFT, S, C, keepbits, keep_words, codes, doc_offsets, P, meta[q].bin_hi,
                                meta[q].bin_scale, candbits, cand_words, keys2, key_stride, hist, emptybits, dense_id, dense_bits, gs,
                                lcand_all[0], lcnt_all[0], plist, n_front, given, mode & 512);
                i = !own_xcd ? i + 1 : (i + 8 < by_xcd ? i + 8 : by_xcd);
            }
            return;
        }
    }
    // This instance's queries, from the lists the probe kernel made: class 1 (1..31 survivors) or 2 (32..63), and with the
    // 32-bit instance class 0 (none) unless s2_union_wide_kernel has produced its candidate and empty-bag words (mode bit
    // 0).  ALL: every query of these classes.  Bit 3: see the launch.  Queries with more survivors belong to the workgroups above.
    // Consecutive workgroups take consecutive queries of one passage range: all queries of a chunk advance together, so that each
    // has a threshold to prune with after its first ranges, and the bitmap rows of the range are shared in the caches.
    const int cls = sizeof(SetT) == 4 ? 1 : 2;
    static_assert(!ALL || sizeof(SetT) == 8, "31 slots do not do for every query");
    const bool single = ALL && (mode & 4);  // one query: number 0, whatever its class
    const int n_first = single ? 1 : (ALL ? qcount[1] : qcount[cls]);
    const int n_second = ALL && !single ? qcount[2] : 0;
    const int n_none = ((cls == 1 || ALL) && !single && !(mode & 1)) ? qcount[0] : 0;
    const int n_all = n_first + n_second + n_none;
    const int rb = (int)(blockIdx.x / (unsigned)nqx);
    for (int qi = (int)(blockIdx.x % (unsigned)nqx); qi < n_all; qi += nqx) {
        const int q = single ? 0 : s2_uniform(qi < n_first ? qlist[(int64_t)(ALL ? 1 : cls) * qlist_stride + qi]
                                              : (qi < n_first + n_second ? qlist[2ll * qlist_stride + qi - n_first]
                                                                         : qlist[qi - n_first - n_second]));
        // everything that does not depend on the number of survivors is requested at once (the tables have room for
        // S2_MAX_KEPT survivors and uniq_stride probes; what lies past their ends is not used)
        const S2Meta mt = meta[q];
        const int kept_lane = tid < S2_MAX_KEPT ? kept_ids[(int64_t)q * S2_MAX_KEPT + tid] : 0;
        const int gain_any = reinterpret_cast<const uint16_t *>(T + (int64_t)q * (S2_MAX_KEPT + 1) * QLEN)[lane];
        const int probed_c = tid < uniq_stride ? uniq[(int64_t)q * uniq_stride + tid] : 0;
        const int K_all = s2_uniform(mt.K);
        if (!ALL && (K_all <= 31) != (sizeof(SetT) == 4)) continue;  // (never: the lists are made from the same K)
        if (K_all > KMAX) continue;  // (a single query of the gather form)
        if (sizeof(SetT) == 8 && !ALL && ((tall >> (K_all - 32)) & 1u) != (TALL ? 1u : 0u)) continue;  // the other 64-bit instance's
        const int lend_most = K_all <= FULL_PLANES ? 0 : (K_all <= 2 * FULL_PLANES ? 1 : 2);
        if (ALL && ((int64_t)rb * IV_WAVES * steps) >> lend_most >= (P + (1ll << len_log) - 1) >> len_log) continue;  // spare
        const int K = K_all;
        const int nu = n_uniq[q];
        __syncthreads();  // the previous query's readers are done
        static_assert(S2_SEEN == 2 * 64 * IV_WAVES && sizeof(area_all) >= S2_SEEN * sizeof(int32_t), "two places a thread, where the planes will be");
        const bool apart = !PLAIN && (mode & 512);  // (launches of fewer than 32 queries)
        if (apart) reinterpret_cast<int2 *>(area_all[0])[tid] = make_int2(-1, -1);
        if (tid < 64) {
            int32_t c = -1, d = -1;
            if (tid < K) {
                c = kept_lane;
                d = dense_id[c];
                kid[tid] = c;
                drow[tid] = d;
            }
            const unsigned long long sm = __ballot(tid < K && d < 0);
            if (tid == 0) {
                n_sparse = __popcll(sm);
                n_front[0] = n_front[1] = 0;
                probed_mask[0] = probed_mask[1] = 0u;
            }
        }
        for (int e = tid; e < K * (QLEN / 4); e += 64 * IV_WAVES)
            *reinterpret_cast<float4 *>(Tl + (e >> 3) * S2_TSTRIDE + 4 * (e & 7)) =
                *reinterpret_cast<const float4 *>(T + (int64_t)q * (S2_MAX_KEPT + 1) * QLEN + QLEN + 4 * e);
        const int gain_lane = lane < K ? gain_any : 0;
        __syncthreads();
        if (tid < K) {  // one survivor in the bag: its row, summed in the same order as in s2_score_rows
            double d = 0.0;
            for (int i = 0; i < QLEN; ++i) d += (double)Tl[tid * S2_TSTRIDE + i];
            rowsum[tid] = (float)d;
        }
        if (!given) {
            static_assert(64 * IV_WAVES >= IV_LISTS, "one thread per probed list");
            if (tid < nu && (!apart || s2_first_probe(reinterpret_cast<int32_t *>(area_all[0]), probed_c))) {
                const int32_t c = probed_c;
                const int32_t d = dense_id[c];
                int slot = -1;
                for (int s = 0; s < K; ++s) slot = kid[s] == c ? s : slot;
                if (slot >= 0) atomicOr(&probed_mask[slot >> 5], 1u << (slot & 31));
                else if (d >= 0) plist[atomicAdd(&n_front[0], 1)] = d;
                else plist[IV_LISTS - 1 - atomicAdd(&n_front[1], 1)] = c;
            }
        }
        __syncthreads();
        const uint32_t pm0 = s2_uniform((int)probed_mask[0]), pm1 = s2_uniform((int)probed_mask[1]);
        const int n_rows = s2_uniform(n_front[0]), n_ss = s2_uniform(n_sparse), n_dense = K - n_ss;
        const int n_sp = s2_uniform(n_front[1]);
        // log2 of the areas that a wave takes
        const int lend = ALL && (mode & 32) && n_ss > FULL_PLANES ? ((mode & 128) && n_ss > 2 * FULL_PLANES ? 2 : 1) : 0;
        uint32_t *area = area_all[(wave << lend) % IV_WAVES];
        // Slots are numbered by list length, so that those with a bitmap come first.  lane i: the row of slot i's / the centroid of
        // the i-th slot without one
        const int dense_row = lane < n_dense ? drow[lane] : 0;
        const int list_c = lane < n_ss ? kid[n_dense + lane] : -1;
        const bool all_probed = (uint32_t)__popc(pm0) + (uint32_t)__popc(pm1) == (uint32_t)K;
        // this workgroup's part of the key list (s2_parts: of a single query, which an instance that takes every query serves), one per XCD
        uint64_t *klist = keys2 + (int64_t)q * key_stride;
        int32_t *count_q = list_counts + (int64_t)q * S2_COUNTS_QUERY;
        if (ALL && (mode & 1024)) {  // uniform
            const int64_t passages = (int64_t)((IV_WAVES >> lend) * steps) << len_log;
            const int64_t at = s2_list_part(rb & (S2_COPIES - 1), passages, P);
            klist += at;
            count_q += (rb & (S2_COPIES - 1)) * S2_COUNT_STRIDE;
            if (rb < S2_COPIES && tid == 0) count_q[1] = (int32_t)at;
        }
        uint32_t *cbq = candbits + (int64_t)q * cand_words;
        uint32_t *ebq = emptybits + (int64_t)q * cand_words;
        int32_t *hist_q = hist + (int64_t)q * SEL_BINS;
        int32_t *coarse_q = hist_q + (!PLAIN && (mode & 8) ? (blockIdx.x & (S2_COPIES - 1)) : 0) * S2_COARSE;
        const int64_t first = ((int64_t)(rb * (IV_WAVES >> lend) + wave) * steps) << len_log;
        int64_t last = first + ((int64_t)steps << len_log) < P ? first + ((int64_t)steps << len_log) : P;
        if (wave >= IV_WAVES >> lend) last = first;  // its area is lent
        const int room = (FULL_PLANES * 64) << lend;  // words
        const int lane0 = lane;
        int len;
        for (int64_t p0 = first; p0 < last; p0 += len) {  // uniform
            int lane = lane0;
            s2_opaque(lane);
            // where the surviving centroids' other lists enter the range; those with an entry in this column of the table get a
            // plane, in the order of the lists (looked at only where the planes may not fit: the loads are used further down)
            const int64_t col = p0 >> SHIFT;
            uint32_t list_a = 0u, list_b = 0u;
            int64_t list_at = 0;
            if (lane < n_ss) {
                list_a = table[(int64_t)list_c * (nr + 1) + col];
                list_b = table[(int64_t)list_c * (nr + 1) + col + 1];
                list_at = ivf_offsets[list_c];
            }
            // The length depends on the column alone: a column's ranges all have the same, so that p0 stays a multiple of it and the
            // wave's last range ends where its part does.
            const unsigned long long has = __ballot(lane < n_ss && list_b > list_a);
            const int n_act = __popcll(has);
            int my_log = len_log;
            if (KMAX > FULL_PLANES)
                while ((n_act << (my_log - 5)) > room) --my_log;
            len = 1 << my_log;
            const int nw = len >> 5;
            const int64_t w0 = p0 >> 5;
            const bool act = lane < nw && w0 + lane < cand_words;  // the lanes that hold a word of the range
            uint32_t valid = 0u;
            if (act) valid = P - (p0 + 32 * lane) >= 32 ? 0xFFFFFFFFu : (1u << (uint32_t)(P - (p0 + 32 * lane))) - 1u;
            // what is known of the scores so far (used below, once the bounds are there)
            const int2 known = s2_coarse_load(coarse_q, lane);
            // bounds, bit-sliced; A[k] bit b = bit k of the gain sum of passage p0 + 32 lane + b.  A range shorter than 2048
            // passages leaves lanes over: groups of nw lanes then take a slot each and add up their sums at the end.
            uint32_t A[S2_UB_BITS];
#pragma unroll
            for (int k = 0; k < S2_UB_BITS; ++k) A[k] = 0u;
            uint32_t any = 0u, cand = given && act ? cbq[w0 + lane] : 0u;
            // a passage with a probed survivor is a candidate; where all survivors are probed (nearly always) `any` tells
            auto add = [&](uint32_t b, int s, int g) {
                any |= b;
                if (!all_probed && (((s < 32 ? pm0 : pm1) >> (s & 31)) & 1u)) cand |= b;
                s2_add_gain(A, b, g);
            };
            const int groups = 64 / nw, grp = lane / nw, gl = lane % nw;
            // The words of the first n_near slots with a bitmap stay in LDS, as far as there is room beside the planes: the bags of
            // the passages that are scored are read from there (search of 150 queries of 8.8 M passages 6198 us with all of
            // them read from memory again, 6097 this way; one 265 / 258; 512 of 400 000 2457 / 2446).
            const int spare = (room >> (my_log - 5)) - n_act, n_near = n_dense < spare ? n_dense : spare;
            const bool gact = w0 + gl < cand_words;
            if (groups == 1) {
                for (int i0 = 0; i0 < n_dense; i0 += 8) {
                    uint32_t v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        v[u] = 0u;
                        if (i0 + u < n_dense && act)
                            v[u] = dense_bits[(int64_t)__builtin_amdgcn_readlane(dense_row, i0 + u) * cand_words + w0 + lane];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (i0 + u < n_dense) {
                            if (i0 + u < n_near) area[(i0 + u) * 64 + lane] = v[u];
                            add(v[u], i0 + u, __builtin_amdgcn_readlane(gain_lane, i0 + u));
                        }
                }
            } else {
                for (int i0 = 0; i0 < n_dense; i0 += 4 * groups) {  // four loads in flight
                    uint32_t v[4];
                    int g[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int i = i0 + u * groups + grp, row = __shfl(dense_row, i & 63);
                        g[u] = __shfl(gain_lane, i & 63);
                        v[u] = i < n_dense && gact ? dense_bits[(int64_t)row * cand_words + w0 + gl] : 0u;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int i = i0 + u * groups + grp;
                        if (i0 + u * groups < n_dense) {  // uniform
                            if (i < n_near) area[i * nw + gl] = v[u];
                            add(v[u], i & 63, g[u]);
                        }
                    }
                }
            }
            // the planes of the survivors' other lists, entry by entry
            const int my_plane = __popcll(has & ((1ull << lane) - 1ull));
            uint32_t *planes = area + n_near * nw;
            for (int i = 0; i < n_act; ++i)
                if (lane < nw) planes[i * nw + lane] = 0u;
            // lane i: the slot of plane i
            if ((has >> lane) & 1ull) lstart[my_plane] = (uint32_t)(n_dense + lane);
            s2_wave_sync();
            const int plane_slot = lane < n_act ? (int)lstart[lane] : 64;
            s2_wave_sync();
            // an entry of the table of lists: start (low 32 bits), start (high bits) << 21 | entries << 7 | plane, 64 = the candidates
            auto put = [&](int at, int64_t start, uint32_t la, uint32_t lb, int plane) {
                start += la;
                lstart[at] = (uint32_t)start;
                // at most 2^13 entries (a list is ascending); lists hold fewer than 2^43 entries together
                lcnt[at] = (uint32_t)((uint64_t)start >> 32) << 21 | (lb > la ? lb - la : 0u) << 7 | (uint32_t)plane;
            };
            // the bits of the entries of nb lists: a quarter of the wave per list, four lists each in flight
            auto walk = [&](int nb) {
                const int sub = lane & 15;
                auto apply = [&](uint32_t pid, int sl) {
                    const uint32_t loc = pid - (uint32_t)p0;
                    if (loc < (uint32_t)len) atomicOr(sl == 64 ? &lcand[loc >> 5] : &planes[sl * nw + (int)(loc >> 5)], 1u << (loc & 31));
                };
                for (int l0 = lane >> 4; l0 < nb; l0 += 16) {
                    int n[4], sl[4];
                    uint32_t pid[4];
                    const int32_t *src[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t pk = l0 + 4 * u < nb ? lcnt[l0 + 4 * u] : 0u;
                        n[u] = (int)((pk >> 7) & 0x3FFFu);
                        sl[u] = (int)(pk & 127u);
                        src[u] = ivf_pids;
                        if (n[u]) src[u] += (uint64_t)(pk >> 21) << 32 | lstart[l0 + 4 * u];
                        if (sub < n[u]) pid[u] = (uint32_t)src[u][sub];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (sub < n[u]) apply(pid[u], sl[u]);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        for (int x = 16 + sub; x < n[u]; x += 16 * MORE) {
                            uint32_t more[MORE];
#pragma unroll
                            for (int y = 0; y < MORE; ++y)
                                if (x + 16 * y < n[u]) more[y] = (uint32_t)src[u][x + 16 * y];
#pragma unroll
                            for (int y = 0; y < MORE; ++y)
                                if (x + 16 * y < n[u]) apply(more[y], sl[u]);
                        }
                }
                s2_wave_sync();
            };
            if ((has >> lane) & 1ull) put(my_plane, list_at, list_a, list_b, my_plane);
            s2_wave_sync();
            walk(n_act);
            if (groups == 1) {
                for (int i0 = 0; i0 < n_act; i0 += 4) {
                    uint32_t b[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) b[u] = i0 + u < n_act ? planes[(i0 + u) * 64 + lane] : 0u;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (i0 + u < n_act) {
                            const int s = __builtin_amdgcn_readlane(plane_slot, i0 + u);
                            add(b[u], s, __builtin_amdgcn_readlane(gain_lane, s));
                        }
                }
            } else {
                const int plane_gain = __shfl(gain_lane, plane_slot & 63);
                for (int i0 = 0; i0 < n_act; i0 += 2 * groups) {
                    uint32_t v[2];
                    int s[2], g[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int i = i0 + u * groups + grp;
                        s[u] = __shfl(plane_slot, i & 63) & 63;
                        g[u] = __shfl(plane_gain, i & 63);
                        v[u] = i < n_act ? planes[i * nw + gl] : 0u;
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (i0 + u * groups < n_act) add(v[u], s[u], g[u]);  // uniform
                }
                for (int d = nw; d < 64; d <<= 1) {
                    uint32_t carry = 0u;
#pragma unroll
                    for (int k = 0; k < S2_UB_BITS; ++k) {
                        const uint32_t x = __shfl_xor(A[k], d), up = __builtin_amdgcn_bitop3_b32(A[k], x, carry, 0xE8);
                        A[k] = __builtin_amdgcn_bitop3_b32(A[k], x, carry, 0x96);
                        carry = up;
                    }
                    cand |= __shfl_xor(cand, d);
                    any |= __shfl_xor(any, d);
                }
            }
            any &= valid;
            cand = (all_probed ? cand | any : cand) & valid;
            // Smallest gain sum whose bound can reach the best m: at least m scores lie in coarse bins 0 .. b, so a bound in a worse
            // bin needs no score.  -1 while fewer than m scores are known.
            auto least_sum = [&](int2 c) -> int {
                const int incl = s2_wave_scan(c.x + c.y);
                const unsigned long long enough0 = __ballot(incl - c.y >= m), enough1 = __ballot(incl >= m);
                if (!enough1) return -1;
                const int l1 = __ffsll((long long)enough1) - 1;
                const int b = 2 * l1 + (((enough0 >> l1) & 1ull) ? 0 : 1);
                const int worst = ((b + 1) << S2_COARSE_SHIFT) - 1;  // last bin of coarse bin b
                // (bins do not rise with the sum)
                auto reaches = [&](int sum) {
                    return plaid_s2_bin(mt.ub_base + mt.ub_unit * (float)sum, mt.bin_hi, mt.bin_scale) <= worst;
                };
                const unsigned long long hi = __ballot(reaches(16 * lane + 15));
                if (!hi) return 1 << S2_UB_BITS;  // no sum does
                const int h = __ffsll((long long)hi) - 1;
                return 16 * h + __ffsll((long long)__ballot(reaches(16 * h + (lane & 15)))) - 1;
            };
            int need = least_sum(known);
            uint32_t left = any;
            if (need >= 0) left = need >> S2_UB_BITS ? 0u : left & s2_sum_reaches(A, need);
            // The probed lists of no surviving centroid, which only make candidates (usually two thirds of the probed lists).  Once m
            // scores are known, what has no survivor cannot be among the best m and nobody reads its bits any more; then the
            // lists matter only to a passage that would be scored and is not known to be a candidate.  (Search of 150 queries of 8.8 M
            // passages, 73 of 106 probed lists without a survivor: 6880 -> 6309 us; 512 of 400 000 2555 -> 2524.)
            if (!given && (need < 0 || (mode & 256) || __any((left & ~cand) != 0u))) {
                for (int d0 = 0; d0 < n_rows; d0 += 8) {
                    uint32_t v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        v[u] = d0 + u < n_rows && act ? dense_bits[(int64_t)s2_uniform(plist[d0 + u]) * cand_words + w0 + lane] : 0u;
#pragma unroll
                    for (int u = 0; u < 8; ++u) cand |= v[u];
                }
                cand &= valid;
                lcand[lane] = cand;
                const int n_lists = __all(cand == valid) ? 0 : n_sp;
                for (int u0 = 0; u0 < n_lists; u0 += 64) {
                    const int e = u0 + lane;
                    if (e < n_lists) {
                        const int32_t c = plist[IV_LISTS - 1 - e];
                        put(lane, ivf_offsets[c], table[(int64_t)c * (nr + 1) + col], table[(int64_t)c * (nr + 1) + col + 1], 64);
                    }
                    s2_wave_sync();
                    walk(n_lists - u0 < 64 ? n_lists - u0 : 64);
                }
                cand = lcand[lane] & valid;
            }
            if ((given || need < 0 || (mode & 256)) && act) {
                cbq[w0 + lane] = cand;
                ebq[w0 + lane] = cand & ~any;
            }
            left &= cand;
            for (int round = 0; __any(left != 0u); ++round) {  // (no round: no candidate with a surviving centroid)
                s2_opaque(lane);
                if (round > 0) {
                    int2 c;
                    // the copies of all XCDs where that pays (see the launch)
                    if (PLAIN || !(mode & 64)) {  // uniform
                        c = s2_coarse_load(coarse_q, lane);
                    } else {
                        int2 v[S2_COPIES];
#pragma unroll
                        for (int x = 0; x < S2_COPIES; ++x) v[x] = s2_coarse_load(hist_q + x * S2_COARSE, lane);
                        c = v[0];
#pragma unroll
                        for (int x = 1; x < S2_COPIES; ++x) {
                            c.x += v[x].x;
                            c.y += v[x].y;
                        }
                    }
                    need = least_sum(c);
                    if (need >> S2_UB_BITS == 1) break;
                    if (need >= 0) left &= s2_sum_reaches(A, need);
                }
                uint32_t sel = left;
                int want = need >= 0 ? 128 : first_batch;
                if (s2_wave_sum(__popc(left)) > 2 * want) {
                    // nothing, or little, to prune with yet: the highest sums (and those that tie with the last of them)
                    uint32_t cur = left;
                    sel = 0u;
#pragma unroll
                    for (int k = S2_UB_BITS - 1; k >= 0; --k) {
                        const uint32_t top = cur & A[k];
                        const int n = s2_wave_sum(__popc(top));
                        if (n >= want) {
                            cur = top;
                        } else {
                            sel |= top;
                            want -= n;
                            cur &= ~A[k];
                        }
                    }
                    sel |= cur;
                }
                left &= ~sel;
                const int pc = __popc(sel);
                const int rank = s2_wave_scan(pc);
                const int total = __builtin_amdgcn_readlane(rank, 63);
                if (total == 0) break;
                // Its round trip overlaps the first batch: the address is one the compiler takes for a lane's own, since it makes of an
                // addition to a uniform one a sum over the wave, and waits for the result at once.
                int base = 0, place = 0;
                s2_opaque(place);
                if (lane == 0) base = atomicAdd(count_q + place, total);
                s2_wave_sync();
                lcnt[lane] = (uint32_t)(rank - pc);
                lcand[lane] = sel;
                lstart[lane] = 0u;
                s2_wave_sync();
                // lane = passage, 64 at a time: by their rank among the selected bits, or, where more than half of the range
                // is selected, in passage order; two lanes per passage when there are at most 32
                constexpr int COLS = SHIFT == 11 || sizeof(SetT) == 4 ? 16 : 4;
                const bool walk_all = 2 * total > len, pairs = COLS == QLEN / 2 && total <= 32;
                const int end = walk_all ? len : total;
                for (int b0 = 0; b0 < end; b0 += 64) {
                    s2_opaque(lane);
                    int w, pos, at;
                    bool live;
                    if (walk_all && !pairs) {
                        w = (b0 + lane) >> 5;
                        pos = lane & 31;
                        const uint32_t word = lcand[w];
                        live = (word >> pos) & 1u;
                        at = (int)lcnt[w] + __popc(word & ((1u << pos) - 1u));
                    } else {
                        at = pairs ? lane >> 1 : b0 + lane;
                        live = at < total;
                        w = 0;
                        pos = 0;
                        if (live) {
#pragma unroll
                            for (int d = 32; d > 0; d >>= 1)
                                if ((int)lcnt[w + d] <= at) w += d;  // the last word whose first selected bit has rank <= at
                            int r = at - (int)lcnt[w];
                            const uint32_t word = lcand[w];
#pragma unroll
                            for (int d = 16; d > 0; d >>= 1) {
                                const int n = __popc((word >> pos) & ((1u << d) - 1u));
                                if (r >= n) {
                                    r -= n;
                                    pos += d;
                                }
                            }
                        }
                    }
                    SetT rows = 0;
                    if (live) {
                        for (int i0 = 0; i0 < n_near; i0 += 8) {
                            uint32_t v[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) v[u] = i0 + u < n_near ? area[(i0 + u) * nw + w] : 0u;
#pragma unroll
                            for (int u = 0; u < 8; ++u) rows |= (SetT)((v[u] >> pos) & 1u) << (i0 + u);
                        }
                        for (int i0 = n_near; i0 < n_dense; i0 += 8) {
                            uint32_t v[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                v[u] = 0u;
                                if (i0 + u < n_dense)
                                    v[u] = dense_bits[(int64_t)__builtin_amdgcn_readlane(dense_row, i0 + u) * cand_words + w0 + w];
                            }
#pragma unroll
                            for (int u = 0; u < 8; ++u) rows |= (SetT)((v[u] >> pos) & 1u) << (i0 + u);
                        }
                        for (int i0 = 0; i0 < n_act; i0 += 8) {
                            uint32_t v[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) v[u] = i0 + u < n_act ? planes[(i0 + u) * nw + w] : 0u;
#pragma unroll
                            for (int u = 0; u < 8; ++u)
                                rows |= (SetT)((v[u] >> pos) & 1u) << (__builtin_amdgcn_readlane(plane_slot, i0 + u) & 63);
                        }
                    }
                    // bags of one member are a look-up, and a wave of nothing else (few survivors) skips the rows
                    const bool one = (rows & (rows - 1)) == 0;
                    float score = live && one ? rowsum[s2_first_bit(rows)] : 0.f;
                    if (__any(!one)) {
                        const float sum = s2_score_rows<COLS>(one ? (SetT)0 : rows, Tl, rowsum, pairs, lane);
                        if (!one) score = sum;
                    }
                    if (pairs) live = live && (lane & 1);
                    const int bin = live ? plaid_s2_bin(score, mt.bin_hi, mt.bin_scale) >> S2_COARSE_SHIFT : -1;
                    // coarse counts in LDS; many equal bins (few survivors: few distinct scores) as one addition
                    const int lead = __builtin_amdgcn_readlane(bin, 1);  // (an odd lane: those score where lanes pair up)
                    const unsigned long long same = __ballot(bin == lead);
                    if (lead >= 0 && __popcll(same) >= 8) {
                        if (lane == 0) atomicAdd(&lstart[lead >> 1], (uint32_t)__popcll(same) << (16 * (lead & 1)));
                    } else if (bin >= 0 && bin == lead) {
                        atomicAdd(&lstart[bin >> 1], 1u << (16 * (bin & 1)));
                    }
                    if (bin >= 0 && bin != lead) atomicAdd(&lstart[bin >> 1], 1u << (16 * (bin & 1)));
                    if (b0 == 0) base = s2_uniform(base);
                    if (live) klist[base + at] = plaid_make_key(score, (uint32_t)(p0 + 32 * w + pos));
                }
                s2_wave_sync();
                // (both of a lane's bins in one addition)
                const uint32_t counts = lstart[lane];
                if (counts)
                    atomicAdd(reinterpret_cast<unsigned long long *>(coarse_q) + lane, (unsigned long long)(counts >> 16) << 32 | (counts & 0xFFFFu));
            }
            s2_wave_sync();  // the next range's planes overwrite what the last batch read
        }
    }
}

// log2 of the passages per wave and step: 2048, fewer for indexes of so few passages that a wave's own chain of steps is all that counts
// and the chip has room for more waves.  512 at least and up to 400 ranges of a query: beyond, what they add to one histogram and score
// before there is a threshold costs more.  us per search with 2048 / 1024 / 512 / 256: one query of 40 000 passages 73 / 70 / 70 / 73, of
// 100 000 85 / 82 / 84 / 82, of 200 000 76 / 78 / 75 / 80, of 400 000 99 / 94 / 99 / 119 (ndocs 4096 131 / 123 / 129 / 148), of a million
// 101 / 112 / 132 / 178; four of 100 000 112 / 106 / 105 / 108, of 200 000 94 / 92 / 93 / 103, of 400 000 120 / 120 / 131 / 151.  Between
// 400 000 and a million (2048 / 1024, k 100): one query of 450 000 93 / 88, of 500 000 94 / 89, of 600 000 90 / 94, of 700 000 91 / 97, of
// 900 000 94 / 99; four of 450 000 113 / 116, of 500 000 112 / 118, of 600 000 117 / 126.
// The smallest collections: down to 128, up to 100 ranges of a query and while the launch then has at most 2560 waves, beyond 8192
// passages only while a wave's share of m is more than 16.  With 512 / 256 / 128 and the first batches below: ndocs a tenth of the
// passages, eight queries of 2000 81 / 77 / 73, of 5000 94 / 89 / 84, of 12 000 95 / 93 / 87, 33 of 5000 121 / 116 / 112, of 8000 140 / 140 /
// 134; a quarter, eight of 5000 110 / 101 / 90, 33 162 / 154 / 145; a fiftieth, eight of 5000 78 / 76 / 75, of 12 000 78 / 75 / 75, one of
// 10 000 66 / 68 / 67, 33 of 8000 100 / 98 / 99.  Of 20 000, ndocs a twentieth, one 78 / 74 / 76, fifteen 104 / 102 / 98.  Beyond: one of
// 30 000, ndocs 1024, 76 / 79 / -; 33 of 10 000 147 / 150 / -; 48 of 12 000 173 / 174 / 179.
static constexpr int s2_range_log(int64_t P, int64_t nq, int64_t m)
{
    const int64_t ranges = (P + 2047) >> 11, waves = nq * ranges;
    int len_log = 11;
    while (len_log > 9 && (ranges << (12 - len_log)) <= 400 && (waves << (12 - len_log)) <= 2560) --len_log;
    while (len_log <= 9 && len_log > 7 && (P <= 8192 || (m << len_log) / P > 16) && (ranges << (12 - len_log)) <= 100 &&
           (waves << (12 - len_log)) <= (len_log == 9 ? 1280 : 2560))
        --len_log;
    // An ndocs so large that a wave has several batches to score in any case (one query of 400 000 passages, ndocs 100 000: stage 2 and
    // selection 208 -> 158 us, all 400 000 345 -> 87; 64 queries 1129 -> 1030 and 1534 -> 910; scored by four waves per range, in the
    // order of the bags' sizes: 115, 58, 695, 529): shorter ranges while the chip has room.
    while (len_log > 9 && (m << len_log) / P > 128 && (waves << (12 - len_log)) <= 2560) --len_log;
    // A collection of which a large share is kept: down to 128, while a wave's share of m is more than 64 and a query has up to 400 ranges
    // (one query of 40 000, half of them kept, 264 / 252 / 246).
    while (len_log > 7 && (m << len_log) / P > 64 && (ranges << (12 - len_log)) <= 400 && (waves << (12 - len_log)) <= 2560) --len_log;
    return len_log;
}

// Ranges that a wave takes one after the other (waves: how many there are with one each).  The set-up of a workgroup (10 us when
// the chip is full) is worth sharing once every SIMD has dozens of waves to run (512 queries of 400 000 passages: 3.12 / 3.11 /
// 3.16 ms with 1 / 2 / 4 steps, 150 of 8.8 M: 13.3 / 12.6 / 12.4 ms).  A single query of somewhat more ranges than the chip holds
// waves (4096): two each, so that no second round of few waves follows the first and the second ranges find a threshold.  With
// more ranges the second round is nearly a whole one and prunes by what the first has found, and half the waves, two ranges each, take
// longer.  us per search with one / two, millions of passages, nprobe 4 and ndocs 4096: 8.8 290 / 276, 10.6 307 / 292, 12 303 / 288,
// 12.8 311 / 297, 14 318 / 319, 16 318 / 340, 20 358 / 390; nprobe 1 and ndocs 256: 226 / 189, 230 / 188, 233 / 211, 227 / 213,
// 246 / 242, 232 / 248, 260 / 284.
static constexpr int s2_steps(int nq, int64_t waves)
{
    return waves >= 16 * 12288 ? 4 : (waves >= 4 * 12288 || (nq == 1 && waves > 4096 && waves <= 7000) ? 2 : 1);
}

// Passages a wave scores before there is a threshold, or its share of m, which has to be scored whatever the bounds say: 24 (and those
// that tie with the last of them), which mostly fit a batch of 32 in which two lanes share a passage, 48 in whole ranges of large searches.
// us per search with 24 / 32 / 48 / 64, ranges of 2048: 33 queries of 400 000 passages, ndocs 4096, 490 / 486 / 479 / 476, ndocs 256 212 /
// 211 / 212 / 213; 128 1379 / 1366 / 1361 / 1365; 33 of 600 000 523 / 514 / 506 / 506; one of 3 M, ndocs 16 384, 315 / 309 / 304 / 300, ndocs 4096
// 172 / 173 / 170 / 170; sixteen of 200 000, ndocs 1024, 128 / 129 / 130 / 133; 32 of 600 000 286 / 287 / 292 / 295.  Shorter ranges: one
// of 400 000, ndocs 4096, 121 / 122 / 123 / 125; of 200 000 107 / 107 / 110 / 110; of 30 000, ndocs 1024, 77 / 78 / 78 / 84.  Of 128, which are
// chosen where much of a small collection is kept, 64: eight of 5000, ndocs 500, 86 / 87 / - / 84, ndocs 1250 95 / 95 / - / 90, ndocs 100 75 / 75 /
// - / 75; 33 153 / 153 / - / 145.
static constexpr int64_t s2_first_batch(int64_t P, int64_t nq, int64_t m, int len_log)
{
    const int64_t share = (m << len_log) / P, few = len_log == 7 ? 64 : len_log == 11 && (nq > 32 || m >= 4096) ? 48 : 24;
    return share > few ? share : few;
}

// Whether a query's key list is in parts.  The waves of a single query reserve their first places at about the same time, and some ten
// nanoseconds after one another where there is one counter: up to 20 us for the last of two thousand.  Parts cost the selection a
// microsecond or two, which reads their numbers first.  us per search with one list / parts, one query, by its number of waves, nprobe 1
// and ndocs 256, 2 and 1024, 4 and 4096: 391 66.6 / 66.6, 71.0 / 72.5, 99.5 / 100.3; 398 71.1 / 71.4, 77.7 / 78.4, 109.7 / 110.1; 416 73.8
// / 74.1, 79.3 / 80.1, 111.1 / 111.6; 440 72.2 / 71.6, 78.8 / 79.6, 111.6 / 111.6; 464 75.1 / 75.0, 80.1 / 81.3, 112.5 / 113.1; 489 72.0 /
// 70.8, 79.1 / 78.9, 113.6 / 113.5; 586 73.9 / 72.2, 79.8 / 79.3, 113.9 / 113.2; 733 77.6 / 75.1, 84.5 / 83.6, 116.6 / 114.8; 977 83.2 /
// 79.8, 91.1 / 89.4, 121.6 / 118.8; shorter ranges (ndocs 60 000 to 300 000): 450 247.5 / 247.2, 782 308 / 302, 977 623 / 615.  Four
// queries of 2 M passages 113 / 110, 133 / 133, 167 / 168, of 4 M 149 / 149; sixteen of 400 000 152 / 155, of 2 M 253 / 260, of 4 M 337 /
// 352.
static constexpr bool s2_parts(int nq, int64_t waves) { return nq == 1 && waves > 480; }

// The numbers of survivors K (bit K - 32) whose queries the TALL instance takes in launches of many workgroups.  share: how
// often a surviving centroid needs a plane (plaid_launch_ivf_plane_share): K of them need K share, give or take the root of K share
// (1 - share).  With 26 planes four workgroups run on a compute unit, with 36 three: the second wins where it goes through whole
// ranges or halves and the first through halves or quarters.  Even lists of 2 M passages, share 0.97, 200 queries, us per search with
// 26 / 36 planes: K = 33 2573 / 2225, 36 2742 / 2337, 40 2977 / 3478, 52 3402 / 4019, 56 4562 / 4141, 62 4885 / 4433; share 0.85: K = 33
// 2383 / 1999, 40 2554 / 2427, 46 2669 / 3131, 62 4101 / 3678; share 0.71: K = 33 2012 / 2024, 36 2314 / 2062, 46 2745 / 2538, 52 2852 /
// 3172.  Popularities as uneven as Zipf(1.1) give 0.4 to 0.5; so few planes leave little to gain, and their launches are spared one
// that is mostly empty.
static constexpr uint32_t s2_tall_queries(double share)
{
    uint32_t set = 0u;
    if (share > 1.0) share = 1.0;
    for (int K = 32; share > 0.65 && K <= S2_MAX_KEPT; ++K) {
        const double n = K * share;
        auto fit = [=](double planes) { return n <= planes && 4.0 * (planes - n) * (planes - n) >= n * (1.0 - share); };
        if ((!fit(S2_PLANES + 0.5) && fit(S2_TALL_PLANES + 0.5)) || !fit(2 * S2_PLANES + 0.5)) set |= 1u << (K - 32);
    }
    return set;
}

bool plaid_launch_stage2_inverted(hipStream_t st, const int32_t *uniq, const int32_t *n_uniq, int uniq_stride,
                                  const int64_t *ivf_offsets, const int32_t *ivf_pids, const uint32_t *table, const float *S,
                                  int64_t C, const uint32_t *keepbits, int64_t keep_words, const int32_t *codes,
                                  const int64_t *doc_offsets, int64_t P, int nq, const Stage2Buffers &b, uint32_t *candbits,
                                  int64_t cand_words, uint64_t *keys2, int64_t key_stride, const int32_t *dense_id,
                                  const uint32_t *dense_bits, double plane_share, int shift, int32_t m, bool all_candidates)
{
    const int64_t nr = (P + (1ll << shift) - 1) >> shift;
    const int64_t nwide = (P + (1ll << UW_SHIFT) - 1) >> UW_SHIFT;
    // One workgroup per query and 2^19 passages pays off once the launch holds enough queries to fill the chip with such
    // workgroups; below that the range kernel also takes the queries without a surviving centroid.
    const int wide = nq >= IVR_WIDE_MIN_QUERIES ? 1 : 0;
    if (wide)
        hipLaunchKernelGGL(s2_union_wide_kernel, dim3((unsigned)nwide, nq), dim3(UW_THREADS), 0, st, uniq, n_uniq, uniq_stride,
                           ivf_offsets, ivf_pids, table, nr, shift, P, b.meta, dense_id, dense_bits, candbits, cand_words,
                           b.emptybits);
    const int base = wide | (all_candidates ? 256 : 0) | (b.probes_apart ? 512 : 0);
    const int given = uniq_stride > IV_LISTS ? 16 : 0;
    if (given)
        hipLaunchKernelGGL(s2_candidates_kernel, dim3((unsigned)((cand_words + 63) / 64), nq), dim3(64 * IV_WAVES), 0, st, uniq, n_uniq,
                           uniq_stride, ivf_offsets, ivf_pids, table, nr, shift, P, b.meta, dense_id, dense_bits, candbits, cand_words,
                           wide);
    const int64_t ranges = (P + 2047) >> 11, waves = (int64_t)nq * ranges;
    const int len_log = s2_range_log(P, nq, m);
    const int steps = s2_steps(nq, waves);
    const int64_t per_block = (int64_t)(IV_WAVES * steps) << len_log;
    const int first_batch = (int)s2_first_batch(P, nq, m, len_log);
    const int64_t blocks = (P + per_block - 1) / per_block;
    // workgroups of the gather form: no more than there are bitmap words to share, and a multiple of eight
    const int64_t words = (nq * cand_words + 7) & ~7ll;
    const unsigned gather = words < S2_GATHER_BLOCKS ? (unsigned)words : S2_GATHER_BLOCKS;
    const unsigned gather_tall = words < 256 * S2_TALL_UNIT_BLOCKS ? (unsigned)words : 256 * S2_TALL_UNIT_BLOCKS;
    const uint32_t tall = shift == 11 ? s2_tall_queries(plane_share) : 0u;
#define S2_INVERT(SH_, T_, PLAIN_, ALL_, TALL_, MODE_, NQX_, BLOCKS_, GATHER_)                                                   \
    hipLaunchKernelGGL((s2_invert_kernel<SH_, T_, PLAIN_, ALL_, TALL_>), dim3((unsigned)((BLOCKS_) * (NQX_)) + (GATHER_)),                    \
                       dim3(64 * IV_WAVES), 0, st, uniq,                                                                      \
                       n_uniq, uniq_stride, ivf_offsets, ivf_pids, table, nr, S, C, keepbits, keep_words, codes, doc_offsets, \
                       P, b.meta, b.kept_ids, b.T, candbits, cand_words, keys2, key_stride, b.hist, b.list_counts,          \
                        b.emptybits, dense_id, dense_bits, MODE_, b.qcount, b.qlist, b.qlist_stride, NQX_, len_log,  \
                       steps, m, first_batch, (unsigned)((BLOCKS_) * (NQX_)), tall)
    // Updates of one histogram from several XCDs travel between their caches (one query of 8.8 M passages: 0.2 ms for the
    // updates alone).  Workgroups are dealt to the eight XCDs in turn: with many queries their number, per passage range,
    // is made a multiple of eight (empty ones added), so that a query's workgroups share an XCD.  With few, that would
    // leave XCDs and, in the end, most of the chip waiting for the query with the most to do: an odd number spreads
    // every query over all XCDs, each of which counts in a copy of its own (mode bit 3).  That copy alone, an eighth of the
    // scores, gives a threshold that lets through up to eight times as many as all copies do: 8 m scores in all, so
    // once that is several per wave, a wave reads the others' copies too after its first batch (mode bit 6; one query,
    // own / all: ndocs 256 of 5.2 M passages 78 / 92 us, 1024 of 4 M 67 / 69, 4096 of 8.8 M 195 / 183, 1024 of 1 M 84 / 76, of
    // 400 000, three queries, 45 / 37).  Stage 2 and selection, us, multiple of eight / spread, copies read singly / all:
    //   7 and 8 queries of 2 M passages (65536 centroids)   311 / 202 / 172    219 / 232 / 166
    //   8, 16, 32 queries of 8.8 M                          1000, 1360, 2350 / - / 600, 950, 1710
    //   40, 64 of 400 000                                   139, 187 / - / 141, 191      of 2 M: 403, 552 / - / 451, 622
    const bool spread = nq <= 32;
    const int nqx = spread ? (nq | 1) : (nq + 7) & ~7;
    const int copies = spread && nq * blocks > 64 ? (4ll * m >= 3 * ((P + (1ll << len_log) - 1) >> len_log) ? 8 | 64 : 8) : 0;
    const bool parts = copies && s2_parts(nq, (P + (1ll << len_log) - 1) >> len_log);
    const int own = copies | given | (parts ? 1024 : 0);
    // Few workgroups, at most S2_FITS_BLOCKS: the 64-bit instance alone, taking every query (same sets, same scores, one launch
    // less, and no waiting of one class for the other: eight queries of 400 000 passages, thresholds 0.45 / 0.38 / 0.36: 83 / 138 /
    // 126 -> 73 / 72 / 102 us; 24 of 200 000, 0.5 / 0.36: 71 / 113 -> 65 / 70); with twice the workgroups, so that queries with
    // more slots than a wave's area holds can have two (mode bit 5), or four times, where they all run at once, for four areas (bit
    // 7; four queries of 400 000 passages, even lists, 62 survivors 192 -> 148 us).  More: the 32-bit instance's scoring wins
    // (eight of 2 M: 232 with two, 327 with one).  The line: 768 and 1024 make no difference beyond 2 % (16 of 400 000: 166 / 164
    // us per search, 32 and 40 of 200 000: 146 / 143 and 155 / 152, eight of 1 M: 160 / 160).
    const bool fits = blocks * nqx <= S2_FITS_BLOCKS;
    if (nq < 8 || fits) {
        const bool fits4 = 4 * blocks * nqx <= 256 * S2_UNIT_BLOCKS;
        const int mode = base | (nq == 1 ? 4 : 0) | own | (fits ? 32 : 0) | (fits4 ? 128 : 0);
        const int64_t all = fits4 ? 4 * blocks : (fits ? 2 * blocks : blocks);
        // (where the second areas do not come from workgroups that run at once, queries of 27 to 36 lists are better off with the
        // planes for them: twelve of 400 000 passages, even lists, K = 33 211 -> 164 us)
        if (tall && fits && 2 * blocks * nqx > 256 * S2_UNIT_BLOCKS)
            S2_INVERT(11, unsigned long long, false, true, true, mode, nqx, all, gather_tall);
        else if (shift == 11) S2_INVERT(11, unsigned long long, false, true, false, mode, nqx, all, gather);
        else S2_INVERT(13, unsigned long long, false, true, false, mode, nqx, all, gather);
    } else {
        // the class of the 64-bit instance is empty or small more often than not: 128 columns of workgroups share it
        const int many = nqx < 128 ? nqx : 128;
        if (shift == 11) {
            if (own) S2_INVERT(11, uint32_t, false, false, false, base | own, nqx, blocks, 0u);
            else S2_INVERT(11, uint32_t, true, false, false, base, nqx, blocks, 0u);
            if (tall) S2_INVERT(11, unsigned long long, false, false, true, base | own, many, blocks, 0u);
            S2_INVERT(11, unsigned long long, false, false, false, base | own, many, blocks, gather);
        } else {
            if (own) S2_INVERT(13, uint32_t, false, false, false, base | own, nqx, blocks, 0u);
            else S2_INVERT(13, uint32_t, true, false, false, base, nqx, blocks, 0u);
            S2_INVERT(13, unsigned long long, false, false, false, base | own, many, blocks, gather);
        }
    }
#undef S2_INVERT
    return parts;
}

// ------------------------------------------------------------------ host side
void plaid_launch_stage2(hipStream_t st, const float *S, int64_t C, const uint32_t *keepbits, int64_t keep_words,
                         const int32_t *probed, int nprobe, const uint32_t *candbits, int64_t cand_words, int64_t P,
                         int64_t N, const int64_t *doc_offsets, const int32_t *codes, int nq, const Stage2Buffers &b,
                         uint64_t *keys2, int64_t key_stride)
{
    (void)probed;
    (void)nprobe;
    // persistent workgroups; enough of them to fill the chip for one query, fewer per query in a large chunk
    const int64_t ntiles = (P + S2W_PASS - 1) / S2W_PASS;
    int64_t gs = (ntiles + 3) / 4;
    const int64_t gcap = nq >= 16 ? 96 : (nq >= 4 ? 320 : 1280);
    if (gs > gcap) gs = gcap;
    hipLaunchKernelGGL(s2_stream_kernel, dim3((unsigned)gs, nq), dim3(S2_THREADS), 0, st, S, C, keepbits, keep_words, codes, N,
                       doc_offsets, P, candbits, cand_words, b.meta, b.kept_ids, b.T, keys2, key_stride, b.hist,
                       b.emptybits);
}
