// Vanilla ColBERTv2 candidate generation (Section 4.1), the baseline PLAID is compared with: the inverted list of a
// centroid holds the ids of the EMBEDDINGS assigned to it, so the candidate passages of a query are found by walking
// the embedding lists of its probed centroids and looking up the passage of every embedding.
#include "plaid_internal.h"

// probebits[q] = bitmap over the centroids of the query's distinct probed centroids (zero on entry); qmask (null: not
// wanted; zero on entry), one word per centroid and 32 queries: bit q & 31 of qmask[(q >> 5) * C + c] = query q probes c;
// work[0] += the lengths of the probed embedding lists, in units of VAN_UNIT entries.
#define VAN_UNIT 512
__global__ __launch_bounds__(256) void van_probe_mask_kernel(const int32_t *__restrict__ uniq, const int32_t *__restrict__ n_uniq,
                                                             int uniq_stride, uint32_t *__restrict__ probebits, int64_t keep_words,
                                                             const int64_t *__restrict__ eoff, int64_t C,
                                                             uint32_t *__restrict__ qmask, uint32_t *__restrict__ work)
{
    const int q = blockIdx.x;
    const int nu = n_uniq[q];
    unsigned long long entries = 0;
    for (int u = threadIdx.x; u < nu; u += blockDim.x) {
        const uint32_t c = (uint32_t)uniq[(int64_t)q * uniq_stride + u];
        atomicOr(&probebits[(int64_t)q * keep_words + (c >> 5)], 1u << (c & 31));
        if (qmask) {
            atomicOr(&qmask[(int64_t)(q >> 5) * C + c], 1u << (q & 31));
            entries += (unsigned long long)(eoff[c + 1] - eoff[c]);
        }
    }
    for (int d = 1; d < 64; d <<= 1) entries += __shfl_xor(entries, d);
    if (qmask && (threadIdx.x & 63) == 0 && entries) atomicAdd(work, (uint32_t)((entries + VAN_UNIT - 1) / VAN_UNIT));
}

// Which of the two kernels below finds the candidates: the walk of the embedding lists costs about 20 ps per entry of a
// probed list, reading every passage's codes 3 ps per token for each 32 queries (both measured on 26 M tokens), and the
// lists of a query hold more than half of the tokens as soon as it probes the centroids that are in nearly every passage.
__device__ __forceinline__ bool van_by_codes(const uint32_t *work, int64_t N, int nq)
{
    return (int64_t)work[0] * VAN_UNIT > N / 4 * ((nq + 31) / 32);
}

// Candidates from the passages' codes: a wave reads the codes of 16 passages, 16 lanes each, and ORs the queries' masks of
// the centroids it meets; the workgroup's 64 passage masks are then turned into 64 bits of every query's bitmap.  Bound by
// the gathers of the masks (4 bytes per token from an L2-resident table).  Sixteen queries on 26 M tokens: 4.7 ms for the
// walk of their lists, 0.1 ms this way.
__global__ __launch_bounds__(256) void van_codes_kernel(const int64_t *__restrict__ doc_offsets, const int32_t *__restrict__ codes,
                                                        int64_t P, int64_t N, int64_t C, int nq, const uint32_t *__restrict__ qmask,
                                                        const uint32_t *__restrict__ work, uint32_t *__restrict__ candbits,
                                                        int64_t cand_words)
{
    if (!van_by_codes(work, N, nq)) return;  // uniform
    __shared__ uint32_t pm[64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t *mask = qmask + (int64_t)blockIdx.y * C;
    for (int64_t b = blockIdx.x; b * 64 < P; b += gridDim.x) {
        for (int r = 0; r < 4; ++r) {
            const int at = 16 * wave + 4 * r + (lane >> 4);
            const int64_t p = b * 64 + at;
            int64_t t0 = 0, t1 = 0;
            if (p < P) {
                t0 = doc_offsets[p];
                t1 = doc_offsets[p + 1];
            }
            uint32_t v = 0u;
            for (int64_t t = t0 + (lane & 15); t < t1; t += 64) {
                int32_t c[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) c[u] = t + 16 * u < t1 ? codes[t + 16 * u] : -1;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c[u] >= 0) v |= mask[c[u]];
            }
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) v |= __shfl_xor(v, d);
            if ((lane & 15) == 0) pm[at] = v;
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t v = pm[lane];
            unsigned long long mine = 0;
#pragma unroll
            for (int k = 0; k < 32; ++k) {
                const unsigned long long bits = __ballot((v >> k) & 1u);
                if (lane == k) mine = bits;
            }
            const int64_t q = 32ll * blockIdx.y + lane;
            if (lane < 32 && q < nq) {
                uint32_t *out = candbits + q * cand_words + 2 * b;
                out[0] = (uint32_t)mine;
                if (2 * b + 1 < cand_words) out[1] = (uint32_t)(mine >> 32);
            }
        }
        __syncthreads();
    }
}

// candbits[q] |= passages owning an embedding of the probed centroids' embedding lists.  The lists of a query form one
// flat range of work (prefix sums of the list lengths in LDS, a thread finds its list by binary search), spread over
// the grid's x dimension.  Consecutive embeddings mostly belong to one passage: a bit already seen set is not set again.
#define VAN_BATCH 256
__global__ __launch_bounds__(256) void van_union_kernel(const int32_t *__restrict__ uniq, const int32_t *__restrict__ n_uniq,
                                                        int uniq_stride, const int64_t *__restrict__ eoff,
                                                        const int32_t *__restrict__ eids, const int32_t *__restrict__ tok2pid,
                                                        uint32_t *__restrict__ candbits, int64_t cand_words,
                                                        const uint32_t *__restrict__ work /* null: always */, int64_t N)
{
    if (work && van_by_codes(work, N, gridDim.y)) return;  // uniform
    __shared__ int64_t start[VAN_BATCH];
    __shared__ int64_t pref[VAN_BATCH + 1];
    const int q = blockIdx.y;
    const int nu = n_uniq[q];
    uint32_t *bits = candbits + (int64_t)q * cand_words;
    for (int u0 = 0; u0 < nu; u0 += VAN_BATCH) {
        const int nb = nu - u0 < VAN_BATCH ? nu - u0 : VAN_BATCH;
        __syncthreads();
        if ((int)threadIdx.x < nb) {
            const int32_t c = uniq[(int64_t)q * uniq_stride + u0 + threadIdx.x];
            start[threadIdx.x] = eoff[c];
            pref[threadIdx.x + 1] = eoff[c + 1] - eoff[c];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            pref[0] = 0;
            for (int t = 0; t < nb; ++t) pref[t + 1] += pref[t];
        }
        __syncthreads();
        const int64_t total = pref[nb];
        for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < total; w += (int64_t)gridDim.x * blockDim.x) {
            int lo = 0, hi = nb;  // largest lo with pref[lo] <= w
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (pref[mid] <= w) lo = mid;
                else hi = mid;
            }
            const uint32_t pid = (uint32_t)tok2pid[eids[start[lo] + (w - pref[lo])]];
            uint32_t *word = bits + (pid >> 5);
            const uint32_t bit = 1u << (pid & 31);
            if ((*word & bit) == 0u) atomicOr(word, bit);  // a stale read only costs a redundant atomic
        }
    }
}

void plaid_launch_vanilla_candidates(hipStream_t st, const int32_t *uniq, const int32_t *n_uniq, int uniq_stride,
                                     const int64_t *eoff, const int32_t *eids, const int32_t *tok2pid, int nq, int64_t keep_words,
                                     uint32_t *probebits, uint32_t *candbits, int64_t cand_words, const int64_t *doc_offsets,
                                     const int32_t *codes, int64_t P, int64_t N, int64_t C, uint32_t *qmask, uint32_t *work)
{
    hipLaunchKernelGGL(van_probe_mask_kernel, dim3(nq), dim3(256), 0, st, uniq, n_uniq, uniq_stride, probebits, keep_words, eoff,
                       C, qmask, work);
    const int gx = nq >= 16 ? 64 : (nq >= 4 ? 256 : 1024);
    hipLaunchKernelGGL(van_union_kernel, dim3(gx, nq), dim3(256), 0, st, uniq, n_uniq, uniq_stride, eoff, eids, tok2pid, candbits,
                       cand_words, qmask ? work : nullptr, N);
    if (qmask) {
        const int64_t blocks = (P + 63) / 64;
        hipLaunchKernelGGL(van_codes_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192), (unsigned)((nq + 31) / 32)), dim3(256),
                           0, st, doc_offsets, codes, P, N, C, nq, qmask, work, candbits, cand_words);
    }
}
