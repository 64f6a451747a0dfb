// Batched top-m selection on unique 64-bit ranking keys (ascending key = better rank).
//
// Every cut of the pipeline (nprobe centroids per token, ndocs after stage 2, ndocs/4 after
// stage 3, k at the end) is "the m smallest keys of a list".  Lists of up to SEL_SORT_CAP keys are
// sorted by one workgroup in LDS.  Longer lists go through a two-level most-significant-digit
// radix selection that starts below the keys' common prefix (the producer accumulates the AND/OR
// of its keys): level 0 histograms an 11-bit digit over the whole list, level 1 over the keys that
// fell into the boundary bin; keys in lower bins are selected for sure, the remaining boundary
// (normally a handful of exact score ties) is resolved by the finishing workgroup, which falls
// back to an in-block radix selection over global memory if that boundary is still long.
// Nothing is read back to the host; all counts live in device memory.
#include "plaid_internal.h"

#include <math.h>

#define SEL_THREADS 256
#define FIN_THREADS 1024

__device__ __forceinline__ SelState *state_of(SelState *base, int seg) { return base + seg; }

// ------------------------------------------------------------------ AND/OR of a list (when the producer has not)
__global__ __launch_bounds__(SEL_THREADS) void sel_andor_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                const int32_t *__restrict__ counts, SelState *state)
{
    const int seg = blockIdx.y;
    const int n = counts[seg];
    const uint64_t *k = keys + (int64_t)seg * key_stride;
    unsigned long long o = 0, no = 0;
    for (int64_t i = (int64_t)blockIdx.x * SEL_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * SEL_THREADS) {
        const unsigned long long v = k[i];
        o |= v;
        no |= ~v;
    }
    for (int d = 1; d < 64; d <<= 1) {
        o |= __shfl_xor(o, d);
        no |= __shfl_xor(no, d);
    }
    if ((threadIdx.x & 63) == 0 && (o | no)) {
        SelState *s = state_of(state, seg);
        atomicOr(&s->key_or, o);
        atomicOr(&s->key_nor, no);
    }
}

__device__ __forceinline__ void digit_plan(const SelState *s, int &shift0, int &width0, int &shift1, int &width1)
{
    const unsigned long long diff = s->key_or & s->key_nor;  // bits in which the keys differ
    const int hi = diff ? 63 - __clzll((long long)diff) : -1;
    width0 = hi + 1 < SEL_RADIX_BITS ? hi + 1 : SEL_RADIX_BITS;
    shift0 = hi + 1 - width0;
    width1 = shift0 < SEL_RADIX_BITS ? shift0 : SEL_RADIX_BITS;
    shift1 = shift0 - width1;
}
__device__ __forceinline__ int digit_of(uint64_t key, int shift, int width)
{
    return (int)((key >> shift) & ((1u << width) - 1u));
}

// ------------------------------------------------------------------ level-0 histogram over the whole list
__global__ __launch_bounds__(SEL_THREADS) void sel_hist0_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                const int32_t *__restrict__ counts, int32_t m,
                                                                SelState *state, int32_t *__restrict__ hist)
{
    __shared__ int32_t lh[SEL_BINS];
    const int seg = blockIdx.y;
    SelState *s = state_of(state, seg);
    const int n = counts[seg];
    int shift0, width0, shift1, width1;
    digit_plan(s, shift0, width0, shift1, width1);
    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) lh[b] = 0;
    __syncthreads();
    const uint64_t *k = keys + (int64_t)seg * key_stride;
    for (int64_t i = (int64_t)blockIdx.x * SEL_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * SEL_THREADS)
        atomicAdd(&lh[digit_of(k[i], shift0, width0)], 1);
    __syncthreads();
    int32_t *gh = hist + (int64_t)seg * 2 * SEL_BINS;
    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS)
        if (lh[b]) atomicAdd(&gh[b], lh[b]);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        s->n_in = n;
        s->m_rem[0] = m < n ? m : n;
        s->shift[0] = shift0;
        s->width[0] = width0;
        s->shift[1] = shift1;
        s->width[1] = width1;
    }
}

// Finds the boundary bin of a histogram: the smallest b with count(bins <= b) >= m_rem.  Every thread of
// the block returns the same (bstar, before).  bstar = SEL_BINS when the whole list is taken.  (BINS: the histogram's
// size; bins past it count as empty.  COPIES of it, one after the other, are added up.)
template <int BINS = SEL_BINS, int COPIES = 1>
__device__ void find_boundary(const int32_t *__restrict__ gh, int32_t m_rem, int32_t *scan /* [SEL_THREADS] */,
                              int32_t *res /* [2] */, int &bstar, int &before, int32_t m_cap = 0x7FFFFFFF)
{
    constexpr int PER = BINS > SEL_THREADS ? BINS / SEL_THREADS : 1;
    int32_t loc[PER];
    int32_t sum = 0;
    // (no condition where every thread has bins: with one per bin the loads, two of 16 bytes, became eight of 4 bytes, each
    // behind a branch, and the boundary pass of 2048 lists of 65536 keys took 427 us for 327)
    const bool has_bins = BINS >= SEL_THREADS || (int)threadIdx.x < BINS;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        loc[j] = 0;
        if (has_bins)
#pragma unroll
            for (int c = 0; c < COPIES; ++c) loc[j] += gh[c * BINS + threadIdx.x * PER + j];
        sum += loc[j];
    }
    // prefix sums: within the wave by shuffles, the waves' totals through LDS (two barriers in all; a scan of all threads in
    // LDS takes eighteen)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t v = __shfl_up(incl, d);
        if (lane >= d) incl += v;
    }
    if (lane == 63) scan[wave] = incl;
    if (threadIdx.x == 0) {
        res[0] = SEL_BINS;
        res[1] = 0;
    }
    __syncthreads();
    int32_t total = 0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
        const int32_t v = scan[w];
        if (w < wave) incl += v;
        total += v;
    }
    const int32_t excl = incl - sum;
    if (m_cap != 0x7FFFFFFF) m_rem = m_cap < total ? m_cap : total;  // min(m, #keys)
    if (m_rem > 0 && excl < m_rem && m_rem <= incl) {
        int32_t run = excl;
        for (int j = 0; j < PER; ++j) {
            if (run + loc[j] >= m_rem) {
                res[0] = threadIdx.x * PER + j;
                res[1] = run;
                scan[SEL_THREADS - 2] = loc[j];
                break;
            }
            run += loc[j];
        }
    }
    if (m_rem <= 0 && threadIdx.x == 0) {
        res[0] = -1;  // take nothing, keep nothing
        res[1] = 0;
    }
    if (threadIdx.x == SEL_THREADS - 1) scan[SEL_THREADS - 1] = total;  // for the callers, and before it the keys of the boundary bin
    __syncthreads();
    bstar = res[0];
    before = res[1];
    if (bstar == SEL_BINS) before = total;
}

// Keys that other workgroups of the same launch write or read (AGENT) go past the second-level caches, which are not coherent between
// the XCDs.
template <bool AGENT>
__device__ __forceinline__ uint64_t sel_key(const uint64_t *p)
{
    return AGENT ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
template <bool AGENT>
__device__ __forceinline__ void sel_put(uint64_t *p, uint64_t key)
{
    if (AGENT) __hip_atomic_store(p, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = key;
}

#define SEL2_GROUPS 8                              // keys a thread takes per step
#define SEL2_STEP (SEL_THREADS * SEL2_GROUPS)     // keys a workgroup takes per step
template <int THREADS>
struct Sel2Place {                                // LDS of sel2_place
    int32_t cnt[2][2][THREADS / 64];              // [parity of the step][selected / boundary][wave]
    int32_t base[2];
    unsigned long long bits[2][THREADS / 64];
};
// Writes a step's keys of class 0 (selected) to out and of class 1 (boundary) to bl; o, no collect the boundary keys' bits and
// their complements.  The workgroup reserves its positions with one update of each counter per step: the counters of a query
// are two words that every workgroup of the launch updates and waits for, one after the other.  One query of 8.8 M passages:
// with an update per wave the bin filter took 27.6 us and the digit filter, 64 keys a wave, 19.9; now 8.1 and 5.8.  All
// threads call this.
template <int THREADS, int GROUPS, bool AGENT>
__device__ __forceinline__ void sel2_place(const uint64_t (&key)[GROUPS], const int (&cls)[GROUPS], int parity, Sel2Place<THREADS> &l,
                                           int32_t *n_sure, int32_t *n_boundary, uint64_t *__restrict__ out,
                                           uint64_t *__restrict__ bl, unsigned long long &o, unsigned long long &no)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long b0[GROUPS], b1[GROUPS];
    int n0 = 0, n1 = 0;
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) {
        b0[u] = __ballot(cls[u] == 0);
        b1[u] = __ballot(cls[u] == 1);
        n0 += __popcll(b0[u]);
        n1 += __popcll(b1[u]);
    }
    if (lane == 0) {
        l.cnt[parity][0][wave] = n0;
        l.cnt[parity][1][wave] = n1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int n = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) n += l.cnt[parity][threadIdx.x][w];
        l.base[threadIdx.x] = n ? atomicAdd(threadIdx.x == 0 ? n_sure : n_boundary, n) : 0;
    }
    __syncthreads();
    int base0 = l.base[0], base1 = l.base[1];
    for (int w = 0; w < wave; ++w) {
        base0 += l.cnt[parity][0][w];
        base1 += l.cnt[parity][1][w];
    }
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int u = 0; u < GROUPS; ++u) {
        if (cls[u] == 0) out[base0 + __popcll(b0[u] & below)] = key[u];
        if (cls[u] == 1) {
            sel_put<AGENT>(&bl[base1 + __popcll(b1[u] & below)], key[u]);
            o |= key[u];
            no |= ~key[u];
        }
        base0 += __popcll(b0[u]);
        base1 += __popcll(b1[u]);
    }
}

// ------------------------------------------------------------------ level kernel: split a list by its digit
// Positions are reserved by the workgroup, once per counter and 2048 keys (sixteen lists of 400 000 keys, the best 16 384 of each: 199 us
// with an update per wave and 64 keys, 24 now; the second level 39 -> 11).
template <int LEVEL>
__global__ __launch_bounds__(SEL_THREADS) void sel_level_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                SelState *state, int32_t *__restrict__ hist,
                                                                uint64_t *__restrict__ sure, int64_t sure_stride,
                                                                uint64_t *__restrict__ list_out, int64_t list_stride)
{
    __shared__ int32_t scan[SEL_THREADS];
    __shared__ int32_t res[2];
    __shared__ int32_t lh[LEVEL == 0 ? SEL_BINS : 1];
    __shared__ Sel2Place<SEL_THREADS> place;
    const int seg = blockIdx.y;
    SelState *s = state_of(state, seg);
    const int n = LEVEL == 0 ? s->n_in : s->n_list[0];
    const int32_t m_rem = s->m_rem[LEVEL];
    const int shift = s->shift[LEVEL], width = s->width[LEVEL];
    const int shift_n = s->shift[1], width_n = s->width[1];
    int bstar, before;
    find_boundary(hist + ((int64_t)seg * 2 + LEVEL) * SEL_BINS, m_rem, scan, res, bstar, before);
    if (blockIdx.x == 0 && threadIdx.x == 0) s->m_rem[LEVEL + 1] = m_rem - before;
    if (LEVEL == 0) {
        for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) lh[b] = 0;
        __syncthreads();
    }
    const uint64_t *k = keys + (int64_t)seg * key_stride;
    uint64_t *my_sure = sure + (int64_t)seg * sure_stride;
    uint64_t *my_out = list_out + (int64_t)seg * list_stride;
    unsigned long long any = 0, none = 0;  // (not used here)
    int parity = 0;
    for (int64_t s0 = (int64_t)blockIdx.x * SEL2_STEP; s0 < n; s0 += (int64_t)gridDim.x * SEL2_STEP, parity ^= 1) {  // uniform
        uint64_t key[SEL2_GROUPS];
        int cls[SEL2_GROUPS];  // 0 = surely selected, 1 = boundary, 2 = dropped
#pragma unroll
        for (int u = 0; u < SEL2_GROUPS; ++u) {
            const int64_t i = s0 + u * SEL_THREADS + threadIdx.x;
            key[u] = i < n ? k[i] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < SEL2_GROUPS; ++u) {
            const int d = digit_of(key[u], shift, width);
            cls[u] = s0 + u * SEL_THREADS + threadIdx.x < n ? (d < bstar ? 0 : (d == bstar ? 1 : 2)) : 2;
            if (LEVEL == 0 && cls[u] == 1) atomicAdd(&lh[digit_of(key[u], shift_n, width_n)], 1);
        }
        sel2_place<SEL_THREADS, SEL2_GROUPS, false>(key, cls, parity, place, &s->n_sure, &s->n_list[LEVEL], my_sure, my_out, any, none);
    }
    if (LEVEL == 0) {
        __syncthreads();
        int32_t *gh = hist + ((int64_t)seg * 2 + 1) * SEL_BINS;
        for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS)
            if (lh[b]) atomicAdd(&gh[b], lh[b]);
    }
}

// ------------------------------------------------------------------ finishing workgroup
__device__ void lds_bitonic_sort(uint64_t *s, int n2)
{
    for (int k = 2; k <= n2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n2; i += FIN_THREADS) {
                const int p = i ^ j;
                if (p > i) {
                    const uint64_t a = s[i], b = s[p];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) {
                        s[i] = b;
                        s[p] = a;
                    }
                }
            }
            __syncthreads();
        }
}
__device__ __forceinline__ int next_pow2(int n)
{
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// DIRECT: the list is the input itself (no levels ran).  Otherwise: sure keys + boundary list1.
template <bool DIRECT>
__global__ __launch_bounds__(FIN_THREADS) void sel_finish_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                 const int32_t *__restrict__ counts, int32_t m,
                                                                 SelState *state, const uint64_t *__restrict__ sure,
                                                                 int64_t sure_stride, const uint64_t *__restrict__ list1,
                                                                 int64_t list_stride, uint64_t *__restrict__ out,
                                                                 int64_t out_stride, int32_t *__restrict__ out_counts,
                                                                 int sorted)
{
    __shared__ uint64_t sk[SEL_SORT_CAP];
    __shared__ int32_t h256[256];
    __shared__ int32_t sh[4];
    const int seg = blockIdx.x;
    const uint64_t *bl;
    const uint64_t *sr = nullptr;
    int nb, n_sure, m_rem, top_bit;
    if (DIRECT) {
        bl = keys + (int64_t)seg * key_stride;
        nb = counts[seg];
        n_sure = 0;
        m_rem = m < nb ? m : nb;
        top_bit = 64;
    } else {
        SelState *s = state_of(state, seg);
        bl = list1 + (int64_t)seg * list_stride;
        sr = sure + (int64_t)seg * sure_stride;
        nb = s->n_list[1];
        n_sure = s->n_sure;
        m_rem = s->m_rem[2];
        top_bit = s->shift[1];  // boundary keys agree on every bit at or above this position
    }
    uint64_t *o = out + (int64_t)seg * out_stride;
    const int total_out = n_sure + m_rem;
    if (threadIdx.x == 0) out_counts[seg] = total_out;

    if (n_sure + nb <= SEL_SORT_CAP) {
        // common case: sort the union; the first total_out keys are the answer, in rank order
        const int tot = n_sure + nb, n2 = next_pow2(tot > 1 ? tot : 1);
        for (int i = threadIdx.x; i < n2; i += FIN_THREADS)
            sk[i] = i < n_sure ? sr[i] : (i < tot ? bl[i - n_sure] : PLAID_KEY_MAX);
        __syncthreads();
        lds_bitonic_sort(sk, n2);
        for (int i = threadIdx.x; i < total_out; i += FIN_THREADS) o[i] = sk[i];
        return;
    }

    // long boundary: find the m_rem-th smallest boundary key by 8-bit radix passes over global memory
    uint64_t prefix = 0, pmask = 0;  // bits decided so far
    int r = m_rem;
    int pos = top_bit;
    while (pos > 0 && r > 0) {
        const int w = pos < 8 ? pos : 8;
        pos -= w;
        for (int b = threadIdx.x; b < 256; b += FIN_THREADS) h256[b] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < nb; i += FIN_THREADS) {
            const uint64_t key = bl[i];
            if ((key & pmask) == prefix) atomicAdd(&h256[(int)((key >> pos) & ((1u << w) - 1u))], 1);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int run = 0, b = 0;
            for (; b < (1 << w); ++b) {
                if (run + h256[b] >= r) break;
                run += h256[b];
            }
            sh[0] = b;
            sh[1] = run;
        }
        __syncthreads();
        prefix |= (uint64_t)sh[0] << pos;
        pmask |= (uint64_t)((1u << w) - 1u) << pos;
        r -= sh[1];
        __syncthreads();
    }
    // keys are unique, so after all bits are decided `prefix` (restricted to pmask) is the threshold key itself
    if (threadIdx.x == 0) sh[2] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n_sure; i += FIN_THREADS) o[i] = sr[i];
    if (m_rem > 0)
        for (int i = threadIdx.x; i < nb; i += FIN_THREADS) {
            const uint64_t key = bl[i];
            if ((key & pmask) <= prefix) o[n_sure + atomicAdd(&sh[2], 1)] = key;
        }
    __syncthreads();
    if (sorted && total_out <= SEL_SORT_CAP) {
        __threadfence_block();
        const int n2 = next_pow2(total_out > 1 ? total_out : 1);
        for (int i = threadIdx.x; i < n2; i += FIN_THREADS) sk[i] = i < total_out ? o[i] : PLAID_KEY_MAX;
        __syncthreads();
        lds_bitonic_sort(sk, n2);
        for (int i = threadIdx.x; i < total_out; i += FIN_THREADS) o[i] = sk[i];
    }
}

// ------------------------------------------------------------------ global bitonic sort (only for m > SEL_SORT_CAP, sorted)
__global__ void sel_pad_copy_kernel(const uint64_t *__restrict__ src, int64_t src_stride, const int32_t *__restrict__ counts,
                                    uint64_t *__restrict__ dst, int64_t n2)
{
    const int seg = blockIdx.y;
    const int n = counts[seg];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += (int64_t)gridDim.x * blockDim.x)
        dst[(int64_t)seg * n2 + i] = i < n ? src[(int64_t)seg * src_stride + i] : PLAID_KEY_MAX;
}
__global__ void sel_bitonic_step_kernel(uint64_t *__restrict__ a, int64_t n2, int64_t k, int64_t j)
{
    uint64_t *s = a + (int64_t)blockIdx.y * n2;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = i ^ j;
        if (p > i) {
            const uint64_t x = s[i], y = s[p];
            const bool up = (i & k) == 0;
            if ((x > y) == up) {
                s[i] = y;
                s[p] = x;
            }
        }
    }
}
__global__ void sel_copy_back_kernel(const uint64_t *__restrict__ src, int64_t n2, const int32_t *__restrict__ counts,
                                     uint64_t *__restrict__ dst, int64_t dst_stride)
{
    const int seg = blockIdx.y;
    const int n = counts[seg];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[(int64_t)seg * dst_stride + i] = src[(int64_t)seg * n2 + i];
}

// ------------------------------------------------------------------ short lists: one workgroup sorts the list in LDS
// Lists of up to SEL_SORT_CAP keys: a workgroup loads the list into LDS padded with PLAID_KEY_MAX to the next power of
// two of its actual length, runs a bitonic network over it (one compare-exchange per thread and pass: thread t owns
// the pair (lo, lo | j) with lo = t with a zero inserted at bit log2(j)), and the first min(m, n) keys are the result
// in rank order.  n log^2 n compare-exchanges instead of the n^2 comparisons of rank counting, and only as much LDS as
// the longest list of the launch needs (the launcher passes it as dynamic shared memory).
// The 64 pairs a wave owns in one pass lie inside one aligned block of 128 keys whenever j <= 64, and a wave owns the
// same blocks in every pass, so those passes (most of the network) need no workgroup barrier: a wave's LDS
// operations complete in program order.  Only the passes with j >= 128 exchange keys between waves.
template <int THREADS>
__device__ __forceinline__ int lds_sort_list(uint64_t *sk, const uint64_t *__restrict__ k, int n)
{
    int n2 = 2;
    while (n2 < n) n2 <<= 1;
    for (int i = threadIdx.x; i < n2; i += THREADS) sk[i] = i < n ? k[i] : PLAID_KEY_MAX;
    __syncthreads();
    const int half = n2 >> 1;
    for (int kk = 2; kk <= n2; kk <<= 1)
        for (int j = kk >> 1; j > 0; j >>= 1) {
            const bool wide = j >= 128;  // uniform over the workgroup
            if (wide)
                __syncthreads();
            else
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int t = threadIdx.x; t < half; t += THREADS) {
                const int lo = ((t & ~(j - 1)) << 1) | (t & (j - 1)), hi = lo | j;
                const uint64_t a = sk[lo], b = sk[hi];
                const bool up = (lo & kk) == 0;
                if ((a > b) == up) {
                    sk[lo] = b;
                    sk[hi] = a;
                }
            }
            if (wide) __syncthreads();
        }
    __syncthreads();
    return n2;
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void sel_sort_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                           const int32_t *__restrict__ counts, int32_t n_cap, int32_t m,
                                                           uint64_t *__restrict__ out, int64_t out_stride,
                                                           int32_t *__restrict__ out_counts)
{
    extern __shared__ uint64_t sel_sort_lds[];
    const int seg = blockIdx.x;
    int n = counts[seg];
    if (n > n_cap) n = n_cap;
    const int n_out = m < n ? m : n;
    if (threadIdx.x == 0) out_counts[seg] = n_out;
    if (n_out == 0) return;
    lds_sort_list<THREADS>(sel_sort_lds, keys + (int64_t)seg * key_stride, n);
    uint64_t *o = out + (int64_t)seg * out_stride;
    for (int i = threadIdx.x; i < n_out; i += THREADS) o[i] = sel_sort_lds[i];
}

// The same for the final ranking: ids and scores go straight to the caller's buffers, best first, and the
// slots beyond min(k, count) are filled with (-1, -infinity).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void sel_sort_output_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                  const int32_t *__restrict__ counts, int32_t n_cap,
                                                                  int32_t k, int32_t *__restrict__ out_ids,
                                                                  float *__restrict__ out_scores)
{
    extern __shared__ uint64_t sel_sort_lds[];
    const int seg = blockIdx.x;
    int n = counts[seg];
    if (n > n_cap) n = n_cap;
    const int n_out = k < n ? k : n;
    int32_t *oi = out_ids + (int64_t)seg * k;
    float *os = out_scores + (int64_t)seg * k;
    for (int j = n_out + threadIdx.x; j < k; j += THREADS) {
        oi[j] = -1;
        os[j] = -INFINITY;
    }
    if (n_out == 0) return;
    lds_sort_list<THREADS>(sel_sort_lds, keys + (int64_t)seg * key_stride, n);
    for (int i = threadIdx.x; i < n_out; i += THREADS) {
        const uint64_t key = sel_sort_lds[i];
        oi[i] = (int32_t)(key & 0xFFFFFFFFu);
        os[i] = plaid_ord_to_score((uint32_t)(key >> 32));
    }
}

// ------------------------------------------------------------------ short lists, few of them: selection by rank counting
// With only a few lists in the launch (single-query latency) one workgroup per list leaves the chip idle and the
// network's passes are a chain of LDS round trips.  Then the n^2 form is quicker: the rank of a key is the number of
// smaller keys (keys are unique), so key j goes to out[rank] when rank < m.  Every workgroup holds the whole list in
// LDS and ranks 32 of its keys, eight lanes sharing the comparisons of one key.
#define RANK_MAX_LISTS 16
#define RANK_KEYS_PER_BLOCK 32
__global__ __launch_bounds__(256) void sel_rank_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                       const int32_t *__restrict__ counts, int32_t n_cap, int32_t m,
                                                       uint64_t *__restrict__ out, int64_t out_stride,
                                                       int32_t *__restrict__ out_counts)
{
    extern __shared__ uint64_t sk[];
    const int seg = blockIdx.y;
    int n = counts[seg];
    if (n > n_cap) n = n_cap;
    if (blockIdx.x == 0 && threadIdx.x == 0) out_counts[seg] = m < n ? m : n;
    const int j0 = blockIdx.x * RANK_KEYS_PER_BLOCK;
    if (j0 >= n) return;
    const uint64_t *k = keys + (int64_t)seg * key_stride;
    for (int i = threadIdx.x; i < n; i += 256) sk[i] = k[i];
    __syncthreads();
    const int j = j0 + (threadIdx.x >> 3), part = threadIdx.x & 7;
    const uint64_t key = j < n ? sk[j] : PLAID_KEY_MAX;
    int rank = 0;
    for (int i = part; i < n; i += 8) rank += sk[i] < key ? 1 : 0;
    rank += __shfl_xor(rank, 1);
    rank += __shfl_xor(rank, 2);
    rank += __shfl_xor(rank, 4);
    if (part == 0 && j < n && rank < m) out[(int64_t)seg * out_stride + rank] = key;
}

// Rank counting for the final ranking.
__global__ __launch_bounds__(256) void sel_rank_output_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                              const int32_t *__restrict__ counts, int32_t n_cap, int32_t k,
                                                              int32_t *__restrict__ out_ids, float *__restrict__ out_scores)
{
    extern __shared__ uint64_t sk[];
    const int seg = blockIdx.y;
    int n = counts[seg];
    if (n > n_cap) n = n_cap;
    int32_t *oi = out_ids + (int64_t)seg * k;
    float *os = out_scores + (int64_t)seg * k;
    if (blockIdx.x == 0)
        for (int j = (n < k ? n : k) + threadIdx.x; j < k; j += 256) {
            oi[j] = -1;
            os[j] = -INFINITY;
        }
    const int j0 = blockIdx.x * RANK_KEYS_PER_BLOCK;
    if (j0 >= n) return;
    const uint64_t *kk = keys + (int64_t)seg * key_stride;
    for (int i = threadIdx.x; i < n; i += 256) sk[i] = kk[i];
    __syncthreads();
    const int j = j0 + (threadIdx.x >> 3), part = threadIdx.x & 7;
    const uint64_t key = j < n ? sk[j] : PLAID_KEY_MAX;
    int rank = 0;
    for (int i = part; i < n; i += 8) rank += sk[i] < key ? 1 : 0;
    rank += __shfl_xor(rank, 1);
    rank += __shfl_xor(rank, 2);
    rank += __shfl_xor(rank, 4);
    if (part == 0 && j < n && rank < k) {
        oi[rank] = (int32_t)(key & 0xFFFFFFFFu);
        os[rank] = plaid_ord_to_score((uint32_t)(key >> 32));
    }
}

// The `take` smallest (in any order) of the n <= SEL_SORT_CAP keys of `bl`, to o; every key agrees at and above bit `high`.
// One workgroup of FIN_THREADS threads, all of which call this; sk, dh, h256, sh, differ: LDS (keys, one digit's histogram, wave
// totals, four words, two words).
// A digit at a time in LDS, the eleven bits from the highest in which the keys differ: keys below the boundary digit are taken,
// its own are left -- a handful, unless the keys tie in their scores: then the next digit lies in the ids.  What is left is
// ranked by counting.  (Sorting a tie group instead, 45 to 78 dependent steps, was the longest query of most launches: 144
// queries of 8.8 M passages 117 -> 52 us, 512 of 400 000 39 -> 20, 23 of 123 457 13.5 -> 7.6.)
#define FIN_RANK (FIN_THREADS / 4)
// One digit: keys from bl (STAGED: from sk); n, take, base, high: those of the keys that are left, which go to sk.
template <bool STAGED, bool AGENT>
__device__ __forceinline__ void sel_pick_digit(const uint64_t *__restrict__ bl, int &n, int &take, uint64_t *__restrict__ o, int &base,
                                               int &high, uint64_t *sk, int32_t *dh, int32_t *h256, int32_t *sh,
                                               unsigned long long *differ)
{
    uint64_t key[SEL_SORT_CAP / FIN_THREADS];
    const int shift = high > SEL_RADIX_BITS ? high - SEL_RADIX_BITS : 0;
    for (int i = threadIdx.x; i < SEL_BINS; i += FIN_THREADS) dh[i] = 0;
    if (threadIdx.x < 2) {
        sh[threadIdx.x] = 0;
        differ[threadIdx.x] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < SEL_SORT_CAP / FIN_THREADS; ++u) {
        const int i = threadIdx.x + u * FIN_THREADS;
        key[u] = i < n ? (STAGED ? sk[i] : sel_key<AGENT>(bl + i)) : PLAID_KEY_MAX;
        if (i < n) atomicAdd(&dh[(int)(key[u] >> shift) & (SEL_BINS - 1)], 1);
    }
    __syncthreads();
    {
        // thread t: bins 2 t and 2 t + 1; sums over the waves before it from the waves' totals
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int c0 = dh[2 * threadIdx.x], c1 = dh[2 * threadIdx.x + 1];
        int incl = c0 + c1;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        if (lane == 63) h256[wave] = incl;
        __syncthreads();
        int ahead = lane < wave ? h256[lane] : 0;  // (sixteen waves)
#pragma unroll
        for (int d = 1; d < FIN_THREADS / 64; d <<= 1) ahead += __shfl_xor(ahead, d);
        const int before = __builtin_amdgcn_readfirstlane(ahead) + incl - c0 - c1;
        if (take > 0 && before < take && before + c0 + c1 >= take) {
            const bool second = before + c0 < take;
            sh[2] = 2 * threadIdx.x + (second ? 1 : 0);
            sh[3] = before + (second ? c0 : 0);
        }
        if (take <= 0 && threadIdx.x == 0) {
            sh[2] = -1;
            sh[3] = 0;
        }
        __syncthreads();
    }
    const int bd = sh[2], below = sh[3];
#pragma unroll
    for (int u = 0; u < SEL_SORT_CAP / FIN_THREADS; ++u) {
        const int i = threadIdx.x + u * FIN_THREADS;
        if (u * FIN_THREADS >= n) break;  // uniform
        const int d = i < n ? (int)(key[u] >> shift) & (SEL_BINS - 1) : SEL_BINS;
        if (d < bd) o[base + atomicAdd(&sh[0], 1)] = key[u];
        if (d == bd) sk[atomicAdd(&sh[1], 1)] = key[u];
    }
    __syncthreads();
    n = sh[1];
    base += below;
    take -= below;
    if (n > FIN_RANK) {  // in which bits the keys that are left differ
        unsigned long long any = 0, none = 0;
#pragma unroll 1
        for (int i = threadIdx.x; i < n; i += FIN_THREADS) {
            any |= sk[i];
            none |= ~sk[i];
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            any |= __shfl_xor(any, d);
            none |= __shfl_xor(none, d);
        }
        if ((threadIdx.x & 63) == 0) {
            atomicOr(&differ[0], any);
            atomicOr(&differ[1], none);
        }
        __syncthreads();
        const unsigned long long diff = differ[0] & differ[1];
        high = diff ? 64 - __builtin_clzll(diff) : 0;
        __syncthreads();  // sh and differ are cleared next
    }
}
template <bool AGENT>
__device__ __forceinline__ void sel_pick_lds(const uint64_t *__restrict__ bl, int n, int take, uint64_t *__restrict__ o, int high,
                                             uint64_t *sk, int32_t *dh, int32_t *h256, int32_t *sh, unsigned long long *differ)
{
    int base = 0;
    if (n > FIN_RANK) {
        sel_pick_digit<false, AGENT>(bl, n, take, o, base, high, sk, dh, h256, sh, differ);
        // (uniform; keys are unique: a digit that ends at bit 0 leaves one)
#pragma unroll 1
        while (n > FIN_RANK) sel_pick_digit<true, AGENT>(bl, n, take, o, base, high, sk, dh, h256, sh, differ);
    } else {
        if ((int)threadIdx.x < n) sk[threadIdx.x] = sel_key<AGENT>(bl + threadIdx.x);
        __syncthreads();
    }
    // few keys: four threads count how many of them precede theirs
    const int i = threadIdx.x >> 2;
    if (i < n) {
        const uint64_t key = sk[i];
        int rank = 0;
#pragma unroll 4
        for (int j = threadIdx.x & 3; j < n; j += 4) rank += sk[j] < key ? 1 : 0;
        rank += __shfl_xor(rank, 1);
        rank += __shfl_xor(rank, 2);
        if ((threadIdx.x & 3) == 0 && rank < take) o[base + rank] = key;
    }
}

// The m smallest keys of each list, in no particular order: a workgroup per list, one digit and a handful of keys to rank.
// Rank counting, its n^2 form for few lists, takes 10 us for 1024 keys and 34 for 4096, this 5 and 7; sorting in LDS, with many
// lists, 14.9 us for 23 of 1000 keys, 9.7 for 256 of 256, 20.7 for 512 of 1024, 37 for 144 of 4096, this 6, 6, 9 and 9.
__global__ __launch_bounds__(FIN_THREADS, 8) void sel_pick_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                               const int32_t *__restrict__ counts, int32_t n_cap, int32_t m,
                                                               uint64_t *__restrict__ out, int64_t out_stride,
                                                               int32_t *__restrict__ out_counts)
{
    __shared__ uint64_t sk[SEL_SORT_CAP];
    __shared__ int32_t dh[SEL_BINS];
    __shared__ int32_t h256[FIN_THREADS / 64];
    __shared__ int32_t sh[4];
    __shared__ unsigned long long differ[2];  // OR over the keys / over their complements
    __shared__ unsigned long long left[2];
    const int seg = blockIdx.x;
    int n = counts[seg];
    if (n > n_cap) n = n_cap;
    const int take = m < n ? m : n;
    if (threadIdx.x == 0) {
        out_counts[seg] = take;
        differ[0] = differ[1] = 0;
    }
    __syncthreads();
    const uint64_t *k = keys + (int64_t)seg * key_stride;
    unsigned long long o = 0, no = 0;
    for (int i = threadIdx.x; i < n; i += FIN_THREADS) {
        o |= k[i];
        no |= ~k[i];
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        o |= __shfl_xor(o, d);
        no |= __shfl_xor(no, d);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicOr(&differ[0], o);
        atomicOr(&differ[1], no);
    }
    __syncthreads();
    const unsigned long long diff = differ[0] & differ[1];
    sel_pick_lds<false>(k, n, take, out + (int64_t)seg * out_stride, diff ? 64 - __builtin_clzll(diff) : 0, sk, dh, h256, sh, left);
}

static inline int64_t sort_pow2(int64_t n)
{
    int64_t p = 2;
    while (p < n) p <<= 1;
    return p;
}

void plaid_launch_rank_output(hipStream_t st, const uint64_t *keys, int64_t key_stride, const int32_t *counts, int nseg,
                              int64_t n_upper, int32_t k, int32_t *out_ids, float *out_scores)
{
    const size_t lds = (size_t)sort_pow2(n_upper) * 8;  // one thread per pair of the padded list, 256 to 1024
    if (nseg <= RANK_MAX_LISTS) {
        const int gx = (int)((n_upper + RANK_KEYS_PER_BLOCK - 1) / RANK_KEYS_PER_BLOCK);
        hipLaunchKernelGGL(sel_rank_output_kernel, dim3(gx > 0 ? gx : 1, nseg), dim3(256), lds, st, keys, key_stride, counts,
                           (int32_t)n_upper, k, out_ids, out_scores);
    } else if (n_upper <= 512)
        hipLaunchKernelGGL(sel_sort_output_kernel<256>, dim3(nseg), dim3(256), lds, st, keys, key_stride, counts,
                           (int32_t)n_upper, k, out_ids, out_scores);
    else if (n_upper <= 1024)
        hipLaunchKernelGGL(sel_sort_output_kernel<512>, dim3(nseg), dim3(512), lds, st, keys, key_stride, counts,
                           (int32_t)n_upper, k, out_ids, out_scores);
    else
        hipLaunchKernelGGL(sel_sort_output_kernel<1024>, dim3(nseg), dim3(1024), lds, st, keys, key_stride, counts,
                           (int32_t)n_upper, k, out_ids, out_scores);
}

// ------------------------------------------------------------------ host side
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static inline int64_t pow2_at_least(int64_t n)
{
    int64_t p = 1;
    while (p < n) p <<= 1;
    return p;
}

// Scratch of one selection instance comes in two parts: a small head (state + histograms) that must be
// zero before the producer of the keys runs, and a body (sure / boundary lists, sort buffer) that needs no
// initialisation.  The body is only needed for lists longer than SEL_SORT_CAP or more than SEL_SORT_CAP
// sorted results.
size_t plaid_select_zero_bytes(int nseg)
{
    return align256((size_t)nseg * sizeof(SelState)) + align256((size_t)nseg * 2 * SEL_BINS * sizeof(int32_t));
}
size_t plaid_select_body_bytes(int nseg, int64_t n_upper, int32_t m)
{
    size_t b = 0;
    const int64_t mm = m < n_upper ? m : n_upper;
    if (n_upper > SEL_SORT_CAP) b += align256((size_t)nseg * mm * 8) + 2 * align256((size_t)nseg * n_upper * 8);
    if (mm > SEL_SORT_CAP) b += align256((size_t)nseg * pow2_at_least(mm) * 8);
    return b;
}
size_t plaid_select_scratch_bytes(int nseg, int64_t n_upper, int32_t m)
{
    return plaid_select_zero_bytes(nseg) + plaid_select_body_bytes(nseg, n_upper, m);
}

SelScratch plaid_select_scratch_carve2(void *zero_base, void *body_base, int nseg, int64_t n_upper, int32_t m)
{
    SelScratch sc{};
    char *z = (char *)zero_base;
    sc.state = (SelState *)z;
    sc.hist = (int32_t *)(z + align256((size_t)nseg * sizeof(SelState)));
    char *p = (char *)body_base;
    const int64_t mm = m < n_upper ? m : n_upper;
    if (n_upper > SEL_SORT_CAP) {
        sc.sure = (uint64_t *)p;
        sc.sure_stride = mm;
        p += align256((size_t)nseg * mm * 8);
        sc.list0 = (uint64_t *)p;
        p += align256((size_t)nseg * n_upper * 8);
        sc.list1 = (uint64_t *)p;
        p += align256((size_t)nseg * n_upper * 8);
        sc.list_stride = n_upper;
    }
    sc.sortbuf = (mm > SEL_SORT_CAP) ? (uint64_t *)p : nullptr;
    return sc;
}
SelScratch plaid_select_scratch_carve(void *base, int nseg, int64_t n_upper, int32_t m)
{
    return plaid_select_scratch_carve2(base, (char *)base + plaid_select_zero_bytes(nseg), nseg, n_upper, m);
}

static int blocks_for(int64_t n, int nseg)
{
    int64_t b = (n + SEL_THREADS * 8 - 1) / (SEL_THREADS * 8);
    const int64_t cap = nseg >= 16 ? 64 : (nseg >= 4 ? 256 : 1024);
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

void plaid_launch_select(hipStream_t st, const uint64_t *keys, int64_t key_stride, const int32_t *counts, int nseg,
                         int64_t n_upper, int32_t m, uint64_t *out, int64_t out_stride, int32_t *out_counts, int sorted,
                         const SelScratch &sc, int state_ready)
{
    // the caller zeroes state + hist (plaid_launch_fill_u32 over the head of the scratch) before the
    // producer runs; see search.hip
    if (n_upper <= SEL_SORT_CAP) {
        const size_t lds = (size_t)sort_pow2(n_upper) * 8;
        if (!sorted && (nseg > RANK_MAX_LISTS || n_upper > 512)) {
            hipLaunchKernelGGL(sel_pick_kernel, dim3(nseg), dim3(FIN_THREADS), 0, st, keys, key_stride, counts, (int32_t)n_upper, m,
                               out, out_stride, out_counts);
        } else if (nseg <= RANK_MAX_LISTS) {
            const int gx = (int)((n_upper + RANK_KEYS_PER_BLOCK - 1) / RANK_KEYS_PER_BLOCK);
            hipLaunchKernelGGL(sel_rank_kernel, dim3(gx > 0 ? gx : 1, nseg), dim3(256), lds, st, keys, key_stride, counts,
                               (int32_t)n_upper, m, out, out_stride, out_counts);
        } else if (n_upper <= 512)
            hipLaunchKernelGGL(sel_sort_kernel<256>, dim3(nseg), dim3(256), lds, st, keys, key_stride, counts,
                               (int32_t)n_upper, m, out, out_stride, out_counts);
        else if (n_upper <= 1024)
            hipLaunchKernelGGL(sel_sort_kernel<512>, dim3(nseg), dim3(512), lds, st, keys, key_stride, counts,
                               (int32_t)n_upper, m, out, out_stride, out_counts);
        else
            hipLaunchKernelGGL(sel_sort_kernel<1024>, dim3(nseg), dim3(1024), lds, st, keys, key_stride, counts,
                               (int32_t)n_upper, m, out, out_stride, out_counts);
        return;
    } else {
        const int gx = blocks_for(n_upper, nseg);
        if (!state_ready)
            hipLaunchKernelGGL(sel_andor_kernel, dim3(gx, nseg), dim3(SEL_THREADS), 0, st, keys, key_stride, counts,
                               sc.state);
        hipLaunchKernelGGL(sel_hist0_kernel, dim3(gx, nseg), dim3(SEL_THREADS), 0, st, keys, key_stride, counts, m,
                           sc.state, sc.hist);
        hipLaunchKernelGGL(sel_level_kernel<0>, dim3(gx, nseg), dim3(SEL_THREADS), 0, st, keys, key_stride, sc.state,
                           sc.hist, sc.sure, sc.sure_stride, sc.list0, sc.list_stride);
        // (the second list is short more often than not: 2048 workgroups for all lists together, if they have no more than the first; 1024
        // lists of 16 384 keys 26 us with eight each)
        const int most1 = (2048 + nseg - 1) / nseg, gx1 = gx < most1 ? (gx > 16 ? 16 : gx) : (most1 > 16 ? 16 : most1);
        hipLaunchKernelGGL(sel_level_kernel<1>, dim3(gx1, nseg), dim3(SEL_THREADS), 0, st, sc.list0, sc.list_stride,
                           sc.state, sc.hist, sc.sure, sc.sure_stride, sc.list1, sc.list_stride);
        hipLaunchKernelGGL(sel_finish_kernel<false>, dim3(nseg), dim3(FIN_THREADS), 0, st, keys, key_stride, counts, m,
                           sc.state, sc.sure, sc.sure_stride, sc.list1, sc.list_stride, out, out_stride, out_counts,
                           sorted);
    }
    const int64_t mm = m < n_upper ? m : n_upper;
    if (sorted && mm > SEL_SORT_CAP) {
        // rare: more than SEL_SORT_CAP results in rank order -> bitonic network in global memory
        uint64_t *buf = sc.sortbuf;
        const int64_t n2 = pow2_at_least(mm);
        const int gx = (int)((n2 + 255) / 256 > 1024 ? 1024 : (n2 + 255) / 256);
        hipLaunchKernelGGL(sel_pad_copy_kernel, dim3(gx, nseg), dim3(256), 0, st, out, out_stride, out_counts, buf, n2);
        for (int64_t k = 2; k <= n2; k <<= 1)
            for (int64_t j = k >> 1; j > 0; j >>= 1)
                hipLaunchKernelGGL(sel_bitonic_step_kernel, dim3(gx, nseg), dim3(256), 0, st, buf, n2, k, j);
        hipLaunchKernelGGL(sel_copy_back_kernel, dim3(gx, nseg), dim3(256), 0, st, buf, n2, out_counts, out, out_stride);
    }
}

// =================================================================================================
// Stage-2 selection: the ndocs best candidates out of up to P keys plus the empty-bag candidates.
//
// The producer has already counted the keys into SEL_BINS score bins (bin 0 = best), so the cut is
// found without another pass: keys in bins before the boundary bin are selected for sure, the
// boundary bin (normally a few hundred keys) is cut by the finishing workgroup, digit by digit.  Exact score
// ties are common (passages with the same surviving centroids score identically), so a boundary
// bin can be long: then one digit pass over its keys -- starting at the highest bit in which they
// differ, which skips the tied score bits and lands in the passage id -- cuts it down first.
// Candidates with an empty bag (-infinity) are appended last, in passage-id order, straight from
// their bitmap.
// =================================================================================================
// The workgroup's boundary bits to the query's.  All threads call this, once.
template <int THREADS>
__device__ __forceinline__ void sel2_place_bits(unsigned long long o, unsigned long long no, Sel2Place<THREADS> &l, unsigned long long *b_or,
                                                unsigned long long *b_nor)
{
    for (int d = 1; d < 64; d <<= 1) {
        o |= __shfl_xor(o, d);
        no |= __shfl_xor(no, d);
    }
    if ((threadIdx.x & 63) == 0) {
        l.bits[0][threadIdx.x >> 6] = o;
        l.bits[1][threadIdx.x >> 6] = no;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long v = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) v |= l.bits[threadIdx.x][w];
        if (v) atomicOr(threadIdx.x == 0 ? b_or : b_nor, v);
    }
}

// A boundary list longer than this goes through a digit pass (all workgroups of the query) before the finishing workgroup
// takes its digits in LDS.  Where the line lies matters little: the stage with 2048 / 4096 / 8192 (all that LDS holds), us, 32
// queries of 400 000 passages 28 / 23 / 23, 512 of them 94 / 90 / 83, of 8.8 M 8 queries 46 / 44 / 47, 150 189 / 186 / 178; the whole searches
// do not differ.  Two such passes can be chained (LEVEL 1 reads the bin filter's list, LEVEL 2 the list
// LEVEL 1 leaves): when a few distinct scores are shared by very many passages, the first digit falls into the score
// bits and leaves one whole tie group, the second falls into the passage-id bits and leaves 2^-11 of it.
#define SEL2_DIGIT_MIN 4096
#define SEL2_SECOND_MIN_PASSAGES (1 << 19)  // indexes with more passages than this get the second digit pass
#define SEL2_SUB 1024                       // digits of either kind that sel2_bins_kernel counts
static_assert(2 * SEL2_SUB <= SEL_BINS, "both kinds of digits in one histogram");
static constexpr int sel2_id_shift(int64_t P)  // passage id -> digit
{
    int bits = 10;
    while ((int64_t)1 << bits < P) ++bits;
    return bits - 10;
}
// The digit of a score within its bin: not falling in the rank, like the bin.
__device__ __forceinline__ int sel2_sub_bin(uint64_t key, const S2Meta &mt, int bin, int bin_shift)
{
    float x = (mt.bin_hi - plaid_ord_to_score((uint32_t)(key >> 32))) * mt.bin_scale;  // (as in plaid_s2_bin)
    x = fminf(fmaxf(x, 0.f), (float)(SEL_BINS - 1));
    x = (x - (float)(bin << bin_shift)) * (float)(SEL2_SUB >> bin_shift);
    return (int)fminf(fmaxf(x, 0.f), (float)(SEL2_SUB - 1));
}
static_assert(SEL2_SUB >> S2_COARSE_SHIFT > 0, "a coarse bin has digits");
// Scores that lie nearer to one another than that tells apart: of a list whose scores are fewer than SEL2_SUB representable
// numbers apart the digit is the number itself, counted by its ten lowest bits (in the half of the fine histogram's place that the
// coarse ones leave free).  Bins that come with the fine histogram have digits near a rounding step as it is.  Two scores 16 numbers
// apart, which share the passages of an index between them, us per search with / without: one query of 100 000 passages 223 / 409, of 400 000
// 403 / 1091, of 8.8 M 404 / 6350, sixteen of 8.8 M 2915 / 12 310 (one score for all: 353 / 360 and 2344 / 2298).
static_assert(S2_COPIES * S2_COARSE + SEL2_SUB <= SEL_BINS, "both in the fine histogram's place");

// Counts the lanes' digits (-1: none).  All lanes call this, one at least has a digit.
__device__ __forceinline__ void sel2_count(int32_t *lh, int digit)
{
    const unsigned long long have = __ballot(digit >= 0);
    const int lane = (int)(threadIdx.x & 63), lead = (int)__builtin_ctzll(have);
    const unsigned long long same = __ballot(digit == __builtin_amdgcn_readlane(digit, lead));
    if (lane == lead) atomicAdd(&lh[digit], __popcll(same));
    else if (digit >= 0 && !((same >> lane) & 1ull)) atomicAdd(&lh[digit], 1);
}
// The same for the scores' digits of either kind: lh[sub], lh[SEL_BINS + low bits of ord], for the lanes with `in`; the lanes of two
// of the scores add as one each.
__device__ __forceinline__ void sel2_count_score(int32_t *lh, bool in, int sub, uint32_t ord)
{
    const int lane = (int)(threadIdx.x & 63);
    unsigned long long left = __ballot(in);
    int n = in ? 1 : 0;
#pragma unroll
    for (int r = 0; r < 2; ++r)
        if (left) {  // uniform
            const int lead = (int)__builtin_ctzll(left);
            const bool equal = ord == (uint32_t)__builtin_amdgcn_readlane((int)ord, lead);
            const unsigned long long same = left & __ballot(equal);
            if (in && equal) n = lane == lead ? __popcll(same) : 0;
            left &= ~same;
        }
    if (n) {
        atomicAdd(&lh[sub], n);
        atomicAdd(&lh[SEL_BINS + (ord & (SEL2_SUB - 1))], n);
    }
}
// DIGITS: where there are more than SEL_SORT_CAP boundary keys, the extremes of their scores take the place of their bits, and their
// digits are counted in hist1 ([nq][SEL_BINS]: the scores', then the passage ids') and, of a list, the scores' lowest bits in low
// ([nq][SEL_BINS]: the last SEL2_SUB).
template <bool DIGITS>
__device__ __forceinline__ void sel2_filter_body(const uint64_t *__restrict__ keys, int64_t key_stride, const uint32_t *__restrict__ candbits,
                                                 int64_t cand_words, int64_t P, int32_t m, const S2Meta *__restrict__ meta,
                                                 const int32_t *__restrict__ hist, Sel2State *state, uint64_t *__restrict__ out,
                                                 int64_t out_stride, uint64_t *__restrict__ blist, int64_t blist_stride, int lists,
                                                 const int32_t *__restrict__ list_counts, int id_shift, int32_t *__restrict__ hist1,
                                                 int32_t *__restrict__ low,
                                                 int32_t *lh /* [SEL_BINS + SEL2_SUB] */)
{
    __shared__ int32_t scan[SEL_THREADS];
    __shared__ int32_t res[2];
    __shared__ Sel2Place<SEL_THREADS> place;
    const int seg = blockIdx.y;
    Sel2State *s = state + seg;
    const S2Meta mt = meta[seg];
    if (mt.K == 0) return;  // no surviving centroid: no valid key, the state stays zero and the fill takes over
    const bool is_list = lists && mt.K <= S2_MAX_KEPT;
    // a list: its keys; in parts (a single query): where they end, one after the other, and the way from there to their places
    int64_t n_items = P;
    int32_t part_end[DIGITS ? S2_COPIES : 1], part_at[DIGITS ? S2_COPIES : 1];
    bool parts = false;
    if (is_list) {  // uniform
        const int32_t *counts = list_counts + (int64_t)seg * S2_COUNTS_QUERY;
        int32_t n = counts[0];
        if constexpr (DIGITS) {
            parts = lists == 2;
            if (parts) {  // uniform
                n = 0;
#pragma unroll
                for (int x = 0; x < S2_COPIES; ++x) {
                    part_at[x] = counts[x * S2_COUNT_STRIDE + 1] - n;
                    n += counts[x * S2_COUNT_STRIDE];
                    part_end[x] = n;
                }
            }
        }
        n_items = n;
    }
    // a list is short next to the passages the grid is sized for: most of its workgroups have nothing to read
    if (blockIdx.x > 0 && (int64_t)blockIdx.x * SEL2_STEP >= n_items) return;
    int bstar, before;
    // takes min(m, number of keys); a list comes with the coarse histogram
    if (is_list) find_boundary<S2_COARSE, S2_COPIES>(hist + (int64_t)seg * SEL_BINS, 0, scan, res, bstar, before, m);
    else find_boundary(hist + (int64_t)seg * SEL_BINS, 0, scan, res, bstar, before, m);
    const int bin_shift = is_list ? S2_COARSE_SHIFT : 0;
    const int32_t n_keys = scan[SEL_THREADS - 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        s->m_rem = (m < n_keys ? m : n_keys) - before;
        s->bin = bstar;
    }
    if (n_keys == 0) return;
    const bool count = DIGITS && scan[SEL_THREADS - 2] > SEL_SORT_CAP;  // uniform
    if (count) {
        for (int b = threadIdx.x; b < SEL_BINS + SEL2_SUB; b += SEL_THREADS) lh[b] = 0;
        __syncthreads();
    }
    uint32_t ord_max = 0, ord_nmin = 0;  // of the boundary keys' scores; the latter's complement
    const uint32_t *k = reinterpret_cast<const uint32_t *>(keys + (int64_t)seg * key_stride);  // score word of passage i
    const uint32_t *cb = candbits + (int64_t)seg * cand_words;
    uint64_t *my_out = out + (int64_t)seg * out_stride;
    uint64_t *my_bl = blist + (int64_t)seg * blist_stride;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned long long o = 0, no = 0;
    int parity = 0;
    for (int64_t s0 = (int64_t)blockIdx.x * SEL2_STEP; s0 < n_items; s0 += (int64_t)gridDim.x * SEL2_STEP, parity ^= 1) {  // uniform
        const int64_t i0 = s0 + 64 * SEL2_GROUPS * wave;  // a wave takes consecutive slots
        uint64_t key[SEL2_GROUPS];
        int cls[SEL2_GROUPS];  // 0 = surely selected, 1 = boundary, 2 = dropped
        if (is_list) {  // uniform
            const uint64_t *kl = keys + (int64_t)seg * key_stride;
#pragma unroll
            for (int u = 0; u < SEL2_GROUPS; ++u) {
                const int64_t i = i0 + 64 * u + lane;
                int32_t at = 0;
                if constexpr (DIGITS)
                    if (parts) {  // uniform
                        at = part_at[0];
#pragma unroll
                        for (int x = 1; x < S2_COPIES; ++x) at = (int32_t)i >= part_end[x - 1] ? part_at[x] : at;
                    }
                key[u] = i < n_items ? kl[i + at] : PLAID_KEY_MAX;
            }
        } else {
            // word i is meaningful only when passage i is a candidate; it then holds its score word or "no score".  The
            // candidate bits and the score words are requested together (a word that means nothing is read and dropped):
            // one round trip to memory per step.
            uint32_t cw[SEL2_GROUPS], sw[SEL2_GROUPS];
#pragma unroll
            for (int u = 0; u < SEL2_GROUPS; ++u) {
                const int64_t i = i0 + 64 * u + lane;
                cw[u] = i < P ? cb[i >> 5] : 0u;
                sw[u] = i < P ? k[i] : PLAID_S2_NO_SCORE;
            }
#pragma unroll
            for (int u = 0; u < SEL2_GROUPS; ++u) {
                const int64_t i = i0 + 64 * u + lane;
                key[u] = PLAID_KEY_MAX;
                if (((cw[u] >> (i & 31)) & 1u) && sw[u] != PLAID_S2_NO_SCORE) key[u] = ((uint64_t)sw[u] << 32) | (uint32_t)i;
            }
        }
#pragma unroll
        for (int u = 0; u < SEL2_GROUPS; ++u) {
            cls[u] = 2;
            if (key[u] != PLAID_KEY_MAX) {
                const int d = plaid_s2_bin(plaid_ord_to_score((uint32_t)(key[u] >> 32)), mt.bin_hi, mt.bin_scale) >> bin_shift;
                cls[u] = d < bstar ? 0 : (d == bstar ? 1 : 2);
            }
        }
        sel2_place<SEL_THREADS, SEL2_GROUPS, false>(key, cls, parity, place, &s->n_sure, &s->n_b, my_out, my_bl, o, no);
        if (count) {
#pragma unroll
            for (int u = 0; u < SEL2_GROUPS; ++u)
                if (__any(cls[u] == 1)) {  // (the keys of a wave mostly share one digit or both: one update for those)
                    const uint32_t ord = (uint32_t)(key[u] >> 32);
                    sel2_count_score(lh, cls[u] == 1, sel2_sub_bin(key[u], mt, bstar, bin_shift), ord);
                    sel2_count(lh + SEL2_SUB, cls[u] == 1 ? (int)((uint32_t)key[u] >> id_shift) : -1);
                    if (cls[u] == 1) {
                        ord_max = max(ord_max, ord);
                        ord_nmin = max(ord_nmin, ~ord);
                    }
                }
        }
    }
    if (!count) {
        sel2_place_bits<SEL_THREADS>(o, no, place, &s->b_or, &s->b_nor);
    } else {
        for (int d = 1; d < 64; d <<= 1) {
            ord_max = max(ord_max, (uint32_t)__shfl_xor((int)ord_max, d));
            ord_nmin = max(ord_nmin, (uint32_t)__shfl_xor((int)ord_nmin, d));
        }
        if (lane == 0) {
            place.bits[0][wave] = ord_max;
            place.bits[1][wave] = ord_nmin;
        }
        __syncthreads();
        int32_t *gh = hist1 + (int64_t)seg * SEL_BINS;
        for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS)
            if (lh[b]) atomicAdd(&gh[b], lh[b]);
        if (is_list) {
            gh = low + (int64_t)(seg + 1) * SEL_BINS - SEL2_SUB;
            for (int b = threadIdx.x; b < SEL2_SUB; b += SEL_THREADS)
                if (lh[SEL_BINS + b]) atomicAdd(&gh[b], lh[SEL_BINS + b]);
        }
        // (one update per workgroup, and last: the workgroups that are still reserving positions wait for this line.  A query of 8.8 M
        // equal scores: 64 us, with the extremes in front of the digits 141, with the bits of the keys in their place 72)
        if (threadIdx.x < 2) {
            uint32_t v = 0;
#pragma unroll
            for (int w = 0; w < SEL_THREADS / 64; ++w) v = max(v, (uint32_t)place.bits[threadIdx.x][w]);
            if (v) atomicMax(threadIdx.x == 0 ? &s->ord_max : &s->ord_nmin, v);
        }
    }
}
__global__ __launch_bounds__(SEL_THREADS, 8) void sel2_filter_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                  const uint32_t *__restrict__ candbits, int64_t cand_words,
                                                                  int64_t P, int32_t m, const S2Meta *__restrict__ meta,
                                                                  const int32_t *__restrict__ hist, Sel2State *state,
                                                                  uint64_t *__restrict__ out, int64_t out_stride,
                                                                  uint64_t *__restrict__ blist, int64_t blist_stride, int lists,
                                                                  const int32_t *__restrict__ list_counts)
{
    sel2_filter_body<false>(keys, key_stride, candbits, cand_words, P, m, meta, hist, state, out, out_stride, blist, blist_stride, lists,
                            list_counts, 0, nullptr, nullptr, nullptr);
}
__global__ __launch_bounds__(SEL_THREADS, 6) void sel2_bins_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                                                const uint32_t *__restrict__ candbits, int64_t cand_words, int64_t P,
                                                                int32_t m, const S2Meta *__restrict__ meta,
                                                                int32_t *hist, Sel2State *state, uint64_t *__restrict__ out,
                                                                int64_t out_stride, uint64_t *__restrict__ blist, int64_t blist_stride,
                                                                int lists, const int32_t *__restrict__ list_counts, int id_shift,
                                                                int32_t *__restrict__ hist1)
{
    __shared__ int32_t lh[SEL_BINS + SEL2_SUB];
    sel2_filter_body<true>(keys, key_stride, candbits, cand_words, P, m, meta, hist, state, out, out_stride, blist, blist_stride, lists,
                           list_counts, id_shift, hist1, hist, lh);
}

template <int LEVEL>
__device__ __forceinline__ int sel2_level_input(const Sel2State *s, int &m_rem)
{
    m_rem = LEVEL == 1 ? s->m_rem : s->m_rem1;
    // (LEVEL 2 has work only when LEVEL 1 had: n_b1 is zero otherwise)
    return LEVEL == 1 ? s->n_b : s->n_b1;
}
template <int LEVEL>
__device__ __forceinline__ void sel2_digit_plan(const Sel2State *s, int &shift, int &width)
{
    const unsigned long long diff = LEVEL == 1 ? s->b_or & s->b_nor : s->b_or1 & s->b_nor1;
    const int hi = diff ? 63 - __clzll((long long)diff) : -1;
    width = hi + 1 < SEL_RADIX_BITS ? hi + 1 : SEL_RADIX_BITS;
    shift = hi + 1 - width;
}

// Digit histogram of a boundary list of more than `least` keys (no-op otherwise).
template <int LEVEL>
__global__ __launch_bounds__(SEL_THREADS) void sel2_digit_hist_kernel(const uint64_t *__restrict__ blist,
                                                                      int64_t blist_stride, Sel2State *state,
                                                                      int32_t *__restrict__ hist1, int least)
{
    __shared__ int32_t lh[SEL_BINS];
    const int seg = blockIdx.y;
    Sel2State *s = state + seg;
    int m_rem;
    const int n = sel2_level_input<LEVEL>(s, m_rem);
    if (n <= least || (int64_t)blockIdx.x * SEL_THREADS >= n) return;
    int shift, width;
    sel2_digit_plan<LEVEL>(s, shift, width);
    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS) lh[b] = 0;
    __syncthreads();
    const uint64_t *k = blist + (int64_t)seg * blist_stride;
    for (int64_t i = (int64_t)blockIdx.x * SEL_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * SEL_THREADS)
        atomicAdd(&lh[digit_of(k[i], shift, width)], 1);
    __syncthreads();
    int32_t *gh = hist1 + (int64_t)seg * SEL_BINS;
    for (int b = threadIdx.x; b < SEL_BINS; b += SEL_THREADS)
        if (lh[b]) atomicAdd(&gh[b], lh[b]);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (LEVEL == 1) s->shift1 = shift, s->width1 = width;
        else s->shift2 = shift, s->width2 = width;
    }
}

// Digit filter of an over-long boundary list (no-op otherwise): smaller digits are selected, the boundary digit
// goes to blist1 (LEVEL 1 also records in which bits the keys it leaves differ, for LEVEL 2's plan).
template <int LEVEL>
__global__ __launch_bounds__(SEL_THREADS) void sel2_digit_filter_kernel(const uint64_t *__restrict__ blist,
                                                                        int64_t blist_stride, Sel2State *state,
                                                                        const int32_t *__restrict__ hist1,
                                                                        uint64_t *__restrict__ out, int64_t out_stride,
                                                                        uint64_t *__restrict__ blist1,
                                                                        int64_t blist1_stride)
{
    __shared__ int32_t scan[SEL_THREADS];
    __shared__ int32_t res[2];
    __shared__ Sel2Place<SEL_THREADS> place;
    const int seg = blockIdx.y;
    Sel2State *s = state + seg;
    int32_t m_rem;
    const int n = sel2_level_input<LEVEL>(s, m_rem);
    if (n <= SEL2_DIGIT_MIN || (int64_t)blockIdx.x * SEL2_STEP >= n) return;
    int shift, width;
    sel2_digit_plan<LEVEL>(s, shift, width);
    int bstar, before;
    find_boundary(hist1 + (int64_t)seg * SEL_BINS, m_rem, scan, res, bstar, before);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (LEVEL == 1) s->m_rem1 = m_rem - before;
        else s->m_rem2 = m_rem - before;
    }
    int32_t *n_left = LEVEL == 1 ? &s->n_b1 : &s->n_b2;
    const uint64_t *k = blist + (int64_t)seg * blist_stride;
    uint64_t *my_out = out + (int64_t)seg * out_stride;
    uint64_t *my_bl = blist1 + (int64_t)seg * blist1_stride;
    unsigned long long o = 0, no = 0;
    int parity = 0;
    for (int64_t s0 = (int64_t)blockIdx.x * SEL2_STEP; s0 < n; s0 += (int64_t)gridDim.x * SEL2_STEP, parity ^= 1) {  // uniform
        uint64_t key[SEL2_GROUPS];
        int cls[SEL2_GROUPS];
#pragma unroll
        for (int u = 0; u < SEL2_GROUPS; ++u) {
            const int64_t i = s0 + u * SEL_THREADS + threadIdx.x;
            key[u] = i < n ? k[i] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < SEL2_GROUPS; ++u) {
            const int d = digit_of(key[u], shift, width);
            cls[u] = s0 + u * SEL_THREADS + threadIdx.x < n ? (d < bstar ? 0 : (d == bstar ? 1 : 2)) : 2;
        }
        sel2_place<SEL_THREADS, SEL2_GROUPS, false>(key, cls, parity, place, &s->n_sure, n_left, my_out, my_bl, o, no);
    }
    if (LEVEL == 1) sel2_place_bits<SEL_THREADS>(o, no, place, &s->b_or1, &s->b_nor1);
}

// The passages of the words [w0, w1) of a bitmap to o[total ..], until m are there; positions from a wave-level prefix sum of the
// popcounts plus the waves' totals (wsum).  PER words per thread and round.  PER = 1: in ascending order.  PER > 1: rounds that
// are taken as a whole, in any order; a round of more passages than are wanted is left to the caller (returns its w0).
// All threads call this.
template <int PER>
__device__ __forceinline__ int64_t sel2_fill(const uint32_t *__restrict__ eb, int64_t w0, int64_t w1, int64_t P, int32_t m,
                                             int32_t *wsum, uint64_t *__restrict__ o, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (; w0 < w1 && total < m; w0 += FIN_THREADS * PER) {
        const int64_t w = w0 + 64 * PER * wave + lane;  // words w, w + 64, ..
        uint32_t v[PER];
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) v[u] = w + 64 * u < w1 ? eb[w + 64 * u] : 0u;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if ((w + 64 * u + 1) * 32 > P) {
                const int64_t keep = P - (w + 64 * u) * 32;
                v[u] = keep <= 0 ? 0u : (keep >= 32 ? v[u] : (v[u] & ((1u << keep) - 1u)));
            }
            cnt += __popc(v[u]);
        }
        int incl = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        __syncthreads();  // the previous round's readers of wsum are done
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int pos = total + incl - cnt, all = 0;
        for (int wv = 0; wv < FIN_THREADS / 64; ++wv) {
            const int t = wsum[wv];
            if (wv < wave) pos += t;
            all += t;
        }
        if (PER > 1 && total + all > m) return w0;  // uniform: every thread adds the same wave totals
#pragma unroll
        for (int u = 0; u < PER; ++u)
            while (v[u] && pos < m) {
                const int bit = __ffs(v[u]) - 1;
                v[u] &= v[u] - 1;
                o[pos++] = plaid_make_key(-INFINITY, (uint32_t)((w + 64 * u) * 32 + bit));
            }
        total = total + all < m ? total + all : m;
    }
    return w0;
}

// The end of a query's selection, by one workgroup: the m_rem best of the nb boundary keys bl, which agree on every bit at or above
// top_bit, behind the n_sure selected ones, then empty-bag candidates in pid order.
struct Sel2Finish {
    uint64_t sk[SEL_SORT_CAP];
    int32_t dh[SEL_BINS];
    int32_t h256[256];
    int32_t sh[4];
    unsigned long long differ[2];
};
template <bool AGENT>
__device__ __forceinline__ void sel2_finish_body(Sel2Finish &l, const uint64_t *bl, int nb, int m_rem, int n_sure, int top_bit,
                                                 const uint32_t *__restrict__ eb, int64_t cand_words, int64_t P, int32_t m, uint64_t *o,
                                                 int32_t *__restrict__ out_count)
{
    int total = n_sure + m_rem;
    if (nb <= SEL_SORT_CAP) {
        sel_pick_lds<AGENT>(bl, nb, m_rem, o + n_sure, top_bit, l.sk, l.dh, l.h256, l.sh, l.differ);
    } else {
        // still long (huge tie groups): radix selection over global memory by this one workgroup.  The keys of such a
        // list mostly share their digit (that is what made the list long), so a wave whose keys all have one digit
        // counts them with a single LDS update instead of 64 updates of one address.
        uint64_t prefix = 0, pmask = 0;
        int r = m_rem;
        int pos = top_bit;
        const int lane = threadIdx.x & 63;
        const int nb_round = (nb + FIN_THREADS - 1) / FIN_THREADS * FIN_THREADS;  // whole waves in every step
        while (pos > 0 && r > 0) {
            const int w = pos < 8 ? pos : 8;
            pos -= w;
            for (int b = threadIdx.x; b < 256; b += FIN_THREADS) l.h256[b] = 0;
            __syncthreads();
            for (int i0 = threadIdx.x; i0 < nb_round; i0 += 4 * FIN_THREADS) {
                uint64_t key[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * FIN_THREADS;
                    key[u] = i < nb ? sel_key<AGENT>(bl + i) : ~prefix;  // a key past the end never matches the prefix
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u * FIN_THREADS;
                    const int dgt = (i < nb && (key[u] & pmask) == prefix) ? (int)((key[u] >> pos) & ((1u << w) - 1u)) : -1;
                    const int first = __builtin_amdgcn_readfirstlane(dgt);
                    const unsigned long long same = __ballot(dgt == first);
                    if (same == __ballot(true)) {  // uniform digit (or no key in play) in this wave
                        if (lane == (int)__builtin_ctzll(same) && first >= 0) atomicAdd(&l.h256[first], __popcll(same));
                    } else if (dgt >= 0) {
                        atomicAdd(&l.h256[dgt], 1);
                    }
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                int run = 0, b = 0;
                for (; b < (1 << w); ++b) {
                    if (run + l.h256[b] >= r) break;
                    run += l.h256[b];
                }
                l.sh[0] = b;
                l.sh[1] = run;
            }
            __syncthreads();
            prefix |= (uint64_t)l.sh[0] << pos;
            pmask |= (uint64_t)((1u << w) - 1u) << pos;
            r -= l.sh[1];
            __syncthreads();
        }
        if (threadIdx.x == 0) l.sh[2] = 0;
        __syncthreads();
        if (m_rem > 0)
            for (int i0 = threadIdx.x; i0 < nb_round; i0 += FIN_THREADS) {
                const uint64_t key = i0 < nb ? sel_key<AGENT>(bl + i0) : 0;
                const bool take = i0 < nb && (key & pmask) <= prefix;
                const unsigned long long tk = __ballot(take);
                if (tk) {  // one counter update per wave
                    int base = 0;
                    if (lane == (int)__builtin_ctzll(tk)) base = atomicAdd(&l.sh[2], __popcll(tk));
                    base = __shfl(base, (int)__builtin_ctzll(tk));
                    if (take) o[n_sure + base + __popcll(tk & ((1ull << lane) - 1ull))] = key;
                }
            }
    }
    __syncthreads();

    // empty-bag candidates: those of the smallest pids, until m slots are filled.  One bitmap word per thread in the first round,
    // which is enough where nearly every passage is one, then rounds of eight (8.8 M passages are 275 000 words, 268 rounds of
    // one) up to the one in which the last of them lies.
    if (total < m) {
        int64_t w0 = sel2_fill<1>(eb, 0, cand_words < FIN_THREADS ? cand_words : FIN_THREADS, P, m, l.h256, o, total);
        w0 = sel2_fill<8>(eb, w0, cand_words, P, m, l.h256, o, total);
        sel2_fill<1>(eb, w0, cand_words, P, m, l.h256, o, total);
    }
    if (threadIdx.x == 0) *out_count = total;
}
__device__ __forceinline__ int sel2_top_bit(unsigned long long any, unsigned long long none)
{
    return any & none ? 64 - __builtin_clzll(any & none) : 0;
}
// One workgroup per query: finish the boundary list, then append empty-bag candidates in pid order.
__global__ __launch_bounds__(FIN_THREADS, 8) void sel2_finish_kernel(const uint64_t *__restrict__ blist, int64_t blist_stride,
                                                                  const uint64_t *__restrict__ blist1,
                                                                  int64_t blist1_stride, const Sel2State *state,
                                                                  const uint32_t *__restrict__ emptybits,
                                                                  int64_t cand_words, int64_t P, int32_t m, int levels,
                                                                  uint64_t *__restrict__ out, int64_t out_stride,
                                                                  int32_t *__restrict__ out_counts)
{
    __shared__ Sel2Finish l;
    const int seg = blockIdx.x;
    const Sel2State *s = state + seg;
    // how many digit filters this query's boundary list went through (levels: how many were launched); the second one
    // writes where the first one read
    const int done = (levels >= 1 && s->n_b > SEL2_DIGIT_MIN) ? ((levels >= 2 && s->n_b1 > SEL2_DIGIT_MIN) ? 2 : 1) : 0;
    const uint64_t *bl = done == 1 ? blist1 + (int64_t)seg * blist1_stride : blist + (int64_t)seg * blist_stride;
    const int nb = done == 2 ? s->n_b2 : (done == 1 ? s->n_b1 : s->n_b);
    const int m_rem = done == 2 ? s->m_rem2 : (done == 1 ? s->m_rem1 : s->m_rem);
    const int top_bit = done == 2 ? s->shift2 : (done == 1 ? sel2_top_bit(s->b_or1, s->b_nor1) : sel2_top_bit(s->b_or, s->b_nor));
    sel2_finish_body<false>(l, bl, nb, m_rem, s->n_sure, top_bit, emptybits + (int64_t)seg * cand_words, cand_words, P, m,
                            out + (int64_t)seg * out_stride, out_counts + seg);
}

// Launches of few queries.  A boundary list longer than what LDS holds goes through a digit pass by all workgroups of the query.  The
// bin filter, which every query goes through in any case, counts the pass's digits: all that it may be, the score within the bin, the
// score itself (scores close together) and the passage id (keys that share their score).  The pass itself, sel2_cut_kernel<1>, takes
// one of them, and the last of its workgroups to arrive cuts what is left; a list that is not too long the query's first workgroup cuts
// at once.  So a selection is two launches (four with the second pass below), of which each costs 4.6 us when it waits for the one
// before, however little it does (a search of
// one query of 10 000 / 200 000 / 400 000 / 8.8 M passages took 71.8 / 81.1 / 104.5 / 279 us with the digits counted, filtered and the
// rest cut by launches of their own, now 68.1 / 78.4 / 101.7 / 269; 23 queries of 123 457 167.0 / 162.4).  In launches of many queries
// the other form wins: its workgroups are small, most find nothing to do, and tie groups do not meet in one histogram's word (512 of
// 400 000: 78 us for the selection, 105 with this one; hardly a survivor 105, 180).
// Two passes can be chained: when a few distinct scores are shared by very many passages, the first digit falls into the score
// and leaves one whole tie group, the second, from the highest bit in which the keys left differ, falls into the passage-id bits and
// leaves 2^-11 of it.
#define SEL2_FEW 32
// The boundary digit of a histogram of PER digits per thread (which starts at digit `first` and comes round): the smallest whose count,
// and those before it, reach r.  Every thread of the workgroup returns the same.
template <int PER>
__device__ __forceinline__ void sel2_boundary(const int32_t *__restrict__ gh, uint32_t first, int r, Sel2Finish &l, int &bstar, int &before)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = gh[PER == 1 ? (threadIdx.x + first) & (FIN_THREADS - 1) : 2 * threadIdx.x], c1 = PER == 2 ? gh[PER * threadIdx.x + 1] : 0;
    int incl = c0 + c1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    if (lane == 63) l.h256[wave] = incl;
    if (threadIdx.x == 0) {
        l.sh[0] = SEL_BINS;
        l.sh[1] = 0;
    }
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += l.h256[w];
    const int excl = incl - c0 - c1;
    if (excl < r && incl >= r) {
        const bool second = excl + c0 < r;
        l.sh[0] = PER * threadIdx.x + (second ? 1 : 0);
        l.sh[1] = excl + (second ? c0 : 0);
    }
    __syncthreads();
    bstar = __builtin_amdgcn_readfirstlane(l.sh[0]);
    before = __builtin_amdgcn_readfirstlane(l.sh[1]);
    __syncthreads();
}

// Digit pass over an over-long boundary list by all of a query's workgroups (smaller digits are selected, the boundary digit's keys
// are left) and, by the last of them to arrive, the end of the selection; a list that LDS holds is cut by the first workgroup
// alone.  LEVEL 1: the bin filter's list; what it leaves goes on to LEVEL 2 if that is launched (second) and LDS does not hold it.
// Nobody waits for anybody; what the last workgroup reads of the others' goes past the XCDs' caches (AGENT).
template <int LEVEL>
__global__ __launch_bounds__(FIN_THREADS, 8) void sel2_cut_kernel(const uint64_t *__restrict__ list, int64_t list_stride, Sel2State *state,
                                                               const int32_t *__restrict__ hist, const int32_t *__restrict__ low,
                                                               const S2Meta *__restrict__ meta, int lists,
                                                               int id_shift, int second, uint64_t *left, int64_t left_stride,
                                                               const uint32_t *__restrict__ emptybits, int64_t cand_words, int64_t P,
                                                               int32_t m, uint64_t *out, int64_t out_stride, int32_t *__restrict__ out_counts)
{
    __shared__ Sel2Finish l;
    __shared__ Sel2Place<FIN_THREADS> place;
    constexpr int GROUPS = SEL2_GROUPS / 2, STEP = FIN_THREADS * GROUPS;
    const int seg = blockIdx.y;
    Sel2State *s = state + seg;
    const uint64_t *bl = list + (int64_t)seg * list_stride;
    uint64_t *o = out + (int64_t)seg * out_stride;
    int n = LEVEL == 1 ? s->n_b : s->n_b1, m_rem = LEVEL == 1 ? s->m_rem : s->m_rem1, n_sure = s->n_sure, top_bit;
    if (LEVEL == 2 && n <= SEL_SORT_CAP) return;  // (uniform) LEVEL 1 has ended the selection
    if (n <= SEL_SORT_CAP) {
        if (blockIdx.x > 0) return;
        top_bit = sel2_top_bit(s->b_or, s->b_nor);
    } else {
        if ((int64_t)blockIdx.x * STEP >= n) return;
        const int n_work = (n + STEP - 1) / STEP < (int)gridDim.x ? (n + STEP - 1) / STEP : (int)gridDim.x;
        // LEVEL 1: the digit of the score, its lowest bits where all lie that near, or the id's where all keys share the score
        const uint32_t ord_min = ~s->ord_nmin, ord_span = s->ord_max - ord_min;
        const bool tie = LEVEL == 1 && ord_span == 0;
        const S2Meta mt = meta[seg];
        const bool is_list = lists && mt.K <= S2_MAX_KEPT;
        const int bin = s->bin, bin_shift = is_list ? S2_COARSE_SHIFT : 0;
        const bool near = LEVEL == 1 && !tie && is_list && ord_span < SEL2_SUB;
        int shift = 0, width = 0, bstar, before;
        if (LEVEL == 2) sel2_digit_plan<2>(s, shift, width);
        const int32_t *gh = near ? low + (int64_t)(seg + 1) * SEL_BINS - SEL2_SUB : hist + (int64_t)seg * SEL_BINS;
        sel2_boundary<LEVEL == 1 ? 1 : 2>(tie ? gh + SEL2_SUB : gh, near ? ord_min : 0u, m_rem, l, bstar, before);
        uint64_t *my_left = left + (int64_t)seg * left_stride;
        unsigned long long any = 0, none = 0;
        int parity = 0;
        // (positions in 32 bits, n + the step of all workgroups < 2^32: with 64 LEVEL 2 spilled a register)
        for (uint32_t s0 = blockIdx.x * STEP; s0 < (uint32_t)n; s0 += (uint32_t)n_work * STEP, parity ^= 1) {  // uniform
            uint64_t key[GROUPS];
            int cls[GROUPS];
#pragma unroll
            for (int u = 0; u < GROUPS; ++u) {
                const uint32_t i = s0 + u * FIN_THREADS + threadIdx.x;
                key[u] = i < (uint32_t)n ? bl[i] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < GROUPS; ++u) {
                const int d = LEVEL == 2 ? digit_of(key[u], shift, width)
                              : tie        ? (int)((uint32_t)key[u] >> id_shift)
                              : near       ? (int)((uint32_t)(key[u] >> 32) - ord_min)
                                           : sel2_sub_bin(key[u], mt, bin, bin_shift);
                cls[u] = s0 + u * FIN_THREADS + threadIdx.x < (uint32_t)n ? (d < bstar ? 0 : (d == bstar ? 1 : 2)) : 2;
            }
            sel2_place<FIN_THREADS, GROUPS, true>(key, cls, parity, place, &s->n_sure, LEVEL == 1 ? &s->n_b1 : &s->n_b2, o, my_left, any, none);
        }
        if (LEVEL == 1) sel2_place_bits<FIN_THREADS>(any, none, place, &s->b_or1, &s->b_nor1);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);  // every store and atomic of this wave has completed
        __syncthreads();
        if (threadIdx.x == 0) l.sh[0] = __hip_atomic_fetch_add(&s->arrived[LEVEL - 1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (l.sh[0] != n_work - 1) return;  // uniform
        auto word = [](const int32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        n = word(LEVEL == 1 ? &s->n_b1 : &s->n_b2);
        n_sure = word(&s->n_sure);
        m_rem -= before;
        if (LEVEL == 1) {
            if (second && n > SEL_SORT_CAP) {  // uniform
                if (threadIdx.x == 0) s->m_rem1 = m_rem;
                return;
            }
            top_bit = sel2_top_bit(__hip_atomic_load(&s->b_or1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                                   __hip_atomic_load(&s->b_nor1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        } else {
            top_bit = shift;
        }
        bl = my_left;
        __syncthreads();
    }
    sel2_finish_body<true>(l, bl, n, m_rem, n_sure, top_bit, emptybits + (int64_t)seg * cand_words, cand_words, P, m, o, out_counts + seg);
}

void plaid_launch_select2(hipStream_t st, uint64_t *keys2, int64_t key_stride, const uint32_t *candbits, int nq, int64_t P,
                          int64_t cand_words, int32_t m, const Stage2Buffers &b, uint64_t *out, int64_t out_stride,
                          int32_t *out_counts, int lists)
{
    const int gx = blocks_for(P, nq);
    // (lists hold some ten thousand keys: with many queries 16 workgroups each, which stride, are enough; 64 each took
    // 86 us for 512 queries, nearly all of them to find that there was nothing for them to do)
    const int gx_filter = lists && nq >= 16 && gx > 16 ? 16 : gx;
    if (nq <= SEL2_FEW && P > SEL_SORT_CAP) {
        // (the second pass as below; a list of no more than LDS holds has not gone through the first)
        const int second = (nq >= 8 || lists) && P > SEL2_SECOND_MIN_PASSAGES ? 1 : 0;
        const int id_shift = sel2_id_shift(P), cut = gx < 2 ? 1 : gx / 2;
        // (more workgroups than below: with 16 a query counting the digits of long lists was slow.  us per search, hardly a survivor, ndocs
        // 4096, with 16 / 32 / 64: sixteen queries of 200 000 passages 231 / 220 / 213, of 400 000 427 / 403 / 389, of 3 M 826 / 640 / 545,
        // 32 1128 / 930 / 844; the other form 223, 397, 721, 1017.  Lists that need no digit pass: 24 of 400 000, ndocs 256, 178 / 178 / 180)
        const int gx_bins = nq > 16 && gx > 32 ? 32 : gx;
        hipLaunchKernelGGL(sel2_bins_kernel, dim3(gx_bins, nq), dim3(SEL_THREADS), 0, st, keys2, key_stride, candbits, cand_words, P, m,
                           b.meta, b.hist, b.state, out, out_stride, b.blist, P, lists, b.list_counts, id_shift, b.hist1);
        hipLaunchKernelGGL(sel2_cut_kernel<1>, dim3(cut, nq), dim3(FIN_THREADS), 0, st, b.blist, P, b.state, b.hist1, b.hist, b.meta, lists,
                           id_shift, second, keys2, key_stride, b.emptybits, cand_words, P, m, out, out_stride, out_counts);
        if (second) {
            hipLaunchKernelGGL(sel2_digit_hist_kernel<2>, dim3(gx, nq), dim3(SEL_THREADS), 0, st, keys2, key_stride, b.state, b.hist2,
                               SEL_SORT_CAP);
            hipLaunchKernelGGL(sel2_cut_kernel<2>, dim3(cut, nq), dim3(FIN_THREADS), 0, st, keys2, key_stride, b.state, b.hist2, b.hist, b.meta,
                               lists, id_shift, 0, b.blist, P, b.emptybits, cand_words, P, m, out, out_stride, out_counts);
        }
        return;
    }
    hipLaunchKernelGGL(sel2_filter_kernel, dim3(gx_filter, nq), dim3(SEL_THREADS), 0, st, keys2, key_stride, candbits, cand_words, P,
                       m, b.meta, b.hist, b.state, out, out_stride, b.blist, P, lists, b.list_counts);
    // Digit filters: only a boundary list longer than SEL2_DIGIT_MIN makes them do anything.  The second pair is worth its
    // two launches for large indexes (a tie group can be as long as the index) in launches of several queries; otherwise
    // the query's finishing workgroup handles a long remainder alone (same result).  keys2 serves as the first
    // filter's output list, b.blist (its input) as the second one's.
    // (the coarse bins of a key list can hold two scores that millions of passages share: then the first digit leaves a whole
    // tie group also in a launch of one query, 2.8 ms for the finishing workgroup alone on 8.8 M passages)
    const int levels = P > SEL2_DIGIT_MIN ? (((nq >= 8 || lists) && P > SEL2_SECOND_MIN_PASSAGES) ? 2 : 1) : 0;
    if (levels >= 1) {
        hipLaunchKernelGGL(sel2_digit_hist_kernel<1>, dim3(gx, nq), dim3(SEL_THREADS), 0, st, b.blist, P, b.state, b.hist1,
                           SEL2_DIGIT_MIN);
        hipLaunchKernelGGL(sel2_digit_filter_kernel<1>, dim3(gx, nq), dim3(SEL_THREADS), 0, st, b.blist, P, b.state, b.hist1,
                           out, out_stride, keys2, key_stride);
    }
    if (levels >= 2) {
        hipLaunchKernelGGL(sel2_digit_hist_kernel<2>, dim3(gx, nq), dim3(SEL_THREADS), 0, st, keys2, key_stride, b.state, b.hist2,
                           SEL2_DIGIT_MIN);
        hipLaunchKernelGGL(sel2_digit_filter_kernel<2>, dim3(gx, nq), dim3(SEL_THREADS), 0, st, keys2, key_stride, b.state,
                           b.hist2, out, out_stride, b.blist, P);
    }
    hipLaunchKernelGGL(sel2_finish_kernel, dim3(nq), dim3(FIN_THREADS), 0, st, b.blist, P, keys2, key_stride, b.state,
                       b.emptybits, cand_words, P, m, levels, out, out_stride, out_counts);
}
