// Small helper kernels: fills, key -> (id, score) conversion, bitmap -> ascending id list.
#include "plaid_internal.h"

#include <math.h>

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, int64_t n, uint32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
void plaid_launch_fill_u32(hipStream_t st, uint32_t *p, int64_t n, uint32_t v)
{
    if (n <= 0) return;
    int64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((int)g), dim3(256), 0, st, p, n, v);
}

// Final ranking -> caller buffers: ids[q][j], scores[q][j] for j < counts[q] (capped at k), (-1, -inf) beyond.
__global__ void keys_to_output_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                      const int32_t *__restrict__ counts, int32_t k, int32_t *__restrict__ out_ids,
                                      float *__restrict__ out_scores)
{
    const int q = blockIdx.y;
    const int n = counts[q] < k ? counts[q] : k;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < k; j += gridDim.x * blockDim.x) {
        int32_t id = -1;
        float sc = -INFINITY;
        if (j < n) {
            const uint64_t key = keys[(int64_t)q * key_stride + j];
            id = (int32_t)(key & 0xFFFFFFFFu);
            sc = plaid_ord_to_score((uint32_t)(key >> 32));
        }
        out_ids[(int64_t)q * k + j] = id;
        out_scores[(int64_t)q * k + j] = sc;
    }
}
void plaid_launch_keys_to_output(hipStream_t st, const uint64_t *keys, int64_t key_stride, const int32_t *counts, int nq,
                                 int32_t k, int32_t *out_ids, float *out_scores)
{
    int g = (k + 255) / 256;
    if (g > 64) g = 64;
    hipLaunchKernelGGL(keys_to_output_kernel, dim3(g, nq), dim3(256), 0, st, keys, key_stride, counts, k, out_ids,
                       out_scores);
}

// Debug dump of a key list as (id, score) pairs; any output pointer may be null.
__global__ void keys_to_pairs_kernel(const uint64_t *__restrict__ keys, int64_t key_stride,
                                     const int32_t *__restrict__ counts, int32_t cap, int32_t *__restrict__ out_ids,
                                     float *__restrict__ out_scores, int32_t *__restrict__ out_counts)
{
    const int q = blockIdx.y;
    const int n = counts[q] < cap ? counts[q] : cap;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        const uint64_t key = keys[(int64_t)q * key_stride + j];
        if (out_ids) out_ids[(int64_t)q * cap + j] = (int32_t)(key & 0xFFFFFFFFu);
        if (out_scores) out_scores[(int64_t)q * cap + j] = plaid_ord_to_score((uint32_t)(key >> 32));
    }
    if (out_counts && blockIdx.x == 0 && threadIdx.x == 0) out_counts[q] = n;
}
void plaid_launch_keys_to_pairs(hipStream_t st, const uint64_t *keys, int64_t key_stride, const int32_t *counts, int nq,
                                int32_t cap, int32_t *out_ids, float *out_scores, int32_t *out_counts)
{
    int g = (cap + 255) / 256;
    if (g > 64) g = 64;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(keys_to_pairs_kernel, dim3(g, nq), dim3(256), 0, st, keys, key_stride, counts, cap, out_ids,
                       out_scores, out_counts);
}

// A workgroup per query; the lists have up to some thousand keys, each passage once.
__global__ __launch_bounds__(256) void keys_of_passages_kernel(const uint64_t *__restrict__ in_keys, int64_t in_stride,
                                                               const int32_t *__restrict__ in_counts, const uint64_t *__restrict__ keys,
                                                               const int32_t *__restrict__ counts, int64_t stride, uint64_t *__restrict__ out)
{
    const int q = blockIdx.x, n = in_counts[q], m = counts[q];
    for (int j = threadIdx.x; j < m; j += 256) {
        const uint32_t pid = (uint32_t)keys[(int64_t)q * stride + j];
        uint64_t found = PLAID_KEY_MAX;
        for (int i = 0; i < n; ++i) {
            const uint64_t key = in_keys[(int64_t)q * in_stride + i];
            found = (uint32_t)key == pid ? key : found;
        }
        out[(int64_t)q * stride + j] = found;
    }
}
void plaid_launch_keys_of_passages(hipStream_t st, const uint64_t *in_keys, int64_t in_stride, const int32_t *in_counts, const uint64_t *keys,
                                   const int32_t *counts, int64_t stride, int nq, uint64_t *out)
{
    hipLaunchKernelGGL(keys_of_passages_kernel, dim3(nq), dim3(256), 0, st, in_keys, in_stride, in_counts, keys, counts, stride, out);
}

// Ascending list of the set bits of bits[q][0..words).  A workgroup lists `chunk` words (a multiple of 1024) and counts the bits of all
// words before them itself, a few loads per thread and no waiting for another workgroup.  A wave writes the ids of 64 passages at a
// time, side by side.  Sixteen queries of 400 000 candidates: 12 us, with one workgroup per query, a scan through LDS and a thread
// per word 239.
__global__ __launch_bounds__(1024) void bitmap_to_list_kernel(const uint32_t *__restrict__ bits, int64_t words,
                                                              int64_t nvalid, int64_t chunk, int32_t *__restrict__ out,
                                                              int64_t out_stride, int32_t *__restrict__ out_counts)
{
    __shared__ int32_t wave_sum[16];
    const int q = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t *b = bits + (int64_t)q * words;
    int32_t *o = out ? out + (int64_t)q * out_stride : nullptr;
    auto valid = [&](int64_t w, uint32_t v) -> uint32_t {  // bits beyond the valid range do not count
        const int64_t keep = nvalid - w * 32;
        return keep >= 32 ? v : (keep <= 0 ? 0u : v & ((1u << keep) - 1u));
    };
    const int64_t first = (int64_t)blockIdx.x * chunk, last = first + chunk < words ? first + chunk : words;
    int cnt = 0;
    for (int64_t w = threadIdx.x; w < first; w += 8 * 1024) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = w + 1024 * u < first ? b[w + 1024 * u] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) cnt += __popc(w + 1024 * u < first ? valid(w + 1024 * u, v[u]) : 0u);
    }
    int incl = cnt;
    // inclusive sums over the waves' lanes; the waves' totals in LDS; what lies before this wave, and the total
    auto totals = [&](int &before, int &all) {
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        before = all = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int t = wave_sum[v];
            if (v < wave) before += t;
            all += t;
        }
        __syncthreads();  // (the sums are written again)
    };
    int before, base;
    totals(before, base);  // base: bits of the words before `first`
    for (int64_t w0 = first; w0 < last; w0 += 1024) {  // uniform
        const int64_t w = w0 + threadIdx.x;
        const uint32_t v = w < last ? valid(w, b[w]) : 0u;
        incl = __popc(v);
        const int mine = incl;
        int all;
        totals(before, all);
        const int at = base + before + incl - mine;  // of this lane's first bit
        auto write = [&](int k) {                    // the ids of words k and k + 1 of the wave's
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, k), hi = (uint32_t)__builtin_amdgcn_readlane((int)v, k + 1);
            const int place = __builtin_amdgcn_readlane(at, k);
            const unsigned long long m = (unsigned long long)hi << 32 | lo;
            if ((m >> lane) & 1ull)
                o[place + __popcll(m & ((1ull << lane) - 1ull))] = (int32_t)((w0 + 64 * wave + k) * 32 + lane);
        };
        const unsigned long long some = __ballot(v != 0u);
        unsigned long long pairs = o ? (some | some >> 1) & 0x5555555555555555ull : 0ull;
        if (__popcll(pairs) > 16) {                  // uniform over the wave
#pragma unroll 4
            for (int k = 0; k < 64; k += 2) write(k);
        } else {                                     // few of them (the probed centroids of a query)
            for (; pairs; pairs &= pairs - 1) write((int)__builtin_ctzll(pairs));
        }
        base += all;
    }
    if (threadIdx.x == 0 && out_counts && blockIdx.x == gridDim.x - 1) out_counts[q] = base;
}
void plaid_launch_bitmap_to_list(hipStream_t st, const uint32_t *bits, int64_t words, int64_t nbits_valid, int nq,
                                 int32_t *out, int64_t out_stride, int32_t *out_counts)
{
    // (64 workgroups per query at most: each reads the words before its own)
    const int64_t parts = (words + 1023) / 1024, most = 64, per = (parts + most - 1) / most;
    const int64_t chunk = 1024 * (per > 1 ? per : 1);
    const int64_t gx = words > chunk ? (words + chunk - 1) / chunk : 1;
    hipLaunchKernelGGL(bitmap_to_list_kernel, dim3((unsigned)gx, nq), dim3(1024), 0, st, bits, words, nbits_valid, chunk, out, out_stride,
                       out_counts);
}

// ------------------------------------------------------------------ structural validation of a device-resident index
// The search kernels index memory with the index's own offsets, codes and passage ids, so an index whose arrays arrive
// in device memory is checked once, when the handle is made: doc_offsets from 0 to N without a decrease, codes in
// [0, C), ivf_offsets from 0 to ivf_len without a decrease, passage ids in [0, P) and strictly ascending inside each
// list.  bad[0] receives the OR of: 1 doc_offsets, 2 codes, 4 ivf_offsets, 8 passage id out of range, 16 list not
// strictly ascending.  Grid-stride loops over each array; the list test looks up the list of entry e by binary search
// in ivf_offsets only when e follows a larger-or-equal id (a list boundary or an error), so it costs one pass over
// the ids.
__global__ __launch_bounds__(256) void index_validate_kernel(const int64_t *__restrict__ doc_offsets, int64_t P, int64_t N,
                                                             const int32_t *__restrict__ codes, int64_t C,
                                                             const int64_t *__restrict__ ivf_offsets,
                                                             const int32_t *__restrict__ ivf_pids, int64_t ivf_len,
                                                             int32_t *__restrict__ bad)
{
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    int flags = 0;
    for (int64_t p = t0; p <= P; p += step) {
        const int64_t o = doc_offsets[p];
        if (o < 0 || o > N || (p == 0 && o != 0) || (p == P && o != N)) flags |= 1;
        if (p < P && doc_offsets[p + 1] < o) flags |= 1;
    }
    for (int64_t j = t0; j < N; j += step) {
        const int32_t c = codes[j];
        if (c < 0 || c >= C) flags |= 2;
    }
    for (int64_t c = t0; c <= C; c += step) {
        const int64_t o = ivf_offsets[c];
        if (o < 0 || o > ivf_len || (c == 0 && o != 0) || (c == C && o != ivf_len)) flags |= 4;
        if (c < C && ivf_offsets[c + 1] < o) flags |= 4;
    }
    for (int64_t e = t0; e < ivf_len; e += step) {
        const int32_t pid = ivf_pids[e];
        if (pid < 0 || pid >= P) flags |= 8;
        if (e > 0 && ivf_pids[e - 1] >= pid) {
            // allowed only when e is the first entry of a list: some offset equals e
            int64_t lo = 0, hi = C;  // largest lo with ivf_offsets[lo] <= e (offsets validated by other threads: a
            while (lo < hi) {        // malformed table can only produce a wrong verdict here, and sets flag 4 there)
                const int64_t mid = (lo + hi + 1) >> 1;
                if (ivf_offsets[mid] <= e) lo = mid;
                else hi = mid - 1;
            }
            if (ivf_offsets[lo] != e) flags |= 16;
        }
    }
    if (flags) atomicOr(bad, flags);
}
void plaid_launch_index_validate(hipStream_t st, const int64_t *doc_offsets, int64_t P, int64_t N, const int32_t *codes,
                                 int64_t C, const int64_t *ivf_offsets, const int32_t *ivf_pids, int64_t ivf_len, int32_t *bad)
{
    int64_t work = N > ivf_len ? N : ivf_len;
    if (work < P + 1) work = P + 1;
    if (work < C + 1) work = C + 1;
    int64_t g = (work + 255) / 256;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(index_validate_kernel, dim3((unsigned)g), dim3(256), 0, st, doc_offsets, P, N, codes, C, ivf_offsets,
                       ivf_pids, ivf_len, bad);
}
