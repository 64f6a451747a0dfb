// Stage 4 (Sections 4.4-4.5): residual decompression fused with exact MaxSim (Eq. 1).
//
// Decompression follows the lookup-table idea of Section 4.5: a packed byte indexes a 256-entry
// table held in LDS.  A reconstructed token is centroid + residual, so its dot product with a query
// token is S_cq[code][i] (already computed, Eq. 2) plus the residual's dot product: the scoring kernel
// gathers the 128-byte S_cq row of each token instead of its 512-byte centroid and contracts only the
// residuals, which take one of 2^nbits bucket weights per dimension.
//
// The contraction runs on the half-precision matrix instruction with both operands split into two fp16
// terms, x = x1 + 2^-11 x2 (|x - x1 - 2^-11 x2| <= 2^-22 |x|): three products per term, each exact in
// fp32, the leading one in one accumulator and the two cross terms in a second, scaled one.  Two tables
// hold, per byte value, the leading and the trailing fp16 terms of the bucket weights of the byte's
// dimensions, in the order the instruction wants them: an LDS read yields half of an operand (2-bit codes)
// or all of it (1-bit codes) in place, and the decoded 32-token x 128 residual tile never leaves registers.
// (One vector instruction per byte, to form the address.  With both terms in one 16-byte entry, registers had to be moved, six
// per byte; picking the terms by byte permutations from registers takes nine per byte.)
// Against fp32 arithmetic the residual's dot product loses at most 3 * 2^-22 |r||q|, far inside the score
// tolerance.
// The standalone decompression kernel below produces the reconstructed vectors themselves
// (centroid + weight, one fp32 addition).
#include "plaid_internal.h"

#include <math.h>
#include <stddef.h>
#include <type_traits>

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 s4_half8 __attribute__((ext_vector_type(8)));
typedef _Float16 s4_half4 __attribute__((ext_vector_type(4)));
#define S4_RESIDENT_BLOCKS 1024
#define S4_SCALE 2048.0f  // 2^11

// The two fp16 terms of x: x1 = fp16(x) (0 below fp16's normal range), x2 = fp16(2^11 (x - x1)).
__device__ __forceinline__ void s4_split(float x, _Float16 &x1, _Float16 &x2)
{
    x1 = fabsf(x) >= 6.103515625e-05f ? (_Float16)x : (_Float16)0.0f;
    x2 = (_Float16)((x - (float)x1) * S4_SCALE);
}

// Table entry (byte v, quad s): weights of dimensions 4s .. 4s+3 of the 8/NBITS dimensions packed in v.
// Bucket indices are stored most-significant first.
template <int NBITS>
__device__ __forceinline__ void build_tables(float4 *wlut, uint32_t *ilut, const float *__restrict__ weights, int tid,
                                             int nthreads)
{
    constexpr int QUADS = NBITS == 2 ? 1 : 2;
    for (int e = tid; e < 256 * QUADS; e += nthreads) {
        const int v = e / QUADS, s = e % QUADS;
        uint32_t idx[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int d = 4 * s + t;  // dimension within the byte
            idx[t] = (v >> (8 - NBITS * (d + 1))) & ((1 << NBITS) - 1);
        }
        wlut[e] = make_float4(weights[idx[0]], weights[idx[1]], weights[idx[2]], weights[idx[3]]);
        if (ilut) ilut[e] = idx[0] | (idx[1] << 8) | (idx[2] << 16) | (idx[3] << 24);
    }
}
// Entry for dimensions 4*quad .. 4*quad+3 of a token whose packed residual starts at r.
template <int NBITS>
__device__ __forceinline__ int table_slot(const uint8_t *__restrict__ r, int quad)
{
    if (NBITS == 2) return r[quad];
    return 2 * r[quad >> 1] + (quad & 1);
}

// Operand tables of the scoring kernels: entry v (S4_SECOND + v) holds the leading (trailing) fp16 terms of the
// weights of the dimensions packed in byte v: four of them (2-bit codes) or eight.
// (257 entries between them: the two halves of a byte are then two LDS reads, each straight to its operand; at a distance one
// instruction can span the compiler makes them one, whose result has to be moved apart.)
#define S4_SECOND 257
template <int NBITS>
struct S4Entry {
    typedef s4_half4 type;
};
template <>
struct S4Entry<1> {
    typedef s4_half8 type;
};
template <int NBITS, bool SECOND = true>
__device__ __forceinline__ void s4_build_tables(typename S4Entry<NBITS>::type *hlut, const float *__restrict__ weights, int tid,
                                                int nthreads)
{
    for (int v = tid; v < 256; v += nthreads) {
        typename S4Entry<NBITS>::type a, b;
#pragma unroll
        for (int d = 0; d < 8 / NBITS; ++d) {
            _Float16 x1, x2;
            s4_split(weights[(v >> (8 - NBITS * (d + 1))) & ((1 << NBITS) - 1)], x1, x2);
            a[d] = x1;
            b[d] = x2;
        }
        hlut[v] = a;
        if (SECOND) hlut[S4_SECOND + v] = b;
    }
}
// A half of the wave (h = lane / 32) contracts half of the 128 dimensions, the 2 NBITS packed words 2 NBITS h .. of a token;
// step s = 0 .. 7 takes two bytes (2-bit codes) or one of them.
__device__ __forceinline__ int s4_dim(int s, int h, int e)  // dimension of element e of the operands of step s, half h
{
    return 64 * h + 8 * s + e;
}
template <int NBITS>
__device__ __forceinline__ void s4_decode(const uint32_t (&rw)[2 * NBITS], int s, const typename S4Entry<NBITS>::type *hlut,
                                          s4_half8 &a1, s4_half8 &a2)
{
    if constexpr (NBITS == 2) {
        const uint32_t w = rw[s >> 1] >> (16 * (s & 1)), b0 = w & 0xFFu, b1 = (w >> 8) & 0xFFu;
        const s4_half4 x0 = hlut[b0], x1 = hlut[b1], y0 = hlut[S4_SECOND + b0], y1 = hlut[S4_SECOND + b1];
        a1 = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
        a2 = __builtin_shufflevector(y0, y1, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
        const uint32_t b = (rw[s >> 2] >> (8 * (s & 3))) & 0xFFu;
        a1 = hlut[b];
        a2 = hlut[S4_SECOND + b];
    }
}
// fmaxf without the canonicalising copies the compiler puts in front of it.
__device__ __forceinline__ float s4_max(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float s4_max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// The two fp16 terms of the query in the operand order of v_mfma_f32_32x32x16_f16, into LDS: lane 32 h + r of step s holds
// query token r, dimensions s4_dim(s, h, 0) .. + 7.  All 256 threads of the workgroup call this, a barrier follows.
template <int TERMS>
__device__ __forceinline__ void s4_stage_query(const float *__restrict__ Qq, s4_half8 (&qs)[TERMS][8][64])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = (int)threadIdx.x + 256 * i, s = e >> 6, l = e & 63;
        s4_half8 t1, t2;
        const float4 *p = reinterpret_cast<const float4 *>(Qq + (l & 31) * DIM + s4_dim(s, l >> 5, 0));
        const float4 u = p[0], w = p[1];
        const float x[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            _Float16 x1, x2;
            s4_split(x[j], x1, x2);
            t1[j] = x1;
            t2[j] = x2;
        }
        qs[0][s][l] = t1;
        if constexpr (TERMS > 1) qs[TERMS - 1][s][l] = t2;
    }
}

// Residual dot products of 32 tokens (packed words rw, this half's) with the 32 query tokens: acc += leading products, acx +=
// cross terms, scaled by 2^11.  TOKENS_A: rows = tokens, columns = query tokens; else the other way round.  The query
// operands are read from LDS in every step, through an index the compiler cannot tell from the last call's (kept across
// calls they would take 64 registers), but for the first H1 of the leading and H2 of the trailing terms, which the caller holds.
// AHEAD: they and the table entries are requested one step of 16 dimensions ahead, for which a kernel of four waves per SIMD lacks
// the registers.
template <int NBITS, bool TOKENS_A, bool AHEAD, int H1, int H2>
__device__ __forceinline__ void s4_products(const uint32_t (&rw)[2 * NBITS], const typename S4Entry<NBITS>::type *hlut,
                                            const s4_half8 (&qs)[2][8][64], const s4_half8 *held1, const s4_half8 *held2, int lane,
                                            floatx16 &acc, floatx16 &acx)
{
    int ql = lane;
    asm volatile("" : "+v"(ql));
    auto first = [&](int s) { return s < H1 ? held1[s] : qs[0][s][ql]; };
    auto second = [&](int s) { return s < H2 ? held2[s] : qs[1][s][ql]; };
    s4_half8 a1, a2, q1 = first(0), q2 = second(0);
    s4_decode<NBITS>(rw, 0, hlut, a1, a2);
    if (AHEAD) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        s4_half8 n1 = a1, n2 = a2, r1 = q1, r2 = q2;
        if (s < 7) {
            r1 = first(s + 1);
            r2 = second(s + 1);
            s4_decode<NBITS>(rw, s + 1, hlut, n1, n2);
        }
        acx = TOKENS_A ? __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, q2, acx, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_f16(q2, a1, acx, 0, 0, 0);
        acc = TOKENS_A ? __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, q1, acc, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_f16(q1, a1, acc, 0, 0, 0);
        acx = TOKENS_A ? __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, q1, acx, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_f16(q1, a2, acx, 0, 0, 0);
        if (AHEAD && s < 7) {
            __builtin_amdgcn_sched_group_barrier(0x002, NBITS, 0);              // the addresses,
            // LDS reads, then the matrix instructions
            if (s + 1 < H1 && s + 1 < H2) __builtin_amdgcn_sched_group_barrier(0x100, NBITS == 2 ? 4 : 2, 0);
            else if (s + 1 < H1 || s + 1 < H2) __builtin_amdgcn_sched_group_barrier(0x100, NBITS == 2 ? 5 : 3, 0);
            else __builtin_amdgcn_sched_group_barrier(0x100, NBITS == 2 ? 6 : 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
        }
        a1 = n1, a2 = n2, q1 = r1, q2 = r2;
        if (AHEAD) __builtin_amdgcn_sched_barrier(0);
    }
}

// The leading products alone, rows = tokens.
template <int NBITS, int H1>
__device__ __forceinline__ void s4_leading_products(const uint32_t (&rw)[2 * NBITS], const typename S4Entry<NBITS>::type *hlut,
                                                    const s4_half8 (&qs)[8][64], const s4_half8 *held1, int lane, floatx16 &acc)
{
    auto decode = [&](int s) -> s4_half8 {
        if constexpr (NBITS == 2) {
            const uint32_t w = rw[s >> 1] >> (16 * (s & 1));
            const s4_half4 x0 = hlut[w & 0xFFu], x1 = hlut[(w >> 8) & 0xFFu];
            return __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return hlut[(rw[s >> 2] >> (8 * (s & 3))) & 0xFFu];
        }
    };
    int ql = lane;
    asm volatile("" : "+v"(ql));
    auto first = [&](int s) { return s < H1 ? held1[s] : qs[s][ql]; };
    s4_half8 a = decode(0), q = first(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        s4_half8 n = a, r = q;
        if (s < 7) {
            r = first(s + 1);
            n = decode(s + 1);
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, q, acc, 0, 0, 0);
        a = n, q = r;
    }
}

// Column maxima of a 32 x 32 result block spread over the wave as the matrix instruction leaves it: lane 32 h + n holds
// mx[v] = the value of query token 8 (v / 4) + 4 h + v % 4 for passage-token column n.  Returns, in lane 32 h + 2 v (and
// its odd neighbour), the maximum over the 32 columns for that query token: a butterfly in which each exchange halves the
// number of values a lane still carries (16 exchanges instead of 16 x 5).
__device__ __forceinline__ float s4_column_maxima(const float (&mx)[16], int lane)
{
    float a8[8], a4[4], a2[2];
    const bool b4 = lane & 16, b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float keep = b4 ? mx[8 + e] : mx[e], send = b4 ? mx[e] : mx[8 + e];
        a8[e] = s4_max(keep, __shfl_xor(send, 16));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float keep = b3 ? a8[4 + e] : a8[e], send = b3 ? a8[e] : a8[4 + e];
        a4[e] = s4_max(keep, __shfl_xor(send, 8));
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float keep = b2 ? a4[2 + e] : a4[e], send = b2 ? a4[e] : a4[2 + e];
        a2[e] = s4_max(keep, __shfl_xor(send, 4));
    }
    const float keep = b1 ? a2[1] : a2[0], send = b1 ? a2[0] : a2[1];
    const float a1 = s4_max(keep, __shfl_xor(send, 2));
    return s4_max(a1, __shfl_xor(a1, 1));
}
// The lane that holds query token i after s4_column_maxima, and the query token of an even lane.
__device__ __forceinline__ constexpr int s4_lane_of_token(int i) { return 32 * ((i >> 2) & 1) + 2 * (4 * (i >> 3) + (i & 3)); }
__device__ __forceinline__ int s4_token_of_lane(int lane)
{
    const int v = (lane >> 1) & 15;
    return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
}

// Passages are scored 32 tokens per step with v_mfma_f32_32x32x16_f16: rows = the 32 query tokens (A operand), columns
// = 32 passage tokens (B operand); lane 32 h + r holds row / column r of its operand, dimensions s4_dim(s, h, 0) .. + 7 at
// step s of the 128 dimensions.  A lane therefore decodes the residual of one passage token, gets the results of that
// token's column (16 query tokens: 8 g + 4 h + 0..3), and adds the centroid's share from its own token's row of S_cq
// (four 16-byte loads, no exchange between lanes).  It keeps 16 running maxima over the steps of a passage; the maxima
// over the columns are taken once per passage (s4_column_maxima).
// COOP = false: one wave scores one passage at a time and the waves of the grid stride over the query's list (many
// passages per wave: throughput).  COOP = true: the four waves of a workgroup share a passage, each taking every
// fourth step, and combine their maxima in LDS (short lists: latency).
// The grid is one-dimensional; with eight queries or more (spread = 0) workgroup L serves query 8 (L / 8 / gx) + L % 8:
// consecutive workgroups go to the chip's eight partitions in turn, so a query's workgroups share one partition's
// second-level cache and the rows of S_cq its passages have in common are fetched once.
// RN: the storage variant in which a reconstructed vector is scaled to unit length: its dot products are multiplied by
// the token's factor inv_norm[token] = 1 / |centroid + residual| (plaid_launch_token_inv_norm).
// WIDE: rows of S_cq need 64-bit offsets (C > 2^25).
template <int NBITS, bool COOP, bool RN, bool WIDE>
__global__ __launch_bounds__(256, COOP ? 3 : 4) void decompress_maxsim_kernel(
    const float *__restrict__ Q, const float *__restrict__ S, int64_t C, const int64_t *__restrict__ doc_offsets,
    const int32_t *__restrict__ codes, const uint8_t *__restrict__ residuals, const float *__restrict__ weights,
    const float *__restrict__ inv_norm,
    const uint64_t *__restrict__ in_keys, int64_t in_stride, const int32_t *__restrict__ in_counts, int nq, int gx,
    int spread, uint64_t *__restrict__ out_keys, int64_t out_stride)
{
    constexpr int RB = 16 * NBITS;
    __shared__ typename S4Entry<NBITS>::type hlut[S4_SECOND + 256];
    __shared__ float wmax[4][QLEN];
    __shared__ s4_half8 qs[2][8][64];  // [term][step of 16 dimensions][lane]
    int q, bx;
    if (spread) {
        q = blockIdx.x / gx;
        bx = blockIdx.x % gx;
    } else {
        const int k = blockIdx.x >> 3;
        q = 8 * (k / gx) + (blockIdx.x & 7);
        bx = k % gx;
    }
    if (q >= nq) return;
    const int count = in_counts[q];
    if (bx * (COOP ? 1 : 4) >= count) return;  // uniform for the workgroup
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    s4_build_tables<NBITS>(hlut, weights, threadIdx.x, 256);
    const float *Qq = Q + (int64_t)q * QLEN * DIM;
    const char *Sq = reinterpret_cast<const char *>(S + (int64_t)q * C * QLEN);
    // A operands: the two fp16 terms of query token r32, dimensions s4_dim(s, h, ..).  They are the same for the four
    // waves and stay in LDS (16 KB), from where each matrix step reads them: 64 registers less per lane, which buys a
    // third wave per SIMD to cover the latency of the gathers.
    s4_stage_query(Qq, qs);
    __syncthreads();

    // In front of a passage's first step stands a chain of dependent loads: its id (from the key list), its token range,
    // its first codes and residuals.  The chain is started three passages ahead and advanced one link per passage, and the
    // first step's operands of the next passage are requested during the last step of this one, so that a wave never
    // waits for the whole chain.  Ids and ranges are the same in every lane; they are still fetched with vector loads
    // (a zero the compiler cannot see through is added to the index), which return in order and are counted apart from
    // LDS reads.  List positions past the end repeat the last passage (loaded, not scored).
    int vz;
    asm volatile("v_mov_b32 %0, 0" : "=v"(vz));
    const uint32_t *ik = reinterpret_cast<const uint32_t *>(in_keys + (int64_t)q * in_stride);  // low word: passage id
    const int j0 = COOP ? bx : bx * 4 + wave, jstride = gx * (COOP ? 1 : 4);
    auto load_id = [&](int n) -> uint32_t {
        const int64_t jj = (int64_t)j0 + (int64_t)n * jstride;
        return ik[2 * (jj < count ? jj : (int64_t)count - 1) + vz];
    };
    auto uniform64 = [](int64_t v) -> int64_t {
        return ((int64_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(v & 0xFFFFFFFFll));
    };
    constexpr int RW = 2 * NBITS;
    auto request = [&](int64_t t0, int len, int b, int32_t &c, float &nf, uint32_t (&r)[RW]) {
        const int row = b + r32;  // this lane's passage token
        const int64_t tok = t0 + (row < len ? row : len - 1);
        c = codes[tok];
        if (RN) nf = inv_norm[tok];
        // this half's half of the token's packed residual
        if (NBITS == 2) {
            const uint4 v = reinterpret_cast<const uint4 *>(residuals + tok * RB)[h];
            r[0] = v.x, r[1] = v.y, r[2 % RW] = v.z, r[3 % RW] = v.w;
        } else {
            const uint2 v = reinterpret_cast<const uint2 *>(residuals + tok * RB)[h];
            r[0] = v.x, r[1] = v.y;
        }
    };
    constexpr int STEP = COOP ? 128 : 32;
    const int base0 = COOP ? 32 * wave : 0;
    // warm-up: passage 0 completely, passage 1 up to its token range, passage 2's id
    uint32_t pid = (uint32_t)__builtin_amdgcn_readfirstlane((int)load_id(0));
    int64_t t0 = uniform64(doc_offsets[(int64_t)pid + vz]);
    int len = (int)(uniform64(doc_offsets[(int64_t)pid + 1 + vz]) - t0);
    int32_t code = 0;
    float nf = 1.0f;  // this lane's token's scaling factor (RN)
    uint32_t rw[RW] = {0};
    if (base0 < len) request(t0, len, base0, code, nf, rw);
    uint32_t pid1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)load_id(1));
    int64_t o1a = doc_offsets[(int64_t)pid1 + vz], o1b = doc_offsets[(int64_t)pid1 + 1 + vz];  // as loaded (same in every lane)
    uint32_t id2 = load_id(2);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the loop's waits then cover only what the loop itself requests

    for (int n = 0; (int64_t)j0 + (int64_t)n * jstride < count; ++n) {
        const int j = j0 + n * jstride;
        // one link further for the passages ahead
        const int64_t t0_next = uniform64(o1a);
        const int len_next = (int)(uniform64(o1b) - t0_next);
        const uint32_t pid2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)id2);
        const int64_t o2a = doc_offsets[(int64_t)pid2 + vz], o2b = doc_offsets[(int64_t)pid2 + 1 + vz];
        const uint32_t id3 = load_id(n + 3);
        int32_t code_next = 0;
        float nf_next = 1.0f;
        uint32_t rw_next[RW] = {0};
        bool next_requested = false;
        float mx[16];  // running maxima of this lane's column class: query token 8 (v / 4) + 4 h + v % 4
#pragma unroll
        for (int v = 0; v < 16; ++v) mx[v] = -INFINITY;
        // The step loop is software-pipelined too: the code and packed residual of the next step and the S_cq values of
        // this step are requested before this step's matrix instructions are issued.
        for (int base = base0; base < len; base += STEP) {
            // the centroid's share of each dot product: the token's row of S_cq, elements 8 g + 4 h .. + 3 (requested now,
            // used after the matrix instructions)
            float4 sv[4];
            {
                typename std::conditional<WIDE, uint64_t, uint32_t>::type off = (uint32_t)code;
                off = off * (uint32_t)(QLEN * 4) + 16u * (uint32_t)h;
#pragma unroll
                for (int g = 0; g < 4; ++g) sv[g] = *reinterpret_cast<const float4 *>(Sq + off + 32u * g);
            }
            if (base + STEP < len) {  // uniform
                request(t0, len, base + STEP, code_next, nf_next, rw_next);
            } else {  // last step: the first step of the next passage
                if (base0 < len_next) request(t0_next, len_next, base0, code_next, nf_next, rw_next);
                next_requested = true;
            }
            floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            floatx16 acx = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};  // cross terms, scaled by 2^11
            s4_products<NBITS, false, COOP, 0, 0>(rw, hlut, qs, nullptr, nullptr, lane, acc, acx);
            const float svf[16] = {sv[0].x, sv[0].y, sv[0].z, sv[0].w, sv[1].x, sv[1].y, sv[1].z, sv[1].w,
                                   sv[2].x, sv[2].y, sv[2].z, sv[2].w, sv[3].x, sv[3].y, sv[3].z, sv[3].w};
            if (base + 32 <= len) {  // (uniform) a full step: every column counts
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = fmaf(acx[v], 1.0f / S4_SCALE, acc[v]) + svf[v];
                    if (RN) x *= nf;
                    mx[v] = s4_max(mx[v], x);
                }
            } else if (base + r32 < len) {  // this lane's column is a token of the passage
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float x = fmaf(acx[v], 1.0f / S4_SCALE, acc[v]) + svf[v];
                    if (RN) x *= nf;
                    mx[v] = s4_max(mx[v], x);
                }
            }
            code = code_next;
            nf = nf_next;
#pragma unroll
            for (int e = 0; e < RW; ++e) rw[e] = rw_next[e];
        }
        if (!next_requested && base0 < len_next) request(t0_next, len_next, base0, code, nf, rw);  // (uniform) no step was taken
        const float cm = s4_column_maxima(mx, lane);  // query token s4_token_of_lane(lane), in even and odd lane alike
        float total;
        if (COOP) {  // j, len are the same in the four waves
            if (!(lane & 1)) wmax[wave][s4_token_of_lane(lane)] = cm;
            __syncthreads();
            const float m = fmaxf(fmaxf(wmax[0][r32], wmax[1][r32]), fmaxf(wmax[2][r32], wmax[3][r32]));
            __syncthreads();
            total = plaid_sum32_in_order(m);
        } else {
            // the sum over the query tokens of Eq. 1, in double, in index order
            double d = 0.0;
#pragma unroll
            for (int i = 0; i < QLEN; ++i)
                d += (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(cm), s4_lane_of_token(i)));
            total = (float)d;
        }
        if (lane == 0 && (!COOP || wave == 0))
            out_keys[(int64_t)q * out_stride + j] = plaid_make_key(len > 0 ? total : -INFINITY, pid);
        // the passages ahead move up
        pid = pid1, t0 = t0_next, len = len_next;
        pid1 = pid2, o1a = o2a, o1b = o2b;
        id2 = id3;
    }
}

// Stage 3's cut and the scores of what it keeps in one launch, for lists of up to CUT_KEYS keys (short launches): a workgroup per key of the
// list, which counts the keys before its own and leaves if there are m of them; otherwise its passage's score goes to the place of that
// number in out_keys.  The four waves share the passage as above.  Bound by the round trips to memory that follow one another (keys, code,
// scores), which a launch's start and a list that goes through memory only add to: one query of 400 000 passages, 1024 keys of which 256
// stay, 5.2 and 6.9 us as two launches, 6.9 us so; 256 keys of which 64 stay 4.2 and 5.5, 4.8 so.
#define CUT_KEYS 1024
template <int NBITS, bool RN, bool WIDE>
__global__ __launch_bounds__(256, 3) void cut_maxsim_kernel(
    const float *__restrict__ Q, const float *__restrict__ S, int64_t C, const int64_t *__restrict__ doc_offsets,
    const int32_t *__restrict__ codes, const uint8_t *__restrict__ residuals, const float *__restrict__ weights,
    const float *__restrict__ inv_norm, const uint64_t *__restrict__ in_keys, int64_t in_stride, const int32_t *__restrict__ in_counts,
    int32_t m, uint64_t *__restrict__ out_keys, int64_t out_stride, int32_t *__restrict__ out_counts)
{
    constexpr int RB = 16 * NBITS, RW = 2 * NBITS, EACH = CUT_KEYS / 256;
    __shared__ typename S4Entry<NBITS>::type hlut[S4_SECOND + 256];
    __shared__ float wmax[4][QLEN];
    __shared__ s4_half8 qs[2][8][64];  // [term][step of 16 dimensions][lane]
    __shared__ int32_t fewer[4];
    const int q = blockIdx.y, j = blockIdx.x;
    const int n = in_counts[q] < CUT_KEYS ? in_counts[q] : CUT_KEYS;
    if (j == 0 && threadIdx.x == 0) out_counts[q] = m < n ? m : n;
    if (j >= n) return;  // uniform
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const uint64_t *keys = in_keys + (int64_t)q * in_stride;
    uint64_t other[EACH];
#pragma unroll
    for (int u = 0; u < EACH; ++u) other[u] = (int)threadIdx.x + 256 * u < n ? keys[threadIdx.x + 256 * u] : PLAID_KEY_MAX;
    const uint64_t mine = keys[j];
    const uint32_t pid = (uint32_t)mine;
    const int64_t t0 = doc_offsets[pid], t1 = doc_offsets[(int64_t)pid + 1];
    int before = 0;
#pragma unroll
    for (int u = 0; u < EACH; ++u) before += __popcll(__ballot(other[u] < mine));
    if (lane == 0) fewer[wave] = before;
    __syncthreads();
    const int rank = fewer[0] + fewer[1] + fewer[2] + fewer[3];
    if (rank >= m) return;  // uniform
    const int len = (int)(t1 - t0);
    int32_t code = 0;
    float nf = 1.0f;
    uint32_t rw[RW] = {0};
    auto request = [&](int b) {
        const int row = b + r32;  // this lane's passage token
        const int64_t tok = t0 + (row < len ? row : len - 1);
        code = codes[tok];
        if (RN) nf = inv_norm[tok];
        if (NBITS == 2) {
            const uint4 v = reinterpret_cast<const uint4 *>(residuals + tok * RB)[h];
            rw[0] = v.x, rw[1] = v.y, rw[2 % RW] = v.z, rw[3 % RW] = v.w;
        } else {
            const uint2 v = reinterpret_cast<const uint2 *>(residuals + tok * RB)[h];
            rw[0] = v.x, rw[1] = v.y;
        }
    };
    if (32 * wave < len) request(32 * wave);
    s4_build_tables<NBITS>(hlut, weights, threadIdx.x, 256);
    s4_stage_query(Q + (int64_t)q * QLEN * DIM, qs);
    __syncthreads();
    const char *Sq = reinterpret_cast<const char *>(S + (int64_t)q * C * QLEN);
    float mx[16];  // running maxima of this lane's column class: query token 8 (v / 4) + 4 h + v % 4
#pragma unroll
    for (int v = 0; v < 16; ++v) mx[v] = -INFINITY;
    for (int base = 32 * wave; base < len; base += 128) {  // uniform for the wave
        float4 sv[4];
        {
            typename std::conditional<WIDE, uint64_t, uint32_t>::type off = (uint32_t)code;
            off = off * (uint32_t)(QLEN * 4) + 16u * (uint32_t)h;
#pragma unroll
            for (int g = 0; g < 4; ++g) sv[g] = *reinterpret_cast<const float4 *>(Sq + off + 32u * g);
        }
        uint32_t now[RW];
#pragma unroll
        for (int e = 0; e < RW; ++e) now[e] = rw[e];
        const float f = nf;
        if (base + 128 < len) request(base + 128);
        floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        floatx16 acx = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};  // cross terms, scaled by 2^11
        s4_products<NBITS, false, true, 0, 0>(now, hlut, qs, nullptr, nullptr, lane, acc, acx);
        const float svf[16] = {sv[0].x, sv[0].y, sv[0].z, sv[0].w, sv[1].x, sv[1].y, sv[1].z, sv[1].w,
                               sv[2].x, sv[2].y, sv[2].z, sv[2].w, sv[3].x, sv[3].y, sv[3].z, sv[3].w};
        if (base + r32 < len) {  // this lane's column is a token of the passage
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float x = fmaf(acx[v], 1.0f / S4_SCALE, acc[v]) + svf[v];
                if (RN) x *= f;
                mx[v] = s4_max(mx[v], x);
            }
        }
    }
    const float cm = s4_column_maxima(mx, lane);  // query token s4_token_of_lane(lane), in even and odd lane alike
    if (!(lane & 1)) wmax[wave][s4_token_of_lane(lane)] = cm;
    __syncthreads();
    const float best = fmaxf(fmaxf(wmax[0][r32], wmax[1][r32]), fmaxf(wmax[2][r32], wmax[3][r32]));
    const float total = plaid_sum32_in_order(best);
    if (threadIdx.x == 0) out_keys[(int64_t)q * out_stride + rank] = plaid_make_key(len > 0 ? total : -INFINITY, pid);
}

// Many passages per wave: the tokens to score are listed in LDS, VP_GROUP passages at a time, each passage's rounded up to
// eight by repeats of its last one, and the steps of 32 tokens run over the list whatever passage a token belongs to.  Rows
// of the matrix instruction are list positions, columns query tokens: lane 32 h + n gets, for query token n, positions
// 8 g + 4 h .. + 3 of the groups of eight g = 0 .. 3, adds the rows of S_cq (two whole rows per load instruction) and keeps
// one running maximum, which goes to LDS where a passage ends; eight lanes then add up the 32 maxima of eight passages.
// Against steps of one passage each this saves the padding (a third of the steps at 20 tokens per passage, a sixth at 65),
// the exchange of maxima between lanes and a wave-wide chain of 32 additions per passage.  The next step's residuals, codes and
// tokens are requested during a step, the next group's codes before the steps of this one.
//
// FILTER = false: the passages of in_keys[q], all of their tokens (stage 4 of long launches).  The grid is laid out as in
// the kernel above.  512 queries of 256 passages: 399 us with a wave-wide step per 32 tokens of one passage and table
// entries of both terms, 344 us; 144 of 1024 543 -> 393 us.
// FILTER = true: vanilla ColBERTv2's pruning of an over-large candidate set (Section 4.1): a candidate's score from the
// embeddings of E alone, E = the tokens whose centroid was probed (probebits: bit c = centroid c probed; staged in LDS up
// to VP_LDS_WORDS words).  Queries whose candidate count does not exceed ncandidates keep every candidate and are not
// scored: their keys get score 0.  cand: [q][cand_stride] ascending candidate pids, in_counts[q] of them; out_keys[q][j] =
// key of cand[q][j].  The candidates of different queries are mostly the same passages: workgroup L takes query
// L / 8 % nq and a share of the (L % 8)-th eighth of its candidates, so that the queries read a passage at about the same
// time through the same partition's cache (16 queries: the counter of fetches, which sees half of the bytes, shows 17 GB with a
// grid column per query, 1.2 GB this way).  16 queries of 400 000 candidates: 8.4 -> 4.9 ms, of which listing the tokens takes 1.9
// (scalar and vector instructions) and the products 2.0 (matrix instructions 1.7).  The list holds a token's number itself, unless
// 32 bits do not hold that (WIDE), and its lanes are taken from the mask as it is: the pruning by coarse scores of 16 queries 3.10
// -> 2.84 ms (before: rows within the passage, and its first token per group of eight positions).  (Rows of S_cq requested a step
// ahead: 2.96 -> 3.07 ms, 144 queries of 1024 passages 414 -> 426 us; eight passages at a time: the same; a table entry per half
// byte in banks of a lane's own, so that look-ups never conflict: 3 to 5 % slower, its reads being twice as many.)
#define VP_GROUP 4
#define VP_CAP 288  // listed positions: what is left of the last list (< 32), one chunk of 64 and its padding always fit
#define VP_SLOTS 16
#define VP_LDS_WORDS 2048
#define VP_RESIDENT_BLOCKS 768
template <bool WIDE>
struct alignas(16) VpAreaOf {  // of one wave
    int32_t code[VP_CAP];
    uint32_t row[VP_CAP];       // token; WIDE: within its passage
    int32_t end[VP_CAP / 8];    // slot of the passage that ends with a group of eight positions, -1 (also in the groups not listed yet)
    int64_t base[WIDE ? VP_CAP / 8 : 1];  // WIDE: first token of a group's passage
    float sums[VP_SLOTS][QLEN + 1];
    int32_t slot_j[VP_SLOTS], slot_pid[VP_SLOTS];
};
typedef VpAreaOf<true> VpArea;
static_assert(offsetof(VpAreaOf<false>, end) % 16 == 0 && sizeof(VpAreaOf<false>) % 16 == 0, "read 16 bytes at a time");

template <int CTRL>
__device__ __forceinline__ double vp_dpp(double d)  // of another lane
{
    const uint64_t u = __builtin_bit_cast(uint64_t, d);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ void vp_sync()  // orders a wave's LDS accesses
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// RN: as above; WIDE: 2^25 centroids or 2^32 tokens are not enough.  COARSE (with FILTER): the leading products only, a third of
// the matrix instructions and half of the table look-ups; every score lies within the bound that van_bounds_kernel computes of the
// full one.
template <int NBITS, bool FILTER, bool RN, bool WIDE, bool COARSE>
__device__ __forceinline__ void maxsim_list_body(
    const float *__restrict__ Q, const float *__restrict__ S, int64_t C, const int64_t *__restrict__ doc_offsets,
    const int32_t *__restrict__ codes, const uint8_t *__restrict__ residuals, const float *__restrict__ weights,
    const float *__restrict__ inv_norm, const uint64_t *__restrict__ in_keys, int64_t in_stride,
    const uint32_t *__restrict__ probebits, int64_t keep_words, const int32_t *__restrict__ cand, int64_t cand_stride,
    const int32_t *__restrict__ in_counts, int32_t ncandidates, int nq, int gx, int spread, uint64_t *__restrict__ out_keys,
    int64_t out_stride)
{
    constexpr int RB = 16 * NBITS, RW = 2 * NBITS;
    __shared__ s4_half8 qs[COARSE ? 1 : 2][8][64];  // [term][step][lane]
    __shared__ typename S4Entry<NBITS>::type hlut[COARSE ? 256 : S4_SECOND + 256];
    __shared__ VpAreaOf<WIDE> areas[4];
    __shared__ __align__(16) float inv_norms[RN ? 4 : 1][RN ? VP_CAP : 1];
    extern __shared__ uint32_t probe_lds[];  // FILTER: keep_words words and one of zeros, when at most VP_LDS_WORDS
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int q, bx;
    if (FILTER) {
        q = (int)(blockIdx.x >> 3) % nq;
        bx = (int)(blockIdx.x >> 3) / nq;
    } else if (spread) {
        q = blockIdx.x / gx;
        bx = blockIdx.x % gx;
    } else {
        const int k = blockIdx.x >> 3;
        q = 8 * (k / gx) + (blockIdx.x & 7);
        bx = k % gx;
    }
    if (q >= nq) return;
    const int total = in_counts[q];
    const int32_t *cq = FILTER ? cand + (int64_t)q * cand_stride : nullptr;
    const uint32_t *ik = FILTER ? nullptr : reinterpret_cast<const uint32_t *>(in_keys + (int64_t)q * in_stride);  // low word: id
    uint64_t *oq = out_keys + (int64_t)q * out_stride;
    // the workgroup's passages: groups bx 4 + wave, + 4 gx, ... of [lo, count)
    int64_t lo = 0, count = total;
    if (FILTER) {
        const int64_t share = ((int64_t)total + 8 * VP_GROUP - 1) / (8 * VP_GROUP) * VP_GROUP;
        lo = share * (blockIdx.x & 7);
        if (lo + share < count) count = lo + share;
        if (total <= ncandidates) {  // (uniform) no pruning for this query
            for (int64_t j = lo + (int64_t)bx * 256 + threadIdx.x; j < count; j += (int64_t)gx * 256)
                oq[j] = plaid_make_key(0.0f, (uint32_t)cq[j]);
            return;
        }
    }
    if (lo + (int64_t)bx * 4 * VP_GROUP >= count) return;  // uniform for the workgroup
    const int r32 = lane & 31, h = lane >> 5;
    s4_build_tables<NBITS, !COARSE>(hlut, weights, threadIdx.x, 256);
    const char *Sq = reinterpret_cast<const char *>(S + (int64_t)q * C * QLEN);
    const uint32_t *pb = FILTER ? probebits + (int64_t)q * keep_words : nullptr;
    const bool pb_in_lds = FILTER && keep_words <= VP_LDS_WORDS;
    if (pb_in_lds)
        for (int w = threadIdx.x; w <= (int)keep_words; w += 256) probe_lds[w] = w < (int)keep_words ? pb[w] : 0u;
    s4_stage_query(Q + (int64_t)q * QLEN * DIM, qs);
    __syncthreads();
    // The query's operands that fit the registers beside the rest, at three waves per SIMD (COARSE: four), are read from LDS once: reads
    // of LDS, the busiest unit, bound the steps.  512 queries of 256 passages 345 us with none held, 334 with the leading terms, 329 so;
    // 144 of 1024 391, 378, 374; the coarse scores of 16 queries 2.77 ms with none, 2.70.  (All of them, at two waves: 380, 411.)
    constexpr int H1 = COARSE ? (NBITS == 2 ? 6 : 5) : 8, H2 = COARSE ? 0 : (RN ? 1 : 3);
    s4_half8 held1[H1 ? H1 : 1], held2[H2 ? H2 : 1];
#pragma unroll
    for (int s = 0; s < H1; ++s) held1[s] = qs[0][s][lane];
#pragma unroll
    for (int s = 0; s < H2; ++s) held2[s] = qs[COARSE ? 0 : 1][s][lane];
    VpAreaOf<WIDE> &A = areas[wave];
    float *anf = inv_norms[RN ? wave : 0];
    if (lane < VP_CAP / 8) A.end[lane] = -1;
    int have = 0;                                // positions listed
    int assigned = 0, completed = 0, summed = 0;  // passages listed, scored, written out
    float m = -INFINITY;                          // the running maximum of the passage at the head of the list

    typedef typename std::conditional<WIDE, int64_t, uint32_t>::type token_t;
    auto token_at = [&](int at) -> token_t {  // of position at + r32
        if constexpr (WIDE) return A.base[(at + r32) >> 3] + A.row[at + r32];
        else return A.row[at + r32];
    };
    auto request = [&](token_t tok, uint32_t (&r)[RW]) {  // this lane's half of the packed residual of a token
        if (NBITS == 2) {
            const uint4 v = reinterpret_cast<const uint4 *>(residuals + (uint64_t)tok * RB)[h];
            r[0] = v.x, r[1] = v.y, r[2 % RW] = v.z, r[3 % RW] = v.w;
        } else {
            const uint2 v = reinterpret_cast<const uint2 *>(residuals + (uint64_t)tok * RB)[h];
            r[0] = v.x, r[1] = v.y;
        }
    };
    auto codes_at = [&](int at, int4 (&cc)[4]) {  // of positions at + 8 g + 4 h .. + 3
#pragma unroll
        for (int g = 0; g < 4; ++g) cc[g] = *reinterpret_cast<const int4 *>(&A.code[at + 8 * g + 4 * h]);
    };
    auto write_out = [&](int n) {  // the next n <= 8 passages
        vp_sync();
        if constexpr (COARSE) {  // eight lanes a passage: the order of these additions is free
            const int s = (summed + (lane >> 3)) & (VP_SLOTS - 1);
            const float *v = &A.sums[s][4 * (lane & 7)];
            double d = ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
            d += vp_dpp<0xB1>(d);   // the neighbour, the other pair,
            d += vp_dpp<0x4E>(d);
            d += vp_dpp<0x141>(d);  // the other four lanes of the eight
            if ((lane & 7) == 0 && (lane >> 3) < n) oq[A.slot_j[s]] = plaid_make_key((float)d, (uint32_t)A.slot_pid[s]);
        } else if (lane < n) {
            const int s = (summed + lane) & (VP_SLOTS - 1);
            double d = 0.0;
#pragma unroll
            for (int i = 0; i < QLEN; ++i) d += (double)A.sums[s][i];
            oq[A.slot_j[s]] = plaid_make_key((float)d, (uint32_t)A.slot_pid[s]);
        }
        summed += n;
        vp_sync();
    };
    // the full steps of the list; what is left moves to its front
    auto drain = [&]() {
        vp_sync();
        int at = 0;
        uint32_t rw[RW];
        int4 cc[4], ends;
        token_t tok_next;
        if (have < 32) return;  // uniform
        request(token_at(0), rw);
        codes_at(0, cc);
        ends = *reinterpret_cast<const int4 *>(&A.end[0]);
        tok_next = token_at(have >= 64 ? 32 : 0);
        for (; have - at >= 32; at += 32) {  // uniform
            // Requested ahead of time: the residuals of the next step, and, from the list, its codes and the tokens of the one
            // after it (while this step's products leave the matrix unit)
            float sv[16];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int32_t c4[4] = {cc[g].x, cc[g].y, cc[g].z, cc[g].w};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (WIDE) sv[4 * g + v] = *reinterpret_cast<const float *>(Sq + (((uint64_t)(uint32_t)c4[v] << 7) | 4u * (uint32_t)r32));
                    else sv[4 * g + v] = *reinterpret_cast<const float *>(Sq + (((uint32_t)c4[v] << 7) | 4u * (uint32_t)r32));
                }
            }
            uint32_t rw_next[RW];
            request(tok_next, rw_next);  // (past the last step: some token of the list again, not used)
            floatx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            floatx16 acx = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};  // cross terms, scaled by 2^11
            if constexpr (COARSE) s4_leading_products<NBITS, H1>(rw, hlut, qs[0], held1, lane, acc);
            else s4_products<NBITS, true, true, H1, H2>(rw, hlut, qs, held1, held2, lane, acc, acx);
            const int32_t end[4] = {ends.x, ends.y, ends.z, ends.w};
            const int next = have - at >= 64 ? at + 32 : at;
            codes_at(next, cc);
            ends = *reinterpret_cast<const int4 *>(&A.end[next >> 3]);
            tok_next = token_at(have - at >= 96 ? at + 64 : next);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = (COARSE ? acc[4 * g + v] : fmaf(acx[4 * g + v], 1.0f / S4_SCALE, acc[4 * g + v])) + sv[4 * g + v];
                if (RN) {
                    const float4 f = *reinterpret_cast<const float4 *>(&anf[at + 8 * g + 4 * h]);
                    x[0] *= f.x, x[1] *= f.y, x[2] *= f.z, x[3] *= f.w;
                }
                m = s4_max3(m, x[0], x[1]);
                m = s4_max3(m, x[2], x[3]);
                const int slot = __builtin_amdgcn_readfirstlane(end[g]);
                if (slot >= 0) {  // uniform
                    // (The exchange needs two wait states after a vector instruction that writes its operands, and the compiler does not
                    // count those in assembly statements, such as the one that made m.  It counts its own copy of m to the second
                    // operand, which comes after that.)
                    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
                    const float mm = s4_max(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
                    if (lane < QLEN) A.sums[slot][lane] = mm;
                    m = -INFINITY;
                    ++completed;
                }
            }
#pragma unroll
            for (int e = 0; e < RW; ++e) rw[e] = rw_next[e];
        }
        {  // fewer than 32 positions, four groups, are left
            const int left = have - at;
            int32_t c = 0;
            uint32_t r = 0u;
            int64_t b = 0;
            int32_t e = -1;
            float f = 1.0f;
            if (lane < left) c = A.code[at + lane], r = A.row[at + lane];
            if (RN && lane < left) f = anf[at + lane];
            if (lane < (left + 7) >> 3) {
                if (WIDE) b = A.base[(at >> 3) + lane];
                e = A.end[(at >> 3) + lane];
            }
            vp_sync();
            if (lane < left) A.code[lane] = c, A.row[lane] = r;
            if (RN && lane < left) anf[lane] = f;
            if (WIDE && lane < (left + 7) >> 3) A.base[lane] = b;
            if (lane < VP_CAP / 8) A.end[lane] = e;
            have = left;
        }
        // at most 4 + VP_GROUP passages are listed and not written out besides these
        if (completed - summed >= 8) write_out(8);
    };

    const int64_t waves = (int64_t)gx * 4, first = (int64_t)bx * 4 + wave;
    // ids and token ranges of a group, in lanes 0 .. VP_GROUP - 1 (repeated in the others); past the end no tokens
    auto load_id = [&](int64_t g) -> int32_t {
        const int64_t j = lo + g * VP_GROUP + (lane & (VP_GROUP - 1));
        return j < count ? (FILTER ? cq[j] : (int32_t)ik[2 * j]) : -1;
    };
    // the code of a lane without a token: one whose bit is never set
    const int32_t none = pb_in_lds ? 32 * (int32_t)keep_words : -1;
    auto wanted = [&](int32_t code, int n) -> unsigned long long {  // the lanes whose token is scored, of n tokens
        if (!FILTER) return n >= 64 ? ~0ull : (n > 0 ? (1ull << n) - 1ull : 0ull);
        const uint32_t w = (uint32_t)code >> 5;
        const uint32_t bits = pb_in_lds ? probe_lds[w] : (code < 0 ? 0u : pb[w]);
        return __ballot(__builtin_amdgcn_ubfe(bits, (uint32_t)code, 1u) != 0u);
    };
    // the first two chunks of 64 codes of a group's passages
    int64_t t0[VP_GROUP];
    int len[VP_GROUP];
    int32_t c[VP_GROUP][2];
    auto request_codes = [&](int64_t o0, int64_t o1) {
#pragma unroll
        for (int k = 0; k < VP_GROUP; ++k) {
            const uint32_t lo32 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)o0, k);
            const uint32_t hi32 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)o0 >> 32), k);
            t0[k] = (int64_t)((uint64_t)hi32 << 32 | lo32);
            len[k] = __builtin_amdgcn_readlane((int)(o1 - o0), k);
#pragma unroll
            for (int u = 0; u < 2; ++u) c[k][u] = 64 * u + lane < len[k] ? codes[t0[k] + 64 * u + lane] : none;
        }
    };
    // the chain id -> token range -> codes is started two groups ahead and advanced one link per group
    int32_t pid = load_id(first), pid1 = load_id(first + waves);
    int64_t o0 = 0, o1 = 0;
    if (pid >= 0) o0 = doc_offsets[pid], o1 = doc_offsets[pid + 1];
    request_codes(o0, o1);
    for (int64_t g = first;; g += waves) {  // uniform
        const bool more = lo + g * VP_GROUP < count;
        const int32_t pid2 = load_id(g + 2 * waves);
        o0 = o1 = 0;
        if (pid1 >= 0) o0 = doc_offsets[pid1], o1 = doc_offsets[pid1 + 1];
        unsigned long long masks[VP_GROUP][2];
#pragma unroll
        for (int k = 0; k < VP_GROUP; ++k)
#pragma unroll
            for (int u = 0; u < 2; ++u) masks[k][u] = wanted(c[k][u], len[k] - 64 * u);
        int k0 = 0, src0 = 0;  // passage and chunk to go on with
        bool any = false, again;
        int32_t last_code = 0;  // of the last position listed
        uint32_t last_row = 0u;
        float last_nf = 1.0f;
        const int32_t j_lane = (int32_t)(lo + g * VP_GROUP) + lane;  // of passage `lane` of the group, whose id is in this lane
        do {
            again = false;
#pragma unroll
            for (int k = 0; k < VP_GROUP; ++k) {
                const int64_t j = lo + g * VP_GROUP + k;
                if (again || k < k0 || j >= count) continue;  // uniform
#pragma unroll 1
                for (int src = src0; src < len[k]; src += 64) {  // uniform
                    int32_t cc = src == 0 ? c[k][0] : c[k][1];
                    unsigned long long mask = src == 0 ? masks[k][0] : masks[k][1];
                    if (src >= 128) {
                        cc = src + lane < len[k] ? codes[t0[k] + src + lane] : none;
                        mask = wanted(cc, len[k] - src);
                    }
                    if (!mask) continue;
                    if (have + 72 > VP_CAP) {
                        again = true;
                        k0 = k;
                        src0 = src;
                        break;
                    }
                    const bool listed = __builtin_amdgcn_inverse_ballot_w64(mask);
                    const int n = __popcll(mask);
                    const int at = FILTER ? (int)__builtin_amdgcn_mbcnt_hi(
                                                (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)have))
                                          : have + lane;
                    const uint32_t row0 = WIDE ? (uint32_t)src : (uint32_t)t0[k] + (uint32_t)src;
                    if (listed) A.code[at] = cc, A.row[at] = row0 + (uint32_t)lane;
                    const int top = 63 - __clzll((long long)mask);
                    last_code = __builtin_amdgcn_readlane(cc, top);
                    last_row = row0 + (uint32_t)top;
                    if (RN) {
                        const float f = src + lane < len[k] ? inv_norm[t0[k] + src + lane] : 0.0f;
                        if (listed) anf[at] = f;
                        last_nf = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(f), top));
                    }
                    if constexpr (WIDE) {
                        const int o = (have >> 3) + lane;
                        if (8 * o < have + n && lane < 9) A.base[o] = t0[k];
                    }
                    have += n;
                    any = true;
                }
                if (again) continue;
                src0 = 0;
                if (!any) {  // uniform
                    if (lane == k) oq[j] = plaid_make_key(-INFINITY, (uint32_t)pid);
                    continue;
                }
                any = false;
                const int fill = -have & 7;  // repeats of the last position
                if (lane < fill) A.code[have + lane] = last_code, A.row[have + lane] = last_row;
                if (RN && lane < fill) anf[have + lane] = last_nf;
                have += fill;
                const int slot = assigned++ & (VP_SLOTS - 1);
                if (lane == k) {
                    A.end[(have >> 3) - 1] = slot;
                    A.slot_j[slot] = j_lane;
                    A.slot_pid[slot] = pid;
                }
            }
            if (!again) {  // the next group's codes, before the steps
                request_codes(o0, o1);
                pid = pid1;
                pid1 = pid2;
            }
            if (!more && have > 0) {  // the remainder, filled up to a whole step
                vp_sync();
                const int32_t lc = A.code[0];
                const uint32_t lr = A.row[0];
                const int64_t lb = WIDE ? A.base[0] : 0;
                if (have + lane < 32) A.code[have + lane] = lc, A.row[have + lane] = lr;
                if (RN && have + lane < 32) anf[have + lane] = 1.0f;
                if (WIDE && (have >> 3) + lane < 4) A.base[(have >> 3) + lane] = lb;
                have = 32;
            }
            if (have >= 32) drain();
        } while (again);
        if (!more) break;
    }
    if (completed > summed) write_out(completed - summed);
}

template <int NBITS, bool FILTER, bool RN, bool WIDE>
__global__ __launch_bounds__(256, 3) void maxsim_list_kernel(
    const float *__restrict__ Q, const float *__restrict__ S, int64_t C, const int64_t *__restrict__ doc_offsets,
    const int32_t *__restrict__ codes, const uint8_t *__restrict__ residuals, const float *__restrict__ weights,
    const float *__restrict__ inv_norm, const uint64_t *__restrict__ in_keys, int64_t in_stride,
    const uint32_t *__restrict__ probebits, int64_t keep_words, const int32_t *__restrict__ cand, int64_t cand_stride,
    const int32_t *__restrict__ in_counts, int32_t ncandidates, int nq, int gx, int spread, uint64_t *__restrict__ out_keys,
    int64_t out_stride)
{
    maxsim_list_body<NBITS, FILTER, RN, WIDE, false>(Q, S, C, doc_offsets, codes, residuals, weights, inv_norm, in_keys, in_stride, probebits,
                                                      keep_words, cand, cand_stride, in_counts, ncandidates, nq, gx, spread, out_keys,
                                                      out_stride);
}
template <int NBITS>
__global__ __launch_bounds__(256, 4) void van_coarse_kernel(
    const float *__restrict__ Q, const float *__restrict__ S, int64_t C, const int64_t *__restrict__ doc_offsets,
    const int32_t *__restrict__ codes, const uint8_t *__restrict__ residuals, const float *__restrict__ weights,
    const float *__restrict__ inv_norm, const uint64_t *__restrict__ in_keys, int64_t in_stride,
    const uint32_t *__restrict__ probebits, int64_t keep_words, const int32_t *__restrict__ cand, int64_t cand_stride,
    const int32_t *__restrict__ in_counts, int32_t ncandidates, int nq, int gx, int spread, uint64_t *__restrict__ out_keys,
    int64_t out_stride)
{
    maxsim_list_body<NBITS, true, false, false, true>(Q, S, C, doc_offsets, codes, residuals, weights, inv_norm, in_keys, in_stride, probebits,
                                                      keep_words, cand, cand_stride, in_counts, ncandidates, nq, gx, spread, out_keys,
                                                      out_stride);
}

// Pruning by coarse scores.  Most candidates lie far from the cut: scores from the leading products decide them, and only
// those within the coarse scores' error of it are scored in full.  With T the ncandidates-th best coarse score and E the largest
// difference between a coarse and a full score of the query, ncandidates full scores are >= T - E, and no more than
// ncandidates - 1 are > T + E: what has a coarse score > T + 2 E is kept, what has one < T - 2 E is not, and the rest compete by
// their full scores for the places left.
// E: of a query token's product with a residual the coarse score misses w1 . q2 + w2 . q1, w2 and q2 being what the trailing
// terms stand for: w - w1 and q - q1 rounded to fp16 at 2^11 times their size, that is by 2^-11 of themselves or, below fp16's
// normal range, by 2^-36.  (Without the latter, queries of components near 2^-36, where a trailing term can be twice what it stands
// for, had passages kept and dropped that full scores rank the other way.)  Both scores' sums of 128 products of size wmax |q| in
// fp32, and the additions of the centroid's share (at most centroid_max sum |q|), are rounded.
struct VanBand {
    float lo, hi;  // coarse scores within [lo, hi] do not decide
};
__global__ __launch_bounds__(1024) void van_bounds_kernel(const float *__restrict__ Q, const float *__restrict__ weights, int nbits,
                                                          float centroid_max, const uint64_t *__restrict__ kept, int64_t kept_stride,
                                                          const int32_t *__restrict__ n_kept, const int32_t *__restrict__ n_cand,
                                                          VanBand *__restrict__ band)
{
    __shared__ double part[16];
    __shared__ unsigned long long worst[16];
    const int q = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float wmax = 0.f, dw = 0.f;
    for (int b = 0; b < 1 << nbits; ++b) {
        _Float16 w1, w2;
        s4_split(weights[b], w1, w2);
        wmax = fmaxf(wmax, fabsf(weights[b]));
        dw = fmaxf(dw, fabsf(weights[b] - (float)w1));
    }
    double e = 0.0;
    for (int i = threadIdx.x; i < QLEN * DIM; i += 1024) {
        const float x = Q[(int64_t)q * QLEN * DIM + i];
        _Float16 x1, x2;
        s4_split(x, x1, x2);
        const double a = fabs((double)x), b = fabs((double)(float)x1);
        const double up = 1.0 + 0x1p-11;  // an fp16 number is at most this times what was rounded to it, above 2^-14
        e += up * (double)wmax * (up * fabs((double)x - (double)(float)x1) + 0x1p-36);  // |w1| <= up wmax
        e += (up * (double)dw + 0x1p-36) * b;
        e += 3.0 * 128.0 * 0x1p-24 * (double)wmax * (a + b);             // the fp32 sums of either score
        e += 0x1p-20 * (a + b) * ((double)centroid_max + (double)wmax);  // the centroid's share, the sums' last rounding
    }
    unsigned long long w = 0;  // the largest key kept: the worst
    for (int j = threadIdx.x; j < n_kept[q]; j += 1024) {
        const uint64_t key = kept[(int64_t)q * kept_stride + j];
        w = key > w ? key : w;
    }
    for (int d = 1; d < 64; d <<= 1) {
        e += __shfl_xor(e, d);
        const unsigned long long o = __shfl_xor(w, d);
        w = o > w ? o : w;
    }
    if (lane == 0) part[wave] = e, worst[wave] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < 16; ++v) {
            e += part[v];
            w = worst[v] > w ? worst[v] : w;
        }
        VanBand r;
        const float T = plaid_ord_to_score((uint32_t)(w >> 32)), E = (float)e * 2.0f * 1.00001f;  // (the factor: this product's own roundings)
        if (n_cand[q] <= n_kept[q]) r.lo = r.hi = -INFINITY;                   // (all are kept: every score is above)
        else if (!(T > -INFINITY && T < INFINITY && E < INFINITY)) r.lo = -INFINITY, r.hi = INFINITY;  // nothing is decided
        else r.lo = nextafterf(T - E, -INFINITY), r.hi = nextafterf(T + E, INFINITY);
        band[q] = r;
    }
}
// Sorts the candidates by their coarse keys: kept for sure (sure, best_stride keys of room, counted in state's n_sure), to be scored (their ids to
// open, counted in n_b), out.  One update of each counter per workgroup and 2048 keys.
__global__ __launch_bounds__(256) void van_band_kernel(const uint64_t *__restrict__ keys, int64_t key_stride, const int32_t *__restrict__ n_cand,
                                                       const VanBand *__restrict__ band, Sel2State *state, uint64_t *__restrict__ sure,
                                                       int64_t sure_stride, int32_t *__restrict__ open, int64_t open_stride)
{
    __shared__ int32_t cnt[2][4], base[2];
    const int q = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = n_cand[q];
    const VanBand b = band[q];
    const uint64_t *k = keys + (int64_t)q * key_stride;
    Sel2State *s = state + q;
    for (int64_t s0 = (int64_t)blockIdx.x * 2048; s0 < n; s0 += (int64_t)gridDim.x * 2048) {  // uniform
        uint64_t key[8];
        unsigned long long m[2][8];
        int mine[2] = {0, 0};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = s0 + 256 * u + threadIdx.x;
            key[u] = i < n ? k[i] : PLAID_KEY_MAX;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = s0 + 256 * u + threadIdx.x < n;
            const float score = plaid_ord_to_score((uint32_t)(key[u] >> 32));
            // (a score that is not a number, and an empty one where everything is kept, go with the open and the kept)
            const bool above = score > b.hi || (b.hi == -INFINITY && b.lo == -INFINITY);
            m[0][u] = __ballot(in && above);
            m[1][u] = __ballot(in && !above && !(score < b.lo));
            mine[0] += __popcll(m[0][u]);
            mine[1] += __popcll(m[1][u]);
        }
        if (lane == 0) cnt[0][wave] = mine[0], cnt[1][wave] = mine[1];
        __syncthreads();
        if (threadIdx.x < 2) {
            int t = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) t += cnt[threadIdx.x][w];
            base[threadIdx.x] = t ? atomicAdd(threadIdx.x == 0 ? &s->n_sure : &s->n_b, t) : 0;
        }
        __syncthreads();
        int at[2] = {base[0], base[1]};
        for (int w = 0; w < wave; ++w) at[0] += cnt[0][w], at[1] += cnt[1][w];
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p0 = at[0] + __popcll(m[0][u] & below), p1 = at[1] + __popcll(m[1][u] & below);
            if (((m[0][u] >> lane) & 1ull) && p0 < sure_stride) sure[(int64_t)q * sure_stride + p0] = key[u];
            if ((m[1][u] >> lane) & 1ull) open[(int64_t)q * open_stride + p1] = (int32_t)(uint32_t)key[u];
            at[0] += __popcll(m[0][u]);
            at[1] += __popcll(m[1][u]);
        }
        __syncthreads();
    }
}
// Behind the places of the open ones: the kept ones, with keys that no full score can beat.  n_open, n_all: what is to be scored, and all
// that the cut chooses from.
__global__ __launch_bounds__(256) void van_join_kernel(const Sel2State *__restrict__ state, const uint64_t *__restrict__ sure, int64_t sure_stride,
                                                       uint64_t *__restrict__ keys, int64_t key_stride, int32_t *__restrict__ n_open,
                                                       int32_t *__restrict__ n_all)
{
    const int q = blockIdx.y, open = state[q].n_b, n = state[q].n_sure < sure_stride ? state[q].n_sure : (int)sure_stride;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        n_open[q] = open;
        n_all[q] = open + n;
    }
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
        keys[(int64_t)q * key_stride + open + i] = plaid_make_key(INFINITY, (uint32_t)sure[(int64_t)q * sure_stride + i]);
}

void plaid_launch_vanilla_coarse(hipStream_t st, const float *Q, const float *S, int64_t C, const int64_t *doc_offsets,
                                 const int32_t *codes, const uint8_t *residuals, const float *bucket_weights, int nbits,
                                 const uint32_t *probebits, int64_t keep_words, int nq, const int32_t *cand, int64_t cand_stride,
                                 const int32_t *n_cand, int64_t n_upper, int32_t ncandidates, uint64_t *out_keys, int64_t out_stride)
{
    // four workgroups per compute unit, four rounds of them
    int64_t gx = (n_upper + 32 * VP_GROUP - 1) / (32 * VP_GROUP);
    const int64_t cap = (4 * 1024 + 8 * nq - 1) / (8 * nq);
    if (gx > cap) gx = cap;
    const size_t lds = keep_words <= VP_LDS_WORDS ? (size_t)keep_words * 4 + 4 : 0;
#define PLAID_VC_LAUNCH(NB)                                                                                                         \
    hipLaunchKernelGGL(van_coarse_kernel<NB>, dim3((unsigned)(8 * nq * gx)), dim3(256), lds, st, Q, S, C, doc_offsets, codes, residuals, \
                       bucket_weights, (const float *)nullptr, (const uint64_t *)nullptr, (int64_t)0, probebits, keep_words, cand,       \
                       cand_stride, n_cand, ncandidates, nq, (int)gx, 0, out_keys, out_stride)
    if (nbits == 2) PLAID_VC_LAUNCH(2);
    else PLAID_VC_LAUNCH(1);
#undef PLAID_VC_LAUNCH
}
void plaid_launch_vanilla_band(hipStream_t st, const float *Q, const float *bucket_weights, int nbits, float centroid_max, int nq, int64_t P,
                               uint64_t *kept, int64_t kept_stride, const int32_t *n_kept, int32_t *n_cand, uint64_t *keys,
                               int64_t key_stride, void *band, Sel2State *state, int32_t *open, int64_t open_stride, int32_t *n_open)
{
    hipLaunchKernelGGL(van_bounds_kernel, dim3(nq), dim3(1024), 0, st, Q, bucket_weights, nbits, centroid_max, kept, kept_stride, n_kept,
                       n_cand, (VanBand *)band);
    const int64_t parts = (P + 2047) / 2048, most = nq >= 16 ? 64 : (nq >= 4 ? 256 : 1024);
    hipLaunchKernelGGL(van_band_kernel, dim3((unsigned)(parts < most ? parts : most), nq), dim3(256), 0, st, keys, key_stride, n_cand,
                       (const VanBand *)band, state, kept, kept_stride, open, open_stride);
    const int64_t joins = (kept_stride + 1023) / 1024;
    hipLaunchKernelGGL(van_join_kernel, dim3((unsigned)(joins < 64 ? joins : 64), nq), dim3(256), 0, st, state, kept, kept_stride, keys, key_stride,
                       n_open, n_cand);
}

void plaid_launch_vanilla_prune(hipStream_t st, const float *Q, const float *S, int64_t C, int64_t N, const int64_t *doc_offsets,
                                const int32_t *codes, const uint8_t *residuals, const float *bucket_weights, int nbits,
                                const uint32_t *probebits, int64_t keep_words, int nq, const int32_t *cand, int64_t cand_stride,
                                const int32_t *n_cand, int64_t n_upper, int32_t ncandidates, uint64_t *out_keys,
                                int64_t out_stride)
{
    if (n_upper <= 0 || nq <= 0) return;
    // three workgroups per compute unit, four rounds of them; at least a workgroup per query and eighth
    int64_t gx = (n_upper + 32 * VP_GROUP - 1) / (32 * VP_GROUP);
    const int64_t cap = (4 * VP_RESIDENT_BLOCKS + 8 * nq - 1) / (8 * nq);
    if (gx > cap) gx = cap;
    const size_t lds = keep_words <= VP_LDS_WORDS ? (size_t)keep_words * 4 + 4 : 0;
#define PLAID_VP_LAUNCH(NB, WIDE)                                                                                              \
    hipLaunchKernelGGL((maxsim_list_kernel<NB, true, false, WIDE>), dim3((unsigned)(8 * nq * gx)), dim3(256), lds, st, Q, S, C, \
                       doc_offsets, codes, residuals, bucket_weights, (const float *)nullptr, (const uint64_t *)nullptr,       \
                       (int64_t)0, probebits, keep_words, cand, cand_stride, n_cand, ncandidates, nq, (int)gx, 0, out_keys,     \
                       out_stride)
    const bool wide = plaid_wide(C, N);
    if (nbits == 2) {
        if (wide) PLAID_VP_LAUNCH(2, true);
        else PLAID_VP_LAUNCH(2, false);
    } else {
        if (wide) PLAID_VP_LAUNCH(1, true);
        else PLAID_VP_LAUNCH(1, false);
    }
#undef PLAID_VP_LAUNCH
}

// Many passages (48 per workgroup of a full chip, three per compute unit) in lists of some length: steps packed across passages, 32
// passages per workgroup.  512 queries of 256 passages 374 -> 344 us (48, 64, 128 per workgroup: 381, 362, 390), 144 of 1024 488 -> 393
// us (421, 401, 438).  Fewer passages: a wave's list of four leaves too few waves (256 queries of 64 48 -> 50 us, 23 of 250 25 -> 46 us,
// 40 of 256 41 -> 49; from about 20 000 on little depends on it: 80 of 256 75 -> 70, 320 of 64 74 -> 72).  Short lists: the remainder of
// each wave's list is filled up to a whole step, and a query has two workgroups that end together.  us of a launch with a passage at a
// time / packed, 30 to 90 tokens and 8 to 180 with unit-length reconstruction, 512 queries: lists of 72 103 / 115, of 96 133 / 130 and
// 159 / 167, of 128 162 / 157 and 193 / 199, of 192 234 / 224 and 281 / 285; 384 queries: of 96 115 / 108 and 134 / 139, of 128 140 / 119
// and 162 / 153.
static constexpr bool s4_packed(int n_upper, int nq) { return n_upper >= 96 && (int64_t)n_upper * nq >= 48ll * VP_RESIDENT_BLOCKS; }

// Whether the cut of lists of up to n_upper keys and the scores of the m best are one launch: the workgroups that only count and leave are
// three of four, each of which reads its query's whole list, so the launch is bound by them from some 8000 keys on, a few for each place
// of the chip.  Whole searches in us, as one launch and as two, with 1024 keys a query of 400 000 passages: 4 queries 97 / 102, 8 queries 115 /
// 120, 12 queries 144 / 138, 31 queries 276 / 244; 40 000 passages: 6 queries 80 / 85, 12 queries 101 / 91, 31 queries 151 / 119; 256 keys a
// query of 200 000 passages: 12 queries 83 / 88, 31 queries 122 / 129, 40 queries 141 / 135, 96 queries 245 / 224.
static constexpr bool s4_cuts(int n_upper, int nq) { return n_upper <= CUT_KEYS && (int64_t)n_upper * nq <= 8192; }
bool plaid_cut_with_scores(int n_upper, int nq) { return n_upper > 0 && nq > 0 && s4_cuts(n_upper, nq); }
void plaid_launch_cut_maxsim(hipStream_t st, const float *Q, const float *S, int64_t C, int64_t N, const int64_t *doc_offsets, const int32_t *codes,
                             const uint8_t *residuals, const float *bucket_weights, int nbits, int nq, const uint64_t *in_keys,
                             int64_t in_stride, const int32_t *in_counts, int n_upper, int32_t m, uint64_t *out_keys, int64_t out_stride,
                             int32_t *out_counts, const float *inv_norm)
{
    const bool wide = plaid_wide(C, N);
#define PLAID_S4_CUT(NB, RN, WIDE)                                                                                              \
    hipLaunchKernelGGL((cut_maxsim_kernel<NB, RN, WIDE>), dim3((unsigned)n_upper, (unsigned)nq), dim3(256), 0, st, Q, S, C,        \
                       doc_offsets, codes, residuals, bucket_weights, inv_norm, in_keys, in_stride, in_counts, m, out_keys,       \
                       out_stride, out_counts)
#define PLAID_S4_CUTS(NB)                                  \
    do {                                                   \
        if (inv_norm && wide) PLAID_S4_CUT(NB, true, true); \
        else if (inv_norm) PLAID_S4_CUT(NB, true, false);   \
        else if (wide) PLAID_S4_CUT(NB, false, true);       \
        else PLAID_S4_CUT(NB, false, false);                \
    } while (0)
    if (nbits == 2) PLAID_S4_CUTS(2);
    else PLAID_S4_CUTS(1);
#undef PLAID_S4_CUTS
#undef PLAID_S4_CUT
}

void plaid_launch_decompress_maxsim(hipStream_t st, const float *Q, const float *S, int64_t C, int64_t N, const int64_t *doc_offsets,
                                    const int32_t *codes, const uint8_t *residuals, const float *bucket_weights,
                                    int nbits, int nq, const uint64_t *in_keys, int64_t in_stride,
                                    const int32_t *in_counts, int n_upper, uint64_t *out_keys, int64_t out_stride,
                                    const float *inv_norm)
{
    if (n_upper <= 0 || nq <= 0) return;
    // Few passages in all (short lists of few queries): a workgroup per passage.  Otherwise waves stride over the lists,
    // several passages each, so that the per-workgroup set-up (table, query operands) is paid rarely.
    const int64_t all = (int64_t)n_upper * nq;
    const bool coop = all <= 2048, pack = s4_packed(n_upper, nq);
    int gx = coop ? n_upper : (pack ? (n_upper + 31) / 32 : (n_upper + 3) / 4);
    // (256 compute units x 4 resident workgroups: one full round of waves, each striding over several passages)
    const int cap = coop ? 2048 : (S4_RESIDENT_BLOCKS + nq - 1) / nq;
    if (!pack && gx > cap) gx = cap;
    const int spread = nq < 8 ? 1 : 0;
    const int64_t slots = spread ? nq : 8 * (((int64_t)nq + 7) / 8);  // query slots of the one-dimensional grid
    if (slots * gx > (1ll << 23)) gx = (int)((1ll << 23) / slots);  // (the waves stride over longer lists)
    if (gx < 1) gx = 1;
    const bool wide = plaid_wide(C, N);
#define PLAID_S4_LAUNCH(NB, CO, RN, WIDE)                                                                                 \
    hipLaunchKernelGGL((decompress_maxsim_kernel<NB, CO, RN, WIDE>), dim3((unsigned)(slots * gx)), dim3(256), 0, st, Q, S, C,      \
                       doc_offsets, codes, residuals, bucket_weights, inv_norm, in_keys, in_stride, in_counts, nq, gx,       \
                       spread, out_keys, out_stride)
#define PLAID_S4_PACK(NB, RN, WIDE)                                                                                          \
    hipLaunchKernelGGL((maxsim_list_kernel<NB, false, RN, WIDE>), dim3((unsigned)(slots * gx)), dim3(256), 0, st, Q, S, C,    \
                       doc_offsets, codes, residuals, bucket_weights, inv_norm, in_keys, in_stride, (const uint32_t *)nullptr,\
                       (int64_t)0, (const int32_t *)nullptr, (int64_t)0, in_counts, 0, nq, gx, spread, out_keys, out_stride)
#define PLAID_S4_FORMS(NB, RN, WIDE)                              \
    do {                                                          \
        if (pack) PLAID_S4_PACK(NB, RN, WIDE);                    \
        else if (coop) PLAID_S4_LAUNCH(NB, true, RN, WIDE);       \
        else PLAID_S4_LAUNCH(NB, false, RN, WIDE);                \
    } while (0)
#define PLAID_S4_WIDTHS(NB, RN)                                   \
    do {                                                          \
        if (wide) PLAID_S4_FORMS(NB, RN, true);                   \
        else PLAID_S4_FORMS(NB, RN, false);                       \
    } while (0)
    if (nbits == 2) {
        if (inv_norm) PLAID_S4_WIDTHS(2, true);
        else PLAID_S4_WIDTHS(2, false);
    } else {
        if (inv_norm) PLAID_S4_WIDTHS(1, true);
        else PLAID_S4_WIDTHS(1, false);
    }
#undef PLAID_S4_WIDTHS
#undef PLAID_S4_FORMS
#undef PLAID_S4_PACK
#undef PLAID_S4_LAUNCH
}

// ------------------------------------------------------------------ decompression alone (parity of the codec)
// Token counts of the listed passages, a passage per thread, to lens, and their prefix sums by the workgroup that arrives last.
// A lane's address each is what a gather of token ranges costs (one compute unit alone takes 15 us for 5000 of them), so a workgroup has
// OFFS_EACH of them until there is one per compute unit.  The rest is a chain: the lengths back from memory, six steps of a wave's sum
// (a thread's four passages are consecutive, so there is one such sum and not four), the waves' sums, the report.  5000 passages: 13.6 us
// with 1024 to a workgroup, four sums a wave and a report that wrote back the L2 first, 8.9 us so; a whole call 77.7 -> 72.8 us, of
// 50 passages 33.0 -> 30.6 us.
// The ids are the caller's: nothing is read by one out of range, and out_offsets is left alone where there is one.  A list
// with such an id, or of more tokens than capacity, leaves its ticket in *refused: the decompression kernel behind this one
// does nothing then.  lens, work and refused are the library's, so that no write to the caller's buffers gets a refused list
// past that.  work (two words, zero before and after): workgroups arrived, and how far from the list's end the first id out of
// range is.  report (memory of the host, which waits for the last word): total, place of that id or -1, the id, 1.
#define OFFS_THREADS 1024
#define OFFS_PER 4
#define OFFS_EACH 64
__global__ __launch_bounds__(OFFS_THREADS) void passage_offsets_kernel(const int64_t *__restrict__ doc_offsets, int64_t P,
                                                                       const int32_t *__restrict__ pids, int n, int64_t *lens,
                                                                       int64_t *__restrict__ out_offsets, int64_t capacity, uint32_t *work,
                                                                       int64_t *refused, int64_t ticket, int64_t *report)
{
    __shared__ int64_t wave_sum[OFFS_THREADS / 64];
    __shared__ uint32_t arrived;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t each = ((int64_t)n + gridDim.x - 1) / gridDim.x, end = ((int64_t)blockIdx.x + 1) * each < n ? ((int64_t)blockIdx.x + 1) * each : n;
    for (int64_t e = (int64_t)blockIdx.x * each + threadIdx.x; e < end; e += OFFS_THREADS) {
        const int32_t pid = pids[e];
        int64_t len = 0;
        if ((uint64_t)(int64_t)pid < (uint64_t)P) len = doc_offsets[(int64_t)pid + 1] - doc_offsets[pid];
        else atomicMax(&work[1], (uint32_t)(n - e));
        __hip_atomic_store(&lens[e], len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);  // this wave's stores and updates have completed
    __syncthreads();
    if (threadIdx.x == 0) arrived = __hip_atomic_fetch_add(&work[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived != gridDim.x - 1) return;  // uniform
    const uint32_t bad = __hip_atomic_load(&work[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int64_t carry = 0;  // the same in every thread
    if (!bad) {         // uniform
        if (threadIdx.x == 0) out_offsets[0] = 0;
        for (int64_t base = 0; base < n; base += OFFS_THREADS * OFFS_PER) {
            // a thread's passages are consecutive
            const int64_t e0 = base + OFFS_PER * threadIdx.x;
            int64_t incl[OFFS_PER];
#pragma unroll
            for (int u = 0; u < OFFS_PER; ++u)
                incl[u] = e0 + u < n ? __hip_atomic_load(&lens[e0 + u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
#pragma unroll
            for (int u = 1; u < OFFS_PER; ++u) incl[u] += incl[u - 1];
            int64_t sum = incl[OFFS_PER - 1];  // of this lane's and the lanes' before it
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t t = __shfl_up(sum, d);
                if (lane >= d) sum += t;
            }
            if (lane == 63) wave_sum[wave] = sum;
            __syncthreads();
            int64_t run = carry + sum - incl[OFFS_PER - 1];
#pragma unroll
            for (int w = 0; w < OFFS_THREADS / 64; ++w) {
                const int64_t t = wave_sum[w];
                if (w < wave) run += t;
                carry += t;
            }
#pragma unroll
            for (int u = 0; u < OFFS_PER; ++u)
                if (e0 + u < n) out_offsets[e0 + u + 1] = run + incl[u];
            __syncthreads();  // the sums are written again in the next round
        }
    }
    if (threadIdx.x == 0) {
        // each word is written through by itself and has arrived before the last one leaves (a release would write back the whole L2)
        if (bad || carry > capacity) __hip_atomic_store(refused, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&work[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&work[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&report[0], carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&report[1], bad ? (int64_t)n - bad : (int64_t)-1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&report[2], bad ? (int64_t)pids[n - bad] : (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        __hip_atomic_store(&report[3], (int64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}
void plaid_launch_passage_offsets(hipStream_t st, const int64_t *doc_offsets, int64_t P, const int32_t *pids, int n, int64_t *lens,
                                  int64_t *out_offsets, int64_t capacity, uint32_t *work, int64_t *refused, int64_t ticket,
                                  int64_t *report)
{
    const int64_t groups = ((int64_t)n + OFFS_EACH - 1) / OFFS_EACH;
    const unsigned grid = groups < 1 ? 1u : groups > 256 ? 256u : (unsigned)groups;
    hipLaunchKernelGGL(passage_offsets_kernel, dim3(grid), dim3(OFFS_THREADS), 0, st, doc_offsets, P, pids, n, lens, out_offsets,
                       capacity, work, refused, ticket, report);
}

// Same table, same lookup and same addition as the fused kernel; a workgroup per passage, a token to 32 threads, 4 dimensions each.
// Bound by its writes and by the centroid rows, 512 bytes a token each.
// Threads of a workgroup: twice as many fetch twice the rows of a long passage at once, but leave fewer passages in flight on a compute
// unit, and what a list's passages are like does not follow from the collection's mean.  us per call with 256 / 512, lists of 50 000
// passages: of 1 to 8 tokens 96 / 125, of 8 to 24 133 / 196, of 24 to 40 290 / 329, of 30 to 100 610 / 596 (of 262 144 centroids 637 /
// 653); of 5000: 23 / 23, 23 / 27, 31 / 31, 51 / 54; 1000 of 100 to 300 36 / 38; 100 of 1000 to 3000, which are too few passages to fill
// the chip, 148 / 94.
#define DUMP_THREADS 256
// Whether what is written goes past the caches (nontemporal stores).  Then they hold more of the rows and codes, but whoever reads the
// vectors next finds none of them there; where they do not fit the 256 MB of the last cache, most would be gone anyway.  Passages of 65
// tokens, vectors and indices, us of a call alone / of the call and a sum over the vectors / of the call and their product with 32 columns,
// through the caches and past them, lists that are not seen again soon: 1000 (42 MB) 23.1, 38.5, 45.2 and 21.3, 41.2, 48.1; 2000 34.7,
// 54.7, 61.1 and 33.4, 60.6, 66.0; 5000 (208 MB) 70.4, 106, 123 and 70.3, 123, 130; 6000 (250 MB) 82.8, 133, 151 and 82.1, 144, 153; 8000
// (333 MB) 118, 197, 210 and 106, 185, 199; 50 000 656, 1084, 1140 and 610, 1054, 1113.  Eight lists of 5000 in turn, whose codes and rows
// the caches can hold: 71.7, 111, 129 and 50.6, 124, 134.
static constexpr __host__ __device__ bool s4_past_caches(int64_t tokens, bool vectors, bool indices)
{
    return tokens * ((vectors ? DIM * 4 : 0) + (indices ? DIM : 0)) > (256ll << 20);
}
typedef float s4_float4 __attribute__((ext_vector_type(4)));
template <bool PAST, typename T, typename U>
__device__ __forceinline__ void s4_store(T value, U *to)
{
    if (PAST) __builtin_nontemporal_store(value, reinterpret_cast<T *>(to));
    else *reinterpret_cast<T *>(to) = value;
}
template <int NBITS>
__global__ __launch_bounds__(DUMP_THREADS) void decompress_dump_kernel(const float *__restrict__ centroids,
                                                                       const int64_t *__restrict__ doc_offsets,
                                                                       const int32_t *__restrict__ codes,
                                                                       const uint8_t *__restrict__ residuals,
                                                                       const float *__restrict__ weights,
                                                                       const int32_t *__restrict__ pids,
                                                                       const int64_t *__restrict__ out_offsets,
                                                                       float *__restrict__ out_vectors,
                                                                       uint8_t *__restrict__ out_indices,
                                                                       const float *__restrict__ inv_norm,
                                                                       const int64_t *refused, int64_t ticket)
{
    constexpr int RB = 16 * NBITS, ROWS = DUMP_THREADS / 32;
    __shared__ float4 wlut[256 * (NBITS == 2 ? 1 : 2)];
    __shared__ uint32_t ilut[256 * (NBITS == 2 ? 1 : 2)];
    // (uniform) refused by passage_offsets_kernel; another call that is refused meanwhile leaves another ticket
    if (*refused == ticket) return;
    build_tables<NBITS>(wlut, ilut, weights, threadIdx.x, DUMP_THREADS);
    __syncthreads();
    const int a = blockIdx.x;
    const int32_t pid = pids[a];
    const int64_t t0 = doc_offsets[pid];
    const int len = (int)(doc_offsets[pid + 1] - t0);
    const int64_t o0 = out_offsets[a];
    const int quad = threadIdx.x & 31;
    // Four rows per thread in flight: code and residual, then the centroid's piece, then the stores.  (A loop for either kind of store: of
    // two that differ in nothing else, on two sides of a branch, the compiler makes one of the plain kind.)
    auto decode = [&](auto past) {
        for (int row0 = threadIdx.x >> 5; row0 < len; row0 += 4 * ROWS) {
            int slot[4];
            int32_t code[4];
            float4 c[4];
            float f[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int row = row0 + ROWS * u < len ? row0 + ROWS * u : row0;  // (a row past the end repeats the first)
                code[u] = codes[t0 + row];
                slot[u] = table_slot<NBITS>(residuals + (t0 + row) * RB, quad);
                f[u] = inv_norm ? inv_norm[t0 + row] : 1.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = *reinterpret_cast<const float4 *>(centroids + (int64_t)code[u] * DIM + 4 * quad);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int row = row0 + ROWS * u;
                if (row >= len) break;
                const float4 w = wlut[slot[u]];
                if (out_vectors) {
                    float4 d = make_float4(c[u].x + w.x, c[u].y + w.y, c[u].z + w.z, c[u].w + w.w);
                    // scaled to unit length: one fp32 factor per token, one rounding per component
                    if (inv_norm) d = make_float4(d.x * f[u], d.y * f[u], d.z * f[u], d.w * f[u]);
                    s4_store<decltype(past)::value>(s4_float4{d.x, d.y, d.z, d.w}, out_vectors + (o0 + row) * DIM + 4 * quad);
                }
                if (out_indices) s4_store<decltype(past)::value>(ilut[slot[u]], out_indices + (o0 + row) * DIM + 4 * quad);
            }
        }
    };
    if (s4_past_caches(out_offsets[gridDim.x], out_vectors, out_indices)) decode(std::true_type{});  // uniform
    else decode(std::false_type{});
}
void plaid_launch_decompress_dump(hipStream_t st, const float *centroids, const int64_t *doc_offsets,
                                  const int32_t *codes, const uint8_t *residuals, const float *bucket_weights,
                                  int nbits, const int32_t *pids, int n, const int64_t *out_offsets, float *out_vectors,
                                  uint8_t *out_indices, const float *inv_norm, const int64_t *refused, int64_t ticket)
{
    if (n <= 0) return;
    if (nbits == 2)
        hipLaunchKernelGGL(decompress_dump_kernel<2>, dim3(n), dim3(DUMP_THREADS), 0, st, centroids, doc_offsets, codes, residuals,
                           bucket_weights, pids, out_offsets, out_vectors, out_indices, inv_norm, refused, ticket);
    else
        hipLaunchKernelGGL(decompress_dump_kernel<1>, dim3(n), dim3(DUMP_THREADS), 0, st, centroids, doc_offsets, codes, residuals,
                           bucket_weights, pids, out_offsets, out_vectors, out_indices, inv_norm, refused, ticket);
}

// Storage variant "reconstructed vectors scaled to unit length" (the other reading of Section 4.5's reconstruction):
// inv_norm[t] = fl32(1 / sqrt(sum_x fl32(centroid[code_t][x] + weight[index(t, x)])^2)), the squares (exact in double)
// added in double in index order; 0 for a zero vector.  One thread per token; run once, when the variant is switched on.
template <int NBITS>
__global__ __launch_bounds__(256) void token_inv_norm_kernel(const float *__restrict__ centroids,
                                                             const int32_t *__restrict__ codes,
                                                             const uint8_t *__restrict__ residuals,
                                                             const float *__restrict__ weights, int64_t N,
                                                             float *__restrict__ inv_norm)
{
    constexpr int RB = 16 * NBITS;
    __shared__ float4 wlut[256 * (NBITS == 2 ? 1 : 2)];
    build_tables<NBITS>(wlut, nullptr, weights, threadIdx.x, 256);
    __syncthreads();
    for (int64_t tok = (int64_t)blockIdx.x * 256 + threadIdx.x; tok < N; tok += (int64_t)gridDim.x * 256) {
        const float *crow = centroids + (int64_t)codes[tok] * DIM;
        const uint8_t *r = residuals + tok * RB;
        double n2 = 0.0;
        for (int quad = 0; quad < DIM / 4; ++quad) {
            const float4 c = *reinterpret_cast<const float4 *>(crow + 4 * quad);
            const float4 w = wlut[table_slot<NBITS>(r, quad)];
            const float d0 = c.x + w.x, d1 = c.y + w.y, d2 = c.z + w.z, d3 = c.w + w.w;
            n2 = fma((double)d0, (double)d0, n2);
            n2 = fma((double)d1, (double)d1, n2);
            n2 = fma((double)d2, (double)d2, n2);
            n2 = fma((double)d3, (double)d3, n2);
        }
        inv_norm[tok] = n2 > 0.0 ? (float)(1.0 / sqrt(n2)) : 0.0f;
    }
}
void plaid_launch_token_inv_norm(hipStream_t st, const float *centroids, const int32_t *codes, const uint8_t *residuals,
                                 const float *bucket_weights, int nbits, int64_t N, float *inv_norm)
{
    if (N <= 0) return;
    int64_t g = (N + 255) / 256;
    if (g > 65536) g = 65536;
    if (nbits == 2)
        hipLaunchKernelGGL(token_inv_norm_kernel<2>, dim3((unsigned)g), dim3(256), 0, st, centroids, codes, residuals,
                           bucket_weights, N, inv_norm);
    else
        hipLaunchKernelGGL(token_inv_norm_kernel<1>, dim3((unsigned)g), dim3(256), 0, st, centroids, codes, residuals,
                           bucket_weights, N, inv_norm);
}
