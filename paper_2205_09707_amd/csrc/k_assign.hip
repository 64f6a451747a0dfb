// Nearest centroids (Section 3.1: code = argmax_c C[c] . x, ties to the smaller id) by screening: ONE product of fp16
// roundings on the matrix instruction proves nearly every vector's winner, and the few vectors it leaves open are decided
// by the double-precision dot products of the rows that can still win.  The result is the exact one for every input.
//
// With c1 = fp16(c), x1 = fp16(x) and residuals dc = c - c1, dx = x - x1:
//     |c.x - c1.x1| = |dc.x + c1.dx| <= |dc| |x| + |c1| |dx|            (Cauchy-Schwarz)
// the norms are those of the actual residuals (measured, not assumed: whatever fp16 cannot hold, flushed small values
// and overflow included, is in them), the largest over the centroids and the vector's own.  The fp32 accumulation of the
// 128 products (128 * 2^-23 |c1| |x1|) and the row number kept in a score's seven lowest bits (2^-16 of it) come on top.
// Call the sum e: a row whose screened score is more than 2 e below the best one cannot be the winner.
//
// Bound by the matrix unit: 2 * 128 * C flop per vector, a third of what scores good enough to be used as such take
// (three products, k_scq16.hip).  585 000 vectors against 32 768 centroids: the scores 12.4 ms and the choice among 32 rows
// by double-precision products 2.5 ms that way.
#include "plaid_internal.h"

#include <math.h>

typedef _Float16 asg_half8 __attribute__((ext_vector_type(8)));
typedef float asg_floatx16 __attribute__((ext_vector_type(16)));

#define ASG_THREADS 256
#define ASG_WAVES (ASG_THREADS / 64)
#define ASG_NT 4                            // 32-row tiles per wave
#define ASG_ROWS (32 * ASG_NT)              // rows whose best two scores a wave reports per vector
#define ASG_STEPS (DIM / 16)
#define ASG_TILE_VEC (ASG_STEPS * 64)       // 16-byte operand vectors per tile of 32 rows
#define ASG_MIN_NORMAL 6.103515625e-05f     // 2^-14: smaller components are taken as zero

__device__ __forceinline__ _Float16 asg_round(float a) { return fabsf(a) >= ASG_MIN_NORMAL ? (_Float16)a : (_Float16)0.0f; }

// dst[tile][step][lane] = operand of v_mfma_f32_32x32x16_f16: row 32 tile + (lane & 31), dimensions 16 step + 8 (lane / 32)
// and the seven that follow.  Rows at or past n_rows are zero.
__global__ __launch_bounds__(256) void asg_operands_kernel(const float *__restrict__ src, int64_t n_rows, int64_t n_tiles,
                                                           asg_half8 *__restrict__ dst)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_tiles * ASG_TILE_VEC; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = e / ASG_TILE_VEC * 32 + (e & 31);
        const int k0 = 16 * ((int)(e >> 6) & (ASG_STEPS - 1)) + 8 * ((int)(e >> 5) & 1);
        asg_half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (row < n_rows) {
            const float4 *p = reinterpret_cast<const float4 *>(src + row * DIM + k0);
            const float4 a = p[0], b = p[1];
            v = asg_half8{asg_round(a.x), asg_round(a.y), asg_round(a.z), asg_round(a.w),
                          asg_round(b.x), asg_round(b.y), asg_round(b.z), asg_round(b.w)};
        }
        dst[e] = v;
    }
}

// stats[0] = largest |component|, [1] = largest squared norm of a row's residual, [2] = of its fp16 part, as bit patterns
// (non-negative floats order like their bits; what is not a number counts as infinite).  Zero on entry.  A row per wave.
__global__ __launch_bounds__(256) void asg_stats_kernel(const float *__restrict__ c, int64_t C, uint32_t *__restrict__ stats)
{
    __shared__ float best[3][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float m0 = 0.f, m1 = 0.f, m2 = 0.f;
    for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < C; r += (int64_t)gridDim.x * 4) {
        const float2 v = *reinterpret_cast<const float2 *>(c + r * DIM + 2 * lane);
        const float a = (float)asg_round(v.x), b = (float)asg_round(v.y), da = v.x - a, db = v.y - b;
        float top = fmaxf(fabsf(v.x), fabsf(v.y)), d2 = da * da + db * db, s2 = a * a + b * b;
        if (!(v.x == v.x) || !(v.y == v.y)) top = INFINITY;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            top = fmaxf(top, __shfl_xor(top, d));
            d2 += __shfl_xor(d2, d);
            s2 += __shfl_xor(s2, d);
        }
        m0 = fmaxf(m0, top);
        m1 = d2 == d2 ? fmaxf(m1, d2) : INFINITY;
        m2 = s2 == s2 ? fmaxf(m2, s2) : INFINITY;
    }
    if (lane == 0) {
        best[0][wave] = m0;
        best[1][wave] = m1;
        best[2][wave] = m2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const float *b = best[threadIdx.x];
        atomicMax(&stats[threadIdx.x], __float_as_uint(fmaxf(fmaxf(b[0], b[1]), fmaxf(b[2], b[3]))));
    }
}

// LDS-only barrier: the operands requested for the next group but one stay in flight across it.
__device__ __forceinline__ void asg_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Grid: x = block of 512 centroids, y = range of qg groups of 32 vectors.  A wave keeps the operands of its 128 rows in
// registers (four tiles: each operand of a group read from LDS feeds four matrix instructions) and walks the groups, whose
// 8 KB of operands pass through LDS, double-buffered.  Per group it reports, for every vector, its best row's score --
// with the row's number in the seven lowest bits -- and the second best one: three vector instructions per score, between the matrix
// instructions of the same wave: the scores of two tiles while the products of the other two are formed, eight vector
// instructions (of 4 cycles) to a matrix instruction (of 32).  117 000 vectors against 32 768 centroids 986 us with the choice after a
// group's products, where only the other wave's hide it, 917 this way.  best2[group][ceil(C / 128)][32].
template <bool WHOLE>
__device__ __forceinline__ void asg_screen_body(asg_half8 (&Bs)[2][ASG_TILE_VEC], const asg_half8 *__restrict__ A, int64_t C,
                                                int64_t tile0, const asg_half8 *__restrict__ B, int g_begin, int g_end,
                                                float2 *__restrict__ best2, int64_t n_blk)
{
    constexpr int NPRE = ASG_TILE_VEC / ASG_THREADS;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
    asg_half8 pre[NPRE];
    const asg_half8 *src = B + (int64_t)g_begin * ASG_TILE_VEC + tid;
#pragma unroll
    for (int k = 0; k < NPRE; ++k) pre[k] = src[k * ASG_THREADS];
    asg_half8 a[ASG_NT][ASG_STEPS];
#pragma unroll
    for (int t = 0; t < ASG_NT; ++t)
#pragma unroll
        for (int s = 0; s < ASG_STEPS; ++s) a[t][s] = A[(tile0 + t) * ASG_TILE_VEC + s * 64 + lane];
#pragma unroll
    for (int k = 0; k < NPRE; ++k) Bs[0][tid + k * ASG_THREADS] = pre[k];
    if (g_begin + 1 < g_end) {
        src += ASG_TILE_VEC;
#pragma unroll
        for (int k = 0; k < NPRE; ++k) pre[k] = src[k * ASG_THREADS];
    }
    asg_lds_barrier();
    const int64_t blk = tile0 / ASG_NT;
    const int rows = C - tile0 * 32 < ASG_ROWS ? (int)(C - tile0 * 32) : ASG_ROWS;  // (not positive: a block past the end)
    // A maximum is the median with infinity, in a register the compiler knows nothing of: fmaxf costs a canonicalising instruction for an
    // operand that was not computed as a float.  (A score that is not a number or infinite comes from a vector whose bound is not finite
    // either, and every row of such a vector is looked at whatever is reported here.)
    float inf;
    asm volatile("s_mov_b32 %0, 0x7f800000" : "=s"(inf));
    asg_floatx16 acc[ASG_NT];
#pragma unroll
    for (int t = 0; t < ASG_NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    float m1 = -INFINITY, m2 = -INFINITY;
    // the matrix work of tiles half, half + 1 for a group, with the choice among the scores of the other two tiles between its instructions
    auto step = [&](const asg_half8 *buf, auto half_) {
        constexpr int half = decltype(half_)::value, other = 2 - half;
        int lim = rows - 4 * h;
        if (!WHOLE) asm volatile("" : "+v"(lim));  // or 64 lane masks would be formed ahead of the loop and kept
        asg_floatx16 n[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) n[t][v] = 0.f;
#pragma unroll
        for (int s = 0; s < ASG_STEPS; ++s) {
            const asg_half8 b = buf[s * 64 + lane];
#pragma unroll
            for (int t = 0; t < 2; ++t) n[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[half + t][s], b, n[t], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int t = other + u;
            float t1 = -INFINITY, t2 = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v >> 2) + (v & 3);  // row 32 t + r + 4 h of the block
                float x = __uint_as_float((__float_as_uint(acc[t][v]) & ~127u) | (uint32_t)r);
                if (!WHOLE && 32 * t + r >= lim) x = -INFINITY;
                t2 = __builtin_amdgcn_fmed3f(t1, t2, x);
                t1 = __builtin_amdgcn_fmed3f(t1, x, inf);
            }
            if (t1 > -INFINITY) t1 = __uint_as_float(__float_as_uint(t1) | (uint32_t)(32 * t));
            m2 = fmaxf(fmaxf(m2, t2), fminf(m1, t1));
            m1 = fmaxf(m1, t1);
        }
        asm volatile("" : "+v"(m1), "+v"(m2));  // (here, or the choice sinks below to where its result is used)
        __builtin_amdgcn_sched_barrier(0);
        acc[half] = n[0];
        acc[half + 1] = n[1];
    };
    auto finish = [&]() {  // m1, m2: over both halves of the wave
        if (m1 > -INFINITY) m1 = __uint_as_float(__float_as_uint(m1) | (uint32_t)(4 * h));
        const float o1 = __shfl_xor(m1, 32), o2 = __shfl_xor(m2, 32);
        m2 = fmaxf(fmaxf(m2, o2), fminf(m1, o1));
        m1 = fmaxf(m1, o1);
    };
    auto report = [&](int g, float r1, float r2) {
        if (h == 0 && rows > 0) best2[((int64_t)g * n_blk + blk) * 32 + lane] = make_float2(r1, r2);
    };
    struct lower { enum { value = 0 }; };
    struct upper { enum { value = 2 }; };
    for (int g = g_begin; g < g_end; ++g) {
        const asg_half8 *buf = Bs[(g - g_begin) & 1];
        step(buf, lower());
        finish();
        const float r1 = m1, r2 = m2;  // of the group before
        m1 = m2 = -INFINITY;
        step(buf, upper());
        if (g > g_begin) report(g - 1, r1, r2);
        asg_half8 *nxt = Bs[(g - g_begin + 1) & 1];
        if (g + 1 < g_end) {
#pragma unroll
            for (int k = 0; k < NPRE; ++k) nxt[tid + k * ASG_THREADS] = pre[k];
        }
        if (g + 2 < g_end) {
            src += ASG_TILE_VEC;
#pragma unroll
            for (int k = 0; k < NPRE; ++k) pre[k] = src[k * ASG_THREADS];
        }
        asg_lds_barrier();  // publishes nxt; every wave is done reading buf
    }
    if (g_begin < g_end) {  // the upper tiles' scores of the last group
        step(Bs[(g_end - 1 - g_begin) & 1], lower());
        finish();
        report(g_end - 1, m1, m2);
    }
}
__global__ __launch_bounds__(ASG_THREADS, 2) void asg_screen_kernel(const asg_half8 *__restrict__ A, int64_t C,
                                                                    const asg_half8 *__restrict__ B, int groups, int qg,
                                                                    float2 *__restrict__ best2, int64_t n_blk)
{
    __shared__ asg_half8 Bs[2][ASG_TILE_VEC];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t tile0 = ((int64_t)blockIdx.x * ASG_WAVES + wave) * ASG_NT;
    const int g0 = blockIdx.y * qg, g1 = g0 + qg < groups ? g0 + qg : groups;
    // (both instances run the same loop over the groups: their barriers meet)
    if ((tile0 + ASG_NT) * 32 <= C) asg_screen_body<true>(Bs, A, C, tile0, B, g0, g1, best2, n_blk);
    else asg_screen_body<false>(Bs, A, C, tile0, B, g0, g1, best2, n_blk);
}

// A workgroup per group of 32 vectors: thread (vector, part) merges the blocks part, part + 8, ...; a vector whose second
// best screened score is within 2 e of the best is decided from the double-precision products of the rows that are not
// further below.  Those are listed first: (vector, row) pairs, a thread each, and (vector, block) pairs where a block's
// second best row is in the running too, so that any of its 128 may be.  Such a block goes to a wave: fp32 products (eight
// lanes a row, whole cache lines), then double for the rows within the fp32 error of the block's best.
// Near rows tend to be neighbours in the table (the leaves of one cluster, a centroid drawn twice), and a thread that
// walked its block's rows alone held up the workgroup for 128 double products in a row.  200 000 vectors, each of 1024
// centroids twice in a row: 62.9 ms that way, 1.6 with the products dealt to the threads (bound by the rows, which a lane
// each reads 16 bytes of at a time), 0.79 now.  Five waves per SIMD: with four (the products unrolled further) vectors whose
// winner is clear, most of them, wait longer for their block maxima (740 000 against 4096 centroids 97 us, 88 with five).
// The block maxima, 256 bytes a group and block of rows, are read once, and by the open vectors, each its own, once more.  The first time
// past the caches (nontemporal loads): 585 000 vectors against 32 768 centroids, six launches, 316 -> 253 us.  Where all vectors are open,
// whose second reading then goes to memory, the products take the time: ms per call with loads through the caches / past them, every
// centroid with a near one in another block 7.59 / 7.58, with seven of them 7.90 / 7.97 (runs of one side differ by 2 %), 200 000 vectors
// against 1024 centroids each twice 0.82 / 0.83.
typedef float asg_float2 __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(256, 5) void asg_pick_kernel(const float *__restrict__ centroids, int64_t C, const float *__restrict__ x,
                                                       int64_t n, const float2 *__restrict__ best2, int64_t n_blk,
                                                       const uint32_t *__restrict__ stats, int32_t *__restrict__ codes)
{
    __shared__ __align__(16) float xs[32][DIM];
    __shared__ float w1[8][32], w2[8][32], thr[32], near[32];
    __shared__ int32_t wb[8][32], open[32];
    __shared__ int32_t n_open, n_one, n_all;
    __shared__ uint64_t one[256], all[256];  // vector << 32 | row / block of rows
    __shared__ unsigned long long key[32];
    const int tid = threadIdx.x, i = tid & 31, part = tid >> 5;
    const int64_t g = blockIdx.x, v0 = g * 32;
    if (tid == 0) n_open = 0;
    for (int e = tid; e < 32 * (DIM / 4); e += 256) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (v0 + (e >> 5) < n) v = *reinterpret_cast<const float4 *>(x + (v0 + (e >> 5)) * DIM + 4 * (e & 31));
        *reinterpret_cast<float4 *>(&xs[e >> 5][4 * (e & 31)]) = v;
    }
    float m1 = -INFINITY, m2 = -INFINITY;
    int mb = 0;
    for (int64_t b0 = part; b0 < n_blk; b0 += 32) {
        float2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            asg_float2 b = {-INFINITY, -INFINITY};
            if (b0 + 8 * u < n_blk) b = __builtin_nontemporal_load(reinterpret_cast<const asg_float2 *>(best2 + (g * n_blk + b0 + 8 * u) * 32 + i));
            v[u] = make_float2(b[0], b[1]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            m2 = fmaxf(fmaxf(m2, v[u].y), fminf(m1, v[u].x));
            if (v[u].x > m1) {
                m1 = v[u].x;
                mb = (int)(b0 + 8 * u);
            }
        }
    }
    w1[part][i] = m1;
    w2[part][i] = m2;
    wb[part][i] = mb;
    __syncthreads();
    {
        // |x| and |x - x1| of vector tid / 8, eight lanes each
        const int vec = tid >> 3;
        float s = 0.f, d = 0.f;
        for (int k = tid & 7; k < DIM; k += 8) {
            const float a = xs[vec][k], r = a - (float)asg_round(a);
            s += a * a;
            d += r * r;
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            s += __shfl_xor(s, o);
            d += __shfl_xor(d, o);
        }
        if ((tid & 7) == 0) {
            const float nx = sqrtf(s), nd = sqrtf(d), dc = sqrtf(__uint_as_float(stats[1])), c1 = sqrtf(__uint_as_float(stats[2]));
            // 128 * 2^-23 + 2^-16 + the rounding of the exact scores to fp32, with room for the roundings of the norms
            // (the constant: what the row number adds to a score of zero, for a vector of norm zero)
            const float e = 1.01f * (dc * nx + c1 * (nd + 4e-5f * (nx + nd))) + 1e-36f;
            float b1 = w1[0][vec], b2 = w2[0][vec];
            int bb = wb[0][vec];
            for (int p = 1; p < 8; ++p) {
                const float o1 = w1[p][vec], o2 = w2[p][vec];
                b2 = fmaxf(fmaxf(b2, o2), fminf(b1, o1));
                if (o1 > b1) {
                    b1 = o1;
                    bb = wb[p][vec];
                }
            }
            const float t = b1 - 2.0f * e;
            if (v0 + vec < n) {
                if (b2 < t && b1 < INFINITY) {  // (false when the bound is not a number)
                    codes[v0 + vec] = (int32_t)((int64_t)bb * ASG_ROWS + (__float_as_uint(b1) & 127u));
                } else {
                    open[atomicAdd(&n_open, 1)] = vec;
                    thr[vec] = t > -INFINITY && b1 < INFINITY ? t : -INFINITY;  // no bound: every row is looked at
                    // twice the error of an fp32 product: 20 roundings of at most |c| |x|, and of the norms' own
                    near[vec] = 4e-6f * nx * (c1 + dc) + 2e-36f;
                }
            }
        }
    }
    if (tid < 32) key[tid] = PLAID_KEY_MAX;
    __syncthreads();
    const int todo = n_open;
    const int64_t pairs = todo * n_blk;  // of an open vector and a block
    for (int64_t e0 = 0; e0 < pairs; e0 += 256) {
        if (tid == 0) n_one = n_all = 0;
        __syncthreads();
        if (e0 + tid < pairs) {
            const int vec = open[(e0 + tid) / n_blk];
            const int64_t b = (e0 + tid) % n_blk;
            const float t = thr[vec];
            const float2 v = best2[(g * n_blk + b) * 32 + vec];
            if (!(v.x < t)) {
                const uint64_t at = (uint64_t)vec << 32;
                if (v.y < t) one[atomicAdd(&n_one, 1)] = at | (uint64_t)(b * ASG_ROWS + (__float_as_uint(v.x) & 127u));
                else all[atomicAdd(&n_all, 1)] = at | (uint64_t)b;
            }
        }
        __syncthreads();
        auto look = [&](int vec, int64_t r) {
            const unsigned long long k = plaid_make_key(plaid_exact_dot(centroids + r * DIM, xs[vec]), (uint32_t)r);
            if (k < key[vec]) atomicMin(&key[vec], k);
        };
        if (tid < n_one) look((int)(one[tid] >> 32), (int64_t)(uint32_t)one[tid]);
        for (int i = tid >> 6; i < n_all; i += 4) {  // uniform per wave
            const int vec = (int)(all[i] >> 32), lane = tid & 63, piece = lane & 7, r = lane >> 3;
            const int64_t r0 = (int64_t)(uint32_t)all[i] * ASG_ROWS;
            float4 xv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[k] = *reinterpret_cast<const float4 *>(&xs[vec][32 * k + 4 * piece]);
            float top = -INFINITY, mine[2] = {-INFINITY, -INFINITY};  // mine: rows 8 piece + r and 64 + 8 piece + r
#pragma unroll 4
            for (int u = 0; u < ASG_ROWS / 8; ++u) {
                const int64_t row = r0 + 8 * u + r < C ? r0 + 8 * u + r : C - 1;  // (the last row again: no change)
                float d = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 c = *reinterpret_cast<const float4 *>(centroids + row * DIM + 32 * k + 4 * piece);
                    d = fmaf(c.x, xv[k].x, d);
                    d = fmaf(c.y, xv[k].y, d);
                    d = fmaf(c.z, xv[k].z, d);
                    d = fmaf(c.w, xv[k].w, d);
                }
                d += __shfl_xor(d, 1);
                d += __shfl_xor(d, 2);
                d += __shfl_xor(d, 4);
                top = fmaxf(top, d);
                if (u == piece) mine[0] = d;
                if (u == piece + 8) mine[1] = d;
            }
#pragma unroll
            for (int o = 8; o < 64; o <<= 1) top = fmaxf(top, __shfl_xor(top, o));
            const float cut = top - near[vec];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t row = r0 + 64 * k + 8 * piece + r;
                if (row < C && !(mine[k] < cut)) look(vec, row);  // (what is not a number is looked at)
            }
        }
        __syncthreads();
    }
    // (a key can only be missing when no score is a number)
    if (tid < todo) codes[v0 + open[tid]] = key[open[tid]] == PLAID_KEY_MAX ? 0 : (int32_t)(key[open[tid]] & 0xFFFFFFFFu);
}

// ------------------------------------------------------------------ host side
size_t plaid_assign_operand_bytes(int64_t rows)
{
    const int64_t per = 32ll * ASG_NT * ASG_WAVES;
    return (size_t)((rows + per - 1) / per * (per / 32) * ASG_TILE_VEC) * sizeof(asg_half8);
}
size_t plaid_assign_best_bytes(int64_t C, int64_t groups) { return (size_t)groups * (size_t)((C + ASG_ROWS - 1) / ASG_ROWS) * 32 * sizeof(float2); }
void plaid_launch_assign_prepare(hipStream_t st, const float *centroids, int64_t C, void *A, uint32_t *stats)
{
    const int64_t tiles = (int64_t)(plaid_assign_operand_bytes(C) / (ASG_TILE_VEC * sizeof(asg_half8)));
    int64_t g = (tiles * ASG_TILE_VEC + 255) / 256;
    hipLaunchKernelGGL(asg_operands_kernel, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(256), 0, st, centroids, C, tiles, (asg_half8 *)A);
    g = (C + 3) / 4;
    hipLaunchKernelGGL(asg_stats_kernel, dim3((unsigned)(g < 512 ? g : 512)), dim3(256), 0, st, centroids, C, stats);
}
void plaid_launch_assign(hipStream_t st, const float *centroids, int64_t C, const void *A, const uint32_t *stats, const float *x,
                         int64_t n, void *B, void *best2, int32_t *codes)
{
    const int64_t groups = (n + 31) / 32, n_blk = (C + ASG_ROWS - 1) / ASG_ROWS;
    int64_t g = (groups * ASG_TILE_VEC + 255) / 256;
    hipLaunchKernelGGL(asg_operands_kernel, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(256), 0, st, x, n, groups, (asg_half8 *)B);
    const unsigned gx = (unsigned)((C + 32 * ASG_NT * ASG_WAVES - 1) / (32 * ASG_NT * ASG_WAVES));
    // groups per workgroup: its centroid operands are loaded once, yet a few thousand workgroups keep the chip even
    int64_t qg = (groups * gx + 4095) / 4096;
    qg = qg < 8 ? 8 : (qg > 64 ? 64 : qg);
    while ((groups + qg - 1) / qg > 65535) qg *= 2;
    hipLaunchKernelGGL(asg_screen_kernel, dim3(gx, (unsigned)((groups + qg - 1) / qg)), dim3(ASG_THREADS), 0, st, (const asg_half8 *)A, C,
                       (const asg_half8 *)B, (int)groups, (int)qg, (float2 *)best2, n_blk);
    hipLaunchKernelGGL(asg_pick_kernel, dim3((unsigned)groups), dim3(256), 0, st, centroids, C, x, n, (const float2 *)best2, n_blk, stats,
                       codes);
}
