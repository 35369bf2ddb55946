// Nucleus (top-p) sampling on materialised logits ("Reasoning Experiments
// details": rollouts are drawn with top-p 0.9 at temperature 0.7).
//
// With p_v = softmax(logits / T), the nucleus is the smallest set of most
// probable tokens whose probability reaches top_p (equal logits kept or dropped
// together); the token is drawn from the renormalised nucleus with the
// Gumbel-max rule and the same counter-based noise as plain sampling,
// argmax_{v in nucleus} (logit_v + T * g_v).
//
// One block per row.  The unrestricted Gumbel-max winner w0 (from the LM-head
// epilogue, or found here) is the answer whenever it lies inside the nucleus,
// which one streaming pass decides: w0 is inside iff the probability mass of
// the strictly larger logits is below top_p.  That holds for about top_p of the
// rows.  Otherwise the cut is located (one-kernel form: by bisection over the
// order-preserving integer image of the logits, at most 32 passes over the row,
// which stays in cache, each a deterministic block reduction), then the Gumbel-max
// is repeated over the kept tokens only.
//
// Re-reading rows from memory is what those passes cost, so the decode step
// splits the work: nucleus_kernel<.., DEFER> makes the streaming pass for every
// row and appends the rows that need the search to a list, and
// nucleus_slow_kernel takes the listed rows one at a time with the row held in
// registers (persistent blocks of 1024 threads, 32 elements per thread), so each
// row is read from memory twice in total.  Larger vocabularies use the
// one-kernel form.
#pragma once
#include "common.hpp"
#include <cfloat>

// Unsigned integers ordered as the floats are; -0 and +0 share a key.
__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int NW>
__device__ __forceinline__ float block_sum(float v, float *red)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.0f;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += red[i];
    __syncthreads();
    return t;
}

template <int NW>
__device__ __forceinline__ float block_max(float v, float *red)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = -INFINITY;
#pragma unroll
    for (int i = 0; i < NW; ++i) t = fmaxf(t, red[i]);
    __syncthreads();
    return t;
}

// (value, index) maximum, lowest index on equal values; every thread gets the result.
template <int NW>
__device__ __forceinline__ int block_argmax(float bv, int bi, float *red, int *redi)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(bv, off, kWave);
        const int oi = __shfl_xor(bi, off, kWave);
        if (arg_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = bv; redi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    float tv = -INFINITY;
    int ti = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < NW; ++i)
        if (arg_better(red[i], redi[i], tv, ti)) { tv = red[i]; ti = redi[i]; }
    __syncthreads();
    return ti;
}

// Calls fn(value, index) for this thread's share of one row.  Rows that allow it
// are read as 16-byte vectors, four independent loads in flight per thread, so a
// pass over a cache-resident row costs a few memory latencies, not one per element.
template <int NT, typename F>
__device__ __forceinline__ void row_foreach(const float *__restrict__ L, int V, F &&fn)
{
    const int tid = threadIdx.x;
    if ((V & 3) == 0 && (reinterpret_cast<uintptr_t>(L) & 15) == 0) {
        const f32x4_t *L4 = reinterpret_cast<const f32x4_t *>(L);
        const int n4 = V >> 2;
        int i = tid;
        for (; i + 3 * NT < n4; i += 4 * NT) {
            const f32x4_t a = L4[i], b = L4[i + NT], c = L4[i + 2 * NT], d = L4[i + 3 * NT];
#pragma unroll
            for (int k = 0; k < 4; ++k) fn(a[k], 4 * i + k);
#pragma unroll
            for (int k = 0; k < 4; ++k) fn(b[k], 4 * (i + NT) + k);
#pragma unroll
            for (int k = 0; k < 4; ++k) fn(c[k], 4 * (i + 2 * NT) + k);
#pragma unroll
            for (int k = 0; k < 4; ++k) fn(d[k], 4 * (i + 3 * NT) + k);
        }
        for (; i < n4; i += NT) {
            const f32x4_t a = L4[i];
#pragma unroll
            for (int k = 0; k < 4; ++k) fn(a[k], 4 * i + k);
        }
    } else {
        int v = tid;
        for (; v + 3 * NT < V; v += 4 * NT) {
            const float a = L[v], b = L[v + NT], c = L[v + 2 * NT], d = L[v + 3 * NT];
            fn(a, v); fn(b, v + NT); fn(c, v + 2 * NT); fn(d, v + 3 * NT);
        }
        for (; v < V; v += NT) fn(L[v], v);
    }
}

// Calls fn(const float (&)[n]) for this thread's share of one row in batches of n = 16 (or 4, or 1, at the end), the
// next batch requested before the current one is used.  Rows that are no whole vectors go by elements, in the same
// batches (one element at a time: a row of 32001 26 -> 34 us).
template <int NT, typename F>
__device__ __forceinline__ void row_batches(const float *__restrict__ L, int V, F &&fn)
{
    const int tid = threadIdx.x;
    if ((V & 3) == 0 && (reinterpret_cast<uintptr_t>(L) & 15) == 0) {
        const f32x4_t *L4 = reinterpret_cast<const f32x4_t *>(L);
        const int n4 = V >> 2;
        f32x4_t nx[4];
        auto request = [&](int i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) nx[q] = L4[i + q * NT];
        };
        int i = tid;
        if (i + 3 * NT < n4) request(i);
        for (; i + 3 * NT < n4; i += 4 * NT) {
            float x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = nx[k >> 2][k & 3];
            if (i + 7 * NT < n4) request(i + 4 * NT);
            fn(x);
        }
        for (; i < n4; i += NT) {
            const f32x4_t a = L4[i];
            const float x[4] = {a[0], a[1], a[2], a[3]};
            fn(x);
        }
    } else {
        float nx[16];
        auto request = [&](int v) {
#pragma unroll
            for (int k = 0; k < 16; ++k) nx[k] = L[v + k * NT];
        };
        int v = tid;
        if (v + 15 * NT < V) request(v);
        for (; v + 15 * NT < V; v += 16 * NT) {
            float x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = nx[k];
            if (v + 31 * NT < V) request(v + 16 * NT);
            fn(x);
        }
        for (; v + 3 * NT < V; v += 4 * NT) {
            const float x[4] = {L[v], L[v + NT], L[v + 2 * NT], L[v + 3 * NT]};
            fn(x);
        }
        for (; v < V; v += NT) {
            const float x[1] = {L[v]};
            fn(x);
        }
    }
}

// logits: [rows][ld] fp32, V <= ld.  tok[rows]: with FIND_W0 = false it holds the
// unrestricted Gumbel-max winner on entry (a negative value marks an idle row,
// which is skipped) and the nucleus sample on exit; with FIND_W0 = true it is
// output only.  Position of the random counter: pos_rows[row], else *pos_dev,
// else pos.  If store is not null the token also goes to
// store[*step_dev * store_stride + row].  If pos_advance is not null the
// position of every non-idle row is incremented at the end (pos_advance may be
// the same array as pos_rows), or set to -1 (idle) if the row's token is
// eos_plus1 - 1 (eos_plus1 = 0: no such token).
// With DEFER, a row that needs the search is appended to slow_list (its count in
// *slow_count, which must be zero at launch) and left to nucleus_slow_kernel,
// which also does that row's store / pos_advance.
template <int NT, bool FIND_W0, bool DEFER = false>
__global__ void __launch_bounds__(NT)
nucleus_kernel(const float *__restrict__ logits, int64_t ld, int V, float temp, float top_p, uint32_t seed, int pos,
               const int *__restrict__ pos_dev, const int *pos_rows, int32_t *__restrict__ tok,
               int32_t *__restrict__ store, const int *__restrict__ step_dev, int64_t store_stride,
               int32_t *pos_advance, int *__restrict__ slow_count = nullptr, int *__restrict__ slow_list = nullptr,
               uint32_t row_base = 0, int eos_plus1 = 0)
{
    constexpr int NW = NT / 64;
    __shared__ float red[NW];
    __shared__ int redi[NW];
    const int64_t row = blockIdx.x;
    const int tid = threadIdx.x;
    const float *__restrict__ L = logits + row * ld;
    int w0 = FIND_W0 ? 0 : tok[row];
    if (!FIND_W0 && w0 < 0) return;                       // idle row (the whole block leaves)
    const uint32_t p = (uint32_t)(pos_rows ? pos_rows[row] : (pos_dev ? *pos_dev : pos));
    const uint32_t rk = srm_rowkey(seed, p, (uint32_t)row + row_base);     // the counter is keyed on the sample index
    const float inv = 1.4426950408889634f / temp;

    if constexpr (FIND_W0) {
        float bv = -INFINITY;
        int bi = 0x7fffffff;
        row_foreach<NT>(L, V, [&](float x, int v) {
            const float s = x + temp * srm_gumbel(rk, (uint32_t)v);
            if (arg_better(s, v, bv, bi)) { bv = s; bi = v; }
        });
        w0 = block_argmax<NW>(bv, bi, red, redi);
    }
    w0 = min(max(w0, 0), V - 1);
    const uint32_t kw = order_key(L[w0]);

    // One pass: row maximum, normaliser Z and the mass above w0, rescaled on the fly, once per batch (a test and a
    // rescaling per element made the pass bound by its instructions: 15.3 -> 9.4 us for 300 rows of 32000).  A
    // logit's key exceeds w0's exactly if the logit is the larger one.  (The maximum stays finite: with an infinite
    // logit Z is infinite, and w0, which it is, lies inside.)
    const float xw = L[w0];
    float mt = -INFINITY, z = 0.0f, fa = 0.0f;
    row_batches<NT>(L, V, [&](const auto &x) {
        constexpr int n = sizeof(x) / sizeof(float);
        float top = mt;
#pragma unroll
        for (int k = 0; k < n; ++k) top = fmaxf(top, x[k]);
        top = fminf(top, FLT_MAX);
        const float sc = top > mt ? __builtin_amdgcn_exp2f((mt - top) * inv) : 1.0f;
        const float base = top == -INFINITY ? 0.0f : top;
        z *= sc;
        fa *= sc;
        mt = top;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const float e = __builtin_amdgcn_exp2f((x[k] - base) * inv);
            z += e;
            fa += x[k] > xw ? e : 0.0f;
        }
    });
    const float M = block_max<NW>(mt, red);
    const float sc = mt == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((mt - M) * inv);
    const float Z = block_sum<NW>(z * sc, red);
    const float FA = block_sum<NW>(fa * sc, red);
    const float target = top_p * Z;

    int result = w0;
    uint32_t lo = kw, hi = order_key(M);
    if (DEFER && !(FA < target) && hi > lo) {
        if (tid == 0) slow_list[atomicAdd(slow_count, 1)] = (int)row;
        return;
    }
    if (!(FA < target) && hi > lo) {
        // invariant: mass{key > lo} >= target, mass{key > hi} < target; kept = {key >= hi} at the end
        while (hi - lo > 1u) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            float f = 0.0f;
            row_foreach<NT>(L, V, [&](float x, int) {
                if (order_key(x) > mid) f += __builtin_amdgcn_exp2f((x - M) * inv);
            });
            f = block_sum<NW>(f, red);
            if (f < target) hi = mid; else lo = mid;
        }
        float bv = -INFINITY;
        int bi = 0x7fffffff;
        row_foreach<NT>(L, V, [&](float x, int v) {
            if (order_key(x) >= hi) {
                const float s = x + temp * srm_gumbel(rk, (uint32_t)v);
                if (arg_better(s, v, bv, bi)) { bv = s; bi = v; }
            }
        });
        result = block_argmax<NW>(bv, bi, red, redi);
        if (result < 0 || result >= V) result = w0;
    }
    if (tid == 0) {
        tok[row] = result;
        if (store) store[(int64_t)(*step_dev) * store_stride + row] = result;
        if (pos_advance) pos_advance[row] = (eos_plus1 && result == eos_plus1 - 1) ? -1 : (int32_t)p + 1;
    }
}

// The rows nucleus_kernel<.., DEFER> listed, each held in registers for the whole search: a thread keeps the logits and
// the probabilities p / p_max of its EPT elements (V <= NT * EPT).  Sums are taken over their images in units of 2^-47
// (nucleus_mass), so they are exact, do not depend on their order, and a long tail counts: with V <= 2^15 elements the
// total is short of the probabilities' by less than 2^-32 p_max, where a float sum rounds by 2^-24 of itself.
// The elements above w0 go into a histogram of masses over equal
// steps of logit value (LDS atomics); the step that the cut lies in holds a few dozen elements of most rows, which are
// gathered, and each of them is asked whether the mass from it upwards reaches the target.  A step of more than kCand
// elements (ties, extreme ranges) is left to a bisection over all elements.
// Bound by the arithmetic on a row's elements (the Gumbel noise above all), one row per CU.  A row of 32000: 44 us with
// 25 - 31 bisection passes and the noise from a second reading of the row, now 36 us; 300 rows 96 -> 75 us.
// Persistent: block i takes list entries i, i + gridDim, ...  Arguments as
// nucleus_kernel; tok[row] holds the unrestricted winner on entry.
__device__ __forceinline__ float key_value(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k); }

// floor(2^47 e) for 0 <= e <= 1: the upper 23 bits, then the rest (both differences are exact); 0 for a NaN
__device__ __forceinline__ unsigned long long nucleus_mass(float e)
{
    const float t = fmaxf(e, 0.0f) * 8388608.0f;                       // 2^23
    const uint32_t hi = (uint32_t)t;
    const uint32_t lo = (uint32_t)((t - (float)hi) * 16777216.0f);     // 2^24
    return (unsigned long long)hi << 24 | lo;
}

constexpr int kCand = 512, kSteps = 1024;
template <int NT, int EPT>
__global__ void __launch_bounds__(NT)
nucleus_slow_kernel(const float *__restrict__ logits, int64_t ld, int V, float temp, float top_p, uint32_t seed, int pos,
                    const int *__restrict__ pos_dev, const int *pos_rows, int32_t *__restrict__ tok,
                    int32_t *__restrict__ store, const int *__restrict__ step_dev, int64_t store_stride,
                    int32_t *pos_advance, const int *__restrict__ slow_count, const int *__restrict__ slow_list,
                    uint32_t row_base, int eos_plus1)
{
    static_assert(EPT % 4 == 0, "EPT must be a multiple of 4");
    static_assert(NT >= kCand && kSteps % 64 == 0, "one thread per candidate; whole steps per lane");
    typedef unsigned long long u64;
    constexpr int NW = NT / 64;
    __shared__ float red[NW];
    __shared__ int redi[NW];
    __shared__ u64 hist[kSteps];
    __shared__ u64 cand_mass[kCand];
    __shared__ uint32_t cand_key[kCand];
    __shared__ u64 group_s[kSteps / 64];
    __shared__ u64 sum_s, above_s;                   // a block sum; the mass above the cut's step
    __shared__ int step_s, count_s;
    __shared__ uint32_t hi_s;
    const int tid = threadIdx.x;
    const int n = *slow_count;
    const float inv = 1.4426950408889634f / temp;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int64_t row = slow_list[i];
        const float *__restrict__ L = logits + row * ld;
        const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(L) & 15) == 0;
        // element k of this thread has index first + 4 NT (k / 4) + (k % 4) next; absent ones are -inf
        const int first = vec ? 4 * tid : tid, next = vec ? 1 : NT;
        float x[EPT];
        float e[EPT];
        float mt = -INFINITY;
        if (vec) {
            const f32x4_t *L4 = reinterpret_cast<const f32x4_t *>(L);
            const int n4 = V >> 2;
#pragma unroll
            for (int k = 0; k < EPT / 4; ++k) {
                const int j = tid + k * NT;
                f32x4_t a;
                if (j < n4) a = L4[j];
                else a[0] = a[1] = a[2] = a[3] = -INFINITY;
#pragma unroll
                for (int c = 0; c < 4; ++c) { x[4 * k + c] = a[c]; mt = fmaxf(mt, a[c]); }
            }
        } else {
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                const int v = tid + k * NT;
                x[k] = v < V ? L[v] : -INFINITY;
                mt = fmaxf(mt, x[k]);
            }
        }
        const int w0 = min(max(tok[row], 0), V - 1);
        const float xw = L[w0];
        const uint32_t p = (uint32_t)(pos_rows ? pos_rows[row] : (pos_dev ? *pos_dev : pos));
        const uint32_t rk = srm_rowkey(seed, p, (uint32_t)row + row_base);
        for (int b = tid; b < kSteps; b += NT) hist[b] = 0;
        if (tid == 0) { sum_s = 0; count_s = 0; hi_s = 0; step_s = -1; }
        const float M = block_max<NW>(mt, red);      // (its barriers also order the stores above)
        // the step of a logit above w0, never smaller for a larger logit: 0 where M - xw overflows (scale 0, and 0 times
        // infinity), the last one where it is so small that scale is infinite
        const float scale = (float)kSteps / (M - xw);
        auto step_of = [](float v, float xw_, float scale_) {
            return (int)fminf(fmaxf((v - xw_) * scale_, 0.0f), (float)(kSteps - 1));
        };
        u64 z = 0;
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            e[k] = __builtin_amdgcn_exp2f((x[k] - M) * inv);           // absent: exp2(-inf) = 0
            const u64 mass = nucleus_mass(e[k]);
            z += mass;
            if (x[k] > xw) atomicAdd(&hist[step_of(x[k], xw, scale)], mass);
        }
        atomicAdd(&sum_s, z);
        __syncthreads();
        const u64 target = (u64)ceil((double)top_p * (double)sum_s);
        // suffix sums over groups of 64 steps, one group per wavefront at a time; then the step whose own mass takes the
        // mass from above across the target
        constexpr int GROUPS = kSteps / 64, PER = GROUPS / NW;
        static_assert(GROUPS % NW == 0, "whole groups per wavefront");
        const int lane = tid & 63, wave = tid >> 6;
        u64 own[PER], from[PER];
#pragma unroll
        for (int g = 0; g < PER; ++g) {
            own[g] = from[g] = hist[(wave * PER + g) * 64 + lane];
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const u64 o = __shfl_down(from[g], off, kWave);
                if (lane + off < 64) from[g] += o;
            }
            if (lane == 0) group_s[wave * PER + g] = from[g];
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < PER; ++g) {
            u64 higher = 0;
#pragma unroll
            for (int q = 0; q < GROUPS; ++q) higher += q > wave * PER + g ? group_s[q] : 0;
            const u64 above = higher + from[g] - own[g];
            if (above < target && above + own[g] >= target) { step_s = (wave * PER + g) * 64 + lane; above_s = above; }
        }
        __syncthreads();
        int result = w0;
        const int cut = step_s;                      // -1: the mass above w0 stays below the target, w0 lies inside
        if (cut >= 0) {
            const u64 above = above_s;
            // (the compiler must not see that these are the values of the loop above: it would keep that loop's 64
            // places and comparisons in registers)
            float xw2 = xw, scale2 = scale;
            asm volatile("" : "+v"(xw2), "+v"(scale2));
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                if (x[k] > xw2 && step_of(x[k], xw2, scale2) == cut) {
                    const int at = atomicAdd(&count_s, 1);
                    if (at < kCand) { cand_key[at] = order_key(x[k]); cand_mass[at] = nucleus_mass(e[k]); }
                }
            }
            __syncthreads();
            const int nc = count_s;
            uint32_t hi;
            if (nc <= kCand) {
                if (tid < nc) {
                    const uint32_t key = cand_key[tid];
                    u64 f = above;
#pragma unroll 4
                    for (int j = 0; j < nc; ++j) f += cand_key[j] >= key ? cand_mass[j] : 0;
                    if (f >= target) atomicMax(&hi_s, key);
                }
                __syncthreads();
                hi = hi_s;
            } else {
                // invariant: mass{key > lo} >= target, mass{key > hi} < target; kept = {key >= hi} at the end
                uint32_t lo = order_key(xw);
                hi = order_key(M);
                while (hi - lo > 1u) {
                    const uint32_t mid = lo + ((hi - lo) >> 1);
                    u64 f = 0;
                    __syncthreads();
                    if (tid == 0) sum_s = 0;
                    __syncthreads();
                    const float above_v = key_value(mid);              // (as floats: 64 keys would be kept over the loop)
#pragma unroll
                    for (int k = 0; k < EPT; ++k) f += x[k] > above_v ? nucleus_mass(e[k]) : 0;
                    atomicAdd(&sum_s, f);
                    __syncthreads();
                    if (sum_s < target) hi = mid; else lo = mid;
                }
            }
            // Gumbel-max over the kept tokens
            const float least = key_value(hi);
            float bv = -INFINITY;
            int bi = 0x7fffffff;
            auto score = [&](int k, int v) {
                if (x[k] >= least) {
                    const float s = x[k] + temp * srm_gumbel(rk, (uint32_t)v);
                    if (arg_better(s, v, bv, bi)) { bv = s; bi = v; }
                }
            };
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                score(k, first + 4 * NT * (k / 4) + k % 4 * next);
            }
            result = block_argmax<NW>(bv, bi, red, redi);
            if (result < 0 || result >= V) result = w0;
        }
        if (tid == 0) {
            tok[row] = result;
            if (store) store[(int64_t)(*step_dev) * store_stride + row] = result;
            if (pos_advance) pos_advance[row] = (eos_plus1 && result == eos_plus1 - 1) ? -1 : (int32_t)p + 1;
        }
        __syncthreads();                             // the shared words are set again for the next row
    }
}
