// Two measuring kernels that give the chip's achievable rates beside its published peaks: a plain
// streaming copy (HBM read + write) and a register-resident chain of bf16 matrix-core instructions.
// Neither is part of the model's path; the benchmark reports the hot kernels against both.
#pragma once
#include "common.hpp"

// dst[i] = src[i] over n16 16-byte words; every lane moves `UNROLL` words per trip, all loads issued
// before the first store, and the grid covers the array once.  NT selects streaming (non-temporal)
// loads and stores.
template <int UNROLL, bool NT>
__global__ __launch_bounds__(256) void probe_copy_kernel(const u32x4_t *__restrict__ src, u32x4_t *__restrict__ dst,
                                                         int64_t n16)
{
    const int64_t base = ((int64_t)blockIdx.x * UNROLL) * 256 + threadIdx.x;
    u32x4_t v[UNROLL];
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
        const int64_t j = base + (int64_t)i * 256;
        if (j < n16) v[i] = NT ? __builtin_nontemporal_load(src + j) : src[j];
    }
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
        const int64_t j = base + (int64_t)i * 256;
        if (j < n16) {
            if (NT) __builtin_nontemporal_store(v[i], dst + j);
            else dst[j] = v[i];
        }
    }
}

// Every wavefront issues `iters` rounds of eight independent 16x16x32 bf16 products, the ones that the
// GEMMs are made of, into eight fp32 accumulator tiles held in registers (no memory traffic inside the
// loop), then writes one sum per lane.  With A = 1 and B = 1 every accumulator element ends at
// 32 * iters, so the written value is 8 * 4 * 32 * iters per lane (4 accumulator registers per tile):
// checkable on the host.  With random_operands the operand elements are pseudo-random values in
// (-1, 1), different per lane and element: the matrix cores draw more power on such data than on
// constants, and the clock the chip holds (hence the rate) is lower; the sums are then only finite,
// not predictable.
__global__ __launch_bounds__(256, 2) void probe_mfma_kernel(float *__restrict__ out, int iters, float a_val,
                                                         int random_operands)
{
    bf16x8_t a, b;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = (bf16)a_val;
        b[i] = (bf16)1.0f;
        if (random_operands) {
            uint32_t h = (threadIdx.x * 2654435761u) ^ (uint32_t)(i * 40503 + 12345);
            h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
            a[i] = (bf16)((float)(int32_t)h * (1.0f / 2147483648.0f));
            h *= 3266489917u; h ^= h >> 16;
            b[i] = (bf16)((float)(int32_t)h * (1.0f / 2147483648.0f));
        }
    }
    f32x4_t c[8] = {};
    // (Room for 256 registers: with more the compiler copies each product from and to accumulation registers.  The empty
    // statement keeps a tile where it is, which else wanders through overlapping registers.  Random operands: 1.33 | 2.22
    // PFLOP/s.)
#pragma clang loop unroll(disable)
    for (int it = 0; it < iters; ++it)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            c[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c[t], 0, 0, 0);
            asm volatile("" : "+v"(c[t]));
        }
    float s = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) s += c[t][i];
    out[(int64_t)blockIdx.x * 256 + threadIdx.x] = s;
}
