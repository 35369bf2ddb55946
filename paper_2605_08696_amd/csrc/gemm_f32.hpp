// fp32 GEMMs of more than a few rows on the matrix cores: out = epilogue(A W^T + bias), fp32 products and sums
// (v_mfma_f32_32x32x2_f32 / v_mfma_f32_16x16x4_f32: a full fp32 multiply-add per element, like v_fma_f32, at twice
// the rate a kernel without packed fp32 arithmetic reaches on the vector units, and with the operand re-use of a tile).
//
// Two kernels, one for each way the work can be short:
//   gemm_f32_slices_kernel<T>  a T x T output tile per work-group, K cut into one slice per wavefront: every wavefront
//                              streams its own slice through its own LDS ring and never waits for another one; the
//                              four partial tiles meet in LDS at the end, added in wavefront order.  For launches
//                              with few tiles, where the time is a tile's trip through K.
//   gemm_f32_tile_kernel       a 64 x 64 tile per work-group, one 32 x 32 quarter per wavefront, operands shared
//                              through an LDS ring of four 32-wide k tiles.  For launches that fill the chip.
// A sequence form of 4 x 256 tokens on a 256-wide, 4-layer model went from 1.32 to 0.37 ms with them, the prefill of a
// request of 8 x 16 tokens from 1.05 to 0.08 ms: gemm_f32_kernel stepped through K sixteen at a time with one tile in
// flight and 4-byte LDS accesses, 28 us for any launch with K = 256 and 98 with K = 1024 (launch_f32_tiles has the
// figures per shape).  What bounds them: the matrix pipe and, around every 32 k, about 0.1 us of LDS reads and tile
// loads that one wavefront per SIMD does not hide (independent sums, or the next tile's operands read under the
// products, changed nothing).
//
// Both read the operands of four MFMAs with one 16-byte LDS read per lane: lane (i, h) holds k = 8 s + 4 h + j for
// j = 0 .. 3 of the s-th group of 8 (16x16: k = 16 s + 4 q + j), the same mapping for A and W, so the contraction
// sees every k once, in another order than the memory's.  The product is formed transposed (W first), so a lane
// holds four consecutive output columns of one row per register quad.
// NA: how many sums a slice of K is kept in, 1 or kFine = 8 (by j and by the half of a 32-wide k tile), added in pairs at
// the end of the slice.  Eight for calls of at most 32 rows: against 64-bit arithmetic the logits of a 256-wide, 4-layer
// model are off by 5.0e-7 of their norm with one sum, by 2.9e-7 with the GEMV that these kernels replaced there (16 lanes
// per dot product) and by 2.8e-7 with eight; up to 0.1 us per launch.  One for larger calls, where gemm_f32_kernel was off
// by 9.7e-7 and one sum is by 5.0e-7 (four: 3.1e-7, but 4096 x 4096 x 256 takes 106 us instead of 99).
// LDS rows are 128 bytes (32 k), 16-byte chunk c of row r at c ^ ((r >> 1) & 7), as in gemm_bf16_kernel.
// Needs K % 4 == 0, 16-byte aligned operands, and outputs aligned so where N % 4 == 0 (launch_f32 falls back to
// gemm_f32_kernel otherwise).
#pragma once
#include "gemm.hpp"

namespace f32gemm {
constexpr int BK = 32;
constexpr int kSlices = 4;                 // slices of K, whose sums are added in order
constexpr int kFine = 8;

__device__ __forceinline__ u32x4_t descriptor(const void *base, int bytes)
{
    u32x4_t rs;
    const unsigned long long a = reinterpret_cast<unsigned long long>(base);
    rs[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
    rs[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));                 // stride 0: raw buffer
    rs[2] = __builtin_amdgcn_readfirstlane((unsigned)bytes);
    rs[3] = 0x00020000u;
    return rs;
}
// 64 x 16 bytes global -> LDS (lane l's to lds_dst + 16 l); offsets at or past the descriptor's size arrive as zeros.
// (asm: known to the compiler as an LDS write, it would wait for every load in flight before the next LDS read)
__device__ __forceinline__ void dma(const u32x4_t &rs, unsigned lds_dst, int voff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds_dst), "v"(voff), "s"(rs)
                 : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }
__device__ __forceinline__ unsigned lds_address(const void *p)
{
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    return __builtin_amdgcn_readfirstlane((unsigned)reinterpret_cast<unsigned long long>((lds_byte *)p));
}
constexpr int kOutside = 0x7ffffff0;       // a byte offset past every descriptor

// The products of one 32-wide k tile on a 32x32 tile, operands as four 16-byte reads per lane (read s holds k = 8 s +
// 4 (lane / 32) + j): two 32x32x2 products for each 16x16x4 one of the 16-wide tile, over the same four k.
template <int NA>
__device__ __forceinline__ void mfma_k32(const f32x4_t (&fw)[4], const f32x4_t (&fa)[4], f32x16_t (&acc)[NA])
{
#pragma unroll
    for (int s = 0; s < 4; s += 2)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f32x16_t &a = acc[(2 * s + j) % NA];
            a = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[s][j], fa[s][j], a, 0, 0, 0);
            a = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[s + 1][j], fa[s + 1][j], a, 0, 0, 0);
        }
}
// element r of a slice's sum
template <int NA, typename ACC>
__device__ __forceinline__ float slice_sum(const ACC (&acc)[NA], int r)
{
    static_assert(NA == 1 || NA == 8, "one sum or eight");
    if constexpr (NA == 1) return acc[0][r];
    else return ((acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r])) + ((acc[4][r] + acc[5][r]) + (acc[6][r] + acc[7][r]));
}
template <int NA, int R, typename ACC>
__device__ __forceinline__ void clear_sums(ACC (&acc)[NA])
{
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[a][r] = 0.0f;
}

// Four consecutive columns of one output row, column tests where the row ends.
template <int EPI>
__device__ __forceinline__ void store_quad(const GemmEpi &ep, int row, int col, int N, float4 v)
{
    if (ep.bias) {
        v.x += ep.bias[min(col, N - 1)]; v.y += ep.bias[min(col + 1, N - 1)];
        v.z += ep.bias[min(col + 2, N - 1)]; v.w += ep.bias[min(col + 3, N - 1)];
    }
    if ((N & 3) == 0 && col + 3 < N) {
        epi_store4<EPI, float>(ep, row, col, v);
    } else {
        if (col < N) epi_store1p<EPI, float>(ep, row, col, v.x);
        if (col + 1 < N) epi_store1p<EPI, float>(ep, row, col + 1, v.y);
        if (col + 2 < N) epi_store1p<EPI, float>(ep, row, col + 2, v.z);
        if (col + 3 < N) epi_store1p<EPI, float>(ep, row, col + 3, v.w);
    }
}
}  // namespace f32gemm

// LNA (T = 16, M <= kLnaRows, K <= 1024, K % 32 == 0): as in gemm_bf16_slices_kernel, the A operand is LayerNorm(ep.ln_x
// rows), made by the work-group: a panel [K / 32][16 rows][32] behind the rings, which then hold W only.
// (launch bounds of two wavefronts per SIMD: the sums then live in VGPRs; as AGPRs, four of the thirty-two were copied
// back and forth around every k tile)
template <int EPI, int T, int NS, int NA, bool LNA = false>
__global__ void __launch_bounds__(f32gemm::kSlices * 64, NA > 1 ? 2 : 1)
gemm_f32_slices_kernel(const float *__restrict__ A, const float *__restrict__ W, int M, int N, int K, GemmEpi ep)
{
    using namespace f32gemm;
    static_assert(T == 16 || T == 32, "the tile of one MFMA");
    static_assert(EPI != EPI_ARGMAX, "partial winners are counted per 64 columns");
    constexpr int NW = kSlices;
    static_assert(!LNA || T == kLnaRows, "the panel holds one row tile");
    constexpr int AR = LNA ? 0 : T;                      // rows of A in a stage
    constexpr int STAGE = (AR + T) * BK;                 // floats: rows of A, T rows of W
    constexpr int LD = (AR + T) / 8;                     // tile loads (8 rows each) per k tile
    constexpr int RS = T + 4;                            // row stride of the reduction area in floats
    static_assert(NW * T * RS <= NW * NS * STAGE, "the reduction area exceeds the rings");
    extern __shared__ __align__(16) float f32_sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nbn = (N + T - 1) / T;
    const int m0 = (int)(blockIdx.x / nbn) * T, n0 = (int)(blockIdx.x % nbn) * T;
    const u32x4_t rs_a = descriptor(A + (size_t)m0 * K, min(T, M - m0) * K * 4);
    const u32x4_t rs_w = descriptor(W + (size_t)n0 * K, min(T, N - n0) * K * 4);
    float *ring = f32_sm + wave * NS * STAGE;
    const unsigned ring_lds = lds_address(ring);

    // load i of a k tile: rows 8i .. 8i+7 of [A; W]; lane (r = l >> 3, slot = l & 7) fetches the chunk that belongs
    // into its slot.  An odd eight of rows swizzles with chunk bit 2 flipped.
    const int ld_r = lane >> 3;
    const int chunk = ((lane & 7) ^ (ld_r >> 1)) * 4;    // first k of this lane's 16 bytes, even eights
    const int kt_all = (K + BK - 1) / BK;
    const int kt0 = kt_all * wave / NW, kt1 = kt_all * (wave + 1) / NW;
    auto issue = [&](int kt, int slot) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int op_i = i % (T / 8);                // eight of rows within its operand
            const int k = kt * BK + (chunk ^ ((op_i & 1) << 4));
            const int voff = k < K ? ((op_i * 8 + ld_r) * K + k) * 4 : kOutside;
            dma(i < AR / 8 ? rs_a : rs_w, ring_lds + (slot * STAGE + i * 8 * BK) * 4, voff);
        }
    };
    const int li = lane % T, lh = lane / T;              // operand row, k group of this lane
    const int sw = swz_of_row(li);
    typedef typename std::conditional<T == 32, f32x16_t, f32x4_t>::type acc_t;
    acc_t acc[NA];
    clear_sums<NA, T * T / 64>(acc);
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (kt0 + s < kt1) issue(kt0 + s, s);
    // this thread's quad of the output: what its epilogue reads from memory is requested behind the first tiles
    const int er = m0 + tid / (T / 4), ec = n0 + tid % (T / 4) * 4;
    const bool owner = tid < T * T / 4 && er < M && ec < N, whole = (N & 3) == 0;
    EpiQuad eq;
    if (owner && whole) eq = epi_quad_request<EPI>(ep, er, ec);
    float *panel = f32_sm + NW * NS * STAGE;
    if constexpr (LNA)
        layernorm_panel<NW>(ep, M, K, wave, lane, [&](int r, int c, float4 o) {
            *reinterpret_cast<float4 *>(panel + (c >> 5) * T * BK + r * BK + ((((c & 31) >> 2) ^ swz_of_row(r)) << 2)) = o;
        });
    int slot = 0;
    for (int kt = kt0; kt < kt1; ++kt) {
        // k tile kt has landed, younger ones may be on their way (behind the last one issued: none)
        if (kt + NS <= kt1) wait_loads<(NS - 1) * LD>();
        else wait_loads<0>();
        const float *ws = ring + slot * STAGE + (AR + li) * BK;
        const float *as = LNA ? panel + kt * T * BK + li * BK : ring + slot * STAGE + li * BK;
        constexpr int G = 64 / T, NR = 8 / G;            // 16-byte chunks per LDS read of a row, reads per k tile
        f32x4_t fa[NR], fw[NR];
#pragma unroll
        for (int s = 0; s < NR; ++s) {
            const int ch = ((s * G + lh) ^ sw) * 4;
            fa[s] = *reinterpret_cast<const f32x4_t *>(as + ch);
            fw[s] = *reinterpret_cast<const f32x4_t *>(ws + ch);
        }
        wait_lds();
        if (kt + NS < kt1) issue(kt + NS, slot);         // the slot is free again
        if constexpr (T == 32) {
            mfma_k32(fw, fa, acc);
        } else {
#pragma unroll
            for (int s = 0; s < NR; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc_t &a = acc[(4 * s + j) % NA];
                    a = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[s][j], fa[s][j], a, 0, 0, 0);
                }
        }
        slot = slot + 1 == NS ? 0 : slot + 1;
    }
    __syncthreads();
    float *red = f32_sm + wave * T * RS;
#pragma unroll
    for (int g = 0; g < T * T / 256; ++g)
        *reinterpret_cast<float4 *>(red + li * RS + (T == 32 ? 8 * g : 0) + 4 * lh) =
            make_float4(slice_sum(acc, 4 * g), slice_sum(acc, 4 * g + 1), slice_sum(acc, 4 * g + 2), slice_sum(acc, 4 * g + 3));
    __syncthreads();
    if (owner) {
        const float *p = f32_sm + (er - m0) * RS + ec - n0;
        float4 v = *reinterpret_cast<const float4 *>(p);
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const float4 t = *reinterpret_cast<const float4 *>(p + w * T * RS);
            v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
        }
        if (whole) {
            v.x += eq.bias.x; v.y += eq.bias.y; v.z += eq.bias.z; v.w += eq.bias.w;
            epi_quad_store<EPI, float>(ep, er, ec, eq, v);
        } else {
            store_quad<EPI>(ep, er, ec, N, v);
        }
    }
}

template <int EPI>
__global__ void __launch_bounds__(256)
gemm_f32_tile_kernel(const float *__restrict__ A, const float *__restrict__ W, int M, int N, int K, GemmEpi ep)
{
    using namespace f32gemm;
    constexpr int B = 64, NS = 4;
    constexpr int STAGE = 2 * B * BK;                    // floats
    constexpr int LD = 4;                                // tile loads per wavefront and k tile
    constexpr int RS = B + 4;
    __shared__ __align__(16) float sm[NS * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nbm = (M + B - 1) / B, nbn = (N + B - 1) / B;
    int bm, bn;
    tile_of_block(nbm, nbn, bm, bn);
    const int m0 = bm * B, n0 = bn * B;
    const u32x4_t rs_a = descriptor(A + (size_t)m0 * K, min(B, M - m0) * K * 4);
    const u32x4_t rs_w = descriptor(W + (size_t)n0 * K, min(B, N - n0) * K * 4);
    const unsigned sm_lds = lds_address(sm);
    const int ld_r = lane >> 3;
    const int chunk = ((lane & 7) ^ (ld_r >> 1)) * 4;
    // wavefronts 0, 1: the halves of A's rows, 2, 3: of W's
    const u32x4_t rs = wave < 2 ? rs_a : rs_w;
    const int row0 = (wave & 1) * 32 + ld_r;
    const int kt_all = (K + BK - 1) / BK;
    auto issue = [&](int kt, int slot) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int k = kt * BK + (chunk ^ ((i & 1) << 4));
            const int voff = k < K ? ((row0 + i * 8) * K + k) * 4 : kOutside;
            dma(rs, sm_lds + (slot * STAGE + (wave * 32 + i * 8) * BK) * 4, voff);
        }
    };
    const int wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31, lk = lane >> 5, sw = swz_of_row(lr);
    // K in the slices of gemm_f32_slices_kernel (with one sum each), one after the other, added in the same order: the two
    // kernels give the same bits, so a row's result does not depend on how many rows the launch has.
    f32x16_t acc[1], sum;
    clear_sums<1, 16>(acc);
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r] = 0.0f;
    int slice = 0, slice_end = 0;
    auto next_slice = [&](int done) {                    // the first slice that ends behind k tile `done`
        while (slice < kSlices && slice_end <= done) slice_end = kt_all * ++slice / kSlices;
    };
    next_slice(0);
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue(s, s);
    for (int kt = 0; kt < kt_all; ++kt) {
        wait_loads<(NS - 2) * LD>();
        wait_lds();
        asm volatile("s_barrier" : : : "memory");        // tile kt is there for everyone, tile kt-1's slot is free
        issue(kt + NS - 1, (kt + NS - 1) & (NS - 1));
        const float *as = sm + (kt & (NS - 1)) * STAGE + (wm * 32 + lr) * BK;
        const float *ws = sm + (kt & (NS - 1)) * STAGE + (B + wn * 32 + lr) * BK;
        f32x4_t fa[4], fw[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int ch = ((s * 2 + lk) ^ sw) * 4;
            fa[s] = *reinterpret_cast<const f32x4_t *>(as + ch);
            fw[s] = *reinterpret_cast<const f32x4_t *>(ws + ch);
        }
        mfma_k32(fw, fa, acc);
        if (kt + 1 == slice_end) {
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[r] += slice_sum(acc, r);
            clear_sums<1, 16>(acc);
            next_slice(kt + 1);
        }
    }
    wait_loads<0>();
    __syncthreads();
    float *stage = sm;                                   // [B][RS]
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4 *>(stage + (wm * 32 + lr) * RS + wn * 32 + 8 * g + 4 * lk) =
            make_float4(sum[4 * g], sum[4 * g + 1], sum[4 * g + 2], sum[4 * g + 3]);
    __syncthreads();
    if (EPI != EPI_ARGMAX || ep.out) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int r = it * 16 + (tid >> 4), c = (tid & 15) * 4;
            if (m0 + r < M && n0 + c < N)
                store_quad<EPI>(ep, m0 + r, n0 + c, N, *reinterpret_cast<const float4 *>(stage + r * RS + c));
        }
    }
    if constexpr (EPI == EPI_ARGMAX) {
        // four lanes per row, sixteen columns each, ascending; ties keep the lowest index
        const int r = tid >> 2, row = m0 + r;
        const uint32_t rk = ep.temp > 0.0f ? srm_rowkey(ep.seed, epi_pos(ep, row, M), (uint32_t)row + ep.row_base) : 0u;
        float bv = -INFINITY;
        int bi = 0x7fffffff;
        for (int c = 0; c < 16; ++c) {
            const int col = n0 + (tid & 3) * 16 + c;
            if (col >= N) break;
            float v = stage[r * RS + (tid & 3) * 16 + c] + (ep.bias ? ep.bias[col] : 0.0f);
            if (ep.temp > 0.0f) v += ep.temp * srm_gumbel(rk, (uint32_t)col);
            if (arg_better(v, col, bv, bi)) { bv = v; bi = col; }
        }
#pragma unroll
        for (int off = 1; off <= 2; off <<= 1) {
            const float ov = __shfl_xor(bv, off, kWave);
            const int oi = __shfl_xor(bi, off, kWave);
            if (arg_better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if ((tid & 3) == 0 && row < M) {
            ep.part_val[(int64_t)bn * M + row] = bv;
            ep.part_idx[(int64_t)bn * M + row] = bi;
        }
    }
}
