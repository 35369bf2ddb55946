// bf16 GEMMs of few output tiles: out = epilogue(A W^T + bias), same contract and epilogues as gemm_bf16_kernel.
//
// A launch with at most one tile per CU takes as long as one tile's trip through K.  In gemm_bf16_kernel that trip is
// a chain: load into LDS, barrier, LDS reads, one MFMA per wavefront and substep.  Here a work-group owns a
// (16 RT) x (16 CT) tile and its eight wavefronts cut K between them: each contracts its own slice of K for the whole
// tile, streaming it through a ring of NS line steps (64 k, a cache line per row) of its own in LDS, so that no
// wavefront waits for another one inside the loop and two wavefronts per SIMD cover each other's LDS reads.  The
// partial tiles meet in LDS and are added in slice order: the result does not depend on scheduling, and all tile
// shapes give the same bits.
// What bounds it: the trip of the first loads and the launch (2.6 us for the smallest), then the rate at which a CU
// takes cache lines.  Loading the MFMA operands straight into registers needs no LDS, but lanes l .. l+3 of such a
// load lie in four rows, and the address unit then takes one lane per clock: four times slower.
// Measured (graph of launches back to back over 16 weight matrices, us, 64x64 tile of gemm_bf16_kernel -> this):
// 1 x 1024 x 1024: 7.2 -> 3.1; 37 x 4096 x 1024: 8.1 -> 4.4; 64 x 1024 x 4096: 17.8 -> 5.2; 509 x 1024 x 4096:
// 18.5 -> 11.7; 256 x 2048 x 512: 6.4 -> 4.4; 1024 x 512 x 2048: 11.3 -> 6.9 (rows x columns x K).
#pragma once
#include "gemm.hpp"

// LDS bytes of one wavefront: its ring, which later holds its partial tile
template <int RT, int CT, int NS, bool LNA>
constexpr int slices_wave_lds()
{
    constexpr int ring = NS * 16 * (LNA ? CT : RT + CT) * 128, part = 16 * RT * (16 * CT + 4) * 4;
    return ring > part ? ring : part;
}

// LNA (tiles of 16 rows, K <= 1024): the A operand is not read from memory but made by the work-group itself,
// A = LayerNorm(ep.ln_x rows) in the arithmetic of ln_kernel, written once as a panel [K / 64][16 rows][64] behind the
// rings, in the layout of a ring's A tile, while the first W loads travel.  Every column block normalises the few rows
// again, which is cheaper than the LayerNorm launch it replaces.  Panel rows >= M feed accumulator rows that no
// epilogue stores.
constexpr int kSliceWaves = 8;
template <int EPI, int RT, int CT, int NS, bool LNA = false>
__global__ void __launch_bounds__(kSliceWaves * 64)
gemm_bf16_slices_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ W, int M, int N, int K, GemmEpi ep)
{
    constexpr int NW = kSliceWaves, BM = 16 * RT, BN = 16 * CT, NTHR = NW * 64;
    static_assert(!LNA || BM == kLnaRows, "the panel holds one row tile");
    constexpr int RS = BN + 4;                       // row stride of a partial tile in LDS, floats
    constexpr int GPR = BN / 4, G = BM * GPR;        // float4 groups per row and per tile
    constexpr int NQ = (G + NTHR - 1) / NTHR;        // groups per thread in the epilogue
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int WAVE_LDS = slices_wave_lds<RT, CT, NS, LNA>();

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    const bool probe = ep.clk != nullptr && (int64_t)blockIdx.x < ep.clk_blocks;      // (see GemmEpi::clk)
    unsigned long long clk_c0 = 0, clk_t0 = 0, clk_c1 = 0, clk_t1 = 0, clk_c2 = 0, clk_t2 = 0;
    if (probe) { clk_c0 = clock64(); clk_t0 = wall_clock64(); }
    const int nbm = (M + BM - 1) / BM, nbn = (N + BN - 1) / BN;
    int bm, bn;
    tile_of_block(nbm, nbn, bm, bn);
    const int m0 = bm * BM, n0 = bn * BN;

    // operands: descriptors of exactly this tile's rows (rows past M or N arrive as zeros)
    auto descriptor = [](const bf16 *base, int bytes) {
        u32x4_t rs;
        const unsigned long long a = reinterpret_cast<unsigned long long>(base);
        rs[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
        rs[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));             // stride 0: raw buffer
        rs[2] = __builtin_amdgcn_readfirstlane((unsigned)bytes);
        rs[3] = 0x00020000u;
        return rs;
    };
    const u32x4_t rs_a = descriptor(A + (size_t)m0 * K, min(BM, M - m0) * K * 2);
    const u32x4_t rs_w = descriptor(W + (size_t)n0 * K, min(BN, N - n0) * K * 2);
    // Tile loads: one instruction moves 8 rows x 128 bytes, lane (r = l >> 3, slot = l & 7) fetches chunk
    // slot ^ swz(row) of its row (the swizzled layout of gemm_bf16_kernel).  They are issued from an asm statement:
    // a load that the compiler knows to write LDS makes it wait for all outstanding loads in front of the next LDS
    // read it cannot prove disjoint.  The waits are the explicit ones below.
    constexpr int LA = LNA ? 0 : BM / 8, LW = BN / 8, LPS = LA + LW;   // loads per line step
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    unsigned char *ring = smem_raw + wave * WAVE_LDS;
    const unsigned ring_lds = __builtin_amdgcn_readfirstlane(
        (unsigned)reinterpret_cast<unsigned long long>((lds_byte *)ring));
    int off[LA > LW ? LA : LW];
#pragma unroll
    for (int i = 0; i < (LA > LW ? LA : LW); ++i) {
        const int r = 8 * i + (lane >> 3);
        off[i] = (r * K + (((lane & 7) ^ swz_of_row(r)) << 3)) * 2;
    }
    // this wavefront's line steps: none if K / 64 < NW leaves it without
    const int kt = K / 64, first = wave * kt / NW, steps = (wave + 1) * kt / NW - first;
    const int kb = first * 128;                      // bytes
    auto dma = [&](const u32x4_t &rs, unsigned lds_dst, int voff, int soff) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(lds_dst), "v"(voff), "s"(rs), "s"(soff)
                     : "memory");
    };
    auto load = [&](int slot, int step) {
        const unsigned dst = ring_lds + slot * (LPS * 1024);
        static_for<0, LW>([&](auto i_) { dma(rs_w, dst + (LA + decltype(i_)::value) * 1024, off[decltype(i_)::value], kb + step * 128); });
        static_for<0, LA>([&](auto i_) { dma(rs_a, dst + decltype(i_)::value * 1024, off[decltype(i_)::value], kb + step * 128); });
    };
    // all but the youngest n loads have landed (loads that the compiler issues in between only make it wait longer)
#define SRM_WAIT_LOADS(n) asm volatile("s_waitcnt vmcnt(%0)" : : "i"(n) : "memory")
    static_for<0, NS>([&](auto d_) {
        if (decltype(d_)::value < steps) load(decltype(d_)::value, decltype(d_)::value);
    });

    // what the epilogue needs from memory, requested behind the first operands
    int row[NQ], col[NQ];
    bool in[NQ];
    EpiQuad eq[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int g = tid + q * NTHR;
        row[q] = m0 + g / GPR;
        col[q] = n0 + g % GPR * 4;
        in[q] = g < G && row[q] < M && col[q] < N;   // N is a multiple of 4 (the launcher checks)
        if (in[q]) eq[q] = epi_quad_request<EPI>(ep, row[q], col[q]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (LNA) layernorm_panel<NW>(ep, min(BM, M - m0), K, wave, lane, [&](int r, int c, float4 o) {
        store4(reinterpret_cast<bf16 *>(smem_raw + NW * WAVE_LDS + (c >> 6) * 2048 + r * 128 +
                                        ((((c & 63) >> 3) ^ swz_of_row(r)) << 4)) + (c & 7), o);
    }, m0);

    f32x4_t acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto products = [&](int slot, int step) {        // transposed: a lane holds four columns of one row
        const unsigned char *ws = ring + slot * (LPS * 1024) + LA * 1024;
        const unsigned char *as = LNA ? smem_raw + NW * WAVE_LDS + (first + step) * (BM * 128) : ring + slot * (LPS * 1024);
        bf16x8_t fa[2][RT], fw[2][CT];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ch = lr * 128 + (((h * 4 + lq) ^ swz_of_row(lr)) << 4);
#pragma unroll
            for (int j = 0; j < CT; ++j) fw[h][j] = *reinterpret_cast<const bf16x8_t *>(ws + j * 2048 + ch);
#pragma unroll
            for (int i = 0; i < RT; ++i) fa[h][i] = *reinterpret_cast<const bf16x8_t *>(as + i * 2048 + ch);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < CT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][j], fa[h][i], acc[i][j], 0, 0, 0);
    };
    if (probe) { clk_c1 = clock64(); clk_t1 = wall_clock64(); }
    int slot = 0, at_step = 0;
    for (int s = NS; s < steps; ++s, ++at_step) {
        SRM_WAIT_LOADS((NS - 1) * LPS);
        products(slot, at_step);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");           // the slot has been read
        load(slot, s);
        slot = slot + 1 == NS ? 0 : slot + 1;
    }
    if (steps < NS) SRM_WAIT_LOADS(0);               // (a ring that was never full: the counts below do not hold)
    static_for<0, NS>([&](auto t_) {
        if (at_step < steps) {
            SRM_WAIT_LOADS((NS - 1 - decltype(t_)::value) * LPS);
            products(slot, at_step);
            slot = slot + 1 == NS ? 0 : slot + 1;
            ++at_step;
        }
    });
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");               // the ring becomes the partial tile
#undef SRM_WAIT_LOADS

    float *mine = reinterpret_cast<float *>(ring);   // [BM][RS]
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
            *reinterpret_cast<f32x4_t *>(mine + (16 * i + lr) * RS + 16 * j + 4 * lq) = acc[i][j];
    __syncthreads();
    if (probe) { clk_c2 = clock64(); clk_t2 = wall_clock64(); }
    const float *part = reinterpret_cast<const float *>(smem_raw);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (!in[q]) continue;
        const float *p = part + (row[q] - m0) * RS + col[q] - n0;
        float4 v = eq[q].bias;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 t = *reinterpret_cast<const float4 *>(p + w * (WAVE_LDS / 4));
            v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
        }
        epi_quad_store<EPI, bf16>(ep, row[q], col[q], eq[q], v);
    }
    if (probe) {
        __builtin_amdgcn_s_waitcnt(0);                // this wave's stores have completed
        if (tid == 0) {
            unsigned long long *p = ep.clk + 8 * (int64_t)blockIdx.x;
            p[0] = clk_t0; p[1] = clk_t1; p[2] = clk_t2; p[3] = wall_clock64(); p[4] = clk_c1; p[5] = clk_c2;
            p[6] = (unsigned long long)__builtin_amdgcn_s_getreg((31 << 11) | 4) |        // HW_ID
                   ((unsigned long long)__builtin_amdgcn_s_getreg((3 << 11) | 20) << 32);  // XCC_ID
            p[7] = clk_c0;
        }
    }
}
