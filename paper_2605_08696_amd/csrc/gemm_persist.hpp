// The 256x256 bf16 MFMA GEMM (same contract and epilogues as gemm_bf16_kernel in gemm.hpp: out = epilogue(A W^T + bias)),
// as a persistent kernel: one work-group per CU walks its output tiles v = blockIdx.x, blockIdx.x + gridDim.x, ... and the
// LDS ring runs from one output tile into the next, so that a tile that is not a CU's first starts its MFMAs at once
// instead of after a work-group launch and a cold round trip to memory.
//
// LDS (160 KB) is a ring of five units of 32 KB, each an A tile or a W tile of 256 rows x 64 k in the swizzled layout of
// gemm_bf16_kernel.  k tile T (counted on through all output tiles) has A in unit 2T mod 5 and W in unit 2T + 1 mod 5:
//     half 0 of T: MFMAs of its first 32 k | operands of its second half | loads of A of T+2 (unit 2T+4: W of T-1 is done)
//     barrier: T+1 has landed, T has been read by all
//     half 1 of T: MFMAs of the other 32 k | operands of T+1's first half | loads of W of T+2 (unit 2T: A of T is done)
// With two and a half tiles instead of two, loads are issued in both halves: a CU takes a load of 1 KB in about 16
// clocks, 1024 per k tile of 2048 clocks of MFMAs, and all in one half they make the wavefronts wait for their turn to
// issue (16384 x 1024 x 4096: 2555 clocks per k tile with the loads in one half, 2405 in both, 2217
// without any).
// The epilogue stages its stores through the unit of the last k tile's W (32 KB, free since that k tile's barrier),
// sixteen rows at a time; everything else keeps filling under it.
#pragma once
#include "gemm.hpp"

constexpr int kPersistLds = 160 * 1024;

// The epilogue: acc[t][j] of lane (lq, lr) is row t*16 + lr, columns j*16 + 4lq .. +3 of the wave tile (128 x 64; 2 x 4
// wave tiles).  Sixteen rows at a time pass through a wave-private stage [16][64] in `stage` (16-byte chunk c of row r at
// chunk c ^ r: writes and reads free of bank conflicts), so that global accesses are 16-byte vectors over 256 bytes of a
// row.  Old values (residual stream, recurrent state) are requested for 32 rows at a time, in front of the stage.
//
// EPI_RESID_LN also makes the LayerNorm of the new rows, which a launch of its own reads again (16384 rows of 1024: 18.2 us): the new
// values stay in the accumulators' registers, the tiles of a row exchange the mean and the squared deviations of their 256
// columns (two-pass within a wavefront's 64, combined by Chan's formula) through memory, and each normalises its own columns.
// The tiles of a row tile are worked on at the same time, next to each other on an XCD, but nothing promises that: a
// work-group asks ln_polls times (kLnBegun times while some tile has not even been begun: where several streams or processes have
// such launches, their work-groups would otherwise hold CUs that each other's wait for: decode steps of 16384 rows on three streams,
// us per step, 9723 | 6993, LayerNorm launches 6824), and if some tile is still missing it leaves its columns to whoever leaves the
// last one.  Both are one atomic on the row tile's word, so that exactly one of them does it.  (16384 x 1024, both kinds of launch, us, with a
// LayerNorm launch behind | this: 98.7 | 92.9, of which the sums and the normalising are about 5, the exchange 2, the stores 5.)
constexpr int kLnTiles = 4;                          // column tiles of a row at most
constexpr unsigned kLnBegun = 32;                    // some 12 us
template <typename BARRIER>
__device__ __forceinline__ unsigned persist_ln_exchange(const GemmEpi &ep, const float2 *part, float2 *rows, int M, int m0, int bm, int bn,
                                                        int nbn, int tid, BARRIER &&lds_barrier)
{
    // part [4 wavefronts of 64 columns][256 rows] -> this tile's pair for the others
    unsigned long long *const stats = reinterpret_cast<unsigned long long *>(ep.ln_stats);
    auto pair = [](unsigned long long v) {
        return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
    };
    if (tid < 256) {
        float mean = 0.0f, dev = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) mean += part[w * 256 + tid].x;
        mean *= 0.25f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float2 t = part[w * 256 + tid];
            dev += t.y + 64.0f * ((t.x - mean) * (t.x - mean));
        }
        if (m0 + tid < M)
            __hip_atomic_store(stats + (size_t)(m0 + tid) * nbn + bn, (unsigned long long)__float_as_uint(dev) << 32 | __float_as_uint(mean),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    lds_barrier();
    unsigned *const word = ep.ln_words + bm, *const said = reinterpret_cast<unsigned *>(rows + 256);
    if (tid == 0) {
        unsigned seen = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
        auto left = [&] { return (seen & 0xff) == (unsigned)nbn; };
        const bool last = left();
        for (unsigned polls = 0; !left() && polls < ep.ln_polls && (polls < kLnBegun || (seen >> 8 & 0xff) == (unsigned)nbn); ++polls)
            seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        said[0] = left();
        said[1] = last ? seen >> 16 : 0;             // whose columns this work-group makes besides its own
    }
    lds_barrier();
    if (__builtin_expect(!said[0], 0)) {             // tired of waiting: what is in memory is for whoever comes last
        if (tid == 0) {
            const unsigned seen = __hip_atomic_fetch_or(word, 0x10000u << bn, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            said[0] = (seen & 0xff) == (unsigned)nbn;
        }
        lds_barrier();
        if (!said[0]) return ~0u;
    }
    const unsigned others = said[1];
    if (tid < 256) {
        const size_t at = (size_t)min(m0 + tid, M - 1) * nbn;
        float2 t[kLnTiles];
        float mean = 0.0f, dev = 0.0f;
#pragma unroll
        for (int b = 0; b < kLnTiles; ++b)
            t[b] = pair(__hip_atomic_load(stats + at + min(b, nbn - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
        for (int b = 0; b < kLnTiles; ++b) mean += b < nbn ? t[b].x : 0.0f;
        mean /= (float)nbn;
#pragma unroll
        for (int b = 0; b < kLnTiles; ++b) dev += b < nbn ? t[b].y + 256.0f * ((t[b].x - mean) * (t[b].x - mean)) : 0.0f;
        rows[tid] = make_float2(mean, 1.0f / sqrtf(dev / (float)(nbn * 256) + ep.ln_eps));
    }
    if (others != 0 && tid == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");     // (of the cache that the wavefronts share)
    lds_barrier();
    return others;
}
// The columns of the tiles `others` of these rows, behind its own (whose values are registers until then): eight rows of a wavefront
// in flight.  (One after the other, in front of its own columns, a tile took some 50 us.)
template <typename TAct>
__device__ __forceinline__ void persist_ln_others(const GemmEpi &ep, const float2 *rows, int M, int m0, unsigned others, int tid)
{
    constexpr int U = 8;
    for (; others; others &= others - 1) {
        const int col = __builtin_ctz(others) * 256 + (tid & 63) * 4;
        const float4 g = load4(ep.ln_g + col), c = load4(ep.ln_b + col);
#pragma unroll 1
        for (int r0 = (tid >> 6) * U; r0 < 256 && m0 + r0 < M; r0 += 8 * U) {
            float4 x[U];
#pragma unroll
            for (int i = 0; i < U; ++i) x[i] = load4(static_cast<const float *>(ep.out) + (int64_t)min(m0 + r0 + i, M - 1) * ep.ldo + col);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const float2 s = rows[r0 + i];
                if (m0 + r0 + i < M)
                    store4(static_cast<TAct *>(ep.ln_out) + (int64_t)(m0 + r0 + i) * ep.ldo + col,
                           make_float4((x[i].x - s.x) * s.y * g.x + c.x, (x[i].y - s.x) * s.y * g.y + c.y,
                                       (x[i].z - s.x) * s.y * g.z + c.z, (x[i].w - s.x) * s.y * g.w + c.w));
            }
        }
    }
}

template <int EPI, typename TAct, bool STORE, typename BARRIER>
__device__ __forceinline__ void persist_epilogue(f32x4_t (&acc)[8][4], unsigned char *stage_base, const GemmEpi &ep, int M, int N,
                                                 int m0, int n0, int bn, const int tid, BARRIER &&lds_barrier)
{
    constexpr int TM = 8, TN = 4, WTM = 128, WTN = 64, WN = 4;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int lr = lane & 15, lq = lane >> 4;
    const int wcol0 = n0 + wn * WTN, wrow0 = m0 + wm * WTM;
    const bool inside = n0 + 256 <= N && m0 + 256 <= M;                // block-uniform
    // EPI_ARGMAX: every lane leaves the best of its sixteen columns of a row in the stage, entry wn*4 + lq of [256 rows][16]
    // (at entry ^ row: no bank conflicts); two lanes per row then take the best of the sixteen.  With logits to store the
    // stage is in use until all rows are through: the winners wait in registers, their codes in four bits each.
    [[maybe_unused]] uint2 *red = reinterpret_cast<uint2 *>(stage_base);
    [[maybe_unused]] float best_val[TM];
    [[maybe_unused]] unsigned best_code = 0;
    [[maybe_unused]] uint32_t key[TM] = {};
    [[maybe_unused]] auto leave = [&](int t, RowBest b, int col0) {
        red[(wm * WTM + t * 16 + lr) * 16 + ((wn * 4 + lq) ^ lr)] = row_best_entry(b, col0);
    };
    [[maybe_unused]] auto choose = [&](auto choice_c, auto t_) {
        constexpr int C = decltype(choice_c)::value, t = decltype(t_)::value;
        best_val[t] = -INFINITY;
        // (no noise for rows past M, whose entries nobody keeps)
        if ((C & CHOICE_NOISE) && wrow0 + t * 16 >= M) return;         // wave-uniform
        // (opaque: what is derived from the columns is formed for each row, not held in registers across all rows,
        // of which the noise had none left: 300 x 32000 x 512 with a temperature 2.7 us shorter)
        int col0 = wcol0 + 4 * lq;
        asm volatile("" : "+v"(col0));
        const RowBest b = row_best<C>(ep, acc[t], key[t], N, col0);
        if constexpr (STORE) {
            best_val[t] = b.val;
            best_code |= (unsigned)b.code << (4 * t);
        } else {
            leave(t, b, col0);
        }
    };
    [[maybe_unused]] auto keys = [&](auto choice_c) {
        if constexpr (decltype(choice_c)::value & CHOICE_NOISE) noise_keys(ep, wrow0 + lr, M, key);
    };
    if constexpr (STORE) {
        f32x4_t *stage = reinterpret_cast<f32x4_t *>(stage_base) + wave * (16 * 16);   // [16 rows][16 chunks]
        const int s_row = lane >> 4, s_chunk = lane & 15;
        const int gcol = wcol0 + s_chunk * 4;
        const unsigned lane_at = (unsigned)s_row * (unsigned)ep.ldo + s_chunk * 4;    // (the rest of an offset is uniform)
        // (EPI_RESID_LN: the tile's rows that exist, the hardware's range check leaves out the others; fewer registers than addresses)
        [[maybe_unused]] const auto x_rs = __builtin_amdgcn_make_buffer_rsrc(
            EPI == EPI_RESID_LN ? static_cast<float *>(ep.out) + (int64_t)m0 * ep.ldo : nullptr, 0, min(256, M - m0) * (int)ep.ldo * 4, 0x00020000);
        [[maybe_unused]] auto x_row = [&](int t, int it) { return ((wm * WTM + t * 16 + it * 4) * (int)ep.ldo + wcol0) * 4; };
        [[maybe_unused]] float2 kept[2];             // EPI_RESID_LN: mean and squared deviations of 64 columns of two rows
        auto slices = [&](auto inside_c, auto choice_c) {
            constexpr bool IN = decltype(inside_c)::value;
            auto row_of = [&](int t, int it) { return (int64_t)wrow0 + t * 16 + it * 4 + s_row; };
            auto exists = [&](int t, int it) { return IN || (row_of(t, it) < M && gcol < N); };
            // where the old values of a quad are read: one that exists
            auto at = [&](int t, int it) {
                if constexpr (IN) return (wrow0 + t * 16 + it * 4) * ep.ldo + wcol0 + (int64_t)lane_at;
                else return min(row_of(t, it), (int64_t)M - 1) * ep.ldo + min(gcol, N - 4);
            };
            static_for<0, TM / 2>([&](auto p_) {
                constexpr int t0 = 2 * decltype(p_)::value;
                [[maybe_unused]] float4 old[2][4];
                if constexpr (EPI == EPI_RESID || EPI == EPI_RESID_LN || EPI == EPI_MIX) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int it = 0; it < 4; ++it) {
                            if constexpr (EPI == EPI_RESID) old[h][it] = load4(static_cast<const float *>(ep.out) + at(t0 + h, it));
                            else if constexpr (EPI == EPI_RESID_LN) old[h][it] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, (int)lane_at * 4, x_row(t0 + h, it), 0));
                            else if (ep.state_half) old[h][it] = load_state4(static_cast<const f16 *>(ep.state), at(t0 + h, it) >> 2);
                            else old[h][it] = load_state4(static_cast<const float *>(ep.state), at(t0 + h, it) >> 2);
                        }
                }
                static_for<0, 2>([&](auto h_) {
                    constexpr int h = decltype(h_)::value, t = t0 + h;
                    [[maybe_unused]] float al[4], be[4], la = 0.0f;
                    [[maybe_unused]] int ps[4];
                    [[maybe_unused]] bool row_repeat = false;
                    if constexpr (EPI == EPI_MIX) {
                        const int hd = min(gcol, N - 4) / ep.dh;       // four consecutive channels lie in one head
                        row_repeat = hd < ep.hrow;
                        la = ep.lam[hd];
#pragma unroll
                        for (int it = 0; it < 4; ++it)
                            ps[it] = (int)(ep.pos_rows ? (uint32_t)ep.pos_rows[IN ? row_of(t, it) : min(row_of(t, it), (int64_t)M - 1)]
                                                       : epi_shared_pos(ep));
#pragma unroll
                        for (int it = 0; it < 4; ++it) {
                            const int pc = ps[it] >= 0 && ps[it] < ep.n_ctx ? ps[it] : 0;
                            al[it] = ep.alpha[(size_t)hd * ep.n_ctx + pc];
                            be[it] = ep.beta[(size_t)hd * ep.n_ctx + pc];
                        }
                    }
                    // (the choice in front of each sixteen rows' stores, which travel under the next rows' noise: a step of 300
                    // rows of a mid-sized model with temperature and logits 251.8 us | 247.1, of 900 for top-p 402.4 | 393.9)
                    if constexpr (EPI == EPI_ARGMAX) choose(choice_c, std::integral_constant<int, t>{});
#pragma unroll
                    for (int j = 0; j < TN; ++j) stage[lr * 16 + ((4 * j + lq) ^ lr)] = acc[t][j];
                    f32x4_t v[4];
#pragma unroll
                    for (int it = 0; it < 4; ++it) v[it] = stage[(it * 4 + s_row) * 16 + (s_chunk ^ (it * 4 + s_row))];
                    if constexpr (EPI == EPI_RESID_LN) {
#pragma unroll
                        for (int it = 0; it < 4; ++it) {               // (the row's first half of acc is in the stage)
                            const float4 o = old[h][it];
                            const f32x4_t w = f32x4_t{o.x + v[it][0], o.y + v[it][1], o.z + v[it][2], o.w + v[it][3]};
                            const float mean = row16_sum((w[0] + w[1]) + (w[2] + w[3])) * (1.0f / 64);
                            const float a = w[0] - mean, b = w[1] - mean, c = w[2] - mean, d = w[3] - mean;
                            const float dev = row16_sum((a * a + b * b) + (c * c + d * d));
                            // row t*16 + it*4 + s_row is kept by lane (4t + it) mod 16 of the sixteen that hold it
                            if (s_chunk == ((t * 4 + it) & 15)) {
                                kept[t / 4].x = mean;
                                kept[t / 4].y = dev;
                            }
                            acc[t][it] = w;
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, w), x_rs, (int)lane_at * 4, x_row(t, it), 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        return;
                    }
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        if (!exists(t, it)) continue;
                        const int64_t row = row_of(t, it);
                        const float4 w = make_float4(v[it][0], v[it][1], v[it][2], v[it][3]);
                        if constexpr (EPI == EPI_RESID) {
                            const float4 o = old[h][it];
                            store4(static_cast<float *>(ep.out) + row * ep.ldo + gcol,
                                   make_float4(o.x + w.x, o.y + w.y, o.z + w.z, o.w + w.w));
                        } else if constexpr (EPI == EPI_MIX) {
                            EpiQuad q;
                            q.old = old[h][it];
                            q.al = al[it]; q.be = be[it]; q.la = la;
                            epi_mix_store<TAct>(ep, row, gcol, q, ps[it] >= 0 && ps[it] < ep.n_ctx, row_repeat, w);
                        } else if constexpr (EPI == EPI_ARGMAX && IN) {
                            // (nontemporal, see epi_store4; the uniform part of the offset apart, which saves the registers of the rest)
                            float *const o = static_cast<float *>(ep.out) + ((wrow0 + t * 16 + it * 4) * ep.ldo + wcol0);
                            __builtin_nontemporal_store(f32x4_t{w.x, w.y, w.z, w.w}, reinterpret_cast<f32x4_t *>(o + lane_at));
                        } else {
                            epi_store4<EPI, TAct>(ep, row, gcol, w);
                        }
                    }
                });
            });
        };
        if constexpr (EPI == EPI_ARGMAX) {
            with_choice(ep, !inside, [&](auto choice_c) {
                keys(choice_c);
                slices(std::integral_constant<bool, !(decltype(choice_c)::value & CHOICE_EDGE)>{}, choice_c);
            });
        } else if constexpr (EPI == EPI_RESID_LN) {
            // (one form for all tiles: of two, whose new values meet behind them, each would have registers of its own for them)
            slices(std::false_type{}, std::integral_constant<int, CHOICE_EDGE>{});
            lds_barrier();                           // the stages have been read back
            float2 *const part = reinterpret_cast<float2 *>(stage_base), *const rows = part + 4 * 256;
#pragma unroll
            for (int q = 0; q < 2; ++q) {            // row 4t + it = s_chunk + 16 q of this lane's
                const int k = s_chunk + 16 * q;
                part[wn * 256 + wm * WTM + (k >> 2) * 16 + (k & 3) * 4 + s_row] = kept[q];
            }
            lds_barrier();
            const unsigned others = persist_ln_exchange(ep, part, rows, M, m0, m0 >> 8, bn, N >> 8, tid, lds_barrier);
            if (others == ~0u) return;
            // (addresses formed anew, from an opaque copy: those of the slices' stores would be held in registers until here)
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int r0 = wm * WTM + (ln >> 4), col = wcol0 + (ln & 15) * 4;
            const float4 gain = load4(ep.ln_g + col), shift = load4(ep.ln_b + col);            // (whole tiles of columns)
            const auto out_rs = __builtin_amdgcn_make_buffer_rsrc(static_cast<TAct *>(ep.ln_out) + (int64_t)m0 * ep.ldo, 0,
                                                                  min(256, M - m0) * (int)ep.ldo * (int)sizeof(TAct), 0x00020000);
            const int to = (r0 * (int)ep.ldo + col) * (int)sizeof(TAct);
            static_for<0, TM>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const float2 s = rows[r0 + t * 16 + it * 4];
                    const f32x4_t x = acc[t][it];
                    const bf16x2_t lo = __builtin_convertvector(f32x2_t{(x[0] - s.x) * s.y * gain.x + shift.x, (x[1] - s.x) * s.y * gain.y + shift.y}, bf16x2_t);
                    const bf16x2_t hi = __builtin_convertvector(f32x2_t{(x[2] - s.x) * s.y * gain.z + shift.z, (x[3] - s.x) * s.y * gain.w + shift.w}, bf16x2_t);
                    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)}, out_rs, to,
                                                          (t * 16 + it * 4) * (int)ep.ldo * (int)sizeof(TAct), 0);
                }
            });
            if (__builtin_expect(others != 0, 0)) persist_ln_others<TAct>(ep, rows, M, m0, others, tid);
        } else if (inside) {
            slices(std::true_type{}, std::integral_constant<int, CHOICE_PLAIN>{});
        } else {
            slices(std::false_type{}, std::integral_constant<int, CHOICE_EDGE>{});
        }
    } else if constexpr (EPI == EPI_ARGMAX) {
        with_choice(ep, wcol0 + WTN > N, [&](auto choice_c) {
            keys(choice_c);
            static_for<0, TM>([&](auto t_) { choose(choice_c, t_); });
        });
    }
    if constexpr (EPI == EPI_ARGMAX) {
        if constexpr (STORE) {
            lds_barrier();                           // the stages have been read back
#pragma unroll
            for (int t = 0; t < TM; ++t)
                leave(t, RowBest{best_val[t], (int)(best_code >> (4 * t) & 15)}, wcol0 + 4 * lq);
        }
        lds_barrier();
        const int row = m0 + (tid >> 1);
        float bv = -INFINITY;
        int bi = 0x7fffffff;
        best_entry<8>(red + tid * 8, bv, bi);
        best_of_lanes<2>(bv, bi);
        if ((tid & 1) == 0 && row < M) {
            ep.part_val[(int64_t)bn * M + row] = bv;
            ep.part_idx[(int64_t)bn * M + row] = bi;
        }
    }
}

template <int EPI, typename TAct>
__global__ void __launch_bounds__(512)
gemm_bf16_persist_kernel(const bf16 *__restrict__ A, const bf16 *__restrict__ W, int M, int N, int K, GemmEpi ep)
{
    constexpr int BM = 256, BN = 256, WM = 2, WN = 4, BK = 64;
    constexpr int NTHR = WM * WN * 64;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int TM = WTM / 16, TN = WTN / 16;
    constexpr int UNITS = 5, UNIT = 256 * BK * 2;    // bytes
    constexpr int LD_IT = UNIT / 16 / NTHR;          // loads per wavefront and unit
    static_assert(UNITS * UNIT <= kPersistLds, "the ring is the LDS");
    static_assert(WM * WN * 16 * WTN * 4 <= UNIT && BM * 16 * 8 <= UNIT, "the epilogue's stage fits a unit");

    extern __shared__ __align__(16) unsigned char smem_raw[];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int lr = lane & 15, lq = lane >> 4;

    const int nbm = (M + BM - 1) / BM, nbn = (N + BN - 1) / BN, nblk = nbm * nbn;
    const int KT = K / BK;                           // >= 2 (the launcher checks)

    // Tile loads: buffer_load ... lds, one wave instruction = 8 rows x 128 bytes, lane (r = l >> 3, slot = l & 7)
    // fetches chunk slot ^ swz(r) of its row.  A descriptor covers exactly one tile's rows of A or W (rows past
    // M or N, and everything of a descriptor of zero bytes, arrive as zeros).  They are issued from an asm
    // statement: a load that the compiler knows to write LDS makes it wait for all outstanding loads in front
    // of the next LDS read it cannot prove disjoint.  The waits are the explicit ones below.
    constexpr int ROWS_PER_IT = NTHR / 8;
    const int ld_r = tid >> 3, ld_c = tid & 7;
    const int ld_voff = (ld_r * K + ((ld_c ^ swz_of_row(ld_r)) << 3)) * 2;       // bytes
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const unsigned ring_lds = __builtin_amdgcn_readfirstlane(
        (unsigned)reinterpret_cast<unsigned long long>((lds_byte *)smem_raw));
    auto descriptor = [](const void *base, int bytes) {
        u32x4_t rs;
        const unsigned long long a = reinterpret_cast<unsigned long long>(base);
        rs[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
        rs[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));             // stride 0: raw buffer
        rs[2] = __builtin_amdgcn_readfirstlane((unsigned)bytes);
        rs[3] = 0x00020000u;
        return rs;
    };
    // load number i of the unit at ring offset `unit`, from k tile kq
    auto dma_one = [&](int i, const u32x4_t &rs, int kq, unsigned unit) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(ring_lds + unit + (i * ROWS_PER_IT + wave * 8) * (BK * 2)), "v"(ld_voff), "s"(rs),
                       "s"((i * ROWS_PER_IT * K + kq * BK) * 2)
                     : "memory");
    };
    auto dma_unit = [&](const u32x4_t &rs, int kq, unsigned unit) {
        static_for<0, LD_IT>([&](auto i_) { dma_one(decltype(i_)::value, rs, kq, unit); });
    };
    struct Tile {
        int m0, n0, bn;
        u32x4_t ra, rw;
    };
    auto tile_at = [&](int v) {
        Tile t;
        const bool exists = v < nblk;
        int bm;
        tile_of_pid(exists ? v : 0, nbm, nbn, bm, t.bn);
        t.m0 = bm * BM;
        t.n0 = t.bn * BN;
        t.ra = descriptor(A + (size_t)t.m0 * K, exists ? min(BM, M - t.m0) * K * 2 : 0);
        t.rw = descriptor(W + (size_t)t.n0 * K, exists ? min(BN, N - t.n0) * K * 2 : 0);
        return t;
    };
    // the bias of this lane's columns n0 + wn*64 + j*16 + 4lq .. +3 (zeros past N, which is a multiple of 4)
    f32x4_t bq[TN];
    auto bias_request = [&](int n0) {
        // (n0 < N always.  A size clamped at zero as well is formed in a vector register, by v_med3, and each load becomes
        // a loop over lanes with a wait for everything in flight, k tiles on their way included)
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(ep.bias ? ep.bias + n0 : nullptr), 0, ep.bias ? min(BN, N - n0) * 4 : 0, 0x00020000);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            bq[j] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rb, (wn * WTN + j * 16 + 4 * lq) * 4, 0, 0));
    };
#define SRM_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
    // a barrier that orders LDS accesses only
    auto lds_barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    // LDS byte offsets of this lane's first operands of half 0 in a unit; those of half 1 lie 64 bytes across
    typedef const __attribute__((address_space(3))) bf16x8_t lds_frag;
    const unsigned a_lds = ring_lds + (wm * WTM + lr) * (BK * 2) + ((lq ^ swz_of_row(lr)) << 4);
    const unsigned b_lds = ring_lds + (wn * WTN + lr) * (BK * 2) + ((lq ^ swz_of_row(lr)) << 4);
    bf16x8_t fa[2][TM], fb[2][TN];                   // one operand set per half of a k tile
    f32x4_t acc[TM][TN];
    // operand number r of half h of the k tile in units ua, ub: the first TM are of A, the rest of W
    auto read_one = [&](auto r_, auto h_, unsigned ua, unsigned ub) {
        constexpr int r = decltype(r_)::value, h = decltype(h_)::value;
        if constexpr (r < TM) fa[h][r] = *(lds_frag *)((a_lds ^ (h * 64)) + ua + r * (16 * BK * 2));
        else fb[h][r - TM] = *(lds_frag *)((b_lds ^ (h * 64)) + ub + (r - TM) * (16 * BK * 2));
    };
    constexpr std::integral_constant<int, 0> h0{};
    constexpr std::integral_constant<int, 1> h1{};
    // MFMAs of half h, transposed (MFMA rows run over N); pinned behind the q-th of them its share of the operand reads
    // of the other half, over the first three quarters, and of the loads of a unit, over the first quarter
    auto half = [&](auto h_, unsigned ua, unsigned ub, const u32x4_t &rs, int kq, unsigned unit) {
        constexpr int S_ = TM * TN, h = decltype(h_)::value;
        static_for<0, S_>([&](auto q_) {
            constexpr int q = decltype(q_)::value;
            acc[q / TN][q % TN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][q % TN], fa[h][q / TN], acc[q / TN][q % TN], 0, 0, 0);
            static_for<0, TM + TN>([&](auto r_) {
                if constexpr (decltype(r_)::value * (S_ * 3 / 4) / (TM + TN) == q)
                    read_one(r_, std::integral_constant<int, 1 - h>{}, ua, ub);
            });
            static_for<0, LD_IT>([&](auto l_) {
                if constexpr (decltype(l_)::value * (S_ / 4) / LD_IT == q) dma_one(decltype(l_)::value, rs, kq, unit);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // the epilogues that hold old values leave no registers for the operands that the last k tile has read ahead
    constexpr bool REREAD = EPI == EPI_RESID || EPI == EPI_RESID_LN || EPI == EPI_MIX;

    int v = blockIdx.x;                              // gridDim.x <= nblk: every work-group has a first tile
    Tile cur = tile_at(v);
    unsigned long long clk_c0 = 0, clk_t0 = 0, clk_c1 = 0, clk_t1 = 0, clk_c2 = 0, clk_t2 = 0;
    if (ep.clk) { clk_c0 = clock64(); clk_t0 = wall_clock64(); }
    bias_request(cur.n0);
    __builtin_amdgcn_sched_barrier(0);
    dma_unit(cur.ra, 0, 0);
    dma_unit(cur.rw, 0, UNIT);
    dma_unit(cur.ra, 1, 2 * UNIT);
    dma_unit(cur.rw, 1, 3 * UNIT);
    SRM_WAIT_VM(2 * LD_IT);                          // loads return in order: the bias and k tile 0 are there
    lds_barrier();
    static_for<0, TM + TN>([&](auto r_) { read_one(r_, h0, 0, UNIT); });

    unsigned u = 0;                                  // unit of A of this k tile; the five units from there on:
    auto at = [&](unsigned k) { const unsigned x = u + k; return (x >= UNITS ? x - UNITS : x) * UNIT; };
    for (;;) {
        const bool probe = ep.clk != nullptr && v < ep.clk_blocks;
        const int vn = v + (int)gridDim.x;
        const Tile nxt = tile_at(vn);                // of zero size behind the last tile
        if constexpr (EPI == EPI_RESID_LN)
            if (threadIdx.x == 0) __hip_atomic_fetch_add(ep.ln_words + (cur.m0 >> 8), 0x100u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < TN; ++j)                 // the accumulators start at the bias of their column
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i][j] = bq[j];
        __builtin_amdgcn_sched_barrier(0);
        if (probe) { clk_c1 = clock64(); clk_t1 = wall_clock64(); }

        for (int kt = 0; kt < KT; ++kt) {
            const bool ahead = kt + 2 >= KT;
            const u32x4_t ra = ahead ? nxt.ra : cur.ra, rw = ahead ? nxt.rw : cur.rw;
            const int kq = ahead ? kt + 2 - KT : kt + 2;
            half(h0, at(0), at(1), ra, kq, at(4));
            SRM_WAIT_VM(LD_IT);                      // k tile T+1 has landed
            lds_barrier();                           // ... for everyone, and T's units are free
            half(h1, at(2), at(3), rw, kq, at(0));
            u = u + 2 >= UNITS ? u + 2 - UNITS : u + 2;
        }
        if (probe) { clk_c2 = clock64(); clk_t2 = wall_clock64(); }

        // (the thread index through an opaque copy: what the epilogue derives from it is computed here, per
        // tile, and not once in front of the tile loop, where it would be held in registers across every k loop)
        int tid_e = threadIdx.x;
        asm volatile("" : "+v"(tid_e));
        auto epilogue = [&](auto store_c) {
            persist_epilogue<EPI, TAct, decltype(store_c)::value>(acc, smem_raw + at(4), ep, M, N, cur.m0, cur.n0, cur.bn, tid_e,
                                                                  lds_barrier);
        };
        // The next bias is requested in front of the epilogue, unless that leaves no registers for it.
        if (EPI == EPI_ARGMAX && ep.out) {
            epilogue(std::true_type{});
            bias_request(nxt.n0);
        } else {
            if constexpr (EPI != EPI_MIX && EPI != EPI_RESID_LN) bias_request(nxt.n0);
            __builtin_amdgcn_sched_barrier(0);
            epilogue(std::integral_constant<bool, EPI != EPI_ARGMAX>{});
        }
        if (probe) {
            __builtin_amdgcn_s_waitcnt(0);           // this wave's stores have completed
            if (tid == 0) {
                unsigned long long *p = ep.clk + 8 * (int64_t)v;
                p[0] = clk_t0; p[1] = clk_t1; p[2] = clk_t2; p[3] = wall_clock64(); p[4] = clk_c1; p[5] = clk_c2;
                p[6] = (unsigned long long)__builtin_amdgcn_s_getreg((31 << 11) | 4) |        // HW_ID
                       ((unsigned long long)__builtin_amdgcn_s_getreg((3 << 11) | 20) << 32);  // XCC_ID
                p[7] = clk_c0;
            }
            clk_c0 = clock64();
            clk_t0 = wall_clock64();
        }
        if (vn >= nblk) break;                       // (block-uniform)
        v = vn;
        cur = nxt;
        if constexpr (EPI == EPI_MIX || EPI == EPI_RESID_LN) bias_request(cur.n0);
        lds_barrier();                               // every wave has read its stage back: the unit can be filled
        if constexpr (REREAD) static_for<0, TM + TN>([&](auto r_) { read_one(r_, h0, at(0), at(1)); });
    }
    SRM_WAIT_VM(0);                                  // (the loads behind the last tile, of zero size)
#undef SRM_WAIT_VM
}

// The words of a pass's EPI_RESID_LN launches
__global__ void __launch_bounds__(256) words_clear_kernel(int *words, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) words[i] = 0;
}
