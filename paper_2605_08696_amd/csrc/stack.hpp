// All layers of a decode step of some dozens to some thousand bf16 rows in ONE persistent kernel.
//
// As kernels such a step is a chain of four to six launches per layer, 6 to 10 us each, of which most is launch, cold start and
// a last wave of work-groups.  The rows of a decode step have nothing to do with each other, so here they are cut into
// kStackGroups groups, one for each XCD, and the kStackPer work-groups of a group (one per CU) walk through all layers with
// waits among themselves only: what they exchange stays in the XCD's L2.  (Exchanges among all CUs instead, through memory: 5 us
// for 32 KB, 1.6 within an XCD.)  d = 512, 8 layers, us per step, step kernels | this: 37 rows 184 | 122, 300: 243 | 176, 1024: 317 |
// 253 (all rows: stack_ok in srm.hip).
//
// What bounds it: a group of rows needs all weights, so every XCD reads all of them, 5.2 MB per layer at the 0.95 TB/s that an XCD
// gets, 5.5 us of the 13 (37 rows) to 24 (1024) a layer takes; four waits of 0.8 us and the skew in front of them; from some
// hundred rows on what a CU takes from L2, 64 bytes per clock: 0.9 MB per layer at 1024 rows.  The weights sit in registers, requested one
// to two phases ahead and only once a phase's own operands are there: in front of them, or in one phase for the next, they
// hold up the operands (37 rows 116 us for the layers instead of 106, 1024: 250 instead of 198).  Reading them ahead into L2 by a
// ninth wavefront: 121 and 216.
//
// Phases of a layer, each ended by a wait of the group (0.8 us: an atomic add and a poll):
//   x -> LayerNorm1 | in-projection, state update (Eq. 2 / Eq. 3)    -> m
//   m               | out-projection, x +=                           -> x
//   x -> LayerNorm2 | MLP up, GELU                                   -> g
//   g               | MLP down, x +=                                 -> x
// A work-group owns CW columns of the in-, out- and down-projection and 4 CW of the up-projection, for tiles of 16 RB rows.
// Its eight wavefronts cut K between them (each holds its own part of the weights and nothing is read twice), and the partial
// products meet in LDS; the up-projection, whose accumulators would not fit that way, cuts columns in four and K in two.  m and g travel in the
// order of MFMA operands, [16 rows][32 k] blocks of 1 KB, so that a wavefront loads them straight into registers; the
// LayerNorm rows, which all wavefronts need, stand in LDS in the same order, 16-byte chunks of a row swizzled against
// bank conflicts.  Who writes x also leaves the mean and the squared deviations of its CW columns of each row, so that
// LayerNorm is a combination of D / CW pairs (Chan's formula) and one pass over the row.  Wavefronts take neighbouring rows and
// blocks of k, so that they read different channels of the L2 at a time (1024 rows: 202 -> 198).
//
// What is written for others is stored plainly where the group lies on one XCD (its L2 is where they read), else written
// through (sc1); loads of it are sc1 in both cases (measured: plain stores between XCDs are not seen, within one always).
//
// Work-groups that wait for each other must be resident at once: the arrival is that of few.hpp.  Its words carry the XCD, from
// which the groups are formed.  Where some work-groups have not started within its bound (what other processes run on the device
// keeps them off their CUs, and may itself wait for these), they are left out: those that have are grouped by the next power of two,
// and each does two or more parts of a phase, with the same tiles and sums; of fewer than eight, the last to leave does all alone.
// (They wait longer until there are four for each group: alone, a step takes 5 to 90 ms.)  The same form serves launches of half or a quarter of the work-groups, for streams that launch such steps side by side
// (few_others in srm.hip).
#pragma once
#include "few.hpp"

constexpr int kStackBlocks = 256, kStackGroups = 8, kStackPer = kStackBlocks / kStackGroups, kStackThreads = 512;
constexpr int kStackLeast = 32;                      // work-groups that go on without the others (four of a group) once tired of waiting
constexpr int kStackMaxPer = 288;                    // rows of a group: their positions are kept in LDS
constexpr int kStackWordBytes = kStackBlocks * 8 + kStackGroups * 128 + 256;
struct StackArgs {
    const FewLayer *layers;                          // [L], device
    const float *lnf_g, *lnf_b;
    int L, dh, hrow, n_ctx;                          // dh: channels per head
    float eps;
    int rows, per, tiles;                            // rows of a group, row tiles of a group
    int pos;                                         // or *pos_dev, or pos_rows[row]
    const int *pos_dev;
    const int32_t *pos_rows;
    unsigned char *state;                            // row 0's of layer 0
    size_t layer_bytes;                              // to the next layer's
    int state_half;
    float *x;                                        // [rows][D] embedded tokens, then the residual stream
    float2 *stats;                                   // [rows][D / CW] mean and squared deviations of CW columns
    bf16 *m, *g;                                     // [groups tiles RB][D / 32 | FF / 32][64][8]
    bf16 *a;                                         // [rows][D] final LayerNorm
    float *hidden;                                   // [rows][D] or null
    few_word *here;                                  // [kStackBlocks] arrivals
    unsigned *count;                                 // [kStackGroups] 128 bytes apart
    unsigned *dead;                                  // a wait has given up (in this launch, or since the call began)
    unsigned *left;                                  // work-groups that have left without arriving all
    unsigned max_polls, arrive_polls;
    int scattered;                                   // for tests: groups by the work-groups' numbers, which lie on different XCDs
};

// mean and squared deviations of the CW columns that CW / 4 neighbouring lanes hold
template <int CW>
__device__ __forceinline__ float stack_lanes_sum(float v)
{
    static_assert(CW == 16 || CW == 32, "four or eight lanes");
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
    if constexpr (CW == 32)
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));  // row_half_mirror
    return v;
}
template <int CW>
__device__ __forceinline__ float2 stack_stats(const float4 &v)
{
    const float mean = stack_lanes_sum<CW>((v.x + v.y) + (v.z + v.w)) * (1.0f / CW);
    const float a = v.x - mean, b = v.y - mean, c = v.z - mean, d = v.w - mean;
    return make_float2(mean, stack_lanes_sum<CW>((a * a + b * b) + (c * c + d * d)));
}

// In front of the kernel: the words of its exchange, the embedded tokens and their statistics.  A wavefront per row.
template <int D, int CW>
__global__ void __launch_bounds__(256)
stack_begin_kernel(const int32_t *__restrict__ tok, const bf16 *__restrict__ embed, int vocab, float *__restrict__ x,
                   float2 *__restrict__ stats, int rows, u32x4_t *words, int starting, int *advance_ctr)
{
    if (blockIdx.x == 0) {                           // (starting: for tests, work-groups behind these are withdrawn from the start)
        auto word = [&](int b) { return b >= starting && b < kStackBlocks ? (unsigned)kFewWithdrawn : 0u; };
        for (int i = threadIdx.x; i < kStackWordBytes / 16; i += 256) words[i] = u32x4_t{word(2 * i), 0, word(2 * i + 1), 0};
        if (advance_ctr && threadIdx.x == 0) {       // the step counters of a generate call (see ln_kernel)
            advance_ctr[0] += 1;
            advance_ctr[1] += 1;
        }
    }
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int t = min(max(tok[row], 0), vocab - 1);
    float4 v[D / 256];
#pragma unroll
    for (int i = 0; i < D / 256; ++i) v[i] = load4(embed + (size_t)t * D + (i * 64 + lane) * 4);
#pragma unroll
    for (int i = 0; i < D / 256; ++i) {
        const int c = (i * 64 + lane) * 4;
        store4(x + (size_t)row * D + c, v[i]);
        const float2 s = stack_stats<CW>(v[i]);
        if (c % CW == 0) stats[(size_t)row * (D / CW) + c / CW] = s;
    }
}

constexpr int stack_red_bytes(int CW, int RB) { return 8 * 16 * RB * (CW * 4 + 16); }
constexpr int stack_lds_bytes(int D, int CW, int RB)
{
    return 16 * RB * D * 2 + stack_red_bytes(CW, RB) + kFewMaxLayers * (int)sizeof(FewLayer) + kStackMaxPer * 4 + 256;
}

// MULTI: a member may have several tiles (else exactly one)
template <int D, int CW, int RB, bool MULTI>
__global__ void __launch_bounds__(kStackThreads) stack_kernel(StackArgs p)
{
    constexpr int FF = 4 * D, KB = D / 32, KF = FF / 32;               // blocks of 32 k
    constexpr int COLT = D / CW, CB = CW / 16, RT = 16 * RB, NW = kStackThreads / 64;
    constexpr int K1 = KB / NW, K4 = KF / NW;                          // ... of a wavefront, in the in- and out- and in the down-projection
    constexpr int NCG = 4, KS3 = NW / NCG, K3 = KB / KS3;              // up: groups of CW columns, parts of K, blocks of 32 k
    constexpr int RS = CW * 4 + 16;                                    // row stride of the partial products, bytes
    constexpr int VL = D / 256, RPW = RT / NW;                         // float4 per lane of a row, rows per wavefront
    constexpr int TSTEP = kStackPer / COLT;                            // members that share a member's columns
    static_assert(D % 256 == 0 && COLT <= kStackPer && kStackPer % COLT == 0 && COLT % 8 == 0, "columns of the members");
    static_assert(KS3 == 2, "halves");
    static_assert(NCG * RB * CB * 1024 <= stack_red_bytes(CW, RB), "the halves of the up-projection meet there too");
    extern __shared__ __align__(16) unsigned char stack_lds[];
    unsigned char *const panel = stack_lds, *const red = panel + RT * D * 2;
    FewLayer *const lay = reinterpret_cast<FewLayer *>(red + stack_red_bytes(CW, RB));
    int *const lpos = reinterpret_cast<int *>(lay + kFewMaxLayers);    // [per] positions of the group's rows
    int *const who = lpos + kStackMaxPer;                              // [8]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x;

    int me = 0;
    if (tid == 0) {
        few_word found;
        few_set(p.here + blk, kFewXcd0 + few_xcd(), found);
        me = (int)found;
    }
    for (int i = tid; i < p.L * (int)(sizeof(FewLayer) / 8); i += kStackThreads)
        reinterpret_cast<few_word *>(lay)[i] = reinterpret_cast<const few_word *>(p.layers)[i];
    if (wave == 0) {
        const FewPlace place = few_place<kStackBlocks>(p.here, gridDim.x, blk, __builtin_amdgcn_readfirstlane(me), lane, kStackLeast,
                                                         p.arrive_polls, p.arrive_polls << 6);
        // as many as there are of a group, or the next power of two below
        int m = kStackPer;
        while (m * kStackGroups > place.arrived) m >>= 1;
        if (lane == 0) {
            who[0] = m;
            who[1] = p.scattered ? place.order : place.at;
            who[2] = m && place.near(m) && !p.scattered;
            who[3] = 0;                              // a wait of this group has given up
            who[4] = me < kFewXcd0;                  // withdrawn
        }
    }
    __syncthreads();
    const bool alone = !__builtin_amdgcn_readfirstlane(who[0]);
    const int at = __builtin_amdgcn_readfirstlane(who[1]);
    if (__builtin_expect(alone, 0)) {
        if (tid == 0)
            who[5] = __hip_atomic_fetch_add(p.left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        __syncthreads();
        if (!who[5]) return;
    } else if (__builtin_amdgcn_readfirstlane(who[4]) || at >= __builtin_amdgcn_readfirstlane(who[0]) * kStackGroups) {
        return;
    }
    const bool pure = __builtin_amdgcn_readfirstlane(who[2]) || alone;
    // the work-groups of a group, and the parts of a phase that this one does: part v of kStackPer, and every `members`-th behind it
    const int members = alone ? 1 : __builtin_amdgcn_readfirstlane(who[0]);
    const int c0 = alone ? 0 : at >> __builtin_ctz(members), c1 = alone ? kStackGroups : c0 + 1;
    const int v0 = alone ? 0 : at & (members - 1);

    // LDS only: loads and stores of global memory stay in flight across it
    auto barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    const auto x_rs = __builtin_amdgcn_make_buffer_rsrc(p.x, 0, (unsigned)p.rows * D * 4, 0x27000);
    const auto st_rs = __builtin_amdgcn_make_buffer_rsrc(p.stats, 0, (unsigned)p.rows * COLT * 8, 0x27000);
    const unsigned frag_rows = (unsigned)((p.rows + p.per - 1) / p.per * p.tiles) * RT;
    const auto m_rs = __builtin_amdgcn_make_buffer_rsrc(p.m, 0, frag_rows * D * 2, 0x27000);
    const auto g_rs = __builtin_amdgcn_make_buffer_rsrc(p.g, 0, frag_rows * FF * 2, 0x27000);
    constexpr int kSc1 = 16;                         // load: not from this CU's cache; store: through the L2
    auto put16 = [&](auto rs, unsigned off, u32x4_t v) {
        if (pure) __builtin_amdgcn_raw_buffer_store_b128(v, rs, off, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b128(v, rs, off, 0, kSc1);
    };
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
    auto put8 = [&](auto rs, unsigned off, u32x2_t v) {
        if (pure) __builtin_amdgcn_raw_buffer_store_b64(v, rs, off, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(v, rs, off, 0, kSc1);
    };
    auto pack4 = [](float4 v) {
        const bf16x2_t lo = __builtin_convertvector(f32x2_t{v.x, v.y}, bf16x2_t);
        const bf16x2_t hi = __builtin_convertvector(f32x2_t{v.z, v.w}, bf16x2_t);
        return u32x2_t{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    };
    auto opaque = [](int i) {                        // (addresses are formed where they are used, see few.hpp)
        asm volatile("" : "+v"(i));
        return i;
    };
    auto uniform = [](const void *q) {
        const unsigned long long a = reinterpret_cast<unsigned long long>(q);
        return reinterpret_cast<const unsigned char *>(((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(a >> 32)) << 32) |
                                                       (unsigned)__builtin_amdgcn_readfirstlane((unsigned)a));
    };
    auto vec4 = [&](const float *q, int i) { 
        return __builtin_bit_cast(float4, few_load(reinterpret_cast<const f32x4_t *>(reinterpret_cast<const float *>(uniform(q)) + i)));
    };
    auto value = [&](const float *q, int i) { return few_load(reinterpret_cast<const float *>(uniform(q)) + i); };
    // Blocks kb .. kb + n - 1 of 32 k of sixteen columns from col on, of a matrix with K inputs as few_pack_kernel leaves it:
    // [columns / 4][K / 128][16 vectors of k][4 columns] of 16 bytes.  Four lanes read 64 consecutive bytes.
    auto weights = [&](auto K_c, const void *W, int col, int kb, auto &w, int step = 2) {
        constexpr int CH = decltype(K_c)::value / 128 * 64, n = sizeof(w) / sizeof(u32x4_t);
        const int ln = opaque(lane);
        const unsigned of = (unsigned)(((ln >> 2) & 3) * CH + (ln >> 4) * 4 + (ln & 3));
        const u32x4_t *base = reinterpret_cast<const u32x4_t *>(uniform(W)) + (size_t)(col / 4) * CH;
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const int k = kb + (j >> 1) * step + (j & 1);              // pairs of blocks, whose lines are one and the same, `step` apart
            w[j] = few_load(base + (k >> 2) * 64 + (k & 3) * 16 + of);
        }
    };
    auto mfma = [](const u32x4_t &w, const u32x4_t &a, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, a), c, 0, 0, 0);
    };
    // everything this work-group has written is there for the others of its group, and theirs for it
    unsigned phase = 0;
    auto meet = [&](int c) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70);          // (the same, for the compiler to know)
        barrier();
        ++phase;
        if (alone) return;
        if (tid == 0 && !who[3]) {
            unsigned *const n = p.count + c * 32;
            const unsigned all = phase * (unsigned)members;
            __hip_atomic_fetch_add(n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (unsigned polls = 0; __hip_atomic_load(n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < all; ++polls) {
                if (polls >= p.max_polls) {
                    who[3] = 1;
                    __hip_atomic_store(p.dead, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
        }
        barrier();
    };

    u32x4_t w_in[CB][K1], w_out[CB][K1], w_up[2][CB][K3 / 2], w_down[CB][K4];
    const int cg = wave % NCG, k3 = wave / NCG * K3;                   // up: this wavefront's columns and k
    auto get_in = [&](int l, int col) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) weights(std::integral_constant<int, D>{}, lay[l].w_in, col + 16 * cb, wave * K1, w_in[cb]);
    };
    auto get_out = [&](int l, int col) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) weights(std::integral_constant<int, D>{}, lay[l].w_out, col + 16 * cb, wave * K1, w_out[cb]);
    };
    auto get_up = [&](int h, int l, int col) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            weights(std::integral_constant<int, D>{}, lay[l].w_up, 4 * col + (cg * CB + cb) * 16, k3 + h * (K3 / 2), w_up[h][cb]);
    };
    auto get_down = [&](int l, int col) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) weights(std::integral_constant<int, FF>{}, lay[l].w_down, col + 16 * cb, 2 * wave, w_down[cb], 2 * NW);
    };
    // LayerNorm of a tile's rows into the panel; behind(): what is to be requested behind the rows
    auto normalise = [&](int base, int last, const float *gain, const float *shift, auto &&behind, auto &&later) __attribute__((always_inline)) {
        const int ln = opaque(lane);
        float4 v[RPW][VL], pg[VL], pb[VL];
        u32x4_t st[COLT / 16];
        const unsigned sr = (unsigned)min(base + min(ln >> 3, RPW - 1) * NW + wave, last);
#pragma unroll
        for (int j = 0; j < COLT / 16; ++j)
            st[j] = __builtin_amdgcn_raw_buffer_load_b128(st_rs, sr * (COLT * 8) + (ln & 7) * COLT + j * 16, 0, kSc1);
#pragma unroll
        for (int j = 0; j < VL; ++j) {
            pg[j] = vec4(gain, (j * 64 + ln) * 4);
            pb[j] = vec4(shift, (j * 64 + ln) * 4);
        }
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const unsigned row = (unsigned)min(base + i * NW + wave, last);
#pragma unroll
            for (int j = 0; j < VL; ++j)
                v[i][j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, (j * 64 + ln) * 16, row * (D * 4), kSc1));
        }
        __builtin_amdgcn_sched_barrier(0);
        behind();
        __builtin_amdgcn_sched_barrier(0);
        float mean = 0.0f, dev = 0.0f;
#pragma unroll
        for (int j = 0; j < COLT / 16; ++j) mean += __uint_as_float(st[j][0]) + __uint_as_float(st[j][2]);
        mean = stack_lanes_sum<32>(mean) * (1.0f / COLT);
#pragma unroll
        for (int j = 0; j < COLT / 16; ++j) {
            const float a = __uint_as_float(st[j][0]) - mean, b = __uint_as_float(st[j][2]) - mean;
            dev += (__uint_as_float(st[j][1]) + __uint_as_float(st[j][3])) + (float)CW * (a * a + b * b);
        }
        const float rstd = 1.0f / sqrtf(stack_lanes_sum<32>(dev) / (float)D + p.eps);
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const float mu = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mean), 8 * i));
            const float rs = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rstd), 8 * i));
            const int r = i * NW + wave;
#pragma unroll
            for (int j = 0; j < VL; ++j) {
                const float4 o = make_float4((v[i][j].x - mu) * rs * pg[j].x + pb[j].x, (v[i][j].y - mu) * rs * pg[j].y + pb[j].y,
                                             (v[i][j].z - mu) * rs * pg[j].z + pb[j].z, (v[i][j].w - mu) * rs * pg[j].w + pb[j].w);
                // k = 256 j + 4 lane: block of 32, chunk of eight in it, half of that
                const int chunk = (r >> 4) * KB * 4 + j * 32 + (ln >> 1);
                *reinterpret_cast<u32x2_t *>(panel + (chunk * 16 + ((r & 15) ^ ((ln >> 1) & 15))) * 16 + (ln & 1) * 8) = pack4(o);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        later();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto from_panel = [&](int ln, int rb, int kb) {
        const int q = kb * 4 + (ln >> 4);
        return *reinterpret_cast<const u32x4_t *>(panel + ((rb * KB * 4 + q) * 16 + ((ln & 15) ^ (q & 15))) * 16);
    };
    // partial products of this wavefront's k, and their sum for a thread's quad of columns
    struct Quad { int r, q; };                       // its row of the tile, its first column
    auto my_quad = [&] {
        const int t = opaque(tid);
        return Quad{t / (CW / 4), t % (CW / 4) * 4};
    };
    const bool quad = wave * 64 < RT * (CW / 4);     // (whole wavefronts)
    auto leave = [&](const f32x4_t (&acc)[RB][CB]) {
        const int ln = opaque(lane);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                *reinterpret_cast<f32x4_t *>(red + (wave * RT + rb * 16 + (ln & 15)) * RS + cb * 64 + (ln >> 4) * 16) = acc[rb][cb];
    };
    auto total = [&](const Quad &e) {
        f32x4_t t[NW];
#pragma unroll
        for (int s = 0; s < NW; ++s) t[s] = *reinterpret_cast<const f32x4_t *>(red + (s * RT + e.r) * RS + e.q * 4);
        return ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    };
    auto clear = [](f32x4_t (&acc)[RB][CB]) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    // x += what a thread's quad adds up to, and the statistics of the new values
    auto add_to_x = [&](int base, int r1, int ct, const float4 &old, const float4 &bias) {
        if (!quad) return;
        const Quad e = my_quad();
        const f32x4_t t = total(e);
        const float4 v = make_float4(old.x + (t[0] + bias.x), old.y + (t[1] + bias.y), old.z + (t[2] + bias.z), old.w + (t[3] + bias.w));
        const float2 s = stack_stats<CW>(v);
        const int row = base + e.r;
        if (row < r1) {
            put16(x_rs, ((unsigned)row * D + ct * CW + e.q) * 4, __builtin_bit_cast(u32x4_t, v));
            if (e.q == 0) put8(st_rs, ((unsigned)row * COLT + ct) * 8, __builtin_bit_cast(u32x2_t, s));
        }
    };
    auto old_x = [&](int base, int r1, int ct) {
        const Quad e = my_quad();
        const unsigned row = (unsigned)min(base + e.r, r1 - 1);
        return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, (row * D + ct * CW + e.q) * 4, 0, kSc1));
    };

    // One group, a part to each member; or (MANY) several, their weights requested where they are used, of all groups where alone.
    auto run = [&](auto MANY) __attribute__((always_inline)) {
    for (int c = c0; c < c1; ++c) {
        const int r0 = c * p.per, r1 = min(p.rows, r0 + p.per);
        if (r0 >= r1) continue;                      // (all members of the group)
        barrier();
        for (int i = tid; i < r1 - r0; i += kStackThreads)
            lpos[i] = p.pos_rows ? few_load(p.pos_rows + r0 + i) : p.pos_dev ? few_load(p.pos_dev) : p.pos;
        barrier();
        if constexpr (!MANY) {
            get_in(0, v0 % COLT * CW);
            get_out(0, v0 % COLT * CW);
        }
        auto parts = [&](auto &&part) __attribute__((always_inline)) {
            if constexpr (MANY) {
#pragma unroll 1
                for (int v = v0; v < kStackPer; v += members) part(v);
            } else {
                part(v0);
            }
        };
        for (int l = 0; l < p.L; ++l) {
            const int next = l + 1 < p.L ? l + 1 : l;
            const FewLayer &y = lay[l];
            // A member's tiles: the first one's loads stand in front of the weights that are requested in this phase.
            auto tiles = [&](int v, auto &&tile) __attribute__((always_inline)) {
                tile(std::true_type{}, v / COLT);
                if constexpr (MULTI)
#pragma unroll 1
                    for (int t = v / COLT + TSTEP; t < p.tiles; t += TSTEP) tile(std::false_type{}, t);
            };
            // ---------------- LayerNorm1, in-projection, state update
            if (l > 0) meet(c);
            parts([&](int v) __attribute__((always_inline)) {
                const int ct = v % COLT;
                if constexpr (MANY) get_in(l, ct * CW);
                unsigned char *const S = p.state + (size_t)l * p.layer_bytes;
                tiles(v, [&](auto first, int t) __attribute__((always_inline)) {
                    const Quad e = my_quad();
                    const int col = ct * CW + e.q, head = col / p.dh;
                    const int base = r0 + t * RT, row = min(base + e.r, r1 - 1), pos = lpos[row - r0], ps = min(max(pos, 0), p.n_ctx - 1);
                    const int64_t at4 = ((int64_t)row * D + col) >> 2;
                    float4 bias, s0;
                    float al, be, la;
                    normalise(base, r1 - 1, y.ln[0], y.ln[1], [&] {
                        bias = vec4(y.b_in, col);
                        la = value(y.lam, head);
                        al = value(y.alpha, head * p.n_ctx + ps);
                        be = value(y.beta, head * p.n_ctx + ps);
                        s0 = p.state_half ? load_state4(reinterpret_cast<const f16 *>(S), at4) : load_state4(reinterpret_cast<const float *>(S), at4);
                    }, [&] { if constexpr (first && !MANY) get_up(0, l, ct * CW); });
                    barrier();
                    const int ln = opaque(lane);
                    f32x4_t acc[RB][CB];
                    clear(acc);
#pragma unroll
                    for (int j = 0; j < K1; ++j)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) {
                            const u32x4_t a = from_panel(ln, rb, wave * K1 + j);
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = mfma(w_in[cb][j], a, acc[rb][cb]);
                        }
                    leave(acc);
                    barrier();
                    if (quad && base + e.r < r1) {
                        const f32x4_t u = total(e);
                        const bool rr = head < p.hrow, active = pos == ps;
                        const float pp = rr ? al : 1.0f, qq = rr ? 1.0f : al;
                        float4 n, mo;
                        n.x = fmaf(la, s0.x, pp * (float)(bf16)(u[0] + bias.x));
                        n.y = fmaf(la, s0.y, pp * (float)(bf16)(u[1] + bias.y));
                        n.z = fmaf(la, s0.z, pp * (float)(bf16)(u[2] + bias.z));
                        n.w = fmaf(la, s0.w, pp * (float)(bf16)(u[3] + bias.w));
                        if (p.state_half) {
                            f16 *sp = reinterpret_cast<f16 *>(S);
                            n = make_float4(to_state(n.x, sp), to_state(n.y, sp), to_state(n.z, sp), to_state(n.w, sp));
                            if (active) store_state4(sp, at4, n);
                        } else if (active) {
                            store_state4(reinterpret_cast<float *>(S), at4, n);
                        }
                        mo = make_float4(fmaf(qq, n.x, be), fmaf(qq, n.y, be), fmaf(qq, n.z, be), fmaf(qq, n.w, be));
                        if (!active) mo = make_float4(0.f, 0.f, 0.f, 0.f);       // outside the context: the state stays, zeros go out
                        const unsigned fb = (unsigned)((c * p.tiles + t) * RB + (e.r >> 4)) * KB + (col >> 5);
                        put8(m_rs, fb * 1024 + ((e.r & 15) + ((col >> 3) & 3) * 16) * 16 + ((col >> 2) & 1) * 8, pack4(mo));
                    }
                });
            });
            // ---------------- out-projection
            meet(c);
            // (the next layer's LayerNorm parameters, 4 x 2 KB, into the L2: the group's rows would wait for them)
            const u32x4_t touched = few_load(reinterpret_cast<const u32x4_t *>(lay[next].ln[tid / (D / 4) & 3]) + tid % (D / 4));
            parts([&](int v) __attribute__((always_inline)) {
                const int ct = v % COLT;
                if constexpr (MANY) get_out(l, ct * CW);
                tiles(v, [&](auto first, int t) __attribute__((always_inline)) {
                    const int base = r0 + t * RT, ln = opaque(lane);
                    u32x4_t a[K1][RB];
                    const unsigned fb = (unsigned)((c * p.tiles + t) * RB) * KB + wave * K1;
#pragma unroll
                    for (int j = 0; j < K1; ++j)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
                            a[j][rb] = __builtin_amdgcn_raw_buffer_load_b128(m_rs, ln * 16, (fb + rb * KB + j) * 1024, kSc1);
                    const float4 old = old_x(base, r1, ct), bias = vec4(y.b_out, ct * CW + my_quad().q);
                    __builtin_amdgcn_sched_barrier(0);
                    f32x4_t acc[RB][CB];
                    clear(acc);
#pragma unroll
                    for (int j = 0; j < K1; ++j)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = mfma(w_out[cb][j], a[j][rb], acc[rb][cb]);
                    if (!first || MANY) barrier();              // (the sums of the tile in front are formed)
                    if constexpr (first && !MANY) get_up(1, l, ct * CW);
                    __builtin_amdgcn_sched_barrier(0);
                    leave(acc);
                    barrier();
                    add_to_x(base, r1, ct, old, bias);
                });
            });
            asm volatile("" : : "v"(touched));
            // ---------------- LayerNorm2, MLP up, GELU
            meet(c);
            parts([&](int v) __attribute__((always_inline)) {
                const int ct = v % COLT;
                if constexpr (MANY) { get_up(0, l, ct * CW); get_up(1, l, ct * CW); }
                tiles(v, [&](auto first, int t_) __attribute__((always_inline)) {
                    if (!first || MANY) barrier();              // (the panel of the tile in front has been read)
                    const int ln = opaque(lane), col = ct * 4 * CW + CW * cg + 4 * (ln >> 4);
                    float4 bias[CB];
                    normalise(r0 + t_ * RT, r1 - 1, y.ln[2], y.ln[3], [&] {
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) bias[cb] = vec4(y.b_up, col + 16 * cb);
                    }, [&] { if constexpr (first && !MANY) get_down(l, ct * CW); });
                    barrier();
                    f32x4_t acc[RB][CB];
                    clear(acc);
#pragma unroll
                    for (int j = 0; j < K3; ++j)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) {
                            const u32x4_t a = from_panel(ln, rb, k3 + j);
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = mfma(w_up[j / (K3 / 2)][cb][j % (K3 / 2)], a, acc[rb][cb]);
                        }
                    // each half of K finishes every other block of sums
                    auto mine = [&](int rb, int cb) { return ((rb * CB + cb) & 1) == wave / NCG; };
                    auto place = [&](int rb, int cb) { return reinterpret_cast<f32x4_t *>(red + (((cg * RB + rb) * CB + cb) * 64 + ln) * 16); };
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb)
                            if (!mine(rb, cb)) *place(rb, cb) = acc[rb][cb];
                    barrier();
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            if (!mine(rb, cb)) continue;
                            const f32x4_t t = acc[rb][cb] + *place(rb, cb);
                            const bf16 *o = nullptr;
                            const float4 v4 = make_float4(gelu_for(o, t[0] + bias[cb].x), gelu_for(o, t[1] + bias[cb].y),
                                                          gelu_for(o, t[2] + bias[cb].z), gelu_for(o, t[3] + bias[cb].w));
                            const int cc = col + 16 * cb;
                            const unsigned fb = (unsigned)((c * p.tiles + t_) * RB + rb) * KF + (cc >> 5);
                            put8(g_rs, fb * 1024 + ((ln & 15) + ((cc >> 3) & 3) * 16) * 16 + ((cc >> 2) & 1) * 8, pack4(v4));
                        }
                });
            });
            // ---------------- MLP down
            meet(c);
            parts([&](int v) __attribute__((always_inline)) {
                const int ct = v % COLT;
                if constexpr (MANY) get_down(l, ct * CW);
                tiles(v, [&](auto first, int t) __attribute__((always_inline)) {
                    const int base = r0 + t * RT, ln = opaque(lane);
                    constexpr int KC = RB >= 3 ? 2 : RB == 2 ? 4 : K4, NC = K4 / KC;         // blocks of k in a request, requests
                    static_assert(K4 % KC == 0 && KC % 2 == 0, "whole requests, pairs");
                    const unsigned fb = (unsigned)((c * p.tiles + t) * RB) * KF + 2 * wave;
                    u32x4_t a[2][KC][RB];
                    auto request = [&](int n, u32x4_t (&to)[KC][RB]) {
#pragma unroll
                        for (int j = 0; j < KC; ++j)
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb)
                                to[j][rb] = __builtin_amdgcn_raw_buffer_load_b128(g_rs, ln * 16, (fb + rb * KF + ((n * KC + j) >> 1) * 2 * NW + (j & 1)) * 1024, kSc1);
                    };
                    request(0, a[0]);
                    __builtin_amdgcn_sched_barrier(0);         // (left alone, the loads sink to their uses)
                    const float4 old = old_x(base, r1, ct), bias = vec4(y.b_down, ct * CW + my_quad().q);
                    f32x4_t acc[RB][CB];
                    clear(acc);
#pragma unroll
                    for (int n = 0; n < NC; ++n) {
                        if (n + 1 < NC) request(n + 1, a[(n + 1) & 1]);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int j = 0; j < KC; ++j)
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                                for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = mfma(w_down[cb][n * KC + j], a[n & 1][j][rb], acc[rb][cb]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (first && !MANY) { get_in(next, ct * CW); get_out(next, ct * CW); }
                    barrier();                 // (the sums of the tile in front are formed)
                    leave(acc);
                    barrier();
                    add_to_x(base, r1, ct, old, bias);
                });
            });
            if (who[3]) return;            // given up: the tokens are -1
        }
        meet(c);
        // ---------------- final LayerNorm, a wavefront per row
        for (int v = v0; v < kStackPer; v += members)
            for (int i = v * NW + wave; i < r1 - r0; i += kStackPer * NW) {
                const unsigned row = (unsigned)(r0 + i);
                float4 o[VL], pg[VL], pb[VL];
                float s = 0.0f, sq = 0.0f;
#pragma unroll
                for (int j = 0; j < VL; ++j) {
                    o[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, (j * 64 + lane) * 16, row * (D * 4), kSc1));
                    pg[j] = load4(p.lnf_g + (j * 64 + lane) * 4);
                    pb[j] = load4(p.lnf_b + (j * 64 + lane) * 4);
                }
#pragma unroll
                for (int j = 0; j < VL; ++j) s += (o[j].x + o[j].y) + (o[j].z + o[j].w);
                const float mu = wave_sum(s) / (float)D;
#pragma unroll
                for (int j = 0; j < VL; ++j) {
                    const float a = o[j].x - mu, b = o[j].y - mu, cc = o[j].z - mu, d = o[j].w - mu;
                    sq += (a * a + b * b) + (cc * cc + d * d);
                }
                const float rs = 1.0f / sqrtf(wave_sum(sq) / (float)D + p.eps);
#pragma unroll
                for (int j = 0; j < VL; ++j) {
                    const size_t to = (size_t)row * D + (j * 64 + lane) * 4;
                    if (p.hidden) store4(p.hidden + to, o[j]);
                    store4(p.a + to, make_float4((o[j].x - mu) * rs * pg[j].x + pb[j].x, (o[j].y - mu) * rs * pg[j].y + pb[j].y,
                                                 (o[j].z - mu) * rs * pg[j].z + pb[j].z, (o[j].w - mu) * rs * pg[j].w + pb[j].w));
                }
            }
    }
    };
    if (members < kStackPer) run(std::true_type{});
    else run(std::false_type{});
}
