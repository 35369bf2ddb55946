// Decode steps of a handful of samples in ONE persistent kernel, for models of a few hundred to a thousand channels.
//
// With so few rows a step is a chain of four dependent products per layer, and as kernels each of them costs a kernel boundary
// and a cold start, 4 to 5 us whatever it computes.  Here D / NWC co-resident work-groups walk through all layers and all G
// steps (figures against the step kernels: few_max_rows in srm.hip).  What bounds it is the exchange of activations between the phases, so that is made of a single trip through
// memory: every value travels as an 8-byte word of the value and the number of the phase it belongs to ("tag"), stored and
// loaded as one atomic, and the reader polls the words themselves until all carry the phase's tag.  No flag follows the
// data, nothing is flushed or invalidated, and no counter is shared.  All-gather of 16 KB among 64 | 128 | 256 work-groups:
// 1.4 | 1.6 | 2.0 us (a barrier of published flags plus the activations behind it: 4 us and more from 64 work-groups on).
//
// Phases of a layer (x: residual stream, fp32), each an all-gather of what the phase before has published:
//   x -> LayerNorm1 | in-projection, state update (Eq. 2 / Eq. 3)    -> m
//   m               | out-projection, x += (in the owner's register) -> x
//   x -> LayerNorm2 | MLP up, GELU                                   -> g
//   g               | MLP down, x +=                                 -> x
// (non-projected layers: LayerNorm1, update, x += m and LayerNorm2 of whole rows by every work-group, two phases); behind
// the last layer x -> final LayerNorm | LM head, the best (score, index) of the work-group's columns -> winners -> next token.
// Every work-group takes part in every phase, so a buffer's words are all read before any of them is written again: whoever
// writes a phase's words has gathered the words of the phase before, which the others publish after having gathered the
// ones in front of that.
//
// Roles in a work-group: NG wavefronts gather (poll, normalise a row each, leave the rows in LDS), NWC wavefronts compute.
// Work-group b owns the columns b NWC .. b NWC + NWC - 1 of the in-, out- and down-projection, whose inputs its wavefronts cut
// into quarters, and four times as many of the up-projection, four to a wavefront.  The weights sit in registers, requested up
// to a layer ahead by the computing wavefronts: the gathering ones would wait for them in front of every poll, since loads
// return in order.  A publication is one store of consecutive words per work-group (a store per wavefront, into lines that
// several work-groups share: 3.2 us per exchange of 8 KB among 256 work-groups instead of 2.0).
//
// Where the time goes (d = 1024, one row, 16 layers, us): 5 for the launch, 2 + 10.2 per layer, of which four
// exchanges 5.4, two LayerNorms 1.4, products, epilogues and waiting for weights 3.4, and 16 for the head, which reads at 4.5
// TB/s.  Extra work-groups that read the next layer ahead into L2 made it 3 % slower at one row and 5 % faster at two and four.
//
// All work-groups must be resident at once, which an ordinary launch cannot promise: other processes, or kernels that wait for
// each other themselves, can hold the CUs.  So the first exchange is an arrival, before anything but scratch is written
// (few_arrived): either every work-group sees that all have started, and then all stay until they end, or every one leaves, and
// the last to leave does all the work alone (few_alone), slowly and with the same bits.  Kernels in groups that take the whole
// device (few_place) go on with the work-groups that have started.
// The waits behind the arrival are bounded all the same: a work-group that gives up raises a flag that ends all other waits, and
// the tokens are -1.
#pragma once
#include "common.hpp"
#include "gemm.hpp"

constexpr int kFewGather = 4;                        // wavefronts that gather
struct FewLayer {
    const float *ln[4];                              // LayerNorm1's gain and bias, LayerNorm2's
    const float *b_in, *alpha, *beta, *lam, *b_out, *b_up, *b_down;
    const void *w_in, *w_out, *w_up, *w_down;
};
struct FewArgs {
    const FewLayer *layers;                          // [L], device
    const void *embed, *head;
    const float *lnf_g, *lnf_b;
    int V, L, dh, hrow, n_ctx;                       // dh: channels per head
    float eps;
    int B, pos0, G;
    int Bs, row0;                                    // in groups (XCD): rows of the call, the group's first; else B and 0
    const int32_t *tok_in;                           // [B] tokens at pos0
    int32_t *tok_out;                                // [B] the last tokens
    int32_t *store;                                  // [G][Bs] or null
    void *state;                                     // [L][Bs][D]
    int state_half;
    float *logits, *hidden;                          // [B][V], [B][D] of the last step, or null
    float temp;                                      // > 0: Gumbel-max sampling
    uint32_t seed;
    few_word *xw, *mw, *gw, *pw;                     // words of x [MB][D], m [MB][D], g [MB][FF words], winners [MB][NB][2]
    unsigned *flag;                                  // a wait has given up; [1]: work-groups that have left without arriving all
    unsigned max_polls, arrive_polls;                // bounds of the waits
    int scattered;                                   // for tests: groups by the work-groups' numbers, which lie on different XCDs
};

// near: who polls for the word shares this XCD's L2, and it need not be written through
__device__ __forceinline__ void few_put(few_word *p, unsigned payload, unsigned tag, bool near = false)
{
    const few_word w = ((few_word)tag << 32) | payload;
    if (near) __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Polls the words at(0) .. at(N - 1) of every lane until all of the wavefront carry `tag`; false: given up.
template <int N, typename AT>
__device__ __forceinline__ bool few_gather(few_word (&v)[N], AT &&at, unsigned tag, const FewArgs &p)
{
    for (unsigned polls = 0;; ++polls) {
        bool ok = true;
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = __hip_atomic_load(at(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < N; ++i) ok = ok && (unsigned)(v[i] >> 32) == tag;
        if (__all(ok)) return true;
        if (polls >= p.max_polls ||
            ((polls & 255) == 255 && __hip_atomic_load(p.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            __hip_atomic_store(p.flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
    }
}

// The arrival of the NB work-groups: word b (`stride` words apart, zero at the launch) becomes 1 when work-group b starts, or
// 2 when another one, tired of waiting, has withdrawn it first.  Each is set once, so all work-groups come to the same answer:
// true where every word is 1.  One wavefront per work-group.
constexpr few_word kFewHere = 1, kFewWithdrawn = 2;
__device__ __forceinline__ void few_set(few_word *p, few_word value, few_word &found)
{
    found = 0;
    __hip_atomic_compare_exchange_strong(p, &found, value, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (found == 0) found = value;
}
template <int NB>
__device__ __forceinline__ bool few_arrived(few_word *words, int stride, int lane, unsigned max_polls)
{
    static_assert(NB % 64 == 0, "as many words for each lane");
    constexpr int N = NB / 64;
    few_word v[N];
    bool here, withdrawn;
    auto look = [&] {
        here = true;
        withdrawn = false;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            here = here && v[i] == kFewHere;
            withdrawn = withdrawn || v[i] == kFewWithdrawn;
        }
    };
    for (unsigned polls = 0;; ++polls) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            v[i] = __hip_atomic_load(words + (i * 64 + lane) * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        look();
        if (__any(withdrawn)) return false;
        if (__all(here)) return true;
        if (polls >= max_polls) break;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) few_set(words + (i * 64 + lane) * stride, kFewWithdrawn, v[i]);
    look();
    return __all(here);
}

// An arrival of `blocks` work-groups, at most NB, whose words say on which XCD one runs (kFewXcd0 plus its number), and which may go
// on without those that are missing: whoever is tired of waiting withdraws them, and every work-group comes to the same answer.
// It is tired after `polls` where at least `least` have arrived, else after `most_polls`.  `me`: this work-group's word.
constexpr int kFewXcd0 = 4;
__device__ __forceinline__ int few_xcd() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15; }          // HW_REG_XCC_ID
struct FewPlace {
    int arrived;             // work-groups; in the order of their XCDs:
    int at, below, same;     // this one's number, how many lie on the XCDs in front of its own and on its own
    int order;               // its number in the order of the launch
    __device__ __forceinline__ bool near(int per) const                // its group of `per`, a power of two, lies on one XCD
    {
        const int first = at & -per;
        return below <= first && first + per <= below + same;
    }
};
constexpr int kFewGroups = 8;
template <int NB>
__device__ __forceinline__ FewPlace few_place(few_word *words, int blocks, int blk, int me, int lane, int least, unsigned polls,
                                              unsigned most_polls)
{
    static_assert(NB % 64 == 0, "as many words for each lane");
    constexpr int N = NB / 64;
    few_word v[N];
    auto waits = [&] {                               // for one that has neither arrived nor been withdrawn
        bool w = false;
#pragma unroll
        for (int i = 0; i < N; ++i) w = w || (v[i] == 0 && i * 64 + lane < blocks);
        return __any(w);
    };
    auto arrived = [&] {
        int n = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) n += __popcll(__ballot(v[i] >= kFewXcd0));
        return n;
    };
    for (unsigned asked = 0;; ++asked) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            v[i] = i * 64 + lane < blocks ? __hip_atomic_load(words + i * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        if (!waits()) break;
        if (asked >= most_polls || (asked >= polls && arrived() >= least)) {
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (v[i] == 0 && i * 64 + lane < blocks) few_set(words + i * 64 + lane, kFewWithdrawn, v[i]);
            break;
        }
    }
    FewPlace p{arrived(), 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int w = (int)v[i], number = i * 64 + lane;
        p.below += __popcll(__ballot(w >= kFewXcd0 && w < me));
        p.same += __popcll(__ballot(w == me));
        p.at += __popcll(__ballot(w == me && number < blk));
        p.order += __popcll(__ballot(w >= kFewXcd0 && number < blk));
    }
    p.at += p.below;
    return p;
}

// A load through a pointer that came from LDS: global memory, which the compiler cannot know (a flat load would count as an
// LDS access too, and LDS reads would wait for weights on their way from HBM).
template <typename T>
__device__ __forceinline__ T few_load(const T *p)
{
    typedef __attribute__((address_space(1))) const T global_t;
    return *(global_t *)(unsigned long long)p;
}

// Products on the matrix cores' sixteen 4 x 4 blocks (v_mfma_f32_4x4x4_16b_bf16, v_mfma_f32_4x4x1_16b_f32): block b of a
// lane 4b + i takes four columns of W (i) and four rows of activations (i again, of the second operand) over its own k, so that
// one to four rows use all of the unit, which a 16 x 16 tile would leave idle, and a vector unit would need twenty times as
// long for (two products of bf16 pairs take 16 clocks there, with or without v_dot2).  The vectors of W are packed so that a
// wavefront reads 1 KB in one piece (few_pack_kernel); those of the activations come from LDS, rows 32 bytes off a multiple
// of 128 apart: no bank conflicts.
constexpr int kFewPad = 32;
template <typename TW> __device__ __forceinline__ f32x4_t few_mfma(const u32x4_t &w, const u32x4_t &a, f32x4_t c, int part);
template <> __device__ __forceinline__ f32x4_t few_mfma<bf16>(const u32x4_t &w, const u32x4_t &a, f32x4_t c, int part)
{
    typedef __attribute__((ext_vector_type(4))) short s16x4_t;
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
    const u32x2_t x = {w[2 * part], w[2 * part + 1]}, y = {a[2 * part], a[2 * part + 1]};
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4_t, x), __builtin_bit_cast(s16x4_t, y), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4_t few_mfma<float>(const u32x4_t &w, const u32x4_t &a, f32x4_t c, int part)
{
    const uint32_t x = w[part], y = a[part];
    return __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(x), __uint_as_float(y), c, 0, 0, 0);
}
__device__ __forceinline__ float few_add32(float a, float b)      // lanes 0..31: a's two halves added, 32..63: b's
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float few_add16(float a, float b)      // even rows of 16 lanes: a's row pairs added, odd: b's
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
template <int SHIFT>
__device__ __forceinline__ float few_add_ror(float v)             // plus the value SHIFT lanes on in the row of 16
{
    return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x120 + SHIFT, 0xF, 0xF, true));
}
// Four columns of N vectors each (w) times the rows of `act` (row stride `stride` bytes, the vectors from number `first` on):
// v[rb] of lane l = row 4 rb + (l & 3), column few_column(l).
__device__ __forceinline__ int few_column(int lane) { return ((lane >> 4) & 1) + 2 * (lane >> 5); }
template <typename TW, int N, int MB>
__device__ __forceinline__ void few_products(const u32x4_t (&w)[N], const unsigned char *act, int stride, int first, int lane,
                                             float (&v)[(MB + 3) / 4])
{
    constexpr int RB = (MB + 3) / 4, PARTS = (int)sizeof(TW);      // products per vector
    constexpr int G = N < 4 ? N : 4;                 // activation vectors in flight
    static_assert(N % G == 0, "whole groups");
    asm volatile("" : "+v"(lane));                   // (addresses formed here, see opaque())
    const unsigned char *at = act + min(lane & 3, MB - 1) * stride + (first * 16 + (lane >> 2)) * 16;
    f32x4_t acc[RB][2];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb][0] = acc[rb][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j0 = 0; j0 < N; j0 += G) {
        u32x4_t a[RB][G];
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) a[rb][k] = *reinterpret_cast<const u32x4_t *>(at + rb * 4 * stride + (j0 + k) * 256);
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int q = 0; q < PARTS; ++q)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc[rb][q & 1] = few_mfma<TW>(w[j0 + k], a[rb][k], acc[rb][q & 1], q);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const f32x4_t t = acc[rb][0] + acc[rb][1];   // [column] of row lane & 3, block lane >> 2
        v[rb] = few_add_ror<4>(few_add_ror<8>(few_add16(few_add32(t[0], t[2]), few_add32(t[1], t[3]))));
    }
}

// Pieces that the exchanging wavefronts and few_alone share.  Element 128 i + 2 lane of a row and the one behind it:
__device__ __forceinline__ int few_elem(int i, int lane) { return 128 * i + 2 * lane; }
template <typename TW, int D, int MB>
__device__ __forceinline__ void few_embed(const TW *embed, const int *tokb, float *xs, int from, int step)      // rows of the tokens
{
    constexpr int V = 16 / (int)sizeof(TW);
    for (int i = from; i < MB * D / V; i += step) {
        const int r = i / (D / V), c = i % (D / V) * V;
        const u32x4_t t = *reinterpret_cast<const u32x4_t *>(embed + (size_t)tokb[r] * D + c);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (sizeof(TW) == 2) {
                xs[r * D + c + 2 * k] = __uint_as_float(t[k] << 16);
                xs[r * D + c + 2 * k + 1] = __uint_as_float(t[k] & 0xffff0000u);
            } else {
                xs[r * D + c + k] = __uint_as_float(t[k]);
            }
        }
    }
}
template <int XL>
__device__ __forceinline__ void few_row(const float *row, int lane, float (&v)[XL])
{
#pragma unroll
    for (int i = 0; i < XL / 2; ++i) {
        const float2 t = *reinterpret_cast<const float2 *>(row + few_elem(i, lane));
        v[2 * i] = t.x;
        v[2 * i + 1] = t.y;
    }
}
// LayerNorm of a row in registers, two-pass statistics; t: gain and bias in LDS
template <int D, int XL>
__device__ __forceinline__ void few_normalise(const float (&v)[XL], const float *t, float eps, int lane, float (&o)[XL])
{
    float s = 0.0f, sq = 0.0f;
#pragma unroll
    for (int i = 0; i < XL; i += 2) s += v[i] + v[i + 1];
    const float mean = wave_sum(s) / (float)D;
#pragma unroll
    for (int i = 0; i < XL; i += 2) {
        const float a = v[i] - mean, c = v[i + 1] - mean;
        sq += a * a + c * c;
    }
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);
#pragma unroll
    for (int i = 0; i < XL / 2; ++i) {
        const float2 g = *reinterpret_cast<const float2 *>(t + few_elem(i, lane)), b = *reinterpret_cast<const float2 *>(t + D + few_elem(i, lane));
        o[2 * i] = (v[2 * i] - mean) * rstd * g.x + b.x;
        o[2 * i + 1] = (v[2 * i + 1] - mean) * rstd * g.y + b.y;
    }
}
template <typename TW, int XL>
__device__ __forceinline__ void few_leave(unsigned char *row, int lane, const float (&o)[XL])
{
#pragma unroll
    for (int i = 0; i < XL / 2; ++i) {
        TW *q = reinterpret_cast<TW *>(row) + few_elem(i, lane);
        if constexpr (sizeof(TW) == 2) *reinterpret_cast<bf16x2_t *>(q) = __builtin_convertvector(f32x2_t{o[2 * i], o[2 * i + 1]}, bf16x2_t);
        else *reinterpret_cast<float2 *>(q) = make_float2(o[2 * i], o[2 * i + 1]);
    }
}
// State and mixer output of a channel: t, the in-projection without its bias
template <typename TW>
__device__ __forceinline__ TW few_mix(float t, float b_in, float s0, float al, float be, float la, bool row_repeat, int half, float &sn)
{
    const float u = (float)(TW)(t + b_in);           // u in the activation type
    const float pp = row_repeat ? al : 1.0f, qq = row_repeat ? 1.0f : al;
    sn = fmaf(la, s0, pp * u);
    if (half) sn = to_state(sn, static_cast<const f16 *>(nullptr));
    return (TW)fmaf(qq, sn, be);
}
// ... and of two channels without projections, whose output goes to the residual stream x; u: their LayerNorm
template <typename TW>
__device__ __forceinline__ void few_mix2(float2 &s, float *x, const float *u, float al, float be, float la, bool row_repeat, int half)
{
    const float pp = row_repeat ? al : 1.0f, qq = row_repeat ? 1.0f : al;
    s.x = fmaf(la, s.x, pp * (float)(TW)u[0]);
    s.y = fmaf(la, s.y, pp * (float)(TW)u[1]);
    if (half) {
        s.x = to_state(s.x, static_cast<const f16 *>(nullptr));
        s.y = to_state(s.y, static_cast<const f16 *>(nullptr));
    }
    x[0] += (float)(TW)fmaf(qq, s.x, be);
    x[1] += (float)(TW)fmaf(qq, s.y, be);
}
__device__ __forceinline__ float2 few_state2(const void *state, size_t at, int half)
{
    if (half) {
        const f16 *S = static_cast<const f16 *>(state) + at;
        return make_float2((float)S[0], (float)S[1]);
    }
    return *reinterpret_cast<const float2 *>(static_cast<const float *>(state) + at);
}
__device__ __forceinline__ void few_keep2(void *state, size_t at, int half, float2 s)
{
    if (half) {
        f16 *S = static_cast<f16 *>(state) + at;
        S[0] = (f16)s.x;
        S[1] = (f16)s.y;
    } else {
        *reinterpret_cast<float2 *>(static_cast<float *>(state) + at) = s;
    }
}
// Logits of group n of four columns (w: its vectors), below g1, and the best of a lane's so far
template <typename TW, int D, int MB>
__device__ __forceinline__ void few_scores(const FewArgs &p, const u32x4_t (&w)[D * (int)sizeof(TW) / 256], const unsigned char *act, int n, int g1,
                                           int pos, bool last, int lane, int ln, float (&bv)[(MB + 3) / 4], int (&bi)[(MB + 3) / 4])
{
    constexpr int RB = (MB + 3) / 4;
    float logit[RB];
    few_products<TW, D * (int)sizeof(TW) / 256, MB>(w, act, D * (int)sizeof(TW) + kFewPad, 0, lane, logit);
    const int c = 4 * n + few_column(ln);
    if (n < g1 && c < p.V && (ln & 12) == 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = 4 * rb + (ln & 3);
            if (row >= p.B) continue;
            if (p.logits && last) p.logits[(size_t)row * p.V + c] = logit[rb];
            const float score = p.temp > 0.0f
                ? logit[rb] + p.temp * srm_gumbel(srm_rowkey(p.seed, (uint32_t)pos, (uint32_t)(row + p.row0)), (uint32_t)c) : logit[rb];
            if (arg_better(score, c, bv[rb], bi[rb])) { bv[rb] = score; bi[rb] = c; }
        }
    }
}
// The best of a row's columns that the wavefronts of a work-group have left in `red`
template <int NWT, int RB>
__device__ __forceinline__ void few_best(const uint2 *red, int r, int lane, float &bv, int &bi)
{
    bv = -INFINITY;
    bi = 0x7fffffff;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint2 t = red[(min(lane, NWT - 1) * RB + r / 4) * 64 + (r & 3) + 16 * c];
        if (arg_better(__uint_as_float(t.x), (int)t.y, bv, bi)) { bv = __uint_as_float(t.x); bi = (int)t.y; }
    }
    best_of_lanes<16>(bv, bi);
}

// What group c of `rows` rows each sees of a call
__device__ __forceinline__ void few_group(FewArgs &p, int c, int rows, int D)
{
    const int r0 = c * rows;
    p.row0 = r0;
    p.B = min(rows, p.Bs - r0);
    p.tok_in += r0;
    p.tok_out += r0;
    if (p.store) p.store += r0;
    p.state = static_cast<unsigned char *>(p.state) + (size_t)r0 * D * (p.state_half ? 2 : 4);
    if (p.logits) p.logits += (size_t)r0 * p.V;
    if (p.hidden) p.hidden += (size_t)r0 * D;
}

constexpr int few_lds_bytes(int ts, int D, int NWC, int MB)
{
    return MB * (D * (4 + 6 * ts) + 3 * kFewPad) + MB * NWC * 4 * (4 + 4 + 1) + (kFewGather + NWC) * ((MB + 3) / 4) * 64 * 8 +
           8 * D * 4 + kFewMaxLayers * (int)sizeof(FewLayer) + 256;
}

// All steps by one work-group, for a launch whose work-groups have not all started (few_arrived): the same products, slices and
// sums as between them, so the same bits.  Bound by what one CU reads (figures at few_arrive_polls in srm.hip).  LDS as in
// few_rows_kernel, cleared; the tokens stand in tokb.
template <typename TW, int D, int NWT, int MB, bool PROJ>
__device__ __forceinline__ void few_alone(const FewArgs &p, const FewLayer *lay, float *xs, unsigned char *act_a, unsigned char *act_m,
                                          unsigned char *act_g, uint2 *red, float *lnp, int *tokb, int tid, int lane, int wave)
{
    constexpr int TS = (int)sizeof(TW), KD = D * TS / 1024, K4 = 4 * KD, RB = (MB + 3) / 4, XL = D / 64;
    constexpr int SD = D * TS + kFewPad, SF = 4 * D * TS + kFewPad;
    const int B = p.B, groups = (p.V + 3) / 4;
    auto opaque = [](int i) {                        // (as in few_rows_kernel: addresses are formed where they are used)
        asm volatile("" : "+v"(i));
        return i;
    };
    // (loads of the next piece are not moved in front of it: the kernel's registers are the other path's)
    auto piece = [] { asm volatile("" : : : "memory"); };
    auto vectors = [&](const void *W, int first, auto &w) {
        constexpr int K = sizeof(w) / sizeof(u32x4_t);
        const unsigned of = opaque(lane);
        const u32x4_t *base = static_cast<const u32x4_t *>(W) + (size_t)first * 64;
#pragma unroll
        for (int j = 0; j < K; ++j) w[j] = few_load(base + j * 64 + of);
    };
    // group n of four columns, the inputs in quarters of N vectors each
    auto quarters = [&](auto n_c, const void *W, int n, const unsigned char *act, int stride, float (&v)[RB]) {
        constexpr int N = decltype(n_c)::value;
        float q[4][RB];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            u32x4_t w[N];
            vectors(W, (n * 4 + k) * N, w);
            few_products<TW, N, MB>(w, act, stride, k * N, lane, q[k]);
            if (k & 1) piece();
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) v[rb] = (q[0][rb] + q[1][rb]) + (q[2][rb] + q[3][rb]);
    };
    // fn(row, its place in v, column) for what a lane holds of group n
    auto each = [&](int n, auto &&fn) {
        const int of = opaque(lane);
        if ((of & 12) == 0)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                if (4 * rb + (of & 3) < B) fn(4 * rb + (of & 3), rb, 4 * n + few_column(of));
    };
    auto parameters = [&](const float *a, const float *b, const float *c, const float *d) {
        for (int i = tid; i < 4 * D; i += NWT * 64) lnp[i] = few_load((i < 2 * D ? (i < D ? a : b) : (i < 3 * D ? c : d)) + i % D);
        __syncthreads();
    };
    auto normalised = [&](const float *t) {
        for (int r = wave; r < B; r += NWT) {
            const int of = opaque(lane);
            float v[XL], o[XL];
            few_row(xs + r * D, of, v);
            few_normalise<D>(v, t, p.eps, of, o);
            few_leave<TW>(act_a + r * SD, of, o);
        }
        __syncthreads();
    };
    for (int g = 0; g < p.G; ++g) {
        const int pos = p.pos0 + g;
        few_embed<TW, D, MB>(static_cast<const TW *>(p.embed), tokb, xs, tid, NWT * 64);
        for (int l = 0; l < p.L; ++l) {
            const FewLayer &y = lay[l];
            parameters(y.ln[0], y.ln[1], y.ln[2], y.ln[3]);
            if constexpr (PROJ) {
                normalised(lnp);
#pragma unroll 1
                for (int n = wave; n < D / 4; n += NWT) {
                    float v[RB];
                    quarters(std::integral_constant<int, KD>{}, y.w_in, n, act_a, SD, v);
                    each(n, [&](int r, int rb, int col) {
                        const int head = col / p.dh;
                        const size_t at = ((size_t)l * p.Bs + r) * D + col;
                        const float s0 = p.state_half ? (float)static_cast<const f16 *>(p.state)[at] : static_cast<const float *>(p.state)[at];
                        float sn;
                        const TW m = few_mix<TW>(v[rb], few_load(y.b_in + col), s0, few_load(y.alpha + (size_t)head * p.n_ctx + pos),
                                                 few_load(y.beta + (size_t)head * p.n_ctx + pos), few_load(y.lam + head), head < p.hrow,
                                                 p.state_half, sn);
                        if (p.state_half) static_cast<f16 *>(p.state)[at] = (f16)sn;
                        else static_cast<float *>(p.state)[at] = sn;
                        reinterpret_cast<TW *>(act_m + r * SD)[col] = m;
                    });
                }
                __syncthreads();
#pragma unroll 1
                for (int n = wave; n < D / 4; n += NWT) {
                    float v[RB];
                    quarters(std::integral_constant<int, KD>{}, y.w_out, n, act_m, SD, v);
                    each(n, [&](int r, int rb, int col) { xs[r * D + col] += v[rb] + few_load(y.b_out + col); });
                }
                __syncthreads();
                normalised(lnp + 2 * D);
            } else {
                for (int r = wave; r < B; r += NWT) {
                    const int of = opaque(lane);
                    float x[XL], u[XL];
                    few_row(xs + r * D, of, x);
                    few_normalise<D>(x, lnp, p.eps, of, u);
#pragma unroll
                    for (int i = 0; i < XL / 2; ++i) {
                        const int e = few_elem(i, of), h = e / p.dh;
                        const size_t at = ((size_t)l * p.Bs + r) * D + e;
                        float2 s = few_state2(p.state, at, p.state_half);
                        few_mix2<TW>(s, x + 2 * i, u + 2 * i, few_load(y.alpha + (size_t)h * p.n_ctx + pos),
                                     few_load(y.beta + (size_t)h * p.n_ctx + pos), few_load(y.lam + h), h < p.hrow, p.state_half);
                        few_keep2(p.state, at, p.state_half, s);
                        *reinterpret_cast<float2 *>(xs + r * D + e) = make_float2(x[2 * i], x[2 * i + 1]);
                        piece();
                    }
                    few_normalise<D>(x, lnp + 2 * D, p.eps, of, u);
                    few_leave<TW>(act_a + r * SD, of, u);
                }
                __syncthreads();
            }
#pragma unroll 1
            for (int n = wave; n < D; n += NWT) {
                u32x4_t w[K4];
                float v[RB];
                vectors(y.w_up, n * K4, w);
                few_products<TW, K4, MB>(w, act_a, SD, 0, lane, v);
                const float b = few_load(y.b_up + 4 * n + few_column(opaque(lane)));
                each(n, [&](int r, int rb, int col) {
                    reinterpret_cast<TW *>(act_g + r * SF)[col] = (TW)gelu_for(static_cast<const TW *>(nullptr), v[rb] + b);
                });
            }
            __syncthreads();
#pragma unroll 1
            for (int n = wave; n < D / 4; n += NWT) {
                float v[RB];
                quarters(std::integral_constant<int, K4>{}, y.w_down, n, act_g, SF, v);
                each(n, [&](int r, int rb, int col) { xs[r * D + col] += v[rb] + few_load(y.b_down + col); });
            }
            __syncthreads();
        }
        parameters(p.lnf_g, p.lnf_b, p.lnf_g, p.lnf_b);
        normalised(lnp);
        const bool last = g == p.G - 1;
        if (p.hidden && last)
            for (int i = tid; i < B * D; i += NWT * 64) p.hidden[i] = xs[i];
        float bv[RB];
        int bi[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            bv[rb] = -INFINITY;
            bi[rb] = 0x7fffffff;
        }
#pragma unroll 1
        for (int n = wave; n < groups; n += NWT) {
            u32x4_t w[K4];
            vectors(p.head, n * K4, w);
            few_scores<TW, D, MB>(p, w, act_a, n, groups, pos, last, lane, opaque(lane), bv, bi);
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) red[(wave * RB + rb) * 64 + lane] = make_uint2(__float_as_uint(bv[rb]), (unsigned)bi[rb]);
        __syncthreads();
        for (int r = wave; r < B; r += NWT) {
            float v;
            int t;
            few_best<NWT, RB>(red, r, lane, v, t);
            if (t < 0 || t >= p.V) t = 0;            // no ordered value: a valid token all the same
            if (lane == 0) {
                tokb[r] = t;
                if (p.store) p.store[(size_t)g * p.Bs + r] = t;
                if (last) p.tok_out[r] = t;
            }
        }
        __syncthreads();
    }
}

// MB: rows that the arithmetic is unrolled for (B <= MB); the rows between travel along as finite filler.
// XCD: MB rows to a group of work-groups, a group for each XCD (see few_group_rows in srm.hip), the groups on their own.
template <typename TW, int D, int NWC, int MB, bool PROJ, bool XCD = false>
__global__ void __launch_bounds__((kFewGather + NWC) * 64) few_rows_kernel(FewArgs p)
{
    constexpr int NG = kFewGather, NT = NG * 64, NWT = NG + NWC, NB = D / NWC, NALL = XCD ? kFewGroups * NB : NB, FF = 4 * D, TS = (int)sizeof(TW);
    // 1 KB vectors of four columns: of a slice (a quarter) of d inputs; of d inputs, or a slice of FF inputs
    constexpr int KD = D * TS / 1024, K4 = 4 * KD, RB = (MB + 3) / 4;
    constexpr int GC = TS == 2 ? 2 * NWC : 4 * NWC;                    // words of g per row and work-group
    constexpr int XL = D / 64, RPW = (MB + NG - 1) / NG;               // elements per lane of a row; rows per gathering wavefront
    constexpr int SD = D * TS + kFewPad, SF = FF * TS + kFewPad;       // row strides of the activations in LDS, bytes
    static_assert(D * TS % 1024 == 0 && D % NWC == 0 && NWC % 4 == 0, "whole vectors, whole groups of columns");
    static_assert(MB * GC <= NT && MB * NWC <= 64, "one word per thread to publish");
    extern __shared__ __align__(16) unsigned char few_lds[];
    float *const xs = reinterpret_cast<float *>(few_lds);                              // [MB][D] the residual stream
    unsigned char *const act_a = few_lds + MB * D * 4, *const act_m = act_a + MB * SD, *const act_g = act_m + MB * SD;
    float *const part = reinterpret_cast<float *>(act_g + MB * SF);                    // [4 slices][MB][NWC] partial products
    unsigned *const stage = reinterpret_cast<unsigned *>(part + 4 * MB * NWC);         // [MB][GC] words of g to publish
    float *const own = reinterpret_cast<float *>(stage + MB * 4 * NWC);                // [MB][NWC] x of the own columns
    uint2 *const red = reinterpret_cast<uint2 *>(own + MB * NWC);                      // [NWT][RB][64] winners per lane
    float *const lnp = reinterpret_cast<float *>(red + NWT * RB * 64);                 // [2][4][D] LayerNorm parameters of two layers
    FewLayer *const lay = reinterpret_cast<FewLayer *>(lnp + 8 * D);                   // [L] (a read of memory per phase is a trip of 1 us)
    int *const tokb = reinterpret_cast<int *>(lay + kFewMaxLayers);                    // [MB]
    int *const dead = tokb + MB;                                                       // [2], then the place in the groups [3]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int blk = blockIdx.x, B = p.B;
    bool near = false;
    const bool gatherer = wave < NG;
    const int cw = wave - NG;                        // number of a computing wavefront
    const TW *const embed = static_cast<const TW *>(p.embed);

    // (arrivals: words of the winners, which nobody writes before all have arrived; groups do not wait for each other, and have
    // theirs behind the winners)
    few_word *const here = XCD ? p.pw + (size_t)kFewGroups * MB * NB * 2 : p.pw;
    int me = 0;
    if (tid == 0) {
        few_word found;
        few_set(here + blk * (XCD ? 1 : MB * 2), XCD ? kFewXcd0 + few_xcd() : kFewHere, found);
        me = (int)found;
    }
    for (int i = tid; i < (MB * D * 4 + 2 * MB * SD + MB * SF) / 16; i += blockDim.x)
        reinterpret_cast<u32x4_t *>(few_lds)[i] = u32x4_t{0, 0, 0, 0};
    for (int i = tid; i < p.L * (int)(sizeof(FewLayer) / 8); i += blockDim.x)
        reinterpret_cast<few_word *>(lay)[i] = reinterpret_cast<const few_word *>(p.layers)[i];
    auto tokens = [&] {
        if (tid < MB) tokb[tid] = tid < B ? min(max(p.tok_in[tid], 0), p.V - 1) : 0;
    };
    if constexpr (!XCD) tokens();
    if (wave == 0) {
        if constexpr (XCD) {
            // (whole groups of those that have started, each of which takes several groups of rows in turn where some are missing)
            const int own = __builtin_amdgcn_readfirstlane(me);
            const FewPlace place = few_place<NALL>(here, NALL, blk, own, lane, NB, p.arrive_polls, p.arrive_polls << 6);
            if (lane == 0) {
                *dead = place.arrived < NB;
                dead[2] = own < kFewXcd0 ? NALL : p.scattered ? place.order : place.at;        // (withdrawn: no group's)
                dead[3] = place.near(NB) && !p.scattered;
                dead[4] = place.arrived / NB;
            }
        } else {
            const bool all = few_arrived<NB>(here, MB * 2, lane, p.arrive_polls);
            if (lane == 0) *dead = !all;
        }
    }
    // LDS only: loads and stores of global memory stay in flight across it
    auto barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    barrier();
    if (__builtin_expect(*dead, 0)) {                // nothing but scratch has been written
        if (tid == 0)
            dead[1] = __hip_atomic_fetch_add(p.flag + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == NALL - 1;
        __syncthreads();
        if (!dead[1]) return;
        if constexpr (XCD) {
#pragma unroll 1
            for (int c = 0; c < kFewGroups && c * MB < p.Bs; ++c) {
                FewArgs q = p;
                few_group(q, c, MB, D);
                B = q.B;
                if (tid < MB) tokb[tid] = tid < B ? min(max(q.tok_in[tid], 0), q.V - 1) : 0;
                __syncthreads();
                few_alone<TW, D, NWT, MB, PROJ>(q, lay, xs, act_a, act_m, act_g, red, lnp, tokb, tid, lane, wave);
                __syncthreads();
            }
        } else {
            few_alone<TW, D, NWT, MB, PROJ>(p, lay, xs, act_a, act_m, act_g, red, lnp, tokb, tid, lane, wave);
        }
        return;
    }
    // All steps of the rows that p sees (*dead: a wait has given up)
    auto steps = [&]() __attribute__((always_inline)) {
    unsigned tag = 0;                                // of the latest exchange, the same in every wavefront
    // (indexes pass through opaque copies where they are used: what is derived from them would otherwise be formed once, in
    // front of all loops, for every phase, and held in registers that do not exist)
    auto opaque = [](int i) {
        asm volatile("" : "+v"(i));
        return i;
    };

    // ---- LM head, by all wavefronts: groups of four columns, NWT groups at a time
    const int groups = (p.V + 3) / 4, per = (groups + NB - 1) / NB, g0 = min(blk * per, groups), g1 = min(g0 + per, groups);
    auto head_at = [&](int n) { return (size_t)min(n, groups - 1) * K4 * 1024; };
    auto head_load = [&](u32x4_t (&w)[K4], int n) {
        const unsigned of = opaque(lane);
        const u32x4_t *base = reinterpret_cast<const u32x4_t *>(static_cast<const unsigned char *>(p.head) + head_at(n));
#pragma unroll
        for (int j = 0; j < K4; ++j) w[j] = (base + j * 64)[of];
    };
    // w, nx: the wavefront's first two groups; leaves every lane's winners in `red`
    auto head_phase = [&](u32x4_t (&w)[K4], u32x4_t (&nx)[K4], int pos, bool last) {
        const int ln = opaque(lane);
        float bv[RB];
        int bi[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            bv[rb] = -INFINITY;
            bi[rb] = 0x7fffffff;
        }
        auto group = [&](u32x4_t (&v)[K4], int n) { few_scores<TW, D, MB>(p, v, act_a, n, g1, pos, last, lane, ln, bv, bi); };
        for (int n = g0 + wave; n < g1; n += 2 * NWT) {
            group(w, n);
            head_load(w, n + 2 * NWT < g1 ? n + 2 * NWT : n);
            group(nx, n + NWT);
            head_load(nx, n + 3 * NWT < g1 ? n + 3 * NWT : n);
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) red[(wave * RB + rb) * 64 + lane] = make_uint2(__float_as_uint(bv[rb]), (unsigned)bi[rb]);
    };

    if (gatherer) {
        // ================================================================ gathering wavefronts
        // word f = (work-group, row, column within both) of all work-groups' words: thread f mod NT's
        auto gather = [&](auto n_c, const few_word *words, auto &&put) {
            constexpr int ALL = decltype(n_c)::value / NT, N = ALL > (NWT > 8 ? 16 : 32) ? (NWT > 8 ? 16 : 32) : ALL;
            static_assert(decltype(n_c)::value % (NT * N) == 0, "whole requests");
            const int t = opaque(tid);
#pragma unroll 1
            for (int i0 = 0; i0 < ALL; i0 += N) {
                few_word v[N];
                if (!few_gather(v, [&](int i) { return (words + (i0 + i) * NT) + (unsigned)t; }, tag, p)) { *dead = 1; return; }
#pragma unroll
                for (int i = 0; i < N; ++i) put((i0 + i) * NT + t, (unsigned)v[i]);
            }
        };
        auto gather_x = [&] {
            gather(std::integral_constant<int, MB * D>{}, p.xw, [&](int f, unsigned v) {
                const int b = f / (MB * NWC), r = f / NWC % MB, c = f % NWC;
                xs[r * D + b * NWC + c] = __uint_as_float(v);
            });
        };
        auto gather_m = [&] {
            gather(std::integral_constant<int, MB * D>{}, p.mw, [&](int f, unsigned v) {
                const int b = f / (MB * NWC), r = f / NWC % MB, at = b * NWC + f % NWC;
                if constexpr (TS == 2) *reinterpret_cast<unsigned short *>(act_m + r * SD + at * 2) = (unsigned short)v;
                else *reinterpret_cast<unsigned *>(act_m + r * SD + at * 4) = v;
            });
        };
        auto gather_g = [&] {
            gather(std::integral_constant<int, MB * GC * NB>{}, p.gw, [&](int f, unsigned v) {
                const int b = f / (MB * GC), r = f / GC % MB, c = f % GC;
                *reinterpret_cast<unsigned *>(act_g + r * SF + (b * GC + c) * 4) = v;
            });
        };
        auto exchange_g = [&] {
            barrier();                               // a is there
            barrier();                               // the words of g are staged
            ++tag;
            if (tid < MB * GC) few_put(p.gw + blk * (MB * GC) + tid, stage[tid], tag, near);
            gather_g();
            barrier();                               // g is there
        };
        auto leave_normalised = [&](const float *t) {
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int r = wave + q * NG;
                if (r >= MB) break;
                float v[XL], o[XL];
                few_row(xs + r * D, opaque(lane), v);
                few_normalise<D>(v, t, p.eps, opaque(lane), o);
                few_leave<TW>(act_a + r * SD, opaque(lane), o);
            }
        };
        for (int g = 0; g < p.G; ++g) {
            const int pos = p.pos0 + g;
            few_embed<TW, D, MB>(embed, tokb, xs, opaque(tid), NT);
            for (int l = 0; l < p.L; ++l) {
                const float *const t1 = lnp + (l & 1) * 4 * D, *const t2 = t1 + 2 * D;
                if (l > 0) gather_x();
                if constexpr (PROJ) {
                    barrier();                       // x is there
                    leave_normalised(t1);
                    barrier();                       // a is there
                    barrier();                       // the partial products are there
                    ++tag;
                    gather_m();
                    barrier();                       // m is there
                    barrier();                       // the partial products are there
                    ++tag;
                    gather_x();
                    barrier();
                    leave_normalised(t2);
                } else {
                    // whole rows: LayerNorm1, state update, x += m, LayerNorm2; everybody the same, and the new state is
                    // written where the next exchange has shown that everybody has read the old one
                    const float *const alpha = lay[l].alpha, *const beta = lay[l].beta, *const lam = lay[l].lam;
                    float2 s[RPW][XL / 2];
                    float al[XL / 2], be[XL / 2], la[XL / 2];
                    bool rr[XL / 2];
                    const int of = opaque(lane);
#pragma unroll
                    for (int i = 0; i < XL / 2; ++i) {
                        const int h = few_elem(i, of) / p.dh;                  // two consecutive channels lie in one head
                        rr[i] = h < p.hrow;
                        al[i] = few_load(alpha + (size_t)h * p.n_ctx + pos);
                        be[i] = few_load(beta + (size_t)h * p.n_ctx + pos);
                        la[i] = few_load(lam + h);
#pragma unroll
                        for (int q = 0; q < RPW; ++q) {
                            s[q][i] = few_state2(p.state, ((size_t)l * p.Bs + min(wave + q * NG, B - 1)) * D + few_elem(i, of), p.state_half);
                        }
                    }
                    barrier();
#pragma unroll
                    for (int q = 0; q < RPW; ++q) {
                        const int r = wave + q * NG;
                        if (r >= MB) break;
                        float x[XL], u[XL];
                        few_row(xs + r * D, opaque(lane), x);
                        few_normalise<D>(x, t1, p.eps, opaque(lane), u);
#pragma unroll
                        for (int i = 0; i < XL / 2; ++i) {
                            few_mix2<TW>(s[q][i], x + 2 * i, u + 2 * i, al[i], be[i], la[i], rr[i], p.state_half);
                            const int e = few_elem(i, of) - blk * NWC;         // (NWC is even: both columns are this work-group's or none)
                            if (e >= 0 && e < NWC) *reinterpret_cast<float2 *>(own + r * NWC + e) = make_float2(x[2 * i], x[2 * i + 1]);
                        }
                        few_normalise<D>(x, t2, p.eps, opaque(lane), u);
                        few_leave<TW>(act_a + r * SD, opaque(lane), u);
                    }
                    exchange_g();
#pragma unroll
                    for (int q = 0; q < RPW; ++q) {
                        if (wave + q * NG >= B) break;
#pragma unroll
                        for (int i = 0; i < XL / 2; ++i) {
                            if (i != blk) continue;                    // (there are at least XL / 2 work-groups)
                            few_keep2(p.state, ((size_t)l * p.Bs + wave + q * NG) * D + few_elem(i, of), p.state_half, s[q][i]);
                        }
                    }
                }
                if constexpr (PROJ) exchange_g();
                barrier();                           // the partial products are there
                if (*dead) goto out;
                ++tag;
            }
            gather_x();
            barrier();
            leave_normalised(lnp + (p.L & 1) * 4 * D);
            u32x4_t hw[K4], hn[K4];
            head_load(hw, g0 + wave);
            head_load(hn, g0 + wave + NWT);
            barrier();
            head_phase(hw, hn, pos, g == p.G - 1);
            barrier();
            ++tag;
            // a row's winners: four lanes of each wavefront, then those of all work-groups, which are the next tokens
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int r = wave + q * NG;
                if (r >= MB) break;
                float bv;
                int bi;
                few_best<NWT, RB>(red, r, lane, bv, bi);
                if (lane < 2) few_put(p.pw + (blk * MB + r) * 2 + lane, lane ? (unsigned)bi : __float_as_uint(bv), tag, near);
            }
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int r = wave + q * NG;
                if (r >= MB) break;
                constexpr int N = (NB + 63) / 64;
                few_word v[2 * N];
                if (!few_gather(v, [&](int i) { return p.pw + (min((i >> 1) * 64 + lane, NB - 1) * MB + r) * 2 + (i & 1); }, tag, p)) {
                    *dead = 1;
                    break;
                }
                float bv = -INFINITY;
                int bi = 0x7fffffff;
#pragma unroll
                for (int i = 0; i < N; ++i)
                    if (arg_better(__uint_as_float((unsigned)v[2 * i]), (int)(unsigned)v[2 * i + 1], bv, bi)) {
                        bv = __uint_as_float((unsigned)v[2 * i]);
                        bi = (int)(unsigned)v[2 * i + 1];
                    }
                best_of_lanes<64>(bv, bi);
                if (bi < 0 || bi >= p.V) bi = 0;     // no ordered value: a valid token all the same
                if (lane == 0) {
                    tokb[r] = bi;
                    if (blk == 0 && r < B) {
                        if (p.store) p.store[(size_t)g * p.Bs + r] = bi;
                        if (g == p.G - 1) p.tok_out[r] = bi;
                    }
                }
            }
            barrier();
            if (*dead) goto out;
        }
        return;
    } else {
        // ================================================================ computing wavefronts
        // Layer l's LayerNorm parameters (behind the last: the final LayerNorm's), straight into LDS: the gathering wavefronts
        // would poll behind these loads.  (Issued from an asm statement, see gemm_persist.hpp.)
        const unsigned lnp_lds = __builtin_amdgcn_readfirstlane(
            (unsigned)reinterpret_cast<unsigned long long>((__attribute__((address_space(3))) unsigned char *)lnp));
        auto uniform = [](const void *q) {
            const unsigned long long a = reinterpret_cast<unsigned long long>(q);
            return reinterpret_cast<const unsigned char *>(((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(a >> 32)) << 32) |
                                                           (unsigned)__builtin_amdgcn_readfirstlane((unsigned)a));
        };
        auto fetch_ln = [&](int l) {
            constexpr int PARTS = D / 256, N = (4 * PARTS + NWC - 1) / NWC;        // of 1 KB; per wavefront
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int q = (i * NWC + cw) % (4 * PARTS), a = q / PARTS;
                const float *const ln = lay[min(l, p.L - 1)].ln[a], *const lnf = a & 1 ? p.lnf_b : p.lnf_g;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                             :
                             : "s"(__builtin_amdgcn_readfirstlane(lnp_lds + (l & 1) * 4 * D * 4 + q * 1024)), "v"(lane * 16), "s"(uniform(l < p.L ? ln : lnf) + q % PARTS * 1024)
                             : "memory");
            }
        };
        // the vectors of this lane, 1 KB apart, from byte `at` of W
        auto weights = [&](const void *W, size_t at, auto &w) {
            constexpr int K = sizeof(w) / sizeof(u32x4_t);
            const unsigned of = opaque(lane);
            const u32x4_t *base = reinterpret_cast<const u32x4_t *>(uniform(W) + at);
#pragma unroll
            for (int j = 0; j < K; ++j) w[j] = few_load(base + j * 64 + of);
        };
        // This wavefront's shares: a quarter of the inputs of a group of four columns of the in-, out- and down-projection, and all
        // inputs of a group of the up-projection's.  The partial products of the quarters meet in LDS; wavefront 0 adds them and
        // makes the epilogue of all rows and columns of the work-group, a lane each.
        constexpr int GROUPS = NWC / 4;
        const int cq = cw % GROUPS, slice = cw / GROUPS;
        const size_t at_d = ((size_t)(blk * GROUPS + cq) * 4 + slice) * KD * 1024, at_f = 4 * at_d, at_up = (size_t)(blk * NWC + cw) * K4 * 1024;
        u32x4_t w_in[KD], w_out[KD], w_up[K4], w_down[K4];
        const bool lead = cw == 0;
        auto leave_partial = [&](const float (&v)[RB]) {
            const int ln = opaque(lane);
            if ((ln & 12) == 0)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    if (MB >= 4 || (ln & 3) < MB) part[(slice * MB + 4 * rb + (ln & 3)) * NWC + 4 * cq + few_column(ln)] = v[rb];
        };
        auto total = [&](int at) { return (part[at] + part[MB * NWC + at]) + (part[2 * MB * NWC + at] + part[3 * MB * NWC + at]); };
        float x_own = 0.0f;                          // lane (row, column) of wavefront 0
        // what its epilogues of a layer need, requested in the layer in front
        struct Epi { float b_in, b_out, b_down, al, be, la; unsigned s; };
        auto epilogue_operands = [&](int l, int pos) {
            const FewLayer &y = lay[l];
            const int ln = min(opaque(lane), MB * NWC - 1), r = min(ln / NWC, B - 1), col = blk * NWC + ln % NWC;
            Epi e{};
            e.b_down = few_load(y.b_down + col);
            if constexpr (PROJ) {
                const size_t at = ((size_t)l * p.Bs + r) * D + col;
                const int head = col / p.dh;
                e.b_in = few_load(y.b_in + col);
                e.b_out = few_load(y.b_out + col);
                e.al = few_load(y.alpha + (size_t)head * p.n_ctx + pos);
                e.be = few_load(y.beta + (size_t)head * p.n_ctx + pos);
                e.la = few_load(y.lam + head);
                e.s = p.state_half ? few_load(static_cast<const unsigned short *>(p.state) + at)
                                   : few_load(static_cast<const unsigned *>(p.state) + at);
            }
            return e;
        };
        auto up_bias = [&](int l) { return few_load(lay[l].b_up + 4 * (blk * NWC + cw) + few_column(opaque(lane))); };
        for (int g = 0; g < p.G; ++g) {
            const int pos = p.pos0 + g;
            Epi e = epilogue_operands(0, pos);
            float b_up = up_bias(0);
            fetch_ln(0);
            if constexpr (PROJ) {
                weights(lay[0].w_in, at_d, w_in);
                weights(lay[0].w_out, at_d, w_out);
            }
            weights(lay[0].w_down, at_f, w_down);
            asm volatile("s_waitcnt vmcnt(%0)" : : "i"(PROJ ? 6 * KD : K4) : "memory");           // the LayerNorm parameters are there
            for (int l = 0; l < p.L; ++l) {
                // The weights (160 KB of a layer and work-group, d = 1024) are requested where nobody polls: those of MLP up and of
                // the projections while the gathering wavefronts normalise, those of MLP down behind its own products.  A CU
                // takes them at 30 to 60 bytes per clock and returns all loads in order, so that every poll or publication behind
                // one waits for it.  (All behind the barriers that end the phases: polls of 2.1 us instead of 1.4.  Without any
                // weights 16 layers of d = 1024 take 136 us instead of 168.)  No branches around the loads: where one path has
                // fewer of them in flight, the compiler waits for more of them on the other.
                const bool more = l + 1 < p.L;
                const int l1 = more ? l + 1 : l;
                const FewLayer &y = lay[l], &nx = lay[l1];
                Epi en;
                float b_up_n;
                float v[RB];
                if constexpr (PROJ) {
                    barrier();                       // x is there
                    weights(y.w_up, at_up, w_up);
                    barrier();                       // a is there
                    few_products<TW, KD, MB>(w_in, act_a, SD, slice * KD, lane, v);
                    leave_partial(v);
                    barrier();                       // the partial products are there
                    ++tag;
                    if (lead) {
                        const int ln = opaque(lane), at = min(ln, MB * NWC - 1), r = at / NWC, col = blk * NWC + at % NWC;
                        if (l == 0) x_own = xs[r * D + col];
                        const float s0 = p.state_half ? (float)__builtin_bit_cast(f16, (unsigned short)e.s) : __uint_as_float(e.s);
                        float sn;
                        const TW m = few_mix<TW>(total(at), e.b_in, s0, e.al, e.be, e.la, col / p.dh < p.hrow, p.state_half, sn);
                        unsigned bits;
                        if constexpr (TS == 2) bits = __builtin_bit_cast(unsigned short, m);
                        else bits = __float_as_uint(m);
                        if (ln < MB * NWC) {
                            few_put(p.mw + blk * (MB * NWC) + ln, bits, tag, near);
                            if (r < B) {
                                const size_t sat = ((size_t)l * p.Bs + r) * D + col;
                                if (p.state_half) static_cast<f16 *>(p.state)[sat] = (f16)sn;
                                else static_cast<float *>(p.state)[sat] = sn;
                            }
                        }
                    }
                    barrier();                       // m is there
                    few_products<TW, KD, MB>(w_out, act_m, SD, slice * KD, lane, v);
                    leave_partial(v);
                    barrier();                       // the partial products are there
                    ++tag;
                    if (lead) {
                        const int ln = opaque(lane);
                        x_own += total(min(ln, MB * NWC - 1)) + e.b_out;
                        if (ln < MB * NWC) few_put(p.xw + blk * (MB * NWC) + ln, __float_as_uint(x_own), tag, near);
                    }
                }
                barrier();                           // x is there
                en = epilogue_operands(l1, pos);
                b_up_n = up_bias(l1);
                fetch_ln(l + 1);
                if constexpr (PROJ) {
                    weights(nx.w_in, at_d, w_in);
                    weights(nx.w_out, at_d, w_out);
                } else {
                    weights(y.w_up, at_up, w_up);
                }
                barrier();                           // a is there
                if constexpr (!PROJ)
                    if (lead) x_own = own[min(opaque(lane), MB * NWC - 1)];
                few_products<TW, K4, MB>(w_up, act_a, SD, 0, lane, v);
                {
                    const int ln = opaque(lane);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const float o = gelu_for(static_cast<const TW *>(nullptr), v[rb] + b_up);
                        if ((ln & 12) == 0 && (MB >= 4 || (ln & 3) < MB))
                            reinterpret_cast<TW *>(stage)[(4 * rb + (ln & 3)) * (4 * NWC) + 4 * cw + few_column(ln)] = (TW)o;
                    }
                }
                barrier();                           // the words of g are staged
                ++tag;
                barrier();                           // g is there
                few_products<TW, K4, MB>(w_down, act_g, SF, slice * K4, lane, v);
                // the next LayerNorms' parameters are there, with at least these loads behind them
                asm volatile("s_waitcnt vmcnt(%0)" : : "i"(PROJ ? 2 * KD : K4) : "memory");
                weights(nx.w_down, at_f, w_down);
                leave_partial(v);
                barrier();                           // the partial products are there
                if (*dead) goto out;
                ++tag;
                if (lead) {
                    const int ln = opaque(lane);
                    x_own += total(min(ln, MB * NWC - 1)) + e.b_down;
                    if (ln < MB * NWC) few_put(p.xw + blk * (MB * NWC) + ln, __float_as_uint(x_own), tag, near);
                }
                e = en;
                b_up = b_up_n;
            }
            if (p.hidden && lead && g == p.G - 1) {
                const int ln = opaque(lane);
                if (ln < B * NWC) p.hidden[(size_t)(ln / NWC) * D + blk * NWC + ln % NWC] = x_own;
            }
            barrier();                               // x is there
            weights(p.head, head_at(g0 + wave), w_up);
            weights(p.head, head_at(g0 + wave + NWT), w_down);
            barrier();                               // a is there
            head_phase(w_up, w_down, pos, g == p.G - 1);
            barrier();
            ++tag;
            barrier();                               // the tokens are there
            if (*dead) goto out;
        }
        return;
    }
out:
    if (tid < B) p.tok_out[tid] = -1;
    };
    if constexpr (XCD) {
        const int at = __builtin_amdgcn_readfirstlane(dead[2]), teams = __builtin_amdgcn_readfirstlane(dead[4]);
        near = __builtin_amdgcn_readfirstlane(dead[3]);
        blk = at % NB;
        if (at / NB >= teams) return;                // (the whole group)
        const FewArgs all = p;
        auto group = [&](int c) __attribute__((always_inline)) {
            few_group(p, c, MB, D);
            p.xw += (size_t)c * MB * D;
            p.mw += (size_t)c * MB * D;
            p.gw += (size_t)c * MB * GC * NB;
            p.pw += (size_t)c * MB * NB * 2;
            B = p.B;
            tokens();
            barrier();
            steps();
        };
        // (the usual case apart: as a loop, what is kept for its next round costs the steps their registers, 38.2 | 38.5 us a token)
        if (__builtin_expect(teams == kFewGroups, 1)) {
            if (at / NB * MB < p.Bs) group(at / NB);
            return;
        }
#pragma unroll 1
        for (int c = at / NB; c * MB < all.Bs; c += teams) {
            p = all;
            group(c);
            if (*dead) {                             // nor will the rest of its rows be right
                for (c += teams; c * MB < all.Bs; c += teams)
                    if (tid < min(MB, all.Bs - c * MB)) all.tok_out[c * MB + tid] = -1;
                return;
            }
            barrier();                               // (nobody reads the tokens any more)
        }
    } else {
        steps();
    }
}

// Words that an earlier call has left in the workspace must not pass for this call's: no tag is zero.  Also the nucleus
// pass's counter, and the token store of a call whose kernel may give up.  n: pairs of words; those from w0 to w1 (of arrivals, for
// tests) are withdrawn from the start.
__global__ void __launch_bounds__(256)
few_reset_kernel(u32x4_t *words, int n, int w0, int w1, int *counter, int32_t *store, int n_store)
{
    const int i0 = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    auto word = [&](int w) { return w >= w0 && w < w1 ? (unsigned)kFewWithdrawn : 0u; };
    for (int i = i0; i < n; i += step) words[i] = u32x4_t{word(2 * i), 0, word(2 * i + 1), 0};
    for (int i = i0; i < n_store; i += step) store[i] = -1;
    if (i0 == 0) *counter = 0;
}

// W [N][K] of elements of TS bytes -> groups of four rows, vectors of 16 bytes: vector (group, chunk, lane) holds row
// 4 group + (lane & 3) (the last row where there is none), elements from 16 bytes x (16 chunk + (lane >> 2)) on.
__global__ void __launch_bounds__(256)
few_pack_kernel(const u32x4_t *__restrict__ W, u32x4_t *__restrict__ out, int N, int row_vectors)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, n = (int64_t)((N + 3) / 4) * 4 * row_vectors;
    if (i >= n) return;
    const int lane = (int)(i & 63), chunks = row_vectors / 16;
    const int64_t t = i >> 6, group = t / chunks, chunk = t % chunks;
    out[i] = W[min(4 * group + (lane & 3), (int64_t)N - 1) * row_vectors + chunk * 16 + (lane >> 2)];
}
