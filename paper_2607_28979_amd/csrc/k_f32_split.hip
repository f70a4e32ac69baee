// fp32 translation path on the bf16 matrix cores, two launches per call:
//
//   layer 1: Hs[u][t][m*hidden+k] = GELU(W1_m z_t + b1_m)[k]  (erf GELU, App. C.2),
//     and in further workgroups of the same launch the router (logits = Wr z +
//     br, g = softmax, Top-K renormalised; paper Sec. 3, Definition
//     "Mixture-of-Translators")
//   layer 2: dst[j][t][o] = sum_{m,k} g_m Hs[u][t][m*hidden+k] W2_m[o][k] + sum_m g_m b2_m[o]
// which equals sum_m g_m (W2_m GELU(W1_m z + b1_m) + b2_m), Eq. mot_definition.
//
// Every fp32 operand x is split exactly into three bf16 values, x = h + m + l
// (each the round-to-nearest of what is left: 8 + 8 + 8 significand bits), and
// a product is eight v_mfma_f32_32x32x16_bf16: hh, hm, mh, mm, hl, lh, ml, lm.
// The term left out (ll) is below 2^-33 of a product.  hh has accumulators of
// its own, the seven small terms share another set, so a product is rounded once
// and a sum once per 16 products (the fp32 matrix core rounds once per 4): against
// 64 bits the result is closer than v_mfma_f32_16x16x4_f32 gives.  Eight bf16
// products cost half of the fp32 matrix core's time for the same fp32 product.
// (Without ml and lm, six products, a single product was off by up to 0.89e-7
// of itself instead of 0.60e-7.)
//
// A 32x32 block is computed again on v_mfma_f32_32x32x2_f32 where the split does
// not hold: where a result is not finite (operands above bf16's largest value,
// 3.39e38; infinities, NaN and overflow come out as plain fp32 gives them), and
// where one is so small beside its row's and column's largest operands that parts
// of operands or products below bf16's or fp32's least value could count
// (finish_block).
//
// Workgroup = 4 waves, TM (hidden or output) rows x TN tokens, K in steps of
// 32: a thread fetches 8 consecutive fp32 of a row (a step ahead), splits them
// and writes one 16-byte chunk per part into LDS, where row r keeps chunk c at
// c ^ ((r >> 2) & 3) (16 lanes reading one chunk of 16 rows touch 16 distinct
// bank groups).
//
// Bound: latency at one token tile (64 tokens: 84.8 -> 45.6 us per call against
// v_mfma_f32_16x16x4_f32 with operands straight from global memory; 42.5 with six
// products), the sum of splitting, LDS and MFMA issue at many (999 tokens: 698 ->
// 318 us, 119 TFLOP/s of fp32 products; 266 with six products and without the row
// maxima).  Error against 64 bits, both sizes: 7.0e-7 -> 2.7e-7.
#include <type_traits>

#include "mot_device.h"
#include "mot_internal.h"
#include "../../include/mot.h"

namespace mot {

namespace {

__device__ __forceinline__ f32x4 ld4(const float* ptr) { return *reinterpret_cast<const f32x4*>(ptr); }

__device__ __forceinline__ size_t src_off(const Problem& p, int i, int tok, int c) {
    const size_t layer = (size_t)i * p.n_tok * p.d_in;
    if (p.src_layout == MOT_LAYOUT_BTHD) return layer + (size_t)tok * p.d_in + c;
    const int b = tok / p.T, t = tok % p.T, hh = c / p.D_src, dd = c % p.D_src;
    return layer + (((size_t)b * p.H_src + hh) * p.T + t) * p.D_src + dd;
}

// max(m, |x|, |y|), NaN left out, in one instruction (fmaxf of loaded values costs
// three more, which quiet signalling NaN)
__device__ __forceinline__ float max_abs(float m, float x, float y) {
    float r;
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(m), "v"(x), "v"(y));
    return r;
}

__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Workgroups go to the 8 XCDs (an L2 each) round-robin by id: XCD k runs the
// k-th contiguous eighth of the n work items (units outer), so a unit's
// weights and rows are fetched into one L2 instead of eight.  Items >= n: none.
__device__ __forceinline__ int xcd_item(int n) { return (blockIdx.x & 7) * ((n + 7) >> 3) + (blockIdx.x >> 3); }

// One tile shape.  WM x WN waves, each MB x NB blocks of 32 x 32; STAGES LDS
// copies of a K step (two forms of the K loop, below).
template <int TM_, int TN_, int WM_, int WN_, int STAGES_>
struct Tile {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, STAGES = STAGES_;
    static constexpr int MB = TM / WM / 32, NB = TN / WN / 32;
    static constexpr int IA = TM * 4 / 256, IB = TN * 4 / 256;   // 8-value items per thread and K step
    static constexpr int PLANE = (TM + TN) * 4;                  // 16-byte chunks of one part
    static constexpr int LDS = STAGES * 3 * PLANE;
    static_assert(WM * WN == 4 && TM % (WM * 32) == 0 && TN % (WN * 32) == 0, "four waves of 32x32 blocks");
    static_assert(STAGES == 1 || STAGES == 2, "forms of the K loop");
    static_assert(TM * 4 % 256 == 0 && TN * 4 % 256 == 0, "whole items per thread");
};

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

template <class T>
struct Acc {
    f32x16 hi[T::MB][T::NB], lo[T::MB][T::NB];
    float big[T::IA + T::IB];   // largest magnitude this thread split of item q's row
};

// v of another lane of the quad
template <int CTRL>
__device__ __forceinline__ float quad_swap(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Row maxima of a tile (TM rows of A, then TN of B) from the threads' shares; ends
// in a barrier
template <class T>
__device__ __forceinline__ void row_maxima(const Acc<T>& acc, float* s_max) {
#pragma unroll
    for (int q = 0; q < T::IA + T::IB; ++q) {
        float v = acc.big[q];
        v = fmaxf(v, quad_swap<0xB1>(v));   // lane ^ 1
        v = fmaxf(v, quad_swap<0x4E>(v));   // lane ^ 2
        const int row = (q < T::IA ? 0 : T::TM) + (threadIdx.x >> 2) + 64 * (q < T::IA ? q : q - T::IA);
        if ((threadIdx.x & 3) == 0) s_max[row] = v;
    }
    __syncthreads();
}

// The K loop of one tile: acc[hi|lo][block] over nk steps of 32.  fetch_a(q,
// v) and fetch_b(q, v) load this thread's item q (the 8 values of chunk tid % 4
// of tile row (tid + 256 q) / 4) in the current step, zeros past K, and advance()
// moves them to the next; with SCALED, fetch_b returns a factor the values are
// multiplied by when they are used.
//
// STAGES = 1, for launches that fill the chip: split the step into LDS, barrier,
// products; three workgroups per CU overlap each other's phases.  (With six
// products, slotting the splitting between the MFMAs, below, measured 289 us
// against 274 us with 128 x 64 tiles, and 128 x 128 tiles 294-334 us: 999 tokens,
// 768 -> 2 x 256 -> 768, 24 units.)
//
// STAGES = 2, for few workgroups, where a CU holds one: a step is two halves (K
// 0..15 and 16..31) of MFMA slots.  The barrier sits between the halves: before
// it the second half's operands of step s have been read and step s + 1 has been
// written whole, so after it the first operands of step s + 1 are read and the
// writing of step s + 2 begins, into the stage of step s.  The vector work of
// splitting a step so spreads over a whole step's MFMAs: three stages per pair of
// values (h and the remainder; m and the remainder; l), a fixed share of them in
// each slot.  (64 tokens, six products: 43.5 against 47.5 us with STAGES = 1.)
//
// Fetches past the last step repeat it; what is split from them is not used.
template <class T, bool SCALED, class FA, class FB, class ADV>
__device__ __forceinline__ void k_loop(u32x4* lds, int nk, FA fetch_a, FB fetch_b, ADV advance, Acc<T>& acc) {
    constexpr int MB = T::MB, NB = T::NB, NI = T::IA + T::IB, STAGE = 3 * T::PLANE;
    constexpr int NM = 16 * MB * NB, H = NM / 2;   // MFMA slots of a step, of a half
    constexpr int NS = NI * 12, HS = NS / 2;       // splitting stages of a step, of a half
    constexpr int NR = 3 * (MB + NB);              // operand reads of a half
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 5, l32 = lane & 31;
    const int wm = w % T::WM, wn = w / T::WM;
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc.hi[a][b][e] = acc.lo[a][b][e] = 0.f;
#pragma unroll
    for (int q = 0; q < NI; ++q) acc.big[q] = 0.f;

    f32x4 raw[NI][2];
    float scale[T::IB];
    int sf = 0;
    auto fetch_item = [&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if constexpr (q < T::IA) fetch_a(q, raw[q]);
        else scale[q - T::IA] = fetch_b(q - T::IA, raw[q]);
        if constexpr (q == NI - 1) advance(++sf < nk);
    };
    // splitting stage t of the fetched step into LDS at stc; an item's next fetch
    // is issued once its last values are taken
    u32x4 ph, pm, pl;
    float rx, ry;
    auto split = [&](auto tc, u32x4* stc) {
        constexpr int t = decltype(tc)::value;
        constexpr int q = t / 12, pr = t / 3 % 4, st = t % 3;
        if constexpr (st == 0) {
            rx = raw[q][pr / 2][2 * (pr & 1)];
            ry = raw[q][pr / 2][2 * (pr & 1) + 1];
            if constexpr (SCALED && q >= T::IA) {
                rx *= scale[q - T::IA];
                ry *= scale[q - T::IA];
            }
            acc.big[q] = max_abs(acc.big[q], rx, ry);
            ph[pr] = pack_bf16x2(rx, ry);
            rx -= bf16_lo(ph[pr]);
            ry -= bf16_hi(ph[pr]);
            if constexpr (pr == 3) fetch_item(std::integral_constant<int, q>{});
        } else if constexpr (st == 1) {
            pm[pr] = pack_bf16x2(rx, ry);
            rx -= bf16_lo(pm[pr]);
            ry -= bf16_hi(pm[pr]);
        } else {
            pl[pr] = pack_bf16x2(rx, ry);
            if constexpr (pr == 3) {
                const int row = (q < T::IA ? 0 : T::TM) + (tid >> 2) + 64 * (q < T::IA ? q : q - T::IA);
                u32x4* at = stc + row * 4 + ((tid & 3) ^ ((row >> 2) & 3));
                at[0] = ph;
                at[T::PLANE] = pm;
                at[2 * T::PLANE] = pl;
            }
        }
    };
    u32x4 fa[2][3][MB], fb[2][3][NB];
    // operand read r (h parts first, the order of use) of half ks from LDS stage st
    auto read = [&](auto rc, auto ksc, const u32x4* stc) {
        constexpr int r = decltype(rc)::value, ks = decltype(ksc)::value, part = r / (MB + NB), o = r % (MB + NB);
        const u32x4* base = stc + part * T::PLANE;
        const int row = o < MB ? (wm * MB + o) * 32 + l32 : T::TM + (wn * NB + o - MB) * 32 + l32;
        const u32x4 v = base[row * 4 + ((2 * ks + g) ^ ((row >> 2) & 3))];
        if constexpr (o < MB) fa[ks][part][o] = v;
        else fb[ks][part][o - MB] = v;
    };
    auto mma = [&](auto ksc, auto kc) {   // slot k of half ks
        constexpr int ks = decltype(ksc)::value, k = decltype(kc)::value, t = k / (MB * NB), a = k / NB % MB, b = k % NB;
        constexpr int PA[8] = {0, 0, 1, 1, 0, 2, 1, 2}, PB[8] = {0, 1, 0, 1, 2, 0, 2, 1};
        f32x16& c = t == 0 ? acc.hi[a][b] : acc.lo[a][b];
        c = mfma_32x32x16(fa[ks][PA[t]][a], fb[ks][PB[t]][b], c);
    };
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    static_for<0, NI>([&](auto qc) { fetch_item(qc); });
    if constexpr (T::STAGES == 1) {
        for (int s = 0; s < nk; ++s) {
            lds_barrier();   // every wave has read the previous step
            static_for<0, NS>([&](auto tc) { split(tc, lds); });
            lds_barrier();
            static_for<0, 2>([&](auto ksc) {
                static_for<0, NR>([&](auto rc) { read(rc, ksc, lds); });
                static_for<0, H>([&](auto kc) { mma(ksc, kc); });
            });
        }
        return;
    }
    // step 0 and the first half of step 1 into LDS
    static_for<0, NS>([&](auto tc) { split(tc, lds); });
    static_for<0, HS>([&](auto tc) { split(tc, lds + STAGE); });
    lds_barrier();
    static_for<0, NR>([&](auto rc) { read(rc, c0, lds); });
    for (int s = 0; s < nk; ++s) {
        u32x4 *cur = lds + (s & 1) * STAGE, *other = lds + ((s & 1) ^ 1) * STAGE;
        static_for<0, 2 * H>([&](auto kc) {
            constexpr int ks = decltype(kc)::value / H, k = decltype(kc)::value % H;
            if constexpr (ks == 1 && k == 0) lds_barrier();
            mma(std::integral_constant<int, ks>{}, std::integral_constant<int, k>{});
            static_for<k * NR / H, (k + 1) * NR / H>([&](auto rc) {
                if constexpr (ks == 0) read(rc, c1, cur);
                else read(rc, c0, other);
            });
            static_for<k * HS / H, (k + 1) * HS / H>([&](auto tc) {
                if constexpr (ks == 0) split(std::integral_constant<int, HS + decltype(tc)::value>{}, other);
                else split(tc, cur);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
}

// hi + lo of a block, or, where the split does not hold for one of its elements,
// the block in plain fp32.  a(k), b(k): 4 values at k of this lane's row and
// column; row_max, col_max: the largest operand of each row, of this lane's column.
//
// A lost part of an operand is below 2^-125 (bf16 values under 2^-126 taken as
// 0) and meets an operand of the other side; a lost product is below 2^-126, and
// each of K has eight.  Against a result of at least 2^-93 K (1 + row_max +
// col_max) all of them together are below 2^-29 of it.  Results of ordinary data
// are far above that (1e-25 for operands around 1), but for exact zeros of rows or
// columns of zeros, where nothing is lost.
template <class FA, class FB>
__device__ __forceinline__ f32x16 finish_block(const f32x16& hi, const f32x16& lo, int K, const float* row_max,
                                               float col_max, FA a, FB b) {
    const int g = (threadIdx.x & 63) >> 5;
    const float least = (float)K * 0x1p-93f;
    f32x16 v;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x4 rm = ld4(row_max + 8 * i + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = 4 * i + r;
            v[e] = hi[e] + lo[e];
            const float mag = fabsf(v[e]);
            bad |= !(mag <= 3.402823466e38f) || (mag < least * (1.0f + rm[r] + col_max) && rm[r] > 0.f && col_max > 0.f);
        }
    }
    if (__any(bad)) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = 0.f;
        // a step of 8: the lanes of half g hold k .. k+3 of their half
#pragma unroll 1
        for (int k = 4 * g; k < K; k += 8) {
            const f32x4 av = a(k), bv = b(k);
#pragma unroll
            for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], bv[e], v, 0, 0, 0);
        }
    }
    return v;
}

// Router of 64 tokens of one unit, on v_mfma_f32_16x16x4_f32: wave w takes the
// 16-wide k blocks kb = w (mod 4) of a 16-row block (Wr rows, zeros from E on)
// for four groups of 16 tokens; the four partial sums are added in wave order
// through LDS.  For a 16-wide block lane l holds k = 4*(l/16) .. +3 of its row.
// Gate rows (zeros outside the Top-K set) go to p.gates, selections to usage.
__device__ __forceinline__ void router_tile(const Problem& p, uint32_t code, int tok0, f32x4 (*s_part)[64][4]) {
    const int j = unit_j(code), x = unit_x(code), i = unit_i(code), gs = unit_gslot(code), E = p.E;
    const size_t unit = (size_t)j * p.streams + x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, q = lane >> 4;
    const float* src = reinterpret_cast<const float*>(p.src[x]);
    const bool rvalid = l16 < E;
    const float* rrow = reinterpret_cast<const float*>(p.wr) + (unit * E + (rvalid ? l16 : 0)) * p.d_in;
    int tokc[4];
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) tokc[tg] = min(tok0 + tg * 16 + l16, p.n_tok - 1);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 racc[4];
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) racc[tg] = zero;
#pragma unroll 4
    for (int kb = w; kb < p.d_in / 16; kb += 4) {
        const int k = kb * 16 + 4 * q;
        const f32x4 a = rvalid ? ld4(rrow + k) : zero;
        f32x4 b[4];
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) b[tg] = ld4(src + src_off(p, i, tokc[tg], k));
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int tg = 0; tg < 4; ++tg)
                racc[tg] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st], b[tg][st], racc[tg], 0, 0, 0);
    }
    // racc[tg]: partial logits of experts 4q .. 4q+3 for token tg*16 + l16
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) s_part[w][tg * 16 + l16][q] = racc[tg];
    __syncthreads();
    const int tl = w * 16 + l16, tok = tok0 + tl;
    f32x4 lg = s_part[0][tl][q];
#pragma unroll
    for (int ww = 1; ww < 4; ++ww) {
        const f32x4 v = s_part[ww][tl][q];
#pragma unroll
        for (int r = 0; r < 4; ++r) lg[r] += v[r];
    }
    float g[MOT_MAX_EXPERTS];
#pragma unroll
    for (int qq = 0; qq < 4; ++qq)
#pragma unroll
        for (int r = 0; r < 4; ++r) g[4 * qq + r] = __shfl(lg[r], 16 * qq + l16, 64);
    const float* br = p.br ? reinterpret_cast<const float*>(p.br) + unit * E : nullptr;
    float mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m)
        if (m < E) {
            g[m] += br ? br[m] : 0.f;
            mx = fmaxf(mx, g[m]);
        }
    float den = 0.f;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) {
        g[m] = m < E ? expf(g[m] - mx) : 0.f;
        den += g[m];
    }
    const float inv = 1.0f / den;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) g[m] *= inv;
    const uint32_t taken = topk_renormalise(g, E, p.top_k);
    const bool owner = q == 0 && tok < p.n_tok;
    if (owner) {
        float* G = p.gates + ((size_t)gs * p.n_tok_pad + tok) * E;
#pragma unroll
        for (int m = 0; m < MOT_MAX_EXPERTS; ++m)
            if (m < E) G[m] = g[m];
    }
    if (p.usage) count_usage(p.usage + unit * E, E, taken, owner);
}

// work items (xcd_item): per unit its router tiles (64 tokens each), then
// (hidden tiles) x (token tiles), hidden fastest.  GENERAL: d_in % 32 == 16, or
// a BHTD source with heads of other than whole 32s
template <class T, bool GENERAL>
__global__ __launch_bounds__(256, 3) void k_f32_split_gemm1(Problem p, UnitTab ut) {
    __shared__ u32x4 s_lds[T::LDS];
    __shared__ __align__(16) float s_max[T::TM + T::TN];
    static_assert(T::LDS >= 4 * 64 * 4, "the router's partial logits fit");
    const int EH = p.E * p.hidden, nA = (EH + T::TM - 1) / T::TM, d_in = p.d_in;
    const int nr = (p.n_tok + 63) / 64, per = nr + nA * ((p.n_tok + T::TN - 1) / T::TN);
    const int item = xcd_item(ut.n * per);
    if (item >= ut.n * per) return;   // uniform over the workgroup
    const int uz = item / per, id = item % per - nr;
    const uint32_t code = ut.code[uz];
    if (id < 0) {   // uniform over the workgroup
        router_tile(p, code, (id + nr) * 64, reinterpret_cast<f32x4(*)[64][4]>(s_lds));
        return;
    }
    const int j = unit_j(code), x = unit_x(code), i = unit_i(code);
    const int hid0 = id % nA * T::TM, tok0 = id / nA * T::TN;
    const size_t unit = (size_t)j * p.streams + x;
    const float* W1 = reinterpret_cast<const float*>(p.w1) + unit * EH * d_in;
    const float* src = reinterpret_cast<const float*>(p.src[x]);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // item rows of this thread, and the walk over K: a BHTD source goes on in
    // the next head every D_src values (head_gap away).  GENERAL: a chunk may
    // lie past the end of K, or its two halves in two heads
    const int c8 = (threadIdx.x & 3) * 8, r4 = threadIdx.x >> 2;
    const int seg = p.src_layout == MOT_LAYOUT_BTHD ? d_in : p.D_src;
    const size_t head_gap = (size_t)(p.T - 1) * seg;
    const float *arow[T::IA], *brow[T::IB];
    int tokq[T::IB], k0 = 0, in_seg = 0;
    size_t koff = 0;
#pragma unroll
    for (int q = 0; q < T::IA; ++q) arow[q] = W1 + (size_t)min(hid0 + r4 + 64 * q, EH - 1) * d_in + c8;
#pragma unroll
    for (int q = 0; q < T::IB; ++q) {
        tokq[q] = min(tok0 + r4 + 64 * q, p.n_tok - 1);
        brow[q] = src + src_off(p, i, tokq[q], 0) + c8;
    }
    Acc<T> acc;
    k_loop<T, false>(
        s_lds, (d_in + 31) / 32,
        [&](int q, f32x4 (&v)[2]) {
            if (GENERAL && k0 + c8 >= d_in) {   // d_in % 16 == 0: all of the chunk
                v[0] = v[1] = zero;
            } else {
                v[0] = ld4(arow[q] + k0);
                v[1] = ld4(arow[q] + k0 + 4);
            }
        },
        [&](int q, f32x4 (&v)[2]) {
            if (GENERAL && k0 + c8 >= d_in) {
                v[0] = v[1] = zero;
            } else if (GENERAL) {   // D_src % 4 == 0: four values in one head
                v[0] = ld4(src + src_off(p, i, tokq[q], k0 + c8));
                v[1] = ld4(src + src_off(p, i, tokq[q], k0 + c8 + 4));
            } else {
                v[0] = ld4(brow[q] + koff);
                v[1] = ld4(brow[q] + koff + 4);
            }
            return 1.0f;
        },
        [&](bool more) {
            const int by = more ? 32 : 0;
            k0 += by;
            in_seg += by;
            const bool next = in_seg == seg && more;   // seg % 32 == 0 unless GENERAL
            koff += by + (next ? head_gap : 0);
            in_seg = next ? 0 : in_seg;
        },
        acc);
    row_maxima(acc, s_max);

    // epilogue: + b1, GELU; a lane holds hidden rows 8e + 4g .. +3 of the block
    // for token l32
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 5, l32 = lane & 31;
    float* H = reinterpret_cast<float*>(p.hbuf) + (size_t)uz * p.n_tok_pad * EH;
    const float* b1 = p.b1 ? reinterpret_cast<const float*>(p.b1) + unit * EH : nullptr;
#pragma unroll
    for (int a = 0; a < T::MB; ++a)
#pragma unroll
        for (int b = 0; b < T::NB; ++b) {
            const int hr = (w % T::WM * T::MB + a) * 32, tc = (w / T::WM * T::NB + b) * 32 + l32;
            const int h0 = hid0 + hr, tok = tok0 + tc, tokc = min(tok, p.n_tok - 1);
            const float* wrow = W1 + (size_t)min(h0 + l32, EH - 1) * d_in;
            const f32x16 s = finish_block(
                acc.hi[a][b], acc.lo[a][b], d_in, s_max + hr, s_max[T::TM + tc], [&](int k) { return ld4(wrow + k); },
                [&](int k) { return ld4(src + src_off(p, i, tokc, k)); });
            if (tok >= p.n_tok) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int h = h0 + 8 * e + 4 * g;
                if (h >= EH) continue;   // EH % 64 == 0
                const f32x4 bias = b1 ? ld4(b1 + h) : zero;
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float y = s[4 * e + r] + bias[r];
                    v[r] = p.act == MOT_ACT_GELU ? gelu_erf(y) : y;
                }
                *reinterpret_cast<f32x4*>(H + (size_t)tok * EH + h) = v;
            }
        }
}

// work items (xcd_item): per unit (output tiles) x (token tiles), outputs fastest
template <class T>
__global__ __launch_bounds__(256, 3) void k_f32_split_gemm2(Problem p, UnitTab ut) {
    __shared__ u32x4 s_lds[T::LDS];
    __shared__ __align__(16) float s_max[T::TM + T::TN];
    const int E = p.E, hidden = p.hidden, EH = E * hidden, d_out = p.d_out, nA = (d_out + T::TM - 1) / T::TM;
    const int per = nA * ((p.n_tok + T::TN - 1) / T::TN), item = xcd_item(ut.n * per);
    if (item >= ut.n * per) return;   // uniform over the workgroup
    const int uz = item / per, id = item % per;
    const uint32_t code = ut.code[uz];
    const int j = unit_j(code), x = unit_x(code), gs = unit_gslot(code);
    const int out0 = id % nA * T::TM, tok0 = id / nA * T::TN;
    const size_t unit = (size_t)j * p.streams + x;
    const float* W2 = reinterpret_cast<const float*>(p.w2) + unit * E * d_out * hidden;
    const float* H = reinterpret_cast<const float*>(p.hbuf) + (size_t)uz * p.n_tok_pad * EH;
    const float* G = p.gates + (size_t)gs * p.n_tok_pad * E;
    const int c8 = (threadIdx.x & 3) * 8, r4 = threadIdx.x >> 2;
    const float *arow[T::IA], *brow[T::IB], *grow[T::IB];
#pragma unroll
    for (int q = 0; q < T::IA; ++q) arow[q] = W2 + (size_t)min(out0 + r4 + 64 * q, d_out - 1) * hidden + c8;
#pragma unroll
    for (int q = 0; q < T::IB; ++q) {
        const int tok = min(tok0 + r4 + 64 * q, p.n_tok - 1);
        brow[q] = H + (size_t)tok * EH + c8;
        grow[q] = G + (size_t)tok * E;
    }
    // hidden % 64 == 0: a step stays in one translator m; its rows of W2 are
    // w2_gap after the previous one's
    const size_t w2_gap = (size_t)(d_out - 1) * hidden;
    int m = 0, kk = 0;
    size_t aoff = 0, boff = 0;
    Acc<T> acc;
    k_loop<T, true>(
        s_lds, EH / 32,
        [&](int q, f32x4 (&v)[2]) {
            v[0] = ld4(arow[q] + aoff);
            v[1] = ld4(arow[q] + aoff + 4);
        },
        [&](int q, f32x4 (&v)[2]) {
            v[0] = ld4(brow[q] + boff);
            v[1] = ld4(brow[q] + boff + 4);
            return grow[q][m];
        },
        [&](bool more) {
            const int by = more ? 32 : 0;
            kk += by;
            const bool next = kk == hidden && more;
            boff += by;
            aoff += by + (next ? w2_gap : 0);
            kk = next ? 0 : kk;
            m += next ? 1 : 0;
        },
        acc);
    row_maxima(acc, s_max);

    // epilogue: + sum_m g_m b2_m; a lane holds outputs 8e + 4g .. +3 of the
    // block for token l32
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 5, l32 = lane & 31;
    float* dst = reinterpret_cast<float*>(p.dst[x]) + (size_t)j * p.n_tok * d_out;
    const float* b2 = p.b2 ? reinterpret_cast<const float*>(p.b2) + unit * E * d_out : nullptr;
#pragma unroll
    for (int a = 0; a < T::MB; ++a)
#pragma unroll
        for (int b = 0; b < T::NB; ++b) {
            const int orel = (w % T::WM * T::MB + a) * 32, tc = (w / T::WM * T::NB + b) * 32 + l32;
            const int o0 = out0 + orel, tok = tok0 + tc;
            const int tokc = min(tok, p.n_tok - 1), orow = min(o0 + l32, d_out - 1);
            const f32x16 y = finish_block(
                acc.hi[a][b], acc.lo[a][b], EH, s_max + orel, s_max[T::TM + tc],
                [&](int k) { return ld4(W2 + ((size_t)(k / hidden) * d_out + orow) * hidden + k % hidden); },
                [&](int k) {
                    const float gate = G[(size_t)tokc * E + k / hidden];
                    f32x4 h = ld4(H + (size_t)tokc * EH + k);
#pragma unroll
                    for (int r = 0; r < 4; ++r) h[r] *= gate;
                    return h;
                });
            if (tok >= p.n_tok) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = o0 + 8 * e + 4 * g;
                if (o >= d_out) continue;   // d_out % 4 == 0
                f32x4 v = {y[4 * e], y[4 * e + 1], y[4 * e + 2], y[4 * e + 3]};
                if (b2) {
                    f32x4 s = {0.f, 0.f, 0.f, 0.f};
                    for (int m = 0; m < E; ++m) {
                        const f32x4 bv = ld4(b2 + (size_t)m * d_out + o);
                        const float gate = G[(size_t)tok * E + m];
#pragma unroll
                        for (int r = 0; r < 4; ++r) s[r] = fmaf(gate, bv[r], s[r]);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] += s[r];
                }
                size_t off;
                if (p.dst_layout == MOT_LAYOUT_BTHD) {
                    off = (size_t)tok * d_out + o;
                } else {   // D_tgt % 4 == 0: o .. o+3 in one head
                    const int bb = tok / p.T, t = tok % p.T, hh = o / p.D_tgt, dd = o % p.D_tgt;
                    off = (((size_t)bb * p.H_tgt + hh) * p.T + t) * p.D_tgt + dd;
                }
                *reinterpret_cast<f32x4*>(dst + off) = v;
            }
        }
}

typedef Tile<128, 64, 2, 2, 1> Large;
typedef Tile<64, 64, 2, 2, 2> Small;

// Large tiles when they make at least a workgroup per CU
constexpr int kCUs = 256;

bool large_tiles(const Problem& p, const UnitTab& ut, int rows) {
    return (int64_t)((rows + Large::TM - 1) / Large::TM) * ((p.n_tok + Large::TN - 1) / Large::TN) * ut.n >= kCUs;
}

template <class T>
void launch1(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    const int EH = p.E * p.hidden;
    const int items = ut.n * ((p.n_tok + 63) / 64 + (EH + T::TM - 1) / T::TM * ((p.n_tok + T::TN - 1) / T::TN));
    const dim3 grid((items + 7) / 8 * 8);
    const bool general = p.d_in % 32 || (p.src_layout != MOT_LAYOUT_BTHD && p.D_src % 32);
    if (general) hipLaunchKernelGGL((k_f32_split_gemm1<T, true>), grid, dim3(256), 0, stream, p, ut);
    else hipLaunchKernelGGL((k_f32_split_gemm1<T, false>), grid, dim3(256), 0, stream, p, ut);
}

template <class T>
void launch2(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    const dim3 grid((ut.n * ((p.d_out + T::TM - 1) / T::TM * ((p.n_tok + T::TN - 1) / T::TN)) + 7) / 8 * 8);
    hipLaunchKernelGGL(k_f32_split_gemm2<T>, grid, dim3(256), 0, stream, p, ut);
}

}  // namespace

bool f32_split_fits(const Problem& p) {
    return p.hidden % 64 == 0 && p.d_in % 16 == 0 && p.d_out % 4 == 0 && p.E <= MOT_MAX_EXPERTS;
}

hipError_t launch_f32_split_gemm1(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    if (ut.n == 0 || p.n_tok == 0) return hipSuccess;
    large_tiles(p, ut, p.E * p.hidden) ? launch1<Large>(p, ut, stream) : launch1<Small>(p, ut, stream);
    return hipGetLastError();
}

hipError_t launch_f32_split_gemm2(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    if (ut.n == 0 || p.n_tok == 0) return hipSuccess;
    large_tiles(p, ut, p.d_out) ? launch2<Large>(p, ut, stream) : launch2<Small>(p, ut, stream);
    return hipGetLastError();
}

}  // namespace mot
