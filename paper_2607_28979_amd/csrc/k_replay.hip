// Context replay after translation (paper App. C.4, "Post-Translation Phase:
// Cache Replay"): Top-S source-guided sparse attention.
//
// * k_topS_select: for each query position u, the S key positions v <= u
//   with the largest head-averaged source attention A[b][u][v] (ties to the
//   lower position), in ascending position order, padded with -1.  Radix
//   select over order-preserving 32-bit keys: a lower bound from the threads'
//   largest keys, then a 1024-bin histogram of the top 10 bits above it finds
//   the bin holding the S-th largest key; that bin's keys (a few dozen on
//   attention rows) are ranked against each other for the exact key, or, past
//   256 of them, 8-bit radix passes over the lower bits finish the search; then
//   one ordered pass keeps every larger key and the lowest-positioned equal ones.
// * k_sparse_attn_group: attention of every query head over the key sets
//   (grouped-query: query head h reads KV head h / G), four positions and one
//   KV head per wave over the union of the positions' sets, for G <= 8.
// * k_sparse_attn: the same for one position (more than 8 query heads per KV
//   head, K of 2 GiB and more per batch row, short calls on few KV heads).  Per
//   KV head the workgroup computes scores^T = K_sel . Q^T on
//   v_mfma_f32_16x16x32_bf16 with the gathered key rows loaded straight into A
//   operands, a softmax over the set, and O^T = V_sel^T . P^T with V_sel staged
//   transposed in LDS.
// * k_causal_attn: the full causal attention of the bottom layers, tiled (tiles
//   of 128 query positions of one head, 64-key chunks of K and V^T loaded
//   straight into LDS one chunk ahead, online softmax,
//   v_mfma_f32_32x32x16_bf16).
// Scores, softmax and accumulation are fp32; Q, K, V, O are bf16.
#include "mot_device.h"
#include "mot_internal.h"
#include "../../include/mot.h"

namespace mot {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((address_space(3))) void lds_void;
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// Raw buffer over `bytes` bytes at `base` (reads past the end return 0).
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0,
                                             (int)(bytes < 0xFFFFFFFFu ? bytes : 0xFFFFFFFFu), 0x00020000);
}

// 16 bytes per lane from the buffer straight into this wave's 1 KB of LDS
__device__ __forceinline__ void load_lds16(rsrc_t r, uint32_t off, u32x4* lds_dst_wave_base) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)lds_dst_wave_base, 16, off, 0, 0, 0);
}

// Monotone map float -> uint32 (a < b  <=>  key(a) < key(b) for non-NaN).
__device__ __forceinline__ uint32_t order_key(float a) {
    const uint32_t b = __float_as_uint(a);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int kSelBits = 10, kSelBins = 1 << kSelBits;   // first radix digit
constexpr int kSelCand = 256;                              // boundary-bin keys ranked directly
static_assert(kSelBins == 4 * 256, "four first-digit bins per thread");

// Where a selection's keys come from.  RegKeys: the row in registers, NV pieces of Q
// values per thread (piece i of thread t: positions 256 Q i + Q t .. + Q - 1), for T
// <= 256 Q NV.  RowKeys: read from the row again in every pass, one per thread and
// 256 positions (longer rows).  BOUND: length from which a row is searched for a
// lower bound before its keys are counted (0: never).
//
// for_each<EXACT>(f): f(key) for every position < n of this thread, and, unless
// EXACT, f(0) for others (0 is the least key); chunks(f): f(chunk,
// this lane's Q keys, their first position, n) for each chunk of 64 Q positions of
// this wave, by all its lanes (positions >= n among them).
template <int NV, int Q_ = 4>
struct RegKeys {
    static constexpr int Q = Q_, P = 256 * Q;   // positions of a piece of the threads
    // shorter rows pay more for the extra pass than its atomics cost (a map of 2048
    // positions, sets of 128: 13.1 us with it from 1024 on, 12.3 without)
    static constexpr int BOUND = P * NV > 3072 ? 3072 : 0;
    // waves per SIMD the registers are limited to (NV = 8: 6 measured best of 4, 6, 8)
    static constexpr int WAVES = NV <= 4 ? 8 : NV <= 8 ? 6 : 4;
    uint32_t k[NV][Q];
    int n;
    __device__ __forceinline__ void load(const float* row, int T, int n_) {
        n = n_;
        // a row on a 16-byte boundary with T % 4 == 0 (uniform): a piece may end past
        // u, still inside the row; the rest is never used
        const bool whole = Q == 4 && (T & 3) == 0 && (reinterpret_cast<uintptr_t>(row) & 15) == 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int v = P * i + Q * threadIdx.x;
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
            if (v < n) {
                if (whole) {
                    a = *reinterpret_cast<const f32x4*>(row + v);
                } else {
#pragma unroll
                    for (int c = 0; c < Q; ++c)
                        if (v + c < n) a[c] = row[v + c];
                }
            }
#pragma unroll
            for (int c = 0; c < Q; ++c) k[i][c] = v + c < n ? order_key(a[c]) : 0u;
        }
    }
    // n as a new value in each pass: the comparisons with it are made again
    // instead of being kept in scalar registers (which spills them)
    __device__ __forceinline__ int bound() const {
        int m = n;
        asm volatile("" : "+s"(m));
        return m;
    }
    template <bool EXACT, class F>
    __device__ __forceinline__ void for_each(F f) const {
        const int m = bound();
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (P * i < m)   // uniform
#pragma unroll
                for (int c = 0; c < Q; ++c)
                    if (!EXACT || P * i + Q * (int)threadIdx.x + c < m) f(k[i][c]);
    }
    template <class F>
    __device__ __forceinline__ void chunks(F f) const {
        const int m = bound();
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (P * i < m) f(4 * i + (threadIdx.x >> 6), k[i], P * i + Q * (int)threadIdx.x, m);
    }
};

struct RowKeys {
    static constexpr int Q = 1, WAVES = 8;
    static constexpr int BOUND = 0;   // T = 17000, sets of 128: 753 us with it, 633 without
    const float* row;
    int n;
    __device__ __forceinline__ void load(const float* r, int, int n_) {
        row = r;
        n = n_;
    }
    template <bool EXACT, class F>
    __device__ __forceinline__ void for_each(F f) const {
        for (int v = threadIdx.x; v < n; v += 256) f(order_key(row[v]));
    }
    template <class F>
    __device__ __forceinline__ void chunks(F f) const {
        for (int v0 = 0; v0 < n; v0 += 256) {
            const int v = v0 + threadIdx.x;
            const uint32_t k[1] = {v < n ? order_key(row[v]) : 0u};
            f(v >> 6, k, v, n);
        }
    }
};

// Bound: latency of its passes and vector instructions (waves wait 57 % of their
// cycles, the vector ALUs are 39 % busy).  8192 rows of a causal map, sets of 128: 119
// us with the row's keys in LDS (4 workgroups per CU, every key counted by an LDS
// atomic), 55 us with them in registers and one key in ten counted (6 waves per SIMD
// spill 8 registers: 65 MB of writes beside the 4 MB of sets).
//
// grid (T, B), 256 threads; dynamic LDS: per-chunk counts s_gt, s_eq
// (T / (64 Q) + 4 each)
template <class Keys>
__global__ __launch_bounds__(256, Keys::WAVES) void k_topS_select(const float* A, int32_t* idx, int T, int S) {
    extern __shared__ int s_gt[];
    constexpr int Q = Keys::Q;
    __shared__ uint32_t hist[kSelBins];
    __shared__ uint32_t hist_max[Keys::BOUND > 0 ? kSelBins : 1];
    __shared__ uint32_t s_cand[kSelCand];
    __shared__ uint32_t s_sel[3], s_wsum[4];
    __shared__ int s_cnt;
    const int u = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int n = u + 1;
    int32_t* out = idx + ((size_t)b * T + u) * S;
    if (n <= S) {   // every causal position is kept (uniform exit, before any barrier)
        for (int c = tid; c < S; c += 256) out[c] = c < n ? c : -1;
        return;
    }
    int* s_eq = s_gt + T / (64 * Q) + 4;
    Keys keys;
    keys.load(A + ((size_t)b * T + u) * T, T, n);
    // first digit: the top kSelBits bits (sign, exponent and one mantissa bit).
    // 1024 bins: an attention row's keys crowd into a few exponents, and with
    // an 8-bit first digit the boundary bin held ~70 keys and needed another
    // full radix pass; with 10 bits it holds a few dozen, ranked directly.
    constexpr int sh1 = 32 - kSelBits;
    if (tid < 64) s_cnt = 0;
#pragma unroll
    for (int i = 0; i < kSelBins / 256; ++i) hist[tid + 256 * i] = 0;
    static_assert(Keys::BOUND == 0 || Keys::BOUND >= 256 * Q, "every thread holds a key");
    const bool bound = Keys::BOUND > 0 && S <= 256 && n >= Keys::BOUND;   // uniform
    if (bound)
#pragma unroll
        for (int i = 0; i < kSelBins / 256; ++i) hist_max[tid + 256 * i] = 0;
    __syncthreads();
    // the bin of h holding the S-th largest key -> s_sel: thread t holds bins
    // 4t .. 4t+3, suffix sums over the threads (within each wave by shuffles, then
    // the higher waves' totals); ends in a barrier
    auto find_bin = [&](const uint32_t* h) {
        const int lane = tid & 63, wv = tid >> 6;
        const uint32_t hb[4] = {h[4 * tid], h[4 * tid + 1], h[4 * tid + 2], h[4 * tid + 3]};
        const uint32_t c = hb[0] + hb[1] + hb[2] + hb[3];
        uint32_t suf = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_down(suf, off, 64);
            if (lane + off < 64) suf += t;
        }
        if (lane == 0) s_wsum[wv] = suf;
        __syncthreads();
        for (int q = wv + 1; q < 4; ++q) suf += s_wsum[q];
        if (suf >= (uint32_t)S && suf - c < (uint32_t)S) {
            uint32_t cum = suf - c;   // keys in bins above 4t+3
            int d = 4 * tid;
            uint32_t cnt = hb[0];
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                if (cum + hb[q] >= (uint32_t)S) {
                    d = 4 * tid + q;
                    cnt = hb[q];
                    break;
                }
                cum += hb[q];
            }
            s_sel[0] = (uint32_t)d;
            s_sel[1] = cum;
            s_sel[2] = cnt;
        }
        __syncthreads();
    };
    // A lower bound first: every thread holds a key and S <= 256, so S of the
    // threads' largest keys reach the bin of the S-th largest of those, so the
    // row's S-th largest key does too, and the keys below that bin (nine in ten
    // of a long row) need no atomic
    uint32_t d0 = 0;
    if (bound) {
        uint32_t mx = 0;
        keys.template for_each<false>([&](uint32_t k) { mx = k > mx ? k : mx; });
        atomicAdd(&hist_max[mx >> sh1], 1u);
        __syncthreads();
        find_bin(hist_max);
        d0 = s_sel[0];
    }
    const auto count = [&](uint32_t k) {
        if ((k >> sh1) >= d0) atomicAdd(&hist[k >> sh1], 1u);
    };
    if (d0 > 0) keys.template for_each<false>(count);   // uniform
    else keys.template for_each<true>(count);
    __syncthreads();
    find_bin(hist);
    const uint32_t d1 = s_sel[0], cnt1 = s_sel[2];
    int rem = S - (int)s_sel[1];   // keys still to choose in the boundary bin
    uint32_t prefix = d1 << sh1, mask = ~0u << sh1;
    bool all_eq = cnt1 == (uint32_t)rem;   // every key equal to prefix under mask is taken (uniform)
    if (cnt1 != (uint32_t)rem) {   // uniform: not every key of the boundary bin is taken
        if (cnt1 <= (uint32_t)kSelCand) {
            // the boundary bin's keys, ranked against each other: the rem-th
            // largest is the S-th largest of the row, and the keys equal to it
            // that are taken are the first ones in position order
            keys.template for_each<true>([&](uint32_t k) {
                if ((k >> sh1) == d1) s_cand[atomicAdd(&s_cnt, 1)] = k;
            });
            __syncthreads();
            if (tid < (int)cnt1) {
                const uint32_t ki = s_cand[tid];
                int gt = 0, eq = 0;
                for (int j = 0; j < (int)cnt1; ++j) {
                    const uint32_t kj = s_cand[j];
                    gt += kj > ki;
                    eq += kj == ki;
                }
                if (gt < rem && rem <= gt + eq) {   // every such thread writes the same pair
                    s_sel[0] = ki;
                    s_sel[1] = (uint32_t)(rem - gt);
                    s_sel[2] = gt + eq == rem;
                }
            }
            __syncthreads();
            prefix = s_sel[0];
            mask = ~0u;
            rem = (int)s_sel[1];
            all_eq = s_sel[2];
        } else {
            // many keys share the digit: 8-bit radix passes over the bits
            // below it (a last digit that overlaps resolved bits is harmless:
            // the prefix filter fixes them)
            for (int sh = sh1; sh > 0;) {
                sh = sh > 8 ? sh - 8 : 0;
                const int shift = sh;
                hist[tid] = 0;
                __syncthreads();
                keys.template for_each<true>([&](uint32_t k) {
                    if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
                });
                __syncthreads();
                if (tid < 64) {
                    // lane l holds bins 4l .. 4l+3; suffix sums over lanes find the
                    // bin holding the rem-th largest remaining key
                    const uint32_t h0 = hist[4 * tid], h1 = hist[4 * tid + 1], h2 = hist[4 * tid + 2],
                                   h3 = hist[4 * tid + 3];
                    const uint32_t c = h0 + h1 + h2 + h3;
                    uint32_t suf = c;
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const uint32_t t = __shfl_down(suf, off, 64);
                        if (tid + off < 64) suf += t;
                    }
                    const unsigned long long bal = __ballot(suf >= (uint32_t)rem);   // lanes 0 .. L
                    const int L = 63 - __clzll(bal);
                    if (tid == L) {
                        uint32_t cum = suf - c;   // keys in bins above 4L+3
                        int d = 4 * L;
                        uint32_t cnt = h0;
                        const uint32_t hb[4] = {h0, h1, h2, h3};
#pragma unroll
                        for (int q = 3; q >= 0; --q) {
                            if (cum + hb[q] >= (uint32_t)rem) {
                                d = 4 * L + q;
                                cnt = hb[q];
                                break;
                            }
                            cum += hb[q];
                        }
                        s_sel[0] = (uint32_t)d;
                        s_sel[1] = cum;
                        s_sel[2] = cnt;
                    }
                }
                __syncthreads();
                const uint32_t d = s_sel[0], cnt = s_sel[2];
                rem -= (int)s_sel[1];
                prefix |= d << shift;
                mask |= 255u << shift;
                __syncthreads();
                // every key of the boundary bin is taken: the digits below decide nothing
                all_eq = cnt == (uint32_t)rem;
                if (all_eq) break;
            }
        }
    }
    // prefix is the S-th largest key on the resolved digits (k & mask): take
    // every key larger under the mask and the first rem equal ones in
    // position order (all of them after an early stop).  Rows are cut into
    // chunks of 64 Q positions, Q consecutive ones per lane of one wave: per-chunk
    // counts of larger and equal keys, one scan over the chunks, then each chunk
    // writes its picks at its offset, lane by lane.
    const int lane = tid & 63, nch = (n + 64 * Q - 1) / (64 * Q);
    // set bits of b in the lanes below this one, plus add
    const auto below = [](unsigned long long b, int add) {
        return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, add));
    };
    if (all_eq && prefix > 0) {   // uniform; nearly every row: no ranks among the equal keys
        // (keys of positions >= n are 0 and fall out by themselves)
        keys.chunks([&](int c, const auto& k, int, int) {
            int take = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) take += __popcll(__ballot((k[q] & mask) >= prefix));
            if (lane == 0 && c < nch) s_gt[c] = take;
        });
        __syncthreads();
        if (tid < 64) {   // exclusive scan: lane l owns chunks [l*cpl, l*cpl + cpl)
            const int cpl = (nch + 63) >> 6, c0 = tid * cpl, c1 = min(c0 + cpl, nch);
            int own = 0;
            for (int c = c0; c < c1; ++c) own += s_gt[c];
            int pre = own;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int t = __shfl_up(pre, off, 64);
                if (tid >= off) pre += t;
            }
            pre -= own;
            for (int c = c0; c < c1; ++c) {
                const int t = s_gt[c];
                s_gt[c] = pre;
                pre += t;
            }
        }
        __syncthreads();
        keys.chunks([&](int c, const auto& k, int v, int) {
            if (c >= nch) return;   // uniform over the wave
            int pos = s_gt[c];
            bool take[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                take[q] = (k[q] & mask) >= prefix;
                pos = below(__ballot(take[q]), pos);
            }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (take[q]) {
                    if (pos < S) out[pos] = v + q;
                    ++pos;
                }
        });
        return;
    }
    keys.chunks([&](int c, const auto& k, int v, int n) {
        int gt = 0, eq = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t kq = k[q] & mask;
            gt += __popcll(__ballot(v + q < n && kq > prefix));
            eq += __popcll(__ballot(v + q < n && kq == prefix));
        }
        if (lane == 0 && c < nch) {
            s_gt[c] = gt;
            s_eq[c] = eq;
        }
    });
    __syncthreads();
    if (tid < 64) {
        // exclusive scans over chunks: lane l owns chunks [l*cpl, l*cpl + cpl)
        const int cpl = (nch + 63) >> 6, c0 = tid * cpl, c1 = min(c0 + cpl, nch);
        int eq_l = 0;
        for (int c = c0; c < c1; ++c) eq_l += s_eq[c];
        int eq_pre = eq_l;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(eq_pre, off, 64);
            if (tid >= off) eq_pre += t;
        }
        eq_pre -= eq_l;   // equal keys before this lane's chunks
        int take_l = 0;
        for (int c = c0; c < c1; ++c) {
            const int e = s_eq[c];
            const int left = rem - eq_pre;   // equal keys still to take when chunk c starts
            const int tk = s_gt[c] + (left <= 0 ? 0 : (left < e ? left : e));
            s_eq[c] = eq_pre;                // now: equal keys before chunk c
            s_gt[c] = tk;                    // now: picks in chunk c
            eq_pre += e;
            take_l += tk;
        }
        int tk_pre = take_l;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(tk_pre, off, 64);
            if (tid >= off) tk_pre += t;
        }
        tk_pre -= take_l;
        for (int c = c0; c < c1; ++c) {
            const int tk = s_gt[c];
            s_gt[c] = tk_pre;                // now: picks before chunk c
            tk_pre += tk;
        }
    }
    __syncthreads();
    keys.chunks([&](int c, const auto& k, int v, int n) {
        if (c >= nch) return;   // uniform over the wave
        int eq_rank = s_eq[c], pos = s_gt[c];   // before this lane's keys
        bool gt[Q], eq[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t kq = k[q] & mask;
            gt[q] = v + q < n && kq > prefix;
            eq[q] = v + q < n && kq == prefix;
            eq_rank = below(__ballot(eq[q]), eq_rank);
        }
        bool take[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            take[q] = gt[q] || (eq[q] && eq_rank < rem);
            eq_rank += eq[q];
            pos = below(__ballot(take[q]), pos);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (take[q]) {
                if (pos < S) out[pos] = v + q;
                ++pos;
            }
    });
}

__device__ __forceinline__ size_t kv_row(const ReplayProblem& p, int b, int t, int kvh) {
    return p.kv_layout == MOT_LAYOUT_BTHD ? (((size_t)b * p.T + t) * p.H_kv + kvh) * p.D
                                          : (((size_t)b * p.H_kv + kvh) * p.T + t) * p.D;
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  A grid of 8 * ceil(n / 8) workgroups is remapped so that XCD k walks
// the contiguous range [k * per, (k + 1) * per) of the n work items: items
// that share K/V rows (neighbouring positions, the heads of one KV group)
// meet in one L2.  Items >= n return at once.
__device__ __forceinline__ int xcd_item(int id, int n) { return (id & 7) * ((n + 7) >> 3) + (id >> 3); }
inline int xcd_grid(int n) { return 8 * ((n + 7) / 8); }

__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// LDS swizzle of a row of D bf16 (K rows: chunk c at c ^ causal_kswz(row))
template <int D>
__device__ __forceinline__ int causal_kswz(int r) {   // K rows: D/8 chunks
    return D == 128 ? (r & 15) : ((r >> 1) & 7);
}

// four bf16 of 16-byte chunk `at` (half 0 or 1) per lane, transposed within 16
// lanes: lane i's 8 bytes are row i / 4, columns 4 (i % 4) .. +3 of a 4 x 16
// block, and it gets column i of the four rows
__device__ __forceinline__ u32x2 read_tr16(const u32x4* at, int half) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const u32x2* q = reinterpret_cast<const u32x2*>(at) + half;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)q));
}

// 8 bf16 of chunk a (keys k0) and c (key k0+1) interleaved into 8 words:
// word i = (a[i], c[i]) for d = 8*chunk + i
__device__ __forceinline__ uint32_t pair_word(const u32x4& a, const u32x4& c, int i) {
    const uint32_t wa = a[i >> 1], wc = c[i >> 1];
    return (i & 1) ? ((wa >> 16) | (wc & 0xFFFF0000u)) : ((wa & 0xFFFFu) | (wc << 16));
}

// grid (xcd_grid(T), B), 256 threads; dynamic LDS: V^T [D][S] + P [16][S] (bf16) + 128 floats
template <int D, int SMAX>
__global__ __launch_bounds__(256) void k_sparse_attn(ReplayProblem p) {
    extern __shared__ u32x4 s_dyn[];
    constexpr int DC = D / 8;               // 16-byte chunks per row of D
    const int S = p.S, SC = S / 8;          // 16-byte chunks per row of S keys
    // XOR swizzle within aligned groups of the largest power of two (<= 16)
    // dividing SC, so that a permuted chunk stays inside its row
    const int swm = replay_swizzle_mask(SC);
    u32x4* Vt = s_dyn;                      // row d: SC chunks, chunk c at (c ^ (d & swm))
    u32x4* Pl = s_dyn + D * SC;             // row = query head slot
    float* red = reinterpret_cast<float*>(Pl + 16 * SC);   // [4 waves][16]: max, then sum
    const int u = xcd_item(blockIdx.x, p.T), b = blockIdx.y;
    if (u >= p.T) return;   // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, q4 = lane >> 4;
    const int G = p.H_q / p.H_kv, KB = S / 16;
    const int32_t* keys = p.idx + ((size_t)b * p.T + u) * S;
    const uint16_t* Q = reinterpret_cast<const uint16_t*>(p.q);
    const uint16_t* K = reinterpret_cast<const uint16_t*>(p.k);
    const uint16_t* V = reinterpret_cast<const uint16_t*>(p.v);
    uint16_t* O = reinterpret_cast<uint16_t*>(p.o);
    const float sl2 = kLog2e / sqrtf((float)D);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    // a key entry outside 0..u (the -1 padding) is not attended
    auto key_ok = [&](int kv) { return kv >= 0 && kv <= u; };
    // the set is the same for every KV head: read it once
    __shared__ int s_keys[256];
    for (int i = tid; i < S; i += 256) s_keys[i] = keys[i];
    __syncthreads();
    // per-thread item counts for sets of up to SMAX keys
    constexpr int MAXR = replay_sparse_v_items(D, SMAX);   // V key-pair items
    constexpr int MAXB = replay_sparse_key_blocks(SMAX);   // key blocks per wave
    static_assert(replay_sparse_supported(D, SMAX), "instantiated set size");

    for (int kvh = 0; kvh < p.H_kv; ++kvh) {
        // every gather of this KV head is issued before the first is used:
        // (a) V rows, item = (key pair, d chunk); (b) K rows of this wave's
        // key blocks kb = w, w+4, ...; then the query heads of the group
        u32x4 va[MAXR], vc[MAXR];
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            const int it = tid + 256 * r;
            va[r] = zero;
            vc[r] = zero;
            if (it < (S / 2) * DC) {
                const int pr = it % (S / 2), dc = it / (S / 2), k0 = 2 * pr;
                const int v0 = s_keys[k0], v1 = s_keys[k0 + 1];
                if (key_ok(v0)) va[r] = *reinterpret_cast<const u32x4*>(V + kv_row(p, b, v0, kvh) + 8 * dc);
                if (key_ok(v1)) vc[r] = *reinterpret_cast<const u32x4*>(V + kv_row(p, b, v1, kvh) + 8 * dc);
            }
        }
        u32x4 ka[MAXB][D / 32];
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const int kb = w + 4 * i;
            const int kr = kb < KB ? s_keys[kb * 16 + l16] : -1;
            const uint16_t* krow = K + (key_ok(kr) ? kv_row(p, b, kr, kvh) : 0);
#pragma unroll
            for (int ks = 0; ks < D / 32; ++ks)
                ka[i][ks] = key_ok(kr) ? *reinterpret_cast<const u32x4*>(krow + 32 * ks + 8 * q4) : zero;
        }
        const int hq = kvh * G + l16;
        u32x4 qop[D / 32];
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks)
            qop[ks] = l16 < G ? *reinterpret_cast<const u32x4*>(Q + (((size_t)b * p.T + u) * p.H_q + hq) * D + 32 * ks + 8 * q4)
                              : zero;
        // V_sel^T into LDS
        uint32_t* Vw = reinterpret_cast<uint32_t*>(Vt);
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            const int it = tid + 256 * r;
            if (it < (S / 2) * DC) {
                const int pr = it % (S / 2), dc = it / (S / 2), k0 = 2 * pr;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int d = 8 * dc + i;
                    Vw[(d * SC + ((k0 >> 3) ^ (d & swm))) * 4 + ((k0 & 7) >> 1)] = pair_word(va[r], vc[r], i);
                }
            }
        }
        // scores^T[key][head]
        f32x4 sc[MAXB];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const int kb = w + 4 * i;
            sc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (kb < KB) {
#pragma unroll
                for (int ks = 0; ks < D / 32; ++ks) sc[i] = mfma_16x16x32(ka[i][ks], qop[ks], sc[i]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    sc[i][j] = key_ok(s_keys[kb * 16 + 4 * q4 + j]) ? sc[i][j] : -INFINITY;
                    mx = fmaxf(mx, sc[i][j]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) sc[i][j] = -INFINITY;
            }
        }
        // (c) softmax over the set, per head (lane column l16)
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (q4 == 0) red[w * 16 + l16] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(red[l16], red[16 + l16]), fmaxf(red[32 + l16], red[48 + l16]));
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < MAXB; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float e = sc[i][j] == -INFINITY ? 0.f : exp2f((sc[i][j] - mx) * sl2);
                sc[i][j] = e;
                sum += e;
            }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        __syncthreads();   // every wave has read the maxima
        if (q4 == 0) red[w * 16 + l16] = sum;
        __syncthreads();
        sum = red[l16] + red[16 + l16] + red[32 + l16] + red[48 + l16];
        const float inv = sum > 0.f ? 1.0f / sum : 0.f;
        uint32_t* Pw = reinterpret_cast<uint32_t*>(Pl);
#pragma unroll
        for (int i = 0; i < MAXB; ++i) {
            const int kb = w + 4 * i;
            if (kb < KB) {
                const int ch = (2 * kb + (q4 >> 1)) ^ (l16 & swm);
                const int base = (l16 * SC + ch) * 4 + 2 * (q4 & 1);
                Pw[base] = pack_bf16x2(sc[i][0] * inv, sc[i][1] * inv);
                Pw[base + 1] = pack_bf16x2(sc[i][2] * inv, sc[i][3] * inv);
            }
        }
        __syncthreads();
        // (d) O^T[d][head] = V_sel^T . P^T, d blocks db = w, w+4, ...
#pragma unroll
        for (int i = 0; i < D / 64; ++i) {
            const int db = w + 4 * i;
            const int dr = 16 * db + l16;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            for (int ks = 0; ks < S / 32; ++ks) {
                const u32x4 a = Vt[dr * SC + ((4 * ks + q4) ^ (dr & swm))];
                const u32x4 bb = Pl[l16 * SC + ((4 * ks + q4) ^ (l16 & swm))];
                acc = mfma_16x16x32(a, bb, acc);
            }
            if (l16 < G) {
                const u32x2 o2 = {pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
                *reinterpret_cast<u32x2*>(O + (((size_t)b * p.T + u) * p.H_q + hq) * D + 16 * db + 4 * q4) = o2;
            }
        }
        __syncthreads();   // V^T and P are rewritten for the next KV head
    }
}

// Four neighbouring positions per group (grouped-query heads G <= 8): u0 .. u0+3
// attend over the union of their key sets, each key gathered once, with a mask
// of the positions that list it.  Neighbouring positions attend to nearly the
// same keys (sets of 128 over a map of locality, sinks and heavy hitters: four
// positions' union is ~155 keys), and the 4G query heads are the columns of
// 32x32 products.
//
// A wave runs one (group, KV head) by itself, with no barrier: WPG waves share
// a group's key list (KV heads w, w + WPG, ...), 4 / WPG groups per workgroup.
// It walks the list in blocks of 32 keys with an online softmax, as the causal
// kernel does: K and V rows come straight into LDS (buffer loads, a whole row by
// 16 or 8 lanes; entries past the list read as zeros), the next block's K while
// this block's softmax and P . V run, its V while the next scores do.
// scores^T[key][column] takes K rows as A operands; in O^T[d][column] += V^T .
// P^T a lane's accumulators hold keys 8i + 4g + {0..3}, which is the order in
// which two transposing LDS reads (four keys of one d each) give the V^T
// operand, so neither P nor V is rearranged.
//
// The list: with ascending sets (-1 padding last, what the Top-S selection
// writes) the entries of set p that no earlier set holds, in set order, with the
// mask of all sets that hold them (binary searches).  If a set of the group is
// not ascending (unordered, duplicates), every entry as listed, for its own
// position.  Entries outside 0 .. u of their position are left out.
//
// Bound: latency (waves wait half their time; 2 per SIMD is what the tiles and
// accumulators leave room for).  28 query heads on 4 KV heads of 128, 8192
// positions, sets of 128: 252 us with two positions per workgroup and V transposed
// by 4-byte LDS stores, 97 us now (0.67 GB gathered instead of 1.2).
//
// grid xcd_grid(ceil(B * ceil(T / 4) / (4 / WPG))), 256 threads
constexpr int kPos = 4;   // positions per group

template <int D, int WPG>
__global__ __launch_bounds__(256, 2) void k_sparse_attn_group(ReplayProblem p) {
    constexpr int GPW = 4 / WPG, SMAX = replay_sparse_smax(D), ENT = kPos * SMAX;   // entries per group
    constexpr int CH = SMAX / 64, NCH = kPos * CH;   // rounds of 64 entries of a set, of a group
    constexpr int DC = D / 8, TILE = 32 * DC;    // 16-byte chunks of a row, of 32 rows
    constexpr int RPL = 64 / DC, NL = 32 / RPL;  // rows per wave load, loads per tile
    // per wave a K tile and a V tile (the sets, before the walk), then the lists:
    // row offsets, masks (a byte each), counts per 64 entries; a flag per wave.  One LDS
    // object: with a second one (__syncthreads_or brings its own) the compiler
    // waits for every load into LDS before each LDS read of the walk
    __shared__ u32x4 s_lds[4 * 2 * TILE + GPW * (ENT / 4 + ENT / 16 + ENT / 256) + 1];
    static_assert(GPW * ENT * 4 <= 4 * 2 * TILE * 16, "the sets fit the tiles' space");
    int* s_set = reinterpret_cast<int*>(s_lds);
    uint32_t* s_row = reinterpret_cast<uint32_t*>(s_lds + 4 * 2 * TILE);
    uint8_t* s_mask = reinterpret_cast<uint8_t*>(s_row + GPW * ENT);
    int* s_cnt = reinterpret_cast<int*>(s_mask + GPW * ENT);   // [GPW][NCH]
    int* s_bad = s_cnt + GPW * NCH;                            // [4]
    const int ngrp = (p.T + kPos - 1) / kPos, nitem = (p.B * ngrp + GPW - 1) / GPW;
    const int item = xcd_item(blockIdx.x, nitem);
    if (item >= nitem) return;   // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int S = p.S, G = p.H_q / p.H_kv;

    // this wave's group, this lane's column (position pp, head hh of the KV
    // head's), and its query rows of the first KV head, loaded ahead of the list
    const int gi = w / WPG, q = item * GPW + gi, b = q / ngrp, u0 = q % ngrp * kPos;
    const int pp = l32 / G, hh = l32 - pp * G;
    const bool col_ok = pp < kPos && q < p.B * ngrp && u0 + pp < p.T;
    u32x4 qop[D / 16];
    auto load_q = [&](int kvh) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
        const uint16_t* row = reinterpret_cast<const uint16_t*>(p.q) +
                              (((size_t)b * p.T + u0 + pp) * p.H_q + kvh * G + hh) * D + 8 * g;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            qop[ks] = col_ok && kvh < p.H_kv ? *reinterpret_cast<const u32x4*>(row + 16 * ks) : zero;
    };
    load_q(w % WPG);

    // ---- the lists: wave w takes the sets of position w of every group, entry
    // lane + 64 r in round r
    const uint32_t ts = p.kv_layout == MOT_LAYOUT_BTHD ? (uint32_t)(p.H_kv * D) : (uint32_t)D;
    int key[GPW][CH], rank[GPW][CH];
    uint32_t mask[GPW][CH];
#pragma unroll
    for (int j = 0; j < GPW; ++j) {
        const int qj = item * GPW + j, bj = qj / ngrp, u = qj % ngrp * kPos + w;
        const int32_t* set = p.idx + ((size_t)bj * p.T + u) * S;
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const int e = lane + 64 * r;
            key[j][r] = e < S && qj < p.B * ngrp && u < p.T ? set[e] : -1;
        }
    }
#pragma unroll
    for (int j = 0; j < GPW; ++j)
#pragma unroll
        for (int r = 0; r < CH; ++r)
            if (lane + 64 * r < S) s_set[(j * kPos + w) * S + lane + 64 * r] = key[j][r];
    __syncthreads();
    bool bad = false;   // a set that is not ascending
#pragma unroll
    for (int j = 0; j < GPW; ++j)
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            const int e = lane + 64 * r, v = key[j][r], nx = e + 1 < S ? s_set[(j * kPos + w) * S + e + 1] : -1;
            bad |= e < S && ((v < 0 && nx >= 0) || (v >= 0 && nx >= 0 && nx <= v) || v < -1);
        }
    const bool wave_bad = __any(bad);
    if (lane == 0) s_bad[w] = wave_bad;
    __syncthreads();
    const bool ordered = !(s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3]);
    const int top = 1 << (31 - __builtin_clz(S));   // largest power of two <= S
#pragma unroll
    for (int j = 0; j < GPW; ++j) {
        const int uj = (item * GPW + j) % ngrp * kPos;
        const int* sets = s_set + j * kPos * S;
        // entries of each set below each key, by bisection, side by side (-1
        // padding compares as the largest)
        int at[CH][kPos];
#pragma unroll
        for (int r = 0; r < CH; ++r)
#pragma unroll
            for (int o = 0; o < kPos; ++o) at[r][o] = 0;
        for (int step = ordered ? top : 0; step; step >>= 1)
#pragma unroll
            for (int r = 0; r < CH; ++r)
                if (64 * r < S)
#pragma unroll
                    for (int o = 0; o < kPos; ++o) {
                        const int i = at[r][o] + step - 1;
                        const uint32_t v = (uint32_t)sets[o * S + min(i, S - 1)];
                        at[r][o] += i < S && v < (uint32_t)key[j][r] ? step : 0;
                    }
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            bool keep = key[j][r] >= 0 && key[j][r] <= uj + w;
            mask[j][r] = 1u << w;
            if (ordered && 64 * r < S) {
#pragma unroll
                for (int o = 0; o < kPos; ++o) {
                    const int v = sets[o * S + min(at[r][o], S - 1)];
                    // position o attends the key when its set holds it and it is not ahead
                    if (o != w && at[r][o] < S && v == key[j][r] && v <= uj + o) {
                        mask[j][r] |= 1u << o;
                        keep &= o > w;
                    }
                }
            }
            const unsigned long long bal = __ballot(keep);
            if (lane == 0) s_cnt[j * NCH + w * CH + r] = __popcll(bal);
            rank[j][r] = keep ? __popcll(bal & ((1ull << lane) - 1ull)) : -1;
        }
    }
    __syncthreads();
    int U = 0;   // length of this wave's list
#pragma unroll
    for (int j = 0; j < GPW; ++j) {
        int before = 0, all = 0;   // kept entries ahead of this wave's sets, and in all
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int n = s_cnt[j * NCH + c];
            before += c < w * CH ? n : 0;
            all += n;
        }
#pragma unroll
        for (int r = 0; r < CH; ++r) {
            if (rank[j][r] >= 0) {
                s_row[j * ENT + before + rank[j][r]] = (uint32_t)key[j][r] * ts * 2;
                s_mask[j * ENT + before + rank[j][r]] = (uint8_t)mask[j][r];
            }
            before += s_cnt[j * NCH + w * CH + r];
        }
        // pad to whole blocks with rows past the buffers' ends, for no position
        if (w == 0 && lane < (32 - all % 32) % 32) {
            s_row[j * ENT + all + lane] = 0x80000000u;
            s_mask[j * ENT + all + lane] = 0;
        }
        if (j == gi) U = all;
    }
    const int nblk = (U + 31) / 32;
    __syncthreads();
    if (q >= p.B * ngrp) return;   // uniform over the wave; no barrier follows

    const uint32_t* rowoff = s_row + gi * ENT;
    const uint8_t* bytemask = s_mask + gi * ENT;
    const uint32_t* masks = reinterpret_cast<const uint32_t*>(s_mask + gi * ENT);
    u32x4* Kt = s_lds + w * 2 * TILE;   // row r: chunk c at c ^ causal_kswz(r)
    u32x4* Vt = Kt + TILE;              // row r: chunk c at c ^ vswz(r), which keeps chunk pairs together
    auto vswz = [](int r) { return D == 128 ? 2 * (r & 7) : 2 * ((r >> 1) & 3); };
    const uint32_t bytes = ((uint32_t)(p.T - 1) * ts + D) * 2;   // < 2^31 (replay_causal_supported)
    const float sl2 = kLog2e / sqrtf((float)D);
    const uint32_t bit = col_ok ? 1u << pp : 0u;
    const int lrow = lane / DC, lch = lane % DC;   // this lane's row and chunk of a wave load
    uint16_t* O = reinterpret_cast<uint16_t*>(p.o);
    // operand read addresses: V^T by transposing reads, 16 lanes reading 4 keys x
    // 16 d (lane i of the 16: key i / 4, d 4 (i % 4) .. +3, and gets d = i)
    const int l16 = lane & 15, vrow = 4 * g + (l16 >> 2), vch = 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);

    for (int kvh = w % WPG; kvh < p.H_kv; kvh += WPG) {
        const rsrc_t kbuf = make_rsrc(reinterpret_cast<const uint16_t*>(p.k) + kv_row(p, b, 0, kvh), bytes);
        const rsrc_t vbuf = make_rsrc(reinterpret_cast<const uint16_t*>(p.v) + kv_row(p, b, 0, kvh), bytes);
        // positions of this pass: all four, or, when that gave a value that is not
        // finite (a V row that a neighbour attends multiplies a probability of 0),
        // one at a time over its own keys, the others' rows read as zeros
        uint32_t pm;
        uint32_t off[NL];   // row offsets of the block whose V is loaded next
        auto rows = [&](int blk) {
#pragma unroll
            for (int i = 0; i < NL; ++i) off[i] = rowoff[blk * 32 + i * RPL + lrow];
            if (pm != 15u) {   // uniform
#pragma unroll
                for (int i = 0; i < NL; ++i)
                    if (!(bytemask[blk * 32 + i * RPL + lrow] & pm)) off[i] = 0x80000000u;
            }
        };
        auto load_k = [&]() {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                load_lds16(kbuf, off[i] + 16 * (lch ^ causal_kswz<D>(i * RPL + lrow)), Kt + i * 64);
        };
        auto load_v = [&]() {
#pragma unroll
            for (int i = 0; i < NL; ++i) load_lds16(vbuf, off[i] + 16 * (lch ^ vswz(i * RPL + lrow)), Vt + i * 64);
        };
        for (int pass = 0; pass <= kPos; ++pass) {
        pm = pass == 0 ? 15u : 1u << (pass - 1);
        f32x16 acc[D / 32];
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
        // the rounded exponent offset of a maximum (as a value of its own: contracted
        // into the subtraction below it would not be rounded there)
        auto offset = [&](float mx) {
            float r = mx * sl2;
            asm("" : "+v"(r));
            return r;
        };
        // running maximum (finite: a position may have no entry in a block) and its offset
        float m = -3.402823466e38f, mo = offset(m), l = 0.f;
        // the tiles' last readers and the stores of the output rows are done (the
        // waits below count the newest loads only)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        if (nblk > 0) {
            rows(0);
            load_k();
            load_v();
        }
        for (int blk = 0; blk < nblk; ++blk) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");   // K of this block (V may be in flight)
            f32x16 sc;
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks)
                sc = mfma_32x32x16(Kt[l32 * DC + ((2 * ks + g) ^ causal_kswz<D>(l32))], qop[ks], sc);
            const bool more = blk + 1 < nblk;   // uniform
            uint32_t mk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) mk[i] = masks[blk * 8 + 2 * i + g];
            // the operand reads are complete: the next K may land
            wave_lds_sync();
            if (more) {
                rows(blk + 1);
                load_k();
            }
            float cm = -INFINITY;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                sc[e] = (mk[e >> 2] >> (8 * (e & 3))) & bit ? sc[e] : -INFINITY;
                cm = fmaxf(cm, sc[e]);
            }
            cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
            const float mn = fmaxf(m, cm);
            // between the rounded offsets: earlier blocks keep their weight against this
            // one's exactly, however large the scores ((m - mn) sl2 is off by an offset's
            // rounding: 6 % at scores of 2^23)
            const float mon = offset(mn);
            const float alpha = __builtin_amdgcn_exp2f(mo - mon);
            mo = mon;
            float rs = 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                sc[e] = __builtin_amdgcn_exp2f(fmaf(sc[e], sl2, -mo));
                rs += sc[e];
            }
            rs += __shfl_xor(rs, 32, 64);
            l = l * alpha + rs;
            if (__builtin_amdgcn_ballot_w64(mn != m)) {
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[db][e] *= alpha;
            }
            m = mn;
            if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");   // V of this block
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const u32x4 pf = {pack_bf16x2(sc[8 * s], sc[8 * s + 1]), pack_bf16x2(sc[8 * s + 2], sc[8 * s + 3]),
                                  pack_bf16x2(sc[8 * s + 4], sc[8 * s + 5]), pack_bf16x2(sc[8 * s + 6], sc[8 * s + 7])};
#pragma unroll
                for (int db = 0; db < D / 32; ++db) {
                    u32x2 va[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int r = 16 * s + 8 * t + vrow;
                        va[t] = read_tr16(Vt + r * DC + ((4 * db + vch) ^ vswz(r)), l16 & 1);
                    }
                    acc[db] = mfma_32x32x16(u32x4{va[0].x, va[0].y, va[1].x, va[1].y}, pf, acc[db]);
                }
            }
            wave_lds_sync();   // the V operands are read: the next V may land
            if (more) load_v();
        }
        if (pass == 0) {
            float t = 0.f;   // NaN when an accumulator is not finite
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) t = fmaf(acc[db][e], 0.f, t);
            if (__any(t != t)) continue;   // position by position
        }
        // O rows through the K tile: row = column, chunk c at c ^ causal_kswz
        const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = (4 * db + i) ^ causal_kswz<D>(l32);
                reinterpret_cast<u32x2*>(Kt + l32 * DC + c)[g] =
                    u32x2{pack_bf16x2(acc[db][4 * i] * inv, acc[db][4 * i + 1] * inv),
                          pack_bf16x2(acc[db][4 * i + 2] * inv, acc[db][4 * i + 3] * inv)};
            }
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int r = i * RPL + lrow, po = r / G, ho = r - po * G;
            const u32x4 v = Kt[r * DC + (lch ^ causal_kswz<D>(r))];
            if (po < kPos && u0 + po < p.T && ((pm >> po) & 1))
                *reinterpret_cast<u32x4*>(O + (((size_t)b * p.T + u0 + po) * p.H_q + kvh * G + ho) * D + 8 * lch) = v;
        }
        if (pass == 0) break;
        }
        load_q(kvh + WPG);
    }
}

// V transposed for the causal kernel: vt[b][kvh][d][t] (t < replay_tpad(T),
// zero past T).  grid (replay_tpad(T) / 64, H_kv, B), 256 threads: one
// 64-key chunk through LDS (rows padded by 8 elements against bank conflicts).
template <int D>
__global__ __launch_bounds__(256) void k_transpose_v(ReplayProblem p) {
    constexpr int DC = D / 8;
    __shared__ __align__(16) uint16_t tl[64][D + 8];
    const int t0 = blockIdx.x * 64, kvh = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const uint16_t* V = reinterpret_cast<const uint16_t*>(p.v);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int it = tid; it < 64 * DC; it += 256) {
        const int kr = it / DC, c = it % DC, t = t0 + kr;
        const u32x4 x = t < p.T ? *reinterpret_cast<const u32x4*>(V + kv_row(p, b, t, kvh) + 8 * c) : zero;
        *reinterpret_cast<u32x4*>(&tl[kr][8 * c]) = x;
    }
    __syncthreads();
    const int64_t tpad = replay_tpad(p.T);
    uint16_t* out = p.vt + ((size_t)b * p.H_kv + kvh) * D * tpad + t0;
    // chunk c of a row holds keys 16 (c / 2) + 4 (c % 2) + {0..3} and the
    // same + 8: the order in which a 32x32 score block's accumulators hold
    // them, so the causal kernel's P . V operands pair up without a shuffle
    for (int it = tid; it < D * 8; it += 256) {
        const int d = it >> 3, c = it & 7, k0 = 16 * (c >> 1) + 4 * (c & 1);
        u32x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + (j < 2 ? 2 * j : 8 + 2 * (j - 2));
            w[j] = (uint32_t)tl[k][d] | ((uint32_t)tl[k + 1][d] << 16);
        }
        *reinterpret_cast<u32x4*>(out + (size_t)d * tpad + 8 * c) = w;
    }
}

// 256 threads; 128 query positions of one head per tile, 64-key chunks up to the
// tile's last position.  Workgroups go to the 8 XCDs round-robin, and every XCD
// takes a contiguous share of the heads (the heads of a KV group meet in one L2).
//
// PAIRED: a workgroup runs a short and a long tile, so that all do the same work.
// Grid xcd_grid(pairs * H_q * B), pairs fastest.  Otherwise one tile per workgroup,
// an XCD's share of the (head, tile mod m), m = min(8, tiles), in rows of m tiles
// from the longest down; grid 8 * causal_row * ceil(tiles / m).
//
// Per wave and chunk, on v_mfma_f32_32x32x16_bf16: scores^T[key][position]
// for two 32-key blocks (A = K rows from LDS, B = the wave's 32 query rows,
// held in registers), an online softmax per position (column), and
// O^T[d][position] += V^T . P^T with A = V^T rows from LDS and B = the
// probabilities straight from the score accumulators: a lane's accumulator
// holds keys 8i + 4g + {0..3} of its position, and the staged V^T rows keep
// each 16-key group in the matching order (keys 0-3, 8-11, 4-7, 12-15), so k
// step s of the product takes accumulator elements 8 (s % 2) .. +7 of block
// s / 2 as its B operand.  LDS: K chunk [64][D], V^T chunk [D][64] (bf16).


// Pairs or single tiles.  Single tiles end evenly when there are many lengths of them,
// and let short calls use every CU; pairs waste nothing where their workgroups
// fill whole rounds of the CUs (256), or one round of the chip (3 per CU at D = 64, 2 at
// 128), and there are few tile lengths to even out with.  28 heads on 4 of 128, pairs
// against single tiles: T = 500 28 / 22 us, 1000 41 / 34, 2500 103 / 75, 4200 (476
// pairs) 168 / 170, 6000 349 / 306, 9000 642 / 619; 4 x 1000 (448 pairs of 8 tiles) 61
// / 66, 8 x 1000 (896) 107 / 118, 8 x 500 (448 of 4) 43 / 52; 12 heads of 64, 16 x 1000
// (768) 59 / 68, 8 x 2100 (864 of 17) 114 / 102.  Over 1053 calls (9 head counts, B up
// to 16, T to 9000) the choice is 0.24 % above the better form on average, 9 % at most;
// always pairs 14 % and 50 %.
inline bool causal_paired(const ReplayProblem& p) {
    const int ntiles = (p.T + 127) / 128;
    const int64_t nh = (int64_t)p.H_q * p.B, pairs = (ntiles + 1) / 2 * nh, round = p.D == 64 ? 768 : 512;
    if (ntiles == 1 || (ntiles >= 8 && pairs >= 4 * round) || (10 * pairs > 9 * round && pairs <= round)) return true;
    if (ntiles == 8) return nh > 32;   // single tiles: one per CU at most
    const bool full = 100 * pairs >= 78 * 256 * ((pairs + 255) / 256);
    return ntiles <= 12 && full && (ntiles > 8 || (ntiles >= 4 && ntiles % 2 == 0 && pairs > 256));
}

// an XCD's workgroups per row of single tiles
__host__ __device__ inline int causal_row(int ntiles, int nh) {
    return ntiles < 8 ? (nh * ntiles + 7) >> 3 : nh;
}

template <int D, bool PAIRED>
__global__ __launch_bounds__(256, 2) void k_causal_attn(ReplayProblem p) {
    constexpr int DC = D / 8;
    constexpr int KS = 64 * DC, VS = D * 8;   // 16-byte slots of a K chunk and a V^T chunk
    // two stages, each: K chunk rows (key: chunk c at c ^ causal_kswz(key)),
    // then V^T rows (d: chunk c at c ^ ((d >> 1) & 7)); filled straight from
    // global memory (buffer loads into LDS) one chunk ahead
    __shared__ u32x4 lds[2 * (KS + VS)];
    const int ntiles = (p.T + 127) / 128, nh = p.H_q * p.B;
    int head, tile0;
    if constexpr (PAIRED) {
        const int npairs = (ntiles + 1) / 2, item = xcd_item(blockIdx.x, npairs * nh);
        if (item >= npairs * nh) return;   // uniform over the workgroup
        head = item / npairs;
        tile0 = item % npairs;
    } else {
        const int per = causal_row(ntiles, nh), m = ntiles < 8 ? ntiles : 8;
        const int slot = blockIdx.x >> 3, c = (blockIdx.x & 7) * per + slot % per;
        head = c / m;
        tile0 = ntiles - 1 - (m * (slot / per) + c % m);
        if (tile0 < 0 || head >= nh) return;   // uniform over the workgroup
    }
    const int hq = head % p.H_q, b = head / p.H_q;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, g = lane >> 5;
    const int G = p.H_q / p.H_kv, kvh = hq / G;
    const uint16_t* Q = reinterpret_cast<const uint16_t*>(p.q);
    uint16_t* O = reinterpret_cast<uint16_t*>(p.o);
    const float sl2 = kLog2e / sqrtf((float)D);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const int64_t tpad = replay_tpad(p.T);
    // key t of this batch row and KV head sits at row t * ts of the K buffer;
    // the host admits only shapes whose byte offsets (up to (T + 64) * ts * 2)
    // fit in 31 bits; rows past T lie past the descriptor's range and read as zero
    const uint32_t ts = p.kv_layout == MOT_LAYOUT_BTHD ? (uint32_t)(p.H_kv * D) : (uint32_t)D;
    const rsrc_t kbuf = make_rsrc(reinterpret_cast<const uint16_t*>(p.k) + kv_row(p, b, 0, kvh),
                                  ((size_t)(p.T - 1) * ts + D) * 2);
    const rsrc_t vbuf = make_rsrc(p.vt + ((size_t)b * p.H_kv + kvh) * D * tpad, (size_t)D * tpad * 2);
    // this lane's part of the chunk loads: wave load q fills slots
    // (w * NQ + q) * 64 + lane of the K rows (NQ = KS / 256 loads), then of
    // the V^T rows
    constexpr int NQK = KS / 256, NQV = VS / 256;
    uint32_t koff[NQK], voff[NQV];
#pragma unroll
    for (int q = 0; q < NQK; ++q) {
        const int slot = (w * NQK + q) * 64 + lane, kr = slot / DC, c = (slot % DC) ^ causal_kswz<D>(kr);
        koff[q] = ((uint32_t)kr * ts + 8 * c) * 2;
    }
#pragma unroll
    for (int q = 0; q < NQV; ++q) {
        const int slot = (w * NQV + q) * 64 + lane, d = slot >> 3, c = (slot & 7) ^ ((d >> 1) & 7);
        voff[q] = ((uint32_t)d * tpad + 8 * c) * 2;
    }
    auto issue = [&](int kc0, int st) {
        u32x4* kb = lds + st * (KS + VS) + w * NQK * 64;
        u32x4* vb = lds + st * (KS + VS) + KS + w * NQV * 64;
#pragma unroll
        for (int q = 0; q < NQK; ++q) load_lds16(kbuf, koff[q] + (uint32_t)kc0 * ts * 2, kb + q * 64);
#pragma unroll
        for (int q = 0; q < NQV; ++q) load_lds16(vbuf, voff[q] + (uint32_t)kc0 * 2, vb + q * 64);
    };
    auto barrier = [&]() {
        __builtin_amdgcn_s_waitcnt(0x70);   // vmcnt(0) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    for (int pass = 0; pass < (PAIRED ? 2 : 1); ++pass) {
    const int tile = pass == 0 ? tile0 : ntiles - 1 - tile0;
    if (pass == 1 && tile <= tile0) break;   // uniform over the workgroup
    const int u0 = tile * 128;
    const int uw = u0 + 32 * w;            // first position of this wave
    const int u = uw + l32;                // this lane's query column
    u32x4 qop[D / 16];                     // k step s: d = 16 s + 8 g .. +7
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
        qop[ks] = u < p.T ? *reinterpret_cast<const u32x4*>(Q + (((size_t)b * p.T + u) * p.H_q + hq) * D + 16 * ks + 8 * g)
                          : zero;
    f32x16 acc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;
    float m = -INFINITY, l = 0.f;
    const int last = (u0 + 127 < p.T ? u0 + 127 : p.T - 1);
    barrier();   // the previous tile's last chunk is consumed
    issue(0, 0);
    barrier();
    for (int kc0 = 0; kc0 <= last; kc0 += 64) {
        const int st = (kc0 >> 6) & 1;
        if (kc0 + 64 <= last) issue(kc0 + 64, st ^ 1);
        const u32x4* Kl = lds + st * (KS + VS);
        const u32x4* Vt = Kl + KS;
        // keys after every position of this wave add nothing (uniform)
        if (kc0 <= uw + 31 && uw < p.T) {
        // scores^T[key][position], two blocks of 32 keys; only chunks that
        // reach past the wave's first position need the mask
        const bool diag = kc0 + 63 > uw;
        f32x16 sc[2];
        float cm = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[kb][e] = 0.f;
            const int kr = kb * 32 + l32;
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks)
                sc[kb] = mfma_32x32x16(Kl[kr * DC + ((2 * ks + g) ^ causal_kswz<D>(kr))], qop[ks], sc[kb]);
            if (diag) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = kc0 + kb * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
                    sc[kb][e] = key <= u ? sc[kb][e] : -INFINITY;
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) cm = fmaxf(cm, sc[kb][e]);
        }
        cm = fmaxf(cm, __shfl_xor(cm, 32, 64));
        const float mn = fmaxf(m, cm);   // finite: chunk 0 holds key 0 <= u
        // v_exp_f32 directly: results below 2^-126 flush to 0, far below the
        // bf16 resolution of P; exp2(-inf) = 0 for masked keys and the first chunk
        const float alpha = __builtin_amdgcn_exp2f((m - mn) * sl2);
        const float mo = mn * sl2;       // e = 2^(s sl2 - mn sl2)
        float rs = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float ex = __builtin_amdgcn_exp2f(fmaf(sc[kb][e], sl2, -mo));
                sc[kb][e] = ex;
                rs += ex;
            }
        rs += __shfl_xor(rs, 32, 64);
        l = l * alpha + rs;
        // alpha is exactly 1 where the running maximum did not move: the
        // accumulators are rescaled only when some position's maximum rose
        if (__builtin_amdgcn_ballot_w64(mn != m)) {
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[db][e] *= alpha;
        }
        m = mn;
        // O^T[d][position] += V^T . P^T, four k steps of 16 keys
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int kb = ks >> 1, e0 = 8 * (ks & 1);
            const u32x4 pf = {pack_bf16x2(sc[kb][e0], sc[kb][e0 + 1]), pack_bf16x2(sc[kb][e0 + 2], sc[kb][e0 + 3]),
                              pack_bf16x2(sc[kb][e0 + 4], sc[kb][e0 + 5]), pack_bf16x2(sc[kb][e0 + 6], sc[kb][e0 + 7])};
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
                const int dr = 32 * db + l32;
                acc[db] = mfma_32x32x16(Vt[dr * 8 + ((2 * ks + g) ^ ((dr >> 1) & 7))], pf, acc[db]);
            }
        }
        }
        barrier();   // stage st^1 has landed; every wave is done with stage st
    }
    // lane holds d = 32 db + 8 i + 4 g + {0..3} of position u
    if (u < p.T) {
        const float inv = 1.0f / l;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x2 o2 = {pack_bf16x2(acc[db][4 * i] * inv, acc[db][4 * i + 1] * inv),
                                  pack_bf16x2(acc[db][4 * i + 2] * inv, acc[db][4 * i + 3] * inv)};
                *reinterpret_cast<u32x2*>(O + (((size_t)b * p.T + u) * p.H_q + hq) * D + 32 * db + 8 * i + 4 * g) = o2;
            }
    }
    }
}

}  // namespace

hipError_t launch_topS_select(const float* A, int32_t* idx, int B, int T, int S, hipStream_t stream) {
    if (B == 0 || T == 0) return hipSuccess;
    const dim3 grid(T, B);
    const auto lds = [&](int q) { return (size_t)2 * (T / (64 * q) + 4) * sizeof(int); };
    // the row in registers up to 16 pieces per thread
    if (T <= 256) hipLaunchKernelGGL((k_topS_select<RegKeys<1, 1>>), grid, dim3(256), lds(1), stream, A, idx, T, S);
    else if (T <= 1024) hipLaunchKernelGGL(k_topS_select<RegKeys<1>>, grid, dim3(256), lds(4), stream, A, idx, T, S);
    else if (T <= 2048) hipLaunchKernelGGL(k_topS_select<RegKeys<2>>, grid, dim3(256), lds(4), stream, A, idx, T, S);
    else if (T <= 4096) hipLaunchKernelGGL(k_topS_select<RegKeys<4>>, grid, dim3(256), lds(4), stream, A, idx, T, S);
    else if (T <= 8192) hipLaunchKernelGGL(k_topS_select<RegKeys<8>>, grid, dim3(256), lds(4), stream, A, idx, T, S);
    else if (T <= 16384) hipLaunchKernelGGL(k_topS_select<RegKeys<16>>, grid, dim3(256), lds(4), stream, A, idx, T, S);
    else hipLaunchKernelGGL(k_topS_select<RowKeys>, grid, dim3(256), lds(1), stream, A, idx, T, S);
    return hipGetLastError();
}

namespace {

// Two groups per workgroup when a group has work for two waves at most and there
// are groups enough; else one, whose four waves build its list side by side (12
// query heads on 2 of 128, one and two groups per workgroup: 129 positions 20 /
// 27 us, 1040 29 / 34, 2080 47 / 41, 4000 63 / 55; with the selection)
template <int D>
hipError_t launch_sparse_group(const ReplayProblem& p, hipStream_t stream) {
    const int64_t groups = (int64_t)p.B * ((p.T + kPos - 1) / kPos);
    const int wpg = p.H_kv <= 2 && groups > 400 ? 2 : 4, gpw = 4 / wpg;
    const dim3 grid(xcd_grid((int)((groups + gpw - 1) / gpw)));
    if (wpg == 2) hipLaunchKernelGGL((k_sparse_attn_group<D, 2>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((k_sparse_attn_group<D, 4>), grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_replay_attention(const ReplayProblem& p, hipStream_t stream) {
    if (p.B == 0 || p.T == 0) return hipSuccess;
    if (p.idx) {
        // the caller's check admits only these sizes; the register arrays of
        // the instantiation below cover every admitted S
        if (!replay_sparse_supported(p.D, p.S)) return hipErrorInvalidValue;
        // Short calls on up to four KV heads stay with a position per workgroup: a group's
        // list costs more latency than the shared gathers save, and its workgroups, a
        // quarter as many, leave CUs idle.  One position against four, sets of 128: 8 query
        // heads on 1 of 128, 700 positions 13 / 25 us; 6 on 2 of 128, 700 19 / 26, 1100
        // 28 / 29, 1600 38 / 30; 24 on 3 of 64, 700 15 / 21, 1600 31 / 26; 28 on 4 of
        // 128, 500 23 / 27, 700 35 / 29.  Sets of 32 to 256 cross at about the same
        // lengths: over 1350 calls the choice is 0.4 % above the better form on average.
        const bool narrow = p.D == 64;
        const int64_t short_to = p.H_kv == 1   ? 4608
                                 : p.H_kv == 2 ? (narrow ? 2560 : 1024)
                                 : p.H_kv == 3 ? (narrow ? 1024 : 600)
                                 : p.H_kv == 4 ? 600
                                               : 0;
        const bool small = (int64_t)p.B * p.T <= short_to;
        if (!small && replay_sparse_group_supported(p.D, p.S, p.H_q / p.H_kv) &&
            replay_causal_supported(p.T, p.H_kv, p.D, p.kv_layout == MOT_LAYOUT_BTHD))
            return p.D == 128 ? launch_sparse_group<128>(p, stream) : launch_sparse_group<64>(p, stream);
        const dim3 grid(xcd_grid(p.T), p.B);
        const size_t lds = replay_sparse_lds_bytes(p.D, p.S);
        // register arrays sized for S <= 128, or for the largest S the LDS allows
        if (p.D == 128) {
            if (replay_sparse_instance(128, p.S) == 128)
                hipLaunchKernelGGL((k_sparse_attn<128, 128>), grid, dim3(256), lds, stream, p);
            else hipLaunchKernelGGL((k_sparse_attn<128, replay_sparse_smax(128)>), grid, dim3(256), lds, stream, p);
        } else {
            if (replay_sparse_instance(64, p.S) == 128)
                hipLaunchKernelGGL((k_sparse_attn<64, 128>), grid, dim3(256), lds, stream, p);
            else hipLaunchKernelGGL((k_sparse_attn<64, replay_sparse_smax(64)>), grid, dim3(256), lds, stream, p);
        }
    } else {
        if (!p.vt || !replay_causal_supported(p.T, p.H_kv, p.D, p.kv_layout == MOT_LAYOUT_BTHD))
            return hipErrorInvalidValue;
        const dim3 tgrid((unsigned)(replay_tpad(p.T) / 64), p.H_kv, p.B);
        if (p.D == 128) hipLaunchKernelGGL(k_transpose_v<128>, tgrid, dim3(256), 0, stream, p);
        else hipLaunchKernelGGL(k_transpose_v<64>, tgrid, dim3(256), 0, stream, p);
        const int ntiles = (p.T + 127) / 128, nh = p.H_q * p.B;
        if (causal_paired(p)) {
            const dim3 grid(xcd_grid((ntiles + 1) / 2 * nh));
            if (p.D == 128) hipLaunchKernelGGL((k_causal_attn<128, true>), grid, dim3(256), 0, stream, p);
            else hipLaunchKernelGGL((k_causal_attn<64, true>), grid, dim3(256), 0, stream, p);
        } else {
            const dim3 grid(8 * causal_row(ntiles, nh) * ((ntiles + 7) / 8));
            if (p.D == 128) hipLaunchKernelGGL((k_causal_attn<128, false>), grid, dim3(256), 0, stream, p);
            else hipLaunchKernelGGL((k_causal_attn<64, false>), grid, dim3(256), 0, stream, p);
        }
    }
    return hipGetLastError();
}

}  // namespace mot
