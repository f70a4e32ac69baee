// Router + softmax: gates[unit][token][m] = softmax_m(Wr_unit z + br_unit),
// then Top-K: the top_k largest kept and renormalised, the rest zero.
// Paper Sec. 3, Definition "Mixture-of-Translators": token-level nonnegative
// gate scores; here softmax of a linear map of the source row.
//
// bf16: k_router_mfma below.  fp32 (the shapes k_f32.hip serves): eight lanes
// share one token row: lane q reads 16-byte chunks q, q+8, ...
// (coalesced 128-byte runs), accumulates E partial dot products in fp32, and
// the eight partials are combined with cross-lane shuffles.  256 threads =
// 32 tokens per pass, 8 passes per workgroup; grid.y enumerates the units.
#include "mot_device.h"
#include "mot_internal.h"
#include "../../include/mot.h"

namespace mot {

namespace {

constexpr int kLanesPerTok = 8;
constexpr int kTokPerBlock = 256 / kLanesPerTok;   // tokens per pass of a workgroup
constexpr int kGroups = 8;                          // passes per workgroup

// fp32 rows, on the vector ALUs: dense gate rows p.gates[gslot][token][E].
// WLDS: the unit's router rows (E x d_in) are staged once in LDS (dynamic
// shared memory, when they fit) instead of being re-read per token.
template <bool WLDS>
__global__ __launch_bounds__(256) void k_router(Problem p, UnitTab ut) {
    constexpr int VN = 4;   // values per 16-byte chunk
    extern __shared__ u32x4 s_wr[];
    const uint32_t code = ut.code[blockIdx.y];
    const int j = unit_j(code), x = unit_x(code), i = unit_i(code), gs = unit_gslot(code);
    const int q = threadIdx.x % kLanesPerTok;
    const void* wr = p.wr;
    size_t wr_base = ((size_t)j * p.streams + x) * p.E * p.d_in;
    if constexpr (WLDS) {
        const int n16 = p.E * p.d_in / VN;   // 16-byte chunks
        const u32x4* g = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(p.wr) +
                                                        wr_base * 4);
        for (int c = threadIdx.x; c < n16; c += 256) s_wr[c] = g[c];
        __syncthreads();
        wr = s_wr;
        wr_base = 0;
    }
    for (int grp = 0; grp < kGroups; ++grp) {
    const int tok = (blockIdx.x * kGroups + grp) * kTokPerBlock + threadIdx.x / kLanesPerTok;
    // the gate rows of the last partial pass are still written by lanes q == 0
    // of valid tokens only; the usage count needs every lane of the wave
    const bool owner = tok < p.n_tok && q == 0;
    const int E = p.E, d_in = p.d_in;
    const size_t unit = (size_t)j * p.streams + x;

    float acc[MOT_MAX_EXPERTS];
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) acc[m] = 0.f;

    if (tok < p.n_tok) {
        const size_t layer = (size_t)i * p.n_tok * d_in;
        const int b = tok / p.T, t = tok % p.T;
        // four 16-byte source chunks in flight per lane before they are used
        constexpr int kStep = kLanesPerTok * VN;
        for (int c0 = q * VN; c0 < d_in; c0 += 4 * kStep) {
            f32x4 zr[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * kStep;
                const int cc = c < d_in ? c : c0;   // in range; unused when c >= d_in
                size_t off;
                if (p.src_layout == MOT_LAYOUT_BTHD) {
                    off = layer + (size_t)tok * d_in + cc;
                } else {
                    const int hh = cc / p.D_src, dd = cc % p.D_src;
                    off = layer + (((size_t)b * p.H_src + hh) * p.T + t) * p.D_src + dd;
                }
                zr[u] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.src[x]) + off);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * kStep;
                if (c < d_in) {
#pragma unroll
                    for (int m = 0; m < MOT_MAX_EXPERTS; ++m)
                        if (m < E) {
                            const f32x4 wv = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(wr) +
                                                                             wr_base + (size_t)m * d_in + c);
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[m] = fmaf(wv[e], zr[u][e], acc[m]);
                        }
                }
            }
        }
    }
    // combine the eight partial sums of each token (lanes of a token are
    // consecutive and aligned to 8)
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) {
        if (m < E) {
            float v = acc[m];
            v += __shfl_xor(v, 1, 64);
            v += __shfl_xor(v, 2, 64);
            v += __shfl_xor(v, 4, 64);
            acc[m] = v;
        }
    }
    // every lane runs the softmax and the selection (lanes without a token
    // work on zeros and write nothing), so the wave can count selections
    float mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) {
        if (m < E) {
            if (p.br) acc[m] += reinterpret_cast<const float*>(p.br)[unit * E + m];
            mx = fmaxf(mx, acc[m]);
        }
    }
    float den = 0.f;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) {
        if (m < E) {
            acc[m] = expf(acc[m] - mx);
            den += acc[m];
        }
    }
    const float inv = 1.0f / den;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m) acc[m] = m < E ? acc[m] * inv : 0.f;
    const uint32_t taken = topk_renormalise(acc, E, p.top_k);
    if (p.usage) count_usage(p.usage + unit * E, E, taken, owner);
    if (!owner) continue;
    float* g = p.gates + ((size_t)gs * p.n_tok_pad + tok) * E;
#pragma unroll
    for (int m = 0; m < MOT_MAX_EXPERTS; ++m)
        if (m < E) g[m] = acc[m];
    }
}

// bf16 rows on the matrix cores: logits = Wr z^T on v_mfma_f32_16x16x32_bf16, a
// wave 16 tokens (B columns; Wr rows from E on are zeros), kStepsAhead k-steps of
// source loads in flight.  Every lane gets its token's E logits by shuffles;
// lanes 0..15 own the tokens.
//
// Bound: the source rows' bytes where rows are wide (2048 values, 16384 tokens, 56
// units: 3.8 GB in 637 us, 6.0 TB/s); at 256 values (4096 tokens, 56 units: 44 us,
// 2.7 TB/s) the shuffles, softmax and Top-K of a token as much (vector ALUs 45 %
// busy).  With the form above on packed bf16 dot products (E LDS reads and 4 E dot
// products per 8 values and token) a Top-1 call over 8 translators of 256-wide rows
// (4096 tokens, 56 units) took 989 us, with this one 930; a dense call on 2048-wide
// rows (2048 tokens, 4 translators) 2524 and 2470.
//
// grid: x = groups of 64 tokens, strided; y = unit; 256 threads
constexpr int kStepsAhead = 8;

template <bool LISTS, bool WLDS>
__global__ __launch_bounds__(256) void k_router_mfma(Problem p, UnitTab ut) {
    extern __shared__ u32x4 s_wr[];   // WLDS: row m, chunk c at c ^ (m & 7)
    const uint32_t code = ut.code[blockIdx.y];
    const int j = unit_j(code), x = unit_x(code), i = unit_i(code), gs = unit_gslot(code);
    const int E = p.E, d_in = p.d_in, nc = d_in / 8;   // d_in % 64 == 0
    const size_t unit = (size_t)j * p.streams + x;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const u32x4* wr = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.wr) + unit * E * d_in);
    if constexpr (WLDS) {
        for (int c = tid; c < E * nc; c += 256) {
            const int m = c / nc, cc = c - m * nc;
            s_wr[m * nc + (cc ^ (m & 7))] = wr[c];
        }
        __syncthreads();
    }
    const uint16_t* src = reinterpret_cast<const uint16_t*>(p.src[x]) + (size_t)i * p.n_tok * d_in;
    const uint16_t* br = p.br ? reinterpret_cast<const uint16_t*>(p.br) + unit * E : nullptr;
    const bool bthd = p.src_layout == MOT_LAYOUT_BTHD;
    for (int t0 = (blockIdx.x * 4 + (tid >> 6)) * 16; t0 < p.n_tok; t0 += gridDim.x * 64) {   // uniform over a wave
        const int tok = t0 + l16, tokc = min(tok, p.n_tok - 1);
        const int b = tokc / p.T, t = tokc - b * p.T;
        const uint16_t* row = bthd ? src + (size_t)tokc * d_in : src + ((size_t)b * p.H_src * p.T + t) * p.D_src;
        f32x4 lg = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < d_in / 32; s0 += kStepsAhead) {
            u32x4 z[kStepsAhead];
#pragma unroll
            for (int s = 0; s < kStepsAhead; ++s) {
                const int k = (s0 + s) * 32 + 8 * q4;
                z[s] = zero;
                if ((s0 + s) * 32 < d_in) {   // uniform
                    size_t off = k;
                    if (!bthd) {   // D_src % 8 == 0: eight values in one head
                        const int hh = k / p.D_src;
                        off = (size_t)hh * p.T * p.D_src + (k - hh * p.D_src);
                    }
                    z[s] = *reinterpret_cast<const u32x4*>(row + off);
                }
            }
#pragma unroll
            for (int s = 0; s < kStepsAhead; ++s) {
                if ((s0 + s) * 32 < d_in) {
                    const int c = (s0 + s) * 4 + q4;
                    u32x4 a = zero;
                    if (l16 < E) a = WLDS ? s_wr[l16 * nc + (c ^ (l16 & 7))] : wr[l16 * nc + c];
                    lg = mfma_16x16x32(a, z[s], lg);
                }
            }
        }
        // lane group q4 holds the logits of experts 4 q4 .. +3 for token l16
        float g[MOT_MAX_EXPERTS];
#pragma unroll
        for (int qq = 0; qq < 4; ++qq)
#pragma unroll
            for (int r = 0; r < 4; ++r) g[4 * qq + r] = __shfl(lg[r], 16 * qq + l16, 64);
        float mx = -INFINITY;
#pragma unroll
        for (int m = 0; m < MOT_MAX_EXPERTS; ++m)
            if (m < E) {
                if (br) g[m] += bf16_to_f32(br[m]);
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
        const bool owner = q4 == 0 && tok < p.n_tok;
        if constexpr (LISTS) {
            // the routed path counts usage in its plan kernel
            if (owner) {
                const size_t base = ((size_t)gs * p.n_tok + tok) * p.top_k;
                topk_list(g, E, p.top_k, p.rt.sel + base, p.rt.gk + base);
            }
        } else {
            const uint32_t taken = topk_renormalise(g, E, p.top_k);
            if (p.usage) count_usage(p.usage + unit * E, E, taken, owner);
            if (owner) {
                float* out = p.gates + ((size_t)gs * p.n_tok_pad + tok) * E;
#pragma unroll
                for (int m = 0; m < MOT_MAX_EXPERTS; ++m)
                    if (m < E) out[m] = g[m];
            }
        }
    }
}

// Translator usage statistics (paper Sec. 4, "MoT Architecture Ablation"),
// one thread per row of counts I[E]: CV^2 = population variance over the
// squared mean, entropy = -sum p ln p with p = I / sum I (0 ln 0 = 0), in
// double; NaN for a row of zeros.
__global__ __launch_bounds__(256) void k_usage_stats(const uint32_t* counts, int n, int E, double* cv2,
                                                     double* entropy) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    const uint32_t* c = counts + (size_t)r * E;
    double total = 0.0;
    for (int m = 0; m < E; ++m) total += (double)c[m];
    const double mean = total / E;
    double var = 0.0;
    for (int m = 0; m < E; ++m) var += ((double)c[m] - mean) * ((double)c[m] - mean);
    var /= E;
    cv2[r] = var / (mean * mean);
    double h = 0.0;
    for (int m = 0; m < E; ++m) {
        if (c[m] == 0) continue;
        const double q = (double)c[m] / total;
        h -= q * log(q);
    }
    entropy[r] = total > 0.0 ? h : __builtin_nan("");
}

constexpr size_t kWrLdsMax = 64 * 1024;   // router rows staged in LDS up to this size

hipError_t launch_f32(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    dim3 grid((p.n_tok + kTokPerBlock * kGroups - 1) / (kTokPerBlock * kGroups), ut.n);
    const size_t wr_bytes = (size_t)p.E * p.d_in * 4;
    if (wr_bytes <= kWrLdsMax) hipLaunchKernelGGL(k_router<true>, grid, dim3(256), wr_bytes, stream, p, ut);
    else hipLaunchKernelGGL(k_router<false>, grid, dim3(256), 0, stream, p, ut);
    return hipGetLastError();
}

template <bool LISTS>
hipError_t launch_bf16(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    // about 4096 workgroups at most: each stages its unit's router rows once
    const int groups = (p.n_tok + 63) / 64, most = 4096 / ut.n > 1 ? 4096 / ut.n : 1;
    const dim3 grid(groups < most ? groups : most, ut.n);
    const size_t wr_bytes = (size_t)p.E * p.d_in * 2;
    if (wr_bytes <= kWrLdsMax)
        hipLaunchKernelGGL((k_router_mfma<LISTS, true>), grid, dim3(256), wr_bytes, stream, p, ut);
    else hipLaunchKernelGGL((k_router_mfma<LISTS, false>), grid, dim3(256), 0, stream, p, ut);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_router(const Problem& p, const UnitTab& ut, bool bf16, hipStream_t stream) {
    if (ut.n == 0 || p.n_tok == 0) return hipSuccess;
    return bf16 ? launch_bf16<false>(p, ut, stream) : launch_f32(p, ut, stream);
}

hipError_t launch_router_lists(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    if (ut.n == 0 || p.n_tok == 0) return hipSuccess;
    return launch_bf16<true>(p, ut, stream);
}

hipError_t launch_usage_stats(const uint32_t* counts, int n, int E, double* cv2, double* entropy,
                              hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_usage_stats, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, counts, n, E, cv2,
                       entropy);
    return hipGetLastError();
}

}  // namespace mot
