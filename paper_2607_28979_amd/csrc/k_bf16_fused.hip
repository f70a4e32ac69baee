// Host side of the fused kernel: shape support and dispatch to the
// per-shape instantiations (k_bf16_fused_inst.hip, built once per shape).
#include "k_bf16_fused_kernel.h"

namespace mot {

#define MOT_DECL(a, b) \
    hipError_t launch_fused_##a##_##b(const Problem& p, const UnitTab& ut, bool routed, hipStream_t stream);
MOT_DECL(128, 128) MOT_DECL(128, 256) MOT_DECL(128, 512)
MOT_DECL(256, 128) MOT_DECL(256, 256) MOT_DECL(256, 512)
MOT_DECL(512, 128) MOT_DECL(512, 256) MOT_DECL(512, 512)
#undef MOT_DECL

namespace {

hipError_t launch_shape(const Problem& p, const UnitTab& ut, bool routed, hipStream_t stream) {
    if (ut.n == 0 || p.n_tok == 0) return hipSuccess;
    const int key = p.d_in * 1000 + p.d_out;
    switch (key) {
        case 128128: return launch_fused_128_128(p, ut, routed, stream);
        case 128256: return launch_fused_128_256(p, ut, routed, stream);
        case 128512: return launch_fused_128_512(p, ut, routed, stream);
        case 256128: return launch_fused_256_128(p, ut, routed, stream);
        case 256256: return launch_fused_256_256(p, ut, routed, stream);
        case 256512: return launch_fused_256_512(p, ut, routed, stream);
        case 512128: return launch_fused_512_128(p, ut, routed, stream);
        case 512256: return launch_fused_512_256(p, ut, routed, stream);
        case 512512: return launch_fused_512_512(p, ut, routed, stream);
        default: return hipErrorNotSupported;
    }
}

}  // namespace

bool fused_supported(const Problem& p) {
    const bool din = p.d_in == 128 || p.d_in == 256 || p.d_in == 512;
    const bool dout = p.d_out == 128 || p.d_out == 256 || p.d_out == 512;
    return din && dout && p.hidden % 64 == 0 && p.E * p.hidden >= 64 && p.E <= MOT_MAX_EXPERTS;
}

namespace {

// Tile rows of the instantiation for (d_in, d_out), and workgroups a CU holds
struct Tile {
    int rows, wgs;
};
Tile fused_tile(const Problem& p) {
    switch (p.d_in * 1000 + p.d_out) {
#define MOT_TILE(a, b) case a * 1000 + b: return {Cfg<a, b>::BM, Cfg<a, b>::WGS};
        MOT_TILE(128, 128) MOT_TILE(128, 256) MOT_TILE(128, 512)
        MOT_TILE(256, 128) MOT_TILE(256, 256) MOT_TILE(256, 512)
        MOT_TILE(512, 128) MOT_TILE(512, 256) MOT_TILE(512, 512)
#undef MOT_TILE
        default: return {0, 0};
    }
}

}  // namespace

int fused_tile_rows(const Problem& p) { return fused_tile(p).rows; }

// When the tiles do not fill whole rounds of the chip, the last round leaves
// CUs idle for a whole walk of E*hidden (a call of one tile per unit keeps 56
// of 256 busy).  The tiles past the last full round are then cut along the
// walk into `parts` workgroups each.  The choice minimises the modelled time
// of those tiles, in chunk iterations: rounds * (chunks per part + a fixed cost
// of 8 for the router, pipeline fill and drain and stores, 6 more for a partial
// tile's fp32 stores) plus the combine (its launch, and the partial tiles written
// and read at 4 TB/s, in iterations of 1.25 us: they take 0.8 us, 256 -> 128, to 1.8,
// 512 -> 512).  Where a CU holds two workgroups, a round of at most one per CU runs its
// chunks in 0.7 of the time (128 -> 128: 0.58 us for one, 1.09 for two).  A split
// must save 2 % of the call.
//
// Measured, 1.5B -> 7B with 37 tokens (56 tiles, 4 parts): 669 -> 271 us, now
// the time to read the 1.4 GB of weights (5.2 TB/s); 7B -> 7B with 1501 tokens (896
// tiles, the last 128 in 2 parts): 3558 -> 3233 us.  Against every count of parts up
// to 16 for 124 calls (11 shapes, 1 to 3000 tokens), the rule's was 0.4 % above the
// best on average and never above the unsplit call.
FusedSplit fused_split_plan(const Problem& p, int n_units, size_t* bytes) {
    constexpr int kCUs = 256, kMaxParts = 16;
    constexpr size_t kMaxBytes = size_t(256) << 20;
    constexpr double kChunkUs = 1.25, kFixed = 8, kPartFixed = 6, kCombineUs = 4, kBytesPerUs = 4e6,
                     kAlone = 0.7;
    FusedSplit sp = {nullptr, 0, 0, 1};
    *bytes = 0;
    const Tile tl = fused_tile(p);
    if (tl.rows == 0 || n_units == 0 || p.n_tok == 0) return sp;
    const int64_t tiles = (int64_t)((p.n_tok + tl.rows - 1) / tl.rows) * n_units;
    const int slots = kCUs * tl.wgs;
    const int tail = (int)(tiles % slots), nch = p.E * p.hidden / 32;
    if (tail == 0 || tiles > (int64_t)1 << 30) return sp;
    // n workgroups of c chunks and a fixed cost f, in rounds
    auto rounds = [&](int64_t n, double c, double f) {
        const int64_t rest = n % slots;
        const double alone = tl.wgs > 1 && rest <= kCUs ? kAlone : 1;
        return (double)(n / slots) * (c + f) + (rest ? c * alone + f : 0);
    };
    const double whole = (double)(tiles / slots) * (nch + kFixed), unsplit = rounds(tail, nch, kFixed);
    const size_t tile_bytes = (size_t)tl.rows * p.d_out * sizeof(float);
    const double rows = (double)(p.n_tok < tl.rows ? p.n_tok : tl.rows);
    double best = unsplit - 0.02 * (whole + unsplit);
    for (int parts = 2; parts <= kMaxParts && parts <= nch / 2; ++parts) {
        const int64_t wgs = (int64_t)tail * parts;
        if (wgs * tile_bytes > kMaxBytes) break;
        const double combine = kCombineUs + 2.0 * wgs * rows * p.d_out * sizeof(float) / kBytesPerUs;
        const double t = rounds(wgs, (double)nch / parts, kFixed + kPartFixed) + combine / kChunkUs;
        if (t < best) {
            best = t;
            sp.parts = parts;
            *bytes = wgs * tile_bytes;
        }
    }
    if (sp.parts > 1) {
        sp.tail = tail;
        sp.full = (int32_t)(tiles - tail);
    }
    return sp;
}

namespace {

// dst rows of the split tiles: the sum of a row's partial tiles in part
// order, rounded once to bf16; 8 outputs per thread, blockIdx.y = tail tile
__global__ __launch_bounds__(256) void k_split_combine(Problem p, UnitTab ut, int tile_rows) {
    const int ntx = (p.n_tok + tile_rows - 1) / tile_rows, t = p.sp.full + blockIdx.y;
    const uint32_t code = ut.code[t / ntx];
    const int j = unit_j(code), x = unit_x(code), per_tok = p.d_out / 8;
    const int it = blockIdx.x * 256 + threadIdx.x, r = it / per_tok, o = it % per_tok * 8;
    const int tok = t % ntx * tile_rows + r;
    if (r >= tile_rows || tok >= p.n_tok) return;
    const size_t tile = (size_t)tile_rows * p.d_out;
    const float* part = p.sp.part + blockIdx.y * tile + (size_t)r * p.d_out + o;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll 4
    for (int s = 0; s < p.sp.parts; ++s) {
        const f32x4* q = reinterpret_cast<const f32x4*>(part + s * p.sp.tail * tile);
        const f32x4 qa = q[0], qb = q[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] += qa[e];
            b[e] += qb[e];
        }
    }
    const u32x4 v = {pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]),
                     pack_bf16x2(b[2], b[3])};
    uint16_t* dst = reinterpret_cast<uint16_t*>(p.dst[x]) + (size_t)j * p.n_tok * p.d_out;
    const size_t off = p.dst_layout == MOT_LAYOUT_BTHD ? (size_t)tok * p.d_out + o
                                                       : bhtd_row(p, tok) + (size_t)(o / p.D_tgt) * p.T * p.D_tgt +
                                                             o % p.D_tgt;
    *reinterpret_cast<u32x4*>(dst + off) = v;
}

}  // namespace

hipError_t launch_bf16_fused(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    hipError_t e = launch_shape(p, ut, false, stream);
    if (e == hipSuccess && p.sp.parts > 1) {
        const int rows = fused_tile_rows(p);
        const dim3 grid((rows * (p.d_out / 8) + 255) / 256, p.sp.tail);
        hipLaunchKernelGGL(k_split_combine, grid, dim3(256), 0, stream, p, ut, rows);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_bf16_fused_routed(const Problem& p, const UnitTab& ut, hipStream_t stream) {
    return launch_shape(p, ut, true, stream);
}

}  // namespace mot
