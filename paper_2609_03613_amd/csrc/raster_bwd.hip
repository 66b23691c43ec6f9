// Backward of the compositing: dL/d(splat) of every Gaussian from dL/d rgb
// and dL/d alpha of the image. The paper has no backward pass (it lists
// training as future work in its Conclusion); this is the derivative of the
// per-pixel step the forward rasters evaluate, over the same entry stream.
//
// Each 64-lane wavefront owns one 8x8 pixel block, as in the forward WAVE
// raster. Pass 1 repeats the forward walk (same staging, culling and blend,
// so the final transmittance and the last composited position come out
// bit-identical to the forward's), unless the forward's saved final
// transmittance and last position are given. Pass 2 walks the range backwards from
// the largest last position in the block, 64 entries at a time, with the
// same block cull and LDS compaction; each lane recovers the transmittance
// in front of an entry by dividing by the same binary32 (1 - alpha) the
// forward multiplied by (a hardware reciprocal, within an ulp). With S the
// colour behind the entry (T_final bg + the sum over later entries of T alpha
// c), the upstream gradient g enters only through the scalar
// R = g . S - g_alpha T_final, which every lane carries: per entry k
//   dL/dc_k     = g T_k alpha_k
//   dL/dalpha_k = T_k (g . c_k) - R / (1 - alpha_k),  R += T_k alpha_k (g . c_k)
// and, when alpha is not capped at 0.99, through alpha = o exp2(q'):
// dL/do = dL/dalpha exp2(q'), dL/dq' = dL/dalpha alpha ln 2, with q' the
// scaled quadratic form of the staged conic.
//
// The sums over the block's 64 pixels: q' is quadratic in the pixel position,
// so the six geometric gradients of an entry are combinations of the moments
// sum_p d(p) X^i Y^j (i + j <= 2) of d = dL/dalpha alpha, and the colour
// gradients are sum_p w(p) g(p) with w = T alpha. Each lane (pixel) only
// writes its d and w of up to kBatch = 8 entries to LDS; then the batch is
// transposed: lane (entry, pixel row) sums its row of 8 pixels in registers
// and the 8 rows are added by lane swaps. The entry's mean and conic turn the
// moments into gradient words, added to the Gaussian's line by float atomics,
// nine lanes per line so that a line is one memory request.
//
// Bound by VALU issue. Summing the nine gradients of every entry over the
// wavefront (33 instructions of recursive halving, after 17 to form them)
// took 233 us on 500k Gaussians at 1297x840 with 32-pixel tiles; the batches
// take 188 us (198 with four workgroups per CU, see BwdLds). The same contraction
// on the matrix cores (16 binary32 16x16x4 products per batch, the monomials as
// the constant operand) took 226 us: a binary32 product occupies its SIMD for 33
// cycles and no vector instruction of another wavefront is issued meanwhile.
#include <math.h>

#include "raster.hpp"

namespace tgs {

namespace {

using namespace raster;

__device__ __forceinline__ int wave_max_i32(int v) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) v = max(v, __shfl_xor(v, d, kWave));
    return v;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBatch = 8;     // entries per batch
constexpr int kWords = 9;     // gradient words per entry
constexpr int kSumLen = 12;   // LDS words per entry of the summed gradient words

// Per-wavefront LDS of the backward walk. At 31744 bytes a workgroup of four
// wavefronts, and under 96 registers, a CU holds five workgroups (LDS is given
// out in pieces of 1280 bytes); with rows padded to 68 words (8288 bytes a
// wavefront) and 106 registers it held four, and blocks of a few entries, which
// are chains of memory latencies, waited for a place: 6 thousand Gaussians on
// 1281x1041 47.6 us, now 42; 500 thousand on 1297x840 with 32-pixel tiles 199,
// now 188. The bank conflicts of the unpadded rows cost nothing measurable.
struct __align__(16) BwdLds {
    union {
        Staged stage[kWave + 2];  // the last two are read ahead, never written
        struct {
            Staged slots[kWave];
            union {
                float row[2 * kBatch * kWave];  // d of the batch's entries, then w; [entry][pixel]
                float sum[kBatch * kSumLen];    // after the row sums: the batch's gradient words
            };
            float g[3][kWave];  // upstream colour gradients of the block's pixels
        };
    };
};
static_assert((4 * sizeof(BwdLds) + 1279) / 1280 * 5 <= 160 * 1024 / 1280, "five workgroups per CU");

// Sums of a over the lane pairs (l, l ^ 32) in the lower half and of b in the
// upper half.
__device__ __forceinline__ float swap_sum32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sums of a over the lane pairs (l, l ^ 16) in the even rows of 16 lanes and
// of b in the odd rows.
__device__ __forceinline__ float swap_sum16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// v + the value of lane l ^ 8.
__device__ __forceinline__ float sum8(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));  // row_ror:8
}

// NW: wavefronts of a workgroup, 1 with 8-pixel tiles (one block each; with the
// LDS of four, only four such wavefronts fit a CU: 200 thousand Gaussians on
// 1200x800 took 414 us, now 155), else 4.
template <int SRC, int NW>
__global__ void __launch_bounds__(NW * kWave, 5) raster_bwd_kernel(RasterArgs A, const float* __restrict__ d_rgb,
                                                         const float* __restrict__ d_alpha,
                                                         const float* __restrict__ trans_in,
                                                         const int32_t* __restrict__ last_in,
                                                         float* __restrict__ d_splats) {
#pragma clang fp contract(off)
    __shared__ BwdLds lds[NW];
    const int w = threadIdx.x / kWave, l = lane();
    WaveBlock wb;
    if (!block_of_wave(A, w, wb)) return;
    const int x0 = wb.tx * A.tile, y0 = wb.ty * A.tile;
    float xa, xb, ya, yb;
    if (!block_box_at(wb.bx, wb.by, x0, y0, A.width, A.height, xa, xb, ya, yb)) return;  // block outside the image
    const int lx = wb.bx + (l & 7), ly = wb.by + (l >> 3);
    const int x = x0 + lx, y = y0 + ly;
    const bool inside = x < A.width && y < A.height;
    const float ox = (float)x0, oy = (float)y0;
    const float px = (float)lx + 0.5f, py = (float)ly + 0.5f;
    const uint32_t begin = tile_begin(A, wb.t);
    const uint32_t end = tile_end(A, wb.t);
    Staged* st = lds[w].stage;

    // pass 1: the forward walk, or the forward's saved T and last (requested
    // before the flag is waited for, and the ids below before the upstream
    // gradients: 6 thousand Gaussians on 1281x1041 47.6 us, 45 so)
    const int64_t pixel = (int64_t)y * A.width + x;
    Pix p{1.0f, 0.f, 0.f, 0.f, -1, 0, 0, 0, !inside};
    if (trans_in && inside) {
        p.T = trans_in[pixel];
        p.last = last_in[pixel];
    }
    if (A.counters[2] != 0) return;  // truncated stream: the forward image is NaN, no gradient
    if (!trans_in) wave_forward<SRC, false>(A, st, wb.bi, begin, end, ox, oy, px, py, xa, xb, ya, yb, p);

    // pass 2: backwards from the last composited entry
    const int hi = wave_max_i32(p.last);
    if (hi < 0) return;
    // Chunks of 64 entries downwards from hi; lane l holds entry top - l. The
    // gathers are software-pipelined as in the forward walk: while chunk i
    // is processed, the splats of chunk i + 1 are in flight and the ids of
    // chunk i + 2 follow once chunk i's ids are staged. Every lane issues
    // every load (lanes below the range read its first entry and are
    // dropped by the range test).
    const float4* sp = reinterpret_cast<const float4*>(A.splats);
    auto id_clamped = [&](int64_t e) { return id_at<SRC>(A, (uint32_t)(e >= (int64_t)begin ? e : (int64_t)begin)); };
    auto gather = [&](uint32_t g, float4& r0, float4& r1, float4& r2) {
        const float4* q = sp + kSplatVec * (int64_t)g;
        r0 = q[0];
        r1 = q[1];
        r2 = q[2];
    };
    float4 a0, a1, a2, b0, b1, b2;
    uint32_t ida = id_clamped((int64_t)hi - l), idb = id_clamped((int64_t)hi - kWave - l);
    float gr = 0.f, gg = 0.f, gb = 0.f, ga = 0.f;
    if (inside) {
        gr = d_rgb[3 * pixel];
        gg = d_rgb[3 * pixel + 1];
        gb = d_rgb[3 * pixel + 2];
        ga = d_alpha ? d_alpha[pixel] : 0.f;
    }
    gather(ida, a0, a1, a2);
    const float Tf = p.T;
    float T = Tf;
    float R = Tf * (gr * A.bg[0] + gg * A.bg[1] + gb * A.bg[2] - ga);
    // A pixel whose upstream gradient is not finite is left out of the
    // transposed colour sums (0 times it would reach entries that it does not
    // see) and adds its own terms one by one below.
    BwdLds& L = lds[w];
    const bool odd = !(isfinite(gr) && isfinite(gg) && isfinite(gb));
    const uint64_t odd_mask = ballot(odd);
    L.g[0][l] = odd ? 0.f : gr;
    L.g[1][l] = odd ? 0.f : gg;
    L.g[2][l] = odd ? 0.f : gb;
    const float cx = (float)wb.bx + 4.0f, cy = (float)wb.by + 4.0f;  // block centre, tile-local
    // the transposed role of this lane: entry l % 8 of the batch, pixel row l / 8
    const int te = l & 7, ty = l >> 3;
    const float Y = (float)ty - 3.5f;
    // where its sums of the first, second and third swapped register go
    const int row16 = l >> 4;
    const int w0 = row16 == 1 ? 2 : row16 == 2 ? 1 : row16;  // words 0, 2, 1, 3
    // the entry and word that this lane adds: nine consecutive lanes per line,
    // so that a line is one memory request (the batch's last line separately)
    const int ae = l < (kBatch - 1) * kWords ? l / kWords : kBatch, aw = l % kWords;
    int nb = 0;        // entries in the batch
    uint32_t bid = 0;  // lane k: id of the batch's entry k
    auto flush = [&]() {
        // the entry's mean and conic, from the line that the walk gathered
        const uint32_t tid = shfl_u32(bid, te);
        float4 e0 = make_float4(0.f, 0.f, 0.f, 0.f), e1 = make_float4(0.f, 0.f, 0.f, 1.f);
        if (te < nb) {
            const float4* q = sp + kSplatVec * (int64_t)tid;
            e0 = q[0];
            e1 = q[1];
        }
        wave_sync();
        float wd[6], cr, cg, cb;
        {
#pragma clang fp contract(fast)
            const f32x4* dp = reinterpret_cast<const f32x4*>(L.row + te * kWave + 8 * ty);
            const f32x4* wp = reinterpret_cast<const f32x4*>(L.row + (kBatch + te) * kWave + 8 * ty);
            const f32x4 d0 = dp[0], d1 = dp[1], v0 = wp[0], v1 = wp[1];
            // dx = u - X and dy = v with (u, v) the mean's offset from the
            // block centre and from the row, from the staged mean: the d are
            // those of its rounded position
            const float u = ((e0.x - ox) + e0.z) - cx, v = (((e0.y - oy) + e0.w) - cy) - Y;
            float m0 = 0.f, m1 = 0.f, m2 = 0.f;  // sums of d, d dx, d dx^2
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float d = i < 4 ? d0[i] : d1[i - 4], dx = u - ((float)i - 3.5f), t = d * dx;
                m0 += d;
                m1 = fmaf(d, dx, m1);
                m2 = fmaf(t, dx, m2);
            }
            // this row's share of the gradient words: q = a dx^2 + 2 b dx dy +
            // c dy^2 and q' ln 2 = -q / 2
            const float my = v * m0;
            wd[0] = -(e1.x * m1 + e1.y * my);
            wd[1] = -(e1.y * m1 + e1.z * my);
            wd[2] = -0.5f * m2;
            wd[3] = -v * m1;
            wd[4] = -0.5f * (v * my);
            wd[5] = m0 * __builtin_amdgcn_rcpf(e1.w);  // d = dL/dalpha o exp2(q')
            auto dot = [&](int ch) {
                const f32x4* gp = reinterpret_cast<const f32x4*>(L.g[ch] + 8 * ty);
                const f32x4 g0 = gp[0], g1 = gp[1];
                float s = v0[0] * g0[0] + v0[1] * g0[1];
                s += v0[2] * g0[2];
                s += v0[3] * g0[3];
                s += v1[0] * g1[0];
                s += v1[1] * g1[1];
                s += v1[2] * g1[2];
                return s + v1[3] * g1[3];
            };
            cr = dot(0);
            cg = dot(1);
            cb = dot(2);
        }
        // over the 8 rows (lanes l ^ 32, l ^ 16, l ^ 8): register p holds
        // words 0, 2, 1, 3 in its four rows of 16 lanes, q words 4, 6, 5, 7
        const float p = sum8(swap_sum16(swap_sum32(wd[0], wd[1]), swap_sum32(wd[2], wd[3])));
        const float q = sum8(swap_sum16(swap_sum32(wd[4], wd[5]), swap_sum32(cr, cg)));
        const float r8 = swap_sum32(cb, cb);
        const float r = sum8(swap_sum16(r8, r8));
        wave_sync();
        if ((l & 8) == 0) {
            float* s = L.sum + te * kSumLen;
            s[w0] = p;
            s[4 + w0] = q;
            s[8] = r;
        }
        wave_sync();
        const uint32_t g0 = shfl_u32(bid, ae < kBatch ? ae : 0);
        if (ae < nb) unsafeAtomicAdd(d_splats + kGradWords * (int64_t)g0 + aw, L.sum[ae * kSumLen + aw]);
        if (nb == kBatch) {
            const uint32_t g1 = (uint32_t)__builtin_amdgcn_readlane((int)bid, kBatch - 1);
            if (l < kWords) unsafeAtomicAdd(d_splats + kGradWords * (int64_t)g1 + l, L.sum[(kBatch - 1) * kSumLen + l]);
        }
        nb = 0;
        wave_sync();
    };
    auto chunk = [&](int64_t top, const float4& q0, const float4& q1, const float4& q2, uint32_t& gcur,
                     uint32_t g_next, float4& n0, float4& n1, float4& n2) {
        const int64_t e = top - l;
        bool keep = e >= (int64_t)begin;
        gather(g_next, n0, n1, n2);
        Staged s;
        if (keep) {
            float s2;
            stage_splat(q0, q1, q2, ox, oy, s.a, s.b, s2);
            s.c = make_float2(s2, __uint_as_float(gcur));
            keep = block_may_touch(s.a.x, s.a.y, q1.x, q1.y, q1.z, q1.w, xa, xb, ya, yb);
        }
        const uint64_t m = ballot(keep);
        if (keep) st[rank_in(m)] = s;
        gcur = id_clamped(e - 2 * kWave);  // this set's next chunk (i + 2)
        if (m == 0) return;
        wave_sync();
        // an entry's position is top - (its lane): composited by this pixel
        // when the lane is at least `first`
        const int first = (int)(top - p.last);
        uint64_t left = m;
        auto step = [&](const Staged& c) {
            const int src = __builtin_ctzll(left);
            left &= left - 1;
            // the forward's per-pixel test, same operations
            const float dx = c.a.x - px;
            const float dy = c.a.y - py;
            const float wq = fmaf(c.a.z, dx, c.a.w * dy);
            const float q2 = fmaf(dx, wq, (c.b.x * dy) * dy);
            const float araw = c.b.y * __builtin_amdgcn_exp2f(q2);
            const bool comp = src >= first && q2 <= 0.0f && araw >= kAlphaMin;
            if (ballot(comp) == 0) return;
            {
#pragma clang fp contract(fast)
                // the gradient arithmetic may fuse (the bars are not bitwise);
                // the compositing decision above repeats the forward exactly
                const float alpha = __builtin_amdgcn_fmed3f(araw, 0.0f, kAlphaMax);
                // 1 / (1 - alpha) to within an ulp (hardware reciprocal);
                // the gradients carry a 1e-3 tolerance, not the forward's
                // bit-exactness
                const float inv = __builtin_amdgcn_rcpf(1.0f - alpha);
                const float Tk = T * inv;
                const float wt = alpha * Tk;
                const float gc = gr * c.b.z + gg * c.b.w + gb * c.c.x;
                const float dLda = Tk * gc - inv * R;
                L.row[nb * kWave + l] = comp && araw <= kAlphaMax ? dLda * araw : 0.f;
                L.row[(kBatch + nb) * kWave + l] = comp ? wt : 0.f;
                R = comp ? R + wt * gc : R;
                T = comp ? Tk : T;
                const uint32_t id = __float_as_uint(c.c.y);
                bid = l == nb ? id : bid;
                if (odd_mask != 0 && odd && comp) {
                    float* line = d_splats + kGradWords * (int64_t)id;
                    unsafeAtomicAdd(line + 6, gr * wt);
                    unsafeAtomicAdd(line + 7, gg * wt);
                    unsafeAtomicAdd(line + 8, gb * wt);
                }
                ++nb;
            }
        };
        // two entries per round, each read while the one before is worked on
        // (slots past the survivors hold stale entries, read and not used)
        const Staged* nx = st;
        Staged ca = nx[0], cb;
        for (;;) {
            cb = nx[1];
            step(ca);
            ca = nx[2];
            if (left != 0) step(cb);
            if (nb >= kBatch - 1) {
                flush();
                ca = nx[2];  // (not kept in registers meanwhile)
            }
            if (left == 0) break;
            nx += 2;
        }
        wave_sync();
    };
    for (int64_t top = hi;;) {
        if (top < (int64_t)begin) break;
        chunk(top, a0, a1, a2, ida, idb, b0, b1, b2);
        top -= kWave;
        if (top < (int64_t)begin) break;
        chunk(top, b0, b1, b2, idb, ida, a0, a1, a2);
        top -= kWave;
    }
    if (nb) flush();
}

}  // namespace

hipError_t launch_raster_backward(const RasterArgs& a, const float* d_rgb, const float* d_alpha,
                                  const float* trans_in, const int32_t* last_in, float* d_splats, hipStream_t s) {
    const int T = a.tiles_x * a.tiles_y;
    if (T == 0) return hipSuccess;
    const int B = blocks_per_tile(a.tile), G = groups_per_tile(a.tile), NW = B < 4 ? 1 : 4;
    const auto kernel = a.vals ? (NW == 1 ? raster_bwd_kernel<SRC_VALS, 1> : raster_bwd_kernel<SRC_VALS, 4>)
                               : (NW == 1 ? raster_bwd_kernel<SRC_PAIRS, 1> : raster_bwd_kernel<SRC_PAIRS, 4>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(T * G)), dim3((unsigned)(NW * kWave)), 0, s, a, d_rgb, d_alpha, trans_in,
                       last_in, d_splats);
    return hipGetLastError();
}

}  // namespace tgs
