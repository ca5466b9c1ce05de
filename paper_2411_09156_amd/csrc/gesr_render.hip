// Tile renderers of the GES rasterizer (gfx950).
//
// Forward: front-to-back alpha blending (Eq. 5 evaluated discretely) of the
// generalized-exponential falloff exp(-kappa q^(beta/2)) (Eq. 3 in screen
// space).  One workgroup per (view, tile) work item, taken in worklist order
// (most work first: the list length, or the positions a previous forward
// evaluated per tile, so the hardware dispatcher schedules greedily by
// load); a wave's lanes cover 8x8 pixel blocks so that they see similar
// footprints.  Splat records are staged through LDS in batches and every lane
// reads them by broadcast.
//
// Backward: the same tile mapping, traversing each pixel's list in reverse
// from its n_contrib and recovering transmittance by division from final_T
// (no per-fragment state is stored in the forward).  Per splat, each wave
// sums its pixels' 10 gradient terms with cross-lane reductions, the waves'
// sums are added in fixed order, and the tile writes one partial per
// instance: no atomics, bitwise reproducible.

#include "gesr_device.h"
#include "gesr_kernels.h"

namespace gesr {

namespace {

template <int TW, int TH>
struct TileMap {
    static constexpr int NT = TW * TH;
    static constexpr int NW = NT / 64;
    static constexpr int WX = TW / 8;
    // pixel offset inside the tile of thread `tid`
    __device__ static __forceinline__ void pixel(int tid, int& lx, int& ly) {
        const int w = tid >> 6, l = tid & 63;
        lx = (w % WX) * 8 + (l & 7);
        ly = (w / WX) * 8 + (l >> 3);
    }
};

struct TileInfo {
    int v;
    int x, y;       // pixel of this thread
    bool inside;
    uint32_t pix;   // index into per-pixel arrays
    uint32_t ch;    // channel stride of the view (H * W)
    uint32_t img;   // index of channel 0 in the image arrays
    uint32_t tx, ty;
    uint32_t r0, r1;  // list range
};

template <int TW, int TH>
__device__ __forceinline__ TileInfo tile_info(const RenderArgs& a, uint32_t t) {
    TileInfo ti;
    ti.v = view_of_tile(a.cams, t);
    const DevView& w = a.cams.v[ti.v];
    const uint32_t lt = t - w.tile_base;
    ti.tx = lt % (uint32_t)w.tiles_x;
    ti.ty = lt / (uint32_t)w.tiles_x;
    int lx, ly;
    TileMap<TW, TH>::pixel(threadIdx.x, lx, ly);
    ti.x = (int)ti.tx * TW + lx;
    ti.y = (int)ti.ty * TH + ly;
    ti.inside = ti.x < w.W && ti.y < w.H;
    const uint32_t local = (uint32_t)ti.y * (uint32_t)w.W + (uint32_t)ti.x;
    ti.pix = w.pix_base + local;
    ti.ch = (uint32_t)w.W * (uint32_t)w.H;
    ti.img = 3u * w.pix_base + local;
    const uint2 r = reinterpret_cast<const uint2*>(a.ranges)[t];
    ti.r0 = r.x;
    ti.r1 = r.y;
    return ti;
}

// Stage record `vi` into LDS as (u, v, L00, L10), (L11, o, beta/2, qmax),
// (r, g, b, -kappa beta); the last is the splat's factor of 2 dL/dq (below).
__device__ __forceinline__ void stage_record(const float* rec, uint32_t vi, float kappa, float4& sa, float4& sb,
                                             float4& sc) {
    const float4* r = reinterpret_cast<const float4*>(rec + (size_t)vi * GESR_REC_FLOATS);
    const float4 b = r[1], c = r[2];
    sa = r[0];
    sb = make_float4(b.x, b.y, 0.5f * b.z, b.w);
    sc = make_float4(c.x, c.y, c.z, -kappa * b.z);
}

// One pixel's upstream gradients (colour; depth and opacity with the extended
// channels) and its state in the reverse traversal: transmittance in front of the
// fragment last visited and what lies behind per unit transmittance.
struct PixelUp {
    float g0, g1, g2, gD, gA;
};
struct PixelAdjoint {
    float T, Br, Bg, Bb, BD, BA;
};

template <bool EXT>
__device__ __forceinline__ PixelUp load_up(const RenderArgs& a, uint32_t pix, uint32_t img, uint32_t ch) {
    PixelUp u{a.dL_dimage[img], a.dL_dimage[img + ch], a.dL_dimage[img + 2 * ch], 0.f, 0.f};
    if (EXT) {
        if (a.dL_ddepth) u.gD = a.dL_ddepth[pix];
        if (a.dL_dalpha) u.gA = a.dL_dalpha[pix];
    }
    return u;
}

// Whether an upstream gradient of the wave's pixels is not finite (or nearly so).
template <bool EXT>
__device__ __forceinline__ bool any_odd(const PixelUp& u) {
    const float s = fabsf(u.g0) + fabsf(u.g1) + fabsf(u.g2) + (EXT ? fabsf(u.gD) : 0.0f);
    return __builtin_amdgcn_ballot_w64(!(s < INFINITY)) != 0ull;
}

// The background has no depth and no opacity.
__device__ __forceinline__ PixelAdjoint behind_all(const DevSettings& st, float T) {
    return PixelAdjoint{T, st.bg[0], st.bg[1], st.bg[2], 0.f, 0.f};
}

// Takes a pixel past one fragment (in reverse): its weight aT = alpha T and
// dl = dL/dalpha where alpha is neither skipped nor capped, 0 elsewhere.  A
// fragment with on = false (not the pixel's, or below alpha_min) has alpha 0: it
// leaves T (rcp(1) = 1) and what lies behind as they are.  With ON every lane's
// fragment is on, and the skip and the cap are so rare inside the footprint that
// a wave-uniform branch around their selects pays (three instructions at half rate:
// 1,900 -> 1,780 us on 500k x 8 mixed views, 1,890 -> 1,770 on 1M flat x 4, 5.62 ->
// 5.50 ms on 3M x 16); where some lanes are off the selects stay.
template <bool EXT, bool ON>
__device__ __forceinline__ void pixel_step(const Fragment& f, bool on, const float4& rc, float z,
                                           const DevSettings& st, const PixelUp& u, PixelAdjoint& px, float& aT,
                                           float& dl) {
    const bool low = f.oG < st.alpha_min, high = f.oG > st.alpha_max;
    uint64_t rare = 0ull;
    float al = f.oG;
    if constexpr (ON) {
        rare = __builtin_amdgcn_ballot_w64(low) | __builtin_amdgcn_ballot_w64(high);
        if (rare != 0ull) {
            al = low ? 0.0f : fminf(f.oG, st.alpha_max);
            asm volatile("" : "+v"(al));  // keeps the branch
        }
    } else {
        al = on && !low ? f.alpha : 0.0f;
    }
    px.T *= hw_rcp(1.0f - al);
    aT = al * px.T;
    const float er = rc.x - px.Br, eg = rc.y - px.Bg, eb = rc.z - px.Bb;
    const float colour = fmaf(eb, u.g2, fmaf(er, u.g0, eg * u.g1));
    float dLda = px.T * colour;
    px.Br = fmaf(al, er, px.Br);
    px.Bg = fmaf(al, eg, px.Bg);
    px.Bb = fmaf(al, eb, px.Bb);
    if (EXT) {
        const float ed = z - px.BD, ea = 1.0f - px.BA;
        // (the channels' product is the rounded one)
        dLda = fmaf(px.T, colour, px.T * fmaf(ed, u.gD, ea * u.gA));
        px.BD = fmaf(al, ed, px.BD);
        px.BA = fmaf(al, ea, px.BA);
    }
    dl = dLda;
    if constexpr (ON) {
        if (rare != 0ull) {
            dl = low || high ? 0.0f : dLda;
            asm volatile("" : "+v"(dl));
        }
    } else {
        dl = on && !low && !high ? dLda : 0.0f;
    }
}

// Adds one fragment's gradient terms to the splat's sums gr.  With
// G = exp(-kappa P), P = q^(beta/2), X = dL/dalpha o G P and d = -kappa beta X / q
// = 2 dL/dq, q = t^2 + w^2, t = L00 dx + L10 dy, w = L11 dy, (dx, dy) = pixel - (u, v):
//   gr = (sum d t, sum d w, sum d t dx, sum d t dy, sum d w dy, sum dL/dalpha G,
//         sum X ln q (-kappa / 2), dL/dr, dL/dg, dL/db)
// The conic factor is the same for all of a tile's pixels, so the centre's
// gradient takes it once, in `splat_partial`.  At q = 0 the footprint and beta terms
// are 0: P and X are, and the legacy product takes 0 times infinity as 0.  A flat
// splat seen edge-on amplifies the rounding of the three footprint sums in its
// scale gradient, so their terms keep this order of products.
// The kernel is bound by these instructions: the products in place of selects and
// the two sums for the centre took 53 instructions to 47 (a compare or select
// takes 4.3 cycles per wave on gfx950, a product 2.3), a step over 3M splats x 16
// views from 20.2 to 19.7 ms and over 1M flat splats x 4 views from 5.00 to 4.90 ms.
struct FragmentTerms {
    float aT, dl, G, xl, tq, wq;  // xl = X log2 q, tq = d t, wq = d w
};
__device__ __forceinline__ FragmentTerms fragment_terms(const Fragment& f, float rcw, float aT, float dl) {
    const float X = dl * f.oG * f.P;
    const float d = mul_legacy(X * rcw, hw_rcp(f.q));
    return FragmentTerms{aT, dl, f.G, mul_legacy(X, f.l2q), d * f.t, d * f.w};
}
template <bool EXT>
__device__ __forceinline__ void add_terms(const FragmentTerms& v, float dx, float dy, float c2, const PixelUp& u,
                                          float (&gr)[GESR_PARTIAL_FLOATS], float& gz) {
    gr[7] = fmaf(v.aT, u.g0, gr[7]);
    gr[8] = fmaf(v.aT, u.g1, gr[8]);
    gr[9] = fmaf(v.aT, u.g2, gr[9]);
    if (EXT) gz = fmaf(v.aT, u.gD, gz);
    gr[5] = fmaf(v.dl, v.G, gr[5]);
    gr[6] = fmaf(v.xl, c2, gr[6]);
    gr[0] += v.tq;
    gr[1] += v.wq;
    gr[2] = fmaf(v.tq, dx, gr[2]);
    gr[3] = fmaf(v.tq, dy, gr[3]);
    gr[4] = fmaf(v.wq, dy, gr[4]);
}

// The instance's partials (layout: d/du, d/dv, d/dL00, d/dL10, d/dL11, d/do,
// d/dbeta, d/dr, d/dg, d/db) from the sums s and the staged record (ra = u, v,
// L00, L10; rb.x = L11).
__device__ __forceinline__ void splat_partial(float (&s)[GESR_PARTIAL_FLOATS + 1], const float4& ra, const float4& rb) {
    const float st = s[0], sw = s[1];
    s[0] = -(st * ra.z);
    s[1] = -fmaf(sw, rb.x, st * ra.w);
}

constexpr uint32_t kNoInstance = 0xFFFFFFFFu;

// Slot of the instance of a pair in tile (tx, ty) in the pair-major order: the
// pair's instance base plus the tile's row-major position in its rectangle.
// When the lists overflowed their capacity the ranges no longer match the
// truncated lists, so a listed splat may not cover the tile or its slot may lie
// beyond the capacity; kNoInstance then suppresses the partial write.
__device__ __forceinline__ uint32_t instance_index(const RenderArgs& a, uint2 r, uint32_t base, uint32_t tx,
                                                   uint32_t ty) {
    const uint32_t tx0 = r.x & 0xFFFFu, ty0 = r.x >> 16, tx1 = r.y & 0xFFFFu, ty1 = r.y >> 16;
    const uint32_t inst = base + (ty - ty0) * (tx1 - tx0 + 1u) + (tx - tx0);
    const bool inside = tx >= tx0 && tx <= tx1 && ty >= ty0 && ty <= ty1;
    return inside && inst < a.m_cap ? inst : kNoInstance;
}

// Partials of one instance (ten terms, dz with the extended channels, in a
// twelve-float slot): written, and its slot's bit set, unless all are zero
// (the segmented sum adding +-0 or skipping the slot gives the same float
// result, since its running sums start at +0).
template <bool EXT>
__device__ __forceinline__ void write_partial(const RenderArgs& a, uint32_t slot, const float* s) {
    constexpr int NT = EXT ? GESR_PARTIAL_FLOATS + 1 : GESR_PARTIAL_FLOATS;
    bool nz = false;
#pragma unroll
    for (int k = 0; k < NT; ++k) nz |= s[k] != 0.0f;
    if (!nz) return;
    float4* dst = reinterpret_cast<float4*>(a.partials + (size_t)slot * kPartialStride);
    dst[0] = make_float4(s[0], s[1], s[2], s[3]);
    dst[1] = make_float4(s[4], s[5], s[6], s[7]);
    dst[2] = make_float4(s[8], s[9], EXT ? s[10] : 0.0f, 0.0f);
    atomicOr(a.visited + (slot >> 5), 1u << (slot & 31u));
}

template <int TW, int TH, bool COUNT>
__global__ __launch_bounds__(TW * TH) void k_render_fwd(RenderArgs a) {
    constexpr int NT = TW * TH;
    __shared__ float4 sA[NT], sB[NT], sC[NT];
    const uint32_t t = a.worklist[blockIdx.x];
    const TileInfo ti = tile_info<TW, TH>(a, t);
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const float px = (float)ti.x + 0.5f, py = (float)ti.y + 0.5f;

    float T = 1.0f, cr = 0.f, cg = 0.f, cb = 0.f;
    uint32_t contrib = 0, listed = 0, hit = 0;
    bool done = !ti.inside;
    uint32_t stop = ti.r1;  // first list position not evaluated
    for (uint32_t base = ti.r0; base < ti.r1; base += NT) {
        if (__syncthreads_count(done) == NT) {
            stop = base;
            break;
        }
        const uint32_t pos = base + threadIdx.x;
        if (pos < ti.r1) stage_record(a.rec, a.val_sorted[pos], st.kappa, sA[threadIdx.x], sB[threadIdx.x], sC[threadIdx.x]);
        __syncthreads();
        const int cnt = (int)min<uint32_t>(NT, ti.r1 - base);
        if (!done) {
            for (int j = 0; j < cnt; ++j) {
                const float4 ra = sA[j];
                const float4 rb = sB[j];
                Fragment f;
                const float q = ges_q(ra, rb.x, px, py, f);
                if (COUNT) ++listed;
                if (q > rb.w) continue;  // beyond the alpha_min footprint
                ges_alpha(q, rb.z, rb.y, nk, amax, f);
                if (f.alpha < st.alpha_min) continue;
                if (COUNT) ++hit;
                const float Tn = T * (1.0f - f.alpha);
                if (Tn < st.t_min) {
                    done = true;
                    break;
                }
                const float4 rc = sC[j];
                const float w = f.alpha * T;
                cr = fmaf(rc.x, w, cr);
                cg = fmaf(rc.y, w, cg);
                cb = fmaf(rc.z, w, cb);
                T = Tn;
                contrib = base + (uint32_t)j + 1u - ti.r0;
            }
        }
    }
    if (a.tile_work && threadIdx.x == 0) a.tile_work[t] = stop - ti.r0;
    if (ti.inside) {
        a.image[ti.img] = fmaf(T, st.bg[0], cr);
        a.image[ti.img + ti.ch] = fmaf(T, st.bg[1], cg);
        a.image[ti.img + 2 * ti.ch] = fmaf(T, st.bg[2], cb);
        a.final_T[ti.pix] = T;
        a.n_contrib[ti.pix] = contrib;
        if (COUNT) {
            a.n_listed[ti.pix] = listed;
            a.n_hit[ti.pix] = hit;
        }
    }
}

// 32x32: at most 64 registers, so that a CU holds two workgroups of 16 waves (200,000
// splats, two views of 1600x1064: 931 us; one workgroup, with 94 registers, 1,365).
template <int TW, int TH, int BATCH>
__global__ __launch_bounds__(TW * TH, TW * TH == 1024 ? 8 : 1) void k_render_bwd(RenderArgs a) {
    constexpr int NT = TW * TH;
    constexpr int NW = NT / 64;
    constexpr int NP = GESR_PARTIAL_FLOATS;
    static_assert(BATCH <= NT, "batch larger than the workgroup");
    static_assert(NP == 10, "wave_sum10 reduces ten values");
    __shared__ float4 sA[BATCH], sB[BATCH], sC[BATCH];
    __shared__ uint32_t sInst[BATCH];
    __shared__ float sRed[NW][BATCH][NP];
    __shared__ uint32_t sMax[NW];

    const uint32_t t = a.worklist[blockIdx.x];
    const TileInfo ti = tile_info<TW, TH>(a, t);
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const float c2 = -0.5f * kLn2 * st.kappa;
    const float px = (float)ti.x + 0.5f, py = (float)ti.y + 0.5f;
    const uint32_t lane = __lane_id(), wave = threadIdx.x >> 6;

    PixelAdjoint pa = behind_all(st, 0.f);
    PixelUp up{};
    uint32_t nc = 0;
    if (ti.inside) {
        pa.T = a.final_T[ti.pix];
        nc = a.n_contrib[ti.pix];
        up = load_up<false>(a, ti.pix, ti.img, ti.ch);
    }

    // deepest list position any pixel of the tile composited
    const uint32_t wmax = wave_max_u32(nc);
    if (lane == 0) sMax[wave] = wmax;
    __syncthreads();
    uint32_t maxnc = 0;
    for (int w = 0; w < NW; ++w) maxnc = max(maxnc, sMax[w]);
    const uint32_t end = ti.r0 + maxnc;  // positions >= end contributed to no pixel
    const int slot = lane < 16 ? wave_sum10_slot(lane) : NP;  // value this lane writes after a reduction

    for (uint32_t hi = end; hi > ti.r0;) {
        const uint32_t lo = (hi - ti.r0 > (uint32_t)BATCH) ? hi - BATCH : ti.r0;
        const int cnt = (int)(hi - lo);
        if ((int)threadIdx.x < cnt) {
            const uint32_t pos = hi - 1u - threadIdx.x;
            const uint32_t vi = a.val_sorted[pos];
            stage_record(a.rec, vi, st.kappa, sA[threadIdx.x], sB[threadIdx.x], sC[threadIdx.x]);
            const float4 r3 = reinterpret_cast<const float4*>(a.rec + (size_t)vi * GESR_REC_FLOATS)[3];
            const uint2 r = make_uint2(__float_as_uint(r3.x), __float_as_uint(r3.y));  // the pair's rectangle
            sInst[threadIdx.x] = instance_index(a, r, a.inst_base[vi], ti.tx, ti.ty);
        }
        __syncthreads();
        for (int j = 0; j < cnt; ++j) {
            const uint32_t prel = hi - 1u - (uint32_t)j - ti.r0;  // 0-based list position
            float gr[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) gr[k] = opaque_zero();
            bool act = false;
            if (prel < nc) {
                const float4 ra = sA[j];
                const float4 rb = sB[j];
                Fragment f;
                const float q = ges_q(ra, rb.x, px, py, f);
                if (q <= rb.w) {
                    ges_alpha(q, rb.z, rb.y, nk, amax, f);
                    act = true;
                    const float4 rc = sC[j];
                    float gz = 0.0f, aT, dl;
                    pixel_step<false, true>(f, true, rc, 0.0f, st, up, pa, aT, dl);
                    add_terms<false>(fragment_terms(f, rc.w, aT, dl), f.dx, f.dy, c2, up, gr, gz);
                }
            }
            if (__ballot(act) != 0ull) {
                const float tot = wave_sum10(gr, lane);
                if (slot < NP) sRed[wave][j][slot] = tot;
            } else if ((int)lane < NP) {
                sRed[wave][j][lane] = 0.f;
            }
        }
        __syncthreads();
        for (int jj = threadIdx.x; jj < cnt; jj += NT) {
            if (sInst[jj] == kNoInstance) continue;
            float s[NP + 1];
#pragma unroll
            for (int k = 0; k < NP; ++k) s[k] = sRed[0][jj][k];
            for (int w = 1; w < NW; ++w)
#pragma unroll
                for (int k = 0; k < NP; ++k) s[k] += sRed[w][jj][k];
            splat_partial(s, sA[jj], sB[jj]);
            write_partial<false>(a, sInst[jj], s);
        }
        __syncthreads();
        hi = lo;
    }
}

// One pixel of the forward traversal.  A terminated pixel (and one outside the
// image) keeps its transmittance with the sign bit set: the sign then fails the
// termination test of every later fragment, so no separate flag is carried.
struct FwdPixel {
    float T, r, g, b, d;
    uint32_t contrib;
};

// Composites one fragment; alpha is 0 where it is skipped (T and the sums then stay
// as they are: colours and depths of kept records are finite and non-negative).
template <bool EXT>
__device__ __forceinline__ void blend(FwdPixel& p, float alpha, bool ok, const float4& rc, float z, uint32_t pos,
                                      float t_min) {
    const float Tn = p.T * (1.0f - alpha);
    const bool keep = !(Tn < t_min);
    const float wgt = keep ? alpha * p.T : 0.0f;
    p.r = fmaf(rc.x, wgt, p.r);
    p.g = fmaf(rc.y, wgt, p.g);
    p.b = fmaf(rc.z, wgt, p.b);
    if (EXT) p.d = fmaf(z, wgt, p.d);
    p.contrib = ok && keep ? pos : p.contrib;
    p.T = keep ? Tn : -fabsf(p.T);
}

template <bool EXT>
__device__ __forceinline__ void write_pixel(const RenderArgs& a, const DevView& w, int x, int y, const FwdPixel& p) {
    const uint32_t ch = (uint32_t)w.W * (uint32_t)w.H;
    const uint32_t local = (uint32_t)y * (uint32_t)w.W + (uint32_t)x;
    const uint32_t pix = w.pix_base + local, img = 3u * w.pix_base + local;
    const float T = fabsf(p.T);
    a.image[img] = fmaf(T, a.st.bg[0], p.r);
    a.image[img + ch] = fmaf(T, a.st.bg[1], p.g);
    a.image[img + 2 * ch] = fmaf(T, a.st.bg[2], p.b);
    a.final_T[pix] = T;
    a.n_contrib[pix] = p.contrib;
    if (EXT) {
        if (a.out_depth) a.out_depth[pix] = p.d;
        if (a.out_alpha) a.out_alpha[pix] = 1.0f - T;
    }
}

// Forward of one 16x16 tile by one wave with 4 pixels per lane (one per 8x8
// quadrant): a staged splat's LDS reads serve 256 pixels; the wave leaves the
// tile once all its pixels have terminated.  sA, sB, sC: the wave's stage.
// EXT: also the extended channels (depth composited over zero, alpha = 1 - T).
template <bool COUNT, int B, bool EXT>
__device__ __forceinline__ void fwd_wave_tile(const RenderArgs& a, uint32_t t, float4* sA, float4* sB, float4* sC) {
    static_assert(B >= 1 && B <= 64, "one staged record per lane");
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const uint32_t lane = __lane_id();
    const int v = view_of_tile(a.cams, t);
    const DevView& w = a.cams.v[v];
    const uint32_t lt = t - w.tile_base;
    const uint32_t tx = lt % (uint32_t)w.tiles_x, ty = lt / (uint32_t)w.tiles_x;
    const uint2 rg = reinterpret_cast<const uint2*>(a.ranges)[t];
    const uint32_t r0 = rg.x, r1 = rg.y;

    const int x0 = (int)tx * 16 + (int)(lane & 7), y0 = (int)ty * 16 + (int)(lane >> 3);
    const float pxb = (float)x0 + 0.5f, pyb = (float)y0 + 0.5f;
    FwdPixel p[4];
    uint32_t listed[4], hit[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = x0 + (q & 1) * 8, y = y0 + (q >> 1) * 8;
        p[q] = FwdPixel{x < w.W && y < w.H ? 1.0f : -1.0f, 0.f, 0.f, 0.f, 0.f, 0u};
        listed[q] = hit[q] = 0;
    }
    // the next batch's records are loaded into registers while the current
    // batch is rendered from LDS
    float4 na = make_float4(0.f, 0.f, 0.f, 0.f), nb = na, nc = na;
    auto fetch = [&](uint32_t b) {
        const uint32_t pos = b + lane;
        if ((int)lane < B && pos < r1) {
            const float4* r = reinterpret_cast<const float4*>(a.rec + (size_t)a.val_sorted[pos] * GESR_REC_FLOATS);
            na = r[0];
            nb = r[1];
            nc = r[2];
        }
    };
    fetch(r0);
    uint32_t stop = r1;  // first list position not evaluated
    for (uint32_t base = r0; base < r1; base += B) {
        if (__ballot(fmaxf(fmaxf(p[0].T, p[1].T), fmaxf(p[2].T, p[3].T)) > 0.0f) == 0ull) {
            stop = base;
            break;
        }
        if ((int)lane < B && base + lane < r1) {
            sA[lane] = na;
            sB[lane] = make_float4(nb.x, nb.y, 0.5f * nb.z, nb.w);
            sC[lane] = nc;
        }
        wave_lds_fence();
        if (base + B < r1) fetch(base + B);
        const int cnt = (int)__builtin_amdgcn_readfirstlane(min<uint32_t>(B, r1 - base));
        uint32_t pos = in_vgpr(base - r0);
        for (int j = 0; j < cnt; ++j) {
            const float4 ra = sA[j];
            const float4 rb = sB[j];
            const float4 rc = sC[j];
            ++pos;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                Fragment f;
                const float qq = ges_q(ra, rb.x, pxb + (float)((q & 1) * 8), pyb + (float)((q >> 1) * 8), f);
                const bool on = p[q].T > 0.0f;
                if (COUNT) listed[q] += on ? 1u : 0u;
                // Beyond the alpha_min footprint or terminated.  Inside it alpha
                // almost never falls below alpha_min and a pixel terminates once:
                // both decisions are selects, one branch per quadrant.
                if (!((int)on & (int)!(qq > rb.w))) continue;
                ges_alpha(qq, rb.z, rb.y, nk, amax, f);
                const bool ok = !(f.alpha < st.alpha_min);
                if (COUNT) hit[q] += ok ? 1u : 0u;
                float al = f.alpha;
                if (__builtin_amdgcn_ballot_w64(!ok) != 0ull) {
                    al = ok ? al : 0.0f;
                    asm volatile("" : "+v"(al));
                }
                blend<EXT>(p[q], al, ok, rc, rc.w, pos, st.t_min);
            }
        }
        wave_lds_fence();
    }
    if (a.tile_work && lane == 0) a.tile_work[t] = stop - r0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = x0 + (q & 1) * 8, y = y0 + (q >> 1) * 8;
        if (x >= w.W || y >= w.H) continue;
        write_pixel<EXT>(a, w, x, y, p[q]);
        if (COUNT) {
            const uint32_t pix = w.pix_base + (uint32_t)y * (uint32_t)w.W + (uint32_t)x;
            a.n_listed[pix] = listed[q];
            a.n_hit[pix] = hit[q];
        }
    }
}

// Whether no pixel centre (u + dx, v + dy), dx in [dx0, dx1], dy in [dy0, dy1],
// can pass the footprint test q <= qmax of record (a, b).  Conservative: the
// ellipse is widened by 1% in q (the renderers' float32 q is off by at most
// u (12 + 8 s) relative, s = |L10| / L11; at s <= 4096 that and the rounding of
// the extents below stay under half of it), the ends by 1e-3 px, and anything
// not finite or more sheared keeps the record.  dx0.. are the renderers' own
// rounded differences.  Over the band of dy the ellipse's right end
// (-L10 dy + sqrt(Q - (L11 dy)^2)) / L00 is largest at its rightmost point
// clamped into the band (the left end mirrors it).
__device__ __forceinline__ bool quad_misses(const float4& a, const float4& b, float dx0, float dx1, float dy0,
                                            float dy1) {
    const float l00 = a.z, l10 = a.w, l11 = b.x;
    const float Q = b.w * 1.01f;
    const float sq = __builtin_amdgcn_sqrtf(Q);
    const float rr = __builtin_amdgcn_sqrtf(l10 * l10 + l11 * l11);
    const float il11 = hw_rcp(l11), il00 = hw_rcp(l00);
    const float ym = sq * il11 + 1e-3f;
    const float dyr = -(l10 * sq) * il11 * hw_rcp(rr);  // dy of the rightmost point
    const float lo = fmaxf(dy0, -ym), hi = fminf(dy1, ym);
    const float tr = fminf(fmaxf(dyr, lo), hi), tl = fminf(fmaxf(-dyr, lo), hi);
    const float wr = l11 * tr, wl = l11 * tl;
    const float xr = (__builtin_amdgcn_sqrtf(fmaxf(Q - wr * wr, 0.f)) - l10 * tr) * il00 + 1e-3f;
    const float xl = (-__builtin_amdgcn_sqrtf(fmaxf(Q - wl * wl, 0.f)) - l10 * tl) * il00 - 1e-3f;
    const bool sound = fabsf(l10) <= 4096.f * l11 && fabsf(dyr) < 1e30f && Q < 1e30f;
    return sound && (lo > hi || dx0 > xr || dx1 < xl);
}

// Forward of one 16x16 tile by the four waves of a workgroup, one 8x8 quadrant
// each (one pixel per lane, no barrier in the list loop).  A wave stages only
// the records that can reach its quadrant and takes them two at a time: their
// falloffs are independent chains, so a tile with a long list is bound by
// far shorter steps than with one wave per tile.  sa, sb, sc: the wave's stage of
// 65 records (an odd count is padded with a record that no pixel passes).
template <bool EXT>
__device__ __forceinline__ void fwd_quad_tile(const RenderArgs& a, uint32_t t, uint32_t wave, float4* sa, float4* sb,
                                              float4* sc, float* sz, uint32_t* s_stop) {
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, amin = st.alpha_min, tmin = st.t_min, nk = in_vgpr(st.neg_kappa_log2e);
    const uint32_t lane = __lane_id();
    const int v = view_of_tile(a.cams, t);
    const DevView& w = a.cams.v[v];
    const uint32_t lt = t - w.tile_base;
    const uint32_t tx = lt % (uint32_t)w.tiles_x, ty = lt / (uint32_t)w.tiles_x;
    const uint2 rg = reinterpret_cast<const uint2*>(a.ranges)[t];
    const uint32_t r0 = rg.x, r1 = rg.y;
    const int qx = (int)tx * 16 + (int)(wave & 1) * 8, qy = (int)ty * 16 + (int)(wave >> 1) * 8;
    const int x = qx + (int)(lane & 7), y = qy + (int)(lane >> 3);
    const bool inside = x < w.W && y < w.H;
    const float px = (float)x + 0.5f, py = (float)y + 0.5f;
    const float qx0 = (float)qx + 0.5f, qx1 = qx0 + 7.0f, qy0 = (float)qy + 0.5f, qy1 = qy0 + 7.0f;
    FwdPixel p{inside ? 1.0f : -1.0f, 0.f, 0.f, 0.f, 0.f, 0u};

    auto value_at = [&](uint32_t pos) { return pos < r1 ? a.val_sorted[pos] : 0u; };
    // a batch's records are loaded while the one before is rendered, its splat
    // ids while the one before that is
    uint32_t vi = value_at(r0 + lane), vi_n = value_at(r0 + 64 + lane);
    float4 na = make_float4(0.f, 0.f, 0.f, 0.f), nb = na, nc = na;
    auto fetch = [&](uint32_t pos, uint32_t id) {
        if (pos < r1) {
            const float4* r = reinterpret_cast<const float4*>(a.rec + (size_t)id * GESR_REC_FLOATS);
            na = r[0];
            nb = r[1];
            nc = r[2];
        }
    };
    fetch(r0 + lane, vi);
    uint32_t stop = r1;  // first list position not evaluated
    for (uint32_t base = r0; base < r1; base += 64) {
        if (__ballot(p.T > 0.0f) == 0ull) {
            stop = base;
            break;
        }
        const bool live = base + lane < r1 && !quad_misses(na, nb, qx0 - na.x, qx1 - na.x, qy0 - na.y, qy1 - na.y);
        const uint64_t mask = __ballot(live);
        const uint32_t cnt = (uint32_t)__popcll(mask);
        if (live) {
            const uint32_t k = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            sa[k] = na;
            sb[k] = make_float4(nb.x, nb.y, 0.5f * nb.z, nb.w);
            sc[k] = make_float4(nc.x, nc.y, nc.z, __uint_as_float(base + lane + 1u - r0));
            if (EXT) sz[k] = nc.w;
        }
        if (lane == 0) {
            sa[cnt] = sc[cnt] = make_float4(0.f, 0.f, 0.f, 0.f);
            sb[cnt] = make_float4(0.f, 0.f, 0.f, -1.f);
            if (EXT) sz[cnt] = 0.f;
        }
        wave_lds_fence();
        vi = vi_n;
        fetch(base + 64 + lane, vi);
        vi_n = value_at(base + 128 + lane);
        for (uint32_t j = 0; j < cnt; j += 2) {
            bool ok[2];
            float al[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                Fragment f;
                const float4 rb = sb[j + u];
                const float q = ges_q(sa[j + u], rb.x, px, py, f);
                ges_alpha(q, rb.z, rb.y, nk, amax, f);
                ok[u] = (int)(q <= rb.w) & (int)!(f.alpha < amin);
                al[u] = ok[u] ? f.alpha : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 rc = sc[j + u];
                blend<EXT>(p, al[u], ok[u], rc, EXT ? sz[j + u] : 0.f, __float_as_uint(rc.w), tmin);
            }
        }
        wave_lds_fence();
    }
    if (a.tile_work) {
        if (lane == 0) s_stop[wave] = stop;
        __syncthreads();
        if (threadIdx.x == 0) a.tile_work[t] = max(max(s_stop[0], s_stop[1]), max(s_stop[2], s_stop[3])) - r0;
    }
    if (inside) write_pixel<EXT>(a, w, x, y, p);
}

// Forward of 16x16 tiles.  The first a.n_split workgroups take one tile each
// (fwd_quad_tile), the others four (a tile per wave, fwd_wave_tile).  The two give
// the same pixels bit for bit.
template <bool EXT>
__global__ __launch_bounds__(256) void k_render_fwd16(RenderArgs a) {
    __shared__ float4 s_a[4][65], s_b[4][65], s_c[4][65];
    __shared__ float s_z[EXT ? 4 : 1][65];
    __shared__ uint32_t s_stop[4];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x < a.n_split) {
        fwd_quad_tile<EXT>(a, a.worklist[blockIdx.x], wave, s_a[wave], s_b[wave], s_c[wave], s_z[EXT ? wave : 0], s_stop);
        return;
    }
    const uint32_t item = a.n_split + 4u * (blockIdx.x - a.n_split) + wave;
    if (item < a.n_items) fwd_wave_tile<false, 64, EXT>(a, a.worklist[item], s_a[wave], s_b[wave], s_c[wave]);
}

// The counting variant: one wave (workgroup) per tile.
template <int B, bool EXT>
__global__ __launch_bounds__(64) void k_render_fwd16_counts(RenderArgs a) {
    __shared__ float4 s_a[B], s_b[B], s_c[B];
    fwd_wave_tile<true, B, EXT>(a, a.worklist[blockIdx.x], s_a, s_b, s_c);
}

// The 64-bit value of lane l (wave-uniform).
__device__ __forceinline__ uint64_t read_lane(uint64_t x, int l) {
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)x, l);
    return (uint64_t)hi << 32 | lo;
}

// Stage of one batch of records of a 16x16 tile's adjoint, and the batch's sums
// (column 10: dz, extended channels).
constexpr int kBwdBatch = 64;
template <bool EXT>
struct BwdStage {
    float4 a[kBwdBatch], b[kBwdBatch], c[kBwdBatch];
    uint32_t inst[kBwdBatch];
    float red[kBwdBatch][GESR_PARTIAL_FLOATS + 1];
    float z[EXT ? kBwdBatch : 1];
};

// One record on its way to the stage: the loads are issued by `load`, what is derived
// from them waits until `store`.
template <bool EXT>
struct BwdRecord {
    float4 a, b, c, r;
    uint32_t base;
    __device__ __forceinline__ void load(const RenderArgs& A, uint32_t vi) {
        const float4* p = reinterpret_cast<const float4*>(A.rec + (size_t)vi * GESR_REC_FLOATS);
        a = p[0];
        b = p[1];
        c = p[2];
        r = p[3];
        base = A.inst_base[vi];
    }
    __device__ __forceinline__ void store(const RenderArgs& A, BwdStage<EXT>& s, uint32_t k, uint32_t tx,
                                          uint32_t ty) const {
        s.a[k] = a;
        s.b[k] = make_float4(b.x, b.y, 0.5f * b.z, b.w);
        s.c[k] = make_float4(c.x, c.y, c.z, -A.st.kappa * b.z);
        s.inst[k] = instance_index(A, make_uint2(__float_as_uint(r.x), __float_as_uint(r.y)), base, tx, ty);
        if (EXT) s.z[k] = c.w;
    }
};

template <bool EXT>
__device__ __forceinline__ void write_batch(const RenderArgs& a, BwdStage<EXT>& s, uint32_t lane, uint32_t cnt) {
    constexpr int NP = GESR_PARTIAL_FLOATS;
    if (lane >= cnt || s.inst[lane] == kNoInstance) return;
    float v[NP + 1];
#pragma unroll
    for (int k = 0; k <= NP; ++k) v[k] = EXT || k < NP ? s.red[lane][k] : 0.0f;
    splat_partial(v, s.a[lane], s.b[lane]);
    write_partial<EXT>(a, s.inst[lane], v);
}

// Sums of a record over the wave's lanes into its row of the batch.
template <bool EXT>
__device__ __forceinline__ void reduce_record(BwdStage<EXT>& s, uint32_t j, const float (&gr)[GESR_PARTIAL_FLOATS],
                                              float gz, uint32_t lane, int slot) {
    static_assert(GESR_PARTIAL_FLOATS == 10, "wave_sum10 reduces ten values");
    const float tot = wave_sum10(gr, lane);
    if (slot < GESR_PARTIAL_FLOATS) s.red[j][slot] = tot;
    if (EXT) {
        const float tz = wave_sum(gz);
        if (lane == 0) s.red[j][GESR_PARTIAL_FLOATS] = tz;
    }
}

struct TilePlace {
    const DevView* w;
    uint32_t tx, ty, ch, r0;
};
__device__ __forceinline__ TilePlace place_tile(const RenderArgs& a, uint32_t t) {
    TilePlace p;
    p.w = &a.cams.v[view_of_tile(a.cams, t)];
    const uint32_t lt = t - p.w->tile_base;
    p.tx = lt % (uint32_t)p.w->tiles_x;
    p.ty = lt / (uint32_t)p.w->tiles_x;
    p.ch = (uint32_t)p.w->W * (uint32_t)p.w->H;
    p.r0 = a.ranges[2 * (size_t)t];
    return p;
}

// Adjoint of one 16x16 tile by one wave: lane l owns pixel (l & 7, l >> 3) of each
// 8x8 quadrant (4 pixels per lane), so a staged splat's LDS reads and its
// 10-value wave reduction serve 256 pixels, and no cross-wave reduction or
// workgroup barrier is needed.  EXT: the extended channels' upstream gradients
// too (depth and opacity as colour channels over a zero background; the depth
// term dz is the eleventh partial value).
template <bool EXT>
__device__ __forceinline__ void bwd_wave_tile(const RenderArgs& a, uint32_t t, BwdStage<EXT>& s) {
    constexpr int NP = GESR_PARTIAL_FLOATS;
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const float c2 = -0.5f * kLn2 * st.kappa;
    const uint32_t lane = __lane_id();
    const TilePlace tp = place_tile(a, t);
    const uint32_t r0 = tp.r0;

    // pixel centres: quadrant q adds (q & 1) * 8 and (q >> 1) * 8 to the lane's base
    const float pxb = (float)(tp.tx * 16 + (lane & 7)) + 0.5f, pyb = (float)(tp.ty * 16 + (lane >> 3)) + 0.5f;
    PixelAdjoint pa[4];
    PixelUp up[4];
    uint32_t nc[4];
    uint32_t mymax = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = (int)tp.tx * 16 + (q & 1) * 8 + (int)(lane & 7);
        const int y = (int)tp.ty * 16 + (q >> 1) * 8 + (int)(lane >> 3);
        pa[q] = behind_all(st, 0.f);
        up[q] = PixelUp{};
        nc[q] = 0;
        if (x < tp.w->W && y < tp.w->H) {
            const uint32_t local = (uint32_t)y * (uint32_t)tp.w->W + (uint32_t)x;
            const uint32_t pix = tp.w->pix_base + local;
            pa[q].T = a.final_T[pix];
            nc[q] = a.n_contrib[pix];
            up[q] = load_up<EXT>(a, pix, 3u * tp.w->pix_base + local, tp.ch);
        }
        mymax = max(mymax, nc[q]);
    }
    const uint32_t maxnc = __builtin_amdgcn_readfirstlane(wave_max_u32(mymax));  // uniform: scalar loop control
    const uint32_t end = r0 + maxnc;  // positions >= end contributed to no pixel
    const int slot = lane < 16 ? wave_sum10_slot(lane) : NP;  // value this lane writes after a reduction

    for (uint32_t hi = end; hi > r0;) {
        const uint32_t cnt = min(hi - r0, (uint32_t)kBwdBatch);
        if (lane < cnt) {
            BwdRecord<EXT> r;
            r.load(a, a.val_sorted[hi - 1u - lane]);
            r.store(a, s, lane, tp.tx, tp.ty);
        }
        wave_lds_fence();
        for (uint32_t j = 0; j < cnt; ++j) {
            const uint32_t prel = hi - 1u - j - r0;  // 0-based list position
            const float4 ra = s.a[j];
            const float4 rb = s.b[j];
            const float4 rc = s.c[j];
            const float z = EXT ? s.z[j] : 0.0f;
            float gr[NP], gz = 0.0f;
#pragma unroll
            for (int k = 0; k < NP; k += 2) opaque_zero2(gr[k], gr[k + 1]);
            if (EXT) gz = opaque_zero();
            bool act = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                Fragment f;
                const float qq = ges_q(ra, rb.x, pxb + (float)((q & 1) * 8), pyb + (float)((q >> 1) * 8), f);
                if (prel >= nc[q] || qq > rb.w) continue;  // behind the pixel's last or beyond the footprint
                // Inside the footprint alpha almost never falls below alpha_min,
                // the alpha cap and a centred pixel are rarer still: those
                // decisions are selects or zero products (a zeroed term leaves the
                // sums as they are), so the wave takes one branch per quadrant.
                ges_alpha(qq, rb.z, rb.y, nk, amax, f);
                act = true;
                float aT, dl;
                pixel_step<EXT, true>(f, true, rc, z, st, up[q], pa[q], aT, dl);
                add_terms<EXT>(fragment_terms(f, rc.w, aT, dl), f.dx, f.dy, c2, up[q], gr, gz);
            }
            if (__ballot(act) != 0ull) reduce_record(s, j, gr, gz, lane, slot);
            else if ((int)lane < (EXT ? NP + 1 : NP)) s.red[j][lane] = 0.f;
        }
        wave_lds_fence();
        write_batch(a, s, lane, cnt);
        wave_lds_fence();
        hi -= cnt;
    }
}

// The fragments' terms of a round of R records.
template <uint32_t R>
struct BwdTerms {
    float4 v0[R][4][64];  // [record][quadrant][lane]: aT, dl, G, xl
    float2 v1[R][4][64];  // tq, wq
};

// The batch's records that can reach the quadrant, a bit each: `left` list positions are
// left, the quadrant's pixels composited the first wmax of the list.
template <bool EXT>
__device__ __forceinline__ uint64_t quad_records(const BwdStage<EXT>& s, uint32_t lane, uint32_t left, uint32_t wmax,
                                                 float qx, float qy) {
    bool can = false;
    if (lane < left && left - 1u - lane < wmax) {
        const float4 la = s.a[lane];
        can = !quad_misses(la, s.b[lane], qx - la.x, (qx + 7.0f) - la.x, qy - la.y, (qy + 7.0f) - la.y);
    }
    return __ballot(can);
}

// Phase 1: the quadrant's pixel (px, py) past the round's records b + k, k the set bits of
// m; `left` list positions were left at the batch's first record, nc of them are the pixel's.
template <bool EXT, uint32_t R>
__device__ __forceinline__ void quad_terms(const DevSettings& st, const BwdStage<EXT>& s, uint32_t b, uint32_t m,
                                           uint32_t left, uint32_t nc, float px, float py, float amax, float nk,
                                           const PixelUp& mine, PixelAdjoint& pa, uint32_t quad, uint32_t lane,
                                           BwdTerms<R>& terms) {
    constexpr uint32_t GRP = 2;  // records side by side
    const uint32_t top = left - 1u - b;
    while (m != 0u) {
        uint32_t k[GRP];
        bool have[GRP];
#pragma unroll
        for (uint32_t u = 0; u < GRP; ++u) {  // past the last record: that one again, off
            have[u] = m != 0u;
            k[u] = have[u] ? (uint32_t)__builtin_ctz(m) : k[u > 0 ? u - 1 : 0];
            m = have[u] ? m & (m - 1) : 0u;
        }
        Fragment f[GRP];
        bool on[GRP];
#pragma unroll
        for (uint32_t u = 0; u < GRP; ++u) {
            const float4 rb = s.b[b + k[u]];
            const float qq = ges_q(s.a[b + k[u]], rb.x, px, py, f[u]);
            on[u] = (int)(top - k[u] < nc) & (int)!(qq > rb.w) & (int)have[u];
            // q = 1 where the fragment is not the pixel's: its terms are exact zeros
            ges_alpha(on[u] ? qq : 1.0f, rb.z, rb.y, nk, amax, f[u]);
        }
#pragma unroll
        for (uint32_t u = 0; u < GRP; ++u) {
            const float4 rc = s.c[b + k[u]];
            float aT, dl;
            pixel_step<EXT, false>(f[u], on[u], rc, EXT ? s.z[b + k[u]] : 0.0f, st, mine, pa, aT, dl);
            if (have[u]) {
                const FragmentTerms v = fragment_terms(f[u], rc.w, aT, dl);
                terms.v0[k[u]][quad][lane] = make_float4(v.aT, v.dl, v.G, v.xl);
                terms.v1[k[u]][quad][lane] = make_float2(v.tq, v.wq);
            }
        }
    }
}

// Phase 2: the sums of the batch's record j, the round's k-th, over the whole tile.
template <bool EXT, uint32_t R>
__device__ __forceinline__ void tile_sums(BwdStage<EXT>& s, const BwdTerms<R>& terms, uint32_t j, uint32_t k,
                                          const uint64_t (&live_of)[4], float pxb, float pyb, float c2,
                                          const PixelUp (&up)[4], uint32_t lane, int slot) {
    constexpr int NP = GESR_PARTIAL_FLOATS;
    if (((live_of[0] | live_of[1] | live_of[2] | live_of[3]) >> j & 1u) == 0u) {
        if ((int)lane < (EXT ? NP + 1 : NP)) s.red[j][lane] = 0.f;
        return;
    }
    const float2 uv = make_float2(s.a[j].x, s.a[j].y);
    float gr[NP], gz = 0.0f;
    // all reads in flight together (a quadrant without the record holds stale terms: not added)
    float4 v0[4];
    float2 v1[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v0[q] = terms.v0[k][q][lane];
        v1[q] = terms.v1[k][q][lane];
    }
#pragma unroll
    for (int i = 0; i < NP; i += 2) opaque_zero2(gr[i], gr[i + 1]);
    if (EXT) gz = opaque_zero();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (!(live_of[q] >> j & 1u)) continue;
        add_terms<EXT>(FragmentTerms{v0[q].x, v0[q].y, v0[q].z, v0[q].w, v1[q].x, v1[q].y},
                       (pxb + (float)((q & 1) * 8)) - uv.x, (pyb + (float)((q >> 1) * 8)) - uv.y, c2, up[q], gr, gz);
    }
    reduce_record(s, j, gr, gz, lane, slot);
}

// Adjoint of one 16x16 tile by the four waves of a workgroup, with the sums of
// bwd_wave_tile bit for bit.  Rounds of four list positions in two phases.  Phase 1:
// wave q takes its quadrant's pixels (one per lane) past the round's records that
// can reach it and leaves each fragment's terms in LDS; the falloffs of two records
// are independent chains, only T and the colour behind are serial.  Phase 2: wave w
// adds the w-th record's terms over the whole tile (4 pixels per lane, quadrants in
// order) and reduces them.
// There a pixel that the record did not reach adds zero times its upstream gradient, so
// a tile with one that is not finite is not taken (false): one wave, which visits a
// record's own pixels only, has to.
template <bool EXT>
struct BwdSplit {
    BwdStage<EXT> s;
    BwdTerms<4> terms;
    uint64_t live[4];
    uint32_t maxnc[4];
};

template <bool EXT>
__device__ __forceinline__ bool bwd_split_tile(const RenderArgs& a, uint32_t t, uint32_t wave, BwdSplit<EXT>& S) {
    constexpr int NP = GESR_PARTIAL_FLOATS;
    constexpr uint32_t R = 4;  // records per round
    BwdStage<EXT>& s = S.s;
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const float c2 = -0.5f * kLn2 * st.kappa;
    const uint32_t lane = __lane_id();
    const TilePlace tp = place_tile(a, t);
    const uint32_t r0 = tp.r0;
    const float pxb = (float)(tp.tx * 16 + (lane & 7)) + 0.5f, pyb = (float)(tp.ty * 16 + (lane >> 3)) + 0.5f;
    const float qx = (float)(tp.tx * 16 + (wave & 1) * 8) + 0.5f, qy = (float)(tp.ty * 16 + (wave >> 1) * 8) + 0.5f;
    const float px = pxb + (float)((wave & 1) * 8), py = pyb + (float)((wave >> 1) * 8);
    PixelUp up[4], mine{};
    PixelAdjoint pa = behind_all(st, 0.f);
    uint32_t nc = 0;
    bool odd = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = (int)tp.tx * 16 + (q & 1) * 8 + (int)(lane & 7);
        const int y = (int)tp.ty * 16 + (q >> 1) * 8 + (int)(lane >> 3);
        up[q] = PixelUp{};
        if (x < tp.w->W && y < tp.w->H) {
            const uint32_t local = (uint32_t)y * (uint32_t)tp.w->W + (uint32_t)x;
            const uint32_t pix = tp.w->pix_base + local;
            up[q] = load_up<EXT>(a, pix, 3u * tp.w->pix_base + local, tp.ch);
            if (q == (int)wave) {
                pa.T = a.final_T[pix];
                nc = a.n_contrib[pix];
                mine = up[q];
            }
        }
        odd |= any_odd<EXT>(up[q]);
    }
    if (odd) return false;  // every wave's finding
    const uint32_t wmax = __builtin_amdgcn_readfirstlane(wave_max_u32(nc));  // this quadrant's deepest position
    if (lane == 0) S.maxnc[wave] = wmax;
    __syncthreads();
    const uint32_t maxnc = __builtin_amdgcn_readfirstlane(max(max(S.maxnc[0], S.maxnc[1]), max(S.maxnc[2], S.maxnc[3])));
    const int slot = lane < 16 ? wave_sum10_slot(lane) : NP;

    // the first wave stages: a batch's records are loaded while the one before is
    // taken, its splat ids while the one before that is
    BwdRecord<EXT> r;
    uint32_t hi = r0 + maxnc, vi = 0;
    auto value_at = [&](uint32_t back) { return back + lane < hi - r0 ? a.val_sorted[hi - 1u - back - lane] : 0u; };
    if (wave == 0) {
        vi = value_at(0);
        if (lane < hi - r0) r.load(a, vi);
        vi = value_at(kBwdBatch);
    }
    while (hi > r0) {
        const uint32_t cnt = min(hi - r0, (uint32_t)kBwdBatch);
        if (wave == 0 && lane < cnt) r.store(a, s, lane, tp.tx, tp.ty);
        __syncthreads();
        if (wave == 0) {
            if (kBwdBatch + lane < hi - r0) r.load(a, vi);
            vi = value_at(2 * kBwdBatch);
        }
        const uint64_t live = quad_records(s, lane, hi - r0, wmax, qx, qy);
        if (lane == 0) S.live[wave] = live;
        __syncthreads();
        const uint64_t own = S.live[lane & 3];
        const uint64_t live_of[4] = {read_lane(own, 0), read_lane(own, 1), read_lane(own, 2), read_lane(own, 3)};
        for (uint32_t b = 0; b < cnt; b += R) {
            quad_terms<EXT, R>(st, s, b, (uint32_t)(live >> b) & ((1u << R) - 1u), hi - r0, nc, px, py, amax, nk, mine, pa,
                               wave, lane, S.terms);
            __syncthreads();
            if (b + wave < cnt) tile_sums<EXT, R>(s, S.terms, b + wave, wave, live_of, pxb, pyb, c2, up, lane, slot);
            __syncthreads();
        }
        if (wave == 0) write_batch(a, s, lane, cnt);
        hi -= cnt;
    }
    return true;
}

// The same tile by eight waves: the first four do phase 1 of a round while the other
// four do phase 2 of the round before (terms, records and sums are held twice), so a
// round lasts as long as the longer phase.  Bound by the phases' serial chains: 92 us
// on 64 tiles (2,000 splats, 128x128) with rounds of eight, 112 with rounds of four, 147
// with four waves and the phases in turn, 124 with the falloffs of four records side by
// side (most are off).
template <bool EXT, uint32_t R>
struct BwdPipe {
    BwdStage<EXT> s[2];
    BwdTerms<R> terms[2];  // of even and odd rounds
    uint64_t live[2][4];
    uint32_t maxnc[4];
    bool odd;
};

template <bool EXT, uint32_t R>  // R records per round
__global__ __launch_bounds__(512) void k_render_bwd16_pipe(RenderArgs a) {
    constexpr int NP = GESR_PARTIAL_FLOATS;
    constexpr uint32_t kRounds = kBwdBatch / R;  // rounds of a full batch
    __shared__ BwdPipe<EXT, R> S;
    const uint32_t t = a.worklist[blockIdx.x];
    const uint32_t w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = w8 & 3u;
    const bool first = w8 < 4u;  // phase 1
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const float c2 = -0.5f * kLn2 * st.kappa;
    const uint32_t lane = __lane_id();
    const TilePlace tp = place_tile(a, t);
    const uint32_t r0 = tp.r0;
    const float pxb = (float)(tp.tx * 16 + (lane & 7)) + 0.5f, pyb = (float)(tp.ty * 16 + (lane >> 3)) + 0.5f;
    const float qx = (float)(tp.tx * 16 + (wave & 1) * 8) + 0.5f, qy = (float)(tp.ty * 16 + (wave >> 1) * 8) + 0.5f;
    const float px = pxb + (float)((wave & 1) * 8), py = pyb + (float)((wave >> 1) * 8);
    PixelUp up[4], mine{};
    PixelAdjoint pa = behind_all(st, 0.f);
    uint32_t nc = 0;
    bool odd = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = (int)tp.tx * 16 + (q & 1) * 8 + (int)(lane & 7);
        const int y = (int)tp.ty * 16 + (q >> 1) * 8 + (int)(lane >> 3);
        up[q] = PixelUp{};
        if (x < tp.w->W && y < tp.w->H && (!first || q == (int)wave)) {
            const uint32_t local = (uint32_t)y * (uint32_t)tp.w->W + (uint32_t)x;
            const uint32_t pix = tp.w->pix_base + local;
            up[q] = load_up<EXT>(a, pix, 3u * tp.w->pix_base + local, tp.ch);
            if (first) {
                pa.T = a.final_T[pix];
                nc = a.n_contrib[pix];
                mine = up[q];
            }
        }
        odd |= any_odd<EXT>(up[q]);
    }
    const uint32_t wmax = __builtin_amdgcn_readfirstlane(wave_max_u32(nc));  // this quadrant's deepest position
    if (first && lane == 0) S.maxnc[wave] = wmax;
    if (w8 == 4 && lane == 0) S.odd = odd;  // of the whole tile
    __syncthreads();
    if (S.odd) {  // see BwdSplit
        if (w8 == 0) bwd_wave_tile<EXT>(a, t, S.s[0]);
        return;
    }
    const uint32_t total = __builtin_amdgcn_readfirstlane(max(max(S.maxnc[0], S.maxnc[1]), max(S.maxnc[2], S.maxnc[3])));
    const int slot = lane < 16 ? wave_sum10_slot(lane) : NP;
    const uint32_t top = r0 + total;  // positions top - 1 .. r0, batch k from top - 64 k

    // the first wave stages: a batch's records are stored while the one before is
    // taken, loaded while the one before that is, its splat ids before that
    BwdRecord<EXT> r;
    uint32_t vi = 0;
    auto value_at = [&](uint32_t back) { return back + lane < total ? a.val_sorted[top - 1u - back - lane] : 0u; };
    if (w8 == 0) {
        vi = value_at(0);
        if (lane < total) {
            r.load(a, vi);
            r.store(a, S.s[0], lane, tp.tx, tp.ty);
        }
        vi = value_at(kBwdBatch);
        if (kBwdBatch + lane < total) r.load(a, vi);
        vi = value_at(2 * kBwdBatch);
    }
    __syncthreads();
    const uint32_t rounds = (total + R - 1) / R;
    uint64_t live = 0, live_of[4] = {0, 0, 0, 0};
    for (uint32_t i = 0; i <= rounds; ++i) {
        if (first) {
            const uint32_t k = i / kRounds, b = i % kRounds * R;
            BwdStage<EXT>& s = S.s[k & 1];
            const uint32_t hi = top - k * kBwdBatch;  // not used past the last round
            if (i < rounds) {
                if (b == 0) {
                    live = quad_records(s, lane, hi - r0, wmax, qx, qy);
                    if (lane == 0) S.live[k & 1][wave] = live;
                }
                quad_terms<EXT, R>(st, s, b, (uint32_t)(live >> b) & ((1u << R) - 1u), hi - r0, nc, px, py, amax, nk, mine,
                                   pa, wave, lane, S.terms[i & 1]);
            }
            // the stage's last use, by batch k - 1, ended with the step before
            if (w8 == 0 && b == 2u * R && (k + 1u) * kBwdBatch < total) {
                if ((k + 1u) * kBwdBatch + lane < total) r.store(a, S.s[(k + 1u) & 1u], lane, tp.tx, tp.ty);
                if ((k + 2u) * kBwdBatch + lane < total) r.load(a, vi);
                vi = value_at((k + 3u) * kBwdBatch);
            }
        } else {
            if (i > 0u) {
                const uint32_t p = i - 1u, k = p / kRounds, b = p % kRounds * R;
                BwdStage<EXT>& s = S.s[k & 1];
                if (b == 0) {
                    const uint64_t own = S.live[k & 1][lane & 3];
#pragma unroll
                    for (int q = 0; q < 4; ++q) live_of[q] = read_lane(own, q);
                }
#pragma unroll 1
                for (uint32_t c = wave; c < R; c += 4u)
                    if (k * kBwdBatch + b + c < total)
                        tile_sums<EXT, R>(s, S.terms[p & 1], b + c, c, live_of, pxb, pyb, c2, up, lane, slot);
            }
            // batch k - 1's last round was summed in the step before
            if (w8 == 4 && i % kRounds == 1u && i > kRounds) write_batch(a, S.s[(i / kRounds - 1u) & 1u], lane, kBwdBatch);
        }
        __syncthreads();
    }
    if (w8 == 4 && rounds != 0u) {
        const uint32_t k = (rounds - 1u) / kRounds;
        write_batch(a, S.s[k & 1], lane, total - k * kBwdBatch);
    }
}

// Adjoint of 16x16 tiles: the first a.n_split workgroups take one tile each, the
// others four (a tile per wave).
template <bool EXT>
__global__ __launch_bounds__(256, EXT ? 4 : 5) void k_render_bwd16(RenderArgs a) {
    __shared__ union {
        BwdStage<EXT> wave[4];
        BwdSplit<EXT> split;
    } S;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t item = a.n_split + 4u * (blockIdx.x - a.n_split) + wave;
    if (blockIdx.x < a.n_split) {
        if (bwd_split_tile<EXT>(a, a.worklist[blockIdx.x], wave, S.split) || wave != 0) return;
        item = blockIdx.x;
    }
    if (item < a.n_items) bwd_wave_tile<EXT>(a, a.worklist[item], S.wave[wave]);
}

// A workgroup of one wave per tile.
template <bool EXT>
__global__ __launch_bounds__(64) void k_render_bwd16_wave(RenderArgs a) {
    __shared__ BwdStage<EXT> S;
    bwd_wave_tile<EXT>(a, a.worklist[blockIdx.x], S);
}

template <int TW, int TH>
hipError_t fwd_shape(const RenderArgs& a, bool counts, hipStream_t s) {
    if (counts)
        hipLaunchKernelGGL((k_render_fwd<TW, TH, true>), dim3(a.n_items), dim3(TW * TH), 0, s, a);
    else
        hipLaunchKernelGGL((k_render_fwd<TW, TH, false>), dim3(a.n_items), dim3(TW * TH), 0, s, a);
    return hipGetLastError();
}

template <int TW, int TH, int BATCH>
hipError_t bwd_shape(const RenderArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((k_render_bwd<TW, TH, BATCH>), dim3(a.n_items), dim3(TW * TH), 0, s, a);
    return hipGetLastError();
}

// Leading worklist tiles (the ones with most work) that the 16x16 forward takes
// with four waves each.  Up to 8,192 tiles all of them: with a wave per tile the
// chip's 8,192 wave slots would be filled once or less and the kernel would last as
// long as its longest list (one wave takes 220 ns per list position): 200 -> 89 us
// on 3,024 tiles (100k splats, 1008x756), 145 -> 31 us on 64 tiles, 290 -> 172 us
// on 8,487.  Above that the first 1,024, which shortens the longest lists: 1,385 ->
// 810 us on 24,842 tiles of views at 1/8 .. 1 of 1600x1064 (its longest list, 6,208
// positions against 300 on average, took all of the former time), 880 -> 837 us
// on 33,948 and unchanged on 130,560 even tiles; with four waves for all tiles these
// take 944, 991 and (2,530 ->) 3,080 us, because a quadrant wave reads every record
// from LDS for 64 pixels instead of 256.
uint32_t fwd_split_tiles(uint32_t n_items) { return n_items <= 8192u ? n_items : 1024u; }

// The 16x16 adjoint's tiles with eight waves each: all of them up to 2,048, where four
// would leave SIMDs idle or with one serial chain each (147 -> 92 us on 64 tiles, 236
// -> 174 on 1,024, 214 -> 207 on 1,936; 2,500 tiles would take 262 us instead of 234,
// 3,024 321 instead of 231).
// Rounds of eight records, half the barriers for twice the LDS and so one workgroup on
// a CU, pay up to 512 tiles (112 -> 92 us on 64, 190 -> 161 on 256, 109 -> 93 on 484;
// 179 -> 197 on 1,024).
// With four waves each: all of them up to 5,500, where one-wave tiles would fill the
// chip's wave slots about once and the kernel would last as long as its longest list
// (one wave takes 300 ns per list position): 360 -> 218 us on 3,024; 198 -> 134 on 4,347,
// 196 -> 162 on 5,292; 185 -> 186 on 5,922, 194 -> 202 on 6,700; up to 4,096 where one
// view has four times another's pixels and the longest lists are few (5,326 tiles of
// views at 1/8 .. 1 of 1468x334: 1,286 us, 1,238 with the worklist's first 256).
// Beyond, those 256 as long as another tile does not hide the longest lists; the others
// of a workgroup's four waves then take a tile each, and free their slots together,
// which costs 2 to 5% on even lists (with the channels 4 to 7%):
//  - Up to 32,768 tiles: 11,442 tiles of views at 1/8 .. 3/4 of 1600x1064 286 us and 693
//    (one-wave workgroups 535, 1,160), 24,842 at 1/8 .. 1 469 and 655 (565, 1,118); even
//    views 9,500 tiles 312 (316), 15,200 of 400x300 349 (376) and of 800x600 453 (440),
//    20,100 572 (562), 30,400 842 (809).  Above, 33,948 tiles take 1,890 us and 130,560
//    5.77 ms, one-wave workgroups 1,790 and 5.55.
//  - With the channels up to 28,672 where one view has four times another's pixels: the
//    splats share fewer tiles in the smaller one, so its lists are longer by that factor,
//    and one of them sets the end (24,842 tiles 608 and 860 us, 667 and 1,344; 31,553 812
//    and 1,097, 756 and 1,030).  Views of nearer resolution have no such lists: up to
//    12,288 tiles (9,500 404 us, 467; 10,332 364, 377; 13,400 463, 443; 20,100 720, 681;
//    30,400 1,097, 1,026).
constexpr uint32_t kBwdPipeMax = 2048u, kBwdPipe8Max = 512u;
constexpr uint32_t kBwdSplitAllMax = 5500u, kBwdSplitAllSkewMax = 4096u, kBwdSplit = 256u;
constexpr uint32_t kBwdMixedMax = 32768u, kBwdMixedExtMax = 12288u, kBwdMixedExtSkewMax = 28672u;

bool views_skewed(const DevCams& c) {
    uint64_t lo = ~0ull, hi = 0;
    for (int v = 0; v < c.V; ++v) {
        const uint64_t pixels = (uint64_t)c.v[v].W * (uint64_t)c.v[v].H;
        lo = pixels < lo ? pixels : lo;
        hi = pixels > hi ? pixels : hi;
    }
    return hi >= 4u * lo;
}

}  // namespace

hipError_t launch_render_fwd(const RenderArgs& a, int tw, int th, bool counts, hipStream_t s) {
    if (a.n_items == 0) return hipSuccess;
    if (tw == 16 && th == 16) {
        if (a.st.variant == 1 && counts) {
            hipLaunchKernelGGL((k_render_fwd<16, 16, true>), dim3(a.n_items), dim3(256), 0, s, a);
            return hipGetLastError();
        }
        const bool small = a.batch == 32, ext = a.out_depth || a.out_alpha;
        if (counts) {
            const dim3 grid(a.n_items), block(64);
            if (ext) {
                if (small) hipLaunchKernelGGL((k_render_fwd16_counts<32, true>), grid, block, 0, s, a);
                else hipLaunchKernelGGL((k_render_fwd16_counts<64, true>), grid, block, 0, s, a);
            } else {
                if (small) hipLaunchKernelGGL((k_render_fwd16_counts<32, false>), grid, block, 0, s, a);
                else hipLaunchKernelGGL((k_render_fwd16_counts<64, false>), grid, block, 0, s, a);
            }
            return hipGetLastError();
        }
        RenderArgs b = a;
        b.n_split = a.st.variant == 1 ? a.n_items : fwd_split_tiles(a.n_items);
        const dim3 grid(b.n_split + (a.n_items - b.n_split + 3) / 4), block(256);
        if (ext) hipLaunchKernelGGL((k_render_fwd16<true>), grid, block, 0, s, b);
        else hipLaunchKernelGGL((k_render_fwd16<false>), grid, block, 0, s, b);
        return hipGetLastError();
    }
    if (tw == 8 && th == 8) return fwd_shape<8, 8>(a, counts, s);
    if (tw == 32 && th == 16) return fwd_shape<32, 16>(a, counts, s);
    if (tw == 32 && th == 32) return fwd_shape<32, 32>(a, counts, s);
    return hipErrorInvalidValue;
}

hipError_t launch_render_bwd(const RenderArgs& a, int tw, int th, int batch, hipStream_t s) {
    if (a.n_items == 0) return hipSuccess;
    if (tw == 16 && th == 16) {
        if (a.st.variant == 1)  // one workgroup of 4 waves per tile
            return batch >= 128 ? bwd_shape<16, 16, 128>(a, s) : bwd_shape<16, 16, 64>(a, s);
        const bool ext = a.dL_ddepth || a.dL_dalpha;
        if (a.n_items <= kBwdPipeMax) {
            const dim3 grid(a.n_items), block(512);
            if (a.n_items <= kBwdPipe8Max) {
                if (ext) hipLaunchKernelGGL((k_render_bwd16_pipe<true, 8>), grid, block, 0, s, a);
                else hipLaunchKernelGGL((k_render_bwd16_pipe<false, 8>), grid, block, 0, s, a);
            } else {
                if (ext) hipLaunchKernelGGL((k_render_bwd16_pipe<true, 4>), grid, block, 0, s, a);
                else hipLaunchKernelGGL((k_render_bwd16_pipe<false, 4>), grid, block, 0, s, a);
            }
            return hipGetLastError();
        }
        const bool skewed = views_skewed(a.cams);
        const uint32_t mixed_max = !ext ? kBwdMixedMax : (skewed ? kBwdMixedExtSkewMax : kBwdMixedExtMax);
        if (a.n_items > mixed_max) {
            const dim3 grid(a.n_items), block(64);
            if (ext) hipLaunchKernelGGL((k_render_bwd16_wave<true>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((k_render_bwd16_wave<false>), grid, block, 0, s, a);
            return hipGetLastError();
        }
        RenderArgs b = a;
        b.n_split = a.n_items <= (skewed ? kBwdSplitAllSkewMax : kBwdSplitAllMax) ? a.n_items : kBwdSplit;
        const dim3 grid(b.n_split + (a.n_items - b.n_split + 3) / 4), block(256);
        if (ext) hipLaunchKernelGGL((k_render_bwd16<true>), grid, block, 0, s, b);
        else hipLaunchKernelGGL((k_render_bwd16<false>), grid, block, 0, s, b);
        return hipGetLastError();
    }
    if (tw == 8 && th == 8) return bwd_shape<8, 8, 64>(a, s);
    if (tw == 32 && th == 16) return batch >= 128 ? bwd_shape<32, 16, 128>(a, s) : bwd_shape<32, 16, 64>(a, s);
    if (tw == 32 && th == 32) return bwd_shape<32, 32, 64>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace gesr
