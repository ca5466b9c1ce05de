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

// One pixel's state of the reverse traversal: transmittance in front of the
// fragment last visited, upstream gradients, and what lies behind per unit
// transmittance (colour; depth and opacity with the extended channels).
struct PixelAdjoint {
    float T, g0, g1, g2, Br, Bg, Bb, gD, gA, BD, BA;
};

// Adds one fragment's gradient terms to the splat's sums gr.  With
// G = exp(-kappa P), P = q^(beta/2), X = dL/dalpha o G P and d = -kappa beta X / q
// = 2 dL/dq, q = t^2 + w^2, t = L00 dx + L10 dy, w = L11 dy, (dx, dy) = pixel - (u, v):
//   gr = (sum d t, sum d w, sum d t dx, sum d t dy, sum d w dy, sum dL/dalpha G,
//         sum X ln q (-kappa / 2), dL/dr, dL/dg, dL/db)
// The conic factor is the same for all of a tile's pixels, so the centre's
// gradient takes it once, in `splat_partial`.  At q = 0 the footprint and beta terms
// are 0: P and X are, and the legacy product takes 0 times infinity as 0.  The
// alpha cap removes the dependence on opacity and footprint; a fragment below
// alpha_min has alpha 0 here, which leaves T (rcp(1) = 1), what lies behind and the
// sums as they are.  A flat splat seen edge-on amplifies the rounding of the three
// footprint sums in its scale gradient, so their terms keep this order of products.
// The kernel is bound by these instructions: the products in place of selects and
// the two sums for the centre took 53 instructions to 47 (a compare or select
// takes 4.3 cycles per wave on gfx950, a product 2.3), a step over 3M splats x 16
// views from 20.2 to 19.7 ms and over 1M flat splats x 4 views from 5.00 to 4.90 ms.
template <bool EXT>
__device__ __forceinline__ void add_fragment(const Fragment& f, const float4& rc, float z, const DevSettings& st,
                                             float c2, PixelAdjoint& px, float (&gr)[GESR_PARTIAL_FLOATS],
                                             float& gz) {
    const bool ok = !(f.alpha < st.alpha_min);
    const float al = ok ? f.alpha : 0.0f;
    px.T *= hw_rcp(1.0f - al);
    const float aT = al * px.T;
    gr[7] = fmaf(aT, px.g0, gr[7]);
    gr[8] = fmaf(aT, px.g1, gr[8]);
    gr[9] = fmaf(aT, px.g2, gr[9]);
    const float er = rc.x - px.Br, eg = rc.y - px.Bg, eb = rc.z - px.Bb;
    float dLda = px.T * fmaf(eb, px.g2, fmaf(er, px.g0, eg * px.g1));
    px.Br = fmaf(al, er, px.Br);
    px.Bg = fmaf(al, eg, px.Bg);
    px.Bb = fmaf(al, eb, px.Bb);
    if (EXT) {
        const float ed = z - px.BD, ea = 1.0f - px.BA;
        dLda = fmaf(px.T, fmaf(ed, px.gD, ea * px.gA), dLda);
        gz = fmaf(aT, px.gD, gz);
        px.BD = fmaf(al, ed, px.BD);
        px.BA = fmaf(al, ea, px.BA);
    }
    const float dl = ok && !(f.oG > st.alpha_max) ? dLda : 0.0f;
    gr[5] = fmaf(dl, f.G, gr[5]);
    const float X = dl * f.oG * f.P;
    gr[6] = fmaf(mul_legacy(X, f.l2q), c2, gr[6]);
    const float d = mul_legacy(X * rc.w, hw_rcp(f.q));
    const float tq = d * f.t, wq = d * f.w;
    gr[0] += tq;
    gr[1] += wq;
    gr[2] = fmaf(tq, f.dx, gr[2]);
    gr[3] = fmaf(tq, f.dy, gr[3]);
    gr[4] = fmaf(wq, f.dy, gr[4]);
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

// Slot of the instance (splat vi, tile (tx, ty)) in the pair-major order: the
// splat's instance base plus the tile's row-major position in its rectangle.
// When the lists overflowed their capacity the ranges no longer match the
// truncated lists, so a listed splat may not cover the tile or its slot may lie
// beyond the capacity; kNoInstance then suppresses the partial write.
__device__ __forceinline__ uint32_t instance_index(const RenderArgs& a, uint2 r, uint32_t vi, uint32_t tx,
                                                   uint32_t ty) {
    const uint32_t tx0 = r.x & 0xFFFFu, ty0 = r.x >> 16, tx1 = r.y & 0xFFFFu, ty1 = r.y >> 16;
    const uint32_t inst = a.inst_base[vi] + (ty - ty0) * (tx1 - tx0 + 1u) + (tx - tx0);
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

template <int TW, int TH, int BATCH>
__global__ __launch_bounds__(TW * TH) void k_render_bwd(RenderArgs a) {
    // The gradient arithmetic may fuse multiply-adds; the alpha, threshold and
    // transmittance evaluation shared with the forward is written with explicit
    // fmaf (or has no multiply-add) and compiles identically in both kernels.
#pragma clang fp contract(fast)
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

    PixelAdjoint pa{};
    pa.Br = st.bg[0];
    pa.Bg = st.bg[1];
    pa.Bb = st.bg[2];
    uint32_t nc = 0;
    if (ti.inside) {
        pa.T = a.final_T[ti.pix];
        nc = a.n_contrib[ti.pix];
        pa.g0 = a.dL_dimage[ti.img];
        pa.g1 = a.dL_dimage[ti.img + ti.ch];
        pa.g2 = a.dL_dimage[ti.img + 2 * ti.ch];
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
            sInst[threadIdx.x] = instance_index(a, r, vi, ti.tx, ti.ty);
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
                    float gz = 0.0f;
                    add_fragment<false>(f, sC[j], 0.0f, st, c2, pa, gr, gz);
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

// Orders a wave's LDS writes before its own later reads of other lanes' data
// (the waves of a workgroup run different tiles: no workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
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
        wave_lds_sync();
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
                blend<EXT>(p[q], ok ? f.alpha : 0.0f, ok, rc, rc.w, pos, st.t_min);
            }
        }
        wave_lds_sync();
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
        wave_lds_sync();
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
        wave_lds_sync();
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

// Backward, one wave per 16x16 tile: lane l owns pixel (l & 7, l >> 3) of each
// 8x8 quadrant (4 pixels per lane), so a staged splat's LDS reads and its
// 10-value wave reduction serve 256 pixels, and no cross-wave reduction or
// workgroup barrier beyond the wave itself is needed.  EXT: the extended
// channels' upstream gradients too (depth and opacity as colour channels over
// a zero background; the depth term dz is the eleventh partial value).
template <int B, bool EXT>
__global__ __launch_bounds__(64) void k_render_bwd_wave16(RenderArgs a) {
    // The gradient arithmetic may fuse multiply-adds; the alpha, threshold and
    // transmittance evaluation shared with the forward is written with explicit
    // fmaf (or has no multiply-add) and compiles identically in both kernels.
#pragma clang fp contract(fast)
    static_assert(B >= 1 && B <= 64, "one staged record per lane");
    constexpr int NP = GESR_PARTIAL_FLOATS;
    static_assert(NP == 10, "wave_sum10 reduces ten values");
    __shared__ float4 sA[B], sB[B], sC[B];
    __shared__ uint32_t sInst[B];
    __shared__ float sRed[B][NP + 1];  // column NP: dz (extended channels)
    __shared__ float sZ[EXT ? B : 1];   // staged splat depths (extended channels)

    const uint32_t t = a.worklist[blockIdx.x];
    const DevSettings& st = a.st;
    const float amax = st.alpha_max, nk = in_vgpr(st.neg_kappa_log2e);
    const float c2 = -0.5f * kLn2 * st.kappa;
    const uint32_t lane = __lane_id();
    const int v = view_of_tile(a.cams, t);
    const DevView& w = a.cams.v[v];
    const uint32_t lt = t - w.tile_base;
    const uint32_t tx = lt % (uint32_t)w.tiles_x, ty = lt / (uint32_t)w.tiles_x;
    const uint2 rg = reinterpret_cast<const uint2*>(a.ranges)[t];
    const uint32_t r0 = rg.x;
    const uint32_t ch = (uint32_t)w.W * (uint32_t)w.H;

    // pixel centres: quadrant q adds (q & 1) * 8 and (q >> 1) * 8 to the lane's base
    const float pxb = (float)(tx * 16 + (lane & 7)) + 0.5f, pyb = (float)(ty * 16 + (lane >> 3)) + 0.5f;
    PixelAdjoint pa[4];
    uint32_t nc[4];
    uint32_t mymax = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = (int)tx * 16 + (q & 1) * 8 + (int)(lane & 7);
        const int y = (int)ty * 16 + (q >> 1) * 8 + (int)(lane >> 3);
        pa[q] = PixelAdjoint{};  // the background has no depth and no opacity
        pa[q].Br = st.bg[0];
        pa[q].Bg = st.bg[1];
        pa[q].Bb = st.bg[2];
        nc[q] = 0;
        if (x < w.W && y < w.H) {
            const uint32_t local = (uint32_t)y * (uint32_t)w.W + (uint32_t)x;
            const uint32_t pix = w.pix_base + local, img = 3u * w.pix_base + local;
            pa[q].T = a.final_T[pix];
            nc[q] = a.n_contrib[pix];
            pa[q].g0 = a.dL_dimage[img];
            pa[q].g1 = a.dL_dimage[img + ch];
            pa[q].g2 = a.dL_dimage[img + 2 * ch];
            if (EXT) {
                if (a.dL_ddepth) pa[q].gD = a.dL_ddepth[pix];
                if (a.dL_dalpha) pa[q].gA = a.dL_dalpha[pix];
            }
        }
        mymax = max(mymax, nc[q]);
    }
    const uint32_t maxnc = __builtin_amdgcn_readfirstlane(wave_max_u32(mymax));  // uniform: scalar loop control
    const uint32_t end = r0 + maxnc;  // positions >= end contributed to no pixel
    const int slot = lane < 16 ? wave_sum10_slot(lane) : NP;  // value this lane writes after a reduction

    for (uint32_t hi = end; hi > r0;) {
        const uint32_t lo = (hi - r0 > (uint32_t)B) ? hi - B : r0;
        const int cnt = (int)(hi - lo);
        if ((int)lane < cnt) {
            const uint32_t pos = hi - 1u - lane;
            const uint32_t vi = a.val_sorted[pos];
            stage_record(a.rec, vi, st.kappa, sA[lane], sB[lane], sC[lane]);
            if (EXT) sZ[lane] = a.rec[(size_t)vi * GESR_REC_FLOATS + 11];
            const float4 r3 = reinterpret_cast<const float4*>(a.rec + (size_t)vi * GESR_REC_FLOATS)[3];
            const uint2 r = make_uint2(__float_as_uint(r3.x), __float_as_uint(r3.y));  // the pair's rectangle
            sInst[lane] = instance_index(a, r, vi, tx, ty);
        }
        __syncthreads();
        for (int j = 0; j < cnt; ++j) {
            const uint32_t prel = hi - 1u - (uint32_t)j - r0;  // 0-based list position
            const float4 ra = sA[j];
            const float4 rb = sB[j];
            const float4 rc = sC[j];
            const float z = EXT ? sZ[j] : 0.0f;
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
                // decisions are selects (a zeroed term leaves the sums as they
                // are), so the wave takes one branch per quadrant.
                ges_alpha(qq, rb.z, rb.y, nk, amax, f);
                act = true;
                add_fragment<EXT>(f, rc, z, st, c2, pa[q], gr, gz);
            }
            if (__ballot(act) != 0ull) {
                const float tot = wave_sum10(gr, lane);
                if (slot < NP) sRed[j][slot] = tot;
                if (EXT) {
                    const float tz = wave_sum(gz);
                    if (lane == 0) sRed[j][NP] = tz;
                }
            } else if ((int)lane < (EXT ? NP + 1 : NP)) {
                sRed[j][lane] = 0.f;
            }
        }
        __syncthreads();
        if ((int)lane < cnt && sInst[lane] != kNoInstance) {
            float s[NP + 1];
#pragma unroll
            for (int k = 0; k <= NP; ++k) s[k] = EXT || k < NP ? sRed[lane][k] : 0.0f;
            splat_partial(s, sA[lane], sB[lane]);
            write_partial<EXT>(a, sInst[lane], s);
        }
        __syncthreads();
        hi = lo;
    }
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
        const dim3 grid(a.n_items), block(64);
        if (ext) {
            if (batch == 32) hipLaunchKernelGGL((k_render_bwd_wave16<32, true>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((k_render_bwd_wave16<64, true>), grid, block, 0, s, a);
        } else {
            if (batch == 32) hipLaunchKernelGGL((k_render_bwd_wave16<32, false>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((k_render_bwd_wave16<64, false>), grid, block, 0, s, a);
        }
        return hipGetLastError();
    }
    if (tw == 8 && th == 8) return bwd_shape<8, 8, 64>(a, s);
    if (tw == 32 && th == 16) return batch >= 128 ? bwd_shape<32, 16, 128>(a, s) : bwd_shape<32, 16, 64>(a, s);
    if (tw == 32 && th == 32) return bwd_shape<32, 32, 64>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace gesr
