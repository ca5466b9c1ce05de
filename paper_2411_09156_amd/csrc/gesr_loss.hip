// Photometric loss of Eq. 8 (Sec. 3.2): L_v = (1 - lambda) mean|X - Y| +
// lambda (1 - mean SSIM) per view, and its gradient with respect to the
// rendered image X, for every view of the batch in one launch per kernel.
//
// SSIM (the paper names it, not its window): an 11 x 11 Gaussian window with
// zero padding, C1 and C2 as given.  With the window sums mu = G*X, m2 = G*X^2,
// mxy = G*(X Y):
//   S = (2 mu_x mu_y + C1)(2 s_xy + C2) / ((mu_x^2 + mu_y^2 + C1)(s_x^2 + s_y^2 + C2)),
//   s_x^2 = m2x - mu_x^2, s_xy = mxy - mu_x mu_y.
// The gradient of sum_p S(p) is the window sum of the moments' adjoints:
//   dS/dX(q) = (G*a)(q) + 2 X(q) (G*b)(q) + Y(q) (G*c)(q)
// with a = dS/dmu_x, b = dS/dm2x, c = dS/dmxy per pixel (the window is
// symmetric, so the adjoint of a zero-padded window sum is the window sum).
//
// Both kernels work on 16 x 16 output tiles, one thread per pixel: the tile's
// 26 x 26 input patch (5 pixels of halo, zero outside the image) is staged in
// LDS, the 11 horizontal taps are summed per row (two neighbours by one thread, which
// share ten of their inputs), then the 11 vertical taps per pixel.  Bound by the
// chain from load to store of each channel where tiles are few, so the next channel's
// patch is loaded during this one's sums and a patch's addresses are found once; the
// weights sit in vector registers, where a multiply-add takes them at full rate.
// 3,024 tiles: forward 33 us (40 without these), backward 30 (41); 64 tiles: 7.8
// (11.9) and 5.6 (13.9).  The forward writes a, b, c and per-tile partial sums of S and
// |X - Y| (fixed-order block reductions); a one-block-per-view kernel sums the
// partials in tile order; the backward adds the L1 term's sign.

#include "gesr_device.h"
#include "gesr_kernels.h"

namespace gesr {

namespace {

constexpr int kR = GESR_LOSS_RADIUS;  // window radius (11 taps)
constexpr int kTile = 16;
constexpr int kPatch = kTile + 2 * kR;  // 26
constexpr int kThreads = kTile * kTile;

__device__ __forceinline__ int view_of_loss_tile(const LossArgs& a, uint32_t t) {
    int v = 0;
    while (v + 1 < a.V && t >= a.v[v + 1].tile_base) ++v;
    return v;
}

// Fixed-order sum over the 256 threads of a block (wave butterflies, then the
// four wave totals in order); every thread receives the total.
__device__ __forceinline__ float block_sum(float x, float* lds4) {
    x = wave_sum(x);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds4[w] = x;
    __syncthreads();
    return ((lds4[0] + lds4[1]) + lds4[2]) + lds4[3];
}

// The patch around a tile: this thread's up to three elements, where they lie in a
// plane of the view (-1: outside, zero) and in LDS.
constexpr int kPitch = kPatch + 1;
constexpr int kElems = (kPatch * kPatch + kThreads - 1) / kThreads;
struct Patch {
    int off[kElems];
    __device__ __forceinline__ Patch(const LossView& w, int tx0, int ty0) {
#pragma unroll
        for (int k = 0; k < kElems; ++k) {
            const int i = threadIdx.x + k * kThreads;
            const int gy = ty0 + i / kPatch - kR, gx = tx0 + i % kPatch - kR;
            const bool in = i < kPatch * kPatch && gx >= 0 && gx < w.W && gy >= 0 && gy < w.H;
            off[k] = in ? gy * w.W + gx : -1;
        }
    }
    __device__ __forceinline__ void load(const float* src, float (&v)[kElems]) const {
#pragma unroll
        for (int k = 0; k < kElems; ++k) v[k] = off[k] >= 0 ? src[off[k]] : 0.0f;
    }
    __device__ __forceinline__ void store(float* dst, const float (&v)[kElems]) const {
#pragma unroll
        for (int k = 0; k < kElems; ++k) {
            const int i = threadIdx.x + k * kThreads;
            if (i < kPatch * kPatch) dst[i / kPatch * kPitch + i % kPatch] = v[k];
        }
    }
};

// The window's weights, in vector registers.
struct Window {
    float w[2 * kR + 1];
    __device__ __forceinline__ explicit Window(const LossArgs& a) {
#pragma unroll
        for (int j = 0; j <= 2 * kR; ++j) w[j] = in_vgpr(a.w[j]);
    }
};

__global__ __launch_bounds__(kThreads) void k_ssim_fwd(LossArgs a) {
    __shared__ float sx[kPatch * kPitch], sy[kPatch * kPitch];
    __shared__ float h[5][kPatch][kTile + 1];
    __shared__ float red[4];
    const uint32_t t = blockIdx.x;
    const int v = view_of_loss_tile(a, t);
    const LossView& w = a.v[v];
    const uint32_t lt = t - w.tile_base;
    const int tiles_x = (w.W + kTile - 1) / kTile;
    const int tx0 = (int)(lt % tiles_x) * kTile, ty0 = (int)(lt / tiles_x) * kTile;
    const int lx = threadIdx.x % kTile, ly = threadIdx.x / kTile;
    const int x = tx0 + lx, y = ty0 + ly;
    const bool inside = x < w.W && y < w.H;
    const size_t HW = (size_t)w.W * w.H;
    float s_sum = 0.0f, l1_sum = 0.0f;
    const Patch patch(w, tx0, ty0);
    const Window win(a);
    const float *image = a.image + 3 * (size_t)w.pix_base, *target = a.target + 3 * (size_t)w.pix_base;
    float nx[kElems], ny[kElems];
    patch.load(image, nx);
    patch.load(target, ny);
    for (int ch = 0; ch < 3; ++ch) {
        const size_t base = 3 * (size_t)w.pix_base + ch * HW;
        __syncthreads();
        patch.store(sx, nx);
        patch.store(sy, ny);
        __syncthreads();
        if (ch < 2) {
            patch.load(image + (ch + 1) * HW, nx);
            patch.load(target + (ch + 1) * HW, ny);
        }
        if (threadIdx.x < kPatch * kTile / 2) {
            const int r = threadIdx.x / (kTile / 2), q = threadIdx.x % (kTile / 2) * 2;
            const float *px = sx + r * kPitch + q, *py = sy + r * kPitch + q;
            float m1x[2] = {0.f, 0.f}, m1y[2] = {0.f, 0.f}, m2x[2] = {0.f, 0.f}, m2y[2] = {0.f, 0.f},
                  mxy[2] = {0.f, 0.f};
#pragma unroll
            for (int j = 0; j <= 2 * kR + 1; ++j) {
                const float xv = px[j], yv = py[j];
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    if (j - o < 0 || j - o > 2 * kR) continue;
                    const float gx = win.w[j - o] * xv;
                    const float gy = win.w[j - o] * yv;
                    m1x[o] += gx;
                    m1y[o] += gy;
                    m2x[o] = fmaf(gx, xv, m2x[o]);
                    m2y[o] = fmaf(gy, yv, m2y[o]);
                    mxy[o] = fmaf(gx, yv, mxy[o]);
                }
            }
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                h[0][r][q + o] = m1x[o];
                h[1][r][q + o] = m1y[o];
                h[2][r][q + o] = m2x[o];
                h[3][r][q + o] = m2y[o];
                h[4][r][q + o] = mxy[o];
            }
        }
        __syncthreads();
        float m[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i <= 2 * kR; ++i)
#pragma unroll
            for (int k = 0; k < 5; ++k) m[k] = fmaf(win.w[i], h[k][ly + i][lx], m[k]);
        if (inside) {
            const float mx = m[0], my = m[1];
            const float sxx = m[2] - mx * mx, syy = m[3] - my * my, sxy = m[4] - mx * my;
            const float N1 = 2.f * mx * my + a.c1, N2 = 2.f * sxy + a.c2;
            const float D1 = mx * mx + my * my + a.c1, D2 = sxx + syy + a.c2;
            const float inv = 1.0f / (D1 * D2);
            const float S = N1 * N2 * inv;
            const float da = 2.f * my * N2 * inv - 2.f * mx * S / D1 + 2.f * mx * S / D2 - 2.f * my * N1 * inv;
            const size_t p = base + (size_t)y * w.W + x;
            a.amap[p] = da;
            a.bmap[p] = -S / D2;
            a.cmap[p] = 2.f * N1 * inv;
            s_sum += S;
            l1_sum += fabsf(sx[(ly + kR) * kPitch + lx + kR] - sy[(ly + kR) * kPitch + lx + kR]);
        }
    }
    const float ts = block_sum(s_sum, red);
    const float tl = block_sum(l1_sum, red);
    if (threadIdx.x == 0) {
        a.partial[2 * (size_t)t] = ts;
        a.partial[2 * (size_t)t + 1] = tl;
    }
}

// One block per view: the view's tile partials summed in tile order (each
// thread a fixed stride, then the block sum), then L_v.
__global__ __launch_bounds__(kThreads) void k_ssim_loss(LossArgs a) {
    __shared__ float red[4];
    const LossView& w = a.v[blockIdx.x];
    const uint32_t tiles = (uint32_t)(((w.W + kTile - 1) / kTile) * ((w.H + kTile - 1) / kTile));
    float s = 0.f, l = 0.f;
    for (uint32_t i = threadIdx.x; i < tiles; i += kThreads) {
        s += a.partial[2 * (size_t)(w.tile_base + i)];
        l += a.partial[2 * (size_t)(w.tile_base + i) + 1];
    }
    s = block_sum(s, red);
    l = block_sum(l, red);
    if (threadIdx.x == 0) a.loss[blockIdx.x] = (1.0f - a.lam) * l * w.inv_n + a.lam * (1.0f - s * w.inv_n);
}

__global__ __launch_bounds__(kThreads) void k_ssim_bwd(LossArgs a) {
    __shared__ float sp[3][kPatch * kPitch];
    __shared__ float h[3][kPatch][kTile + 1];
    const uint32_t t = blockIdx.x;
    const int v = view_of_loss_tile(a, t);
    const LossView& w = a.v[v];
    const uint32_t lt = t - w.tile_base;
    const int tiles_x = (w.W + kTile - 1) / kTile;
    const int tx0 = (int)(lt % tiles_x) * kTile, ty0 = (int)(lt / tiles_x) * kTile;
    const int lx = threadIdx.x % kTile, ly = threadIdx.x / kTile;
    const int x = tx0 + lx, y = ty0 + ly;
    const bool inside = x < w.W && y < w.H;
    const size_t HW = (size_t)w.W * w.H;
    const float l1s = (1.0f - a.lam) * w.inv_n, ss = a.lam * w.inv_n;
    const Patch patch(w, tx0, ty0);
    const Window win(a);
    const size_t first = 3 * (size_t)w.pix_base;
    float n0[kElems], n1[kElems], n2[kElems];
    patch.load(a.amap + first, n0);
    patch.load(a.bmap + first, n1);
    patch.load(a.cmap + first, n2);
    for (int ch = 0; ch < 3; ++ch) {
        const size_t base = first + ch * HW;
        const size_t p = base + (size_t)y * w.W + x;
        __syncthreads();
        patch.store(sp[0], n0);
        patch.store(sp[1], n1);
        patch.store(sp[2], n2);
        const float X = inside ? a.image[p] : 0.f, Y = inside ? a.target[p] : 0.f;
        __syncthreads();
        if (ch < 2) {
            patch.load(a.amap + base + HW, n0);
            patch.load(a.bmap + base + HW, n1);
            patch.load(a.cmap + base + HW, n2);
        }
        if (threadIdx.x < kPatch * kTile / 2) {
            const int r = threadIdx.x / (kTile / 2), q = threadIdx.x % (kTile / 2) * 2;
            float s[3][2] = {};
#pragma unroll
            for (int j = 0; j <= 2 * kR + 1; ++j)
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float v = sp[k][r * kPitch + q + j];
#pragma unroll
                    for (int o = 0; o < 2; ++o)
                        if (j - o >= 0 && j - o <= 2 * kR) s[k][o] = fmaf(win.w[j - o], v, s[k][o]);
                }
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int o = 0; o < 2; ++o) h[k][r][q + o] = s[k][o];
        }
        __syncthreads();
        float ga = 0.f, gb = 0.f, gc = 0.f;
#pragma unroll
        for (int i = 0; i <= 2 * kR; ++i) {
            ga = fmaf(win.w[i], h[0][ly + i][lx], ga);
            gb = fmaf(win.w[i], h[1][ly + i][lx], gb);
            gc = fmaf(win.w[i], h[2][ly + i][lx], gc);
        }
        if (inside) {
            const float d = X - Y;
            const float sgn = (d > 0.f) ? 1.f : ((d < 0.f) ? -1.f : 0.f);
            const float dS = ga + 2.f * X * gb + Y * gc;
            a.grad[p] = l1s * sgn - ss * dS;
        }
    }
}

}  // namespace

hipError_t launch_ssim_loss(const LossArgs& a, uint32_t n_tiles, bool want_loss, hipStream_t stream) {
    if (n_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ssim_fwd, dim3(n_tiles), dim3(kThreads), 0, stream, a);
    if (want_loss) hipLaunchKernelGGL(k_ssim_loss, dim3(a.V), dim3(kThreads), 0, stream, a);
    hipLaunchKernelGGL(k_ssim_bwd, dim3(n_tiles), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace gesr

// --------------------------------------------------------------------------
// Surface-alignment regulariser of the flattened-splat workload: per splat,
// with k* the axis of the smallest scale (lowest index on ties), n = R(q) e_k*
// and m the true surface normal,
//   L = w_scale / N sum_i s_ik* + w_normal / N sum_i (1 - <n_i, m_i>^2);
// its gradient is added to the scale and quaternion gradients (one thread per
// splat: an HBM-bound pass) and its two sums are reduced in a fixed order.
namespace gesr {

namespace {

__global__ __launch_bounds__(256) void k_surface_align(AlignArgs a) {
    __shared__ float red[4];
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const size_t n = (size_t)a.n;
    float ls = 0.f, ln = 0.f;
    if (i < (uint32_t)a.n) {
        const float s0 = a.scale[i], s1 = a.scale[n + i], s2 = a.scale[2 * n + i];
        const int k = (s0 <= s1 && s0 <= s2) ? 0 : (s1 <= s2 ? 1 : 2);
        const float qw0 = a.quat[i], qx0 = a.quat[n + i], qy0 = a.quat[2 * n + i], qz0 = a.quat[3 * n + i];
        const float inv = 1.0f / sqrtf(qw0 * qw0 + qx0 * qx0 + qy0 * qy0 + qz0 * qz0);
        const float w = qw0 * inv, x = qx0 * inv, y = qy0 * inv, z = qz0 * inv;
        // column k of R(q) and its derivative with respect to (w, x, y, z)
        float c[3], J[3][4];
        if (k == 0) {
            c[0] = 1.f - 2.f * (y * y + z * z); c[1] = 2.f * (x * y + w * z); c[2] = 2.f * (x * z - w * y);
            J[0][0] = 0.f;        J[0][1] = 0.f;       J[0][2] = -4.f * y;  J[0][3] = -4.f * z;
            J[1][0] = 2.f * z;    J[1][1] = 2.f * y;   J[1][2] = 2.f * x;   J[1][3] = 2.f * w;
            J[2][0] = -2.f * y;   J[2][1] = 2.f * z;   J[2][2] = -2.f * w;  J[2][3] = 2.f * x;
        } else if (k == 1) {
            c[0] = 2.f * (x * y - w * z); c[1] = 1.f - 2.f * (x * x + z * z); c[2] = 2.f * (y * z + w * x);
            J[0][0] = -2.f * z;   J[0][1] = 2.f * y;   J[0][2] = 2.f * x;   J[0][3] = -2.f * w;
            J[1][0] = 0.f;        J[1][1] = -4.f * x;  J[1][2] = 0.f;       J[1][3] = -4.f * z;
            J[2][0] = 2.f * x;    J[2][1] = 2.f * w;   J[2][2] = 2.f * z;   J[2][3] = 2.f * y;
        } else {
            c[0] = 2.f * (x * z + w * y); c[1] = 2.f * (y * z - w * x); c[2] = 1.f - 2.f * (x * x + y * y);
            J[0][0] = 2.f * y;    J[0][1] = 2.f * z;   J[0][2] = 2.f * w;   J[0][3] = 2.f * x;
            J[1][0] = -2.f * x;   J[1][1] = -2.f * w;  J[1][2] = 2.f * z;   J[1][3] = 2.f * y;
            J[2][0] = 0.f;        J[2][1] = -4.f * x;  J[2][2] = -4.f * y;  J[2][3] = 0.f;
        }
        const float m0 = a.normal[i], m1 = a.normal[n + i], m2 = a.normal[2 * n + i];
        const float d = c[0] * m0 + c[1] * m1 + c[2] * m2;
        ls = k == 0 ? s0 : (k == 1 ? s1 : s2);
        ln = 1.f - d * d;
        // dL/dn = -2 d w_normal / N m, then through the column and the normalisation
        const float gsc = -2.f * d * a.w_normal_n;
        const float gn[3] = {gsc * m0, gsc * m1, gsc * m2};
        float gq[4];
        for (int j = 0; j < 4; ++j) gq[j] = gn[0] * J[0][j] + gn[1] * J[1][j] + gn[2] * J[2][j];
        const float dot = gq[0] * w + gq[1] * x + gq[2] * y + gq[3] * z;
        a.g_quat[i] += (gq[0] - dot * w) * inv;
        a.g_quat[n + i] += (gq[1] - dot * x) * inv;
        a.g_quat[2 * n + i] += (gq[2] - dot * y) * inv;
        a.g_quat[3 * n + i] += (gq[3] - dot * z) * inv;
        a.g_scale[(size_t)k * n + i] += a.w_scale_n;
    }
    const float ts = block_sum(ls, red);
    const float tn = block_sum(ln, red);
    if (a.partial && threadIdx.x == 0) {
        a.partial[2 * (size_t)blockIdx.x] = ts;
        a.partial[2 * (size_t)blockIdx.x + 1] = tn;
    }
}

// One block: the block partials summed in block order, scaled by the weights.
__global__ __launch_bounds__(256) void k_surface_align_sum(AlignArgs a, uint32_t blocks) {
    __shared__ float red[4];
    float s = 0.f, t = 0.f;
    for (uint32_t b = threadIdx.x; b < blocks; b += 256) {
        s += a.partial[2 * (size_t)b];
        t += a.partial[2 * (size_t)b + 1];
    }
    s = block_sum(s, red);
    t = block_sum(t, red);
    if (threadIdx.x == 0) {
        a.losses[0] = s * a.w_scale_n;
        a.losses[1] = t * a.w_normal_n;
    }
}

}  // namespace

hipError_t launch_surface_align(const AlignArgs& a, hipStream_t stream) {
    if (a.n <= 0) return hipSuccess;
    const uint32_t blocks = (uint32_t)((a.n + 255) / 256);
    hipLaunchKernelGGL(k_surface_align, dim3(blocks), dim3(256), 0, stream, a);
    if (a.losses) hipLaunchKernelGGL(k_surface_align_sum, dim3(1), dim3(256), 0, stream, a, blocks);
    return hipGetLastError();
}

}  // namespace gesr
