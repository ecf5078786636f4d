// gfx950 (CDNA4) kernels of the Gaussian-splatting rasterizer used by RT-GuIDE
// (arXiv 2409.18122): projection and culling, prefix sums, an LSD radix sort,
// tile binning, front-to-back compositing of RGB / depth / alpha /
// uncertainty, the L1 mapping loss, the reverse-mode kernels, and the
// persistent view scorer.
//
// The file is compiled without floating-point contraction: every fused
// multiply-add below is an explicit fmaf/fma, so a value computed in two
// kernels (a splat's alpha in the forward and the backward, the camera depth
// used as sort key) is bit-identical in both.
#include "rtg_internal.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace rtg {

namespace {

constexpr double LOG2E = 1.4426950408889634;

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    uint32_t l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ------------------------------------------------------------------ fill

// Orders a wave's LDS stores and loads (a compiler's matter: the hardware keeps them in order).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

// ------------------------------------------------------------- projection
// Sec. III (Gaussian Splatting paragraph): t = R^T (mu - T), d = t_z,
// mu_2D = (fx t_x / d + cx, fy t_y / d + cy); the 2D covariance is the EWA
// form J R^T Sigma R J^T of the cited 3DGS work, with Sigma = Rq S^2 Rq^T,
// or, for the paper's isotropic Gaussians, diag((fx r / d)^2, (fy r / d)^2)
// (r_2D = f r / d; one log-radius per Gaussian, no quaternion).

struct GPre {
    double mu[3];
    double Rq[9];
    double s[3];
    double o, rho2;
    float mu_f[3];
    float reach;           // rho * max scale: bound on the support radius in 3D
    float rho_f, rho2_f;   // binary32 rho = sqrt(2 ln(o / alpha_min)) and rho^2, for the bound
};

// The isotropic form: s = (r, r, r) and Rq = I; only the first n log-scale values are read.
__device__ inline bool pre_gauss_iso(const GaussDev& g, int64_t i, const SetDev& st, GPre& P) {
    const int64_t n = g.n;
    const float m0 = g.means[i], m1 = g.means[n + i], m2 = g.means[2 * n + i];
    const float lr = g.log_scales[i];
    const float op = g.opacity[i];
    if (!(isfinite(m0) && isfinite(m1) && isfinite(m2) && isfinite(lr) && isfinite(op))) return false;
    if (op < st.alpha_min) return false;
#pragma unroll
    for (int k = 0; k < 9; k++) P.Rq[k] = (k % 4 == 0) ? 1.0 : 0.0;
    const double r = exp((double)lr);
    P.s[0] = r;
    P.s[1] = r;
    P.s[2] = r;
    P.mu[0] = m0; P.mu[1] = m1; P.mu[2] = m2;
    P.mu_f[0] = m0; P.mu_f[1] = m1; P.mu_f[2] = m2;
    P.o = op;
    P.rho2 = 2.0 * log((double)op / (double)st.alpha_min);
    P.reach = (float)(sqrt(P.rho2) * r);
    P.rho_f = (float)sqrt(P.rho2);
    P.rho2_f = (float)P.rho2;
    return true;
}

__device__ inline bool pre_gauss(const GaussDev& g, int64_t i, const SetDev& st, GPre& P) {
    if (st.isotropic) return pre_gauss_iso(g, i, st, P);
    const int64_t n = g.n;
    float m0 = g.means[i], m1 = g.means[n + i], m2 = g.means[2 * n + i];
    float l0 = g.log_scales[i], l1 = g.log_scales[n + i], l2 = g.log_scales[2 * n + i];
    float q0 = g.quats[i], q1 = g.quats[n + i], q2 = g.quats[2 * n + i], q3 = g.quats[3 * n + i];
    float op = g.opacity[i];
    bool fin = isfinite(m0) && isfinite(m1) && isfinite(m2) && isfinite(l0) && isfinite(l1) &&
               isfinite(l2) && isfinite(q0) && isfinite(q1) && isfinite(q2) && isfinite(q3) &&
               isfinite(op);
    if (!fin) return false;
    if (op < st.alpha_min) return false;
    double w = q0, x = q1, y = q2, z = q3;
    double qn = sqrt(w * w + x * x + y * y + z * z);
    if (!(qn > 0.0)) return false;
    double inv = 1.0 / qn;
    w *= inv; x *= inv; y *= inv; z *= inv;
    double xx = x * x, yy = y * y, zz = z * z;
    double xy = x * y, xz = x * z, yz = y * z, wx = w * x, wy = w * y, wz = w * z;
    P.Rq[0] = 1.0 - 2.0 * (yy + zz); P.Rq[1] = 2.0 * (xy - wz);       P.Rq[2] = 2.0 * (xz + wy);
    P.Rq[3] = 2.0 * (xy + wz);       P.Rq[4] = 1.0 - 2.0 * (xx + zz); P.Rq[5] = 2.0 * (yz - wx);
    P.Rq[6] = 2.0 * (xz - wy);       P.Rq[7] = 2.0 * (yz + wx);       P.Rq[8] = 1.0 - 2.0 * (xx + yy);
    P.s[0] = exp((double)l0);
    P.s[1] = exp((double)l1);
    P.s[2] = exp((double)l2);
    P.mu[0] = m0; P.mu[1] = m1; P.mu[2] = m2;
    P.mu_f[0] = m0; P.mu_f[1] = m1; P.mu_f[2] = m2;
    P.o = op;
    P.rho2 = 2.0 * log((double)op / (double)st.alpha_min);
    double smax = fmax(P.s[0], fmax(P.s[1], P.s[2]));
    P.reach = (float)(sqrt(P.rho2) * smax);
    P.rho_f = (float)sqrt(P.rho2);
    P.rho2_f = (float)P.rho2;
    return true;
}

// Bounds hi and lo of the singular values of a camera's matrix, which may be any finite one, from the row sums
// of R^T R; both 1 for a rotation (within 1e-3, which the screens' constants cover).
__device__ __forceinline__ float2 camera_norms(const ViewDev& V) {
    float hi = 0.0f, lo = INFINITY, off = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        float diag = 0.0f, rest = 0.0f;
#pragma unroll
        for (int b = 0; b < 3; b++) {
            const float dot = V.Rf[a] * V.Rf[b] + V.Rf[3 + a] * V.Rf[3 + b] + V.Rf[6 + a] * V.Rf[6 + b];
            if (a == b) diag = dot;
            else rest += fabsf(dot);
        }
        off = fmaxf(off, fmaxf(fabsf(diag - 1.0f), rest));
        hi = fmaxf(hi, diag + rest);
        lo = fminf(lo, diag - rest);
    }
    if (off <= 1e-3f) return make_float2(1.0f, 1.0f);
    return make_float2(sqrtf(hi) * 1.00001f, sqrtf(fmaxf(lo - 1e-5f * hi, 0.0f)) * 0.99999f);
}

// Conservative binary32 test: false only if the exact binary64 projection is
// certain to be culled (behind the near plane, or its support box cannot meet
// the image).  The half extent of the support box is bounded through
// Sigma_xx <= s_max^2 |J_row0|^2 = s_max^2 fx^2 / t_z^2 (1 + t_x^2 / t_z^2), times the square of the largest
// singular value of R where that is no rotation (the isotropic extent does not see R).
// The binary32 camera values the test reads, packed in five 16-byte words:
// the columns of R with the camera centre, (fx, fy, cx, cy), (W - 1, H - 1,
// the factors of the depth's error and of the extent).
struct CullView {
    float4 c0, c1, c2, k, wh;
};

__device__ __forceinline__ CullView cull_view(const ViewDev& V, const SetDev& st) {
    CullView f;
    f.c0 = make_float4(V.Rf[0], V.Rf[3], V.Rf[6], V.Tf[0]);
    f.c1 = make_float4(V.Rf[1], V.Rf[4], V.Rf[7], V.Tf[1]);
    f.c2 = make_float4(V.Rf[2], V.Rf[5], V.Rf[8], V.Tf[2]);
    f.k = make_float4(V.fxf, V.fyf, V.cxf, V.cyf);
    const float norm = camera_norms(V).x;
    f.wh = make_float4((float)(V.W - 1), (float)(V.H - 1), norm, st.isotropic ? 1.0f : norm);
    return f;
}

__device__ inline bool may_be_visible(const GPre& P, const CullView& V, const SetDev& st) {
    float dx = P.mu_f[0] - V.c0.w;
    float dy = P.mu_f[1] - V.c1.w;
    float dz = P.mu_f[2] - V.c2.w;
    float mag = fabsf(dx) + fabsf(dy) + fabsf(dz) + 1.0f;
    float tz = dx * V.c2.x + dy * V.c2.y + dz * V.c2.z;
    float err = 1e-5f * mag * V.wh.z;
    if (tz + err <= st.z_near) return false;
    if (tz <= 0.5f * st.z_near) return true;  // let the exact test decide
    float tx = dx * V.c0.x + dy * V.c0.y + dz * V.c0.z;
    float ty = dx * V.c1.x + dy * V.c1.y + dz * V.c1.z;
    // hardware reciprocal and square root (within an ulp or two): the slack
    // below is a relative 1e-3 plus a pixel
    float iz = __builtin_amdgcn_rcpf(tz);
    float ux = tx * iz, uy = ty * iz;
    float fx = V.k.x, fy = V.k.y;
    float ax = fx * ux + V.k.z;
    float ay = fy * uy + V.k.w;
    const float reach = P.reach * V.wh.w;
    float rx = reach * fx * iz, ry = reach * fy * iz;
    const float ep = 2.0f * P.rho_f * st.eps2d + st.eps2d * P.rho2_f;
    float hx = __builtin_amdgcn_sqrtf(rx * rx * (1.0f + ux * ux) + ep);
    float hy = __builtin_amdgcn_sqrtf(ry * ry * (1.0f + uy * uy) + ep);
    float slack_x = 1e-3f * (fabsf(ax - V.k.z) + hx) + 1.0f + err * fx * iz * 4.0f;
    float slack_y = 1e-3f * (fabsf(ay - V.k.w) + hy) + 1.0f + err * fy * iz * 4.0f;
    if (ax + hx + slack_x < 0.0f) return false;
    if (ax - hx - slack_x > V.wh.x) return false;
    if (ay + hy + slack_y < 0.0f) return false;
    if (ay - hy - slack_y > V.wh.y) return false;
    return true;
}

struct GProj {
    double t[3];
    double A[9];  // R^T Rq
    double j0, j2, j4, j5;  // nonzero entries of the perspective Jacobian
    double cxx, cxy, cyy;
    double mx, my;
    int u0, u1, v0, v1;
};

// A camera in binary64, from the binary32 values of the table: every lane of a wave may have its own camera, and five
// 16-byte loads visit a quarter of the cache lines that the table's binary64 copy would.
struct Cam {
    double R[9], T[3], fx, fy, cx, cy;
    int W, H;
};

__device__ __forceinline__ Cam load_cam(const ViewDev* v) {
    static_assert(offsetof(ViewDev, Rf) % 16 == 0 && sizeof(ViewDev) % 16 == 0 &&
                      offsetof(ViewDev, W) == offsetof(ViewDev, Rf) + 64, "the camera's 18 words in five 16-byte loads");
    const float4* p = reinterpret_cast<const float4*>(v->Rf);
    const float4 a = p[0], b = p[1], c = p[2], d = p[3];
    const int2 wh = *reinterpret_cast<const int2*>(&v->W);
    Cam V;
    V.R[0] = a.x; V.R[1] = a.y; V.R[2] = a.z; V.R[3] = a.w;
    V.R[4] = b.x; V.R[5] = b.y; V.R[6] = b.z; V.R[7] = b.w;
    V.R[8] = c.x; V.T[0] = c.y; V.T[1] = c.z; V.T[2] = c.w;
    V.fx = d.x; V.fy = d.y; V.cx = d.z; V.cy = d.w;
    V.W = wh.x; V.H = wh.y;
    return V;
}

// Exact binary64 projection.  The camera depth is evaluated in the fixed
// order ((dx R02 + dy R12) + dz R22): its binary32 rounding is the sort key.
__device__ inline bool project_exact(const GPre& P, const Cam& V, const SetDev& st, GProj& q) {
    double dx = P.mu[0] - V.T[0];
    double dy = P.mu[1] - V.T[1];
    double dz = P.mu[2] - V.T[2];
    const double* R = V.R;
    double tx = (dx * R[0] + dy * R[3]) + dz * R[6];
    double ty = (dx * R[1] + dy * R[4]) + dz * R[7];
    double tz = (dx * R[2] + dy * R[5]) + dz * R[8];
    if (!(tz > (double)st.z_near)) return false;
    q.t[0] = tx; q.t[1] = ty; q.t[2] = tz;
    double iz = 1.0 / tz;
    q.j0 = V.fx * iz;
    q.j4 = V.fy * iz;
    if (st.isotropic) {
        // Sigma_2D = diag(j0^2, j4^2) r^2: the EWA form below with A = I and
        // no off-axis Jacobian terms (which the backward then treats as constant)
#pragma unroll
        for (int k = 0; k < 9; k++) q.A[k] = (k % 4 == 0) ? 1.0 : 0.0;
        q.j2 = 0.0;
        q.j5 = 0.0;
    } else {
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++)
                q.A[a * 3 + b] = fma(R[0 * 3 + a], P.Rq[0 * 3 + b],
                                     fma(R[1 * 3 + a], P.Rq[1 * 3 + b], R[2 * 3 + a] * P.Rq[2 * 3 + b]));
        q.j2 = -V.fx * tx * iz * iz;
        q.j5 = -V.fy * ty * iz * iz;
    }
    // B = J A scaled by s per column; cov = B S^2 B^T
    double cxx = 0.0, cxy = 0.0, cyy = 0.0;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        double b0 = fma(q.j0, q.A[0 * 3 + k], q.j2 * q.A[2 * 3 + k]) * P.s[k];
        double b1 = fma(q.j4, q.A[1 * 3 + k], q.j5 * q.A[2 * 3 + k]) * P.s[k];
        cxx = fma(b0, b0, cxx);
        cxy = fma(b0, b1, cxy);
        cyy = fma(b1, b1, cyy);
    }
    cxx += (double)st.eps2d;
    cyy += (double)st.eps2d;
    double det = cxx * cyy - cxy * cxy;
    if (!(det > 0.0) || !isfinite(det)) return false;
    q.cxx = cxx; q.cxy = cxy; q.cyy = cyy;
    q.mx = fma(V.fx * tx, iz, V.cx);
    q.my = fma(V.fy * ty, iz, V.cy);
    double hx = sqrt(P.rho2 * cxx), hy = sqrt(P.rho2 * cyy);
    double ulo = ceil(q.mx - hx), uhi = floor(q.mx + hx);
    double vlo = ceil(q.my - hy), vhi = floor(q.my + hy);
    if (!(ulo <= uhi) || !(vlo <= vhi)) return false;
    ulo = fmax(ulo, 0.0);
    vlo = fmax(vlo, 0.0);
    uhi = fmin(uhi, (double)(V.W - 1));
    vhi = fmin(vhi, (double)(V.H - 1));
    if (ulo > uhi || vlo > vhi) return false;
    q.u0 = (int)ulo; q.u1 = (int)uhi; q.v0 = (int)vlo; q.v1 = (int)vhi;
    return true;
}


// The binary32 screen of the projection.  Camera coordinates scaled to pixels are affine in the mean,
// (U, V, z) = (fx t_x + cx t_z, fy t_y + cy t_z, t_z), taken relative to the first camera's centre, so that
// their rounding follows the spread of map and cameras and not the distance from the world's origin.  With
// a = U / z the support box's half extent is bounded above through
// Sigma_xx <= s_max^2 |J_row0|^2 = (s_max / z)^2 (fx^2 + (a - cx)^2), and below by s_min fx / z.
struct ScreenView {
    float4 u, v, z;   // coefficients of the offset from the first camera's centre, and the constant
    float4 kx, ky;    // (cx, fx^2, (W - 1) / 2, slack in pixels), (cy, fy^2, (H - 1) / 2, min(fx, fy))
};

__device__ __forceinline__ ScreenView screen_view(const ViewDev& V, const float* T0) {
    ScreenView f;
    double w[3];
#pragma unroll
    for (int k = 0; k < 3; k++) w[k] = V.T[k] - (double)T0[k];
    double U[4], Y[4], Z[4];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        U[k] = V.fx * V.R[3 * k] + V.cx * V.R[3 * k + 2];
        Y[k] = V.fy * V.R[3 * k + 1] + V.cy * V.R[3 * k + 2];
        Z[k] = V.R[3 * k + 2];
    }
    U[3] = -(U[0] * w[0] + U[1] * w[1] + U[2] * w[2]);
    Y[3] = -(Y[0] * w[0] + Y[1] * w[1] + Y[2] * w[2]);
    Z[3] = -(Z[0] * w[0] + Z[1] * w[1] + Z[2] * w[2]);
    f.u = make_float4((float)U[0], (float)U[1], (float)U[2], (float)U[3]);
    f.v = make_float4((float)Y[0], (float)Y[1], (float)Y[2], (float)Y[3]);
    f.z = make_float4((float)Z[0], (float)Z[1], (float)Z[2], (float)Z[3]);
    const float fx = fabsf(V.fxf), fy = fabsf(V.fyf), wx = (float)(V.W - 1), wy = (float)(V.H - 1);
    // a field of view beyond 71 degrees to a side or pixels far from square would spoil the bounds in the image: such
    // a view's pairs are settled by the near plane alone
    const bool plain = fx <= 2.0f * fy && fy <= 2.0f * fx && fmaxf(fabsf(V.cxf), fabsf(wx - V.cxf)) <= 3.0f * fx &&
                       fmaxf(fabsf(V.cyf), fabsf(wy - V.cyf)) <= 3.0f * fy;
    const float slack = plain ? 0.05f + 4e-4f * fmaxf(fx + 2.0f * fabsf(V.cxf), fy + 2.0f * fabsf(V.cyf)) : INFINITY;
    f.kx = make_float4(V.cxf, fx * fx, 0.5f * wx, slack);
    f.ky = make_float4(V.cyf, fy * fy, 0.5f * wy, fminf(fx, fy));
    return f;
}

// What the screen knows of a Gaussian.  z is off by less than 3.5e-7 m, m = |offset|_1 + the largest |camera
// offset|_1, and U, V by that times (f + |c|); err is 2e-6 m.  For z >= 1e3 err the pixel offset a - c is
// then off by less than 2e-4 (f + 2 |c| + |a - c|) and the extent by less than a relative 1e-3: the
// slack, 4e-4 |a - c| and 0.003 of the extent cover both.  That holds for rotations; where a camera of
// the batch has another matrix, err and hi are taken times the largest singular value and lo times the smallest.
struct ScreenGauss {
    float dx, dy, dz;  // offset from the first camera's centre
    float hi, lo;      // bounds of rho s_max and rho s_min, rho^2 = 2 ln(o / alpha_min)
    float ep;          // bound of rho^2 eps2d
    float zlo, zhi;
};

// False if the binary64 form is invalid (pre_gauss returns false).
__device__ __forceinline__ bool screen_gauss(const GaussDev& g, int64_t i, const SetDev& st, const float* T0,
                                             ScreenGauss& G) {
    const int64_t n = g.n;
    const float m0 = g.means[i], m1 = g.means[n + i], m2 = g.means[2 * n + i];
    const float op = g.opacity[i];
    const float l0 = g.log_scales[i];
    bool ok = isfinite(m0) && isfinite(m1) && isfinite(m2) && isfinite(l0) && isfinite(op) && op >= st.alpha_min;
    float lmax = l0, lmin = l0;
    if (!st.isotropic) {
        const float l1 = g.log_scales[n + i], l2 = g.log_scales[2 * n + i];
        const float q0 = g.quats[i], q1 = g.quats[n + i], q2 = g.quats[2 * n + i], q3 = g.quats[3 * n + i];
        ok = ok && isfinite(l1) && isfinite(l2) && isfinite(q0) && isfinite(q1) && isfinite(q2) && isfinite(q3) &&
             (q0 != 0.0f || q1 != 0.0f || q2 != 0.0f || q3 != 0.0f);
        lmax = fmaxf(l0, fmaxf(l1, l2));
        lmin = fminf(l0, fminf(l1, l2));
    }
    G.dx = m0 - T0[0];
    G.dy = m1 - T0[1];
    G.dz = m2 - T0[2];
    // hardware logarithm and exponential, to about 1e-6 absolute and 1e-5 relative
    const float rho2 = 1.38629436f * __builtin_amdgcn_logf(op / st.alpha_min);
    const float rho2_hi = rho2 * 1.0001f + 1e-5f, rho2_lo = fmaxf(rho2 * 0.9999f - 1e-5f, 0.0f);
    G.hi = __builtin_amdgcn_sqrtf(rho2_hi) * 1.0003f * fast_exp2(1.44269504f * lmax);
    G.lo = __builtin_amdgcn_sqrtf(rho2_lo) * 0.9997f * fast_exp2(1.44269504f * lmin);
    G.ep = rho2_hi * st.eps2d;
    return ok;
}

// culled: the binary64 projection is certain to reject the pair; certain: it is certain to keep it.  That is
// when the half extents are above 0.55 and reach half a pixel and every rounding into the image (so that
// the box holds a pixel of it), and det Sigma cannot round to zero: extents below 1.1e6 (0.03 of them
// is within the image or the lower bound) and above 0.55 keep (s_max / s_min)^2 below 4e12, so det, at least
// (s_min f / z)^2 max(Sigma_xx, Sigma_yy), is above 2e-15 Sigma_xx Sigma_yy 30 times over.
// Neither: the binary64 projection decides.
__device__ __forceinline__ void screen_pair(const ScreenGauss& G, const ScreenView& V, bool& culled, bool& certain) {
    const float z = fmaf(V.z.x, G.dx, fmaf(V.z.y, G.dy, fmaf(V.z.z, G.dz, V.z.w)));
    const float U = fmaf(V.u.x, G.dx, fmaf(V.u.y, G.dy, fmaf(V.u.z, G.dz, V.u.w)));
    const float Y = fmaf(V.v.x, G.dx, fmaf(V.v.y, G.dy, fmaf(V.v.z, G.dz, V.v.w)));
    // hardware reciprocal and square root: within an ulp or two
    const float iz = __builtin_amdgcn_rcpf(z);
    const float r = G.hi * iz, r2 = r * r;
    const float ax = U * iz, ay = Y * iz;
    const float dx = ax - V.kx.x, dy = ay - V.ky.x;
    const float hx = __builtin_amdgcn_sqrtf(fmaf(r2, fmaf(dx, dx, V.kx.y), G.ep));
    const float hy = __builtin_amdgcn_sqrtf(fmaf(r2, fmaf(dy, dy, V.ky.y), G.ep));
    const float sx = fmaf(4e-4f, fabsf(dx), V.kx.w), sy = fmaf(4e-4f, fabsf(dy), V.kx.w);
    const float gx = fabsf(ax - V.kx.z) - V.kx.z, gy = fabsf(ay - V.ky.z) - V.ky.z;  // beyond the image's edge
    const float lo = fmaf(G.lo * iz, V.ky.w, -0.56f);
    const bool far = z >= G.zhi;  // no comparison holds for a NaN: binary64 decides
    culled = (z <= G.zlo) | (far & ((fmaf(-1.003f, hx, gx) > sx) | (fmaf(-1.003f, hy, gy) > sy)));
    certain = far & (lo >= 0.0f) & (fmaf(0.03f, hx, gx) < lo - sx) & (fmaf(0.03f, hy, gy) < lo - sy);  // not inf < inf
}

// ------------------------------------------------------- support extents
// A splat's support {alpha >= alpha_min} in the whitened form is
// w1^2 + w2^2 <= log2(o / alpha_min) with w1 = a dx, w2 = b dx + c dy
// (geo1 = (a, b, c, o), d = pixel - mean): the ellipse with
// Q = [[a^2 + b^2, b c], [b c, c^2]], det Q = (a c)^2.  On a horizontal
// slice at offset dy it spans dx = (-B dy +/- sqrt(A l - D dy^2)) / A
// (A = a^2 + b^2, B = b c, D = det Q).  The right end is concave in dy with
// its maximum at dy_r = -(b / (a c)) sqrt(l), the left end convex with its
// minimum at -dy_r, so the x extent over a band of rows is the two slices at
// the offsets clamped into the band.
//
// The test is conservative in binary32: l exceeds log2(o / alpha_min) by the
// binary64 refinement band of the alpha_min test, by the binary32 rounding of
// a pixel's own exponent (which grows with |b dx| + c |dy|, bounded here
// through X and Y, the largest |dx| and |dy| in question) and by a relative
// 1e-4; the extents are widened by a relative 1e-3 plus 1e-3 pixel.
// Returns false if the rows [r0, r1] miss the support.
// m = (a, b, c, log2 o).
__device__ __forceinline__ bool support_span(float mx, float my, float4 m, float log2_amin, float X, int r0, int r1,
                                             float& xl, float& xr) {
    const float a = m.x, b = m.y, c = m.z;
    const float dy0 = (float)r0 - my, dy1 = (float)r1 - my;
    const float Y = fmaxf(fabsf(dy0), fabsf(dy1));
    const float l = (m.w - log2_amin) * 1.0001f + 0.004f + 4e-7f * fmaf(fabsf(b), X, c * Y);
    const float A = fmaf(a, a, b * b);
    const float ac = a * c;
    if (!(A > 0.0f) || !(ac > 0.0f) || !(l > 0.0f) || !(A < 3e38f)) {  // not expected: no culling
        xl = -3e38f;
        xr = 3e38f;
        return true;
    }
    const float D = ac * ac;
    const float B = b * c;
    const float dyr = -b * __builtin_amdgcn_rcpf(ac) * __builtin_amdgcn_sqrtf(l);
    const float yr = fminf(fmaxf(dyr, dy0), dy1);
    const float yl = fminf(fmaxf(-dyr, dy0), dy1);
    const float Al = A * l;
    const float dr = fmaf(-D * yr, yr, Al);
    const float dl = fmaf(-D * yl, yl, Al);
    if (dr < -1e-4f * Al) return false;
    const float ia = __builtin_amdgcn_rcpf(A);
    const float R = (__builtin_amdgcn_sqrtf(fmaxf(dr, 0.0f)) - B * yr) * ia;
    const float L = (-__builtin_amdgcn_sqrtf(fmaxf(dl, 0.0f)) - B * yl) * ia;
    const float mg = 1e-3f * (fabsf(R) + fabsf(L)) + 1e-3f;
    xl = mx + L - mg;
    xr = mx + R + mg;
    return true;
}

// Whether a splat's support can reach a pixel of the rectangle [c0, c1] x
// [r0, r1] (a prefilter; the per-pixel tests decide).  The mean (mx, my) and
// the rectangle are in any common pixel frame.
__device__ __forceinline__ bool support_meets_rect(float mx, float my, float4 m, float log2_amin, int c0, int c1, int r0,
                                                   int r1) {
    const float X = fmaxf(fabsf((float)c0 - mx), fabsf((float)c1 - mx));
    float xl, xr;
    if (!support_span(mx, my, m, log2_amin, X, r0, r1, xl, xr)) return false;
    return xl <= (float)c1 && xr >= (float)c0;
}

// Per-record constants of the support rows: on a slice at offset dy the
// ellipse spans [-sqrt(P - Qc dy^2) - Bc dy, sqrt(P - Qc dy^2) - Bc dy]
// (P = l / A, Qc = D / A^2, Bc = B / A in the notation of support_span), l
// taken with X and Y bounding |dx| and |dy| over the whole pixel box.
struct SupportRows {
    float mx, my, dyr, P, Qc, Bc;
    uint32_t pb_x, pb_y;  // pixel box
    int all;              // 1: no culling (degenerate form, not expected)
};

// Pair counting and pair emission both evaluate support_setup and support_row on the same stored record values
// (geo0, geo1, pixel box); the code is compiled without contraction and reassociation, so they agree exactly.
__device__ __forceinline__ SupportRows support_setup(float4 g0, float4 g1, uint2 pb, float log2_amin) {
    SupportRows S;
    const float a = g1.x, b = g1.y, c = g1.z;
    S.mx = g0.x + g0.z;
    S.my = g0.y + g0.w;
    S.pb_x = pb.x;
    S.pb_y = pb.y;
    const float u0 = (float)(pb.x & 0xffffu), u1 = (float)(pb.x >> 16);
    const float v0 = (float)(pb.y & 0xffffu), v1 = (float)(pb.y >> 16);
    const float X = fmaxf(fabsf(u0 - S.mx), fabsf(u1 - S.mx));
    const float Y = fmaxf(fabsf(v0 - S.my), fabsf(v1 - S.my));
    const float l = (__builtin_amdgcn_logf(g1.w) - log2_amin) * 1.0001f + 0.004f + 4e-7f * fmaf(fabsf(b), X, c * Y);
    const float A = fmaf(a, a, b * b);
    const float ac = a * c;
    S.all = !(A > 0.0f) || !(ac > 0.0f) || !(l > 0.0f) || !(A < 3e38f);
    const float ia = __builtin_amdgcn_rcpf(A);
    S.dyr = -b * __builtin_amdgcn_rcpf(ac) * __builtin_amdgcn_sqrtf(l);
    S.P = l * ia;
    S.Qc = (ac * ia) * (ac * ia);
    S.Bc = (b * c) * ia;
    return S;
}

// Tiles of tile row ty (tiles 2^tws x 2^ths) that a record's support meets
// inside its pixel box, as (first column, count).
__device__ __forceinline__ uint2 support_row(const SupportRows& S, uint32_t ty, int tws, int ths) {
    const int u0 = (int)(S.pb_x & 0xffffu), u1 = (int)(S.pb_x >> 16);
    const int v0 = (int)(S.pb_y & 0xffffu), v1 = (int)(S.pb_y >> 16);
    const int y0 = max((int)(ty << ths), v0), y1 = min((int)((ty + 1) << ths) - 1, v1);
    const uint32_t f0 = (uint32_t)u0 >> tws;
    if (y0 > y1) return make_uint2(f0, 0u);
    if (S.all) return make_uint2(f0, ((uint32_t)u1 >> tws) - f0 + 1);
    const float dy0 = (float)y0 - S.my, dy1 = (float)y1 - S.my;
    const float yr = fminf(fmaxf(S.dyr, dy0), dy1);
    const float yl = fminf(fmaxf(-S.dyr, dy0), dy1);
    const float er = fmaf(-S.Qc * yr, yr, S.P);
    const float el = fmaf(-S.Qc * yl, yl, S.P);
    if (er < -1e-4f * S.P) return make_uint2(f0, 0u);  // the rows miss the support
    const float R = __builtin_amdgcn_sqrtf(fmaxf(er, 0.0f)) - S.Bc * yr;
    const float L = -__builtin_amdgcn_sqrtf(fmaxf(el, 0.0f)) - S.Bc * yl;
    const float mg = 1e-3f * (fabsf(R) + fabsf(L)) + 1e-3f;
    const float cl = fmaxf(ceilf(S.mx + L - mg), (float)u0);
    const float cr = fminf(floorf(S.mx + R + mg), (float)u1);
    if (!(cl <= cr)) return make_uint2(f0, 0u);
    const uint32_t first = (uint32_t)cl >> tws;
    return make_uint2(first, ((uint32_t)cr >> tws) - first + 1);
}

// Few views (one word of them): a thread per Gaussian forms its binary64 form, screens the views and decides each
// candidate.  The line to the queued kernel below: at 1 and 8 views this one took 9 and 57 us (200 k and 1 M
// Gaussians), the queue 18 and 75 (its second reading of a Gaussian is not shared by enough views); at
// 64 and 256 views (500 k and 2 M) this way took 135 and 1,460 us, the queue 94 and 1,040.
constexpr int PC_FEW = 32;

__global__ __launch_bounds__(256) void k_project_count(GaussDev g, const ViewDev* __restrict__ views,
                                                       const Header* __restrict__ hdr, SetDev st,
                                                       uint32_t* __restrict__ cnt, uint32_t* __restrict__ mask,
                                                       uint32_t* __restrict__ zero, int n_zero) {
    if (blockIdx.x == 0 && (int)threadIdx.x < n_zero) zero[threadIdx.x] = 0u;
    // the cameras' test values, staged in LDS (every thread reads the same camera at a time)
    __shared__ CullView s_vf[PC_FEW];
    const int nv = min((int)hdr->n_views, PC_FEW);
    if ((int)threadIdx.x < nv) s_vf[threadIdx.x] = cull_view(views[threadIdx.x], st);
    __syncthreads();
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    GPre P;
    uint32_t vis = 0;
    if (pre_gauss(g, i, st, P)) {
        uint32_t cand = 0;
        for (int b = 0; b < nv; b++)
            if (may_be_visible(P, s_vf[b], st)) cand |= 1u << b;
        while (cand) {
            int b = __ffs(cand) - 1;
            cand &= cand - 1;
            GProj q;
            if (project_exact(P, load_cam(views + b), st, q)) vis |= 1u << b;
        }
    }
    mask[i] = vis;
    cnt[i] = __popc(vis);
}

// Visible views of every Gaussian, as bits (mask[word][Gaussian]) and a count.  VIEWS cameras at a time lie in
// LDS; the binary32 screen settles most pairs (98% of 2 M Gaussians in 256 views; 7% are visible), and the rest
// go through a queue of the wave, so that the binary64 projection runs on 64 pairs at once instead of on the one or two
// lanes of a wave whose pair is open.  Bound by the screen's instructions (about 50 per 64 pairs, two pairs
// a lane in flight) and, at four waves per SIMD (128 VGPRs, 8 spilled), by the latency of the binary64 part: 2 M Gaussians
// in 256 views 1,020 us (970 with bounds that held for rotations alone).
constexpr int PC_VIEWS = 256;
constexpr int PC_STEP = 2;

// The binary64 decision.  Not inlined: its registers and constants stay out of the screen's loop.
__device__ __noinline__ bool pair_visible(const GaussDev& g, int64_t i, const ViewDev* V, const SetDev& st) {
    GPre P;
    GProj q;
    return pre_gauss(g, i, st, P) && project_exact(P, load_cam(V), st, q);
}

template <int VIEWS, int NT>
__global__ __launch_bounds__(NT, 4) void k_project_count_queued(GaussDev g, const ViewDev* __restrict__ views,
                                                         const Header* __restrict__ hdr, int words, SetDev st,
                                                         uint32_t* __restrict__ cnt, uint32_t* __restrict__ mask,
                                                         uint32_t* __restrict__ zero, int n_zero) {
    if (blockIdx.x == 0 && (int)threadIdx.x < n_zero) zero[threadIdx.x] = 0u;
    static_assert(VIEWS <= NT && VIEWS % 32 == 0 && VIEWS <= 256, "a thread stages a camera; a queue entry holds 8 bits of it");
    __shared__ ScreenView s_v[VIEWS];
    __shared__ uint32_t s_vis[VIEWS / 32][NT];
    __shared__ uint16_t s_q[NT / 64][64 * (PC_STEP + 1)];  // lane | view << 6
    // bits of the largest |camera offset|_1 and of the cameras' largest and smallest singular value
    __shared__ uint32_t s_spread, s_hi, s_lo;
    const int nv = (int)hdr->n_views;
    const int tid = threadIdx.x, wv = tid >> 6, lane = (int)lane_id();
    const int64_t i0 = (int64_t)blockIdx.x * NT + 64 * wv, i = i0 + lane;
    float T0[3] = {0.0f, 0.0f, 0.0f};
    if (nv > 0)
#pragma unroll
        for (int k = 0; k < 3; k++) T0[k] = views[0].Tf[k];
    ScreenGauss G{};
    const bool ok = i < g.n && screen_gauss(g, i, st, T0, G);
    const float hi1 = G.hi, lo1 = G.lo;
    uint32_t c = 0;
    for (int base = 0; base < 32 * words; base += VIEWS) {
        const int lim = max(0, min(VIEWS, nv - base));
        if (tid == 0) {
            s_spread = s_hi = 0u;
            s_lo = 0x7f800000u;
        }
        __syncthreads();
        if (tid < lim) {
            const ViewDev& V = views[base + tid];
            s_v[tid] = screen_view(V, T0);
            atomicMax(&s_spread, __float_as_uint(fabsf(V.Tf[0] - T0[0]) + fabsf(V.Tf[1] - T0[1]) + fabsf(V.Tf[2] - T0[2])));
            const float2 norms = camera_norms(V);
            atomicMax(&s_hi, __float_as_uint(norms.x));
            atomicMin(&s_lo, __float_as_uint(norms.y));
        }
        __syncthreads();
        const float norm = __uint_as_float(s_hi);
        const float err = 2e-6f * norm * (fabsf(G.dx) + fabsf(G.dy) + fabsf(G.dz) + __uint_as_float(s_spread));
        if (!st.isotropic) {  // the isotropic extent does not see the matrix
            G.hi = hi1 * norm;
            G.lo = lo1 * __uint_as_float(s_lo);
        }
        G.zlo = st.z_near - err;
        G.zhi = fmaxf(st.z_near + err, 1e3f * err);
        uint32_t nq = 0;  // queued pairs of the wave
        for (int w = 0; 32 * w < lim; w++) {
            s_vis[w][tid] = 0u;
            uint32_t vis = 0;
            const int n = min(32, lim - 32 * w);
            for (int b = 0; b < n; b += PC_STEP) {
                // the screens of a step first: independent work that hides its latencies
                bool culled[PC_STEP], certain[PC_STEP];
#pragma unroll
                for (int k = 0; k < PC_STEP; k++) screen_pair(G, s_v[32 * w + b + k], culled[k], certain[k]);
#pragma unroll
                for (int k = 0; k < PC_STEP; k++) {
                    const bool here = ok & (b + k < n);
                    vis |= here & certain[k] ? 1u << (b + k) : 0u;
                    const bool open = here & !culled[k] & !certain[k];
                    const uint64_t m = __ballot(open);
                    if (open) s_q[wv][nq + (uint32_t)__popcll(m & lanemask_lt())] = (uint16_t)(lane | (32 * w + b + k) << 6);
                    nq += (uint32_t)__popcll(m);
                }
                const bool last = 32 * w + b + PC_STEP >= lim;
                while (nq >= 64u || (last && nq > 0u)) {
                    const uint32_t take = min(nq, 64u);
                    wave_lds_order();
                    uint32_t e = 0;
                    uint32_t rest[PC_STEP];
#pragma unroll
                    for (int k = 0; k < PC_STEP; k++) rest[k] = s_q[wv][64 * (k + 1) + lane];
                    e = s_q[wv][lane];
                    const uint32_t src = e & 63u, v = e >> 6;
                    if ((uint32_t)lane < take && pair_visible(g, i0 + src, views + base + v, st))
                        atomicOr(&s_vis[v >> 5][64 * wv + src], 1u << (v & 31));
                    wave_lds_order();
#pragma unroll
                    for (int k = 0; k < PC_STEP; k++) s_q[wv][64 * k + lane] = (uint16_t)rest[k];
                    nq -= take;
                }
            }
            atomicOr(&s_vis[w][tid], vis);
        }
        wave_lds_order();
        for (int w = 0; w < VIEWS / 32 && base / 32 + w < words; w++) {
            const uint32_t vis = 32 * w < lim ? s_vis[w][tid] : 0u;
            if (i < g.n) mask[(int64_t)(base / 32 + w) * g.n + i] = vis;
            c += __popc(vis);
        }
        __syncthreads();
    }
    if (i < g.n) cnt[i] = c;
}

// -------------------------------------------------------------- prefix sum

constexpr int SC_THREADS = 256;
constexpr int SC_IPT = 8;  // two 16-byte loads per lane and tile
constexpr int SC_TILE = SC_THREADS * SC_IPT;
constexpr int SC_MAX_BLOCKS = 1024;

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    uint32_t l = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(v, o, 64);
        if (l >= (uint32_t)o) v += y;
    }
    return v;
}

// Exclusive scan of one value per thread over a 256-thread block.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* ws, uint32_t& total) {
    uint32_t inc = wave_incl_scan(x);
    int wv = threadIdx.x >> 6;
    if (lane_id() == 63) ws[wv] = inc;
    __syncthreads();
    uint32_t base = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < SC_THREADS / 64; k++) {
        uint32_t t = ws[k];
        if (k < wv) base += t;
        total += t;
    }
    __syncthreads();
    return base + inc - x;
}

__device__ __forceinline__ void chunk_of(uint32_t n, int nblocks, uint32_t& begin, uint32_t& end) {
    uint32_t per = (uint32_t)(((uint64_t)n + nblocks - 1) / nblocks);
    per = (per + SC_TILE - 1) / SC_TILE * SC_TILE;
    uint64_t b = (uint64_t)blockIdx.x * per;
    begin = (uint32_t)min<uint64_t>(b, n);
    end = (uint32_t)min<uint64_t>(b + per, n);
}

// Items [at, at + 4) and [at + gap, at + gap + 4), 0 from `end` on; at and gap are multiples of four and the array is
// 16-byte aligned.
__device__ __forceinline__ void scan_load(const uint32_t* in, uint32_t at, uint32_t gap, uint32_t end, uint32_t (&v)[8]) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const uint32_t i = at + h * gap;
        uint4 q = make_uint4(0u, 0u, 0u, 0u);
        if ((uint64_t)i + 4 <= end) {
            q = *reinterpret_cast<const uint4*>(in + i);
        } else {
            if (i < end) q.x = in[i];
            if ((uint64_t)i + 1 < end) q.y = in[i + 1];
            if ((uint64_t)i + 2 < end) q.z = in[i + 2];
        }
        v[4 * h] = q.x;
        v[4 * h + 1] = q.y;
        v[4 * h + 2] = q.z;
        v[4 * h + 3] = q.w;
    }
}

// Multi-block exclusive scan of n = min(*n_dev, cap) items (n = cap when n_dev is
// null): per-block totals here, then k_scan_down.  34 M counts: 86 + 134 us with 4-byte loads and stores of eight
// consecutive items per lane, 36 + 48 with 16-byte ones.  Totals are formed in 64 bits; a block total is stored
// saturated at SCAN_LIMIT, so that k_scan_down can tell a sum of 2^31 or more
// from one that merely wrapped.
constexpr uint64_t SCAN_LIMIT = 0x80000000ull;

__device__ __forceinline__ uint64_t block_sum64(uint64_t x, uint64_t* ws) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += (uint64_t)__shfl_xor((unsigned long long)x, o, 64);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = x;
    __syncthreads();
    uint64_t t = 0;
#pragma unroll
    for (int k = 0; k < SC_THREADS / 64; k++) t += ws[k];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(SC_THREADS) void k_scan_reduce(const uint32_t* __restrict__ in,
                                                            const uint32_t* __restrict__ n_dev,
                                                            uint32_t cap, uint32_t* __restrict__ partial) {
    __shared__ uint64_t ws[SC_THREADS / 64];
    const uint32_t n = n_dev ? min(*n_dev, cap) : cap;
    uint32_t begin, end;
    chunk_of(n, gridDim.x, begin, end);
    uint64_t acc = 0;
    // a tile (begin is a multiple of one) as two 16-byte loads per lane
    for (uint32_t t0 = begin; t0 < end; t0 += SC_TILE) {
        uint32_t v[SC_IPT];
        scan_load(in, t0 + 4 * threadIdx.x, 4 * SC_THREADS, end, v);
#pragma unroll
        for (int j = 0; j < SC_IPT; j++) acc += v[j];
    }
    const uint64_t total = block_sum64(acc, ws);
    if (threadIdx.x == 0) partial[blockIdx.x] = (uint32_t)min(total, SCAN_LIMIT);
}


// What a scan leaves beside the offsets (all nullable): the total, on the device and in pinned host memory
// with the flags word (mirror[0], mirror[1]; a copy would be a launch of its own), and for the records of each Gaussian
// the owners of the chunk ends (chunk_owners).
struct ScanOut {
    uint32_t* total;
    uint32_t* flags;
    uint32_t* mirror;
    uint32_t* chunk_g;
    uint32_t rec_cap;
};

// The Gaussians that own the first and the last record of every chunk of
// PE_CHUNK records (chunk_g[2c], chunk_g[2c + 1]): each Gaussian i, of c records from a, writes the
// chunk ends that fall among its records, so every entry has one writer.
// Record p is owned by the Gaussian i with rec_off[i] <= p < rec_off[i] +
// cnt[i], which is the last Gaussian whose first record is at or before p.
__device__ __forceinline__ void chunk_owners(uint32_t i, uint32_t a, uint32_t c, uint32_t R, uint32_t* chunk_g) {
    if (c == 0 || a >= R) return;
    const uint32_t b = (uint32_t)min<uint64_t>((uint64_t)a + c, R);  // records [a, b)
    for (uint32_t k = a / PE_CHUNK; k <= (b - 1) / PE_CHUNK; k++) {
        const uint32_t first = k * PE_CHUNK;
        const uint32_t last = (uint32_t)min<uint64_t>((uint64_t)first + PE_CHUNK - 1, R - 1);
        if (first >= a) chunk_g[2 * k] = i;
        if (last < b) chunk_g[2 * k + 1] = i;
    }
}

// partial[b] holds block b's total (k_scan_reduce); each block adds up the
// totals before it, and block 0 writes the grand total.  Without partial a single block adds up its
// items itself.
// A grand total of 2^31 or more is not representable by the 32-bit offsets:
// then the total is 0, flags gets FLAG_COUNT_OVERFLOW and nothing is
// written to out, so every consumer of the total sees an empty list.
// in and out may be the same array (each item is read and written by one thread).
__global__ __launch_bounds__(SC_THREADS) void k_scan_down(const uint32_t* in, uint32_t* out,
                                                          const uint32_t* __restrict__ n_dev, uint32_t cap,
                                                          const uint32_t* __restrict__ partial, ScanOut o) {
    __shared__ uint32_t ws[SC_THREADS / 64];
    __shared__ uint64_t ws64[SC_THREADS / 64];
    const uint32_t n = n_dev ? min(*n_dev, cap) : cap;
    uint32_t begin, end;
    chunk_of(n, gridDim.x, begin, end);
    uint64_t before = 0, all = 0;
    if (partial) {
        for (uint32_t t = threadIdx.x; t < gridDim.x; t += SC_THREADS) {
            const uint64_t p = partial[t];
            all += p;
            before += t < blockIdx.x ? p : 0u;
        }
    } else {
        for (uint32_t i = begin + threadIdx.x; i < end; i += SC_THREADS) all += in[i];
    }
    uint32_t run = (uint32_t)block_sum64(before, ws64);
    all = block_sum64(all, ws64);
    const bool over = all >= SCAN_LIMIT;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint32_t total = over ? 0u : (uint32_t)all;
        if (o.total) *o.total = total;
        if (o.flags && over) atomicOr(o.flags, FLAG_COUNT_OVERFLOW);
        if (o.mirror) {
            __hip_atomic_store(o.mirror, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(o.mirror + 1, (over ? FLAG_COUNT_OVERFLOW : 0u) | (o.flags ? *o.flags : 0u), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    if (over) return;
    const uint32_t R = (uint32_t)min<uint64_t>(all, o.rec_cap);
    for (uint32_t t0 = begin; t0 < end; t0 += SC_TILE) {
        // thread owns SC_IPT consecutive items
        uint32_t v[SC_IPT];
        uint32_t first = t0 + threadIdx.x * SC_IPT;
        uint32_t sum = 0;
        scan_load(in, first, 4, end, v);
#pragma unroll
        for (int j = 0; j < SC_IPT; j++) sum += v[j];
        uint32_t total;
        uint32_t ex = block_excl_scan(sum, ws, total) + run;
        uint32_t e[SC_IPT];
#pragma unroll
        for (int j = 0; j < SC_IPT; j++) {
            e[j] = ex;
            if (o.chunk_g && first + j < end) chunk_owners(first + j, ex, v[j], R, o.chunk_g);
            ex += v[j];
        }
#pragma unroll
        for (int h = 0; h < SC_IPT; h += 4) {
            if ((uint64_t)first + h + 4 <= end) {
                *reinterpret_cast<uint4*>(out + first + h) = make_uint4(e[h], e[h + 1], e[h + 2], e[h + 3]);
            } else {
#pragma unroll
                for (int j = h; j < h + 4; j++)
                    if (first + j < end) out[first + j] = e[j];
            }
        }
        run += total;
    }
}

// ------------------------------------------------------------- radix sort
// Stable LSD sort with digits of up to 8 bits.  A fixed grid of blocks splits the input into equal chunks; per
// pass: per-block digit histograms (upsweep, one LDS atomic add per item into per-wave tables), the offsets of
// every (digit, block), and a scatter in which every wave ranks its items with 64-lane ballots (peers with the
// same digit), preserving input order within the block; the block then sorts its tile in LDS and writes each
// digit's run from consecutive lanes.  Up to RS_FUSED_BLOCKS blocks add up their offsets themselves from the
// block-major table (5.6 us for the scatter of 2 k items, launch included); for more blocks k_rs_columns scans a
// digit-major table: 196 blocks that each read the whole table took 13.7 us, with the third launch 4.4 + 7.5.
//
// Items per lane and tile: 16 on large inputs (a digit's run per step is twice as long as with 8, so fewer of
// the scatter's writes are partial cache lines: measured 3% faster on 192 M pairs, 6% on 40 M); 4 or 8 where
// those fit RS_MAX_BLOCKS blocks, because a pass over a small input is a chain of latencies (1.0 M pairs: 16 per lane
// 16.3 us a scatter, 8 11.3; 1.5 M: 17.9 and 12.6; 200 k: 15 and, with 4, 7.5).  Inputs of at least RS_BIG_ITEMS
// take blocks of 512 threads (runs twice as long again); smaller ones keep 256, which gives them twice as many blocks.
constexpr int RS_THREADS = 256;
constexpr int RS_THREADS_BIG = 512;
constexpr int RS_IPT = 16;
constexpr int RS_MAX_BLOCKS = 1024;
constexpr uint64_t RS_BIG_ITEMS = (uint64_t)RS_MAX_BLOCKS * RS_THREADS_BIG * RS_IPT;
constexpr int RS_FUSED_BLOCKS = 32;
constexpr int RS_DB = 8;

__device__ __forceinline__ uint64_t digit_peers(uint32_t d, uint64_t valid) {
    uint64_t m = valid;
#pragma unroll
    for (int b = 0; b < RS_DB; b++) {
        uint32_t bit = (d >> b) & 1u;
        uint64_t bal = __ballot(bit);
        m &= bit ? bal : ~bal;
    }
    return m;
}

template <int TILE>
__device__ __forceinline__ void rs_chunk(uint32_t n, uint32_t& begin, uint32_t& end) {
    uint32_t per = (uint32_t)(((uint64_t)n + gridDim.x - 1) / gridDim.x);
    per = (per + TILE - 1) / TILE * TILE;
    uint64_t b = (uint64_t)blockIdx.x * per;
    begin = (uint32_t)min<uint64_t>(b, n);
    end = (uint32_t)min<uint64_t>(b + per, n);
}

// Exclusive sum over the NT threads of a block.
template <int NT>
__device__ __forceinline__ uint32_t rs_block_excl(uint32_t x, uint32_t* ws) {
    const uint32_t inc = wave_incl_scan(x);
    const int wv = threadIdx.x >> 6;
    if (lane_id() == 63) ws[wv] = inc;
    __syncthreads();
    uint32_t base = inc - x;
#pragma unroll
    for (int w = 0; w < NT / 64; w++)
        if (w < wv) base += ws[w];
    __syncthreads();
    return base;
}

// Digit of this pass: `bits` (<= RS_DB) bits from `shift`.
// hist layout: block-major [block][d] when block_major, digit-major [d][block] otherwise.
template <int NT, int IPT>
__global__ __launch_bounds__(NT) void k_rs_upsweep(const uint32_t* __restrict__ keys,
                                                   const uint32_t* __restrict__ n_dev, uint32_t cap, int shift,
                                                   int bits, uint32_t* __restrict__ hist, int block_major) {
    constexpr int NB = 1 << RS_DB;
    constexpr int WAVES = NT / 64, TILE = NT * IPT;
    // each wave counts into CP copies of its table (lane l into copy l % CP),
    // so that a skewed digit (few tiles or views dominating a pass) does not
    // serialise a whole wave's atomics on one LDS word
    constexpr int CP = 4;
    __shared__ uint32_t h[WAVES * CP][NB];
    const int tid = threadIdx.x, wv = tid >> 6;
    const int cp = wv * CP + (int)(lane_id() % CP);
    const uint32_t mask = (1u << bits) - 1u;
    for (int i = tid; i < WAVES * CP * NB; i += NT) (&h[0][0])[i] = 0;
    __syncthreads();
    uint32_t n = min(*n_dev, cap);
    uint32_t begin, end;
    rs_chunk<TILE>(n, begin, end);
    // the scatter's tiling: IPT coalesced loads per lane in flight, then
    // their IPT additions to the wave's table
    for (uint32_t t0 = begin; t0 < end; t0 += TILE) {
        const uint32_t seg = t0 + wv * (64 * IPT);
        uint32_t k[IPT];
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            const uint32_t idx = seg + j * 64 + lane_id();
            k[j] = idx < end ? keys[idx] : 0u;
        }
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            const uint32_t idx = seg + j * 64 + lane_id();
            if (idx < end) atomicAdd(&h[cp][(k[j] >> shift) & mask], 1u);
        }
    }
    __syncthreads();
    for (int d = tid; d < NB; d += NT) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < WAVES * CP; w++) c += h[w][d];
        if (block_major)
            hist[(uint64_t)blockIdx.x * NB + d] = c;
        else
            hist[(uint64_t)d * gridDim.x + blockIdx.x] = c;
    }
}

// Exclusive sums, in place, of each digit's nb <= RS_MAX_BLOCKS block counts (a block per digit), and the digit's total.
__global__ __launch_bounds__(256) void k_rs_columns(uint32_t* __restrict__ hist, int nb, uint32_t* __restrict__ totals) {
    static_assert(RS_MAX_BLOCKS == 4 * 256, "four blocks' counts per thread");
    __shared__ uint32_t ws[4];
    uint32_t* col = hist + (uint64_t)blockIdx.x * nb;
    const int i0 = 4 * (int)threadIdx.x;
    uint32_t c[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        c[j] = i0 + j < nb ? col[i0 + j] : 0u;
        sum += c[j];
    }
    uint32_t run = rs_block_excl<256>(sum, ws);
    if (threadIdx.x == 255) totals[blockIdx.x] = run + sum;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        if (i0 + j < nb) col[i0 + j] = run;
        run += c[j];
    }
}

// Values of a sort that orders the items' positions and lays out their counts in that order: the first pass makes
// them (no values are read), as the position, with the count in the spare bits above `pb` position bits (the largest
// value there stands for a count that does not fit); the last pass takes them apart, and looks up the
// few counts that did not fit.  pb = 32: no spare bits, every count is looked up.
struct RsCounts {
    const uint32_t* count;  // null: plain values
    int pb;
};

template <int NT, int IPT>
__global__ __launch_bounds__(NT, 4) void k_rs_scatter(const uint32_t* __restrict__ kin,
                                                   const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                   uint32_t* __restrict__ vout, const uint32_t* __restrict__ n_dev,
                                                   uint32_t cap, int shift, int bits,
                                                   const uint32_t* __restrict__ hist,
                                                   const uint32_t* __restrict__ totals, RsCounts rc,
                                                   uint32_t* __restrict__ gout) {
    constexpr int NB = 1 << RS_DB;
    constexpr int WAVES = NT / 64, TILE = NT * IPT;
    static_assert(NB <= NT && TILE >= 4 * NB, "a thread per digit; the staging buffer holds four partial tables");
    __shared__ uint32_t wh[WAVES][NB];
    __shared__ uint32_t bbase[NB], lst[NB], tcnt[NB];
    __shared__ uint32_t ws[WAVES];
    __shared__ uint32_t s_k[TILE], s_v[TILE];  // the tile in sorted order
    const int tid = threadIdx.x, wv = tid >> 6;
    const uint32_t lane = lane_id();
    const uint32_t mask = (1u << bits) - 1u;
    uint32_t n = min(*n_dev, cap);
    uint32_t begin, end;
    rs_chunk<TILE>(n, begin, end);
    if (begin >= end) return;
    const uint32_t sat = rc.pb < 32 ? (1u << (32 - rc.pb)) - 1u : 0u;
    uint32_t k[IPT], v[IPT];
    auto load = [&](uint32_t seg) {
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            const uint32_t idx = seg + j * 64 + lane;
            const bool valid = idx < end;
            k[j] = valid ? kin[idx] : 0u;
            if (vin) v[j] = valid ? vin[idx] : 0u;
            else v[j] = valid && rc.pb < 32 ? idx | min(rc.count[idx], sat) << rc.pb : idx;
        }
    };
    load(begin + wv * (64 * IPT));  // in flight while the offsets are formed
    // offset of digit d for this block = count of smaller digits in all blocks + count of digit d in earlier blocks
    if (totals) {
        const uint32_t base = rs_block_excl<NT>(tid < NB ? totals[tid] : 0u, ws);
        if (tid < NB) bbase[tid] = base + hist[(uint64_t)tid * gridDim.x + blockIdx.x];
    } else if constexpr (NT == NB) {
        // each wave adds up every fourth block's counts, four digits a lane, many loads in flight
        uint4 tot = make_uint4(0u, 0u, 0u, 0u), pre = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll 16
        for (uint32_t b = wv; b < gridDim.x; b += WAVES) {
            const uint4 c = *reinterpret_cast<const uint4*>(hist + (uint64_t)b * NB + 4 * lane);
            const uint32_t earlier = b < blockIdx.x ? 0xffffffffu : 0u;
            tot.x += c.x;
            tot.y += c.y;
            tot.z += c.z;
            tot.w += c.w;
            pre.x += c.x & earlier;
            pre.y += c.y & earlier;
            pre.z += c.z & earlier;
            pre.w += c.w & earlier;
        }
        reinterpret_cast<uint4*>(&wh[wv][0])[lane] = tot;
        reinterpret_cast<uint4*>(s_k + wv * NB)[lane] = pre;
        __syncthreads();
        uint32_t t = 0, q = 0;
#pragma unroll
        for (int w = 0; w < WAVES; w++) {
            t += wh[w][tid];
            q += s_k[w * NB + tid];
        }
        bbase[tid] = rs_block_excl<NT>(t, ws) + q;
    }
    for (uint32_t t0 = begin; t0 < end; t0 += TILE) {
        __syncthreads();
        for (int i = tid; i < WAVES * NB; i += NT) (&wh[0][0])[i] = 0;
        __syncthreads();
        const uint32_t seg = t0 + wv * (64 * IPT);
        uint32_t pos[IPT];
        if (t0 != begin) load(seg);
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            uint32_t idx = seg + j * 64 + lane;
            bool valid = idx < end;
            uint32_t d = (k[j] >> shift) & mask;
            uint64_t vm = __ballot(valid);
            uint64_t m = digit_peers(d, vm);
            uint32_t before = valid ? wh[wv][d] : 0u;
            pos[j] = before + (uint32_t)__popcll(m & lanemask_lt());
            if (valid && lane == (uint32_t)__builtin_ctzll(m)) wh[wv][d] = before + (uint32_t)__popcll(m);
        }
        __syncthreads();
        // per digit: the waves' offsets inside the tile's run of the digit, and the run's length and start
        uint32_t run = 0;
        if (tid < NB) {
#pragma unroll
            for (int w = 0; w < WAVES; w++) {
                uint32_t c = wh[w][tid];
                wh[w][tid] = run;
                run += c;
            }
            tcnt[tid] = run;
        }
        const uint32_t start = rs_block_excl<NT>(run, ws);
        if (tid < NB) lst[tid] = start;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            uint32_t idx = seg + j * 64 + lane;
            if (idx < end) {
                uint32_t d = (k[j] >> shift) & mask;
                const uint32_t lp = lst[d] + wh[wv][d] + pos[j];
                s_k[lp] = k[j];
                s_v[lp] = v[j];
            }
        }
        __syncthreads();
        const uint32_t tn = min<uint32_t>(TILE, end - t0);
        for (uint32_t i = tid; i < tn; i += NT) {
            const uint32_t kk = s_k[i];
            const uint32_t d = (kk >> shift) & mask;
            const uint32_t dst = bbase[d] + (i - lst[d]);
            uint32_t vv = s_v[i];
            if (kout) kout[dst] = kk;
            if (gout) {
                uint32_t c = sat;
                if (rc.pb < 32) {
                    c = vv >> rc.pb;
                    vv &= (1u << rc.pb) - 1u;
                }
                gout[dst] = c == sat ? rc.count[vv] : c;
            }
            vout[dst] = vv;
        }
        __syncthreads();
        if (tid < NB) bbase[tid] += tcnt[tid];
    }
}

// The whole sort of up to RS_ONE items in one block: every pass ranks as above and moves the items through LDS.
constexpr int RS_ONE_THREADS = 1024, RS_ONE_IPT = 4;
constexpr uint32_t RS_ONE = RS_ONE_THREADS * RS_ONE_IPT;

__global__ __launch_bounds__(RS_ONE_THREADS) void k_rs_one(const uint32_t* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin,
                                                           uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                           const uint32_t* __restrict__ n_dev, uint32_t cap, int nbits,
                                                           const uint32_t* __restrict__ count,
                                                           uint32_t* __restrict__ gout) {
    constexpr int NB = 1 << RS_DB, WAVES = RS_ONE_THREADS / 64, IPT = RS_ONE_IPT;
    __shared__ uint32_t wh[WAVES][NB];
    __shared__ uint32_t ws[WAVES];
    __shared__ uint32_t s_k[RS_ONE], s_v[RS_ONE];
    const int tid = threadIdx.x, wv = tid >> 6;
    const uint32_t lane = lane_id(), n = min(min(*n_dev, cap), RS_ONE), seg = wv * (64 * IPT);
    uint32_t k[IPT], v[IPT], pos[IPT];
#pragma unroll
    for (int j = 0; j < IPT; j++) {
        const uint32_t idx = seg + j * 64 + lane;
        k[j] = idx < n ? kin[idx] : 0u;
        v[j] = count ? idx : idx < n ? vin[idx] : 0u;
    }
    for (int shift = 0; shift < nbits; shift += RS_DB) {
        const uint32_t mask = (1u << min(RS_DB, nbits - shift)) - 1u;
        for (int i = tid; i < WAVES * NB; i += RS_ONE_THREADS) (&wh[0][0])[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            const bool valid = seg + j * 64 + lane < n;
            const uint32_t d = (k[j] >> shift) & mask;
            const uint64_t m = digit_peers(d, __ballot(valid));
            const uint32_t before = valid ? wh[wv][d] : 0u;
            pos[j] = before + (uint32_t)__popcll(m & lanemask_lt());
            if (valid && lane == (uint32_t)__builtin_ctzll(m)) wh[wv][d] = before + (uint32_t)__popcll(m);
        }
        __syncthreads();
        uint32_t run = 0;
        if (tid < NB)
#pragma unroll
            for (int w = 0; w < WAVES; w++) run += wh[w][tid];
        uint32_t at = rs_block_excl<RS_ONE_THREADS>(run, ws);
        if (tid < NB)
#pragma unroll
            for (int w = 0; w < WAVES; w++) {
                const uint32_t c = wh[w][tid];
                wh[w][tid] = at;
                at += c;
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; j++)
            if (seg + j * 64 + lane < n) {
                const uint32_t lp = wh[wv][(k[j] >> shift) & mask] + pos[j];
                s_k[lp] = k[j];
                s_v[lp] = v[j];
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; j++) {
            const uint32_t idx = seg + j * 64 + lane;
            k[j] = idx < n ? s_k[idx] : 0u;
            v[j] = idx < n ? s_v[idx] : 0u;
        }
    }
#pragma unroll
    for (int j = 0; j < IPT; j++) {
        const uint32_t idx = seg + j * 64 + lane;
        if (idx < n) {
            kout[idx] = k[j];
            vout[idx] = v[j];
            if (gout) gout[idx] = count[v[j]];
        }
    }
}

// ---------------------------------------------------------------- binning

__device__ __forceinline__ uint32_t last_le(const uint32_t* a, uint32_t n, uint32_t x) {
    // largest i < n with a[i] <= x (a[0] == 0 <= x)
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        uint32_t mid = lo + (hi - lo + 1) / 2;
        if (a[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The same search over global memory by one wave in 64-way steps: the lanes
// probe 64 evenly spaced positions of the current range; the probes with
// a[p] <= x form a prefix of the lanes (a is non-decreasing), so their count
// narrows the range 64-fold per step.  All values are wave-uniform.
__device__ __forceinline__ uint32_t wave_last_le(const uint32_t* __restrict__ a, uint32_t n, uint32_t x) {
    uint32_t lo = 0, hi = n - 1;  // a[lo] <= x; the answer lies in [lo, hi]
    const uint32_t lane = lane_id();
    while (hi > lo) {
        const uint32_t step = (hi - lo + 63) / 64;
        const uint64_t p = (uint64_t)lo + (uint64_t)step * (lane + 1);
        const bool le = p <= hi && a[p] <= x;
        const uint32_t c = (uint32_t)__popcll(__ballot(le));
        const uint32_t nlo = lo + step * c;
        hi = (uint32_t)min<uint64_t>(hi, (uint64_t)lo + (uint64_t)step * (c + 1) - 1);
        lo = nlo;
    }
    return lo;
}

// The tile rows of a wave's records, laid out one after another and taken 64 at a time, a lane a row.  A
// record's support constants wait in LDS at its rank among the records that have rows.
struct RowRec {
    float4 s0;   // mx, my, dyr, P
    float4 s1;   // Qc, Bc, pixel box
};

__device__ __forceinline__ RowRec row_rec(const SupportRows& S) {
    return {make_float4(S.mx, S.my, S.dyr, S.P), make_float4(S.Qc, S.Bc, __uint_as_float(S.pb_x), __uint_as_float(S.pb_y))};
}

__device__ __forceinline__ SupportRows support_rows(const RowRec& r) {
    SupportRows S;
    S.mx = r.s0.x;
    S.my = r.s0.y;
    S.dyr = r.s0.z;
    S.P = r.s0.w;
    S.Qc = r.s1.x;
    S.Bc = r.s1.y;
    S.pb_x = __float_as_uint(r.s1.z);
    S.pb_y = __float_as_uint(r.s1.w);
    S.all = 0;
    return S;
}

// Lanes mark positions [0, 64 W) of a window (`mark` lanes, distinct positions) and every lane gets the marks of each
// 64 as a mask: the rank of a lane's owner is then a population count, where a search would be a chain of LDS reads.
template <int W>
__device__ __forceinline__ void window_marks(uint32_t* bits, bool mark, uint32_t at, uint64_t (&m)[W]) {
    wave_lds_order();
    if (lane_id() < 2 * W) bits[lane_id()] = 0u;
    wave_lds_order();
    if (mark) atomicOr(&bits[at >> 5], 1u << (at & 31u));
    wave_lds_order();
#pragma unroll
    for (int w = 0; w < W; w++) m[w] = (uint64_t)bits[2 * w] | (uint64_t)bits[2 * w + 1] << 32;
}

__device__ __forceinline__ uint64_t lanemask_le() { return ~0ull >> (63 - lane_id()); }

// Record emission, one thread per record so that the record arrays are
// written in contiguous runs: the records of Gaussian i are rec_off[i] ...
// rec_off[i] + cnt[i] - 1, one per visible view in view order.  A block finds
// the Gaussians spanning its records with two wave searches and stages their
// offsets in LDS (a span wider than PE_LDS, i.e. a long run of culled
// Gaussians, is searched in global memory instead).
constexpr int PE_THREADS = 256;
constexpr uint32_t PE_LDS = 2048;
constexpr uint32_t PE_PRE = 64;
// Visibility mask words a record's view search loads at once.
constexpr int PE_MASK_WORDS = 8;

// Position of the k-th (from 0) set bit of x (k < popcount(x)), by halving.
__device__ __forceinline__ int nth_set_bit(uint32_t x, uint32_t k) {
    int pos = 0;
#pragma unroll
    for (int h = 16; h > 0; h >>= 1) {
        const uint32_t c = (uint32_t)__popc(x & ((1u << h) - 1u));
        const bool up = k >= c;
        k = up ? k - c : k;
        x = up ? x >> h : x;
        pos += up ? h : 0;
    }
    return pos;
}

static_assert(PE_THREADS == PE_CHUNK, "a block step of the record emission is one chunk");

// The chunk ends' owners where the record buffers are sized only after the scan.
__global__ __launch_bounds__(256) void k_chunk_owners(const uint32_t* __restrict__ cnt,
                                                      const uint32_t* __restrict__ rec_off, int64_t n,
                                                      const uint32_t* __restrict__ R_dev, uint32_t rec_cap,
                                                      uint32_t* __restrict__ chunk_g) {
    const uint32_t R = min(*R_dev, rec_cap);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        chunk_owners((uint32_t)i, rec_off[i], cnt[i], R, chunk_g);
}

// Bound by the instructions of the binary64 form (two divisions and two square roots beyond the projection's own) and
// its registers: three waves per SIMD; four spill 42 of them (1,870 -> 2,050 us).  With the rows counted by
// the wave together, where each lane walked up to four of its own and the wave the rest record by record:
// 256 views of 2 M Gaussians 2,230 -> 1,870 us, 8 frames of 1 M 141 -> 71, one of 300 k 50 -> 24.
__global__ __launch_bounds__(PE_THREADS, 3) void k_project_emit(GaussDev g, const ViewDev* __restrict__ views,
                                                             int words, SetDev st, int tws, int ths,
                                                             const uint32_t* __restrict__ mask,
                                                             const uint32_t* __restrict__ rec_off,
                                                             const uint32_t* __restrict__ R_dev, uint32_t rec_cap,
                                                             Records rec, uint32_t* __restrict__ sortkey, int write_attr,
                                                             const uint32_t* __restrict__ chunk_g,
                                                             uint32_t* __restrict__ flags) {
    __shared__ uint32_t s_off[PE_LDS];
    __shared__ GPre s_pre[PE_PRE];
    __shared__ RowRec s_rows[PE_THREADS];
    __shared__ uint2 s_row0[PE_THREADS];    // first row of the record among the wave's, its first tile row
    __shared__ uint32_t s_nt[PE_THREADS];   // pairs
    __shared__ uint32_t s_bits[PE_THREADS / 64][2];
    const int lane = (int)lane_id(), wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), wb = 64 * wv;
    const uint32_t Rall = *R_dev;
    if (blockIdx.x == 0 && threadIdx.x == 0 && Rall > rec_cap) atomicOr(flags, FLAG_REC_OVERFLOW);
    const uint32_t R = min(Rall, rec_cap);
    const uint32_t n = (uint32_t)g.n;
    for (uint32_t k0 = blockIdx.x * PE_THREADS; k0 < R; k0 += gridDim.x * PE_THREADS) {
        const uint32_t k1 = min(k0 + PE_THREADS, R);  // exclusive
        __syncthreads();
        // the Gaussians owning the chunk's first and last records
        const uint32_t lo = chunk_g[2 * (k0 / PE_CHUNK)], ng = chunk_g[2 * (k0 / PE_CHUNK) + 1] - lo + 1;
        const bool staged = ng <= PE_LDS;
        if (staged)
            for (uint32_t j = threadIdx.x; j < ng; j += PE_THREADS) s_off[j] = rec_off[lo + j];
        // the per-Gaussian part of the projection, once per Gaussian when few
        // Gaussians own the block's records (many views see each)
        const bool shared_pre = ng <= PE_PRE;
        if (shared_pre && threadIdx.x < ng) pre_gauss(g, lo + threadIdx.x, st, s_pre[threadIdx.x]);
        __syncthreads();
        const uint32_t pos = k0 + threadIdx.x;
        const bool valid = pos < k1;
        SupportRows S{};
        uint32_t ty0 = 0, nrow = 0, ntiles = 1;
        EmitRec e;
        if (valid) {
            // owner Gaussian: the last one whose first record is at or before pos
            const uint32_t ii = staged ? last_le(s_off, ng, pos) : last_le(rec_off + lo, ng, pos);
            const uint32_t i = lo + ii;
            // its (pos - rec_off[i])-th visible view; the mask words are
            // loaded eight at a time (256 views), all in flight together,
            // then scanned for the word that holds it
            uint32_t kk = pos - (staged ? s_off[ii] : rec_off[i]);
            int v = 0;
            bool found = false;
            for (int w0 = 0; w0 < words && !found; w0 += PE_MASK_WORDS) {
                uint32_t vis[PE_MASK_WORDS];
#pragma unroll
                for (int q = 0; q < PE_MASK_WORDS; q++)
                    vis[q] = w0 + q < words ? mask[(int64_t)(w0 + q) * n + i] : 0u;
                uint32_t word = 0;
                int wsel = 0;
#pragma unroll
                for (int q = 0; q < PE_MASK_WORDS; q++) {
                    const uint32_t c = (uint32_t)__popc(vis[q]);
                    const bool here = !found && kk < c;
                    word = here ? vis[q] : word;
                    wsel = here ? w0 + q : wsel;
                    kk = !found && !here ? kk - c : kk;
                    found = found || here;
                }
                if (found) v = 32 * wsel + nth_set_bit(word, kk);
            }
            GPre P;
            if (shared_pre) P = s_pre[i - lo];
            else pre_gauss(g, i, st, P);
            GProj q;
            project_exact(P, load_cam(views + v), st, q);
            float mxh = (float)q.mx, myh = (float)q.my;
            const float4 g0 = make_float4(mxh, myh, (float)(q.mx - (double)mxh), (float)(q.my - (double)myh));
            const double det = q.cxx * q.cyy - q.cxy * q.cxy;
            const double idet = 1.0 / det, icxx = 1.0 / q.cxx;
            // Sigma_2D = C C^T (Cholesky); M = sqrt(log2e / 2) C^-1 = sl [[1 / c00, 0], [-c10 / (c00 c11), 1 / c11]]
            const double sl = sqrt(0.5 * LOG2E);
            const double m11 = sl * sqrt(q.cxx * idet);
            const float4 g1 = make_float4((float)(sl * sqrt(icxx)), (float)(-q.cxy * icxx * m11), (float)m11, (float)P.o);
            rec.q64[pos] = make_double4(q.cyy * idet, -q.cxy * idet, q.cxx * idet, P.rho2);
            float depth = (float)q.t[2];
            const int64_t gi = i;
            if (write_attr) {
                if (g.colors)
                    rec.attr[pos] = make_float4(g.colors[gi], g.colors[g.n + gi], g.colors[2 * g.n + gi], depth);
                else
                    rec.attr[pos] = make_float4(0.0f, 0.0f, 0.0f, depth);
            }
            const uint32_t tx0 = (uint32_t)q.u0 >> tws, tx1 = (uint32_t)q.u1 >> tws;
            ty0 = (uint32_t)q.v0 >> ths;
            const uint32_t ty1 = (uint32_t)q.v1 >> ths;
            const uint2 pb = make_uint2((uint32_t)q.u0 | ((uint32_t)q.u1 << 16),
                                        (uint32_t)q.v0 | ((uint32_t)q.v1 << 16));
            sortkey[pos] = __float_as_uint(depth);
            S = support_setup(g0, g1, pb, st.log2_amin);
            ntiles = (tx1 - tx0 + 1) * (ty1 - ty0 + 1);
            // the only tile of a box is the record's pair in any case, and a degenerate form is not culled
            nrow = ntiles > 1u && !S.all ? ty1 - ty0 + 1 : 0u;
            e.g0 = g0;
            e.g1 = g1;
            e.pbox = pb;
            e.rect = make_uint2(tx0 | (tx1 << 16), ty0 | (ty1 << 16));
            e.view = (uint32_t)v;
            e.unc = __float_as_uint(g.uncert ? g.uncert[gi] : 0.0f);
            e.gid = i;
        }
        // the pairs of a record, the tiles its support meets: the wave takes the rows of its records 64 at a time
        // (integer counts, so their sum does not depend on the split)
        const uint64_t has = __ballot(nrow > 0u);
        if (has) {
            const uint32_t first = wave_incl_scan(nrow) - nrow;
            const uint32_t rows = (uint32_t)__builtin_amdgcn_readlane((int)(first + nrow), 63);
            const int rank = (int)__popcll(has & lanemask_lt());
            if (nrow > 0u) {
                s_rows[wb + rank] = row_rec(S);
                s_row0[wb + rank] = make_uint2(first, ty0);
                s_nt[wb + rank] = 0u;
            }
            int before = 0;  // records that start before the window
            for (uint32_t t0 = 0; t0 < rows; t0 += 64) {
                uint64_t m[1];
                window_marks<1>(s_bits[wv], nrow > 0u && first - t0 < 64u, first - t0, m);
                const int own = wb + before + (int)__popcll(m[0] & lanemask_le()) - 1;
                before += (int)__popcll(m[0]);
                if (t0 + (uint32_t)lane < rows) {
                    const uint2 r0 = s_row0[own];
                    const uint32_t n = support_row(support_rows(s_rows[own]), r0.y + (t0 + (uint32_t)lane - r0.x), tws, ths).y;
                    if (n) atomicAdd(&s_nt[own], n);
                }
            }
            wave_lds_order();
            if (nrow > 0u) {
                ntiles = s_nt[wb + rank];
                if (ntiles == 0u) {
                    // a support that meets no tile still owns one pair, its box's first tile
                    ntiles = 1u;
                    e.rect = make_uint2((e.rect.x & 0xffffu) * 0x10001u, (e.rect.y & 0xffffu) * 0x10001u);
                }
            }
            wave_lds_order();
        }
        if (valid) {
            e.ntiles = ntiles;
            rec.ntiles[pos] = ntiles;
            rec.emit[pos] = e;
        }
    }
}

// Pair emission.  A wave takes a contiguous run of the pairs and walks the depth-ordered records that own them, 64 at a
// time, a lane a record; then their tile rows, 64 at a time, a lane a row (every row of a record whose pairs are
// all the tiles of its rectangle, the support's columns of a row otherwise); then the rows' pairs, 128
// at a time, so that wide rows and tall records cost what their pairs cost.
// Nothing is staged for a whole block, so no barrier holds a wave up.  Bound by the gather of the records in depth
// order (a cache line for 64 bytes) and the pairs' stores.  192 M pairs of 256 views: 2,300 us with blocks that tabulated
// the rows of 1,024 pairs and found each pair's record and row by binary search in LDS, 1,350 now (2 x 768 MB
// written); 39.7 M pairs of 8 frames 408 -> 110; 1.0 M of one frame 17.6 -> 14.5.
constexpr int EM_THREADS = 256;
constexpr int EM_WAVES = EM_THREADS / 64;
constexpr uint32_t EM_RUN = 256;  // the smallest run of a wave
constexpr unsigned EM_BLOCKS = 16384;

struct EmitMeta {
    uint32_t tile, tiles_x;  // the rectangle's first tile; tiles per row of the view
    uint32_t tx, ty0;        // tx0 | nx << 16; first tile row, or 0xffffffff if every tile of the rectangle is a pair
};

__global__ __launch_bounds__(EM_THREADS, 6) void k_emit_instances(const uint32_t* __restrict__ order,
                                                               const uint32_t* __restrict__ R_dev, uint32_t rec_cap,
                                                               const uint32_t* __restrict__ K_dev, Records rec,
                                                               const ViewDev* __restrict__ views,
                                                               const uint32_t* __restrict__ inst_off,
                                                               int tws, int ths, float log2_amin,
                                                               uint32_t inst_cap, uint32_t* __restrict__ tile_key,
                                                               uint32_t* __restrict__ inst_rec,
                                                               uint2* __restrict__ ranges, uint32_t tiles_cap,
                                                               uint32_t* __restrict__ flags) {
    __shared__ RowRec s_rows[EM_THREADS];
    __shared__ EmitMeta s_meta[EM_THREADS];
    __shared__ uint4 s_own[EM_THREADS];   // record id, first row among the wave's, the next record's first row and first pair
    __shared__ uint4 s_run[EM_THREADS];   // rows with pairs: first pair, its tile, record id
    __shared__ uint32_t s_bits[EM_WAVES][4];
    // every tile starts empty; k_tile_ranges later fills the occupied ones
    // (nothing reads the ranges in between), and an overflow leaves them empty
    for (uint32_t t = blockIdx.x * EM_THREADS + threadIdx.x; t < tiles_cap; t += gridDim.x * EM_THREADS)
        ranges[t] = make_uint2(0u, 0u);
    if (*flags & (FLAG_REC_OVERFLOW | FLAG_COUNT_OVERFLOW)) return;
    const uint32_t R = min(*R_dev, rec_cap);
    const uint32_t Kall = *K_dev;
    if (threadIdx.x == 0 && blockIdx.x == 0 && Kall > inst_cap) atomicOr(flags, FLAG_INST_OVERFLOW);
    const uint32_t K = min(Kall, inst_cap);
    if (R == 0) return;
    const uint32_t lane = lane_id(), wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), wb = 64 * wv;
    const uint64_t waves = (uint64_t)gridDim.x * EM_WAVES;
    const uint64_t per = (((uint64_t)K + waves - 1) / waves + EM_RUN - 1) / EM_RUN * EM_RUN;
    const uint64_t w0 = ((uint64_t)blockIdx.x * EM_WAVES + wv) * per;
    const uint32_t kbeg = (uint32_t)min<uint64_t>(w0, K), kend = (uint32_t)min<uint64_t>(w0 + per, K);
    if (kbeg >= kend) return;  // no barrier below
    uint32_t base = kbeg;      // first pair of the next row
    for (uint32_t r0 = wave_last_le(inst_off, R, kbeg); r0 < R && base < kend; r0 += 64) {
        const uint32_t idx = r0 + lane;
        const uint32_t off = idx < R ? inst_off[idx] : 0xffffffffu;
        const uint32_t end = idx + 1 < R ? inst_off[idx + 1] : Kall;
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
        const bool valid = idx < R && off < kend;
        uint32_t nrow = 0;
        wave_lds_order();
        if (valid) {
            const uint32_t rid = order[idx];
            const EmitRec e = rec.emit[rid];
            const ViewDev& V = views[e.view];
            const uint32_t tx0 = e.rect.x & 0xffffu, ty0 = e.rect.y & 0xffffu;
            const uint32_t nx = (e.rect.x >> 16) - tx0 + 1;
            nrow = (e.rect.y >> 16) - ty0 + 1;
            EmitMeta md;
            md.tiles_x = (uint32_t)V.tiles_x;
            md.tile = V.tile_off + ty0 * (uint32_t)V.tiles_x;
            md.tx = tx0 | (nx << 16);
            md.ty0 = e.ntiles == nx * nrow ? 0xffffffffu : ty0;
            s_meta[wb + lane] = md;
            s_rows[wb + lane] = row_rec(support_setup(e.g0, e.g1, e.pbox, log2_amin));
            s_own[wb + lane].x = rid;
        }
        const uint32_t next = wave_incl_scan(nrow), first = next - nrow;
        if (valid) {
            s_own[wb + lane].y = first;
            s_own[wb + lane].z = next;
            s_own[wb + lane].w = end;
        }
        const uint32_t rows = (uint32_t)__builtin_amdgcn_readlane((int)next, 63);
        uint32_t before = 0;  // records that start before the window
        for (uint32_t t0 = 0; t0 < rows && base < kend; t0 += 64) {
            uint64_t m[1];
            window_marks<1>(s_bits[wv], valid && first - t0 < 64u, first - t0, m);
            const uint32_t own = wb + before + (uint32_t)__popcll(m[0] & lanemask_le()) - 1u;
            before += (uint32_t)__popcll(m[0]);
            const uint32_t t = t0 + lane;
            uint32_t n = 0, tile = 0, rid = 0, own_next = 0, own_end = 0;
            if (t < rows) {
                const EmitMeta md = s_meta[own];
                const uint4 o = s_own[own];
                rid = o.x;
                own_next = o.z;
                own_end = o.w;
                const uint32_t r = t - o.y;
                uint2 fc;
                if (md.ty0 == 0xffffffffu) fc = make_uint2(md.tx & 0xffffu, md.tx >> 16);
                else fc = support_row(support_rows(s_rows[own]), md.ty0 + r, tws, ths);
                n = fc.y;
                tile = md.tile + r * md.tiles_x + fc.x;
            }
            const uint32_t upto = wave_incl_scan(n), pos = base + upto - n;
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
            // a record's rows have to end where the next record's pairs begin
            if (t < rows && t + 1 == own_next && pos + n != own_end) atomicOr(flags, FLAG_BIN_MISMATCH);
            const uint64_t some = __ballot(n > 0u);
            if (n > 0u) s_run[wb + (uint32_t)__popcll(some & lanemask_lt())] = make_uint4(pos, tile, rid, 0u);
            const uint32_t p1 = min(base + total, kend);
            for (uint32_t p0 = max(base, kbeg); p0 < p1; p0 += 128) {
                // the rows that start in the window, at its second pair or later
                const uint32_t at = pos - p0;
                uint64_t mk[2];
                window_marks<2>(s_bits[wv], n > 0u && pos > p0 && at < 128u, at, mk);
                const uint32_t started = (uint32_t)__popcll(__ballot(n > 0u && pos <= p0));
                const uint32_t c0 = wb + started - 1u + (uint32_t)__popcll(mk[0] & lanemask_le());
                const uint32_t c1 = wb + started - 1u + (uint32_t)__popcll(mk[0]) + (uint32_t)__popcll(mk[1] & lanemask_le());
                const uint32_t p = p0 + lane, q = p + 64;
                if (p < p1) {
                    const uint4 run = s_run[c0];
                    tile_key[p] = run.y + (p - run.x);
                    inst_rec[p] = run.z;
                }
                if (q < p1) {
                    const uint4 run = s_run[c1];
                    tile_key[q] = run.y + (q - run.x);
                    inst_rec[q] = run.z;
                }
            }
            base += total;
        }
    }
}

// A tile's range starts where the sorted key changes from the previous one
// and ends where it changes to the next.  Each thread reads four consecutive
// keys with one 16-byte load; the neighbours across thread boundaries come
// from the adjacent lanes (lane 0 and lane 63 load theirs).  Keys are stored
// 16-byte aligned.
__device__ __forceinline__ void range_edges(uint32_t i, uint32_t t, uint32_t prev, uint32_t next, uint32_t K,
                                            uint2* __restrict__ ranges, uint32_t tiles_cap) {
    if (t >= tiles_cap) return;
    if (i == 0 || prev != t) ranges[t].x = i;
    if (i + 1 == K || next != t) ranges[t].y = i + 1;
}

__global__ __launch_bounds__(256) void k_tile_ranges(const uint32_t* __restrict__ key,
                                                     const uint32_t* __restrict__ K_dev, uint32_t cap,
                                                     uint2* __restrict__ ranges, uint32_t tiles_cap,
                                                     const uint32_t* __restrict__ flags) {
    if (*flags) return;  // an overflowed binning leaves the ranges empty
    const uint32_t K = min(*K_dev, cap);
    const uint32_t n4 = K / 4;  // whole groups of four keys
    const uint32_t lane = lane_id();
    const uint32_t stride = gridDim.x * blockDim.x;
    // the loop bound is rounded up to whole waves so that every lane of a
    // wave takes part in the shuffles of every round
    const uint32_t nwave = (n4 + 63) / 64 * 64;
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < nwave; g += stride) {
        const bool live = g < n4;
        const uint32_t i = 4 * g;
        const uint4 k = live ? *reinterpret_cast<const uint4*>(key + i) : make_uint4(0u, 0u, 0u, 0u);
        uint32_t prev = (uint32_t)__shfl_up((int)k.w, 1, 64);
        uint32_t next = (uint32_t)__shfl_down((int)k.x, 1, 64);
        if (live && lane == 0 && i > 0) prev = key[i - 1];
        if (live && (lane == 63 || g + 1 == n4)) next = i + 4 < K ? key[i + 4] : 0u;
        if (live) {
            range_edges(i, k.x, prev, k.y, K, ranges, tiles_cap);
            range_edges(i + 1, k.y, k.x, k.z, K, ranges, tiles_cap);
            range_edges(i + 2, k.z, k.y, k.w, K, ranges, tiles_cap);
            range_edges(i + 3, k.w, k.z, next, K, ranges, tiles_cap);
        }
    }
    // the last K % 4 keys
    const uint32_t i = 4 * n4 + blockIdx.x * blockDim.x + threadIdx.x;
    if (i < K) range_edges(i, key[i], i > 0 ? key[i - 1] : 0u, i + 1 < K ? key[i + 1] : 0u, K, ranges, tiles_cap);
}

// ---------------------------------------------------------- tile order
// The compositing kernels take the tiles in descending order of their pair
// counts, bucketed by powers of two, so that long tiles start first and no
// long tile is left for the end of a launch.  A counting sort over 33
// buckets: bucket 0 holds the tiles with 2^31 or more pairs, bucket 31 those
// with one, bucket 32 the empty ones; within a bucket the order is
// arbitrary, since every tile's result is independent of when it runs.
constexpr int TO_BUCKETS = 33;
static_assert(TILE_ORDER_WS == 2 * TO_BUCKETS, "the scratch holds the bucket sizes and the cursors");

__device__ __forceinline__ int tile_bucket(uint2 rg) {
    const uint32_t c = rg.y - rg.x;
    return c ? __clz((int)c) : 32;
}

__global__ __launch_bounds__(256) void k_tile_order_count(const uint2* __restrict__ ranges,
                                                          const Header* __restrict__ hdr, uint32_t tiles_cap,
                                                          uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[TO_BUCKETS];
    for (int i = threadIdx.x; i < TO_BUCKETS; i += blockDim.x) h[i] = 0;
    __syncthreads();
    const uint32_t n = min(hdr->tiles_total, tiles_cap);
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
        atomicAdd(&h[tile_bucket(ranges[t])], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < TO_BUCKETS; i += blockDim.x)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

// hist: the bucket sizes; cursor: per bucket, the places already taken
// (zero before the launch).
__global__ __launch_bounds__(256) void k_tile_order_place(const uint2* __restrict__ ranges,
                                                          const Header* __restrict__ hdr, uint32_t tiles_cap,
                                                          const uint32_t* __restrict__ hist,
                                                          uint32_t* __restrict__ cursor,
                                                          uint32_t* __restrict__ order) {
    __shared__ uint32_t start[TO_BUCKETS], h[TO_BUCKETS], base[TO_BUCKETS];
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int i = 0; i < TO_BUCKETS; i++) {
            start[i] = run;
            run += hist[i];
        }
    }
    const uint32_t n = min(hdr->tiles_total, tiles_cap);
    for (uint32_t t0 = blockIdx.x * blockDim.x; t0 < n; t0 += gridDim.x * blockDim.x) {
        for (int i = threadIdx.x; i < TO_BUCKETS; i += blockDim.x) h[i] = 0;
        __syncthreads();
        const uint32_t t = t0 + threadIdx.x;
        int b = 0;
        uint32_t rank = 0;
        if (t < n) {
            b = tile_bucket(ranges[t]);
            rank = atomicAdd(&h[b], 1u);
        }
        __syncthreads();
        if (threadIdx.x < TO_BUCKETS && h[threadIdx.x]) base[threadIdx.x] = atomicAdd(&cursor[threadIdx.x], h[threadIdx.x]);
        __syncthreads();
        if (t < n) order[start[b] + base[b] + rank] = t;
        __syncthreads();
    }
}

// The same in one block, for up to TO_ONE tiles: the sizes of the buckets, then the places.
constexpr uint32_t TO_ONE = 8192;

__global__ __launch_bounds__(1024) void k_tile_order_one(const uint2* __restrict__ ranges,
                                                         const Header* __restrict__ hdr, uint32_t tiles_cap,
                                                         uint32_t* __restrict__ order) {
    __shared__ uint32_t h[TO_BUCKETS];
    if (threadIdx.x < TO_BUCKETS) h[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t n = min(hdr->tiles_total, tiles_cap);
    int b[TO_ONE / 1024];
#pragma unroll
    for (uint32_t j = 0; j < TO_ONE / 1024; j++) {
        const uint32_t t = j * 1024 + threadIdx.x;
        b[j] = t < n ? tile_bucket(ranges[t]) : -1;
    }
#pragma unroll
    for (uint32_t j = 0; j < TO_ONE / 1024; j++)
        if (b[j] >= 0) atomicAdd(&h[b[j]], 1u);
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t c = threadIdx.x < TO_BUCKETS ? h[threadIdx.x] : 0u;
        const uint32_t start = wave_incl_scan(c) - c;
        if (threadIdx.x < TO_BUCKETS) h[threadIdx.x] = start;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < TO_ONE / 1024; j++)
        if (b[j] >= 0) order[atomicAdd(&h[b[j]], 1u)] = j * 1024 + threadIdx.x;
}

// ------------------------------------------------------------ compositing
// Sec. III: C(p) = sum_i c_i a_i T_i with T_i = prod_{j<i} (1 - a_j); the
// depth image replaces c_i by d_i; the uncertainty image by u_i (Sec. IV-A).

__device__ __forceinline__ uint32_t view_of_tile(const ViewDev* views, int nv, uint32_t tile) {
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_off <= tile) lo = mid;
        else hi = mid - 1;
    }
    return (uint32_t)lo;
}

// Pixel arithmetic of the compositing loops is done relative to an origin
// fixed per 32 x 16 pixel block (a multiple of every tile shape, so no
// pixel's arithmetic depends on the tile): a pixel's coordinates are then
// small exact integers and a splat's mean, staged once per tile as
// (mean hi - origin) + mean lo, is rounded at the magnitude of its distance
// from the block, far below what the alpha test needs.
__device__ __forceinline__ int origin_x(int x) { return x & ~31; }
__device__ __forceinline__ int origin_y(int y) { return y & ~15; }
__device__ __forceinline__ float4 rel_mean(float4 g0, int ox, int oy) {
    return make_float4((g0.x - (float)ox) + g0.z, (g0.y - (float)oy) + g0.w, 0.0f, 0.0f);
}

// alpha of one splat at the pixel (lx, ly) of the block whose origin the
// staged mean (mx, my) is relative to: G = exp2(-|M d|^2), d = p - mean.
// CLAMP = false leaves out the clamp at alpha_max, for splats whose opacity
// is at most alpha_max: G <= 1, so their rounded o G never exceeds it and
// the result is the same.
template <bool CLAMP = true>
__device__ __forceinline__ float splat_alpha(float mx, float my, float4 g1, float lx, float ly, float amax, float& G,
                                             float& dx, float& dy, float& w1, float& w2) {
    dx = lx - mx;
    dy = ly - my;
    w1 = g1.x * dx;
    w2 = fmaf(g1.y, dx, g1.z * dy);
    float pw = fmaf(w1, w1, w2 * w2);
    G = fast_exp2(-pw);
    // o G >= 0, so the median of (o G, 0, alpha_max) is min(alpha_max, o G)
    // (one instruction, with no quieting of its operands)
    return CLAMP ? __builtin_amdgcn_fmed3f(g1.w * G, 0.0f, amax) : g1.w * G;
}

template <bool V>
struct BoolC {
    static constexpr bool value = V;
};

// Splat box meets the pixel rectangle [c0, c1] x [r0, r1].
__device__ __forceinline__ bool box_meets(uint2 b, int c0, int c1, int r0, int r1) {
    return (int)(b.x & 0xffffu) <= c1 && (int)(b.x >> 16) >= c0 && (int)(b.y & 0xffffu) <= r1 &&
           (int)(b.y >> 16) >= r0;
}


// Where the support-ellipse prefilter runs.  It pays in scoring (many
// elongated splats seen close up from arbitrary poses); on mapping frames
// the box test alone is faster in the forward and backward passes.
constexpr bool FWD_ELL = false, SCORE_ELL = true;

// Splats evaluated per step of the front-to-back loops: their alphas are
// independent of the pixel state, so they overlap; the updates follow in order.
constexpr int FWD_STEP = 2;
// The scoring loop's (it keeps only T and one sum per pixel).
constexpr int SCORE_STEP = 2;
// Half width of the band around alpha_min inside which a splat's skip decision is re-taken in binary64:
// twice the rounding of its binary32 alpha or more.  With m the staged mean (relative to the block's origin, so a
// pixel's offset is below |m| + 32) and M = [[a, 0], [b, c]], the whitened offset w = M d is off by at most
// 5 2^-24 E, E = (a + |b|) (|m_x| + 32) + c (|m_y| + 32), so near the threshold, where |w|^2 = log2(o /
// alpha_min), alpha is off by a relative 2 ln 2 sqrt(log2(1 / alpha_min)) 5 2^-24 E, plus a few 2^-24 for the
// squares, the exponential and the opacity: st.band_e E + st.band_c (absolute; to_dev in
// rtg_abi.hip forms both).
// A relative 2e-3 for every splat, which covers needles whose mean is thousands of pixels away, sent one
// alpha in 1,400 to the binary64 branch: every third step of the backward's 512 alphas.
__device__ __forceinline__ float amin_band(float mx, float my, float a, float b, float c, const SetDev& st) {
    const float E = fmaf(a + fabsf(b), fabsf(mx) + 32.0f, c * (fabsf(my) + 32.0f));
    return fmaf(st.band_e, E, st.band_c);
}

// Whether binary32 alpha a lies in that band.
__device__ __forceinline__ bool near_amin(float a, float amin, float band) { return fabsf(a - amin) <= band; }

// A uniform value in a vector register: an instruction that reads a scalar register takes four cycles
// a wave where one of vector registers and constants takes two (additions, products and their fusions).
__device__ __forceinline__ float in_vgpr(float x) {
    asm("" : "+v"(x));
    return x;
}

// The alpha_min test: a splat with alpha < alpha_min at a pixel is skipped
// there.  Where binary32 alpha lies within the splat's band of alpha_min
// the decision is re-taken in binary64 from the binary64 conic
// (kept64), as the definition states it.  No pixel box test is needed: the
// box is the exact bounding box of the support, so outside it alpha <
// alpha_min already.  The loops take the rare binary64 branch once per
// step, for all the splats of the step.

// alpha >= alpha_min, i.e. o exp(-power / 2) >= alpha_min (alpha_max is above it), is taken as power <= 2 ln(o /
// alpha_min), the bound that the projection formed for the support box (q64.w): no exponential, whose
// temporaries set the compositing kernels' register count.
__device__ __forceinline__ bool kept64(float4 g0, const double4* __restrict__ q64, uint32_t r, float px, float py) {
    const double4 q = q64[r];
    const double dx = ((double)px - (double)g0.x) - (double)g0.z;
    const double dy = ((double)py - (double)g0.y) - (double)g0.w;
    const double pw = (q.x * dx * dx + 2.0 * q.y * dx * dy) + q.z * dy * dy;
    return pw <= q.w;
}

// Staged form of a splat for the pair loops of the forward and scoring
// kernels: p = (mean x, mean y relative to the block origin, M00, M10),
// q = (M11, opacity or its log2 (LOG), u, band of alpha_min).  Slot NB of the staged arrays holds
// the null splat (opacity 0, log2 opacity -3e38, band 0): alpha 0 at every pixel, so it never
// contributes.
template <bool LOG>
__device__ __forceinline__ void stage_splat(const EmitRec& e, int ox, int oy, const SetDev& st, float4& p, float4& q) {
    const float4 m = rel_mean(e.g0, ox, oy);
    p = make_float4(m.x, m.y, e.g1.x, e.g1.y);
    q = make_float4(e.g1.z, LOG ? __builtin_amdgcn_logf(e.g1.w) : e.g1.w, __uint_as_float(e.unc),
                    amin_band(m.x, m.y, e.g1.x, e.g1.y, e.g1.z, st));
}

template <int NB, bool LOG>
__device__ __forceinline__ void stage_null_splat(float4* s_p, float4* s_q) {
    if (threadIdx.x == 0) {
        s_p[NB] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        s_q[NB] = make_float4(0.0f, LOG ? -3e38f : 0.0f, 0.0f, 0.0f);
    }
}

// The staged splats that can reach the calling wave's pixel rectangle
// [c0, c1] x [r0, r1] (relative to the block origin (ox, oy)): their box
// meets it and, with ELL, so does their support ellipse.  Written to list as
// LDS byte offsets of their staged entries, in ascending order (so a step
// reads its offsets with one load and no unpacking); two entries past the
// end name the null splat, so the loops run in whole steps of two without
// checks.  Returns the count (wave-uniform).
template <int NB, bool ELL>
__device__ __forceinline__ int splat_list(const uint2* s_pb, const float4* s_p, const float4* s_q, float log2_amin,
                                          int cnt, int c0, int c1, int r0, int r1, int ox, int oy,
                                          uint32_t* list) {
    const int lane = (int)lane_id();
    int n = 0;
#pragma unroll
    for (int c = 0; c < (NB + 63) / 64; c++) {
        const int e = c * 64 + lane;
        bool hit = e < cnt && box_meets(s_pb[e], c0 + ox, c1 + ox, r0 + oy, r1 + oy);
        if (ELL && hit) {
            const float4 p = s_p[e], q = s_q[e];
            hit = support_meets_rect(p.x, p.y, make_float4(p.z, p.w, q.x, q.y), log2_amin, c0, c1, r0, r1);
        }
        const uint64_t m = __ballot(hit);
        if (hit) list[n + (int)__popcll(m & lanemask_lt())] = (uint32_t)(e * sizeof(float4));
        n += (int)__popcll(m);
    }
    if (lane < 2) list[n + lane] = (uint32_t)(NB * sizeof(float4));
    return n;
}

// The binary64 re-decision of a splat whose binary32 alpha fell within the
// band around alpha_min: a splat it keeps enters with alpha at least
// alpha_min (its binary32 alpha lies within the band, below the binary64
// value), one it drops with alpha 0.
__device__ __forceinline__ float redecide(float a, const Records& rec, uint32_t r, int u, int v, const SetDev& st) {
    return kept64(rec.emit[r].g0, rec.q64, r, (float)u, (float)v) ? fmaxf(a, st.alpha_min) : 0.0f;
}

// B splats are staged per batch (B <= TW * TH; threads below B load them).
// UNC: the uncertainty image is requested (otherwise it is not composited).
// COUNT: the contributing splats are counted (out.contrib), per wave and by the scalar unit, whose two instructions
// a splat cost 1 to 2 %; captured iterations, whose counts nobody can read, leave them out.
//
// Front to back over the wave's list, FWD_STEP splats per step: their alphas
// are independent of the pixel state, the updates follow in order.  A pixel
// whose next transmittance would fall below T_min stops there; its T is then
// kept negated (|T| is the final transmittance), which no later update
// passes, so the loop carries no per-pixel flags; the pixels still live are those of the last
// update's comparison, a scalar mask.  A splat below alpha_min
// enters with alpha 0 (T unchanged, exactly).
//
// Bound by instruction issue (cycles per wave: additions, products and their fusions 2; comparisons, selects,
// minima and maxima, and anything with a scalar register 4; exp2 8).  So the thresholds sit in vector
// registers, and a batch whose splats are all at most alpha_max opaque leaves the clamp out.
// 8 keyframes of 1280x720, with the narrower band of the binary64 branch and 64 instead of 80 VGPRs (eight waves per SIMD): 1,172 -> 1,027 us.
template <int TW, int TH, int B, bool UNC, bool COUNT>
__global__ __launch_bounds__(TW * TH, 8) void k_render_fwd(const ViewDev* __restrict__ views, int n_views,
                                                        const uint2* __restrict__ ranges,
                                                        const uint32_t* __restrict__ tile_order,
                                                        const uint32_t* __restrict__ inst_rec,
                                                        Records rec, SetDev st, RenderOut out,
                                                        const uint32_t* __restrict__ flags) {
    constexpr int NT = TW * TH;
    static_assert(B <= NT, "batch larger than the tile");
    static_assert(32 % TW == 0 && 16 % TH == 0, "tiles must divide the 32 x 16 origin block");
    static_assert(FWD_STEP == 2, "the list is padded for steps of two");
    if (flags && *flags) return;
    __shared__ float4 s_p[B + 1], s_q[B + 1], s_at[B + 1];
    __shared__ uint32_t s_r[B + 1];
    __shared__ uint2 s_pb[B];
    __shared__ __align__(8) uint32_t s_list[NT / 64 * (B + 2)];
    stage_null_splat<B, false>(s_p, s_q);
    if (threadIdx.x == 0) s_at[B] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const uint32_t tile = tile_order[blockIdx.x];
    const uint32_t vi = view_of_tile(views, n_views, tile);
    const ViewDev& V = views[vi];
    const int W = V.W, H = V.H;
    const uint32_t lt = tile - V.tile_off;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const int u = tx * TW + (int)(threadIdx.x % TW), v = ty * TH + (int)(threadIdx.x / TW);
    const int ox = origin_x(tx * TW), oy = origin_y(ty * TH);
    // this wave's pixel rectangle (64 consecutive threads = 64 / TW rows of
    // the tile), relative to the origin
    const int wc0 = tx * TW - ox, wc1 = wc0 + TW - 1;
    const int wr0 = ty * TH + (int)(threadIdx.x >> 6) * (64 / TW) - oy, wr1 = wr0 + 64 / TW - 1;
    const bool inside = u < W && v < H;
    const float lx = (float)(u - ox), ly = (float)(v - oy);
    const float amin = in_vgpr(st.alpha_min), tmin = in_vgpr(st.T_min), amax = st.alpha_max;
    const char* sp = reinterpret_cast<const char*>(s_p);
    const char* sq = reinterpret_cast<const char*>(s_q);
    const char* sa = reinterpret_cast<const char*>(s_at);
    const uint2 rg = ranges[tile];
    float T = inside ? 1.0f : -1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, dd = 0.0f, uu = 0.0f;
    uint32_t last = 0;
    uint64_t contrib = 0;  // of the wave's pixels
    for (uint32_t b = rg.x; b < rg.y; b += B) {
        if (__builtin_amdgcn_readfirstlane(__syncthreads_count(T > 0.0f)) == 0) break;
        uint32_t idx = b + threadIdx.x;
        bool opaque = false;
        if (threadIdx.x < (uint32_t)B && idx < rg.y) {
            uint32_t r = inst_rec[idx];
            s_r[threadIdx.x] = r;
            const EmitRec e = rec.emit[r];
            s_pb[threadIdx.x] = e.pbox;
            opaque = e.g1.w > amax;
            stage_splat<false>(e, ox, oy, st, s_p[threadIdx.x], s_q[threadIdx.x]);
            s_at[threadIdx.x] = rec.attr[r];
        }
        const bool clamped = __builtin_amdgcn_readfirstlane(__syncthreads_or(opaque));
        const int cnt = (int)min<uint32_t>(B, rg.y - b);
        uint32_t* my = s_list + (threadIdx.x >> 6) * (B + 2);
        int nl = 0;
        uint64_t alive = __ballot(T > 0.0f);
        if (alive)
            nl = splat_list<B, FWD_ELL>(s_pb, s_p, s_q, st.log2_amin, cnt, wc0, wc1, wr0, wr1, ox, oy, my);
        __syncthreads();  // the wave's list is in LDS
        // LDS offset of the last splat this lane took in this batch
        uint32_t lastoff = 0xffffffffu;
        uint32_t taken = 0;  // contributors among the wave's pixels and this batch's splats, in a scalar register
        auto walk = [&](auto clamp) {
            for (int i = 0; i < nl && alive; i += FWD_STEP) {
                uint32_t ko[FWD_STEP];
                float as[FWD_STEP], bs[FWD_STEP];
                bool need = false;
#pragma unroll
                for (int q = 0; q < FWD_STEP; q++) {
                    ko[q] = my[i + q];
                    const float4 pp = *reinterpret_cast<const float4*>(sp + ko[q]);
                    const float4 qq = *reinterpret_cast<const float4*>(sq + ko[q]);
                    float G, dx, dy, w1, w2;
                    as[q] = splat_alpha<decltype(clamp)::value>(pp.x, pp.y, make_float4(pp.z, pp.w, qq.x, qq.y), lx, ly,
                                                                amax, G, dx, dy, w1, w2);
                    bs[q] = qq.w;
                    need = need | near_amin(as[q], amin, bs[q]);
                }
                if (__ballot(need)) {
#pragma unroll
                    for (int q = 0; q < FWD_STEP; q++)
                        if (near_amin(as[q], amin, bs[q]))
                            as[q] = redecide(as[q], rec, s_r[ko[q] / sizeof(float4)], u, v, st);
                }
#pragma unroll
                for (int q = 0; q < FWD_STEP; q++) {
                    const bool ok = as[q] >= amin;
                    const float a0 = ok ? as[q] : 0.0f;
                    const float Tn = fmaf(-a0, T, T);
                    const bool live = Tn >= tmin;
                    const bool use = ok & live;
                    if (COUNT) taken += (uint32_t)__popcll(__ballot(ok) & __ballot(live));
                    // weight 0 where the splat is skipped (a0 = 0) or the pixel
                    // stops: fmaf(x, 0, c) = c for the finite staged attributes,
                    // so the sums need no per-channel select
                    const float w = live ? a0 * T : 0.0f;
                    const float4 at = *reinterpret_cast<const float4*>(sa + ko[q]);
                    c0 = fmaf(at.x, w, c0);
                    c1 = fmaf(at.y, w, c1);
                    c2 = fmaf(at.z, w, c2);
                    dd = fmaf(at.w, w, dd);
                    if (UNC) {
                        const float uk = *reinterpret_cast<const float*>(sq + ko[q] + 8);
                        uu = fmaf(uk, w, uu);
                    }
                    lastoff = use ? ko[q] : lastoff;
                    T = live ? Tn : -fabsf(T);
                    if (q + 1 == FWD_STEP) alive = __ballot(live);
                }
            }
        };
        if (clamped) walk(BoolC<true>{});
        else walk(BoolC<false>{});
        if (COUNT) contrib += (uint32_t)__builtin_amdgcn_readfirstlane((int)taken);
        if (lastoff != 0xffffffffu) last = b - rg.x + 1 + lastoff / (uint32_t)sizeof(float4);
    }
    if (COUNT && lane_id() == 0) out.contrib[(uint64_t)tile * (NT / 64) + (threadIdx.x >> 6)] = contrib;
    if (!inside) return;
    T = fabsf(T);
    const uint64_t P = (uint64_t)W * H;
    const uint64_t pix = V.pix_off + (uint64_t)v * W + u;
    if (out.rgb) {
        float* base = out.rgb + 3 * V.pix_off + (uint64_t)v * W + u;
        base[0] = c0;
        base[P] = c1;
        base[2 * P] = c2;
    }
    if (out.depth) out.depth[pix] = dd;
    if (out.alpha) out.alpha[pix] = 1.0f - T;
    if (out.unc) out.unc[pix] = uu;
    if (out.T_final) out.T_final[pix] = T;
    if (out.n_last) out.n_last[pix] = last;
}

// ----------------------------------------------------------------- loss
// Sec. III eq. (4), L1 terms: (1/P) sum_p (sum_ch |C - C*| + w_d |D - D*|).

__device__ __forceinline__ float sgnf(float e) { return e > 0.0f ? 1.0f : (e < 0.0f ? -1.0f : 0.0f); }

__device__ __forceinline__ double wave_sum_d(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ __forceinline__ float wave_sum_f(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__global__ __launch_bounds__(256) void k_loss(const ViewDev* __restrict__ views, const float* __restrict__ rgb,
                                              const float* __restrict__ depth, const float* __restrict__ trgb,
                                              const float* __restrict__ tdepth, float w_depth,
                                              float* __restrict__ d_rgb, float* __restrict__ d_depth,
                                              double* __restrict__ partial) {
    __shared__ double ws[4];
    const ViewDev& V = views[blockIdx.y];
    const uint64_t P = (uint64_t)V.W * V.H;
    const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double l = 0.0;
    if (p < P) {
        const float invP = (float)(1.0 / (double)P);
        const uint64_t c = 3 * V.pix_off + p;
        const uint64_t q = V.pix_off + p;
        float acc = 0.0f;
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            float e = rgb[c + ch * P] - trgb[c + ch * P];
            acc += fabsf(e);
            if (d_rgb) d_rgb[c + ch * P] = sgnf(e) * invP;
        }
        float e = depth[q] - tdepth[q];
        if (d_depth) d_depth[q] = w_depth * sgnf(e) * invP;
        l = ((double)acc + (double)w_depth * (double)fabsf(e)) / (double)P;
    }
    l = wave_sum_d(l);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) partial[(uint64_t)blockIdx.y * gridDim.x + blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// One block; each thread keeps four running sums over entries 4096 apart, so
// that four loads are in flight per step (the order is fixed: the total is
// the same on every run).
constexpr int SP_THREADS = 1024;
__global__ __launch_bounds__(SP_THREADS) void k_sum_partials(const double* __restrict__ partial, int n,
                                                             double* __restrict__ out) {
    __shared__ double ws[SP_THREADS / 64];
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < n; i += 4 * SP_THREADS) {
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (i + k * SP_THREADS < n) a[k] += partial[i + k * SP_THREADS];
    }
    double s = wave_sum_d((a[0] + a[1]) + (a[2] + a[3]));
    if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < SP_THREADS / 64; w++) t += ws[w];
        *out = t;
    }
}

// ------------------------------------------------------------ backward
// Reverse mode of the compositing, walking each tile back to front; the
// transmittance before splat i is recovered as T_{i+1} / (1 - a_i).

// Words between the rows of the backward's reduction in LDS: rows r to r + 15 start 4 banks apart each, so
// 16-byte reads of 16 rows meet no bank twice.
constexpr int RED_STRIDE = 68;

// One pixel's step of the reverse compositing recursion for a kept splat i.
// With T = T_{i+1} (transmittance behind it), T_i = T / (1 - a_i) and the
// splat's weight w = a_i T_i; for an image channel with colour c_i and pixel
// gradient g, dL/da_i = g (c_i T_i - S / (1 - a_i)), S = sum_{j > i} c_j w_j.
// The channels enter only through GA = sum_ch g_ch c_i,ch, so the pixel
// carries one running sum D = sum_ch g_ch S_ch (D += w GA) instead of one per
// channel: dL/da_i = T_i GA - D / (1 - a_i).  Since a_i <= alpha_max < 1,
// 1 - a_i is a normal number well away from zero and the hardware reciprocal
// (within 1 ulp) stands in for the correctly rounded division; T only scales
// gradient terms here and decides nothing.
// The sums over the pixels (the record's gradient slots, in this order), with
// t = dL/da a_g, where a_g = o G is the splat's alpha where it is not clamped
// at alpha_max (then da/dpower = -a_g / 2 and da/do = a_g / o) and 0 where it
// is (no gradient flows through the clamp):
//   0, 1: sum t dx, sum t dy, with d = pixel - mean; the projection backward
//         scales them by -1/2 into sum dpow dx, sum dpow dy (dpow = dL/dpower,
//         power = d^T Q d, G = exp(-power / 2)) and forms the mean's gradient
//         -2 Q (sum dpow d) per record in binary64;
//   2, 3, 4: sum t dx^2, sum t dx dy, sum t dy^2, likewise (dL/dQ);
//   5: sum t, which the projection backward divides by o (dL/do);
//   6..9: sum g_ch w (colour and depth).
// A splat with a = 0 and a_g = 0 leaves T (1 / (1 - 0) = 1 exactly), D and
// every sum unchanged, for finite pixel gradients and colours.
// AU: the alpha and uncertainty images carry gradients too (colour 1 and u
// in GA; otherwise their terms are left out altogether).
// FIRST: the lane's first pixel starts the sums.
template <bool AU, bool FIRST>
__device__ __forceinline__ void bwd_pixel(float a, float ag, float dx, float dy, float4 at, float ui, float gr, float gg,
                                          float gb, float gd, float ga, float gu, float& T, float& D, float* acc) {
    const float inv = __builtin_amdgcn_rcpf(1.0f - a);
    const float Ti = T * inv;
    const float w = a * Ti;
    float GA = gr * at.x;
    GA = fmaf(gg, at.y, GA);
    GA = fmaf(gb, at.z, GA);
    GA = fmaf(gd, at.w, GA);
    if constexpr (AU) {
        GA += ga;
        GA = fmaf(gu, ui, GA);
    }
    const float da = fmaf(Ti, GA, -(D * inv));
    D = fmaf(w, GA, D);
    T = Ti;
    const float t = da * ag, tx = t * dx, ty = t * dy;
    acc[0] = FIRST ? tx : acc[0] + tx;
    acc[1] = FIRST ? ty : acc[1] + ty;
    acc[2] = FIRST ? tx * dx : fmaf(tx, dx, acc[2]);
    acc[3] = FIRST ? tx * dy : fmaf(tx, dy, acc[3]);
    acc[4] = FIRST ? ty * dy : fmaf(ty, dy, acc[4]);
    acc[5] = FIRST ? t : acc[5] + t;
    acc[6] = FIRST ? gr * w : fmaf(gr, w, acc[6]);
    acc[7] = FIRST ? gg * w : fmaf(gg, w, acc[7]);
    acc[8] = FIRST ? gb * w : fmaf(gb, w, acc[8]);
    acc[9] = FIRST ? gd * w : fmaf(gd, w, acc[9]);
}

// One wave takes a tile, or one of the NSUB bands of 8x8 pixel blocks a tile is cut into (a workgroup each), and a
// lane the same pixel of each of its PPT blocks.  The staging lanes keep only the splats whose box meets the
// band and write them compacted, in ascending order, to LDS; the walk back to front is a countdown over them,
// two per step.  Slot B holds the null splat: position 0xffffffff (no pixel takes it), zero geometry and
// colour.
//
// Bound by instruction issue (cycles per wave as at k_render_fwd; a DPP addition 4, a row swap 8).  The 20 sums of a
// step are added up over the lanes through LDS, which is otherwise idle: about 90 cycles of vector
// instructions; halving them lane by lane with DPP additions and selects took about 250.  The sums cancel for needle-
// shaped splats, whose gradients depend on the rounding of the products and on the tree of lanes:
// both are the ones of a halving by lanes (i, 15 - i, 7 - i, i ^ 2, i ^ 1, then the rows).  Moments of a row of
// four pixels, 13 instructions instead of 32, took 1,940 us where these take 2,120, but moved such gradients by up to 2e-3.
// 8 keyframes of 1280x720, with the narrower band of the binary64 branch, thresholds in vector registers and four waves
// per SIMD (128 VGPRs with 9 spilled, 13 at 32x8; 158 before): 2,264 -> 2,120 us, of which the atomics are 70 us; one
// 640x480 frame in two bands: 134 -> 113 us.
template <int TW, int TH, int NSUB, bool AU>
__global__ __launch_bounds__(64, AU ? 3 : 4) void k_render_bwd(const ViewDev* __restrict__ views, int n_views,
                                                        const uint2* __restrict__ ranges,
                                                        const uint32_t* __restrict__ tile_order,
                                                        const uint32_t* __restrict__ inst_rec, Records rec,
                                                        SetDev st, const float* __restrict__ T_final,
                                                        const uint32_t* __restrict__ n_last,
                                                        const float* __restrict__ d_rgb,
                                                        const float* __restrict__ d_depth,
                                                        const float* __restrict__ d_alpha,
                                                        const float* __restrict__ d_unc, double* __restrict__ g2d,
                                                        const uint32_t* __restrict__ flags) {
    constexpr int PPT = TW * TH / 64 / NSUB;
    constexpr int RW = PPT * 8 < TW ? PPT * 8 : TW, RH = PPT * 64 / RW;  // the band
    constexpr int B = 64;
    static_assert(PPT >= 1 && PPT <= 4 && RW * RH == PPT * 64, "a wave must hold the band, one to four blocks");
    if (flags && *flags) return;
    // s_p = (mean x, mean y relative to the origin, record id bits, position bits)
    __shared__ float4 s_p[B + 1], s_g1[B + 1], s_at[B + 1];
    __shared__ float s_u[B + 1], s_band[B + 1];
    __shared__ float s_red[20 * RED_STRIDE];
    const uint32_t tile = tile_order[blockIdx.x / NSUB];
    const uint32_t vi = view_of_tile(views, n_views, tile);
    const ViewDev& V = views[vi];
    const int W = V.W, H = V.H;
    const uint32_t lt = tile - V.tile_off;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const uint2 rg = ranges[tile];
    const uint64_t P = (uint64_t)W * H;
    const int lane = (int)threadIdx.x;
    if (lane == 0) {
        s_p[B] = make_float4(0.0f, 0.0f, 0.0f, __uint_as_float(0xffffffffu));
        s_g1[B] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        s_at[B] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        s_u[B] = 0.0f;
        s_band[B] = 0.0f;
    }

    const int ox = origin_x(tx * TW), oy = origin_y(ty * TH);
    // the band's pixels, and the lane's: (u0 + bx(j), v0 + by(j))
    const int first = (int)(blockIdx.x % NSUB) * PPT;
    const int c0 = tx * TW + first % (TW / 8) * 8, c1 = c0 + RW - 1, r0 = ty * TH + first / (TW / 8) * 8, r1 = r0 + RH - 1;
    const int u0 = c0 + (lane & 7), v0 = r0 + (lane >> 3);
    const float px0 = (float)(u0 - ox), py0 = (float)(v0 - oy);
    auto bx = [](int j) { return j % (RW / 8) * 8; };
    auto by = [](int j) { return j / (RW / 8) * 8; };
    float T[PPT];
    uint32_t last[PPT];
    float gr[PPT], gg[PPT], gb[PPT], gd[PPT], ga[PPT], gu[PPT];
    float D[PPT];
    uint32_t mylast = 0;
#pragma unroll
    for (int j = 0; j < PPT; j++) {
        const int u = u0 + bx(j), v = v0 + by(j);
        T[j] = 1.0f;
        last[j] = 0;
        gr[j] = gg[j] = gb[j] = gd[j] = ga[j] = gu[j] = 0.0f;
        D[j] = 0.0f;
        if (u < W && v < H) {
            const uint64_t pix = V.pix_off + (uint64_t)v * W + u;
            T[j] = T_final[pix];
            last[j] = n_last[pix];
            if (d_rgb) {
                const float* cb = d_rgb + 3 * V.pix_off + (uint64_t)v * W + u;
                gr[j] = cb[0];
                gg[j] = cb[P];
                gb[j] = cb[2 * P];
            }
            if (d_depth) gd[j] = d_depth[pix];
            if (AU && d_alpha) ga[j] = d_alpha[pix];
            if (AU && d_unc) gu[j] = d_unc[pix];
        }
        mylast = max(mylast, last[j]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mylast = max(mylast, (uint32_t)__shfl_xor((int)mylast, o, 64));
    const uint32_t maxlast = mylast;
    const float amin = in_vgpr(st.alpha_min), amax = st.alpha_max;

    for (int64_t bend = maxlast; bend > 0; bend -= B) {
        const int64_t bstart = bend - B > 0 ? bend - B : 0;
        __syncthreads();
        bool hit = false;
        float4 p, q1, at;
        float uv = 0.0f;
        {
            const int64_t e = bstart + lane;
            if (e < bend) {
                const uint32_t r = inst_rec[rg.x + (uint32_t)e];
                const EmitRec er = rec.emit[r];
                hit = box_meets(er.pbox, c0, c1, r0, r1);
                const float4 m = rel_mean(er.g0, ox, oy);
                p = make_float4(m.x, m.y, __uint_as_float(r), __uint_as_float((uint32_t)e));
                q1 = er.g1;
                at = rec.attr[r];
                if (AU) uv = __uint_as_float(er.unc);
            }
        }
        const uint64_t hm = __ballot(hit);
        const int n = (int)__popcll(hm);
        if (hit) {
            const int slot = (int)__popcll(hm & lanemask_lt());
            s_p[slot] = p;
            s_g1[slot] = q1;
            s_at[slot] = at;
            s_band[slot] = amin_band(p.x, p.y, q1.x, q1.y, q1.z, st);
            if (AU) s_u[slot] = uv;
        }
        __syncthreads();
        // back to front over slots n - 1, n - 2, ..., two per step
        for (int i = n - 1; i >= 0; i -= 2) {
            float4 cp[2], cg[2];
            int slot[2];
#pragma unroll
            for (int q = 0; q < 2; q++) {
                slot[q] = i - q >= 0 ? i - q : B;
                cp[q] = s_p[slot[q]];
                cg[q] = s_g1[slot[q]];
            }
            uint32_t sr[2], spos[2];
#pragma unroll
            for (int q = 0; q < 2; q++) {
                sr[q] = __float_as_uint(cp[q].z);
                spos[q] = __float_as_uint(cp[q].w);
            }
            float acc[20];
            bool any[2];
#pragma unroll
            for (int q = 0; q < 2; q++) any[q] = false;
            // every alpha of the step first (one block of independent work),
            // then the rare binary64 re-decisions, then the ordered updates.
            // CL: a splat of the step is more opaque than alpha_max, so its
            // alpha may be clamped and then carries no gradient; otherwise
            // alpha = o G carries it at every pixel (a_g = a)
            auto step = [&](auto clamp) {
                constexpr bool CL = decltype(clamp)::value;
                float a[PPT][2], G[PPT][2], dx[PPT][2], dy[PPT][2];
                const float bands[2] = {s_band[slot[0]], s_band[slot[1]]};
                bool need = false;
#pragma unroll
                for (int j = 0; j < PPT; j++)
#pragma unroll
                    for (int q = 0; q < 2; q++) {
                        float w1, w2;
                        a[j][q] = splat_alpha<CL>(cp[q].x, cp[q].y, cg[q], px0 + (float)bx(j), py0 + (float)by(j), amax,
                                                  G[j][q], dx[j][q], dy[j][q], w1, w2);
                        need = need | near_amin(a[j][q], amin, bands[q]);
                    }
                if (__ballot(need)) {
                    // one copy of the binary64 code: a loop over the step's alphas, each taken out
                    // and put back by selects
#pragma unroll 1
                    for (int k = 0; k < 2 * PPT; k++) {
                        float x = 0.0f;
                        uint32_t l = 0;
#pragma unroll
                        for (int j = 0; j < PPT; j++) {
                            x = k == 2 * j ? a[j][0] : k == 2 * j + 1 ? a[j][1] : x;
                            l = k >> 1 == j ? last[j] : l;
                        }
                        if ((((k & 1) ? spos[1] : spos[0]) < l) & near_amin(x, amin, (k & 1) ? bands[1] : bands[0]))
                            x = redecide(x, rec, (k & 1) ? sr[1] : sr[0], u0 + bx(k >> 1), v0 + by(k >> 1), st);
#pragma unroll
                        for (int j = 0; j < PPT; j++) {
                            a[j][0] = k == 2 * j ? x : a[j][0];
                            a[j][1] = k == 2 * j + 1 ? x : a[j][1];
                        }
                    }
                }
                // the colours are read here, not with the geometry: fewer registers live above
                asm volatile("" ::: "memory");
                float4 ca[2];
                float cu[2];
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    ca[q] = s_at[slot[q]];
                    cu[q] = AU ? s_u[slot[q]] : 0.0f;
                }
#pragma unroll
                for (int j = 0; j < PPT; j++) {
#pragma unroll
                    for (int q = 0; q < 2; q++) {
                        const bool ok = (spos[q] < last[j]) & (a[j][q] >= amin);
                        any[q] = any[q] | ok;
                        const float a0 = ok ? a[j][q] : 0.0f;
                        const float ag = CL ? (cg[q].w * G[j][q] <= amax ? a0 : 0.0f) : a0;
                        if (j == 0)
                            bwd_pixel<AU, true>(a0, ag, dx[j][q], dy[j][q], ca[q], cu[q], gr[j], gg[j], gb[j], gd[j], ga[j],
                                                gu[j], T[j], D[j], acc + 10 * q);
                        else
                            bwd_pixel<AU, false>(a0, ag, dx[j][q], dy[j][q], ca[q], cu[q], gr[j], gg[j], gb[j], gd[j], ga[j],
                                                 gu[j], T[j], D[j], acc + 10 * q);
                    }
                }
            };
            // opacities and alpha_max are positive: their bits order as they do
            const uint32_t amax_bits = __float_as_uint(amax);
            if (__ballot((__float_as_uint(cg[0].w) > amax_bits) | (__float_as_uint(cg[1].w) > amax_bits)))
                step(BoolC<true>{});
            else
                step(BoolC<false>{});
            bool t[2];
#pragma unroll
            for (int q = 0; q < 2; q++) t[q] = __ballot(any[q]) != 0;
            // reduced unconditionally (a step that no pixel takes is rare), so
            // that the per-pixel sums are formed pixel by pixel instead of
            // being held back behind a branch
            // totals: value k of every lane in row k of LDS, and lanes r and r + 32 each add up half of
            // row r (r < 20; the spare lanes repeat row 19)
            wave_lds_order();
#pragma unroll
            for (int k = 0; k < 20; k++) s_red[k * RED_STRIDE + lane] = acc[k];
            wave_lds_order();
            const int row = min(lane & 31, 19);
            const float4* half = reinterpret_cast<const float4*>(s_red + row * RED_STRIDE + (lane & 32));
            float4 h[8];
#pragma unroll
            for (int k = 0; k < 8; k++) h[k] = half[k];
            // a tree in every 16 lanes (lane i with 15 - i, 7 - i, i ^ 2, i ^ 1), then the rows of lanes
            float row16[2];
#pragma unroll
            for (int k = 0; k < 2; k++) {
                const float4 p = h[4 * k], q = h[4 * k + 1], r = h[4 * k + 2], s4 = h[4 * k + 3];
                const float a0 = p.x + s4.w, a1 = p.y + s4.z, a2 = p.z + s4.y, a3 = p.w + s4.x;
                const float a4 = q.x + r.w, a5 = q.y + r.z, a6 = q.z + r.y, a7 = q.w + r.x;
                row16[k] = ((a0 + a7) + (a2 + a5)) + ((a1 + a6) + (a3 + a4));
            }
            const float part = row16[0] + row16[1];
            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(part), __float_as_uint(part), false, false);
            const float tot = __uint_as_float(both[0]) + __uint_as_float(both[1]);
            // one binary64 atomic of 20 lanes
            if (lane < 20 && (lane >= 10 ? t[1] : t[0]))
                unsafeAtomicAdd(g2d + (uint64_t)(lane >= 10 ? sr[1] : sr[0]) * G2D_STRIDE + (lane >= 10 ? lane - 10 : lane),
                                (double)tot);
        }
    }
}

// Chain rule from the screen-space gradients of a Gaussian's records to its
// parameters, in binary64, summed over the views that see it.
__global__ __launch_bounds__(256) void k_project_bwd(GaussDev g, const ViewDev* __restrict__ views, SetDev st,
                                                     const uint32_t* __restrict__ rec_off,
                                                     const uint32_t* __restrict__ cnt,
                                                     const EmitRec* __restrict__ emit,
                                                     const double* __restrict__ g2d,
                                                     float* __restrict__ d_means, float* __restrict__ d_ls,
                                                     float* __restrict__ d_quats, float* __restrict__ d_op,
                                                     float* __restrict__ d_col, const uint32_t* __restrict__ flags,
                                                     uint32_t* __restrict__ flag_host) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (flag_host && i == 0) __hip_atomic_store(flag_host, *flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (i >= g.n) return;
    if (flags && *flags) return;
    uint32_t c = cnt[i];
    if (c == 0) return;
    GPre P;
    if (!pre_gauss(g, i, st, P)) return;
    const int64_t n = g.n;
    double gm[3] = {0, 0, 0}, gs[3] = {0, 0, 0}, gR[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    double go = 0.0, gc[3] = {0, 0, 0};
    uint32_t r0 = rec_off[i];
    for (uint32_t r = r0; r < r0 + c; r++) {
        const Cam V = load_cam(views + emit[r].view);
        GProj q;
        project_exact(P, V, st, q);
        const double* G2 = g2d + (uint64_t)r * G2D_STRIDE;
        go += G2[5];  // divided by the opacity below
        gc[0] += G2[6];
        gc[1] += G2[7];
        gc[2] += G2[8];
        double gdepth = G2[9];
        double det = q.cxx * q.cyy - q.cxy * q.cxy;
        double Qxx = q.cyy / det, Qxy = -q.cxy / det, Qyy = q.cxx / det;
        // the 2D mean: power = d^T Q d with d = pixel - mean, so
        // dL/dmean = -2 Q sum_p dpow d, and slots 0 and 1 hold -2 times that
        // sum (dpow = -t / 2)
        double gmx = Qxx * G2[0] + Qxy * G2[1];
        double gmy = Qxy * G2[0] + Qyy * G2[1];
        // conic gradient (slots 2..4 times -1/2: dL/dQxx, dL/dQxy of the xy
        // term taken once, dL/dQyy) -> symmetric matrix gradient
        double Gq00 = -0.5 * G2[2], Gq01 = -0.5 * G2[3], Gq11 = -0.5 * G2[4];
        // G_cov = -Q G_Q Q
        double m00 = Gq00 * Qxx + Gq01 * Qxy, m01 = Gq00 * Qxy + Gq01 * Qyy;
        double m10 = Gq01 * Qxx + Gq11 * Qxy, m11 = Gq01 * Qxy + Gq11 * Qyy;
        double C00 = -(Qxx * m00 + Qxy * m10);
        double C01 = -(Qxx * m01 + Qxy * m11);
        double C11 = -(Qxy * m01 + Qyy * m11);
        // cov = Bs Bs^T with Bs = J A diag(s)
        double B0[3], B1[3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            B0[k] = fma(q.j0, q.A[0 * 3 + k], q.j2 * q.A[2 * 3 + k]);
            B1[k] = fma(q.j4, q.A[1 * 3 + k], q.j5 * q.A[2 * 3 + k]);
        }
        double GB0[3], GB1[3];  // dL/dB (B = J A)
#pragma unroll
        for (int k = 0; k < 3; k++) {
            double gbs0 = 2.0 * (C00 * B0[k] + C01 * B1[k]) * P.s[k];  // dL/dBs row 0
            double gbs1 = 2.0 * (C01 * B0[k] + C11 * B1[k]) * P.s[k];
            gs[k] += gbs0 * B0[k] + gbs1 * B1[k];
            GB0[k] = gbs0 * P.s[k];
            GB1[k] = gbs1 * P.s[k];
        }
        // B = J A:  G_J = G_B A^T, G_A = J^T G_B
        double GJ00 = 0, GJ02 = 0, GJ11 = 0, GJ12 = 0;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            GJ00 += GB0[k] * q.A[0 * 3 + k];
            GJ02 += GB0[k] * q.A[2 * 3 + k];
            GJ11 += GB1[k] * q.A[1 * 3 + k];
            GJ12 += GB1[k] * q.A[2 * 3 + k];
        }
        double GA[9];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            GA[0 * 3 + k] = q.j0 * GB0[k];
            GA[1 * 3 + k] = q.j4 * GB1[k];
            GA[2 * 3 + k] = q.j2 * GB0[k] + q.j5 * GB1[k];
        }
        // A = R^T Rq:  G_Rq = R G_A
        const double* R = V.R;
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++)
                gR[a * 3 + b] += R[a * 3 + 0] * GA[0 * 3 + b] + R[a * 3 + 1] * GA[1 * 3 + b] +
                                 R[a * 3 + 2] * GA[2 * 3 + b];
        // camera-frame mean
        double tx = q.t[0], ty = q.t[1], tz = q.t[2];
        double iz = 1.0 / tz, iz2 = iz * iz;
        double gtx = 0, gty = 0, gtz = 0;
        gtz += GJ00 * (-V.fx * iz2);
        gtx += GJ02 * (-V.fx * iz2);
        gtz += GJ02 * (2.0 * V.fx * tx * iz2 * iz);
        gtz += GJ11 * (-V.fy * iz2);
        gty += GJ12 * (-V.fy * iz2);
        gtz += GJ12 * (2.0 * V.fy * ty * iz2 * iz);
        gtx += gmx * V.fx * iz;
        gtz -= gmx * V.fx * tx * iz2;
        gty += gmy * V.fy * iz;
        gtz -= gmy * V.fy * ty * iz2;
        gtz += gdepth;
#pragma unroll
        for (int a = 0; a < 3; a++) gm[a] += R[a * 3 + 0] * gtx + R[a * 3 + 1] * gty + R[a * 3 + 2] * gtz;
    }
    // slot 5 summed dL/da a_g = o dL/do over the pixels (o >= alpha_min > 0)
    go /= P.o;
    if (st.isotropic) {
        // one radius for the three axes; no rotation
        if (d_means) {
            d_means[i] += (float)gm[0];
            d_means[n + i] += (float)gm[1];
            d_means[2 * n + i] += (float)gm[2];
        }
        if (d_ls) d_ls[i] += (float)((gs[0] + gs[1] + gs[2]) * P.s[0]);
        if (d_op) d_op[i] += (float)go;
        if (d_col) {
            d_col[i] += (float)gc[0];
            d_col[n + i] += (float)gc[1];
            d_col[2 * n + i] += (float)gc[2];
        }
        return;
    }
    // rotation matrix -> normalised quaternion -> raw quaternion
    double w = g.quats[i], x = g.quats[n + i], y = g.quats[2 * n + i], z = g.quats[3 * n + i];
    double qn = sqrt(w * w + x * x + y * y + z * z);
    double inv = 1.0 / qn;
    w *= inv; x *= inv; y *= inv; z *= inv;
    double gw = 2.0 * (-z * gR[1] + y * gR[2] + z * gR[3] - x * gR[5] - y * gR[6] + x * gR[7]);
    double gx = 2.0 * (y * gR[1] + z * gR[2] + y * gR[3] - 2.0 * x * gR[4] - w * gR[5] + z * gR[6] +
                       w * gR[7] - 2.0 * x * gR[8]);
    double gy = 2.0 * (-2.0 * y * gR[0] + x * gR[1] + w * gR[2] + x * gR[3] + z * gR[5] - w * gR[6] +
                       z * gR[7] - 2.0 * y * gR[8]);
    double gz = 2.0 * (-2.0 * z * gR[0] - w * gR[1] + x * gR[2] + w * gR[3] - 2.0 * z * gR[4] + y * gR[5] +
                       x * gR[6] + y * gR[7]);
    double dot = w * gw + x * gx + y * gy + z * gz;
    if (d_quats) {
        d_quats[i] += (float)((gw - w * dot) * inv);
        d_quats[n + i] += (float)((gx - x * dot) * inv);
        d_quats[2 * n + i] += (float)((gy - y * dot) * inv);
        d_quats[3 * n + i] += (float)((gz - z * dot) * inv);
    }
    if (d_means) {
        d_means[i] += (float)gm[0];
        d_means[n + i] += (float)gm[1];
        d_means[2 * n + i] += (float)gm[2];
    }
    if (d_ls) {
        d_ls[i] += (float)(gs[0] * P.s[0]);
        d_ls[n + i] += (float)(gs[1] * P.s[1]);
        d_ls[2 * n + i] += (float)(gs[2] * P.s[2]);
    }
    if (d_op) d_op[i] += (float)go;
    if (d_col) {
        d_col[i] += (float)gc[0];
        d_col[n + i] += (float)gc[1];
        d_col[2 * n + i] += (float)gc[2];
    }
}

// ---------------------------------------------------------------- scoring
// Rendered form of the trace proxy of Sec. IV-A eq. (7): per view, the sum
// over pixels of the composited uncertainty sum_i u_i a_i T_i.  Only alpha,
// transmittance and uncertainty are composited; nothing is written per pixel.

// mode 0: sum_i u_i a_i T_i (the rendered proxy); mode 1: sum of u_i over
// the contributing splats (the binary-J trace).
//
// The pair loop is cut to the arithmetic the proxy needs.  Staged per splat:
// the mean relative to an origin fixed per 32 x 16 pixel block (a multiple
// of every tile shape, so no pixel's arithmetic depends on the tile), the
// whitening M, log2(opacity) and u; a pixel's offset is then one subtraction
// from a small exact integer, and alpha = min(alpha_max, exp2(log2 o - |Md|^2)).
// Bound by instruction issue, as k_render_fwd: with the thresholds in vector registers, one select
// instead of two per splat, the narrower band of the binary64 branch (which also freed the registers for eight
// waves per SIMD instead of six) 256 uneven views went from 3,536 to 2,816 us, 64 views of 320x240 from
// 891 to 698 us.
// Termination is carried by T itself: a pixel whose next transmittance
// would fall below T_min stops with T = 0, after which every splat leaves it
// unchanged, so the loop needs no per-pixel flags; a splat below alpha_min
// enters the update with alpha 0 (T unchanged, exactly).
template <int MODE>
__device__ __forceinline__ float score_weight(float a0, float T) {
    return MODE ? 1.0f : a0 * T;
}

template <int TW, int TH, int B, int MODE>
__device__ __forceinline__ void score_one_tile(const ViewDev* __restrict__ views, int n_views, uint32_t tile,
                                               const uint2* __restrict__ ranges,
                                               const uint32_t* __restrict__ inst_rec, const Records& rec,
                                               const SetDev& st, double* __restrict__ partial,
                                               float4* s_p, float4* s_q, uint32_t* s_r, uint2* s_pb,
                                               double* ws, uint32_t* s_list) {
    constexpr int NT = TW * TH;
    static_assert(32 % TW == 0 && 16 % TH == 0, "tiles must divide the 32 x 16 origin block");
    static_assert(SCORE_STEP == 2, "the list is padded for steps of two");
    const uint32_t vi = view_of_tile(views, n_views, tile);
    const ViewDev& V = views[vi];
    const uint32_t lt = tile - V.tile_off;
    const int tx = (int)(lt % (uint32_t)V.tiles_x), ty = (int)(lt / (uint32_t)V.tiles_x);
    const int u = tx * TW + (int)(threadIdx.x % TW), v = ty * TH + (int)(threadIdx.x / TW);
    const int ox = origin_x(tx * TW), oy = origin_y(ty * TH);
    // this wave's pixel rectangle (64 consecutive threads = 64 / TW rows of
    // the tile), relative to the origin
    const int wc0 = tx * TW - ox, wc1 = wc0 + TW - 1;
    const int wr0 = ty * TH + (int)(threadIdx.x >> 6) * (64 / TW) - oy, wr1 = wr0 + 64 / TW - 1;
    const bool inside = u < V.W && v < V.H;
    const float lx = (float)(u - ox), ly = (float)(v - oy);
    const float amin = in_vgpr(st.alpha_min), amax = in_vgpr(st.alpha_max), tmin = in_vgpr(st.T_min);
    const uint2 rg = ranges[tile];
    const char* sp = reinterpret_cast<const char*>(s_p);
    const char* sq = reinterpret_cast<const char*>(s_q);
    float T = inside ? 1.0f : 0.0f, uu = 0.0f;
    for (uint32_t b = rg.x; b < rg.y; b += B) {
        if (__syncthreads_count(T > 0.0f) == 0) break;
        uint32_t idx = b + threadIdx.x;
        bool odd = false;
        if (threadIdx.x < (uint32_t)B && idx < rg.y) {
            uint32_t r = inst_rec[idx];
            s_r[threadIdx.x] = r;
            const EmitRec e = rec.emit[r];
            s_pb[threadIdx.x] = e.pbox;
            odd = !isfinite(__uint_as_float(e.unc));
            stage_splat<true>(e, ox, oy, st, s_p[threadIdx.x], s_q[threadIdx.x]);
        }
        // an uncertainty that is not finite must not meet the weight 0 below (MODE 1 needs the barrier alone)
        if (MODE != 0) __syncthreads();
        const bool select = MODE != 0 || __builtin_amdgcn_readfirstlane(__syncthreads_or(odd));
        const int cnt = (int)min<uint32_t>(B, rg.y - b);
        uint32_t* my = s_list + (threadIdx.x >> 6) * (B + 2);
        int nl = 0;
        uint64_t alive = __ballot(T > 0.0f);
        if (alive)
            nl = splat_list<B, SCORE_ELL>(s_pb, s_p, s_q, st.log2_amin, cnt, wc0, wc1, wr0, wr1, ox, oy, my);
        __syncthreads();  // the wave's list is in LDS
        auto walk = [&](auto selected) {
            for (int i = 0; i < nl && alive; i += SCORE_STEP) {
                uint32_t ko[SCORE_STEP];
                float as[SCORE_STEP], us[SCORE_STEP], bs[SCORE_STEP];
                bool need = false;
#pragma unroll
                for (int q = 0; q < SCORE_STEP; q++) {
                    ko[q] = my[i + q];
                    const float4 p = *reinterpret_cast<const float4*>(sp + ko[q]);
                    const float4 g = *reinterpret_cast<const float4*>(sq + ko[q]);
                    const float dx = lx - p.x, dy = ly - p.y;
                    const float w1 = p.z * dx, w2 = fmaf(p.w, dx, g.x * dy);
                    const float ex = fmaf(w1, w1, fmaf(w2, w2, -g.y));
                    const float a = __builtin_amdgcn_fmed3f(fast_exp2(-ex), 0.0f, amax);
                    as[q] = a;
                    us[q] = g.z;
                    bs[q] = g.w;
                    need = need | near_amin(a, amin, bs[q]);
                }
                if (__ballot(need)) {
#pragma unroll
                    for (int q = 0; q < SCORE_STEP; q++)
                        if (near_amin(as[q], amin, bs[q]))
                            as[q] = redecide(as[q], rec, s_r[ko[q] / sizeof(float4)], u, v, st);
                }
#pragma unroll
                for (int q = 0; q < SCORE_STEP; q++) {
                    const bool ok = as[q] >= amin;
                    const float a0 = ok ? as[q] : 0.0f;
                    const float Tn = fmaf(-a0, T, T);
                    const bool live = Tn >= tmin;
                    if constexpr (decltype(selected)::value) {
                        const float w = score_weight<MODE>(a0, T);
                        uu = (ok & live) ? fmaf(us[q], w, uu) : uu;
                        T = live ? Tn : 0.0f;
                    } else {
                        // one select: a pixel that stops takes T = 0 first, so that its weight and
                        // its next T are 0; a skipped splat's weight is 0 through a0
                        const float T0 = live ? T : 0.0f;
                        uu = fmaf(us[q], a0 * T0, uu);
                        T = fmaf(-a0, T0, T0);
                    }
                    if (q + 1 == SCORE_STEP) alive = __ballot(live);
                }
            }
        };
        if (select) walk(BoolC<true>{});
        else walk(BoolC<false>{});
    }
    float s = wave_sum_f(uu);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = (double)s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double acc = 0.0;
        for (int w = 0; w < NT / 64; w++) acc += ws[w];
        partial[tile] = acc;
    }
    __syncthreads();
}

template <int TW, int TH, int B>
__global__ __launch_bounds__(TW * TH) void k_score_plain(const ViewDev* __restrict__ views, int n_views,
                                                         uint32_t tile_begin, const uint2* __restrict__ ranges,
                                                         const uint32_t* __restrict__ inst_rec, Records rec,
                                                         SetDev st, int mode, double* __restrict__ partial) {
    constexpr int NT = TW * TH;
    static_assert(B <= NT, "batch larger than the tile");
    __shared__ float4 s_p[B + 1], s_q[B + 1];
    __shared__ uint32_t s_r[B + 1];
    __shared__ uint2 s_pb[B];
    __shared__ double ws[NT / 64];
    __shared__ __align__(8) uint32_t s_list[NT / 64 * (B + 2)];
    stage_null_splat<B, true>(s_p, s_q);
    if (mode)
        score_one_tile<TW, TH, B, 1>(views, n_views, tile_begin + blockIdx.x, ranges, inst_rec, rec, st, partial,
                                     s_p, s_q, s_r, s_pb, ws, s_list);
    else
        score_one_tile<TW, TH, B, 0>(views, n_views, tile_begin + blockIdx.x, ranges, inst_rec, rec, st, partial,
                                     s_p, s_q, s_r, s_pb, ws, s_list);
}

template <int TW, int TH, int B>
__global__ __launch_bounds__(TW * TH) __attribute__((amdgpu_waves_per_eu(8))) void k_score_persistent(const ViewDev* __restrict__ views,
                                                              const Header* __restrict__ hdr,
                                                              const uint2* __restrict__ ranges,
                                                              const uint32_t* __restrict__ tile_order,
                                                              const uint32_t* __restrict__ inst_rec, Records rec,
                                                              SetDev st, int mode, double* __restrict__ partial,
                                                              uint32_t* __restrict__ queue,
                                                              const uint32_t* __restrict__ flags) {
    constexpr int NT = TW * TH;
    static_assert(B <= NT, "batch larger than the tile");
    if (*flags) return;  // overflowed binning: results are reported invalid
    __shared__ float4 s_p[B + 1], s_q[B + 1];
    __shared__ uint32_t s_r[B + 1];
    __shared__ uint2 s_pb[B];
    __shared__ double ws[NT / 64];
    __shared__ __align__(8) uint32_t s_list[NT / 64 * (B + 2)];
    stage_null_splat<B, true>(s_p, s_q);
    __shared__ uint32_t s_item;
    const uint32_t total = hdr->tiles_total;
    const int nv = (int)hdr->n_views;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t item = s_item;
        __syncthreads();
        if (item >= total) break;
        const uint32_t tile = tile_order ? tile_order[item] : item;
        if (mode)
            score_one_tile<TW, TH, B, 1>(views, nv, tile, ranges, inst_rec, rec, st, partial, s_p, s_q, s_r, s_pb,
                                         ws, s_list);
        else
            score_one_tile<TW, TH, B, 0>(views, nv, tile, ranges, inst_rec, rec, st, partial, s_p, s_q, s_r, s_pb,
                                         ws, s_list);
    }
}

__global__ __launch_bounds__(256) void k_score_reduce(const ViewDev* __restrict__ views,
                                                      const Header* __restrict__ hdr,
                                                      const double* __restrict__ partial,
                                                      double* __restrict__ scores,
                                                      const uint32_t* __restrict__ flags,
                                                      uint32_t* __restrict__ flag_host) {
    __shared__ double ws[4];
    const uint32_t v = blockIdx.x;
    if (flag_host && v == 0 && threadIdx.x == 0)
        __hip_atomic_store(flag_host, *flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (v >= hdr->n_views) return;
    if (*flags) {  // an overflowed or inconsistent binning: the scores are invalid
        if (threadIdx.x == 0) scores[v] = __builtin_nan("");
        return;
    }
    const ViewDev& V = views[v];
    const uint32_t nt = (uint32_t)(V.tiles_x * V.tiles_y);
    double s = 0.0;
    for (uint32_t t = threadIdx.x; t < nt; t += 256) s += partial[V.tile_off + t];
    s = wave_sum_d(s);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) scores[v] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

__global__ __launch_bounds__(256) void k_export(const uint32_t* __restrict__ tile_key,
                                                const uint32_t* __restrict__ inst_rec,
                                                const uint32_t* __restrict__ K_dev, uint32_t cap, Records rec,
                                                uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    uint32_t K = min(*K_dev, cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < K; i += gridDim.x * blockDim.x) {
        uint32_t r = inst_rec[i];
        if (keys) keys[i] = ((uint64_t)tile_key[i] << 32) | __float_as_uint(rec.attr[r].w);
        if (vals) vals[i] = rec.emit[r].gid;
    }
}

// Planar copies of the record fields for inspection (all outputs nullable).
__global__ __launch_bounds__(256) void k_export_records(const uint32_t* __restrict__ R_dev, uint32_t cap, Records rec,
                                                        double* __restrict__ mean2d, double* __restrict__ conic,
                                                        int32_t* __restrict__ pbox, uint32_t* __restrict__ depth_bits,
                                                        uint32_t* __restrict__ gid, uint32_t* __restrict__ view,
                                                        uint32_t* __restrict__ ntiles) {
    const uint32_t R = min(*R_dev, cap);
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < R; r += gridDim.x * blockDim.x) {
        const EmitRec e = rec.emit[r];
        if (mean2d) {
            mean2d[r] = (double)e.g0.x + (double)e.g0.z;
            mean2d[(uint64_t)R + r] = (double)e.g0.y + (double)e.g0.w;
        }
        if (conic) {
            const double4 q = rec.q64[r];
            conic[r] = q.x;
            conic[(uint64_t)R + r] = q.y;
            conic[2 * (uint64_t)R + r] = q.z;
        }
        if (pbox) {
            pbox[r] = (int32_t)(e.pbox.x & 0xffffu);
            pbox[(uint64_t)R + r] = (int32_t)(e.pbox.x >> 16);
            pbox[2 * (uint64_t)R + r] = (int32_t)(e.pbox.y & 0xffffu);
            pbox[3 * (uint64_t)R + r] = (int32_t)(e.pbox.y >> 16);
        }
        if (depth_bits) depth_bits[r] = __float_as_uint(rec.attr[r].w);
        if (gid) gid[r] = e.gid;
        if (view) view[r] = e.view;
        if (ntiles) ntiles[r] = e.ntiles;
    }
}

__global__ __launch_bounds__(256) void k_sum_counts(const uint64_t* __restrict__ a, uint64_t na,
                                                    const uint32_t* __restrict__ b, uint64_t nb,
                                                    unsigned long long* __restrict__ out) {
    __shared__ unsigned long long ws[2][4];
    unsigned long long sa = 0, sb = 0;
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = i0; i < na; i += stride) sa += a[i];
    for (uint64_t i = i0; i < nb; i += stride) sb += b[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sa += __shfl_xor(sa, o, 64);
        sb += __shfl_xor(sb, o, 64);
    }
    if (lane_id() == 0) {
        ws[0][threadIdx.x >> 6] = sa;
        ws[1][threadIdx.x >> 6] = sb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(out, ws[0][0] + ws[0][1] + ws[0][2] + ws[0][3]);
        atomicAdd(out + 1, ws[1][0] + ws[1][1] + ws[1][2] + ws[1][3]);
    }
}

// ------------------------------------------------ view utility of eq. (8)
// Sec. IV-B: v(x, g) = 1 when the Gaussian is in the field of view (camera
// depth in (z_near, range], projected mean inside the image, no occlusion);
// xi = |H visible| - lambda |L visible| with H / L the Gaussians above / below
// the uncertainty thresholds.  The visibility test runs in binary32 and falls
// back to the exact binary64 expression within a margin of every border.

constexpr int UT_THREADS = 256;
constexpr double FIX_SCALE = 1099511627776.0;  // 2^40: uncertainty sums in fixed point

__device__ __forceinline__ bool fov_exact(double mx0, double my0, double mz0, const ViewDev& V, double z_near,
                                          double range) {
    double dx = mx0 - V.T[0], dy = my0 - V.T[1], dz = mz0 - V.T[2];
    const double* R = V.R;
    double tx = (dx * R[0] + dy * R[3]) + dz * R[6];
    double ty = (dx * R[1] + dy * R[4]) + dz * R[7];
    double tz = (dx * R[2] + dy * R[5]) + dz * R[8];
    if (!(tz > z_near) || !(tz <= range)) return false;
    double mx = V.fx * tx / tz + V.cx;
    double my = V.fy * ty / tz + V.cy;
    return mx >= 0.0 && mx <= (double)(V.W - 1) && my >= 0.0 && my <= (double)(V.H - 1);
}

// Screen of the field-of-view test.  With p the mean, d = R^T (p - T) its camera coordinates and
// h = (W - 1) / 2, the projection lies inside the image's columns where |s_x| <= d_z, s_x = (fx d_x +
// (cx - h) d_z) / h, for d_z > 0: s_x is a linear form of (p, 1); likewise s_y; and the depth is in
// (z_near, range].  So one number e = max(|s_x| - d_z, |s_y| - d_z, z_near - d_z, d_z - range)
// decides: visible where e < -m, not where e > m, and the binary64 test between.
// m = k |p|_1 + c bounds the rounding of the forms: a coefficient's (2^-24), the two
// products of third parts that are left out (2^-23) and at most 26 roundings or truncations
// (2^-23) of sums below k |p|_1 + c; UT_EPS is over twice that.  (The rounding of a large range
// matters only near d_z = range, where |p|_1 or |T| is as large.)  A coefficient or a mean beyond
// UT_HUGE, or an image one pixel wide or high, gets an infinite m, which leaves the decision to
// the binary64 test.
constexpr float UT_EPS = 8e-6f;
constexpr float UT_HUGE = 1e15f;

struct ViewScreen {
    float row[4][4];  // s_x, s_y, d_z as forms of (x, y, z, 1); the fourth is 0
    float k, c;       // margin
};

__device__ inline ViewScreen view_screen(const ViewDev& V, double z_near) {
    const double h[2] = {0.5 * (V.W - 1), 0.5 * (V.H - 1)};
    const double along[2] = {V.fx / h[0], V.fy / h[1]}, off[2] = {(V.cx - h[0]) / h[0], (V.cy - h[1]) / h[1]};
    double kmax = 0.0, cmax = 0.0;
    ViewScreen s;
    for (int r = 0; r < 3; r++) {
        double bias = 0.0, k = 0.0, c = z_near;
        for (int a = 0; a < 3; a++) {
            const double z = V.R[3 * a + 2], f = r < 2 ? along[r] * V.R[3 * a + r] + off[r] * z : z;
            bias -= f * V.T[a];
            s.row[r][a] = (float)f;
            // the form's own terms and those of the d_z it is compared with
            k = fmax(k, fabs(f) + fabs(z));
            c += (fabs(f) + fabs(z)) * fabs(V.T[a]);
        }
        s.row[r][3] = (float)bias;
        // the negated test also takes a NaN
        kmax = k < UT_HUGE ? fmax(kmax, k) : HUGE_VAL;
        cmax = c < UT_HUGE ? fmax(cmax, c) : HUGE_VAL;
    }
    for (int a = 0; a < 4; a++) s.row[3][a] = 0.0f;
    s.k = UT_EPS * (float)kmax;
    s.c = UT_EPS * (float)cmax;
    if (!(kmax < UT_HUGE) || !(cmax < UT_HUGE)) {
        for (int r = 0; r < 3; r++)
            for (int a = 0; a < 4; a++) s.row[r][a] = 0.0f;
        s.k = 0.0f;
        s.c = __builtin_inff();
    }
    return s;
}

// The forms of four views at 16 Gaussians are one matrix product: 16 rows (three forms per view and a
// spare one) by the columns (x, y, z, 1), each binary32 number the exact sum of three bfloat16
// parts (high, mid, low) and each product the six leading products of parts, 24 of the 32 columns of
// v_mfma_f32_16x16x32_bf16.  Lane l then holds the forms of view l / 16 at Gaussian l % 16.
// Measured for 576 views x 2M Gaussians: one projection per lane with a reciprocal and
// twelve compares (about 65 vector instructions a test) 1,823 us; the product in binary32
// (v_mfma_f32_16x16x4_f32, which the vector unit does not overlap) 755 us; this 501 us, of which the
// tests' eight vector instructions take most.
// A block takes UT_VB views (their forms in registers) and a share of the Gaussians, 64 per
// wave and step; counts and fixed-point sums stay in registers, per lane and view, until the
// end.  They are integers: the result does not depend on the order.
constexpr int UT_GROUPS = 8;  // of four views
constexpr int UT_VB = 4 * UT_GROUPS;
constexpr int64_t UT_LANE_MAX = 60000;  // Gaussians per lane and view: the two counts share a word

constexpr int UT_CHUNK = 4;
static_assert(UT_GROUPS % UT_CHUNK == 0 && UT_CHUNK == 4, "whole chunks, four minima");

// Maxima without the quieting of their operands that fmaxf asks for (it would double their count).
__device__ __forceinline__ float max2(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// max(|a|, |b|, c), c uniform, of matrix-core results a and b.  `after`, unused, was formed from the same
// result by ordinary code, which has waited for it.
__device__ __forceinline__ float max_abs(float a, float b, float c, float after) {
    float r;
    asm("v_max3_f32 %0, |%1|, |%2|, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c), "v"(after));
    return r;
}
// The least magnitude of four.
__device__ __forceinline__ float min_abs4(float a, float b, float c, float d) {
    float r;
    asm("v_min3_f32 %0, |%1|, |%2|, |%3|\n\tv_min_f32 %0, %0, |%4|" : "=&v"(r) : "v"(a), "v"(b), "v"(c), "v"(d));
    return r;
}

// a += x and b += y in the lanes of m (two vector instructions under the mask instead of the five of
// two sums and three selects).
__device__ __forceinline__ void add_where(uint64_t m, uint32_t& a, uint32_t x, unsigned long long& b,
                                          unsigned long long y) {
    uint64_t keep;
    asm volatile("s_and_saveexec_b64 %2, %3\n\tv_add_u32 %0, %0, %4\n\tv_lshl_add_u64 %1, %5, 0, %1\n\ts_mov_b64 exec, %2"
                 : "+v"(a), "+v"(b), "=&s"(keep)
                 : "s"(m), "v"(x), "v"(y)
                 : "scc");
}

using f32x4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;
using bf16x8 = __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16;

// A binary32 number as three bfloat16 parts (their exact sum): .x = mid << 16 | high, .y = high << 16 | low.
__device__ __forceinline__ uint2 split_bf16(float x) {
    const uint32_t h = __float_as_uint(x) & 0xffff0000u;
    const float r = x - __uint_as_float(h);
    const uint32_t m = __float_as_uint(r) & 0xffff0000u;
    const uint32_t l = __float_as_uint(r - __uint_as_float(m));
    return make_uint2(h >> 16 | m, l >> 16 | h);
}
// One component's eight columns: A (h, h, m, m, l, h, 0, 0) against B (h, m, h, m, h, l, 0, 0).
__device__ __forceinline__ bf16x8 operand_a(uint2 p) {
    const uint32_t h = p.x & 0xffffu, m = p.x >> 16;
    const uint4 v = make_uint4(h | h << 16, m | m << 16, (p.y & 0xffffu) | h << 16, 0u);
    return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ bf16x8 operand_b(uint2 p) {
    return __builtin_bit_cast(bf16x8, make_uint4(p.x, p.x, p.y >> 16 | p.y << 16, 0u));
}

__global__ __launch_bounds__(UT_THREADS, 4) void k_view_utility(GaussDev g, const ViewDev* __restrict__ views, int nv,
                                                             float z_near, float range,
                                                             const double* __restrict__ lo_hi,
                                                             unsigned long long* __restrict__ cnt_h,
                                                             unsigned long long* __restrict__ cnt_l,
                                                             unsigned long long* __restrict__ fix_u) {
    constexpr int WAVES = UT_THREADS / 64;
    __shared__ float s_row[UT_VB][4][4];
    __shared__ float2 s_h[UT_VB];  // margins
    __shared__ uint2 s_x[WAVES][3][64];  // the split mean
    __shared__ uint4 s_d[WAVES][64];     // counts' increments, fixed-point u (two words), margin
    __shared__ unsigned long long s_sum[3][UT_VB];
    __shared__ uint16_t s_ask[WAVES][64 * UT_GROUPS];  // Gaussian of the step | view << 6
    const int v0 = (int)blockIdx.y * UT_VB;
    const int nvb = min(UT_VB, nv - v0), ngr = (nvb + 3) / 4;
    const int lane = (int)lane_id(), wv = (int)threadIdx.x >> 6, col = lane & 15, quad = lane >> 4;
    if ((int)threadIdx.x < UT_VB) {
        ViewScreen s;
        if ((int)threadIdx.x < nvb) {
            s = view_screen(views[v0 + threadIdx.x], (double)z_near);
        } else {  // sees nothing
            for (int r = 0; r < 4; r++)
                for (int a = 0; a < 4; a++) s.row[r][a] = 0.0f;
            s.row[2][3] = -1e38f;
            s.k = s.c = 0.0f;
        }
        for (int r = 0; r < 4; r++)
            for (int a = 0; a < 4; a++) s_row[threadIdx.x][r][a] = s.row[r][a];
        s_h[threadIdx.x] = make_float2(s.k, s.c);
        s_sum[0][threadIdx.x] = s_sum[1][threadIdx.x] = s_sum[2][threadIdx.x] = 0ull;
    }
    __syncthreads();
    bf16x8 A[UT_GROUPS];
    uint32_t cnt[UT_GROUPS];
    unsigned long long su[UT_GROUPS];
#pragma unroll
    for (int q = 0; q < UT_GROUPS; q++) {
        // operand A: row lane % 16 (view of four, form), columns of component lane / 16
        A[q] = operand_a(split_bf16(s_row[4 * q + (col >> 2)][col & 3][quad]));
        cnt[q] = 0u;
        su[q] = 0ull;
    }
    // one margin for the block's views
    float mk = 0.0f, mc = 0.0f;
    for (int v = 0; v < nvb; v++) {
        mk = fmaxf(mk, s_h[v].x);
        mc = fmaxf(mc, s_h[v].y);
    }
    const double lo = lo_hi[0], hi = lo_hi[1];
    const int64_t n = g.n;
    const int64_t stride = (int64_t)gridDim.x * UT_THREADS;
    int64_t base = (int64_t)blockIdx.x * UT_THREADS + wv * 64;
    int nask = 0;
    float raw[4];
    auto fetch = [&](int64_t i0) {
        const int64_t i = min(i0 + lane, n - 1);
        raw[0] = g.means[i];
        raw[1] = g.means[n + i];
        raw[2] = g.means[2 * n + i];
        raw[3] = g.uncert[i];
    };
    if (base < n) fetch(base);
    for (; base < n; base += stride) {
        const float u = raw[3];
        // a Gaussian past the end or without a finite mean counts nothing
        const bool ok = base + lane < n && isfinite(raw[0]) && isfinite(raw[1]) && isfinite(raw[2]);
        const uint32_t inc = !ok ? 0u : ((double)u > hi ? 1u : 0u) | ((double)u < lo ? 0x10000u : 0u);
        const unsigned long long fu =
            ok && isfinite(u) && u > 0.0f ? (unsigned long long)((double)u * FIX_SCALE) : 0ull;
        const float mag = fabsf(raw[0]) + fabsf(raw[1]) + fabsf(raw[2]);
        const bool tame = ok && mag < UT_HUGE;
#pragma unroll
        for (int a = 0; a < 3; a++) s_x[wv][a][lane] = split_bf16(tame ? raw[a] : 0.0f);
        // 0 <= mk, mc; one that counts nothing needs no second look
        const float margin = !ok ? 0.0f : tame ? fmaf(mk, mag, mc) : __builtin_inff();
        s_d[wv][lane] = make_uint4(inc, (uint32_t)fu, (uint32_t)(fu >> 32), __float_as_uint(margin));
        if (base + stride < n) fetch(base + stride);  // in flight during this step
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int s = 0; s < 4; s++) {
            // operand B: columns of component lane / 16 (the fourth is 1) of Gaussian lane % 16
            const uint2 bx = s_x[wv][min(quad, 2)][16 * s + col];
            const bf16x8 B = operand_b(quad < 3 ? bx : make_uint2(0x3f80u, 0x3f800000u));
            const uint4 d = s_d[wv][16 * s + col];
            const float m = __uint_as_float(d.w);
            const unsigned long long du = (unsigned long long)d.z << 32 | d.y;
            // UT_CHUNK products in flight, then their tests; groups past the last view see nothing
#pragma unroll
            for (int q0 = 0; q0 < UT_GROUPS; q0 += UT_CHUNK) {
                if (q0 >= ngr) break;
                f32x4 f[UT_CHUNK];
#pragma unroll
                for (int k = 0; k < UT_CHUNK; k++)
                    f[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[q0 + k], B, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
                float e[UT_CHUNK];
                uint64_t vis[UT_CHUNK];
#pragma unroll
                for (int k = 0; k < UT_CHUNK; k++) {
                    const float beyond = f[k][2] - range;
                    e[k] = max2(max_abs(f[k][0], f[k][1], z_near, beyond) - f[k][2], beyond);
                    vis[k] = __ballot(e[k] < -m);
                }
                // the least |e| tells whether any test is undecided (also with an infinite m)
                if (__ballot(!(min_abs4(e[0], e[1], e[2], e[3]) > m))) {
#pragma unroll
                    for (int k = 0; k < UT_CHUNK; k++) {
                        const uint64_t um = __ballot(!(e[k] > m)) & ~vis[k];
                        if ((um >> lane) & 1ull)
                            s_ask[wv][nask + (int)__popcll(um & lanemask_lt())] =
                                (uint16_t)(16 * s + col + ((4 * (q0 + k) + quad) << 6));
                        nask += (int)__popcll(um);
                    }
                }
#pragma unroll
                for (int k = 0; k < UT_CHUNK; k++) add_where(vis[k], cnt[q0 + k], d.x, su[q0 + k], du);
            }
            // the undecided tests of this turn, a pair (Gaussian, view) per lane; rare, so they go to
            // the block's sums one by one
            if (nask == 0) continue;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int a = lane; a < nask; a += 64) {
                const int j = s_ask[wv][a] & 63, v = s_ask[wv][a] >> 6;
                const int64_t i = base + j;
                if (i >= n || v >= nvb) continue;
                if (!fov_exact((double)g.means[i], (double)g.means[n + i], (double)g.means[2 * n + i], views[v0 + v],
                               (double)z_near, (double)range))
                    continue;
                const uint4 e = s_d[wv][j];
                atomicAdd(&s_sum[0][v], (unsigned long long)(e.x & 0xffffu));
                atomicAdd(&s_sum[1][v], (unsigned long long)(e.x >> 16));
                atomicAdd(&s_sum[2][v], (unsigned long long)e.z << 32 | e.y);
            }
            nask = 0;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int q = 0; q < UT_GROUPS; q++) {
        uint32_t h = cnt[q] & 0xffffu, l = cnt[q] >> 16;
        unsigned long long t = su[q];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            h += (uint32_t)__shfl_xor((int)h, o, 64);
            l += (uint32_t)__shfl_xor((int)l, o, 64);
            t += __shfl_xor(t, o, 64);
        }
        if (col == 0) {
            atomicAdd(&s_sum[0][4 * q + quad], (unsigned long long)h);
            atomicAdd(&s_sum[1][4 * q + quad], (unsigned long long)l);
            atomicAdd(&s_sum[2][4 * q + quad], t);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nvb) {
        const int v = v0 + (int)threadIdx.x;
        if (s_sum[0][threadIdx.x]) atomicAdd(cnt_h + v, s_sum[0][threadIdx.x]);
        if (s_sum[1][threadIdx.x]) atomicAdd(cnt_l + v, s_sum[1][threadIdx.x]);
        if (s_sum[2][threadIdx.x]) atomicAdd(fix_u + v, s_sum[2][threadIdx.x]);
    }
}

__global__ void k_utility_finish(int nv, const unsigned long long* __restrict__ cnt_h,
                                 const unsigned long long* __restrict__ cnt_l,
                                 const unsigned long long* __restrict__ fix_u, double lambda,
                                 int64_t* __restrict__ n_high, int64_t* __restrict__ n_low,
                                 double* __restrict__ sum_u, double* __restrict__ xi) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
        if (n_high) n_high[v] = (int64_t)cnt_h[v];
        if (n_low) n_low[v] = (int64_t)cnt_l[v];
        if (sum_u) sum_u[v] = (double)fix_u[v] / FIX_SCALE;
        if (xi) xi[v] = (double)cnt_h[v] - lambda * (double)cnt_l[v];
    }
}

// Mean and population standard deviation of u, binary64, fixed reduction order: the
// blocks' partial sums (MO_BLOCKS of them at most), then the partial sums of the squared deviations
// from the mean, which every block forms from the first pass's partial sums itself.
constexpr int MO_BLOCKS = 512;

// The sum of partial[0 .. nb), the same in every block of 256 threads that forms it.
__device__ __forceinline__ double sum_partials_256(const double* __restrict__ partial, int nb, double* ws) {
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) s += partial[b];
    s = wave_sum_d(s);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    s = (ws[0] + ws[1]) + (ws[2] + ws[3]);
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(256) void k_moments(const float* __restrict__ u, int64_t n, int pass,
                                                 const double* __restrict__ sums, double* __restrict__ partial) {
    __shared__ double ws[4];
    const double mean = pass ? sum_partials_256(sums, (int)gridDim.x, ws) / (double)n : 0.0;
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        double d = (double)u[i] - mean;
        s += pass ? d * d : (double)u[i];
    }
    s = wave_sum_d(s);
    if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

__global__ __launch_bounds__(256) void k_moments_finish(const double* __restrict__ sums, const double* __restrict__ sq,
                                                        int nb, int64_t n, double k, double* __restrict__ lo_hi) {
    __shared__ double ws[4];
    const double mean = n > 0 ? sum_partials_256(sums, nb, ws) / (double)n : 0.0;
    const double sd = n > 0 ? sqrt(sum_partials_256(sq, nb, ws) / (double)n) : 0.0;
    if (threadIdx.x == 0) {
        lo_hi[0] = mean - k * sd;
        lo_hi[1] = mean + k * sd;
    }
}

// eq. (10): utility of trajectory t = sum of xi over its states
// [off[t], off[t+1]) in order; best = first trajectory of maximal utility.
// One block, a trajectory per thread (one thread for all of them waited for 576 loads in turn:
// 39 us), TS_BATCH of its loads in flight and added in order (one trajectory of 100,000 states: 6,620 us with one
// load at a time, 1,000 now).  A NaN utility is never greater, and nothing is greater than a NaN first one.
constexpr int TS_BATCH = 16;

__global__ __launch_bounds__(256) void k_traj_select(const double* __restrict__ xi, const int32_t* __restrict__ off,
                                                     int n_traj, double* __restrict__ util,
                                                     int32_t* __restrict__ best) {
    __shared__ double s_v[256];
    __shared__ int s_t[256];
    __shared__ int s_nan;
    int b = n_traj;  // none
    double bv = 0.0;
    for (int t = threadIdx.x; t < n_traj; t += 256) {
        double s = 0.0;
        const int end = off[t + 1];
        int k = off[t];
        for (; k <= end - TS_BATCH; k += TS_BATCH) {
            double x[TS_BATCH];
#pragma unroll
            for (int j = 0; j < TS_BATCH; j++) x[j] = xi[k + j];
#pragma unroll
            for (int j = 0; j < TS_BATCH; j++) s += x[j];
        }
        for (; k < end; k++) s += xi[k];
        if (util) util[t] = s;
        if (t == 0) s_nan = s != s;
        if (s == s && (b == n_traj || s > bv)) {
            b = t;
            bv = s;
        }
    }
    s_v[threadIdx.x] = bv;
    s_t[threadIdx.x] = b;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            const int t2 = s_t[threadIdx.x + o], t1 = s_t[threadIdx.x];
            const double v2 = s_v[threadIdx.x + o], v1 = s_v[threadIdx.x];
            if (t2 < n_traj && (t1 == n_traj || v2 > v1 || (v2 == v1 && t2 < t1))) {
                s_t[threadIdx.x] = t2;
                s_v[threadIdx.x] = v2;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *best = s_nan ? 0 : s_t[0];
}

inline unsigned grid_for(uint64_t n, unsigned block, unsigned cap = 65535u * 16u) {
    uint64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

// ------------------------------------------------- uncertainty bookkeeping
// Sec. IV-A: the uncertainty of a Gaussian is the magnitude of the change of
// its mean over a map update (squared for the -sq variant); a Gaussian whose
// mean did not change keeps its previous value.  Formed in binary64 as
// sqrt((dx dx + dy dy) + dz dz) and rounded once to binary32.

__global__ __launch_bounds__(256) void k_uncertainty_update(int64_t n, const float* __restrict__ prev,
                                                            const float* __restrict__ cur,
                                                            const float* u_prev, int squared, float* u_out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double dx = (double)cur[i] - (double)prev[i];
        const double dy = (double)cur[n + i] - (double)prev[n + i];
        const double dz = (double)cur[2 * n + i] - (double)prev[2 * n + i];
        float u;
        if (dx == 0.0 && dy == 0.0 && dz == 0.0) {
            u = u_prev[i];
        } else {
            const double s2 = (dx * dx + dy * dy) + dz * dz;
            u = (float)(squared ? s2 : sqrt(s2));
        }
        u_out[i] = u;
    }
}

// ---------------------------------------------------------- region utility
// Sec. IV-B (high-level planner; the 2.5 m edge is set in Sec. IV-C): cuboid
// regions of edge `size` over the box [lo, lo + dims size);
// a Gaussian belongs to region (ix, iy, iz), index ix + nx (iy + ny iz), with
// i = floor((mu - lo) / size) in binary64.  Counts are exact; sums are in
// fixed point with 2^-32 resolution (|u| < 2^20 per value), so the result
// does not depend on the order of the atomics.  A non-finite or out-of-range
// u marks its region (its sum and mean become NaN).

constexpr double RG_FIX = 4294967296.0;  // 2^32
constexpr int RG_LDS = 2048;             // regions privatised in LDS per block

__device__ __forceinline__ int64_t region_of(float mx, float my, float mz, double lx, double ly, double lz, double size,
                                             int nx, int ny, int nz) {
    const double fx = floor(((double)mx - lx) / size);
    const double fy = floor(((double)my - ly) / size);
    const double fz = floor(((double)mz - lz) / size);
    if (!(fx >= 0.0 && fx < (double)nx && fy >= 0.0 && fy < (double)ny && fz >= 0.0 && fz < (double)nz)) return -1;
    return (int64_t)fx + (int64_t)nx * ((int64_t)fy + (int64_t)ny * (int64_t)fz);
}

// Bound by the latency of a thread's turns (few blocks, so that few add their tables up at the end): RG_BATCH
// Gaussians a turn, all their loads in flight, and by the blocks that add their tables up at the end: 2 M Gaussians, 128
// regions: 256 blocks of 1,024 threads 16.4 us, 128 20.7, 512 18.1; blocks of 256 threads that took one Gaussian a turn:
// 34 us with 488 of them, 47 with 1,953.
constexpr int RG_BATCH = 4;
constexpr int RG_THREADS = 1024;
constexpr unsigned RG_BLOCKS = 256;

__global__ __launch_bounds__(RG_THREADS) void k_region_utility(int64_t n, const float* __restrict__ means,
                                                        const float* __restrict__ u, double lx, double ly,
                                                        double lz, double size, int nx, int ny, int nz,
                                                        unsigned long long* __restrict__ cnt,
                                                        unsigned long long* __restrict__ fix,
                                                        unsigned int* __restrict__ bad) {
    __shared__ unsigned long long s_cnt[RG_LDS], s_fix[RG_LDS];
    const int64_t nr = (int64_t)nx * ny * nz;
    const bool lds = nr <= RG_LDS;
    if (lds) {
        for (int r = threadIdx.x; r < nr; r += blockDim.x) s_cnt[r] = s_fix[r] = 0ull;
        __syncthreads();
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += RG_BATCH * stride) {
        float m[RG_BATCH][4];
#pragma unroll
        for (int k = 0; k < RG_BATCH; k++) {
            const int64_t i = i0 + k * stride;
            const bool in = i < n;
            m[k][0] = in ? means[i] : 0.0f;
            m[k][1] = in ? means[n + i] : 0.0f;
            m[k][2] = in ? means[2 * n + i] : 0.0f;
            m[k][3] = in ? u[i] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < RG_BATCH; k++) {
            const int64_t r = region_of(m[k][0], m[k][1], m[k][2], lx, ly, lz, size, nx, ny, nz);
            if (r < 0 || i0 + k * stride >= n) continue;
            const float v = m[k][3];
            const bool ok = isfinite(v) && fabsf(v) < 1048576.0f;
            const long long f = ok ? __double2ll_rn((double)v * RG_FIX) : 0ll;
            if (!ok) atomicOr(&bad[r], 1u);
            if (lds) {
                atomicAdd(&s_cnt[r], 1ull);
                atomicAdd(&s_fix[r], (unsigned long long)f);  // two's complement: signed sums wrap correctly
            } else {
                atomicAdd(&cnt[r], 1ull);
                atomicAdd(&fix[r], (unsigned long long)f);
            }
        }
    }
    if (lds) {
        __syncthreads();
        for (int r = threadIdx.x; r < nr; r += blockDim.x) {
            if (s_cnt[r]) {
                atomicAdd(&cnt[r], s_cnt[r]);
                atomicAdd(&fix[r], s_fix[r]);
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_region_finish(int64_t nr, const unsigned long long* __restrict__ cnt,
                                                       const unsigned long long* __restrict__ fix,
                                                       const unsigned int* __restrict__ bad,
                                                       int64_t* __restrict__ count, double* __restrict__ sum,
                                                       double* __restrict__ mean) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nr; r += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = (int64_t)cnt[r];
        const double sm = bad[r] ? __longlong_as_double(0x7ff8000000000000ll) : (double)(long long)fix[r] / RG_FIX;
        if (count) count[r] = c;
        if (sum) sum[r] = sm;
        if (mean) mean[r] = c ? sm / (double)c : 0.0;
    }
}

}  // namespace

// ================================================================ launchers

#define RTG_TILE_DISPATCH(TW_, TH_, CALL)                      \
    if (tw == 8 && th == 8) {                                  \
        constexpr int TW_ = 8, TH_ = 8;                        \
        CALL;                                                  \
    } else if (tw == 32 && th == 8) {                          \
        constexpr int TW_ = 32, TH_ = 8;                       \
        CALL;                                                  \
    } else {                                                   \
        constexpr int TW_ = 16, TH_ = 16;                      \
        CALL;                                                  \
    }


// Tile and staging batch: batch 0 means one splat per thread of the tile;
// otherwise one of 32, 64, 128, 256 not above the tile's pixel count
// (checked by the library before any launch).
#define RTG_BATCH_DISPATCH(TW_, TH_, B_, CALL)                 \
    RTG_TILE_DISPATCH(TW_, TH_, {                              \
        const int bsel_ = batch > 0 ? batch : TW_ * TH_;       \
        if (bsel_ == 32) {                                     \
            constexpr int B_ = 32;                             \
            CALL;                                              \
        } else if (bsel_ == 64 || TW_ * TH_ == 64) {           \
            constexpr int B_ = 64;                             \
            CALL;                                              \
        } else if (bsel_ == 128) {                             \
            constexpr int B_ = (TW_ * TH_ >= 128) ? 128 : 64;  \
            CALL;                                              \
        } else {                                               \
            constexpr int B_ = (TW_ * TH_ >= 256) ? 256 : 64;  \
            CALL;                                              \
        }                                                      \
    })

int score_persistent_blocks(int tw, int th, int batch) {
    int per_cu = 0;
    hipError_t e = hipSuccess;
    RTG_BATCH_DISPATCH(TW, TH, B,
                       (e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_score_persistent<TW, TH, B>,
                                                                         TW * TH, 0)));
    if (e != hipSuccess || per_cu < 1) per_cu = 1;
    return per_cu * device_cu_count();
}

void view_utility(const GaussDev& g, const ViewDev* views, int nv, float z_near, float range, const double* lo_hi,
                  unsigned long long* acc, double lambda, int64_t* n_high, int64_t* n_low, double* sum_u, double* xi,
                  hipStream_t s) {
    fill_u32(reinterpret_cast<uint32_t*>(acc), 0u, (uint64_t)6 * nv, s);
    if (g.n > 0) {
        // about 2048 blocks over (Gaussian shares) x (groups of UT_VB views), more where a lane's
        // share would not fit its counters (a step gives each lane four Gaussians a view)
        const unsigned gy = (unsigned)((nv + UT_VB - 1) / UT_VB);
        const unsigned gmax = grid_for((uint64_t)g.n, UT_THREADS, 1u << 30);
        const unsigned gfit = (unsigned)(g.n * 4 / (UT_THREADS * UT_LANE_MAX) + 1);
        const unsigned gx = std::max(gfit, std::min(gmax, (2048u + gy - 1) / gy));
        k_view_utility<<<dim3(gx, gy), UT_THREADS, 0, s>>>(g, views, nv, z_near, range, lo_hi, acc, acc + nv,
                                                           acc + 2 * nv);
    }
    k_utility_finish<<<(nv + 255) / 256, 256, 0, s>>>(nv, acc, acc + nv, acc + 2 * nv, lambda, n_high, n_low, sum_u,
                                                      xi);
}

void uncertainty_thresholds(const float* u, int64_t n, double k, double* scratch, double* lo_hi, hipStream_t s) {
    const int nb = (int)grid_for((uint64_t)std::max<int64_t>(n, 1), 256, MO_BLOCKS);
    double* sums = scratch;
    double* sq = scratch + MO_BLOCKS;
    k_moments<<<nb, 256, 0, s>>>(u, n, 0, nullptr, sums);
    k_moments<<<nb, 256, 0, s>>>(u, n, 1, sums, sq);
    k_moments_finish<<<1, 256, 0, s>>>(sums, sq, nb, n, k, lo_hi);
}

void trajectory_select(const double* xi, const int32_t* offsets, int n_traj, double* util, int32_t* best,
                       hipStream_t s) {
    k_traj_select<<<1, 256, 0, s>>>(xi, offsets, n_traj, util, best);
}

int device_cu_count() {
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cu;
}

void fill_u32(uint32_t* p, uint32_t v, uint64_t n, hipStream_t s) {
    if (n == 0) return;
    k_fill_u32<<<grid_for(n, 256, 4096), 256, 0, s>>>(p, v, n);
}

void project_count(const GaussDev& g, const ViewDev* views, const Header* hdr, int n_views_cap, SetDev st,
                   uint32_t* cnt, uint32_t* mask, uint32_t* zero, int n_zero, hipStream_t s) {
    if (g.n == 0) {
        fill_u32(zero, 0u, n_zero, s);
        return;
    }
    int words = (n_views_cap + 31) / 32;
    // one thread per Gaussian: the grid covers every n below 2^31
    if (n_views_cap <= PC_FEW)
        k_project_count<<<grid_for(g.n, 256, 0xffffffffu), 256, 0, s>>>(g, views, hdr, st, cnt, mask, zero, n_zero);
    else
        k_project_count_queued<PC_VIEWS, 512><<<grid_for(g.n, 512, 0xffffffffu), 512, 0, s>>>(g, views, hdr, words, st, cnt, mask, zero,
                                                                                               n_zero);
}

// log2 of a power-of-two tile side (8, 16 or 32)
static int ilog2(int x) {
    int k = 0;
    while ((1 << (k + 1)) <= x) k++;
    return k;
}

void project_emit(const GaussDev& g, const ViewDev* views, const Header* hdr, int n_views_cap, SetDev st,
                  int tw, int th, const uint32_t* mask, const uint32_t* cnt, const uint32_t* rec_off,
                  const uint32_t* R_dev, uint32_t rec_cap, Records rec, uint32_t* sortkey,
                  bool write_attr, uint32_t* chunk_g, bool owners, uint32_t* flags, hipStream_t s) {
    (void)hdr;
    if (g.n == 0 || rec_cap == 0) return;
    int words = (n_views_cap + 31) / 32;
    if (!owners)
        k_chunk_owners<<<grid_for(g.n, 256, 16384), 256, 0, s>>>(cnt, rec_off, g.n, R_dev, rec_cap, chunk_g);
    k_project_emit<<<grid_for(rec_cap, PE_THREADS, 32768), PE_THREADS, 0, s>>>(
        g, views, words, st, ilog2(tw), ilog2(th), mask, rec_off, R_dev, rec_cap, rec, sortkey,
        write_attr ? 1 : 0, chunk_g, flags);
}

int scan_blocks(uint64_t cap) {
    uint64_t b = (cap + SC_TILE - 1) / SC_TILE;
    if (b < 1) b = 1;
    if (b > SC_MAX_BLOCKS) b = SC_MAX_BLOCKS;
    return (int)b;
}

// One launch up to SCAN_ONE items (a block reads 16 k of them twice in 9 us; the two launches take 10).
constexpr uint32_t SCAN_ONE = 8 * SC_TILE;

void scan_u32(const uint32_t* in, uint32_t* out, const uint32_t* n_dev, uint32_t cap, uint32_t* total, uint32_t* flags,
              ScanWs ws, hipStream_t s, uint32_t* mirror, uint32_t* chunk_g, uint32_t rec_cap) {
    const ScanOut o{total, flags, mirror, chunk_g, rec_cap};
    if (cap <= SCAN_ONE) {
        k_scan_down<<<1, SC_THREADS, 0, s>>>(in, out, n_dev, cap, nullptr, o);
        return;
    }
    int nb = scan_blocks(cap);
    k_scan_reduce<<<nb, SC_THREADS, 0, s>>>(in, n_dev, cap, ws.partial);
    k_scan_down<<<nb, SC_THREADS, 0, s>>>(in, out, n_dev, cap, ws.partial, o);
}

// The form of a pass over at most cap items: items per lane, threads and blocks (one per tile, up to RS_MAX_BLOCKS).
struct RsForm {
    int ipt, threads, blocks;
};

static RsForm sort_form(uint64_t cap) {
    const uint64_t small = (uint64_t)RS_MAX_BLOCKS * RS_THREADS;
    RsForm f;
    f.ipt = cap <= 4 * small ? 4 : cap <= 8 * small ? 8 : RS_IPT;
    f.threads = cap >= RS_BIG_ITEMS ? RS_THREADS_BIG : RS_THREADS;
    const uint64_t tile = (uint64_t)f.ipt * f.threads;
    f.blocks = (int)std::min<uint64_t>(std::max<uint64_t>((cap + tile - 1) / tile, 1), RS_MAX_BLOCKS);
    return f;
}

// Histograms (a table per block) and the digits' totals, for every input of up to cap items: the smallest tile
// bounds the blocks of any.
size_t sort_hist_words(uint64_t cap) {
    const uint64_t tile = 4 * RS_THREADS;
    return ((size_t)1 << RS_DB) * (size_t)(std::min<uint64_t>((cap + tile - 1) / tile + 1, RS_MAX_BLOCKS) + 1);
}

template <int NT, int IPT>
static void rs_pass(uint32_t* ki, const uint32_t* vi, uint32_t* ko, uint32_t* vo, const uint32_t* n_dev, uint32_t cap,
                    int shift, int bits, int nb, SortWs ws, RsCounts rc, uint32_t* gout, hipStream_t s) {
    const bool fused = NT == RS_THREADS && nb <= RS_FUSED_BLOCKS;
    k_rs_upsweep<NT, IPT><<<nb, NT, 0, s>>>(ki, n_dev, cap, shift, bits, ws.hist, fused);
    uint32_t* totals = nullptr;
    if (!fused) {
        totals = ws.hist + ((size_t)nb << RS_DB);
        k_rs_columns<<<1 << RS_DB, 256, 0, s>>>(ws.hist, nb, totals);
    }
    k_rs_scatter<NT, IPT><<<nb, NT, 0, s>>>(ki, vi, ko, vo, n_dev, cap, shift, bits, ws.hist, totals, rc, gout);
}

// The nbits are split into the fewest passes of at most RS_DB bits, as evenly as possible.  Two 9-bit passes in place
// of three over 192 M pairs took 1,220 us each (the 8-bit ones 700 to 930): twice the buckets, half the runs.
int radix_sort(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, const uint32_t* n_dev, uint32_t cap,
               int nbits, SortWs ws, hipStream_t s, const uint32_t* count, uint32_t* gout) {
    if (cap <= RS_ONE) {
        // the passes of 2 k items in one launch of 16 us; 8 launches took 31 and the gaps between them
        k_rs_one<<<1, RS_ONE_THREADS, 0, s>>>(k0, v0, k1, v1, n_dev, cap, nbits, count, gout);
        return 1;
    }
    const RsForm f = sort_form(cap);
    const int passes = std::max(1, (nbits + RS_DB - 1) / RS_DB);
    RsCounts rc{count, 32};
    if (count) {
        int pb = 1;
        while (((uint64_t)1 << pb) < cap) pb++;
        if (pb <= 29) rc.pb = pb;  // at least three bits for the counts
    }
    uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
    int shift = 0;
    for (int p = 0; p < passes; p++) {
        // with count k0 stays as it is (the same frame may be sorted again): the keys go by k1 and, until the last
        // pass fills it, gout, and the last pass reads them from k1 and leaves them out
        if (count) ko = p + 1 == passes ? nullptr : (passes - p) % 2 == 0 ? k1 : gout;
        const int bits = std::max(nbits / passes + (p < nbits % passes ? 1 : 0), 1);
        const uint32_t* vin = count && p == 0 ? nullptr : vi;
        uint32_t* go = p + 1 == passes ? gout : nullptr;
        auto pass = [&](auto nt, auto ipt) {
            rs_pass<decltype(nt)::value, decltype(ipt)::value>(ki, vin, ko, vo, n_dev, cap, shift, bits, f.blocks, ws, rc,
                                                               go, s);
        };
        using std::integral_constant;
        using Small = integral_constant<int, RS_THREADS>;
        using Big = integral_constant<int, RS_THREADS_BIG>;
        if (f.threads == RS_THREADS_BIG) pass(Big{}, integral_constant<int, RS_IPT>{});
        else if (f.ipt == 4) pass(Small{}, integral_constant<int, 4>{});
        else if (f.ipt == 8) pass(Small{}, integral_constant<int, 8>{});
        else pass(Small{}, integral_constant<int, RS_IPT>{});
        shift += bits;
        uint32_t* t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
    }
    return passes & 1;
}

void emit_instances(const uint32_t* order, const uint32_t* R_dev, uint32_t rec_cap, const uint32_t* K_dev,
                    Records rec, const ViewDev* views, const uint32_t* inst_off, int tw, int th, SetDev st,
                    uint32_t inst_cap, uint32_t* tile_key, uint32_t* inst_rec, uint2* ranges, uint32_t tiles_cap,
                    uint32_t* flags, hipStream_t s) {
    const unsigned grid = grid_for(std::max<uint32_t>(inst_cap, 1), EM_WAVES * EM_RUN, EM_BLOCKS);
    k_emit_instances<<<grid, EM_THREADS, 0, s>>>(order, R_dev, rec_cap, K_dev, rec, views, inst_off, ilog2(tw),
                                                 ilog2(th), st.log2_amin, inst_cap, tile_key, inst_rec, ranges,
                                                 tiles_cap, flags);
}

void tile_ranges(const uint32_t* tile_key, const uint32_t* K_dev, uint32_t inst_cap, uint2* ranges,
                 uint32_t tiles_cap, const uint32_t* flags, hipStream_t s) {
    k_tile_ranges<<<grid_for((inst_cap + 3) / 4, 256, 16384), 256, 0, s>>>(tile_key, K_dev, inst_cap, ranges,
                                                                           tiles_cap, flags);
}

void tile_order(const uint2* ranges, const Header* hdr, uint32_t tiles_cap, uint32_t* ws, uint32_t* order,
                hipStream_t s) {
    if (tiles_cap == 0) return;
    if (tiles_cap <= TO_ONE) {
        // one launch of 5 us instead of three
        k_tile_order_one<<<1, 1024, 0, s>>>(ranges, hdr, tiles_cap, order);
        return;
    }
    fill_u32(ws, 0u, 2 * TO_BUCKETS, s);
    const unsigned grid = grid_for(tiles_cap, 256, 1024);
    k_tile_order_count<<<grid, 256, 0, s>>>(ranges, hdr, tiles_cap, ws);
    k_tile_order_place<<<grid, 256, 0, s>>>(ranges, hdr, tiles_cap, ws, ws + TO_BUCKETS, order);
}

void render_forward(int tw, int th, int batch, const ViewDev* views, int n_views,
                    uint32_t tiles_total, const uint2* ranges, const uint32_t* tile_order, const uint32_t* inst_rec,
                    Records rec, SetDev st, RenderOut out, const uint32_t* flags, hipStream_t s) {
    if (tiles_total == 0) return;
    auto launch = [&](auto kernel) {
        kernel<<<tiles_total, tw * th, 0, s>>>(views, n_views, ranges, tile_order, inst_rec, rec, st, out, flags);
    };
    if (!out.contrib) {  // captured iterations, which composite no uncertainty
        RTG_BATCH_DISPATCH(TW, TH, B, (launch(k_render_fwd<TW, TH, B, false, false>)));
    } else if (out.unc) {
        RTG_BATCH_DISPATCH(TW, TH, B, (launch(k_render_fwd<TW, TH, B, true, true>)));
    } else {
        RTG_BATCH_DISPATCH(TW, TH, B, (launch(k_render_fwd<TW, TH, B, false, true>)));
    }
}

void loss_l1(const ViewDev* views, int n_views, int max_pix, const float* rgb, const float* depth,
             const float* trgb, const float* tdepth, float w_depth, float* d_rgb, float* d_depth, double* partial,
             int partial_cap, double* loss, hipStream_t s) {
    unsigned bx = grid_for((uint64_t)max_pix, 256, 1u << 30);
    (void)partial_cap;
    dim3 grid(bx, n_views);
    k_loss<<<grid, 256, 0, s>>>(views, rgb, depth, trgb, tdepth, w_depth, d_rgb, d_depth, partial);
    k_sum_partials<<<1, SP_THREADS, 0, s>>>(partial, (int)(bx * n_views), loss);
}

// Bands per tile for the backward: frames of few tiles leave most SIMDs with a wave or none, and then
// more, shorter walks win until their atomics (one set per band and splat) cost more.  Isotropic maps, in us
// (with alpha gradients), for one, two and four bands on 256 CUs:
//     336 tiles   266 (323)   146 (189)    98 (132)
//     690         139 (168)    97 (124)    81 (100)
//     980         126 (150)    95 (112)    95 (108)
//   1,200         122 (141)    97 (115)   106 (131)
//   2,400         159 (186)   124 (140)   181 (188)
//   7,200         217 (250)   342 (355)   604 (642)
// so four below 3.5 tiles per CU, two below 16, one from there on.  Maps of needle-shaped splats never take four: the
// sums of a splat over a tile cancel, and are added up over two bands as they always were.  RTG_BWD_WAVES overrides.
static int backward_bands(int tw, int th, uint32_t tiles, bool isotropic) {
    static int forced = -1;
    if (forced < 0) {
        const char* e = getenv("RTG_BWD_WAVES");
        forced = e ? atoi(e) : 0;
    }
    const int nb8 = tw * th / 64;
    int nw = 1;
    if (forced == 1 || forced == 2 || forced == 4) nw = forced;
    else {
        const uint32_t cu = (uint32_t)std::max(device_cu_count(), 1);
        nw = isotropic && 2 * (uint64_t)tiles < 7 * cu ? 4 : tiles < 16 * cu ? 2 : 1;
    }
    while (nw > nb8) nw >>= 1;
    return nw;
}

void render_backward(int tw, int th, int batch, const ViewDev* views, int n_views, uint32_t tiles_total,
                     const uint2* ranges, const uint32_t* tile_order, const uint32_t* inst_rec, Records rec,
                     SetDev st, const float* T_final,
                     const uint32_t* n_last, const float* d_rgb, const float* d_depth, const float* d_alpha,
                     const float* d_unc, double* g2d, const uint32_t* flags, hipStream_t s) {
    (void)batch;  // the backward stages 64 splats per wave
    if (tiles_total == 0) return;
    const int nw = backward_bands(tw, th, tiles_total, st.isotropic != 0);
    const bool au = d_alpha != nullptr || d_unc != nullptr;
    auto launch = [&](auto kernel) {
        kernel<<<tiles_total * (unsigned)nw, 64, 0, s>>>(views, n_views, ranges, tile_order, inst_rec, rec, st,
                                                         T_final, n_last, d_rgb, d_depth, d_alpha, d_unc, g2d, flags);
    };
    auto bands = [&](auto w, auto h) {
        constexpr int TW = decltype(w)::value, TH = decltype(h)::value;
        if constexpr (TW * TH > 64) {
            if (nw == 4) return au ? launch(k_render_bwd<TW, TH, 4, true>) : launch(k_render_bwd<TW, TH, 4, false>);
            if (nw == 2) return au ? launch(k_render_bwd<TW, TH, 2, true>) : launch(k_render_bwd<TW, TH, 2, false>);
        }
        return au ? launch(k_render_bwd<TW, TH, 1, true>) : launch(k_render_bwd<TW, TH, 1, false>);
    };
    using std::integral_constant;
    if (tw == 8 && th == 8) bands(integral_constant<int, 8>{}, integral_constant<int, 8>{});
    else if (tw == 32 && th == 8) bands(integral_constant<int, 32>{}, integral_constant<int, 8>{});
    else bands(integral_constant<int, 16>{}, integral_constant<int, 16>{});
}

void project_backward(const GaussDev& g, const ViewDev* views, SetDev st, const uint32_t* rec_off,
                      const uint32_t* cnt, const EmitRec* emit, const double* g2d, float* d_means,
                      float* d_log_scales, float* d_quats, float* d_opacity, float* d_colors, const uint32_t* flags,
                      hipStream_t s, uint32_t* flag_host) {
    if (g.n == 0) return;
    k_project_bwd<<<grid_for(g.n, 256, 0xffffffffu), 256, 0, s>>>(g, views, st, rec_off, cnt, emit, g2d, d_means,
                                                     d_log_scales, d_quats, d_opacity, d_colors, flags, flag_host);
}

void score_tiles(int tw, int th, int batch, int mode, bool persistent, int grid_persistent, const ViewDev* views,
                 int n_views, const Header* hdr, uint32_t tile_begin, uint32_t n_tiles,
                 const uint2* ranges, const uint32_t* tile_order, const uint32_t* inst_rec, Records rec, SetDev st,
                 double* partial, uint32_t* queue, const uint32_t* flags, hipStream_t s) {
    if (persistent) {
        fill_u32(queue, 0u, 1, s);
        RTG_BATCH_DISPATCH(TW, TH, B,
                           (k_score_persistent<TW, TH, B><<<grid_persistent, TW * TH, 0, s>>>(views, hdr, ranges,
                                                                                             tile_order, inst_rec,
                                                                                             rec, st,
                                                                                             mode, partial, queue,
                                                                                             flags)));
    } else {
        if (n_tiles == 0) return;
        RTG_BATCH_DISPATCH(TW, TH, B,
                           (k_score_plain<TW, TH, B><<<n_tiles, TW * TH, 0, s>>>(views, n_views, tile_begin,
                                                                                ranges, inst_rec, rec, st, mode,
                                                                                partial)));
    }
}

void score_reduce(const ViewDev* views, const Header* hdr, int n_views_cap, const double* partial,
                  double* scores, const uint32_t* flags, hipStream_t s, uint32_t* flag_host) {
    k_score_reduce<<<n_views_cap, 256, 0, s>>>(views, hdr, partial, scores, flags, flag_host);
}

void sum_counts(const uint64_t* a, uint64_t na, const uint32_t* b, uint64_t nb, unsigned long long* out, hipStream_t s) {
    const uint64_t n = std::max(na, nb);
    if (n == 0) return;
    k_sum_counts<<<grid_for(n, 256, 2048), 256, 0, s>>>(a, na, b, nb, out);
}

void uncertainty_update(int64_t n, const float* prev, const float* cur, const float* u_prev, int squared,
                        float* u_out, hipStream_t s) {
    if (n <= 0) return;
    k_uncertainty_update<<<grid_for((uint64_t)n, 256, 1u << 20), 256, 0, s>>>(n, prev, cur, u_prev, squared, u_out);
}

void region_utility(int64_t n, const float* means, const float* u, const double* lo, double size, const int* dims,
                    unsigned long long* cnt, int64_t* count, double* sum, double* mean, hipStream_t s) {
    const int64_t nr = (int64_t)dims[0] * dims[1] * dims[2];
    unsigned long long* fix = cnt + nr;
    unsigned int* bad = reinterpret_cast<unsigned int*>(fix + nr);
    fill_u32(reinterpret_cast<uint32_t*>(cnt), 0u, 5 * (uint64_t)nr, s);
    if (n > 0) {
        const unsigned grid = grid_for((uint64_t)n, RG_THREADS * RG_BATCH, RG_BLOCKS);
        k_region_utility<<<grid, RG_THREADS, 0, s>>>(n, means, u, lo[0], lo[1], lo[2], size, dims[0], dims[1], dims[2], cnt,
                                                     fix, bad);
    }
    k_region_finish<<<grid_for((uint64_t)nr, 256, 4096), 256, 0, s>>>(nr, cnt, fix, bad, count, sum, mean);
}

void export_pairs(const uint32_t* tile_key, const uint32_t* inst_rec, const uint32_t* K_dev, Records rec,
                  uint64_t* keys, uint32_t* vals, uint32_t cap, hipStream_t s) {
    k_export<<<grid_for(cap, 256, 8192), 256, 0, s>>>(tile_key, inst_rec, K_dev, cap, rec, keys, vals);
}

void export_records(const uint32_t* R_dev, uint32_t cap, Records rec, double* mean2d, double* conic, int32_t* pbox,
                    uint32_t* depth_bits, uint32_t* gid, uint32_t* view, uint32_t* ntiles, hipStream_t s) {
    k_export_records<<<grid_for(std::max<uint32_t>(cap, 1), 256, 8192), 256, 0, s>>>(
        R_dev, cap, rec, mean2d, conic, pbox, depth_bits, gid, view, ntiles);
}

}  // namespace rtg
