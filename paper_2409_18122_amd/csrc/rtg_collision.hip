// gfx950 (CDNA4) collision check of RT-GuIDE's trajectory planner (arXiv
// 2409.18122, Sec. IV-B, trajectory planner, Collision Checking paragraph):
// points sampled on motion primitives against every Gaussian of the map, each taken as a sphere of lambda_g times its principal
// axis.  Compiled without floating-point contraction, like the rasterizer.
#include "rtg_internal.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

namespace rtg {

namespace {

// Sec. IV-B (trajectory planner, Collision Checking): a sampled point (a
// sphere of radius r_robot) collides with a Gaussian whose mean is closer than r_robot + lambda_g r, r = the Gaussian's
// principal axis exp(max log-scale); the clearance is min_i (||p - mu_i|| - w_i), w_i = lambda_g r_i.
//
// Two things bound the check: reading the map once, and the pair tests.  Testing every pair of a
// 3M-Gaussian map with 8,256 points is 2.5e10 pairs (7.5 ms at the FP32 vector rate), but a
// Gaussian can matter to a point only if it lies within the point's clearance.  So:
//   k_cc_points puts the points of a batch in spatial order and covers every 64 of them (one per
//     lane) with a ball (c, R);
//   k_cc_bound gives every point an upper bound of its clearance from a strided sample of the map, above the
//     exact clearance of the pair that sets it by more than every rounding;
//   k_cc_check streams the map once per slab of points: a lane takes a Gaussian and tests it against the
//     balls; one that is nearer to c than R + w + the largest bound of the group's points is tested
//     against the group's 64 points, a point per lane.
// What is left out is further from all 64 points than the bounds, so it sets no minimum; and no flag that the
// pair of the bound does not set too, since that pair's exact clearance is the smaller one and it is always
// tested itself.  So the results do not depend on the grouping.  (A binary32 clearance would not do as
// the bound: that of an axis of 100 m is off by 1e-5 m, and its pair may miss a point that it seems to hold.)
// Points far apart or in no order cost more tests, at worst all pairs (check_dense).
// Flags are decided in binary32 outside a relative CC_BAND of the bound (r_robot + w)^2, which is formed in binary64
// and rounded once, and inside it in binary64 (from the original parameters, in the oracle's order).  A clearance is a minimum of
// binary32 values (the hardware square root, within an ulp), the same in every order.

constexpr double CC_BAND = 4e-6;  // relative band re-taken in binary64 (d^2 error < 4e-7)
constexpr float CC_INF = __builtin_inff();

// Points of a batch (one block of k_cc_points) and their spatial order: 2^CP_BITS bins, the box
// halved along its longest side each time, so that bins stay near cubes for points on a
// plane or a line too.
constexpr int CP_THREADS = 1024;
constexpr int CP_IPT = 4;
constexpr int CP_BATCH = CP_THREADS * CP_IPT;
constexpr int CP_BITS = 12;
constexpr int CP_BINS = 1 << CP_BITS;
constexpr int CP_BPT = CP_BINS / CP_THREADS;

// k_cc_check: a block holds a slab of up to CK_GROUPS groups of 64 points in LDS and takes
// CK_THREADS Gaussians a step.
constexpr int CK_THREADS = 768;
constexpr int CK_GROUPS = 44;
constexpr int CK_UNROLL = 4;  // balls tested per branch

// Sorted points of one call, planar; index: the point's place in the caller's arrays.  Places past a
// batch's finite points hold NaN coordinates, which no comparison passes.
struct CcPoints {
    float *x, *y, *z;
    float* ub;  // bound of the clearance (k_cc_bound)
    uint32_t* index;
    float4 *ball, *sub;  // per 64 and per 8 points: centre, radius (NaN centre: no finite point)
};

// Minimum of *p and v (v never -0: then +0 would not order below negative bits).  Binary32
// values order as their bits do, negative ones in reverse.
__device__ __forceinline__ void atomic_min_float(float* p, float v) {
    if (v >= 0.0f) atomicMin(reinterpret_cast<int*>(p), __float_as_int(v));
    else atomicMax(reinterpret_cast<unsigned*>(p), __float_as_uint(v));
}

// The next number above x (x never -0; infinity stays).
__device__ __forceinline__ float next_up(float x) {
    const int b = __float_as_int(x);
    return x < CC_INF ? __int_as_float(b < 0 ? b - 1 : b + 1) : x;
}

__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// w = lambda_g r of one Gaussian, from its mean and log-scales.
__device__ __forceinline__ double cc_axis(const float (&v)[6], float lambda_g) {
    return (double)lambda_g * exp((double)fmaxf(fmaxf(v[3], v[4]), v[5]));
}

// Its mean and w, rounded once; an ignored one (a non-finite mean or log-scale) gets a NaN mean, which no
// comparison passes.
__device__ __forceinline__ float4 cc_gauss(const float (&v)[6], double w) {
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 6; k++) ok = ok && isfinite(v[k]);
    return make_float4(ok ? v[0] : __builtin_nanf(""), v[1], v[2], (float)w);
}

// The squared bound of its collisions, a band below and above.
__device__ __forceinline__ float2 cc_band(double w, float r_robot) {
    const double gm = (double)r_robot + w, g2 = gm * gm;
    return make_float2((float)(g2 * (1.0 - CC_BAND)), (float)(g2 * (1.0 + CC_BAND)));
}

// Block b orders the points [b per, (b + 1) per) of the caller's planar arrays (stride np_all) and
// clears their results.  One block per batch: a counting sort over the bins in LDS; the order within a
// bin is arbitrary, and nothing depends on it.
__global__ __launch_bounds__(CP_THREADS) void k_cc_points(const float* __restrict__ pts, int64_t np_all, int np,
                                                          int per, CcPoints P, int32_t* __restrict__ collide,
                                                          float* __restrict__ clearance) {
    __shared__ uint32_t hist[CP_BINS];
    __shared__ float s_lo[3][CP_THREADS / 64], s_hi[3][CP_THREADS / 64];
    __shared__ uint32_t s_w[CP_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int begin = blockIdx.x * per, end = min(begin + per, np);
    for (int i = tid; i < CP_BINS; i += CP_THREADS) hist[i] = 0;
    float x[CP_IPT][3];
    uint32_t live = 0;
    float lo[3] = {CC_INF, CC_INF, CC_INF}, hi[3] = {-CC_INF, -CC_INF, -CC_INF};
#pragma unroll
    for (int k = 0; k < CP_IPT; k++) {
        const int i = begin + tid + k * CP_THREADS;
#pragma unroll
        for (int a = 0; a < 3; a++) x[k][a] = i < end ? pts[a * np_all + i] : 0.0f;
        if (i >= end) continue;
        collide[i] = 0;
        if (clearance) clearance[i] = CC_INF;
        if (!(isfinite(x[k][0]) && isfinite(x[k][1]) && isfinite(x[k][2]))) continue;
        live |= 1u << k;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fminf(lo[a], x[k][a]);
            hi[a] = fmaxf(hi[a], x[k][a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
        if (lane == 0) {
            s_lo[a][wv] = lo[a];
            s_hi[a][wv] = hi[a];
        }
    }
    __syncthreads();
    float size[3], scale[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        for (int w = 0; w < CP_THREADS / 64; w++) {
            lo[a] = fminf(lo[a], s_lo[a][w]);
            hi[a] = fmaxf(hi[a], s_hi[a][w]);
        }
        // an extent of 0 or beyond binary32 is not split
        size[a] = hi[a] - lo[a];
        if (!(size[a] > 0.0f && size[a] < 1e38f)) size[a] = 0.0f;
        scale[a] = size[a] > 0.0f ? 1.0f / size[a] : 0.0f;
    }
    // the halvings, first to last: axis of split s in bits 2 s of `axes`; levels per axis
    uint32_t axes = 0;
    int lev[3] = {0, 0, 0};
#pragma unroll
    for (int s = 0; s < CP_BITS; s++) {
        const int a = size[0] >= size[1] ? (size[0] >= size[2] ? 0 : 2) : (size[1] >= size[2] ? 1 : 2);
        axes |= (uint32_t)a << (2 * s);
#pragma unroll
        for (int b = 0; b < 3; b++)
            if (b == a) {
                size[b] *= 0.5f;
                lev[b]++;
            }
    }
    uint32_t bin[CP_IPT], rank[CP_IPT];
#pragma unroll
    for (int k = 0; k < CP_IPT; k++) {
        bin[k] = rank[k] = 0;
        if (!((live >> k) & 1u)) continue;
        uint32_t q[3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const float cells = (float)(1u << lev[a]);
            // cell within the axis, its bits left-aligned so that each split takes the next one
            const uint32_t c = (uint32_t)fminf((x[k][a] - lo[a]) * scale[a] * cells, cells - 1.0f);
            q[a] = c << (CP_BITS - lev[a]);
        }
        uint32_t code = 0;
#pragma unroll
        for (int s = 0; s < CP_BITS; s++) {
            const uint32_t a = (axes >> (2 * s)) & 3u;
            const uint32_t qa = a == 0 ? q[0] : a == 1 ? q[1] : q[2];
            code = 2 * code + ((qa >> (CP_BITS - 1)) & 1u);
            q[0] = a == 0 ? q[0] << 1 : q[0];
            q[1] = a == 1 ? q[1] << 1 : q[1];
            q[2] = a == 2 ? q[2] << 1 : q[2];
        }
        bin[k] = code;
        rank[k] = atomicAdd(&hist[code], 1u);
    }
    __syncthreads();
    // exclusive scan of the bins, CP_BPT consecutive ones per thread
    uint32_t c[CP_BPT], mine = 0;
#pragma unroll
    for (int j = 0; j < CP_BPT; j++) {
        c[j] = hist[tid * CP_BPT + j];
        mine += c[j];
    }
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) s_w[wv] = inc;
    __syncthreads();
    uint32_t run = inc - mine, total = 0;
    for (int w = 0; w < CP_THREADS / 64; w++) {
        if (w < wv) run += s_w[w];
        total += s_w[w];
    }
#pragma unroll
    for (int j = 0; j < CP_BPT; j++) {
        hist[tid * CP_BPT + j] = run;
        run += c[j];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CP_IPT; k++) {
        if (!((live >> k) & 1u)) continue;
        const uint32_t at = (uint32_t)begin + hist[bin[k]] + rank[k];
        P.x[at] = x[k][0];
        P.y[at] = x[k][1];
        P.z[at] = x[k][2];
        P.index[at] = (uint32_t)(begin + tid + k * CP_THREADS);
    }
    const float nan = __builtin_nanf("");
    if (clearance)
        for (int i = tid; i < per; i += CP_THREADS) P.ub[begin + i] = CC_INF;
    for (uint32_t i = total + tid; i < (uint32_t)per; i += CP_THREADS) {
        P.x[begin + i] = nan;
        P.y[begin + i] = nan;
        P.z[begin + i] = nan;
        P.index[begin + i] = 0;
    }
    __syncthreads();  // the block's own stores are read below
    for (int gr = wv; gr < per / 64; gr += CP_THREADS / 64) {
        const int at = begin + gr * 64 + lane;
        const bool in = (uint32_t)(gr * 64 + lane) < total;
        const float p0 = P.x[at], p1 = P.y[at], p2 = P.z[at];
        float mn[3] = {in ? p0 : CC_INF, in ? p1 : CC_INF, in ? p2 : CC_INF};
        float mx[3] = {in ? p0 : -CC_INF, in ? p1 : -CC_INF, in ? p2 : -CC_INF};
        // the ball over the 2^level lanes around this one (no points: inf - inf gives NaN)
        auto ball = [&](int from, int to) {
            for (int o = from; o < to; o <<= 1)
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    mn[a] = fminf(mn[a], __shfl_xor(mn[a], o, 64));
                    mx[a] = fmaxf(mx[a], __shfl_xor(mx[a], o, 64));
                }
            float4 c = make_float4(0.5f * mn[0] + 0.5f * mx[0], 0.5f * mn[1] + 0.5f * mx[1],
                                   0.5f * mn[2] + 0.5f * mx[2], 0.0f);
            const float dx = p0 - c.x, dy = p1 - c.y, dz = p2 - c.z;
            c.w = in ? sqrtf(dx * dx + dy * dy + dz * dz) : 0.0f;
            for (int o = 1; o < to; o <<= 1) c.w = fmaxf(c.w, __shfl_xor(c.w, o, 64));
            return c;
        };
        const float4 b8 = ball(1, 8), b64 = ball(8, 64);
        if ((lane & 7) == 0) P.sub[at / 8] = b8;
        if (lane == 0) P.ball[at / 64] = b64;
    }
}

// Upper bounds of the clearances: 256 PPL ordered points of a block against `per` Gaussians of the
// sample (sample s is Gaussian s n / m), staged 256 at a time.  Each LDS read of a Gaussian serves PPL
// tests; below 65,536 points one test each, which gives four times as many waves (8,256 points and
// 4,096 Gaussians: 18 us, against 22 us with PPL = 4).
// The bound is d (1 + 1e-6) - w (1 - 1e-6): d is off by a relative 3.6e-7 at most (its differences, sum and root), w and the
// result by 6e-8.  An axis beyond binary32 counts as 3e38, so the bound is finite wherever d is.
template <int PPL>
__global__ __launch_bounds__(256) void k_cc_bound(GaussDev g, int m, int per, float lambda_g, CcPoints P, int npad) {
    __shared__ float4 s_c[256];
    const float nan = __builtin_nanf("");
    float px[PPL], py[PPL], pz[PPL], best[PPL];
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        const int j = (blockIdx.x * PPL + k) * 256 + threadIdx.x;
        px[k] = j < npad ? P.x[j] : nan;
        py[k] = j < npad ? P.y[j] : nan;
        pz[k] = j < npad ? P.z[j] : nan;
        best[k] = CC_INF;
    }
    const int s0 = blockIdx.y * per, s1 = min(s0 + per, m);
    for (int s = s0; s < s1; s += 256) {
        __syncthreads();
        float4 c = make_float4(nan, nan, nan, 0.0f);
        if (s + (int)threadIdx.x < s1) {
            const int64_t i = (int64_t)(s + threadIdx.x) * g.n / m;
            const float v[6] = {g.means[i],      g.means[g.n + i],      g.means[2 * g.n + i],
                                g.log_scales[i], g.log_scales[g.n + i], g.log_scales[2 * g.n + i]};
            c = cc_gauss(v, cc_axis(v, lambda_g));
            if (c.w == CC_INF) c.w = 3e38f;
            c.w *= 0.999999f;
        }
        s_c[threadIdx.x] = c;
        __syncthreads();
#pragma unroll 8
        for (int t = 0; t < 256; t++) {
            const float4 q = s_c[t];
#pragma unroll
            for (int k = 0; k < PPL; k++) {
                const float dx = px[k] - q.x, dy = py[k] - q.y, dz = pz[k] - q.z;
                const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                best[k] = fminf(best[k], fmaf(__builtin_amdgcn_sqrtf(d2), 1.000001f, -q.w));
            }
        }
    }
#pragma unroll
    for (int k = 0; k < PPL; k++) {  // a place past the points has found nothing
        const int j = (blockIdx.x * PPL + k) * 256 + threadIdx.x;
        if (best[k] < CC_INF) atomic_min_float(&P.ub[j], best[k]);
    }
}

// binary64 test of point (px, py, pz) against Gaussian i, as the oracle takes it
__device__ __forceinline__ bool collide64(const GaussDev& g, int64_t i, float px, float py, float pz, float r_robot,
                                       float lambda_g) {
    const double l0 = g.log_scales[i], l1 = g.log_scales[g.n + i], l2 = g.log_scales[2 * g.n + i];
    double lm = l0 > l1 ? l0 : l1;
    lm = lm > l2 ? lm : l2;
    const double r = exp(lm);
    const double dx = (double)px - (double)g.means[i];
    const double dy = (double)py - (double)g.means[g.n + i];
    const double dz = (double)pz - (double)g.means[2 * g.n + i];
    const double d2 = (dx * dx + dy * dy) + dz * dz;
    const double gm = (double)r_robot + (double)lambda_g * r;
    return d2 < gm * gm;
}

// A tile of Gaussians in LDS: mean and w, and the band of the squared bound.
struct CcTile {
    float4* c;
    float *lo, *hi;
};

// Gaussian i (past the last one: an ignored one) as the tile's entry at.
__device__ __forceinline__ void stage_gauss(const GaussDev& g, int64_t i, float r_robot, float lambda_g, const CcTile& s,
                                            int at) {
    float4 c = make_float4(__builtin_nanf(""), 0.0f, 0.0f, 0.0f);
    float2 b = make_float2(0.0f, 0.0f);
    if (i < g.n) {
        const float v[6] = {g.means[i],      g.means[g.n + i],      g.means[2 * g.n + i],
                            g.log_scales[i], g.log_scales[g.n + i], g.log_scales[2 * g.n + i]};
        const double w = cc_axis(v, lambda_g);
        c = cc_gauss(v, w);
        b = cc_band(w, r_robot);
    }
    s.c[at] = c;
    s.lo[at] = b.x;
    s.hi[at] = b.y;
}

// PPL points per lane against the tile's entries [u0, u1) in whole steps of CC_STEP (entry 0 is Gaussian `first`); hit: a
// lane mask per point.  No branch but the one for the rare step that holds a hit or a binary64 decision: a clearance
// costs 13 cycles (root, difference, half a minimum of three), a test whether it is lower 11 and a branch that is
// taken often.  31 cycles a pair of 64 points.
constexpr int CC_STEP = 4;

template <bool CLR, int PPL>
__device__ __forceinline__ void walk_pairs(const GaussDev& g, int64_t first, float r_robot, float lambda_g, const CcTile& s,
                                           int u0, int u1, const float (&px)[PPL], const float (&py)[PPL],
                                           const float (&pz)[PPL], float (&best)[PPL], uint64_t (&hit)[PPL]) {
    for (int u = u0; u < u1; u += CC_STEP) {
        float d2[PPL][CC_STEP];
        uint64_t near[PPL] = {}, rare = 0;
#pragma unroll
        for (int k = 0; k < CC_STEP; k++) {
            const float4 q = s.c[u + k];
            const float hi = s.hi[u + k];
#pragma unroll
            for (int p = 0; p < PPL; p++) {
                const float dx = px[p] - q.x, dy = py[p] - q.y, dz = pz[p] - q.z;
                d2[p][k] = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                near[p] |= __ballot(d2[p][k] <= hi);
                if (CLR) best[p] = fminf(best[p], __builtin_amdgcn_sqrtf(d2[p][k]) - q.w);
            }
        }
#pragma unroll
        for (int p = 0; p < PPL; p++) rare |= near[p] & ~hit[p];
        if (rare) {
#pragma unroll
            for (int p = 0; p < PPL; p++) {
                bool h = hit[p] >> (threadIdx.x & 63) & 1u;
#pragma unroll
                for (int k = 0; k < CC_STEP; k++)
                    if (!h && d2[p][k] <= s.hi[u + k])
                        h = d2[p][k] < s.lo[u + k] ||
                            collide64(g, first + u + k, px[p], py[p], pz[p], r_robot, lambda_g);
                hit[p] = __ballot(h);
            }
        }
    }
}

// Every point against every Gaussian, for maps too small for the grouping to pay (pairs_pay).  A block of 16 waves takes
// 64 PPL points for every SPLIT waves, PPL per lane, and shares out the Gaussians between these waves, 1,024 at a time in
// LDS; the shares' minima meet at the end, so one launch does it all.  Few points need the waves (SPLIT 16: a chain
// a sixteenth as long); for many, two per lane halve the reads of LDS.  Bound by issue.  Two blocks a CU at 64 VGPRs (the
// binary64 decision spills five of them; one block: 719 us for 2,000 Gaussians and 2^20 points instead of 634).
// 100 Gaussians and 100,000 points 23 us, where the groups took 118 to 450 and a loop over all pairs in four launches 31.
template <bool CLR, int SPLIT, int PPL>
__global__ __launch_bounds__(CP_THREADS, 8) void k_cc_pairs(GaussDev g, float r_robot, float lambda_g,
                                                         const float* __restrict__ pts, int64_t np,
                                                         int32_t* __restrict__ collide, float* __restrict__ clearance) {
    constexpr int WAVES = CP_THREADS / 64;
    __shared__ float4 s_c[CP_THREADS];
    __shared__ float s_hi[CP_THREADS], s_lo[CP_THREADS];
    const CcTile s{s_c, s_lo, s_hi};
    __shared__ float s_best[WAVES][PPL][64];
    __shared__ uint64_t s_hit[WAVES][PPL];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t j0 = ((int64_t)blockIdx.x * (WAVES / SPLIT) + wv / SPLIT) * (64 * PPL) + lane;
    const float nan = __builtin_nanf("");
    float px[PPL], py[PPL], pz[PPL], best[PPL];
    uint64_t hit[PPL];
#pragma unroll
    for (int p = 0; p < PPL; p++) {
        const int64_t j = j0 + 64 * p;
        px[p] = j < np ? pts[j] : nan;
        py[p] = j < np ? pts[np + j] : nan;
        pz[p] = j < np ? pts[2 * np + j] : nan;
        best[p] = CC_INF;
        hit[p] = 0;
    }
    for (int64_t t0 = 0; t0 < g.n; t0 += CP_THREADS) {
        __syncthreads();
        stage_gauss(g, t0 + tid, r_robot, lambda_g, s, tid);
        __syncthreads();
        // the wave's share, in whole steps (a step may reach into the next share or past the last Gaussian: no harm)
        const int cnt = (int)min<int64_t>(CP_THREADS, g.n - t0);
        const int per = (cnt + SPLIT * CC_STEP - 1) / (SPLIT * CC_STEP) * CC_STEP;
        const int u0 = wv % SPLIT * per;
        walk_pairs<CLR, PPL>(g, t0, r_robot, lambda_g, s, u0, min(u0 + per, cnt), px, py, pz, best, hit);
    }
    if constexpr (SPLIT > 1) {
#pragma unroll
        for (int p = 0; p < PPL; p++) {
            if (lane == 0) s_hit[wv][p] = hit[p];
            s_best[wv][p][lane] = best[p];
        }
        __syncthreads();
        if (wv % SPLIT) return;
#pragma unroll
        for (int w = 1; w < SPLIT; w++)
#pragma unroll
            for (int p = 0; p < PPL; p++) {
                hit[p] |= s_hit[wv + w][p];
                best[p] = fminf(best[p], s_best[wv + w][p][lane]);
            }
    }
#pragma unroll
    for (int p = 0; p < PPL; p++) {
        const int64_t j = j0 + 64 * p;
        if (j >= np) continue;
        collide[j] = (int32_t)(hit[p] >> lane & 1u);
        if (CLR) clearance[j] = best[p];
    }
}

// Orders a wave's LDS stores before its later LDS loads (its own lanes' queues below).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Whether a block's minimum for place `at` is worth an atomic: no Gaussian above the point's bound is its nearest, the one
// that set the bound is in some block, and most blocks hold none below it.
__device__ __forceinline__ bool lower(float v, const CcPoints& P, int at, float found) {
    return v < next_up(P.ub[at]) && v < found;
}

// All pairs of a block's Gaussians (every gridDim.x-th step) and its slab of ng groups from g0: a wave takes four
// groups, a point of each per lane, and where that leaves waves over they share the Gaussians.
template <bool CLR>
__device__ __forceinline__ void check_dense(const GaussDev& g, float r_robot, float lambda_g, const CcPoints& P, int g0,
                                            int ng, float4* lds, int32_t* collide, float* clearance) {
    constexpr int PPL = 4;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CcTile s{lds, reinterpret_cast<float*>(lds + CK_THREADS), reinterpret_cast<float*>(lds + CK_THREADS) + CK_THREADS};
    const int units = (ng + PPL - 1) / PPL, split = CK_THREADS / 64 / units, share = wv / units;
    const float nan = __builtin_nanf("");
    float px[PPL], py[PPL], pz[PPL], best[PPL];
    uint64_t hit[PPL];
#pragma unroll
    for (int p = 0; p < PPL; p++) {
        const int gr = wv % units * PPL + p, at = (g0 + gr) * 64 + lane;
        px[p] = gr < ng ? P.x[at] : nan;
        py[p] = gr < ng ? P.y[at] : nan;
        pz[p] = gr < ng ? P.z[at] : nan;
        best[p] = CC_INF;
        hit[p] = 0;
    }
    for (int64_t t0 = (int64_t)blockIdx.x * CK_THREADS; t0 < g.n; t0 += (int64_t)gridDim.x * CK_THREADS) {
        __syncthreads();
        stage_gauss(g, t0 + tid, r_robot, lambda_g, s, tid);
        __syncthreads();
        const int cnt = (int)min<int64_t>(CK_THREADS, g.n - t0);
        const int per = (cnt + split * CC_STEP - 1) / (split * CC_STEP) * CC_STEP;
        const int u0 = share * per;  // none for the waves past the shares
        if (share < split) walk_pairs<CLR, PPL>(g, t0, r_robot, lambda_g, s, u0, min(u0 + per, cnt), px, py, pz, best, hit);
    }
#pragma unroll
    for (int p = 0; p < PPL; p++) {
        if (!(px[p] == px[p])) continue;
        const uint32_t i = P.index[(g0 + wv % units * PPL + p) * 64 + lane];
        if (hit[p] >> lane & 1u) collide[i] = 1;  // every writer writes 1
        if (CLR && lower(best[p], P, (g0 + wv % units * PPL + p) * 64 + lane, clearance[i])) atomic_min_float(&clearance[i], best[p]);
    }
}

// grid: x over the Gaussians (a block takes every gridDim.x-th step), y over slabs of `gps` groups (CkGrid).
// CLR: the clearance is wanted; otherwise a group's reach is r_robot alone.
//
// A wave takes 64 Gaussians, one per lane, and tests them against the slab's balls of 64 points; a
// pair (Gaussian, ball) that passes goes into the wave's queue q1.  Of 64 such pairs at a time, a pair
// per lane, the eight balls of 8 points inside are tested into q2, and of 64 of these the
// 8 points.  Few Gaussians pass a ball (on a lot, one in 40), so without the queues
// nearly every lane of the later tests would be idle: testing all 64 points of a ball (a point
// per lane) for each passing Gaussian took 931 us for 8,256 points and 3M Gaussians, with the queues 445 to 476 us.
// Bound by instruction issue there (about 2.0e8 vector and 1.4e8 scalar wave instructions); for few points
// by the one pass over the map (129 points, 3M Gaussians: 33 us, 2.2 TB/s).
// Where points lie far from the map or from each other most pairs pass the balls, and 8 points of a queue's entry, read
// from as many places of LDS, cost 65 cycles a pair of 64 lanes, where a plain walk costs 31: a block whose first Gaussians pass
// more than half of the balls of 8 takes check_dense instead (8,256 points in a cube of 400 m: 12,400 -> 5,900 us, the
// former loop over all pairs 7,600).
// Slabs of 44 groups: 63 KB of LDS, two blocks of twelve waves a CU at 80 VGPRs (512 threads and 24
// groups, which read the map twice as often: 533 us).
template <bool CLR>
__global__ __launch_bounds__(CK_THREADS, 6) void k_cc_check(GaussDev g, float r_robot, float lambda_g, CcPoints P,
                                                         int ngroups, int gps, int32_t* __restrict__ collide,
                                                         float* clearance) {
    extern __shared__ float4 s_all[];
    const int ngp = (gps + CK_UNROLL - 1) / CK_UNROLL * CK_UNROLL;  // ck_lds_bytes
    float4* s_pt = s_all;             // x, y, z and the least clearance so far, at first above its bound
    float4* s_sub = s_pt + ngp * 64;  // balls of 8 points: centre and reach (radius + bound)
    float4* s_ball = s_sub + ngp * 8;  // of 64
    unsigned long long* s_hit = reinterpret_cast<unsigned long long*>(s_ball + ngp);
    __shared__ uint16_t s_q1[CK_THREADS / 64][64 * (CK_UNROLL + 1)], s_q2[CK_THREADS / 64][128];
    __shared__ uint32_t s_near;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) s_near = 0u;
    const int g0 = blockIdx.y * gps, ng = min(gps, ngroups - g0);
    const float nan = __builtin_nanf("");
    // a reach, widened by more than the rounding of the test (passes adds that of the Gaussian's own axis)
    auto reach_of = [](float r, float ub) { return (r + ub) + 1e-5f * (r + fabsf(ub)); };
    for (int gr = wv; gr < ngp; gr += CK_THREADS / 64) {
        float4 ball = make_float4(nan, nan, nan, 0.0f);
        if (gr < ng) {
            const int at = (g0 + gr) * 64 + lane;
            const float x = P.x[at], y = P.y[at], z = P.z[at];
            float b = r_robot;
            if (CLR) b = x == x ? P.ub[at] : -CC_INF;
            s_pt[gr * 64 + lane] = make_float4(x, y, z, CLR ? next_up(b) : b);
            float4 sub = P.sub[at / 8];
            ball = P.ball[at / 64];
            for (int o = 1; CLR && o < 8; o <<= 1) b = fmaxf(b, __shfl_xor(b, o, 64));
            sub.w = reach_of(sub.w, b);
            if ((lane & 7) == 0) s_sub[gr * 8 + (lane >> 3)] = sub;
            for (int o = 8; CLR && o < 64; o <<= 1) b = fmaxf(b, __shfl_xor(b, o, 64));
            ball.w = reach_of(ball.w, b);
        }
        if (lane == 0) {
            s_ball[gr] = ball;
            s_hit[gr] = 0ull;
        }
    }
    __syncthreads();
    uint16_t *q1 = s_q1[wv], *q2 = s_q2[wv];
    int n1 = 0, n2 = 0;
    auto passes = [&](float4 b, float4 q) {
        const float dx = q.x - b.x, dy = q.y - b.y, dz = q.z - b.z;
        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        // below 0 where a bound lies deeper inside another Gaussian than this one is wide: nothing passes
        const float reach = fmaf(q.w, 1.00001f, b.w);
        return d2 <= reach * fabsf(reach);
    };
    // appends the entries of the lanes in m
    auto push = [&](uint16_t* queue, int& n, bool pass, uint64_t m, uint32_t entry) {
        const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (pass) queue[n + (int)at] = (uint16_t)entry;
        n += (int)__popcll(m);
    };
    const int64_t stride = (int64_t)gridDim.x * CK_THREADS;
    float raw[6] = {nan, nan, nan, 0.0f, 0.0f, 0.0f};
    auto fetch = [&](int64_t i0) {
        const int64_t i = min(i0 + lane, g.n - 1);
#pragma unroll
        for (int k = 0; k < 3; k++) {
            raw[k] = g.means[k * g.n + i];
            raw[3 + k] = g.log_scales[k * g.n + i];
        }
    };
    int64_t base = (int64_t)blockIdx.x * CK_THREADS + wv * 64;
    if (base < g.n) fetch(base);
    // two pairs of a Gaussian of the first step and a ball of 8 points per lane tell whether the balls sort anything out
    // (1.5 us; up to 256 points the queues cost no more than the walk)
    if (ngroups > 4) {
        float4 q = cc_gauss(raw, cc_axis(raw, lambda_g));
        if (base + lane >= g.n) q.x = nan;
        uint32_t near = 0;
        for (int t = 0; t < 2; t++) near += (uint32_t)__popcll(__ballot(passes(s_sub[(lane + 64 * t) * ng / 16], q)));
        if (lane == 0) atomicAdd(&s_near, near);
        __syncthreads();
        const int64_t first = (int64_t)blockIdx.x * CK_THREADS;
        if (s_near > (uint32_t)min<int64_t>(CK_THREADS, g.n - first)) {
            check_dense<CLR>(g, r_robot, lambda_g, P, g0, ng, s_all, collide, clearance);
            return;
        }
    }
    for (; base < g.n; base += stride) {
        const double w = cc_axis(raw, lambda_g);
        float4 q = cc_gauss(raw, w);
        const float2 band = cc_band(w, r_robot);
        if (base + lane >= g.n) q.x = nan;
        if (base + stride < g.n) fetch(base + stride);  // in flight during this step
        for (int gr0 = 0; gr0 < ng; gr0 += CK_UNROLL) {
            bool pass[CK_UNROLL];
            uint64_t m[CK_UNROLL], some = 0;
#pragma unroll
            for (int k = 0; k < CK_UNROLL; k++) {
                pass[k] = passes(s_ball[gr0 + k], q);
                m[k] = __ballot(pass[k]);
                some |= m[k];
            }
            if (some) {
#pragma unroll
                for (int k = 0; k < CK_UNROLL; k++)
                    push(q1, n1, pass[k], m[k], (uint32_t)lane | (uint32_t)(gr0 + k) << 6);
            }
            // 64 entries at a time; the queues name this step's lanes, so they end with it
            const bool last = gr0 + CK_UNROLL >= ng;
            while (n1 >= 64 || (last && n1 + n2 > 0)) {
                wave_lds_fence();
                const int t1 = min(n1, 64);
                n1 -= t1;
                const uint32_t e1 = lane < t1 ? q1[n1 + lane] : 0u;  // (lane of the Gaussian, ball of 64)
                const int src1 = (int)(e1 & 63u);
                float4 u;
                u.x = __shfl(q.x, src1, 64);
                u.y = __shfl(q.y, src1, 64);
                u.z = __shfl(q.z, src1, 64);
                u.w = __shfl(q.w, src1, 64);
#pragma unroll 1
                for (int k = 0; k < 8; k++) {
                    // lanes start at different balls (and points below): those of one place would share its banks
                    const uint32_t sub = (e1 >> 6) * 8 + ((k + lane) & 7);
                    const bool ps = lane < t1 && passes(s_sub[sub], u);
                    push(q2, n2, ps, __ballot(ps), (uint32_t)src1 | sub << 6);
                    while (n2 >= 64 || (last && n1 == 0 && k == 7 && n2 > 0)) {
                        wave_lds_fence();
                        const int t2 = min(n2, 64);
                        n2 -= t2;
                        const uint32_t e2 = lane < t2 ? q2[n2 + lane] : 0u;  // (lane of the Gaussian, ball of 8)
                        const int src = (int)(e2 & 63u);
                        float4 c;
                        c.x = __shfl(q.x, src, 64);
                        c.y = __shfl(q.y, src, 64);
                        c.z = __shfl(q.z, src, 64);
                        c.w = CLR ? __shfl(q.w, src, 64) : 0.0f;
                        const float lo = __shfl(band.x, src, 64), hi = __shfl(band.y, src, 64);
                        wave_lds_fence();
                        uint32_t amb = 0;  // points in the band
                        if (lane < t2) {
#pragma unroll
                            for (int j = 0; j < 8; j++) {
                                const int i = (int)(e2 >> 6) * 8 + ((j + lane) & 7);
                                const float4 p = s_pt[i];
                                const float dx = p.x - c.x, dy = p.y - c.y, dz = p.z - c.z;
                                const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                                if (CLR) {
                                    const float v = __builtin_amdgcn_sqrtf(d2) - c.w;
                                    if (v < p.w) atomic_min_float(&s_pt[i].w, v);
                                }
                                if (d2 <= hi) {
                                    const unsigned long long bit = 1ull << (i & 63);
                                    if (!(s_hit[i >> 6] & bit)) {
                                        if (d2 < lo) atomicOr(&s_hit[i >> 6], bit);
                                        else amb |= 1u << j;
                                    }
                                }
                            }
                        }
                        if (__ballot(amb != 0)) {
                            for (; amb; amb &= amb - 1) {
                                const int i = (int)(e2 >> 6) * 8 + ((__builtin_ctz(amb) + lane) & 7);
                                const float4 p = s_pt[i];
                                if (collide64(g, base + src, p.x, p.y, p.z, r_robot, lambda_g))
                                    atomicOr(&s_hit[i >> 6], 1ull << (i & 63));
                            }
                        }
                    }
                }
            }
        }
    }
    __syncthreads();
    for (int gr = wv; gr < ng; gr += CK_THREADS / 64) {
        const float4 p = s_pt[gr * 64 + lane];
        if (!(p.x == p.x)) continue;
        const uint32_t i = P.index[(g0 + gr) * 64 + lane];
        if ((s_hit[gr] >> lane) & 1ull) collide[i] = 1;  // every writer writes 1
        if (CLR && lower(p.w, P, (g0 + gr) * 64 + lane, clearance[i])) atomic_min_float(&clearance[i], p.w);
    }
}

// Points of one set of launches; more are taken in turn (their scratch is shared, in stream order).
constexpr int64_t CC_MAX_POINTS = (int64_t)1 << 20;
// Most Gaussians of the bounds' sample.  A 40 m lot's points are then bounded to half a metre on
// average; four times as many cost 30 us more for 8,256 points and leave a tenth fewer pairs.
constexpr int64_t CC_SAMPLE = 4096;

// Whether all pairs in one launch beat the grouping, whose launches take 35 (129 points) to 100 us (8,256) however few the
// Gaussians, 170 (100,000 close by) to 350 (scattered): while the pairs take no longer (8.7e8: 240 us; without
// clearances the groups need less, 2^27), and neither does a wave's chain (a sixteenth of the Gaussians; 8,192: 27 us).  More
// points than that keep the groups, which are faster by 2 where points lie close, from 2,048 Gaussians on.
bool pairs_pay(int64_t n, int64_t np, bool clearance) {
    if (!clearance) return n <= 8192 && n * np <= (int64_t)1 << 27;
    if (n <= 8192) return n <= 2048 || n * np <= (int64_t)13 << 26;
    return n <= 12288 && np >= 8192 && n * np <= (int64_t)1 << 29;
}

// LDS of k_cc_check for slabs of gps groups.
size_t ck_lds_bytes(int gps) {
    const int ngp = (gps + CK_UNROLL - 1) / CK_UNROLL * CK_UNROLL;
    const size_t groups = (size_t)ngp * ((64 + 8 + 1) * sizeof(float4) + sizeof(unsigned long long));
    return std::max(groups, CK_THREADS * (sizeof(float4) + 2 * sizeof(float)));  // check_dense's tile
}

// Batches of k_cc_points for np points: their number and (equal) size, whole groups.
struct CcBatches {
    int blocks, per, groups;
    explicit CcBatches(int64_t np) {
        blocks = (int)((np + CP_BATCH - 1) / CP_BATCH);
        per = (int)(((np + blocks - 1) / blocks + 63) / 64 * 64);
        groups = blocks * per / 64;
    }
};

// Grid of k_cc_check: ny slabs of gps groups (numbers that check_dense deals out to twelve waves) and nx blocks over the
// Gaussians.  512 blocks run at a time; the least of their rounds and turns is taken, in units of a group's tests
// of a step: a step costs about two more, setting up and ending a block sixteen (their atomics too, so that more,
// shorter blocks lose: 30,000 Gaussians and 100,000 points 250 us as 504 blocks, 374 as 1,440).
struct CkGrid {
    int gps = 0, ny = 0, nx = 0;
    CkGrid(int groups, int64_t n) {
        const int64_t steps = (n + CK_THREADS - 1) / CK_THREADS;
        int64_t least = INT64_MAX;
        for (int s : {CK_GROUPS, 24, 16, 12, 8, 4}) {
            const int64_t slabs = (groups + s - 1) / s;
            for (int r = 1; r <= 4; r++) {
                const int64_t blocks = std::min<int64_t>(steps, std::max<int64_t>(1, 512 * r / slabs));
                const int64_t rounds = (blocks * slabs + 511) / 512, turns = (steps + blocks - 1) / blocks;
                const int64_t cost = rounds * (turns * (s + 2) + 16);
                if (cost >= least) continue;
                least = cost;
                gps = s;
                ny = (int)slabs;
                nx = (int)blocks;
            }
        }
    }
};

}  // namespace

size_t collision_ws_bytes(int64_t np) {
    if (np <= 0) return 256;
    // the largest set of launches; a smaller last one needs no more
    const CcBatches b(std::min(np, CC_MAX_POINTS));
    return (size_t)b.groups * (64 * 20 + 9 * 16);
}

void collision_check(const GaussDev& g, const float* pts, int64_t np_all, float r_robot, float lambda_g, void* ws,
                     int32_t* collide, float* clearance, hipStream_t s) {
    if (pairs_pay(g.n, np_all, clearance != nullptr)) {
        auto launch = [&](auto kernel, int64_t points) {
            kernel<<<(unsigned)((np_all + points - 1) / points), CP_THREADS, 0, s>>>(g, r_robot, lambda_g, pts, np_all,
                                                                                     collide, clearance);
        };
        // 64 points per block until that is two blocks a CU, then 256, then 1,024
        auto split = [&](auto clr) {
            constexpr bool CLR = decltype(clr)::value;
            if (np_all < 32768) launch(k_cc_pairs<CLR, 16, 1>, 64);
            else if (np_all < 262144) launch(k_cc_pairs<CLR, 8, 2>, 256);
            else launch(k_cc_pairs<CLR, 2, 2>, 1024);
        };
        if (clearance) split(std::true_type{});
        else split(std::false_type{});
        return;
    }
    for (int64_t p0 = 0; p0 < np_all; p0 += CC_MAX_POINTS) {
        const int np = (int)std::min(np_all - p0, CC_MAX_POINTS);
        const CcBatches b(np);
        const int npad = b.groups * 64;
        CcPoints P;
        P.ball = static_cast<float4*>(ws);
        P.sub = P.ball + b.groups;
        P.x = reinterpret_cast<float*>(P.sub + 8 * b.groups);
        P.y = P.x + npad;
        P.z = P.y + npad;
        P.ub = P.z + npad;
        P.index = reinterpret_cast<uint32_t*>(P.ub + npad);
        int32_t* hit = collide + p0;
        float* clr = clearance ? clearance + p0 : nullptr;
        k_cc_points<<<b.blocks, CP_THREADS, 0, s>>>(pts + p0, np_all, np, b.per, P, hit, clr);
        if (clr) {
            const int m = (int)std::min<int64_t>(g.n, std::max<int64_t>(1024, std::min<int64_t>(CC_SAMPLE, g.n / 128)));
            const bool wide = npad >= 65536;  // enough points for 256 blocks with four per lane
            const int gx = (npad + (wide ? 1023 : 255)) / (wide ? 1024 : 256);
            // about 1,024 blocks, each with whole rounds of 256 Gaussians
            const int rounds = (m + 255) / 256;
            const int gy = std::max(1, std::min(rounds, 1024 / gx));
            const int per = (rounds + gy - 1) / gy * 256;
            const dim3 grid((unsigned)gx, (unsigned)((m + per - 1) / per));
            if (wide) k_cc_bound<4><<<grid, 256, 0, s>>>(g, m, per, lambda_g, P, npad);
            else k_cc_bound<1><<<grid, 256, 0, s>>>(g, m, per, lambda_g, P, npad);
        }
        const CkGrid k(b.groups, g.n);
        const dim3 grid((unsigned)k.nx, (unsigned)k.ny);
        const size_t lds = ck_lds_bytes(k.gps);
        if (clr) k_cc_check<true><<<grid, CK_THREADS, lds, s>>>(g, r_robot, lambda_g, P, b.groups, k.gps, hit, clr);
        else k_cc_check<false><<<grid, CK_THREADS, lds, s>>>(g, r_robot, lambda_g, P, b.groups, k.gps, hit, clr);
    }
}

}  // namespace rtg
