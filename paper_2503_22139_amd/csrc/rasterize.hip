// rasterize.hip -- the X-ray Gaussian rasterizer of Stage 1 (Sec. 2.2,
// Eq. 7-9) and its adjoint.
//
// Per view, each 3-D Gaussian (mean p, Sigma = R(q) diag(s^2) R(q)^T, density
// rho) is mapped to a 2-D Gaussian on the detector by the local affine
// approximation of the projective map phi (Eq. 8): t = W (p - o) in the
// source-centred frame (u, v, central ray), phi(t) = (SDD t_u / (t_d du) +
// cu, SDD t_v / (t_d dv) + cv, |t|), J = d phi / d t at t, Sigma~ = J W Sigma
// W^T J^T; integrating along the ray coordinate (Eq. 9) leaves centre
// phi_01(t), covariance Sigma^ (top-left 2 x 2 of Sigma~) and amplitude
// rho sqrt(2 pi |Sigma~| / |Sigma^|).  A pixel's value is the sum of the
// 2-D Gaussians at its centre, each truncated to (x - mu)^T Sigma^-1 (x - mu)
// <= k^2 (k = inf: untruncated); Gaussians not in front of the source are
// skipped.  Geometry and pixel centres are those of the ray-march projector.
//
// Forward: per-(view, Gaussian) set-up in double, tile binning (16 x 16-pixel
// tiles, a counting sort by chunks of Gaussians; a Gaussian whose truncation
// box covers more than RS_TMAX tiles goes to a list of large splats), then one
// workgroup per tile: Gaussians staged in LDS, one pixel per thread, summed in
// fixed point (bit-reproducible), the large splats that reach the tile with
// its list.  Adjoint: one wave per splat walks the pixels of its box and
// reduces the six moments of g e over them (fixed order, no atomics); per
// (view, Gaussian) the chain rule goes from these back to (p, s, q, rho) in
// double, summed over views in order.
#include <math.h>

#include <algorithm>

#include "pmf_internal.h"

namespace pmf {

constexpr int RS_T = 16;                // tile edge (pixels)
constexpr int RS_THREADS = RS_T * RS_T;
constexpr int RS_TMAX = 16;             // tiles per Gaussian on the tile path
constexpr int RS_W = 12288;             // tiles per window of counts (48 KB of LDS)
constexpr int RS_CT = 512;              // threads (and Gaussians a pass) per chunk

// 2-D splat of one (view, Gaussian): centre, conic (Sigma^-1 = [[a, b], [b, c]]),
// amplitude, and its pixel box (empty when lo > hi).
struct alignas(16) SplatP {
    float mu_u, mu_v, a, b;
    float c, rho;
    uint16_t u0, v0, u1, v1;
};

// The box's tiles.
struct SplatTiles {
    int tu0, tv0, tu1, tv1, area;       // area 0: none
};
__device__ __forceinline__ SplatTiles splat_tiles(const SplatP &P) {
    SplatTiles t;
    t.tu0 = P.u0 / RS_T;
    t.tv0 = P.v0 / RS_T;
    t.tu1 = P.u1 / RS_T;
    t.tv1 = P.v1 / RS_T;
    t.area = P.u0 <= P.u1 && P.v0 <= P.v1 ? (t.tu1 - t.tu0 + 1) * (t.tv1 - t.tv0 + 1) : 0;
    return t;
}

struct RastGeo {
    double sad, sdd, du, dv, off_u, off_v;
    int nu, nv, tiles_u, tiles_v;
    float k;        // truncation radius (inf: none)
};

// Per (view, Gaussian) quantities in double: the view frame, J, Sigma~.
struct SplatD {
    bool ok;
    double t[3], nt, W[3][3], J[3][3], M[3][3], R[3][3], Sig[3][3], St[3][3];
    double mu[2], Sh[3];       // Sigma^ (s00, s01, s11)
    double det2, det3, amp;    // amp = sqrt(2 pi det3 / det2)
    double qh[4], qn;
};

__device__ void splat_setup(const RastGeo &G, double th, const float *p, const float *s,
                            const float *q, SplatD &D) {
    const double ct = cos(th), st = sin(th);
    const double o[3] = {G.sad * ct, G.sad * st, 0.0};
    const double W[3][3] = {{-st, ct, 0.0}, {0.0, 0.0, 1.0}, {-ct, -st, 0.0}};
    double x[3];
    for (int a = 0; a < 3; ++a) x[a] = (double)p[a] - o[a];
    for (int r = 0; r < 3; ++r) {
        D.t[r] = W[r][0] * x[0] + W[r][1] * x[1] + W[r][2] * x[2];
        for (int c = 0; c < 3; ++c) D.W[r][c] = W[r][c];
    }
    D.ok = D.t[2] > 0.0;
    const double td = D.ok ? D.t[2] : 1.0;
    const double su = G.sdd / G.du, sv = G.sdd / G.dv;
    D.nt = sqrt(D.t[0] * D.t[0] + D.t[1] * D.t[1] + D.t[2] * D.t[2]);
    D.mu[0] = su * D.t[0] / td + 0.5 * (G.nu - 1) - G.off_u;
    D.mu[1] = sv * D.t[1] / td + 0.5 * (G.nv - 1) - G.off_v;
    double J[3][3] = {{su / td, 0.0, -su * D.t[0] / (td * td)},
                      {0.0, sv / td, -sv * D.t[1] / (td * td)},
                      {D.t[0] / D.nt, D.t[1] / D.nt, D.t[2] / D.nt}};
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            D.J[r][c] = J[r][c];
            D.M[r][c] = J[r][0] * W[0][c] + J[r][1] * W[1][c] + J[r][2] * W[2][c];
        }
    // Sigma = R diag(s^2) R^T, normalised quaternion (w, x, y, z)
    D.qn = sqrt((double)q[0] * q[0] + (double)q[1] * q[1] + (double)q[2] * q[2] + (double)q[3] * q[3]);
    for (int k = 0; k < 4; ++k) D.qh[k] = q[k] / D.qn;
    const double w = D.qh[0], xq = D.qh[1], y = D.qh[2], z = D.qh[3];
    const double R[3][3] = {{1 - 2 * (y * y + z * z), 2 * (xq * y - w * z), 2 * (xq * z + w * y)},
                            {2 * (xq * y + w * z), 1 - 2 * (xq * xq + z * z), 2 * (y * z - w * xq)},
                            {2 * (xq * z - w * y), 2 * (y * z + w * xq), 1 - 2 * (xq * xq + y * y)}};
    const double s2[3] = {(double)s[0] * s[0], (double)s[1] * s[1], (double)s[2] * s[2]};
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            D.R[r][c] = R[r][c];
            D.Sig[r][c] = R[r][0] * s2[0] * R[c][0] + R[r][1] * s2[1] * R[c][1] + R[r][2] * s2[2] * R[c][2];
        }
    double MS[3][3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
            MS[r][c] = D.M[r][0] * D.Sig[0][c] + D.M[r][1] * D.Sig[1][c] + D.M[r][2] * D.Sig[2][c];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
            D.St[r][c] = MS[r][0] * D.M[c][0] + MS[r][1] * D.M[c][1] + MS[r][2] * D.M[c][2];
    D.Sh[0] = D.St[0][0];
    D.Sh[1] = D.St[0][1];
    D.Sh[2] = D.St[1][1];
    D.det2 = D.Sh[0] * D.Sh[2] - D.Sh[1] * D.Sh[1];
    D.det3 = D.St[0][0] * (D.St[1][1] * D.St[2][2] - D.St[1][2] * D.St[2][1]) -
             D.St[0][1] * (D.St[1][0] * D.St[2][2] - D.St[1][2] * D.St[2][0]) +
             D.St[0][2] * (D.St[1][0] * D.St[2][1] - D.St[1][1] * D.St[2][0]);
    D.ok = D.ok && D.det2 > 0.0 && D.det3 > 0.0;
    D.amp = D.ok ? sqrt(2.0 * M_PI * D.det3 / D.det2) : 0.0;
}

// ------------------------------------------------------------------ binning
// A counting sort of the (splat, tile) pairs by tile.  A view's Gaussians are
// cut into chunks, one workgroup each: k_splat_prep builds the chunk's splats
// and counts its pairs per tile in LDS (an atomic's old value is the pair's
// place among the chunk's), k_splat_chunks turns the chunks' counts of a tile
// into places and totals, k_rast_scan scans the totals into the lists' offsets
// and k_splat_fill writes each pair to its place and lists the large splats.
// (Counts in global memory took a device-scope atomic per pair: 75 us with the
// clears for 200k Gaussians on 512 x 384, now 39 us.)  Counts are held for
// RS_W tiles at a time; a larger detector walks its splats again per window.
struct SplatBins {
    int V, nch, T;                     // views, chunks per view, tiles per view
    int64_t m, chunk;                  // Gaussians, Gaussians per chunk
};

// A launch of n < 2^32 workgroups, over two grid dimensions: one of them holds
// fewer than 2^32 threads (2^22 workgroups of 1,024), and the runtime does not
// refuse more.
static dim3 many_blocks(int64_t n) {
    const int64_t x = std::min<int64_t>(std::max<int64_t>(n, 1), 1 << 21);
    return dim3((unsigned)x, (unsigned)((n + x - 1) / x));
}
// The workgroup's number (the last ones may lie past n).
__device__ __forceinline__ uint32_t flat_block() { return blockIdx.y * gridDim.x + blockIdx.x; }

// Pixel box of the ellipse of D: its half-extents k sqrt(Sigma^_aa), widened
// by a bound on the rounding errors that the pixels' float arithmetic makes of
// the conic (about 2^-24 s00 s11 / det2 of k^2) and of the centre.
__device__ __forceinline__ void splat_box(const RastGeo &G, const SplatD &D, SplatP &P) {
    double u0 = 0.0, u1 = G.nu - 1, v0 = 0.0, v1 = G.nv - 1;
    if (isfinite(G.k)) {
        const double wide = G.k * (1.0 + 2e-6 * (D.Sh[0] * D.Sh[2] / D.det2));
        const double ru = wide * sqrt(D.Sh[0]) + 0.01 + 1e-6 * (fabs(D.mu[0]) + G.nu);
        const double rv = wide * sqrt(D.Sh[2]) + 0.01 + 1e-6 * (fabs(D.mu[1]) + G.nv);
        u0 = fmax(u0, ceil(D.mu[0] - ru));
        u1 = fmin(u1, floor(D.mu[0] + ru));
        v0 = fmax(v0, ceil(D.mu[1] - rv));
        v1 = fmin(v1, floor(D.mu[1] + rv));
    }
    if (u0 <= u1 && v0 <= v1) {
        P.u0 = (uint16_t)u0;
        P.u1 = (uint16_t)u1;
        P.v0 = (uint16_t)v0;
        P.v1 = (uint16_t)v1;
    }
}

// Calls f(tile - w0, k) for the pairs k = 0.. (row by row) of a splat with a
// tile in [w0, w0 + RS_W).
template <class F>
__device__ __forceinline__ void each_tile(const SplatTiles &t, int tiles_u, int w0, F &&f) {
    int k = 0;
    for (int ty = t.tv0; ty <= t.tv1; ++ty)
        for (int tx = t.tu0; tx <= t.tu1; ++tx, ++k) {
            const int w = ty * tiles_u + tx - w0;
            if (w >= 0 && w < RS_W) f(w, k);
        }
}

__global__ __launch_bounds__(RS_CT) void k_splat_prep(const float *__restrict__ mean,
                                                      const float *__restrict__ scale,
                                                      const float *__restrict__ quat,
                                                      const float *__restrict__ value,
                                                      SplatBins B, RastGeo G,
                                                      const float *__restrict__ angles,
                                                      SplatP *__restrict__ sp,
                                                      int *__restrict__ part,
                                                      int *__restrict__ slot,
                                                      int *__restrict__ nlarge) {
    extern __shared__ int hist[];
    const uint32_t blk = flat_block(), nch = (uint32_t)B.nch;
    const int v = (int)(blk / nch), ch = (int)(blk - (uint32_t)v * nch);
    if (v >= B.V) return;
    const int64_t g0 = ch * B.chunk, g1 = min(g0 + B.chunk, B.m);
    int *const row = part + (int64_t)blk * B.T;
    const int64_t mv = B.m * B.V;
    if (blk == 0 && threadIdx.x == 0) *nlarge = 0;
    for (int w0 = 0; w0 < B.T; w0 += RS_W) {
        const int nw = min(RS_W, B.T - w0);
        for (int t = threadIdx.x; t < nw; t += RS_CT) hist[t] = 0;
        __syncthreads();
        for (int64_t g = g0 + threadIdx.x; g < g1; g += RS_CT) {
            const int64_t i = (int64_t)v * B.m + g;
            SplatP P;
            if (w0 > 0) {
                P = sp[i];
            } else {
                SplatD D;
                splat_setup(G, (double)angles[v], mean + 3 * g, scale + 3 * g, quat + 4 * g, D);
                P.mu_u = P.mu_v = P.a = P.b = P.c = P.rho = 0.0f;
                P.u0 = P.v0 = 1;
                P.u1 = P.v1 = 0;
                if (D.ok) {
                    P.mu_u = (float)D.mu[0];
                    P.mu_v = (float)D.mu[1];
                    P.a = (float)(D.Sh[2] / D.det2);
                    P.b = (float)(-D.Sh[1] / D.det2);
                    P.c = (float)(D.Sh[0] / D.det2);
                    P.rho = (float)((double)value[g] * D.amp);
                    splat_box(G, D, P);
                }
                sp[i] = P;
            }
            const SplatTiles t = splat_tiles(P);
            if (t.area > 0 && t.area <= RS_TMAX)
                each_tile(t, G.tiles_u, w0, [&](int w, int k) {
                    slot[k * mv + i] = atomicAdd(&hist[w], 1);
                });
        }
        __syncthreads();
        for (int t = threadIdx.x; t < nw; t += RS_CT) row[w0 + t] = hist[t];
        __syncthreads();
    }
}

// Per tile: the chunks' counts -> the places of their first pairs in the tile's
// list, in place, and the tile's total.  A workgroup takes 64 tiles of a view (a
// lane each), its sixteen waves a sixteenth of the chunks each.
__global__ __launch_bounds__(1024) void k_splat_chunks(int *__restrict__ part, SplatBins B,
                                                       int *__restrict__ total) {
    __shared__ int sums[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t blk = flat_block(), nb = (uint32_t)(B.T + 63) / 64;
    const int v = (int)(blk / nb);
    if (v >= B.V) return;
    const int t = (int)(blk - (uint32_t)v * nb) * 64 + lane;
    int *const p = part + (int64_t)v * B.nch * B.T + t;
    const int c0 = (int)((int64_t)B.nch * w / 16), c1 = (int)((int64_t)B.nch * (w + 1) / 16);
    int s = 0;
    if (t < B.T) {
#pragma unroll 8
        for (int c = c0; c < c1; ++c) s += p[(int64_t)c * B.T];
    }
    sums[w][lane] = s;
    __syncthreads();
    if (t >= B.T) return;
    int run = 0;
    for (int k = 0; k < w; ++k) run += sums[k][lane];
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
        const int x = p[(int64_t)c * B.T];
        p[(int64_t)c * B.T] = run;
        run += x;
    }
    if (w == 15) total[(int64_t)v * B.T + t] = run;
}

// Exclusive prefix sum of n totals (one workgroup, chunks of 1024).
__global__ __launch_bounds__(1024) void k_rast_scan(const int *__restrict__ total, int64_t n,
                                                    int *__restrict__ offsets) {
    __shared__ int wsum[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int carry = 0;
    for (int64_t b = 0; b < n; b += 1024) {
        const int64_t i = b + threadIdx.x;
        const int x = i < n ? total[i] : 0;
        const int incl = wave_incl_sum(x);
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        int base = carry;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (k < w) base += wsum[k];
            carry += wsum[k];
        }
        if (i < n) offsets[i] = base + incl - x;
        __syncthreads();
    }
    if (threadIdx.x == 0) offsets[n] = carry;
}

__global__ __launch_bounds__(RS_CT) void k_splat_fill(const SplatP *__restrict__ sp, SplatBins B,
                                                      int tiles_u, const int *__restrict__ part,
                                                      const int *__restrict__ offsets,
                                                      const int *__restrict__ slot,
                                                      int *__restrict__ list,
                                                      int *__restrict__ large,
                                                      int *__restrict__ nlarge) {
    extern __shared__ int base[];
    const uint32_t blk = flat_block(), nch = (uint32_t)B.nch;
    const int v = (int)(blk / nch), ch = (int)(blk - (uint32_t)v * nch);
    if (v >= B.V) return;
    const int64_t g0 = ch * B.chunk, g1 = min(g0 + B.chunk, B.m);
    const int *const row = part + (int64_t)blk * B.T;
    const int64_t mv = B.m * B.V;
    for (int w0 = 0; w0 < B.T; w0 += RS_W) {
        const int nw = min(RS_W, B.T - w0);
        for (int t = threadIdx.x; t < nw; t += RS_CT)
            base[t] = offsets[(int64_t)v * B.T + w0 + t] + row[w0 + t];
        __syncthreads();
        for (int64_t g = g0 + threadIdx.x; g < g1; g += RS_CT) {
            const int64_t i = (int64_t)v * B.m + g;
            const SplatTiles t = splat_tiles(sp[i]);
            if (t.area > RS_TMAX) {
                // (the order of the large list changes no result)
                if (w0 == 0) large[atomicAdd(nlarge, 1)] = (int)i;
            } else if (t.area > 0) {
                each_tile(t, tiles_u, w0, [&](int w, int k) {
                    list[base[w] + slot[k * mv + i]] = (int)i;
                });
            }
        }
        __syncthreads();
    }
}

// e^(-m/2) of splat P at pixel (x, y), 0 outside the ellipse.  (-log2(e) / 2
// rounds to half of log2(e)'s float: the product is that of e^x's own.)
__device__ __forceinline__ float splat_at(const SplatP &P, float x, float y, float k2, float &du,
                                          float &dv) {
    du = x - P.mu_u;
    dv = y - P.mu_v;
    const float m = fmaf(P.a * du, du, fmaf(2.0f * P.b * du, dv, P.c * dv * dv));
    return m <= k2 ? __builtin_amdgcn_exp2f(-0.72134752044f * m) : 0.0f;
}

// ------------------------------------------------------------------ forward
// Whether splat P may pass m <= k2 at a pixel of the 8 x 8 block from (x0, y0):
// the least m over the block lies on an edge that faces the centre.  The
// pixels' m carry rounding errors below 1e-6 of the terms' sizes.
__device__ __forceinline__ bool splat_reaches(const SplatP &P, float x0, float y0, float k2) {
    const float u0 = x0 - P.mu_u, u1 = u0 + 7.0f, v0 = y0 - P.mu_v, v1 = v0 + 7.0f;
    const float cu = fmaxf(u0, fminf(0.0f, u1)), cv = fmaxf(v0, fminf(0.0f, v1));
    const float b2 = 2.0f * P.b;
    const float pv = fminf(fmaxf(-P.b * cu * __builtin_amdgcn_rcpf(P.c), v0), v1);
    const float pu = fminf(fmaxf(-P.b * cv * __builtin_amdgcn_rcpf(P.a), u0), u1);
    const float m1 = P.a * cu * cu + b2 * cu * pv + P.c * pv * pv;
    const float m2 = P.a * pu * pu + b2 * pu * cv + P.c * cv * cv;
    const float du = fmaxf(-u0, u1), dv = fmaxf(-v0, v1);
    const float terms = P.a * du * du + fabsf(b2) * du * dv + P.c * dv * dv;
    return !(fminf(m1, m2) > k2 + 4e-6f * (terms + k2));
}

// One workgroup per (view, tile); a wave has one 8 x 8 block of the tile, one
// pixel per lane, and one PARTS-th of the staged splats.  Each pixel sums
// its splats in 32-bit fixed point with the tile's scale 2^30 / S, S = (number
// of splats reaching the tile: its list and the view's large Gaussians) x
// (their largest |amplitude|), so every pixel's sum stays below 2^30: neither
// the integer sums nor S depend on the order in which the binning's atomics
// filled the list, nor on the parts, so the images repeat bit for bit.  The
// large Gaussians (no tile entries) are staged by every tile, after its list,
// like the list's: a thread tests one against the tile and its blocks (200k
// on 2048 x 2048: 338 ms with every wave on every one, 674 with a quarter of
// them per wave of sixteen, now 9.4).
//
// The walk is bound by VALU issue, so a staged splat is tested once per block
// and the waves visit only the splats that reach theirs (a bit mask per
// block): 200k Gaussians of about 20 pixels on 512 x 384: 130 us with every
// wave on every splat of its tile, now 67 (with two parts 70, with one 81).
//
// Four parts pay where the tiles are few and their lists long; else the
// sixteen waves of a tile only wait for its start and end.  Kernel alone, four
// parts / one: 512x384 (768 tiles) one view, 10,000 Gaussians of s to 2 voxels
// 14 / 10 us, 50,000 21 / 22, 200,000 52 / 65; 256x192 (192) 2,000 7.6 / 7.1, 10,000
// 8.9 / 9.7; 64x48 (12) 300 7.2 / 7.2, 2,000 8.0 / 9.6; 512x384 four views, 50,000
// 63 / 52; 1024x768 one view, 200,000 467 / 471, 10 Gaussians 12 / 8.
constexpr int64_t RF_FEW = 1024;        // tiles of all views
constexpr int64_t RF_LONG = 40;         // Gaussians per tile of a view

template <int PARTS>
__global__ __launch_bounds__(RS_THREADS * PARTS) void k_splat_fwd(const SplatP *__restrict__ sp, int64_t m, int V,
                                                    RastGeo G,
                                                    const int *__restrict__ offsets,
                                                    const int *__restrict__ list,
                                                    const int *__restrict__ large,
                                                    const int *__restrict__ nlarge,
                                                    float *__restrict__ proj) {
    constexpr int RF_T = RS_THREADS * PARTS;
    __shared__ SplatP sh[RF_T + 1];              // the last one adds nothing
    __shared__ uint64_t mask[4][RF_T / 64];
    __shared__ float red[RF_T / 64];
    __shared__ int cnt[RF_T / 64];
    __shared__ int sum[RS_THREADS];
    const uint32_t T = (uint32_t)(G.tiles_u * G.tiles_v), tix = flat_block();
    const int v = (int)(tix / T), t = (int)(tix - (uint32_t)v * T);
    if (v >= V) return;
    const int tx = t % G.tiles_u, ty = t / G.tiles_u;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int blk = wave & 3, part = wave >> 2;
    const int x = tx * RS_T + (blk & 1) * 8 + (lane & 7);
    const int y = ty * RS_T + (blk >> 1) * 8 + (lane >> 3);
    const float fx = (float)x, fy = (float)y;
    const float k2 = G.k * G.k;
    const int b = offsets[tix], e = offsets[tix + 1];
    const int nl = *nlarge;
    if (b == e && nl == 0) {                     // nothing here
        if (part == 0 && x < G.nu && y < G.nv) proj[((int64_t)v * G.nv + y) * G.nu + x] = 0.0f;
        return;
    }
    auto reaches = [&](const SplatP &P) {
        const SplatTiles q = splat_tiles(P);
        return q.area > 0 && q.tu0 <= tx && tx <= q.tu1 && q.tv0 <= ty && ty <= q.tv1;
    };
    // S = (splats reaching the tile) x (their largest |amplitude|): an
    // order-independent bound of every pixel's sum
    float mx = 0.0f;
    int nh = 0;
    for (int q = b + (int)threadIdx.x; q < e; q += RF_T) mx = fmaxf(mx, fabsf(sp[list[q]].rho));
    for (int q = (int)threadIdx.x; q < nl; q += RF_T) {
        const int i = large[q];
        if (i >= v * m && i < (v + 1) * m && reaches(sp[i])) {
            mx = fmaxf(mx, fabsf(sp[i].rho));
            ++nh;
        }
    }
    mx = wave_max(mx);
    for (int o = 32; o > 0; o >>= 1) nh += __shfl_xor(nh, o, 64);
    if (lane == 0) {
        red[wave] = mx;
        cnt[wave] = nh;
    }
    if (threadIdx.x < RS_THREADS) sum[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        SplatP z = {};
        sh[RF_T] = z;
    }
    __syncthreads();
    int reach = e - b;
    mx = 0.0f;
#pragma unroll
    for (int w = 0; w < RF_T / 64; ++w) {
        reach += cnt[w];
        mx = fmaxf(mx, red[w]);
    }
    const float S = (float)reach * mx;
    const float scale = S > 0.0f ? 1073741824.0f / (S * 1.0001f) : 0.0f;
    int acc = 0;
    auto add = [&](int j) {
        const SplatP P = sh[j];
        float du, dv;
        acc += __float2int_rn(P.rho * splat_at(P, fx, fy, k2, du, dv));
    };
    // adds up to RF_T splats, one per thread
    auto add_staged = [&](int n, bool on, SplatP P) {
        if (on) {
            P.rho *= scale;
            sh[threadIdx.x] = P;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t bits = __ballot(on && splat_reaches(P, (float)(tx * RS_T + (q & 1) * 8),
                                                               (float)(ty * RS_T + (q >> 1) * 8), k2));
            if (lane == 0) mask[q][wave] = bits;
        }
        __syncthreads();
        for (int w = part; w * 64 < n; w += PARTS) {
            uint64_t bits = mask[blk][w];
            bits = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)bits) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(bits >> 32)) << 32;
            while (bits) {                       // uniform; four at a time
                int j[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    j[k] = bits ? w * 64 + __builtin_ctzll(bits) : RF_T;
                    bits &= bits - 1;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) add(j[k]);
            }
        }
        __syncthreads();
    };
    for (int c0 = b; c0 < e; c0 += RF_T) {
        const int n = min(RF_T, e - c0);
        const bool on = (int)threadIdx.x < n;
        SplatP P = {};
        if (on) P = sp[list[c0 + threadIdx.x]];
        add_staged(n, on, P);
    }
    for (int c0 = 0; c0 < nl; c0 += RF_T) {
        const int n = min(RF_T, nl - c0);
        bool on = (int)threadIdx.x < n;
        SplatP P = {};
        if (on) {
            const int i = large[c0 + threadIdx.x];
            on = i >= v * m && i < (v + 1) * m;
            if (on) P = sp[i];
            on = on && reaches(P);
        }
        add_staged(n, on, P);
    }
    if constexpr (PARTS > 1) {
        atomicAdd(&sum[blk * 64 + lane], acc);
        __syncthreads();
        if (part > 0) return;
        acc = sum[blk * 64 + lane];
    }
    if (x < G.nu && y < G.nv)
        proj[((int64_t)v * G.nv + y) * G.nu + x] = scale > 0.0f ? (float)acc / scale : 0.0f;
}

// ------------------------------------------------------------------ adjoint
// Moments of ge = g e over a splat's pixels: ge, ge du, ge dv, ge du^2,
// ge du dv, ge dv^2; the chain rule turns them into the gradients of
// amplitude, centre and conic.
struct SplatSums {
    float s[6];
};
__device__ __forceinline__ void splat_moments(const SplatP &P, float x, float y, float k2, float g,
                                              SplatSums &o) {
    float du, dv;
    const float ge = g * splat_at(P, x, y, k2, du, dv), gu = ge * du, gv = ge * dv;
    o.s[0] += ge;
    o.s[1] += gu;
    o.s[2] += gv;
    o.s[3] = fmaf(gu, du, o.s[3]);
    o.s[4] = fmaf(gu, dv, o.s[4]);
    o.s[5] = fmaf(gv, dv, o.s[5]);
}

// One wave per (view, Gaussian): the pixels of its box laid over the lanes 64
// at a time, row by row, and the six sums reduced over the wave once.  Splats
// on the large list are left to k_splat_large_bwd.
// Bound by VALU issue (25 per 64 pixels, 45 for set-up and reduction): 200k
// Gaussians of about 20 x 20 pixels on 512 x 384.  By tile -- every pixel of
// the five tiles a splat reaches, and a wave reduction per tile and wave -- it
// took 275 us and 21 to gather the tiles' partials, now 73 us.
__global__ __launch_bounds__(256) void k_splat_bwd(const SplatP *__restrict__ sp, int64_t m, int V, int nb,
                                                   RastGeo G, const float *__restrict__ g_proj,
                                                   float *__restrict__ acc6) {
    const uint32_t blk = flat_block();
    const int v = (int)(blk / (uint32_t)nb);
    const int64_t g = (int64_t)(blk - (uint32_t)v * (uint32_t)nb) * 4 +
                      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (v >= V || g >= m) return;
    const int64_t i = (int64_t)v * m + g;
    const int lane = threadIdx.x & 63;
    SplatP P = sp[i];
    const int area = splat_tiles(P).area;
    if (area > RS_TMAX) return;
    SplatSums o = {};
    if (area > 0) {
        const float k2 = in_vgpr(G.k * G.k);
        const int w = P.u1 - P.u0 + 1, n = w * (P.v1 - P.v0 + 1);
        // pixel p = lane + 64 k is (p % w, p / w): w <= 256, so the float
        // quotients of p + 1/2 are exact after truncation
        const float rw = __builtin_amdgcn_rcpf((float)w);
        const int ly = (int)(((float)lane + 0.5f) * rw), sy = (int)(64.5f * rw);
        const int lx = lane - ly * w, sx = 64 - sy * w;
        float x = (float)(P.u0 + lx), y = (float)(P.v0 + ly);
        // the step to the lane's next pixel, and past the end of a row
        const float dx0 = in_vgpr((float)sx), dx1 = in_vgpr((float)(sx - w));
        const float dy0 = in_vgpr((float)sy), dy1 = in_vgpr((float)(sy + 1));
        const float end = in_vgpr((float)(P.u1 - sx));
        const int st0 = 4 * (sy * G.nu + sx), st1 = st0 + 4 * (G.nu - w);
        const int dp0 = in_vgpr(st0), dp1 = in_vgpr(st1);
        const char *const base = (const char *)(g_proj + ((int64_t)v * G.nv + P.v0) * G.nu + P.u0);
        uint32_t p = 4u * (uint32_t)(ly * G.nu + lx);
        P.mu_u = in_vgpr(P.mu_u);
        P.mu_v = in_vgpr(P.mu_v);
        P.a = in_vgpr(P.a);
        P.b = in_vgpr(P.b);
        P.c = in_vgpr(P.c);
        auto at = [&]() { return *(const float *)(base + p); };
        auto next = [&]() {
            const bool wrap = x > end;
            x += wrap ? dx1 : dx0;
            y += wrap ? dy1 : dy0;
            p += (uint32_t)(wrap ? dp1 : dp0);
        };
        int k = 0;
#pragma unroll 2
        for (; k + 64 <= n; k += 64) {
            splat_moments(P, x, y, k2, at(), o);
            next();
        }
        if (k + lane < n) splat_moments(P, x, y, k2, at(), o);
    }
    const float z = 0.0f;
    const float lo = wave_sum4(o.s[0], o.s[1], o.s[2], o.s[3]);
    const float hi = wave_sum4(o.s[4], o.s[5], z, z);
    const int q = sum4_index(lane);
    if ((lane & 15) == 0) {
        acc6[i * 6 + q] = lo;
        if (q < 2) acc6[i * 6 + 4 + q] = hi;
    }
}

// Large-list Gaussians: one workgroup sums its box's contributions.
__global__ __launch_bounds__(256) void k_splat_large_bwd(const SplatP *__restrict__ sp, int64_t m,
                                                         RastGeo G, const int *__restrict__ large,
                                                         const int *__restrict__ nlarge,
                                                         const float *__restrict__ g_proj,
                                                         float *__restrict__ acc6) {
    __shared__ float red[4][6];
    const float k2 = G.k * G.k;
    const int n = *nlarge;
    for (int li = blockIdx.x; li < n; li += gridDim.x) {
        const int64_t i = large[li];
        const SplatP P = sp[i];
        const int v = (int)(i / m);
        const int w = P.u1 - P.u0 + 1;
        const int64_t npx = (int64_t)w * (P.v1 - P.v0 + 1);
        SplatSums o = {};
        for (int64_t p = threadIdx.x; p < npx; p += blockDim.x) {
            const int x = P.u0 + (int)(p % w), y = P.v0 + (int)(p / w);
            splat_moments(P, (float)x, (float)y, k2, g_proj[((int64_t)v * G.nv + y) * G.nu + x], o);
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) o.s[q] = wave_sum_lane63(o.s[q]);
        if ((threadIdx.x & 63) == 63)
#pragma unroll
            for (int q = 0; q < 6; ++q) red[threadIdx.x >> 6][q] = o.s[q];
        __syncthreads();
        if (threadIdx.x < 6)
            acc6[i * 6 + threadIdx.x] = (red[0][threadIdx.x] + red[1][threadIdx.x]) +
                                        (red[2][threadIdx.x] + red[3][threadIdx.x]);
        __syncthreads();
    }
}

// Chain rule per Gaussian, views in order (double): from the 2-D splat's
// moments to the mean, scale, quaternion and density.
__global__ __launch_bounds__(256) void k_splat_chain(const float *__restrict__ mean,
                                                     const float *__restrict__ scale,
                                                     const float *__restrict__ quat,
                                                     const float *__restrict__ value, int64_t m,
                                                     int V, RastGeo G,
                                                     const float *__restrict__ angles,
                                                     const float *__restrict__ acc6,
                                                     float *__restrict__ g_mean,
                                                     float *__restrict__ g_scale,
                                                     float *__restrict__ g_quat,
                                                     float *__restrict__ g_value) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= m) return;
    double gm[3] = {0, 0, 0}, gs[3] = {0, 0, 0}, gq[4] = {0, 0, 0, 0}, gv = 0.0;
    for (int v = 0; v < V; ++v) {
        const float *A6 = acc6 + ((int64_t)v * m + g) * 6;
        if (A6[0] == 0.0f && A6[1] == 0.0f && A6[2] == 0.0f && A6[3] == 0.0f && A6[4] == 0.0f &&
            A6[5] == 0.0f)
            continue;
        SplatD D;
        splat_setup(G, (double)angles[v], mean + 3 * g, scale + 3 * g, quat + 4 * g, D);
        if (!D.ok) continue;
        const double rho_hat = (double)value[g] * D.amp;
        const double grho = A6[0];
        gv += grho * D.amp;
        // conic A = Sigma^-1 (entries a, b (twice), c): dL/dSigma^ = -A Gc A
        const double Ai[2][2] = {{D.Sh[2] / D.det2, -D.Sh[1] / D.det2},
                                 {-D.Sh[1] / D.det2, D.Sh[0] / D.det2}};
        // the moments -> the gradients of the centre and of the conic
        const double gmu[2] = {rho_hat * (Ai[0][0] * A6[1] + Ai[0][1] * A6[2]),
                               rho_hat * (Ai[1][0] * A6[1] + Ai[1][1] * A6[2])};
        const double gb = -0.5 * rho_hat * A6[4];
        const double Gc[2][2] = {{-0.5 * rho_hat * A6[3], gb}, {gb, -0.5 * rho_hat * A6[5]}};
        double T2[2][2], GSh[2][2];
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 2; ++c) T2[r][c] = Gc[r][0] * Ai[0][c] + Gc[r][1] * Ai[1][c];
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 2; ++c) GSh[r][c] = -(Ai[r][0] * T2[0][c] + Ai[r][1] * T2[1][c]);
        // amplitude: rho^ = rho sqrt(2 pi det3 / det2): d/dSigma~ = rho^/2 Sigma~^-1,
        // d/dSigma^ = -rho^/2 Sigma^-1
        double Sti[3][3];
        {
            const double(*S)[3] = D.St;
            Sti[0][0] = (S[1][1] * S[2][2] - S[1][2] * S[2][1]) / D.det3;
            Sti[0][1] = (S[0][2] * S[2][1] - S[0][1] * S[2][2]) / D.det3;
            Sti[0][2] = (S[0][1] * S[1][2] - S[0][2] * S[1][1]) / D.det3;
            Sti[1][0] = (S[1][2] * S[2][0] - S[1][0] * S[2][2]) / D.det3;
            Sti[1][1] = (S[0][0] * S[2][2] - S[0][2] * S[2][0]) / D.det3;
            Sti[1][2] = (S[0][2] * S[1][0] - S[0][0] * S[1][2]) / D.det3;
            Sti[2][0] = (S[1][0] * S[2][1] - S[1][1] * S[2][0]) / D.det3;
            Sti[2][1] = (S[0][1] * S[2][0] - S[0][0] * S[2][1]) / D.det3;
            Sti[2][2] = (S[0][0] * S[1][1] - S[0][1] * S[1][0]) / D.det3;
        }
        const double hr = 0.5 * grho * rho_hat;
        double GSt[3][3];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) GSt[r][c] = hr * Sti[r][c];
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 2; ++c) GSt[r][c] += GSh[r][c] - hr * Ai[r][c];
        // Sigma~ = M Sigma M^T: dL/dSigma = M^T G M, dL/dM = 2 G M Sigma
        double GM[3][3], GSig[3][3], MS[3][3], GMM[3][3];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c)
                GM[r][c] = GSt[r][0] * D.M[0][c] + GSt[r][1] * D.M[1][c] + GSt[r][2] * D.M[2][c];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c)
                GSig[r][c] = D.M[0][r] * GM[0][c] + D.M[1][r] * GM[1][c] + D.M[2][r] * GM[2][c];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c)
                MS[r][c] = GM[r][0] * D.Sig[0][c] + GM[r][1] * D.Sig[1][c] + GM[r][2] * D.Sig[2][c];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) GMM[r][c] = 2.0 * MS[r][c];
        // M = J W: dL/dJ = dL/dM W^T
        double GJ[3][3];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c)
                GJ[r][c] = GMM[r][0] * D.W[c][0] + GMM[r][1] * D.W[c][1] + GMM[r][2] * D.W[c][2];
        // dL/dt: through the centre (rows 0, 1 of J) and through J(t)
        const double su = G.sdd / G.du, sv = G.sdd / G.dv;
        const double tu = D.t[0], tv = D.t[1], td = D.t[2], n = D.nt;
        double gt[3];
        for (int k = 0; k < 3; ++k) gt[k] = D.J[0][k] * gmu[0] + D.J[1][k] * gmu[1];
        gt[2] += GJ[0][0] * (-su / (td * td)) + GJ[1][1] * (-sv / (td * td));
        gt[0] += GJ[0][2] * (-su / (td * td));
        gt[2] += GJ[0][2] * (2.0 * su * tu / (td * td * td));
        gt[1] += GJ[1][2] * (-sv / (td * td));
        gt[2] += GJ[1][2] * (2.0 * sv * tv / (td * td * td));
        for (int c = 0; c < 3; ++c)
            for (int k = 0; k < 3; ++k)
                gt[k] += GJ[2][c] * (((c == k) ? 1.0 : 0.0) - D.t[c] * D.t[k] / (n * n)) / n;
        // t = W (p - o): dL/dp = W^T dL/dt
        for (int a = 0; a < 3; ++a) gm[a] += D.W[0][a] * gt[0] + D.W[1][a] * gt[1] + D.W[2][a] * gt[2];
        // Sigma = R diag(s^2) R^T: dL/ds_k = 2 s_k (R^T G R)_kk, dL/dR = 2 G R diag(s^2)
        const double s_[3] = {scale[3 * g], scale[3 * g + 1], scale[3 * g + 2]};
        double GR[3][3];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) {
                const double gr = GSig[r][0] * D.R[0][c] + GSig[r][1] * D.R[1][c] + GSig[r][2] * D.R[2][c];
                GR[r][c] = 2.0 * gr * s_[c] * s_[c];
            }
        for (int k = 0; k < 3; ++k) {
            double d = 0.0;
            for (int r = 0; r < 3; ++r)
                for (int c = 0; c < 3; ++c) d += D.R[r][k] * GSig[r][c] * D.R[c][k];
            gs[k] += 2.0 * s_[k] * d;
        }
        const double w = D.qh[0], x = D.qh[1], y = D.qh[2], z = D.qh[3];
        double gqh[4];
        gqh[0] = 2 * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] + x * GR[2][1]);
        gqh[1] = 2 * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - 2 * x * GR[1][1] - w * GR[1][2] +
                      z * GR[2][0] + w * GR[2][1] - 2 * x * GR[2][2]);
        gqh[2] = 2 * (-2 * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] + z * GR[1][2] -
                      w * GR[2][0] + z * GR[2][1] - 2 * y * GR[2][2]);
        gqh[3] = 2 * (-2 * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] - 2 * z * GR[1][1] +
                      y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
        const double dot = gqh[0] * w + gqh[1] * x + gqh[2] * y + gqh[3] * z;
        for (int k = 0; k < 4; ++k) gq[k] += (gqh[k] - D.qh[k] * dot) / D.qn;
    }
    for (int a = 0; a < 3; ++a) {
        g_mean[3 * g + a] = (float)gm[a];
        g_scale[3 * g + a] = (float)gs[a];
    }
    for (int k = 0; k < 4; ++k) g_quat[4 * g + k] = (float)gq[k];
    g_value[g] = (float)gv;
}

// ---------------------------------------------------------------- launchers
static RastGeo rast_geo(const pmf_cone_t &c, float k) {
    RastGeo G;
    G.sad = c.sad;
    G.sdd = c.sdd;
    G.du = c.du;
    G.dv = c.dv;
    G.off_u = c.off_u;
    G.off_v = c.off_v;
    G.nu = c.nu;
    G.nv = c.nv;
    G.tiles_u = (c.nu + RS_T - 1) / RS_T;
    G.tiles_v = (c.nv + RS_T - 1) / RS_T;
    G.k = k;
    return G;
}

// Chunks per view: of RS_CT Gaussians (a pass of their workgroup), at most 512
// a view and about 2,048 in all, and no more than 2^24 (chunk, tile) counts.
static SplatBins rast_bins(int64_t m, const RastGeo &G, int V) {
    SplatBins B;
    B.V = V;
    B.m = m;
    B.T = G.tiles_u * G.tiles_v;
    B.nch = (int)std::max<int64_t>(
        1, std::min<int64_t>({512, (m + RS_CT - 1) / RS_CT, std::max(1, 2048 / V),
                              (1 << 24) / std::max<int64_t>(1, (int64_t)B.T * V)}));
    B.chunk = (m + B.nch - 1) / B.nch;
    return B;
}

namespace {
struct RastWs {
    SplatP *sp;
    int *bins, *total, *offsets, *list, *large, *nlarge, *slot;
    float *acc6;
    size_t bytes;
};

RastWs rast_ws(void *base, int64_t m, const RastGeo &G, int V) {
    RastWs w;
    const SplatBins B = rast_bins(m, G, V);
    const size_t T = (size_t)B.T * (size_t)V;
    const size_t mv = (size_t)m * (size_t)V;
    char *p = (char *)base;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *r = p ? p + off : nullptr;
        off += align256(bytes);
        return r;
    };
    w.sp = (SplatP *)take(sizeof(SplatP) * mv);
    w.bins = (int *)take(sizeof(int) * (size_t)B.nch * T);      // the chunks' counts
    w.total = (int *)take(sizeof(int) * T);
    w.offsets = (int *)take(sizeof(int) * (T + 1));
    w.list = (int *)take(sizeof(int) * mv * RS_TMAX);
    w.large = (int *)take(sizeof(int) * mv);
    w.nlarge = (int *)take(sizeof(int));
    w.acc6 = (float *)take(sizeof(float) * 6 * mv);
    w.slot = (int *)take(sizeof(int) * mv * RS_TMAX);
    w.bytes = off;
    return w;
}
}  // namespace

size_t rasterize_workspace(int64_t m, const pmf_cone_t &c, int V) {
    return rast_ws(nullptr, m, rast_geo(c, 3.0f), V).bytes;
}

static hipError_t rast_bin(const pmf_gauss_t &gs, const RastGeo &G, const float *angles, int V,
                           const RastWs &w, hipStream_t s) {
    const SplatBins B = rast_bins(gs.m, G, V);
    const int64_t T = (int64_t)B.T * V;
    const dim3 nb = many_blocks((int64_t)B.nch * V);
    const size_t lds = sizeof(int) * (size_t)std::min(B.T, RS_W);
    hipError_t e;
    ProfScope prof_("rasterize_bin", s);
    k_splat_prep<<<nb, RS_CT, lds, s>>>(gs.mean, gs.scale, gs.quat, gs.value, B, G, angles, w.sp,
                                        w.bins, w.slot, w.nlarge);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_splat_chunks<<<many_blocks((int64_t)((B.T + 63) / 64) * V), 1024, 0, s>>>(w.bins, B, w.total);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_rast_scan<<<1, 1024, 0, s>>>(w.total, T, w.offsets);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_splat_fill<<<nb, RS_CT, lds, s>>>(w.sp, B, G.tiles_u, w.bins, w.offsets, w.slot, w.list,
                                        w.large, w.nlarge);
    return hipGetLastError();
}

hipError_t launch_rasterize(const pmf_gauss_t &gs, const pmf_cone_t &c, const float *angles,
                            int V, float k, float *proj, void *ws, hipStream_t s) {
    const RastGeo G = rast_geo(c, k);
    const RastWs w = rast_ws(ws, gs.m, G, V);
    hipError_t e = rast_bin(gs, G, angles, V, w, s);
    if (e != hipSuccess) return e;
    const int64_t T = (int64_t)G.tiles_u * G.tiles_v * V;
    {
        ProfScope prof_("rasterize", s);
        if (T <= RF_FEW && gs.m >= RF_LONG * (T / V))
            k_splat_fwd<4><<<many_blocks(T), 4 * RS_THREADS, 0, s>>>(w.sp, gs.m, V, G, w.offsets, w.list,
                                                                     w.large, w.nlarge, proj);
        else
            k_splat_fwd<1><<<many_blocks(T), RS_THREADS, 0, s>>>(w.sp, gs.m, V, G, w.offsets, w.list,
                                                                 w.large, w.nlarge, proj);
    }
    return hipGetLastError();
}

// rebin = false: ws already holds the binning of a pmf_rasterize call on the
// same inputs (splat records, tile lists, list positions), which is reused.
hipError_t launch_rasterize_bwd(const pmf_gauss_t &gs, const pmf_cone_t &c, const float *angles,
                                int V, float k, const float *g_proj, const pmf_gauss_grad_t &gg,
                                void *ws, hipStream_t s, bool rebin) {
    const RastGeo G = rast_geo(c, k);
    const RastWs w = rast_ws(ws, gs.m, G, V);
    hipError_t e = rebin ? rast_bin(gs, G, angles, V, w, s) : hipSuccess;
    if (e != hipSuccess) return e;
    {
        ProfScope prof_("rasterize_bwd", s);
        const int nb = (int)((gs.m + 3) / 4);
        if (gs.m > 0) {
            k_splat_bwd<<<many_blocks((int64_t)nb * V), 256, 0, s>>>(w.sp, gs.m, V, nb, G, g_proj,
                                                                     w.acc6);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        k_splat_large_bwd<<<1024, 256, 0, s>>>(w.sp, gs.m, G, w.large, w.nlarge, g_proj, w.acc6);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_splat_chain<<<(unsigned)((gs.m + 255) / 256), 256, 0, s>>>(
            gs.mean, gs.scale, gs.quat, gs.value, gs.m, V, G, angles, w.acc6, gg.mean, gg.scale,
            gg.quat, gg.value);
    }
    return hipGetLastError();
}

}  // namespace pmf
