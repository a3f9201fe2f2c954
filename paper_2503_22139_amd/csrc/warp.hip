// warp.hip -- the motion-compensated warp of Eq. 2 and its adjoint.
//
// One thread per voxel of the output grid; the sample point x_j + d is taken
// in voxel units as i_a + t_a, t_a = d_a / h_a, its cell decided from t_a
// (disp_cell).  The adjoint writes g_dvf directly (one owner per entry) and
// scatters g_ref onto the 8 corners of each sample in 64-bit fixed point
// (scale from the largest |g_out|), so g_ref does not depend on the order of
// the additions: bricks of voxels add into an LDS box with a halo, the boxes
// are staged, and a last pass sums the boxes that cover a voxel and converts
// to float.  Displacements that leave the halo add into a global 64-bit
// volume (the last pass adds it in).
#include <algorithm>

#include "pmf_internal.h"

namespace pmf {

__global__ __launch_bounds__(256) void k_warp(const float *__restrict__ ref, GridK g,
                                              const float *__restrict__ dvf, int V,
                                              float *__restrict__ out) {
    const int64_t N = grid_size(g);
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    const int iz = (int)(j % g.n[2]);
    const int iy = (int)((j / g.n[2]) % g.n[1]);
    const int ix = (int)(j / ((int64_t)g.n[2] * g.n[1]));
    for (int v = 0; v < V; ++v) {
        const float *d = dvf + (int64_t)v * 3 * N;
        const float t0 = d[j] * g.inv_h[0], t1 = d[N + j] * g.inv_h[1],
                    t2 = d[2 * N + j] * g.inv_h[2];
        out[(int64_t)v * N + j] = sample_disp(ref, g.n, ix, iy, iz, t0, t1, t2);
    }
}

// Bricks of the adjoint: 8 x 8 x 32 voxels, two per thread (lanes along axis
// 2: 128-byte rows), and a halo of 3 voxels (plus the upper corner) around
// the brick.  One global atomic per corner (67 M a view at 256x256x128, about
// 54 G/s) took 1.25 ms a view; the box takes them to LDS (70 KB, two
// workgroups of 16 waves per CU) and leaves its 64-bit words as the main
// traffic (4.3 per voxel, written and read once): 0.17 + 0.10 ms.
constexpr int WA0 = 8, WA1 = 8, WA2 = 32, WHALO = 3;
constexpr int WX0 = WA0 + 2 * WHALO + 1, WX1 = WA1 + 2 * WHALO + 1, WX2 = WA2 + 2 * WHALO + 1;
constexpr int WX = WX0 * WX1 * WX2;
constexpr int WB_THREADS = WA0 * WA1 * WA2 / 2;

// The double product x scale (|x| <= M, scale = 2^40 / M: below 2^41) rounded to
// the nearest integer, as 64 bits: the product plus 1.5 2^52 holds it in its low
// bits.  (fix_add's integer without its conversion; a split into two words in
// float loses the low ones of a negative term.)
__device__ __forceinline__ unsigned long long warp_fix(float x, double scale) {
#pragma clang fp contract(off)
    constexpr double MAGIC52 = 6755399441055744.0;
    const double p = (double)x * scale;
    return (unsigned long long)(__double_as_longlong(p + MAGIC52) -
                                __double_as_longlong(MAGIC52));
}

// One voxel's share of every view: g_dvf, and the terms of its corners into the
// box at (B0, B1, B2) where they lie in it (BOX), else into the 64-bit volume.
template <bool BOX>
__device__ __forceinline__ void warp_bwd_voxel(const float *__restrict__ ref, const GridK &g,
                                               const float *__restrict__ dvf, int V,
                                               const float *__restrict__ g_out, double fscale, int ix,
                                               int iy, int iz, int B0, int B1, int B2,
                                               unsigned long long *__restrict__ wbox,
                                               unsigned long long *__restrict__ fix,
                                               float *__restrict__ g_dvf) {
    const int64_t N = grid_size(g);
    const int s1 = g.n[2], s0 = g.n[1] * g.n[2];
    const int64_t j = ((int64_t)ix * g.n[1] + iy) * g.n[2] + iz;
    for (int v = 0; v < V; ++v) {
        const float *d = dvf + (int64_t)v * 3 * N;
        const float t0 = d[j] * g.inv_h[0], t1 = d[N + j] * g.inv_h[1],
                    t2 = d[2 * N + j] * g.inv_h[2];
        const float go = g_out[(int64_t)v * N + j];
        float *gd = g_dvf + (int64_t)v * 3 * N;
        int i0, i1, i2;
        float f0, f1, f2;
        if (!disp_cell(ix, t0, g.n[0], i0, f0) || !disp_cell(iy, t1, g.n[1], i1, f1) ||
            !disp_cell(iz, t2, g.n[2], i2, f2)) {
            gd[j] = 0.0f;
            gd[N + j] = 0.0f;
            gd[2 * N + j] = 0.0f;
            continue;
        }
        const int64_t base = ((int64_t)i0 * g.n[1] + i1) * g.n[2] + i2;
        const float *p = ref + base;
        const float c000 = p[0], c001 = p[1], c010 = p[s1], c011 = p[s1 + 1];
        const float c100 = p[s0], c101 = p[s0 + 1], c110 = p[s0 + s1], c111 = p[s0 + s1 + 1];
        // derivative of the trilinear blend along each axis (per voxel unit)
        const float a00 = lerp1(c000, c001, f2), a01 = lerp1(c010, c011, f2);
        const float a10 = lerp1(c100, c101, f2), a11 = lerp1(c110, c111, f2);
        const float dx = lerp1(a10, a11, f1) - lerp1(a00, a01, f1);
        const float dy = lerp1(a01, a11, f0) - lerp1(a00, a10, f0);
        const float b00 = lerp1(c000, c010, f1), b01 = lerp1(c001, c011, f1);
        const float b10 = lerp1(c100, c110, f1), b11 = lerp1(c101, c111, f1);
        const float dz = lerp1(b01, b11, f0) - lerp1(b00, b10, f0);
        gd[j] = go * dx * g.inv_h[0] * disp_free(ix, t0, g.n[0]);
        gd[N + j] = go * dy * g.inv_h[1] * disp_free(iy, t1, g.n[1]);
        gd[2 * N + j] = go * dz * g.inv_h[2] * disp_free(iz, t2, g.n[2]);
        if (go == 0.0f || !isfinite(go)) continue;     // (an infinite M leaves the scale 0)
        const float w0[2] = {1.0f - f0, f0}, w1[2] = {1.0f - f1, f1}, w2[2] = {1.0f - f2, f2};
        const int l0 = i0 - (B0 - WHALO), l1 = i1 - (B1 - WHALO), l2 = i2 - (B2 - WHALO);
        const bool inbox = BOX && l0 >= 0 && l0 + 1 < WX0 && l1 >= 0 && l1 + 1 < WX1 && l2 >= 0 &&
                           l2 + 1 < WX2;
        const int o = (l0 * WX1 + l1) * WX2 + l2;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const unsigned long long x = warp_fix(go * w0[a] * w1[b] * w2[c], fscale);
                    if (inbox) atomicAdd(&wbox[o + (a * WX1 + b) * WX2 + c], x);
                    else atomicAdd(&fix[base + a * s0 + b * s1 + c], x);
                }
    }
}

__global__ __launch_bounds__(WB_THREADS) void k_warp_bwd(const float *__restrict__ ref, GridK g,
                                                         const float *__restrict__ dvf, int V,
                                                         const float *__restrict__ g_out,
                                                         const uint32_t *__restrict__ gmax, int nb1,
                                                         int nb2, int first,
                                                         unsigned long long *__restrict__ fix,
                                                         unsigned long long *__restrict__ stage,
                                                         float *__restrict__ g_dvf) {
    __shared__ unsigned long long wbox[WX];
    const int local = xcd_block((int)blockIdx.x, (int)gridDim.x), blk = first + local;
    const int b2 = blk % nb2, b1 = (blk / nb2) % nb1, b0 = blk / (nb2 * nb1);
    const int B0 = b0 * WA0, B1 = b1 * WA1, B2 = b2 * WA2;
    for (int i = threadIdx.x; i < WX; i += WB_THREADS) wbox[i] = 0;
    __syncthreads();
    const double fscale = fix_scale(*gmax);
    const int iz = B2 + (int)threadIdx.x % WA2, iy = B1 + ((int)threadIdx.x / WA2) % WA1;
    for (int q = 0; q < 2; ++q) {
        const int ix = B0 + (int)threadIdx.x / (WA1 * WA2) + q * (WA0 / 2);
        if (ix >= g.n[0] || iy >= g.n[1] || iz >= g.n[2]) continue;
        warp_bwd_voxel<true>(ref, g, dvf, V, g_out, fscale, ix, iy, iz, B0, B1, B2, wbox, fix, g_dvf);
    }
    __syncthreads();
    unsigned long long *st = stage + (int64_t)local * WX;
    for (int i = threadIdx.x; i < WX; i += WB_THREADS) st[i] = wbox[i];
}

// A voxel per thread and every term straight into the 64-bit volume: grids whose
// bricks hold next to nothing (warp_direct).
__global__ __launch_bounds__(256) void k_warp_bwd_direct(const float *__restrict__ ref, GridK g,
                                                         const float *__restrict__ dvf, int V,
                                                         const float *__restrict__ g_out,
                                                         const uint32_t *__restrict__ gmax,
                                                         unsigned long long *__restrict__ fix,
                                                         float *__restrict__ g_dvf) {
    const unsigned j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= (unsigned)grid_size(g)) return;                // < 2^31
    const unsigned q = j / (unsigned)g.n[2];
    const int ix = (int)(q / (unsigned)g.n[1]);
    warp_bwd_voxel<false>(ref, g, dvf, V, g_out, fix_scale(*gmax), ix,
                          (int)(q - (unsigned)ix * (unsigned)g.n[1]), (int)(j - q * (unsigned)g.n[2]), 0,
                          0, 0, nullptr, fix, g_dvf);
}

// The staged boxes of bricks [first, first + count) (ALL: of every brick) that
// cover voxel j (at most two per axis), summed in 64 bits.
template <bool ALL>
__device__ __forceinline__ unsigned long long warp_boxes(const unsigned long long *__restrict__ stage,
                                                         const GridK &g, int nb0, int nb1, int nb2,
                                                         int first, int count, unsigned j) {
    const unsigned q = j / (unsigned)g.n[2];
    const int p2 = (int)(j - q * (unsigned)g.n[2]);
    const int p0 = (int)(q / (unsigned)g.n[1]);
    const int p1 = (int)(q - (unsigned)p0 * (unsigned)g.n[1]);
    // boxes b with b WA - WHALO <= p <= b WA + WA + WHALO
    const int a0 = max(0, (p0 - WHALO - 1) / WA0), e0 = min(nb0 - 1, (p0 + WHALO) / WA0);
    const int a1 = max(0, (p1 - WHALO - 1) / WA1), e1 = min(nb1 - 1, (p1 + WHALO) / WA1);
    const int a2 = max(0, (p2 - WHALO - 1) / WA2), e2 = min(nb2 - 1, (p2 + WHALO) / WA2);
    unsigned long long s = 0;
    for (int b0 = a0; b0 <= e0; ++b0)
        for (int b1 = a1; b1 <= e1; ++b1)
            for (int b2 = a2; b2 <= e2; ++b2) {
                const int blk = (b0 * nb1 + b1) * nb2 + b2 - (ALL ? 0 : first);
                if (!ALL && (blk < 0 || blk >= count)) continue;
                const int l0 = p0 - (b0 * WA0 - WHALO), l1 = p1 - (b1 * WA1 - WHALO),
                          l2 = p2 - (b2 * WA2 - WHALO);
                s += stage[(int64_t)blk * WX + (l0 * WX1 + l1) * WX2 + l2];
            }
    return s;
}

__device__ __forceinline__ float warp_unfix(unsigned long long s, uint32_t gmax) {
    const double sc = fix_scale(gmax);
    const double inv = sc > 0.0 ? 1.0 / sc : 0.0;       // 0 or infinite M: zeros
    return (float)((double)(long long)s * inv);
}

// g_ref[j] = the boxes of all bricks and the halo overflow, as a float.
__global__ __launch_bounds__(256) void k_warp_gather(
    const unsigned long long *__restrict__ stage, GridK g, int nb0, int nb1, int nb2,
    const unsigned long long *__restrict__ fix, const uint32_t *__restrict__ gmax,
    float *__restrict__ g_ref) {
    const unsigned j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= (unsigned)grid_size(g)) return;                // < 2^31
    g_ref[j] = warp_unfix(fix[j] + warp_boxes<true>(stage, g, nb0, nb1, nb2, 0, 0, j), *gmax);
}

// A round's boxes added to the 64-bit volume, voxels [j0, j0 + n).
__global__ __launch_bounds__(256) void k_warp_add_boxes(
    const unsigned long long *__restrict__ stage, GridK g, int nb0, int nb1, int nb2, int first,
    int count, unsigned j0, unsigned n, unsigned long long *__restrict__ fix) {
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const unsigned long long s =
        warp_boxes<false>(stage, g, nb0, nb1, nb2, first, count, j0 + i);
    if (s != 0) fix[j0 + i] += s;
}

__global__ __launch_bounds__(256) void k_warp_convert(const unsigned long long *__restrict__ fix,
                                                      unsigned n, const uint32_t *__restrict__ gmax,
                                                      float *__restrict__ g_ref) {
    const unsigned j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) g_ref[j] = warp_unfix(fix[j], *gmax);
}

hipError_t launch_warp(const float *ref, const GridK &g, const float *dvf, int V, float *out,
                       hipStream_t s) {
    const int64_t N = grid_size(g);
    {
        ProfScope prof_("warp", s);
        k_warp<<<(unsigned)((N + 255) / 256), 256, 0, s>>>(ref, g, dvf, V, out);
    }
    return hipGetLastError();
}

struct WarpBricks {
    int nb[3];
    int64_t n;
};
static WarpBricks warp_bricks(const GridK &g) {
    WarpBricks b{{(g.n[0] + WA0 - 1) / WA0, (g.n[1] + WA1 - 1) / WA1, (g.n[2] + WA2 - 1) / WA2}, 0};
    b.n = (int64_t)b.nb[0] * b.nb[1] * b.nb[2];
    return b;
}

// Bricks that are nearly empty cost their boxes' traffic for little (512x512x2,
// one view, displacements of 12 voxels 129 us by voxels, 187 by bricks; 512x512x4
// 273 / 262, smaller displacements 265 / 152), and on grids of a few bricks a
// thread's atomics past its box wait for each other (24^3, four views, 12 voxels
// 38 / 50 us; 32^3, 16 bricks, 66 / 70, smaller displacements 53 / 29).
static bool warp_direct(const GridK &g, const WarpBricks &b) {
    return b.n < 12 || grid_size(g) * 10 < (int64_t)(WA0 * WA1 * WA2) * b.n;
}

// Bricks of a round: all, unless their boxes (34 bytes per voxel) would take
// more than 1 GiB; then each round's boxes are added to the 64-bit volume (the
// sums are of integers: the same bits).
constexpr int64_t WSTAGE_BYTES = (int64_t)1 << 30;
static int warp_round(const WarpBricks &b) {
    return (int)std::min<int64_t>(b.n, WSTAGE_BYTES / (int64_t)(sizeof(long long) * WX));
}

// Workspace: the 64-bit fixed-point halo overflow, a round's staged boxes,
// then the largest |g_out|.
size_t warp_bwd_workspace(const GridK &g) {
    return align256(sizeof(long long) * (size_t)grid_size(g)) +
           align256(sizeof(long long) * WX * (size_t)warp_round(warp_bricks(g))) +
           align256(sizeof(uint32_t));
}

hipError_t launch_warp_bwd(const float *ref, const GridK &g, const float *dvf, int V,
                           const float *g_out, float *g_ref, float *g_dvf, void *ws,
                           hipStream_t s) {
    const int64_t N = grid_size(g);
    const WarpBricks b = warp_bricks(g);
    const int round = warp_round(b);
    unsigned long long *fix = (unsigned long long *)ws;
    unsigned long long *stage =
        (unsigned long long *)((char *)ws + align256(sizeof(long long) * (size_t)N));
    uint32_t *gmax =
        (uint32_t *)((char *)stage + align256(sizeof(long long) * WX * (size_t)round));
    hipError_t e = launch_fill_i32((int32_t *)fix, 2 * N, 0, s);
    if (e != hipSuccess) return e;
    if ((e = launch_absmax(g_out, N * V, gmax, s)) != hipSuccess) return e;
    if (warp_direct(g, b)) {
        const unsigned nb = (unsigned)((N + 255) / 256);
        {
            ProfScope prof_("warp_bwd", s);
            k_warp_bwd_direct<<<nb, 256, 0, s>>>(ref, g, dvf, V, g_out, gmax, fix, g_dvf);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        ProfScope prof_("warp_gather", s);
        k_warp_convert<<<nb, 256, 0, s>>>(fix, (unsigned)N, gmax, g_ref);
        return hipGetLastError();
    }
    const int plane = b.nb[1] * b.nb[2];
    const int64_t row = (int64_t)g.n[1] * g.n[2];
    for (int64_t first = 0; first < b.n; first += round) {
        const int count = (int)std::min<int64_t>(round, b.n - first);
        {
            ProfScope prof_("warp_bwd", s);
            k_warp_bwd<<<(unsigned)count, WB_THREADS, 0, s>>>(ref, g, dvf, V, g_out, gmax, b.nb[1],
                                                              b.nb[2], (int)first, fix, stage, g_dvf);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (round == b.n) break;
        // the rows along axis 0 that the round's boxes reach
        const int64_t x0 = std::max<int64_t>(0, first / plane * WA0 - WHALO);
        const int64_t x1 = std::min<int64_t>(g.n[0], ((first + count - 1) / plane + 1) * WA0 + WHALO + 1);
        const unsigned n = (unsigned)((x1 - x0) * row);
        {
            ProfScope prof_("warp_gather", s);
            k_warp_add_boxes<<<(n + 255) / 256, 256, 0, s>>>(stage, g, b.nb[0], b.nb[1], b.nb[2],
                                                             (int)first, count, (unsigned)(x0 * row), n,
                                                             fix);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    {
        ProfScope prof_("warp_gather", s);
        const unsigned nb = (unsigned)((N + 255) / 256);
        if (round == b.n)
            k_warp_gather<<<nb, 256, 0, s>>>(stage, g, b.nb[0], b.nb[1], b.nb[2], fix, gmax, g_ref);
        else
            k_warp_convert<<<nb, 256, 0, s>>>(fix, (unsigned)N, gmax, g_ref);
    }
    return hipGetLastError();
}

}  // namespace pmf
