// voxelize.hip -- Eq. 5 (Gaussian voxelization) and its gradient.
//
// Forward: tile-binned.  Each Gaussian's truncation ellipsoid is bounded by
// a box of voxels; Gaussians are binned into the tiles their box overlaps
// (a counting sort).  One workgroup owns a tile.  One-channel sets (the
// reference, ~150 Gaussians per tile) are splatted: the waves lay the
// (Gaussian, column) pairs of batches of the tile's Gaussians over their
// lanes and add into an LDS copy of the tile in fixed point.  Three- and
// nine-channel sets (the MBC bases, ~10 Gaussians per tile) on more than
// VOX_FEW tiles are gathered: each thread owns a few voxels and keeps their
// channel sums in registers.
// Either way the tile is stored once with plain writes -- no global atomics
// -- and the integer sums do not depend on the order in which the binning's
// atomics filled the tile lists.  Gaussians whose box spans more tiles than
// the bin capacity (e.g. untruncated ones) go to a separate list in
// ascending order, which every tile walks after its own list, adding in
// float per voxel in that order.
//
// Backward: Gaussian owner.  A workgroup takes a batch of Gaussians; each of
// its waves walks one's voxel box at a time, accumulates the sums in registers
// and reduces them across the wave; one lane per Gaussian applies the chain rule
// through Sigma = R diag(s^2) R^T and the quaternion normalisation.
#include <math.h>

#include <algorithm>

#include "pmf_internal.h"

namespace pmf {

constexpr int MAXC_VOX = 16;     // channels per Gaussian set (voxelize_workspace checks)

struct alignas(16) GaussK {
    float mu[3];
    float a00;
    float a01, a02, a11, a12;
    float a22;
    int lo0, lo1, lo2;
    int hi0, hi1, hi2;
    uint32_t rim;               // the binning's box: 4 bits per side beyond lo0, hi0, lo1, ...
    int pad;
};

struct GaussFull {
    float mu[3], s[3], qh[4], qn;
    float R[3][3];
    float A[3][3];
    int lo[3], hi[3];           // voxels that may lie inside (none: lo > hi on some axis)
    uint32_t rim;               // GaussK
};

// Rounding allowance of a grid position along axis a, in voxels.
__device__ __forceinline__ float voxel_margin(const GridK &g, int a, float c) {
    return fmaf(1e-6f, fmaf(2.0f * fabsf(g.c0[a]), g.inv_h[a], fabsf(c) + (float)g.n[a]), 0.01f);
}

// Sigma^-1 = R diag(s^-2) R^T and the voxel box of the ellipsoid m <= k^2
// (half-extent k sqrt(Sigma_aa) per axis).  The box holds every voxel whose
// computed m passes m <= k^2: the rounding errors of m and of Sigma_aa are a
// few 2^-24 (s_max / s_min)^2 of k^2, the half-extent is widened by 1e-5
// (s_max / s_min)^2 (an ill-conditioned Gaussian takes its outermost voxels
// plus one).  The tiles' lists, whose lengths and largest values set the scales
// of their fixed-point sums, go by a box of one voxel more on each side
// (`rim`).  Exact boxes and column ranges matter: with one voxel more on
// each side, 200k Gaussians of about 7 x 7 x 5 voxels walked twice the columns
// and three times the voxels (256x256x128: k_vox_tile 243 -> 111 us, k_vox_bwd
// 228 -> 147 us, and 109 with its walks of today).
__device__ __forceinline__ void gauss_full(const float *__restrict__ mean,
                                           const float *__restrict__ scale,
                                           const float *__restrict__ quat, int64_t i, float k,
                                           const GridK &g, GaussFull &G) {
    for (int a = 0; a < 3; ++a) {
        G.mu[a] = mean[3 * i + a];
        G.s[a] = scale[3 * i + a];
    }
    float q[4];
    for (int c = 0; c < 4; ++c) q[c] = quat[4 * i + c];
    const float qn = sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    G.qn = qn;
    for (int c = 0; c < 4; ++c) G.qh[c] = q[c] / qn;
    const float w = G.qh[0], x = G.qh[1], y = G.qh[2], z = G.qh[3];
    G.R[0][0] = 1.0f - 2.0f * (y * y + z * z);
    G.R[0][1] = 2.0f * (x * y - w * z);
    G.R[0][2] = 2.0f * (x * z + w * y);
    G.R[1][0] = 2.0f * (x * y + w * z);
    G.R[1][1] = 1.0f - 2.0f * (x * x + z * z);
    G.R[1][2] = 2.0f * (y * z - w * x);
    G.R[2][0] = 2.0f * (x * z - w * y);
    G.R[2][1] = 2.0f * (y * z + w * x);
    G.R[2][2] = 1.0f - 2.0f * (x * x + y * y);
    float is2[3], s2[3];
    for (int c = 0; c < 3; ++c) {
        s2[c] = G.s[c] * G.s[c];
        is2[c] = 1.0f / s2[c];
    }
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            G.A[a][b] = G.R[a][0] * G.R[b][0] * is2[0] + G.R[a][1] * G.R[b][1] * is2[1] +
                        G.R[a][2] * G.R[b][2] * is2[2];
    const float smax = fmaxf(fmaxf(fabsf(G.s[0]), fabsf(G.s[1])), fabsf(G.s[2]));
    const float smin = fminf(fminf(fabsf(G.s[0]), fabsf(G.s[1])), fabsf(G.s[2]));
    const float widen = fmaf(1e-5f, (smax / smin) * (smax / smin), 1.0f);
    G.rim = 0;
    bool outside = false;
    for (int a = 0; a < 3; ++a) {
        if (isinf(k)) {
            G.lo[a] = 0;
            G.hi[a] = g.n[a] - 1;
            continue;
        }
        const float var = G.R[a][0] * G.R[a][0] * s2[0] + G.R[a][1] * G.R[a][1] * s2[1] +
                          G.R[a][2] * G.R[a][2] * s2[2];
        const float ext = k * sqrtf(var);
        const float c = (G.mu[a] - g.c0[a]) * g.inv_h[a];
        const float we = ext * widen * g.inv_h[a] + voxel_margin(g, a, c);
        const float wl = fmaxf(floorf((G.mu[a] - ext - g.c0[a]) * g.inv_h[a]) - 1.0f, 0.0f);
        const float wu = fminf(ceilf((G.mu[a] + ext - g.c0[a]) * g.inv_h[a]) + 1.0f,
                               (float)(g.n[a] - 1));
        outside = outside || !(wl <= wu);
        // (fmaxf and fminf drop a NaN: then the wide box holds)
        const float l = fminf(fmaxf(ceilf(c - we), wl), wl + 15.0f);
        const float u = fmaxf(fminf(floorf(c + we), wu), wu - 15.0f);
        G.lo[a] = (int)l;
        G.hi[a] = (int)u;
        G.rim |= (uint32_t)(l - wl) << (8 * a) | (uint32_t)(wu - u) << (8 * a + 4);
    }
    if (outside) {
        G.rim = 0;
        for (int a = 0; a < 3; ++a) {
            G.lo[a] = 1;
            G.hi[a] = 0;
        }
    }
}

// Cheap test that Gaussian i's voxel box is empty without building it: the
// ellipsoid's half-extent on any axis is at most k max(s), and the box adds
// one voxel on each side (one more of margin here).  False when unsure
// (untruncated sets, NaN parameters), so callers then build the box.
__device__ __forceinline__ bool far_from_grid(const float *__restrict__ mean,
                                              const float *__restrict__ scale, int64_t i, float k,
                                              const GridK &g) {
    if (isinf(k)) return false;
    const float smax = fmaxf(fmaxf(fabsf(scale[3 * i]), fabsf(scale[3 * i + 1])),
                             fabsf(scale[3 * i + 2]));
    const float ext = 1.001f * k * smax;
    bool far = false;
    for (int a = 0; a < 3; ++a) {
        const float d = mean[3 * i + a] - g.c0[a];
        far = far || d + ext < -3.0f * g.h[a] || d - ext > (float)(g.n[a] + 2) * g.h[a];
    }
    return far;
}

// ---------------------------------------------------------------- binning
// A counting sort of the (Gaussian, tile) pairs by tile.  The set is cut into
// chunks, one workgroup each: k_vox_bin builds the chunk's Gaussians and counts
// its pairs per tile in LDS (an atomic's old value is the pair's place among
// the chunk's), k_vox_chunks turns the chunks' counts of a tile into places
// and totals, and k_vox_fill scans the totals and writes each pair to its
// place.  (Counting in global memory took a device-scope atomic per pair, which
// contend per cache line: 100 + 19 us of 150 for the 200k set, and eight
// launches; now three and 48 us.)  Counts are held for BIN_W tiles; a grid of
// more has a workgroup per chunk and window of them (grid dimension y), and
// k_vox_chunks adds up the windows' totals.  (Windows walked one after the
// other by the chunk's workgroup, few chunks where tiles are many: 2.5 ms for
// 200k Gaussians in 1024x1024x800, 34 windows, now 0.36.)
struct VoxTiles {                      // a set's tiles and chunks
    int T0, T1, T2, nt1, nt2, ntiles;
    int maxtiles;                      // more tiles than this: a large Gaussian
    int64_t chunk;                     // Gaussians per chunk
};

constexpr int BIN_W = 12288;           // tiles per window (48 KB of LDS)
constexpr int BIN_T = 512;             // threads per chunk

// A Gaussian's tile box [t*a, t*b], of its voxel box and rim; the pairs are numbered
// q = 0.. with axis 2 fastest.
struct TileBox {
    int a0, b0, a1, b1, a2, b2;
    int64_t count;                     // 0: no voxel
};
__device__ __forceinline__ TileBox tile_box(const GaussK &r, int T0, int T1, int T2) {
    TileBox t{};
    const int lo0 = r.lo0 - (int)(r.rim & 15), hi0 = r.hi0 + (int)(r.rim >> 4 & 15);
    const int lo1 = r.lo1 - (int)(r.rim >> 8 & 15), hi1 = r.hi1 + (int)(r.rim >> 12 & 15);
    const int lo2 = r.lo2 - (int)(r.rim >> 16 & 15), hi2 = r.hi2 + (int)(r.rim >> 20 & 15);
    if (lo0 > hi0 || lo1 > hi1 || lo2 > hi2) return t;
    t.a0 = lo0 / T0;
    t.b0 = hi0 / T0;
    t.a1 = lo1 / T1;
    t.b1 = hi1 / T1;
    t.a2 = lo2 / T2;
    t.b2 = hi2 / T2;
    t.count = (int64_t)(t.b0 - t.a0 + 1) * (t.b1 - t.a1 + 1) * (t.b2 - t.a2 + 1);
    return t;
}

// Calls f(tile - w0, q) for the box's pairs with a tile in [w0, w0 + BIN_W).
template <class F>
__device__ __forceinline__ void each_pair(const TileBox &t, const VoxTiles &p, int w0, F &&f) {
    int q = 0;
    for (int a = t.a0; a <= t.b0; ++a)
        for (int b = t.a1; b <= t.b1; ++b)
            for (int c = t.a2; c <= t.b2; ++c, ++q) {
                const int w = (a * p.nt1 + b) * p.nt2 + c - w0;
                if (w >= 0 && w < BIN_W) f(w, q);
            }
}

// Windows win0 + blockIdx.y; the first builds the records that the others read.
// (COUNT = false: the records and the large Gaussians only.)
template <bool COUNT>
__global__ __launch_bounds__(BIN_T) void k_vox_bin(pmf_gauss_t gs, GridK g, float k, VoxTiles p,
                                                   GaussK *__restrict__ rec,
                                                   int32_t *__restrict__ part,
                                                   int32_t *__restrict__ slot,
                                                   int32_t *__restrict__ nlarge, int win0,
                                                   int32_t *__restrict__ wtotal) {
    extern __shared__ int32_t hist[];
    __shared__ int32_t nl;
    const int64_t i0 = (int64_t)blockIdx.x * p.chunk, i1 = min(i0 + p.chunk, gs.m);
    int32_t *const row = part + (int64_t)blockIdx.x * p.ntiles;
    const int win = win0 + (int)blockIdx.y, w0 = win * BIN_W;
    const int nw = min(BIN_W, p.ntiles - w0);
    if (threadIdx.x == 0) {
        nl = 0;
        if (COUNT && blockIdx.x == 0) wtotal[win] = 0;
    }
    if (COUNT)
        for (int t = threadIdx.x; t < nw; t += BIN_T) hist[t] = 0;
    __syncthreads();
    for (int64_t i = i0 + threadIdx.x; i < i1; i += BIN_T) {
        GaussK r = {};
        if (win > 0) {
            r = rec[i];                           // an earlier launch's
        } else {
            if (far_from_grid(gs.mean, gs.scale, i, k, g)) {
                r.lo0 = r.lo1 = r.lo2 = 1;        // empty box: no tile, no voxel
            } else {
                GaussFull G;
                gauss_full(gs.mean, gs.scale, gs.quat, i, k, g, G);
                for (int a = 0; a < 3; ++a) r.mu[a] = G.mu[a];
                r.a00 = G.A[0][0];
                r.a01 = G.A[0][1];
                r.a02 = G.A[0][2];
                r.a11 = G.A[1][1];
                r.a12 = G.A[1][2];
                r.a22 = G.A[2][2];
                r.lo0 = G.lo[0];
                r.lo1 = G.lo[1];
                r.lo2 = G.lo[2];
                r.hi0 = G.hi[0];
                r.hi1 = G.hi[1];
                r.hi2 = G.hi[2];
                r.rim = G.rim;
            }
            rec[i] = r;
        }
        const TileBox t = tile_box(r, p.T0, p.T1, p.T2);
        if (t.count > p.maxtiles) {
            if (win == 0) atomicAdd(&nl, 1);
        } else if (COUNT && t.count > 0) {
            each_pair(t, p, w0, [&](int w, int q) {
                slot[(int64_t)q * gs.m + i] = atomicAdd(&hist[w], 1);
            });
        }
    }
    __syncthreads();
    if (COUNT)
        for (int t = threadIdx.x; t < nw; t += BIN_T) row[w0 + t] = hist[t];
    if (win == 0 && threadIdx.x == 0) nlarge[1 + blockIdx.x] = nl;
}

// Per tile: the chunks' counts -> the places of their first pairs in the tile's
// list, in place, and the tile's total.  A workgroup takes 64 tiles (a lane
// each), its sixteen waves a sixteenth of the chunks each.  With several windows
// their totals are added up too.
__global__ __launch_bounds__(1024) void k_vox_chunks(int32_t *__restrict__ part, int ntiles, int nch,
                                                    int32_t *__restrict__ total,
                                                    int32_t *__restrict__ wtotal) {
    __shared__ int32_t sums[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = blockIdx.x * 64 + lane;
    const int per = (nch + 15) / 16, c0 = min(w * per, nch), c1 = min(c0 + per, nch);
    int32_t s = 0;
    if (t < ntiles) {
#pragma unroll 8
        for (int c = c0; c < c1; ++c) s += part[(int64_t)c * ntiles + t];
    }
    sums[w][lane] = s;
    __syncthreads();
    if (w == 0 && ntiles > BIN_W) {
        static_assert(BIN_W % 64 == 0, "a workgroup's tiles lie in one window");
        int32_t all = 0;
        for (int k = 0; k < 16; ++k) all += sums[k][lane];
        for (int o = 32; o > 0; o >>= 1) all += __shfl_xor(all, o, 64);
        if (lane == 0) atomicAdd(&wtotal[(int)blockIdx.x * 64 / BIN_W], all);
    }
    if (t >= ntiles) return;
    int32_t run = 0;
    for (int k = 0; k < w; ++k) run += sums[k][lane];
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
        const int32_t x = part[(int64_t)c * ntiles + t];
        part[(int64_t)c * ntiles + t] = run;
        run += x;
    }
    if (w == 15) total[t] = run;
}

// Exclusive scan of v over the workgroup (BIN_T threads), the sum added to carry.
__device__ __forceinline__ int32_t block_excl_sum(int32_t v, int32_t *wsum, int32_t &carry) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t incl = wave_incl_sum(v);
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int32_t base = carry, sum = 0;
#pragma unroll
    for (int k = 0; k < BIN_T / 64; ++k) {
        if (k < w) base += wsum[k];
        sum += wsum[k];
    }
    carry += sum;
    __syncthreads();
    return base + incl - v;
}

// Each chunk scans the tiles' totals (the first one stores them as the lists'
// offsets) and writes its pairs to their places, and its large Gaussians, in
// ascending order, to the large list.
// With SHORT it also sums the chunks' counts itself: up to BIN_SHORT (chunk,
// tile) counts of one window that costs less than k_vox_chunks' launch.
constexpr int BIN_SHORT = 1 << 14;

template <bool SHORT>
__global__ __launch_bounds__(BIN_T) void k_vox_fill(int64_t m, const GaussK *__restrict__ rec,
                                                    VoxTiles p, const int32_t *__restrict__ part,
                                                    const int32_t *__restrict__ total,
                                                    const int32_t *__restrict__ slot,
                                                    int32_t *__restrict__ nlarge,
                                                    const int32_t *__restrict__ wtotal,
                                                    int32_t *__restrict__ off,
                                                    int32_t *__restrict__ list,
                                                    int32_t *__restrict__ large) {
    extern __shared__ int32_t base[];
    __shared__ int32_t wsum[BIN_T / 64];
    const int64_t i0 = (int64_t)blockIdx.x * p.chunk, i1 = min(i0 + p.chunk, m);
    const int32_t *const row = part + (int64_t)blockIdx.x * p.ntiles;
    const bool first = blockIdx.x == 0;
    const int w0 = (int)blockIdx.y * BIN_W, nw = min(BIN_W, p.ntiles - w0);
    int32_t carry = 0;
    for (int k = 0; k < (int)blockIdx.y; ++k) carry += wtotal[k];
    for (int t0 = 0; SHORT && t0 < nw; t0 += BIN_T) {
        const int t = t0 + (int)threadIdx.x;
        int32_t all = 0, before = 0;
        if (t < nw) {
#pragma unroll 8
            for (int c = 0; c < (int)gridDim.x; ++c) {
                const int32_t x = part[(int64_t)c * p.ntiles + t];
                all += x;
                before += c < (int)blockIdx.x ? x : 0;
            }
        }
        const int32_t o = block_excl_sum(all, wsum, carry);
        if (t < nw) {
            if (first) off[t] = o;
            base[t] = o + before;
        }
    }
    for (int t0 = 0; !SHORT && t0 < nw; t0 += 4 * BIN_T) {
        // four neighbouring tiles per thread
        const int t = t0 + 4 * (int)threadIdx.x;
        int32_t v[4], s = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = t + k < nw ? total[w0 + t + k] : 0;
            s += v[k];
        }
        int32_t o = block_excl_sum(s, wsum, carry);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (t + k < nw) {
                if (first) off[w0 + t + k] = o;
                base[t + k] = o + row[w0 + t + k];
                o += v[k];
            }
    }
    __syncthreads();
    for (int64_t i = i0 + threadIdx.x; i < i1; i += BIN_T) {
        const TileBox t = tile_box(rec[i], p.T0, p.T1, p.T2);
        if (t.count == 0 || t.count > p.maxtiles) continue;
        each_pair(t, p, w0, [&](int w, int q) {
            list[base[w] + slot[(int64_t)q * m + i]] = (int32_t)i;
        });
    }
    __syncthreads();
    if (first && w0 + nw == p.ntiles && threadIdx.x == 0) off[p.ntiles] = carry;
    if (blockIdx.y > 0) return;
    // the large list: this chunk's place in it, then its entries by ballots
    int32_t before = 0, all = 0;
    for (int c0 = 0; c0 < (int)gridDim.x; c0 += BIN_T) {
        const int c = c0 + (int)threadIdx.x;
        const int32_t x = c < (int)gridDim.x ? nlarge[1 + c] : 0;
        const int32_t e = block_excl_sum(x, wsum, all);
        if (c == (int)blockIdx.x) base[0] = e;      // the pairs are written: base is free
    }
    __syncthreads();
    before = base[0];
    if (first && threadIdx.x == 0) nlarge[0] = all;
    if (nlarge[1 + blockIdx.x] == 0) return;
    for (int64_t j0 = i0; j0 < i1; j0 += BIN_T) {
        const int64_t i = j0 + threadIdx.x;
        const bool f = i < i1 && tile_box(rec[i], p.T0, p.T1, p.T2).count > p.maxtiles;
        const int32_t e = block_excl_sum(f ? 1 : 0, wsum, before);
        if (f) large[e] = (int32_t)i;
    }
}

// ------------------------------------------------------------ tile splat
// On a column (d0, d1 fixed) the quadratic form is m(d2) = a22 d2^2 + b2 d2
// + cq; the forward and the adjoint evaluate it in this form, so both take
// the same mask decisions.
__device__ __forceinline__ void col_coeffs(float a00, float a01, float a02, float a11, float a12,
                                           float d0, float d1, float &b2, float &cq) {
    b2 = 2.0f * fmaf(a02, d0, a12 * d1);
    cq = fmaf(a00 * d0, d0, fmaf(2.0f * a01 * d0, d1, a11 * d1 * d1));
}

// e^(-m/2).  (-log2(e) / 2 rounds to half of log2(e)'s float: the product is
// that of e^x's own.)
__device__ __forceinline__ float half_exp(float m) {
    return __builtin_amdgcn_exp2f(-0.72134752044f * m);
}

__device__ __forceinline__ float col_quad(float a22, float b2, float cq, float d2) {
    return fmaf(fmaf(a22, d2, b2), d2, cq);
}

// z range [za, zb] of a column that the truncation ellipsoid m <= k2 can
// reach, clipped to [lo2, hi2]; false when the column's quadratic stays above
// k2.  The range holds every voxel whose computed col_quad passes m <= k2: with
// u = -b2 / (2 a22) the roots are u +- sqrt(disc), the rounding errors of
// col_quad and of disc are below 1e-6 of u^2 + (|cq| + k2) / a22, and disc is
// raised by 1e-4 of that.  zc: the Gaussian's centre in voxels; zm: the margin
// of a voxel's position.  Untruncated sets take the whole range.
__device__ __forceinline__ bool col_range(float a22, float b2, float cq, float zc, float zm,
                                          float inv_h2, float k2, bool untrunc, int lo2, int hi2,
                                          int &za, int &zb) {
    za = lo2;
    zb = hi2;
    if (untrunc) return true;
    const float ra = __builtin_amdgcn_rcpf(a22);
    const float u = -0.5f * b2 * ra;
    const float bound = fmaf(u, u, (fabsf(cq) + k2) * ra);
    const float disc = fmaf(1e-4f, bound, fmaf(u, u, (k2 - cq) * ra));
    if (disc < 0.0f) return false;
    const float r = __builtin_amdgcn_sqrtf(disc);
    // (fmaxf and fminf drop a NaN: then the box's bound holds)
    za = (int)fmaxf(ceilf(fmaf(u - r, inv_h2, zc - zm)), (float)lo2);
    zb = (int)fminf(floorf(fmaf(u + r, inv_h2, zc + zm)), (float)hi2);
    return za <= zb;
}

// One workgroup per tile.  Accumulation is in 32-bit fixed point with
// integer LDS atomics, so the sums do not depend on their order: per channel
// the scale is 2^30 / S with S = (Gaussians reaching the tile) x (their
// largest |value|), which bounds every voxel's sum since each Gaussian adds
// value * e (e <= 1) at most once per voxel, and is itself independent of
// the list's order.
//
// Work layout: each wave takes batches of up to VB of the tile's Gaussians
// (lane j < VB reads batch entry j, clips its box to the tile and stages it
// in LDS), then lays the batch's (Gaussian, column) pairs out over its
// lanes, 64 at a time: a lane finds its pair by a search over the batch's
// column offsets, walks the column's z range (col_range: nearly every voxel
// it visits is inside the ellipsoid) and adds value x e^(-m/2) of each
// in-mask voxel.  The lanes are spread over the columns of many Gaussians,
// not one Gaussian's few.
//
// NW waves per workgroup: 4, or 16 (in smaller batches) where the grid has so
// few tiles that each tile's list is a long serial walk (VOX_FEW).
struct VoxB {                 // one Gaussian of a wave's batch, box clipped to the tile
    float mu[3];
    float a00, a01, a02, a11, a12, a22;
    int lo0, lo1, lo2, hi2, ny, cend;    // its columns are [cend - ncols, cend)
    int ncols;
};

// Workgroup b runs on XCD b % 8, and with a power of two of tiles along axis 2
// that would give each XCD the tiles of one axis-2 slab (and the middle slabs
// of a body hold most of the Gaussians: CUs were busy 59% of the time, 73%
// now), so the axis-2 tile index is rotated from column to column.
__device__ __forceinline__ int rotated_tile(int b, int nt1, int nt2) {
    const int c = b / nt2, z = b - c * nt2;
    const int tx = c / nt1, ty = c - tx * nt1;
    return c * nt2 + (z + tx + ty / 2) % nt2;
}

// SCAN: a small set on few tiles has no lists; each workgroup finds its tile's
// Gaussians among all of them (nlarge then holds the chunks' counts of large
// ones behind its first word), which costs less than the launch that would write
// the lists.  Every tile reads every record, so the line falls with the tiles:
// up to VOX_SCAN (a tile's list in 16 KB of LDS) on one tile per CU, 1,000 on
// more.  Whole call, lists / search: 32^3 (64 tiles) 1,000 Gaussians 27 / 17 us,
// 4,096 35 / 27; 64^3 (256) 24 / 18 at 4,096 (12,000 34 / 33 with 64 KB); 128x128x64
// (512) 500 25 / 19, 1,000 25 / 21, 2,000 26 / 25, 4,096 26 / 30, three channels 500
// 27 / 26, 1,000 28 / 29, 4,096 30 / 38.
constexpr int VOX_SCAN = 4096;
constexpr int VOX_SCAN_MANY = 1000;

template <int T0, int T1, int T2, int CT, int NW, int VB, bool SCAN>
__global__ __launch_bounds__(64 * NW, 8) void k_vox_tile(const GaussK *__restrict__ rec, int m, int nch,
                                                  int maxtiles,
                                                  const float *__restrict__ value, int Crt, GridK g,
                                                  float k2, int nt1, int nt2,
                                                  const int32_t *__restrict__ off,
                                                  const int32_t *__restrict__ list,
                                                  const int32_t *__restrict__ large,
                                                  const int32_t *__restrict__ nlarge,
                                                  float *__restrict__ vol) {
    constexpr int TV = T0 * T1 * T2;
    constexpr int NT = 64 * NW;
    constexpr int CM = CT > 0 ? CT : MAXC_VOX;
    const int C = CT > 0 ? CT : Crt;
    extern __shared__ int acc[];          // C tile planes
    __shared__ float cs[NW][CM];
    __shared__ float scale[CM];
    __shared__ VoxB bt[NW][VB];
    __shared__ float bv[NW][VB][CM];      // value x scale per batch entry
    __shared__ int32_t slist[SCAN ? VOX_SCAN : 1];
    __shared__ int scount[NW];            // [0]: Gaussians found
    for (int i = threadIdx.x; i < C * TV; i += NT) acc[i] = 0;
    const int t = rotated_tile((int)blockIdx.x, nt1, nt2);
    const int tz = t % nt2, ty = (t / nt2) % nt1, tx = t / (nt2 * nt1);
    const int b0 = tx * T0, b1 = ty * T1, b2 = tz * T2;
    const int e0 = min(b0 + T0, g.n[0]) - 1, e1 = min(b1 + T1, g.n[1]) - 1,
              e2 = min(b2 + T2, g.n[2]) - 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int beg, end, nl = 0;
    if constexpr (SCAN) {
        if (threadIdx.x == 0) scount[0] = 0;
        __syncthreads();
        for (int i0 = wave * 64; i0 < m; i0 += NT) {                  // uniform
            bool in = false;
            if (i0 + lane < m) {
                const TileBox q = tile_box(rec[i0 + lane], T0, T1, T2);
                in = q.count > 0 && q.count <= maxtiles && q.a0 <= tx && tx <= q.b0 &&
                     q.a1 <= ty && ty <= q.b1 && q.a2 <= tz && tz <= q.b2;
            }
            const uint64_t hits = __ballot(in);
            if (hits == 0) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(&scount[0], __popcll(hits));
            at = __builtin_amdgcn_readfirstlane(at);
            if (in) slist[at + __popcll(hits & ((1ull << lane) - 1))] = i0 + lane;
        }
        for (int c = 0; c < nch; ++c) nl += nlarge[1 + c];
        __syncthreads();
        beg = 0;
        end = scount[0];
    } else {
        beg = off[t];
        end = off[t + 1];
        nl = *nlarge;
    }
    auto entry = [&](int e) { return SCAN ? slist[e] : list[e]; };
    // per-channel bound S = (the tile's list length) x (the list's largest
    // |value|): every voxel's sum stays below it, and unlike a float sum of
    // the |values| it does not depend on the order the binning's atomics gave
    // the list, so neither does the scale (results repeat bit for bit)
    for (int c = 0; c < C; ++c) {
        float mx = 0.0f;
        for (int e = beg + (int)threadIdx.x; e < end; e += NT)
            mx = fmaxf(mx, fabsf(value[(int64_t)entry(e) * C + c]));
        mx = wave_max(mx);
        if (lane == 0) cs[wave][c] = mx;
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)C) {
        float mx = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) mx = fmaxf(mx, cs[w][threadIdx.x]);
        const float S = (float)(end - beg) * mx;
        scale[threadIdx.x] = S > 0.0f ? 1073741824.0f / (S * 1.0001f) : 0.0f;
    }
    __syncthreads();
    const bool untrunc = isinf(k2);
    const float inv_h2 = g.inv_h[2];
    const float h2 = in_vgpr(g.h[2]), o2 = in_vgpr(g.c0[2]), kk = in_vgpr(k2);
    VoxB *const B = bt[wave];
    for (int eb = beg + wave * VB; eb < end; eb += NW * VB) {     // uniform per wave
        const int nb = min(VB, end - eb);
        int ncols = 0;
        VoxB q;
        if (lane < nb) {
            const int gi = entry(eb + lane);
            const GaussK p = rec[gi];
            const int lo0 = max(p.lo0, b0), lo1 = max(p.lo1, b1), lo2 = max(p.lo2, b2);
            const int hi0 = min(p.hi0, e0), hi1 = min(p.hi1, e1), hi2 = min(p.hi2, e2);
            if (lo0 <= hi0 && lo1 <= hi1 && lo2 <= hi2) ncols = (hi0 - lo0 + 1) * (hi1 - lo1 + 1);
            for (int a = 0; a < 3; ++a) q.mu[a] = p.mu[a];
            q.a00 = p.a00;
            q.a01 = p.a01;
            q.a02 = p.a02;
            q.a11 = p.a11;
            q.a12 = p.a12;
            q.a22 = p.a22;
            q.lo0 = lo0;
            q.lo1 = lo1;
            q.lo2 = lo2;
            q.hi2 = hi2;
            q.ny = hi1 - lo1 + 1;
            q.ncols = ncols;
            const float *vv = value + (int64_t)gi * C;
            for (int c = 0; c < C; ++c) bv[wave][lane][c] = vv[c] * scale[c];
        }
        const int cend = wave_incl_sum(ncols);          // lanes >= nb add 0
        const int total = __builtin_amdgcn_readlane(cend, VB - 1);
        if (lane < nb) {
            q.cend = cend;
            B[lane] = q;
        } else if (lane < VB) {          // the search reads every entry's cend
            B[lane].cend = cend;
            B[lane].ncols = 0;
        }
        wave_lds_sync();
        for (int cb = 0; cb < total; cb += 64) {           // uniform per wave
            const int qc = cb + lane;
            if (qc >= total) continue;
            // batch entry: the smallest j with cend_j > qc
            int j = 0;
#pragma unroll
            for (int step = VB / 2; step > 0; step >>= 1)
                if (B[j + step - 1].cend <= qc) j += step;
            const VoxB &q = B[j];
            const int ql = qc - (q.cend - q.ncols);
            // column ql of the clipped box, y fastest (exact: ql < 256, ny <= 16)
            const int cx = (int)(((float)ql + 0.5f) * __builtin_amdgcn_rcpf((float)q.ny));
            const int ix = q.lo0 + cx, iy = q.lo1 + (ql - cx * q.ny);
            const float d0 = fmaf((float)ix, g.h[0], g.c0[0]) - q.mu[0];
            const float d1 = fmaf((float)iy, g.h[1], g.c0[1]) - q.mu[1];
            float cb2, cq;
            col_coeffs(q.a00, q.a01, q.a02, q.a11, q.a12, d0, d1, cb2, cq);
            int za, zb;
            const float zc = (q.mu[2] - g.c0[2]) * inv_h2;
            if (!col_range(q.a22, cb2, cq, zc, voxel_margin(g, 2, zc), inv_h2, k2, untrunc, q.lo2,
                           q.hi2, za, zb))
                continue;
            const float a22 = q.a22, mu2 = q.mu[2];
            float vs[CM];
#pragma unroll
            for (int c = 0; c < CM; ++c) vs[c] = c < C ? bv[wave][j][c] : 0.0f;
            int li = ((ix - b0) * T1 + (iy - b1)) * T2 + (za - b2);
            float fz = (float)za;
            for (int n = zb - za; n >= 0; --n, ++li, fz += 1.0f) {
                const float d2 = fmaf(fz, h2, o2) - mu2;
                const float mm = col_quad(a22, cb2, cq, d2);
                if (!(mm <= kk)) continue;
                const float ev = half_exp(mm);
#pragma unroll
                for (int c = 0; c < CM; ++c)
                    if (c < C) atomicAdd(&acc[c * TV + li], __float2int_rn(vs[c] * ev));
            }
        }
        wave_lds_sync();
    }
    __syncthreads();
    // fixed point -> float, in place
    float *const accf = (float *)acc;
    for (int i = threadIdx.x; i < C * TV; i += NT) {
        const float sc = scale[i / TV];
        accf[i] = sc > 0.0f ? (float)acc[i] / sc : 0.0f;
    }
    // Gaussians too large for the bins (e.g. untruncated sets): each thread
    // owns voxels of the tile and adds them in float, in the list's ascending
    // order (a fixed order: the results repeat bit for bit)
    if (nl > 0) {
        __syncthreads();
        if constexpr (SCAN) {
            // their list, in ascending order, in the found ones' place
            int n = 0;
            for (int i0 = 0; i0 < m; i0 += NT) {                      // uniform
                const int i = i0 + (int)threadIdx.x;
                const bool f = i < m && tile_box(rec[i], T0, T1, T2).count > maxtiles;
                const uint64_t hits = __ballot(f);
                if (lane == 0) scount[wave] = __popcll(hits);
                __syncthreads();
                int at = n;
                for (int w = 0; w < NW; ++w) {
                    if (w < wave) at += scount[w];
                    n += scount[w];
                }
                if (f) slist[at + __popcll(hits & ((1ull << lane) - 1))] = i;
                __syncthreads();
            }
        }
        // 64 at a time, those that reach the tile in the batches' LDS, their boxes' hi0 and hi1 in place of
        // ncols and ny (one record after the other, from global memory: 300
        // Gaussians of s = 12 in 128x128x64, three channels, 314 us, now 88)
        constexpr int K = TV > NT ? TV / NT : 1;       // a thread's voxels, along axis 2
        static_assert(T2 % K == 0, "a thread's voxels lie in one column");
        static_assert(NW * VB >= 64 && TV % (64 * K) == 0, "a wave's entries; whole waves of voxels");
        constexpr int LU = K > 2 ? 1 : 4;
        VoxB *const lb = bt[0];
        float(*const lv)[CM] = bv[0];
        const int li = (int)threadIdx.x * K;
        const int ix = b0 + li / (T1 * T2), iy = b1 + (li / T2) % T1, iz = b2 + li % T2;
        const bool on = li < TV && ix <= e0 && iy <= e1;
        const float d0g = fmaf((float)ix, g.h[0], g.c0[0]);
        const float d1g = fmaf((float)iy, g.h[1], g.c0[1]);
        float d2g[K], out[K][CT > 0 ? CT : 1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            d2g[k] = fmaf((float)(iz + k), g.h[2], g.c0[2]);
#pragma unroll
            for (int c = 0; c < CT; ++c) out[k][c] = on ? accf[c * TV + li + k] : 0.0f;
        }
        for (int f = 0; f < nl; f += 64) {                            // uniform
            __syncthreads();              // slist is there, the entries before are used
            if (wave == 0) {              // those that reach the tile, in order
                bool hit = false;
                GaussK p = {};
                int gi = 0;
                if (f + lane < nl) {
                    gi = SCAN ? slist[f + lane] : large[f + lane];
                    p = rec[gi];
                    hit = max(p.lo0, b0) <= min(p.hi0, e0) && max(p.lo1, b1) <= min(p.hi1, e1) &&
                          max(p.lo2, b2) <= min(p.hi2, e2);
                }
                const uint64_t hits = __ballot(hit);
                if (hit) {
                    const int j = __popcll(hits & ((1ull << lane) - 1));
                    VoxB q;
                    for (int a = 0; a < 3; ++a) q.mu[a] = p.mu[a];
                    q.a00 = p.a00;
                    q.a01 = p.a01;
                    q.a02 = p.a02;
                    q.a11 = p.a11;
                    q.a12 = p.a12;
                    q.a22 = p.a22;
                    q.lo0 = p.lo0;
                    q.lo1 = p.lo1;
                    q.lo2 = p.lo2;
                    q.hi2 = p.hi2;
                    q.ny = p.hi1;
                    q.ncols = p.hi0;
                    q.cend = 0;
                    lb[j] = q;
                    for (int c = 0; c < C; ++c) lv[j][c] = value[(int64_t)gi * C + c];
                }
                if (lane == 0) scount[0] = __popcll(hits);
            }
            __syncthreads();
            const int n = scount[0];
            // (without branches, so that several entries' reads are in flight)
#pragma unroll LU
            for (int e = 0; wave * 64 * K < TV && e < n; ++e) {      // uniform
                const VoxB p = lb[e];
                float cb2, cq;
                col_coeffs(p.a00, p.a01, p.a02, p.a11, p.a12, d0g - p.mu[0], d1g - p.mu[1], cb2, cq);
                const bool col = ix >= p.lo0 && ix <= p.ncols && iy >= p.lo1 && iy <= p.ny;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float mm = col_quad(p.a22, cb2, cq, d2g[k] - p.mu[2]);
                    const bool in = col && iz + k >= p.lo2 && iz + k <= p.hi2 && mm <= k2;
                    const float ev = half_exp(mm);
                    if constexpr (CT > 0) {
#pragma unroll
                        for (int c = 0; c < CT; ++c) {
                            const float t = fmaf(lv[e][c], ev, out[k][c]);
                            out[k][c] = in ? t : out[k][c];
                        }
                    } else if (on && in) {
                        for (int c = 0; c < C; ++c) accf[c * TV + li + k] += lv[e][c] * ev;
                    }
                }
            }
        }
        if (on)
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int c = 0; c < CT; ++c) accf[c * TV + li + k] = out[k][c];
    }
    __syncthreads();
    const int64_t N = grid_size(g);
    for (int i = threadIdx.x; i < C * TV; i += NT) {
        const int c = i / TV, li = i % TV;
        const int z = li % T2, y = (li / T2) % T1, x = li / (T2 * T1);
        const int gx = b0 + x, gy = b1 + y, gz = b2 + z;
        if (gx < g.n[0] && gy < g.n[1] && gz < g.n[2])
            vol[(int64_t)c * N + ((int64_t)gx * g.n[1] + gy) * g.n[2] + gz] = accf[i];
    }
}

// Multi-channel sets (the MBC bases: few Gaussians per tile, 3 or 9
// channels): voxel owners.  A thread owns SEG consecutive voxels of one
// column of the tile and keeps their channel sums in registers, in the same
// 32-bit fixed point and with the same per-term rounding as k_vox_tile (so
// the two give the same bits, and the sums do not depend on the order of the
// tile's list); the tile's Gaussians are staged in LDS a chunk at a time and
// every thread tests each against its voxels.  No LDS accumulator, no
// atomics: the kernel holds little LDS and keeps many tiles in flight (six per
// CU; at 256x256x128, 16k Gaussians of nine channels, 110 us with five and divisions, 90
// with six, 121 with seven, which spill; its 302 MB take 63 at the copy rate).
constexpr int VG_CHUNK = 64;

template <int T0, int T1, int T2, int CT>
__global__ __launch_bounds__(256, 6) void k_vox_gather(const GaussK *__restrict__ rec,
                                                   const float *__restrict__ value, GridK g,
                                                   float k2, int nt1, int nt2,
                                                   const int32_t *__restrict__ off,
                                                   const int32_t *__restrict__ list,
                                                   const int32_t *__restrict__ large,
                                                   const int32_t *__restrict__ nlarge,
                                                   float *__restrict__ vol) {
    constexpr int TV = T0 * T1 * T2;
    constexpr int NT = 256;
    constexpr int SEG = TV / NT;            // voxels per thread (along z)
    constexpr int NS = T2 / SEG;            // threads per column
    constexpr int NW = NT / 64;
    static_assert(SEG >= 1 && T2 % SEG == 0 && TV % NT == 0, "tile shape");
    __shared__ GaussK gsh[VG_CHUNK];
    __shared__ float gvs[VG_CHUNK][CT];
    __shared__ int nsh;
    __shared__ float cs[NW][CT];
    __shared__ float scale[CT];
    const int t = rotated_tile((int)blockIdx.x, nt1, nt2);
    const int tz = t % nt2, ty = (t / nt2) % nt1, tx = t / (nt2 * nt1);
    const int b0 = tx * T0, b1 = ty * T1, b2 = tz * T2;
    const int e0 = min(b0 + T0, g.n[0]) - 1, e1 = min(b1 + T1, g.n[1]) - 1,
              e2 = min(b2 + T2, g.n[2]) - 1;
    const int beg = off[t], end = off[t + 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int seg = threadIdx.x % NS, col = threadIdx.x / NS;
    const int ix = b0 + col / T1, iy = b1 + col % T1, z0 = b2 + seg * SEG;
    // x range of the wave's columns (a wave-uniform cull of each Gaussian)
    const int wx0 = b0 + (wave * 64 / NS) / T1, wx1 = b0 + ((wave * 64 + 63) / NS) / T1;
    // lane's entry of a chunk, staged in LDS if it has voxels in the tile (one wave)
    auto stage = [&](bool on, const GaussK &p, const float (&v)[CT]) {
        const bool hit = on && max(p.lo0, b0) <= min(p.hi0, e0) &&
                         max(p.lo1, b1) <= min(p.hi1, e1) && max(p.lo2, b2) <= min(p.hi2, e2);
        const uint64_t hits = __ballot(hit);
        if (hit) {
            const int j = __popcll(hits & ((1ull << lane) - 1));
            gsh[j] = p;
#pragma unroll
            for (int c = 0; c < CT; ++c) gvs[j][c] = v[c];
        }
        if (lane == 0) nsh = __popcll(hits);
    };
    auto scale_of = [&](float mx) {
        const float S = (float)(end - beg) * mx;
        return S > 0.0f ? 1073741824.0f / (S * 1.0001f) : 0.0f;
    };
    // A list of one chunk (the usual case) is read once, by one wave: its
    // largest values and its staging need no second chain of loads.
    const bool one = end - beg <= VG_CHUNK;                       // uniform
    if (one) {
        if (wave == 0) {
            const bool on = beg + lane < end;
            GaussK p = {};
            float v[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) v[c] = 0.0f;
            if (on) {
                const int gi = list[beg + lane];
#pragma unroll
                for (int c = 0; c < CT; ++c) v[c] = value[(int64_t)gi * CT + c];
                p = rec[gi];
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const float sc = scale_of(wave_max(fabsf(v[c])));
                v[c] *= sc;
                if (lane == 0) scale[c] = sc;
            }
            stage(on, p, v);
        }
    } else {
        // one pass over the list: each entry's channels load together
        float mx[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) mx[c] = 0.0f;
        for (int e = beg + (int)threadIdx.x; e < end; e += NT) {
            const float *vv = value + (int64_t)list[e] * CT;
#pragma unroll
            for (int c = 0; c < CT; ++c) mx[c] = fmaxf(mx[c], fabsf(vv[c]));
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float m = wave_max(mx[c]);
            if (lane == 0) cs[wave][c] = m;
        }
        __syncthreads();
        if (threadIdx.x < (unsigned)CT) {
            float m = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) m = fmaxf(m, cs[w][threadIdx.x]);
            scale[threadIdx.x] = scale_of(m);
        }
    }
    const float d0g = fmaf((float)ix, g.h[0], g.c0[0]);
    const float d1g = fmaf((float)iy, g.h[1], g.c0[1]);
    float d2g[SEG];
#pragma unroll
    for (int s = 0; s < SEG; ++s) d2g[s] = fmaf((float)(z0 + s), g.h[2], g.c0[2]);
    int acc[SEG][CT];
#pragma unroll
    for (int s = 0; s < SEG; ++s)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[s][c] = 0;
    __syncthreads();                      // scale and, of one chunk, the staged entries are there
    for (int cb = beg; cb < end; cb += VG_CHUNK) {
        if (!one) {
            if (cb > beg) __syncthreads();        // the previous chunk is consumed
            if (wave == 0) {
                const bool on = cb + lane < end;
                const int gi = list[on ? cb + lane : cb];
                float v[CT];
#pragma unroll
                for (int c = 0; c < CT; ++c) v[c] = value[(int64_t)gi * CT + c] * scale[c];
                const GaussK p = rec[gi];
                stage(on, p, v);
            }
            __syncthreads();
        }
        const int n = nsh;
        for (int e = 0; e < n; ++e) {
            const GaussK p = gsh[e];
            if (p.hi0 < wx0 || p.lo0 > wx1) continue;         // uniform
            if (ix < p.lo0 || ix > p.hi0 || iy < p.lo1 || iy > p.hi1 || z0 > p.hi2 ||
                z0 + SEG - 1 < p.lo2)
                continue;
            float cb2, cq;
            col_coeffs(p.a00, p.a01, p.a02, p.a11, p.a12, d0g - p.mu[0], d1g - p.mu[1], cb2, cq);
#pragma unroll
            for (int s = 0; s < SEG; ++s) {
                const float mm = col_quad(p.a22, cb2, cq, d2g[s] - p.mu[2]);
                if (z0 + s >= p.lo2 && z0 + s <= p.hi2 && mm <= k2) {
                    const float ev = half_exp(mm);
#pragma unroll
                    for (int c = 0; c < CT; ++c) acc[s][c] += __float2int_rn(gvs[e][c] * ev);
                }
            }
        }
    }
    float out[SEG][CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        // a correctly rounded quotient by one residual step on a product with
        // the correctly rounded reciprocal (Markstein), a third of a division's
        // instructions, where neither can leave the normal numbers
        const float sc = scale[c], y = 1.0f / sc;
        const bool plain = sc > 0x1p-90f && sc < 0x1p90f;            // uniform
#pragma unroll
        for (int s = 0; s < SEG; ++s) {
            const float x = (float)acc[s][c], q = x * y;
            out[s][c] = fmaf(fmaf(-sc, q, x), y, q);
        }
        if (!plain) {
#pragma unroll
            for (int s = 0; s < SEG; ++s) out[s][c] = sc > 0.0f ? (float)acc[s][c] / sc : 0.0f;
        }
    }
    // Gaussians too large for the bins, in float, in the list's ascending
    // order (as k_vox_tile)
    const int nl = *nlarge;
    for (int f = 0; f < nl; f += VG_CHUNK) {                      // uniform
        __syncthreads();                  // the entries before are used
        if (wave == 0) {
            const bool in = f + lane < nl;
            const int gi = large[in ? f + lane : f];
            float v[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) v[c] = value[(int64_t)gi * CT + c];
            const GaussK p = rec[gi];
            stage(in, p, v);              // in order
        }
        __syncthreads();
        const int n = nsh;
        for (int e = 0; e < n; ++e) {
            const GaussK p = gsh[e];
            if (p.hi0 < wx0 || p.lo0 > wx1) continue;             // uniform
            if (ix < p.lo0 || ix > p.hi0 || iy < p.lo1 || iy > p.hi1) continue;
            float cb2, cq;
            col_coeffs(p.a00, p.a01, p.a02, p.a11, p.a12, d0g - p.mu[0], d1g - p.mu[1], cb2, cq);
#pragma unroll
            for (int s = 0; s < SEG; ++s) {
                if (z0 + s < p.lo2 || z0 + s > p.hi2) continue;
                const float mm = col_quad(p.a22, cb2, cq, d2g[s] - p.mu[2]);
                if (!(mm <= k2)) continue;
                const float ev = half_exp(mm);
#pragma unroll
                for (int c = 0; c < CT; ++c) out[s][c] += gvs[e][c] * ev;
            }
        }
    }
    if (ix > e0 || iy > e1) return;
    const int64_t N = grid_size(g);
    float *const vb = vol + ((int64_t)ix * g.n[1] + iy) * g.n[2];
    if constexpr (SEG == 4) {
        // a thread's four voxels as one 16-byte store per channel when the
        // rows and the volume are 16-byte aligned (z0 is a multiple of 4)
        if ((g.n[2] & 3) == 0 && ((uintptr_t)vol & 15) == 0 && z0 + 3 <= e2) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
                *(float4 *)(vb + (int64_t)c * N + z0) =
                    make_float4(out[0][c], out[1][c], out[2][c], out[3][c]);
            return;
        }
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int s = 0; s < SEG; ++s)
            if (z0 + s <= e2) vb[(int64_t)c * N + z0 + s] = out[s][c];
}

// Up to this many tiles (two per CU) k_vox_tile has 16 waves per tile, not
// four: with fewer tiles than CUs can hold the longest list's walk is what the
// launch takes (4,096 Gaussians in 64^3, 256 tiles: 59 us with 4 waves, 22 with
// 16; a 32^3 block of 200k Gaussians, 64 tiles: 43 and 21).  With more the CUs
// are full either way, and the smaller batches cost.
constexpr int64_t VOX_FEW = 512;

VoxPlan vox_plan(int64_t m, int c, const GridK &g) {
    VoxPlan p;
    int T[3];
    if (c <= 1) {
        // fewest columns cut at z faces; 8x16x32 and 8x8x64 leave fewer,
        // longer lists, and their LDS atomics contend (200k Gaussians into
        // 256x256x128, binning + tiles: 8x8x32 0.49 ms, 8x16x16 0.50, 8x16x32
        // 0.66, 8x8x64 0.63; 0.15 ms now with the binning and boxes of today)
        T[0] = 8; T[1] = 8; T[2] = 32;
    } else if (c <= 4) {
        T[0] = 8; T[1] = 16; T[2] = 16;
    } else if (c <= 9) {
        T[0] = 8; T[1] = 8; T[2] = 16;
    } else {
        T[0] = 8; T[1] = 8; T[2] = 8;
    }
    // small grids (a TV sub-volume): halve the longest tile edge, down to 8,
    // until there are at least 256 tiles to spread over the CUs
    auto ntiles_of = [&](const int *t) {
        int64_t n = 1;
        for (int a = 0; a < 3; ++a) n *= (g.n[a] + t[a] - 1) / t[a];
        return n;
    };
    while (ntiles_of(T) < 256) {
        int a = 0;
        for (int b = 1; b < 3; ++b)
            if (T[b] > T[a]) a = b;
        if (T[a] <= 8) break;
        T[a] /= 2;
    }
    p.ntiles = 1;
    for (int a = 0; a < 3; ++a) {
        p.T[a] = T[a];
        p.nt[a] = (g.n[a] + T[a] - 1) / T[a];
        p.ntiles *= p.nt[a];
    }
    p.maxtiles = 32;
    p.cap = m * p.maxtiles;
    // chunks of at least 128 Gaussians, at most 256 of them (one per CU) or,
    // if that is more, of 512 Gaussians (a pass of their threads), and no
    // more than 2^24 (chunk, tile) counts unless that leaves fewer than 8
    const int64_t most = std::max<int64_t>(256, std::min<int64_t>(512, (m + BIN_T - 1) / BIN_T));
    p.nch = (int)std::max<int64_t>(1, std::min<int64_t>({most, (m + 127) / 128,
                                                         std::max<int64_t>(8, (1 << 24) / p.ntiles)}));
    return p;
}

namespace {
struct VoxWs {
    GaussK *rec;
    int32_t *part, *total, *wtotal, *off, *list, *large, *nlarge, *slot;
    size_t bytes;
};
VoxWs vox_ws(void *base, const VoxPlan &p, int64_t m) {
    VoxWs w;
    char *const b = (char *)base;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *r = b ? b + o : nullptr;
        o += align256(bytes);
        return r;
    };
    const size_t n = (size_t)std::max<int64_t>(m, 1), cap = (size_t)std::max<int64_t>(p.cap, 1);
    w.rec = (GaussK *)take(sizeof(GaussK) * n);                                  // records
    w.part = (int32_t *)take(sizeof(int32_t) * (size_t)p.nch * (size_t)p.ntiles);   // chunks' counts
    w.total = (int32_t *)take(sizeof(int32_t) * (size_t)p.ntiles);               // tiles' totals
    w.wtotal = (int32_t *)take(sizeof(int32_t) * (size_t)((p.ntiles + BIN_W - 1) / BIN_W));  // windows'
    w.off = (int32_t *)take(sizeof(int32_t) * (size_t)(p.ntiles + 1));           // lists' offsets
    w.list = (int32_t *)take(sizeof(int32_t) * cap);
    w.large = (int32_t *)take(sizeof(int32_t) * n);                              // large list
    w.nlarge = (int32_t *)take(sizeof(int32_t) * (size_t)(p.nch + 1));           // its length, per chunk
    w.slot = (int32_t *)take(sizeof(int32_t) * cap);                             // pairs' places
    w.bytes = o;
    return w;
}
}  // namespace

size_t vox_workspace(const VoxPlan &p, int64_t m) { return vox_ws(nullptr, p, m).bytes; }

hipError_t launch_voxelize(const pmf_gauss_t &gs, const GridK &g, float k, float *vol,
                           const VoxPlan &p, void *ws, hipStream_t s) {
    const int64_t m = gs.m;
    const VoxWs w = vox_ws(ws, p, m);
    GaussK *const rec = w.rec;
    int32_t *const off = w.off, *const list = w.list, *const large = w.large,
                  *const nlarge = w.nlarge;
    const float k2 = isinf(k) ? INFINITY : k * k;
    hipError_t e;
    const bool few = p.ntiles <= VOX_FEW, scan = few && m > 0 && m <= (p.ntiles <= 256 ? VOX_SCAN : VOX_SCAN_MANY);
    if (m == 0) {
        if ((e = launch_fill_i32(off, p.ntiles + 1, 0, s)) != hipSuccess) return e;
        if ((e = launch_fill_i32(nlarge, 1, 0, s)) != hipSuccess) return e;
    } else {
        VoxTiles t;
        t.T0 = p.T[0];
        t.T1 = p.T[1];
        t.T2 = p.T[2];
        t.nt1 = p.nt[1];
        t.nt2 = p.nt[2];
        t.ntiles = (int)p.ntiles;
        t.maxtiles = p.maxtiles;
        t.chunk = (m + p.nch - 1) / p.nch;
        const size_t hist = sizeof(int32_t) * (size_t)std::min<int64_t>(p.ntiles, BIN_W);
        const unsigned nwin = (unsigned)((p.ntiles + BIN_W - 1) / BIN_W);
        {
            ProfScope prof_("voxelize_bin", s);
            if (scan) {
                k_vox_bin<false><<<(unsigned)p.nch, BIN_T, 0, s>>>(gs, g, k, t, rec, w.part, w.slot,
                                                                   nlarge, 0, w.wtotal);
            } else {
                k_vox_bin<true><<<(unsigned)p.nch, BIN_T, hist, s>>>(gs, g, k, t, rec, w.part, w.slot,
                                                                     nlarge, 0, w.wtotal);
                if (nwin > 1)
                    k_vox_bin<true><<<dim3((unsigned)p.nch, nwin - 1), BIN_T, hist, s>>>(
                        gs, g, k, t, rec, w.part, w.slot, nlarge, 1, w.wtotal);
            }
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const bool brief = nwin == 1 && (int64_t)p.nch * p.ntiles <= BIN_SHORT;
        if (!brief && !scan) {
            ProfScope prof_("voxelize_chunks", s);
            k_vox_chunks<<<(unsigned)((p.ntiles + 63) / 64), 1024, 0, s>>>(w.part, t.ntiles, p.nch,
                                                                          w.total, w.wtotal);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (!scan) {
            ProfScope prof_("voxelize_fill", s);
            if (brief)
                k_vox_fill<true><<<(unsigned)p.nch, BIN_T, hist, s>>>(
                    m, rec, t, w.part, w.total, w.slot, nlarge, w.wtotal, off, list, large);
            else
                k_vox_fill<false><<<dim3((unsigned)p.nch, nwin), BIN_T, hist, s>>>(
                    m, rec, t, w.part, w.total, w.slot, nlarge, w.wtotal, off, list, large);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const size_t lds = sizeof(float) * (size_t)gs.c * (p.T[0] * p.T[1] * p.T[2]);
    {
        ProfScope prof_("voxelize_tile", s);
        const int sel = (p.T[1] == 16 ? 2 : 0) + (p.T[2] == 16 ? 1 : 0);
        const int cs = gs.c;
        // one channel: the LDS splat (many Gaussians per tile); 3 or 9
        // channels: voxel owners, but sixteen waves of the LDS splat on few
        // tiles (1,000 to 16,000 Gaussians of three channels on 32x32x32 to
        // 128x128x64, 64 to 512 tiles: 21, 21 and 66 us with voxel owners, 8,
        // 10 and 21 with the splat; on 8,192 tiles of nine channels 110 us
        // against 152); other channel counts: the LDS splat
#define VOX_TILE_W(T1_, T2_, CT_, NW_, VB_, SCAN_)                                                 \
    k_vox_tile<8, T1_, T2_, CT_, NW_, VB_, SCAN_><<<(unsigned)p.ntiles, 64 * NW_, lds, s>>>(      \
        rec, (int)m, p.nch, p.maxtiles, gs.value, gs.c, g, k2, p.nt[1], p.nt[2], off, list,       \
        large, nlarge, vol)
#define VOX_FEW_TILES(T1_, T2_, CT_)                                                              \
    do {                                                                                          \
        if (scan) VOX_TILE_W(T1_, T2_, CT_, 16, 8, true);                                         \
        else VOX_TILE_W(T1_, T2_, CT_, 16, 8, false);                                             \
    } while (0)
#define VOX_TILE(T1_, T2_, CT_)                                                                   \
    do {                                                                                          \
        if (few) VOX_FEW_TILES(T1_, T2_, CT_);                                                    \
        else VOX_TILE_W(T1_, T2_, CT_, 4, 16, false);                                             \
    } while (0)
#define VOX_GATHER(T1_, T2_, CT_)                                                                 \
    do {                                                                                          \
        if (few) VOX_FEW_TILES(T1_, T2_, CT_);                                                    \
        else                                                                                      \
            k_vox_gather<8, T1_, T2_, CT_><<<(unsigned)p.ntiles, 256, 0, s>>>(                    \
                rec, gs.value, g, k2, p.nt[1], p.nt[2], off, list, large, nlarge, vol);           \
    } while (0)
#define VOX_TILE_C(T1_, T2_)                                                                      \
    do {                                                                                          \
        if (cs == 1) VOX_TILE(T1_, T2_, 1);                                                       \
        else if (cs == 3) VOX_GATHER(T1_, T2_, 3);                                                \
        else if (cs == 9) VOX_GATHER(T1_, T2_, 9);                                                \
        else VOX_TILE(T1_, T2_, 0);                                                               \
    } while (0)
        if (cs == 1 && p.T[1] == 8 && p.T[2] == 32) VOX_TILE(8, 32, 1);   // one channel
        else switch (sel) {
            case 3: VOX_TILE_C(16, 16); break;
            case 2: VOX_TILE_C(16, 8); break;
            case 1: VOX_TILE_C(8, 16); break;
            default: VOX_TILE_C(8, 8); break;
        }
#undef VOX_TILE_C
#undef VOX_GATHER
#undef VOX_TILE
#undef VOX_FEW_TILES
#undef VOX_TILE_W
    }
    return hipGetLastError();
}

// ------------------------------------------------------------- backward

// Adjoint, Gaussian owner.  A workgroup takes `per` consecutive Gaussians: its
// lanes j < per build their geometry and stage what the walks need in LDS, its
// waves walk the voxel boxes of those that reach the grid, one Gaussian of a
// wave at a time, and the lanes j < per apply the chain rule to the sums.  (With
// set-up and chain by each wave for its own eight Gaussians, or its one, most of
// its lanes were idle for half of the instructions: 200k Gaussians of which few
// reach a 32^3 block 48 us, now 12.)  Fetches bound the walks of sets in no
// order: 640 MB in 109 us for 200k Gaussians in 256x256x128 (147 before), and
// for 16k of nine channels (117 us, 129 before), whose volume is 302 MB.  A walk sums, over the
// voxels inside the ellipsoid, with t = e sum_c v_c g_c:
//   sum e g_c (value gradients),
//   sum t d    (mean gradient A sum t d),
//   sum t d d^T (the gradient of the quadratic form),
// in an order that only the Gaussian itself sets, and reduces them over the
// wave; the chain rule goes on through Sigma^-1 = R diag(s^-2) R^T and the
// quaternion normalisation.
constexpr int BW_NS = 9;       // sums besides the channels: P0..P2, M00 M01 M02 M11 M12 M22
constexpr int BW_WAVES = 4;    // waves per workgroup
constexpr int BW_SLOTS = 512;  // voxels per window of a walk over several channels

struct VoxG {                  // one Gaussian of the workgroup's batch
    float mu[3];
    float a00, a01, a02, a11, a12, a22;
    int lo0, lo1, lo2, hi0, hi1, hi2;
};

// Column `col` of the box of q (axis 1 fastest): its offsets, its quadratic's
// coefficients and its z range [za, zb] (za > zb: empty).
struct VoxCol {
    float d0, d1, b2, cq;
    int ix, iy, za, zb;
};
__device__ __forceinline__ VoxCol vox_col(const VoxG &q, const GridK &g, int col, int ny, float rny,
                                          float zc, float zm, float k2, bool untrunc) {
    VoxCol c;
    // col = cx * ny + cy (the float quotient is corrected to exact)
    int cx = (int)(((float)col + 0.5f) * rny);
    int cy = col - cx * ny;
    if (cy < 0) {
        --cx;
        cy += ny;
    } else if (cy >= ny) {
        ++cx;
        cy -= ny;
    }
    c.ix = q.lo0 + cx;
    c.iy = q.lo1 + cy;
    c.d0 = fmaf((float)c.ix, g.h[0], g.c0[0]) - q.mu[0];
    c.d1 = fmaf((float)c.iy, g.h[1], g.c0[1]) - q.mu[1];
    col_coeffs(q.a00, q.a01, q.a02, q.a11, q.a12, c.d0, c.d1, c.b2, c.cq);
    if (!col_range(q.a22, c.b2, c.cq, zc, zm, g.inv_h[2], k2, untrunc, q.lo2, q.hi2, c.za, c.zb)) {
        c.za = 0;
        c.zb = -1;
    }
    return c;
}

// Sums of x[0..N) over the wave -> out[0..n), in LDS.
template <int N>
__device__ __forceinline__ void wave_sums(const float (&x)[N], int n, int lane, float *out) {
    const int q = sum4_index(lane);
#pragma unroll
    for (int k = 0; k < N; k += 4) {
        const float z = 0.0f;
        const float t = wave_sum4(x[k], k + 1 < N ? x[k + 1 < N ? k + 1 : 0] : z,
                                  k + 2 < N ? x[k + 2 < N ? k + 2 : 0] : z,
                                  k + 3 < N ? x[k + 3 < N ? k + 3 : 0] : z);
        if ((lane & 15) == 0 && k + q < n) out[k + q] = t;
    }
}

// One channel: a lane per column, 64 columns at a time; a lane walks its
// column's z range S voxels at a time (whole steps by one wide load: a lane's
// column is a cache line of its own) and keeps only sum e g, sum e g d2 and
// sum e g d2^2 of it, folded into the others when it leaves the column (the
// factor v_0 of t waits for the chain rule).  Steps of 2, 4 and 8, 256x256x128:
// 300 Gaussians of s = 12 voxels 757 / 531 / 432 us (495 with four loads in
// flight before), 50,000 of s = 4 (25 tall) 1.02 / 0.88 / 0.67 ms, of s = 2 (13 tall)
// 155 / 146 us with 2 and 4; with more than 64 registers the reference set's 107 us
// became 119.
template <int S>
__device__ __forceinline__ void walk_columns(const VoxG &q, const GridK &g, float k2, bool untrunc,
                                             const float *__restrict__ g_vol, int lane,
                                             float *out) {
    float x[1 + BW_NS];
#pragma unroll
    for (int k = 0; k < 1 + BW_NS; ++k) x[k] = 0.0f;
    const int ny = q.hi1 - q.lo1 + 1;
    const int ncol = (q.hi0 - q.lo0 + 1) * ny;
    const float rny = __builtin_amdgcn_rcpf((float)ny);
    const float zc = (q.mu[2] - g.c0[2]) * g.inv_h[2], zm = voxel_margin(g, 2, zc);
    const float h2 = in_vgpr(g.h[2]), o2 = in_vgpr(g.c0[2]), kk = in_vgpr(k2);
    for (int c0 = 0; c0 < ncol; c0 += 64) {
        const int col = c0 + lane;
        if (col >= ncol) continue;
        const VoxCol c = vox_col(q, g, col, ny, rny, zc, zm, k2, untrunc);
        const float *gz = g_vol + ((int64_t)c.ix * g.n[1] + c.iy) * g.n[2] + c.za;
        float St = 0.0f, Sz = 0.0f, Szz = 0.0f, fz = (float)c.za;
        auto voxel = [&](float z, float gl, bool in) {
            const float d2 = fmaf(z, h2, o2) - q.mu[2];
            const float mm = col_quad(q.a22, c.b2, c.cq, d2);
            const float t = gl * (in && mm <= kk ? half_exp(mm) : 0.0f);
            St += t;
            const float td = t * d2;
            Sz += td;
            Szz = fmaf(td, d2, Szz);
        };
        int n = c.zb - c.za + 1;
        if constexpr (S > 2) {
            for (; n >= S; n -= S, gz += S, fz += (float)S) {
                typedef float vec __attribute__((ext_vector_type(S), aligned(4)));
                const vec gl = *(const vec *)gz;
#pragma unroll
                for (int k = 0; k < S; ++k) voxel(fz + (float)k, gl[k], true);
            }
        }
        for (; n > 0; n -= 2, gz += 2, fz += 2.0f) {
            const float g0 = gz[0], g1 = gz[n > 1 ? 1 : 0];
            voxel(fz, g0, true);
            voxel(fz + 1.0f, g1, n > 1);
        }
        x[0] += St;
        x[1] = fmaf(c.d0, St, x[1]);
        x[2] = fmaf(c.d1, St, x[2]);
        x[3] += Sz;
        x[4] = fmaf(c.d0 * St, c.d0, x[4]);
        x[5] = fmaf(c.d0 * St, c.d1, x[5]);
        x[6] = fmaf(c.d0, Sz, x[6]);
        x[7] = fmaf(c.d1 * St, c.d1, x[7]);
        x[8] = fmaf(c.d1, Sz, x[8]);
        x[9] += Szz;
    }
    wave_sums(x, 1 + BW_NS, lane, out);
}

// Several channels: a voxel loads C values, and lanes on different columns
// would touch a cache line per lane and channel, so the voxels of 64 columns
// are laid over the lanes in order (z fastest): each column's lane writes its
// number to the places of its voxels, BW_SLOTS at a time, and a voxel's lane
// reads its column from there.
struct VoxSlots {
    float4 q[64];                       // d0, d1, b2, cq of a column
    int2 at[64];                        // volume offset and z index of place 0, if the column began there
    uint8_t col[BW_SLOTS];
};
template <int CT>
__device__ __forceinline__ void walk_voxels(const VoxG &q, const GridK &g, float k2, bool untrunc,
                                            const float *__restrict__ g_vol, int C,
                                            const float *val, VoxSlots &sl, int lane, float *out) {
    constexpr int CM = CT > 0 ? CT : MAXC_VOX;
    float x[CM + BW_NS], v[CM];
#pragma unroll
    for (int k = 0; k < CM + BW_NS; ++k) x[k] = 0.0f;
#pragma unroll
    for (int c = 0; c < CM; ++c) v[c] = c < C ? val[c] : 0.0f;
    float *const m = x + CM;
    const int64_t N = grid_size(g);
    const int ny = q.hi1 - q.lo1 + 1;
    const int ncol = (q.hi0 - q.lo0 + 1) * ny;
    const float rny = __builtin_amdgcn_rcpf((float)ny);
    const float zc = (q.mu[2] - g.c0[2]) * g.inv_h[2], zm = voxel_margin(g, 2, zc);
    const float h2 = in_vgpr(g.h[2]), o2 = in_vgpr(g.c0[2]), kk = in_vgpr(k2);
    for (int c0 = 0; c0 < ncol; c0 += 64) {                     // uniform
        VoxCol c;
        c.za = 0;
        c.zb = -1;
        if (c0 + lane < ncol) c = vox_col(q, g, c0 + lane, ny, rny, zc, zm, k2, untrunc);
        const int len = c.zb - c.za + 1;
        const int end = wave_incl_sum(len), beg = end - len;
        const int total = __builtin_amdgcn_readlane(end, 63);
        // the box's corner column begins at g_vol + box: offsets from it are int
        if (len > 0) {
            sl.q[lane] = make_float4(c.d0, c.d1, c.b2, c.cq);
            sl.at[lane] = make_int2((c.ix - q.lo0) * g.n[1] + (c.iy - q.lo1), c.za - beg);
        }
        for (int w0 = 0; w0 < total; w0 += BW_SLOTS) {          // uniform
            const int e = min(end - w0, BW_SLOTS);
            for (int k = max(beg - w0, 0); k < e; ++k) sl.col[k] = (uint8_t)lane;
            wave_lds_sync();
            const int nw = min(total - w0, BW_SLOTS);
            for (int p = lane; p < nw; p += 64) {
                const int j = sl.col[p];
                const float4 cf = sl.q[j];
                const int2 at = sl.at[j];
                const int iz = at.y + w0 + p;
                const float *gp = g_vol + (((int64_t)q.lo0 * g.n[1] + q.lo1 + at.x) * g.n[2] + iz);
                float gl[CM];
#pragma unroll
                for (int ch = 0; ch < CM; ++ch) gl[ch] = ch < C ? gp[ch * N] : 0.0f;
                const float d2 = fmaf((float)iz, h2, o2) - q.mu[2];
                const float mm = col_quad(q.a22, cf.z, cf.w, d2);
                const float ev = mm <= kk ? half_exp(mm) : 0.0f;
                float G = 0.0f;
#pragma unroll
                for (int ch = 0; ch < CM; ++ch) {
                    if (ch < C) {
                        x[ch] = fmaf(gl[ch], ev, x[ch]);
                        G = fmaf(v[ch], gl[ch], G);
                    }
                }
                const float t = G * ev;
                const float t0 = t * cf.x, t1 = t * cf.y, t2 = t * d2;
                m[0] += t0;
                m[1] += t1;
                m[2] += t2;
                m[3] = fmaf(t0, cf.x, m[3]);
                m[4] = fmaf(t0, cf.y, m[4]);
                m[5] = fmaf(t0, d2, m[5]);
                m[6] = fmaf(t1, cf.y, m[6]);
                m[7] = fmaf(t1, d2, m[7]);
                m[8] = fmaf(t2, d2, m[8]);
            }
            wave_lds_sync();
        }
    }
    wave_sums(x, CM + BW_NS, lane, out);
}

template <int CT>
__global__ __launch_bounds__(64 * BW_WAVES, CT == 1 ? 8 : 1) void k_vox_bwd(pmf_gauss_t gs, GridK g, float k, int per,
                                                           const float *__restrict__ g_vol,
                                                           pmf_gauss_grad_t gr) {
    constexpr int CM = CT > 0 ? CT : MAXC_VOX;
    const int C = CT > 0 ? CT : gs.c;
    extern __shared__ float4 bwd_smem[];
    float(*const sums)[CM + BW_NS] = (float(*)[CM + BW_NS])bwd_smem;
    VoxG *const gb = (VoxG *)(sums + per);
    __shared__ int near[64], nnear;
    const int t = (int)threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), nwaves = (int)blockDim.x / 64;
    const int64_t g0 = (int64_t)blockIdx.x * per;
    const float k2 = isinf(k) ? INFINITY : k * k;
    const bool untrunc = isinf(k2);
    bool hit = false;
    if (wave == 0) {
        const int64_t gi = g0 + lane;
        if (lane < per && gi < gs.m && !far_from_grid(gs.mean, gs.scale, gi, k, g)) {
            GaussFull G;
            gauss_full(gs.mean, gs.scale, gs.quat, gi, k, g, G);
            VoxG q;
            for (int a = 0; a < 3; ++a) q.mu[a] = G.mu[a];
            q.a00 = G.A[0][0];
            q.a01 = G.A[0][1];
            q.a02 = G.A[0][2];
            q.a11 = G.A[1][1];
            q.a12 = G.A[1][2];
            q.a22 = G.A[2][2];
            q.lo0 = G.lo[0];
            q.lo1 = G.lo[1];
            q.lo2 = G.lo[2];
            q.hi0 = G.hi[0];
            q.hi1 = G.hi[1];
            q.hi2 = G.hi[2];
            hit = q.lo0 <= q.hi0 && q.lo1 <= q.hi1 && q.lo2 <= q.hi2;
            gb[lane] = q;
        }
        const uint64_t hits = __ballot(hit);
        if (hit) near[__popcll(hits & ((1ull << lane) - 1))] = lane;
        if (lane == 0) nnear = __popcll(hits);
    }
    __syncthreads();
    for (int i = wave; i < nnear; i += nwaves) {               // uniform
        const int j = near[i];
        const VoxG q = gb[j];
        if constexpr (CT == 1) {
            // steps of the box's height: a tall column's loads merge into wide
            // ones, a low one has no whole step
            const int nz = q.hi2 - q.lo2 + 1;
            if (nz <= 8) walk_columns<2>(q, g, k2, untrunc, g_vol, lane, sums[j]);
            else if (nz <= 16) walk_columns<4>(q, g, k2, untrunc, g_vol, lane, sums[j]);
            else walk_columns<8>(q, g, k2, untrunc, g_vol, lane, sums[j]);
        } else {
            __shared__ VoxSlots slots[BW_WAVES];
            walk_voxels<CT>(q, g, k2, untrunc, g_vol, C, gs.value + (g0 + j) * C, slots[wave], lane,
                            sums[j]);
        }
    }
    __syncthreads();
    // chain rule: lane j for Gaussian g0 + j
    const int64_t gi = g0 + t;
    if (t >= per || gi >= gs.m) return;
    float *const o = sums[t];
    if (!hit) {                           // no voxel: zero gradients (t < per: a lane of wave 0)
        for (int c = 0; c < C; ++c) gr.value[gi * C + c] = 0.0f;
        for (int a = 0; a < 3; ++a) {
            gr.mean[3 * gi + a] = 0.0f;
            gr.scale[3 * gi + a] = 0.0f;
        }
        for (int c = 0; c < 4; ++c) gr.quat[4 * gi + c] = 0.0f;
        return;
    }
    GaussFull G;
    gauss_full(gs.mean, gs.scale, gs.quat, gi, k, g, G);
    for (int c = 0; c < C; ++c) gr.value[gi * C + c] = o[c];
    if constexpr (CT == 1) {
        const float v = gs.value[gi];
        for (int c = 1; c <= BW_NS; ++c) o[c] *= v;
    }
    const float P[3] = {o[CM + 0], o[CM + 1], o[CM + 2]};
    // mean: d/dmu of -m/2 is A d, so dL/dmu = A sum t d
    for (int a = 0; a < 3; ++a)
        gr.mean[3 * gi + a] = G.A[a][0] * P[0] + G.A[a][1] * P[1] + G.A[a][2] * P[2];
    // d/dA of -m/2 is -d d^T / 2
    const float M[3][3] = {{-0.5f * o[CM + 3], -0.5f * o[CM + 4], -0.5f * o[CM + 5]},
                           {-0.5f * o[CM + 4], -0.5f * o[CM + 6], -0.5f * o[CM + 7]},
                           {-0.5f * o[CM + 5], -0.5f * o[CM + 7], -0.5f * o[CM + 8]}};
    float MR[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            MR[a][b] = M[a][0] * G.R[0][b] + M[a][1] * G.R[1][b] + M[a][2] * G.R[2][b];
    for (int kk = 0; kk < 3; ++kk) {
        const float d = G.R[0][kk] * MR[0][kk] + G.R[1][kk] * MR[1][kk] + G.R[2][kk] * MR[2][kk];
        gr.scale[3 * gi + kk] = -2.0f * d / (G.s[kk] * G.s[kk] * G.s[kk]);
    }
    float GR[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) GR[a][b] = 2.0f * MR[a][b] / (G.s[b] * G.s[b]);
    const float w = G.qh[0], x = G.qh[1], y = G.qh[2], z = G.qh[3];
    float gq[4];
    gq[0] = 2.0f * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] +
                    x * GR[2][1]);
    gq[1] = 2.0f * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - 2.0f * x * GR[1][1] -
                    w * GR[1][2] + z * GR[2][0] + w * GR[2][1] - 2.0f * x * GR[2][2]);
    gq[2] = 2.0f * (-2.0f * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] +
                    z * GR[1][2] - w * GR[2][0] + z * GR[2][1] - 2.0f * y * GR[2][2]);
    gq[3] = 2.0f * (-2.0f * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] -
                    2.0f * z * GR[1][1] + y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
    const float dot = gq[0] * w + gq[1] * x + gq[2] * y + gq[3] * z;
    for (int c = 0; c < 4; ++c) gr.quat[4 * gi + c] = (gq[c] - G.qh[c] * dot) / G.qn;
}

hipError_t launch_voxelize_bwd(const pmf_gauss_t &gs, const GridK &g, float k, const float *g_vol,
                               const pmf_gauss_grad_t &gr, hipStream_t s) {
    if (gs.m <= 0) return hipSuccess;
    {
        ProfScope prof_("voxelize_bwd", s);
        // Gaussians per workgroup: as many as leave about 2,000 workgroups (64
        // fill the lanes of the set-up and the chain rule), at least one per wave
        int per = BW_WAVES;
        const int choice = tune_get(KNOB_VOXELIZE_BWD);
        if (choice > 0)
            per = 1 << (choice - 1);
        else
            while (per < 64 && gs.m / (2 * per) >= 2000) per *= 2;
        const unsigned nb = (unsigned)((gs.m + per - 1) / per), nt = 64u * std::min(per, BW_WAVES);
        const int cm = gs.c == 1 || gs.c == 3 || gs.c == 9 ? gs.c : MAXC_VOX;
        const size_t lds = (size_t)per * (sizeof(VoxG) + sizeof(float) * (cm + BW_NS));
        if (gs.c == 1)
            k_vox_bwd<1><<<nb, nt, lds, s>>>(gs, g, k, per, g_vol, gr);
        else if (gs.c == 3)
            k_vox_bwd<3><<<nb, nt, lds, s>>>(gs, g, k, per, g_vol, gr);
        else if (gs.c == 9)
            k_vox_bwd<9><<<nb, nt, lds, s>>>(gs, g, k, per, g_vol, gr);
        else
            k_vox_bwd<0><<<nb, nt, lds, s>>>(gs, g, k, per, g_vol, gr);
    }
    return hipGetLastError();
}

}  // namespace pmf
