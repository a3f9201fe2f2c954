// combine.hip -- the low-rank DVF of Eq. 3 and its adjoint.
//
// Forward: one thread per output voxel.  For each level the trilinear
// stencil on the level grid is computed once and shared by its 3B channels;
// the L*B*3 sampled basis values stay in registers while the V views'
// displacements are formed from the (wave-uniform) coefficients.
//
// Adjoint, coefficients: the same per-voxel basis samples dotted with g_dvf,
// reduced per workgroup into a partial buffer and summed in a second pass
// (fixed order, deterministic).
//
// Adjoint, bases: the trilinear upsampling is a tensor product of three 1-D
// interpolation matrices (fine index -> level index per axis, zero rows
// outside the box), so its transpose is applied as up to three 1-D gather
// passes, each recomputing the forward's 1-D weights.  Axes on which the
// level grid equals the output grid are skipped.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "pmf_internal.h"

namespace pmf {

template <int L, int B>
__global__ __launch_bounds__(256) void k_combine(LevelsK lv, const float *__restrict__ coeff,
                                                 int V, GridK out, float *__restrict__ dvf) {
    const int64_t N = grid_size(out);
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= N) return;
    const int iz = (int)(j % out.n[2]);
    const int iy = (int)((j / out.n[2]) % out.n[1]);
    const int ix = (int)(j / ((int64_t)out.n[2] * out.n[1]));
    float sv[L][B][3];
    basis_samples<L, B>(lv, ix, iy, iz, sv);
    for (int v = 0; v < V; ++v) {
        const float *cv = coeff + (int64_t)v * L * B * 3;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float d = 0.0f;
#pragma unroll
            for (int l = 0; l < L; ++l)
#pragma unroll
                for (int b = 0; b < B; ++b) d = fmaf(cv[(l * B + b) * 3 + k], sv[l][b][k], d);
            dvf[((int64_t)v * 3 + k) * N + j] = d;
        }
    }
}

// ------------------------------------------------------- basis samples by block
// A wave's block of output voxels: 4 x 4 columns of 64 along axis 2 (lanes),
// which share the level's cells.  Per channel the coarse columns under the
// block are read and interpolated along axis 2 once (9 of them at a ratio of
// 4 x 4, 16 at 2 x 2 or on the level's own grid, where 16 outputs taken alone
// read 64), then along axis 1 per coarse plane, then along axis 0: the
// arithmetic of stencil_read in its order.  All loads of a channel are issued
// together.  (Walking the columns and reusing each as the next needs it reads
// no more but waits for every column in turn: 703 us where this takes
// 172.)  Cells and fractions of axes 0 and 1 are wave-uniform.
constexpr int CXY = 16;

struct BlockAxis {              // the block's four outputs along one axis
    int c0, n;                  // first output's cell, level size
    int r[4];                   // cells relative to c0
    float f[4];
    bool in[4];
};

// axis_cell of four consecutive outputs of n_out; one outside the level's box
// takes the cell of the nearest inside point (its value is not used, nor that
// of one past the output grid: the level may go on there).
__device__ __forceinline__ BlockAxis block_axis(const AxisMap &m, int a, int i0, int n_out) {
    BlockAxis x;
    x.n = m.n[a];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float u = level_coord(m, a, i0 + q);
        x.in[q] = u >= -0.5f && u <= (float)m.n[a] - 0.5f && i0 + q < n_out;
        const float uc = fminf(fmaxf(u, 0.0f), (float)(m.n[a] - 1));
        const int c = __builtin_amdgcn_readfirstlane(min((int)floorf(uc), m.n[a] - 2));
        x.f[q] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(uc - (float)c)));
        if (q == 0) x.c0 = c;
        x.r[q] = c - x.c0;
    }
    return x;
}

// Coarse values that four outputs of an axis can touch, by the level's
// spacing: their coordinates span at most 3 scale, so cells at most
// 1 + floor(3 scale) + 1 apart (0: too many for a block).  An axis on the
// level's own grid has integer coordinates.
__host__ __device__ inline int axis_span(const AxisMap &m, int a) {
    if (m.ident[a]) return 5;
    return m.scale[a] <= 0.25f ? 3 : m.scale[a] <= 0.5f ? 4 : m.scale[a] <= 0.99f ? 5 : 0;
}

struct LevelBlock {
    BlockAxis x, y;
    int cz, s0, s1, span;
    float fz;
    bool inz, direct;           // direct: outputs lie on the level's columns
};

__device__ __forceinline__ LevelBlock level_block(const AxisMap &m, const GridK &out, int ix0,
                                                  int iy0, int iz, bool on) {
    LevelBlock b;
    b.x = block_axis(m, 0, ix0, out.n[0]);
    b.y = block_axis(m, 1, iy0, out.n[1]);
    int i = 0;
    float f = 0.0f;
    b.inz = axis_cell(level_coord(m, 2, iz), m.n[2], i, f) && on;
    b.cz = b.inz ? i : 0;
    b.fz = b.inz ? f : 0.0f;
    b.s1 = m.n[2];
    b.s0 = m.n[1] * m.n[2];
    b.span = max(axis_span(m, 0), axis_span(m, 1));
    // (past the level's last interior voxel the cell is the one below, f = 1)
    b.direct = m.ident[0] && m.ident[1] && ix0 + 3 < m.n[0] - 1 && iy0 + 3 < m.n[1] - 1;
    return b;
}

// lerp1 that returns a where f is 0 (fma(0, b - a, a) = a, also with b not finite)
__device__ __forceinline__ float lerp0(float a, float b, float f) {
    return f == 0.0f ? a : lerp1(a, b, f);
}

typedef float zpair __attribute__((ext_vector_type(2), aligned(4)));

// z[i] for a wave-uniform i < N
template <int N>
__device__ __forceinline__ float pick(const float (&z)[N], int o, int i) {
    float v = z[o];
#pragma unroll
    for (int k = 1; k + o < N; ++k) v = i == k ? z[o + k] : v;
    return v;
}

template <int N, class F>
__device__ __forceinline__ void block_samples_n(const float *__restrict__ E, const LevelBlock &b,
                                                F &&f) {
    zpair p[N][N];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j)
            p[i][j] = *(const zpair *)(E + min(b.x.c0 + i, b.x.n - 1) * b.s0 +
                                       min(b.y.c0 + j, b.y.n - 1) * b.s1 + b.cz);
    float Y[4][N];              // [y output][plane]
#pragma unroll
    for (int i = 0; i < N; ++i) {
        float z[N];
#pragma unroll
        for (int j = 0; j < N; ++j) z[j] = lerp0(p[i][j].x, p[i][j].y, b.fz);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            Y[r][i] = lerp0(pick(z, 0, b.y.r[r]), pick(z, 1, b.y.r[r]), b.y.f[r]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float v = lerp0(pick(Y[r], 0, b.x.r[q]), pick(Y[r], 1, b.x.r[q]), b.x.f[q]);
            f(4 * q + r, b.x.in[q] && b.y.in[r] && b.inz ? v : 0.0f);
        }
}

// f(4 q + r, value) for every output (x q, y r) of the block.
template <class F>
__device__ __forceinline__ void block_samples(const float *__restrict__ E, const LevelBlock &b, F &&f) {
    if (b.direct) {
        zpair p[CXY];
#pragma unroll
        for (int i = 0; i < CXY; ++i)
            p[i] = *(const zpair *)(E + (b.x.c0 + i / 4) * b.s0 + (b.y.c0 + i % 4) * b.s1 + b.cz);
#pragma unroll
        for (int i = 0; i < CXY; ++i) f(i, b.inz ? lerp0(p[i].x, p[i].y, b.fz) : 0.0f);
    } else if (b.span == 3) {
        block_samples_n<3>(E, b, f);
    } else if (b.span == 4) {
        block_samples_n<4>(E, b, f);
    } else {
        block_samples_n<5>(E, b, f);
    }
}

static bool block_levels(const LevelsK &lv) {
    for (int l = 0; l < lv.L; ++l)
        if (axis_span(lv.map[l], 0) == 0 || axis_span(lv.map[l], 1) == 0) return false;
    return true;
}

// Blocks of a grid, z fastest, and a wave's place in them.
struct BlockGrid {
    int nx, ny, nz;
    int n;
};
static BlockGrid block_grid(const GridK &g) {
    BlockGrid b{(g.n[0] + 3) / 4, (g.n[1] + 3) / 4, (g.n[2] + 63) / 64, 0};
    b.n = b.nx * b.ny * b.nz;
    return b;
}

// Whether the outputs fill the blocks well enough (a block takes the same time
// with few of its lanes on a voxel) and the blocks the chip: at least `fill` of
// a block's 1,024 outputs and `waves` blocks, by the number of bases that share
// a block's geometry.
struct BlockCut {
    int fill;
    int64_t waves;
};
static bool use_blocks(const LevelsK &lv, const GridK &out, const BlockGrid &bg, int64_t waves,
                       BlockCut one, BlockCut more) {
    const BlockCut c = lv.B == 1 ? one : more;
    return block_levels(lv) && waves >= c.waves && grid_size(out) >= c.fill * (int64_t)bg.n;
}

template <int VG>
__global__ __launch_bounds__(256) void k_combine_block(LevelsK lv, const float *__restrict__ coeff,
                                                       GridK out, BlockGrid bg,
                                                       float *__restrict__ dvf) {
    const int wave = __builtin_amdgcn_readfirstlane(
        xcd_block((int)blockIdx.x, (int)gridDim.x) * 4 + (int)(threadIdx.x >> 6));
    if (wave >= bg.n) return;
    const int bz = wave % bg.nz, by = (wave / bg.nz) % bg.ny, bx = wave / (bg.nz * bg.ny);
    const int ix0 = bx * 4, iy0 = by * 4, iz = bz * 64 + (int)(threadIdx.x & 63);
    const bool on = iz < out.n[2];
    const int64_t N = grid_size(out);
    const int k = (int)blockIdx.y;
    float d[VG][CXY];
#pragma unroll
    for (int w = 0; w < VG; ++w)
#pragma unroll
        for (int i = 0; i < CXY; ++i) d[w][i] = 0.0f;
#pragma unroll 1
    for (int l = 0; l < lv.L; ++l) {
        const AxisMap &m = lv.map[l];
        const LevelBlock b = level_block(m, out, ix0, iy0, iz, on);
        const int64_t Nl = (int64_t)m.n[0] * m.n[1] * m.n[2];
#pragma unroll 1
        for (int bb = 0; bb < lv.B; ++bb) {
            float c[VG];
#pragma unroll
            for (int w = 0; w < VG; ++w)
                c[w] = coeff[((w * lv.L + l) * lv.B + bb) * 3 + k];
            block_samples(lv.E[l] + (int64_t)(bb * 3 + k) * Nl, b, [&](int i, float x) {
#pragma unroll
                for (int w = 0; w < VG; ++w) d[w][i] = fmaf(c[w], x, d[w][i]);
            });
        }
    }
    if (!on) return;
#pragma unroll
    for (int w = 0; w < VG; ++w)
#pragma unroll
        for (int i = 0; i < CXY; ++i) {
            const int ix = ix0 + i / 4, iy = iy0 + i % 4;
            if (ix < out.n[0] && iy < out.n[1])
                dvf[(w * 3 + k) * N + ((int64_t)ix * out.n[1] + iy) * out.n[2] + iz] = d[w][i];
        }
}

// One or two views take the block kernel, which reads the bases once per call;
// from three on the per-voxel kernel's samples serve every view.  Three levels
// (64^3, 128^3, 256x256x128), per voxel against blocks: B = 3 one view
// 370 / 172 us, two 391 / 210, three 415 / 373 (two passes); B = 1 one view 123 / 89, two
// 164 / 116; at 128x128x64, B = 3, one view 52 / 34, three 54 / 61.  The cuts
// (k_combine alone, one view): 256 x 256 x 40 (640 outputs per block) B = 1
// 47 / 48, B = 3 121 / 90; x 32 (512) 39 / 48 and 98 / 88, two views 40 / 54 and
// 98 / 98; x 96 (768) B = 1 two views 96 / 98; 512x512x2 13 / 149 and 29 / 284;
// 64^3 (256 blocks) 11 / 15 and 18 / 22; 88x88x64 (484) 16 / 16 and 32 / 27;
// 112x112x64 (784) B = 1 two views 21 / 22.
hipError_t launch_combine(const LevelsK &lv, const float *coeff, int V, const GridK &out, float *dvf,
                          hipStream_t s) {
    const int64_t N = grid_size(out);
    const BlockGrid bg = block_grid(out);
    // (a grid of 2^26 blocks, flat along axis 2, has more threads than one
    // dimension of a launch)
    if (V <= 2 && bg.n < 1 << 26 && use_blocks(lv, out, bg, bg.n, {800, 784}, {576, 480})) {
        const dim3 nb((unsigned)((bg.n + 3) / 4), 3);
        ProfScope prof_("combine", s);
        if (V == 1) k_combine_block<1><<<nb, 256, 0, s>>>(lv, coeff, out, bg, dvf);
        else k_combine_block<2><<<nb, 256, 0, s>>>(lv, coeff, out, bg, dvf);
        return hipGetLastError();
    }
    return dispatch_lb(lv.L, lv.B, [&](auto Lc, auto Bc) {
        constexpr int L = decltype(Lc)::value, B = decltype(Bc)::value;
        {
            ProfScope prof_("combine", s);
            k_combine<L, B><<<(unsigned)((N + 255) / 256), 256, 0, s>>>(lv, coeff, V, out, dvf);
        }
        return hipGetLastError();
    });
}

// ------------------------------------------------------- coefficient adjoint
constexpr int NLB = MAXL * MAXB * 3;
constexpr int CB_BLOCKS = 1024;

template <int L, int B>
__global__ __launch_bounds__(256) void k_combine_bwd_coeff(LevelsK lv, GridK out,
                                                           const float *__restrict__ g_dvf,
                                                           float *__restrict__ partial) {
    const int64_t N = grid_size(out);
    const int v = blockIdx.y;
    float acc[L][B][3];
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int k = 0; k < 3; ++k) acc[l][b][k] = 0.0f;
    const float *gd = g_dvf + (int64_t)v * 3 * N;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < N;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int iz = (int)(j % out.n[2]);
        const int iy = (int)((j / out.n[2]) % out.n[1]);
        const int ix = (int)(j / ((int64_t)out.n[2] * out.n[1]));
        float sv[L][B][3];
        basis_samples<L, B>(lv, ix, iy, iz, sv);
        const float g[3] = {gd[j], gd[N + j], gd[2 * N + j]};
#pragma unroll
        for (int l = 0; l < L; ++l)
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int k = 0; k < 3; ++k) acc[l][b][k] = fmaf(g[k], sv[l][b][k], acc[l][b][k]);
    }
    __shared__ float red[4][NLB];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float t = wave_sum_lane63(acc[l][b][k]);
                if (lane == 63) red[wave][(l * B + b) * 3 + k] = t;
            }
    __syncthreads();
    if (threadIdx.x < L * B * 3) {
        const int idx = threadIdx.x;
        const float t = (red[0][idx] + red[1][idx]) + (red[2][idx] + red[3][idx]);
        partial[((int64_t)v * gridDim.x + blockIdx.x) * NLB + idx] = t;
    }
}

// One wave per block of outputs in turn (block_samples), one view per
// blockIdx.y and one component k per blockIdx.z: the lanes' products with
// g_dvf are kept per channel in LDS (each lane its own word), reduced over the
// wave and the workgroup at the end.  One view, B = 3, three levels at
// 256x256x128: 489 us with a voxel per thread, now 202 us.  Where the blocks
// are not filled or few, a voxel per thread is faster (k_combine_bwd_coeff
// first): 256 x 256 x 44 (704 outputs per block) B = 1 one view 62 / 53, three
// 143 / 140; x 40 129 / 139 (three); x 32 (512) B = 2 76 / 74, three views 193 / 199;
// 512x512x2 B = 1 eight views 0.26 / 1.45 ms the call; 64^3 (256 blocks) B = 1 one
// view 11 / 14, two 16 / 16; 32x32x64 (64) eight views 16 / 16; 88x88x64 (484) 17 / 16.
__global__ __launch_bounds__(256) void k_combine_bwd_coeff_block(
    LevelsK lv, GridK out, BlockGrid bg, const float *__restrict__ g_dvf,
    float *__restrict__ partial) {
    __shared__ float csum[4][MAXL * MAXB][64];
    __shared__ float red[4][MAXL * MAXB];
    const int nc = lv.L * lv.B;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int c = 0; c < nc; ++c) csum[wave][c][lane] = 0.0f;
    const int64_t N = grid_size(out);
    const int v = blockIdx.y, k = blockIdx.z;
    const float *gd = g_dvf + ((int64_t)v * 3 + k) * N;
    for (int w = (int)blockIdx.x * 4 + wave; w < bg.n; w += (int)gridDim.x * 4) {
        const int bz = w % bg.nz, by = (w / bg.nz) % bg.ny, bx = w / (bg.nz * bg.ny);
        const int ix0 = bx * 4, iy0 = by * 4, iz = bz * 64 + lane;
        const bool on = iz < out.n[2];
        float g[CXY];
#pragma unroll
        for (int i = 0; i < CXY; ++i) {
            const int ix = ix0 + i / 4, iy = iy0 + i % 4;
            const bool ok = on && ix < out.n[0] && iy < out.n[1];
            g[i] = ok ? gd[((int64_t)ix * out.n[1] + iy) * out.n[2] + iz] : 0.0f;
        }
#pragma unroll 1
        for (int l = 0; l < lv.L; ++l) {
            const AxisMap &m = lv.map[l];
            const LevelBlock b = level_block(m, out, ix0, iy0, iz, on);
            const int64_t Nl = (int64_t)m.n[0] * m.n[1] * m.n[2];
#pragma unroll 1
            for (int bb = 0; bb < lv.B; ++bb) {
                float t = 0.0f;
                block_samples(lv.E[l] + (int64_t)(bb * 3 + k) * Nl, b,
                              [&](int i, float x) { t = fmaf(g[i], x, t); });
                csum[wave][l * lv.B + bb][lane] += t;
            }
        }
    }
    for (int c = 0; c < nc; ++c) {
        const float t = wave_sum_lane63(csum[wave][c][lane]);
        if (lane == 63) red[wave][c] = t;
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < nc)
        partial[((int64_t)v * gridDim.x + blockIdx.x) * NLB + c * 3 + k] =
            (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

// g_coeff[v][l][b][k] = sum over blocks of the partials: one workgroup per
// output entry, fixed-order tree (deterministic).
__global__ __launch_bounds__(256) void k_reduce_coeff(const float *__restrict__ partial, int nblk,
                                                      int per, float *__restrict__ g_coeff) {
    const int t = blockIdx.x;
    const int v = t / per, idx = t % per;
    float s = 0.0f;
    for (int i = threadIdx.x; i < nblk; i += blockDim.x)
        s += partial[((int64_t)v * nblk + i) * NLB + idx];
    __shared__ float red[4];
    s = wave_sum_lane63(s);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) g_coeff[t] = (red[0] + red[1]) + (red[2] + red[3]);
}

// ----------------------------------------------------------- basis adjoint
// Source of the first pass without an input array: channel c of level l is
//   sum_v coeff[v][l][b][k] g_dvf[v][k][j]   (c = b*3 + k).
struct AdjSrc {
    const float *g_dvf;
    const float *coeff;
    int V, L, B, l;
    int64_t N;
};

__device__ __forceinline__ float adj_src(const AdjSrc &src, int c, int64_t j) {
    const int b = c / 3, k = c % 3;
    float s = 0.0f;
    for (int v = 0; v < src.V; ++v)
        s = fmaf(src.coeff[(((int64_t)v * src.L + src.l) * src.B + b) * 3 + k],
                 src.g_dvf[((int64_t)v * 3 + k) * src.N + j], s);
    return s;
}

struct Shape4 {
    int c, d[3];
};

// One 1-D transpose pass along axis `ax`, out[c][..p..] = sum_j W(j,p)
// in[c][..j..] with W(j,p) the forward's linear weight of level index p for
// fine index j.  Each line along `ax` is cut into nseg segments of outputs
// [p0, p1), one thread each (short or few lines would otherwise leave the
// pass latency-bound): the thread walks the line's input values from the
// first one that reaches p0, in order, each split between its two level
// cells (weights 1 - f and f, as the forward reads them), and emits its
// outputs in order (a cell is complete once the walk has passed it).  Every
// output sums its terms in ascending fine order whatever nseg is.
// SRC: the first pass without an input array (in: the others').
template <bool SRC>
__global__ __launch_bounds__(256) void k_adj_line(Shape4 in_s, int ax, int nc, float scale,
                                                  float off, int nseg,
                                                  const float *__restrict__ in, AdjSrc src,
                                                  float *__restrict__ out) {
    // lines: all index tuples of (c, d0, d1, d2) with the ax index fixed to 0
    int ld[3] = {in_s.d[0], in_s.d[1], in_s.d[2]};
    ld[ax] = 1;
    const int64_t nlines = (int64_t)in_s.c * ld[0] * ld[1] * ld[2];
    const int64_t tt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tt >= nlines * nseg) return;
    // segment-major, so neighbouring threads take neighbouring lines
    const int seg = (int)(tt / nlines);
    int64_t r = tt - (int64_t)seg * nlines;
    const int per = (nc + nseg - 1) / nseg;
    const int p0 = seg * per, p1 = min(nc, p0 + per);
    if (p0 >= p1) return;
    int idx[3];
    idx[2] = (int)(r % ld[2]);
    r /= ld[2];
    idx[1] = (int)(r % ld[1]);
    r /= ld[1];
    idx[0] = (int)(r % ld[0]);
    const int c = (int)(r / ld[0]);
    const int nf = in_s.d[ax];
    // input strides and base (channel-major [c][d0][d1][d2])
    const int64_t ist = ax == 2 ? 1 : (ax == 1 ? in_s.d[2] : (int64_t)in_s.d[1] * in_s.d[2]);
    const int64_t ibase = ((int64_t)idx[0] * in_s.d[1] + idx[1]) * in_s.d[2] + idx[2];
    const int64_t cbase = (int64_t)c * in_s.d[0] * in_s.d[1] * in_s.d[2];
    // output shape: ax dimension nc
    int od[3] = {in_s.d[0], in_s.d[1], in_s.d[2]};
    od[ax] = nc;
    const int64_t ost = ax == 2 ? 1 : (ax == 1 ? od[2] : (int64_t)od[1] * od[2]);
    const int64_t obase = (((int64_t)c * od[0] + idx[0]) * od[1] + idx[1]) * od[2] + idx[2];
    auto emit = [&](int p, float v) {
        if (p >= p0 && p < p1) out[obase + (int64_t)p * ost] = v;
    };
    // a value at cell i feeds outputs i and i + 1: start a little below the
    // first fine index whose cell is p0 - 1 (values below it are skipped)
    const int jlo = p0 == 0 ? 0 : max(0, (int)floorf(((float)(p0 - 1) - off) / scale) - 2);
    int next = p0;          // first output not yet written
    int cur = -1;           // cell of the pending pair (cur, cur + 1)
    float a0 = 0.0f, a1 = 0.0f;
    bool done = false;
    // The line's values are fetched ADJ_U at a time ahead of the walk (whose
    // branches would otherwise leave one load in flight per wave).
    constexpr int ADJ_U = 8;
    for (int j0 = jlo; j0 < nf && !done; j0 += ADJ_U) {
        float xs[ADJ_U];
#pragma unroll
        for (int u = 0; u < ADJ_U; ++u) {
            const int64_t jj = min(j0 + u, nf - 1);     // past the end: in range, unused
            if constexpr (SRC) xs[u] = adj_src(src, c, ibase + jj * ist);
            else xs[u] = in[cbase + ibase + jj * ist];
        }
#pragma unroll
        for (int u = 0; u < ADJ_U; ++u) {
            const int j = j0 + u;
            if (j >= nf) break;
            int i;
            float f;
            if (!axis_cell(fmaf((float)j, scale, off), nc, i, f)) continue;
            if (i < p0 - 1) continue;           // reaches no output of this segment
            if (i >= p1) {                      // nor does anything past it
                done = true;
                break;
            }
            if (i != cur) {
                // cells below i are complete: write them (zeros for cells no value reached)
                if (cur >= 0) {
                    emit(cur, a0);
                    next = cur + 1;
                    a0 = (cur + 1 == i) ? a1 : 0.0f;
                    if (cur + 1 < i) {
                        emit(cur + 1, a1);
                        next = cur + 2;
                    }
                } else {
                    a0 = 0.0f;
                }
                for (; next < i; ++next) emit(next, 0.0f);
                a1 = 0.0f;
                cur = i;
            }
            const float x = xs[u];
            a0 = fmaf(1.0f - f, x, a0);
            a1 = fmaf(f, x, a1);
        }
    }
    if (cur >= 0) {
        emit(cur, a0);
        emit(cur + 1, a1);
        next = max(next, cur + 2);
    }
    for (; next < p1; ++next) emit(next, 0.0f);
}

// out[b * 3 + k][i] = sum_v coeff[v][l][b][k] in[v * 3 + k][i], i < n: the
// bases' share of every view.  Component k per blockIdx.y; a value is read once
// for its B bases (a thread per output read it B times, with 64-bit divisions:
// 173 us for one view and three bases at 256x256x128, now 75 us).  VEC: n a
// multiple of 4 and both arrays 16-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(256) void k_adj_mix(const float *__restrict__ in,
                                                 const float *__restrict__ coeff, int V, int L,
                                                 int B, int l, int64_t n, float *__restrict__ out) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    using T = std::conditional_t<VEC, f4, float>;
    const int k = (int)blockIdx.y;
    const int64_t m = VEC ? n / 4 : n;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    T acc[MAXB];
#pragma unroll
    for (int b = 0; b < MAXB; ++b) acc[b] = T(0.0f);
    for (int v = 0; v < V; ++v) {
        const T x = ((const T *)in)[(v * 3 + k) * m + i];
        const float *c = coeff + ((int64_t)v * L + l) * B * 3 + k;
#pragma unroll
        for (int b = 0; b < MAXB; ++b)
            if (b < B) acc[b] = __builtin_elementwise_fma(T(c[b * 3]), x, acc[b]);
    }
#pragma unroll
    for (int b = 0; b < MAXB; ++b)
        if (b < B) ((T *)out)[(b * 3 + k) * m + i] = acc[b];
}

static hipError_t launch_adj_mix(const float *in, const float *coeff, int V, const LevelsK &lv, int l,
                                 int64_t n, float *out, hipStream_t s) {
    const bool vec = (n & 3) == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
    const dim3 nb((unsigned)(((vec ? n / 4 : n) + 255) / 256), 3);
    ProfScope prof_("upsample_adjoint", s);
    if (vec) k_adj_mix<true><<<nb, 256, 0, s>>>(in, coeff, V, lv.L, lv.B, l, n, out);
    else k_adj_mix<false><<<nb, 256, 0, s>>>(in, coeff, V, lv.L, lv.B, l, n, out);
    return hipGetLastError();
}

static void adj_plan(const GridK &out, const AxisMap &m, int C, int order[3], int &np,
                     size_t &bufA, size_t &bufB) {
    np = 0;
    for (int a = 0; a < 3; ++a)
        if (!m.ident[a]) order[np++] = a;
    int d[3] = {out.n[0], out.n[1], out.n[2]};
    size_t sz[3] = {0, 0, 0};
    for (int p = 0; p < np; ++p) {
        d[order[p]] = m.n[order[p]];
        sz[p] = (size_t)C * d[0] * d[1] * d[2];
    }
    bufA = np >= 2 ? sz[0] : 0;
    bufB = np >= 3 ? sz[1] : 0;
}

size_t upsample_adjoint_workspace(int C, const GridK &lvl_grid, const GridK &out, const AxisMap &m) {
    (void)lvl_grid;
    int order[3], np;
    size_t a, b;
    adj_plan(out, m, C, order, np, a, b);
    return align256(a * sizeof(float)) + align256(b * sizeof(float));
}

hipError_t launch_upsample_adjoint(const LevelsK &lv, int l, const GridK &lvl_grid,
                                   const float *coeff, int V, const GridK &out, const float *g_dvf,
                                   const float *G, float *g_base, void *ws, hipStream_t s) {
    (void)lvl_grid;
    const AxisMap &m = lv.map[l];
    const int C = 3 * lv.B;
    AdjSrc src;
    src.g_dvf = g_dvf;
    src.coeff = coeff;
    src.V = V;
    src.L = lv.L;
    src.B = lv.B;
    src.l = l;
    src.N = grid_size(out);
    int order[3], np;
    size_t a, b;
    adj_plan(out, m, C, order, np, a, b);
    // level grid equals the output grid: the mix of the views is the answer
    // (G then already is the answer and the caller does not ask)
    if (np == 0) return launch_adj_mix(g_dvf, coeff, V, lv, l, src.N, g_base, s);
    float *bufA = (float *)ws;
    float *bufB = (float *)((char *)ws + align256(a * sizeof(float)));
    // As many views as bases or fewer: the map is linear, so the views' own 3 V
    // channels go through it and are mixed on the level's grid.
    const bool mix = !G && V <= lv.B;
    float *const last = mix ? (float *)((char *)bufB + align256(b * sizeof(float))) : g_base;
    Shape4 sh;
    sh.c = mix ? 3 * V : C;
    sh.d[0] = out.n[0];
    sh.d[1] = out.n[1];
    sh.d[2] = out.n[2];
    const float *in = mix ? g_dvf : G;
    for (int p = 0; p < np; ++p) {
        const int ax = order[p];
        float *dst = (p == np - 1) ? last : (p == 0 ? bufA : bufB);
        Shape4 os = sh;
        os.d[ax] = m.n[ax];
        const int64_t lines = (int64_t)sh.c * sh.d[0] * sh.d[1] * sh.d[2] / sh.d[ax];
        // segments per line: enough threads to cover the pass's latency
        // (about 2^20: measured against 2^18 to 2^22), at least 8 outputs each
        int nseg = 1;
        while (2 * nseg <= m.n[ax] / 8 && lines * nseg < (1 << 20)) nseg *= 2;
        const int64_t threads = lines * nseg;
        {
            ProfScope prof_("upsample_adjoint", s);
            const unsigned nb = (unsigned)((threads + 255) / 256);
            if (in)
                k_adj_line<false><<<nb, 256, 0, s>>>(sh, ax, m.n[ax], m.scale[ax], m.off[ax], nseg, in, src, dst);
            else
                k_adj_line<true><<<nb, 256, 0, s>>>(sh, ax, m.n[ax], m.scale[ax], m.off[ax], nseg, in, src, dst);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        in = dst;
        sh = os;
    }
    return mix ? launch_adj_mix(last, coeff, V, lv, l, (int64_t)sh.d[0] * sh.d[1] * sh.d[2], g_base, s)
               : hipSuccess;
}

size_t combine_bwd_workspace(const LevelsK &lv, const GridK *lvl_grids, int V, const GridK &out) {
    size_t part = align256(sizeof(float) * (size_t)CB_BLOCKS * (size_t)V * NLB);
    size_t adj = 0;
    for (int l = 0; l < lv.L; ++l) {
        // the passes' buffers, then the views' channels on the level's grid
        const AxisMap &m = lv.map[l];
        size_t w = upsample_adjoint_workspace(3 * lv.B, lvl_grids[l], out, m);
        if (V <= lv.B && !(m.ident[0] && m.ident[1] && m.ident[2]))
            w += align256(sizeof(float) * 3 * (size_t)lv.B * (size_t)grid_size(lvl_grids[l]));
        if (w > adj) adj = w;
    }
    return part + adj;
}

hipError_t launch_combine_bwd(const LevelsK &lv, const GridK *lvl_grids, const float *coeff, int V,
                              const GridK &out, const float *g_dvf, float *const *g_bases,
                              float *g_coeff, void *ws, hipStream_t s) {
    const int per = lv.L * lv.B * 3;
    float *partial = (float *)ws;
    char *adjws = (char *)ws + align256(sizeof(float) * (size_t)CB_BLOCKS * (size_t)V * NLB);
    hipError_t e;
    int nblk;
    const BlockGrid bg = block_grid(out);
    if (use_blocks(lv, out, bg, (int64_t)bg.n * V, {704, 480}, {576, 480})) {
        nblk = std::min((bg.n + 3) / 4, CB_BLOCKS);
        ProfScope prof_("combine_bwd_coeff", s);
        k_combine_bwd_coeff_block<<<dim3((unsigned)nblk, (unsigned)V, 3), 256, 0, s>>>(
            lv, out, bg, g_dvf, partial);
        e = hipGetLastError();
    } else {
        nblk = (int)std::min<int64_t>((grid_size(out) + 255) / 256, CB_BLOCKS);
        e = dispatch_lb(lv.L, lv.B, [&](auto Lc, auto Bc) {
            constexpr int L = decltype(Lc)::value, B = decltype(Bc)::value;
            ProfScope prof_("combine_bwd_coeff", s);
            k_combine_bwd_coeff<L, B>
                <<<dim3((unsigned)nblk, (unsigned)V), 256, 0, s>>>(lv, out, g_dvf, partial);
            return hipGetLastError();
        });
    }
    if (e != hipSuccess) return e;
    const int tot = V * per;
    {
        ProfScope prof_("combine_bwd_reduce", s);
        k_reduce_coeff<<<(unsigned)tot, 256, 0, s>>>(partial, nblk, per, g_coeff);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int l = 0; l < lv.L; ++l) {
        e = launch_upsample_adjoint(lv, l, lvl_grids[l], coeff, V, out, g_dvf, nullptr, g_bases[l],
                                    adjws, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace pmf
