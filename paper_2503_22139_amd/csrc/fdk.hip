// fdk.hip -- FDK reconstruction (Feldkamp et al. 1984), the motion-averaged
// CBCT from which the Gaussians are initialised (Sec. 2.3.2).
//
// Circular orbit, flat detector, in the projector's geometry, written on the
// virtual detector through the isocentre (pitches scaled by SAD / SDD):
// cosine weighting SDD / sqrt(SDD^2 + a^2 + b^2); ramp filtering of each
// detector row with the discrete Ram-Lak kernel of the virtual pitch tau
// (h[0] = 1 / (4 tau^2), h[n odd] = -1 / (pi n tau)^2, rows zero-padded),
// q = tau (h * p~); voxel-driven back-projection f(x) = 1/2 sum_views
// dtheta (SAD / U)^2 q(a', b'), U the depth of x along the central ray,
// (a', b') = SAD (t_u, t_v) / U, bilinear between pixel centres (0 off the
// detector), dtheta = 2 pi / V.  The plain Ram-Lak kernel, linear
// interpolation and full-scan weighting 1/2 are the readings of the paper's
// "quick FDK reconstruction".
//
// Layout of the filtered projections (workspace): per view a zero-bordered
// plane of (nv + 2) x (nu + 3) pairs; pair (j, c) holds qp(j, c), qp(j + 1, c)
// of the padded image qp(j, c) = q[j - 1][c - 1] (0 on the border and beyond),
// so the 2 x 2 taps at (j, c) are the 16 contiguous bytes of pairs c and c + 1.
// A back-projection sample clamps its padded pixel coordinates into
// [0, nu + 1] x [0, nv + 1] -- any sample that leaves the detector then reads
// zero taps, exactly as the definition asks -- and fetches its whole 2 x 2
// neighbourhood with one 16-byte load, with no bounds test.  (Quads of all
// four taps, 16 bytes per pixel, took the same load but twice the memory: a
// workgroup's patch of a view, 45 KB, then missed the 32 KB L1.)
#include <math.h>

#include <algorithm>

#include "pmf_internal.h"

namespace pmf {

constexpr int BP_ZC = 16;              // voxels along axis 2 per back-projection thread

// ---------------------------------------------------------------- filter
// The ramp filter of a row, q[n] = sum_m h[n - m] p~[m] (h[0] = 1 / (4 tau),
// h[d odd] = -1 / (pi^2 tau d^2)), as a circular convolution of length M =
// 2^P >= 2 nu - 1 by FFT.  h is even, so its transform is real, and two rows
// are filtered at once as the real and imaginary parts of one sequence.  All
// of it is double: for smooth rows on fine pixels q is a small difference of
// large terms.  The transform's errors go by the larger of its two rows, so the
// second is first scaled by a power of two to the first's size (exact; beside a
// dead pixel of 3e38 nothing would be left of the other row).  The direct sum
// over odd lags (~nu / 2 double FMAs per output, issue-bound) took 1.6 ms for
// 660 views of 512x384; the transforms' ~90 per output leave 1.0 ms.
//
// Transform: 16 points per thread; in-place decimation-in-frequency passes of
// radix 16 and a last one of radix 2^(P mod 4) (16 when that is 1), whose
// digit-reversed output is what the inverse's passes, the same in reverse,
// take as input -- no reordering, and the last forward pass, the product and
// the first inverse pass stay in registers.  LDS holds the sequence between
// passes; its index is XORed so that 16 neighbouring lanes hit distinct 16-byte
// banks in every pass (measured on the 1024-point passes, strides 64, 4 and 1).
typedef double2 cplx;

__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
    return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return {a.x - b.x, a.y - b.y}; }

// In-place DFTs (INV: the conjugate transform, unscaled).  X[k] lands at
// dft_slot<R>(k).
template <bool INV>
__device__ __forceinline__ void dft2(cplx &a, cplx &b) {
    const cplx s = cadd(a, b);
    b = csub(a, b);
    a = s;
}
template <bool INV>
__device__ __forceinline__ void dft4(cplx &a, cplx &b, cplx &c, cplx &d) {
    const cplx t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), u = csub(b, d);
    const cplx t3 = INV ? cplx{-u.y, u.x} : cplx{u.y, -u.x};      // -+i (b - d)
    a = cadd(t0, t2);
    b = cadd(t1, t3);
    c = csub(t0, t2);
    d = csub(t1, t3);
}
// a * exp(-+2 pi i k / 16)
template <bool INV, int K>
__device__ __forceinline__ cplx rot16(cplx a) {
    constexpr double C[16] = {1.0, 0.92387953251128675613, 0.70710678118654752440,
                              0.38268343236508977173, 0.0, -0.38268343236508977173,
                              -0.70710678118654752440, -0.92387953251128675613, -1.0,
                              -0.92387953251128675613, -0.70710678118654752440,
                              -0.38268343236508977173, 0.0, 0.38268343236508977173,
                              0.70710678118654752440, 0.92387953251128675613};
    if constexpr (K == 0) return a;
    else return cmul(a, cplx{C[K], INV ? C[(K + 12) % 16] : -C[(K + 12) % 16]});
}
template <int R>
__device__ constexpr int dft_slot(int k) {
    return R == 16 ? 4 * (k % 4) + k / 4 : R == 8 ? 2 * (k % 4) + k / 4 : k;
}
// The 16-point DFT, in two levels of dft4.  HALF: its upper eight inputs are 0
// (forward) or its upper eight outputs are not wanted (inverse), as in the
// pass that holds the row: the row fills at most half of the transform.
template <bool INV, bool HALF>
__device__ __forceinline__ void dft16(cplx *x) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if constexpr (HALF && !INV) {
            const cplx a = x[j], b = x[j + 4], ib = {b.y, -b.x};        // -i b
            x[j] = cadd(a, b);
            x[j + 4] = cadd(a, ib);
            x[j + 8] = csub(a, b);
            x[j + 12] = csub(a, ib);
        } else {
            dft4<INV>(x[j], x[j + 4], x[j + 8], x[j + 12]);
        }
    }
    x[5] = rot16<INV, 1>(x[5]);
    x[9] = rot16<INV, 2>(x[9]);
    x[13] = rot16<INV, 3>(x[13]);
    x[6] = rot16<INV, 2>(x[6]);
    x[10] = rot16<INV, 4>(x[10]);
    x[14] = rot16<INV, 6>(x[14]);
    x[7] = rot16<INV, 3>(x[7]);
    x[11] = rot16<INV, 6>(x[11]);
    x[15] = rot16<INV, 9>(x[15]);
#pragma unroll
    for (int k = 0; k < 16; k += 4) {
        if constexpr (HALF && INV) {            // outputs k / 4 and k / 4 + 4 only
            const cplx a = x[k], b = x[k + 1], c = x[k + 2], d = x[k + 3];
            const cplx u = csub(b, d);
            x[k] = cadd(cadd(a, c), cadd(b, d));
            x[k + 1] = cadd(csub(a, c), cplx{-u.y, u.x});
        } else {
            dft4<INV>(x[k], x[k + 1], x[k + 2], x[k + 3]);
        }
    }
}

template <bool INV, int R>
__device__ __forceinline__ void dft(cplx *x) {
    if constexpr (R == 2) {
        dft2<INV>(x[0], x[1]);
    } else if constexpr (R == 4) {
        dft4<INV>(x[0], x[1], x[2], x[3]);
    } else if constexpr (R == 8) {
        dft4<INV>(x[0], x[2], x[4], x[6]);
        dft4<INV>(x[1], x[3], x[5], x[7]);
        x[3] = rot16<INV, 2>(x[3]);
        x[5] = rot16<INV, 4>(x[5]);
        x[7] = rot16<INV, 6>(x[7]);
#pragma unroll
        for (int k = 0; k < 8; k += 2) dft2<INV>(x[k], x[k + 1]);
    } else {
        dft16<INV, false>(x);
    }
}

// A copy of u that the compiler cannot connect with it: addresses derived from
// it are computed where they are used.  (Kept across the passes and the loop
// over rows they took 150 registers, and with them two waves in three.)
__device__ __forceinline__ int fresh(int u) {
    asm volatile("" : "+v"(u));
    return u;
}

__device__ __forceinline__ int fft_at(int i) { return i ^ ((i >> 4) & 3) ^ (((i >> 6) & 3) << 2); }

template <int P>
struct Fft {
    static constexpr int M = 1 << P;
    static constexpr int TPP = M / 16;                          // threads per transform
    static constexpr int NP = P % 4 == 0 ? P / 4 - 1 : P / 4;   // radix-16 passes
    static constexpr int LR = P % 4 == 0 ? 16 : 1 << (P % 4);   // radix of the last pass
    static constexpr int G = 16 / LR;                           // its groups per thread
    static constexpr int THREADS = TPP < 64 ? 64 : TPP;
    static constexpr int PER = THREADS / TPP;                   // transforms per workgroup
    static constexpr int WAVES = P <= 10 ? 3 : 2;               // per SIMD: LDS (16 bytes a point) leaves 2.5

    // first point and spacing of thread u's 16 points in pass p
    static __device__ __forceinline__ int first(int p, int u) {
        const int S = (M >> (4 * p)) / 16;
        return (u / S) * 16 * S + u % S;
    }
    static __device__ __forceinline__ constexpr int step(int p) { return (M >> (4 * p)) / 16; }

    // x[k] *= exp(-+2 pi i t k / L), L = M >> 4p the pass's block, t the
    // thread's place in its sixteenth
    template <bool INV>
    static __device__ __forceinline__ void twiddle(cplx *x, const cplx *__restrict__ tw, int p,
                                                   int u, const int *slot) {
        const int t = u % step(p);
        auto root = [&](int k) {
            const cplx w = tw[(t * k) << (4 * p)];
            return cplx{w.x, INV ? -w.y : w.y};
        };
        auto mul = [&](int k, cplx w) { x[slot[k]] = cmul(x[slot[k]], w); };
        // four roots read, the others as products (at most two deep)
        const cplx w1 = root(1), w2 = root(2), w3 = cmul(w1, w2);
        mul(1, w1);
        mul(2, w2);
        mul(3, w3);
#pragma unroll
        for (int h = 4; h < 16; h += 4) {
            const cplx w = h < 12 ? root(h) : cmul(root(4), root(8));
            mul(h, w);
            mul(h + 1, cmul(w, w1));
            mul(h + 2, cmul(w, w2));
            mul(h + 3, cmul(w, w3));
        }
    }

    // x: the thread's points of pass 0 on entry (HALF: x[8..] are 0 and not
    // read), of the last pass on return (in slot order)
    template <bool HALF>
    static __device__ __forceinline__ void forward(cplx *x, cplx *sh, const cplx *__restrict__ tw,
                                                   int id) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int u = fresh(id);
            constexpr int slot[16] = {0, 4, 8, 12, 1, 5, 9, 13, 2, 6, 10, 14, 3, 7, 11, 15};
            const int b = first(p, u), S = step(p);
            if (p > 0) {
#pragma unroll
                for (int j = 0; j < 16; ++j) x[j] = sh[fft_at(b + j * S)];
            }
            if (p == 0) dft16<false, HALF>(x);
            else dft16<false, false>(x);
            twiddle<false>(x, tw, p, u, slot);
#pragma unroll
            for (int k = 0; k < 16; ++k) sh[fft_at(b + k * S)] = x[slot[k]];
            __syncthreads();
        }
        const int u = fresh(id);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int b = (u + q * TPP) * LR;
#pragma unroll
            for (int j = 0; j < LR; ++j) x[q * LR + j] = sh[fft_at(b + j)];
            dft<false, LR>(x + q * LR);
        }
    }

    // the inverse, from the last pass's points (slot order) to the lower eight
    // of pass 0's (point j at dft_slot<16>(j))
    static __device__ __forceinline__ void inverse(cplx *x, cplx *sh, const cplx *__restrict__ tw,
                                                   int id) {
        constexpr int same[16] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15};
        const int ul = fresh(id);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int b = (ul + q * TPP) * LR;
            cplx y[LR];
#pragma unroll
            for (int k = 0; k < LR; ++k) y[k] = x[q * LR + dft_slot<LR>(k)];
            dft<true, LR>(y);
#pragma unroll
            for (int j = 0; j < LR; ++j) sh[fft_at(b + j)] = y[dft_slot<LR>(j)];
        }
        __syncthreads();
#pragma unroll
        for (int p = NP - 1; p >= 0; --p) {
            const int u = fresh(id);
            const int b = first(p, u), S = step(p);
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = sh[fft_at(b + k * S)];
            twiddle<true>(x, tw, p, u, same);
            if (p == 0) {
                dft16<true, true>(x);
            } else {
                dft16<true, false>(x);
#pragma unroll
                for (int j = 0; j < 16; ++j) sh[fft_at(b + j * S)] = x[dft_slot<16>(j)];
                __syncthreads();
            }
        }
    }
};

struct FdkView {
    float ct, st, sx, sy;    // cos, sin, source position SAD (cos, sin)
};

// Views' sources, and the FFT's twiddles exp(-2 pi i m / M), m < M.
__global__ void k_fdk_tables(const float *__restrict__ angles, int V, float sad,
                             FdkView *__restrict__ out, int M, cplx *__restrict__ tw) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < V) {
        const double th = angles[i], ct = cos(th), st = sin(th);
        out[i] = {(float)ct, (float)st, (float)(sad * ct), (float)(sad * st)};
    }
    if (i < M) {
        double s, c;
        sincospi(2.0 * i / M, &s, &c);
        tw[i] = {c, -s};
    }
}

// 1 / sqrt(s) for a positive s: the hardware's estimate and two Newton steps
// (each squares its relative error), a few ulp.
__device__ __forceinline__ double rsqrt_nr(double s) {
    double y = __builtin_amdgcn_rsq(s);
#pragma unroll
    for (int k = 0; k < 2; ++k) y = fma(0.5 * y, fma(-(s * y), y, 1.0), y);
    return y;
}

// Transform of the filter's taps over M (real), in the order of the last
// pass's points.  One workgroup.
template <int P>
__global__ __launch_bounds__(Fft<P>::THREADS) void k_fdk_ramp(double tau, int nu,
                                                              const cplx *__restrict__ tw,
                                                              double *__restrict__ H) {
    using F = Fft<P>;
    __shared__ cplx sh[F::PER * F::M];
    const int u = threadIdx.x % F::TPP;
    cplx x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int m = F::first(0, u) + j * F::step(0);
        const int d = m < nu ? m : F::M - m;            // lag; |lag| < nu or no tap
        const double dd = (double)d;
        x[j] = {d >= nu ? 0.0 : d == 0 ? 0.25 / tau : (d & 1) ? -1.0 / (M_PI * M_PI * tau * dd * dd) : 0.0,
                0.0};
    }
    F::template forward<false>(x, sh + (threadIdx.x / F::TPP) * F::M, tw, u);
    if ((int)threadIdx.x >= F::TPP) return;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        H[(u + (i / F::LR) * F::TPP) * F::LR + i % F::LR] = x[i].x / (double)F::M;
}

// 2^e, |e| < 1022.
__device__ __forceinline__ double pow2(int e) {
    return __longlong_as_double((long long)(1023 + e) << 52);
}
// The top word of |x|: ordered like |x|, its upper 11 bits the exponent.
__device__ __forceinline__ uint32_t top_word(double x) { return (uint32_t)__double2hiint(x) & 0x7fffffffu; }

// The values of a thread's eight points of two rows that are not finite.  Every
// tap of an odd lag is negative, so such a value adds -+infinity (or NaN) to
// every output of the other parity, whatever the lag, and to its own place the
// centre tap's +-infinity.
struct BadPixels {
    uint32_t own = 0;       // 2 bits per point and row: 1 +infinity, 2 -infinity, 3 NaN
    uint32_t kinds = 0;     // the rows': 3 bits per row and parity, one per code
    __device__ __forceinline__ void take(double x, int row, int k, int parity) {
        if (top_word(x) < 0x7ff00000u) return;
        const uint32_t code = x != x ? 3u : x > 0.0 ? 1u : 2u;
        own |= code << (4 * k + 2 * row);
        kinds |= 1u << (6 * row + 3 * parity + code - 1);
    }
    // what they add to the output at point k
    __device__ __forceinline__ float term(int row, int k, int parity) const {
        const uint32_t code = own >> (4 * k + 2 * row) & 3u, other = kinds >> (6 * row + 3 * (1 - parity));
        float t = code == 1u ? INFINITY : code == 2u ? -INFINITY : code == 3u ? NAN : 0.0f;
        if (other & 1u) t -= INFINITY;
        if (other & 2u) t += INFINITY;
        return other & 4u ? NAN : t;
    }
};

// Filters `rows` rows of one view per transform slot, two at a time, and
// writes them into the padded plane's pairs: padded row i + 1 holds rows i and
// i + 1, so a row is kept until the next one is there, and only the slot's
// first and last padded rows are written by halves (the neighbours write the
// others).  The plane's border columns and rows are written too.
constexpr int FDK_ROWS = 8;
constexpr int64_t FDK_FEW = 2560;      // workgroups that the chip holds at once

template <int P>
__global__ __launch_bounds__(Fft<P>::THREADS)
__attribute__((amdgpu_waves_per_eu(Fft<P>::WAVES))) void k_fdk_filter(const float *__restrict__ proj,
                                                                pmf_cone_t c, double tau,
                                                                const cplx *__restrict__ tw,
                                                                const double *__restrict__ H, int rows,
                                                                float2 *__restrict__ qq) {
    using F = Fft<P>;
    __shared__ cplx smem[F::PER * F::M];
    __shared__ ushort2 wexp[F::THREADS / 64];       // the pair's largest exponents, by wave
    static_assert(F::step(0) % 2 == 0, "a thread's outputs have one parity");
    const int nu = c.nu, nv = c.nv, pitch = nu + 3;
    const int u = threadIdx.x % F::TPP, v = blockIdx.y;
    cplx *const sh = smem + (threadIdx.x / F::TPP) * F::M;
    const int r0 = ((int)blockIdx.x * F::PER + (int)threadIdx.x / F::TPP) * rows;
    const int r1 = min(r0 + rows, nv);          // r0 >= nv: the slot only keeps the barriers
    float2 *const plane = qq + (int64_t)v * (nv + 2) * pitch;
    const double sdd = c.sdd;
    constexpr int S = F::step(0);
    // padded row j, columns 1 .. nu at this thread's points, and the border
    // columns; HALF: 0 both of a pair, 1 the first, 2 the second
    auto store = [&](int j, int half, const float *top, const float *bot) {
        float2 *const row = plane + (int64_t)j * pitch;
        const int b0 = F::first(0, fresh(u));
        auto put = [&](int col, float a, float b) {
            if (half == 0) row[col] = make_float2(a, b);
            else if (half == 1) row[col].x = a;
            else row[col].y = b;
        };
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int n = b0 + k * S;
            if (n < nu) put(n + 1, top[k], bot[k]);
        }
        if (u < 3) put(u == 0 ? 0 : nu + u, 0.0f, 0.0f);
    };
    float prev[8], zero[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) prev[k] = zero[k] = 0.0f;
#pragma unroll 1
    for (int q = 0; q < rows; q += 2) {
        const int i = r0 + q;
        auto pixel = [&](int i, int n) {            // cosine-weighted rows i, i + 1
            const double ba = ((double)i - 0.5 * (nv - 1) + c.off_v) * c.dv;
            const double bb = ((double)(i + 1) - 0.5 * (nv - 1) + c.off_v) * c.dv;
            const double sa = sdd * sdd + ba * ba, sb = sdd * sdd + bb * bb;
            const float *row = proj + ((int64_t)v * nv + i) * nu;
            const double a = ((double)n - 0.5 * (nu - 1) + c.off_u) * c.du, aa = a * a;
            return cplx{i < r1 ? (double)row[n] * (sdd * rsqrt_nr(sa + aa)) : 0.0,
                        i + 1 < r1 ? (double)row[nu + n] * (sdd * rsqrt_nr(sb + aa)) : 0.0};
        };
        cplx x[16];
        uint32_t ma = 0, mb = 0;
        const int b0 = F::first(0, fresh(u));
#pragma unroll
        for (int k = 0; k < 8; ++k) {           // n < M / 2 covers the row
            const int n = b0 + k * S;
            x[k] = n < nu ? pixel(i, n) : cplx{0.0, 0.0};
            ma = max(ma, top_word(x[k].x));
            mb = max(mb, top_word(x[k].y));
        }
        // the rows' largest exponents, as they stand in the top words
        typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
        u16x2 ex;
        auto row_exponents = [&]() {
            ex = u16x2{(uint16_t)(ma >> 20), (uint16_t)(mb >> 20)};
#pragma unroll
            for (int o = 1; o < (F::TPP < 64 ? F::TPP : 64); o <<= 1)
                ex = __builtin_elementwise_max(
                    ex, __builtin_bit_cast(u16x2, __shfl_xor(__builtin_bit_cast(int, ex), o, 64)));
            if (F::TPP > 64 && (threadIdx.x & 63) == 0) wexp[threadIdx.x >> 6] = make_ushort2(ex.x, ex.y);
        };
        row_exponents();
        // (not finite; a workgroup of one wave needs no barrier's vote)
        const bool any = ex.x == 0x7ff || ex.y == 0x7ff;
        const bool bad = F::THREADS == 64 ? __ballot(any) != 0
                                          : __builtin_amdgcn_readfirstlane(__syncthreads_or(any)) != 0;
        if (bad) {
            // Values that are not finite would spread over both rows of the
            // transform: they are left out of it and their terms added after it.
            __syncthreads();
            ma = mb = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (top_word(x[k].x) >= 0x7ff00000u) x[k].x = 0.0;
                if (top_word(x[k].y) >= 0x7ff00000u) x[k].y = 0.0;
                ma = max(ma, top_word(x[k].x));
                mb = max(mb, top_word(x[k].y));
            }
            row_exponents();
            __syncthreads();
        }
        int ea = ex.x, eb = ex.y;
        if constexpr (F::TPP > 64) {
#pragma unroll
            for (int w = 0; w < F::THREADS / 64; ++w) {
                ea = max(ea, (int)wexp[w].x);
                eb = max(eb, (int)wexp[w].y);
            }
        }
        // (a row of zeros counts as 2^-300, below any float: the other's
        // errors then round to zero in it)
        ea = max(ea, 1023 - 300);
        eb = max(eb, 1023 - 300);
        const double down = pow2(ea - eb);
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k].y *= down;
        F::template forward<true>(x, sh, tw, u);
        const int uh = fresh(u);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const double h = H[(uh + (k / F::LR) * F::TPP) * F::LR + k % F::LR];
            x[k].x *= h;
            x[k].y *= h;
        }
        F::inverse(x, sh, tw, u);
        __syncthreads();                        // sh is free for the next two rows
        const double up = pow2(eb - ea);
        float qa[8], qb[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            qa[k] = (float)x[dft_slot<16>(k)].x;
            qb[k] = (float)(x[dft_slot<16>(k)].y * up);
        }
        if (bad) {
            // (the rows are read again, and the transform's LDS used: nothing of
            // this is kept through the passes)
            const int bn = F::first(0, fresh(u)), ii = fresh(i);
            BadPixels bp;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (bn + k * S >= nu) continue;
                const cplx p = pixel(ii, bn + k * S);
                bp.take(p.x, 0, k, bn & 1);
                bp.take(p.y, 1, k, bn & 1);
            }
            uint32_t *const kinds = (uint32_t *)sh;
            if (u == 0) *kinds = 0;
            __syncthreads();
            if (bp.kinds) atomicOr(kinds, bp.kinds);
            __syncthreads();
            bp.kinds = *kinds;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                qa[k] += bp.term(0, k, bn & 1);
                qb[k] += bp.term(1, k, bn & 1);
            }
            __syncthreads();                    // sh is free again
        }
        if (i < r1) {
            store(i, q > 0 || i == 0 ? 0 : 2, prev, qa);
            if (i + 1 < r1) store(i + 1, 0, qa, qb);
#pragma unroll
            for (int k = 0; k < 8; ++k) prev[k] = i + 1 < r1 ? qb[k] : qa[k];
        }
    }
    if (r0 >= nv) return;
    store(r1, r1 == nv ? 0 : 1, prev, zero);
    if (r1 == nv) store(nv + 1, 0, zero, zero);
}

// Smallest transform that holds a row's linear convolution.
static int fdk_log2(int nu) {
    int P = 6;
    while ((1 << P) < 2 * nu - 1) ++P;
    return P;
}

template <int P>
static hipError_t fdk_filter(const float *proj, const pmf_cone_t &c, int V, double tau,
                             const cplx *tw, double *H, float2 *qq, hipStream_t s) {
    using F = Fft<P>;
    k_fdk_ramp<P><<<1, F::THREADS, 0, s>>>(tau, c.nu, tw, H);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // eight rows per slot (whole padded rows are stored for all but its ends),
    // two where that leaves the chip idle: a slot's pairs wait for each other
    // (whole call, eight / two rows: one view of 512x384 49 / 28 us, four 61 / 42)
    const int64_t pairs = (int64_t)(c.nv + 1) / 2 * V;
    const int rows = pairs <= FDK_FEW * F::PER ? 2 : FDK_ROWS;
    const int slots = (c.nv + rows - 1) / rows;
    ProfScope prof_("fdk_filter", s);
    k_fdk_filter<P><<<dim3((unsigned)((slots + F::PER - 1) / F::PER), (unsigned)V), F::THREADS, 0, s>>>(
        proj, c, tau, tw, H, rows, qq);
    return hipGetLastError();
}

struct FdkBp {
    float sad, inv_tu, inv_tv, cu, cv, umax, vmax, wsc, hz;
    unsigned row_bytes;      // (nu + 3) * 8
    int64_t plane_bytes;     // (nv + 2) * row_bytes
    int tx, ty;              // 16 x 16 column tiles along axes 0, 1
};

typedef float taps __attribute__((ext_vector_type(4), aligned(8)));

// Workgroup = 16 x 16 voxel columns (each wave an 8 x 8 patch, so one wave's
// samples of a view fall on a few neighbouring detector cache lines) x
// BP_ZC voxels along axis 2 per thread.  Per view the column's geometry
// (depth U, magnification, u coordinate) is computed once; along the column
// only v moves, linearly.  Views are summed in order.  Workgroups are
// numbered so that each XCD gets a contiguous slab along axis 2 (one band of
// detector rows in every view).  Threads past the grid edge compute on
// clamped positions and store nothing.
// Bound by the L1: a load of 64 lanes takes a tag lookup per cache line that
// each four lanes touch and two cycles more per miss (22.3 lookups and 2.6
// misses: 4.31 ms for 660 views onto 256x256x128; with lanes row by row
// instead of in Morton order 24.6 lookups, 4.37 ms; with 16-byte quads per
// pixel 4.71 ms).  Lanes along the rays (views in two groups) measured no
// fewer lookups.
__global__ __launch_bounds__(256, 8) void k_fdk_bp(const float2 *__restrict__ qq, FdkBp p,
                                                const FdkView *__restrict__ views, int V, GridK g,
                                                float *__restrict__ vol) {
    const int b = xcd_block(blockIdx.x, gridDim.x);
    const int tiles = p.tx * p.ty;
    const int zc = b / tiles, tile = b - zc * tiles;
    const int tyi = tile / p.tx, txi = tile - tyi * p.tx;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // the lane's column of the wave's 8 x 8, in Morton order
    const int mx = (lane & 1) | ((lane >> 1) & 2) | ((lane >> 2) & 4);
    const int my = ((lane >> 1) & 1) | ((lane >> 2) & 2) | ((lane >> 3) & 4);
    const int ix = txi * 16 + (w & 1) * 8 + mx, iy = tyi * 16 + (w >> 1) * 8 + my;
    const int iz0 = zc * BP_ZC;
    const float x = g.c0[0] + min(ix, g.n[0] - 1) * g.h[0];
    const float y = g.c0[1] + min(iy, g.n[1] - 1) * g.h[1];
    const float z0 = g.c0[2] + iz0 * g.h[2];
    float acc[BP_ZC];
#pragma unroll
    for (int k = 0; k < BP_ZC; ++k) acc[k] = 0.0f;
    const char *pl = (const char *)qq;
    for (int v = 0; v < V; ++v, pl += p.plane_bytes) {
        const FdkView w = views[v];
        const float dx = x - w.sx, dy = y - w.sy;
        const float tu = fmaf(-w.st, dx, w.ct * dy);
        const float U = -fmaf(w.ct, dx, w.st * dy);
        const float r = p.sad / U;
        const float fu = __builtin_amdgcn_fmed3f(fmaf(r * tu, p.inv_tu, p.cu), 0.0f, p.umax);
        const float wu = __builtin_amdgcn_fractf(fu);
        const unsigned colb = (unsigned)(int)fu * 8u;
        const float wr2 = p.wsc * r * r;
        const float rv = r * p.inv_tv;
        const float fv0 = fmaf(rv, z0, p.cv), dfv = rv * p.hz;
#pragma unroll
        for (int k = 0; k < BP_ZC; ++k) {
            const float fv = __builtin_amdgcn_fmed3f(fmaf((float)k, dfv, fv0), 0.0f, p.vmax);
            const float wv = __builtin_amdgcn_fractf(fv);
            const unsigned off = __umul24((unsigned)(int)fv, p.row_bytes) + colb;
            // qp(j, c), (j + 1, c), (j, c + 1), (j + 1, c + 1)
            const taps e = *(const taps *)(pl + off);
            const float top = fmaf(wu, e.z - e.x, e.x), bot = fmaf(wu, e.w - e.y, e.y);
            acc[k] = fmaf(wr2, fmaf(wv, bot - top, top), acc[k]);
        }
    }
    if (ix >= g.n[0] || iy >= g.n[1]) return;
    float *o = vol + ((int64_t)ix * g.n[1] + iy) * g.n[2];
#pragma unroll
    for (int k = 0; k < BP_ZC; ++k)
        if (iz0 + k < g.n[2]) o[iz0 + k] = acc[k];
}

static size_t fdk_plane_bytes(const pmf_cone_t &c) {
    return sizeof(float2) * (size_t)(c.nu + 3) * (c.nv + 2);
}

// Workspace: the views' planes, the views, the FFT's twiddles and the ramp's
// transform.
size_t fdk_workspace(const pmf_cone_t &c, int V) {
    const size_t M = (size_t)1 << fdk_log2(c.nu);
    return align256(fdk_plane_bytes(c) * V) + align256(sizeof(FdkView) * (size_t)V) +
           align256(sizeof(cplx) * M) + align256(sizeof(double) * M);
}

hipError_t launch_fdk(const float *proj, const pmf_cone_t &c, const float *angles, int V,
                      const GridK &g, float *vol, void *ws, hipStream_t s) {
    char *w = (char *)ws;
    float2 *qq = (float2 *)w;
    w += align256(fdk_plane_bytes(c) * V);
    FdkView *views = (FdkView *)w;
    w += align256(sizeof(FdkView) * (size_t)V);
    const int P = fdk_log2(c.nu), M = 1 << P;
    cplx *tw = (cplx *)w;
    w += align256(sizeof(cplx) * (size_t)M);
    double *H = (double *)w;
    const double tau = (double)c.du * c.sad / c.sdd;
    hipError_t e;
    k_fdk_tables<<<(unsigned)((std::max(V, M) + 255) / 256), 256, 0, s>>>(angles, V, c.sad, views, M, tw);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    switch (P) {
        case 6: e = fdk_filter<6>(proj, c, V, tau, tw, H, qq, s); break;
        case 7: e = fdk_filter<7>(proj, c, V, tau, tw, H, qq, s); break;
        case 8: e = fdk_filter<8>(proj, c, V, tau, tw, H, qq, s); break;
        case 9: e = fdk_filter<9>(proj, c, V, tau, tw, H, qq, s); break;
        case 10: e = fdk_filter<10>(proj, c, V, tau, tw, H, qq, s); break;
        case 11: e = fdk_filter<11>(proj, c, V, tau, tw, H, qq, s); break;
        case 12: e = fdk_filter<12>(proj, c, V, tau, tw, H, qq, s); break;
        default: e = fdk_filter<13>(proj, c, V, tau, tw, H, qq, s); break;   // rows of at most 4096
    }
    if (e != hipSuccess) return e;
    FdkBp p;
    p.sad = c.sad;
    p.inv_tu = (float)((double)c.sdd / ((double)c.du * c.sad));
    p.inv_tv = (float)((double)c.sdd / ((double)c.dv * c.sad));
    p.cu = (float)(0.5 * (c.nu - 1) - c.off_u + 1.0);
    p.cv = (float)(0.5 * (c.nv - 1) - c.off_v + 1.0);
    p.umax = (float)(c.nu + 1);
    p.vmax = (float)(c.nv + 1);
    p.wsc = (float)(M_PI / V);
    p.hz = g.h[2];
    p.row_bytes = 8u * (unsigned)(c.nu + 3);
    p.plane_bytes = (int64_t)fdk_plane_bytes(c);
    p.tx = (g.n[0] + 15) / 16;
    p.ty = (g.n[1] + 15) / 16;
    const int64_t nb = (int64_t)p.tx * p.ty * ((g.n[2] + BP_ZC - 1) / BP_ZC);
    {
        ProfScope prof_("fdk_backproject", s);
        k_fdk_bp<<<(unsigned)nb, 256, 0, s>>>(qq, p, views, V, g, vol);
    }
    return hipGetLastError();
}

// Grid-based sampling of the FDK volume into initial Gaussians (Sec.
// 2.3.2): a lattice of m0 x m1 x m2 points evenly filling the volume box
// (point k at box_lo + (k + 1/2) box_len / m per axis, axis 2 fastest); each
// point keeps its position and the volume's trilinear value there as its
// density; isotropic scale s, identity rotation.
__global__ void k_grid_init(const float *__restrict__ vol, GridK g, int m0, int m1, int m2,
                            float s, float *__restrict__ mean, float *__restrict__ scale,
                            float *__restrict__ quat, float *__restrict__ value) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)m0 * m1 * m2) return;
    const int k2 = (int)(k % m2), k1 = (int)((k / m2) % m1), k0 = (int)(k / ((int64_t)m2 * m1));
    const int kk[3] = {k0, k1, k2}, mm[3] = {m0, m1, m2};
    float u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // voxel-unit coordinate of the point (voxel 0's centre at 0)
        const double ua = ((double)kk[a] + 0.5) * g.n[a] / mm[a] - 0.5;
        u[a] = (float)ua;
        mean[3 * k + a] = (float)(g.c0d[a] + ua * g.hd[a]);
        scale[3 * k + a] = s;
    }
    quat[4 * k + 0] = 1.0f;
    quat[4 * k + 1] = 0.0f;
    quat[4 * k + 2] = 0.0f;
    quat[4 * k + 3] = 0.0f;
    value[k] = sample_u(vol, g.n, u[0], u[1], u[2]);
}

hipError_t launch_grid_init(const float *vol, const GridK &g, const int m[3], float s,
                            float *mean, float *scale, float *quat, float *value, hipStream_t st) {
    const int64_t M = (int64_t)m[0] * m[1] * m[2];
    k_grid_init<<<(unsigned)((M + 255) / 256), 256, 0, st>>>(vol, g, m[0], m[1], m[2], s, mean,
                                                              scale, quat, value);
    return hipGetLastError();
}

}  // namespace pmf
