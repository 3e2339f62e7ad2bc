// History part (Section 5): type-1 NUFFT of the quadrature sources, the
// multiplier of eq. (sh_fourier), type-2 NUFFT at the targets.
//
//   spread    g_m = sum_j q_j phi(x_m - x_j) on a periodic fine grid of step h
//             (q = w sigma, w' f, w nu_x mu, w nu_y mu: eqs. (disrete_sigma_hat),
//             (rhs_vol) and the D transform of Section 5.1);
//   FFT       rocFFT real-to-complex, in place;
//   multiply  c_l = (h^4/P^2) m(k_l) G_l / phihat(k_l)^2 for S and V, and
//             (h^4/P^2) m(k_l) (-i k_l . G_l) / phihat(k_l)^2 for D, where
//             m(k) = exp(-delta(alpha^2 + |k|^2))/(alpha^2 + |k|^2) (eq. (sh))
//             and c_l = 0 outside the square |k_x|, |k_y| <= k_max;
//   FFT       rocFFT complex-to-real, in place;
//   interp    u(x) = sum_m phi(x - x_m) U_m.
//
// Spreading: one workgroup owns one 16x16 block of the fine grid and adds the
// windows of the sources that meet it (listed per block at plan time) as
// rank-4 updates on the FP64 matrix cores: every grid value is written
// exactly once, with no atomics and in a fixed summation order.
// Interpolation: where the targets are dense on the grid, one wavefront per
// non-empty block of grid cells on the matrix cores; else one workgroup per
// non-empty target tile stages the tile plus its window halo of the three
// result grids in LDS with coalesced row reads.
#include <type_traits>

#include "mhk_internal.h"

namespace mhk {

// threads per interpolation / spreading workgroup: a busy tile holds a few
// hundred targets, one per thread; a spreading block's list is dealt to NWV
// wavefronts in batches of 32
constexpr int HB = 256;
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int INTERP_NB = 4;   // densities per interpolation wavefront, sharing its window values
// doubles of LDS per spreading wavefront: 64 rows of W + 2 window values, the
// strengths of 32 sources in NF fields, 64 window corners
constexpr int SPREAD_LDS(int W, int NF) { return 64 * (W + 2) + NF * 32 + 32; }

template <typename T>
struct SpreadArgs {
    int64_t n, field, nb, nv;
    int nblk, B;           // blocks per grid row
    int64_t nvw;           // workgroups of the volume: (active block, group of NV densities)
    int nvt, nbt;          // density groups of the volume and of the boundary (ND densities each)
    const int32_t *vact, *bact;
    const double *bgx, *bgy, *bw, *bwx, *bwy;
    const int32_t *bidx, *blofs, *blist;
    const double *vgx, *vgy, *vw;
    const int32_t *vidx, *vlofs, *vlist;
    const T *sigma, *mu, *f_vol;
    const T *wcoef;
    T *grid;               // [4][B][field]: S, V, Dx, Dy sources
};

// a b + c with c taken from scalar registers (the compiler copies a scalar
// addend into vector registers first: two more instructions per FP64 step)
__device__ inline double fma_s(double a, double b, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}
__device__ inline float fma_s(float a, float b, float c)
{
    float r;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// Window values phi(z_k), z_k = (m0 + k - g) 2/W, at the W grid points from
// m0 = ceil(g - W/2), from the per-point polynomials in t = 2(m0 - g + W/2) - 1
// (degree W + 3; the offset is formed in FP64).
// Window values at the W grid points of both axes of one source.  The
// window is even, so point W-1-k at offset t is point k at -t: with the
// polynomial of point k split into even and odd parts, p_k(t) = E(t^2) +
// t O(t^2), the pair is E +- t O, and half the polynomials serve all W
// points.  The coefficients are loaded with scalar loads inside the
// caller's loop (the empty asm keeps the compiler from hoisting all of them
// into vector registers), and each is used for both axes.
template <int W, typename T>
__device__ inline void window_weights2(double gx, double gy, const T *__restrict__ cf, int &mx0, int &my0, T *wx,
                                       T *wy)
{
    constexpr int D = W + 3;           // degree
    constexpr int NE = D / 2 + 1;      // even coefficients c_0, c_2, ...
    constexpr int NO = (D + 1) / 2;    // odd coefficients c_1, c_3, ...
    typedef const __attribute__((address_space(4))) T *ConstPtr;   // scalar-loadable
    ConstPtr cc = (ConstPtr)cf;
    asm volatile("" : "+s"(cc));
    mx0 = (int)ceil(gx - 0.5 * W);
    my0 = (int)ceil(gy - 0.5 * W);
    const T tx = (T)(2.0 * ((double)mx0 - gx + 0.5 * W) - 1.0);
    const T ty = (T)(2.0 * ((double)my0 - gy + 0.5 * W) - 1.0);
    const T sx = tx * tx, sy = ty * ty;
#pragma unroll
    for (int k = 0; k < (W + 1) / 2; ++k) {
        // the next point's coefficients are loaded only after this point's
        // inputs exist, which keeps 16 (not 8 W) coefficients live in SGPRs
        if (k > 0) asm volatile("" : "+s"(cc) : "v"(wx[k - 1]), "v"(wy[k - 1]));
        ConstPtr c = cc + k * (D + 1);
        T ex = c[2 * (NE - 1)], ey = ex;
#pragma unroll
        for (int j = NE - 2; j >= 0; --j) {
            ex = fma_s(ex, sx, c[2 * j]);
            ey = fma_s(ey, sy, c[2 * j]);
        }
        T ox = c[2 * (NO - 1) + 1], oy = ox;
#pragma unroll
        for (int j = NO - 2; j >= 0; --j) {
            ox = fma_s(ox, sx, c[2 * j + 1]);
            oy = fma_s(oy, sy, c[2 * j + 1]);
        }
        wx[k] = fma(tx, ox, ex);
        wy[k] = fma(ty, oy, ey);
        if (W - 1 - k != k) {
            wx[W - 1 - k] = fma(-tx, ox, ex);
            wy[W - 1 - k] = fma(-ty, oy, ey);
        }
    }
}

// Window values along one axis of one source, as above with one offset.
template <int W, typename T>
__device__ inline void window_weights1(double g, const T *__restrict__ cf, int &m0, T *w)
{
    constexpr int D = W + 3, NE = D / 2 + 1, NO = (D + 1) / 2;
    typedef const __attribute__((address_space(4))) T *ConstPtr;   // scalar-loadable
    ConstPtr cc = (ConstPtr)cf;
    asm volatile("" : "+s"(cc));
    m0 = (int)ceil(g - 0.5 * W);
    const T t = (T)(2.0 * ((double)m0 - g + 0.5 * W) - 1.0), s = t * t;
#pragma unroll
    for (int k = 0; k < (W + 1) / 2; ++k) {
        // two points' coefficients in flight
        if (k > 1) asm volatile("" : "+s"(cc) : "v"(w[k - 2]));
        ConstPtr c = cc + k * (D + 1);
        T e = c[2 * (NE - 1)];
#pragma unroll
        for (int j = NE - 2; j >= 0; --j) e = fma_s(e, s, c[2 * j]);
        T o = c[2 * (NO - 1) + 1];
#pragma unroll
        for (int j = NO - 2; j >= 0; --j) o = fma_s(o, s, c[2 * j + 1]);
        w[k] = fma(t, o, e);
        if (W - 1 - k != k) w[W - 1 - k] = fma(-t, o, e);
    }
}

// LDS exchange among the lanes of one wavefront
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The list [e0, e1) of one block into NF fields: sum_s q_f(s) w_y(s) (x) w_x(s),
// a product of a 16 x K matrix of y-window values, a diagonal of strengths and
// a K x 16 matrix of x-window values, four sources at a time on
// v_mfma_f64_16x16x4 (A: lane l holds row l % 16 of source l / 16, B: column
// l % 16 of source l / 16, D: rows 4 v + l / 16, column l % 16).  Each of the
// NWV wavefronts takes every NWV-th batch of 32 sources: lane l evaluates
// the W window values of axis l / 32 of source l % 32 (half the lanes' work
// of one thread per source, with scalar coefficients) into LDS rows of W + 2,
// the first and last of them zero, so that a row clamped to [-1, W] reads
// zero outside its window.  The windows of a list's sources cover 44% of the
// block's rows and columns (W = 12); skipping the rest would cost more than
// the matrix cores take.
template <int W, typename T, int NF, bool VOL, int NWV>
__device__ inline void spread_block(const SpreadArgs<T> &A, int b0, int nf, int x0, int y0, int e0, int e1,
                                    double *lds)
{
    constexpr int RW = W + 2;
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    double *row = lds + wave * SPREAD_LDS(W, NF);
    double *qs = row + 64 * RW;                       // [NF][32]
    int *ms = reinterpret_cast<int *>(qs + NF * 32);  // [2][32]
    d4 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = d4{0.0, 0.0, 0.0, 0.0};
    row[lane * RW] = 0.0;
    row[lane * RW + W + 1] = 0.0;
    const int axis = lane / 32, sl = lane % 32, i = lane % 16, k = lane / 16;
    const double *__restrict__ gc = axis ? (VOL ? A.vgy : A.bgy) : (VOL ? A.vgx : A.bgx);
    const int32_t *__restrict__ list = VOL ? A.vlist : A.blist, *__restrict__ idx = VOL ? A.vidx : A.bidx;
    // the volume's densities alternate between the two halves of the
    // wavefront; the lower half forms the boundary's strengths
    constexpr int NQ = VOL ? (NF + 1) / 2 : NF;
    const int step = 32 * NWV;
    struct Src {
        double g, w[3], f[NQ];
    };
    // loads run ahead of their use: the coordinate and the densities of the
    // next batch while this one is summed, the list entry one batch further
    auto load = [&](int s, Src &r) {
        const int id = idx[s];
        r.g = gc[s];
        if (VOL) {
            r.w[0] = A.vw[s];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int f = 2 * q + axis;
                r.f[q] = f < nf ? (double)A.f_vol[(size_t)(b0 + f) * A.nv + id] : 0.0;
            }
        } else {
            r.w[0] = A.bw[s];
            r.w[1] = A.bwx[s];
            r.w[2] = A.bwy[s];
#pragma unroll
            for (int d = 0; d < NF / 3; ++d) {
                const size_t o = (size_t)(b0 + d) * A.nb + id;
                r.f[3 * d] = A.sigma && 3 * d < nf ? (double)A.sigma[o] : 0.0;
                r.f[3 * d + 1] = r.f[3 * d + 2] = A.mu && 3 * d < nf ? (double)A.mu[o] : 0.0;
            }
        }
    };
    int e = e0 + 32 * wave + sl;
    Src cur{}, nxt{};
    int s1 = 0;
    if (e < e1) load(list[e], cur);
    if (e + step < e1) s1 = list[e + step];
    for (int base = e0 + 32 * wave; base < e1; base += step, e += step) {
        int s2 = 0;
        if (e + 2 * step < e1) s2 = list[e + 2 * step];
        if (e + step < e1) load(s1, nxt);
        int m = 1 << 20;                              // past the list's end: a window far outside, strength zero
        if (e < e1) {
            T w[W];
            window_weights1<W, T>(cur.g, A.wcoef, m, w);
            m -= axis ? y0 : x0;
#pragma unroll
            for (int q = 0; q < W; ++q) row[lane * RW + 1 + q] = (double)w[q];
        }
        const bool in = e < e1;
        if (VOL) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (2 * q + axis < NF) qs[(2 * q + axis) * 32 + sl] = in ? (double)(T)(cur.w[0] * cur.f[q]) : 0.0;
        } else if (axis == 0) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) qs[q * 32 + sl] = in ? (double)(T)(cur.w[q % 3] * cur.f[q]) : 0.0;
        }
        ms[lane] = m;
        // the wavefront's own LDS region: its lanes' writes are read below
        wave_sync();
#pragma unroll
        for (int g = 0; g < 32; g += 4) {
            const int src = g + k;
            const int ix = min(max(i - ms[src], -1), W) + 1, iy = min(max(i - ms[32 + src], -1), W) + 1;
            const double bx = row[src * RW + ix], ay = row[(32 + src) * RW + iy];
#pragma unroll
            for (int f = 0; f < NF; ++f)
                acc[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay, bx * qs[f * 32 + src], acc[f], 0, 0, 0);
        }
        wave_sync();
        cur = nxt;
        s1 = s2;
    }
    // the wavefronts' sums, in order, one field at a time
    const size_t fs = (size_t)A.B * A.field;
    const size_t o = (size_t)(y0 + tid / 16) * (A.n + 2) + x0 + tid % 16;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        if (f >= nf) break;
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) lds[wave * 256 + (4 * v + k) * 16 + i] = acc[f][v];
        __syncthreads();
        if (tid >= 256) continue;
        double sum = lds[tid];
#pragma unroll
        for (int q = 1; q < NWV; ++q) sum += lds[256 * q + tid];
        if (VOL) {
            A.grid[fs + (size_t)(b0 + f) * A.field + o] = (T)sum;
        } else {
            const int c = f % 3;                      // S in slot 0, D_x in 2, D_y in 3
            if (c == 0 ? A.sigma != nullptr : A.mu != nullptr)
                A.grid[(size_t)(c == 0 ? 0 : c + 1) * fs + (size_t)(b0 + f / 3) * A.field + o] = (T)sum;
        }
    }
}

// One workgroup per (active 16 x 16 block, group of densities): NV volume
// densities or ND boundary densities (S, D_x and D_y each).  The accumulators
// are FP64 at both precisions.  Bound by latency with the VALU a third and the
// matrix cores a fifth busy (waves wait for memory or LDS 58% of their cycles):
// per batch of 32 sources gathered loads and an LDS exchange around some 120
// instructions of window values, 90 of LDS addressing and 512 cycles of the
// matrix cores.  Measured alone, 1.04M volume
// and 16384 boundary sources on 1920^2, W = 12: 126 us (LDS atomic adds over
// 32 x 32 tiles: 312 us); 16 densities on 2880^2: 741 us (3013); 4.09M sources
// on 3840^2, W = 8, FP32: 215 us (430).  Blocks that no window meets are not
// launched: a workgroup each to write their zeros cost 50 us at 1920^2 and
// 70 us at 3840^2; the row transforms skip them by their flags.
template <int W, typename T, int NV, int ND, int NWV>
__global__ void __launch_bounds__(64 * NWV) k_spread(SpreadArgs<T> A)
{
    constexpr int NM = NV > 3 * ND ? NV : 3 * ND;
    constexpr int SZ = SPREAD_LDS(W, NM) * NWV;
    __shared__ double lds[SZ > 256 * NWV ? SZ : 256 * NWV];
    const bool vol = (int64_t)blockIdx.x < A.nvw;
    const int id = (int)(blockIdx.x - (vol ? 0 : A.nvw)), nt = vol ? A.nvt : A.nbt;
    const int blk = (vol ? A.vact : A.bact)[id / nt], b0 = id % nt * (vol ? NV : ND);
    const int nd = min(vol ? NV : ND, A.B - b0);
    const int x0 = blk % A.nblk * SPB, y0 = blk / A.nblk * SPB;
    if (vol)
        spread_block<W, T, NV, true, NWV>(A, b0, nd, x0, y0, A.vlofs[blk], A.vlofs[blk + 1], lds);
    else
        spread_block<W, T, 3 * ND, false, NWV>(A, b0, 3 * nd, x0, y0, A.blofs[blk], A.blofs[blk + 1], lds);
}

// Fourier multiplier on the half spectrum [n][n/2+1] of each field; the
// multiplier is formed in FP64 in both precision paths (it peaks at 1/alpha^2
// near k = 0).
template <typename T>
__global__ void __launch_bounds__(256) k_multiply(int64_t n, int B, int64_t field, T *grid,
                                                  const double *__restrict__ fac, double c, double alpha2,
                                                  double dk, const double *__restrict__ mtab, int lmax)
{
    const int64_t nh = n / 2 + 1;
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= n * nh * B) return;
    const int64_t lx = id % nh;
    const int64_t ly = (id / nh) % n;
    const int b = (int)(id / (nh * n));
    const int64_t fy = ly <= n / 2 ? ly : ly - n;
    const double ax = fac[lx], ay = fac[fy < 0 ? -fy : fy];
    const size_t fs = (size_t)B * field / 2;                  // complex values per field group
    typedef typename Vec2<T>::type T2;
    T2 *F = reinterpret_cast<T2 *>(grid) + (size_t)b * (field / 2) + ly * nh + lx;
    T2 zS = {0, 0}, zV = {0, 0}, zD = {0, 0};
    double M = 0.0;
    if (mtab) {
        if (lx <= lmax && fy >= -lmax && fy <= lmax) M = mtab[(fy + lmax) * (lmax + 1) + lx];
    } else if (ax != 0.0 && ay != 0.0) {
        const double kx = dk * lx, ky = dk * fy;
        M = c * ax * ay / (alpha2 + kx * kx + ky * ky);
    }
    if (M != 0.0) {
        const double kx = dk * lx, ky = dk * fy;
        const T2 s = F[0], v = F[fs], gx = F[2 * fs], gy = F[3 * fs];
        zS.x = (T)(M * s.x); zS.y = (T)(M * s.y);
        zV.x = (T)(M * v.x); zV.y = (T)(M * v.y);
        // -i (kx Gx + ky Gy)
        const double re = kx * gx.x + ky * gy.x, im = kx * gx.y + ky * gy.y;
        zD.x = (T)(M * im); zD.y = (T)(-M * re);
    }
    F[0] = zS;
    F[fs] = zV;
    F[2 * fs] = zD;
}

// ---------------------------------------------------------------------------
// Column transforms fused with the multiplier.  After the row transforms
// (real-to-complex along x, below), every column l_x of the half spectrum is
// an independent length-n sequence along y; the multiplier is applied between
// the forward and the inverse column transforms, so one workgroup takes a
// column from HBM into LDS, transforms it, multiplies, transforms back and
// writes it: the 2D transforms' two column passes, their transposes and the
// multiplier pass become one read and one write of each column.  Columns
// with l_x beyond the multiplier's support are neither written by the
// forward row transforms nor touched here; the inverse row transforms take
// them as zero.
//
// Transforms: self-sorting (Stockham) passes of radix 8, 9, 6, 4, 2, 3 or 5 on the
// LDS copy; each pass reads every butterfly's inputs into registers, waits,
// and writes the outputs in place.  Twiddles e^{-2 pi i m/n} come from a
// table (conjugated for the inverse); both directions are unnormalised, like
// the rocFFT row transforms.
// ---------------------------------------------------------------------------
template <typename T2>
__device__ inline T2 c2(decltype(T2::x) x, decltype(T2::x) y)
{
    T2 r;
    r.x = x;
    r.y = y;
    return r;
}
template <typename T2> __device__ inline T2 cadd(T2 a, T2 b) { return c2<T2>(a.x + b.x, a.y + b.y); }
template <typename T2> __device__ inline T2 csub(T2 a, T2 b) { return c2<T2>(a.x - b.x, a.y - b.y); }
template <typename T2> __device__ inline T2 cmul(T2 a, T2 b)
{
    return c2<T2>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <typename T2> __device__ inline T2 cscale(T2 a, decltype(T2::x) s) { return c2<T2>(a.x * s, a.y * s); }
// -i z (forward) or +i z (inverse)
template <bool INV, typename T2> __device__ inline T2 rot(T2 z)
{
    return INV ? c2<T2>(-z.y, z.x) : c2<T2>(z.y, -z.x);
}

// DFT of R points, y_k = sum_t x_t e^{-+2 pi i t k / R}
template <int R, bool INV, typename T2> __device__ inline void dft(T2 *x)
{
    typedef decltype(T2::x) T;
    if constexpr (R == 2) {
        const T2 a = x[0];
        x[0] = cadd(a, x[1]);
        x[1] = csub(a, x[1]);
    } else if constexpr (R == 3) {
        const T c = (T)-0.5, s = (T)0.86602540378443864676;
        const T2 a = cadd(x[1], x[2]), d = csub(x[1], x[2]);
        const T2 r = cadd(x[0], cscale(a, c)), i = rot<INV>(cscale(d, s));
        x[0] = cadd(x[0], a);
        x[1] = cadd(r, i);
        x[2] = csub(r, i);
    } else if constexpr (R == 4) {
        const T2 t0 = cadd(x[0], x[2]), t1 = csub(x[0], x[2]), t2 = cadd(x[1], x[3]), t3 = rot<INV>(csub(x[1], x[3]));
        x[0] = cadd(t0, t2);
        x[2] = csub(t0, t2);
        x[1] = cadd(t1, t3);
        x[3] = csub(t1, t3);
    } else if constexpr (R == 6) {
        // two DFTs of 3 on the even and odd points, combined with w6^k
        T2 e[3] = {x[0], x[2], x[4]}, o[3] = {x[1], x[3], x[5]};
        dft<3, INV>(e);
        dft<3, INV>(o);
        const T h = (T)0.86602540378443864676;
        // w6 = e^{-+ i pi/3} = 1/2 -+ i sqrt(3)/2, w6^2 = -1/2 -+ i sqrt(3)/2
        const T sg = INV ? (T)1 : (T)-1;
        const T2 o1 = c2<T2>((T)0.5 * o[1].x - sg * h * o[1].y, (T)0.5 * o[1].y + sg * h * o[1].x);
        const T2 o2 = c2<T2>((T)-0.5 * o[2].x - sg * h * o[2].y, (T)-0.5 * o[2].y + sg * h * o[2].x);
        x[0] = cadd(e[0], o[0]);
        x[3] = csub(e[0], o[0]);
        x[1] = cadd(e[1], o1);
        x[4] = csub(e[1], o1);
        x[2] = cadd(e[2], o2);
        x[5] = csub(e[2], o2);
    } else if constexpr (R == 9) {
        // three DFTs of 3 on the points t = 3u + r, twiddles w9^(r k), then
        // DFTs of 3 across r
        T2 a[3][3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            a[r][0] = x[r];
            a[r][1] = x[r + 3];
            a[r][2] = x[r + 6];
            dft<3, INV>(a[r]);
        }
        const T c1 = (T)0.76604444311897803520, s1 = (T)0.64278760968653932632;   // 2 pi / 9
        const T c2v = (T)0.17364817766693034885, s2 = (T)0.98480775301220805936;  // 4 pi / 9
        const T c4 = (T)-0.93969262078590838405, s4 = (T)0.34202014332566873304;  // 8 pi / 9
        const T sg = INV ? (T)1 : (T)-1;
        auto tw9 = [&](T2 z, T c, T sn) { return c2<T2>(c * z.x - sg * sn * z.y, c * z.y + sg * sn * z.x); };
        a[1][1] = tw9(a[1][1], c1, s1);     // w9^1
        a[1][2] = tw9(a[1][2], c2v, s2);    // w9^2
        a[2][1] = tw9(a[2][1], c2v, s2);    // w9^2
        a[2][2] = tw9(a[2][2], c4, s4);     // w9^4
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            T2 b[3] = {a[0][k], a[1][k], a[2][k]};
            dft<3, INV>(b);
            x[k] = b[0];
            x[k + 3] = b[1];
            x[k + 6] = b[2];
        }
    } else if constexpr (R == 8) {
        // two DFTs of 4 on the even and odd points, combined with w8^k
        T2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
        dft<4, INV>(e);
        dft<4, INV>(o);
        const T h = (T)0.70710678118654752440;
        // w8^k o_k, w8 = e^{-+ i pi/4}
        const T2 o1 = INV ? c2<T2>(h * (o[1].x - o[1].y), h * (o[1].x + o[1].y))
                          : c2<T2>(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
        const T2 o2 = rot<INV>(o[2]);
        const T2 o3 = INV ? c2<T2>(-h * (o[3].x + o[3].y), h * (o[3].x - o[3].y))
                          : c2<T2>(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
        x[0] = cadd(e[0], o[0]);
        x[4] = csub(e[0], o[0]);
        x[1] = cadd(e[1], o1);
        x[5] = csub(e[1], o1);
        x[2] = cadd(e[2], o2);
        x[6] = csub(e[2], o2);
        x[3] = cadd(e[3], o3);
        x[7] = csub(e[3], o3);
    } else {
        static_assert(R == 5, "radix");
        const T c1 = (T)0.30901699437494742410, c2v = (T)-0.80901699437494742410;
        const T s1 = (T)0.95105651629515357212, s2 = (T)0.58778525229247312917;
        const T2 a1 = cadd(x[1], x[4]), b1 = csub(x[1], x[4]), a2 = cadd(x[2], x[3]), b2 = csub(x[2], x[3]);
        const T2 r1 = cadd(x[0], cadd(cscale(a1, c1), cscale(a2, c2v)));
        const T2 r2 = cadd(x[0], cadd(cscale(a1, c2v), cscale(a2, c1)));
        const T2 i1 = rot<INV>(cadd(cscale(b1, s1), cscale(b2, s2)));
        const T2 i2 = rot<INV>(csub(cscale(b1, s2), cscale(b2, s1)));
        x[0] = cadd(x[0], cadd(a1, a2));
        x[1] = cadd(r1, i1);
        x[4] = csub(r1, i1);
        x[2] = cadd(r2, i2);
        x[3] = csub(r2, i2);
    }
}

// Position of transform point i in LDS (lengths are multiples of 8): the low
// bits of an aligned group of eight points turned by the group's number, so that
// the first pass's writes, R points apart from lane to lane, spread over the
// banks (radix 8 unturned: 128 bytes apart, four times the cycles).
__device__ inline int lds_at(int i) { return i ^ (i >> 3 & 7); }

// Twiddles of a radix-R butterfly: x_t times w^t, the powers by repeated
// products in FP64 (R - 2 roundings of 1e-16), each rounded once to the
// transform's precision.
template <int R, typename T2> __device__ inline void twiddle(T2 *x, double2 w)
{
    typedef decltype(T2::x) T;
    double2 wt = w;
#pragma unroll
    for (int t = 1; t < R; ++t) {
        x[t] = cmul(x[t], c2<T2>((T)wt.x, (T)wt.y));
        if (t + 1 < R) wt = cmul(wt, w);
    }
}

// j % Ns for j < 8192 (the quotient by FP32, at least 0.4/Ns from the next
// whole number; an integer division takes some 20 instructions)
__device__ inline int mod_small(int j, int Ns, float inv) { return j - Ns * (int)(((float)j + 0.5f) * inv); }

// One radix-R pass of a length-N transform by NT threads (N <= NMAX); Ns =
// product of the radices of the passes before it.  Input i comes from get(i),
// output i goes to put(i, .): LDS, or on a transform's first and last pass global
// memory.  PRE: every thread's inputs are read before any output is written;
// POST: the outputs are visible to all at the end.  The twiddle table holds
// e^{-2 pi i m / (N ts)}, read at stride ts.
template <int R, bool INV, int NT, int NMAX, bool PRE, bool POST, typename T2, typename Get, typename Put>
__device__ inline void fft_pass(Get get, Put put, const double2 *__restrict__ tw, int ts, int N, int Ns)
{
    constexpr int MB = (NMAX / R + NT - 1) / NT;
    const int nb = N / R, step = N / (Ns * R) * ts;
    const float inv = 1.0f / (float)Ns;
    // formed anew in every pass: left to itself the compiler keeps the addresses
    // of all the passes and radices in registers
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    T2 v[MB][R];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int j = tid + i * NT;
        if (j < nb) {
            // one twiddle load per butterfly, issued before the reads of LDS
            double2 w = make_double2(1.0, 0.0);
            if (Ns > 1) {
                w = tw[mod_small(j, Ns, inv) * step];
                if (INV) w.y = -w.y;
            }
#pragma unroll
            for (int t = 0; t < R; ++t) v[i][t] = get(j + t * nb);
            if (Ns > 1) twiddle<R>(v[i], w);
        }
    }
    if (PRE) __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int j = tid + i * NT;
        if (j < nb) {
            dft<R, INV>(v[i]);
            const int k = mod_small(j, Ns, inv), o = (j - k) * R + k;
#pragma unroll
            for (int t = 0; t < R; ++t) put(o + t * Ns, v[i][t]);
        }
    }
    if (POST) __syncthreads();
}

template <bool INV, int NT, int NMAX, bool PRE, bool POST, typename T2, typename Get, typename Put>
__device__ inline void fft_pass_any(int r, Get get, Put put, const double2 *__restrict__ tw, int ts, int N, int Ns)
{
    if (r == 8) fft_pass<8, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
    else if (r == 9) fft_pass<9, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
    else if (r == 6) fft_pass<6, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
    else if (r == 4) fft_pass<4, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
    else if (r == 2) fft_pass<2, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
    else if (r == 3) fft_pass<3, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
    else fft_pass<5, INV, NT, NMAX, PRE, POST, T2>(get, put, tw, ts, N, Ns);
}

// ---------------------------------------------------------------------------
// Row transforms (x direction), real to complex and back, one row per
// workgroup, in place on the padded rows: the n reals of a row are n/2
// complex points z_m = x_2m + i x_2m+1, transformed in LDS (length n/2,
// twiddles of the length-n table at stride 2) and untangled:
//   X_k = (Z_k + conj Z_{n/2-k})/2 - i e^{-2 pi i k/n} (Z_k - conj Z_{n/2-k})/2,
// k = 0..n/2; the inverse forms Z_k = (X_k + conj X_{n/2-k}) + i e^{2 pi i k/n}
// (X_k - conj X_{n/2-k}) and transforms back (unnormalised, as the column
// transforms).
// ---------------------------------------------------------------------------
template <typename T>
struct RowArgs {
    int64_t n;
    int r0, nrow;                  // rows r0 .. r0 + nrow - 1 of every field of the launch
    int m0, m1;                    // forward: complex points [m0, m1) of a row can be nonzero;
                                   // inverse: complex points [m0, m1) are written back
    int B, nblk;                   // densities; blocks per grid row
    int8_t grp[4];                 // field groups of the launch: forward S, V, D_x, D_y sources, inverse S, V, D
    const uint8_t *vflag, *bflag;  // forward: blocks holding volume / boundary sources; the others are zero, unwritten
    int ncol;                      // half-spectrum entries k < ncol can be nonzero after the multiplier
    int npass;
    int8_t radix[COL_MAXPASS];     // of n/2
    T *grid;                       // rows of n + 2 reals, consecutive
    const double2 *tw;             // e^{-2 pi i m / n}, FP64 at both precisions
};

// The first pass takes its inputs from global memory, tangled on the way for
// the inverse, and the inverse's last pass writes there: a row's points go
// through LDS once per two passes and once for the untangling.
template <bool INV, typename T, int NMAX>
__global__ void __launch_bounds__(NMAX / 16) k_rows(RowArgs<T> A)
{
    typedef typename Vec2<T>::type T2;
    constexpr int RT = NMAX / 16, HM = NMAX / 2;         // threads (one radix-8 butterfly each); longest transform
    extern __shared__ double lds_row[];
    T2 *buf = reinterpret_cast<T2 *>(lds_row);
    auto get = [&](int i) { return buf[lds_at(i)]; };
    auto put = [&](int i, T2 z) { buf[lds_at(i)] = z; };
    const int n = (int)A.n, h = n / 2;
    const int gb = (int)(blockIdx.x / A.nrow), grp = A.grp[gb / A.B];
    const size_t slot = (size_t)grp * A.B + gb % A.B, row = A.r0 + blockIdx.x % A.nrow;
    T2 *c = reinterpret_cast<T2 *>(A.grid + (slot * (size_t)n + row) * (size_t)(n + 2));   // h + 1 complex
    const int tid = threadIdx.x;
    if (!INV) {
        // the row is zero outside the blocks of the sources' windows
        const T2 zero = c2<T2>((T)0, (T)0);
        const uint8_t *__restrict__ flag =
            (grp == 1 ? A.vflag : A.bflag) + (row / SPB) * (size_t)A.nblk;
        auto on = [&](int m) { return m >= A.m0 && m < A.m1 && flag[2 * m / SPB]; };
        int any = 0;
        for (int m = tid * (SPB / 2); m < h; m += RT * (SPB / 2)) any |= flag[2 * m / SPB];
        if (!__syncthreads_or(any)) {
            for (int k = tid; k < A.ncol; k += RT) c[k] = zero;
            return;
        }
        auto row_in = [&](int m) { return on(m) ? c[m] : zero; };
        fft_pass_any<false, RT, HM, false, true, T2>(A.radix[0], row_in, put, A.tw, 2, h, 1);
        int Ns = A.radix[0];
        for (int p = 1; p < A.npass; Ns *= A.radix[p], ++p)
            fft_pass_any<false, RT, HM, true, true, T2>(A.radix[p], get, put, A.tw, 2, h, Ns);
        // only the columns that the multiplier keeps are read again
        for (int k = tid; k < A.ncol; k += RT) {
            const T2 zk = get(k == h ? 0 : k), zc = get(k == 0 ? 0 : h - k);
            const double2 wd64 = A.tw[k];                                    // e^{-2 pi i k/n}
            const T2 w = c2<T2>((T)wd64.x, (T)wd64.y);
            const T2 sp = c2<T2>(zk.x + zc.x, zk.y - zc.y);                  // Z_k + conj Z_{h-k}
            const T2 dm = c2<T2>(zk.x - zc.x, zk.y + zc.y);                  // Z_k - conj Z_{h-k}
            const T2 wd = cmul(w, dm);
            c[k] = c2<T2>((T)0.5 * (sp.x + wd.y), (T)0.5 * (sp.y - wd.x));   // (sp - i w dm)/2
        }
    } else {
        // entries k >= ncol are zero (the column transforms leave them unwritten)
        const T2 zero = c2<T2>((T)0, (T)0);
        auto row_in = [&](int k) {
            const T2 a = k < A.ncol ? c[k] : zero, bb = h - k < A.ncol ? c[h - k] : zero;
            const T2 sp = c2<T2>(a.x + bb.x, a.y - bb.y);                    // X_k + conj X_{h-k}
            const T2 dm = c2<T2>(a.x - bb.x, a.y + bb.y);                    // X_k - conj X_{h-k}
            const double2 wd64 = A.tw[k];
            const T2 wd = cmul(c2<T2>((T)wd64.x, (T)-wd64.y), dm);           // e^{+2 pi i k/n} dm
            return c2<T2>(sp.x - wd.y, sp.y + wd.x);                         // sp + i wd
        };
        fft_pass_any<true, RT, HM, false, true, T2>(A.radix[0], row_in, put, A.tw, 2, h, 1);
        int Ns = A.radix[0], p = 1;
        for (; p + 1 < A.npass; Ns *= A.radix[p], ++p)
            fft_pass_any<true, RT, HM, true, true, T2>(A.radix[p], get, put, A.tw, 2, h, Ns);
        // only the points the interpolation windows use (the barrier above: every
        // thread has read its points of the row)
        auto row_out = [&](int m, T2 z) {
            if (m >= A.m0 && m < A.m1) c[m] = z;
        };
        fft_pass_any<true, RT, HM, false, false, T2>(A.radix[p], get, row_out, A.tw, 2, h, Ns);
    }
}

template <typename T>
struct ColArgs {
    int64_t n, field;
    int B, ncol, npass;
    int8_t grp[3];         // outputs of the launch: 0 S, 1 V, 2 D
    int iy0, iy1;          // rows [iy0, iy1) of the input columns can be nonzero (the sources' windows)
    int oy0, oy1;          // rows [oy0, oy1) of the output columns are written (the targets' windows)
    int8_t radix[COL_MAXPASS];
    T *grid;
    const double2 *tw;             // e^{-2 pi i m / n}, FP64 at both precisions
    const double *fac, *mtab;
    double c, alpha2, dk;
    int lmax;
};

// One workgroup per (column, density, output): 0 S, 1 V, 2 D (from the D_x
// and D_y spectra: -i (k_x Gx + k_y Gy) M, two forward transforms and one
// inverse).  The first forward pass reads global memory and the last inverse
// one writes it; the last forward pass, the multiplier and the first inverse
// pass, all on the same eight points of a thread, stay in registers: 2 (npass -
// 1) exchanges through LDS per pair of transforms instead of 2 npass + 2, and three
// transforms per D output instead of four.  Alone: D on 3840^2 217 -> 127 us, 16
// densities on 2880^2 2.60 -> 1.81 ms.
template <typename T, int NMAX>
__global__ void __launch_bounds__(NMAX / 8, 4) k_columns(ColArgs<T> A)
{
    typedef typename Vec2<T>::type T2;
    constexpr int CT = NMAX / 8;       // threads: one radix-8 butterfly each
    extern __shared__ double lds_col[];
    T2 *buf = reinterpret_cast<T2 *>(lds_col);
    auto get = [&](int i) { return buf[lds_at(i)]; };
    auto put = [&](int i, T2 z) { buf[lds_at(i)] = z; };
    const int n = (int)A.n, nh = n / 2 + 1;
    // consecutive columns on one XCD (workgroups are dealt to the 8 XCDs in
    // turn), so that neighbouring columns share the XCD's L2 lines; only the
    // columns l_x < ncol that the multiplier keeps (the inverse row
    // transforms take the others as zero)
    const int per = (A.ncol + 7) / 8;
    const int lx = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (lx >= A.ncol) return;
    const int b = blockIdx.y, grp = A.grp[blockIdx.z];
    const size_t fs = (size_t)A.B * (A.field / 2);              // complex values per slot
    T2 *base = reinterpret_cast<T2 *>(A.grid) + (size_t)b * (A.field / 2) + lx;
    T2 *out = base + (size_t)grp * fs;
    const double ax = A.fac[lx];
    const double kx = A.dk * lx;
    auto mult = [&](int ly) -> double {
        const int fy = ly <= n / 2 ? ly : ly - n;
        if (A.mtab) {
            if (lx <= A.lmax && fy >= -A.lmax && fy <= A.lmax) return A.mtab[(fy + A.lmax) * (A.lmax + 1) + lx];
            return 0.0;
        }
        const double ay = A.fac[fy < 0 ? -fy : fy];
        if (ax == 0.0 || ay == 0.0) return 0.0;
        const double ky = A.dk * fy;
        return A.c * ax * ay / (A.alpha2 + kx * kx + ky * ky);
    };
    const T2 zero = c2<T2>((T)0, (T)0);
    const int nparts = grp == 2 ? 2 : 1, last = A.npass - 1, nb = n / 8;
    // the spectrum's points j + t nb of thread j: outputs of the last forward
    // pass (radix 8) and inputs of the first inverse one
    int j = threadIdx.x;
    T2 u[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) u[t] = zero;
    for (int part = 0; part < nparts; ++part) {
        const T2 *in = base + (size_t)(grp == 2 ? 2 + part : grp) * fs;
        auto col_in = [&](int y) { return y >= A.iy0 && y < A.iy1 ? in[(size_t)y * nh] : zero; };
        fft_pass_any<false, CT, NMAX, false, true, T2>(A.radix[0], col_in, put, A.tw, 1, n, 1);
        int Ns = A.radix[0];
        for (int p = 1; p < last; Ns *= A.radix[p], ++p)
            fft_pass_any<false, CT, NMAX, true, true, T2>(A.radix[p], get, put, A.tw, 1, n, Ns);
        asm volatile("" : "+v"(j));
        if (j < nb) {
            T2 z[8];
            const double2 w = A.tw[j];
#pragma unroll
            for (int t = 0; t < 8; ++t) z[t] = get(j + t * nb);
            twiddle<8>(z, w);
            dft<8, false>(z);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int ly = j + t * nb;
                const double M = mult(ly);
                if (grp < 2) {
                    u[t] = c2<T2>((T)(M * z[t].x), (T)(M * z[t].y));
                } else {
                    // -i k M z with k = k_x (part 0) or k_y (part 1)
                    const int fy = ly <= n / 2 ? ly : ly - n;
                    const double kM = (part == 0 ? kx : A.dk * fy) * M;
                    u[t] = cadd(u[t], c2<T2>((T)(kM * z[t].y), (T)(-kM * z[t].x)));
                }
            }
        }
        __syncthreads();
    }
    if (j < nb) {
        dft<8, true>(u);
#pragma unroll
        for (int t = 0; t < 8; ++t) put(8 * j + t, u[t]);
    }
    __syncthreads();
    int Ns = 8, p = last - 1;
    for (; p > 0; Ns *= A.radix[p], --p)
        fft_pass_any<true, CT, NMAX, true, true, T2>(A.radix[p], get, put, A.tw, 1, n, Ns);
    auto col_out = [&](int y, T2 z) {
        if (y >= A.oy0 && y < A.oy1) out[(size_t)y * nh] = z;
    };
    fft_pass_any<true, CT, NMAX, false, false, T2>(A.radix[0], get, col_out, A.tw, 1, n, Ns);
}

template <typename T>
struct InterpArgs {
    int64_t n, field, nout;
    int ntile, B;          // tiles (or blocks) per grid row
    int nrun;              // non-empty tiles (or blocks)
    int gx0, gx1, gy0, gy1;   // grid values [gx0, gx1) x [gy0, gy1) are set
    double beta, ox, oy, h;
    const int32_t *tile_xy, *tile_rng;
    const double *tx, *ty;
    const T *grid;         // [3][B][field]: S, V, D results
    const T *wcoef;
    T *acc;                // [3][B][nout]: S, D, V
    int want_s, want_d, want_v;
};

template <int W, typename T>
__global__ void __launch_bounds__(HB) k_interp(InterpArgs<T> A)
{
    constexpr int RS = TILE + W + 2;
    __shared__ T reg[3][RS * RS];
    const int t = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int tile = A.tile_xy[t];
    const int tx = tile % A.ntile, ty = tile / A.ntile;
    const int rx0 = tx * TILE - W / 2 - 1, ry0 = ty * TILE - W / 2 - 1;
    const size_t fs = (size_t)A.B * A.field;
    const T *g0 = A.grid + (size_t)b * A.field;
    for (int i = tid; i < RS * RS; i += HB) {
        // the staged region exceeds the grid by less than one period
        int gy = ry0 + i / RS, gx = rx0 + i % RS;
        gy += gy < 0 ? (int)A.n : gy >= A.n ? -(int)A.n : 0;
        gx += gx < 0 ? (int)A.n : gx >= A.n ? -(int)A.n : 0;
        const size_t o = (size_t)gy * (A.n + 2) + gx;
        reg[0][i] = A.want_s ? g0[o] : (T)0;
        reg[1][i] = A.want_v ? g0[fs + o] : (T)0;
        reg[2][i] = A.want_d ? g0[2 * fs + o] : (T)0;
    }
    __syncthreads();
    const int s0 = A.tile_rng[t], s1 = A.tile_rng[t + 1];
    for (int s = s0 + tid; s < s1; s += HB) {
        const double gx = (A.tx[s] - A.ox) / A.h, gy = (A.ty[s] - A.oy) / A.h;
        int mx0, my0;
        T wx[W], wy[W];
        window_weights2<W, T>(gx, gy, A.wcoef, mx0, my0, wx, wy);
        const int lx = min(max(mx0 - rx0, 0), RS - W), ly = min(max(my0 - ry0, 0), RS - W);
        T uS = 0, uV = 0, uD = 0;
#pragma unroll 1
        for (int ky = 0; ky < W; ++ky) {
            const int o = (ly + ky) * RS + lx;
            T rS = 0, rV = 0, rD = 0;
#pragma unroll
            for (int kx = 0; kx < W; ++kx) {
                rS = fma(wx[kx], reg[0][o + kx], rS);
                rV = fma(wx[kx], reg[1][o + kx], rV);
                rD = fma(wx[kx], reg[2][o + kx], rD);
            }
            uS = fma(wy[ky], rS, uS);
            uV = fma(wy[ky], rV, uV);
            uD = fma(wy[ky], rD, uD);
        }
        const size_t ob = (size_t)b * A.nout + s, cs = (size_t)A.B * A.nout;
        if (A.want_s) A.acc[ob] = uS;
        if (A.want_d) A.acc[cs + ob] = uD;
        if (A.want_v) A.acc[2 * cs + ob] = uV;
    }
}

// Interpolation on the matrix cores, for targets dense on the grid.  The windows
// of the targets of an E x E block of grid cells (E + W <= 16) lie in one 16 x
// 16 region U of each result grid, so u_j = sum_y w_y(j, y) sum_x U(y, x) w_x(j,
// x) is, for 16 targets, a 16 x 16 x 16 product (four v_mfma_16x16x4 in the
// plan's precision, A: U with lane l holding row l % 16 and columns 4 (l / 16) +
// s of step s, B: the x-window values) and a dot product of each column with
// the target's y-window values.  A wavefront owns a block: U stays in its
// registers, the window values of 32 targets at a time go through LDS as in the
// spreading.  One thread per target instead reads 3 W^2 values at addresses
// that differ from lane to lane, bound by LDS bank conflicts.  Measured (three
// results, W = 12, alone): 1.02M targets, 45 per block, 138 by tiles -> 71 us; 4608
// targets, 23 per block, 45 -> 8 us; 16 densities, 1000 -> 846 us.
template <typename T> struct Frag;
template <> struct Frag<double> { typedef d4 type; };
template <> struct Frag<float> { typedef float type __attribute__((ext_vector_type(4))); };
__device__ inline d4 mma16(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ inline Frag<float>::type mma16(float a, float b, Frag<float>::type c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int W, typename T>
__global__ void __launch_bounds__(HB) k_interp_mm(InterpArgs<T> A)
{
    typedef typename Frag<T>::type F;
    constexpr int RW = W + 2, E = interp_edge(W);
    __shared__ T rows[HB / 64][64 * RW];
    __shared__ int corner[HB / 64][64];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int run = (int)blockIdx.x * (HB / 64) + wave;
    if (run >= A.nrun) return;                        // wavefronts are independent: no workgroup barrier below
    T *row = rows[wave];
    int *ms = corner[wave];
    const int blk = A.tile_xy[run], s0 = A.tile_rng[run], s1 = A.tile_rng[run + 1];
    // the lowest window corner of the block's targets
    const int x0 = blk % A.ntile * E - W / 2, y0 = blk / A.ntile * E - W / 2;
    const int j = lane % 16, k = lane / 16, axis = lane / 32, sl = lane % 32;
    const size_t fs = (size_t)A.B * A.field, cs = (size_t)A.B * A.nout;
    const bool want[3] = {A.want_s != 0, A.want_v != 0, A.want_d != 0};
    T u[3][4];
    // values outside the set part of the grid are zero (their weights are, too)
    auto region = [&](int b) {
        const int gy = y0 + j, gx = x0 + 4 * k;
        const bool iny = gy >= A.gy0 && gy < A.gy1;
        const T *g = A.grid + (size_t)b * A.field + (size_t)gy * (A.n + 2) + gx;
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                u[f][s] = want[f] && iny && gx + s >= A.gx0 && gx + s < A.gx1 ? g[f * fs + s] : (T)0;
    };
    row[lane * RW] = (T)0;
    row[lane * RW + W + 1] = (T)0;
    const int b0 = (int)blockIdx.y * INTERP_NB, b1 = min(A.B, b0 + INTERP_NB);
    if (b1 - b0 == 1) region(b0);
    for (int p = s0; p < s1; p += 32) {
        const int s = p + sl;
        int m = 1 << 20;                              // no target: a window far outside
        if (s < s1) {
            const double g = axis ? (A.ty[s] - A.oy) / A.h : (A.tx[s] - A.ox) / A.h;
            T w[W];
            window_weights1<W, T>(g, A.wcoef, m, w);
            m -= axis ? y0 : x0;
#pragma unroll
            for (int q = 0; q < W; ++q) row[lane * RW + 1 + q] = w[q];
        }
        ms[lane] = m;
        wave_sync();
        const int cnt = min(32, s1 - p);
        for (int b = b0; b < b1; ++b) {
            if (b1 - b0 > 1) region(b);
            for (int q0 = 0; q0 < cnt; q0 += 16) {
                const int src = q0 + j, mx = ms[src], my = ms[32 + src];
                T wx[4], wy[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    // D: row 4 v + k in FP64, 4 k + v in FP32
                    const int y = sizeof(T) == 8 ? 4 * v + k : 4 * k + v;
                    wx[v] = row[src * RW + min(max(4 * k + v - mx, -1), W) + 1];
                    wy[v] = row[(32 + src) * RW + min(max(y - my, -1), W) + 1];
                }
                T r[3];
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    F c = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
                    for (int v = 0; v < 4; ++v) c = mma16(u[f][v], wx[v], c);
                    r[f] = wy[0] * c[0];
#pragma unroll
                    for (int v = 1; v < 4; ++v) r[f] = fma(wy[v], c[v], r[f]);
                    r[f] += __shfl_xor(r[f], 16, 64);
                    r[f] += __shfl_xor(r[f], 32, 64);
                }
                if (lane < 16 && q0 + lane < cnt) {
                    const size_t o = (size_t)b * A.nout + p + q0 + lane;
                    if (want[0]) A.acc[o] = r[0];
                    if (want[2]) A.acc[cs + o] = r[2];
                    if (want[1]) A.acc[2 * cs + o] = r[1];
                }
            }
        }
        wave_sync();
    }
}

// Interpolation of few targets far apart: sixteen lanes per target, one per
// window column, read the W rows of the window straight from the grid (a tile
// of 46 x 46 values staged for one or two targets took 65 us for 8065 targets
// on 4858 tiles, one result; this takes 7 us).
template <int W, typename T>
__global__ void __launch_bounds__(HB) k_interp_few(InterpArgs<T> A)
{
    const int64_t s = ((int64_t)blockIdx.x * HB + threadIdx.x) / 16;
    const int kx = threadIdx.x % 16, b = blockIdx.y;
    if (s >= A.nout) return;                          // whole groups of sixteen lanes
    const double gx = (A.tx[s] - A.ox) / A.h, gy = (A.ty[s] - A.oy) / A.h;
    int mx0, my0;
    T wx[W], wy[W];
    window_weights2<W, T>(gx, gy, A.wcoef, mx0, my0, wx, wy);
    T w = (T)0;
#pragma unroll
    for (int q = 0; q < W; ++q) w = kx == q ? wx[q] : w;
    const size_t fs = (size_t)A.B * A.field, cs = (size_t)A.B * A.nout, o = (size_t)b * A.nout + s;
    // windows lie inside the grid (its origin is W/2 + 3 points below the points)
    const T *g = A.grid + (size_t)b * A.field + (size_t)my0 * (A.n + 2) + mx0 + kx;
    auto one = [&](int f) {
        T v = (T)0;
        if (kx < W)
#pragma unroll
            for (int ky = 0; ky < W; ++ky) v = fma(wy[ky], g[f * fs + (size_t)ky * (A.n + 2)], v);
        v *= w;
#pragma unroll
        for (int m = 8; m >= 1; m /= 2) v += __shfl_xor(v, m, 16);
        return v;
    };
    if (A.want_s) {
        const T v = one(0);
        if (kx == 0) A.acc[o] = v;
    }
    if (A.want_v) {
        const T v = one(1);
        if (kx == 0) A.acc[2 * cs + o] = v;
    }
    if (A.want_d) {
        const T v = one(2);
        if (kx == 0) A.acc[cs + o] = v;
    }
}

// The smoothly truncated history kernel on the grid is a sum of products of one
// factor per axis: G^H(r) = int_delta^inf H(t, r) dt (eq. (sl_sh)) with t = delta
// e^{-u} is
//   (1/4pi) int_{-inf}^0 exp(-a e^u - b e^{-u}) du,  a = r^2/(4 delta), b = alpha^2 delta,
// and under a quadrature in u every node's exp(-a e^u) splits into its x and y
// parts.  So do its cosine transforms: one transform per node instead of one per
// row of the samples, and the spectrum is their sum of products.

// Factor of every node q < Q at x = m h, m < M: exp(-x^2 su_q) chi(x), su_q =
// e^{u_q}/(4 delta), chi(x) = erfc((x - rmid) slope)/2, row-major [q][m].
__global__ void __launch_bounds__(256) k_trunc_factors(double *__restrict__ buf, int64_t M, int64_t Q, double h,
                                                       double rmid, double slope, const double *__restrict__ su)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= M * Q) return;
    const double x = (double)(id % M) * h;
    buf[id] = exp(-x * x * su[id / M]) * 0.5 * erfc((x - rmid) * slope);
}

// COS: the cosine transforms of even sequences,
//   out[a][b] = sum_{k < K} c_k cos(2 pi a k / n) in[b][k],  c_0 = 1, c_k = 2
// (the +-k pairs folded into c_k; the cosines from a table of cos(2 pi m / n) at m
// = a k mod n); else the weighted products
//   out[a][b] = sum_{k < K} w_k in[a][k] in[b][k],
// for a < NA, b < NB.  Tiles of 32 x 32 outputs per 256-thread workgroup, 2 x 2
// per thread (64 x 64 are too few tiles for the chip), both inputs staged through
// LDS 32 values of k at a time.
constexpr int CS_T = 32, CS_K = 32;
template <bool COS>
__global__ void __launch_bounds__(256) k_cos_step(const double *__restrict__ in, int64_t K, int64_t NA, int64_t NB,
                                                  int n, const double *__restrict__ tab, double *__restrict__ out)
{
    constexpr int E = CS_K * CS_T / 256, R = CS_T / 16;
    __shared__ double ca[CS_K][CS_T + 1];
    __shared__ double ib[CS_K][CS_T + 1];
    const int tid = threadIdx.x;
    const int64_t a0 = (int64_t)blockIdx.x * CS_T, b0 = (int64_t)blockIdx.y * CS_T;
    const int ta = tid / 16, tb = tid % 16;
    // COS: table positions a k mod n of this thread's elements, and their steps
    int pos[E], step[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int e = tid + 256 * i;
        const int64_t a = a0 + e % CS_T;
        pos[i] = COS ? (int)(a * (e / CS_T) % n) : 0;
        step[i] = COS ? (int)(a * CS_K % n) : 0;
    }
    double acc[R][R] = {};
    for (int64_t k0 = 0; k0 < K; k0 += CS_K) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const int e = tid + 256 * i;
            const int bb = e / CS_K, kk = e % CS_K;
            const int64_t k = k0 + kk;
            ib[kk][bb] = k < K && b0 + bb < NB ? in[(b0 + bb) * K + k] : 0.0;
            if (!COS) ca[kk][bb] = k < K && a0 + bb < NA ? tab[k] * in[(a0 + bb) * K + k] : 0.0;
        }
        if (COS) {
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int e = tid + 256 * i;
                const int64_t k = k0 + e / CS_T;
                ca[e / CS_T][e % CS_T] = k < K && a0 + e % CS_T < NA ? (k == 0 ? 1.0 : 2.0) * tab[pos[i]] : 0.0;
                pos[i] += step[i];
                if (pos[i] >= n) pos[i] -= n;
            }
        }
        __syncthreads();
#pragma unroll 8
        for (int kk = 0; kk < CS_K; ++kk) {
            double av[R], bv[R];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                av[i] = ca[kk][ta + 16 * i];
                bv[i] = ib[kk][tb + 16 * i];
            }
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < R; ++j) acc[i][j] = fma(av[i], bv[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int64_t a = a0 + ta + 16 * i, b = b0 + tb + 16 * j;
            if (a < NA && b < NB) out[a * NB + b] = acc[i][j];
        }
}

// Multiplier table on the kept modes |l_x|, |l_y| <= lmax from the cosine
// transform tr[l_y][l_x] (l >= 0; the kernel's transform is real and even).
__global__ void __launch_bounds__(256) k_trunc_table(const double *__restrict__ tr, int lmax,
                                                     const double *__restrict__ phi2inv, double c,
                                                     double *__restrict__ mtab)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t w = lmax + 1;
    if (id >= (2 * (int64_t)lmax + 1) * w) return;
    const int64_t lx = id % w, fy = id / w - lmax, ly = fy < 0 ? -fy : fy;
    mtab[id] = c * tr[ly * w + lx] * phi2inv[lx] * phi2inv[ly];
}

hipError_t launch_trunc_factors(double *buf, int64_t M, int64_t Q, double h, double rmid, double slope,
                                const double *su, hipStream_t s)
{
    hipLaunchKernelGGL(k_trunc_factors, dim3((unsigned)((M * Q + 255) / 256)), dim3(256), 0, s, buf, M, Q, h, rmid,
                       slope, su);
    return hipGetLastError();
}

hipError_t launch_cos_step(bool cosines, const double *in, int64_t K, int64_t NA, int64_t NB, int n, const double *tab,
                           double *out, hipStream_t s)
{
    const dim3 grid((unsigned)((NA + CS_T - 1) / CS_T), (unsigned)((NB + CS_T - 1) / CS_T));
    if (cosines)
        hipLaunchKernelGGL(k_cos_step<true>, grid, dim3(256), 0, s, in, K, NA, NB, n, tab, out);
    else
        hipLaunchKernelGGL(k_cos_step<false>, grid, dim3(256), 0, s, in, K, NA, NB, n, tab, out);
    return hipGetLastError();
}

hipError_t launch_trunc_table(const double *tr, int lmax, const double *phi2inv, double c, double *mtab,
                              hipStream_t s)
{
    const int64_t tot = (2 * (int64_t)lmax + 1) * (lmax + 1);
    hipLaunchKernelGGL(k_trunc_table, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, tr, lmax, phi2inv, c,
                       mtab);
    return hipGetLastError();
}

template <int W, typename T>
static hipError_t spread_w(mhk_plan *P, SpreadArgs<T> &A)
{
    const History &G = P->hist;
    const bool vol = A.f_vol, bnd = A.sigma || A.mu;
    const int64_t blocks = (vol ? G.nvact : 0) + (bnd ? G.nbact : 0);
    if (blocks == 0) return hipSuccess;
    // Several densities share the window values of a workgroup (8 accumulators of
    // the volume or 6 of the boundary, 4 doubles a lane each, stay in registers
    // beside them) where single ones already fill the chip: beyond 1024 workgroups of
    // one density each, or 4096 up to 3 densities, as a workgroup's 8 of the volume
    // take the matrix cores' time of 8 whatever their number, while single ones form
    // the window values once each, beside level sums that need the VALU too.  By
    // eights against one each, history part: FP64 V of 2 on 720 blocks 320 / 229 us, of
    // 8 548 / 628, of 16 on 122 blocks 301 / 307 (1952 workgroups); whole evaluations:
    // FP64 of 2 (834 workgroups) 300 / 275 us, of 3 (1251) 355 / 334, of 5 (2085) 479 /
    // 484, of 7 (2919) 593 / 615.  Without V the boundary's short lists gain nothing (S
    // and D of 3 on 101 blocks 125 / 126).
    const bool one = A.B == 1 || (vol && blocks * A.B <= (A.B <= 3 ? 4096 : 1024));
    const int nv = one ? 1 : 8, nd = one ? 1 : 2;
    A.nvt = (A.B + nv - 1) / nv;
    A.nbt = (A.B + nd - 1) / nd;
    A.nvw = vol ? G.nvact * A.nvt : 0;
    const int64_t wg = A.nvw + (bnd ? G.nbact * A.nbt : 0);
    // wavefronts per block: few blocks leave the chip idle behind their long
    // lists, so they take 16 (up to two workgroups per CU) or 8; many blocks
    // fill it, and four shorter-lived wavefronts each finish more evenly.
    // Measured with 4 / 8 / 16, alone: 40 workgroups 25 / 16 / 12 us, 476
    // workgroups (FP32) 26 / 18 / 14 us, 2236 workgroups 126 / 107 / 122 us,
    // 7149 workgroups (FP32) 219 / 234 / 287 us; 16 densities 750 / 843 us.  At
    // 2236 the gain alone is lost beside the level sums, which the larger LDS
    // share keeps out (whole evaluation 1288 / 1315 us).  8 FP32 densities of V on
    // 14 blocks (history part): 87 us by eights with 4, 51 one each with 16.
    if (!one)
        hipLaunchKernelGGL((k_spread<W, T, 8, 2, 4>), dim3((unsigned)wg), dim3(256), 0, P->stream, A);
    else if (wg <= 512)
        hipLaunchKernelGGL((k_spread<W, T, 1, 1, 16>), dim3((unsigned)wg), dim3(1024), 0, P->stream, A);
    else if (wg <= 1024)
        hipLaunchKernelGGL((k_spread<W, T, 1, 1, 8>), dim3((unsigned)wg), dim3(512), 0, P->stream, A);
    else
        hipLaunchKernelGGL((k_spread<W, T, 1, 1, 4>), dim3((unsigned)wg), dim3(256), 0, P->stream, A);
    return hipGetLastError();
}

template <int W, typename T>
static hipError_t interp_w(mhk_plan *P, const InterpArgs<T> &A)
{
    if (P->hist.n_ttiles == 0) return hipSuccess;
    if constexpr (interp_edge(W) > 0) {
        if (P->hist.iedge > 0) {
            dim3 grid((unsigned)((A.nrun + HB / 64 - 1) / (HB / 64)), (unsigned)((A.B + INTERP_NB - 1) / INTERP_NB));
            hipLaunchKernelGGL((k_interp_mm<W, T>), grid, dim3(HB), 0, P->stream, A);
            return hipGetLastError();
        }
    }
    if (P->nout <= INTERP_FEW * (int64_t)P->hist.n_ttiles) {
        dim3 grid((unsigned)((P->nout * 16 + HB - 1) / HB), (unsigned)A.B);
        hipLaunchKernelGGL((k_interp_few<W, T>), grid, dim3(HB), 0, P->stream, A);
        return hipGetLastError();
    }
    dim3 grid((unsigned)P->hist.n_ttiles, (unsigned)A.B);
    hipLaunchKernelGGL((k_interp<W, T>), grid, dim3(HB), 0, P->stream, A);
    return hipGetLastError();
}

#define MHK_W_SWITCH(w, F, T, ...)              \
    switch (w) {                                \
    case 4: return F<4, T>(__VA_ARGS__);        \
    case 5: return F<5, T>(__VA_ARGS__);        \
    case 6: return F<6, T>(__VA_ARGS__);        \
    case 7: return F<7, T>(__VA_ARGS__);        \
    case 8: return F<8, T>(__VA_ARGS__);        \
    case 9: return F<9, T>(__VA_ARGS__);        \
    case 10: return F<10, T>(__VA_ARGS__);      \
    case 11: return F<11, T>(__VA_ARGS__);      \
    case 12: return F<12, T>(__VA_ARGS__);      \
    case 13: return F<13, T>(__VA_ARGS__);      \
    case 14: return F<14, T>(__VA_ARGS__);      \
    case 15: return F<15, T>(__VA_ARGS__);      \
    case 16: return F<16, T>(__VA_ARGS__);      \
    default: return hipErrorInvalidValue;       \
    }

template <typename T>
static hipError_t spread_t(mhk_plan *P, const void *sigma, const void *mu, const void *f_vol)
{
    const History &G = P->hist;
    SpreadArgs<T> A;
    A.n = G.n;
    A.field = G.field;
    A.nb = P->nb;
    A.nv = P->nv;
    A.nblk = (int)(G.n / SPB);
    A.B = P->bat;
    A.vact = G.vact;
    A.bact = G.bact;
    A.bgx = G.bgx; A.bgy = G.bgy; A.bw = G.bw; A.bwx = G.bwx; A.bwy = G.bwy;
    A.bidx = G.bidx; A.blofs = G.blofs; A.blist = G.blist;
    A.vgx = G.vgx; A.vgy = G.vgy; A.vw = G.vw; A.vidx = G.vidx; A.vlofs = G.vlofs; A.vlist = G.vlist;
    A.sigma = (const T *)sigma;
    A.mu = (const T *)mu;
    A.f_vol = (const T *)f_vol;
    A.grid = (T *)G.grid;
    A.wcoef = (const T *)G.wcoef;
    MHK_W_SWITCH(G.w, spread_w, T, P, A);
}

hipError_t launch_spread(mhk_plan *P, const void *sigma, const void *mu, const void *f_vol)
{
    return P->p.prec == MHK_FP64 ? spread_t<double>(P, sigma, mu, f_vol) : spread_t<float>(P, sigma, mu, f_vol);
}

template <typename T>
static hipError_t multiply_t(mhk_plan *P)
{
    const History &G = P->hist;
    const int64_t tot = G.n * (G.n / 2 + 1) * P->bat;
    hipLaunchKernelGGL(k_multiply<T>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, P->stream, G.n,
                       P->bat, G.field, (T *)G.grid, G.fac, G.mult_c, P->p.alpha * P->p.alpha,
                       2.0 * M_PI / G.period, G.trunc ? G.mtab : nullptr, G.lmax);
    return hipGetLastError();
}

template <typename T>
static hipError_t columns_t(mhk_plan *P, bool want_s, bool want_d, bool want_v)
{
    const History &G = P->hist;
    ColArgs<T> A;
    // the D spectra take two transforms: first, so that the long workgroups start first
    int ng = 0;
    if (want_d) A.grp[ng++] = 2;
    if (want_s) A.grp[ng++] = 0;
    if (want_v) A.grp[ng++] = 1;
    if (ng == 0) return hipSuccess;
    A.n = G.n;
    A.field = G.field;
    A.B = P->bat;
    A.ncol = G.ncol;
    A.npass = G.npass;
    for (int i = 0; i < COL_MAXPASS; ++i) A.radix[i] = G.radix[i];
    A.grid = (T *)G.grid;
    A.tw = (const double2 *)G.tw;
    A.fac = G.fac;
    A.mtab = G.trunc ? G.mtab : nullptr;
    A.c = G.mult_c;
    A.alpha2 = P->p.alpha * P->p.alpha;
    A.dk = 2.0 * M_PI / G.period;
    A.lmax = G.lmax;
    A.iy0 = G.sy0;
    A.iy1 = G.sy1;
    A.oy0 = G.ty0;
    A.oy1 = G.ty1;
    const size_t lds = sizeof(typename Vec2<T>::type) * (size_t)G.n;
    if (G.ncol == 0) return hipSuccess;     // the multiplier is zero everywhere
    dim3 grid((unsigned)(((G.ncol + 7) / 8) * 8), (unsigned)P->bat, (unsigned)ng);
    // threads and register arrays for the longest column of the variant
    auto go = [&](auto nmax) {
        constexpr int NMAX = decltype(nmax)::value;
        const void *fn = (const void *)k_columns<T, NMAX>;
        if (lds > 64 * 1024) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL((k_columns<T, NMAX>), grid, dim3(NMAX / 8), lds, P->stream, A);
        return hipGetLastError();
    };
    if (G.n <= COL_NMAX / 4) return go(std::integral_constant<int, COL_NMAX / 4>());
    if (G.n <= COL_NMAX / 2) return go(std::integral_constant<int, COL_NMAX / 2>());
    return go(std::integral_constant<int, COL_NMAX>());
}

template <bool INV, typename T>
static hipError_t rows_t(mhk_plan *P, bool want_s, bool want_d, bool want_v)
{
    const History &G = P->hist;
    RowArgs<T> A;
    int ng = 0;
    if (want_s) A.grp[ng++] = 0;
    if (want_v) A.grp[ng++] = 1;
    if (want_d) A.grp[ng++] = 2;
    if (want_d && !INV) A.grp[ng++] = 3;
    A.n = G.n;
    A.ncol = G.ncol;
    A.npass = G.rnpass;
    for (int i = 0; i < COL_MAXPASS; ++i) A.radix[i] = G.rradix[i];
    A.grid = (T *)G.grid;
    A.tw = (const double2 *)G.tw;
    // forward: the rows and columns of the sources' windows; inverse: those
    // of the targets' windows
    A.r0 = INV ? G.ty0 : G.sy0;
    A.nrow = INV ? G.ty1 - G.ty0 : G.sy1 - G.sy0;
    A.m0 = (INV ? G.tx0 : G.sx0) / 2;
    A.m1 = ((INV ? G.tx1 : G.sx1) + 1) / 2;
    A.B = P->bat;
    A.nblk = (int)(G.n / SPB);
    A.vflag = G.vflag;
    A.bflag = G.bflag;
    const size_t lds = sizeof(typename Vec2<T>::type) * (size_t)(G.n / 2);
    const int64_t rows = ng * (int64_t)P->bat * A.nrow;
    if (rows <= 0) return hipSuccess;
    auto go = [&](auto nmax) {
        constexpr int NMAX = decltype(nmax)::value;
        hipLaunchKernelGGL((k_rows<INV, T, NMAX>), dim3((unsigned)rows), dim3(NMAX / 16), lds, P->stream, A);
        return hipGetLastError();
    };
    if (G.n <= COL_NMAX / 4) return go(std::integral_constant<int, COL_NMAX / 4>());
    if (G.n <= COL_NMAX / 2) return go(std::integral_constant<int, COL_NMAX / 2>());
    return go(std::integral_constant<int, COL_NMAX>());
}

// only the fields of the densities given are transformed
hipError_t launch_rows(mhk_plan *P, bool inverse, bool s, bool d, bool v)
{
    if (P->p.prec == MHK_FP64)
        return inverse ? rows_t<true, double>(P, s, d, v) : rows_t<false, double>(P, s, d, v);
    return inverse ? rows_t<true, float>(P, s, d, v) : rows_t<false, float>(P, s, d, v);
}

hipError_t launch_columns(mhk_plan *P, bool s, bool d, bool v)
{
    return P->p.prec == MHK_FP64 ? columns_t<double>(P, s, d, v) : columns_t<float>(P, s, d, v);
}

hipError_t launch_multiply(mhk_plan *P)
{
    return P->p.prec == MHK_FP64 ? multiply_t<double>(P) : multiply_t<float>(P);
}

template <typename T>
static hipError_t interp_t(mhk_plan *P, bool want_s, bool want_d, bool want_v)
{
    const History &G = P->hist;
    InterpArgs<T> A;
    A.n = G.n;
    A.field = G.field;
    A.nout = P->nout;
    A.ntile = G.iedge > 0 ? (int)(G.n / G.iedge) : G.ntile;
    A.nrun = G.n_ttiles;
    A.gx0 = G.colpath ? G.tx0 : 0;
    A.gx1 = G.colpath ? G.tx1 : (int)G.n;
    A.gy0 = G.colpath ? G.ty0 : 0;
    A.gy1 = G.colpath ? G.ty1 : (int)G.n;
    A.B = P->bat;
    A.beta = G.beta;
    A.ox = G.ox;
    A.oy = G.oy;
    A.h = G.h;
    A.tile_xy = G.ttile_xy;
    A.tile_rng = G.ttile_rng;
    A.tx = P->tx;
    A.ty = P->ty;
    A.grid = (const T *)G.grid;
    A.wcoef = (const T *)G.wcoef;
    A.acc = (T *)P->acc;
    A.want_s = want_s;
    A.want_d = want_d;
    A.want_v = want_v;
    MHK_W_SWITCH(G.w, interp_w, T, P, A);
}

hipError_t launch_interp(mhk_plan *P, bool want_s, bool want_d, bool want_v)
{
    return P->p.prec == MHK_FP64 ? interp_t<double>(P, want_s, want_d, want_v)
                                 : interp_t<float>(P, want_s, want_d, want_v);
}

}  // namespace mhk
