// Boundary integral equations of Section 3.2 on the device: the dense Nystrom
// matrix of the double-layer operator, its matrix-vector product, restarted
// GMRES, and the Dirichlet and Neumann solves that combine them with the
// potential evaluation of a plan.
//
// Layout: off the diagonal K_ij = S_ij w_j (x_i - x_j).nu_j with S_ij = alpha
// K_1(alpha r)/(2 pi r) symmetric, so only S's lower triangle is kept, as FP64
// tiles of 64 x 128 (1.1 GB at N_B = 16384, 17 GB at 65536), resident in HBM for
// the life of the object, with the nodes' geometry and the diagonal of K.  The
// product y = (shift I + K) x streams the tiles once per call, each element
// serving rows i and j (HBM bound: 4 N_B^2 bytes); every other GMRES step is
// O(N_B m).
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "mhk_internal.h"

// partial sums of one product in flight: the object's own calls
// (mhk_nystrom_apply), its solves and the allocation-free solves may run on
// different streams, so each has its own
struct NysPart {
    double *cp = nullptr;       // [tiles][128] column sums
    double *rp = nullptr;       // [items][64] row sums
};

struct mhk_nystrom {
    int64_t n = 0, np = 0;      // nodes; padded to whole tile columns
    double alpha = 0;
    hipStream_t stream = nullptr;
    double *S = nullptr;        // [tiles][64][128]
    double *geo = nullptr;      // [6][np]: x, y, nu_x, nu_y, w, diagonal of K
    int64_t nstrip = 0, ntile = 0, nitem = 0;
    int run = 1;                // tiles per work item
    int2 *item = nullptr;       // [nitem] strip and first tile column
    int32_t *item_ofs = nullptr;  // [nstrip + 1] items of each strip
    NysPart prod[3];            // NYS_APPLY, NYS_SOLVE, NYS_NOALLOC
    std::mutex apply_mu;        // a product's two launches, which share prod[NYS_APPLY]
    double *na_part = nullptr;  // gpart of the allocation-free solves (restart <= NOALLOC_MAX_RESTART)
    // GMRES workspace (grown on demand)
    int m_cap = 0;
    int nblk = 0;
    double *V = nullptr;        // [m_cap + 1][n] Krylov basis
    double *wv = nullptr;       // [n]
    double *rv = nullptr;       // [n] residual / right-hand side
    double *part = nullptr;     // [(m_cap + 1) nblk] partial sums
    double *gpart = nullptr;    // [2][m_cap + 1][np/TC] partial sums of the Gram-Schmidt passes
    double *hd = nullptr;       // [2 (m_cap + 1) + 1] h (two passes) and |w|^2
    double *yd = nullptr;       // [m_cap] least-squares solution
    double *hh = nullptr;       // pinned host mirror of hd / yd
    // scratch of the Dirichlet and Neumann solves, [2][work_n]
    double *work = nullptr;
    int64_t work_n = 0;
    int64_t ws_bytes = 0;       // GMRES workspace
    double ms_assemble = 0;
    int64_t bytes() const
    {
        return (int64_t)sizeof(double) * (ntile * 64 * 128 + 6 * np + 3 * (ntile * 128 + nitem * 64) + np + 2 * work_n) +
               nitem * 8 + (nstrip + 1) * 4 + ws_bytes;
    }
};

namespace mhk {

#define BIE_HIP(call)                                                                     \
    do {                                                                                  \
        hipError_t e_ = (call);                                                           \
        if (e_ != hipSuccess) {                                                           \
            set_error(std::string("HIP error in ") + #call + ": " + hipGetErrorString(e_)); \
            return MHK_EHIP;                                                              \
        }                                                                                 \
    } while (0)

#define BIE_TRY(x)                        \
    do {                                  \
        mhk_status s_ = (x);              \
        if (s_ != MHK_OK) return s_;      \
    } while (0)

constexpr int BT = 256;         // threads per block of the vector kernels
constexpr int TR = 64, TC = 128;   // rows and columns of a tile
enum { NYS_APPLY, NYS_SOLVE, NYS_NOALLOC };

// tiles of the strips before strip I (strip k holds k/2 + 1 tile columns)
__host__ __device__ inline int64_t tile_ofs(int64_t I) { return I > 0 ? I + (I - 1) * (I - 1) / 4 : 0; }

// z e^z K_1(z) as a table of polynomials: eight segments of equal width per
// binade of z from 2^-52 to 2^10 (below, the function is 1 to rounding; above,
// e^{-z} underflows), degree 10 in the segment's local variable.  The function
// is smooth but for its logarithm at z = 0, at least 17 half-widths from the
// middle of a segment, so the interpolant errs by about 34^-11 = 1e-17.  The
// values come from the power series (DLMF 10.31.1) for z <= 1 and beyond from
// the trapezoidal rule (Trefethen and Weideman, SIAM Review 56 (2014), Section
// 5) on e^z K_1(z) = int_0^inf exp(-2 z sinh^2(t/2)) cosh t dt, both in long
// double, once per process.  The sum itself at every matrix element (20 to 90
// terms of sinh, exp and cosh) took 11.2 ms for 8192^2 elements; the table
// takes 0.31 ms and errs by 2.2e-16 instead of 8.5e-16 (relative, z in [1e-6, 700]).
constexpr int K1_LO = -52, K1_SEG = 8 * 62, K1_NC = 11;

static long double k1_scaled(long double z)
{
    if (z <= 1.0L) {
        // K_1 = 1/z + ln(z/2) I_1 - (z/4) sum (psi(k+1) + psi(k+2)) (z^2/4)^k / (k! (k+1)!)
        const long double q = z * z / 4, euler = 0.57721566490153286060651209L;
        long double term = 1, i1 = 0, s = 0, h = 0;      // term = q^k/(k! (k+1)!), h = H_k
        for (int k = 0; k < 24; ++k) {
            i1 += term;
            s += term * (2 * (h - euler) + 1.0L / (k + 1));
            h += 1.0L / (k + 1);
            term *= q / ((long double)(k + 1) * (k + 2));
        }
        return expl(z) * (1 + z * (logl(z / 2) * (z / 2) * i1 - (z / 4) * s));
    }
    const long double st = std::min(0.2L, 0.6L / sqrtl(z));
    const int n = (int)ceill(acoshl(1 + 50 / z) / st);
    long double s = 0.5L;
    for (int k = 1; k <= n; ++k) {
        const long double sh = sinhl(k * st / 2);
        s += expl(-2 * z * sh * sh) * coshl(k * st);
    }
    return z * st * s;
}

static const std::vector<double> &k1_table()
{
    static const std::vector<double> tab = [] {
        std::vector<double> t((size_t)K1_SEG * K1_NC);
        std::vector<long double> f(K1_NC), mono(K1_NC), tp(K1_NC), tc(K1_NC), tn(K1_NC);
        for (int sg = 0; sg < K1_SEG; ++sg) {
            const long double e = ldexpl(1.0L, K1_LO + sg / 8), z0 = e * (1 + sg % 8 / 8.0L), hw = e / 16;
            for (int i = 0; i < K1_NC; ++i) f[i] = k1_scaled(z0 + hw * (1 + cosl(M_PIl * (i + 0.5L) / K1_NC)));
            // Chebyshev coefficients to monomials
            std::fill(mono.begin(), mono.end(), 0.0L);
            std::fill(tp.begin(), tp.end(), 0.0L);
            std::fill(tc.begin(), tc.end(), 0.0L);
            tp[0] = 1;
            tc[1] = 1;
            for (int m = 0; m < K1_NC; ++m) {
                long double c = 0;
                for (int i = 0; i < K1_NC; ++i) c += f[i] * cosl(M_PIl * m * (i + 0.5L) / K1_NC);
                c *= (m == 0 ? 1.0L : 2.0L) / K1_NC;
                const std::vector<long double> &p = m == 0 ? tp : tc;
                for (int k = 0; k < K1_NC; ++k) mono[k] += c * p[k];
                if (m == 0) continue;
                for (int k = 0; k < K1_NC; ++k) tn[k] = (k > 0 ? 2 * tc[k - 1] : 0) - tp[k];
                tp = tc;
                tc = tn;
            }
            for (int k = 0; k < K1_NC; ++k) t[(size_t)sg * K1_NC + k] = (double)mono[k];
        }
        return t;
    }();
    return tab;
}

// z e^z K_1(z) from the table in LDS: the segment is the exponent and the
// three highest bits of the fraction, the local variable the others
__device__ inline double k1_scaled_dev(const double *tab, double z)
{
    const long long bits = __double_as_longlong(z);
    const int sg = min(K1_SEG - 1, max(0, (int)(bits >> 49) - ((1023 + K1_LO) << 3)));
    const double v = fma(2.0, __longlong_as_double(((bits << 3) & 0x000fffffffffffffll) | 0x3ff0000000000000ll), -3.0);
    const double *c = tab + sg * K1_NC;
    double p = c[K1_NC - 1];
#pragma unroll
    for (int k = K1_NC - 2; k >= 0; --k) p = fma(p, v, c[k]);
    return p;
}

// The tiles of S_ij = alpha K_1(alpha r)/(2 pi r), i > j (zero elsewhere and in
// the padding): K_ij = w_j S_ij (x_i - x_j).nu_j for i != j (Section 3.2; K_ii =
// -w_i kappa_i/(4 pi), the diagonal limit of eq. (dlp_diag_limit), is kept
// apart).  One workgroup per work item, a row per wavefront at a time, two
// columns per lane.
__global__ void __launch_bounds__(BT) k_nys_assemble(int64_t n, int64_t np, double alpha,
                                                     const double *__restrict__ geo, const double *__restrict__ tab,
                                                     const int2 *__restrict__ item, int run, double *__restrict__ S)
{
    __shared__ double k1[K1_SEG * K1_NC];
    for (int t = threadIdx.x; t < K1_SEG * K1_NC; t += BT) k1[t] = tab[t];
    __syncthreads();
    const int64_t I = item[blockIdx.x].x;
    const int c0 = item[blockIdx.x].y, c1 = min(c0 + run, (int)(I / 2 + 1));
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const double *x = geo, *y = geo + np;
    for (int c = c0; c < c1; ++c) {
        const int64_t j = (int64_t)c * TC + 2 * lane;
        const double2 xj = *reinterpret_cast<const double2 *>(x + j), yj = *reinterpret_cast<const double2 *>(y + j);
        double *tile = S + (tile_ofs(I) + c) * (TR * TC) + 2 * lane;
        for (int r = wave; r < TR; r += BT / 64) {
            const int64_t i = I * TR + r;
            auto elem = [&](double xv, double yv, int64_t jj) -> double {
                if (jj >= i || i >= n) return 0.0;
                const double dx = x[i] - xv, dy = y[i] - yv, r2 = dx * dx + dy * dy, z = alpha * sqrt(r2);
                return k1_scaled_dev(k1, z) * exp(-z) / (2.0 * M_PI * r2);
            };
            double2 v;
            v.x = elem(xj.x, yj.x, j);
            v.y = elem(xj.y, yj.y, j + 1);
            *reinterpret_cast<double2 *>(tile + r * TC) = v;
        }
    }
}

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Products of the tiles of one work item (a run of tile columns of one strip)
// with x.  A wavefront takes 16 rows of the strip, two columns per lane: every
// element adds to its row's sum (in registers over the run, reduced over the
// lanes at its end) and to its column's sum (reduced over the four wavefronts
// per tile).  Bound by HBM: 16384 nodes 0.206 ms (5.2 TB/s of tiles) against
// 0.356 with the dense matrix (6.0 TB/s), 8192 nodes 57 against 102 us; the ten
// FP64 instructions per element are a fifth of that.
__global__ void __launch_bounds__(BT, 3) k_symv(int64_t n, int64_t np, const double *__restrict__ S,
                                             const double *__restrict__ geo, const int2 *__restrict__ item, int run,
                                             const double *__restrict__ x, double *__restrict__ cp,
                                             double *__restrict__ rp)
{
    constexpr int RW = TR / (BT / 64);
    __shared__ double col[2][BT / 64][TC];
    __shared__ double row[TR][6];              // x, y, nu, w x of the strip's rows (broadcast reads)
    const int64_t I = item[blockIdx.x].x;
    const int c0 = item[blockIdx.x].y, c1 = min(c0 + run, (int)(I / 2 + 1));
    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const double *__restrict__ gx = geo, *__restrict__ gy = geo + np, *__restrict__ gnx = geo + 2 * np,
                               *__restrict__ gny = geo + 3 * np, *__restrict__ gw = geo + 4 * np;
    if (tid < TR) {
        const int64_t i = I * TR + tid;
        row[tid][0] = gx[i];
        row[tid][1] = gy[i];
        row[tid][2] = gnx[i];
        row[tid][3] = gny[i];
        row[tid][4] = i < n ? gw[i] * x[i] : 0.0;
    }
    __syncthreads();
    double acc[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) acc[r] = 0.0;
    // loads run half a tile ahead: the second half of the wavefront's rows while
    // the first is summed, the next tile's first half and columns while the
    // second is
    struct Cols {
        double2 x, y, nx, ny, w;
    };
    auto cols = [&](int c, Cols &q) {
        const int64_t j = (int64_t)c * TC + 2 * lane;
        auto two = [&](const double *g) { return *reinterpret_cast<const double2 *>(g + j); };
        q.x = two(gx);
        q.y = two(gy);
        q.nx = two(gnx);
        q.ny = two(gny);
        q.w = two(gw);
        // nodes come in panels of 16, so a lane's two columns are both nodes or both padding
        q.w.x *= j < n ? x[j] : 0.0;
        q.w.y *= j < n ? x[j + 1] : 0.0;
    };
    const double *tile = S + (tile_ofs(I) + c0) * (TR * TC) + wave * RW * TC + 2 * lane;
    auto half = [&](const double *p, double2 *s) {
#pragma unroll
        for (int r = 0; r < RW / 2; ++r) s[r] = *reinterpret_cast<const double2 *>(p + r * TC);
    };
    double2 s[RW / 2], s2[RW / 2];
    Cols q;
    half(tile, s);
    cols(c0, q);
    for (int c = c0; c < c1; ++c, tile += TR * TC) {
        half(tile + RW / 2 * TC, s2);
        double cs0 = 0.0, cs1 = 0.0;
        // diag: the tile holds the diagonal, and its elements from there on, zero in
        // S, are no part of the sums (nor is zero times an infinite x)
        auto one = [&](auto diag, int r, double2 sv) {
            const double *g = row[wave * RW + r];
            const double2 p = *reinterpret_cast<const double2 *>(g), nu = *reinterpret_cast<const double2 *>(g + 2);
            const double wi = g[4];
            const double dx0 = p.x - q.x.x, dy0 = p.y - q.y.x, dx1 = p.x - q.x.y, dy1 = p.y - q.y.y;
            // columns 2 lane and 2 lane + 1 of the tile, row wave RW + r of the strip's half
            const int below = wave * RW + r + (int)(I % 2) * TR - 2 * lane;      // i - j of the first column
            if (!diag || below > 0) {
                acc[r] = fma(sv.x * fma(dx0, q.nx.x, dy0 * q.ny.x), q.w.x, acc[r]);
                cs0 = fma(sv.x * fma(dx0, nu.x, dy0 * nu.y), wi, cs0);
            }
            if (!diag || below > 1) {
                acc[r] = fma(sv.y * fma(dx1, q.nx.y, dy1 * q.ny.y), q.w.y, acc[r]);
                cs1 = fma(sv.y * fma(dx1, nu.x, dy1 * nu.y), wi, cs1);
            }
            // the sums are formed here: left to itself the compiler moves them
            // past the barrier below, with their operands in scratch
            asm volatile("" : "+v"(acc[r]), "+v"(cs0), "+v"(cs1));
        };
        const bool dg = c == (int)(I / 2);
        if (dg) {
#pragma unroll
            for (int r = 0; r < RW / 2; ++r) one(std::true_type(), r, s[r]);
        } else {
#pragma unroll
            for (int r = 0; r < RW / 2; ++r) one(std::false_type(), r, s[r]);
        }
        // (the last tile once more at the end of the run)
        const int cn = min(c + 1, c1 - 1);
        half(tile + (cn - c) * (TR * TC), s);
        if (dg) {
#pragma unroll
            for (int r = 0; r < RW / 2; ++r) one(std::true_type(), RW / 2 + r, s2[r]);
        } else {
#pragma unroll
            for (int r = 0; r < RW / 2; ++r) one(std::false_type(), RW / 2 + r, s2[r]);
        }
        cols(cn, q);
        double(*cl)[TC] = col[c & 1];
        cl[wave][2 * lane] = cs0;
        cl[wave][2 * lane + 1] = cs1;
        __syncthreads();
        // the other buffer is written next: its readers passed the barrier above
        if (tid < TC)
            cp[(tile_ofs(I) + c) * TC + tid] = -(((cl[0][tid] + cl[1][tid]) + cl[2][tid]) + cl[3][tid]);
    }
    // the 16 rows' sums over the lanes, halving the rows a lane holds at each
    // step: 17 exchanges instead of 96; the row is bits 5..2 of the lane
    static_assert(RW == 16, "rows per wavefront");
#pragma unroll
    for (int h = RW / 2, m = 32; h >= 1; h /= 2, m /= 2) {
        const bool up = (lane & m) != 0;
#pragma unroll
        for (int r = 0; r < h; ++r) {
            const double keep = up ? acc[r + h] : acc[r], give = up ? acc[r] : acc[r + h];
            acc[r] = keep + __shfl_xor(give, m, 64);
        }
    }
    double v = acc[0] + __shfl_xor(acc[0], 2, 64);
    v += __shfl_xor(v, 1, 64);
    if ((lane & 3) == 0) rp[(int64_t)blockIdx.x * TR + wave * RW + lane / 4] = v;
}

// y_i = (shift + K_ii) x_i + the row sums of its strip's items + the column
// sums of the tiles below it, in a fixed order: 128 outputs per workgroup, the
// tiles dealt to eight groups of threads.  With a basis V (count > 0) the
// workgroup also leaves its share of the dot products V_k . y, part[k nblk +
// block].
constexpr int SG = 8;
__global__ void __launch_bounds__(TC * SG) k_symv_sum(int64_t n, int64_t np, int64_t nstrip,
                                                      const double *__restrict__ geo,
                                                      const int32_t *__restrict__ item_ofs,
                                                      const double *__restrict__ cp, const double *__restrict__ rp,
                                                      double shift, const double *__restrict__ x,
                                                      double *__restrict__ y, const double *__restrict__ V, int count,
                                                      double *__restrict__ part)
{
    __shared__ double sh[SG][TC];
    const int cc = threadIdx.x % TC, g = threadIdx.x / TC;
    const int64_t J = blockIdx.x, i = J * TC + cc;
    double s = 0.0;
#pragma unroll 4
    for (int64_t I = 2 * J + g; I < nstrip; I += SG) s += cp[(tile_ofs(I) + J) * TC + cc];
    const int64_t strip = i / TR;
    if (strip < nstrip)
        for (int it = item_ofs[strip] + g; it < item_ofs[strip + 1]; it += SG) s += rp[(int64_t)it * TR + i % TR];
    sh[g][cc] = s;
    __syncthreads();
    double yi = 0.0;
    if (g == 0 && i < n) {
        double v = sh[0][cc];
#pragma unroll
        for (int q = 1; q < SG; ++q) v += sh[q][cc];
        const double xi = x[i];
        yi = fma(shift, xi, fma(geo[5 * np + i], xi, v));
        y[i] = yi;
    }
    if (count == 0) return;
    __syncthreads();
    if (g == 0) sh[0][cc] = yi;
    __syncthreads();
    // one basis vector per wavefront at a time, two outputs per lane
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const double y0 = sh[0][lane], y1 = sh[0][64 + lane];
    const int64_t i0 = J * TC + lane;
    for (int k = wave; k < count; k += TC * SG / 64) {
        const double *v = V + (int64_t)k * n;
        double d = i0 < n ? v[i0] * y0 : 0.0;
        if (i0 + 64 < n) d = fma(v[i0 + 64], y1, d);
        d = wave_sum(d);
        if (lane == 0) part[(int64_t)k * gridDim.x + J] = d;
    }
}

// y = shift x + K x with nothing kept between launches, for products recorded
// into a graph: its replays may run beside the object's other products, whose
// partial sums k_symv keeps in the object; and one launch instead of two for
// products of few nodes.  One workgroup per 8 QW rows i forms their whole sums: of
// the triangle's rows for j < i and of its columns for j > i, so every element is
// read twice, by the workgroups of its row and of its column.  At step t
// workgroups of the 128 rows R take the elements of columns K = t - R (modulo the
// number of such groups), so both read a tile at the same time and one of the
// reads can come from the memory-side cache.  QW wavefronts a step (8 rows, or
// 128/QW rows of the columns, each), G steps at a time.  Bound by load latency
// (up to some 4096 nodes), then HBM.  Against the dense matrix, which has the same
// bytes in one pass: 512 nodes 4.9 us (4.9), 2048 10.2 (9.3), 4096 24 (26), 5632
// 42 (39), 8192 79 (97), 10240 131 (141), 16384 327 (354).
template <int QW, int G>
__global__ void __launch_bounds__(64 * QW * G) k_nys_rows(int64_t n, int64_t np, int64_t nstrip,
                                                      const double *__restrict__ S, const double *__restrict__ geo,
                                                      double shift, const double *__restrict__ x,
                                                      double *__restrict__ y)
{
    constexpr int RW = 8, NR = RW * QW, JW = TC / QW, LR = NR / 2, JL = 64 / LR;
    static_assert(JW <= TR && JW == RW * JL, "a wavefront's rows j lie in one strip");
    const int64_t i0 = (int64_t)blockIdx.x * NR;
    const int R = (int)(i0 / TC), NK = (int)(np / TC);
    const double *__restrict__ gx = geo, *__restrict__ gy = geo + np, *__restrict__ gnx = geo + 2 * np,
                               *__restrict__ gny = geo + 3 * np, *__restrict__ gw = geo + 4 * np;
    __shared__ __align__(16) double jd[QW * G][JW][6];     // x, y, nu, w x of a wavefront's rows j
    __shared__ double rs[QW * G][RW], cs[QW * G][NR];
    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64), qw = wave % QW;
    // rows j < i: this wavefront's 8 rows, two columns per lane; columns i of the
    // rows j > i: two columns per lane, JL rows per load
    const int64_t ir = i0 + RW * qw;
    const int c = 2 * (lane % LR), jr = lane / LR;
    const double *rowp = S + tile_ofs(i0 / TR) * (TR * TC) + (ir % TR) * TC + 2 * lane;
    // step t < NK: columns K = t - R; step NK: the columns of the tiles that hold the
    // diagonal, whose rows step 2R (modulo NK) took
    auto col_of = [&](int t) { return t == NK ? R : t >= R ? t - R : t - R + NK; };
    auto fetch = [&](int t, double2 *s) {
        const int K = col_of(t);
        const double *p = rowp + (int64_t)K * (TR * TC);
        int64_t step = TC;
        if (t == NK || K > R) {
            // (the last tile column's second strip may be missing: not summed below)
            const int64_t j0 = (int64_t)K * TC + JW * qw, strip = min(j0 / TR, nstrip - 1);
            p = S + (tile_ofs(strip) + R) * (TR * TC) + (j0 % TR + jr) * TC + i0 % TC + c;
            step = JL * TC;
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) s[r] = *reinterpret_cast<const double2 *>(p + r * step);
    };
    int t = wave / QW;
    double2 s[RW], ahead[RW];
    if (t <= NK) fetch(t, s);
    double xr[RW], yr[RW], acc[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        xr[r] = gx[ir + r];
        yr[r] = gy[ir + r];
        acc[r] = 0.0;
    }
    const double2 xc = *reinterpret_cast<const double2 *>(gx + i0 + c), yc = *reinterpret_cast<const double2 *>(gy + i0 + c);
    double a0 = 0.0, a1 = 0.0;
    // diag: the tile holds the diagonal; its other elements are no part of the
    // sums (nor is zero times an infinite x)
    auto rows = [&](auto diag, int K) {
        const int64_t j = (int64_t)K * TC + 2 * lane;
        auto two = [&](const double *g) { return *reinterpret_cast<const double2 *>(g + j); };
        const double2 xj = two(gx), yj = two(gy), nx = two(gnx), ny = two(gny);
        double2 w = two(gw);
        w.x *= j < n ? x[j] : 0.0;
        w.y *= j < n ? x[j + 1] : 0.0;
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            if (!diag || j < ir + r) acc[r] = fma(s[r].x * fma(xr[r] - xj.x, nx.x, (yr[r] - yj.x) * ny.x), w.x, acc[r]);
            if (!diag || j + 1 < ir + r)
                acc[r] = fma(s[r].y * fma(xr[r] - xj.y, nx.y, (yr[r] - yj.y) * ny.y), w.y, acc[r]);
        }
    };
    auto cols = [&](auto diag, int K) {
        const int64_t j0 = (int64_t)K * TC + JW * qw;
        if (j0 / TR >= nstrip) return;
        if (lane < JW) {
            const int64_t j = j0 + lane;
            double *d = jd[wave][lane];
            d[0] = gx[j];
            d[1] = gy[j];
            d[2] = gnx[j];
            d[3] = gny[j];
            d[4] = j < n ? gw[j] * x[j] : 0.0;
        }
        // the wavefront's own rows: its lanes' writes are read below, and again
        // overwritten at its next step
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int q = 0; q < RW; ++q) {
            const double *d = jd[wave][JL * q + jr];
            const double2 g = *reinterpret_cast<const double2 *>(d), nu = *reinterpret_cast<const double2 *>(d + 2);
            const double w = d[4];
            const int64_t below = j0 + JL * q + jr - (i0 + c);      // j - i of the first column
            if (!diag || below > 0) a0 = fma(s[q].x * fma(xc.x - g.x, nu.x, (yc.x - g.y) * nu.y), w, a0);
            if (!diag || below > 1) a1 = fma(s[q].y * fma(xc.y - g.x, nu.x, (yc.y - g.y) * nu.y), w, a1);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the next step's elements are loaded while this one's are summed
    for (; t <= NK; t += G) {
        if (t + G <= NK) fetch(t + G, ahead);
        const int K = col_of(t);
        if (t == NK)
            cols(std::true_type(), K);
        else if (K > R)
            cols(std::false_type(), K);
        else if (K < R)
            rows(std::false_type(), K);
        else
            rows(std::true_type(), K);
#pragma unroll
        for (int r = 0; r < RW; ++r) s[r] = ahead[r];
    }
    // the rows' sums over the lanes, halving the rows a lane holds at each step;
    // the row is bits 5..3 of the lane
#pragma unroll
    for (int h = RW / 2, m = 32; h >= 1; h /= 2, m /= 2) {
        const bool up = (lane & m) != 0;
#pragma unroll
        for (int r = 0; r < h; ++r) {
            const double keep = up ? acc[r + h] : acc[r], give = up ? acc[r] : acc[r + h];
            acc[r] = keep + __shfl_xor(give, m, 64);
        }
    }
    double v = acc[0];
#pragma unroll
    for (int m = 4; m >= 1; m /= 2) v += __shfl_xor(v, m, 64);
    if (lane % 8 == 0) rs[wave][lane / 8] = v;
#pragma unroll
    for (int m = LR; m < 64; m *= 2) {
        a0 += __shfl_xor(a0, m, 64);
        a1 += __shfl_xor(a1, m, 64);
    }
    if (lane < LR) {
        cs[wave][c] = a0;
        cs[wave][c + 1] = a1;
    }
    __syncthreads();
    if (tid < NR && i0 + tid < n) {
        v = 0.0;
#pragma unroll
        for (int g = 0; g < G; ++g) v += rs[QW * g + tid / RW][tid % RW];
#pragma unroll
        for (int q = 0; q < QW * G; ++q) v += cs[q][tid];
        const double xi = x[i0 + tid];
        y[i0 + tid] = fma(shift, xi, fma(geo[5 * np + i0 + tid], xi, v));
    }
}

__device__ inline double block_sum(double v, double *sh)
{
    const int tid = threadIdx.x;
    v = wave_sum(v);
    if ((tid & 63) == 0) sh[tid >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < BT / 64; ++q) s += sh[q];
    __syncthreads();
    return s;
}

// part[i nblk + b] = partial dot product of basis vector i with w over the
// b-th slice of the index range; grid (nblk, count)
__global__ void __launch_bounds__(BT) k_dots(int64_t n, const double *__restrict__ V, const double *__restrict__ w,
                                             int nblk, double *__restrict__ part)
{
    __shared__ double sh[BT / 64];
    const int i = blockIdx.y;
    const double *v = V + (int64_t)i * n;
    double s = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * BT + threadIdx.x; t < n; t += (int64_t)nblk * BT) s = fma(v[t], w[t], s);
    s = block_sum(s, sh);
    if (threadIdx.x == 0) part[(int64_t)i * nblk + blockIdx.x] = s;
}

// out[i] = sum_b part[i nblk + b], one block per i, fixed order
__global__ void __launch_bounds__(BT) k_reduce(const double *__restrict__ part, int nblk, double *__restrict__ out)
{
    __shared__ double sh[BT / 64];
    const int i = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += BT) s += part[(int64_t)i * nblk + b];
    s = block_sum(s, sh);
    if (threadIdx.x == 0) out[i] = s;
}

// One Gram-Schmidt pass of GMRES over 128 entries of w per workgroup, as the
// products leave them: h = the sums of the partial dot products of the pass
// before (every workgroup forms them, in the same order; the first one stores
// them), w -= sum_k h_k V_k, then its share of the next pass's dot products
// V_k . w, or (norm) of w . w.  A pass is one launch instead of the three of a
// reduction, an update and a dot product, four launches an iteration with the
// normalisation instead of ten: a solve of 24 iterations at 8192 nodes went
// from 3.9 to 3.5 ms with the matrix, a heat step at 16384 nodes from 6.4 to 5.9.
__global__ void __launch_bounds__(TC * SG) k_gs_pass(int64_t n, const double *__restrict__ V, int count,
                                                     const double *__restrict__ pin, double *__restrict__ h,
                                                     double *__restrict__ w, int norm, double *__restrict__ pout)
{
    extern __shared__ double hs[];                    // [count], then [SG][TC]
    double(*sh)[TC] = reinterpret_cast<double(*)[TC]>(hs + count);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, nblk = gridDim.x;
    for (int k = wave; k < count; k += TC * SG / 64) {
        double d = 0.0;
        for (int b = lane; b < nblk; b += 64) d += pin[(int64_t)k * nblk + b];
        d = wave_sum(d);
        if (lane == 0) {
            hs[k] = d;
            if (blockIdx.x == 0) h[k] = d;
        }
    }
    __syncthreads();
    const int cc = threadIdx.x % TC, g = threadIdx.x / TC;
    const int64_t i = (int64_t)blockIdx.x * TC + cc;
    double s = 0.0;
    if (i < n)
        for (int k = g; k < count; k += SG) s = fma(-hs[k], V[(int64_t)k * n + i], s);
    sh[g][cc] = s;
    __syncthreads();
    if (g == 0) {
        double v = i < n ? w[i] : 0.0;
#pragma unroll
        for (int q = 0; q < SG; ++q) v += sh[q][cc];
        if (i < n) w[i] = v;
        sh[0][cc] = i < n ? v : 0.0;
    }
    __syncthreads();
    const double y0 = sh[0][lane], y1 = sh[0][64 + lane];
    const int64_t i0 = (int64_t)blockIdx.x * TC + lane;
    if (norm) {
        if (wave == 0) {
            const double d = wave_sum(fma(y0, y0, y1 * y1));
            if (lane == 0) pout[blockIdx.x] = d;
        }
        return;
    }
    for (int k = wave; k < count; k += TC * SG / 64) {
        const double *v = V + (int64_t)k * n;
        double d = i0 < n ? v[i0] * y0 : 0.0;
        if (i0 + 64 < n) d = fma(v[i0 + 64], y1, d);
        d = wave_sum(d);
        if (lane == 0) pout[(int64_t)k * nblk + blockIdx.x] = d;
    }
}

// v = w / |w| with |w|^2 the sum of the partial sums (stored in *nrm2 by the
// first workgroup); zero when the norm vanishes: breakdown, v unused
__global__ void __launch_bounds__(BT) k_normalize(int64_t n, const double *__restrict__ w,
                                                  const double *__restrict__ pin, int nblk, double *__restrict__ nrm2,
                                                  double *__restrict__ v)
{
    __shared__ double sh[BT / 64];
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += BT) s += pin[b];
    s = block_sum(s, sh);
    const int64_t t = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (t == 0) *nrm2 = s;
    if (t < n) v[t] = s > 0.0 ? w[t] / sqrt(s) : 0.0;
}

// x += sum_{i < count} y[i] V_i
__global__ void __launch_bounds__(BT) k_combine(int64_t n, const double *__restrict__ V, int count,
                                                const double *__restrict__ yv, double *__restrict__ x)
{
    const int64_t t = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (t >= n) return;
    double s = x[t];
    for (int i = 0; i < count; ++i) s = fma(yv[i], V[(int64_t)i * n + t], s);
    x[t] = s;
}

__global__ void __launch_bounds__(BT) k_fill(int64_t n, double v, double *out)
{
    const int64_t t = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (t < n) out[t] = v;
}

// out = a p + b q (out may alias p or q)
__global__ void __launch_bounds__(BT) k_axpby(int64_t n, double a, const double *p, double b, const double *q,
                                              double *out)
{
    const int64_t t = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (t >= n) return;
    out[t] = a * p[t] + (q ? b * q[t] : 0.0);
}

// Dirichlet: u = V + D[mu] at the targets, the interior limit V + D[mu] - mu/2
// on the boundary nodes (jump relation, eq. (jumprel)).
__global__ void __launch_bounds__(BT) k_dirichlet_u(int64_t nt, int64_t nout, const double *__restrict__ d,
                                                    const double *__restrict__ mu, double *__restrict__ u)
{
    const int64_t s = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (s >= nout) return;
    double v = u[s] + d[s];
    if (s >= nt) v -= 0.5 * mu[s - nt];
    u[s] = v;
}

// Neumann: u = V + S[g] - D[u_b] at the targets, u_b on the boundary nodes.
__global__ void __launch_bounds__(BT) k_neumann_u(int64_t nt, int64_t nout, const double *__restrict__ sg,
                                                  const double *__restrict__ d, const double *__restrict__ ub,
                                                  double *__restrict__ u)
{
    const int64_t s = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (s >= nout) return;
    u[s] = s < nt ? u[s] + sg[s] - d[s] : ub[s - nt];
}

// f = alpha^2 u + F (F may be NULL): the source of one implicit-Euler step
__global__ void __launch_bounds__(BT) k_heat_source(int64_t n, double a2, const double *__restrict__ u,
                                                    const double *__restrict__ F, double *__restrict__ f)
{
    const int64_t s = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (s >= n) return;
    f[s] = a2 * u[s] + (F ? F[s] : 0.0);
}

// rhs[i] = a * p[off + i] + b * q[off + i]  (q may be NULL)
__global__ void __launch_bounds__(BT) k_rhs(int64_t n, int64_t off, double a, const double *p, double b,
                                            const double *q, double *rhs)
{
    const int64_t i = (int64_t)blockIdx.x * BT + threadIdx.x;
    if (i >= n) return;
    rhs[i] = a * p[off + i] + (q ? b * q[off + i] : 0.0);
}

static inline unsigned nb_of(int64_t n) { return (unsigned)((n + BT - 1) / BT); }

// GMRES workspace: device vectors and the host mirror of the small ones.
// The object's own workspace (nys_workspace) or the fixed scratch array of
// mhk_nystrom_solve_noalloc.
struct GmresWs {
    int set = NYS_SOLVE;        // partial sums of the products
    int nblk = 0;               // blocks of the two-stage dot products
    double *V = nullptr;        // [m + 1][n] Krylov basis
    double *wv = nullptr;       // [n]
    double *rv = nullptr;       // [n] residual / right-hand side
    double *part = nullptr;     // [(m + 1) nblk] partial sums
    double *gpart = nullptr;    // [2][m + 1][np/TC] partial sums of the Gram-Schmidt passes
    double *hd = nullptr;       // [2 (m + 1) + 1] h (two passes) and |w|^2
    double *yd = nullptr;       // [m] least-squares solution
    double *hh = nullptr;       // host, [2 (m + 1) + 1 + m]: mirror of hd, then y
    // host arrays of the least-squares problem: H [(m + 1) m], cs, sn, yv [m], g [m + 1]
    double *H = nullptr, *cs = nullptr, *sn = nullptr, *g = nullptr, *yv = nullptr;
};

static inline int gmres_nblk(int64_t n) { return (int)std::min<int64_t>(256, std::max<int64_t>(1, (n + BT - 1) / BT)); }

// Device buffers of a Nystrom object are allocated and freed in the order
// of its stream (hipFree would wait for every stream of the device, i.e.
// for other plans' work); an allocation is waited for on that stream before
// use, since the solves run on the plan's stream.
static mhk_status nys_alloc(mhk_nystrom *N, double **p, int64_t count)
{
    *p = nullptr;
    if (hipMallocAsync((void **)p, sizeof(double) * (size_t)std::max<int64_t>(count, 1), N->stream) != hipSuccess ||
        hipStreamSynchronize(N->stream) != hipSuccess) {
        (void)hipGetLastError();
        if (*p) (void)hipFreeAsync(*p, N->stream);
        *p = nullptr;
        set_error("device allocation of " + std::to_string(sizeof(double) * count) + " bytes failed");
        return MHK_ENOMEM;
    }
    return MHK_OK;
}

static void nys_free(mhk_nystrom *N, double **p)
{
    if (*p) (void)hipFreeAsync(*p, N->stream);
    *p = nullptr;
}

static void nys_free_ws(mhk_nystrom *N)
{
    for (double **p : {&N->V, &N->wv, &N->rv, &N->part, &N->gpart, &N->hd, &N->yd}) nys_free(N, p);
    delete[] N->hh;
    N->hh = nullptr;
    N->ws_bytes = 0;
    N->m_cap = 0;
}

static mhk_status nys_workspace(mhk_nystrom *N, int m)
{
    if (m <= N->m_cap) return MHK_OK;
    nys_free_ws(N);
    N->nblk = gmres_nblk(N->n);
    BIE_TRY(nys_alloc(N, &N->V, (int64_t)(m + 1) * N->n));
    BIE_TRY(nys_alloc(N, &N->wv, N->n));
    BIE_TRY(nys_alloc(N, &N->rv, N->n));
    BIE_TRY(nys_alloc(N, &N->part, (int64_t)(m + 1) * N->nblk));
    BIE_TRY(nys_alloc(N, &N->gpart, 2 * (int64_t)(m + 1) * (N->np / TC)));
    BIE_TRY(nys_alloc(N, &N->hd, 2 * (m + 1) + 1));
    BIE_TRY(nys_alloc(N, &N->yd, m));
    // host mirror of the few Arnoldi values copied back per iteration
    // (pageable: pinned host memory would have to be released with
    // hipHostFree, which waits for the whole device)
    N->hh = new double[(size_t)(2 * (m + 1) + 1 + m)];
    N->m_cap = m;
    N->ws_bytes = (int64_t)sizeof(double) * ((int64_t)(m + 3) * N->n + (int64_t)(m + 1) * (N->nblk + 2 * (N->np / TC)) + 3 * (m + 1));
    return MHK_OK;
}

// The object's own workspace as a GmresWs, with host arrays for restart m.
struct OwnWs {
    GmresWs W;
    std::vector<double> H, cs, sn, g, yv;
};

static mhk_status own_workspace(mhk_nystrom *N, int m, OwnWs &o)
{
    BIE_TRY(nys_workspace(N, m));
    o.H.assign((size_t)(m + 1) * m, 0.0);
    o.cs.assign(m, 0.0);
    o.sn.assign(m, 0.0);
    o.g.assign(m + 1, 0.0);
    o.yv.assign(m, 0.0);
    GmresWs &W = o.W;
    W.nblk = N->nblk;
    W.V = N->V; W.wv = N->wv; W.rv = N->rv; W.part = N->part; W.gpart = N->gpart; W.hd = N->hd; W.yd = N->yd; W.hh = N->hh;
    W.H = o.H.data(); W.cs = o.cs.data(); W.sn = o.sn.data(); W.g = o.g.data(); W.yv = o.yv.data();
    return MHK_OK;
}

static mhk_status nys_scratch(mhk_nystrom *N, int64_t nout)
{
    if (nout <= N->work_n) return MHK_OK;
    nys_free(N, &N->work);
    N->work_n = 0;
    BIE_TRY(nys_alloc(N, &N->work, 2 * nout));
    N->work_n = nout;
    return MHK_OK;
}

// y = (shift I + K) x with partial sums in set `set`
// (and, with a basis, the partial dot products of y with its count vectors)
static hipError_t product(const mhk_nystrom *N, int set, double shift, const double *x, double *y, hipStream_t st,
                          const double *V = nullptr, int count = 0, double *part = nullptr)
{
    const NysPart &p = N->prod[set];
    hipLaunchKernelGGL(k_symv, dim3((unsigned)N->nitem), dim3(BT), 0, st, N->n, N->np, (const double *)N->S,
                       (const double *)N->geo, (const int2 *)N->item, N->run, x, p.cp, p.rp);
    hipLaunchKernelGGL(k_symv_sum, dim3((unsigned)(N->np / TC)), dim3(TC * SG), 0, st, N->n, N->np, N->nstrip,
                       (const double *)N->geo, (const int32_t *)N->item_ofs, (const double *)p.cp,
                       (const double *)p.rp, shift, x, y, V, count, part);
    return hipGetLastError();
}

// out[0..count) = dot products of V_0..V_{count-1} with w (device result)
static hipError_t dots(const mhk_nystrom *N, const GmresWs &W, const double *V, int count, const double *w,
                       double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_dots, dim3((unsigned)W.nblk, (unsigned)count), dim3(BT), 0, st, N->n, V, w, W.nblk,
                       W.part);
    hipLaunchKernelGGL(k_reduce, dim3((unsigned)count), dim3(BT), 0, st, W.part, W.nblk, out);
    return hipGetLastError();
}

// host copy of a device scalar
static mhk_status fetch(mhk_nystrom *N, const double *d, int count, double *h, hipStream_t st)
{
    BIE_HIP(hipMemcpyAsync(h, d, sizeof(double) * count, hipMemcpyDeviceToHost, st));
    BIE_HIP(hipStreamSynchronize(st));
    return MHK_OK;
}

// Restarted GMRES(m) for (shift I + K) x = b, x = 0 initially; classical
// Gram-Schmidt with one re-orthogonalisation on the device, Givens rotations
// of the small Hessenberg matrix on the host.  Converged when the true
// residual |b - A x| <= tol |b| at the end of a cycle.
static mhk_status gmres(mhk_nystrom *N, const GmresWs &W, double shift, const double *b, double *x, double tol,
                        int m, int maxit, hipStream_t st, mhk_solve_info *info)
{
    const int64_t n = N->n;
    double *hh = W.hh, *h1 = W.hd, *h2 = W.hd + (m + 1), *nrm = W.hd + 2 * (m + 1);
    hipLaunchKernelGGL(k_fill, dim3(nb_of(n)), dim3(BT), 0, st, n, 0.0, x);
    BIE_HIP(hipGetLastError());
    BIE_HIP(dots(N, W, b, 1, b, nrm, st));
    double bn2;
    BIE_TRY(fetch(N, nrm, 1, &bn2, st));
    const double bnorm = sqrt(bn2);
    info->iters = 0;
    info->resid = 0.0;
    info->converged = 1;
    if (!(bnorm > 0.0)) return MHK_OK;
    if (!std::isfinite(bnorm)) {
        set_error("right-hand side is not finite");
        return MHK_EINVAL;
    }
    const int gblk = (int)(N->np / TC);               // workgroups of the Gram-Schmidt passes
    double *H = W.H, *cs = W.cs, *sn = W.sn, *g = W.g, *yv = W.yv;
    int total = 0;
    bool first = true;
    for (;;) {
        // r = b - A x
        if (first) {
            BIE_HIP(hipMemcpyAsync(W.rv, b, sizeof(double) * n, hipMemcpyDeviceToDevice, st));
        } else {
            BIE_HIP(product(N, W.set, shift, x, W.wv, st));
            hipLaunchKernelGGL(k_axpby, dim3(nb_of(n)), dim3(BT), 0, st, n, 1.0, b, -1.0, (const double *)W.wv,
                               W.rv);
            BIE_HIP(hipGetLastError());
        }
        first = false;
        BIE_HIP(dots(N, W, W.rv, 1, W.rv, nrm, st));
        double r2;
        BIE_TRY(fetch(N, nrm, 1, &r2, st));
        const double beta = sqrt(r2);
        info->resid = beta / bnorm;
        if (!std::isfinite(beta)) {
            set_error("GMRES residual is not finite");
            return MHK_EHIP;
        }
        if (beta <= tol * bnorm) {
            info->converged = 1;
            break;
        }
        if (total >= maxit) {
            info->converged = 0;
            break;
        }
        // nrm holds |r|^2 (its own only partial sum here)
        hipLaunchKernelGGL(k_normalize, dim3(nb_of(n)), dim3(BT), 0, st, n, (const double *)W.rv,
                           (const double *)nrm, 1, W.part, W.V);
        BIE_HIP(hipGetLastError());
        std::fill(g, g + m + 1, 0.0);
        g[0] = beta;
        int jend = 0;
        for (int j = 0; j < m; ++j) {
            const double *vj = W.V + (int64_t)j * n;
            // the passes' partial sums alternate between the halves of `gpart`
            double *p0 = W.gpart, *p1 = W.gpart + (int64_t)(m + 1) * gblk;
            const size_t lds = sizeof(double) * (size_t)(j + 1 + SG * TC);
            BIE_HIP(product(N, W.set, shift, vj, W.wv, st, W.V, j + 1, p0));
            hipLaunchKernelGGL(k_gs_pass, dim3((unsigned)gblk), dim3(TC * SG), lds, st, n, (const double *)W.V, j + 1,
                               (const double *)p0, h1, W.wv, 0, p1);
            hipLaunchKernelGGL(k_gs_pass, dim3((unsigned)gblk), dim3(TC * SG), lds, st, n, (const double *)W.V, j + 1,
                               (const double *)p1, h2, W.wv, 1, p0);
            hipLaunchKernelGGL(k_normalize, dim3(nb_of(n)), dim3(BT), 0, st, n, (const double *)W.wv,
                               (const double *)p0, gblk, nrm, W.V + (int64_t)(j + 1) * n);
            BIE_HIP(hipGetLastError());
            BIE_TRY(fetch(N, W.hd, 2 * (m + 1) + 1, hh, st));
            double *col = &H[(size_t)j * (m + 1)];
            for (int i = 0; i <= j; ++i) col[i] = hh[i] + hh[(m + 1) + i];
            const double hn = sqrt(std::max(0.0, hh[2 * (m + 1)]));
            col[j + 1] = hn;
            for (int i = 0; i < j; ++i) {
                const double a = col[i], c = col[i + 1];
                col[i] = cs[i] * a + sn[i] * c;
                col[i + 1] = -sn[i] * a + cs[i] * c;
            }
            const double den = hypot(col[j], col[j + 1]);
            cs[j] = den > 0 ? col[j] / den : 1.0;
            sn[j] = den > 0 ? col[j + 1] / den : 0.0;
            col[j] = den;
            col[j + 1] = 0.0;
            g[j + 1] = -sn[j] * g[j];
            g[j] = cs[j] * g[j];
            ++total;
            jend = j + 1;
            if (fabs(g[j + 1]) <= tol * bnorm || total >= maxit || !(hn > 0.0)) break;
        }
        // back substitution H y = g, then x += V y
        for (int i = jend - 1; i >= 0; --i) {
            double s = g[i];
            for (int k = i + 1; k < jend; ++k) s -= H[(size_t)k * (m + 1) + i] * yv[k];
            const double d = H[(size_t)i * (m + 1) + i];
            yv[i] = d != 0.0 ? s / d : 0.0;
        }
        double *yh = hh + 2 * (m + 1) + 1;
        for (int i = 0; i < jend; ++i) yh[i] = yv[i];
        BIE_HIP(hipMemcpyAsync(W.yd, yh, sizeof(double) * jend, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_combine, dim3(nb_of(n)), dim3(BT), 0, st, n, (const double *)W.V, jend,
                           (const double *)W.yd, x);
        BIE_HIP(hipGetLastError());
        // the pinned buffer is reused by the next fetch: wait for the copy
        BIE_HIP(hipStreamSynchronize(st));
    }
    info->iters = total;
    return MHK_OK;
}

// Scratch of mhk_nystrom_solve_noalloc: one fixed device array of
// NOALLOC_DOUBLES doubles (32 MiB), held by every GPU the library runs on
// until the process ends.  Host code never passes the array's name to a
// kernel (on the host it stands for no device address): the address of each
// device's copy is looked up once, with that device current, and kept.
constexpr int64_t NOALLOC_DOUBLES = (int64_t)4 << 20;
constexpr int NOALLOC_MAX_RESTART = 64;
constexpr int NOALLOC_MAX_DEVICES = 64;
static __device__ __align__(256) double scratch[NOALLOC_DOUBLES];
static std::mutex g_scratch_mu;
static double *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

static mhk_status scratch_base(double **out)
{
    int dev = 0;
    BIE_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) {
        set_error("device index out of the range of the scratch table");
        return MHK_EUNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error(std::string("hipGetSymbolAddress of the scratch array: ") + hipGetErrorString(e));
            return MHK_EHIP;
        }
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return MHK_OK;
}

static inline int64_t round256(int64_t count) { return (count + 31) / 32 * 32; }   // doubles -> 256 B

static mhk_status check_solve(mhk_plan *P, mhk_nystrom *N, const void *g, const void *f_vol, const void *f_trg,
                              double tol, int restart, int maxit, const void *dens, const void *u)
{
    if (!P || !N || !g || !dens || !u) {
        set_error("null plan, Nystrom matrix, data or output pointer");
        return MHK_EINVAL;
    }
    if (P->p.prec != MHK_FP64 || P->p.batch != 1 || P->p.local_order >= 2) {
        set_error("the boundary integral solves need an FP64 plan with batch 1 and first-order local expansions");
        return MHK_EUNSUPPORTED;
    }
    if (P->nout != P->nt + P->nb) {
        set_error("the boundary integral solves need a plan with on-surface targets");
        return MHK_EINVAL;
    }
    if (P->nb != N->n || P->p.alpha != N->alpha) {
        set_error("plan and Nystrom matrix differ in boundary size or alpha");
        return MHK_EINVAL;
    }
    if ((f_vol == nullptr) != (f_trg == nullptr)) {
        set_error("f_vol and f_trg must be given together");
        return MHK_EINVAL;
    }
    if (f_vol && P->nv == 0) {
        set_error("volume source given but the plan has no volume nodes");
        return MHK_EINVAL;
    }
    if (!(tol > 0.0 && tol < 1.0) || restart < 1 || restart > 1000 || maxit < 1) {
        set_error("need 0 < tol < 1, 1 <= restart <= 1000, maxit >= 1");
        return MHK_EINVAL;
    }
    return MHK_OK;
}

}  // namespace mhk

using namespace mhk;

extern "C" {

mhk_status mhk_nystrom_create(double alpha, const mhk_boundary *b, void *hip_stream, mhk_nystrom **out)
{
    if (!out) {
        set_error("null output handle");
        return MHK_EINVAL;
    }
    *out = nullptr;
    if (!b || !(alpha > 0.0) || !std::isfinite(alpha) || b->n_panels < 1 || !b->x || !b->y || !b->nx || !b->ny ||
        !b->w || !b->kappa) {
        set_error("need alpha > 0 and a boundary with panels and all node arrays");
        return MHK_EINVAL;
    }
    const int64_t n = b->n_panels * NGL;
    if (n > (int64_t)1 << 20) {
        set_error("boundary too large for a dense Nystrom matrix");
        return MHK_EUNSUPPORTED;
    }
    mhk_nystrom *N = new mhk_nystrom();
    N->n = n;
    N->np = (n + TC - 1) / TC * TC;
    N->alpha = alpha;
    N->stream = (hipStream_t)hip_stream;
    N->nstrip = (n + TR - 1) / TR;
    N->ntile = tile_ofs(N->nstrip);
    // tiles per work item: as many items as keep the device busy to the end
    // (4096: four workgroups on each of 256 CUs, four times over)
    N->run = (int)std::min<int64_t>(8, std::max<int64_t>(1, N->ntile / 4096));
    std::vector<int2> item;
    std::vector<int32_t> item_ofs((size_t)N->nstrip + 1, 0);
    for (int64_t I = N->nstrip - 1; I >= 0; --I) item_ofs[(size_t)I + 1] = (int32_t)((I / 2 + N->run) / N->run);
    for (int64_t I = 0; I < N->nstrip; ++I) {
        item_ofs[(size_t)I + 1] += item_ofs[(size_t)I];
        for (int64_t c = 0; c < I / 2 + 1; c += N->run) item.push_back(make_int2((int)I, (int)c));
    }
    N->nitem = (int64_t)item.size();
    const std::vector<double> &k1 = k1_table();
    double *tab = nullptr, *ia = nullptr, *io = nullptr;
    mhk_status st = nys_alloc(N, &N->S, N->ntile * TR * TC);
    if (st == MHK_OK) st = nys_alloc(N, &N->geo, 6 * N->np);
    if (st == MHK_OK) st = nys_alloc(N, &N->na_part, 2 * (int64_t)(NOALLOC_MAX_RESTART + 1) * (N->np / TC));
    if (st == MHK_OK) st = nys_alloc(N, &tab, (int64_t)k1.size());
    if (st == MHK_OK) st = nys_alloc(N, &ia, N->nitem);
    N->item = reinterpret_cast<int2 *>(ia);
    if (st == MHK_OK) st = nys_alloc(N, &io, (N->nstrip + 2) / 2);
    N->item_ofs = reinterpret_cast<int32_t *>(io);
    for (NysPart &p : N->prod) {
        if (st == MHK_OK) st = nys_alloc(N, &p.cp, N->ntile * TC);
        if (st == MHK_OK) st = nys_alloc(N, &p.rp, N->nitem * TR);
    }
    if (st != MHK_OK) {
        nys_free(N, &tab);
        mhk_nystrom_destroy(N);
        return st;
    }
    std::vector<double> h(6 * (size_t)N->np, 0.0);
    const double *src[5] = {b->x, b->y, b->nx, b->ny, b->w};
    for (int k = 0; k < 5; ++k) memcpy(&h[(size_t)(k * N->np)], src[k], sizeof(double) * n);
    for (int64_t i = 0; i < n; ++i) h[(size_t)(5 * N->np + i)] = -b->w[i] * b->kappa[i] / (4.0 * M_PI);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto up = [&](void *d, const void *s, size_t bytes) {
        return hipMemcpyAsync(d, s, bytes, hipMemcpyHostToDevice, N->stream);
    };
    hipError_t e = up(N->geo, h.data(), sizeof(double) * h.size());
    if (e == hipSuccess) e = up(tab, k1.data(), sizeof(double) * k1.size());
    if (e == hipSuccess) e = up(N->item, item.data(), sizeof(int2) * item.size());
    if (e == hipSuccess) e = up(N->item_ofs, item_ofs.data(), sizeof(int32_t) * item_ofs.size());
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = hipEventRecord(e0, N->stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_nys_assemble, dim3((unsigned)N->nitem), dim3(BT), 0, N->stream, n, N->np, alpha,
                           (const double *)N->geo, (const double *)tab, (const int2 *)N->item, N->run, N->S);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipEventRecord(e1, N->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(N->stream);
    float ms = 0;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    nys_free(N, &tab);
    if (e != hipSuccess) {
        set_error(std::string("Nystrom assembly: ") + hipGetErrorString(e));
        mhk_nystrom_destroy(N);
        return MHK_EHIP;
    }
    N->ms_assemble = ms;
    *out = N;
    return MHK_OK;
}

mhk_status mhk_nystrom_info(const mhk_nystrom *N, mhk_nys_info *info)
{
    if (!N || !info) {
        set_error("null Nystrom matrix or info");
        return MHK_EINVAL;
    }
    info->n = N->n;
    info->alpha = N->alpha;
    info->device_bytes = N->bytes();
    info->ms_assemble = N->ms_assemble;
    return MHK_OK;
}

mhk_status mhk_nystrom_apply(mhk_nystrom *N, double shift, const double *x, double *y)
{
    if (!N || !x || !y || x == y) {
        set_error("null Nystrom matrix or vector, or x aliases y");
        return MHK_EINVAL;
    }
    // products that must keep no partial sums in the object: recorded ones, and
    // those of threads that each have a stream of their own under this handle; and
    // those of few nodes, where the triangle's two launches take longer (128 nodes
    // 7.9 us against 3.9, 1536 9.1 against 7.6, 2048 10.3 against 10.2)
    bool alone = N->n <= 2048 || N->stream == hipStreamPerThread;
    if (!alone && N->stream) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        BIE_HIP(hipStreamIsCapturing(N->stream, &cap));
        alone = cap == hipStreamCaptureStatusActive;
    }
    if (alone) {
        auto rows = [&](auto qw, auto g) {
            constexpr int QW = decltype(qw)::value, G = decltype(g)::value;
            hipLaunchKernelGGL((k_nys_rows<QW, G>), dim3((unsigned)((N->n + 8 * QW - 1) / (8 * QW))), dim3(64 * QW * G),
                               0, N->stream, N->n, N->np, N->nstrip, (const double *)N->S, (const double *)N->geo,
                               shift, x, y);
        };
        // few rows a workgroup while the chip has room for all (2048 nodes 10.2 us, 14
        // with <4, 3>, as 4096 24 and 28); 32 of them with as many wavefronts as fit a
        // CU (8192: 79, 81 with <2, 6>); beyond 256 such workgroups several small ones
        // on a CU, which leave the CUs evenly loaded (10240: 131 against 169); and
        // large ones again once those are many too (14336: 262 against 298; 16384:
        // 327 against 377)
        if (N->n <= 4096)
            rows(std::integral_constant<int, 2>(), std::integral_constant<int, 6>());
        else if (N->n > 8192 && N->n <= 12288)
            rows(std::integral_constant<int, 2>(), std::integral_constant<int, 2>());
        else
            rows(std::integral_constant<int, 4>(), std::integral_constant<int, 3>());
        BIE_HIP(hipGetLastError());
        return MHK_OK;
    }
    std::lock_guard<std::mutex> lock(N->apply_mu);
    BIE_HIP(product(N, NYS_APPLY, shift, x, y, N->stream));
    return MHK_OK;
}

mhk_status mhk_nystrom_solve(mhk_nystrom *N, double shift, const double *rhs, double *x, double tol, int restart,
                             int maxit, mhk_solve_info *info)
{
    if (!N || !rhs || !x || !info || rhs == x) {
        set_error("null Nystrom matrix, vector or info, or rhs aliases x");
        return MHK_EINVAL;
    }
    if (!(tol > 0.0 && tol < 1.0) || restart < 1 || restart > 1000 || maxit < 1) {
        set_error("need 0 < tol < 1, 1 <= restart <= 1000, maxit >= 1");
        return MHK_EINVAL;
    }
    memset(info, 0, sizeof(*info));
    OwnWs o;
    BIE_TRY(own_workspace(N, restart, o));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    BIE_HIP(hipEventCreate(&e0));
    BIE_HIP(hipEventCreate(&e1));
    BIE_HIP(hipEventRecord(e0, N->stream));
    mhk_status st = gmres(N, o.W, shift, rhs, x, tol, restart, maxit, N->stream, info);
    if (st == MHK_OK) {
        BIE_HIP(hipEventRecord(e1, N->stream));
        BIE_HIP(hipEventSynchronize(e1));
        float ms = 0;
        BIE_HIP(hipEventElapsedTime(&ms, e0, e1));
        info->ms_gmres = ms;
        info->ms_total = ms;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return st;
}

mhk_status mhk_nystrom_solve_noalloc(mhk_nystrom *N, double shift, const double *rhs, double *x, double tol,
                                     int restart, int maxit, mhk_solve_info *info)
{
    if (!N || !rhs || !x || !info || rhs == x) {
        set_error("null Nystrom matrix, vector or info, or rhs aliases x");
        return MHK_EINVAL;
    }
    if (!(tol > 0.0 && tol < 1.0) || restart < 1 || restart > NOALLOC_MAX_RESTART || maxit < 1) {
        set_error("need 0 < tol < 1, 1 <= restart <= " + std::to_string(NOALLOC_MAX_RESTART) + ", maxit >= 1");
        return MHK_EINVAL;
    }
    const int m = restart;
    const int64_t n = N->n;
    const int nblk = gmres_nblk(n);
    const int64_t nV = round256((int64_t)(m + 1) * n), nvec = round256(n), npart = round256((int64_t)(m + 1) * nblk),
                  nhd = round256(2 * (m + 1) + 1), nyd = round256(m);
    const int64_t need = nV + 2 * nvec + npart + nhd + nyd;
    if (need > NOALLOC_DOUBLES) {
        set_error("GMRES needs " + std::to_string(need * 8) + " bytes of scratch at N_B = " + std::to_string(n) +
                  " and restart " + std::to_string(m) + "; the fixed scratch holds " +
                  std::to_string(NOALLOC_DOUBLES * 8));
        return MHK_EINVAL;
    }
    double *base = nullptr;
    BIE_TRY(scratch_base(&base));
    GmresWs W;
    W.set = NYS_NOALLOC;
    W.nblk = nblk;
    W.V = base;
    W.wv = W.V + nV;
    W.rv = W.wv + nvec;
    W.part = W.rv + nvec;
    W.gpart = N->na_part;
    W.hd = W.part + npart;
    W.yd = W.hd + nhd;
    // host side of the least-squares problem on the stack (restart <= 64)
    double hh[2 * (NOALLOC_MAX_RESTART + 1) + 1 + NOALLOC_MAX_RESTART];
    double H[(NOALLOC_MAX_RESTART + 1) * NOALLOC_MAX_RESTART];
    double cs[NOALLOC_MAX_RESTART], sn[NOALLOC_MAX_RESTART], g[NOALLOC_MAX_RESTART + 1], yv[NOALLOC_MAX_RESTART];
    W.hh = hh;
    W.H = H;
    W.cs = cs;
    W.sn = sn;
    W.g = g;
    W.yv = yv;
    memset(info, 0, sizeof(*info));
    const auto t0 = std::chrono::steady_clock::now();
    const mhk_status st = gmres(N, W, shift, rhs, x, tol, m, maxit, N->stream, info);
    if (st == MHK_OK) {
        // GMRES ends with the stream synchronised
        const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        info->ms_gmres = ms;
        info->ms_total = ms;
    }
    return st;
}

static mhk_status solve_common(mhk_plan *P, mhk_nystrom *N, int neumann, const double *g, const double *f_vol,
                               const double *f_trg, double tol, int restart, int maxit, double *dens, double *u,
                               mhk_solve_info *info)
{
    BIE_TRY(check_solve(P, N, g, f_vol, f_trg, tol, restart, maxit, dens, u));
    if (!info) {
        set_error("null solve info");
        return MHK_EINVAL;
    }
    memset(info, 0, sizeof(*info));
    hipStream_t st = P->stream;
    const int64_t nt = P->nt, nb = P->nb, nout = P->nout;
    BIE_TRY(nys_scratch(N, nout));
    OwnWs o;
    BIE_TRY(own_workspace(N, restart, o));
    double *w1 = N->work, *w2 = N->work + N->work_n;
    hipEvent_t ev[4] = {};
    for (auto &e : ev) BIE_HIP(hipEventCreate(&e));
    mhk_status rc = MHK_OK;
#define SOLVE_HIP(call)                                                                       \
    if ((call) != hipSuccess) {                                                               \
        set_error(std::string("HIP error in the boundary integral solve: ") + #call);         \
        rc = MHK_EHIP;                                                                        \
        break;                                                                                \
    }
    do {
        SOLVE_HIP(hipEventRecord(ev[0], st));
        // right-hand side: Dirichlet g - V on the boundary, Neumann V + S[g]
        if (neumann) {
            rc = mhk_eval_parts(P, MHK_PART_ALL, g, nullptr, f_vol, f_trg, w1, nullptr, f_vol ? u : nullptr);
            if (rc != MHK_OK) break;
            if (!f_vol) hipLaunchKernelGGL(k_fill, dim3(nb_of(nout)), dim3(BT), 0, st, nout, 0.0, u);
            hipLaunchKernelGGL(k_rhs, dim3(nb_of(nb)), dim3(BT), 0, st, nb, nt, 1.0, (const double *)u, 1.0,
                               (const double *)w1, o.W.rv);
        } else {
            if (f_vol) {
                rc = mhk_eval_parts(P, MHK_PART_ALL, nullptr, nullptr, f_vol, f_trg, nullptr, nullptr, u);
                if (rc != MHK_OK) break;
            } else {
                hipLaunchKernelGGL(k_fill, dim3(nb_of(nout)), dim3(BT), 0, st, nout, 0.0, u);
            }
            hipLaunchKernelGGL(k_rhs, dim3(nb_of(nb)), dim3(BT), 0, st, nb, (int64_t)0, 1.0, g, -1.0,
                               (const double *)(u + nt), o.W.rv);
        }
        SOLVE_HIP(hipGetLastError());
        SOLVE_HIP(hipEventRecord(ev[1], st));
        // GMRES on (-/+ 1/2 I + K); the right-hand side lives in the
        // residual vector, which GMRES overwrites, so it is first copied to w2
        SOLVE_HIP(hipMemcpyAsync(w2, o.W.rv, sizeof(double) * nb, hipMemcpyDeviceToDevice, st));
        rc = gmres(N, o.W, neumann ? 0.5 : -0.5, w2, dens, tol, restart, maxit, st, info);
        if (rc != MHK_OK) break;
        SOLVE_HIP(hipEventRecord(ev[2], st));
        // representation at every output
        rc = mhk_eval_parts(P, MHK_PART_ALL, nullptr, dens, nullptr, nullptr, nullptr, w2, nullptr);
        if (rc != MHK_OK) break;
        if (neumann)
            hipLaunchKernelGGL(k_neumann_u, dim3(nb_of(nout)), dim3(BT), 0, st, nt, nout, (const double *)w1,
                               (const double *)w2, (const double *)dens, u);
        else
            hipLaunchKernelGGL(k_dirichlet_u, dim3(nb_of(nout)), dim3(BT), 0, st, nt, nout, (const double *)w2,
                               (const double *)dens, u);
        SOLVE_HIP(hipGetLastError());
        SOLVE_HIP(hipEventRecord(ev[3], st));
        SOLVE_HIP(hipEventSynchronize(ev[3]));
        float a = 0, b = 0, c = 0;
        (void)hipEventElapsedTime(&a, ev[0], ev[1]);
        (void)hipEventElapsedTime(&b, ev[1], ev[2]);
        (void)hipEventElapsedTime(&c, ev[2], ev[3]);
        info->ms_eval = a + c;
        info->ms_gmres = b;
        info->ms_total = a + b + c;
    } while (0);
#undef SOLVE_HIP
    for (auto &e : ev) (void)hipEventDestroy(e);
    return rc;
}

mhk_status mhk_solve_dirichlet(mhk_plan *plan, mhk_nystrom *nys, const double *g, const double *f_vol,
                               const double *f_trg, double tol, int restart, int maxit, double *mu, double *u,
                               mhk_solve_info *info)
{
    return solve_common(plan, nys, 0, g, f_vol, f_trg, tol, restart, maxit, mu, u, info);
}

mhk_status mhk_solve_neumann(mhk_plan *plan, mhk_nystrom *nys, const double *g, const double *f_vol,
                             const double *f_trg, double tol, int restart, int maxit, double *u_b, double *u,
                             mhk_solve_info *info)
{
    return solve_common(plan, nys, 1, g, f_vol, f_trg, tol, restart, maxit, u_b, u, info);
}

mhk_status mhk_heat_step(mhk_plan *P, mhk_nystrom *N, const double *u_n, const double *F, const double *g_next,
                         double tol, int restart, int maxit, double *u_next, double *mu, mhk_solve_info *info)
{
    if (!P || !N || !u_n || !u_next || u_n == u_next) {
        set_error("null plan, Nystrom matrix or state, or u_n aliases u_next");
        return MHK_EINVAL;
    }
    if (!P->targets_are_volume) {
        set_error("the heat step needs a plan whose targets are its volume nodes, in the same order");
        return MHK_EINVAL;
    }
    BIE_TRY(check_solve(P, N, g_next, u_n, u_n, tol, restart, maxit, mu, u_next));
    const int64_t nout = P->nout;
    BIE_TRY(nys_scratch(N, nout));
    // f at the outputs (volume nodes, then boundary nodes) in the first
    // scratch half, which the Dirichlet solve leaves untouched; its first N_V
    // entries are f at the volume nodes
    double *f = N->work;
    hipLaunchKernelGGL(k_heat_source, dim3(nb_of(nout)), dim3(BT), 0, P->stream, nout, P->p.alpha * P->p.alpha,
                       u_n, F, f);
    BIE_HIP(hipGetLastError());
    return solve_common(P, N, 0, g_next, f, f, tol, restart, maxit, mu, u_next, info);
}

void mhk_nystrom_destroy(mhk_nystrom *N)
{
    if (!N) return;
    (void)hipStreamSynchronize(N->stream);
    nys_free_ws(N);
    for (double **p : {&N->S, &N->geo, &N->na_part, &N->work}) nys_free(N, p);
    for (NysPart &p : N->prod) {
        nys_free(N, &p.cp);
        nys_free(N, &p.rp);
    }
    if (N->item) (void)hipFreeAsync(N->item, N->stream);
    if (N->item_ofs) (void)hipFreeAsync(N->item_ofs, N->stream);
    (void)hipStreamSynchronize(N->stream);
    delete N;
}

}  // extern "C"
