// Dyadic difference-kernel levels (Section 4.2, eqs. (sld), (dld)).
//
// Level j sums, for every target x,
//   S_j(x) = sum_q w_q sigma_q K_j^S(|x - x_q|),
//   D_j(x) = sum_q w_q mu_q nu_q.(x - x_q) K_j^D(|x - x_q|),
// over the child nodes q of the panels bisected up to j times.  The kernels come
// from one piecewise-polynomial table of K_j^S in a = r^2/(4 delta_j) held in
// LDS: Horner's rule gives the polynomial and its derivative together, and
// K_j^D is a constant times dK_j^S/da, applied once per target at the end
// (the table reads serve both kernels).  Pairs with a >= a_max are below
// the requested accuracy and skipped (a lane beyond it reads the table's
// zero segment).  Target and source coordinates are scaled by sqrt(seg_inv / (4 delta_j)),
// so that the squared separation is the segment coordinate a seg_inv itself;
// the double-layer sum is rescaled once per target.
//
// Work decomposition: a wavefront owns 64 consecutive targets of the Morton
// order, one per lane, and one piece of the flat list (built at plan time) of
// the sources within R_j of its targets' bounding box.  It reads the list 64
// sources at a time with vector loads (lane l holds source l) -- the next
// batch is loaded while the current one is summed -- and hands each source to
// all lanes with readlane; each lane keeps its target's sums in registers: no
// atomics, no barriers in the loop, deterministic summation order (the local
// part adds the pieces in order).  The lists are cut because a whole one is a
// serial chain: a few thousand wavefronts (or 72, for 4608 targets) with lists
// of up to several thousand sources left the chip idle behind the longest
// ones.  All levels go in one launch.  Measured with whole lists and a launch
// per level against pieces of 128 to 1024 sources: 618 against 111 us at 4608
// targets and 512 boundary nodes, 1895 against 930 us at 466 thousand targets
// and 65536 boundary nodes (beside the history part).  Sources
// are taken two at a time with no branch per lane, and a pair of sources out
// of range of every lane is skipped as a whole.  The two polynomial
// evaluations are independent, so their table reads and multiply-adds
// interleave.  The kernel table sits in LDS (shared by the wavefronts of a
// workgroup) in rows of 48 bytes, an odd multiple of 16, read as aligned
// 16-byte loads, so that neighbouring segments fall in different bank
// groups.
//
// Precision: T = double (FP64 path) or float (FP32 path).  In the FP32 path
// the separation x - x_q is formed in FP64 from FP64 positions and rounded
// once, so that its relative error is that of one rounding even when the
// separation is far smaller than the coordinates; the table (degree 7), the
// kernel evaluation and the accumulation are FP32.  The FP64 path keeps its
// table's three highest coefficients, each below 4e-8 of K_j(0), as floats
// and starts Horner's rule over them in FP32 (52 bytes of table per pair
// instead of 64); the rest is FP64.
#include <type_traits>

#include "mhk_internal.h"

namespace mhk {

// Child-node strengths of every level for the current densities: q_S = w
// sigma, q_Dx = w nu_x mu, q_Dy = w nu_y mu, with sigma, mu at the child node
// interpolated from the parent panel's 16 nodal values.  One launch for all
// levels (workgroup ranges qblk0).  Layout [3][B][n_src], or for the sums on the
// matrix cores (bp > 0) [3][n_src][bp], the densities of a node side by side and
// zeros up to bp.
template <typename T>
__global__ void __launch_bounds__(256) k_level_q(const LevelDesc *__restrict__ desc, int J, int B, int bp, int64_t nb,
                                                 const T *__restrict__ sigma, const T *__restrict__ mu)
{
    int j = 0;
    while (j + 1 < J && (int)blockIdx.x >= desc[j + 1].qblk0) ++j;
    const LevelDesc &L = desc[j];
    const int64_t n_src = L.n_src;
    int64_t s = (int64_t)((int)blockIdx.x - L.qblk0) * blockDim.x + threadIdx.x;
    if (s >= n_src) return;
    T *q = (T *)L.q;
    int c = L.code[s];
    int k = c % NGL;
    int pc = c / NGL;
    int child = pc % L.nchild;
    int64_t panel = pc / L.nchild;
    const double *row = L.interp + ((size_t)child * NGL + k) * NGL;
    double r[NGL];
#pragma unroll
    for (int i = 0; i < NGL; ++i) r[i] = row[i];
    const double w = L.sw[s], wx = L.swx[s], wy = L.swy[s];
    const size_t cs = (size_t)(bp > 0 ? bp : B) * n_src, bs = bp > 0 ? 1 : n_src;
    q += bp > 0 ? (size_t)s * bp : (size_t)s;
    for (int b = 0; b < B; ++b) {
        if (sigma) {
            const T *f = sigma + (size_t)b * nb + panel * NGL;
            double v = 0;
#pragma unroll
            for (int i = 0; i < NGL; ++i) v = fma(r[i], (double)f[i], v);
            q[b * bs] = (T)(w * v);
        }
        if (mu) {
            const T *f = mu + (size_t)b * nb + panel * NGL;
            double v = 0;
#pragma unroll
            for (int i = 0; i < NGL; ++i) v = fma(r[i], (double)f[i], v);
            q[cs + b * bs] = (T)(wx * v);
            q[2 * cs + b * bs] = (T)(wy * v);
        }
    }
    for (int b = B; b < bp; ++b) {
        if (sigma) q[b] = (T)0;
        if (mu) q[cs + b] = q[2 * cs + b] = (T)0;
    }
}

struct LevelArgs {
    const LevelDesc *desc;
    int lev0, nlev;       // levels [lev0, lev0 + nlev) of the launch
    int64_t nout;
    const double *tx, *ty;
    int B, ncomp;         // densities; components of an item's part (2: S and D, 1: S)
    int want_s, want_d;
    int *counter;         // persistent launch: next work item, zero at the launch
};

// Value of lane k (wave-uniform k) for the whole wave.
__device__ inline double bcast(double v, int k)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), k);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
    return __hiloint2double(hi, lo);
}
__device__ inline float bcast(float v, int k)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// x - floor(x) for x >= 0 (exact), one instruction
__device__ inline double frac_part(double x) { return __builtin_amdgcn_fract(x); }
__device__ inline float frac_part(float x) { return __builtin_amdgcn_fractf(x); }

// One batch of up to 64 sources held one per lane: positions and strengths.
template <typename T, int BCH>
struct SrcBatch {
    double x, y;
    T qs[BCH], qx[BCH], qy[BCH];
};

// Source k of a batch against the lane's target: separation, table segment
// (the zero segment out of range), local variable.
template <typename T>
struct PairGeo {
    T dx, dy, v;
    const T *c;          // the segment's row
    const float *c7;     // FP64 table: the segment's c_7
};

template <typename T, int STRIDE>
__device__ inline PairGeo<T> pair_geo(double x, double y, double sxv, double syv, T f_max, T f_zero,
                                      const T *s_tab, const float *s_c7, bool &in)
{
    PairGeo<T> g;
    g.dx = (T)(x - sxv);
    g.dy = (T)(y - syv);
    // coordinates are scaled so that |dx|^2 is the segment coordinate
    // f = a seg_inv; a pair beyond the cut-off reads the zero segment f_zero
    // (at v = -1), which adds exactly nothing
    const T f = g.dx * g.dx + g.dy * g.dy;
    in = f < f_max;
    const T fc = in ? f : f_zero;
    const int sg = (int)fc;
    g.v = (T)2 * frac_part(fc) - (T)1;
    g.c = s_tab + __umul24((unsigned)sg, (unsigned)STRIDE);
    if constexpr (std::is_same<T, double>::value) g.c7 = s_c7 + sg;
    return g;
}

// p(v) and p'(v) of a table segment by Horner's rule for two sources at
// once (K_j^S and, up to the factor d_scale, K_j^D); the derivative's first
// step is c_7.  FP32 table: eight floats, read as two 16-byte LDS loads.
struct Row32 {
    float c[TABF_NC];
};
__device__ inline Row32 load_row(const PairGeo<float> &g)
{
    const float4 *r = reinterpret_cast<const float4 *>(g.c);
    const float4 a = r[0], b = r[1];
    return Row32{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ inline void horner2(const PairGeo<float> &g0, const PairGeo<float> &g1, float &ks0, float &kd0,
                               float &ks1, float &kd1)
{
    const Row32 w0 = load_row(g0), w1 = load_row(g1);
    kd0 = w0.c[TABF_NC - 1];
    kd1 = w1.c[TABF_NC - 1];
    ks0 = fmaf(kd0, g0.v, w0.c[TABF_NC - 2]);
    ks1 = fmaf(kd1, g1.v, w1.c[TABF_NC - 2]);
#pragma unroll
    for (int m = TABF_NC - 3; m >= 0; --m) {
        kd0 = fmaf(kd0, g0.v, ks0);
        kd1 = fmaf(kd1, g1.v, ks1);
        ks0 = fmaf(ks0, g0.v, w0.c[m]);
        ks1 = fmaf(ks1, g1.v, w1.c[m]);
    }
}

// FP64 table row (48 bytes, 16-byte aligned): c_0..c_4 as doubles and c_5,
// c_6 as two floats, read as three 16-byte LDS loads; c_7 (float) from the
// array after the rows.  The high part goes through Horner's rule in FP32
// and the result continues in FP64 (the same order as the plan's accuracy
// check of the table).
struct Row64 {
    double c[TAB_NC64];
    float c5, c6, c7;
};
__device__ inline Row64 load_row(const PairGeo<double> &g)
{
    const double2 *r = reinterpret_cast<const double2 *>(g.c);
    const double2 a = r[0], b = r[1], h = r[2];
    Row64 w;
    w.c[0] = a.x;
    w.c[1] = a.y;
    w.c[2] = b.x;
    w.c[3] = b.y;
    w.c[4] = h.x;
    w.c5 = __int_as_float(__double2loint(h.y));
    w.c6 = __int_as_float(__double2hiint(h.y));
    w.c7 = *g.c7;
    return w;
}
__device__ inline void horner_hi(const Row64 &w, double v, float &ks, float &kd)
{
    const float vf = (float)v;
    kd = w.c7;
    ks = fmaf(kd, vf, w.c6);
    kd = fmaf(kd, vf, ks);
    ks = fmaf(ks, vf, w.c5);
}
__device__ inline void horner2(const PairGeo<double> &g0, const PairGeo<double> &g1, double &ks0, double &kd0,
                               double &ks1, double &kd1)
{
    const Row64 w0 = load_row(g0), w1 = load_row(g1);
    float hs0, hd0, hs1, hd1;
    horner_hi(w0, g0.v, hs0, hd0);
    horner_hi(w1, g1.v, hs1, hd1);
    ks0 = hs0;
    kd0 = hd0;
    ks1 = hs1;
    kd1 = hd1;
#pragma unroll
    for (int m = TAB_NC64 - 1; m >= 0; --m) {
        kd0 = fma(kd0, g0.v, ks0);
        kd1 = fma(kd1, g1.v, ks1);
        ks0 = fma(ks0, g0.v, w0.c[m]);
        ks1 = fma(ks1, g1.v, w1.c[m]);
    }
}
__device__ inline void horner1(const PairGeo<float> &g, float &ks, float &kd)
{
    const Row32 w = load_row(g);
    kd = w.c[TABF_NC - 1];
    ks = fmaf(kd, g.v, w.c[TABF_NC - 2]);
#pragma unroll
    for (int m = TABF_NC - 3; m >= 0; --m) {
        kd = fmaf(kd, g.v, ks);
        ks = fmaf(ks, g.v, w.c[m]);
    }
}
__device__ inline void horner1(const PairGeo<double> &g, double &ks, double &kd)
{
    const Row64 w = load_row(g);
    float hs, hd;
    horner_hi(w, g.v, hs, hd);
    ks = hs;
    kd = hd;
#pragma unroll
    for (int m = TAB_NC64 - 1; m >= 0; --m) {
        kd = fma(kd, g.v, ks);
        ks = fma(ks, g.v, w.c[m]);
    }
}

// One work item: the LV_WAVE targets of a wavefront against one piece of its
// candidate list, for the densities of chunk `chunk` (BCH of them).
template <int BCH, typename T, int STRIDE>
__device__ inline void level_item(const LevelArgs &A, const LevelDesc &L, const T *s_tab, const float *s_c7, int lane,
                                  int item, int chunk)
{
    const int wave = __builtin_amdgcn_readfirstlane(L.item_wave[item]);
    const int64_t t = (int64_t)wave * LV_WAVE + lane;
    const double ps = L.pscale;
    double x = 0.0, y = 0.0;
    if (t < A.nout) {
        x = A.tx[t] * ps;
        y = A.ty[t] * ps;
    }
    const int b0 = chunk * BCH, nbh = min(BCH, A.B - b0);
    const T f_max = (T)L.f_max, f_zero = (T)L.nseg;
    const double *__restrict__ sx = L.sx, *__restrict__ sy = L.sy;
    const int32_t *__restrict__ wave_src = L.wave_src;
    T S[BCH], D[BCH];
    // FP32 path: the sums of each batch of 64 sources are added into FP64
    // totals (a volume level sums thousands of nodes per target, where one
    // running FP32 sum would lose about sqrt(N) roundings)
    double S64[BCH], D64[BCH];
#pragma unroll
    for (int b = 0; b < BCH; ++b) S[b] = D[b] = (T)0, S64[b] = D64[b] = 0.0;
    // strengths of density b0 + b: q[c][b0 + b][s] for c = S, D_x, D_y
    const size_t n_src = (size_t)L.n_src, fstride = (size_t)A.B * n_src;
    const T *__restrict__ q0 = (const T *)L.q + (size_t)b0 * n_src;
    // lane l of a batch holds source l of the list; lanes past its end hold a
    // far-away source of zero strength
    auto load = [&](int pos, int end, SrcBatch<T, BCH> &sb) {
        if (pos < end) {
            const int s = wave_src[pos];
            sb.x = sx[s] * ps;
            sb.y = sy[s] * ps;
#pragma unroll
            for (int b = 0; b < BCH; ++b) {
                const T *qb = q0 + (size_t)min(b, nbh - 1) * n_src + s;
                sb.qs[b] = A.want_s ? qb[0] : (T)0;
                sb.qx[b] = A.want_d ? qb[fstride] : (T)0;
                sb.qy[b] = A.want_d ? qb[2 * fstride] : (T)0;
            }
        } else {
            sb.x = sb.y = 1e30;
#pragma unroll
            for (int b = 0; b < BCH; ++b) sb.qs[b] = sb.qx[b] = sb.qy[b] = (T)0;
        }
    };
    auto accumulate = [&](const SrcBatch<T, BCH> &sb, int k, const PairGeo<T> &g, T ks, T kd) {
#pragma unroll
        for (int b = 0; b < BCH; ++b) {
            const T qsv = bcast(sb.qs[b], k), qxv = bcast(sb.qx[b], k), qyv = bcast(sb.qy[b], k);
            S[b] = fma(qsv, ks, S[b]);
            D[b] = fma(fma(qxv, g.dx, qyv * g.dy), kd, D[b]);
        }
    };
    // the item's piece of the list
    const int l0 = L.wave_ofs[wave], l1 = L.wave_ofs[wave + 1];
    const int i0 = L.item_ofs[wave], i1 = L.item_ofs[wave + 1];
    const int size = level_piece(l1 - l0, i1 - i0);
    const int c0 = __builtin_amdgcn_readfirstlane(l0 + (item - i0) * size);
    const int c1 = __builtin_amdgcn_readfirstlane(min(l1, c0 + size));
    SrcBatch<T, BCH> cur, nxt;
    load(c0 + lane, c1, cur);
    for (int base = c0; base < c1; base += LV_WAVE) {
        load(base + LV_WAVE + lane, c1, nxt);            // next batch in flight while this one is summed
        const int cnt = __builtin_amdgcn_readfirstlane(min(LV_WAVE, c1 - base));
        if (BCH == 1) {
            for (int k = 0; k < cnt; k += 2) {
                // sources k and k + 1 (past the batch's end: a lane holding
                // the far-away source of zero strength)
                bool in0, in1;
                const PairGeo<T> g0 = pair_geo<T, STRIDE>(x, y, bcast(cur.x, k), bcast(cur.y, k), f_max, f_zero,
                                                          s_tab, s_c7, in0);
                const PairGeo<T> g1 = pair_geo<T, STRIDE>(x, y, bcast(cur.x, k + 1), bcast(cur.y, k + 1), f_max,
                                                          f_zero, s_tab, s_c7, in1);
                if (__ballot(in0 || in1) == 0) continue;
                T ks0, kd0, ks1, kd1;
                horner2(g0, g1, ks0, kd0, ks1, kd1);
                accumulate(cur, k, g0, ks0, kd0);
                accumulate(cur, k + 1, g1, ks1, kd1);
            }
        } else {
            // several densities: the strengths of one source already fill
            // the registers, so one source at a time
            for (int k = 0; k < cnt; ++k) {
                bool in0;
                const PairGeo<T> g0 = pair_geo<T, STRIDE>(x, y, bcast(cur.x, k), bcast(cur.y, k), f_max, f_zero,
                                                          s_tab, s_c7, in0);
                if (__ballot(in0) == 0) continue;
                T ks0, kd0;
                horner1(g0, ks0, kd0);
                accumulate(cur, k, g0, ks0, kd0);
            }
        }
        if constexpr (std::is_same<T, float>::value) {
#pragma unroll
            for (int b = 0; b < BCH; ++b) {
                S64[b] += (double)S[b];
                D64[b] += (double)D[b];
                S[b] = D[b] = 0.0f;
            }
        }
        cur = nxt;
    }
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
        for (int b = 0; b < BCH; ++b) {
            S[b] = (float)S64[b];
            D[b] = (float)(D64[b] * L.d_scale);
        }
    } else {
#pragma unroll
        for (int b = 0; b < BCH; ++b) D[b] *= L.d_scale;
    }
    T *part = (T *)L.part + (size_t)item * A.ncomp * A.B * LV_WAVE + lane;
#pragma unroll
    for (int b = 0; b < BCH; ++b) {
        if (b < nbh) {
            if (A.want_s) part[(size_t)(b0 + b) * LV_WAVE] = S[b];
            if (A.want_d) part[(size_t)(A.B + b0 + b) * LV_WAVE] = D[b];
        }
    }
}

// The level's kernel table is loaded into LDS once per workgroup.  PERSIST =
// false: one launch over all levels, one work item per wavefront (the level
// and the item from the launch position, density chunk from blockIdx.y), the
// long items of a level first.  PERSIST = true: one launch per level, a grid
// sized to fill the device once; every wavefront takes work items (item-major:
// the density chunks of one item follow each other, so its candidates stay in
// cache) from a counter in device memory, zeroed before the launch, until
// none is left -- the exit every wavefront reaches.
template <int BCH, typename T, int STRIDE, int NB, bool PERSIST>
__global__ void __launch_bounds__(NB) k_level_sums(LevelArgs A)
{
    extern __shared__ double lds[];
    int j = A.lev0;
    if (!PERSIST)
        while (j + 1 < A.lev0 + A.nlev && (int)blockIdx.x >= A.desc[j + 1].blk0) ++j;
    const LevelDesc &L = A.desc[j];
    T *s_tab = reinterpret_cast<T *>(lds);                // [nseg + 1][STRIDE], the last segment zero
    const int tid = threadIdx.x, nseg = L.nseg;
    const T *__restrict__ tab = (const T *)L.tab;
    for (int i = tid; i < (nseg + 1) * STRIDE; i += NB) s_tab[i] = i < nseg * STRIDE ? tab[i] : (T)0;
    // FP64 table: c_7 of every segment (the zero segment's last) after the rows
    float *s_c7 = nullptr;
    if constexpr (std::is_same<T, double>::value) {
        s_c7 = reinterpret_cast<float *>(s_tab + (nseg + 1) * STRIDE);
        const float *g7 = reinterpret_cast<const float *>(tab + (size_t)nseg * STRIDE);
        for (int i = tid; i <= nseg; i += NB) s_c7[i] = i < nseg ? g7[i] : 0.0f;
    }
    __syncthreads();
    const int lane = tid % LV_WAVE;
    if (!PERSIST) {
        // the item number is wave-uniform
        const int64_t pos = (int64_t)((int)blockIdx.x - L.blk0) * (NB / LV_WAVE) + tid / LV_WAVE;
        if (pos >= L.n_items) return;
        const int item = __builtin_amdgcn_readfirstlane(L.item_order[pos]);
        level_item<BCH, T, STRIDE>(A, L, s_tab, s_c7, lane, item, blockIdx.y);
        return;
    }
    const int nchunk = (A.B + BCH - 1) / BCH;
    const int64_t nitems = L.n_items * nchunk;
    for (;;) {
        int pos = 0;
        if (lane == 0) pos = atomicAdd(A.counter, 1);
        pos = __builtin_amdgcn_readfirstlane(__shfl(pos, 0));
        if (pos >= nitems) break;
        const int item = __builtin_amdgcn_readfirstlane(L.item_order[pos / nchunk]);
        level_item<BCH, T, STRIDE>(A, L, s_tab, s_c7, lane, item, pos % nchunk);
    }
}

// The same sums for LV_MM_MIN or more densities, 16 of them per pass, as
// products on the matrix cores: one kernel value per lane for 16 targets (lane %
// 16) and 4 sources (lane / 16) is the 16 x 4 operand of v_mfma_f64_16x16x4, the
// four sources' strengths the 4 x 16 one (D as K dx times q_Dx plus K dy times
// q_Dy), and the sums of 16 targets by 16 densities the result (rows 4 v + lane /
// 16, column lane % 16).  A table evaluation serves 16 densities instead of lv_bch,
// no source is handed from lane to lane, and out-of-range pairs are skipped 16
// targets by 4 sources at a time.  Per 64 pairs 192 cycles of the matrix cores
// beside about 150 of the VALU, whatever the number of densities up to 16: whole
// evaluations of S and D at 200 thousand targets, 16384 boundary nodes, with 16
// densities 4.69 -> 3.64 ms, 8 2.42 -> 2.15, 5 1.87 -> 1.64; four take one table
// evaluation of k_level_sums anyway (1.25 ms).  16 densities at 1.03M outputs,
// 32768 boundary and 1M volume nodes: 11.8 -> 7.9 ms.
// FP32: 8 densities at 366 thousand outputs, 65536 boundary nodes 1.87 -> 1.78 ms;
// at 200 thousand targets, 16384 boundary nodes 8 as before (1.02 against 1.01 ms),
// 5 723 -> 712 us.
// FP32 plans form the kernel values in FP32, as above, and their products and sums
// in FP64 (the FP32 matrix instructions would need their sums moved to FP64 every
// 64 sources).
typedef double d4 __attribute__((ext_vector_type(4)));
template <typename T, int STRIDE>
__global__ void __launch_bounds__(256, 3) k_level_mm(LevelArgs A, int bp)
{
    extern __shared__ double lds[];
    int j = 0;
    while (j + 1 < A.nlev && (int)blockIdx.x >= A.desc[j + 1].mblk0) ++j;
    const LevelDesc &L = A.desc[j];
    const int tid = threadIdx.x, nseg = L.nseg;
    T *s_tab = reinterpret_cast<T *>(lds);
    const T *__restrict__ tab = (const T *)L.tab;
    for (int i = tid; i < (nseg + 1) * STRIDE; i += 256) s_tab[i] = i < nseg * STRIDE ? tab[i] : (T)0;
    float *s_c7 = nullptr;
    if constexpr (std::is_same<T, double>::value) {
        s_c7 = reinterpret_cast<float *>(s_tab + (nseg + 1) * STRIDE);
        const float *g7 = reinterpret_cast<const float *>(tab + (size_t)nseg * STRIDE);
        for (int i = tid; i <= nseg; i += 256) s_c7[i] = i < nseg ? g7[i] : 0.0f;
    }
    __syncthreads();
    const int64_t pos = (int64_t)((int)blockIdx.x - L.mblk0) * (256 / LV_WAVE) + tid / LV_WAVE;
    if (pos >= L.n_items) return;
    const int lane = tid % LV_WAVE, r = lane % 16, k = lane / 16;
    const int item = __builtin_amdgcn_readfirstlane(L.item_order[pos]);
    const int wave = __builtin_amdgcn_readfirstlane(L.item_wave[item]);
    const double ps = L.pscale;
    const T f_max = (T)L.f_max, f_zero = (T)nseg;
    double tx[4], ty[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int64_t t = (int64_t)wave * LV_WAVE + 16 * g + r;
        tx[g] = t < A.nout ? A.tx[t] * ps : 0.0;
        ty[g] = t < A.nout ? A.ty[t] * ps : 0.0;
    }
    // the item's piece of the list
    const int l0 = L.wave_ofs[wave], l1 = L.wave_ofs[wave + 1];
    const int i0 = L.item_ofs[wave], i1 = L.item_ofs[wave + 1];
    const int size = level_piece(l1 - l0, i1 - i0);
    const int c0 = __builtin_amdgcn_readfirstlane(l0 + (item - i0) * size);
    const int c1 = __builtin_amdgcn_readfirstlane(min(l1, c0 + size));
    const double *__restrict__ sx = L.sx, *__restrict__ sy = L.sy;
    const int32_t *__restrict__ wave_src = L.wave_src;
    const int b0 = (int)blockIdx.y * 16;
    const size_t cs = (size_t)bp * L.n_src;
    const T *__restrict__ q0 = (const T *)L.q + b0 + r;
    // lane's source k of four (past the list's end a far one of zero strength),
    // its strengths for density r; loaded one step ahead, the list entry two
    struct Src {
        double x, y, qs, qx, qy;
    };
    constexpr double far = 1e15;
    auto load = [&](int p, int id) {
        Src v{far, far, 0.0, 0.0, 0.0};
        if (p < c1) {
            v.x = sx[id] * ps;
            v.y = sy[id] * ps;
            const T *q = q0 + (size_t)id * bp;
            if (A.want_s) v.qs = q[0];
            if (A.want_d) {
                v.qx = q[cs];
                v.qy = q[2 * cs];
            }
        }
        return v;
    };
    d4 S[4], D[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) S[g] = D[g] = d4{0.0, 0.0, 0.0, 0.0};
    auto entry = [&](int p) { return p < c1 ? wave_src[p] : 0; };
    Src cur = load(c0 + k, entry(c0 + k));
    int id = entry(c0 + 4 + k);
    for (int p = c0; p < c1; p += 4) {
        const int id2 = entry(p + 8 + k);
        const Src nxt = load(p + 4 + k, id);
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
            bool in0, in1;
            const PairGeo<T> g0 = pair_geo<T, STRIDE>(tx[g], ty[g], cur.x, cur.y, f_max, f_zero, s_tab, s_c7, in0);
            const PairGeo<T> g1 =
                pair_geo<T, STRIDE>(tx[g + 1], ty[g + 1], cur.x, cur.y, f_max, f_zero, s_tab, s_c7, in1);
            if (!__any(in0 || in1)) continue;
            T s0, d0, s1, d1;
            horner2(g0, g1, s0, d0, s1, d1);
            const double ks0 = s0, kd0 = d0, ks1 = s1, kd1 = d1;
            if (A.want_s) {
                S[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(ks0, cur.qs, S[g], 0, 0, 0);
                S[g + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ks1, cur.qs, S[g + 1], 0, 0, 0);
            }
            if (A.want_d) {
                D[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(kd0 * g0.dx, cur.qx, D[g], 0, 0, 0);
                D[g + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(kd1 * g1.dx, cur.qx, D[g + 1], 0, 0, 0);
                D[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(kd0 * g0.dy, cur.qy, D[g], 0, 0, 0);
                D[g + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(kd1 * g1.dy, cur.qy, D[g + 1], 0, 0, 0);
            }
        }
        cur = nxt;
        id = id2;
    }
    if (b0 + r >= A.B) return;
    T *part = (T *)L.part + ((size_t)item * A.ncomp * A.B + b0 + r) * LV_WAVE + k;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (A.want_s) part[16 * g + 4 * v] = (T)S[g][v];
            if (A.want_d) part[(size_t)A.B * LV_WAVE + 16 * g + 4 * v] = (T)(D[g][v] * L.d_scale);
        }
}

// LDS bytes of a level's table: the rows of nseg + 1 segments (the last zero)
// and, FP64, their c_7 as floats
template <typename T, int STRIDE>
static size_t level_lds(int nseg)
{
    size_t b = sizeof(T) * (size_t)(nseg + 1) * STRIDE;
    if (std::is_same<T, double>::value) b += sizeof(float) * (size_t)(nseg + 2);
    return b;
}

template <typename T>
static hipError_t level_q(mhk_plan *P, hipStream_t st, const void *sigma, const void *mu)
{
    if (P->levq_grid == 0) return hipSuccess;
    hipLaunchKernelGGL(k_level_q<T>, dim3(P->levq_grid), dim3(256), 0, st, P->lev_desc, P->J, P->bat,
                       level_mm(P, P->bat) ? level_bp(P->bat) : 0, P->nb,
                       (const T *)sigma, (const T *)mu);
    return hipGetLastError();
}

hipError_t launch_level_densities(mhk_plan *P, hipStream_t st, const void *sigma, const void *mu)
{
    return P->p.prec == MHK_FP64 ? level_q<double>(P, st, sigma, mu) : level_q<float>(P, st, sigma, mu);
}

mhk_status level_descs(mhk_plan *P, bool vol, std::vector<LevelDesc> &out)
{
    out.assign((size_t)P->J, LevelDesc{});
    const bool f64 = P->p.prec == MHK_FP64;
    const int per = P->p.lv_block / LV_WAVE;
    int64_t blk = 0, qblk = 0, mblk = 0;
    for (int j = 0; j < P->J; ++j) {
        const Level &L = P->lev[j];
        LevelDesc &d = out[(size_t)j];
        const LevelItems &I = vol ? P->vlev[j].items : L.items;
        d.wave_ofs = vol ? P->vlev[j].wave_ofs : L.wave_ofs;
        d.wave_src = vol ? P->vlev[j].wave_src : L.wave_src;
        d.item_ofs = I.ofs;
        d.item_wave = I.wave;
        d.item_order = I.order;
        d.part = I.part;
        d.n_items = I.n;
        d.sx = vol ? P->vlev[j].sx : L.sx;
        d.sy = vol ? P->vlev[j].sy : L.sy;
        d.q = vol ? P->vlev[j].q : L.q;
        d.n_src = vol ? P->vlev[j].n_src : L.n_src;
        d.tab = L.tab_dev;
        d.nseg = L.nseg;
        d.nchild = L.nchild;
        d.code = L.code;
        d.interp = L.interp;
        d.sw = L.sw;
        d.swx = L.swx;
        d.swy = L.swy;
        d.pscale = sqrt(L.inv4d * L.seg_inv);
        d.d_scale = level_d_scale(L) / d.pscale;       // D is summed over scaled separations
        d.f_max = L.a_max * L.seg_inv;
        d.blk0 = (int)blk;
        d.qblk0 = (int)qblk;
        d.mblk0 = (int)mblk;
        blk += (I.n + per - 1) / per;
        mblk += (I.n + 256 / LV_WAVE - 1) / (256 / LV_WAVE);
        qblk += (d.n_src + 255) / 256;
        const size_t lds = f64 ? level_lds<double, TAB_STRIDE>(L.nseg) : level_lds<float, TABF_STRIDE>(L.nseg);
        P->lev_lds = std::max(P->lev_lds, lds);
    }
    if (P->lev_lds > 160 * 1024 || mblk > INT32_MAX || qblk > INT32_MAX) {
        set_error("level tables or work-item lists too large");
        return MHK_EUNSUPPORTED;
    }
    if (vol) {
        P->vlev_grid = (unsigned)blk;
    } else {
        P->lev_grid = (unsigned)blk;
        P->levm_grid = (unsigned)mblk;
        P->levq_grid = (unsigned)qblk;
    }
    return MHK_OK;
}

template <int BCH, typename T, int STRIDE, int NB>
static hipError_t level_launch(mhk_plan *P, LevelArgs A, bool vol, hipStream_t st)
{
    const size_t lds = P->lev_lds;
    const unsigned nby = (unsigned)((A.B + BCH - 1) / BCH);
    if (!P->p.lv_persist) {
        const void *fn = (const void *)k_level_sums<BCH, T, STRIDE, NB, false>;
        if (lds > 64 * 1024) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        const unsigned grid = vol ? P->vlev_grid : P->lev_grid;
        if (grid == 0) return hipSuccess;
        A.lev0 = 0;
        A.nlev = P->J;
        hipLaunchKernelGGL((k_level_sums<BCH, T, STRIDE, NB, false>), dim3(grid, nby), dim3(NB), lds, st, A);
        return hipGetLastError();
    }
    const void *fn = (const void *)k_level_sums<BCH, T, STRIDE, NB, true>;
    if (lds > 64 * 1024) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    // as many workgroups as are resident at once, at most one per item
    int per_cu = 0, dev = 0, ncu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NB, lds) != hipSuccess || per_cu < 1) per_cu = 1;
    for (int j = 0; j < P->J; ++j) {
        const int64_t items = (vol ? P->vlev[j].items.n : P->lev[j].items.n) * nby;
        if (items == 0) continue;
        const int64_t wg = std::min<int64_t>((int64_t)per_cu * std::max(ncu, 1), (items + NB / LV_WAVE - 1) / (NB / LV_WAVE));
        hipError_t e = launch_fill_int(P->lv_counter, 1, st);
        if (e != hipSuccess) return e;
        A.lev0 = j;
        A.nlev = 1;
        hipLaunchKernelGGL((k_level_sums<BCH, T, STRIDE, NB, true>), dim3((unsigned)wg), dim3(NB), lds, st, A);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int BCH, typename T, int STRIDE>
static hipError_t level_launch_nb(mhk_plan *P, const LevelArgs &A, bool vol, hipStream_t st)
{
    return P->p.lv_block == 512 ? level_launch<BCH, T, STRIDE, 512>(P, A, vol, st)
                                : level_launch<BCH, T, STRIDE, 256>(P, A, vol, st);
}

// vol: the volume potential's levels -- the same kernel tables, the volume
// level nodes as sources (single-layer sums only)
template <typename T, int STRIDE>
static hipError_t level_sums(mhk_plan *P, hipStream_t st, bool vol, bool want_s, bool want_d)
{
    LevelArgs A{};
    A.desc = vol ? P->vlev_desc : P->lev_desc;
    A.nout = P->nout;
    A.tx = P->tx;
    A.ty = P->ty;
    A.B = P->bat;
    A.ncomp = vol ? 1 : 2;
    A.want_s = want_s;
    A.want_d = want_d;
    A.counter = P->lv_counter;
    if (!vol && level_mm(P, A.B)) {
        if (P->levm_grid == 0) return hipSuccess;
        A.nlev = P->J;
        const void *fn = (const void *)k_level_mm<T, STRIDE>;
        if (P->lev_lds > 64 * 1024)
            (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)P->lev_lds);
        const int bp = level_bp(A.B);
        hipLaunchKernelGGL((k_level_mm<T, STRIDE>), dim3(P->levm_grid, (unsigned)(bp / 16)), dim3(256), P->lev_lds, st,
                           A, bp);
        return hipGetLastError();
    }
    // densities per pass: the plan's lv_bch, or fewer for a smaller batch
    // (rounded up to an instantiated size; missing densities of the last
    // pass are skipped)
    const int want = std::min(A.B, P->p.lv_bch);
    if (want <= 1) return level_launch_nb<1, T, STRIDE>(P, A, vol, st);
    if (want <= 2) return level_launch_nb<2, T, STRIDE>(P, A, vol, st);
    if (want <= 4) return level_launch_nb<4, T, STRIDE>(P, A, vol, st);
    return level_launch_nb<8, T, STRIDE>(P, A, vol, st);
}

hipError_t launch_level_sums(mhk_plan *P, hipStream_t st, bool vol, bool want_s, bool want_d)
{
    if (P->p.prec == MHK_FP64) return level_sums<double, TAB_STRIDE>(P, st, vol, want_s, want_d);
    return level_sums<float, TABF_STRIDE>(P, st, vol, want_s, want_d);
}

}  // namespace mhk
