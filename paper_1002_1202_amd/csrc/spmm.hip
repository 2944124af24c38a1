// Block-sparse products with H and S for many right-hand sides at once.
//
// One workgroup walks one block row for 64 lanes of columns, its four waves a
// quarter of the stored blocks each, or four rows, one a wave, in launches of many
// short rows (spmm.h, geometry.h); the B x B blocks of S and H are
// wave-uniform (scalar loads), the gathered x rows are 64 contiguous values
// per orbital (one coalesced 1 KiB transaction per orbital row).  No MFMA: per
// stored value the product does 2 (S only) or 4 (S and H) FMAs per complex
// column against >= 16 bytes of vector traffic, far below the FP64 ridge.
#include <algorithm>
#include <cstring>

#include "spmm.h"

namespace gsc {

namespace {

// sums of the four waves of a workgroup, lane by lane, written by wave 0
template <typename P>
__device__ inline void wave_sums_store(P v, P (*red)[64], int w, int lane, P *out, bool write = true) {
    red[w][lane] = v;
    __syncthreads();
    if (w == 0 && write) {
        P s = red[0][lane];
#pragma unroll
        for (int k = 1; k < kWavesPerBlock; ++k) s = s + red[k][lane];
        *out = s;
    }
}

}  // namespace

// q = zs_c * (S p) - H p for every active column c and the per-column
// unconjugated partial dot  sum_i p_i q_i  (the denominator of alpha,
// eq. CGp:r with the S-bilinear form) of this row group.
template <typename T, int B, int SPLIT>
__global__ __launch_bounds__(kBlock) void k_spmm_seed(
    int nb, int Rp, bool ragged, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const T *__restrict__ Sv, const T *__restrict__ Hv, const cpx<T> *__restrict__ p,
    cpx<T> *__restrict__ q, const c128 *__restrict__ z, const int *__restrict__ seed,
    const int *__restrict__ skip, c128 *__restrict__ partial) {
    using V = cpx<T>;
    __shared__ RowSums<V, B, SPLIT> red;
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int col = cx * 64 + lane;
    const size_t ld = Rp;
    const V *pc = p + cx * 64;
    V *qc = q + cx * 64;
    const bool act = !skip[col];
    const c128 zs = act ? z[seed[col]] : c128{0, 0};
    const V zt = ccast<T>(zs);
    c128 dot{0.0, 0.0};
    walk_rows<SPLIT, true, false>(
        act, nb, g, w, lane, rowptr, colidx, Sv, Hv, pc, ld, red, red,
        [&](size_t row) { return (pc + row * ld)[lane]; },
        [&](V(&aS)[B], V(&aH)[B]) {
#pragma unroll
            for (int a = 0; a < B; ++a) aS[a] = zt * aS[a] - aH[a];
        },
        [&](size_t row, V v, V, V own) {
            (qc + row * ld)[lane] = v;
            dot = dot + ccast<double>(own) * ccast<double>(v);
        });
    __shared__ c128 redd[kWavesPerBlock][64];
    wave_sums_store(dot, redd, w, lane, partial + static_cast<size_t>(g) * Rp + col);
}

// The same product for a caller's own X and Y, R columns wide: rows of any
// length, the lanes beyond the last column masked, and the columns' factors in
// the kernel's arguments.  Against padded copies of X and Y around the kernel
// above and factors copied to the device: 64 Si x 8 columns 41.7 -> 22.5 us a call,
// 8,192 Si x 250 307 -> 191 us.  Four waves share a row at every size (one wave a
// row: 102 against 85 us for 8,192 Si x 128); without the dots there is nothing to
// load beside the product.
constexpr int kFactors = 128;
struct Factors { c128 z[kFactors]; };
template <int B>
__global__ __launch_bounds__(kBlock) void k_product(int nb, int R, int ncols, bool ragged,
                                                    const int32_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ colidx,
                                                    const double *__restrict__ Sv, const double *__restrict__ Hv,
                                                    const c128 *__restrict__ X, c128 *__restrict__ Y, int same,
                                                    const c128 *__restrict__ many, Factors f) {
    constexpr int SPLIT = kSplit<double>;
    __shared__ RowSums<c128, B, SPLIT> red;
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int col = cx * 64 + lane;
    const c128 *x = X + cx * 64;
    c128 *y = Y + cx * 64;
    const size_t ld = R;
    const bool act = col < ncols;
    const int at = same || !act ? 0 : col;
    const c128 z = many != nullptr ? many[at] : f.z[at % kFactors];
    struct None {};
    walk_rows<SPLIT, true, false>(
        act, nb, g, w, lane, rowptr, colidx, Sv, Hv, x, ld, red, red, [](size_t) { return None{}; },
        [&](c128(&aS)[B], c128(&aH)[B]) {
#pragma unroll
            for (int a = 0; a < B; ++a) aS[a] = z * aS[a] - aH[a];
        },
        [&](size_t row, c128 v, c128, None) { (y + row * ld)[lane] = v; });
}

void launch_product(hipStream_t st, const Pair &pr, int R, const double *factors, const c128 *X, c128 *Y,
                    c128 *room) {
    const c128 *z = reinterpret_cast<const c128 *>(factors);
    bool same = true;
    for (int c = 1; c < R && same; ++c) same = std::memcmp(z, z + c, sizeof(c128)) == 0;
    const c128 *many = nullptr;
    if (!same && R > kProductFactors) {
        GSC_HIP(hipMemcpyAsync(room, z, R * sizeof(c128), hipMemcpyHostToDevice, st));
        many = room;
    }
    for (int c0 = 0; c0 < R;) {
        const int n = same || many ? R : std::min(R - c0, kFactors);
        Factors f{};
        if (!many) std::memcpy(f.z, z + c0, (same ? 1 : n) * sizeof(c128));
        TileDims td{};
        td.nb = static_cast<int>(pr.nb);
        td.Rp = (n + 63) / 64 * 64;
        set_spmm_geometry(td, pr, false);
        const dim3 grid(td.Rp / 64, td.Gw);
        const bool ragged = ragged_end(td.Rp, n, 64);
#define GSC_PRODUCT(BB)                                                                                           \
    k_product<BB><<<grid, kBlock, 0, st>>>(td.nb, R, n, ragged, pr.rowptr.get(), pr.colidx.get(), pr.S.get(),  \
                                           pr.H.get(), X + c0, Y + c0, same, many, f)
        if (pr.B == 4) GSC_PRODUCT(4);
        else GSC_PRODUCT(6);
#undef GSC_PRODUCT
        GSC_HIP(hipGetLastError());
        c0 += n;
    }
}

// w = S d for the columns whose inner solve is still running, plus the
// per-column partial  Re(d^H S d)  (the CG curvature; S real symmetric).
template <typename T, int B, int SPLIT>
__global__ __launch_bounds__(kBlock) void k_spmm_S(
    int nb, int Rp, bool ragged, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const T *__restrict__ Sv, const cpx<T> *__restrict__ d, cpx<T> *__restrict__ wout,
    const int *__restrict__ skip, double *__restrict__ partial) {
    using V = cpx<T>;
    __shared__ RowSums<V, B, SPLIT> red;
    __shared__ double redd[kWavesPerBlock][64];
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int col = cx * 64 + lane;
    const size_t ld = Rp;
    const V *dc = d + cx * 64;
    V *wc = wout + cx * 64;
    const bool act = !skip[col];
    double dot = 0.0;
    walk_rows<SPLIT, false, false>(
        act, nb, g, w, lane, rowptr, colidx, Sv, Sv, dc, ld, red, red,
        [&](size_t row) { return (dc + row * ld)[lane]; }, NoCombine{},
        [&](size_t row, V v, V, V own) {
            (wc + row * ld)[lane] = v;
            dot += static_cast<double>(own.re) * v.re + static_cast<double>(own.im) * v.im;
        });
    wave_sums_store(dot, redd, w, lane, partial + static_cast<size_t>(g) * Rp + col);
}

// ------------------------------------------------------------------ Chebyshev step
// One step of the Chebyshev iteration for S y = r on the interval
// [theta - delta, theta + delta] fused with the product, in the three-term
// form (see cheb_next): one gathered vector (y_k, or r in the first
// step), r and y_{k-1} streamed, y_{k+1} written over y_{k-1}.  A launch covers
// the columns [col0, col0 + 64 gridDim.x) of the Rp-wide tile.  OUT 1: also a
// partial ||r - S y_k||^2.  OUT 2: the step is a column's last, and
// the partial of y_{k+1}^T r (unconjugated: the next rho of the outer
// iteration, eq. CGp:p) goes to dpart as well, for every column
// (dot_active_only = 0) or only for the columns that take this step.
template <typename T, int B, int SPLIT, int MODE, bool NT, int OUT>
__global__ __launch_bounds__(kBlock) void k_cheb_step(
    int nb, int Rp, int col0, bool ragged, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const T *__restrict__ Sv, const cpx<T> *__restrict__ y, const cpx<T> *__restrict__ r,
    cpx<T> *__restrict__ yio, const int *__restrict__ skip, T inv_theta, T c1, T c2,
    double *__restrict__ partial, c128 *__restrict__ dpart, int dot_active_only) {
    using V = cpx<T>;
    __shared__ RowSums<V, B, SPLIT> red;
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int cb = col0 + cx * 64, col = cb + lane;
    const size_t ld = Rp;
    const bool act = !skip[col];
    double acc2 = 0.0;
    c128 dacc{0.0, 0.0};
    const V *x = (MODE == 0 ? r : y) + cb;
    const V *rb = r + cb;
    V *yb = yio + cb;
    struct Elem { V own, r, yprev; };
    walk_rows<SPLIT, false, false>(
        act, nb, g, w, lane, rowptr, colidx, Sv, Sv, x, ld, red, red,
        [&](size_t row) {
            const size_t e = row * ld + lane;
            Elem v{x[e], {}, {}};
            if constexpr (MODE != 0) v.r = ld_cpx<T, NT>(rb + e);
            if constexpr (MODE == 2) v.yprev = ld_cpx<T, NT>(yb + e);
            return v;
        },
        NoCombine{},
        [&](size_t row, V s, V, Elem v) {
            double res2;
            const V ynew = cheb_next<T, MODE>(v.own, s, v.r, v.yprev, inv_theta, c1, c2, res2);
            st_cpx<T, NT>(ynew, yb + row * ld + lane);
            if constexpr (OUT >= 1) acc2 += res2;
            if constexpr (OUT == 2) dacc = dacc + ccast<double>(ynew) * ccast<double>(v.r);
        });
    if constexpr (OUT >= 1) {
        __shared__ double redd[kWavesPerBlock][64];
        wave_sums_store(acc2, redd, w, lane, partial + static_cast<size_t>(g) * Rp + col);
    }
    if constexpr (OUT == 2) {
        __shared__ c128 redc[kWavesPerBlock][64];
        wave_sums_store(dacc, redc, w, lane, dpart + static_cast<size_t>(g) * Rp + col, act || !dot_active_only);
    }
}

template <typename T>
void launch_cheb_step(hipStream_t st, const Pair &pr, const TileDims &td, int mode, int col0, int ncols,
                      const T *Sv, const cpx<T> *y, const cpx<T> *r, cpx<T> *yio, const int *skip,
                      double inv_theta, double c1, double c2, double *partial, c128 *dpart, int dot_mode) {
    GSC_REQUIRE(col0 % 64 == 0 && ncols % 64 == 0 && ncols > 0 && col0 + ncols <= td.Rp,
                "Chebyshev column block outside the tile");
    GSC_REQUIRE(dot_mode == 0 || (dpart != nullptr && partial != nullptr), "the fused dot needs its partials");
    const int waves = kSplit<T> == 1 ? 1 : step_waves(td.nb, ncols / 64, td.row_orbitals, false);
    dim3 grid(ncols / 64, partial ? td.Gs : waves == 1 ? td.G1 : td.Gw), block(kBlock);
    const bool ragged = ragged_end(col0 + ncols, td.R, 64);
    const T it = static_cast<T>(inv_theta), a = static_cast<T>(c1), b = static_cast<T>(c2);
#define GSC_CHEB_D(BB, SP, M, N, D)                                                                               \
    k_cheb_step<T, BB, SP, M, N, D><<<grid, block, 0, st>>>(td.nb, td.Rp, col0, ragged, pr.rowptr.get(),          \
                                                            pr.colidx.get(), Sv, y, r, yio, skip, it, a, b,       \
                                                            partial, dpart, dot_mode == 2)
#define GSC_CHEB(BB, SP, M, N)                      \
    if (dot_mode) GSC_CHEB_D(BB, SP, M, N, 2);      \
    else if (partial) GSC_CHEB_D(BB, SP, M, N, 1);  \
    else GSC_CHEB_D(BB, SP, M, N, 0);
#define GSC_CHEB_N(BB, SP, M) \
    if (td.nt) { GSC_CHEB(BB, SP, M, true) } else { GSC_CHEB(BB, SP, M, false) }
#define GSC_CHEB_M(BB, SP)                    \
    if (mode == 0) { GSC_CHEB_N(BB, SP, 0) }  \
    else if (mode == 1) { GSC_CHEB_N(BB, SP, 1) } else { GSC_CHEB_N(BB, SP, 2) }
#define GSC_CHEB_B(BB) \
    if (waves == 1) { GSC_CHEB_M(BB, 1) } else { GSC_CHEB_M(BB, kSplit<T>) }
    if (pr.B == 4) { GSC_CHEB_B(4) } else { GSC_CHEB_B(6) }
#undef GSC_CHEB_B
#undef GSC_CHEB_M
#undef GSC_CHEB_N
#undef GSC_CHEB
#undef GSC_CHEB_D
    GSC_HIP(hipGetLastError());
}

template void launch_cheb_step<double>(hipStream_t, const Pair &, const TileDims &, int, int, int, const double *,
                                       const c128 *, const c128 *, c128 *, const int *, double, double, double,
                                       double *, c128 *, int);
template void launch_cheb_step<float>(hipStream_t, const Pair &, const TileDims &, int, int, int, const float *,
                                      const c64 *, const c64 *, c64 *, const int *, double, double, double,
                                      double *, c128 *, int);

// ------------------------------------------------------------------ mixed inner solve
// Complex64 rounds of the inner solve S Y = r refined in FP64 (iterative
// refinement).  Inside a round the iterates y live in complex64 and each step
// runs in FP32 arithmetic against the FP32 copy of S, solving S y = f for the
// round's right-hand side f (complex64).  The round's last step (FIN) does not
// store its iterate: it adds it to the FP64 solution Y (FIN 1: Y = y, FIN 2:
// Y += y); OUT as in k_cheb_step, with the partial of Y^T r (unconjugated,
// FP64: the next rho of the outer iteration, eq. CGp:p) from the FP64 r.
// Between rounds k_mx_resid forms the next right-hand side f = r - S Y in
// FP64, so rounding in the complex64 rounds limits only how fast the
// refinement converges, not where it ends.
//
// V = c64x2: two adjacent columns a lane, 128 a launch column (every load
// 16 bytes a lane); V = c64: one, for the 64-column tail.
template <typename V> struct mx_lane;
template <> struct mx_lane<c64> {
    static constexpr int W = 1;
    static __device__ c64 &at(c64 &v, int) { return v; }
};
template <> struct mx_lane<c64x2> {
    static constexpr int W = 2;
    static __device__ c64 &at(c64x2 &v, int h) { return h ? v.b : v.a; }
};

template <typename V, int B, int SPLIT, int MODE, int FIN, int OUT>
__global__ __launch_bounds__(kBlock) void k_cheb_mx(
    int nb, int Rp, int col0, bool ragged, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *__restrict__ Sv, const c64 *__restrict__ y, const c64 *__restrict__ f, c64 *__restrict__ yio,
    c128 *__restrict__ Y, const c128 *__restrict__ r, const int *__restrict__ skip, float inv_theta, float c1,
    float c2, double *__restrict__ partial, c128 *__restrict__ dpart, int dot_active_only) {
    using L = mx_lane<V>;
    constexpr int W = L::W;
    __shared__ RowSums<V, B, SPLIT> red;
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int cb = col0 + cx * 64 * W, col = cb + W * lane;
    const size_t ld = Rp / W;      // in V
    bool on[W], act = false;
#pragma unroll
    for (int h = 0; h < W; ++h) { on[h] = !skip[col + h]; act = act || on[h]; }
    double acc2[W];
    c128 dacc[W];
#pragma unroll
    for (int h = 0; h < W; ++h) { acc2[h] = 0.0; dacc[h] = {0.0, 0.0}; }
    const V *x = reinterpret_cast<const V *>((MODE == 0 ? f : y) + cb);
    const V *fb = reinterpret_cast<const V *>(f + cb);
    V *yb = reinterpret_cast<V *>(yio + cb);
    struct Elem { V own, f, yprev; };
    walk_rows<SPLIT, false, false>(
        act, nb, g, w, lane, rowptr, colidx, Sv, Sv, x, ld, red, red,
        [&](size_t row) {
            const size_t e = row * ld + lane;
            Elem v{x[e], {}, {}};
            if constexpr (MODE != 0) v.f = fb[e];
            if constexpr (MODE == 2) v.yprev = yb[e];
            return v;
        },
        NoCombine{},
        [&](size_t row, V s, V, Elem v) {
            V nw = s;
            bool all = true;
#pragma unroll
            for (int h = 0; h < W; ++h) {
                double res2;
                const c64 ynew = cheb_next<float, MODE>(L::at(v.own, h), L::at(s, h), L::at(v.f, h),
                                                        L::at(v.yprev, h), inv_theta, c1, c2, res2);
                L::at(nw, h) = ynew;
                all = all && on[h];
                if (!on[h]) continue;
                if constexpr (OUT >= 1) acc2[h] += res2;
                if constexpr (FIN != 0) {
                    const size_t e = row * Rp + col + h;
                    c128 sum = ccast<double>(ynew);
                    if constexpr (FIN == 2) sum = Y[e] + sum;
                    Y[e] = sum;
                    if constexpr (OUT == 2) dacc[h] = dacc[h] + sum * r[e];
                }
            }
            if constexpr (FIN == 0) {
                if (all) {
                    yb[row * ld + lane] = nw;
                } else {
#pragma unroll
                    for (int h = 0; h < W; ++h)
                        if (on[h]) yio[row * Rp + col + h] = L::at(nw, h);
                }
            }
        });
    if constexpr (OUT >= 1) {
        __shared__ double redd[W][kWavesPerBlock][64];
#pragma unroll
        for (int h = 0; h < W; ++h)
            wave_sums_store(acc2[h], redd[h], w, lane, partial + static_cast<size_t>(g) * Rp + col + h);
    }
    if constexpr (OUT == 2) {
        __shared__ c128 redc[W][kWavesPerBlock][64];
#pragma unroll
        for (int h = 0; h < W; ++h)
            wave_sums_store(dacc[h], redc[h], w, lane, dpart + static_cast<size_t>(g) * Rp + col + h,
                            on[h] || !dot_active_only);
    }
}

// f = r - S Y in FP64 (S, Y, r in FP64), stored in complex64 as the
// right-hand side of the next complex64 round.
template <int B, int SPLIT>
__global__ __launch_bounds__(kBlock) void k_mx_resid(
    int nb, int Rp, int col0, bool ragged, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const double *__restrict__ Sv, const c128 *__restrict__ Y, const c128 *__restrict__ r, c64 *__restrict__ f,
    const int *__restrict__ skip) {
    using V = c128;
    __shared__ RowSums<V, B, SPLIT> red;
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int cb = col0 + cx * 64;
    const size_t ld = Rp;
    walk_rows<SPLIT, false, false>(
        !skip[cb + lane], nb, g, w, lane, rowptr, colidx, Sv, Sv, Y + cb, ld, red, red,
        [&](size_t row) { return r[row * ld + cb + lane]; }, NoCombine{},
        [&](size_t row, V s, V, V rv) { f[row * ld + cb + lane] = ccast<float>(rv - s); });
}

void launch_cheb_mx(hipStream_t st, const Pair &pr, const TileDims &td, int mode, int fin, bool dot, int col0,
                    int ncols, const float *Sv, const c64 *y, const c64 *f, c64 *yio, c128 *Y, const c128 *r,
                    const int *skip, double inv_theta, double c1, double c2, double *partial, c128 *dpart,
                    int dot_active_only) {
    GSC_REQUIRE(col0 % 64 == 0 && ncols % 64 == 0 && ncols > 0 && col0 + ncols <= td.Rp,
                "Chebyshev column block outside the tile");
    GSC_REQUIRE(mode >= 0 && mode <= 2 && fin >= 0 && fin <= 2, "bad mixed Chebyshev step");
    GSC_REQUIRE(!dot || (fin > 0 && dpart != nullptr && r != nullptr && partial != nullptr),
                "the fused dot needs a final step and its partials");
    GSC_REQUIRE(fin == 0 || Y != nullptr, "a final step needs the FP64 solution");
    GSC_REQUIRE(fin != 0 || partial == nullptr, "only a final step leaves partial sums");
    const float it = static_cast<float>(inv_theta), a = static_cast<float>(c1), b = static_cast<float>(c2);
    // 128-column pieces with two columns per lane, a 64-column tail with one
    const int n2 = ncols / 128 * 128;
#define GSC_MX(V, BB, SP, M, F, O)                                                                          \
    k_cheb_mx<V, BB, SP, M, F, O><<<grid, kBlock, 0, st>>>(td.nb, td.Rp, c0, ragged, pr.rowptr.get(),       \
                                                           pr.colidx.get(), Sv, y, f, yio, Y, r, skip, it,  \
                                                           a, b, partial, dpart, dot_active_only)
#define GSC_MX_O(V, BB, SP, M, F)                     \
    if (dot) GSC_MX(V, BB, SP, M, F, 2);              \
    else if (partial) GSC_MX(V, BB, SP, M, F, 1);     \
    else GSC_MX(V, BB, SP, M, F, 0);
#define GSC_MX_F(V, BB, SP, M)                   \
    if (fin == 0) { GSC_MX(V, BB, SP, M, 0, 0); } \
    else if (fin == 1) { GSC_MX_O(V, BB, SP, M, 1) } else { GSC_MX_O(V, BB, SP, M, 2) }
#define GSC_MX_M(V, BB, SP)                    \
    if (mode == 0) { GSC_MX_F(V, BB, SP, 0) }  \
    else if (mode == 1) { GSC_MX_F(V, BB, SP, 1) } else { GSC_MX_F(V, BB, SP, 2) }
    if (n2 > 0) {
        const dim3 grid(n2 / 128, partial ? td.Gs : td.Gw);
        const int c0 = col0;
        const bool ragged = ragged_end(c0 + n2, td.R, 128);
        if (pr.B == 4) { GSC_MX_M(c64x2, 4, 4) } else { GSC_MX_M(c64x2, 6, 4) }
    }
    if (n2 < ncols) {
        const int waves = step_waves(td.nb, 1, td.row_orbitals, true);
        const dim3 grid(1, partial ? td.Gs : waves == 1 ? td.G1 : td.Gw);
        const int c0 = col0 + n2;
        const bool ragged = false;      // one chunk
        if (pr.B == 4) { if (waves == 1) { GSC_MX_M(c64, 4, 1) } else { GSC_MX_M(c64, 4, 4) } }
        else { if (waves == 1) { GSC_MX_M(c64, 6, 1) } else { GSC_MX_M(c64, 6, 4) } }
    }
#undef GSC_MX_M
#undef GSC_MX_F
#undef GSC_MX_O
#undef GSC_MX
    GSC_HIP(hipGetLastError());
}

void launch_mx_resid(hipStream_t st, const Pair &pr, const TileDims &td, int col0, int ncols, const double *Sv,
                     const c128 *Y, const c128 *r, c64 *f, const int *skip) {
    GSC_REQUIRE(col0 % 64 == 0 && ncols % 64 == 0 && ncols > 0 && col0 + ncols <= td.Rp,
                "Chebyshev column block outside the tile");
    const int waves = step_waves(td.nb, ncols / 64, td.row_orbitals, false);
    dim3 grid(ncols / 64, waves == 1 ? td.G1 : td.Gw), block(kBlock);
    const bool ragged = ragged_end(col0 + ncols, td.R, 64);
#define GSC_RESID(BB, SP)                                                                                       \
    k_mx_resid<BB, SP><<<grid, block, 0, st>>>(td.nb, td.Rp, col0, ragged, pr.rowptr.get(), pr.colidx.get(), Sv, \
                                               Y, r, f, skip)
    if (pr.B == 4) { if (waves == 1) GSC_RESID(4, 1); else GSC_RESID(4, 4); }
    else { if (waves == 1) GSC_RESID(6, 1); else GSC_RESID(6, 4); }
#undef GSC_RESID
    GSC_HIP(hipGetLastError());
}

// ------------------------------------------------------------------ launchers
void set_spmm_geometry(TileDims &td, const Pair &pr, bool one_wave) {
    const int w = td.cb > 0 && td.cb < td.Rp ? td.cb : td.Rp;   // width of a Chebyshev launch
    td.row_orbitals = static_cast<int>(pr.nnzb * pr.B / pr.nb);
    static_cast<RowGroups &>(td) = row_groups(td.nb, td.Rp / 64, std::max(1, w / 64), td.row_orbitals, one_wave);
}

template <typename T>
void launch_spmm_seed(hipStream_t st, const Pair &pr, const TileDims &td, const T *Sv, const T *Hv,
                      const cpx<T> *p, cpx<T> *q, const c128 *z, const int *seed, const int *skip,
                      c128 *partial) {
    dim3 grid(td.Rp / 64, td.G2), block(kBlock);
    const bool ragged = ragged_end(td.Rp, td.R, 64);
#define GSC_SEED(BB, SP)                                                                                         \
    k_spmm_seed<T, BB, SP><<<grid, block, 0, st>>>(td.nb, td.Rp, ragged, pr.rowptr.get(), pr.colidx.get(), Sv, Hv,   \
                                                   p, q, z, seed, skip, partial)
#define GSC_SEED_S(BB) \
    if (td.waves2 == 1) GSC_SEED(BB, 1); else GSC_SEED(BB, kSplit<T>);
    if (pr.B == 4) { GSC_SEED_S(4) } else { GSC_SEED_S(6) }
#undef GSC_SEED_S
#undef GSC_SEED
    GSC_HIP(hipGetLastError());
}

template <typename T>
void launch_spmm_S(hipStream_t st, const Pair &pr, const TileDims &td, const T *Sv, const cpx<T> *d,
                   cpx<T> *w, const int *skip, double *partial) {
    dim3 grid(td.Rp / 64, td.G2), block(kBlock);
    const bool ragged = ragged_end(td.Rp, td.R, 64);
#define GSC_S(BB, SP)                                                                                            \
    k_spmm_S<T, BB, SP><<<grid, block, 0, st>>>(td.nb, td.Rp, ragged, pr.rowptr.get(), pr.colidx.get(), Sv, d, w, \
                                                skip, partial)
    if (pr.B == 4) { if (td.waves2 == 1) GSC_S(4, 1); else GSC_S(4, kSplit<T>); }
    else { if (td.waves2 == 1) GSC_S(6, 1); else GSC_S(6, kSplit<T>); }
#undef GSC_S
    GSC_HIP(hipGetLastError());
}

template void launch_spmm_seed<double>(hipStream_t, const Pair &, const TileDims &, const double *,
                                       const double *, const c128 *, c128 *, const c128 *, const int *,
                                       const int *, c128 *);
template void launch_spmm_seed<float>(hipStream_t, const Pair &, const TileDims &, const float *,
                                      const float *, const c64 *, c64 *, const c128 *, const int *,
                                      const int *, c128 *);
template void launch_spmm_S<double>(hipStream_t, const Pair &, const TileDims &, const double *,
                                    const c128 *, c128 *, const int *, double *);
template void launch_spmm_S<float>(hipStream_t, const Pair &, const TileDims &, const float *, const c64 *,
                                   c64 *, const int *, double *);

}  // namespace gsc
