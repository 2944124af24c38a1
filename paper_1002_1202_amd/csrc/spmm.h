#pragma once
#include "kernels.h"

namespace gsc {

// row groups (TileDims) of the product kernels; one_wave: all of them walk a
// block row with one wave (kSplit 1)
void set_spmm_geometry(TileDims &td, const Pair &pr, bool one_wave);

// ------------------------------------------------------------------ one block row in a workgroup
// The four waves of a workgroup share one block row at a time: each takes a
// quarter of the row's stored blocks for the workgroup's 64 lanes of columns,
// the four sums meet in LDS and every wave finishes its own orbitals.  A row
// walked by one wave is a chain of 17 to 27 dependent loads (index, then x and
// S); a quarter of it ends over four times sooner, four times as many waves are
// there to hide it, and they need fewer rows in flight, whose x stays in L2.
// Average Chebyshev step of a whole solve, one wave a row -> four (before the next
// index was read ahead, see row_blocks): 24 H2O x 192
// columns 14.9 -> 6.5 us, 256 H2O x 1536 57.5 -> 47.4, 3,000 H2O x 128 (mixed)
// 34.9 -> 28.4, 633 Si x 128 (mixed) 9.8 -> 6.3, 4,096 Si x 128 32.5 -> 30.0,
// 4,096 Si x 256 55.2 -> 54.7.  What is left at the large end is the issue of
// vector loads: a wave load of 1 KiB takes 18 cycles of a CU's address path,
// from L1 or L2 alike (35 TB/s over the card).
//
// V is what one lane holds of a row: one column (c128, c64) or two adjacent
// complex64 columns (c64x2: 16-byte loads, half the loads per byte).
struct alignas(16) c64x2 { c64 a, b; };
template <typename V> struct scalar_of { using type = double; };
template <> struct scalar_of<c64> { using type = float; };
template <> struct scalar_of<c64x2> { using type = float; };
template <typename V> using scalar_t = typename scalar_of<V>::type;

template <typename T> __device__ inline void mac(cpx<T> &a, T s, cpx<T> x) {
    a.re = fma(s, x.re, a.re);
    a.im = fma(s, x.im, a.im);
}
__device__ inline void mac(c64x2 &a, float s, c64x2 x) {
    mac(a.a, s, x.a);
    mac(a.b, s, x.b);
}
__device__ inline c64x2 operator+(c64x2 p, c64x2 q) { return {p.a + q.a, p.b + q.b}; }

// Pattern and matrix values are read through the scalar cache: the constant
// address space says that nothing writes them while the kernel runs, which the
// compiler cannot see across the barriers of the row loop.
template <typename T> using const_mem = const T __attribute__((address_space(4))) *;
template <typename T> __device__ inline const_mem<T> as_const(const T *p) {
    return reinterpret_cast<const_mem<T>>(reinterpret_cast<uintptr_t>(p));
}

// x rows of block column J: a uniform base and the lane's offset
template <typename V, int B> __device__ inline void load_block(V (&x)[B], const V *base, int J, size_t ld, int lane) {
#pragma unroll
    for (int c = 0; c < B; ++c) x[c] = (base + (static_cast<size_t>(J) * B + c) * ld)[lane];
}
template <typename V, int B> __device__ inline void mac_block(V (&acc)[B], const_mem<scalar_t<V>> m, const V (&x)[B]) {
#pragma unroll
    for (int a = 0; a < B; ++a)
#pragma unroll
        for (int c = 0; c < B; ++c) mac(acc[a], m[a * B + c], x[c]);
}

// acc += M x over the n stored blocks from s0 on (TWO: acc2 += M2 x as well).
// What other waves there are hides the loop's latencies better than registers
// spent on loads in flight (x of one block ahead or two blocks at a time, against
// none: 256 H2O x 1536 columns 60.6 and 49.2 against 47.4 us a step, 3,000 H2O x
// 96 mixed 32.6 and 29.5 against 28.4).  The index of the next block is the
// exception (AHEAD): scalar loads end together, so an index waits for M's values
// of its block, and the x loads for both (whole solves without and with it: 256
// H2O x 1536 360 -> 340 ms, 3,000 H2O x 96 mixed 892 -> 847, 4,096 Si x 256 745 ->
// 741; one wave a row of 27 blocks, complex64 throughout: 3,000 H2O x 64 9.0 -> 8.0, 256
// H2O x 1300 13.7 -> 12.8).  It reads one index past the row, which the pattern's array
// has room for.  Short rows of one wave load the x of two blocks together instead
// (18,432 Si x 190 mixed 200 | 202 with the index ahead).
template <typename V, int B, bool AHEAD, bool TWO>
__device__ inline void row_blocks(V (&acc)[B], V (&acc2)[B], int s0, int n, const int32_t *colidx,
                                  const scalar_t<V> *M, const scalar_t<V> *M2, const V *base, size_t ld, int lane) {
    const_mem<int32_t> ci = as_const(colidx + s0);
    const_mem<scalar_t<V>> m = as_const(M + static_cast<size_t>(s0) * B * B);
    const_mem<scalar_t<V>> m2 = as_const(M2 + static_cast<size_t>(s0) * B * B);
    auto block = [&](int J) {
        V x[B];
        load_block<V, B>(x, base, J, ld, lane);
        return [=](V(&a1)[B], V(&a2)[B]) {
            mac_block<V, B>(a1, m, x);
            if constexpr (TWO) mac_block<V, B>(a2, m2, x);
        };
    };
    if constexpr (AHEAD) {
        int J = ci[0];
#pragma unroll 1
        for (int j = 0; j < n; ++j) {
            const auto add = block(J);
            int Jn = ci[j + 1];
            add(acc, acc2);
            m += B * B;
            if constexpr (TWO) m2 += B * B;
            asm("" : "+s"(Jn));       // keeps its load up there
            J = Jn;
        }
    } else {
#pragma unroll(B == 4 ? 2 : 1)
        for (int j = 0; j < n; ++j) {
            block(ci[j])(acc, acc2);
            m += B * B;
            if constexpr (TWO) m2 += B * B;
        }
    }
}

// Waves that share a block row.  The all-complex64 seed process keeps one wave
// a row: at its accuracy floor the convergence of single columns hangs on the
// order of summation, and its results stay what they are.
template <typename T> constexpr int kSplit = sizeof(T) == 8 ? kWavesPerBlock : 1;

// Sums of the orbitals that another wave of the row finishes, through LDS.
template <typename V, int B, int SPLIT> struct RowSums { V v[SPLIT == 1 ? 1 : kWavesPerBlock][B][64]; };

// acc[a] of the SPLIT waves, added in pairs
template <int SPLIT, typename V, int B>
__device__ inline V total_sum(V mine, const RowSums<V, B, SPLIT> &red, int a, int w, int lane) {
    if constexpr (SPLIT == 1) return mine;
    static_assert(SPLIT == 1 || SPLIT == 4, "sums of one or four waves");
    V t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = k == w ? mine : red.v[k][a][lane];
    return (t[0] + t[1]) + (t[2] + t[3]);
}

// Walks the block rows of row group g: wave w takes its part of each, and for
// every orbital it finishes calls done(row, (M x)_row, (M2 x)_row, load(row)),
// row = I B + a.  load fetches what the orbital needs beside the product: of a
// shared row, and where it is more than one FP64 value (the Chebyshev step), while the
// row is walked (18,432 Si x 190 columns FP64, loads one by one between the stores |
// together after the walk | before it 252 | 249 | 244 ms), else all after it (mixed
// 200 | 200 | 201).  combine(acc, acc2)
// runs on the wave's sums before they are shared; acc2 is shared too when
// SECOND.  Waves of finished columns (act false) skip the walk.  Beside columns at
// work, the lane of a finished one (or of one beyond the last) walks with the first
// that works: its own lines are not fetched, and its sums are dropped.  Masked off
// instead, it makes the wave slow: with 8 lanes or fewer at work the walk took up to
// twice the time of one with all (4,096 Si x 8 columns, truncated runs, masked | not:
// mixed 13.0 | 10.2 ms, FP64 10.4 | 9.2; x 130 mixed 25.5 | 22.9; 3,000 H2O x 8 18.8 |
// 14.4).  A branch round the loads alone costs all lanes the loads of several
// blocks at a time (3,000 H2O x 64 17.6 -> 22.2).
template <int SPLIT, bool TWO, bool SECOND, typename V, int B, typename Load, typename Combine, typename Done>
__device__ inline void walk_rows(bool act, int nb, int g, int w, int lane, const int32_t *rowptr,
                                 const int32_t *colidx, const scalar_t<V> *M, const scalar_t<V> *M2, const V *base,
                                 size_t ld, RowSums<V, B, SPLIT> &red, RowSums<V, B, SPLIT> &red2, Load load,
                                 Combine combine, Done done) {
    const unsigned long long on = __ballot(act);
    if (on == 0) return;
    const int from = act ? lane : __builtin_ctzll(on);
    constexpr int kOwn = (B + SPLIT - 1) / SPLIT;
    const int q = w % SPLIT, step = kWavesPerBlock / SPLIT * static_cast<int>(gridDim.y);
    for (int I = kWavesPerBlock / SPLIT * g + w / SPLIT; I < nb; I += step) {
        V acc[B], acc2[B];
#pragma unroll
        for (int a = 0; a < B; ++a) { acc[a] = V{}; acc2[a] = V{}; }
        const_mem<int32_t> rp = as_const(rowptr + I);
        const int b0 = rp[0], len = rp[1] - b0;
        const int lo = len * q / SPLIT, hi = len * (q + 1) / SPLIT;
        const size_t row = static_cast<size_t>(I) * B;
        using Extra = decltype(load(row));
        Extra ex[kOwn];
        constexpr bool kFirst = SPLIT > 1 || (sizeof(V) == 16 && sizeof(Extra) > 16);
        if (kFirst && act) {
#pragma unroll
            for (int o = 0; o < kOwn; ++o)
                if (B % SPLIT == 0 || q + o * SPLIT < B) ex[o] = load(row + q + o * SPLIT);
        }
        row_blocks<V, B, (SPLIT > 1 || B == 6), TWO>(acc, acc2, b0 + lo, hi - lo, colidx, M, M2, base, ld, from);
        combine(acc, acc2);
        if constexpr (SPLIT == 1) {
            if (act) {
                if constexpr (!kFirst) {
#pragma unroll
                    for (int a = 0; a < B; ++a) ex[a] = load(row + a);
                }
#pragma unroll
                for (int a = 0; a < B; ++a) done(row + a, acc[a], acc2[a], ex[a]);
            }
        } else {
#pragma unroll
            for (int a = 0; a < B; ++a) {
                if (a % SPLIT == q) continue;
                red.v[w][a][lane] = acc[a];
                if constexpr (SECOND) red2.v[w][a][lane] = acc2[a];
            }
        }
        if constexpr (SPLIT > 1) {
            __syncthreads();
            if (act) {
#pragma unroll
                for (int a = 0; a < B; ++a) {
                    if (a % SPLIT != q) continue;
                    const V s = total_sum<SPLIT>(acc[a], red, a, w, lane);
                    const V s2 = SECOND ? total_sum<SPLIT>(acc2[a], red2, a, w, lane) : V{};
                    done(row + a, s, s2, ex[a / SPLIT]);
                }
            }
            if (I + step < nb) __syncthreads();
        }
    }
}
struct NoCombine {
    template <typename A> __device__ void operator()(A &, A &) const {}
};

// Y = factor_c S X - H X, X and Y [N][R] of the caller (not overlapping),
// factors [R] complex in host memory.  More than kProductFactors columns with
// factors of their own take one launch and a device copy of the factors in room
// [R], instead of a launch for each 128 (64 block rows, 1000 columns: 36 against 87 us).
constexpr int kProductFactors = 512;
void launch_product(hipStream_t st, const Pair &pr, int R, const double *factors, const c128 *X, c128 *Y, c128 *room);

// with the dots' partials
template <typename T>
void launch_spmm_seed(hipStream_t st, const Pair &pr, const TileDims &td, const T *Sv, const T *Hv,
                      const cpx<T> *p, cpx<T> *q, const c128 *z, const int *seed, const int *skip,
                      c128 *partial);

template <typename T>
void launch_spmm_S(hipStream_t st, const Pair &pr, const TileDims &td, const T *Sv, const cpx<T> *d,
                   cpx<T> *w, const int *skip, double *partial);

// partial == nullptr: a step whose residual nobody asks for (dot_mode 0)
template <typename T>
void launch_cheb_step(hipStream_t st, const Pair &pr, const TileDims &td, int mode, int col0, int ncols, const T *Sv,
                      const cpx<T> *y, const cpx<T> *r, cpx<T> *yio, const int *skip, double inv_theta,
                      double c1, double c2, double *partial, c128 *dpart = nullptr, int dot_mode = 0);

// mixed inner solve: one complex64 Chebyshev step (FP32 S, FP32 arithmetic)
// for S y = f, mode as launch_cheb_step; fin 0 stores y_{k+1} over y_{k-1},
// fin 1 writes Y = y_{k+1}, fin 2 adds Y += y_{k+1} (Y complex128), with dot
// also the partials of Y^T r into dpart (partial == nullptr: neither).
// launch_mx_resid: f = r - S Y (FP64) in complex64.
void launch_cheb_mx(hipStream_t st, const Pair &pr, const TileDims &td, int mode, int fin, bool dot, int col0,
                    int ncols, const float *Sv, const c64 *y, const c64 *f, c64 *yio, c128 *Y, const c128 *r,
                    const int *skip, double inv_theta, double c1, double c2, double *partial, c128 *dpart,
                    int dot_active_only);
void launch_mx_resid(hipStream_t st, const Pair &pr, const TileDims &td, int col0, int ncols, const double *Sv,
                     const c128 *Y, const c128 *r, c64 *f, const int *skip);

// h = H u and s = S u with the split dots of two packed real Lanczos
// processes per column
template <typename T>
void launch_lz_hprod(hipStream_t st, const Pair &pr, const TileDims &td, const T *Hv, const T *Sv, const cpx<T> *u,
                     cpx<T> *h, cpx<T> *su, const int *skip, double *part);

}  // namespace gsc
