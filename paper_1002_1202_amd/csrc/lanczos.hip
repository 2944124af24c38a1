// Products of the generalised Lanczos step (Sec. 3.2, eq. 1.13): h = H u and
// s = S u in one gather pass.  s is formed afresh every step: propagating it
// by the three-term recursion instead would carry the inner solve's error
// through a recursion that amplifies it by about |a_n| / b_n per step.
//
// The Lanczos vectors are real (S, H and the start vectors e_j are real), so
// two processes share one complex column: process 2c in the real parts and
// process 2c + 1 in the imaginary parts of column c.  Every linear operation
// of the step (the product with H, the solve with S) acts on the two parts
// separately; only the dot products must be split, which this kernel does:
// per column it leaves the partial sums of u_re h_re, u_im h_im (a_n of the
// two processes) and |h|^2 (the scale of the inner solve's tolerance).
// Layout, block order and the row's split over the waves are those of the row
// product kernels.
#include "spmm.h"

namespace gsc {

template <typename T, int B, int SPLIT>
__global__ __launch_bounds__(kBlock) void k_lz_hprod(int nb, int Rp, bool ragged, int G2,
                                                     const int32_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ colidx, const T *__restrict__ Hv,
                                                     const T *__restrict__ Sv, const cpx<T> *__restrict__ u,
                                                     cpx<T> *__restrict__ h, cpx<T> *__restrict__ su,
                                                     const int *__restrict__ skip, double *__restrict__ part) {
    using V = cpx<T>;
    __shared__ RowSums<V, B, SPLIT> redH, redS;
    int cx, g;
    xcd_remap_chunks(ragged, cx, g);
    const int lane = threadIdx.x & 63;
    const int wv = wave_id();
    const int col = cx * 64 + lane;
    const size_t ld = Rp;
    const V *uc = u + cx * 64;
    const bool act = !skip[col];
    double dre = 0.0, dim = 0.0, nrm = 0.0;
    walk_rows<SPLIT, true, true>(
        act, nb, g, wv, lane, rowptr, colidx, Hv, Sv, uc, ld, redH, redS,
        [&](size_t row) { return (uc + row * ld)[lane]; }, NoCombine{},
        [&](size_t row, V hv, V sv, V own) {
            h[row * ld + col] = hv;
            su[row * ld + col] = sv;
            dre += static_cast<double>(own.re) * hv.re;
            dim += static_cast<double>(own.im) * hv.im;
            nrm += static_cast<double>(hv.re) * hv.re + static_cast<double>(hv.im) * hv.im;
        });
    __shared__ double red[3][kWavesPerBlock][64];
    red[0][wv][lane] = dre;
    red[1][wv][lane] = dim;
    red[2][wv][lane] = nrm;
    __syncthreads();
    if (threadIdx.x < 64) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < kWavesPerBlock; ++k) t += red[q][k][lane];
            part[(static_cast<size_t>(q) * G2 + g) * Rp + col] = t;
        }
    }
}

template <typename T>
void launch_lz_hprod(hipStream_t st, const Pair &pr, const TileDims &td, const T *Hv, const T *Sv, const cpx<T> *u,
                     cpx<T> *h, cpx<T> *su, const int *skip, double *part) {
    dim3 grid(td.Rp / 64, td.G2), block(kBlock);
    const bool ragged = ragged_end(td.Rp, td.R, 64);
#define GSC_LZ(BB, SP)                                                                                           \
    k_lz_hprod<T, BB, SP><<<grid, block, 0, st>>>(static_cast<int>(pr.nb), td.Rp, ragged, td.G2, pr.rowptr.get(), \
                                                  pr.colidx.get(), Hv, Sv, u, h, su, skip, part)
    if (pr.B == 4) { if (td.waves2 == 1) GSC_LZ(4, 1); else GSC_LZ(4, kSplit<T>); }
    else { if (td.waves2 == 1) GSC_LZ(6, 1); else GSC_LZ(6, kSplit<T>); }
#undef GSC_LZ
    GSC_HIP(hipGetLastError());
}

template void launch_lz_hprod<double>(hipStream_t, const Pair &, const TileDims &, const double *, const double *,
                                      const c128 *, c128 *, c128 *, const int *, double *);
template void launch_lz_hprod<float>(hipStream_t, const Pair &, const TileDims &, const float *, const float *,
                                     const c64 *, c64 *, c64 *, const int *, double *);

}  // namespace gsc
