// The outer iteration of small systems: one workgroup runs one right-hand side
// from its first step to its last (Sec. 3.3, the steps and eqs. listed at the
// top of solver.hip).
//
// A column is an independent Krylov process, and for a few hundred orbitals its
// vectors fit one CU: a quad of lanes works on two orbitals and keeps their
// elements of r, p and the Chebyshev iterates in registers; only the gathered
// vector goes through LDS (two buffers, one barrier a step).  S and H sit in
// registers as far as they fit and stream from L2 otherwise.  The launch per
// kernel of the tiled path, about 24 an outer iteration with 4 to 7 us each
// however small the system, becomes a barrier, and no status is read back
// between iterations.
//
// What bounds it is one CU's product: the chain of LDS reads and fmas of a
// Chebyshev step (about 1 us at N = 256).  Measured, the tiled path
// that it replaced -> this kernel, 64 shifts: Green's functions N 256 R 8 47 -> 8.3
// ms, charges N 144 R 144 32 -> 4.6 ms, gradients of a loss N 384 R 130 221 -> 60 ms,
// of the band energy N 384 R 384 255 -> 114 ms (the product of the tiles has become
// faster since: 37, 27, - and 158 ms there).
// One row a lane read LDS twice as often; unpacked S and H cost a gather of
// 8-byte values; more blocks in registers spilled (rows below: the fastest of
// a scan, in blocks a lane keeps of S and of H).
//
// The inner solve is the FP64 Chebyshev iteration for GSC_MIXED too: with the
// vectors on chip complex64 rounds save no bandwidth, and the refinement passes
// would cost more than they replace.
#include <algorithm>

#include "small.h"

namespace gsc {

namespace {

constexpr int kSmallMax = 1024;      // threads of a workgroup
constexpr int kSmallRows = 512;      // largest N of this path (1024 threads)
// Largest N times rounds of columns over the CUs, one column a CU at a time.
// Measured on both sides, this kernel and the tiles (ms, 64 shifts): charges
// N 368 R 100 12.6 | 39, N 512 R 100 18.3 | 33; gradients N 504 R 130 78 | 102,
// N 384 R 384 (768) 111 | 142, N 504 R 504 (1008) 89 | 71; band charges N 504
// R 504 68 | 55; Green's functions N 512 R 500 (1024) 66 | 65.
constexpr int kSmallRowRounds = 768;
constexpr int kFlushSteps = 8;       // r' elements a lane holds in a shift-update pass

// `v` as a value the compiler cannot trace out of the loop: without it the
// addresses of every (shift, column) array stay in registers from one outer
// iteration to the next, and the rows of S are spilled for them
__device__ inline int here(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// a value that is the same in every lane, in scalar registers
__device__ inline double uni(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<int>(u & 0xffffffffull));
    const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<int>(u >> 32));
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}
__device__ inline c128 uni(c128 v) { return {uni(v.re), uni(v.im)}; }
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// sums over the workgroup of NV values a lane, in every lane; red: 16 * NV
template <int NV>
__device__ inline void group_sum(double (&v)[NV], double *red, int nw) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], o);
    const int w = threadIdx.x >> 6;
    __syncthreads();                 // the last sums have been read
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) red[w * NV + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double s = 0.0;
        for (int j = 0; j < nw; ++j) s += red[j * NV + k];
        v[k] = uni(s);
    }
}

// Gathered vectors lie in LDS by orbital slot, x[slot * nb + block]: the lanes
// of a wave read one slot of different blocks at a time, which this spreads
// over the banks (16 bytes a block; by rows, B * 16 apart, four blocks of sp3
// share a bank).
__device__ inline int lds_at(int i, int B, int nb) { return i % B * nb + i / B; }

// the value of the lane 1 or 2 over in its quad
template <int X> __device__ inline double quad_xor(double v) {
    constexpr int kPerm = X == 1 ? 0xB1 : 0x4E;      // quad_perm [1,0,3,2] or [2,3,0,1]
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_mov_dpp(static_cast<int>(u & 0xffffffffull), kPerm, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_mov_dpp(static_cast<int>(u >> 32), kPerm, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

// Two rows of one block row of a matrix, orbital slots a and a + 1, held by the
// four lanes of a quad, which take its stored blocks [b0, b1) in turn (two rows a
// lane halve the LDS reads of x per value).  The matrix comes packed by lanes:
// value pair e of the lane's jth block at pk[(j * B + e) * nt], so a wave load is
// 1 KiB without a gap; blocks beyond the row are zeros.  The first NBL blocks of
// a lane stay in registers for the whole solve, the rest stream from L2 at every
// product.
struct alignas(16) d2 { double x, y; };
template <int B> __device__ inline void load_pair(const d2 *pk, int j, int nt, double (&v)[2][B]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < B; c += 2) {
            const d2 t = pk[static_cast<size_t>(j * B + (h * B + c) / 2) * nt];
            v[h][c] = t.x;
            v[h][c + 1] = t.y;
        }
}
template <int B, int NBL> struct RowPair {
    double v[NBL > 0 ? NBL : 1][2][B];
    __device__ void load(const d2 *pk, int nt, int nj) {
#pragma unroll
        for (int j = 0; j < NBL; ++j) {
            if (j < nj) {
                load_pair<B>(pk, j, nt, v[j]);
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int c = 0; c < B; ++c) v[j][h][c] = 0.0;
            }
        }
    }
    // (M x) of row a + (lane & 1); col: block columns of the lane's blocks
    __device__ c128 times(const d2 *pk, int nt, int nj, const uint16_t *lcol, int bq, int b1, const c128 *x,
                          int nb) const {
        c128 s0{0, 0}, s1{0, 0};
        auto add = [&](const double (&m)[2][B], int j) {
            const int b = bq + 4 * j;
            const c128 *xb = x + (b < b1 ? lcol[b] : 0);
#pragma unroll
            for (int c = 0; c < B; ++c) {
                const c128 t = xb[c * nb];
                s0.re = fma(m[0][c], t.re, s0.re);
                s0.im = fma(m[0][c], t.im, s0.im);
                s1.re = fma(m[1][c], t.re, s1.re);
                s1.im = fma(m[1][c], t.im, s1.im);
            }
        };
#pragma unroll
        for (int j = 0; j < NBL; ++j) add(v[j], j);
#pragma unroll 1
        for (int j = NBL; j < nj; ++j) {
            double m[2][B];
            load_pair<B>(pk, j, nt, m);
            add(m, j);
        }
        // each lane passes the neighbour's row on and keeps its own
        const bool odd = threadIdx.x & 1;
        const c128 mine = odd ? s1 : s0, give = odd ? s0 : s1;
        c128 t{mine.re + quad_xor<1>(give.re), mine.im + quad_xor<1>(give.im)};
        return {t.re + quad_xor<2>(t.re), t.im + quad_xor<2>(t.im)};
    }
};

// the packed form of a matrix (RowPair), one block of threads a lane block j
template <int B>
__global__ void k_small_pack(int nb, int nt, const int32_t *rowptr, const double *S, const double *H, d2 *pS, d2 *pH) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (t >= nt) return;
    const int unit = t >> 2, I = unit / (B / 2), a = 2 * (unit % (B / 2));
    const int b = I < nb ? rowptr[I] + (t & 3) + 4 * j : 0;
    const bool in = I < nb && b < rowptr[I + 1];
    for (int e = 0; e < B; ++e) {
        const size_t o = static_cast<size_t>(j * B + e) * nt + t;
        const size_t m = (static_cast<size_t>(b) * B + a) * B + 2 * e;
        pS[o] = in ? d2{S[m], S[m + 1]} : d2{0.0, 0.0};
        pH[o] = in ? d2{H[m], H[m + 1]} : d2{0.0, 0.0};
    }
}

// Pending steps [n0, n1) of the shifted recurrences on x^k and p^k of column c
// (as k_flush): a wave group of ceil(N / 64) waves takes a shift at a time.
__device__ inline void flush_column(const SmallSolve &s, int c, int n0, int n1, int nw) {
    const int wg = (s.N + 63) / 64, groups = nw / wg;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = w / wg, i = here((w % wg) * 64 + (threadIdx.x & 63));
    if (grp >= groups || i >= s.N) return;
    const size_t base = static_cast<size_t>(c) * s.N + i;
    const size_t NR = static_cast<size_t>(s.N) * s.Rp;
    for (int t0 = n0; t0 < n1; t0 += kFlushSteps) {
        const int cnt = min(kFlushSteps, n1 - t0);
        c128 rr[kFlushSteps];
#pragma unroll
        for (int j = 0; j < kFlushSteps; ++j)
            rr[j] = j < cnt ? s.ringT[((t0 + j) % s.m) * NR + base] : c128{0, 0};
        for (int k = grp; k < s.K; k += groups) {
            const int last = s.ss.last[shift_at(s.K, k, c)];
            const int kc = min(cnt, last >= n1 ? cnt : last + 1 - t0);
            if (kc <= 0) continue;
            const size_t ox = static_cast<size_t>(k) * s.ldx + base, op = static_cast<size_t>(k) * s.ldp + base;
            c128 pv{0, 0}, xv{0, 0};
            if (t0 > 0) {            // before step 0 both are zero and not read
                pv = s.P[op];
                xv = s.X[ox];
            }
#pragma unroll
            for (int j = 0; j < kFlushSteps; ++j) {
                if (j < kc) {
                    const size_t f = coef_at(s.ss, k, c, (t0 + j) % s.m);
                    pv = s.ss.ra[f] * rr[j] + s.ss.rb[f] * pv;
                    xv = xv + s.ss.rc[f] * pv;
                }
            }
            s.P[op] = pv;
            s.X[ox] = xv;
        }
    }
}

template <int B, int NBS, int NBH, int MAXT>
__global__ __launch_bounds__(MAXT) void k_small_solve(SmallSolve s) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int N = s.N, Rp = s.Rp, K = s.K, tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6;
    const int M = s.Mu + s.srow;
    c128 *buf0 = reinterpret_cast<c128 *>(lds), *buf1 = buf0 + N, *rpb = buf1 + N;   // gathered x (two), r'_n
    c128 *cr = rpb + N;                                                              // projections of r'_n
    double *red = reinterpret_cast<double *>(cr + M);                                // 16 x 4
    uint16_t *col = reinterpret_cast<uint16_t *>(red + 64);                          // block columns
    const int nb = s.nb;
    const int c = blockIdx.x;
    if (c >= s.R || s.cs.done[c]) return;
    const int nnzb = s.rowptr[s.nb];
    for (int b = tid; b < nnzb; b += nt) col[b] = static_cast<uint16_t>(s.colidx[b]);
    // the quad's block row and its two orbitals; the lane's own is i, and lanes
    // 0 and 1 of a quad speak for theirs
    const int unit = tid >> 2, I = min(unit / (B / 2), s.nb - 1);
    const bool own = unit / (B / 2) < s.nb, first = own && (tid & 2) == 0;
    const int i = I * B + 2 * (unit % (B / 2)) + (tid & 1);
    const int b0 = own ? s.rowptr[I] : 0, b1 = own ? s.rowptr[I + 1] : 0;
    c128 p{0, 0}, r{0, 0}, rp{0, 0};
    if (own) {
        const size_t e = static_cast<size_t>(i) * Rp + c;
        p = s.p[e];
        r = s.r[e];
        rp = s.rp[e];
    }
    const int at = lds_at(i, B, nb);
    if (first) {
        buf0[at] = p;
        rpb[at] = rp;
    }
    const size_t ring_ld = static_cast<size_t>(N) * Rp, ring_at = static_cast<size_t>(c) * N + i;
    // scalars of the column, the same in every lane
    c128 rho = uni(s.cs.rho[c]), alpha_prev{1.0, 0.0}, beta_prev{0.0, 0.0};
    const double bn = uni(s.cs.bnorm[c]);
    int seed = uni(s.cs.seed[c]), flags = 0, iters = 0, n0 = 0, switches = 0;
    long long shift_iters = 0;
    bool done = false;
    // z-derivative carry (k_proj_update_vjp): projection vm's sums over the
    // shifts k = vset (mod sets), kept through the solve and added in set order
    int sets = 0;
    if (s.dh != nullptr && M > 0)
        for (sets = 1; sets * 2 * M <= nt && sets < 16;) sets *= 2;
    const int vm = M > 0 ? tid % M : 0, vset = M > 0 ? tid / M : 0;
    c128 ag{0, 0}, ad{0, 0}, az{0, 0};
    const double inv_theta = 1.0 / s.theta, sigma = s.theta / s.delta;
    __syncthreads();
    const d2 *pS = reinterpret_cast<const d2 *>(s.packed) + tid, *pH = pS + static_cast<size_t>(s.nj) * B * nt;
    const int nj = s.nj, bq = b0 + (tid & 3);
    RowPair<B, NBS> Sr;
    RowPair<B, NBH> Hr;
    Sr.load(pS, nt, nj);
    Hr.load(pH, nt, nj);
    for (int n = 0; n < s.max_iter && !done; ++n) {
        const int slot = n % s.m, tk = here(tid);
        // ---- q = z_s S p - H p, mu = p^T q, alpha
        const c128 zs = uni(s.ss.z[seed]);
        const c128 aS = Sr.times(pS, nt, nj, col, bq, b1, buf0, nb);
        const c128 aH = Hr.times(pH, nt, nj, col, bq, b1, buf0, nb);
        const c128 q = zs * aS - aH, pq = p * q;
        double mv[2] = {first ? pq.re : 0.0, first ? pq.im : 0.0};
        group_sum<2>(mv, red, nw);
        const c128 mu{mv[0], mv[1]}, alpha = uni(cdiv(rho, mu));
        if (!cfinite(mu) || !cfinite(alpha)) {
            flags |= cfinite(mu) ? FLAG_BREAKDOWN : FLAG_NAN;
            break;
        }
        if (cabs(mu) == 0.0 || cabs(alpha) == 0.0) {
            flags |= FLAG_BREAKDOWN;
            break;
        }
        // ---- shift coefficients of step n (k_ctrl)
        const c128 tail = uni(cdiv(alpha * beta_prev, alpha_prev));
        int cnt = 0;
        for (int k = tk; k < K; k += nt) {
            const size_t idx = shift_at(K, k, c);
            if (s.ss.last[idx] != kFrozenNever) continue;
            ++cnt;
            const c128 pi = s.ss.pi[idx], pim = s.ss.pi_prev[idx];
            const c128 lead = c128{1.0, 0.0} + alpha * (s.ss.z[k] - zs);
            const c128 pin = lead * pi + tail * (pi - pim);
            s.ss.pi_next[idx] = pin;
            const c128 qq = cdiv(pim, pi);
            const c128 ak = cdiv(alpha * pi, pin);
            const size_t f = coef_at(s.ss, k, c, slot);
            s.ss.ra[f] = cdiv(c128{1.0, 0.0}, pi);
            s.ss.rb[f] = (qq * qq) * beta_prev;
            s.ss.rc[f] = s.ss.omega[idx] * ak;
            if (s.ss.dpi != nullptr) {
                const c128 dpi = s.ss.dpi[idx], dpim = s.ss.dpi_prev[idx];
                const c128 dpin = alpha * pi + lead * dpi + tail * (dpi - dpim);
                s.ss.dpi_next[idx] = dpin;
                const c128 dak = cdiv(alpha * (dpi * pin - pi * dpin), pin * pin);
                s.ss.rda[f] = cdiv(c128{-dpi.re, -dpi.im}, pi * pi);
                s.ss.rdb[f] = cdiv(2.0 * beta_prev * qq * (dpim * pi - pim * dpi), pi * pi);
                s.ss.rdc[f] = s.ss.domega[idx] * ak + s.ss.omega[idx] * dak;
            }
        }
        ++iters;
        // ---- r <- r - alpha q, ||r||^2 (and the active shifts)
        r = r - alpha * q;
        double rv[2] = {first ? cabs2(r) : 0.0, static_cast<double>(cnt)};
        if (first) buf1[at] = r;
        group_sum<2>(rv, red, nw);   // its barriers publish buf1 and the coefficients
        const double rn2 = rv[0];
        shift_iters += static_cast<long long>(rv[1]);
        // ---- projections of r'_n and their carry (k_proj_update)
        if (s.X == nullptr) {
            for (int mm = tk; mm < s.Mu; mm += nt) cr[mm] = rpb[lds_at(s.pidx[static_cast<size_t>(c) * s.Mu + mm], B, nb)];
            if (s.srow) {
                const int64_t ao = s.rhs[c];
                const int Ia = static_cast<int>(ao / B), aa = static_cast<int>(ao % B);
                if (tid < 64) {
                    const int c0 = s.rowptr[Ia], len = (s.rowptr[Ia + 1] - c0) * B;
                    c128 v{0, 0};
                    for (int t = tid; t < len; t += 64)
                        v = v + s.S[(static_cast<size_t>(c0 + t / B) * B + aa) * B + t % B] *
                                    rpb[t % B * nb + col[c0 + t / B]];
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) {
                        v.re += __shfl_xor(v.re, o);
                        v.im += __shfl_xor(v.im, o);
                    }
                    if (tid == 0) cr[s.Mu] = v;
                }
            }
            __syncthreads();
            if (s.dh == nullptr) {
                for (int t = tk; t < K * M; t += nt) {
                    const int k = t / M, mm = t % M;
                    const size_t idx = shift_at(K, k, c);
                    if (s.ss.last[idx] != kFrozenNever) continue;
                    const size_t f = coef_at(s.ss, k, c, slot), o = idx * M + mm;
                    const c128 hv = s.ss.ra[f] * cr[mm] + s.ss.rb[f] * s.h[o];
                    s.h[o] = hv;
                    s.g[o] = s.g[o] + s.ss.rc[f] * hv;
                }
            } else {
                if (vset < sets) {
                    const c128 crm = cr[vm];
                    for (int k = here(vset); k < K; k += sets) {
                        const size_t idx = shift_at(K, k, c);
                        if (s.ss.last[idx] != kFrozenNever) continue;
                        const size_t f = coef_at(s.ss, k, c, slot), o = idx * M + vm;
                        const c128 hold = s.h[o], dhold = s.dh[o];
                        const c128 hv = s.ss.ra[f] * crm + s.ss.rb[f] * hold;
                        const c128 dhv = s.ss.rda[f] * crm + s.ss.rdb[f] * hold + s.ss.rb[f] * dhold;
                        s.h[o] = hv;
                        s.dh[o] = dhv;
                        const c128 dg = s.ss.rc[f] * hv;
                        const c128 ddg = s.ss.rdc[f] * hv + s.ss.rc[f] * dhv;
                        const double we = s.wE[k];
                        ag = ag + we * dg;
                        ad = ad + we * ddg;
                        az = az + we * (s.ss.z[k] * ddg);
                    }
                }
            }
        }
        // ---- S r' = r: Chebyshev steps (cheb_next), y_1 = r / theta
        const double rstop = s.inner_tol / s.rho;
        c128 yc = inv_theta * r, yp{0, 0}, *xg = buf1, *xn = buf0;
        double rho_c = 1.0 / sigma, rr2 = 0.0;
        c128 rho_new{0, 0};
        bool ok = rn2 == 0.0;
        for (int st = 1; !ok;) {
            // steps up to `end`, the residual of the last one checked
            const int end = st < s.steps ? s.steps : st + 2;
            for (; st < end; ++st) {
                const double rh = 1.0 / (2.0 * sigma - rho_c);
                const double c1 = rh * rho_c, c2 = 2.0 * rh / s.delta;
                rho_c = rh;
                c128 Sy = Sr.times(pS, nt, nj, col, bq, b1, xg, nb);
                if (st == 1) Sy = inv_theta * Sy;    // the gathered vector of step 1 is r
                const c128 res = r - Sy;
                const c128 yn = yc + c1 * (yc - yp) + c2 * res;
                yp = yc;
                yc = yn;
                if (st + 1 < end) {
                    if (first) xn[at] = yc;
                    __syncthreads();
                    c128 *t = xg;
                    xg = xn;
                    xn = t;
                } else {
                    const c128 d = yc * r;
                    double v[3] = {first ? cabs2(res) : 0.0, first ? d.re : 0.0, first ? d.im : 0.0};
                    if (first) xn[at] = yc;
                    group_sum<3>(v, red, nw);
                    c128 *t = xg;
                    xg = xn;
                    xn = t;
                    rr2 = v[0];
                    rho_new = {v[1], v[2]};
                }
            }
            if (!isfinite(rr2)) {
                flags |= FLAG_NAN;
                break;
            }
            const bool again = st > s.steps;
            const double thr = again ? s.inner_tol : rstop;
            ok = rr2 <= thr * thr * rn2;
            if (again && !ok) {
                flags |= FLAG_INNER;     // inexact S^{-1} r for this iteration
                ok = true;
            }
        }
        if (!isfinite(rn2) || (flags & FLAG_NAN)) {
            flags |= FLAG_NAN;
            break;
        }
        rp = rn2 == 0.0 ? c128{0, 0} : yc;
        // ---- beta, pi, freezing (k_post)
        const double rn = sqrt(rn2);
        double best = -1.0;
        int bestk = 0x7fffffff, left = 0;
        for (int k = tk; k < K; k += nt) {
            const size_t idx = shift_at(K, k, c);
            if (s.ss.last[idx] != kFrozenNever) continue;
            const c128 pin = s.ss.pi_next[idx];
            s.ss.pi_prev[idx] = s.ss.pi[idx];
            s.ss.pi[idx] = pin;
            if (s.ss.dpi != nullptr) {
                s.ss.dpi_prev[idx] = s.ss.dpi[idx];
                s.ss.dpi[idx] = s.ss.dpi_next[idx];
            }
            const double rs = cabs(s.ss.omega[idx]) * rn / (cabs(pin) * bn);
            s.ss.res[idx] = rs;
            if (!(rs > s.tol)) {
                s.ss.last[idx] = n;
            } else {
                ++left;
                if (rs > best) { best = rs; bestk = k; }
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double b2 = __shfl_xor(best, o);
            const int k2 = __shfl_xor(bestk, o);
            if (b2 > best || (b2 == best && k2 < bestk)) { best = b2; bestk = k2; }
            left += __shfl_xor(left, o);
        }
        __syncthreads();
        if ((tid & 63) == 0) {
            red[(tid >> 6) * 3] = best;
            red[(tid >> 6) * 3 + 1] = bestk;
            red[(tid >> 6) * 3 + 2] = left;
        }
        __syncthreads();
        best = red[0];
        bestk = static_cast<int>(red[1]);
        left = static_cast<int>(red[2]);
        for (int j = 1; j < nw; ++j) {
            const double b2 = red[3 * j];
            const int k2 = static_cast<int>(red[3 * j + 1]);
            if (b2 > best || (b2 == best && k2 < bestk)) { best = b2; bestk = k2; }
            left += static_cast<int>(red[3 * j + 2]);
        }
        best = uni(best);
        bestk = uni(bestk);
        left = uni(left);
        const c128 beta = uni(cdiv(rho_new, rho));
        c128 swc{1.0, 0.0};
        int sw = 0;
        if (left == 0) {
            done = true;
        } else if (!cfinite(rho_new) || !cfinite(beta)) {
            flags |= FLAG_NAN;
            break;
        } else if (cabs(rho_new) == 0.0) {
            flags |= FLAG_BREAKDOWN;
            break;
        } else if (s.ss.last[shift_at(K, seed, c)] != kFrozenNever) {
            sw = s.X != nullptr ? 1 : 2;
        }
        alpha_prev = alpha;
        beta_prev = beta;
        rho = rho_new;
        if (s.X != nullptr) {
            if (n + 1 - n0 == s.m || sw != 0 || done) {
                flush_column(s, c, n0, n + 1, nw);
                n0 = n + 1;
                __syncthreads();     // the ring has been read
            }
            // r' of step n + 1 for the shift updates
            if (!done && sw == 0 && first) s.ringT[((n + 1) % s.m) * ring_ld + ring_at] = rp;
        }
        if (done) break;
        if (sw != 0) {
            ++switches;
            const size_t ix = shift_at(K, bestk, c);
            const c128 cc = uni(s.ss.pi[ix]), ccm = uni(s.ss.pi_prev[ix]);
            __syncthreads();         // read before the rescale; P of the flush is visible
            if (sw == 1) {
                const c128 qq = cdiv(ccm, cc);
                rho = uni(cdiv(rho_new, cc * cc));
                beta_prev = uni((qq * qq) * beta);
                alpha_prev = uni(alpha * qq);
                swc = uni(cdiv(c128{1.0, 0.0}, cc));
                for (int k = tk; k < K; k += nt) {
                    const size_t idx = shift_at(K, k, c);
                    s.ss.pi[idx] = cdiv(s.ss.pi[idx], cc);
                    s.ss.pi_prev[idx] = cdiv(s.ss.pi_prev[idx], ccm);
                }
            } else {
                alpha_prev = {1.0, 0.0};
                beta_prev = {0.0, 0.0};
                for (int k = tk; k < K; k += nt) {
                    const size_t idx = shift_at(K, k, c);
                    if (s.ss.last[idx] == kFrozenNever) {
                        const c128 pik = s.ss.pi[idx];
                        if (s.ss.dpi != nullptr)
                            s.ss.domega[idx] =
                                cdiv(s.ss.domega[idx], pik) - cdiv(s.ss.omega[idx] * s.ss.dpi[idx], pik * pik);
                        s.ss.omega[idx] = cdiv(s.ss.omega[idx], pik);
                    }
                    s.ss.pi[idx] = {1.0, 0.0};
                    s.ss.pi_prev[idx] = {1.0, 0.0};
                    if (s.ss.dpi != nullptr) {
                        s.ss.dpi[idx] = {0.0, 0.0};
                        s.ss.dpi_prev[idx] = {0.0, 0.0};
                    }
                }
                for (int t = tk; t < K * M; t += nt) {
                    const size_t o = shift_at(K, t / M, c) * M + t % M;
                    s.h[o] = {0, 0};
                    if (s.dh != nullptr) s.dh[o] = {0, 0};
                }
            }
            seed = bestk;
        }
        // ---- p <- r' + beta p (k_p_update)
        if (sw == 1) {
            rp = swc * rp;
            r = swc * r;
            const c128 Ps = own ? s.P[static_cast<size_t>(seed) * s.ldp + ring_at] : c128{0, 0};
            p = rp + beta_prev * Ps;
            if (first) s.ringT[((n + 1) % s.m) * ring_ld + ring_at] = rp;
        } else {
            p = sw == 2 ? rp : rp + beta_prev * p;
        }
        __syncthreads();             // buf0 and r'_n have been read
        if (first) {
            buf0[at] = p;
            rpb[at] = rp;
        }
        __syncthreads();
    }
    // a column that ran out of iterations keeps its pending steps
    if (s.X != nullptr && iters > n0) flush_column(s, c, n0, iters, nw);
    for (int j = 0; j < sets; ++j) {
        if (vset == j) {
            c128 *A = s.acc + (static_cast<size_t>(c) * M + vm) * 3;
            A[0] = A[0] + ag;
            A[1] = A[1] + ad;
            A[2] = A[2] + az;
        }
        __syncthreads();
    }
    if (tid == 0) {
        s.cs.done[c] = done || (flags & ~FLAG_INNER) != 0 ? 1 : 0;
        s.cs.flags[c] |= flags;
        s.cs.iters[c] = iters;
        s.cs.shift_iters[c] = shift_iters;
        s.cs.wres[c] = -1.0;
        if (switches) atomicAdd(s.switches, switches);
    }
}

int small_threads(int N) { return (2 * N + 63) / 64 * 64; }

size_t small_lds(int N, int64_t nnzb, int M) {
    return (3 * static_cast<size_t>(N) + M) * sizeof(c128) + 64 * sizeof(double) + nnzb * sizeof(uint16_t);
}

}  // namespace

bool small_fits(const Pair &pr, int K, bool full, int M, int R, int num_cu) {
    if (pr.n > kSmallRows || (full && !small_full_carry(pr.n, K))) return false;
    const int N = static_cast<int>(pr.n);
    if (static_cast<int64_t>(N) * div_up(R, num_cu) > kSmallRowRounds) return false;
    return small_lds(N, pr.nnzb, M) <= size_t{64} << 10 && M <= small_threads(N);
}

int small_lane_blocks(const Pair &pr) {
    int64_t len = 0;
    for (int64_t I = 0; I < pr.nb; ++I) len = std::max(len, pr.h_rowptr[I + 1] - pr.h_rowptr[I]);
    return static_cast<int>((len + 3) / 4);
}

size_t small_packed(const Pair &pr, int nj) {
    return 2 * static_cast<size_t>(nj) * pr.B * small_threads(static_cast<int>(pr.n)) * 2;
}

void launch_small_solve(hipStream_t st, const Pair &pr, const SmallSolve &a) {
    const int nt = small_threads(a.N);
    GSC_REQUIRE(nt <= kSmallMax && a.Mu + a.srow <= nt, "system too large for one workgroup");
    const dim3 pg((nt + 255) / 256, a.nj);
    d2 *pS = reinterpret_cast<d2 *>(a.packed), *pH = pS + static_cast<size_t>(a.nj) * a.B * nt;
    if (a.B == 4) k_small_pack<4><<<pg, 256, 0, st>>>(a.nb, nt, a.rowptr, a.S, a.H, pS, pH);
    else k_small_pack<6><<<pg, 256, 0, st>>>(a.nb, nt, a.rowptr, a.S, a.H, pS, pH);
    const size_t lds = small_lds(a.N, pr.nnzb, a.Mu + a.srow);
#define GSC_SMALL(BB, NS, NH, MT) k_small_solve<BB, NS, NH, MT><<<a.R, nt, lds, st>>>(a)
    if (a.B == 4) {
        if (nt <= 256) GSC_SMALL(4, 5, 5, 256);
        else if (nt <= 512) GSC_SMALL(4, 4, 1, 512);
        else if (nt <= 768) GSC_SMALL(4, 3, 0, 768);
        else GSC_SMALL(4, 2, 0, 1024);
    } else {
        if (nt <= 256) GSC_SMALL(6, 7, 0, 256);
        else if (nt <= 512) GSC_SMALL(6, 4, 0, 512);
        else if (nt <= 768) GSC_SMALL(6, 2, 0, 768);
        else GSC_SMALL(6, 2, 0, 1024);
    }
#undef GSC_SMALL
    GSC_HIP(hipGetLastError());
}

}  // namespace gsc
