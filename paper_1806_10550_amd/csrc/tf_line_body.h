// Bodies of the whole-line sweeps of the ADI-Newton iteration (gfx950, FP64;
// Lam, Cummings & Kondic, arXiv:1806.10550, eqs. JacobianSystem1-3, NewtonError): one kernel per
// sweep, one or several waves per line (core and layout: tf_line.h, tf_internal.h; kernels: tf_line.hip for
// one film, tf_line_ens.hip for ensembles).
//
//   k_xline  x sweep: a wave holds one grid row (up to 1024 cells; longer rows two to eight waves);
//            everything a wave alone on its row touches in LDS is its own, so it has no barrier at all. Reads u_k (the row and its two neighbours) and w once, writes
//            u_{k+1} once.
//   k_yline  y sweep: a workgroup holds four neighbouring columns, one per wave, and stages their
//            u tile (two columns more on each side) and b^n with coalesced loads; each wave forms
//            the residual and the bands of its column and solves it; w goes out through LDS in
//            32-byte row pieces. Reads u_k and b^n, writes w.
//
// What bounds them: at small sizes the latency of one wave's serial elimination, reduction and
// memory round trips (kernel trace, x + y of 128^2: 5.7 + 7.2 us; 512^2: 7.8 + 11 us; the same sweeps by tile passes
// and record tree took 25 + 35 and 23 + 35 us between events), at large ones two waves per SIMD that neither stream
// nor compute all the time: of 699 us for the x sweep of 8192^2 (kernel trace of 120 passes; 2.3 TB/s of the 24 B per cell, 41 % of
// the vector issue slots), 432 remain when only loads, staging and stores are left, cells and elimination
// add 109 and the reduced system 158 (8192 columns of 1000: 89 us against 141 us for the partitioned
// passes). The waves of different lines share nothing, so the
// loads of one line overlap the arithmetic of others.
#pragma once

#include "tf_line.h"

namespace tf {

// Whether this launch of a batch stands down (PassParams::ctl); the y sweep of an iteration decides
// from the previous iteration's record, one copy per lane. Uniform over the launch.
__device__ __forceinline__ bool stands_down(const PassParams &p, bool decide)
{
    if (p.ctl == nullptr) return false;
    if (p.ctl[0] == p.epoch) return true;
    if (!decide || p.chk == nullptr) return false;
    const unsigned long long *w = p.chk + (size_t)(threadIdx.x & 63) * RES_WORDS;
    const double e = wave_max(__longlong_as_double((long long)w[RES_EMAX]));
    const unsigned f = wave_or((unsigned)w[RES_FLAGS]);
    if (f == 0u && !(e < p.tol)) return false;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        p.ctl[1] = p.it - 1;
        p.ctl[0] = p.epoch;
    }
    return true;
}

// ------------------------------------------------------------------------------------
// x sweep of grid row j. sU, s2: the wave's LDS rows (ln_row, ln_row2 doubles). rec: index of the
// wave's reduction copy and mass record. AL: the row fills its lanes (CPL divides nx), so that its first cell
// is some lane's position 0; the elimination is then one straight block of code instead of one cut by a
// test for the first cell at every position (8192 rows of 1024: 75 -> 65 us).
// ------------------------------------------------------------------------------------
template <int KM, int CPL, bool MW, bool AL>
__device__ __forceinline__ void xline_body(const PassParams &p, int j, int rec, int W, double *sU, double *s2,
                                           double *bnd)
{
    const int nx = p.nx, ny = p.ny;
    const int lane = threadIdx.x & 63;
    const int wv = MW ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0; // wave of the line
    const int w0 = 64 * CPL * wv;                                             // its first position
    const int sh = 64 * CPL * W - nx;
    double *const priv = s2 + (size_t)wv * ln_priv(CPL);
    const double ka = p.ka;
    const double *uc = p.u + (size_t)j * nx;
    const double *un = p.u + (size_t)crefl(j - 1, ny) * nx;
    const double *us = p.u + (size_t)crefl(j + 1, ny) * nx;
    const double *wrow = p.in2 + (size_t)j * nx;
    // stage w through the second row (each lane then takes its own CPL positions), u(j) and
    // u(j-1) + u(j+1); positions before the line repeat its first cells
    double wr[CPL];
    {
        double vu[CPL], vx[CPL], vw[CPL], eu = 0.0, ex = 0.0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const int q = w0 + lane + 64 * k - sh;
            vw[k] = wrow[max(q, 0)];
            const int c = q >= 0 ? q : -1 - max(q, -2);
            vu[k] = uc[c];
            vx[k] = us[c] + un[c];
        }
        // the two positions on each side of the line's span: w = -2, -1 and 64 W CPL + 0, 1
        const int we = lane < 2 ? lane - 2 : 64 * CPL * W + lane - 2;
        const bool ends = wv == 0 && lane < 4;
        if (ends) {
            const int c = crefl(max(we - sh, -2), nx);
            eu = uc[c];
            ex = us[c] + un[c];
        }
        if (stands_down(p, false)) return;
#pragma unroll
        for (int k = 0; k < CPL; ++k) s2[ln_at<CPL>(w0 + lane + 64 * k)] = vw[k];
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < CPL; ++k) wr[k] = s2[ln_at<CPL>(w0 + CPL * lane) + k];
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            sU[ln_at<CPL>(w0 + lane + 64 * k)] = vu[k];
            s2[ln_at<CPL>(w0 + lane + 64 * k)] = vx[k];
        }
        if (ends) {
            sU[ln_at<CPL>(we)] = eu;
            s2[ln_at<CPL>(we)] = ex;
        }
        if (MW) __syncthreads();
        else wave_lds_sync();
    }
    double fa[CPL], fb[CPL], fz[CPL], fph[CPL], fps[CPL];
    {
        const double *bu = sU + ln_at<CPL>(w0 + CPL * lane), *bx = s2 + ln_at<CPL>(w0 + CPL * lane);
        auto cell = [&](int t) {
            const double uq = bu[ln_off<CPL>(t)];
            return cell_core<KM>(p, uq, __builtin_fma(-4.0, uq, (bu[ln_off<CPL>(t + 1)] + bu[ln_off<CPL>(t - 1)])
                                                                    + bx[ln_off<CPL>(t)]));
        };
        // slot and position of the line's first cell; the last slot holds its end at k = CPL-2, CPL-1
        const int lz = sh / CPL, kz = AL ? 0 : sh % CPL, slot = 64 * wv + lane;
        const bool re = slot == 64 * W - 1;
        CellS c0 = cell(0);
        FaceS fm = face_s<false>(cell(-1), c0, true, ka);
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const CellS cp = cell(k + 1);
            const FaceS fp = face_s<false>(c0, cp, !(k == CPL - 1 && re), ka);
            if (k == kz && slot == lz) fm = FaceS{0.0, 0.0, 0.0, 0.0}; // no flux through x = 0
            Band B = xr_band(fm, fp);
            if (k >= CPL - 2 && re) fold_right(B, CPL - 1 - k);
            if (k == kz && slot == lz) fold_left(B, 0);
            if (k == (kz + 1) % CPL && slot == lz + (kz == CPL - 1 ? 1 : 0)) fold_left(B, 1);
            xr_elim<CPL>(k, B, wr[k], fa, fb, fz, fph, fps);
            c0 = cp;
            fm = fp;
        }
    }
    double B0, B1, l1, l2;
    double2 *const xch = reinterpret_cast<double2 *>(priv);
    if constexpr (MW) ln_pairs_mw<CPL>(xch, bnd, lane, wv, W, sh / CPL, fa, fb, fz, fph, fps, B0, B1, l1, l2);
    else ln_pairs<CPL>(xch, lane, (nx + CPL - 1) / CPL, fa, fb, fz, fph, fps, B0, B1, l1, l2);
    {
        // back-substitution from the lane's pair and its left neighbour's; v goes to the wave's space
        double *v2 = priv + (CPL + 1) * lane;
        __asm__ volatile("" ::: "memory");
        double x1 = B0, x2 = B1;
        v2[CPL - 1] = B1;
        v2[CPL - 2] = B0;
#pragma unroll
        for (int k = CPL - 3; k >= 0; --k) {
            const double v = fz[k] + fph[k] * l1 + fps[k] * l2 - fa[k] * x1 - fb[k] * x2;
            v2[k] = v;
            x2 = x1;
            x1 = v;
        }
        wave_lds_sync();
    }
    // output: u_{k+1} = u_k + v, update ratio, flags, mass diagnostic (coalesced)
    double emax = 0.0;
    unsigned flags = 0;
    const bool diag = p.mass != nullptr;
    double ms = 0.0, mc = 0.0, mmin = __builtin_inf();
    double *orow = p.out + (size_t)j * nx;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        const int i = lane + 64 * k, q = w0 + i - sh;
        if (q >= 0) {
            const double v = priv[i + i / CPL], uk = sU[ln_at<CPL>(w0 + i)];
            const double u1 = uk + v;
            emax = fmax(emax, fabs(v) * rcp(fabs(uk)));
            if (!(u1 > 0.0)) flags |= (u1 != u1 || v != v) ? FLAG_NAN : FLAG_NONPOS;
            orow[q] = u1;
            if (diag) {
                two_sum_acc(ms, mc, u1);
                mmin = fmin(mmin, u1);
            }
        }
    }
    const double wm = wave_max(emax);
    const unsigned wf = wave_or(flags);
    if (lane == 0 && p.res != nullptr) {
        unsigned long long *rs = p.res + (size_t)((unsigned)(rec * W + wv) % (unsigned)p.res_spread) * RES_WORDS;
        atomicMax(&rs[RES_EMAX], (unsigned long long)__double_as_longlong(wm));
        if (wf) atomicOr(&rs[RES_FLAGS], (unsigned long long)wf);
    }
    if (diag) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) { // fixed-order butterfly
            comp_add(ms, mc, __shfl_xor(ms, o), __shfl_xor(mc, o));
            mmin = fmin(mmin, __shfl_xor(mmin, o));
        }
        if (lane == 0) {
            double *o = p.mass + 4 * ((size_t)rec * W + wv);
            o[0] = ms;
            o[1] = mc;
            o[2] = mmin;
            o[3] = 0.0;
        }
    }
}

// ------------------------------------------------------------------------------------
// y sweep of the columns i0 .. i0 + LN_COLS - 1 (W waves each). sU: LDS of lny_u2 doubles that holds
// b^n on its way to the lanes, then the u tile, then the waves' exchange records and solutions:
// with a single region the workgroups of a CU fill its registers (8 waves of 16 positions per lane).
// ------------------------------------------------------------------------------------
template <int KM, int CPL, int W>
__device__ __forceinline__ void yline_body(const PassParams &p, int i0, int rec, double *sU, double *bnd)
{
    constexpr bool MW = W > 1;
    constexpr int RB = ln_row(CPL, W), NT = 64 * LN_COLS * W, NP = 64 * CPL * W;
    const int nx = p.nx, ny = p.ny;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = MW ? wave / W : wave, wv = MW ? wave % W : 0; // column and wave of its line
    const int sh = NP - ny, slot = 64 * wv + lane;
    const double ka = p.ka;
    double br[CPL]; // b^n of this lane's positions
    {
        // u: LN_UC columns x (NP + 4) positions, NT / LN_UC positions per round; b^n: LN_COLS
        // columns. All loads of a thread are issued before its first LDS store.
        constexpr int RU = NT / LN_UC, KU = (NP + 4 + RU - 1) / RU, RW = NT / LN_COLS, KW = NP / RW;
        const int cu = tid % LN_UC, ru = tid / LN_UC, cb = tid % LN_COLS, rb = tid / LN_COLS;
        const unsigned gu = (unsigned)crefl(i0 - 2 + cu, nx), gb = (unsigned)min(i0 + cb, nx - 1);
        double vu[KU], vb[KW];
#pragma unroll
        for (int k = 0; k < KU; ++k) {
            const int w = ru + RU * k - 2;
            if (w < NP + 2) vu[k] = p.u[(size_t)crefl(max(w - sh, -2), ny) * nx + gu];
        }
#pragma unroll
        for (int k = 0; k < KW; ++k) vb[k] = p.in2[(size_t)max(rb + RW * k - sh, 0) * nx + gb];
        if (stands_down(p, true)) return;
        if (p.res_clear != nullptr && blockIdx.x == 0)
            for (int e = tid; e < p.res_spread * RES_WORDS; e += NT) p.res_clear[e] = 0ull;
#pragma unroll
        for (int k = 0; k < KW; ++k) sU[cb * RB + ln_at<CPL>(rb + RW * k)] = vb[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < CPL; ++k) br[k] = sU[col * RB + ln_at<CPL>(CPL * slot) + k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KU; ++k) {
            const int w = ru + RU * k - 2;
            if (w < NP + 2) sU[lny_at<CPL>(w) + cu] = vu[k];
        }
    }
    __syncthreads();
    const int gl = i0 + col; // grid column of this wave
    double fa[CPL], fb[CPL], fz[CPL], fph[CPL], fps[CPL];
    double rmax = 0.0;
    unsigned flags = 0;
    {
        const double *bu = sU + lny_at<CPL>(CPL * slot) + 2 + col;
        // cell quantities at column offset dc, position t; the neighbouring columns' cells enter the
        // residual's x faces only (their derivatives are not formed)
        auto cell = [&](int dc, int t) {
            const double *b = bu + dc;
            const double uq = b[lny_off<CPL>(t)];
            return cell_core<KM>(p, uq, __builtin_fma(-4.0, uq, (b[lny_off<CPL>(t) + 1] + b[lny_off<CPL>(t) - 1])
                                                                    + (b[lny_off<CPL>(t + 1)] + b[lny_off<CPL>(t - 1)])));
        };
        auto flux = [&](const CellS &L, const CellS &R) {
            return __builtin_fma(L.f0 + R.f0, R.lap - L.lap, (L.f1 + R.f1) * (R.u - L.u));
        };
        const int lz = sh / CPL, kz = sh % CPL;
        const bool re = slot == 64 * W - 1;
        CellS c0 = cell(0, 0);
        FaceS fm = face_s<true>(cell(0, -1), c0, true, ka);
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const CellS cp = cell(0, k + 1);
            const FaceS fp = face_s<true>(c0, cp, !(k == CPL - 1 && re), ka);
            if (k == kz && slot == lz) fm = FaceS{0.0, 0.0, 0.0, 0.0};
            const double Fe = gl < nx - 1 ? flux(c0, cell(1, k)) : 0.0;
            const double Fw = gl > 0 ? flux(cell(-1, k), c0) : 0.0;
            const double D = (Fe - Fw) + (fp.F - fm.F);
            const double G = __builtin_fma(ka, D, c0.u - br[k]);
            if (CPL * slot + k >= sh) {
                rmax = fmax(rmax, fabs(G));
                if (G != G) flags |= FLAG_NAN;
            }
            Band B = xr_band(fm, fp);
            if (k >= CPL - 2 && re) fold_right(B, CPL - 1 - k);
            if (k == kz && slot == lz) fold_left(B, 0);
            if (k == (kz + 1) % CPL && slot == lz + (kz == CPL - 1 ? 1 : 0)) fold_left(B, 1);
            xr_elim<CPL>(k, B, -G, fa, fb, fz, fph, fps);
            c0 = cp;
            fm = fp;
        }
    }
    if (p.res != nullptr) {
        const double wm = wave_max(gl < nx ? rmax : 0.0);
        const unsigned wf = wave_or(gl < nx ? flags : 0u);
        if (lane == 0) {
            const unsigned copy = (unsigned)(rec * LN_COLS * W + wave) % (unsigned)p.res_spread;
            unsigned long long *rs = p.res + (size_t)copy * RES_WORDS;
            atomicMax(&rs[RES_RMAX], (unsigned long long)__double_as_longlong(wm));
            if (wf) atomicOr(&rs[RES_FLAGS], (unsigned long long)wf);
        }
    }
    // the u tile is consumed (after a barrier): its space holds the waves' exchange records
    // and then their solutions
    double *const priv = sU + wave * ln_priv(CPL);
    double2 *const xch = reinterpret_cast<double2 *>(priv);
    double B0, B1, l1, l2;
    if constexpr (MW) {
        ln_pairs_mw<CPL>(xch, bnd + col * W * LN_BND, lane, wv, W, sh / CPL, fa, fb, fz, fph, fps,
                         B0, B1, l1, l2);
    } else {
        __syncthreads();
        ln_pairs<CPL>(xch, lane, (ny + CPL - 1) / CPL, fa, fb, fz, fph, fps, B0, B1, l1, l2);
    }
    {
        double *v2 = priv + (CPL + 1) * lane;
        __asm__ volatile("" ::: "memory");
        double x1 = B0, x2 = B1;
        v2[CPL - 1] = B1;
        v2[CPL - 2] = B0;
#pragma unroll
        for (int k = CPL - 3; k >= 0; --k) {
            const double v = fz[k] + fph[k] * l1 + fps[k] * l2 - fa[k] * x1 - fb[k] * x2;
            v2[k] = v;
            x2 = x1;
            x1 = v;
        }
    }
    __syncthreads();
    {
        constexpr int RW = NT / LN_COLS, KW = NP / RW;
        const int cb = tid % LN_COLS, rb = tid / LN_COLS;
        if (i0 + cb < nx) {
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                const int w = rb + RW * k, q = w - sh, i = w % (64 * CPL);
                if (q >= 0) p.out[(size_t)q * nx + i0 + cb] = sU[(cb * W + w / (64 * CPL)) * ln_priv(CPL) + i + i / CPL];
            }
        }
    }
}

} // namespace tf
