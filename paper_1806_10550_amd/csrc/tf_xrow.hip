// Whole-line solves on stored bands (gfx950, FP64): the adjoint's transposed row and column solves
// and a variant of tf_penta_solve. One kernel; the lines lie across the lanes of one to four waves and
// are solved by the core of the forward whole-line sweeps (tf_line.h).
#include "tf_line.h"

namespace tf {

// A x = r (TRANS: A^T x = r) for nl lines of np cells with the five bands a..e of A stored
// per line: line-major (PM false: element (line j, position i) at j np + i; the row solves
// of the adjoint's preconditioner) or position-major (PM true: at i nl + j; the layout of
// tf_penta_solve and of the adjoint's column solves), bands back to back (band k at
// k nl np). MODE 0: out = x; MODE 1: out += x and red[0], red[1] take max|x|, max|out|
// (atomic maxima of the bit patterns). Row p of A^T is (e_{p-2}, d_{p-1}, c_p, b_{p+1}, a_{p+2});
// entries that reach outside the line are taken as zero. Positions before the line (the padding of
// its first lanes) are identity rows with a zero right-hand side, and the first real rows have no
// coupling to them.
//
// A workgroup holds L lines of W waves. The six input arrays reach the lanes
// through LDS with loads that run along the contiguous index (one position of the workgroup's
// lines for the position-major layout), sb_round(CPL) arrays at a time, so that two workgroups of
// one-wave lines fit on a CU. Latency bound at the sizes it is chosen for: 512 lines of 512 cells
// 13.4 us (position-major, MODE 1) and 8.8 us (line-major), where 16 cells per lane, loads
// strided by line and a record tree took 26 and 21.
// Lines of a workgroup: four waves' worth, and for lines of several waves twice that once they fill
// the GPU (wider pieces of each position: 4096 lines of 2048 277 -> 213 us, 512 of 4096 81 -> 69; with few
// lines the smaller workgroups start sooner, 256 of 2048 24 against 31 us).
constexpr int sb_lines(int W, bool many) { return W == 1 ? 4 : (W == 2 ? 2 : 1) * (many ? 2 : 1); }
constexpr int sb_round(int cpl) { return cpl == 4 ? 6 : (cpl == 8 ? 3 : 2); }

template <bool TRANS, bool PM, int MODE, int CPL, int W, int L>
__global__ void __launch_bounds__(64 * W * L) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_sbline(int nl, int np, const double *bands, const double *rhs, double *out, unsigned long long *red, int nblocks,
         const unsigned long long *stop)
{
    if (stop != nullptr && *stop != 0ull) return; // a converged iteration (the whole workgroup leaves)
    constexpr int NW = L * W, NT = 64 * NW, NP = 64 * CPL * W, RB = ln_row(CPL, W), R = sb_round(CPL);
    constexpr int NLDS = R * L * RB > NW * ln_priv(CPL) ? R * L * RB : NW * ln_priv(CPL);
    __shared__ __align__(16) double lds[NLDS];
    __shared__ double bnd[W > 1 ? NW * LN_BND : 1];
    __shared__ double sRed[NW][2];
    const int j0 = xcd_tile(blockIdx.x, nblocks) * L; // first line
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = W > 1 ? wave / W : wave, wv = W > 1 ? wave % W : 0, slot = 64 * wv + lane;
    const int sh = NP - np;
    const size_t N = (size_t)nl * np;
    // element (position q, line j0 + l); lines past the last one repeat it and are not stored
    auto at = [&](int q, int l) -> size_t {
        const int j = min(j0 + l, nl - 1);
        return PM ? (size_t)q * nl + j : (size_t)j * np + q;
    };
    constexpr int K = NP * L / NT; // = CPL elements per thread and array
    auto el = [&](int k, int &w, int &l) { // element k of this thread: position w of line l
        const int e = tid + NT * k;
        if (PM) { l = e % L; w = e / L; }
        else { l = e / NP; w = e % NP; }
    };
    // array t of the solve (a..e, rhs) at this thread's elements, from the stored band and its offset
    auto fetch = [&](int t, double (&x)[K]) {
        constexpr int dq[5] = {-2, -1, 0, 1, 2};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int w, l;
            el(k, w, l);
            const int q = w - sh;
            const int qn = t < 5 ? q + dq[t < 5 ? t : 0] : q;
            const int qc = min(max(TRANS && t < 5 ? qn : q, 0), np - 1);
            const double y = t == 5 ? rhs[at(qc, l)] : bands[(size_t)(TRANS ? 4 - t : t) * N + at(qc, l)];
            if (t == 5) x[k] = q >= 0 ? y : 0.0;
            else if (t == 2) x[k] = q >= 0 ? y : 1.0;
            else x[k] = q >= 0 && qn >= 0 && qn < np ? y : 0.0;
        }
    };
    double v[6][CPL]; // this lane's a..e and right-hand side
    // with few positions per lane every load is issued at once, else one round at a time
    constexpr int SR = CPL <= 8 ? 6 : R;
    double st[SR][K];
    if (SR == 6)
#pragma unroll
        for (int t = 0; t < SR; ++t) fetch(t, st[t]);
#pragma unroll
    for (int t0 = 0; t0 < 6; t0 += R) {
        if (SR != 6)
#pragma unroll
            for (int t = 0; t < R; ++t) fetch(t0 + t, st[t]);
        if (t0 > 0) __syncthreads();
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                int w, l;
                el(k, w, l);
                lds[(t * L + l) * RB + ln_at<CPL>(w)] = st[(SR == 6 ? t0 : 0) + t][k];
            }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
            for (int k = 0; k < CPL; ++k) v[t0 + t][k] = lds[(t * L + ln) * RB + ln_at<CPL>(CPL * slot) + k];
    }
    // MODE 1: the values to update are on their way while the lines are solved
    double prev[MODE == 1 && CPL <= 8 ? K : 1];
    if (MODE == 1 && CPL <= 8)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int w, l;
            el(k, w, l);
            prev[k] = out[at(max(w - sh, 0), l)];
        }
    double fa[CPL], fb[CPL], fz[CPL], fph[CPL], fps[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k)
        xr_elim<CPL>(k, Band{v[0][k], v[1][k], v[2][k], v[3][k], v[4][k]}, v[5][k], fa, fb, fz, fph, fps);
    // (a barrier frees the staging space:) the waves' exchange records, then their solutions
    double *const priv = lds + wave * ln_priv(CPL);
    double2 *const xch = reinterpret_cast<double2 *>(priv);
    double B0, B1, l1, l2;
    if constexpr (W > 1) {
        ln_pairs_mw<CPL, true>(xch, bnd + ln * W * LN_BND, lane, wv, W, sh / CPL, fa, fb, fz, fph, fps, B0, B1, l1,
                               l2);
    } else {
        __syncthreads();
        ln_pairs<CPL, true>(xch, lane, (np + CPL - 1) / CPL, fa, fb, fz, fph, fps, B0, B1, l1, l2);
    }
    {
        double *v2 = priv + (CPL + 1) * lane;
        __asm__ volatile("" ::: "memory");
        double x1 = B0, x2 = B1;
        v2[CPL - 1] = B1;
        v2[CPL - 2] = B0;
#pragma unroll
        for (int k = CPL - 3; k >= 0; --k) {
            const double x = fz[k] + fph[k] * l1 + fps[k] * l2 - fa[k] * x1 - fb[k] * x2;
            v2[k] = x;
            x2 = x1;
            x1 = x;
        }
    }
    __syncthreads();
    double xm = 0.0, om = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int w, l;
        el(k, w, l);
        const int q = w - sh, i = w % (64 * CPL);
        if (q >= 0 && j0 + l < nl) {
            const double x = lds[(l * W + w / (64 * CPL)) * ln_priv(CPL) + i + i / CPL];
            const size_t o = at(q, l);
            if (MODE == 0) {
                out[o] = x;
            } else {
                const double y = (CPL <= 8 ? prev[CPL <= 8 ? k : 0] : out[o]) + x;
                out[o] = y;
                xm = max_nan(xm, fabs(x));
                om = max_nan(om, fabs(y));
            }
        }
    }
    if (MODE == 1) {
        const double wx = wave_max_nan(xm), wo = wave_max_nan(om);
        if (lane == 0) { sRed[wave][0] = wx; sRed[wave][1] = wo; }
        __syncthreads();
        if (tid == 0) {
            double a = 0.0, b = 0.0;
            for (int w = 0; w < NW; ++w) { a = max_nan(a, sRed[w][0]); b = max_nan(b, sRed[w][1]); }
            atomicMax(&red[0], (unsigned long long)__double_as_longlong(a));
            atomicMax(&red[1], (unsigned long long)__double_as_longlong(b));
        }
    }
}

bool sbline_supported(int np) { return np >= 4 && np <= XR_ROW4_MAX_NX; }

template <bool TRANS, bool PM, int MODE>
static hipError_t launch_sb(int nl, int np, const double *bands, const double *rhs, double *out,
                            unsigned long long *red, hipStream_t s, const unsigned long long *stop)
{
    // (not the forward sweeps' finer choice: these kernels are latency bound)
    const LineGeom g = {np <= 256 ? 4 : (np <= 512 ? 8 : 16), (np + 1023) / 1024};
    const bool many = (long long)nl * g.W > 1024;
    const int L = sb_lines(g.W, many), nb = (nl + L - 1) / L;
    const dim3 grid(nb), block(64 * L * g.W);
#define TF_SB(C, V, M) \
    case 1000 * V + 10 * C + M: \
        k_sbline<TRANS, PM, MODE, C, V, sb_lines(V, M)><<<grid, block, 0, s>>>(nl, np, bands, rhs, out, red, nb, stop); \
        break
    switch (1000 * g.W + 10 * g.cpl + (g.W > 1 && many)) {
    TF_SB(4, 1, 0); TF_SB(8, 1, 0); TF_SB(16, 1, 0);
    TF_SB(16, 2, 0); TF_SB(16, 3, 0); TF_SB(16, 4, 0); TF_SB(16, 2, 1); TF_SB(16, 3, 1); TF_SB(16, 4, 1);
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_sbline(bool trans, bool pm, int mode, int nl, int np, const double *bands, const double *rhs,
                         double *out, unsigned long long *red, hipStream_t s, const unsigned long long *stop)
{
    if (nl < 1 || !sbline_supported(np) || (mode == 1 && red == nullptr) || (!pm && (!trans || mode != 0)))
        return hipErrorInvalidValue;
    if (!pm) return launch_sb<true, false, 0>(nl, np, bands, rhs, out, red, s, stop);
    if (trans) return mode == 0 ? launch_sb<true, true, 0>(nl, np, bands, rhs, out, red, s, stop)
                                : launch_sb<true, true, 1>(nl, np, bands, rhs, out, red, s, stop);
    return mode == 0 ? launch_sb<false, true, 0>(nl, np, bands, rhs, out, red, s, stop)
                     : launch_sb<false, true, 1>(nl, np, bands, rhs, out, red, s, stop);
}

} // namespace tf
