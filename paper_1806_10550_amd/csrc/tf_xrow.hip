// Whole-row x sweep (gfx950, FP64): the second half of one ADI-Newton iteration
// (Lam, Cummings & Kondic, arXiv:1806.10550, eqs. JacobianSystem2-3, NewtonError),
//   (I + c J_x(u_k)) v = w   per grid row,   u_{k+1} = u_k + v,   e = max|v/u_k|,
// in ONE kernel that reads u_k and w once and writes u_{k+1} once.
//
// A workgroup owns whole rows (one row of up to 8192 cells, or several shorter rows).
// Each lane owns a sub-segment of at most XR_CPL consecutive cells of its row:
//   phase 1  stage u_k(row) and u_k(row-1) + u_k(row+1) in LDS; every lane assembles the
//            five bands of its sub-segment and eliminates it with its outer unknowns (the
//            two cells before and the two after) kept symbolic -> a relation record
//            expressing its first and last cell pairs in those outer unknowns;
//   tree     the records of a row are merged pairwise in LDS (log2 levels): merging two
//            neighbouring blocks eliminates the two cell pairs at their junction; the
//            junction's solution, affine in the merged block's outer pairs, stays in the
//            right child's slot. Walking back down gives every sub-segment its outer pairs;
//   back-substitution  every lane finishes its sub-segment from the factors of phase 1
//            (held in registers; one of the five arrays waits in the u row's LDS while
//            the tree runs) and its outer pairs;
//   output   v through LDS, u_{k+1} = u_k + v, max|v/u_k|, h <= 0 / NaN flags and the
//            mass diagnostic of u_{k+1} in one coalesced store loop.
// No band, factor or interface record goes to HBM: 24 algorithmic bytes per cell (u_k is
// read twice, the second time for the update, mostly from L2).
#include "tf_line.h"

namespace tf {

// ---- record algebra of the row tree ---------------------------------------------------
// A block [a, e] of sub-segments has the record
//   T_a = t + Tl Bo + Tr To,   B_e = b + Bl Bo + Br To
// with Bo = B_{a-1} (the last pair before the block) and To = T_{e+1} (the first pair after
// it); a leaf record is the relation record (Rel) of one sub-segment. Records live in LDS
// as structure of arrays: field f of slot s at rec[f * S + s] (the Rel order T[0][0..4],
// T[1][0..4], B[0][0..4], B[1][0..4]).
__device__ __forceinline__ void rec_load(const double *rec, int S, int s, Rel &R)
{
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            R.T[i][j] = rec[(i * 5 + j) * S + s];
            R.B[i][j] = rec[(10 + i * 5 + j) * S + s];
        }
}
__device__ __forceinline__ M2 madd(const M2 &x, const M2 &y) { return {x.a + y.a, x.b + y.b, x.c + y.c, x.d + y.d}; }
// Merge of the blocks in slots a (left, [a, m]) and c = m+1 (right, [c, e]): the junction
// pairs Bm = B_m and Tm = T_c solve
//   Bm = bL + BlL Bo + BrL Tm,   Tm = tR + TlR Bm + TrR To,
// so with K = (I - BrL TlR)^-1:  Bm = K (bL + BrL tR) + K BlL Bo + K BrL TrR To and
// Tm = tR + TlR Bm + TrR To. The merged record goes to slot a; the junction forms (Bm in
// the B fields, Tm in the T fields) to slot c.
__device__ __forceinline__ M2 ld_m2(const double *rec, int S, int s, int f) // fields f, f+1, f+5, f+6
{
    return {rec[f * S + s], rec[(f + 1) * S + s], rec[(f + 5) * S + s], rec[(f + 6) * S + s]};
}
__device__ __forceinline__ void st_form(double *rec, int S, int s, int f0, double c0, double c1, const M2 &L,
                                        const M2 &Rr) // fields f0 .. f0 + 9 (one pair form)
{
    double *r = rec + s;
    r[(f0 + 0) * S] = c0; r[(f0 + 1) * S] = L.a; r[(f0 + 2) * S] = L.b; r[(f0 + 3) * S] = Rr.a; r[(f0 + 4) * S] = Rr.b;
    r[(f0 + 5) * S] = c1; r[(f0 + 6) * S] = L.c; r[(f0 + 7) * S] = L.d; r[(f0 + 8) * S] = Rr.c; r[(f0 + 9) * S] = Rr.d;
}
__device__ __forceinline__ void rec_merge(double *rec, int S, int a, int c)
{
    // junction: B fields of slot a (left) and T fields of slot c (right)
    const M2 BrL = ld_m2(rec, S, a, 13), TlR = ld_m2(rec, S, c, 1);
    const double bL0 = rec[10 * S + a], bL1 = rec[15 * S + a], tR0 = rec[0 * S + c], tR1 = rec[5 * S + c];
    const M2 K = inv_i_minus(mul(BrL, TlR));
    const double s0 = bL0 + BrL.a * tR0 + BrL.b * tR1;
    const double s1 = bL1 + BrL.c * tR0 + BrL.d * tR1;
    const double b0 = K.a * s0 + K.b * s1, b1 = K.c * s0 + K.d * s1;
    const M2 TrR = ld_m2(rec, S, c, 3), BlL = ld_m2(rec, S, a, 11);
    const M2 b_l = mul(K, BlL), b_r = mul(K, mul(BrL, TrR));
    const double t0 = tR0 + TlR.a * b0 + TlR.b * b1, t1 = tR1 + TlR.c * b0 + TlR.d * b1;
    const M2 t_l = mul(TlR, b_l), t_r = madd(mul(TlR, b_r), TrR);
    // merged record: T from slot a's T fields, B from slot c's B fields
    {
        const M2 TlL = ld_m2(rec, S, a, 1), TrL = ld_m2(rec, S, a, 3);
        const double tL0 = rec[0 * S + a], tL1 = rec[5 * S + a];
        st_form(rec, S, a, 0, tL0 + TrL.a * t0 + TrL.b * t1, tL1 + TrL.c * t0 + TrL.d * t1, madd(TlL, mul(TrL, t_l)),
                mul(TrL, t_r));
    }
    {
        const M2 BlR = ld_m2(rec, S, c, 11), BrR = ld_m2(rec, S, c, 13);
        const double bR0 = rec[10 * S + c], bR1 = rec[15 * S + c];
        st_form(rec, S, a, 10, bR0 + BlR.a * b0 + BlR.b * b1, bR1 + BlR.c * b0 + BlR.d * b1, mul(BlR, b_l),
                madd(mul(BlR, b_r), BrR));
    }
    // junction forms: Tm in the T fields, Bm in the B fields of slot c
    st_form(rec, S, c, 0, t0, t1, t_l, t_r);
    st_form(rec, S, c, 10, b0, b1, b_l, b_r);
}

// Down the tree: the block in slot a with outer pairs (Bo, To) in rec[0..3][a] splits at
// c; the junction forms in slot c give Bm and Tm, and the children get (Bo, Tm) in slot a
// and (Bm, To) in slot c (fields 0..3 of a slot hold its outer pairs on the way down).
__device__ __forceinline__ void rec_split(double *rec, int S, int a, int c)
{
    const double bo0 = rec[0 * S + a], bo1 = rec[1 * S + a], to0 = rec[2 * S + a], to1 = rec[3 * S + a];
    Rel J;
    rec_load(rec, S, c, J);
    const double tm0 = J.T[0][0] + J.T[0][1] * bo0 + J.T[0][2] * bo1 + J.T[0][3] * to0 + J.T[0][4] * to1;
    const double tm1 = J.T[1][0] + J.T[1][1] * bo0 + J.T[1][2] * bo1 + J.T[1][3] * to0 + J.T[1][4] * to1;
    const double bm0 = J.B[0][0] + J.B[0][1] * bo0 + J.B[0][2] * bo1 + J.B[0][3] * to0 + J.B[0][4] * to1;
    const double bm1 = J.B[1][0] + J.B[1][1] * bo0 + J.B[1][2] * bo1 + J.B[1][3] * to0 + J.B[1][4] * to1;
    rec[2 * S + a] = tm0;
    rec[3 * S + a] = tm1;
    rec[0 * S + c] = bm0;
    rec[1 * S + c] = bm1;
    rec[2 * S + c] = to0;
    rec[3 * S + c] = to1;
}

// The relation record of slot s from the factors of its sub-segment (Rel layout, field f at
// rec[f * S + s]). Top pair: x_{p0} = sum_k g_k Z_k, x_{p0+1} = sum_k h_k Z_k with g, h the
// first two rows of the inverse of the unit upper factor (g_k = -al_{k-1} g_{k-1} -
// be_{k-2} g_{k-2}) and Z_k = z_k + ph_k l1 + ps_k l2 the eliminated right-hand sides;
// bottom pair x_{e-1} = Z_{e-1} - al1 r1 - be1 r2, x_{e-2} = Z_{e-2} - al2 x_{e-1} - be2 r1.
template <int CPL>
__device__ __forceinline__ void xr_record(double *rec, int S, int s, const double (&fa)[CPL], const double (&fb)[CPL],
                                          const double (&fz)[CPL], const double (&fph)[CPL], const double (&fps)[CPL])
{
    double g1 = 0.0, g2 = 0.0, h1 = 0.0, h2 = 0.0;
    double sgz = 0.0, sgph = 0.0, sgps = 0.0, shz = 0.0, shph = 0.0, shps = 0.0;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        const double gg = k == 0 ? 1.0 : -fa[k - 1] * g1 - (k >= 2 ? fb[k - 2] : 0.0) * g2;
        const double hh = k == 1 ? 1.0 : (k == 0 ? 0.0 : -fa[k - 1] * h1 - (k >= 2 ? fb[k - 2] : 0.0) * h2);
        sgz += gg * fz[k]; sgph += gg * fph[k]; sgps += gg * fps[k];
        shz += hh * fz[k]; shph += hh * fph[k]; shps += hh * fps[k];
        g2 = g1; g1 = gg; h2 = h1; h1 = hh;
    }
    constexpr int L = CPL - 1;
    double *r = rec + s;
    r[0 * S] = sgz; r[1 * S] = sgph; r[2 * S] = sgps;
    r[3 * S] = -g2 * fb[L - 1] - g1 * fa[L]; r[4 * S] = -g1 * fb[L];
    r[5 * S] = shz; r[6 * S] = shph; r[7 * S] = shps;
    r[8 * S] = -h2 * fb[L - 1] - h1 * fa[L]; r[9 * S] = -h1 * fb[L];
    r[10 * S] = fz[L - 1] - fa[L - 1] * fz[L];
    r[11 * S] = fph[L - 1] - fa[L - 1] * fph[L];
    r[12 * S] = fps[L - 1] - fa[L - 1] * fps[L];
    r[13 * S] = -fb[L - 1] + fa[L - 1] * fa[L];
    r[14 * S] = fa[L - 1] * fb[L];
    r[15 * S] = fz[L]; r[16 * S] = fph[L]; r[17 * S] = fps[L]; r[18 * S] = -fa[L]; r[19 * S] = -fb[L];
}

// Tree over the S records of a row (called by every thread of the workgroup; tr: the
// thread's index within its row group, row_ok: the group holds a row). Level l merges the
// blocks starting at slots b * 2^l and b * 2^l + 2^(l-1); merge b is done by thread b of the
// row group, so only the first waves work at the low levels and wave 0 alone at the top
// (nm <= 64 merges: no workgroup barrier needed there, only ordering of this wave's LDS
// accesses). On return, fields 0..3 of slot s hold the outer pairs of sub-segment s.
__device__ __forceinline__ void xr_tree(double *rec, int S, int tr, bool row_ok)
{
    int levels = 0;
    while ((1 << levels) < S) ++levels;
    auto nmerge = [&](int l) { const int half = 1 << (l - 1); return (S - half + 2 * half - 1) / (2 * half); };
    int lw = levels + 1; // first level done by wave 0 alone
    for (int l = 1; l <= levels; ++l)
        if (nmerge(l) <= 64) { lw = l; break; }
    for (int l = 1; l < lw; ++l) {
        const int half = 1 << (l - 1);
        if (row_ok && tr < nmerge(l)) rec_merge(rec, S, tr * 2 * half, tr * 2 * half + half);
        __syncthreads();
    }
    if (row_ok && tr < 64) {
        for (int l = lw; l <= levels; ++l) {
            const int half = 1 << (l - 1);
            if (tr < nmerge(l)) rec_merge(rec, S, tr * 2 * half, tr * 2 * half + half);
            wave_lds_sync();
        }
        // the row's outer pairs are the ghost-folded ends: zero
        if (tr == 0) { rec[0 * S] = 0.0; rec[1 * S] = 0.0; rec[2 * S] = 0.0; rec[3 * S] = 0.0; }
        wave_lds_sync();
        for (int l = levels; l >= lw; --l) {
            const int half = 1 << (l - 1);
            if (tr < nmerge(l)) rec_split(rec, S, tr * 2 * half, tr * 2 * half + half);
            wave_lds_sync();
        }
    }
    __syncthreads();
    for (int l = lw - 1; l >= 1; --l) {
        const int half = 1 << (l - 1);
        if (row_ok && tr < nmerge(l)) rec_split(rec, S, tr * 2 * half, tr * 2 * half + half);
        __syncthreads();
    }
}

// Back-substitution of slot s from its outer pairs (fields 0..3 of the slot after the tree);
// the coefficient ps of l2 waits in the LDS slot of each position (parked there before the
// tree) and the solution replaces it.
template <int CPL>
__device__ __forceinline__ void xr_backsub(const double *rec, int S, int s, double *slots,
                                           const double (&fa)[CPL], const double (&fb)[CPL], const double (&fz)[CPL],
                                           const double (&fph)[CPL])
{
    // slots: this lane's block (position k at slots[k]); positions before the row are
    // identity rows and solve to zero
    const double l1 = rec[0 * S + s], l2 = rec[1 * S + s];
    double x1 = rec[2 * S + s], x2 = rec[3 * S + s];
#pragma unroll
    for (int k = CPL - 1; k >= 0; --k) {
        double *slot = slots + k;
        const double v = fz[k] + fph[k] * l1 + *slot * l2 - fa[k] * x1 - fb[k] * x2;
        *slot = v;
        x2 = x1;
        x1 = v;
    }
}

// ---- stored-band whole-line solve -------------------------------------------------------
// A x = r (TRANS: A^T x = r) for nl lines of np cells with the five bands a..e of A stored
// per line: line-major (PM false: element (line j, position i) at j np + i; the row solves
// of the adjoint's preconditioner) or position-major (PM true: at i nl + j; the layout of
// tf_penta_solve and of the adjoint's column solves), bands back to back (band k at
// k nl np). MODE 0: out = x; MODE 1: out += x and red[0], red[1] take max|x|, max|out|
// (atomic maxima of the bit patterns). One kernel instead of the partitioned solver's three:
// the elimination, relation records, tree and back-substitution are those of the forward
// whole-row sweep. Row p of A^T is (e_{p-2}, d_{p-1}, c_p, b_{p+1}, a_{p+2}); entries that
// reach outside the line are taken as zero. Padding positions before the line (lane 0, when
// XR_CPL does not divide np) are identity rows with a zero right-hand side, and the first
// real rows have no coupling to them.
template <bool TRANS, bool PM, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_sbline(int nl, int np, const double *bands, const double *rhs, double *out, unsigned long long *red, XRowGeom g,
         int nblocks, const unsigned long long *stop)
{
    if (stop != nullptr && *stop != 0ull) return; // a converged iteration (the whole workgroup leaves)
    __shared__ double lds[xr_lds(4)];
    __shared__ double sRed[4][2];
    constexpr int CPL = XR_CPL;
    const int rb = xcd_tile(blockIdx.x, nblocks);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave / g.W;                       // line group of this wave (uniform)
    const int s = (wave - rg * g.W) * 64 + lane;     // slot (sub-segment) of this lane in its line
    const int nthr = 64 * g.W;
    const int j = rb * g.R + rg;
    const bool row_ok = rg < g.R && j < nl;
    double *const sV = lds + (size_t)rg * (g.pu + g.p2); // parked factor, then the solution
    double *const rec = sV + g.pu;
    const int S = g.S;
    const bool act = row_ok && s < S;
    const int p0 = np - CPL * (S - s);
    const size_t N = (size_t)nl * np;
    // element (position q, this line), 0 <= q < np
    auto at = [&](int q) -> size_t { return PM ? (size_t)q * nl + j : (size_t)j * np + q; };
    double fa[CPL], fb[CPL], fz[CPL], fph[CPL], fps[CPL];
    if (act) {
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const int q = p0 + k;
            const bool real = q >= 0;
            // every load stays inside the line (clamped position); entries outside it are
            // selected away afterwards
            double va, vb, vc, vd, ve;
            if (TRANS) {
                va = bands[4 * N + at(max(q - 2, 0))];
                vb = bands[3 * N + at(max(q - 1, 0))];
                vc = bands[2 * N + at(max(q, 0))];
                vd = bands[N + at(min(max(q + 1, 0), np - 1))];
                ve = bands[at(min(max(q + 2, 0), np - 1))];
            } else {
                const size_t o = at(max(q, 0));
                va = bands[o]; vb = bands[N + o]; vc = bands[2 * N + o]; vd = bands[3 * N + o]; ve = bands[4 * N + o];
            }
            const double rr = rhs[at(max(q, 0))];
            Band B;
            B.a = q >= 2 ? va : 0.0;
            B.b = q >= 1 ? vb : 0.0;
            B.c = real ? vc : 1.0;
            B.d = real && q + 1 < np ? vd : 0.0;
            B.e = real && q + 2 < np ? ve : 0.0;
            xr_elim(k, B, real ? rr : 0.0, fa, fb, fz, fph, fps);
        }
        xr_record(rec, S, s, fa, fb, fz, fph, fps);
#pragma unroll
        for (int k = 0; k < CPL; ++k) sV[xr_base(s) + k] = fps[k];
    }
    __syncthreads();
    xr_tree(rec, S, s, row_ok);
    if (act) xr_backsub(rec, S, s, sV + xr_base(s), fa, fb, fz, fph);
    __syncthreads();
    double xm = 0.0, om = 0.0;
    if (row_ok) {
        for (int i = s; i < np; i += nthr) {
            const double x = sV[xr_at(i + CPL * S - np)];
            const size_t o = at(i);
            if (MODE == 0) {
                out[o] = x;
            } else {
                const double v = out[o] + x;
                out[o] = v;
                xm = max_nan(xm, fabs(x));
                om = max_nan(om, fabs(v));
            }
        }
    }
    if (MODE == 1) {
        const double wx = wave_max_nan(xm), wo = wave_max_nan(om);
        if (lane == 0) { sRed[wave][0] = wx; sRed[wave][1] = wo; }
        __syncthreads();
        if (tid == 0) {
            double a = 0.0, b = 0.0;
            for (int w = 0; w < (int)(blockDim.x >> 6); ++w) { a = max_nan(a, sRed[w][0]); b = max_nan(b, sRed[w][1]); }
            atomicMax(&red[0], (unsigned long long)__double_as_longlong(a));
            atomicMax(&red[1], (unsigned long long)__double_as_longlong(b));
        }
    }
}

bool sbline_supported(int np) { return np <= XR_ROW4_MAX_NX && xrow_supported(np); }

hipError_t launch_sbline(bool trans, bool pm, int mode, int nl, int np, const double *bands, const double *rhs,
                         double *out, unsigned long long *red, hipStream_t s, const unsigned long long *stop)
{
    if (nl < 1 || !sbline_supported(np) || (mode == 1 && red == nullptr) || (!pm && (!trans || mode != 0)))
        return hipErrorInvalidValue;
    const XRowGeom g = xrow_geom(np); // 4-wave workgroups for lines of at most XR_ROW4_MAX_NX cells
    const int nb = (nl + g.R - 1) / g.R;
    const dim3 grid(nb), block(64 * g.W * g.R);
    if (!pm) k_sbline<true, false, 0><<<grid, block, 0, s>>>(nl, np, bands, rhs, out, red, g, nb, stop);
    else if (trans && mode == 0) k_sbline<true, true, 0><<<grid, block, 0, s>>>(nl, np, bands, rhs, out, red, g, nb, stop);
    else if (trans) k_sbline<true, true, 1><<<grid, block, 0, s>>>(nl, np, bands, rhs, out, red, g, nb, stop);
    else if (mode == 0) k_sbline<false, true, 0><<<grid, block, 0, s>>>(nl, np, bands, rhs, out, red, g, nb, stop);
    else k_sbline<false, true, 1><<<grid, block, 0, s>>>(nl, np, bands, rhs, out, red, g, nb, stop);
    return hipGetLastError();
}

} // namespace tf
