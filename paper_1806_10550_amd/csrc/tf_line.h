// Core of the whole-line solvers in which one wave holds one line (tf_line.hip): the LU step of a
// lane's sub-segment, the reduced system of the lanes' last pairs, its parallel cyclic reduction
// across the wave and the back-substitution.
//
// Lane s owns CPL consecutive positions; its last two are the separator pair B_s. The forward
// elimination of the sub-segment carries its two left outer unknowns l = B_{s-1} symbolically
// (x_k = z_k + ph_k l1 + ps_k l2 - al_k x_{k+1} - be_k x_{k+2}). Two relations follow:
//   bottom pair   B_s = b + Bl B_{s-1} + Br T_{s+1}      (T: the first pair of a lane)
//   top pair      T_s = t + Tl B_{s-1} + Tb B_s          (interior back-substituted from B_s)
// With T_{s+1} from the right neighbour the lanes' pairs satisfy the block tridiagonal system
//   B_s = r_s + A_s B_{s-1} + C_s B_{s+1},
// which log2(64) steps of cyclic reduction decouple: no tree to walk back down, every lane works in
// every step, ten doubles per lane are exchanged and no barrier is needed inside the wave.
#pragma once

#include "tf_sweep.h"

namespace tf {

// Orders this wave's LDS writes before its later LDS reads by other lanes of the same wave:
// the wave's LDS operations complete in issue order once the counter drains, and the empty
// asm statement keeps the compiler from moving memory accesses across the point.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0)
    __asm__ volatile("" ::: "memory");
}

// Bands of row p of I + c J from the faces p-1/2 (fm) and p+1/2 (fp).
struct Band {
    double a, b, c, d, e;
};
__device__ __forceinline__ Band xr_band(const FaceS &fm, const FaceS &fp)
{
    Band B;
    B.a = fm.kA;
    B.b = __builtin_fma(-3.0, fm.kA, -fp.kA) - fm.P;
    B.c = __builtin_fma(3.0, fp.kA + fm.kA, 1.0) + (fp.P - fm.Q);
    B.d = __builtin_fma(-3.0, fp.kA, fp.Q) - fm.kA;
    B.e = fp.kA;
    return B;
}
// Ghost columns folded back (even reflection of the perturbation) at the line ends.
__device__ __forceinline__ void fold_left(Band &B, int pos) // pos: 0 or 1
{
    if (pos == 0) { B.c += B.b; B.d += B.a; B.b = 0.0; B.a = 0.0; }
    else { B.b += B.a; B.a = 0.0; }
}
__device__ __forceinline__ void fold_right(Band &B, int pos) // pos: n-1 (0) or n-2 (1)
{
    if (pos == 0) { B.c += B.d; B.b += B.e; B.d = 0.0; B.e = 0.0; }
    else { B.d += B.e; B.e = 0.0; }
}

// LU step at position k of a lane's sub-segment with the outer unknowns l1 = x_{p0-2},
// l2 = x_{p0-1} kept symbolic (z: constant part, ph: coefficient of l1, ps: of l2); the
// factors of every position stay in the arrays for the back-substitution. The pivots' reciprocals are good to the
// last bits: with one refinement (rcp_pivot, as in the tiles) the lanes' pairs lose twice the tiles' digits on stiff
// films (largest error of an iterate at dt = 50, 128^2: tiles 5.0e-13, one refinement 9.9e-13, two 3.4e-13; 512 x 300
// at dt = 100: 5.1e-9, 5.3e-9, 1.5e-9) for up to 2 % of a sweep (y + x of 1637^2 NLC 127.3 -> 129.3 us, of 2048^2 109.5 -> 111.3; a call at 128^2
// 28.2 -> 28.3, at 8192^2 1563 -> 1566).
template <int CPL>
__device__ __forceinline__ void xr_elim(int k, const Band &B, double rhs, double (&fa)[CPL], double (&fb)[CPL],
                                        double (&fz)[CPL], double (&fph)[CPL], double (&fps)[CPL])
{
    const double al2 = k >= 2 ? fa[k - 2] : 0.0, be2 = k >= 2 ? fb[k - 2] : 0.0;
    const double al1 = k >= 1 ? fa[k - 1] : 0.0, be1 = k >= 1 ? fb[k - 1] : 0.0;
    const double z2 = k >= 2 ? fz[k - 2] : 0.0, z1 = k >= 1 ? fz[k - 1] : 0.0;
    // rows p0-2 and p0-1 stand for the outer unknowns l1 (ph = 1) and l2 (ps = 1)
    const double ph2 = k >= 2 ? fph[k - 2] : (k == 0 ? 1.0 : 0.0), ph1 = k >= 1 ? fph[k - 1] : 0.0;
    const double ps2 = k >= 2 ? fps[k - 2] : (k == 1 ? 1.0 : 0.0), ps1 = k >= 1 ? fps[k - 1] : 1.0;
    const double gam = B.b - B.a * al2;
    const double mu = B.c - B.a * be2 - gam * al1;
    const double rm = rcp(mu);
    fa[k] = (B.d - gam * be1) * rm;
    fb[k] = B.e * rm;
    fz[k] = (rhs - B.a * z2 - gam * z1) * rm;
    fph[k] = (-B.a * ph2 - gam * ph1) * rm;
    fps[k] = (-B.a * ps2 - gam * ps1) * rm;
}

__device__ __forceinline__ M2 m2_ma(const M2 &x, const M2 &y, const M2 &z) // x y + z
{
    return {__builtin_fma(x.a, y.a, __builtin_fma(x.b, y.c, z.a)), __builtin_fma(x.a, y.b, __builtin_fma(x.b, y.d, z.b)),
            __builtin_fma(x.c, y.a, __builtin_fma(x.d, y.c, z.c)), __builtin_fma(x.c, y.b, __builtin_fma(x.d, y.d, z.d))};
}

// Exchange records of a wave: pair f (0..4) of lane s at xch[LN_XS f + s]; 16-byte accesses, a
// wave's lanes contiguous. Slots 64 and 65 hold the records of the pairs outside a wave that is
// one of several on its line (see ln_pairs_mw).
__device__ __forceinline__ void ln_put(double2 *xch, int s, const M2 &A, const M2 &C, double r0, double r1)
{
    xch[s] = make_double2(A.a, A.b);
    xch[LN_XS + s] = make_double2(A.c, A.d);
    xch[2 * LN_XS + s] = make_double2(C.a, C.b);
    xch[3 * LN_XS + s] = make_double2(C.c, C.d);
    xch[4 * LN_XS + s] = make_double2(r0, r1);
}
__device__ __forceinline__ void ln_get(const double2 *xch, int s, M2 &A, M2 &C, double &r0, double &r1)
{
    const double2 v0 = xch[s], v1 = xch[LN_XS + s], v2 = xch[2 * LN_XS + s], v3 = xch[3 * LN_XS + s],
                  v4 = xch[4 * LN_XS + s];
    A = {v0.x, v0.y, v1.x, v1.y};
    C = {v2.x, v2.y, v3.x, v3.y};
    r0 = v4.x;
    r1 = v4.y;
}
// The same record in ten consecutive doubles.
__device__ __forceinline__ void ln_put1(double *b, const M2 &A, const M2 &C, double r0, double r1)
{
    b[0] = A.a; b[1] = A.b; b[2] = A.c; b[3] = A.d;
    b[4] = C.a; b[5] = C.b; b[6] = C.c; b[7] = C.d;
    b[8] = r0; b[9] = r1;
}
__device__ __forceinline__ void ln_get1(const double *b, M2 &A, M2 &C, double &r0, double &r1)
{
    A = {b[0], b[1], b[2], b[3]};
    C = {b[4], b[5], b[6], b[7]};
    r0 = b[8];
    r1 = b[9];
}

// (A, C, r) with the left neighbour's record (lA, lC, l0, l1) and the right one's substituted:
// one step of cyclic reduction of B = r + A B_left + C B_right.
__device__ __forceinline__ void ln_step(M2 &A, M2 &C, double &r0, double &r1, const double2 *xch, int left, int right)
{
    M2 nA, nC;
    double n0, n1;
    ln_get(xch, left, nA, nC, n0, n1);
    M2 D = mul(A, nC);
    const M2 lA = mul(A, nA);
    double s0 = __builtin_fma(A.a, n0, __builtin_fma(A.b, n1, r0));
    double s1 = __builtin_fma(A.c, n0, __builtin_fma(A.d, n1, r1));
    ln_get(xch, right, nA, nC, n0, n1);
    D = m2_ma(C, nA, D);
    s0 = __builtin_fma(C.a, n0, __builtin_fma(C.b, n1, s0));
    s1 = __builtin_fma(C.c, n0, __builtin_fma(C.d, n1, s1));
    const M2 lC = mul(C, nC);
    const M2 K = inv_i_minus(D);
    A = mul(K, lA);
    C = mul(K, lC);
    r0 = K.a * s0 + K.b * s1;
    r1 = K.c * s0 + K.d * s1;
}

// High word of the largest |entry| of a block (its exponent and leading bits); NaN and infinity above all.
__device__ __forceinline__ unsigned hi_word(double x) { return (unsigned)__double2hiint(x) & 0x7fffffffu; }
__device__ __forceinline__ unsigned ln_word(const M2 &x)
{
    return max(max(hi_word(x.a), hi_word(x.b)), max(hi_word(x.c), hi_word(x.d)));
}
constexpr unsigned LN_DECOUPLED = (1023u - 100u) << 20; // 2^-100
// Couplings from which a reduction is not trusted: 16. While the matrix is definite they stay below about 8,
// and the reduction is as exact as an elimination. Once the film's growing modes make I + c J indefinite they
// pass 1e2 to 1e6 in its steps and the (I - D)^-1 lose as many digits (lines of 777 cells at dt = 1000, worst
// of 200: 6e-4 of the solution where elimination in order keeps 1e-7); such lines are solved again in order
// (ln_in_order). 0.2 <= dt <= 50: no line of a noise film, dt = 70 a tenth to a half, dt >= 100 all.
constexpr unsigned LN_GROWN = (1023u + 4u) << 20;

// Whether the wave's couplings (ma, mc: ln_word of A and C, 0 where they reach no lane of the wave) are all below
// 2^-100. They square with every step of the reduction (for I + c J they fall like exp(-distance / (4 c)^(1/4)),
// distance in cells), and an update is compared with u > 0 only in the sum u + v: below 2^-100 of the largest one
// nothing of the rest of the line reaches it. NaN and infinity, in the right-hand side r too, count as coupled:
// they spread over the line as in an elimination.
__device__ __forceinline__ bool ln_decoupled(unsigned ma, unsigned mc, double r0, double r1)
{
    return __all(max(hi_word(r0), hi_word(r1)) < 0x7ff00000u && max(ma, mc) < LN_DECOUPLED);
}

// Value of lane s (uniform over the wave).
__device__ __forceinline__ double ln_bcast(double x, int s)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)b, s), hi = __builtin_amdgcn_readlane((int)(b >> 32), s);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// One chain of equations in order over the records at xch[at(0)] .. xch[at(n - 1)], B_i = r + A B_{i-1} + C B_{i+1}: each
// is left as B_i = r + A (what lies before the first) + C (what lies beyond the last); OUTER false: there is nothing
// there and A is not formed. Every lane carries a recurrence (its own chain's: at depends on the lane), `put` the
// one that writes; the records stay in the exchange space, so that the path takes few registers from the usual one.
template <bool OUTER, class At>
__device__ __forceinline__ void ln_chain(double2 *xch, int n, bool put, At at)
{
    wave_lds_sync();
    M2 a, c;
    double q0, q1;
    ln_get(xch, at(0), a, c, q0, q1);
#pragma unroll 1
    for (int i = 1; i < n; ++i) {
        M2 eA, eC;
        double e0, e1;
        ln_get(xch, at(i), eA, eC, e0, e1);
        const M2 K = inv_i_minus(mul(eA, c));
        const double s0 = __builtin_fma(eA.a, q0, __builtin_fma(eA.b, q1, e0));
        const double s1 = __builtin_fma(eA.c, q0, __builtin_fma(eA.d, q1, e1));
        q0 = K.a * s0 + K.b * s1;
        q1 = K.c * s0 + K.d * s1;
        if (OUTER) a = mul(K, mul(eA, a));
        c = mul(K, eC);
        __asm__ volatile("" ::: "memory"); // (read by every lane of the chain before it is written)
        if (put) ln_put(xch, at(i), a, c, q0, q1);
    }
#pragma unroll 1
    for (int i = n - 2; i >= 0; --i) {
        M2 eA, eC;
        double e0, e1;
        __asm__ volatile("" ::: "memory");
        ln_get(xch, at(i), eA, eC, e0, e1);
        const double s0 = __builtin_fma(eC.a, q0, __builtin_fma(eC.b, q1, e0));
        q1 = __builtin_fma(eC.c, q0, __builtin_fma(eC.d, q1, e1));
        q0 = s0;
        if (OUTER) a = m2_ma(eC, a, eA);
        c = mul(eC, c);
        __asm__ volatile("" ::: "memory");
        if (put) ln_put(xch, at(i), a, c, q0, q1);
    }
    wave_lds_sync();
}

// The equations of lanes 0 .. 62 by elimination in order, for waves whose couplings grow: afterwards B_s = r + A L + C G
// with L what lies before lane 0 and G the pair of lane 63, which keeps its equation. Lanes before `first` hold no part
// of the line. In two levels of eight, so that the serial length is a fifth of the wave's: the seven lanes between
// two separators (lanes 7, 15, .. 55) in terms of them, all groups at once, then the separators in terms of L and G
// (one iteration of such a film, polymer at dt = 0.2, 2048^2: lane after lane 357 us, this 205, the reduction alone 154;
// 512^2: 89, 54, 40; the tile passes take 195 and 78). No digit lost against lane after lane beyond the spread of films.
__device__ __forceinline__ void ln_in_order(double2 *xch, int lane, int first, M2 &A, M2 &C, double &r0, double &r1)
{
    const M2 zero = {0.0, 0.0, 0.0, 0.0};
    const int g8 = lane & ~7;
    if (lane < first) {
        A = C = zero;
        r0 = r1 = 0.0;
    }
    __asm__ volatile("" ::: "memory");
    ln_put(xch, lane, A, C, r0, r1);
    if (lane < 2) {
        const double i = lane == 0 ? 1.0 : 0.0;
        ln_put(xch, 64 + lane, M2{i, 0.0, 0.0, i}, M2{1.0 - i, 0.0, 0.0, 1.0 - i}, 0.0, 0.0);
    }
    ln_chain<true>(xch, 7, (lane & 7) == 0, [&](int i) { return g8 + i; });
    // a separator's equation with its two neighbours' in terms of the separators (own records are read again rather
    // than held in registers meanwhile)
    if ((lane & 7) == 7 && lane < 63) {
        ln_get(xch, lane, A, C, r0, r1);
        ln_step(A, C, r0, r1, xch, lane - 1, lane + 1);
        ln_put(xch, lane, A, C, r0, r1);
    }
    ln_chain<true>(xch, 7, lane == 0, [&](int i) { return 8 * i + 7; });
    ln_get(xch, lane, A, C, r0, r1);
    if ((lane & 7) != 7) {
        M2 nA, nC;
        double n0, n1;
        const M2 a = A, c = C;
        ln_get(xch, lane < 8 ? 64 : g8 - 1, nA, nC, n0, n1);
        A = mul(a, nA);
        C = mul(a, nC);
        r0 = __builtin_fma(a.a, n0, __builtin_fma(a.b, n1, r0));
        r1 = __builtin_fma(a.c, n0, __builtin_fma(a.d, n1, r1));
        ln_get(xch, lane >= 56 ? 65 : g8 + 7, nA, nC, n0, n1);
        A = m2_ma(c, nA, A);
        C = m2_ma(c, nC, C);
        r0 = __builtin_fma(c.a, n0, __builtin_fma(c.b, n1, r0));
        r1 = __builtin_fma(c.c, n0, __builtin_fma(c.d, n1, r1));
    }
}

// Top pair record of a lane: x_0 = sum g_k Z_k, x_1 = sum h_k Z_k over the interior (g, h: the
// first two rows of the inverse of the unit upper factor), minus the coupling of the last interior
// rows to the lane's own pair.
template <int CPL>
__device__ __forceinline__ void ln_top(const double (&fa)[CPL], const double (&fb)[CPL], const double (&fz)[CPL],
                                       const double (&fph)[CPL], const double (&fps)[CPL], M2 &Tl, M2 &Tb, double &t0,
                                       double &t1)
{
    constexpr int E = CPL - 3; // last interior position
    double g1 = 0.0, g2 = 0.0, h1 = 0.0, h2 = 0.0;
    t0 = 0.0;
    t1 = 0.0;
    Tl = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k <= E; ++k) {
        const double gg = k == 0 ? 1.0 : -fa[k - 1] * g1 - (k >= 2 ? fb[k - 2] : 0.0) * g2;
        const double hh = k == 1 ? 1.0 : (k == 0 ? 0.0 : -fa[k - 1] * h1 - (k >= 2 ? fb[k - 2] : 0.0) * h2);
        t0 += gg * fz[k]; Tl.a += gg * fph[k]; Tl.b += gg * fps[k];
        t1 += hh * fz[k]; Tl.c += hh * fph[k]; Tl.d += hh * fps[k];
        g2 = g1; g1 = gg; h2 = h1; h1 = hh;
    }
    Tb = {-g2 * fb[E - 1] - g1 * fa[E], -g1 * fb[E], -h2 * fb[E - 1] - h1 * fa[E], -h1 * fb[E]};
}

// Bottom pair of a lane, B_s = b + Bl B_{s-1} + Br T_{s+1}; last: no right neighbour.
template <int CPL>
__device__ __forceinline__ void ln_bottom(const double (&fa)[CPL], const double (&fb)[CPL], const double (&fz)[CPL],
                                          const double (&fph)[CPL], const double (&fps)[CPL], bool last, M2 &Bl, M2 &Br,
                                          double &b0, double &b1)
{
    constexpr int L = CPL - 1;
    Bl = {fph[L - 1] - fa[L - 1] * fph[L], fps[L - 1] - fa[L - 1] * fps[L], fph[L], fps[L]};
    Br = {last ? 0.0 : -fb[L - 1] + fa[L - 1] * fa[L], last ? 0.0 : fa[L - 1] * fb[L], last ? 0.0 : -fa[L],
          last ? 0.0 : -fb[L]};
    b0 = fz[L - 1] - fa[L - 1] * fz[L];
    b1 = fz[L];
}

// Equation of a lane's pair, B_s = r + A B_{s-1} + C B_{s+1}, from its factors and the right
// neighbour's top pair record (nTl, nTb, n0, n1); last: no right neighbour.
template <int CPL>
__device__ __forceinline__ void ln_equation(const double (&fa)[CPL], const double (&fb)[CPL], const double (&fz)[CPL],
                                            const double (&fph)[CPL], const double (&fps)[CPL], bool last, const M2 &nTl,
                                            const M2 &nTb, double n0, double n1, M2 &A, M2 &C, double &r0, double &r1)
{
    M2 Bl, Br;
    double b0, b1;
    ln_bottom<CPL>(fa, fb, fz, fph, fps, last, Bl, Br, b0, b1);
    const M2 K = inv_i_minus(mul(Br, nTl));
    const double s0 = __builtin_fma(Br.a, n0, __builtin_fma(Br.b, n1, b0));
    const double s1 = __builtin_fma(Br.c, n0, __builtin_fma(Br.d, n1, b1));
    r0 = K.a * s0 + K.b * s1;
    r1 = K.c * s0 + K.d * s1;
    A = mul(K, Bl);
    C = mul(K, mul(Br, nTb));
}

// The pair's own equation once more, with the neighbours' solutions: where the couplings are below one the
// rounding errors of the reduction's steps shrink by them (stored-band solves of 248 cells, four a lane:
// 3.1e-16 -> 2.3e-16 of the solution's norm). Not for grown lines, whose errors they would multiply.
__device__ __forceinline__ void ln_again(const M2 &A, const M2 &C, double r0, double r1, double l0, double l1, double n0,
                                         double n1, double &B0, double &B1)
{
    B0 = __builtin_fma(A.a, l0, __builtin_fma(A.b, l1, __builtin_fma(C.a, n0, __builtin_fma(C.b, n1, r0))));
    B1 = __builtin_fma(A.c, l0, __builtin_fma(A.d, l1, __builtin_fma(C.c, n0, __builtin_fma(C.d, n1, r1))));
}

// The factors behind an opaque barrier: what is formed from them again afterwards is not kept in registers
// from the first time.
template <int CPL>
__device__ __forceinline__ void ln_launder(double (&fa)[CPL], double (&fb)[CPL], double (&fz)[CPL], double (&fph)[CPL],
                                           double (&fps)[CPL])
{
#pragma unroll
    for (int k = 0; k < CPL; ++k)
        __asm__ volatile("" : "+v"(fa[k]), "+v"(fb[k]), "+v"(fz[k]), "+v"(fph[k]), "+v"(fps[k]));
}

// Equation (A, C, r) of every lane's pair for a line held by one wave.
template <int CPL>
__device__ __forceinline__ void ln_own(double2 *xch, int lane, const double (&fa)[CPL], const double (&fb)[CPL],
                                       const double (&fz)[CPL], const double (&fph)[CPL], const double (&fps)[CPL],
                                       M2 &A, M2 &C, double &r0, double &r1)
{
    if constexpr (CPL == 2) {
        // the pair is the whole lane: its two relations are the equation (T_{s+1} = B_{s+1})
        ln_bottom<CPL>(fa, fb, fz, fph, fps, lane == 63, A, C, r0, r1);
    } else {
        M2 Tl, Tb;
        double n0, n1;
        ln_top<CPL>(fa, fb, fz, fph, fps, Tl, Tb, n0, n1);
        __asm__ volatile("" ::: "memory"); // earlier reads of this LDS space stay before the writes
        ln_put(xch, lane, Tl, Tb, n0, n1);
        wave_lds_sync();
        ln_get(xch, min(lane + 1, 63), Tl, Tb, n0, n1);
        ln_equation<CPL>(fa, fb, fz, fph, fps, lane == 63, Tl, Tb, n0, n1, A, C, r0, r1);
    }
    if (lane == 0) A = {0.0, 0.0, 0.0, 0.0};
}

// The separator pair (B0, B1) of every lane and its left neighbour's (l1, l2) for a line held by
// one wave. nsub: lanes that hold part of the line (the last nsub of the wave). Every lane calls it.
// FULL: all steps of the reduction (the stored-band solves, whose results are the answer at every
// magnitude); else it ends when the lanes are decoupled, of an ordinary film after three of
// the six steps at 16 positions per lane (x sweep of 8192^2 771 -> 705 us, x + y of 2048^2 111 -> 102). Lanes
// of two or four cells decouple a step early at best, which the test costs (lines of 256; 128^2 when it still had four a lane, a
// call: 29.0 us with all steps, 29.4 with the test): they take all steps.
// Lines whose couplings grow past LN_GROWN are solved in order instead.
template <int CPL, bool FULL = false>
__device__ __forceinline__ void ln_pairs(double2 *xch, int lane, int nsub, double (&fa)[CPL],
                                         double (&fb)[CPL], double (&fz)[CPL], double (&fph)[CPL], double (&fps)[CPL],
                                         double &B0, double &B1, double &l1, double &l2)
{
    M2 A, C;
    double r0, r1;
    ln_own<CPL>(xch, lane, fa, fb, fz, fph, fps, A, C, r0, r1);
    const M2 A0 = A, C0 = C;
    const double q0 = r0, q1 = r1;
    unsigned grown = lane >= 64 - nsub ? max(ln_word(A), ln_word(C)) : 0u;
    for (int d = 1; d < nsub; d <<= 1) {
        __asm__ volatile("" ::: "memory");
        ln_put(xch, lane, A, C, r0, r1);
        wave_lds_sync();
        // past the wave's ends A or C is zero
        ln_step(A, C, r0, r1, xch, max(lane - d, 0), min(lane + d, 63));
        const unsigned ma = ln_word(A), mc = ln_word(C);
        if (lane >= 64 - nsub) grown = max(grown, max(ma, mc));
        if (!FULL && CPL > 4 && ln_decoupled(ma, mc, r0, r1)) break;
    }
    const bool again = __any(grown >= LN_GROWN);
    if (__builtin_expect(again, 0)) {
        if (FULL) {
            A = A0;
            C = C0;
            r0 = q0;
            r1 = q1;
        } else {
            ln_launder<CPL>(fa, fb, fz, fph, fps);
            ln_own<CPL>(xch, lane, fa, fb, fz, fph, fps, A, C, r0, r1);
        }
        ln_in_order(xch, lane, 64 - nsub, A, C, r0, r1);
        // lane 63: B = r + A B_62 and B_62 = r_62 + C_62 B
        const M2 c = {ln_bcast(C.a, 62), ln_bcast(C.b, 62), ln_bcast(C.c, 62), ln_bcast(C.d, 62)}, a = {
            ln_bcast(A.a, 63), ln_bcast(A.b, 63), ln_bcast(A.c, 63), ln_bcast(A.d, 63)};
        const double s0 = ln_bcast(r0, 62), s1 = ln_bcast(r1, 62);
        const M2 K = inv_i_minus(mul(a, c));
        const double t0 = __builtin_fma(a.a, s0, __builtin_fma(a.b, s1, ln_bcast(r0, 63)));
        const double t1 = __builtin_fma(a.c, s0, __builtin_fma(a.d, s1, ln_bcast(r1, 63)));
        const double g0 = K.a * t0 + K.b * t1, g1 = K.c * t0 + K.d * t1;
        r0 = lane == 63 ? g0 : __builtin_fma(C.a, g0, __builtin_fma(C.b, g1, r0));
        r1 = lane == 63 ? g1 : __builtin_fma(C.c, g0, __builtin_fma(C.d, g1, r1));
    }
    B0 = r0;
    B1 = r1;
    if (FULL && !again) ln_again(A0, C0, q0, q1, lane_prev(r0), lane_prev(r1), lane_next(r0), lane_next(r1), B0, B1);
    l1 = lane_prev(B0);
    l2 = lane_prev(B1);
}

// The same for a line held by W consecutive waves (wv: this wave's place on the line, bnd: LN_BND
// doubles per wave of the line, shared by its waves, disjoint from xch; lz: the first lane of the line's first
// wave that holds part of it). The pairs of each wave's lane 63 (G) are the separators of the upper level:
// cyclic reduction inside a wave keeps G_{wv-1} and G_wv symbolic, because a neighbour beyond lane 0 is the
// record "itself" (A = I) and one beyond lane 62 likewise (C = I). Each wave then solves the W equations of
// the G's in its first lanes. A wave whose couplings grow solves its own lanes in order, and likewise the G's; the
// other waves of the line take no notice. Every thread of the workgroup calls it; on entry the factors of every lane are
// done and xch is still in use by other waves (the first barrier below frees it).
template <int CPL, bool FULL = false>
__device__ __forceinline__ void ln_pairs_mw(double2 *xch, double *bnd, int lane, int wv, int W, int lz,
                                            double (&fa)[CPL], double (&fb)[CPL], double (&fz)[CPL],
                                            double (&fph)[CPL], double (&fps)[CPL], double &B0, double &B1, double &l1,
                                            double &l2)
{
    double *const mb = bnd + (size_t)wv * LN_BND;
    M2 A, C;
    double r0, r1;
    // a lane's equation from its own and the next lane's top pair (lane 63: the next wave's lane 0)
    auto equation = [&] {
        M2 Tl, Tb;
        double n0, n1;
        if (lane < 63) ln_get(xch, lane + 1, Tl, Tb, n0, n1);
        else ln_get1(wv + 1 < W ? mb + LN_BND : mb, Tl, Tb, n0, n1);
        ln_equation<CPL>(fa, fb, fz, fph, fps, lane == 63 && wv == W - 1, Tl, Tb, n0, n1, A, C, r0, r1);
        if (lane == 0 && wv == 0) A = {0.0, 0.0, 0.0, 0.0};
    };
    {
        M2 Tl, Tb;
        double n0, n1;
        ln_top<CPL>(fa, fb, fz, fph, fps, Tl, Tb, n0, n1);
        if (lane == 0) ln_put1(mb, Tl, Tb, n0, n1);
        __syncthreads();
        ln_put(xch, lane, Tl, Tb, n0, n1);
    }
    if (lane < 2) {
        const double i = lane == 0 ? 1.0 : 0.0;
        ln_put(xch, 64 + lane, M2{i, 0.0, 0.0, i}, M2{1.0 - i, 0.0, 0.0, 1.0 - i}, 0.0, 0.0);
    }
    wave_lds_sync();
    equation();
    if (lane == 63) ln_put1(mb + 30, A, C, r0, r1);
    const M2 A0 = A, C0 = C;
    const double q0 = r0, q1 = r1;
    const int first = wv == 0 ? lz : 0;
    unsigned grown = lane >= first && lane < 63 ? max(ln_word(A), ln_word(C)) : 0u;
#pragma unroll 1
    for (int d = 1; d < 64; d <<= 1) {
        __asm__ volatile("" ::: "memory");
        ln_put(xch, lane, A, C, r0, r1);
        wave_lds_sync();
        ln_step(A, C, r0, r1, xch, lane >= d ? lane - d : 64, lane + d < 63 ? lane + d : 65);
        // lanes whose A or C reaches a lane of the wave (the others hold G's)
        const bool a = lane >= 2 * d && lane < 63, c = lane + 2 * d < 63;
        const unsigned ma = ln_word(A), mc = ln_word(C);
        if (lane >= first && lane < 63) grown = max(grown, max(ma, mc));
        if (!FULL && ln_decoupled(a ? ma : 0u, c ? mc : 0u, r0, r1)) {
            if (a) A = {0.0, 0.0, 0.0, 0.0};
            if (c) C = {0.0, 0.0, 0.0, 0.0};
            break;
        }
    }
    const bool again = __any(grown >= LN_GROWN);
    if (__builtin_expect(again, 0)) {
        if (FULL) {
            A = A0;
            C = C0;
            r0 = q0;
            r1 = q1;
        } else {
            ln_launder<CPL>(fa, fb, fz, fph, fps);
            M2 Tl, Tb;
            double n0, n1;
            ln_top<CPL>(fa, fb, fz, fph, fps, Tl, Tb, n0, n1);
            __asm__ volatile("" ::: "memory");
            ln_put(xch, lane, Tl, Tb, n0, n1);
            wave_lds_sync();
            equation();
        }
        ln_in_order(xch, lane, first, A, C, r0, r1);
    }
    if (lane == 0) ln_put1(mb + 10, A, C, r0, r1);
    if (lane == 62) ln_put1(mb + 20, A, C, r0, r1);
    __syncthreads();
    // equation of G_i on lane i: lane 63's own with lane 62's and the next wave's lane 0's records
    {
        const int i = min(lane, W - 1);
        M2 gA, gC;
        double g0, g1;
        auto outer = [&] {
            const double *b = bnd + (size_t)i * LN_BND;
            M2 nA, nC;
            double n0, n1;
            ln_get1(b + 30, gA, gC, g0, g1);
            ln_get1(b + 20, nA, nC, n0, n1);
            M2 D = mul(gA, nC);
            const M2 lA = mul(gA, nA);
            double s0 = __builtin_fma(gA.a, n0, __builtin_fma(gA.b, n1, g0));
            double s1 = __builtin_fma(gA.c, n0, __builtin_fma(gA.d, n1, g1));
            ln_get1((i + 1 < W ? b + LN_BND : b) + 10, nA, nC, n0, n1); // the last wave's C is zero
            D = m2_ma(gC, nA, D);
            s0 = __builtin_fma(gC.a, n0, __builtin_fma(gC.b, n1, s0));
            s1 = __builtin_fma(gC.c, n0, __builtin_fma(gC.d, n1, s1));
            const M2 K = inv_i_minus(D);
            gA = mul(K, lA);
            gC = mul(K, mul(gC, nC));
            if (i == 0) gA = {0.0, 0.0, 0.0, 0.0};
            g0 = K.a * s0 + K.b * s1;
            g1 = K.c * s0 + K.d * s1;
        };
        outer();
        unsigned gw = max(ln_word(gA), ln_word(gC));
#pragma unroll 1
        for (int d = 1; d < W; d <<= 1) {
            if (!FULL && ln_decoupled(ln_word(gA), ln_word(gC), g0, g1)) break;
            __asm__ volatile("" ::: "memory");
            ln_put(xch, lane, gA, gC, g0, g1);
            wave_lds_sync();
            ln_step(gA, gC, g0, g1, xch, max(i - d, 0), min(i + d, W - 1));
            gw = max(gw, max(ln_word(gA), ln_word(gC)));
        }
        if (__builtin_expect(__any(gw >= LN_GROWN), 0)) {
            __asm__ volatile("" ::: "memory");
            outer();
            ln_put(xch, lane, gA, gC, g0, g1);
            ln_chain<false>(xch, W, lane == 0, [](int w) { return w; });
            ln_get(xch, i, gA, gC, g0, g1);
        }
        __asm__ volatile("" ::: "memory");
        xch[lane] = make_double2(g0, g1);
        wave_lds_sync();
    }
    const double2 gl = xch[max(wv - 1, 0)], gr = xch[wv];
    const double p0 = wv > 0 ? gl.x : 0.0, p1 = wv > 0 ? gl.y : 0.0;
    B0 = __builtin_fma(A.a, p0, __builtin_fma(A.b, p1, __builtin_fma(C.a, gr.x, __builtin_fma(C.b, gr.y, r0))));
    B1 = __builtin_fma(A.c, p0, __builtin_fma(A.d, p1, __builtin_fma(C.c, gr.x, __builtin_fma(C.d, gr.y, r1))));
    if (lane == 63) {
        B0 = gr.x;
        B1 = gr.y;
    }
    l1 = lane_prev(B0); // on every lane, before the select
    l2 = lane_prev(B1);
    l1 = lane == 0 ? p0 : l1;
    l2 = lane == 0 ? p1 : l2;
    if (FULL && !again) {
        double b0, b1;
        ln_again(A0, C0, q0, q1, l1, l2, lane_next(B0), lane_next(B1), b0, b1);
        B0 = lane == 63 ? B0 : b0; // (its right neighbour is another wave's)
        B1 = lane == 63 ? B1 : b1;
        l1 = lane_prev(B0);
        l2 = lane_prev(B1);
        l1 = lane == 0 ? p0 : l1;
        l2 = lane == 0 ? p1 : l2;
    }
}

} // namespace tf
