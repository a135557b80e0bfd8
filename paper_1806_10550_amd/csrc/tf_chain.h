// Interface systems of the partitioned line solvers by cyclic reduction.
//
// The P segments of a line satisfy (T, B: a segment's first and last pair)
//   T_q = t_q + Tl_q B_{q-1} + Tr_q T_{q+1},   B_q = b_q + Bl_q B_{q-1} + Br_q T_{q+1}
// with nothing beyond the line's ends. The unknowns of the junction q | q+1 are x_q = (B_q, T_{q+1});
// eliminating each from the other's equation gives
//   x_q = R_q + A_q B_{q-1} + C_q T_{q+2}       (A, C: 4 x 2),
// which couples x_q to the B half of its left and the T half of its right neighbour: log2(P - 1) steps of
// cyclic reduction, each a 4 x 4 solve in 2 x 2 blocks, leave x_q alone. The couplings of an ordinary film span
// 64 cells and vanish after one or two steps; a line then takes no more (stored-band solves take all). Lines whose
// couplings grow (LN_GROWN) are eliminated in order instead. One lane
// per junction; a workgroup holds CH_LINES lines so that records move in 64-byte pieces.
#pragma once

#include "tf_line.h"

namespace tf {

constexpr int CH_LINES = 4;
constexpr int CH_MAXP = 129;                                 // junctions of two waves
__host__ __device__ constexpr int ch_pitch(int WJ) { return 64 * WJ + 1; }
__host__ __device__ constexpr int ch_lds(int WJ) { return CH_LINES * (NREL / 2) * ch_pitch(WJ); } // double2

// Equation of a junction: B half (rb, Ab, Cb), T half (rt, At, Ct).
struct Junction {
    double rb0, rb1, rt0, rt1;
    M2 Ab, Cb, At, Ct;
};

__device__ __forceinline__ void ch_mv(const M2 &x, double v0, double v1, double &o0, double &o1) // o += x v
{
    o0 = __builtin_fma(x.a, v0, __builtin_fma(x.b, v1, o0));
    o1 = __builtin_fma(x.c, v0, __builtin_fma(x.d, v1, o1));
}
__device__ __forceinline__ M2 m2_neg(const M2 &x) { return {-x.a, -x.b, -x.c, -x.d}; }

// One line's system in order (the recurrence of the tiles' chain, tf_device.h), by one wave that fetches the records once
// more; leaves (B_q, T_{q+1}) in the pairs 8 and 9 of column q. In two levels, so that the serial length is a fifth of
// the line's: lane j takes the segments 8 j .. 8 j + 7 in terms of its outer pairs l = B_{8j-1} and T beyond, then the
// groups are chained with all lanes carrying the recurrence, then lane j goes back through its segments (64 lines of 128
// segments, the iteration of a 64 x 8192 film: segment after segment 228 us, this 142).
template <int PP>
__device__ __forceinline__ void chain_in_order(const ChainParams &c, int line, double2 *rec)
{
    constexpr int NP = NREL / 2, G = 8;
    const size_t NL = (size_t)c.nlines;
    const int P = c.P, lane = threadIdx.x & 63, ng = (P + G - 1) / G;
    for (int e = lane; e < NP * P; e += 64)
        rec[(e % NP) * PP + e / NP] = rec_get2(c.rel + (size_t)(e / NP) * NREL * NL + 2 * (size_t)line, NL, e % NP);
    wave_lds_sync();
    const M2 zero = {0.0, 0.0, 0.0, 0.0};
    const int first = G * min(lane, ng - 1), last = min(first + G, P) - 1;
    // the group's first pair T = F + Fl l + Fr T'' and last pair B = b + bl l + M T'', T'' the pair beyond its last segment
    double F0 = 0.0, F1 = 0.0, b0 = 0.0, b1 = 0.0;
    M2 Fl = zero, Fr = {1.0, 0.0, 0.0, 1.0}, bl = {1.0, 0.0, 0.0, 1.0}, M = zero;
    if (lane < ng) {
#pragma unroll 1
        for (int q = first; q <= last; ++q) {
            double T[10], B[10];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const double2 v = rec[k * PP + q], w = rec[(5 + k) * PP + q];
                T[2 * k] = v.x; T[2 * k + 1] = v.y;
                B[2 * k] = w.x; B[2 * k + 1] = w.y;
            }
            const M2 Tl = {T[1], T[2], T[6], T[7]}, Tr = {T[3], T[4], T[8], T[9]};
            const M2 Bl = {B[1], B[2], B[6], B[7]}, Br = {B[3], B[4], B[8], B[9]};
            // B_{q-1} = b + bl l + M T_q gives T_q = t + tl l + N T_{q+1}, then B_q
            const M2 K = inv_i_minus(mul(Tl, M)), N = mul(K, Tr), tl = mul(K, mul(Tl, bl));
            double s0 = T[0], s1 = T[5];
            ch_mv(Tl, b0, b1, s0, s1);
            const double t0 = K.a * s0 + K.b * s1, t1 = K.c * s0 + K.d * s1;
            ch_mv(M, t0, t1, b0, b1);
            double n0 = B[0], n1 = B[5];
            ch_mv(Bl, b0, b1, n0, n1);
            b0 = n0;
            b1 = n1;
            bl = mul(Bl, m2_ma(M, tl, bl));
            M = m2_ma(mul(Bl, M), N, Br);
            ch_mv(Fr, t0, t1, F0, F1);
            Fl = m2_ma(Fr, tl, Fl);
            Fr = mul(Fr, N);
            rec[0 * PP + q] = make_double2(t0, t1);
            rec[1 * PP + q] = make_double2(tl.a, tl.b);
            rec[2 * PP + q] = make_double2(tl.c, tl.d);
            rec[3 * PP + q] = make_double2(N.a, N.b);
            rec[4 * PP + q] = make_double2(N.c, N.d);
            rec[5 * PP + q] = make_double2(b0, b1);
            rec[6 * PP + q] = make_double2(bl.a, bl.b);
            rec[7 * PP + q] = make_double2(bl.c, bl.d);
            rec[8 * PP + q] = make_double2(M.a, M.b);
            rec[9 * PP + q] = make_double2(M.c, M.d);
        }
    }
    auto bc = [](const M2 &x, int j) { return M2{ln_bcast(x.a, j), ln_bcast(x.b, j), ln_bcast(x.c, j), ln_bcast(x.d, j)}; };
    // over the groups: T = t + N T'' and, of the group before, B = p + Q T (kept by the group's lane)
    double t0 = 0.0, t1 = 0.0, p0 = 0.0, p1 = 0.0;
    M2 N = zero, Q = zero;
    {
        double B0 = 0.0, B1 = 0.0;
        M2 BM = zero;
#pragma unroll 1
        for (int j = 0; j < ng; ++j) {
            const M2 Tl = bc(Fl, j), Bl = bc(bl, j);
            const M2 K = inv_i_minus(mul(Tl, BM)), n = mul(K, bc(Fr, j));
            double s0 = ln_bcast(F0, j), s1 = ln_bcast(F1, j);
            ch_mv(Tl, B0, B1, s0, s1);
            const double u0 = K.a * s0 + K.b * s1, u1 = K.c * s0 + K.d * s1;
            if (lane == j) {
                t0 = u0;
                t1 = u1;
                p0 = B0;
                p1 = B1;
                N = n;
                Q = BM;
            }
            ch_mv(BM, u0, u1, B0, B1);
            double n0 = ln_bcast(b0, j), n1 = ln_bcast(b1, j);
            ch_mv(Bl, B0, B1, n0, n1);
            B0 = n0;
            B1 = n1;
            BM = m2_ma(mul(Bl, BM), n, bc(M, j));
        }
    }
    double l0 = 0.0, l1 = 0.0, x0 = 0.0, x1 = 0.0; // the group's outer pairs
    {
        double y0 = 0.0, y1 = 0.0; // nothing beyond the last segment
#pragma unroll 1
        for (int j = ng - 1; j >= 0; --j) {
            if (lane == j) {
                x0 = y0;
                x1 = y1;
            }
            double z0 = ln_bcast(t0, j), z1 = ln_bcast(t1, j);
            ch_mv(bc(N, j), y0, y1, z0, z1);
            y0 = z0;
            y1 = z1;
            if (lane == j) {
                l0 = p0;
                l1 = p1;
                ch_mv(Q, y0, y1, l0, l1);
            }
        }
    }
    __asm__ volatile("" ::: "memory");
    if (lane < ng) {
#pragma unroll 1
        for (int q = last; q >= first; --q) {
            const double2 t = rec[q], u0 = rec[PP + q], u1 = rec[2 * PP + q], n0 = rec[3 * PP + q], n1 = rec[4 * PP + q];
            const double2 b = rec[5 * PP + q], v0 = rec[6 * PP + q], v1 = rec[7 * PP + q], m0 = rec[8 * PP + q],
                          m1 = rec[9 * PP + q];
            double s0 = b.x, s1 = b.y, y0 = t.x, y1 = t.y;
            ch_mv(M2{v0.x, v0.y, v1.x, v1.y}, l0, l1, s0, s1);
            ch_mv(M2{m0.x, m0.y, m1.x, m1.y}, x0, x1, s0, s1);
            ch_mv(M2{u0.x, u0.y, u1.x, u1.y}, l0, l1, y0, y1);
            ch_mv(M2{n0.x, n0.y, n1.x, n1.y}, x0, x1, y0, y1);
            rec[8 * PP + q] = make_double2(s0, s1);
            rec[9 * PP + q] = make_double2(x0, x1);
            x0 = y0;
            x1 = y1;
        }
    }
    wave_lds_sync();
}

// State of a wave's junctions before a step: its largest coupling's word (down to which of the limits it reaches) and
// whether its right-hand sides are finite.
struct ChainState {
    unsigned m, finite;
};
__device__ __forceinline__ bool ch_decoupled(const ChainState &s) { return s.m < LN_DECOUPLED && s.finite != 0u; }

// Lines l0 .. l0 + CH_LINES - 1, WJ waves per line (P - 1 <= 64 WJ); buf: ch_lds(WJ) double2, state: WJ CH_LINES words of LDS.
template <int WJ>
__device__ __forceinline__ void chain_reduce(const ChainParams &c, int l0, double2 *buf, ChainState *state)
{
    constexpr int PP = ch_pitch(WJ), NT = 64 * WJ * CH_LINES, NP = NREL / 2;
    const size_t NL = (size_t)c.nlines;
    const int P = c.P, tid = threadIdx.x;
    // records: pair f of segment q of line l at buf[(l NP + f) PP + q]
    for (int e = tid; e < CH_LINES * NP * P; e += NT) {
        const int l = e % CH_LINES, f = (e / CH_LINES) % NP, q = e / (CH_LINES * NP);
        if (l0 + l < c.nlines)
            buf[(l * NP + f) * PP + q] = rec_get2(c.rel + (size_t)q * NREL * NL + 2 * (size_t)(l0 + l), NL, f);
    }
    __syncthreads();
    const int ln = tid / (64 * WJ), q = tid % (64 * WJ), nj = P - 1; // junction q of line ln
    const int qc = min(q, max(nj - 1, 0));
    double2 *const rec = buf + ln * NP * PP;
    Junction J;
    {
        // B half of segment q (fields 10..19), T half of segment q + 1 (fields 0..9)
        double B[10], T[10];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const double2 v = rec[(5 + k) * PP + qc], w = rec[k * PP + min(qc + 1, P - 1)];
            B[2 * k] = v.x; B[2 * k + 1] = v.y;
            T[2 * k] = w.x; T[2 * k + 1] = w.y;
        }
        const M2 Bl = {B[1], B[2], B[6], B[7]}, Br = {B[3], B[4], B[8], B[9]};
        const M2 Tl = {T[1], T[2], T[6], T[7]};
        M2 Tr = {T[3], T[4], T[8], T[9]};
        if (qc == nj - 1) Tr = {0.0, 0.0, 0.0, 0.0};
        const M2 K = inv_i_minus(mul(Br, Tl));
        double s0 = B[0], s1 = B[5];
        ch_mv(Br, T[0], T[5], s0, s1);
        J.rb0 = K.a * s0 + K.b * s1;
        J.rb1 = K.c * s0 + K.d * s1;
        J.Ab = qc == 0 ? M2{0.0, 0.0, 0.0, 0.0} : mul(K, Bl);
        J.Cb = mul(K, mul(Br, Tr));
        J.rt0 = T[0];
        J.rt1 = T[5];
        ch_mv(Tl, J.rb0, J.rb1, J.rt0, J.rt1);
        J.At = mul(Tl, J.Ab);
        J.Ct = m2_ma(Tl, J.Cb, Tr);
    }
    auto sync = [&] {
        if (WJ > 1) __syncthreads();
        else wave_lds_sync();
    };
    // junction q's B half at pairs 0..4, its T half at pairs 5..9 of column q
    const bool in = q < nj;
    bool grown = false, any_grown = false; // this line; any line of the workgroup (WJ > 1)
    for (int d = 1; d < nj; d <<= 1) {
        // a line takes steps until its junctions are decoupled or its couplings have grown, whatever the lines beside it
        const unsigned m = in ? max(max(ln_word(J.Ab), ln_word(J.Cb)), max(ln_word(J.At), ln_word(J.Ct))) : 0u;
        const unsigned r = in ? max(max(hi_word(J.rb0), hi_word(J.rb1)), max(hi_word(J.rt0), hi_word(J.rt1))) : 0u;
        const ChainState st = {__any(m >= LN_GROWN) ? LN_GROWN : (__any(m >= LN_DECOUPLED) ? LN_DECOUPLED : 0u),
                               __all(r < 0x7ff00000u) ? 1u : 0u};
        bool go;
        if (WJ > 1) {
            if ((tid & 63) == 0) state[tid / 64] = st;
            __syncthreads(); // (also: the records / the last step's halves have been read)
            bool any = false;
            go = false;
            for (int l = 0; l < CH_LINES; ++l) {
                ChainState s = state[l * WJ];
                for (int w = 1; w < WJ; ++w) {
                    const ChainState o = state[l * WJ + w];
                    s = {max(s.m, o.m), s.finite & o.finite};
                }
                const bool g = s.m >= LN_GROWN && l0 + l < c.nlines; // (and stays so: it takes no more steps)
                const bool step = s.m < LN_GROWN && l0 + l < c.nlines && (c.full || !ch_decoupled(s));
                any_grown |= g;
                any |= step;
                if (l == ln) {
                    grown = g;
                    go = step;
                }
            }
            if (!any) break;
        } else {
            grown = st.m >= LN_GROWN && l0 + ln < c.nlines;
            go = st.m < LN_GROWN && l0 + ln < c.nlines && (c.full || !ch_decoupled(st));
            if (!go) break;
        }
        __asm__ volatile("" ::: "memory");
        rec[0 * PP + q] = make_double2(J.rb0, J.rb1);
        rec[1 * PP + q] = make_double2(J.Ab.a, J.Ab.b);
        rec[2 * PP + q] = make_double2(J.Ab.c, J.Ab.d);
        rec[3 * PP + q] = make_double2(J.Cb.a, J.Cb.b);
        rec[4 * PP + q] = make_double2(J.Cb.c, J.Cb.d);
        rec[5 * PP + q] = make_double2(J.rt0, J.rt1);
        rec[6 * PP + q] = make_double2(J.At.a, J.At.b);
        rec[7 * PP + q] = make_double2(J.At.c, J.At.d);
        rec[8 * PP + q] = make_double2(J.Ct.a, J.Ct.b);
        rec[9 * PP + q] = make_double2(J.Ct.c, J.Ct.d);
        sync();
        if (!go) continue;
        // past the line's ends A or C is zero and any junction's halves will do
        const double2 *L = rec + max(qc - d, 0), *R = rec + min(qc + d, nj - 1);
        const double2 l0v = L[0], l1 = L[PP], l2 = L[2 * PP], l3 = L[3 * PP], l4 = L[4 * PP];
        const M2 lA = {l1.x, l1.y, l2.x, l2.y}, lC = {l3.x, l3.y, l4.x, l4.y};
        const double2 r0v = R[5 * PP], r1 = R[6 * PP], r2 = R[7 * PP], r3 = R[8 * PP], r4 = R[9 * PP];
        const M2 rA = {r1.x, r1.y, r2.x, r2.y}, rC = {r3.x, r3.y, r4.x, r4.y};
        // [M_BB M_BT; M_TB M_TT] x = f + F B'' + G T''
        const M2 Mbt = m2_neg(mul(J.Ab, lC)), Mtb = m2_neg(mul(J.Ct, rA));
        const M2 Pb = inv_i_minus(mul(J.Cb, rA));
        const M2 U = mul(Pb, Mbt);
        // S = M_TT - M_TB U = I - (A_T lC + M_TB U)
        const M2 Si = inv_i_minus(m2_ma(Mtb, U, mul(J.At, lC)));
        double fb0 = J.rb0, fb1 = J.rb1, ft0 = J.rt0, ft1 = J.rt1;
        ch_mv(J.Ab, l0v.x, l0v.y, fb0, fb1);
        ch_mv(J.Cb, r0v.x, r0v.y, fb0, fb1);
        ch_mv(J.At, l0v.x, l0v.y, ft0, ft1);
        ch_mv(J.Ct, r0v.x, r0v.y, ft0, ft1);
        {
            const double g0 = Pb.a * fb0 + Pb.b * fb1, g1 = Pb.c * fb0 + Pb.d * fb1;
            const double h0 = ft0 - (Mtb.a * g0 + Mtb.b * g1), h1 = ft1 - (Mtb.c * g0 + Mtb.d * g1);
            J.rt0 = Si.a * h0 + Si.b * h1;
            J.rt1 = Si.c * h0 + Si.d * h1;
            J.rb0 = g0 - (U.a * J.rt0 + U.b * J.rt1);
            J.rb1 = g1 - (U.c * J.rt0 + U.d * J.rt1);
        }
        auto solve = [&](const M2 &Fb, const M2 &Ft, M2 &Xb, M2 &Xt) {
            const M2 G = mul(Pb, Fb);
            Xt = mul(Si, m2_ma(m2_neg(Mtb), G, Ft));
            Xb = m2_ma(m2_neg(U), Xt, G);
        };
        const M2 Fb = mul(J.Ab, lA), Ft = mul(J.At, lA), Gb = mul(J.Cb, rC), Gt = mul(J.Ct, rC);
        solve(Fb, Ft, J.Ab, J.At);
        solve(Gb, Gt, J.Cb, J.Ct);
    }
    if (grown && tid % (64 * WJ) < 64) chain_in_order<PP>(c, l0 + ln, rec);
    if (WJ > 1 && any_grown) __syncthreads();
    if (grown && in) {
        const double2 b = rec[8 * PP + q], t = rec[9 * PP + q];
        J.rb0 = b.x;
        J.rb1 = b.y;
        J.rt0 = t.x;
        J.rt1 = t.y;
    }
    // boundary records: segment s takes l = B_{s-1} and r = T_{s+1}; through LDS so that a position's lines
    // are stored together
    __syncthreads();
    double *const eo = reinterpret_cast<double *>(buf); // [segment][field][line]
    if (q < nj) {
        eo[((q + 1) * NEXT + 0) * CH_LINES + ln] = J.rb0;
        eo[((q + 1) * NEXT + 1) * CH_LINES + ln] = J.rb1;
        eo[(q * NEXT + 2) * CH_LINES + ln] = J.rt0;
        eo[(q * NEXT + 3) * CH_LINES + ln] = J.rt1;
    }
    if (q == 0) {
        eo[0 * CH_LINES + ln] = 0.0;
        eo[1 * CH_LINES + ln] = 0.0;
        eo[((P - 1) * NEXT + 2) * CH_LINES + ln] = 0.0;
        eo[((P - 1) * NEXT + 3) * CH_LINES + ln] = 0.0;
    }
    __syncthreads();
    for (int e = tid; e < CH_LINES * NEXT * P; e += NT) {
        const int l = e % CH_LINES;
        if (l0 + l < c.nlines) c.ext[(size_t)(e / CH_LINES) * NL + l0 + l] = eo[e];
    }
}

} // namespace tf
