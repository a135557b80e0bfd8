// Host-side bounds check of the whole-line kernels' layout (tf_internal.h, tf_line_body.h, tf_xrow.hip, tf_chain.h): for
// every line length the geometry the library chooses, the LDS offsets of the staged rows and columns, the
// exchange and solution regions, the staged reads, and the interface reduction's records. The geometry rules are the
// library's own (linked); staging loops are restated from the kernels. Prints the (positions, waves) pairs in use
// for the caller to compare with the kernels compiled, then "line geometry check: ok" or the first failures.
#include "../paper_1806_10550_amd/csrc/tf_chain.h"

#include <cstdio>
#include <set>
#include <vector>

using namespace tf;

static int failures = 0;
#define CHECK(cond, ...)                                                                    \
    do {                                                                                    \
        if (!(cond)) {                                                                      \
            if (failures++ < 20) {                                                          \
                std::printf("FAIL %s:%d: %s: ", __FILE__, __LINE__, #cond);                 \
                std::printf(__VA_ARGS__);                                                   \
                std::printf("\n");                                                          \
            }                                                                               \
        }                                                                                   \
    } while (0)

constexpr int LDS_BYTES = 160 * 1024;

// Offsets that depend on (CPL, W) only: rows of W 64 CPL positions, a lane's block, the y sweep's column tile.
template <int CPL>
static void check_offsets(int W)
{
    const int NP = 64 * CPL * W, RB = ln_row(CPL, W);
    std::vector<int> seen(RB, 0);
    for (int w = -2; w < NP + 2; ++w) {
        const int a = ln_at<CPL>(w);
        CHECK(a >= 0 && a < RB, "cpl=%d W=%d w=%d at %d", CPL, W, w, a);
        if (a >= 0 && a < RB) CHECK(seen[a]++ == 0, "cpl=%d W=%d slot %d twice", CPL, W, a);
    }
    for (int s = 0; s < 64 * W; ++s)
        for (int t = -2; t <= CPL + 1; ++t) { // cells -1 .. CPL read one position beyond
            CHECK(ln_at<CPL>(CPL * s) + ln_off<CPL>(t) == ln_at<CPL>(CPL * s + t), "cpl=%d s=%d t=%d", CPL, s, t);
            CHECK(lny_at<CPL>(CPL * s) + lny_off<CPL>(t) == lny_at<CPL>(CPL * s + t), "cpl=%d s=%d t=%d", CPL, s, t);
            if (t >= 0 && t < CPL) CHECK(ln_off<CPL>(t) == t, "cpl=%d t=%d", CPL, t);
        }
    const int U = lny_u(CPL, W);
    std::vector<int> tile(U, 0);
    for (int w = -2; w < NP + 2; ++w)
        for (int c = 0; c < LN_UC; ++c) {
            const int a = lny_at<CPL>(w) + c;
            CHECK(a >= 0 && a < U, "cpl=%d W=%d w=%d column %d at %d", CPL, W, w, c, a);
            if (a >= 0 && a < U) CHECK(tile[a]++ == 0, "cpl=%d W=%d tile slot %d twice", CPL, W, a);
        }
    // a wave's own space: exchange records of its lanes and the two outer ones, then its solution; 16-byte accesses
    CHECK(LN_XS >= 66 && 10 * LN_XS <= ln_priv(CPL) && ln_priv(CPL) % 2 == 0, "cpl=%d", CPL);
    CHECK(64 * (CPL + 1) <= ln_priv(CPL), "cpl=%d", CPL);
    const int last = 64 * CPL - 1;
    CHECK(last + last / CPL < ln_priv(CPL), "cpl=%d", CPL);
    CHECK(W * ln_priv(CPL) <= ln_row2(CPL, W) && RB <= ln_row2(CPL, W), "cpl=%d W=%d", CPL, W);
    CHECK(LN_COLS * W * ln_priv(CPL) <= lny_u2(CPL, W) && LN_COLS * RB <= lny_u2(CPL, W) && U <= lny_u2(CPL, W),
          "cpl=%d W=%d", CPL, W);
    CHECK(LN_BND >= 40, "top pair, lanes 0 and 62, lane 63");
}

static void check_offsets(int cpl, int W)
{
    switch (cpl) {
    case 2: check_offsets<2>(W); break;
    case 4: check_offsets<4>(W); break;
    case 6: check_offsets<6>(W); break;
    case 8: check_offsets<8>(W); break;
    case 10: check_offsets<10>(W); break;
    case 12: check_offsets<12>(W); break;
    case 14: check_offsets<14>(W); break;
    case 16: check_offsets<16>(W); break;
    default: CHECK(false, "cpl=%d", cpl);
    }
}

// Right alignment, folds and staged reads of a line of n cells.
static void check_line(int n, LineGeom g)
{
    const int NP = 64 * g.cpl * g.W, sh = NP - n;
    CHECK(sh >= 0 && sh < 64 * g.cpl, "n=%d cpl=%d W=%d: the line starts past its first wave", n, g.cpl, g.W);
    // lanes that hold part of the line, and the slot of its first cell
    const int nsub = (n + g.cpl - 1) / g.cpl;
    CHECK(sh / g.cpl == 64 * g.W - nsub, "n=%d cpl=%d W=%d", n, g.cpl, g.W);
    CHECK(n % g.cpl != 0 || sh % g.cpl == 0, "n=%d cpl=%d: a filled row starts inside a lane", n, g.cpl);
    for (int w = 0; w < NP; ++w) {
        const int q = w - sh, c = q >= 0 ? q : -1 - (q > -2 ? q : -2), r = crefl(q > -2 ? q : -2, n);
        CHECK(c >= 0 && c < n && r >= 0 && r < n, "n=%d w=%d reads %d, %d", n, w, c, r);
    }
    const int ends[4] = {-2, -1, NP, NP + 1};
    for (int w : ends) {
        const int c = crefl(w - sh > -2 ? w - sh : -2, n);
        CHECK(c >= 0 && c < n, "n=%d w=%d reads %d", n, w, c);
    }
}

static void check_sweeps()
{
    std::set<int> xs, ys;
    for (int n = 4; n <= XR_MAX_NX; ++n) {
        const LineGeom g = xline_geom(n);
        CHECK(xrow_supported(n) && g.W >= 1 && g.W <= 8, "nx=%d W=%d", n, g.W);
        if (n <= XR_ROW4_MAX_NX) CHECK(g.W <= XL_MAXW, "nx=%d W=%d", n, g.W);
        check_line(n, g);
        xs.insert(100 * g.W + g.cpl);
    }
    for (int n = XR_MAX_NX + 1; n < XR_MAX_NX + 40; ++n) CHECK(xline_geom(n).W == 0, "nx=%d", n);
    for (int n = 0; n < 4; ++n) CHECK(xline_geom(n).W == 0 && yline_geom(KM_P32, 64, n).W == 0, "n=%d", n);
    const int kms[5] = {KM_P32, KM_POWER, KM_LINEAR, KM_NLC, KM_POLYMER};
    for (int km : kms)
        for (int ny = 4; ny <= 2100; ++ny)
            for (int nx : {4, 63, 700, 1100, 1637, 2048, 3000, 4096, 4097, 8192}) {
                const LineGeom g = yline_geom(km, nx, ny);
                if (g.W == 0) continue;
                CHECK(g.W <= YL_MAXW, "nx=%d ny=%d W=%d", nx, ny, g.W);
                if (ys.insert(100 * g.W + g.cpl).second || nx == 4) check_line(ny, g);
            }
    for (int v : xs) {
        const int cpl = v % 100, W = v / 100;
        check_offsets(cpl, W);
        const int bytes = 8 * (ln_row2(cpl, W) + ln_row(cpl, W) + (W > 1 ? W * LN_BND : 1));
        CHECK(bytes <= LDS_BYTES, "x cpl=%d W=%d: %d bytes of LDS", cpl, W, bytes);
        std::printf("x %d %d\n", cpl, W);
    }
    for (int v : ys) {
        const int cpl = v % 100, W = v / 100, NT = 64 * LN_COLS * W, NP = 64 * cpl * W;
        check_offsets(cpl, W);
        const int bytes = 8 * (lny_u2(cpl, W) + (W > 1 ? LN_COLS * W * LN_BND : 1));
        CHECK(bytes <= LDS_BYTES && NT <= 1024, "y cpl=%d W=%d: %d bytes of LDS", cpl, W, bytes);
        // staging rounds: u by NT / LN_UC positions, b^n and w by NT / LN_COLS
        const int RU = NT / LN_UC, KU = (NP + 4 + RU - 1) / RU, RW = NT / LN_COLS;
        CHECK(NT % LN_UC == 0 && KU * RU >= NP + 4 && NP % RW == 0, "y cpl=%d W=%d", cpl, W);
        std::printf("y %d %d\n", cpl, W);
    }
    // columns a wave reads around its own in the tile: its two neighbours' cells and their neighbours
    CHECK(2 + 0 - 2 >= 0 && 2 + (LN_COLS - 1) + 2 < LN_UC, "tile columns");
}

// Stored-band lines (launch_sb, k_sbline).
static void check_stored()
{
    std::set<int> used;
    for (int n = 4; n <= XR_ROW4_MAX_NX; ++n) {
        CHECK(sbline_supported(n), "n=%d", n);
        const LineGeom g = {n <= 256 ? 4 : (n <= 512 ? 8 : 16), (n + 1023) / 1024};
        CHECK(64 * g.cpl * g.W >= n, "n=%d", n);
        const int sh = 64 * g.cpl * g.W - n;
        CHECK(sh < 64 * g.cpl && sh / g.cpl == 64 * g.W - (n + g.cpl - 1) / g.cpl, "n=%d", n);
        used.insert(100 * g.W + g.cpl);
    }
    CHECK(!sbline_supported(3) && !sbline_supported(XR_ROW4_MAX_NX + 1), "lengths");
    for (int v : used) {
        const int cpl = v % 100, W = v / 100;
        check_offsets(cpl, W);
        for (int many = 0; many < (W > 1 ? 2 : 1); ++many) {
            const int L = W == 1 ? 4 : (W == 2 ? 2 : 1) * (many ? 2 : 1), NW = L * W, NT = 64 * NW;
            const int R = cpl == 4 ? 6 : (cpl == 8 ? 3 : 2);
            const int stage = R * L * ln_row(cpl, W), own = NW * ln_priv(cpl);
            const int bytes = 8 * ((stage > own ? stage : own) + (W > 1 ? NW * LN_BND : 1) + 2 * NW);
            CHECK(bytes <= LDS_BYTES && NT <= 1024, "cpl=%d W=%d L=%d: %d bytes", cpl, W, L, bytes);
            CHECK(6 % R == 0 && 64 * cpl * W * L == NT * cpl, "cpl=%d W=%d L=%d", cpl, W, L);
            std::printf("s %d %d %d\n", cpl, W, many);
        }
    }
}

// Interface reduction: records of P segments and the boundary records written over them.
static void check_chain()
{
    for (int P = 1; P <= CH_MAXP; ++P) {
        CHECK(chain_reduced(P, 64) && chain_lines(P, 64) == CH_LINES, "P=%d", P);
        for (int WJ = P <= 65 ? 1 : 2; WJ <= 2; ++WJ) {
            const int PP = ch_pitch(WJ), NP = NREL / 2;
            CHECK(P <= PP && P - 1 <= 64 * WJ, "P=%d WJ=%d", P, WJ);
            // last pair of the last line; column q of a junction's halves (every thread writes one)
            CHECK(((CH_LINES - 1) * NP + NP - 1) * PP + PP - 1 < ch_lds(WJ) && 64 * WJ - 1 < PP, "P=%d WJ=%d", P, WJ);
            CHECK(((P - 1) * NEXT + NEXT - 1) * CH_LINES + CH_LINES - 1 < 2 * ch_lds(WJ), "P=%d WJ=%d", P, WJ);
            CHECK(16 * ch_lds(WJ) <= LDS_BYTES, "WJ=%d", WJ);
        }
    }
    CHECK(!chain_reduced(CH_MAXP + 1, 64) && chain_lines(CH_MAXP + 1, 64) == 64, "longest chain");
}

int main()
{
    check_sweeps();
    check_stored();
    check_chain();
    if (failures) {
        std::printf("line geometry check: %d failures\n", failures);
        return 1;
    }
    std::printf("line geometry check: ok\n");
    return 0;
}
