// Whole-line sweep kernels of one film (bodies: tf_line_body.h) and the geometry rules they share with the
// ensemble's (tf_line_ens.hip).
#include "tf_line_body.h"

namespace tf {

bool xrow_supported(int nx) { return nx >= 4 && nx <= XR_MAX_NX; }

// Positions per lane and waves per line: as few waves as hold the line with 16 positions per lane, then the
// fewest positions (an even number) that hold it with those. Few positions make short lines fast: the
// elimination is a serial chain over them and small launches do not fill the GPU (128^2 and 512^2: 8 and
// 11 us a sweep with 4 and 8, where 16 took 29 and 23); two leave nothing to eliminate, the pair being the
// whole lane (128^2: x + y 18.3 -> 16.4 us). For long lines 16 positions in few waves beat 8 in
// twice as many, whose cyclic reduction costs twice as much per cell (rows of 1000 cells, 8192 of them: 68
// against 89 us; 4096^2: 164 against 263). Lengths between the powers of two leave no lanes idle (600^2:
// 35 -> 27 us for both sweeps, 3001 x 700 polymer 74 -> 60). The partitioned x sweep takes longer at every
// length and number of rows (2048^2: 87 against 45 us, 8192 rows of 4096: 485 against 344).
static int line_positions(int n, int W)
{
    return W > 4 ? 16 : (n <= 128 ? 2 : n <= 256 ? 4 : 2 * ((n + 128 * W - 1) / (128 * W)));
}
LineGeom xline_geom(int nx)
{
    if (!xrow_supported(nx)) return {0, 0};
    const int W = (nx + 1023) / 1024;
    return {line_positions(nx, W), W};
}
// Columns of more than 1024 cells need a workgroup of 8 waves and up to 135 KB of LDS, one per CU, that
// overlaps nothing: with many of them the partitioned passes stream better (8192 x 2048: 268 against
// 251 us; 4096 x 2048: 127 against 142; 2048^2: 65 against 86). The NLC model, whose cells cost most, also
// evaluates its neighbouring columns' cells, and its time goes by rounds of one workgroup per CU (1300 rows:
// 68 us from 1100 to 1450 columns, 100 from 2200 to 3072): whole columns gain where the last round leaves the GPU well filled
// (700 x 1300: 37 against 53 us partitioned, 1637^2 79 against 91, 2700 x 1637 114 against 124, 4000 x 1500
// 135 against 151; 1100 x 1300 70 against 69, 2200 x 1300 100 against 95) and, with 16 positions per lane,
// in at most two rounds (2048^2 108 against 114, 3000 x 2000 157 against 145).
// Short columns in wide films: the partitioned passes stream them better once four-column workgroups are many
// (power law, whole / partitioned y sweep in us: 12000 x 64 38/41, 16384 x 64 49/42, 65536 x 64 164/80, 65536 x 4 94/45;
// 12000 x 128 42/51, 16384 x 128 53/52, 65536 x 128 175/130; 16384 x 129 66/67, 32768 x 129 121/105), from four tile
// rows on never (65536 x 200 221/233, 65536 x 1000 whole 0.7 of the time).
LineGeom yline_geom(int km, int nx, int ny)
{
    if (ny <= 3 * TILE && nx > (ny <= TILE ? 12288 : 16384)) return {0, 0};
    if (ny < 4 || ny > 2048 || (ny > 1024 && nx > 4096)) return {0, 0};
    if (km == KM_NLC && ny > 1024) {
        constexpr int round = 256 * LN_COLS; // columns
        const int n = (nx + round - 1) / round;
        if (n > 1 && (4 * nx < 3 * round * n || (ny > 1792 && n > 2))) return {0, 0};
    }
    const int W = (ny + 1023) / 1024;
    return {line_positions(ny, W), W};
}

// Waves per SIMD the line kernels are compiled for: with 10 and more positions a lane holds 50 to 80
// factors (2 waves), with 6 and 8 up to 40 (3 waves).
constexpr int line_waves(int cpl) { return cpl >= 10 ? 2 : (cpl >= 6 ? 3 : 4); }
#define TF_LINE_ATTR(CPL) __attribute__((amdgpu_waves_per_eu(line_waves(CPL), line_waves(CPL))))

template <int KM, int CPL, int W, bool AL>
__global__ void __launch_bounds__(64 * W) TF_LINE_ATTR(CPL) k_xline(PassParams p)
{
    __shared__ __align__(16) double s2[ln_row2(CPL, W)];
    __shared__ double sU[ln_row(CPL, W)];
    __shared__ double bnd[W > 1 ? W * LN_BND : 1];
    const int j = xcd_tile(blockIdx.x, p.ny);
    xline_body<KM, CPL, (W > 1), AL>(p, j, j, W, sU, s2, bnd);
}

template <int KM, int CPL, int W>
__global__ void __launch_bounds__(64 * LN_COLS * W) TF_LINE_ATTR(CPL) k_yline(PassParams p, int nblocks)
{
    __shared__ __align__(16) double sU[lny_u2(CPL, W)];
    __shared__ double bnd[W > 1 ? LN_COLS * W * LN_BND : 1];
    const int b = xcd_tile(blockIdx.x, nblocks);
    yline_body<KM, CPL, W>(p, b * LN_COLS, b, sU, bnd);
}

template <int KM>
static hipError_t launch_line_km(int dir, const PassParams &p, hipStream_t s)
{
    const int nb = (p.nx + LN_COLS - 1) / LN_COLS;
    const LineGeom g = dir == 0 ? yline_geom(KM, p.nx, p.ny) : xline_geom(p.nx);
    const dim3 gx(p.ny), gy(nb), bx(64 * g.W), by(64 * LN_COLS * g.W);
#define TF_XL(C, V) \
    case 100 * V + C: \
        if (p.nx % C == 0) k_xline<KM, C, V, true><<<gx, bx, 0, s>>>(p); \
        else k_xline<KM, C, V, false><<<gx, bx, 0, s>>>(p); \
        break
#define TF_YL(C, V) case 100 * V + C: k_yline<KM, C, V><<<gy, by, 0, s>>>(p, nb); break
    if (dir == 0) {
        switch (100 * g.W + g.cpl) {
        TF_YL(2, 1); TF_YL(4, 1); TF_YL(6, 1); TF_YL(8, 1); TF_YL(10, 1); TF_YL(12, 1); TF_YL(14, 1); TF_YL(16, 1);
        TF_YL(10, 2); TF_YL(12, 2); TF_YL(14, 2); TF_YL(16, 2);
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (100 * g.W + g.cpl) {
        TF_XL(2, 1); TF_XL(4, 1); TF_XL(6, 1); TF_XL(8, 1); TF_XL(10, 1); TF_XL(12, 1); TF_XL(14, 1); TF_XL(16, 1);
        TF_XL(10, 2); TF_XL(12, 2); TF_XL(14, 2); TF_XL(16, 2);
        TF_XL(12, 3); TF_XL(14, 3); TF_XL(16, 3); TF_XL(14, 4); TF_XL(16, 4);
        TF_XL(16, 5); TF_XL(16, 6); TF_XL(16, 7); TF_XL(16, 8);
        default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

hipError_t launch_line(int dir, const PassParams &p, hipStream_t s)
{
    switch (p.M.kind) {
    case MODEL_LINEAR: return launch_line_km<KM_LINEAR>(dir, p, s);
    case MODEL_NLC: return launch_line_km<KM_NLC>(dir, p, s);
    case MODEL_POLYMER: return launch_line_km<KM_POLYMER>(dir, p, s);
    default:
        return p.M.p32 ? launch_line_km<KM_P32>(dir, p, s) : launch_line_km<KM_POWER>(dir, p, s);
    }
}

} // namespace tf
