// Whole-line sweep kernels of the ensemble (bodies: tf_line_body.h).
#include "tf_line_body.h"

namespace tf {

// Ensemble versions: block -> (film, four columns / one row) from the work list of the films with W waves
// per line, whatever their positions per lane: one launch has no gaps and no nearly empty last waves
// between the sizes (24 films of five sizes: 262 us an iteration with a launch per size, 219 with this). Films
// that are not iterating exit at once (before any barrier: the test is uniform over the block).
template <int KM, int W, bool AL>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) k_xline_ens(EnsParams e)
{
    __shared__ __align__(16) double s2[ln_row2(16, W)];
    __shared__ double sU[ln_row(16, W)];
    __shared__ double bnd[W > 1 ? W * LN_BND : 1];
    const int f = e.items[3 * blockIdx.x], j = e.items[3 * blockIdx.x + 1], cpl = e.items[3 * blockIdx.x + 2];
    if (f < 0) return;
    FilmState *st = e.state + f;
    if (!st->active) return;
    const PassParams p = ens_pass_params(e, e.desc[f], st, 1);
#define TF_XC(C) case C: xline_body<KM, C, (W > 1), AL>(p, j, j, W, sU, s2, bnd); break
    if constexpr (W == 1) {
        switch (cpl) { TF_XC(2); TF_XC(4); TF_XC(6); TF_XC(8); TF_XC(10); TF_XC(12); TF_XC(14); default: TF_XC(16); }
    } else if constexpr (W == 2) {
        switch (cpl) { TF_XC(10); TF_XC(12); TF_XC(14); default: TF_XC(16); }
    } else if constexpr (W == 3) {
        switch (cpl) { TF_XC(12); TF_XC(14); default: TF_XC(16); }
    } else {
        switch (cpl) { TF_XC(14); default: TF_XC(16); }
    }
}

template <int KM, int W>
__global__ void __launch_bounds__(64 * LN_COLS * W) __attribute__((amdgpu_waves_per_eu(2, 2))) k_yline_ens(EnsParams e)
{
    __shared__ __align__(16) double sU[lny_u2(16, W)];
    __shared__ double bnd[W > 1 ? LN_COLS * W * LN_BND : 1];
    const int f = e.items[3 * blockIdx.x], b = e.items[3 * blockIdx.x + 1], cpl = e.items[3 * blockIdx.x + 2];
    if (f < 0) return;
    FilmState *st = e.state + f;
    if (!st->active) return;
    const PassParams p = ens_pass_params(e, e.desc[f], st, 0);
#define TF_YC(C) case C: yline_body<KM, C, W>(p, b * LN_COLS, b, sU, bnd); break
    if constexpr (W == 1) {
        switch (cpl) { TF_YC(2); TF_YC(4); TF_YC(6); TF_YC(8); TF_YC(10); TF_YC(12); TF_YC(14); default: TF_YC(16); }
    } else {
        switch (cpl) { TF_YC(10); TF_YC(12); TF_YC(14); default: TF_YC(16); }
    }
}

// Rows that fill their lanes (aligned) have a launch of their own: with both bodies of every size in one
// kernel its code took 24 films from 20.9 to 24.0 ms.
template <int KM, int W>
static void launch_xline_ens(bool aligned, const EnsParams &e, hipStream_t s)
{
    if (aligned) k_xline_ens<KM, W, true><<<dim3(e.nitems), dim3(64 * W), 0, s>>>(e);
    else k_xline_ens<KM, W, false><<<dim3(e.nitems), dim3(64 * W), 0, s>>>(e);
}

template <int KM>
static hipError_t launch_line_ens_km(int dir, int W, bool aligned, const EnsParams &e, hipStream_t s)
{
    const dim3 grid(e.nitems), by(64 * LN_COLS * W);
    if (dir == 0) {
        if (W == 1) k_yline_ens<KM, 1><<<grid, by, 0, s>>>(e);
        else if (W == 2) k_yline_ens<KM, 2><<<grid, by, 0, s>>>(e);
        else return hipErrorInvalidValue;
    } else {
        if (W == 1) launch_xline_ens<KM, 1>(aligned, e, s);
        else if (W == 2) launch_xline_ens<KM, 2>(aligned, e, s);
        else if (W == 3) launch_xline_ens<KM, 3>(aligned, e, s);
        else if (W == 4) launch_xline_ens<KM, 4>(aligned, e, s);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_line_ens(int dir, int W, bool aligned, int km, const EnsParams &e, hipStream_t s)
{
    switch (km) {
    case KM_P32: return launch_line_ens_km<KM_P32>(dir, W, aligned, e, s);
    case KM_POWER: return launch_line_ens_km<KM_POWER>(dir, W, aligned, e, s);
    case KM_LINEAR: return launch_line_ens_km<KM_LINEAR>(dir, W, aligned, e, s);
    case KM_NLC: return launch_line_ens_km<KM_NLC>(dir, W, aligned, e, s);
    default: return launch_line_ens_km<KM_POLYMER>(dir, W, aligned, e, s);
    }
}

} // namespace tf
