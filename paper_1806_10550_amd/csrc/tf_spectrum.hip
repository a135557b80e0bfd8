// Radial Fourier spectrum of a film (App. "Radial Fourier Transform"; see include/thinfilm.h,
// tf_radial_spectrum and tf_spectrum_maxima).
//
// Device part (steps 1-4): the film minus H0 is transformed by hipFFT, in place and real to complex (half
// spectrum, the other half by conjugate symmetry): the rows, then only the columns kx that the window
// below reads, brought together by a transpose (a window of 5 q_m reads a twentieth to an eighth of the
// columns of the paper's films; the full 2D transform runs when it reads more than half of the half
// spectrum). The magnitudes are gathered into a window of the wavenumber plane that covers the disk
// |k|^2 <= M plus the Gaussian's reach (indices taken modulo n, so the smoothing is the periodic
// convolution over the whole plane); two separable passes smooth the window; the smoothed values of
// each group m = kx^2 + ky^2 (all its wavevectors have the same |q|) are averaged in a fixed order (an
// index of the window by group, built once per window on the host), so spectra are bit-reproducible.
// Only the row transforms touch all n^2 values; the window holds (2 sqrt(M) + 2 r + 1)^2 values. Bound
// by the row transforms: 2674^2 (a length with a prime factor 191) 173 of 383 us, where transforming every
// column took another 185 and reading sums and counts of empty groups back to pageable memory 70.
//
// Host part (steps 5-7): the fit has about N/10 unknowns, the smoothed curve 400 points: a
// tridiagonal normal-equation solve and a few passes over 400 doubles, done in plain C++.
#include "tf_internal.h"
#include "../../include/thinfilm.h"

#include <hipfft/hipfft.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace tf {

// buf[j * pitch + i] = h[j * n + i] - h0: the film minus H0 in the padded row layout of an
// in-place real-to-complex transform (pitch = 2 (n/2 + 1) doubles).
__global__ void __launch_bounds__(256) k_spec_load(const double *__restrict__ h, double h0, int n, int pitch,
                                                   double *__restrict__ buf)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (i >= n) return;
    buf[(size_t)j * pitch + i] = h[(size_t)j * n + i] - h0;
}

// T[c][j] = F[j][c] for the columns c < nc of the half spectrum (rows of pitch2 complex values), through
// a 32 x 32 LDS tile; zero for nc <= c < nb, which the column plan transforms with the rest (what an earlier,
// wider window left there would grow by each transform).
__global__ void __launch_bounds__(256) k_spec_columns(const hipfftDoubleComplex *__restrict__ F, int n, int pitch2,
                                                      int nc, int nb, hipfftDoubleComplex *__restrict__ T)
{
    __shared__ hipfftDoubleComplex t[32][33];
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32, x = threadIdx.x & 31, y = threadIdx.x >> 5;
#pragma unroll
    for (int r = y; r < 32; r += 8)
        t[r][x] = r0 + r < n && c0 + x < nc ? F[(size_t)(r0 + r) * pitch2 + c0 + x] : hipfftDoubleComplex{0.0, 0.0};
    __syncthreads();
#pragma unroll
    for (int c = y; c < 32; c += 8)
        if (c0 + c < nb && r0 + x < n) T[(size_t)(c0 + c) * n + r0 + x] = t[x][c];
}

// A[(wy + E) * W + (wx + E)] = |F(wx mod n, wy mod n)| / n^2 for wx, wy in [-E, E], from the
// half spectrum of the real transform: the other half follows from F(-k) = conj F(k). Element (ix,
// iy), ix <= n/2, at F[ix * sx + iy * sy].
__global__ void __launch_bounds__(256) k_spec_window(const hipfftDoubleComplex *__restrict__ F, size_t sx, size_t sy,
                                                     int n, int E, double inv_n2, double *__restrict__ A)
{
    const int W = 2 * E + 1;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= W * W) return;
    const int wx = t % W - E, wy = t / W - E;
    int ix = ((wx % n) + n) % n, iy = ((wy % n) + n) % n;
    if (ix > n / 2) {
        ix = n - ix;
        iy = (n - iy) % n;
    }
    const hipfftDoubleComplex c = F[ix * sx + iy * sy];
    A[t] = sqrt(c.x * c.x + c.y * c.y) * inv_n2;
}

// One separable smoothing pass over a window of side W (input) into a window of side
// W - 2r (output), along x (DIR 0) or y (DIR 1); the other index keeps its range when
// DIR says so: out is (Wo x Wi) with Wi = W along the untouched axis.
template <int DIR>
__global__ void __launch_bounds__(256) k_spec_smooth(const double *__restrict__ in, int Win_x, int Win_y,
                                                     const double *__restrict__ w, int r, double *__restrict__ out)
{
    const int Wo_x = DIR == 0 ? Win_x - 2 * r : Win_x;
    const int Wo_y = DIR == 1 ? Win_y - 2 * r : Win_y;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= Wo_x * Wo_y) return;
    const int ox = t % Wo_x, oy = t / Wo_x;
    double s = 0.0;
    for (int d = 0; d <= 2 * r; ++d) {
        const int ix = DIR == 0 ? ox + d : ox;
        const int iy = DIR == 1 ? oy + d : oy;
        s = fma(w[d], in[(size_t)iy * Win_x + ix], s);
    }
    out[t] = s;
}

// Group means over the disk: S is the smoothed window of side 2R+1 centred on k = 0. SG lanes per
// nonempty group of m = kx^2 + ky^2 (1 <= m <= M; a dozen wavevectors on average): lane i adds the values i,
// i + SG, ... of the index (window positions sorted by group, then by position) and the lanes' sums are
// added in a fixed tree, so the means do not depend on scheduling.
constexpr int SG = 8;
__global__ void __launch_bounds__(256) k_spec_groups(const double *__restrict__ S, const int *__restrict__ perm,
                                                     const int *__restrict__ off, int ng, double *__restrict__ mean)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x, g = t / SG;
    const bool live = g < ng;
    const int b = live ? off[g] : 0, e = live ? off[g + 1] : 0;
    double acc = 0.0;
    for (int i = b + t % SG; i < e; i += SG) acc += S[perm[i]];
#pragma unroll
    for (int o = SG / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (live && t % SG == 0) mean[g] = acc / (e - b);
}

} // namespace tf

namespace {

tf_status sfail(tf_status s, const std::string &msg)
{
    tf_detail::set_error(msg);
    return s;
}

// Plans and scratch of one (device, n), kept until tf_spectrum_release: the padded real /
// half-complex buffer of the in-place transform and the small window and group arrays
// (grown on demand).
struct SpecWork {
    hipfftHandle full = 0, rows = 0;                // 2D transform; row transforms
    bool has_full = false, has_rows = false;
    std::map<int, hipfftHandle> cols;               // column transforms by batch (64, 128, 256, ...)
    double *buf = nullptr;
    hipfftDoubleComplex *colbuf = nullptr;          // transposed columns
    size_t col_cap = 0;
    double *small = nullptr; // A | B | C | weights | means, doubles
    size_t small_cap = 0;
    double *hmean = nullptr; // pinned host copy of the means
    size_t hmean_cap = 0;
    // index of the window by group for the last (M, R): the nonempty groups in increasing m
    // (gm), perm lists window positions sorted by m = kx^2 + ky^2 (then by position), group g owns
    // perm[off[g] .. off[g+1])
    int *perm = nullptr, *off = nullptr;
    std::vector<int> gm, goff;
    long long idx_M = -1;
    int idx_R = -1;
};
struct WorkKey {
    int device, n;
    bool operator<(const WorkKey &o) const { return device != o.device ? device < o.device : n < o.n; }
};
std::mutex g_spec_mu;
std::map<WorkKey, SpecWork> g_spec;

void free_work(SpecWork &w)
{
    if (w.has_full) (void)hipfftDestroy(w.full);
    if (w.has_rows) (void)hipfftDestroy(w.rows);
    for (auto &kv : w.cols) (void)hipfftDestroy(kv.second);
    if (w.buf) (void)hipFree(w.buf);
    if (w.colbuf) (void)hipFree(w.colbuf);
    if (w.small) (void)hipFree(w.small);
    if (w.hmean) (void)hipHostFree(w.hmean);
    if (w.perm) (void)hipFree(w.perm);
    if (w.off) (void)hipFree(w.off);
    w = SpecWork{};
}

// The window index for the groups 1..M over a window of half side R (n x n spectrum), built on
// the host by a counting sort over m (positions in increasing order within a group) and kept
// until the next call with another (M, R). Called with g_spec_mu held.
tf_status get_index(SpecWork &w, int n, int R, long long M)
{
    if (w.idx_M == M && w.idx_R == R) return TF_OK;
    const int Wr = 2 * R + 1;
    const int lo = -(n / 2), hi = (n - 1) / 2;
    const long long npos = (long long)Wr * Wr;
    auto group = [&](long long t) -> long long {
        const int kx = (int)(t % Wr) - R, ky = (int)(t / Wr) - R;
        if (kx < lo || kx > hi || ky < lo || ky > hi) return 0;
        const long long m = (long long)kx * kx + (long long)ky * ky;
        return m <= M ? m : 0;
    };
    std::vector<int> at(M + 1, 0); // members, then the compact number, of each group
    for (long long t = 0; t < npos; ++t) {
        const long long m = group(t);
        if (m > 0) ++at[m];
    }
    w.gm.clear();
    w.goff.assign(1, 0);
    for (long long m = 1; m <= M; ++m) {
        if (at[m] == 0) continue;
        w.goff.push_back(w.goff.back() + at[m]);
        at[m] = (int)w.gm.size();
        w.gm.push_back((int)m);
    }
    std::vector<int> perm((size_t)w.goff.back()), next(w.goff.begin(), w.goff.end() - 1);
    for (long long t = 0; t < npos; ++t) {
        const long long m = group(t);
        if (m > 0) perm[(size_t)next[at[m]]++] = (int)t;
    }
    if (w.perm) (void)hipFree(w.perm);
    if (w.off) (void)hipFree(w.off);
    w.perm = nullptr;
    w.off = nullptr;
    w.idx_M = -1;
    if (hipMalloc(&w.perm, std::max<size_t>(perm.size(), 1) * sizeof(int)) != hipSuccess
        || hipMalloc(&w.off, w.goff.size() * sizeof(int)) != hipSuccess) {
        if (w.perm) (void)hipFree(w.perm);
        w.perm = nullptr;
        w.off = nullptr;
        return sfail(TF_ENOMEM, "spectrum index allocation failed");
    }
    if (hipMemcpy(w.perm, perm.data(), perm.size() * sizeof(int), hipMemcpyHostToDevice) != hipSuccess
        || hipMemcpy(w.off, w.goff.data(), w.goff.size() * sizeof(int), hipMemcpyHostToDevice) != hipSuccess)
        return sfail(TF_EDEVICE, "spectrum index upload failed");
    w.idx_M = M;
    w.idx_R = R;
    return TF_OK;
}

// Batch of the column plan that covers nc columns.
int col_batch(int nc)
{
    int b = 64;
    while (b < nc) b *= 2;
    return b;
}

// Plans, buffers and scratch of one call. groups: nonempty groups, whose means come back through pinned memory;
// nc: columns of the half spectrum to transform, or 0 for the full 2D transform. Called with g_spec_mu held.
tf_status get_work(SpecWork &w, int n, size_t small_doubles, size_t groups, int nc)
{
    if (nc == 0 && !w.has_full) {
        if (hipfftPlan2d(&w.full, n, n, HIPFFT_D2Z) != HIPFFT_SUCCESS) return sfail(TF_EDEVICE, "hipfftPlan2d failed");
        w.has_full = true;
    }
    if (nc > 0 && !w.has_rows) {
        int len = n, in = 2 * (n / 2 + 1), on = n / 2 + 1;
        if (hipfftPlanMany(&w.rows, 1, &len, &in, 1, in, &on, 1, on, HIPFFT_D2Z, n) != HIPFFT_SUCCESS)
            return sfail(TF_EDEVICE, "hipfftPlanMany (rows) failed");
        w.has_rows = true;
    }
    if (nc > 0 && w.cols.find(col_batch(nc)) == w.cols.end()) {
        int len = n;
        hipfftHandle h = 0;
        if (hipfftPlanMany(&h, 1, &len, &len, 1, n, &len, 1, n, HIPFFT_Z2Z, col_batch(nc)) != HIPFFT_SUCCESS)
            return sfail(TF_EDEVICE, "hipfftPlanMany (columns) failed");
        w.cols[col_batch(nc)] = h;
    }
    if (w.buf == nullptr
        && hipMalloc(&w.buf, (size_t)n * (n / 2 + 1) * sizeof(hipfftDoubleComplex)) != hipSuccess) {
        w.buf = nullptr;
        return sfail(TF_ENOMEM, "spectrum buffer allocation failed");
    }
    const size_t col_need = nc > 0 ? (size_t)col_batch(nc) * n : 0;
    if (w.col_cap < col_need) {
        if (w.colbuf) (void)hipFree(w.colbuf);
        w.colbuf = nullptr;
        w.col_cap = 0;
        if (hipMalloc(&w.colbuf, col_need * sizeof(hipfftDoubleComplex)) != hipSuccess) {
            w.colbuf = nullptr;
            return sfail(TF_ENOMEM, "spectrum buffer allocation failed");
        }
        w.col_cap = col_need;
    }
    if (w.small_cap < small_doubles) {
        if (w.small) (void)hipFree(w.small);
        w.small = nullptr;
        w.small_cap = 0;
        if (hipMalloc(&w.small, small_doubles * sizeof(double)) != hipSuccess) {
            w.small = nullptr;
            return sfail(TF_ENOMEM, "spectrum scratch allocation failed");
        }
        w.small_cap = small_doubles;
    }
    if (w.hmean_cap < groups) {
        if (w.hmean) (void)hipHostFree(w.hmean);
        w.hmean = nullptr;
        w.hmean_cap = 0;
        if (hipHostMalloc(&w.hmean, groups * sizeof(double), hipHostMallocDefault) != hipSuccess) {
            w.hmean = nullptr;
            return sfail(TF_ENOMEM, "spectrum host buffer allocation failed");
        }
        w.hmean_cap = groups;
    }
    return TF_OK;
}

// Waits for the stream on every exit, so that no work of a failed call is left queued.
struct StreamDrain {
    hipStream_t s;
    ~StreamDrain() { (void)hipStreamSynchronize(s); }
};

} // namespace

extern "C" {

tf_status tf_radial_spectrum(const double *h, int n, double ds, double h0, double sigma, double qmax, void *stream,
                             double *q_out, double *s_out, int *count_out, int capacity, int *npoints)
{
    if (h == nullptr || npoints == nullptr) return sfail(TF_EINVAL, "NULL argument");
    if (n < 4 || n > (1 << 14)) return sfail(TF_EINVAL, "need 4 <= n <= 16384");
    if (!(ds > 0.0) || !std::isfinite(ds) || !std::isfinite(h0)) return sfail(TF_EINVAL, "need finite ds > 0 and h0");
    if (!(sigma >= 0.0) || sigma > 64.0) return sfail(TF_EINVAL, "need 0 <= sigma <= 64");
    if (!(qmax > 0.0) || !std::isfinite(qmax)) return sfail(TF_EINVAL, "need finite qmax > 0");
    const double L = n * ds;
    const double kmax = qmax * L / (2.0 * M_PI);
    // groups beyond the spectrum's largest |k|^2 are empty
    const double mcap = 2.0 * (double)(n / 2) * (double)(n / 2);
    long long M = (long long)std::floor(std::min(kmax * kmax * (1.0 + 1e-12), mcap));
    if (M < 1) {
        *npoints = 0;
        return TF_OK;
    }
    if (M > (1LL << 26)) return sfail(TF_EINVAL, "qmax too large: more than 2^26 wavenumber groups");
    const int R = std::min((int)std::floor(std::sqrt((double)M)), n / 2);
    const int r = sigma > 0.0 ? (int)std::ceil(4.0 * sigma) : 0;
    const int E = R + r, W = 2 * E + 1, Wr = 2 * R + 1;
    std::vector<double> w(2 * r + 1, 1.0);
    if (r > 0) {
        double z = 0.0;
        for (int d = -r; d <= r; ++d) z += (w[d + r] = std::exp(-(double)d * d / (2.0 * sigma * sigma)));
        for (double &v : w) v /= z;
    }
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lk(g_spec_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return sfail(TF_EDEVICE, "hipGetDevice failed");
    SpecWork *const wk = &g_spec[WorkKey{dev, n}];
    tf_status st = get_index(*wk, n, R, M);
    if (st != TF_OK) return st;
    const int ng = (int)wk->gm.size();
    // small scratch: A (W x W) | B (Wr x W) | C (Wr x Wr) | weights | group means
    const size_t oA = 0, oB = oA + (size_t)W * W, oC = oB + (size_t)W * Wr, oW = oC + (size_t)Wr * Wr,
                 oS = oW + w.size(), small = oS + ng;
    // The columns 0 .. E (and their mirror images) are all the window reads. Up to half of the half spectrum they win
    // over the full transform, batches rounded up to a power of two included (whole call, us, columns / full: 2674^2 with
    // 80 columns 326 / 537, 401 491 / 652, 602 712 / 785, 669 760 / 843; 1637^2 409 columns 376 / 484; 4096^2 122
    // 241 / 309, 1024 946 / 991; 1024^2 51 75 / 77, 256 126 / 129), up to n = 512 only for lengths with larger prime
    // factors (401^2 79 / 86): there one launch more costs powers of two 3 to 5 us (512^2 58 / 52, 128^2 57 / 54).
    const int nc = 2 * (E + 1) <= n / 2 + 1 ? E + 1 : 0;
    if ((st = get_work(*wk, n, small, ng, nc)) != TF_OK) return st;
    StreamDrain drain{s};
    double *A = wk->small + oA, *B = wk->small + oB, *C = wk->small + oC, *wd = wk->small + oW,
           *mean = wk->small + oS;
    const int pitch = 2 * (n / 2 + 1);
    if (hipMemcpyAsync(wd, w.data(), w.size() * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
        return sfail(TF_EDEVICE, "spectrum scratch setup failed");
    tf::k_spec_load<<<dim3((n + 255) / 256, n), 256, 0, s>>>(h, h0, n, pitch, wk->buf);
    if (hipGetLastError() != hipSuccess) return sfail(TF_EDEVICE, "spectrum load launch failed");
    auto *F = (hipfftDoubleComplex *)wk->buf;
    const hipfftHandle first = nc > 0 ? wk->rows : wk->full;
    if (hipfftSetStream(first, s) != HIPFFT_SUCCESS || hipfftExecD2Z(first, wk->buf, F) != HIPFFT_SUCCESS)
        return sfail(TF_EDEVICE, "hipfftExecD2Z failed");
    size_t sx = 1, sy = n / 2 + 1;
    if (nc > 0) {
        const int nb = col_batch(nc);
        tf::k_spec_columns<<<dim3((nb + 31) / 32, (n + 31) / 32), 256, 0, s>>>(F, n, n / 2 + 1, nc, nb, wk->colbuf);
        if (hipGetLastError() != hipSuccess) return sfail(TF_EDEVICE, "spectrum transpose launch failed");
        const hipfftHandle col = wk->cols[nb];
        F = wk->colbuf;
        if (hipfftSetStream(col, s) != HIPFFT_SUCCESS || hipfftExecZ2Z(col, F, F, HIPFFT_FORWARD) != HIPFFT_SUCCESS)
            return sfail(TF_EDEVICE, "hipfftExecZ2Z failed");
        sx = n;
        sy = 1;
    }
    const double inv_n2 = 1.0 / ((double)n * (double)n);
    tf::k_spec_window<<<(W * W + 255) / 256, 256, 0, s>>>(F, sx, sy, n, E, inv_n2, A);
    tf::k_spec_smooth<0><<<(Wr * W + 255) / 256, 256, 0, s>>>(A, W, W, wd, r, B);
    tf::k_spec_smooth<1><<<(Wr * Wr + 255) / 256, 256, 0, s>>>(B, Wr, W, wd, r, C);
    tf::k_spec_groups<<<(unsigned)(((size_t)ng * tf::SG + 255) / 256), 256, 0, s>>>(C, wk->perm, wk->off, ng, mean);
    if (hipGetLastError() != hipSuccess) return sfail(TF_EDEVICE, "spectrum kernel launch failed");
    if (hipMemcpyAsync(wk->hmean, mean, ng * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess
        || hipStreamSynchronize(s) != hipSuccess)
        return sfail(TF_EDEVICE, "spectrum readback failed");
    int np = 0;
    for (int g = 0; g < ng; ++g) {
        const double q = 2.0 * M_PI * std::sqrt((double)wk->gm[g]) / L;
        if (q > qmax) continue;
        if (np < capacity && q_out != nullptr && s_out != nullptr) {
            q_out[np] = q;
            s_out[np] = wk->hmean[g];
            if (count_out != nullptr) count_out[np] = wk->goff[g + 1] - wk->goff[g];
        }
        ++np;
    }
    *npoints = np;
    if (np > capacity || (np > 0 && (q_out == nullptr || s_out == nullptr)))
        return sfail(TF_EINVAL, "output capacity too small (npoints holds the number needed)");
    return TF_OK;
}

tf_status tf_spectrum_release(void)
{
    std::lock_guard<std::mutex> lk(g_spec_mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (auto &kv : g_spec) {
        (void)hipSetDevice(kv.first.device);
        (void)hipDeviceSynchronize();
        free_work(kv.second);
    }
    g_spec.clear();
    (void)hipSetDevice(cur);
    return TF_OK;
}

tf_status tf_spectrum_maxima(const double *q, const double *s, int npoints, double qmax, int nfine, double *curve_out,
                             double *peak_q, double *peak_s, int capacity, int *npeaks)
{
    if (q == nullptr || s == nullptr || npeaks == nullptr) return sfail(TF_EINVAL, "NULL argument");
    if (npoints < 1 || nfine < 8 || !(qmax > 0.0)) return sfail(TF_EINVAL, "need npoints >= 1, nfine >= 8, qmax > 0");
    for (int p = 0; p < npoints; ++p)
        if (!(q[p] > 0.0) || q[p] > qmax || (p > 0 && !(q[p] > q[p - 1])) || !std::isfinite(s[p]))
            return sfail(TF_EINVAL, "q must increase strictly within (0, qmax] and s be finite");
    // knots: 0, q[9], q[19], ..., qmax; unknowns: the values at knots 1..K
    const int per = 10;
    const int K = std::max(1, npoints / per);
    std::vector<double> t(K + 1);
    t[0] = 0.0;
    for (int k = 1; k < K; ++k) t[k] = q[per * k - 1];
    t[K] = qmax;
    // normal equations of the hat basis: tridiagonal (K x K), unknown j <-> knot j + 1
    std::vector<double> dg(K, 0.0), up(K, 0.0), rhs(K, 0.0);
    int k = 0;
    for (int p = 0; p < npoints; ++p) {
        while (k < K - 1 && q[p] >= t[k + 1]) ++k;
        const double u = (q[p] - t[k]) / (t[k + 1] - t[k]);
        const double wl = 1.0 - u, wr = u; // weights of knots k and k+1
        if (k >= 1) {
            dg[k - 1] += wl * wl;
            up[k - 1] += wl * wr;
            rhs[k - 1] += wl * s[p];
        }
        dg[k] += wr * wr;
        rhs[k] += wr * s[p];
    }
    // symmetric tridiagonal solve (sub-diagonal = up shifted)
    std::vector<double> c(K, 0.0), d(K, 0.0);
    for (int j = 0; j < K; ++j) {
        const double sub = j > 0 ? up[j - 1] : 0.0;
        const double den = dg[j] - (j > 0 ? sub * c[j - 1] : 0.0);
        if (!(std::fabs(den) > 0.0)) return sfail(TF_EINVAL, "degenerate fit (an interval holds no data)");
        c[j] = up[j] / den;
        d[j] = (rhs[j] - (j > 0 ? sub * d[j - 1] : 0.0)) / den;
    }
    std::vector<double> a(K + 1, 0.0);
    for (int j = K - 1; j >= 0; --j) a[j + 1] = d[j] - (j < K - 1 ? c[j] * a[j + 2] : 0.0);
    // the fit on nfine equispaced points of [0, qmax]
    const double hstep = qmax / (nfine - 1);
    std::vector<double> x(nfine), v(nfine), tmp(nfine);
    k = 0;
    for (int j = 0; j < nfine; ++j) {
        x[j] = j == nfine - 1 ? qmax : j * hstep;
        while (k < K - 1 && x[j] >= t[k + 1]) ++k;
        const double u = (x[j] - t[k]) / (t[k + 1] - t[k]);
        v[j] = (1.0 - u) * a[k] + u * a[k + 1];
    }
    // moving averages, half widths 3, 2, 1, windows truncated at the ends
    for (int half : {3, 2, 1}) {
        for (int j = 0; j < nfine; ++j) {
            const int lo = std::max(0, j - half), hi = std::min(nfine - 1, j + half);
            double acc = 0.0;
            for (int i = lo; i <= hi; ++i) acc += v[i];
            tmp[j] = acc / (hi - lo + 1);
        }
        v.swap(tmp);
    }
    if (curve_out != nullptr) std::copy(v.begin(), v.end(), curve_out);
    // maxima: derivative by second-order differences, sign change + to -, second difference < 0
    std::vector<double> dv(nfine);
    for (int j = 1; j < nfine - 1; ++j) dv[j] = (v[j + 1] - v[j - 1]) / (2.0 * hstep);
    dv[0] = (-3.0 * v[0] + 4.0 * v[1] - v[2]) / (2.0 * hstep);
    dv[nfine - 1] = (3.0 * v[nfine - 1] - 4.0 * v[nfine - 2] + v[nfine - 3]) / (2.0 * hstep);
    int np = 0;
    for (int j = 0; j < nfine - 1; ++j) {
        if (!(dv[j] > 0.0 && dv[j + 1] <= 0.0)) continue;
        const double u = dv[j] / (dv[j] - dv[j + 1]);
        int jj = u < 0.5 ? j : j + 1;
        jj = std::min(std::max(jj, 1), nfine - 2);
        if (!(v[jj + 1] - 2.0 * v[jj] + v[jj - 1] < 0.0)) continue;
        if (np < capacity && peak_q != nullptr && peak_s != nullptr) {
            peak_q[np] = x[j] + u * hstep;
            peak_s[np] = v[j] + u * (v[j + 1] - v[j]);
        }
        ++np;
    }
    *npeaks = np;
    if (np > capacity) return sfail(TF_EINVAL, "peak capacity too small (npeaks holds the number found)");
    return TF_OK;
}

} // extern "C"
