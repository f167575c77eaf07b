// Design-field front end (Sec. 2.1): the linear density filter
//   chi_fil_e = sum_i w_ei chi_i / sum_i w_ei,   w_ei = max(0, r_fil - |x_e - x_i|)
// over element centroids x_e = ((i + 1/2)/nx, (j + 1/2)/ny), followed by the
// threshold projection
//   chi_phys = (tanh(beta (chi_fil - eta)) + tanh(beta eta))
//              / (tanh(beta (1 - eta)) + tanh(beta eta)),
// and its adjoint: grad_chi = H^T (P'(chi_fil) o grad_phys). The weights are
// symmetric in (e, i), so H^T y at i is sum_e w_ei y_e / W_e over the same
// neighbourhood.
//
// Both directions are one weighted sum over the neighbourhood (k_filter_sum)
// with FP64 FMAs as the bound: about 2 pi r^2 nx ny flops per element. W_e depends
// on the element's distance to the edges only and comes from sums of the weights
// over rectangles.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "pt.h"

namespace {

struct Geom {
    int nx, ny, Rx, Ry;
    double r;
};

constexpr int kBX = 16, kBY = 16;
constexpr long long kMaxWindow = 1ll << 18;  // neighbourhood cells per element

__device__ __forceinline__ double cone(const Geom &g, int di, int dj) {
    const double dx = (double)di / g.nx, dy = (double)dj / g.ny;
    return fmax(0.0, g.r - sqrt(dx * dx + dy * dy));
}

__device__ __forceinline__ double weight_sum(const Geom &g, int i, int j) {
    double W = 0.0;
    for (int dj = max(-g.Ry, -j); dj <= min(g.Ry, g.ny - 1 - j); ++dj)
        for (int di = max(-g.Rx, -i); di <= min(g.Rx, g.nx - 1 - i); ++di) W += cone(g, di, dj);
    return W;
}

__device__ __forceinline__ double proj(double f, double beta, double eta) {
    if (!(beta > 0.0)) return f;
    const double den = tanh(beta * (1.0 - eta)) + tanh(beta * eta);
    return (tanh(beta * (f - eta)) + tanh(beta * eta)) / den;
}

__device__ __forceinline__ double proj_deriv(double f, double beta, double eta) {
    if (!(beta > 0.0)) return 1.0;
    const double den = tanh(beta * (1.0 - eta)) + tanh(beta * eta);
    const double t = tanh(beta * (f - eta));
    return beta * (1.0 - t * t) / den;
}

// ---------------------------------------------------------------------------
// Windows that fit the LDS in pieces
// ---------------------------------------------------------------------------

constexpr int kTX = 64, kThr = 512;      // output columns, threads of a block
constexpr int kWaves = kThr / 64;        // output rows: T per wave
constexpr int kMinRows = 32;             // rows staged at once, at least
constexpr size_t kLdsMax = 158 * 1024;

// Doubles of the sums of weights over rectangles: prefix sums over 1..Rx x 1..Ry
// and along both axes.
__host__ __device__ inline size_t rect_doubles(const Geom &g) {
    return (size_t)(g.Rx + 1) * (g.Ry + 1) + (g.Rx + 1) + (g.Ry + 1);
}

// Fills P with Q[a][b] = sum of w(1..a, 1..b), X[a] = sum of w(1..a, 0) and
// Y[b] = sum of w(0, 1..b); all threads of the block call it.
__device__ void rect_sums(const Geom &g, double *P) {
    const int nb = g.Ry + 1;
    double *X = P + (size_t)(g.Rx + 1) * nb, *Y = X + g.Rx + 1;
    for (int k = threadIdx.x; k < (g.Rx + 1) * nb; k += kThr) {
        const int a = k / nb, b = k - a * nb;
        P[k] = a > 0 && b > 0 ? cone(g, a, b) : 0.0;
    }
    for (int a = threadIdx.x; a <= g.Rx; a += kThr) X[a] = a > 0 ? cone(g, a, 0) : 0.0;
    for (int b = threadIdx.x; b <= g.Ry; b += kThr) Y[b] = b > 0 ? cone(g, 0, b) : 0.0;
    __syncthreads();
    for (int a = threadIdx.x; a <= g.Rx + 2; a += kThr) {
        double *p = a <= g.Rx ? P + (size_t)a * nb : a == g.Rx + 1 ? X : Y;
        const int m = a <= g.Rx ? g.Ry : a == g.Rx + 1 ? g.Rx : g.Ry;
        double v = 0.0;
        for (int b = 1; b <= m; ++b) p[b] = v += p[b];
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += kThr) {
        double v = 0.0;
        for (int a = 1; a <= g.Rx; ++a) P[(size_t)a * nb + b] = v += P[(size_t)a * nb + b];
    }
    __syncthreads();
}

// W of element (i, j): the window reaches a0, a1 columns and b0, b1 rows.
__device__ __forceinline__ double rect_weight(const Geom &g, const double *P, int i, int j) {
    const int nb = g.Ry + 1;
    const double *X = P + (size_t)(g.Rx + 1) * nb, *Y = X + g.Rx + 1;
    const int a0 = min(g.Rx, i), a1 = min(g.Rx, g.nx - 1 - i);
    const int b0 = min(g.Ry, j), b1 = min(g.Ry, g.ny - 1 - j);
    return cone(g, 0, 0) + (X[a0] + X[a1]) + (Y[b0] + Y[b1]) +
           ((P[a0 * nb + b0] + P[a0 * nb + b1]) + (P[a1 * nb + b0] + P[a1 * nb + b1]));
}

// The direct sum at one element.
__device__ double direct_sum(const Geom &g, const double *x, int i, int j) {
    double s = 0.0;
    for (int dj = max(-g.Ry, -j); dj <= min(g.Ry, g.ny - 1 - j); ++dj) {
        const double *row = x + (size_t)(j + dj) * g.nx + i;
        for (int di = max(-g.Rx, -i); di <= min(g.Rx, g.nx - 1 - i); ++di)
            s += cone(g, di, dj) * row[di];
    }
    return s;
}

// out_e = sum_i w_ei x_i (ADJ), or that over W_e and its projection. A wave holds
// T rows of 64 columns; the block's input and halo are in LDS (rc_max rows at a
// time), rows of x(+di) + x(-di) are formed once for T outputs, and the weights of
// a column distance lie in LDS too, formed once by all threads (two buffers, one
// barrier per distance). Bound by the LDS: per input row and column distance a
// thread reads two values and about two weights for T FMAs. Eight waves of 8 rows
// hide its latency better than four of 16 on the same tile (0.32 against 0.36 ms).
// 1024^2 elements, r = 0.03 (2965 weights): forward and backward 13.5 -> 0.32 ms
// against one thread per element with weights formed in place.
template <int T, bool ADJ>
__global__ void __launch_bounds__(kThr)
k_filter_sum(Geom g, double beta, double eta, int rc_max, const double *__restrict__ x,
             double *__restrict__ fil, double *__restrict__ out) {
    extern __shared__ double lds[];
    const int LW = kTX + 2 * g.Rx, WL = 2 * g.Ry + 4 * T;
    double *wt = lds, *buf = lds + 2 * WL;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = blockIdx.x * kTX, j0 = blockIdx.y * (kWaves * T);
    const int rows = kWaves * T + 2 * g.Ry;
    double acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = 0.0;
    bool odd = false;  // values that a zero weight or a pair's sum would change
    for (int c0 = 0; c0 < rows; c0 += rc_max) {
        const int rc = min(rc_max, rows - c0);
        __syncthreads();
        // rows c0 .. c0 + rc - 1 of the window and T rows of zeros
        for (int r = wave; r < rc + T; r += kWaves) {
            const int y = j0 - g.Ry + c0 + r;
            const bool in = r < rc && y >= 0 && y < g.ny;
            for (int c = lane; c < LW; c += 64) {
                const int xx = i0 - g.Rx + c;
                double v = 0.0;
                if (in && xx >= 0 && xx < g.nx) v = x[(size_t)y * g.nx + xx];
                odd |= !(fabs(v) <= 1e300);
                buf[r * LW + c] = v;
            }
        }
        for (int di = 0; di <= g.Rx; ++di) {
            // rows beyond H have weight 0 (one more for the rounding of the root)
            const double dx = (double)di / g.nx;
            const int H = min(g.Ry, (int)(g.ny * sqrt(fmax(0.0, g.r * g.r - dx * dx))) + 1);
            double *w = wt + (di & 1) * WL;
            for (int k = threadIdx.x; k < 2 * H + 4 * T - 3; k += kThr)
                w[k] = (di == 0 ? 0.5 : 1.0) * cone(g, di, k - (H + 2 * T - 2));
            __syncthreads();
            // row q of the wave's outputs lies at row base + q of the piece
            const int base = wave * T + g.Ry - c0;
            const int lo = max(-H, -base), hi = min(T - 1 + H, rc - 1 - base);
            for (int q = lo; q <= hi; q += T) {
                const double *b0 = buf + (base + q) * LW + lane + g.Rx;
                const double *wq = w + (q + H + T - 1);
                double xr[T], wv[2 * T - 1];
#pragma unroll
                for (int u = 0; u < T; ++u) xr[u] = b0[u * LW + di] + b0[u * LW - di];
#pragma unroll
                for (int m = 0; m < 2 * T - 1; ++m) wv[m] = wq[m];
#pragma unroll
                for (int u = 0; u < T; ++u)
#pragma unroll
                    for (int t = 0; t < T; ++t) acc[t] += wv[u - t + T - 1] * xr[u];
            }
        }
    }
    const bool direct = __syncthreads_or(odd) != 0;
    if constexpr (!ADJ) rect_sums(g, lds);
    const int i = i0 + lane;
    if (i >= g.nx) return;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int j = j0 + wave * T + t;
        if (j >= g.ny) break;
        const double s = direct ? direct_sum(g, x, i, j) : acc[t];
        const size_t e = (size_t)j * g.nx + i;
        if constexpr (ADJ) {
            out[e] = s;
        } else {
            const double f = s / rect_weight(g, lds, i, j);
            if (fil) fil[e] = f;
            out[e] = proj(f, beta, eta);
        }
    }
}

// work_e = P'(chi_fil_e) grad_phys_e / W_e, every block with its own sums of weights
__global__ void __launch_bounds__(kThr)
k_filter_scale_rect(Geom g, double beta, double eta, const double *__restrict__ fil,
                    const double *__restrict__ grad_phys, double *__restrict__ work) {
    extern __shared__ double lds[];
    rect_sums(g, lds);
    const size_t n = (size_t)g.nx * g.ny;
    for (size_t e = (size_t)blockIdx.x * kThr + threadIdx.x; e < n; e += (size_t)gridDim.x * kThr) {
        const int j = (int)(e / g.nx), i = (int)(e - (size_t)j * g.nx);
        work[e] = proj_deriv(fil[e], beta, eta) * grad_phys[e] / rect_weight(g, lds, i, j);
    }
}

// ---------------------------------------------------------------------------
// Larger windows, and few elements: one thread per element, the neighbourhood
// through the caches
// ---------------------------------------------------------------------------

__global__ void k_filter_forward(Geom g, double beta, double eta, const double *__restrict__ chi,
                                 double *__restrict__ fil, double *__restrict__ phys) {
    const int i = blockIdx.x * kBX + threadIdx.x;
    const int j = blockIdx.y * kBY + threadIdx.y;
    if (i >= g.nx || j >= g.ny) return;
    double s = 0.0, W = 0.0;
    for (int dj = max(-g.Ry, -j); dj <= min(g.Ry, g.ny - 1 - j); ++dj) {
        const double *row = chi + (size_t)(j + dj) * g.nx + i;
        for (int di = max(-g.Rx, -i); di <= min(g.Rx, g.nx - 1 - i); ++di) {
            const double w = cone(g, di, dj);
            s += w * row[di];
            W += w;
        }
    }
    const double f = s / W;
    const size_t e = (size_t)j * g.nx + i;
    if (fil) fil[e] = f;
    phys[e] = proj(f, beta, eta);
}

// work_e = P'(chi_fil_e) grad_phys_e / W_e
__global__ void k_filter_scale(Geom g, double beta, double eta, const double *__restrict__ fil,
                               const double *__restrict__ grad_phys, double *__restrict__ work) {
    const int i = blockIdx.x * kBX + threadIdx.x;
    const int j = blockIdx.y * kBY + threadIdx.y;
    if (i >= g.nx || j >= g.ny) return;
    const size_t e = (size_t)j * g.nx + i;
    work[e] = proj_deriv(fil[e], beta, eta) * grad_phys[e] / weight_sum(g, i, j);
}

// grad_chi_i = sum_e w_ei work_e
__global__ void k_filter_adjoint(Geom g, const double *__restrict__ work,
                                 double *__restrict__ grad_chi) {
    const int i = blockIdx.x * kBX + threadIdx.x;
    const int j = blockIdx.y * kBY + threadIdx.y;
    if (i >= g.nx || j >= g.ny) return;
    grad_chi[(size_t)j * g.nx + i] = direct_sum(g, work, i, j);
}

bool make_geom(const pt_filter *f, Geom &g) {
    if (!f) return false;
    if (f->nx < 1 || f->ny < 1 || f->nx > 16384 || f->ny > 16384) return false;
    if (!(f->r_fil > 0.0) || !std::isfinite(f->r_fil)) return false;
    if (!std::isfinite(f->beta) || !std::isfinite(f->eta) || f->eta < 0.0 || f->eta > 1.0)
        return false;
    g.nx = f->nx;
    g.ny = f->ny;
    g.r = f->r_fil;
    // |di|/nx < r for a positive weight; beyond the grid nothing is read
    const double rx = std::floor(f->r_fil * f->nx), ry = std::floor(f->r_fil * f->ny);
    g.Rx = (int)std::fmin(rx, (double)(f->nx - 1));
    g.Ry = (int)std::fmin(ry, (double)(f->ny - 1));
    if ((long long)(2 * g.Rx + 1) * (2 * g.Ry + 1) > kMaxWindow) return false;
    return true;
}

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
    if (!a || !b) return false;
    const char *pa = (const char *)a, *pb = (const char *)b;
    return pa < pb + nb && pb < pa + na;
}

// Rows per wave, rows staged at once and LDS of k_filter_sum; T = 0 where the window
// is too large. 8 rows where the blocks fill the device (4 rows read as much LDS per
// row for half the outputs); 4 below, where half the blocks would idle.
struct SumPlan {
    int T, rc;
    size_t lds;
};

SumPlan sum_plan(const Geom &g) {
    auto blocks = [&](int T) {
        return (long long)((g.nx + kTX - 1) / kTX) * ((g.ny + kWaves * T - 1) / (kWaves * T));
    };
    SumPlan P{0, 0, 0};
    if (rect_doubles(g) * sizeof(double) > kLdsMax) return P;
    for (int T : {8, 4}) {
        if (T == 8 && blocks(8) < 200) continue;
        const size_t row = sizeof(double) * (kTX + 2 * (size_t)g.Rx);
        const size_t wts = sizeof(double) * 2 * (2 * (size_t)g.Ry + 4 * T);
        if (wts + row * (kMinRows + T) > kLdsMax) continue;
        P.T = T;
        P.rc = (int)std::fmin((double)(kWaves * T + 2 * g.Ry), (double)((kLdsMax - wts) / row - T));
        P.lds = std::max(wts + row * (P.rc + T), sizeof(double) * rect_doubles(g));
        break;
    }
    return P;
}

// Whether one thread per element takes less time than the tiles, for a direction of
// `sums` sums per element (the backward one also sums the weights). Where the tiles do
// not fill the device both are chains: one thread's terms, each 0.11 us or, with many
// elements, the time of them all; a tile's column distances, 1 us and 0.17 us per T
// rows of the window, for each piece of rows that is staged. Forward, us, one thread
// per element against tiles:
//    100^2, r = 0.03 (49 terms, the paper's filter)   11 against 16
//    199 x 150, r = 0.03 (99)                         16 against 28
//    16384 x 1, r = 0.01 (327 in a row)               40 against 287
//    300 x 12, r = 0.8 (3600)                        404 against 707
//    256^2, r = 0.03 (225)                            31 against 25
//    64^2, r = 0.2 (625)                              74 against 38
bool direct_pays(const Geom &g, const SumPlan &P, int sums) {
    const int rows = kWaves * P.T;
    const long long tiles = (long long)((g.nx + kTX - 1) / kTX) * ((g.ny + rows - 1) / rows);
    if (tiles > 256) return false;
    const double terms = (double)std::min(2 * g.Rx + 1, g.nx) * std::min(2 * g.Ry + 1, g.ny);
    const double term = std::max(0.11, 1.33e-6 * (double)g.nx * g.ny);
    const int pieces = (rows + 2 * g.Ry + P.rc - 1) / P.rc;
    const double tile = 8.5 + pieces * (g.Rx + 1) * (1.0 + 0.17 * ((2 * g.Ry + 2 * P.T - 1) / P.T));
    return sums * (5.0 + terms * term) < tile + 4.0 * (sums - 1);
}

template <bool ADJ>
int launch_sum(const Geom &g, const SumPlan &P, double beta, double eta, const double *x,
               double *fil, double *out, hipStream_t stream) {
    auto kern = P.T == 8 ? k_filter_sum<8, ADJ> : k_filter_sum<4, ADJ>;
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)P.lds) != hipSuccess)
        return PT_EHIP;
    const dim3 grid((g.nx + kTX - 1) / kTX, (g.ny + kWaves * P.T - 1) / (kWaves * P.T));
    hipLaunchKernelGGL(kern, grid, dim3(kThr), P.lds, stream, g, beta, eta, P.rc, x, fil, out);
    return hipGetLastError() == hipSuccess ? PT_OK : PT_EHIP;
}

int launched() { return hipGetLastError() == hipSuccess ? PT_OK : PT_EHIP; }

}  // namespace

extern "C" int pt_filter_validate(const pt_filter *f) {
    Geom g;
    return make_geom(f, g) ? PT_OK : PT_EINVAL;
}

extern "C" int pt_filter_projection(const pt_filter *f, const double *chi, double *chi_fil,
                                    double *chi_phys, hipStream_t stream) {
    Geom g;
    if (!make_geom(f, g) || !chi || !chi_phys) return PT_EINVAL;
    const size_t n = (size_t)g.nx * g.ny * sizeof(double);
    if (overlap(chi, n, chi_phys, n) || overlap(chi, n, chi_fil, n) ||
        overlap(chi_fil, n, chi_phys, n))
        return PT_EINVAL;
    const SumPlan P = sum_plan(g);
    if (P.T > 0 && !direct_pays(g, P, 1))
        return launch_sum<false>(g, P, f->beta, f->eta, chi, chi_fil, chi_phys, stream);
    const dim3 grid((g.nx + kBX - 1) / kBX, (g.ny + kBY - 1) / kBY), block(kBX, kBY);
    hipLaunchKernelGGL(k_filter_forward, grid, block, 0, stream, g, f->beta, f->eta, chi, chi_fil,
                       chi_phys);
    return launched();
}

extern "C" int pt_filter_projection_backward(const pt_filter *f, const double *chi_fil,
                                             const double *grad_phys, double *work,
                                             double *grad_chi, hipStream_t stream) {
    Geom g;
    if (!make_geom(f, g) || !chi_fil || !grad_phys || !work || !grad_chi) return PT_EINVAL;
    const size_t n = (size_t)g.nx * g.ny * sizeof(double);
    if (overlap(work, n, grad_chi, n) || overlap(work, n, chi_fil, n) ||
        overlap(work, n, grad_phys, n) || overlap(grad_chi, n, chi_fil, n) ||
        overlap(grad_chi, n, grad_phys, n))
        return PT_EINVAL;
    const SumPlan P = sum_plan(g);
    if (P.T > 0 && !direct_pays(g, P, 2)) {
        const size_t lds = sizeof(double) * rect_doubles(g);
        if (hipFuncSetAttribute((const void *)k_filter_scale_rect,
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return PT_EHIP;
        const long long n1 = ((long long)g.nx * g.ny + 4 * kThr - 1) / (4 * kThr);
        hipLaunchKernelGGL(k_filter_scale_rect, dim3((unsigned)std::min(n1, 1024ll)), dim3(kThr),
                           lds, stream, g, f->beta, f->eta, chi_fil, grad_phys, work);
        if (hipGetLastError() != hipSuccess) return PT_EHIP;
        return launch_sum<true>(g, P, 0.0, 0.0, work, nullptr, grad_chi, stream);
    }
    const dim3 grid((g.nx + kBX - 1) / kBX, (g.ny + kBY - 1) / kBY), block(kBX, kBY);
    hipLaunchKernelGGL(k_filter_scale, grid, block, 0, stream, g, f->beta, f->eta, chi_fil,
                       grad_phys, work);
    hipLaunchKernelGGL(k_filter_adjoint, grid, block, 0, stream, g, work, grad_chi);
    return launched();
}
