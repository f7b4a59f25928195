// bte_direct.hip -- the diffusion operators of a geometry without pores and
// with one conductivity per axis, solved by their eigenvectors.
//
// Such an operator (heat-diffusion guess, synthetic correction) is a sum of
// one-dimensional ones, L = sum_a L_a, each with constant couplings
// c = k_a / h_a^2 and one boundary condition per end, so L is diagonal in the
// products of the axes' eigenvectors: x = V ((V^T b) / lambda), one dense
// product per axis and direction.  The products are 4 launches in 2D whatever
// the conditioning; CG takes about 600 iterations at 3.0 us on 97 x 83 cells
// (relative residual 1e-10) and 1 660 at 4.0 us for the guess on 256^2 (1e-13).
//
// Eigenpairs in closed form: with v_(-1) = a v_0 and v_n = b v_(n-1) at the
// ends (a, b = 1 - the wall's share of c; 1: zero flux, -1: fixed value at the
// face), v_i = sin((i + 1) t) - a sin(i t), lambda = 4 c sin^2(t / 2), and the
// n values of t in [0, pi) solve
//   (n - 1) t + arg(e^(i t) - a) + arg(e^(i t) - b) = m pi,  m = 1 .. n
// (the left side grows with t for |a|, |b| <= 1).  Periodic axes: cosines and
// sines.
#include "bte_internal.h"

#include <algorithm>
#include <cmath>

namespace bte {

// t of eigenvector m of one axis of n cells; al, ar: wall conductance at the
// ends in units of c (0: zero flux, at most 2).
double axis_angle(int n, bool periodic, double al, double ar, int m)
{
    if (periodic) return 2.0 * M_PI * ((m + 1) / 2) / n;
    const double a = 1.0 - al, b = 1.0 - ar;
    if (a == 1.0 && b == 1.0) return M_PI * m / n;
    auto phase = [&](double th) {
        // arg(e^(i th) - 1) = (th + pi) / 2 and arg(e^(i th) + 1) = th / 2 also
        // at 0 and pi
        auto arg = [&](double z) {
            return z == 1.0 ? 0.5 * (th + M_PI) : z == -1.0 ? 0.5 * th : std::atan2(std::sin(th), std::cos(th) - z);
        };
        return (n - 1) * th + arg(a) + arg(b) - (m + 1) * M_PI;
    };
    double lo = 0.0, hi = M_PI;
    for (int k = 0; k < 60; ++k) {
        const double mid = 0.5 * (lo + hi);
        (phase(mid) < 0.0 ? lo : hi) = mid;
    }
    return 0.5 * (lo + hi);
}

// V[n][n] (column m: eigenvector m, unit length) and lambda[n] of one axis.
void axis_eigen(int n, double c, bool periodic, double al, double ar, double *V, double *lambda)
{
    const double a = 1.0 - al, b = 1.0 - ar;
    for (int m = 0; m < n; ++m) {
        double *col = V + m;
        const double t = axis_angle(n, periodic, al, ar, m);
        if (periodic) {
            for (int i = 0; i < n; ++i) col[(size_t)i * n] = (m & 1) || m == 0 ? std::cos(t * i) : std::sin(t * i);
        } else if (a == 1.0) {
            for (int i = 0; i < n; ++i) col[(size_t)i * n] = std::cos(t * (i + 0.5));
        } else if (b == 1.0) {
            for (int i = 0; i < n; ++i) col[(size_t)i * n] = std::cos(t * (n - 1 - i + 0.5));
        } else if (a == -1.0) {
            for (int i = 0; i < n; ++i) col[(size_t)i * n] = std::sin(t * (i + 0.5));
        } else if (b == -1.0) {
            for (int i = 0; i < n; ++i) col[(size_t)i * n] = std::sin(t * (n - 1 - i + 0.5));
        } else {
            for (int i = 0; i < n; ++i) col[(size_t)i * n] = std::sin((i + 1) * t) - a * std::sin(i * t);
        }
        double s = 0.0;
        for (int i = 0; i < n; ++i) s += col[(size_t)i * n] * col[(size_t)i * n];
        s = 1.0 / std::sqrt(s);
        for (int i = 0; i < n; ++i) col[(size_t)i * n] *= s;
        const double h = std::sin(0.5 * t);
        lambda[m] = 4.0 * c * h * h;
    }
}

namespace {

constexpr int kDT = 16;   // outputs of a block along the transformed axis and across it

typedef double double4_t __attribute__((ext_vector_type(4)));

// One axis: out[o][j][q] = sum_i M[j][i] in[o][i][q], M = V^T (fwd) or V;
// columns are numbered o inner + q.  The last forward axis divides by the
// eigenvalue of the operator (0 for its null vector).  The last axis back
// (fin) gives 0 where the sum is not finite, that is everywhere if one value
// of b is not: CG, too, returns 0 for such a b.
// A block takes 16 x 16 outputs on the FP64 matrix cores (16 x 16 x 4); its
// four wavefronts split the sum over i, so that the few outputs of a line or a
// small plane still keep loads in flight, straight from the caches: both
// factors are read once or a few times and are small.  Correction (the
// products and the update of T_L) of a line of 200 cells, 97 x 83, 256^2, 64^3,
// 128^3: 50, 63, 155, 76, 295 us with tiles of 32 x 32 through LDS on the vector
// units, 16, 21, 29, 52, 250 us here.
__global__ __launch_bounds__(256) void k_axis_product(const double *__restrict__ in, double *__restrict__ out,
                                                      const double *__restrict__ V, int n, int inner, int cols, int fwd,
                                                      const double *__restrict__ lx, const double *__restrict__ ly,
                                                      const double *__restrict__ lz, int n0, int n1, double zero, int fin)
{
    constexpr int U = 8;   // steps of 4 in flight
    __shared__ double sm[4][kDT][kDT + 1];
    const int j0 = blockIdx.x * kDT, q0 = blockIdx.y * kDT;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
    // operands of this lane: M[j0 + l16][i], in[i][column q0 + l16], i = 4 step + l4
    const int ja = min(j0 + l16, n - 1), qa = min(q0 + l16, cols - 1);
    const double *pa = fwd ? V + ja : V + (size_t)ja * n;
    const double *pb = in + (size_t)(qa / inner) * n * inner + qa % inner;
    const size_t sa = fwd ? n : 1, sb = inner;
    const int steps = (n + 3) / 4;
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    for (int s0 = wave; s0 < steps; s0 += 4 * U) {
        double a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = 4 * (s0 + 4 * u) + l4, ic = min(i, n - 1);
            a[u] = pa[ic * sa];
            b[u] = pb[ic * sb];
            if (i >= n) a[u] = b[u] = 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
    // element r of a lane: row 4 r + l4, column l16
#pragma unroll
    for (int r = 0; r < 4; ++r) sm[wave][4 * r + l4][l16] = acc[r];
    __syncthreads();
    const int hi = threadIdx.x >> 4, lo = threadIdx.x & 15;   // consecutive threads along memory
    const int jr = inner == 1 ? lo : hi, qr = inner == 1 ? hi : lo, j = j0 + jr, q = q0 + qr;
    if (j >= n || q >= cols) return;
    const size_t at = ((size_t)(q / inner) * n + j) * inner + q % inner;
    double v = (sm[0][jr][qr] + sm[1][jr][qr]) + (sm[2][jr][qr] + sm[3][jr][qr]);
    if (lx) {
        const int i = (int)at;
        const double l = lx[i % n0] + (ly ? ly[i / n0 % n1] : 0.0) + (lz ? lz[i / (n0 * n1)] : 0.0);
        v = l > zero ? v / l : 0.0;
    }
    out[at] = fin && !isfinite(v) ? 0.0 : v;
}

}  // namespace

// x = L^-1 b (the part of b in L's null space dropped).  V, lam: device, axis
// after axis (n_a^2 and n_a values); tmp: two buffers of nc doubles; zero:
// eigenvalues up to it are the null vector's.
hipError_t launch_direct(int dim, const int *n, const double *V, const double *lam, const double *b, double *x,
                         double *tmp0, double *tmp1, double zero, hipStream_t s)
{
    const double *Va[3] = {V, V + (size_t)n[0] * n[0], V + (size_t)n[0] * n[0] + (size_t)n[1] * n[1]};
    const double *la[3] = {lam, lam + n[0], lam + n[0] + n[1]};
    const int nc = n[0] * n[1] * n[2], inner[3] = {1, n[0], n[0] * n[1]};
    const double *src = b;
    for (int k = 0; k < 2 * dim; ++k) {
        const int a = k < dim ? k : k - dim;
        const bool fwd = k < dim, last = k == dim - 1;
        double *dst = k == 2 * dim - 1 ? x : (k & 1) ? tmp1 : tmp0;
        const int cols = nc / n[a];
        hipLaunchKernelGGL(k_axis_product, dim3((n[a] + kDT - 1) / kDT, (cols + kDT - 1) / kDT), dim3(256), 0, s, src, dst,
                           Va[a], n[a], inner[a], cols, fwd ? 1 : 0, last ? la[0] : nullptr,
                           last && dim > 1 ? la[1] : nullptr, last && dim > 2 ? la[2] : nullptr, n[0], n[1], zero,
                           k == 2 * dim - 1 ? 1 : 0);
        src = dst;
    }
    return hipGetLastError();
}

}  // namespace bte
