// Device parts of the thin-plate smoothing of the prior grid shared by the finalize
// kernels and the run kernel: the parity basis of the grid and the GCV score.
#pragma once

#include "m2m_device.h"

namespace m2m {
namespace {

// GCV score (RSS/n) / (1 - tr(A)/n)^2 of the spectral smoother at P values
// of lambda, summed by one wave over the n eigenvalues (in g2) and the
// transformed data (in wh); 1 / (1 + t) is a hardware reciprocal refined by two Newton
// steps (within an ulp or two), as the score only ranks the lambdas.
template <int P>
__device__ __forceinline__ void gcv_points(const double* g2, const double* wh, int n, int lane,
                                           const double* lam, double* out) {
    double rss[P], den[P];
#pragma unroll
    for (int j = 0; j < P; ++j) rss[j] = den[j] = 0.0;
    for (int c = lane; c < n; c += 64) {
        const double g = g2[c], w = wh[c];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const double t = lam[j] * g;
            const double d = 1.0 + t;
            double iv = __builtin_amdgcn_rcp(d);
            iv = fma(iv, fma(-d, iv, 1.0), iv);
            iv = fma(iv, fma(-d, iv, 1.0), iv);
            const double r = t * iv;
            const double e = r * w;
            rss[j] = fma(e, e, rss[j]);
            den[j] += r;
        }
    }
#pragma unroll
    for (int j = 0; j < P; ++j) {
        for (int off = 32; off >= 1; off >>= 1) {
            rss[j] += __shfl_xor(rss[j], off, 64);
            den[j] += __shfl_xor(den[j], off, 64);
        }
        out[j] = (rss[j] / n) / ((den[j] / n) * (den[j] / n));
    }
}

// Parity blocks of an axis of n cells: (n+1)/2 even and n/2 odd vectors.
// Coefficient of cell k in vector i of parity p (cells i and n-1-i).
__device__ __forceinline__ double fold_coef(int n, int p, int i, int k) {
    const int i2 = n - 1 - i;
    if (i == i2) return (p == 0 && k == i) ? 1.0 : 0.0;
    const double s = 0.70710678118654752440;
    if (k == i) return s;
    if (k == i2) return p == 0 ? s : -s;
    return 0.0;
}

// The four parity blocks of an n_E x n_x grid: block b = 2 pE + pX holds
// mE(pE) mX(pX) folded coefficients from off(b) and its eigenvectors from
// qoff(b) in the basis (scalars and selects, no indexed arrays, so that
// nothing goes to scratch memory).
struct SmBlocks {
    int mE0, mE1, mX0, mX1;
    int o1, o2, o3, o4;  // off(1..4); off(0) = 0
    int q0, q1, q2, q3;  // qoff(0..3)
    __device__ int mE(int p) const { return p ? mE1 : mE0; }
    __device__ int mX(int p) const { return p ? mX1 : mX0; }
    __device__ int off(int b) const {
        return b == 0 ? 0 : (b == 1 ? o1 : (b == 2 ? o2 : (b == 3 ? o3 : o4)));
    }
    __device__ int qoff(int b) const { return b == 0 ? q0 : (b == 1 ? q1 : (b == 2 ? q2 : q3)); }
    // the block of folded index c (0 <= c < n_E n_x)
    __device__ int block_of(int c) const { return c < o1 ? 0 : (c < o2 ? 1 : (c < o3 ? 2 : 3)); }
};

__device__ __forceinline__ SmBlocks sm_blocks(int nE, int nx) {
    SmBlocks B;
    B.mE0 = (nE + 1) / 2;
    B.mE1 = nE / 2;
    B.mX0 = (nx + 1) / 2;
    B.mX1 = nx / 2;
    const int m0 = B.mE0 * B.mX0, m1 = B.mE0 * B.mX1, m2 = B.mE1 * B.mX0, m3 = B.mE1 * B.mX1;
    B.o1 = m0;
    B.o2 = m0 + m1;
    B.o3 = m0 + m1 + m2;
    B.o4 = m0 + m1 + m2 + m3;
    B.q0 = nE * nx;
    B.q1 = B.q0 + m0 * m0;
    B.q2 = B.q1 + m1 * m1;
    B.q3 = B.q2 + m2 * m2;
    return B;
}

// Fold: folded coefficient c from its (up to) four cells (k, l) with
// k in {i, nE-1-i}, l in {j, nx-1-j}; w0(q) the data of cell q.
template <typename F>
__device__ __forceinline__ double fold_cell(const SmBlocks& B, int nE, int nx, int c, F w0) {
    const int b = B.block_of(c), pE = b >> 1, pX = b & 1;
    const int r = c - B.off(b), i = r / B.mX(pX), j = r - i * B.mX(pX);
    const int k1 = nE - 1 - i, l1 = nx - 1 - j;
    const double ce0 = fold_coef(nE, pE, i, i), ce1 = k1 != i ? fold_coef(nE, pE, i, k1) : 0.0;
    const double cx0 = fold_coef(nx, pX, j, j), cx1 = l1 != j ? fold_coef(nx, pX, j, l1) : 0.0;
    double v = ce0 * cx0 * w0(i * nx + j);
    if (l1 != j) v += ce0 * cx1 * w0(i * nx + l1);
    if (k1 != i) {
        v += ce1 * cx0 * w0(k1 * nx + j);
        if (l1 != j) v += ce1 * cx1 * w0(k1 * nx + l1);
    }
    return v;
}

// Unfold: cell (k, l) from the vectors of both parities that touch it; s(bb, i, j)
// the folded coefficient (i, j) of parity block bb.
template <typename F>
__device__ __forceinline__ double unfold_cell(const SmBlocks& B, int nE, int nx, int k, int l, F s) {
    const int i = min(k, nE - 1 - k), j = min(l, nx - 1 - l);
    double v = 0.0;
    for (int pE = 0; pE < 2; ++pE) {
        if (i >= B.mE(pE)) continue;
        const double ce = fold_coef(nE, pE, i, k);
        if (ce == 0.0) continue;
        for (int pX = 0; pX < 2; ++pX) {
            if (j >= B.mX(pX)) continue;
            const double cx = fold_coef(nx, pX, j, l);
            if (cx == 0.0) continue;
            v += ce * cx * s(2 * pE + pX, i, j);
        }
    }
    return v;
}

}  // namespace
}  // namespace m2m
