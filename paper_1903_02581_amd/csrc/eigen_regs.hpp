// Hermitian (or real symmetric) tridiagonalisation by one workgroup with the
// matrix in registers, and Sturm counts of the result (FP64).
//
// A 1024-thread block holds the matrix as a 32 x 32 thread grid with cyclic
// ownership: thread (tr, tc) keeps elements (tr + 32 a, tc + 32 b), a, b < NB, so
// every thread stays busy as the active window shrinks and NB = 4 carries 128 x
// 128 complex values in 64 VGPRs of each of the 1024 threads; LDS only moves the
// two vectors of a step.  (The matrix itself does not fit 160 KB of LDS at 128 x
// 128 complex, and a pass over it in L2 per step is what bounds larger sizes,
// tridiag_global below.)
//
// Step s, with x the column s below the diagonal: the reflector
// H = 1 - tau v v^H, v = x + (x_0 / |x_0|) ||x|| e_0, tau = 1 / (||x||^2 + |x_0| ||x||)
// (Golub and Van Loan, Householder tridiagonalisation) maps x to
// -(x_0 / |x_0|) ||x|| e_0; with p = A v and w = tau p - (tau^2 / 2) (v^H p) v the
// window becomes A - v w^H - w v^H.  Two barriers per step: one after the
// column is in LDS, one after p is.  Each wavefront forms ||x||^2 and v^H p for
// itself, from the same LDS values in the same order, so that every thread holds
// the same bits and takes the same branches.  The chain of these steps, not the
// arithmetic, bounds it: one block, 2 barriers and 2 wavefront reductions a step.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dft_regs.hpp"

namespace hom4d_impl {
namespace eig {
using namespace hom4d_dev;

constexpr int kThreads = 1024;  // 32 x 32 threads
constexpr int kRegMax = 128;    // largest matrix held in registers (NB = 4)
constexpr int kMax = 256;       // largest matrix
// squared norms below this (of a column; the matrices are of order 1 or larger)
// count as zero: dropping such a column changes an eigenvalue by less than 1e-140
constexpr double kTiny2 = 1e-280;

// The element operations, for double and double2 (complex).
__device__ __forceinline__ double zero_of(double) { return 0.0; }
__device__ __forceinline__ double2 zero_of(double2) { return make_double2(0.0, 0.0); }
__device__ __forceinline__ double real_of(double a) { return a; }
__device__ __forceinline__ double real_of(double2 a) { return a.x; }
__device__ __forceinline__ double conj_of(double a) { return a; }
__device__ __forceinline__ double2 conj_of(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double abs2(double a) { return a * a; }
__device__ __forceinline__ double abs2(double2 a) { return fma(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ double scaled(double a, double s) { return a * s; }
__device__ __forceinline__ double2 scaled(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
// c + a b
__device__ __forceinline__ double madd(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ double2 madd(double2 a, double2 b, double2 c) {
    return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
// c - a conj(b)
__device__ __forceinline__ double msubc(double a, double b, double c) { return fma(-a, b, c); }
__device__ __forceinline__ double2 msubc(double2 a, double2 b, double2 c) {
    return make_double2(fma(-a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(-a.y, b.x, c.y)));
}
// c - s a with real s
__device__ __forceinline__ double msubr(double s, double a, double c) { return fma(-s, a, c); }
__device__ __forceinline__ double2 msubr(double s, double2 a, double2 c) {
    return make_double2(fma(-s, a.x, c.x), fma(-s, a.y, c.y));
}
// Re(conj(a) b)
__device__ __forceinline__ double redot(double a, double b) { return a * b; }
__device__ __forceinline__ double redot(double2 a, double2 b) { return fma(a.x, b.x, a.y * b.y); }

// x + (x of the lane that the DPP control names)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return x + __hiloint2double(hi, lo);
}
// Sums over aligned groups of 32 lanes and over the wavefront, valid in every lane
// (all lanes active): quad_perm, half-mirror and mirror within 16 lanes.
__device__ __forceinline__ double sum32(double x) {
    x = dpp_add<0xB1>(x);   // quad_perm 1 0 3 2
    x = dpp_add<0x4E>(x);   // quad_perm 2 3 0 1
    x = dpp_add<0x141>(x);  // row_half_mirror
    x = dpp_add<0x140>(x);  // row_mirror
    return x + __shfl_xor(x, 16, 64);
}
__device__ __forceinline__ double2 sum32(double2 x) { return make_double2(sum32(x.x), sum32(x.y)); }
__device__ __forceinline__ double sum64(double x) {
    x = sum32(x);
    return x + __shfl_xor(x, 32, 64);
}

// LDS of one tridiagonalisation.
template <class T>
struct Work {
    T x[2][kMax];  // the current column / reflector (two steps alternate)
    T p[kMax];     // A v
};

// The reflector of the column x (entries s + 1 .. m - 1, zeros at and below s):
// entry s + 1 of v, tau, and the off-diagonal element it leaves.  NL: entries per
// lane.  tau = 0: the column is already zero below s + 1.
template <class T, int NL>
struct Reflector {
    T v0, e;
    double tau;
    T mine[NL];  // v at entries lane + 64 l
    __device__ __forceinline__ Reflector(const T* x, int s) {
        const int lane = threadIdx.x & 63;
        double n2 = 0.0;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            mine[l] = x[lane + 64 * l];
            if (lane + 64 * l != s + 1) n2 += abs2(mine[l]);
        }
        n2 = sum64(n2);
        const T x0 = x[s + 1];
        const double a2 = abs2(x0);
        if (!(n2 > kTiny2)) {
            tau = 0.0;
            v0 = zero_of(x0);
            e = x0;
            return;
        }
        const double nrm = sqrt(n2 + a2), a = sqrt(a2);
        if constexpr (std::is_same<T, double>::value) {
            const double sg = x0 < 0.0 ? -1.0 : 1.0;
            v0 = x0 + sg * nrm;
            e = -sg * nrm;
        } else {
            T ph;  // x0 / |x0|
            if (a2 > kTiny2) {
                ph = scaled(x0, 1.0 / a);
            } else {
                ph = zero_of(x0);
                ph.x = 1.0;
            }
            v0 = make_double2(fma(ph.x, nrm, x0.x), fma(ph.y, nrm, x0.y));
            e = scaled(ph, -nrm);
        }
        tau = 1.0 / (n2 + a2 + a * nrm);
#pragma unroll
        for (int l = 0; l < NL; ++l)
            if (lane + 64 * l == s + 1) mine[l] = v0;
    }
    // v^H p
    __device__ __forceinline__ double dot(const T* p) const {
        const int lane = threadIdx.x & 63;
        double g = 0.0;
#pragma unroll
        for (int l = 0; l < NL; ++l) g += redot(mine[l], p[lane + 64 * l]);
        return sum64(g);
    }
};

// Tridiagonalise the m x m matrix of the registers (elements at and past m zero;
// m <= 32 NB): d[0 .. m-1] gets the diagonal, step(s, e, tau, v) is called by every
// thread for each column s = 0 .. m - 2 with the off-diagonal element e, and with
// the reflector in LDS where tau != 0 (v[s + 1 ..], entries at and below s zero).
template <class T, int NB, class Step>
__device__ __forceinline__ void tridiag_regs(T (&A)[NB][NB], int m, Work<T>& wk, double* d, Step step) {
    constexpr int NL = (NB + 1) / 2;  // entries per lane of a vector of 32 NB
    const int tid = threadIdx.x, tr = tid >> 5, tc = tid & 31;
    sfor<0, NB>([&](auto cbc) {
        constexpr int CB = decltype(cbc)::value;
        const int s1 = m < 32 * (CB + 1) ? m : 32 * (CB + 1);
        for (int s = 32 * CB; s < s1; ++s) {
            T* x = wk.x[s & 1];
            if (tc == (s & 31)) {
#pragma unroll
                for (int a = 0; a < NB; ++a) {
                    const int i = tr + 32 * a;
                    const T v = A[a][CB];
                    if (i == s) d[s] = real_of(v);
                    x[i] = i > s ? v : zero_of(v);
                }
                // a vector of 32 entries (NB = 1) is read 64 wide
                if constexpr (NB % 2 == 1) x[32 * NB + tr] = zero_of(A[0][0]);
            }
            __syncthreads();
            if (s == m - 1) break;
            const Reflector<T, NL> h(x, s);
            if (h.tau != 0.0) {
                T vc[NB];
#pragma unroll
                for (int b = CB; b < NB; ++b) {
                    const int j = tc + 32 * b;
                    vc[b] = j == s + 1 ? h.v0 : x[j];
                }
#pragma unroll
                for (int a = CB; a < NB; ++a) {
                    T acc = zero_of(vc[CB]);
#pragma unroll
                    for (int b = CB; b < NB; ++b) acc = madd(A[a][b], vc[b], acc);
                    acc = sum32(acc);
                    if (tc == 0) wk.p[tr + 32 * a] = acc;
                }
                if (NB % 2 == 1 && tid < 32) wk.p[32 * NB + tid] = zero_of(vc[CB]);
                // rows below the window's first block hold no part of v
                if constexpr (CB > 0) {
                    if (tid < 32 * CB) wk.p[tid] = zero_of(vc[CB]);
                }
                __syncthreads();
                const double half = 0.5 * h.tau * h.tau * h.dot(wk.p);
                T wc[NB];
#pragma unroll
                for (int b = CB; b < NB; ++b) wc[b] = msubr(half, vc[b], scaled(wk.p[tc + 32 * b], h.tau));
#pragma unroll
                for (int a = CB; a < NB; ++a) {
                    const int i = tr + 32 * a;
                    const T vr = i == s + 1 ? h.v0 : x[i];
                    const T wr = msubr(half, vr, scaled(wk.p[i], h.tau));
#pragma unroll
                    for (int b = CB; b < NB; ++b) A[a][b] = msubc(wr, vc[b], msubc(vr, wc[b], A[a][b]));
                }
            }
            step(s, h.e, h.tau, h.v0, x);
        }
    });
}

// The first n_steps steps on an m x m matrix in global memory (row-major, both
// halves kept; m <= kMax), for matrices past the registers: each step reads the
// window for p = A v and reads and writes it for the update.
template <class T, class Step>
__device__ __forceinline__ void tridiag_global(T* A, int m, int n_steps, Work<T>& wk, double* d, Step step) {
    constexpr int NL = kMax / 64;
    const int tid = threadIdx.x, tr = tid >> 5, tc = tid & 31;
    for (int s = 0; s < n_steps; ++s) {
        T* x = wk.x[s & 1];
        if (tid < kMax) {
            // column s as the conjugate of row s
            T v = zero_of(wk.p[0]);
            if (tid >= s && tid < m) v = conj_of(A[(size_t)s * m + tid]);
            if (tid == s) d[s] = real_of(v);
            x[tid] = tid > s ? v : zero_of(v);
        }
        __syncthreads();
        const Reflector<T, NL> h(x, s);
        if (h.tau != 0.0) {
            const int b0 = s >> 5;
            for (int i = tr + 32 * b0; i < m; i += 32) {
                T acc = zero_of(h.v0);
                for (int j = tc + 32 * b0; j < m; j += 32) acc = madd(A[(size_t)i * m + j], j == s + 1 ? h.v0 : x[j], acc);
                acc = sum32(acc);
                if (tc == 0) wk.p[i] = acc;
            }
            // p outside the window meets zeros of v only
            if (tid < 32 * b0 || (tid >= m && tid < kMax)) wk.p[tid] = zero_of(h.v0);
            __syncthreads();
            const double half = 0.5 * h.tau * h.tau * h.dot(wk.p);
            for (int i = tr + 32 * b0; i < m; i += 32) {
                const T vr = i == s + 1 ? h.v0 : x[i];
                const T wr = msubr(half, vr, scaled(wk.p[i], h.tau));
                for (int j = tc + 32 * b0; j < m; j += 32) {
                    const T vj = j == s + 1 ? h.v0 : x[j];
                    const T wj = msubr(half, vj, scaled(wk.p[j], h.tau));
                    T* q = A + (size_t)i * m + j;
                    *q = msubc(wr, vj, msubc(vr, wj, *q));
                }
            }
        }
        step(s, h.e, h.tau, h.v0, x);
        __syncthreads();  // the next column is read by other threads
    }
}

// Eigenvalues below x of the tridiagonal matrix with diagonal d and squared
// off-diagonals e2: sign changes of the leading minors p_{i+1} = (d_i - x) p_i -
// e2_{i-1} p_{i-1} (Givens), rescaled every four rows.  The recurrence takes two
// dependent FP64 operations a row where the quotient form takes a division.
__device__ __forceinline__ int sturm_count(const double* d, const double* e2, int m, double x) {
    double p0 = 1.0, p1 = d[0] - x;
    int count = p1 < 0.0 ? 1 : 0;
    bool neg = p1 < 0.0;
    for (int i = 1; i < m; i += 4) {
        const int n = fmax(fabs(p0), fabs(p1)) > 0.0 ? -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1))) : 0;
        p0 = ldexp(p0, n);
        p1 = ldexp(p1, n);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i + q < m) {
                // a vanishing coupling still separates the minors' signs
                const double p2 = fma(d[i + q] - x, p1, -fmax(e2[i + q - 1], kTiny2) * p0);
                // a zero minor takes the sign opposite to its predecessor's
                const bool n2 = p2 < 0.0 || (p2 == 0.0 && !neg);
                count += n2 != neg ? 1 : 0;
                neg = n2;
                p0 = p1;
                p1 = p2;
            }
        }
    }
    return count;
}

// The k-th smallest eigenvalue (k from 0) by a wavefront, every lane the same
// value: 64 points a round split [lo, hi] in 65 parts.
__device__ __forceinline__ double sturm_select(const double* d, const double* e2, int m, int k, double lo, double hi,
                                               int rounds) {
    const int lane = threadIdx.x & 63;
    for (int r = 0; r < rounds; ++r) {
        const double h = (hi - lo) * (1.0 / 65.0);
        const double x = fma((double)(lane + 1), h, lo);
        const bool above = sturm_count(d, e2, m, x) > k;  // the eigenvalue lies below x
        const unsigned long long b = __ballot(above);
        const int first = b ? __ffsll((long long)b) - 1 : 64;
        const double nlo = fma((double)first, h, lo);
        if (first < 64) hi = fma((double)(first + 1), h, lo);
        lo = nlo;
    }
    return 0.5 * (lo + hi);
}

}  // namespace eig
}  // namespace hom4d_impl
