// Hermitian (or real symmetric) tridiagonalisation by one workgroup with the
// matrix in registers, and Sturm counts of the result (FP64).
//
// A block of TR x 16 threads holds the matrix with cyclic ownership: thread
// (tr, tc) keeps elements (tr + TR a, tc + 16 b), so every thread stays busy as the
// active window shrinks; 512 threads carry 128 x 128 complex values in 128 VGPRs
// each.  LDS only moves the two vectors of a step, once per wavefront: a lane holds the
// entries of its number, and a thread's columns of the matrix come from the four rows of its
// own wavefront by lane swaps.  (The matrix itself does not fit
// 160 KB of LDS at 128 x 128 complex, and a pass over it in L2 per step is what
// bounds larger sizes, tridiag_global below.)
//
// Step s, with x the column s below the diagonal: the reflector
// H = 1 - tau v v^H, v = x + (x_0 / |x_0|) ||x|| e_0, tau = 1 / (||x||^2 + |x_0| ||x||)
// (Golub and Van Loan, Householder tridiagonalisation) maps x to
// -(x_0 / |x_0|) ||x|| e_0; with p = A v and w = tau p - (tau^2 / 2) (v^H p) v the
// window becomes A - v w^H - w v^H.  Two barriers per step: one after the
// column is in LDS, one after p is.  Each wavefront forms ||x||^2 and v^H p for
// itself, from the same LDS values in the same order, so that every thread holds
// the same bits and takes the same branches.
//
// The chain of m - 1 steps on one CU bounds it, and in a step the instructions that its one or
// two wavefronts per SIMD issue.  What a step costs beyond its 12 FP64 operations per element
// is work every wavefront repeats, so there are as few wavefronts as the registers allow,
// a large matrix goes on in the form of fewer wavefronts once it has shrunk to 64 rows,
// the sums stay in DPP and lane swaps, the vectors' entries are kept from the product to the
// update, and square root and reciprocals are the hardware estimates with two Newton
// steps.  128 x 128 complex: 239 us (278 us with the columns' entries read from LDS, the
// reflector's first put in by selects, and one form to the end; 421 us with 1024 threads,
// 32-lane shuffles and library square roots and divisions); 64 x 64: 75 us (92; 152); 128
// wave numbers' 96 x 96 real matrices, one per CU: about 100 of the 184 us of k_edge_state.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dft_regs.hpp"
#include "estimates.hpp"

namespace hom4d_impl {
namespace eig {
using namespace hom4d_dev;
using dev::rcp_of;
using dev::rsqrt_of;

constexpr int kRegMax = 128;  // largest matrix held in registers
constexpr int kMax = 256;     // largest matrix
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

// the value of the lane that the DPP control names (within 16 lanes)
constexpr int kXor15 = 0x140, kXor7 = 0x141, kXor3 = 0x1B, kXor1 = 0xB1;  // mirror, half mirror, quad_perm
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ double2 dpp(double2 x) { return make_double2(dpp<CTRL>(x.x), dpp<CTRL>(x.y)); }
__device__ __forceinline__ double add(double a, double b) { return a + b; }
__device__ __forceinline__ double2 add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }

// The lane swaps between a wavefront's rows of 16 lanes: of x twice, out[0] gets rows
// (0, 1, 0, 1) and out[1] rows (2, 3, 2, 3) from swap32, rows (0, 0, 2, 2) and
// (1, 1, 3, 3) from swap16 (all lanes active).
__device__ __forceinline__ void swap32(double x, double* out) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
    out[0] = __hiloint2double(hi[0], lo[0]);
    out[1] = __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ void swap16(double x, double* out) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
    out[0] = __hiloint2double(hi[0], lo[0]);
    out[1] = __hiloint2double(hi[1], lo[1]);
}
// out[r]: x of the lane of row r with the same number within its 16
__device__ __forceinline__ void rows_of(double x, double* out) {
    double h[2];
    swap32(x, h);
    swap16(h[0], out);
    swap16(h[1], out + 2);
}
__device__ __forceinline__ void rows_of(double2 x, double2* out) {
    double re[4], im[4];
    rows_of(x.x, re);
    rows_of(x.y, im);
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = make_double2(re[r], im[r]);
}
// Sum over the wavefront, the same in every lane (all lanes active).
__device__ __forceinline__ double sum64(double x) {
    x += dpp<kXor15>(x);
    x += dpp<kXor7>(x);
    x += dpp<kXor3>(x);
    x += dpp<kXor1>(x);
    double h[2];
    swap32(x, h);
    swap16(h[0] + h[1], h);
    return h[0] + h[1];
}

// Sums of C values each over 16 lanes, by halves: a stage sends the half of the
// values that the partner keeps, until a lane holds one of the sums.
template <int C, int CTRL, int BIT, class T>
__device__ __forceinline__ void reduce_stage(T* acc, int lane, int& row) {
    if constexpr (C > 1) {
        constexpr int H = C / 2;
        const bool up = (lane & BIT) != 0;
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const T lo = acc[k], hi = acc[k + H];
            acc[k] = add(up ? hi : lo, dpp<CTRL>(up ? lo : hi));
        }
        if (up) row += H;
    } else {
        acc[0] = add(acc[0], dpp<CTRL>(acc[0]));
    }
}
// acc[0] becomes the sum of value `row` (returned) of the lane's group of 16; the
// lanes whose bits below 16 / C are zero hold each sum once.
template <int C, class T>
__device__ __forceinline__ int reduce16(T* acc) {
    static_assert((C & (C - 1)) == 0 && C <= 16, "a power of two");
    const int lane = threadIdx.x & 15;
    int row = 0;
    reduce_stage<C, kXor15, 8>(acc, lane, row);
    reduce_stage<(C > 2 ? C / 2 : 1), kXor7, 4>(acc, lane, row);
    reduce_stage<(C > 4 ? C / 4 : 1), kXor3, 2>(acc, lane, row);
    reduce_stage<(C > 8 ? C / 8 : 1), kXor1, 1>(acc, lane, row);
    return row;
}

// LDS of one tridiagonalisation; cleared before the first step (clear()).
template <class T>
struct Work {
    T x[2][kMax];  // the current column / reflector (two steps alternate)
    T p[kMax];     // A v
    __device__ __forceinline__ void clear() {
        double* q = reinterpret_cast<double*>(this);
        for (int i = threadIdx.x; i < (int)(sizeof(Work) / sizeof(double)); i += blockDim.x) q[i] = 0.0;
        __syncthreads();
    }
};

// The reflector of the column x (entries s + 1 .. m - 1, zeros elsewhere): entry
// s + 1 of v, tau, and the off-diagonal element it leaves.  NL: entries per lane.
// tau = 0: the column is already zero below s + 1.
template <class T, int NL>
struct Reflector {
    T v0, e;
    double tau;
    T mine[NL];  // v at entries lane + 64 l
    __device__ __forceinline__ Reflector(const T* x, int s) {
        const int lane = threadIdx.x & 63;
        const T x0 = x[s + 1];
        double n2 = 0.0;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            mine[l] = x[lane + 64 * l];
            if (lane + 64 * l != s + 1) n2 += abs2(mine[l]);
        }
        n2 = sum64(n2);
        if (!(n2 > kTiny2)) {
            tau = 0.0;
            v0 = zero_of(x0);
            e = x0;
            return;
        }
        const double a2 = abs2(x0), t2 = n2 + a2;
        const double nrm = t2 * rsqrt_of(t2);
        double a;
        if constexpr (std::is_same<T, double>::value) {
            a = fabs(x0);
            e = x0 < 0.0 ? nrm : -nrm;
            v0 = x0 - e;
        } else {
            T ph = make_double2(1.0, 0.0);  // x0 / |x0|
            a = 0.0;
            if (a2 > kTiny2) {
                const double r = rsqrt_of(a2);
                a = a2 * r;
                ph = scaled(x0, r);
            }
            e = scaled(ph, -nrm);
            v0 = make_double2(x0.x - e.x, x0.y - e.y);
        }
        tau = rcp_of(fma(a, nrm, t2));
#pragma unroll
        for (int l = 0; l < NL; ++l)
            if (lane + 64 * l == s + 1) mine[l] = v0;
    }
    // (tau^2 / 2) v^H p; w: w at entries lane + 64 l
    __device__ __forceinline__ double half_dot(const T* p, T (&w)[NL]) const {
        const int lane = threadIdx.x & 63;
        double g = 0.0;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            w[l] = p[lane + 64 * l];
            g += redot(mine[l], w[l]);
        }
        const double half = 0.5 * tau * tau * sum64(g);
#pragma unroll
        for (int l = 0; l < NL; ++l) w[l] = msubr(half, mine[l], scaled(w[l], tau));
        return half;
    }
};

// The first n steps of the tridiagonalisation of the m x m matrix of the registers
// (n < m <= N = TR RA = 16 CB, n <= 16 CE; elements at and past m zero): step(s, h, x) is
// called by every thread for each column s = 0 .. n - 1 with its Reflector and the
// column in LDS (the reflector's entries past s + 1); d[0 .. n-1], and d[n] for n = m - 1,
// gets the diagonal at the end (from the registers: a store to memory within a step
// would be waited for at its barriers).  Rows and columns n .. m - 1 then hold what is
// left to reduce.
template <class T, int TR, int RA, int CB, int CE = CB, class Step>
__device__ __forceinline__ void tridiag_regs(T (&A)[RA][CB], int m, int n, Work<T>& wk, double* d, Step step) {
    static_assert(TR * RA == 16 * CB, "a square matrix");
    constexpr int N = TR * RA, NL = (N + 63) / 64;
    const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15;
    sfor<0, CE>([&](auto cbc) {
        constexpr int C0 = decltype(cbc)::value, A0 = 16 * C0 / TR;  // first active blocks
        const int s1 = n < 16 * (C0 + 1) ? n : 16 * (C0 + 1);
        for (int s = 16 * C0; s < s1; ++s) {
            T* x = wk.x[s & 1];
            if (tc == (s & 15)) {
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    const int i = tr + TR * a;
                    x[i] = i > s ? A[a][C0] : zero_of(A[a][C0]);
                }
            }
            __syncthreads();
            const Reflector<T, NL> h(x, s);
            if (h.tau != 0.0) {
                T vc[4 * NL];  // v at this thread's columns tc + 16 b
                sfor<C0 / 4, NL>([&](auto lc) { rows_of(h.mine[decltype(lc)::value], vc + 4 * decltype(lc)::value); });
                {
                    T acc[RA];
#pragma unroll
                    for (int a = 0; a < RA; ++a) acc[a] = zero_of(h.v0);
#pragma unroll
                    for (int b = C0; b < CB; ++b)
#pragma unroll
                        for (int a = A0; a < RA; ++a) acc[a] = madd(A[a][b], vc[b], acc[a]);
                    const int row = reduce16<RA>(acc);
                    if ((tc & (16 / RA - 1)) == 0) wk.p[tr + TR * row] = acc[0];
                }
                __syncthreads();
                T w[NL], vr[RA], wr[RA];
                const double half = h.half_dot(wk.p, w);
#pragma unroll
                for (int a = A0; a < RA; ++a) {
                    const int i = tr + TR * a;
                    vr[a] = x[i];
                    if (a <= A0 + 1 && i == s + 1) vr[a] = h.v0;
                    wr[a] = msubr(half, vr[a], scaled(wk.p[i], h.tau));
                }
                sfor<C0 / 4, NL>([&](auto lc) {
                    constexpr int l = decltype(lc)::value;
                    T wj[4];
                    rows_of(w[l], wj);
#pragma unroll
                    for (int b = 4 * l < C0 ? C0 : 4 * l; b < (4 * l + 4 < CB ? 4 * l + 4 : CB); ++b)
#pragma unroll
                        for (int a = A0; a < RA; ++a)
                            A[a][b] = msubc(wr[a], vc[b], msubc(vr[a], wj[b - 4 * l], A[a][b]));
                });
            }
            step(s, h, x);
        }
    });
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
            if (tr + TR * a == tc + 16 * b && tr + TR * a < (n == m - 1 ? m : n)) d[tr + TR * a] = real_of(A[a][b]);
}

// The first n_steps steps on an m x m matrix in global memory (row-major, both
// halves kept; m <= kMax), for matrices past the registers: each step reads the
// window for p = A v and reads and writes it for the update.  TR: threads / 16.
template <class T, int TR, class Step>
__device__ __forceinline__ void tridiag_global(T* A, int m, int n_steps, Work<T>& wk, double* d, Step step) {
    constexpr int NL = kMax / 64;
    const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15;
    for (int s = 0; s < n_steps; ++s) {
        T* x = wk.x[s & 1];
        for (int i = tid; i < kMax; i += 16 * TR) {
            // column s as the conjugate of row s
            T v = zero_of(wk.p[0]);
            if (i >= s && i < m) v = conj_of(A[(size_t)s * m + i]);
            if (i == s) d[s] = real_of(v);
            x[i] = i > s ? v : zero_of(v);
        }
        __syncthreads();
        const Reflector<T, NL> h(x, s);
        if (h.tau != 0.0) {
            const int j0 = s & ~15, i0 = s / TR * TR;
            for (int i = tr + i0; i < m; i += TR) {
                T acc = zero_of(h.v0);
                for (int j = tc + j0; j < m; j += 16) acc = madd(A[(size_t)i * m + j], j == s + 1 ? h.v0 : x[j], acc);
                reduce16<1>(&acc);
                if (tc == 0) wk.p[i] = acc;
            }
            __syncthreads();
            T w[NL];
            const double half = h.half_dot(wk.p, w);
            for (int i = tr + i0; i < m; i += TR) {
                const T vr = i == s + 1 ? h.v0 : x[i];
                const T wr = msubr(half, vr, scaled(wk.p[i], h.tau));
                for (int j = tc + j0; j < m; j += 16) {
                    const T vj = j == s + 1 ? h.v0 : x[j];
                    const T wj = msubr(half, vj, scaled(wk.p[j], h.tau));
                    T* q = A + (size_t)i * m + j;
                    *q = msubc(wr, vj, msubc(vr, wj, *q));
                }
            }
        }
        step(s, h, x);
        __syncthreads();  // the next column is read by other threads
    }
}

// A tridiagonal matrix as Sturm counts read it: entry i holds the diagonal d_i and
// the squared off-diagonal e2_{i-1} before it (at least kTiny2: a vanishing coupling
// still separates the minors' signs), padded to whole groups of eight with rows
// above every eigenvalue.
constexpr int kSturmRows = (kMax + 7) / 8 * 8;
__device__ __forceinline__ double2 sturm_row(double d, double e2) { return make_double2(d, fmax(e2, kTiny2)); }
__device__ __forceinline__ double2 sturm_pad(double above) { return make_double2(above, kTiny2); }

// Eigenvalues below x: sign changes of the leading minors p_{i+1} = (d_i - x) p_i -
// e2_{i-1} p_{i-1} (Givens), rescaled every eight rows.  One dependent FP64
// operation a row, where the quotient form takes a division.  A zero minor counts
// one change in all whatever its sign, since the next one is opposite to its predecessor.
__device__ __forceinline__ int sturm_count(const double2* t, int m, double x) {
    double p0 = 0.0, p1 = 1.0;
    int count = 0;
    for (int i = 0; i < m; i += 8) {
        double2 r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = t[i + q];
        const int n = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
        p0 = ldexp(p0, n);
        p1 = ldexp(p1, n);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double p2 = fma(r[q].x - x, p1, -r[q].y * p0);
            count += (unsigned)(__double2hiint(p2) ^ __double2hiint(p1)) >> 31;
            p0 = p1;
            p1 = p2;
        }
    }
    return count;
}

// Bracket [lo, hi] of the k-th smallest eigenvalue (k from 0) by a wavefront, every
// lane the same: 64 points a round split it in 65 parts.
__device__ __forceinline__ void sturm_select(const double2* t, int m, int k, double& lo, double& hi, int rounds) {
    const int lane = threadIdx.x & 63;
    for (int r = 0; r < rounds; ++r) {
        const double h = (hi - lo) * (1.0 / 65.0);
        const double x = fma((double)(lane + 1), h, lo);
        const unsigned long long b = __ballot(sturm_count(t, m, x) > k);  // it lies below x
        const int first = b ? __ffsll((long long)b) - 1 : 64;
        const double base = lo;
        lo = fma((double)first, h, base);
        if (first < 64) hi = fma((double)(first + 1), h, base);
    }
}

}  // namespace eig
}  // namespace hom4d_impl
