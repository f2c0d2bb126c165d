// Edge states and Gaussian edge-state wave packets on the GPU: the one-electron
// inputs of the two-electron propagation (arXiv 1903.02581 Sec. II.A,
// Eq. (H_effective); Sec. II.B, Eq. (singlepwp)).
//
// In the gauge A = (-B y, 0) an electron with wave number k along x sees the
// transverse Hamiltonian
//     H(k) = kappa [ -d^2/dy^2 + (k - y eB/hbar)^2 ] + v(y),
// with the second derivative spectral on the periodic y grid: the circulant
// matrix c[(i - j) mod ny], c[d] = (kappa / ny) sum_m ky_m^2 cos(2 pi m d / ny),
// whose first row the host computes.  k_edge_state finds the lowest eigenpair of
// H(k) for every grid k, one workgroup per k: Householder tridiagonalisation with
// the matrix in registers (eigen_regs.hpp), bisection from Sturm counts, the
// tridiagonal eigenvector from a twisted factorisation (Fernando; Parlett and
// Dhillon), the reflectors applied to it in reverse, and its sign fixed so that the
// largest-magnitude component is positive.  Only the lowest pair is wanted, so
// this takes one reduction where the full Jacobi diagonalisation it replaces took
// 7-9 sweeps of 3 barriers per rotation step over a matrix in L2: 20.4 -> 0.17 ms
// at nx = 128, ny = 96.
//
// k_edge_sum forms psi(x_i, y_j) = sum_m exp(-sigma^2 (k_m - k0)^2)
// exp(i k_m (x_i - xc)) phi_m(y_j) with the m sum in grid order, where k0 is the
// grid wave number (on the requested side: k > 0 for the top edge, k < 0 for the
// bottom) whose edge-state energy is closest to hbar omega_c / 2 + e_above;
// k_edge_scale normalises it on the grid.  All arithmetic is FP64.
#include "axis_pass.hpp"
#include "eigen_regs.hpp"
#include "hom4d_internal.hpp"

namespace hom4d_impl {
namespace {

using namespace dev;

constexpr int kThreads = 256;
constexpr int kTR = kThreads / 16;

// Reflector s of an m x m reduction: entries s + 1 .. m - 1, packed.
__device__ __forceinline__ int reflector_at(int s, int m) { return s * (m - 1) - s * (s - 1) / 2 - (s + 1); }

// One workgroup per wave number.  MEM: ny > eig::kRegMax, the matrix and the
// reflectors in global memory (work: ny^2, then ny (ny - 1) / 2 doubles per k);
// otherwise the matrix is in registers and the reflectors in LDS.
template <int RA, int CB, bool MEM>
__global__ void __launch_bounds__(kThreads) k_edge_state(EdgeArgs g) {
    __shared__ eig::Work<double> wk;
    __shared__ double2 t[eig::kSturmRows];                     // Sturm rows
    __shared__ double circ[eig::kMax], d[eig::kMax], e[eig::kMax], tau[eig::kMax];
    __shared__ double piv[2][eig::kMax], z[eig::kMax];
    extern __shared__ double lds_refl[];
    const int m = g.ny, tid = threadIdx.x, lane = tid & 63, tr = tid >> 4, tc = tid & 15;
    const double k = g.kx[blockIdx.x];
    double* A = MEM ? g.work + (size_t)blockIdx.x * ((size_t)m * m + (size_t)m * (m - 1) / 2) : nullptr;
    double* refl = MEM ? A + (size_t)m * m : lds_refl;
    if (tid < m) circ[tid] = g.circ[tid];
    wk.clear();

    auto element = [&](int i, int j) {
        double a = circ[i >= j ? i - j : i - j + m];
        if (i == j) {
            const double u = k - (g.y0 + g.dy * i) * g.inv_lb2;
            a += g.kappa * u * u + g.vcol[i];
        }
        return a;
    };
    int s0 = 0;
    auto keep = [&](int sl, const auto& h, const double* x) {
        const int s = s0 + sl, i = s0 + tid;
        if (h.tau != 0.0 && tid > sl && i < m) refl[reflector_at(s, m) + i] = tid == sl + 1 ? h.v0 : x[tid];
        if (tid == 0) {
            e[s] = h.e;
            tau[s] = h.tau;
        }
    };
    if constexpr (MEM) {
        for (int q = tid; q < m * m; q += kThreads) A[q] = element(q / m, q % m);
        __syncthreads();
        eig::tridiag_global<double, kTR>(A, m, m - eig::kRegMax, wk, d, keep);
        s0 = m - eig::kRegMax;
        wk.clear();
    }
    {
        double M[RA][CB];
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int i = s0 + tr + kTR * a, j = s0 + tc + 16 * b;
                M[a][b] = 0.0;
                if (i < m && j < m) M[a][b] = MEM ? A[(size_t)i * m + j] : element(i, j);
            }
        if constexpr (CB <= 4) {
            eig::tridiag_regs<double, kTR, RA, CB>(M, m, m - 1, wk, d, keep);
        } else {
            // down to 64 rows, then the form of 64 rows: a step of it moves half the vectors
            // (m = 96: the kernel 184 -> 172 us)
            __shared__ double rest[64 * 64];
            const int n = m - s0 - 64;
            eig::tridiag_regs<double, kTR, RA, CB, CB / 2>(M, m - s0, n, wk, d + s0, keep);
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b) {
                    const int i = tr + kTR * a - n, j = tc + 16 * b - n;
                    if (i >= 0 && j >= 0 && i < 64 && j < 64) rest[i * 64 + j] = M[a][b];
                }
            __syncthreads();
            s0 += n;
            double L[4][4];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) L[a][b] = rest[(tr + kTR * a) * 64 + tc + 16 * b];
            eig::tridiag_regs<double, kTR, 4, 4>(L, 64, 63, wk, d + s0, keep);
        }
    }
    __syncthreads();

    // lowest eigenvalue: between the Gershgorin bound and the smallest diagonal entry
    double lo = 1e300, hi = 1e300, top = -1e300;
    for (int i = lane; i < m; i += 64) {
        const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i < m - 1 ? fabs(e[i]) : 0.0);
        lo = fmin(lo, d[i] - r);
        hi = fmin(hi, d[i]);
        top = fmax(top, d[i] + r);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, 64));
        hi = fmin(hi, __shfl_xor(hi, o, 64));
        top = fmax(top, __shfl_xor(top, o, 64));
    }
    const double span = top - lo;
    t[tid] = tid < m ? eig::sturm_row(d[tid], tid > 0 ? e[tid - 1] * e[tid - 1] : 0.0) : eig::sturm_pad(top + span + 1.0);
    __syncthreads();
    // (every wavefront the same rounds, so that they stay together for the barriers below)
    lo -= 1e-15 * span;
    eig::sturm_select(t, m, 0, lo, hi, 10);

    // Eigenvector of the tridiagonal matrix at a shift l: the pivots of the
    // factorisations from the top (lane 0) and from the bottom (lane 1), joined at
    // the row where they leave the smallest residual gamma.  From the lower end of
    // the bracket T - l is positive definite; a second pass at the Rayleigh-corrected
    // shift takes out the bracket's rounding.
    double shift = lo;
    const double tiny = 1e-30 * span;
    for (int pass = 0; pass < 2; ++pass) {
        if (tid < 2) {
            double p = 1.0, c2 = 0.0;
            for (int q = 0; q < m; ++q) {
                const int i = tid == 0 ? q : m - 1 - q;
                p = fma(-c2, eig::rcp_of(p), d[i] - shift);
                if (fabs(p) < tiny) p = p < 0.0 ? -tiny : tiny;
                piv[tid][i] = p;
                if (q < m - 1) {
                    const double c = e[tid == 0 ? i : i - 1];
                    c2 = c * c;
                }
            }
        }
        __syncthreads();
        double best = 1e300;
        int at = 0;
        for (int i = lane; i < m; i += 64) {
            const double gm = fabs(piv[0][i] + piv[1][i] - (d[i] - shift));
            if (gm < best) {
                best = gm;
                at = i;
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const double ob = __shfl_xor(best, o, 64);
            const int oa = __shfl_xor(at, o, 64);
            if (ob < best || (ob == best && oa < at)) {
                best = ob;
                at = oa;
            }
        }
        const double gamma = piv[0][at] + piv[1][at] - (d[at] - shift);
        __syncthreads();
        // the ratio of each row to its neighbour on the side of row `at`
        if (tid < m) z[tid] = tid < at ? -e[tid] * eig::rcp_of(piv[0][tid]) : tid > at ? -e[tid - 1] * eig::rcp_of(piv[1][tid]) : 1.0;
        __syncthreads();
        if (tid == 0) {
            double p = 1.0;
            for (int i = at - 1; i >= 0; --i) z[i] = p *= z[i];
        } else if (tid == 1) {
            double p = 1.0;
            for (int i = at + 1; i < m; ++i) z[i] = p *= z[i];
        }
        __syncthreads();
        double n2 = 0.0;
        for (int i = lane; i < m; i += 64) n2 = fma(z[i], z[i], n2);
        const double next = shift + gamma * eig::rcp_of(eig::sum64(n2));
        if (pass == 1) {
            if (tid == 0) g.e1[blockIdx.x] = next;
        }
        shift = next;
    }

    // back to the grid: reflectors in reverse, by the first wavefront
    if (tid >= 64) return;
    constexpr int NL = MEM ? eig::kMax / 64 : (16 * CB + 63) / 64;
    double y[NL], v[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) y[l] = lane + 64 * l < m ? z[lane + 64 * l] : 0.0;
    auto fetch = [&](int s) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int i = lane + 64 * l;
            v[l] = s >= 0 && i > s && i < m ? refl[reflector_at(s, m) + i] : 0.0;
        }
    };
    fetch(m - 2);
    for (int s = m - 2; s >= 0; --s) {
        double w[NL], dot = 0.0;
        const double ts = tau[s];
#pragma unroll
        for (int l = 0; l < NL; ++l) w[l] = v[l];
        fetch(s - 1);
        if (ts != 0.0) {
#pragma unroll
            for (int l = 0; l < NL; ++l) dot = fma(w[l], y[l], dot);
            dot = ts * eig::sum64(dot);
#pragma unroll
            for (int l = 0; l < NL; ++l) y[l] = fma(-dot, w[l], y[l]);
        }
    }
    double n2 = 0.0, big = 0.0;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        n2 = fma(y[l], y[l], n2);
        big = fmax(big, fabs(y[l]));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
    double scale = 1.0 / sqrt(eig::sum64(n2));
    // the first component of the largest magnitude is positive
    bool found = false;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const unsigned long long b = __ballot(fabs(y[l]) == big);
        if (!found && b != 0) {
            found = true;
            if (__shfl(y[l], __ffsll((long long)b) - 1, 64) < 0.0) scale = -scale;
        }
    }
#pragma unroll
    for (int l = 0; l < NL; ++l)
        if (lane + 64 * l < m) g.phi[(size_t)blockIdx.x * m + lane + 64 * l] = scale * y[l];
}

// rows: grid rows per block (x_i), each on ny threads; the amplitudes and phases of
// a row's waves are staged in LDS once instead of formed by each of its ny threads
// (128 x 96: 67 -> 10 us).
constexpr int kWaves = 1024;  // rows nx staged waves at most
__global__ void __launch_bounds__(kThreads) k_edge_sum(EdgeArgs g, int rows) {
    __shared__ double s_gap[kThreads];
    __shared__ int s_at[kThreads];
    __shared__ double2 wave[kWaves];
    __shared__ double red[kThreads / 64];
    const int tid = threadIdx.x, nx = g.nx, ny = g.ny;
    // first grid index on the requested side whose level is closest to the target
    double gap = 1e300;
    int at = nx;
    for (int m = tid; m < nx; m += kThreads) {
        const double k = g.kx[m];
        const double d = fabs(g.e1[m] - g.target);
        if ((g.top ? k > 0.0 : k < 0.0) && (at == nx || d < gap)) {
            gap = d;
            at = m;
        }
    }
    s_gap[tid] = gap;
    s_at[tid] = at;
    __syncthreads();
    for (int o = kThreads / 2; o >= 1; o >>= 1) {
        if (tid < o) {
            const double og = s_gap[tid + o];
            const int oa = s_at[tid + o];
            if (oa < nx && (s_at[tid] == nx || og < s_gap[tid] || (og == s_gap[tid] && oa < s_at[tid]))) {
                s_gap[tid] = og;
                s_at[tid] = oa;
            }
        }
        __syncthreads();
    }
    const int best = s_at[0] < nx ? s_at[0] : 0;  // every supported nx has wave numbers of both signs
    const double k0 = g.kx[best];
    if (blockIdx.x == 0 && tid == 0) {
        g.info[0] = k0;
        g.info[1] = g.e1[best];
        g.info[2] = g.target;
    }
    const int i0 = blockIdx.x * rows;
    for (int q = tid; q < rows * nx; q += kThreads) {
        const int m = q % nx;
        const double k = g.kx[m], d = k - k0;
        const double amp = exp(-g.sigma * g.sigma * d * d);
        double sn, cs;
        sincos(k * (g.x0 + g.dx * (i0 + q / nx) - g.xc), &sn, &cs);
        wave[q] = make_double2(amp * cs, amp * sn);
    }
    __syncthreads();
    const int r = tid / ny, j = tid % ny, i = i0 + r;
    double n2 = 0.0;
    if (r < rows && i < nx) {
        double re = 0.0, im = 0.0;
#pragma unroll 8
        for (int m = 0; m < nx; ++m) {
            const double f = g.phi[(size_t)m * ny + j];
            const double2 w = wave[r * nx + m];
            re = fma(w.x, f, re);
            im = fma(w.y, f, im);
        }
        g.psi[(size_t)i * ny + j] = make_double2(re, im);
        n2 = re * re + im * im;
    }
    const double s = block_sum(n2, red);
    if (tid == 0) g.part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kThreads) k_edge_scale(double2* psi, const double* part, int nparts, int count) {
    __shared__ double red[kThreads / 64];
    __shared__ double s_inv;
    const int tid = threadIdx.x;
    double a = 0.0;
    for (int q = tid; q < nparts; q += kThreads) a += part[q];
    const double s = block_sum(a, red);
    if (tid == 0) s_inv = 1.0 / sqrt(s);
    __syncthreads();
    const int idx = blockIdx.x * kThreads + tid;
    if (idx < count) psi[idx] = cscale(psi[idx], s_inv);
}

template <int RA, int CB, bool MEM>
hipError_t launch_edge_state(const EdgeArgs& e, hipStream_t s) {
    const size_t lds = MEM ? 0 : (size_t)e.ny * (e.ny - 1) / 2 * sizeof(double);
    auto fn = k_edge_state<RA, CB, MEM>;
    if (lds > 8 * 1024) {
        // with its static LDS (56 KB for more than 64 rows) the block may be past 64 KB,
        // which has to be allowed
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(fn, dim3(e.nx), dim3(kThreads), lds, s, e);
    return hipGetLastError();
}

}  // namespace

size_t edge_work_doubles(int nx, int ny) {
    return ny > eig::kRegMax ? (size_t)nx * ((size_t)ny * ny + (size_t)ny * (ny - 1) / 2) : 0;
}

hipError_t launch_edge_packet(const EdgeArgs& e, hipStream_t s) {
    if (e.nx <= 0 || e.nx > kWaves / 4 || e.ny < 4 || e.ny > eig::kMax) return hipErrorInvalidValue;
    hipError_t err = e.ny <= 32    ? launch_edge_state<2, 2, false>(e, s)
                     : e.ny <= 64  ? launch_edge_state<4, 4, false>(e, s)
                     : e.ny <= 128 ? launch_edge_state<8, 8, false>(e, s)
                                   : launch_edge_state<8, 8, true>(e, s);
    if (err != hipSuccess) return err;
    int rows = kThreads / e.ny;
    if (rows > kWaves / e.nx) rows = kWaves / e.nx;
    const int nblocks = (e.nx + rows - 1) / rows, count = e.nx * e.ny;
    hipLaunchKernelGGL(k_edge_sum, dim3(nblocks), dim3(kThreads), 0, s, e, rows);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_edge_scale, dim3((count + kThreads - 1) / kThreads), dim3(kThreads), 0, s, e.psi, e.part,
                       nblocks, count);
    return hipGetLastError();
}

}  // namespace hom4d_impl
