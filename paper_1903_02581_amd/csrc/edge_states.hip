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
// Dhillon), the reflectors applied to it in reverse, one step of refinement with H itself,
// and its sign fixed so that the largest-magnitude component is positive.  Only the
// lowest pair is wanted, so this takes one reduction where a full Jacobi diagonalisation
// took 7-9 sweeps of 3 barriers per rotation step over a matrix in L2: 20.4 -> 0.18 ms
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

// Entries of a stored reflector: whole turns of 64 lanes, zeros outside s + 1 .. m - 1.
__host__ __device__ constexpr int reflector_stride(int m) { return (m + 63) / 64 * 64; }

__host__ __device__ constexpr size_t edge_work_per_k(int m) { return (size_t)m * m + (size_t)m * reflector_stride(m); }

// One workgroup per wave number.  MEM: ny > eig::kRegMax, the matrix and the
// reflectors in global memory (work: ny^2 doubles each per k); otherwise the matrix is in
// registers and the reflectors in LDS.
template <int RA, int CB, bool MEM>
__global__ void __launch_bounds__(kThreads) k_edge_state(EdgeArgs g) {
    __shared__ eig::Work<double> wk;
    __shared__ double2 t[eig::kSturmRows];  // Sturm rows, the minors' rows, ratios and reciprocal pivots
    __shared__ double circ[eig::kMax], d[eig::kMax], e[eig::kMax], tau[eig::kMax];
    // (entry kMax takes the stores past the last row)
    __shared__ double piv[2][eig::kMax + 1], z[eig::kMax + 1], w[eig::kMax], before[2][eig::kMax / 8], link[eig::kMax / 2];
    extern __shared__ double lds_refl[];
    constexpr int NL = MEM ? eig::kMax / 64 : (16 * CB + 63) / 64;  // entries of a vector per lane
    constexpr int STRIDE = 64 * NL;
    const int m = g.ny, tid = threadIdx.x, lane = tid & 63, tr = tid >> 4, tc = tid & 15;
    const double k = g.kx[blockIdx.x];
    double* A = MEM ? g.work + (size_t)blockIdx.x * edge_work_per_k(m) : nullptr;
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
        const int s = s0 + sl;
        if (tid < STRIDE) {
            const double v = tid > s && tid < m && h.tau != 0.0 ? x[tid - s0] : 0.0;
            refl[s * STRIDE + tid] = tid == s + 1 && h.tau != 0.0 ? h.v0 : v;
        }
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
            // (12 us less at m = 96), through the places of its reflectors
            const int n = m - s0 - 64;
            double* rest = lds_refl + (MEM ? 0 : n * STRIDE);
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
    // A pivot is the ratio of two leading minors, whose recurrence (as in sturm_count) is two
    // operations a row where the pivots' own takes a reciprocal; all the rest of a row is done by
    // its own thread, since one lane's chain costs as many issue slots as it has instructions.
    double shift = lo;
    const double tiny = 1e-30 * span;
    int row = 0;  // where the second pass joins them
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        double e2[2] = {0.0, 0.0}, diag = 0.0;  // of row tid: couplings before it from either end
        if (tid < m) {
            diag = d[tid] - shift;
            if (tid > 0) e2[0] = e[tid - 1] * e[tid - 1];
            if (tid < m - 1) e2[1] = e[tid] * e[tid];
            t[tid] = make_double2(e2[0], diag);
            w[tid] = e2[1];
        }
        __syncthreads();
        if (tid < 2) {
            double p0 = 0.0, p1 = 1.0;
            const int end = tid == 0 ? 0 : m - 1, by = tid == 0 ? 1 : -1;
#pragma unroll 1
            for (int q0 = 0; q0 < m; q0 += 8) {
                const int n = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
                p0 = ldexp(p0, n);
                p1 = ldexp(p1, n);
                before[tid][q0 >> 3] = p1;  // the minor before the group, in its scale
                batched<8, 8>(
                    [&](int q) {
                        const int i = end + by * (q0 + q < m ? q0 + q : m - 1);
                        return make_double2(tid == 0 ? t[i].x : w[i], t[i].y);
                    },
                    [&](int q, double2 f) {
                        const double p2 = fma(f.y, p1, -f.x * p0);
                        piv[tid][q0 + q < m ? end + by * (q0 + q) : eig::kMax] = p2;
                        p0 = p1;
                        p1 = p2;
                    });
            }
        }
        __syncthreads();
        double p[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int u = side == 0 ? tid : m - 1 - tid;  // the row's number from its end
            if (tid < m) {
                const double num = piv[side][tid];
                const double den = u % 8 == 0 ? before[side][u >> 3] : piv[side][side == 0 ? tid - 1 : tid + 1];
                // after a minor that vanishes: the pivot that a tiny one before it leaves
                p[side] = den != 0.0 ? num / den : diag - e2[side] / tiny;
                if (fabs(p[side]) < tiny) p[side] = p[side] < 0.0 ? -tiny : tiny;
            }
        }
        __syncthreads();
        if (tid < m) {
            piv[0][tid] = p[0];
            piv[1][tid] = p[1];
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
        // the ratio of each row to its neighbour on the side of row `at`, and the reciprocal pivot
        if (tid < m) {
            const double r = eig::rcp_of(piv[tid < at ? 0 : 1][tid]);
            z[tid] = tid < at ? -e[tid] * r : tid > at ? -e[tid - 1] * r : 1.0;
            t[tid] = make_double2(z[tid], r);
        }
        __syncthreads();
        if (tid < 2) {
            const int by = tid == 0 ? -1 : 1, count = tid == 0 ? at : m - 1 - at;
            double p = 1.0;
#pragma unroll 1
            for (int q0 = 1; q0 <= count; q0 += 8)
                batched<8, 8>([&](int q) { return z[at + by * (q0 + q <= count ? q0 + q : count)]; },
                              [&](int q, double f) { z[q0 + q <= count ? at + by * (q0 + q) : eig::kMax] = p *= f; });
        }
        __syncthreads();
        double n2 = 0.0;
        for (int i = lane; i < m; i += 64) n2 = fma(z[i], z[i], n2);
        shift = fma(gamma, eig::rcp_of(eig::sum64(n2)), shift);
        row = at;
    }

    // The reflectors in reverse (Q; forwards, its transpose) on a vector over the lanes of the
    // first wavefront, two at a time, so that one sum over the lanes waits while the other
    // runs: (1 - a u u^T)(1 - b v v^T) x needs u . x, v . x and u . v, and the last is there
    // before (link, by all wavefronts).  Reflector m - 2 acts on one entry and is 1.  What a
    // turn costs is the instructions of its one wavefront, about 8 cycles each: stored with
    // zeros in whole turns of 64 lanes the reflectors need no masks (m = 96: packed 15 us a turn,
    // so 10).
    auto fetch = [&](int s, double (&v)[NL]) {
#pragma unroll
        for (int l = 0; l < NL; ++l) v[l] = refl[s * STRIDE + lane + 64 * l];
        return tau[s];
    };
    auto dot = [&](const double (&a)[NL], const double (&b)[NL]) {
        double c = 0.0;
#pragma unroll
        for (int l = 0; l < NL; ++l) c = fma(a[l], b[l], c);
        return eig::sum64(c);
    };
    const int pairs = (m - 2) / 2;
    for (int p = tid >> 6; p < pairs; p += kThreads / 64) {
        double u[NL], v[NL];
        fetch(2 * p, u);
        fetch(2 * p + 1, v);
        const double c = dot(u, v);
        if (lane == 0) link[p] = c;
    }
    __syncthreads();
    auto reflect = [&](double (&x)[NL], bool forwards) {
        double u[NL], v[NL], tu, tv, c;  // the next pair in the order of application
        auto take = [&](int p) {
            tu = fetch(2 * p + (forwards ? 0 : 1), u);
            tv = fetch(2 * p + (forwards ? 1 : 0), v);
            c = link[p];
        };
        int p = forwards ? 0 : pairs - 1;
        take(p);
        for (int q = 0; q < pairs; ++q) {
            double a = 0.0, b = 0.0, u0[NL], v0[NL];
            const double ta = tu, tb = tv, ab = c;
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                a = fma(u0[l] = u[l], x[l], a);
                b = fma(v0[l] = v[l], x[l], b);
            }
            if (q + 1 < pairs) take(p += forwards ? 1 : -1);
            a = ta * eig::sum64(a);
            b = tb * fma(-a, ab, eig::sum64(b));
#pragma unroll
            for (int l = 0; l < NL; ++l) x[l] = fma(-b, v0[l], fma(-a, u0[l], x[l]));
        }
    };
    auto read = [&](double (&x)[NL]) {
#pragma unroll
        for (int l = 0; l < NL; ++l) x[l] = lane + 64 * l < m ? z[lane + 64 * l] : 0.0;
    };
    auto write = [&](const double (&x)[NL]) {
#pragma unroll
        for (int l = 0; l < NL; ++l)
            if (lane + 64 * l < m) z[lane + 64 * l] = x[l];
    };
    double y[NL], r[NL], x[NL];
    if (tid < 64) {
        read(y);
        reflect(y, false);
        const double c = 1.0 / sqrt(dot(y, y));
#pragma unroll
        for (int l = 0; l < NL; ++l) y[l] *= c;
        write(y);
    }
    __syncthreads();

    // One step of refinement on H itself.  The reduction's rounding is that of the largest
    // entry, so behind walls of V the pair comes out good to eps V only (a level of 4.6 meV behind
    // walls of 1e4 meV: 4e-13, 1e8: 8e-10), where H's own rows, whose large entries meet small
    // components, tell it to rounding.  With r = (H - level) y and y . r = 0 the
    // correction is d = -Q (T - shift)^-1 Q^T r on the rest of the space, solved with row `row`
    // held at zero from the pivots that are there, and the level gains d . r.  At walls of 1e8 meV
    // the packet then is 9e-16 off (1.2e-10 without); the kernel takes 184 us at 128 x 96 (177
    // without it, and with masked reflectors and pivots by reciprocals).
    const int parts = kThreads / m;
    if (tid < parts * m) {
        const int i = tid % m, p = tid / m;
        double a = 0.0;
        for (int j0 = p; j0 < m; j0 += 8 * parts)
            batched<8, 8>(
                [&](int q) {
                    const int j = j0 + q * parts < m ? j0 + q * parts : m - 1, at = i - j;
                    return make_double2(circ[at < 0 ? at + m : at], j0 + q * parts < m ? z[j] : 0.0);
                },
                [&](int, double2 f) { a = fma(f.x, f.y, a); });
        piv[0][tid] = p == 0 ? fma(element(i, i) - circ[0] - shift, z[i], a) : a;
    }
    __syncthreads();
    if (tid >= 64) return;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        r[l] = 0.0;
        if (lane + 64 * l < m)
            for (int p = 0; p < parts; ++p) r[l] += piv[0][p * m + lane + 64 * l];
    }
    const double mu = dot(y, r);
    double level = shift + mu;
#pragma unroll
    for (int l = 0; l < NL; ++l) x[l] = -(r[l] = fma(-mu, y[l], r[l]));
    reflect(x, true);
    write(x);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // rows above `row` by one lane, rows below it by another: elimination towards it, then back,
    // w = ratio w_before + z (over the pivot); eight rows are read ahead of the chain
    if (lane < 2) {
        const int dir = lane == 0 ? 1 : -1, end = lane == 0 ? 0 : m - 1;
        const int count = (row - end) * dir;
        for (int back = 0; back < 2; ++back) {
            const int at = back ? row - dir : end, by = back ? -dir : dir;
            double w = 0.0;
            for (int q0 = 0; q0 < count; q0 += 8)
                batched<8, 8>(
                    [&](int q) {
                        const int k = q0 + q < count ? q0 + q : count - 1, i = at + by * k;
                        const double2 f = t[back || k == 0 ? i : i - by];
                        return make_double2(f.x, back ? z[i] * f.y : z[i]);
                    },
                    [&](int q, double2 f) {
                        w = fma(f.x, w, f.y);
                        z[q0 + q < count ? at + by * (q0 + q) : eig::kMax] = w;
                    });
        }
    }
    if (lane == 0) z[row] = 0.0;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    read(x);
    reflect(x, false);
    const double along = dot(y, x);
#pragma unroll
    for (int l = 0; l < NL; ++l) x[l] = fma(-along, y[l], x[l]);
    // a large one comes from a level next to this one that rounding does not tell apart
    if (dot(x, x) < 1e-6) {
        level += dot(x, r);
#pragma unroll
        for (int l = 0; l < NL; ++l) y[l] += x[l];
    }
    if (tid == 0) g.e1[blockIdx.x] = level;
    double big = 0.0;
#pragma unroll
    for (int l = 0; l < NL; ++l) big = fmax(big, fabs(y[l]));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
    double scale = 1.0 / sqrt(dot(y, y));
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
    // the reflectors; with ny > kRegMax the rest of the matrix between the two register forms
    const size_t lds = (MEM ? 64 * 64 : (size_t)(e.ny - 1) * reflector_stride(e.ny)) * sizeof(double);
    auto fn = k_edge_state<RA, CB, MEM>;
    if (lds > 8 * 1024) {
        // with its static LDS (29 KB) the block may be past 64 KB, which has to be allowed
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(fn, dim3(e.nx), dim3(kThreads), lds, s, e);
    return hipGetLastError();
}

}  // namespace

size_t edge_work_doubles(int nx, int ny) {
    return ny > eig::kRegMax ? (size_t)nx * edge_work_per_k(ny) : 0;
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
