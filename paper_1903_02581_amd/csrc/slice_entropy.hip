// Von Neumann entropy of a slice phi(a, b) = Psi(x1_a, y1, x2_b, y2) on the GPU
// (arXiv 1903.02581 Sec. III.C, Eq. (reduced_density)): rho = phi phi^dagger over
// the smaller side, normalised, S = -sum lambda ln lambda over its eigenvalues.
//
// Five kernels: the gather (with the slice's squared norm in partial sums), the
// Gram matrix, its tridiagonalisation by one workgroup with the matrix in
// registers (eigen_regs.hpp), the eigenvalues by bisection, a wavefront each, and
// the sum.  All arithmetic is FP64, sums in a fixed order.  Only (S, norm) leave
// the GPU.  Measured: 4 + 12 + 239 + 26 + 4 us at m = 128, 4 + 8 + 75 + 14 + 4 us at
// m = 64, the tridiagonalisation's chain of steps bounding both.  On the host, with the 2m x 2m real embedding and cyclic Jacobi, one call took
// 15 ms at m = 64 and 0.7-1.0 s at m = 128.
#include "axis_pass.hpp"
#include "eigen_regs.hpp"
#include "hom4d_internal.hpp"

namespace hom4d_impl {
namespace {

using namespace dev;

constexpr int kTile = 16;    // Gram tile
constexpr int kChunk = 32;   // its steps along the long side

// Row p of out: phi[p][.] (left) or the conjugate of column p of phi (right), so
// that rho = out out^dagger in either case.  part: the block's sum of |phi|^2.
template <class S>
__global__ void k_slice_gather(const S* psi, SliceIndex ix, int m, int kd, int left, int jy1, int jy2, int nx, int ny,
                               double2* out, double* part) {
    __shared__ double red[4];
    const int idx = blockIdx.x * 256 + threadIdx.x;
    double n2 = 0.0;
    if (idx < m * kd) {
        const int p = idx / kd, k = idx % kd;
        const int64_t nxy = (int64_t)nx * ny;
        const int i1 = ix.a[left ? p : k], i2 = ix.b[left ? k : p];
        double2 v = ld<S>(psi + ((int64_t)i1 * ny + jy1) * nxy + (int64_t)i2 * ny + jy2);
        n2 = v.x * v.x + v.y * v.y;
        if (!left) v.y = -v.y;
        out[idx] = v;
    }
    const double s = block_sum(n2, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Sum of the gather's partial sums (at most 256), the same in every thread of a
// 256-thread block.
__device__ double slice_norm(const double* part, int nparts, double* red) {
    const double s = block_sum((int)threadIdx.x < nparts ? part[threadIdx.x] : 0.0, red);
    if (threadIdx.x == 0) red[4] = s;
    __syncthreads();
    return red[4];
}

// rho[i][j] = sum_k a[i][k] conj(a[j][k]) / norm, 16 x 16 elements per block, lower
// tiles only; the upper ones are their conjugates.
__global__ void __launch_bounds__(256) k_slice_gram(const double2* a, int m, int kd, const double* part, int nparts,
                                                    double2* rho) {
    __shared__ double red[5];
    __shared__ double2 ti[kTile][kChunk + 1], tj[kTile][kChunk + 1];
    if (blockIdx.y > blockIdx.x) return;
    const double inv = 1.0 / sqrt(slice_norm(part, nparts, red));
    const int tid = threadIdx.x, r = tid / kTile, c = tid % kTile;
    const int i0 = blockIdx.x * kTile, j0 = blockIdx.y * kTile;
    double2 acc = make_double2(0.0, 0.0);
    for (int k0 = 0; k0 < kd; k0 += kChunk) {
        for (int q = tid; q < kTile * kChunk; q += 256) {
            const int row = q / kChunk, k = k0 + q % kChunk;
            const bool in = k < kd;
            const double2 zero = make_double2(0.0, 0.0);
            ti[row][q % kChunk] = in && i0 + row < m ? cscale(a[(i0 + row) * kd + k], inv) : zero;
            tj[row][q % kChunk] = in && j0 + row < m ? cscale(a[(j0 + row) * kd + k], inv) : zero;
        }
        __syncthreads();
#pragma unroll 8
        for (int k = 0; k < kChunk; ++k) {
            const double2 x = ti[r][k], y = tj[c][k];
            acc = make_double2(fma(x.x, y.x, fma(x.y, y.y, acc.x)), fma(x.y, y.x, fma(-x.x, y.y, acc.y)));
        }
        __syncthreads();
    }
    const int i = i0 + r, j = j0 + c;
    if (i < m && j < m && (blockIdx.x != blockIdx.y || j <= i)) {
        if (i == j) acc.y = 0.0;
        rho[i * m + j] = acc;
        if (i != j) rho[j * m + i] = conjd(acc);
    }
}

// One block of TR x 16 threads: diagonal d and squared off-diagonals e2 of the
// tridiagonal form of rho, steps s0 .. s0 + n - 1 of it; the rest of the matrix goes back to
// memory if the steps end short of the last.  With more than eig::kRegMax rows the
// first steps run on the matrix in memory.
template <int TR, int RA, int CB, int CE = CB>
__global__ void __launch_bounds__(16 * TR) k_slice_tridiag(double2* rho, int m, int s0, int n, double* d, double* e2) {
    __shared__ eig::Work<double2> wk;
    __shared__ double off[eig::kMax];  // in LDS first: a step's barriers would wait for its store to memory
    const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15, first = s0, end = s0 + n;
    auto keep = [&](int s, const auto& h, const double2*) {
        if (tid == 0) off[s0 + s] = eig::abs2(h.e);
    };
    wk.clear();
    if constexpr (TR * RA == eig::kRegMax) {
        if (m > eig::kRegMax) {
            eig::tridiag_global<double2, TR>(rho, m, m - eig::kRegMax, wk, d, keep);
            s0 = m - eig::kRegMax;
            wk.clear();
        }
    }
    double2 A[RA][CB];
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int i = s0 + tr + TR * a, j = s0 + tc + 16 * b;
            A[a][b] = i < m && j < m ? rho[(size_t)i * m + j] : make_double2(0.0, 0.0);
        }
    eig::tridiag_regs<double2, TR, RA, CB, CE>(A, m - s0, end - s0, wk, d + s0, keep);
    if constexpr (CE < CB) {
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int i = s0 + tr + TR * a, j = s0 + tc + 16 * b;
                if (i >= end && j >= end && i < m && j < m) rho[(size_t)i * m + j] = A[a][b];
            }
    }
    __syncthreads();
    if (tid >= first && tid < end) e2[tid] = off[tid];
}

// Eigenvalue k per wavefront.  rho is positive with unit trace, so they lie in
// [0, 1] up to rounding; ten rounds of 65 leave an interval below 1e-18.
__global__ void __launch_bounds__(256) k_slice_spectrum(const double* d, const double* e2, int m, double* lam) {
    __shared__ double2 t[eig::kSturmRows];
    const int tid = threadIdx.x;
    t[tid] = tid < m ? eig::sturm_row(d[tid], tid > 0 ? e2[tid - 1] : 0.0) : eig::sturm_pad(3.0);
    __syncthreads();
    const int k = blockIdx.x * 4 + (tid >> 6);
    if (k >= m) return;
    double lo = -1e-9, hi = 1.0 + 1e-9;
    eig::sturm_select(t, m, k, lo, hi, 10);
    if ((tid & 63) == 0) lam[k] = 0.5 * (lo + hi);
}

__global__ void k_slice_entropy(const double* lam, int m, const double* part, int nparts, double* out) {
    __shared__ double red[5];
    const double nrm = slice_norm(part, nparts, red);
    const double x = (int)threadIdx.x < m ? lam[threadIdx.x] : 0.0;
    __syncthreads();
    const double s = block_sum(x > 0.0 ? -x * log(x) : 0.0, red);
    if (threadIdx.x == 0) {
        out[0] = s;
        out[1] = nrm;
    }
}

}  // namespace

hipError_t launch_slice_entropy(const void* psi, bool mixed, const SliceIndex& ix, int n1, int jy1, int n2, int jy2,
                                int nx, int ny, double2* phi, double2* rho, double* scratch, double* out,
                                hipStream_t s) {
    if (n1 < 1 || n1 > eig::kMax || n2 < 1 || n2 > eig::kMax) return hipErrorInvalidValue;
    const int left = n1 <= n2 ? 1 : 0;
    const int m = left ? n1 : n2, kd = left ? n2 : n1;
    const int nparts = (m * kd + 255) / 256;  // at most 256
    double* part = scratch;
    double* d = scratch + 256;
    double* e2 = d + 256;
    double* lam = e2 + 256;
    if (mixed)
        hipLaunchKernelGGL(k_slice_gather<float2>, dim3(nparts), dim3(256), 0, s, (const float2*)psi, ix, m, kd, left, jy1,
                           jy2, nx, ny, phi, part);
    else
        hipLaunchKernelGGL(k_slice_gather<double2>, dim3(nparts), dim3(256), 0, s, (const double2*)psi, ix, m, kd, left,
                           jy1, jy2, nx, ny, phi, part);
    const int nt = (m + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_slice_gram, dim3(nt, nt), dim3(256), 0, s, phi, m, kd, part, nparts, rho);
    // the smallest register form that holds the matrix, on as few wavefronts as hold it;
    // from 128 rows down to 64 in the one, the rest in the other, whose four wavefronts do
    // a step in 1.2 us where eight take 1.6 (m = 128: 252 -> 239 us)
    int s0 = 0;
    if (m > 64) {
        s0 = m - 64;
        hipLaunchKernelGGL((k_slice_tridiag<32, 4, 8, 4>), dim3(1), dim3(512), 0, s, rho, m, 0, s0, d, e2);
    }
    if (m <= 32)
        hipLaunchKernelGGL((k_slice_tridiag<16, 2, 2>), dim3(1), dim3(256), 0, s, rho, m, 0, m - 1, d, e2);
    else
        hipLaunchKernelGGL((k_slice_tridiag<16, 4, 4>), dim3(1), dim3(256), 0, s, rho, m, s0, m - 1 - s0, d, e2);
    hipLaunchKernelGGL(k_slice_spectrum, dim3((m + 3) / 4), dim3(256), 0, s, d, e2, m, lam);
    hipLaunchKernelGGL(k_slice_entropy, dim3(1), dim3(256), 0, s, lam, m, part, nparts, out);
    return hipGetLastError();
}

}  // namespace hom4d_impl
