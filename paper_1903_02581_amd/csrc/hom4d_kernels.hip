// Launchers of the pass kernels and the elementwise / reduction kernels of the
// two-electron split-step propagator (gfx950, wave64).
//
// The pass kernels (axis_pass.hpp, axis3_pass.hpp, plane_pass.hpp) apply one
// batched transform round trip along a coordinate of Psi[x1][y1][x2][y2] with
// the diagonal kinetic phase of that coordinate in reciprocal space (Appendix A
// of arXiv 1903.02581: T_x diagonal in (k_x, y), T_y diagonal in k_y), and on
// the passes that carry it the real-space potential factor
// exp(-i tau (V1 + V2 + V12) / hbar) (Sec. II.C Eq. (evoloperat); Sec. III.B
// Eq. (coulomb)).  A thread loads its elements of a line straight from HBM
// (for strided axes consecutive lanes read consecutive lines, so every row
// access of a wavefront is one contiguous run), runs register DFTs, exchanges
// through LDS between radix stages, applies the phase at known wave numbers and
// runs the transposed network back to its own elements, which it stores in
// place.  All arithmetic is FP64; the state is stored as complex128 or complex64.
//
// This file also holds the launch logic (kernel choice per line length,
// storage type, state count and potential-factor form) and the FP64
// reductions, whose partial sums are combined in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <unordered_set>

#include "axis_pass.hpp"
#include "hom4d_internal.hpp"

using namespace hom4d_dev;

namespace hom4d_impl {

using dev::AxisKernel;
AxisKernel pick_axis_f64_1(int axis, int n, int vk, bool nt, int* t);
AxisKernel pick_axis_f64_2(int axis, int n, int vk, bool nt, int* t);
AxisKernel pick_axis_f32_1(int axis, int n, int vk, bool nt, int* t);
AxisKernel pick_axis_f32_2(int axis, int n, int vk, bool nt, int* t);
AxisKernel pick_axis3_f64(int axis, int n, int vk, int nst, bool nt, bool pers, int w, int* t);
AxisKernel pick_axis3_f32(int axis, int n, int vk, int nst, bool nt, bool pers, int w, int* t);
AxisKernel pick_plane_f64(int nx, int ny, int vk, int* nt);
AxisKernel pick_plane_f32(int nx, int ny, int vk, int* nt);
AxisKernel pick_plane_regs(int nx, int ny, bool nt, int* threads, size_t* lds);
AxisKernel pick_plane1_f64(int nx, int ny, int vk, Plane1Launch* p);
AxisKernel pick_plane1_f32(int nx, int ny, int vk, Plane1Launch* p);

namespace {

using namespace dev;

// --------------------------------------------------------------------------------------
// Elementwise / reduction kernels over all pairs (r1, r2).  A block takes one chunk of
// r2 and a strided set of rows r1: every thread keeps its r2 table entries
// (weights, orbitals) in registers over its rows and moves 16 bytes of state per
// load or store, K of them per row, where one pair per thread and load re-read the
// tables for every point and kept one 8- or 16-byte access in flight.  Bound by HBM
// (init_norm by its FP64 products): 128x96 complex128 init_write 576 -> 438 us (5.5
// TB/s), init_norm 230 -> 111; 256x128 complex64 2.67 -> 1.57 ms and 1.55 -> 0.77;
// 128x64 complex64 obs 164 -> 131 us, loss_lambda 246 -> 182.  The summation order
// depends only on the launch shape: results are bitwise repeatable.

constexpr int kPairThreads = 256;
constexpr int kPairBlocks = 2048;  // eight 256-thread blocks per CU
template <class S>
constexpr int kVec = 16 / (int)sizeof(S);  // state elements per access

template <class S>
__device__ __forceinline__ void ld16(const S* p, double2* v) {
    if constexpr (std::is_same<S, double2>::value) {
        v[0] = *p;
    } else {
        const float4 f = *reinterpret_cast<const float4*>(p);
        v[0] = make_double2((double)f.x, (double)f.y);
        v[1] = make_double2((double)f.z, (double)f.w);
    }
}
template <class S>
__device__ __forceinline__ void st16(S* p, const double2* v) {
    if constexpr (std::is_same<S, double2>::value)
        *p = v[0];
    else
        *reinterpret_cast<float4*>(p) = make_float4((float)v[0].x, (float)v[0].y, (float)v[1].x, (float)v[1].y);
}

// The r2 positions of a thread: K groups of kVec<S> consecutive ones (every supported nxy is a
// multiple of 4, so a group is inside the row or outside it).
template <class S, int K>
struct PairTile {
    int pos[K];
    bool in[K];
    __device__ __forceinline__ explicit PairTile(int nxy) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            pos[k] = (((int)blockIdx.x * K + k) * kPairThreads + (int)threadIdx.x) * kVec<S>;
            in[k] = pos[k] < nxy;
        }
    }
};

// psi_a(r1) psi_b(r2) + sym psi_b(r1) psi_a(r2)
__device__ __forceinline__ double2 pair_value(double2 a1, double2 b1, double2 a2, double2 b2, int sym) {
    double2 p = cmul(a1, b2);
    if (sym != 0) {
        const double2 q = cmul(b1, a2);
        p = make_double2(p.x + sym * q.x, p.y + sym * q.y);
    }
    return p;
}

// For sym != 0 the sum is symmetric in (r1, r2), so a tile of r2 takes only half of the
// others as its r1, those up to half way round from it: each pair of tiles is visited from
// one side and counts twice, a tile with itself and the one opposite (from both sides) once.
// FP64 operations bound it: 128x96 109 us with all pairs, 69 so.
template <int K>
__global__ void __launch_bounds__(kPairThreads) k_init_norm(const double2* pa, const double2* pb, int sym, int nxy,
                                                            double* part) {
    __shared__ double red[kPairThreads / 64];
    const PairTile<double2, K> tile(nxy);
    double2 a2[K], b2[K];
#pragma unroll
    for (int k = 0; k < K; ++k) a2[k] = b2[k] = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tile.in[k]) {
            a2[k] = pa[tile.pos[k]];
            b2[k] = pb[tile.pos[k]];
        }
    double acc = 0.0;
    constexpr int T = K * kPairThreads;
    const int tiles = gridDim.x, visits = sym != 0 ? tiles / 2 + 1 : tiles;
    for (int r = blockIdx.y; r < visits * T; r += gridDim.y) {
        const int turn = r / T;
        int r1 = r + blockIdx.x * T;
        if (r1 >= tiles * T) r1 -= tiles * T;
        if (r1 >= nxy) continue;
        const double weight = sym != 0 && turn != 0 && 2 * turn != tiles ? 2.0 : 1.0;
        const double2 a1 = pa[r1], b1 = pb[r1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double2 p = pair_value(a1, b1, a2[k], b2[k], sym);
            if (tile.in[k]) acc += weight * (p.x * p.x + p.y * p.y);
        }
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// The same norm for complex64 states, rows r1 over blocks and r2 over threads.  Its
// last bit sets the last bit of every initial value, a few of which then round to the other
// complex64 neighbour, and within a step or two the rounding of every pass follows: a
// complex64 run is reproducible only with this order of summation.  It re-reads the
// orbitals for every pair (128x64 108 us against 57, 256x128 1.55 ms against 0.77).
constexpr int kNormRows = 1024;
__global__ void k_init_norm_rows(const double2* pa, const double2* pb, int sym, int nxy, double* part) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int r1 = blockIdx.x; r1 < nxy; r1 += gridDim.x) {
        const double2 a1 = pa[r1], b1 = pb[r1];
        for (int r2 = threadIdx.x; r2 < nxy; r2 += blockDim.x) {
            const double2 p = pair_value(a1, b1, pa[r2], pb[r2], sym);
            acc += p.x * p.x + p.y * p.y;
        }
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

template <class S, int K>
__global__ void __launch_bounds__(kPairThreads) k_init_write(S* psi, const double2* pa, const double2* pb, int sym,
                                                             int nxy, double scale) {
    constexpr int V = kVec<S>;
    const PairTile<S, K> tile(nxy);
    double2 a2[K][V], b2[K][V];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int q = 0; q < V; ++q) {
            a2[k][q] = b2[k][q] = make_double2(0.0, 0.0);
            if (tile.in[k]) {
                a2[k][q] = pa[tile.pos[k] + q];
                b2[k][q] = pb[tile.pos[k] + q];
            }
        }
    for (int r1 = blockIdx.y; r1 < nxy; r1 += gridDim.y) {
        const double2 a1 = pa[r1], b1 = pb[r1];
        S* row = psi + (int64_t)r1 * nxy;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double2 v[V];
#pragma unroll
            for (int q = 0; q < V; ++q) v[q] = cscale(pair_value(a1, b1, a2[k][q], b2[k][q], sym), scale);
            if (tile.in[k]) st16<S>(row + tile.pos[k], v);
        }
    }
}

template <class S, int K>
__global__ void __launch_bounds__(kPairThreads) k_obs(const S* psi, const double* w, int nxy, double* part) {
    constexpr int V = kVec<S>;
    __shared__ double red[kPairThreads / 64];
    const PairTile<S, K> tile(nxy);
    double w2[K][V];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int q = 0; q < V; ++q) w2[k][q] = tile.in[k] ? w[tile.pos[k] + q] : 0.0;
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int r1 = blockIdx.y; r1 < nxy; r1 += gridDim.y) {
        const S* row = psi + (int64_t)r1 * nxy;
        double2 p[K][V];
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int q = 0; q < V; ++q) p[k][q] = make_double2(0.0, 0.0);
            if (tile.in[k]) ld16<S>(row + tile.pos[k], p[k]);
        }
        // the row's sums over this thread's r2: all, top and bottom weighted
        double all = 0.0, top = 0.0, bottom = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const double d = p[k][q].x * p[k][q].x + p[k][q].y * p[k][q].y;
                all += d;
                top += w2[k][q] * d;
                bottom += (1.0 - w2[k][q]) * d;
            }
        const double w1 = w[r1];
        acc[0] += all;
        acc[1] += w1 * top;
        acc[2] += w1 * bottom;
        acc[3] += (1.0 - w1) * top;
        acc[4] += (1.0 - w1) * bottom;
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const double s = block_sum(acc[q], red);
        if (threadIdx.x == 0) part[(blockIdx.y * gridDim.x + blockIdx.x) * 5 + q] = s;
    }
}

struct LossCoeffs {
    double c[4];
};

template <class S, int K>
__global__ void __launch_bounds__(kPairThreads) k_loss_lambda(const S* psi, S* lam, const double* w, LossCoeffs cf,
                                                              int nxy, double* part) {
    constexpr int V = kVec<S>;
    __shared__ double red[kPairThreads / 64];
    const PairTile<S, K> tile(nxy);
    double w2[K][V];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int q = 0; q < V; ++q) w2[k][q] = tile.in[k] ? w[tile.pos[k] + q] : 0.0;
    double acc = 0.0;
    for (int r1 = blockIdx.y; r1 < nxy; r1 += gridDim.y) {
        const int64_t o = (int64_t)r1 * nxy;
        double2 p[K][V];
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int q = 0; q < V; ++q) p[k][q] = make_double2(0.0, 0.0);
            if (tile.in[k]) ld16<S>(psi + o + tile.pos[k], p[k]);
        }
        const double w1 = w[r1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double2 v[V];
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const double wl = cf.c[0] * w1 * w2[k][q] + cf.c[1] * w1 * (1.0 - w2[k][q]) +
                                  cf.c[2] * (1.0 - w1) * w2[k][q] + cf.c[3] * (1.0 - w1) * (1.0 - w2[k][q]);
                acc += wl * (p[k][q].x * p[k][q].x + p[k][q].y * p[k][q].y);
                v[q] = cscale(p[k][q], wl);
            }
            if (tile.in[k]) st16<S>(lam + o + tile.pos[k], v);
        }
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// out[block * width + q] = sum of part[b * width + q] over the block's share of the
// partial sums, fixed order; grid (width, blocks).  Bound by the latency of its loads: eight in
// flight take the observables of 32x32 complex64 states from 29.9 to 28.5 us.
__global__ void __launch_bounds__(256) k_reduce_parts(const double* part, int nparts, int width, double* out) {
    __shared__ double red[4];
    const int q = blockIdx.x;
    double acc = 0.0;
    const int step = gridDim.y * 256;
    for (int b0 = blockIdx.y * 256 + threadIdx.x; b0 < nparts; b0 += 8 * step)
        batched<8, 8>(
            [&](int i) { return b0 + i * step < nparts ? part[(int64_t)(b0 + i * step) * width + q] : 0.0; },
            [&](int i, double v) { acc = b0 + i * step < nparts ? acc + v : acc; });
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) out[blockIdx.y * width + q] = s;
}

template <class S>
__global__ void k_gather(const S* psi, const int32_t* ix1, int n1, int jy1, const int32_t* ix2, int n2, int jy2,
                         int nx, int ny, double2* out) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n1 * n2) return;
    const int a = idx / n2, b = idx % n2;
    const int64_t nxy = (int64_t)nx * ny;
    const int64_t off = ((int64_t)ix1[a] * ny + jy1) * nxy + (int64_t)ix2[b] * ny + jy2;
    out[idx] = ld<S>(psi + off);
}

// out[r1] = sum_r2 |psi(r1, r2)|^2: one block per r1 over its contiguous plane.
template <class S>
__global__ void k_marginal(const S* psi, int nxy, double* out) {
    __shared__ double red[256];
    const int r1 = blockIdx.x;
    const S* row = psi + (int64_t)r1 * nxy;
    double acc = 0.0;
    for (int r2 = threadIdx.x; r2 < nxy; r2 += blockDim.x) {
        const double2 p = ld<S>(row + r2);
        acc += p.x * p.x + p.y * p.y;
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) out[r1] = s;
}

// out[r1] = |psi(r1, r2)|^2 for one fixed r2.
template <class S>
__global__ void k_conditional(const S* psi, int nxy, int r2, double* out) {
    const int r1 = blockIdx.x * blockDim.x + threadIdx.x;
    if (r1 >= nxy) return;
    const double2 p = ld<S>(psi + (int64_t)r1 * nxy + r2);
    out[r1] = p.x * p.x + p.y * p.y;
}

__global__ void k_zero(double* p, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// dL/dV from the marginals: 16 table entries per 256-thread block, 16 threads sharing
// the terms of each (one thread per entry summed up to nx + ny terms in a serial
// chain of loads on a few blocks: 128x64 82 -> 10 us).  g1 then g2, each in thread order.
constexpr int kFinishEntries = 16;
__global__ void __launch_bounds__(256) k_grad_finish(const double* m_x2, int bpr_x2, const double* m_y2, int bpr_y2,
                                                     const double* m_y1, const double* m_x1, int nx, int ny,
                                                     double gscale, double* dldv) {
    __shared__ double sum[16][kFinishEntries + 1];
    const int nxy = nx * ny;
    const int c = threadIdx.x % kFinishEntries, t = threadIdx.x / kFinishEntries;
    const int r = blockIdx.x * kFinishEntries + c;
    double g = 0.0;
    if (r < nxy) {  // the last block is partial on grids of 4 and 6 by 6 and 12 points
        for (int q = t; q < bpr_x2; q += 16) g += m_x2[(int64_t)r * bpr_x2 + q];
        for (int q = t; q < bpr_y2; q += 16) g += m_y2[(int64_t)r * bpr_y2 + q];
        for (int i = t; i < nx; i += 16) g += m_y1[(int64_t)i * nxy + r];
        for (int j = t; j < ny; j += 16) g += m_x1[(int64_t)j * nxy + r];
    }
    sum[t][c] = g;
    __syncthreads();
    if (t == 0 && r < nxy) {
        double a = 0.0;
        for (int q = 0; q < 16; ++q) a += sum[q][c];
        dldv[r] = gscale * a;
    }
}

// Grid of a pair kernel: four accesses per thread and row where they fill at least two thirds
// of their chunks of r2, one otherwise (48x48 complex64 fills 56% of two chunks: observables
// 43 us, with one access 38; 48x24 complex128 30 and 29; at 75% four are as fast); chunks by groups
// of rows, about kPairBlocks blocks, of the same number of rows each where that is up to
// four (32x24 complex128: 28 -> 25.5 us).  Fixed by the sizes alone.
template <class S>
int pair_chunks(int nxy, int k) {
    const int span = k * kPairThreads * kVec<S>;
    return (nxy + span - 1) / span;
}
template <class S>
bool pair_k4(int nxy) {
    constexpr int span = 4 * kPairThreads * kVec<S>;
    return nxy >= span && 3 * nxy >= 2 * span * pair_chunks<S>(nxy, 4);
}
template <class S>
dim3 pair_grid(int nxy) {
    const int chunks = pair_chunks<S>(nxy, pair_k4<S>(nxy) ? 4 : 1);
    const int groups = std::min(nxy, std::max(1, kPairBlocks / chunks)), rows = (nxy + groups - 1) / groups;
    return dim3(chunks, rows <= 4 ? (nxy + rows - 1) / rows : groups);
}
inline int blocks_of(dim3 g) { return (int)(g.x * g.y); }

}  // namespace

int axis3_threads(int n, int nst) {
    if (nst != 1 && nst != 2) return 0;
    switch (n) {
        case 96: return 8;
        case 128: return 16;
        case 256: return 32;
        default: return 0;
    }
}

bool fft_shape(int n, FftShape* out) {
    switch (n) {
        case 4: *out = {4, 1, 1}; return true;
        case 6: *out = {6, 1, 1}; return true;
        case 8: *out = {8, 1, 1}; return true;
        case 12: *out = {12, 1, 1}; return true;
        case 16: *out = {4, 4, 4}; return true;
        case 24: *out = {12, 2, 2}; return true;
        case 32: *out = {8, 4, 4}; return true;
        case 48: *out = {12, 4, 4}; return true;
        case 64: *out = {8, 8, 8}; return true;
        case 96: *out = {12, 8, 4}; return true;
        case 128: *out = {16, 8, 8}; return true;
        case 256: *out = {16, 16, 16}; return true;
        default: return false;
    }
}

// Blocks of fn (threads, dynamic LDS) resident on the whole device at once:
// blocks per CU times the CU count, cached per kernel and shape.
hipError_t resident_blocks(AxisKernel fn, int threads, size_t lds_bytes, int* out) {
    static std::mutex mu;
    static std::map<std::tuple<const void*, int, size_t>, int> cache;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_tuple(reinterpret_cast<const void*>(fn), threads, lds_bytes);
    auto it = cache.find(key);
    if (it != cache.end()) {
        *out = it->second;
        return hipSuccess;
    }
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(fn), threads,
                                                         lds_bytes);
    if (e != hipSuccess) return e;
    *out = per_cu * cus;
    cache[key] = *out;
    return hipSuccess;
}

// Dynamic LDS above 64 KB has to be enabled per kernel, once.
static hipError_t allow_lds(AxisKernel fn, size_t lds_bytes) {
    if (lds_bytes <= 64 * 1024) return hipSuccess;
    static std::mutex mu;
    static std::unordered_set<const void*> raised;
    std::lock_guard<std::mutex> lock(mu);
    const void* key = reinterpret_cast<const void*>(fn);
    if (!raised.count(key)) {
        hipError_t e = hipFuncSetAttribute(key, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised.insert(key);
    }
    return hipSuccess;
}

hipError_t launch_axis(int axis, int n, bool mixed, int nst, bool pers, const PassArgs& a, int64_t nlines,
                       size_t lds_bytes, hipStream_t s) {
    int t = 0;
    AxisKernel fn = nullptr;
    const int vk = a.vmode == 0 ? 0 : (a.vdirect ? 2 : 1);
    const bool nt = a.nt != 0;
    if (axis3_threads(n, nst) > 0)
        fn = mixed ? pick_axis3_f32(axis, n, vk, nst, nt, pers, a.W, &t)
                   : pick_axis3_f64(axis, n, vk, nst, nt, pers, a.W, &t);
    else if (pers)
        return hipErrorInvalidValue;  // only the three-stage passes have a persistent form
    else if (!mixed)
        fn = (nst == 2) ? pick_axis_f64_2(axis, n, vk, nt, &t) : pick_axis_f64_1(axis, n, vk, nt, &t);
    else
        fn = (nst == 2) ? pick_axis_f32_2(axis, n, vk, nt, &t) : pick_axis_f32_1(axis, n, vk, nt, &t);
    if (!fn || a.W <= 0 || nlines % a.W != 0) return hipErrorInvalidValue;
    const int64_t nblocks = nlines / a.W;
    const int max_threads = axis3_threads(n, nst) > 0 ? axis3_block_threads(axis, n, nst, mixed) : 256;
    if (nblocks > 0x7fffffff || t * a.W > max_threads || lds_bytes > 160 * 1024) return hipErrorInvalidValue;
    if (axis3_threads(n, nst) > 0) {
        if (lds_bytes < axis3_pass_lds_bytes(n, a.W, nst, mixed, pers)) return hipErrorInvalidValue;
    } else {
        FftShape sh;
        if (!fft_shape(n, &sh)) return hipErrorInvalidValue;
        const size_t need = axis_xchg_bytes(axis, sh.n2 > 1 ? n : 0, a.W, nst, axis_xchg_c64(axis, mixed)) + 3u * (size_t)n * 16u;
        if (lds_bytes < need) return hipErrorInvalidValue;
    }
    hipError_t le = allow_lds(fn, lds_bytes);
    if (le != hipSuccess) return le;
    int64_t grid = nblocks;
    if (pers) {
        // persistent pass: the blocks that fit the device at once walk the
        // a.ntiles tiles
        if (a.ntiles != (uint32_t)nblocks) return hipErrorInvalidValue;
        int resident = 0;
        hipError_t e = resident_blocks(fn, t * a.W, lds_bytes, &resident);
        if (e != hipSuccess) return e;
        if (resident > 0) grid = std::min<int64_t>(nblocks, resident);
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(t * a.W), lds_bytes, s, a);
    return hipGetLastError();
}

bool plane_available(int nx, int ny) {
    constexpr int sizes[][2] = {{16, 16}, {24, 24}, {32, 32}, {48, 48}, {64, 64}, {48, 16}, {16, 48}};
    for (const auto& q : sizes)
        if (nx == q[0] && ny == q[1]) return true;
    return false;
}

hipError_t launch_plane(int nx, int ny, bool mixed, const PassArgs& a, hipStream_t s) {
    int nt = 0;
    const int vk = a.vdirect ? 2 : 1;
    AxisKernel fn = mixed ? pick_plane_f32(nx, ny, vk, &nt) : pick_plane_f64(nx, ny, vk, &nt);
    if (!fn || nt <= 0 || nt > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, dim3((unsigned)(nx * ny)), dim3(nt), 0, s, a);
    return hipGetLastError();
}

bool pair_available(int nx, int ny, bool mixed) {
    Plane1Launch p{};
    return (mixed ? pick_plane1_f32(nx, ny, 1, &p) : pick_plane1_f64(nx, ny, 1, &p)) != nullptr;
}

hipError_t launch_plane1(int nx, int ny, bool mixed, const PassArgs& a, hipStream_t s) {
    Plane1Launch p{};
    const int vk = a.vdirect ? 2 : 1;
    AxisKernel fn = mixed ? pick_plane1_f32(nx, ny, vk, &p) : pick_plane1_f64(nx, ny, vk, &p);
    if (!fn || p.lds > 160 * 1024 || (nx * ny) % p.w != 0) return hipErrorInvalidValue;
    hipError_t e = allow_lds(fn, p.lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3((unsigned)(nx * ny / p.w)), dim3(p.threads), p.lds, s, a);
    return hipGetLastError();
}

bool plane_regs_available(int nx, int ny) {
    int threads = 0;
    size_t lds = 0;
    return pick_plane_regs(nx, ny, false, &threads, &lds) != nullptr;
}

hipError_t launch_plane_regs(int nx, int ny, const PassArgs& a, hipStream_t s) {
    int threads = 0;
    size_t lds = 0;
    AxisKernel fn = pick_plane_regs(nx, ny, a.nt != 0, &threads, &lds);
    if (!fn || a.vdirect || lds > 160 * 1024) return hipErrorInvalidValue;
    hipError_t e = allow_lds(fn, lds);
    if (e != hipSuccess) return e;
    int resident = 0;
    e = resident_blocks(fn, threads, lds, &resident);
    if (e != hipSuccess) return e;
    const int grid = resident > 0 ? std::min(nx * ny, resident) : nx * ny;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(threads), lds, s, a);
    return hipGetLastError();
}

int reduction_parts(int nxy, bool mixed) {
    return mixed ? std::max(std::min(nxy, kNormRows), blocks_of(pair_grid<float2>(nxy)))
                 : blocks_of(pair_grid<double2>(nxy));
}

hipError_t launch_init_norm(const double2* pa, const double2* pb, bool mixed, int sym, int nxy, double* part,
                            int* nparts, hipStream_t s) {
    if (mixed) {
        *nparts = std::min(nxy, kNormRows);
        hipLaunchKernelGGL(k_init_norm_rows, dim3(*nparts), dim3(256), 0, s, pa, pb, sym, nxy, part);
        return hipGetLastError();
    }
    const dim3 g = pair_grid<double2>(nxy);
    *nparts = blocks_of(g);
    auto fn = pair_k4<double2>(nxy) ? k_init_norm<4> : k_init_norm<1>;
    hipLaunchKernelGGL(fn, g, dim3(kPairThreads), 0, s, pa, pb, sym, nxy, part);
    return hipGetLastError();
}

template <class S>
static void init_write(S* psi, const double2* pa, const double2* pb, int sym, int nxy, double scale, hipStream_t s) {
    auto fn = pair_k4<S>(nxy) ? k_init_write<S, 4> : k_init_write<S, 1>;
    hipLaunchKernelGGL(fn, pair_grid<S>(nxy), dim3(kPairThreads), 0, s, psi, pa, pb, sym, nxy, scale);
}
hipError_t launch_init_write(void* psi, bool mixed, const double2* pa, const double2* pb, int sym, int nxy,
                             double scale, hipStream_t s) {
    if (mixed)
        init_write((float2*)psi, pa, pb, sym, nxy, scale, s);
    else
        init_write((double2*)psi, pa, pb, sym, nxy, scale, s);
    return hipGetLastError();
}

template <class S>
static int obs(const S* psi, const double* w, int nxy, double* part, hipStream_t s) {
    const dim3 g = pair_grid<S>(nxy);
    auto fn = pair_k4<S>(nxy) ? k_obs<S, 4> : k_obs<S, 1>;
    hipLaunchKernelGGL(fn, g, dim3(kPairThreads), 0, s, psi, w, nxy, part);
    return blocks_of(g);
}
hipError_t launch_obs(const void* psi, bool mixed, const double* w, int nxy, double* part, int* nparts,
                      hipStream_t s) {
    *nparts = mixed ? obs((const float2*)psi, w, nxy, part, s) : obs((const double2*)psi, w, nxy, part, s);
    return hipGetLastError();
}

template <class S>
static int loss_lambda(const S* psi, S* lam, const double* w, const LossCoeffs& cf, int nxy, double* part,
                       hipStream_t s) {
    const dim3 g = pair_grid<S>(nxy);
    auto fn = pair_k4<S>(nxy) ? k_loss_lambda<S, 4> : k_loss_lambda<S, 1>;
    hipLaunchKernelGGL(fn, g, dim3(kPairThreads), 0, s, psi, lam, w, cf, nxy, part);
    return blocks_of(g);
}
hipError_t launch_loss_lambda(const void* psi, void* lam, bool mixed, const double* w, const double* coeffs, int nxy,
                              double* part, int* nparts, hipStream_t s) {
    const LossCoeffs cf{{coeffs[0], coeffs[1], coeffs[2], coeffs[3]}};
    *nparts = mixed ? loss_lambda((const float2*)psi, (float2*)lam, w, cf, nxy, part, s)
                    : loss_lambda((const double2*)psi, (double2*)lam, w, cf, nxy, part, s);
    return hipGetLastError();
}

hipError_t launch_reduce_parts(const double* part, int nparts, int width, double* scratch, double* out,
                               hipStream_t s) {
    // one block per sum takes 256 parts per round of dependent loads; past 16 rounds a
    // first stage of kReduceBlocks blocks pays for its launch (the reverse sweep's
    // dL/dB: 65536 parts at 128x64, 90 -> 5 us)
    if (nparts > 4096) {
        if (width != 1) return hipErrorInvalidValue;  // scratch holds one sum per block
        hipLaunchKernelGGL(k_reduce_parts, dim3(1, kReduceBlocks), dim3(256), 0, s, part, nparts, 1, scratch);
        part = scratch;
        nparts = kReduceBlocks;
    }
    hipLaunchKernelGGL(k_reduce_parts, dim3(width), dim3(256), 0, s, part, nparts, width, out);
    return hipGetLastError();
}

hipError_t launch_gather(const void* psi, bool mixed, const int32_t* ix1, int n1, int jy1, const int32_t* ix2, int n2,
                         int jy2, int nx, int ny, double2* out, hipStream_t s) {
    const int tot = n1 * n2;
    const int nb = (tot + 255) / 256;
    if (mixed)
        hipLaunchKernelGGL(k_gather<float2>, dim3(nb), dim3(256), 0, s, (const float2*)psi, ix1, n1, jy1, ix2, n2,
                           jy2, nx, ny, out);
    else
        hipLaunchKernelGGL(k_gather<double2>, dim3(nb), dim3(256), 0, s, (const double2*)psi, ix1, n1, jy1, ix2, n2,
                           jy2, nx, ny, out);
    return hipGetLastError();
}

hipError_t launch_marginal(const void* psi, bool mixed, int nxy, double* out, hipStream_t s) {
    if (mixed)
        hipLaunchKernelGGL(k_marginal<float2>, dim3(nxy), dim3(256), 0, s, (const float2*)psi, nxy, out);
    else
        hipLaunchKernelGGL(k_marginal<double2>, dim3(nxy), dim3(256), 0, s, (const double2*)psi, nxy, out);
    return hipGetLastError();
}

hipError_t launch_conditional(const void* psi, bool mixed, int nxy, int r2, double* out, hipStream_t s) {
    const int nb = (nxy + 255) / 256;
    if (mixed)
        hipLaunchKernelGGL(k_conditional<float2>, dim3(nb), dim3(256), 0, s, (const float2*)psi, nxy, r2, out);
    else
        hipLaunchKernelGGL(k_conditional<double2>, dim3(nb), dim3(256), 0, s, (const double2*)psi, nxy, r2, out);
    return hipGetLastError();
}

hipError_t launch_zero(double* p, int64_t count, hipStream_t s) {
    hipLaunchKernelGGL(k_zero, dim3(1024), dim3(256), 0, s, p, count);
    return hipGetLastError();
}

// Gradient partials of the reverse sweep for callers that cannot allocate
// (hom4d_grad_backward_noalloc): a fixed array in device memory, one copy per
// GPU that loads the library.  Host code never names it: each device's address
// is taken once, with that device current, and kept in scratch_ptrs.
namespace {
static __device__ __align__(256) double scratch[kScratchDoubles];
std::mutex scratch_mu;
double* scratch_ptrs[kMaxDevices] = {};
}  // namespace

hipError_t init_scratch(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (scratch_ptrs[device]) return hipSuccess;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;  // the caller makes the device current
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_ptrs[device] = static_cast<double*>(ptr);
    return hipSuccess;
}

double* scratch_on(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mu);
    return scratch_ptrs[device];
}

hipError_t launch_grad_finish(const double* m_x2, int bpr_x2, const double* m_y2, int bpr_y2, const double* m_y1,
                              const double* m_x1, int nx, int ny, double gscale, double* dldv, hipStream_t s) {
    const int nxy = nx * ny;
    hipLaunchKernelGGL(k_grad_finish, dim3((nxy + kFinishEntries - 1) / kFinishEntries), dim3(256), 0, s, m_x2, bpr_x2,
                       m_y2, bpr_y2, m_y1, m_x1, nx, ny, gscale, dldv);
    return hipGetLastError();
}

}  // namespace hom4d_impl
