// Fused (x2, y2) plane pass for planes whose complex128 image does not fit LDS beside a
// second workgroup: the plane lives in registers, sixteen elements per thread.
//
// One workgroup owns the contiguous nx * ny plane of one r1 and applies X2(tau), V(dt/2),
// Y2(dt) (arXiv 1903.02581, Sec. II.C Eq. (evoloperat); Appendix A) in one HBM read
// and one HBM write, where the per-axis passes take two of each.  Lines are 64 or 128
// points, n = n1 * 8, on eight consecutive lanes: a thread holds 8 or 16 elements of one
// line (or of two 64-point ones), a wavefront whole lines, so that every exchange of a
// transform stays inside the wavefront.  LDS holds one component of the plane, 8 bytes per
// element: an exchange moves the real parts, then the imaginary parts, through the same
// places, and the hand-off from columns to rows does the same between barriers.  Global
// accesses are runs of eight complex128 values, whole 128-byte lines.
//
// Places (in 8-byte slots, 32 to a turn of the banks): element p of line l at l S + p + p / 8
// with S = 8 or 24 mod 32, so that a half wavefront's writes (8 consecutive slots of 4
// lines) and reads (stride 9, 4 lines) each meet every bank once; the hand-off's
// rows are 12 mod 32 apart, conflict-free to write by columns and two-way in half the slots to read.  All of
// them, and the twiddles staged by (k, t), are one base per thread and immediate offsets.
#pragma once

#include "axis_pass.hpp"

namespace hom4d_impl {
namespace dev {

constexpr int plane_regs_threads(int nx, int ny) { return nx * ny / 16; }
constexpr int plane_regs_stride(int n) { return n / 8 * 9 + (n == 128 ? 8 : 0); }
constexpr int plane_regs_row(int ny) { return ny + 12; }
// LDS: the largest of the column, hand-off and row images, twiddles of both axes, the y
// kinetic factor.
constexpr size_t plane_regs_lds(int nx, int ny) {
    const int c = ny * plane_regs_stride(nx), h = nx * plane_regs_row(ny), r = nx * plane_regs_stride(ny);
    return (size_t)(c > h ? (c > r ? c : r) : (h > r ? h : r)) * sizeof(double) + (size_t)(nx + 2 * ny) * sizeof(double2);
}

// Walks a table from a 32-bit offset: the offset passes through an empty asm, so that the
// addresses formed from it are not formed ahead of this place (and held in registers, or
// spilled, until they are used).
struct TableWalk {
    const char* base;
    uint32_t off;
    __device__ __forceinline__ TableWalk(const double2* table, int index)
        : base(reinterpret_cast<const char*>(table)), off((uint32_t)index * (uint32_t)sizeof(double2)) {
        asm volatile("" : "+v"(off));
    }
    __device__ __forceinline__ double2 next(int step) {
        const double2 f = *reinterpret_cast<const double2*>(base + off);
        off += (uint32_t)(step * (int)sizeof(double2));
        return f;
    }
};

// One line of N = N1 * 8 points on eight lanes: the transform, a factor in reciprocal
// space, the inverse.  v[n1] is the element at n1 * 8 + t; L: the line's places; tw: the
// twiddle of (k, t) at 8 k + t.
template <int N, class Kin>
__device__ __forceinline__ void line_regs(double2* v, int t, double* L, const double2* tw, Kin&& kin) {
    constexpr int N1 = N / 8, IB = N1 / 8;
    double* La = L + t;      // element 8 k + t at 9 k
    double* Lb = L + 9 * t;  // element 8 (t + 8 ii) + j at 72 ii + j
    const double2* tl = tw + t;
    auto sync = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    dft<N1, -1>(v);
    after_loads();
    batched<N1, 4>([&](int k) { return tl[8 * k]; }, [&](int k, double2 w) { if (k > 0) v[k] = cmul(v[k], w); });
    after_loads();
#pragma unroll
    for (int k = 0; k < N1; ++k) La[9 * k] = v[k].x;
    sync();
    double re[N1];
#pragma unroll
    for (int e = 0; e < N1; ++e) re[e] = Lb[72 * (e / 8) + e % 8];
    sync();
#pragma unroll
    for (int k = 0; k < N1; ++k) La[9 * k] = v[k].y;
    sync();
#pragma unroll
    for (int e = 0; e < N1; ++e) v[e] = make_double2(re[e], Lb[72 * (e / 8) + e % 8]);
    sync();
#pragma unroll
    for (int ii = 0; ii < IB; ++ii) {
        dft<8, -1>(&v[8 * ii]);
        after_loads();
        kin(ii, &v[8 * ii]);  // wave numbers t + 8 ii + N1 k2
        after_loads();
        dft<8, 1>(&v[8 * ii]);
        after_loads();
    }
#pragma unroll
    for (int e = 0; e < N1; ++e) Lb[72 * (e / 8) + e % 8] = v[e].x;
    sync();
#pragma unroll
    for (int k = 0; k < N1; ++k) re[k] = La[9 * k];
    sync();
#pragma unroll
    for (int e = 0; e < N1; ++e) Lb[72 * (e / 8) + e % 8] = v[e].y;
    sync();
#pragma unroll
    for (int k = 0; k < N1; ++k) v[k] = make_double2(re[k], La[9 * k]);
    sync();
    batched<N1, 4>([&](int k) { return tl[8 * k]; }, [&](int k, double2 w) { if (k > 0) v[k] = cmulc(v[k], w); });
    after_loads();
    dft<N1, 1>(v);
    after_loads();
}

template <int NX, int NY, bool NT>
__global__ void __launch_bounds__(plane_regs_threads(NX, NY)) k_plane_regs(const PassArgs a) {
    constexpr int THREADS = plane_regs_threads(NX, NY), LINES = THREADS / 8;  // lines at a time
    constexpr int EX = NX / 8, EY = NY / 8, QX = NY / LINES, QY = NX / LINES;
    static_assert(QX * EX == 16 && QY * EY == 16, "sixteen elements a thread in either stage");
    constexpr int PB = THREADS == 1024 ? 2 : 4;  // potential-factor loads ahead: 128 registers a thread
    extern __shared__ double2 lds_raw[];
    double2* twx = lds_raw;
    double2* twy = twx + NX;
    double2* ky = twy + NY;
    double* L = reinterpret_cast<double*>(ky + NY);

    const int tid = threadIdx.x;
    int t = tid % 8, line = tid / 8;
    for (int i = tid; i < NX + NY; i += THREADS) {
        // twiddle of (k, t) at 8 k + t
        const int q = i < NX ? i : i - NX, jk = (q / 8) * (q % 8);
        lds_raw[i] = i < NX ? a.tw[jk] : a.tw2[jk];
    }
    __syncthreads();
    // Planes blockIdx.x, + gridDim.x, ...  Only the hand-off needs the workgroup: from one
    // hand-off to the next -- rows, stores, the next plane's loads, columns -- a wavefront of
    // a square plane keeps to its own lines' places, so that some wait for HBM while others
    // transform (one plane per block: 64x128 1.69 -> 1.62 ms per step, 128x128 6.71 -> 6.63).
    for (int r1 = blockIdx.x; r1 < NX * NY; r1 += gridDim.x) {
        // addresses are formed anew for each plane rather than held across the loop
        asm volatile("" : "+v"(t), "+v"(line));
        const int i1 = r1 / NY, j1 = r1 % NY;
        double2* base = reinterpret_cast<double2*>(a.psi) + (int64_t)r1 * (NX * NY);

        // X2 stage: column c = line + LINES q, element n1 at x2 = 8 n1 + t
        double2 v[16];
#pragma unroll
        for (int q = 0; q < QX; ++q)
#pragma unroll
            for (int n1 = 0; n1 < EX; ++n1)
                v[q * EX + n1] = ld<double2, NT>(base + (8 * n1 + t) * NY + line + LINES * q);
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            const int c = line + LINES * q;
            line_regs<NX>(
                &v[q * EX], t, L + c * plane_regs_stride(NX), twx,
                [&](int ii, double2* u) {
                    TableWalk kt(a.ktab, (t + 8 * ii) * NY + c);  // k-major: [k][y2]
                    batched<8, 4>([&](int) { return kt.next(EX * NY); },
                                  [&](int k, double2 f) { u[k] = cmul(u[k], f); });
                });
            // potential factor at (x2 = 8 n1 + t, y2 = c), without electron 1's one-body factor
            TableWalk one(a.a1, t * NY + c), two(a.ac, (i1 - t + NX - 1) * (2 * NY - 1) + (j1 - c + NY - 1));
            batched<EX, PB>(
                [&](int) {
                    VLoad l;
                    l.q = one.next(8 * NY);
                    l.r = two.next(-8 * (2 * NY - 1));
                    return l;
                },
                [&](int n1, const VLoad& l) { v[q * EX + n1] = cmul(v[q * EX + n1], cmul(l.q, l.r)); });
        }

        // columns to rows, one component at a time: row r = line + LINES q, element n1 at
        // y2 = 8 n1 + t.  The y kinetic factor takes electron 1's one-body factor, one number
        // for the plane, here, where no wavefront reads it (by every thread, some writing the same
        // value: behind a branch the compiler sinks the whole potential factor past it, spilling).
        double* Hw = L + t * plane_regs_row(NY) + line;
        double* Hr = L + line * plane_regs_row(NY) + t;
        auto at_w = [](int e) { return 8 * (e % EX) * plane_regs_row(NY) + LINES * (e / EX); };
        auto at_r = [](int e) { return LINES * (e / EY) * plane_regs_row(NY) + 8 * (e % EY); };
        double re[16];
        __syncthreads();
        ky[tid % NY] = cmul(a.ktab2[tid % NY], a.a1[r1]);
#pragma unroll
        for (int e = 0; e < 16; ++e) Hw[at_w(e)] = v[e].x;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) re[e] = Hr[at_r(e)];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) Hw[at_w(e)] = v[e].y;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = make_double2(re[e], Hr[at_r(e)]);
        __syncthreads();

        // Y2 stage
#pragma unroll
        for (int q = 0; q < QY; ++q) {
            const int r = line + LINES * q;
            line_regs<NY>(
                &v[q * EY], t, L + r * plane_regs_stride(NY), twy,
                [&](int ii, double2* u) {
                    batched<8, 4>([&](int k) { return ky[t + 8 * ii + EY * k]; },
                                  [&](int k, double2 f) { u[k] = cmul(u[k], f); });
                });
#pragma unroll
            for (int n1 = 0; n1 < EY; ++n1) st<double2, NT>(base + r * NY + 8 * n1 + t, v[q * EY + n1]);
        }
        // a wavefront's columns of the next plane take the places of its rows of this one on
        // square planes only
        if constexpr (NX != NY) __syncthreads();
    }
}

}  // namespace dev
}  // namespace hom4d_impl
