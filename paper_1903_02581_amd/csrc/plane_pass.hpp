// Fused pass over the contiguous (x2, y2) plane of one electron-1 position.
//
// For fixed r1 = (x1, y1) the nx*ny values Psi(r1, x2, y2) are contiguous in
// the [x1][y1][x2][y2] layout.  One workgroup owns one such plane and applies,
// in one HBM read and one HBM write,
//     X2(tau):  transform along x2, kinetic phase of (k_x2, y2), inverse,
//     V(dt/2):  exp(-i dt/2 (V(r1) + V(r2) + V12(r1 - r2)) / hbar),
//     Y2(dt):   transform along y2, kinetic phase of k_y2, inverse,
// i.e. three consecutive factors of the Strang step (arXiv 1903.02581,
// Sec. II.C Eq. (evoloperat); the x and y kinetic terms of Appendix A).  The
// plane stays in LDS between the stages, in the storage precision (Xchg); the
// arithmetic is FP64.  Each line transform is the same register/LDS four-step
// network as the per-axis pass.
#pragma once

#include "axis_pass.hpp"

namespace hom4d_impl {
namespace dev {

template <int N>
struct Shape;
template <> struct Shape<4> { static constexpr int n1 = 4, n2 = 1, t = 1; };
template <> struct Shape<6> { static constexpr int n1 = 6, n2 = 1, t = 1; };
template <> struct Shape<8> { static constexpr int n1 = 8, n2 = 1, t = 1; };
template <> struct Shape<12> { static constexpr int n1 = 12, n2 = 1, t = 1; };
template <> struct Shape<16> { static constexpr int n1 = 4, n2 = 4, t = 4; };
template <> struct Shape<24> { static constexpr int n1 = 12, n2 = 2, t = 2; };
template <> struct Shape<32> { static constexpr int n1 = 8, n2 = 4, t = 4; };
template <> struct Shape<48> { static constexpr int n1 = 12, n2 = 4, t = 4; };
template <> struct Shape<64> { static constexpr int n1 = 8, n2 = 8, t = 8; };
template <> struct Shape<96> { static constexpr int n1 = 12, n2 = 8, t = 4; };
template <> struct Shape<128> { static constexpr int n1 = 16, n2 = 8, t = 8; };

// LDS row layout of the plane: element p of row r at r * row + (p ^ ((p / 8) % 8)),
// row = NY + NY / 8.  The XOR permutes each aligned group of 8 slots, so the
// image stays in bounds.  For 16-byte accesses, 16 consecutive lanes must hit
// 16 different 16-byte bank groups: the x stage (lanes along a row, stride 1),
// the y stage's row reads (8 lanes along each of two rows) and its sub-row
// reads (stride 8 along two rows) all do at 64 x 64, where row = 72 puts the
// two rows of a lane group half a bank cycle apart.
// Rows of 12 (not whole groups of 8) are padded by one slot.
template <int NY>
struct PlaneLds {
    static constexpr int row = NY % 8 == 0 ? NY + NY / 8 : NY + 1;
    __device__ static __forceinline__ int at(int r, int p) {
        return r * row + (NY % 8 == 0 ? (p ^ ((p >> 3) & 7)) : p);
    }
};

// One plane per workgroup, grid = nx * ny.  Barriers: one after every LDS write
// that other wavefronts read back (the row exchanges of the Y2 stage stay
// inside one wavefront and only wait for its own writes); none before a write,
// because each exchange writes exactly the positions the same thread read in
// the previous one.
template <class S, int NX, int NY, int NT, int VK>
__global__ void __launch_bounds__(NT) k_plane2(const PassArgs a) {
    using SX_ = Shape<NX>;
    using SY_ = Shape<NY>;
    using LY = PlaneLds<NY>;
    constexpr int A1 = SX_::n1, A2 = SX_::n2, TX = SX_::t;
    constexpr int B1 = SY_::n1, B2 = SY_::n2, TY = SY_::t;
    constexpr int EX = NX / TX;
    constexpr int JAX = A2 / TX, IBX = A1 / TX;
    constexpr int JAY = B2 / TY, IBY = B1 / TY;
    constexpr int SLX = NY * TX, QX = (SLX + NT - 1) / NT;
    constexpr int SLY = NX * TY, QY = (SLY + NT - 1) / NT;
    using X = Xchg<S>;
    // Where the potential factor is applied: at the end of the X2 stage (FP64
    // storage) or as the Y2 stage reads its rows (complex64 storage, where the
    // smaller register footprint buys a resident wavefront per SIMD).
    constexpr bool V_IN_Y = !std::is_same<S, double2>::value;
    __shared__ typename X::T L[NX * LY::row];
    __shared__ double2 TW[NX + 2 * NY];  // x twiddles, y twiddles, y kinetic factor

    const int tid = threadIdx.x;
    const int r1 = blockIdx.x;
    const int i1 = r1 / NY, j1 = r1 % NY;
    // The one-body factor of electron 1 is one number for the whole plane, so it
    // is folded into the y kinetic factor here instead of multiplying each point.
    const double2 v1 = (VK == 1) ? a.a1[r1] : make_double2(1.0, 0.0);
    for (int i = tid; i < NX + 2 * NY; i += NT) {
        double2 v;
        if (i < NX) v = a.tw[i];
        else if (i < NX + NY) v = a.tw2[i - NX];
        else {
            v = a.ktab2[i - NX - NY];
            if constexpr (VK == 1) v = cmul(v, v1);
        }
        TW[i] = v;
    }

    // X2 stage slot of this thread: column c (= y2) and thread-in-line t
    auto slot_x = [&](int q, int* c, int* t) {
        const int s = tid + NT * q;
        *c = s % NY;
        *t = s / NY;
        return s < SLX;
    };

    S* base = reinterpret_cast<S*>(a.psi) + (int64_t)r1 * (NX * NY);
    double2 vx[QX][EX];
#pragma unroll
    for (int q = 0; q < QX; ++q) {
        int c, t;
        if (slot_x(q, &c, &t)) {
#pragma unroll
            for (int jj = 0; jj < JAX; ++jj)
#pragma unroll
                for (int n1 = 0; n1 < A1; ++n1) vx[q][jj * A1 + n1] = ld<S>(base + (n1 * A2 + t + TX * jj) * NY + c);
        }
    }
    __syncthreads();  // TW staged
    {
        const double2* twx = TW;
        const double2* twy = TW + NX;
        const double2* ky = TW + NX + NY;
        const double2* kx = a.ktab;
        const PassArgs& av = a;

        // ---------------- X2 stage A: DFT_A1 on the loaded columns, twiddles
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            int c, t;
            if (slot_x(q, &c, &t)) {
#pragma unroll
                for (int jj = 0; jj < JAX; ++jj) {
                    dft<A1, -1>(&vx[q][jj * A1]);
                    if constexpr (A2 > 1) {
                        const int jc = t + TX * jj;
#pragma unroll
                        for (int k1 = 1; k1 < A1; ++k1)
                            vx[q][jj * A1 + k1] = cmul(vx[q][jj * A1 + k1], twx[(jc * k1) % NX]);
                    }
                }
            }
        }
        double2 vb[QX][EX];  // stage-B / real-space values of the X2 stage
        if constexpr (A2 > 1) {
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                int c, t;
                if (slot_x(q, &c, &t)) {
#pragma unroll
                    for (int jj = 0; jj < JAX; ++jj)
#pragma unroll
                        for (int k1 = 0; k1 < A1; ++k1) L[LY::at(k1 * A2 + t + TX * jj, c)] = X::put(vx[q][jj * A1 + k1]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                int c, t;
                if (slot_x(q, &c, &t)) {
#pragma unroll
                    for (int ii = 0; ii < IBX; ++ii)
#pragma unroll
                        for (int j = 0; j < A2; ++j) vb[q][ii * A2 + j] = X::get(L[LY::at((t + TX * ii) * A2 + j, c)]);
#pragma unroll
                    for (int ii = 0; ii < IBX; ++ii) dft<A2, -1>(&vb[q][ii * A2]);
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < QX; ++q)
#pragma unroll
                for (int e = 0; e < EX; ++e) vb[q][e] = vx[q][e];
        }
        // kinetic x phase at (k_x2, y2), then the inverse transform
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            int c, t;
            if (slot_x(q, &c, &t)) {
                const double2* kt = kx + c;  // k-major table: [k][y2]
#pragma unroll
                for (int ii = 0; ii < IBX; ++ii)
#pragma unroll
                    for (int k2 = 0; k2 < A2; ++k2) {
                        double2 f = kt[(t + TX * ii + A1 * k2) * NY];
                        vb[q][ii * A2 + k2] = cmul(vb[q][ii * A2 + k2], f);
                    }
                if constexpr (A2 > 1) {
#pragma unroll
                    for (int ii = 0; ii < IBX; ++ii) dft<A2, 1>(&vb[q][ii * A2]);
                }
            }
        }
        if constexpr (A2 > 1) {
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                int c, t;
                if (slot_x(q, &c, &t)) {
#pragma unroll
                    for (int ii = 0; ii < IBX; ++ii)
#pragma unroll
                        for (int j = 0; j < A2; ++j) L[LY::at((t + TX * ii) * A2 + j, c)] = X::put(vb[q][ii * A2 + j]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                int c, t;
                if (slot_x(q, &c, &t)) {
#pragma unroll
                    for (int jj = 0; jj < JAX; ++jj)
#pragma unroll
                        for (int k1 = 0; k1 < A1; ++k1) vb[q][jj * A1 + k1] = X::get(L[LY::at(k1 * A2 + t + TX * jj, c)]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            int c, t;
            if (slot_x(q, &c, &t)) {
#pragma unroll
                for (int jj = 0; jj < JAX; ++jj) {
                    if constexpr (A2 > 1) {
                        const int jc = t + TX * jj;
#pragma unroll
                        for (int k1 = 1; k1 < A1; ++k1)
                            vb[q][jj * A1 + k1] = cmulc(vb[q][jj * A1 + k1], twx[(jc * k1) % NX]);
                    }
                    dft<A1, 1>(&vb[q][jj * A1]);
                }
                if constexpr (!V_IN_Y) {
                    // potential factor in real space at (x2 = n1 * A2 + t + TX * jj, y2 = c)
#pragma unroll
                    for (int jj = 0; jj < JAX; ++jj)
#pragma unroll
                        for (int n1 = 0; n1 < A1; ++n1) {
                            const double2 f = vfactor<VK == 1 ? 3 : VK, false>(av, i1, j1, n1 * A2 + t + TX * jj, c);
                            vb[q][jj * A1 + n1] = cmul(vb[q][jj * A1 + n1], f);
                        }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < QX; ++q) {
            int c, t;
            if (slot_x(q, &c, &t)) {
#pragma unroll
                for (int jj = 0; jj < JAX; ++jj)
#pragma unroll
                    for (int n1 = 0; n1 < A1; ++n1) L[LY::at(n1 * A2 + t + TX * jj, c)] = X::put(vb[q][jj * A1 + n1]);
            }
        }
        __syncthreads();

        // ---------------- Y2 stage: lines along y2, one per x2 (row of the plane)
        // When every row's TY threads sit in one wavefront and each wavefront owns
        // whole rows, the row exchanges stay inside the wavefront: it waits for its
        // own LDS writes before it reads (the memory clobber keeps the compiler
        // from moving or forwarding LDS accesses across the wait); no workgroup
        // barrier.  (The column exchanges of the X2 stage span wavefronts: a
        // column-per-wavefront thread mapping measured slower, 127 -> 150 us.)
        // Each sub-transform reads and writes back the same LDS slots, so the
        // stages take one sub-transform at a time and hold only its values in
        // registers.
        constexpr bool Y_WAVE = (QY == 1) && (64 % TY == 0);
        auto y_sync = [&]() {
            if constexpr (Y_WAVE)
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            else
                __syncthreads();
        };
        if constexpr (B2 > 1) {
            // stage A: DFT_B1 and twiddles, in place
#pragma unroll
            for (int q = 0; q < QY; ++q) {
                const int s = tid + NT * q;
                if (s < SLY) {
                    const int t = s % TY, row = s / TY;
#pragma unroll
                    for (int jj = 0; jj < JAY; ++jj) {
                        double2 u[B1];
#pragma unroll
                        for (int n1 = 0; n1 < B1; ++n1) u[n1] = X::get(L[LY::at(row, n1 * B2 + t + TY * jj)]);
                        if constexpr (V_IN_Y) {
                            // potential factor in real space at (x2 = row, y2)
#pragma unroll
                            for (int n1 = 0; n1 < B1; ++n1)
                                u[n1] = cmul(u[n1], vfactor<VK == 1 ? 3 : VK, false>(av, i1, j1, row, n1 * B2 + t + TY * jj));
                        }
                        dft<B1, -1>(u);
                        const int jc = t + TY * jj;
#pragma unroll
                        for (int k1 = 1; k1 < B1; ++k1) u[k1] = cmul(u[k1], twy[(jc * k1) % NY]);
#pragma unroll
                        for (int k1 = 0; k1 < B1; ++k1) L[LY::at(row, k1 * B2 + t + TY * jj)] = X::put(u[k1]);
                    }
                }
            }
            y_sync();
            // stage B: DFT_B2, kinetic y phase, inverse DFT_B2, in place
#pragma unroll
            for (int q = 0; q < QY; ++q) {
                const int s = tid + NT * q;
                if (s < SLY) {
                    const int t = s % TY, row = s / TY;
#pragma unroll
                    for (int ii = 0; ii < IBY; ++ii) {
                        double2 u[B2];
#pragma unroll
                        for (int j = 0; j < B2; ++j) u[j] = X::get(L[LY::at(row, (t + TY * ii) * B2 + j)]);
                        dft<B2, -1>(u);
#pragma unroll
                        for (int k2 = 0; k2 < B2; ++k2) u[k2] = cmul(u[k2], ky[t + TY * ii + B1 * k2]);
                        dft<B2, 1>(u);
#pragma unroll
                        for (int j = 0; j < B2; ++j) L[LY::at(row, (t + TY * ii) * B2 + j)] = X::put(u[j]);
                    }
                }
            }
            y_sync();
            // stage A inverse: conjugate twiddles, inverse DFT_B1, store
#pragma unroll
            for (int q = 0; q < QY; ++q) {
                const int s = tid + NT * q;
                if (s < SLY) {
                    const int t = s % TY, row = s / TY;
#pragma unroll
                    for (int jj = 0; jj < JAY; ++jj) {
                        double2 u[B1];
#pragma unroll
                        for (int k1 = 0; k1 < B1; ++k1) u[k1] = X::get(L[LY::at(row, k1 * B2 + t + TY * jj)]);
                        const int jc = t + TY * jj;
#pragma unroll
                        for (int k1 = 1; k1 < B1; ++k1) u[k1] = cmulc(u[k1], twy[(jc * k1) % NY]);
                        dft<B1, 1>(u);
#pragma unroll
                        for (int n1 = 0; n1 < B1; ++n1) st<S>(base + row * NY + n1 * B2 + t + TY * jj, u[n1]);
                    }
                }
            }
        } else {
            // a whole row per thread: DFT, kinetic y phase, inverse DFT
#pragma unroll
            for (int q = 0; q < QY; ++q) {
                const int s = tid + NT * q;
                if (s < SLY) {
                    const int row = s / TY;
                    double2 u[B1];
#pragma unroll
                    for (int n1 = 0; n1 < B1; ++n1) {
                        u[n1] = X::get(L[LY::at(row, n1)]);
                        if constexpr (V_IN_Y) u[n1] = cmul(u[n1], vfactor<VK == 1 ? 3 : VK, false>(av, i1, j1, row, n1));
                    }
                    dft<B1, -1>(u);
#pragma unroll
                    for (int k1 = 0; k1 < B1; ++k1) u[k1] = cmul(u[k1], ky[k1]);
                    dft<B1, 1>(u);
#pragma unroll
                    for (int n1 = 0; n1 < B1; ++n1) st<S>(base + row * NY + n1, u[n1]);
                }
            }
        }
    }
}

// Fused pass over the strided (x1, y1) plane of W consecutive electron-2 positions.
//
// For fixed r2 the values Psi(x1, y1, r2) lie nx*ny apart; a workgroup takes W
// consecutive r2 (runs of W elements) and applies, in one read and one write,
//     Y1(dt), V(dt/2), X1(tau):
// the three factors of the Strang step that follow the (x2, y2) plane pass, so that
// the two plane passes make a whole step.  The operations on a line are those of
// the per-axis passes in the same order: with complex128 storage the result is the same
// bit for bit.
//
// A line's threads are W apart on consecutive lanes with W T | 64, so every
// exchange of either stage stays inside one wavefront; the workgroup meets once, at the
// hand-off from the y lines to the x lines.  LDS holds the W planes in the storage
// type, position (x, y) of column w at (x NY + swizzle(x, y)) W + w: n2 = T for every
// length, so the XOR moves a stage-B access (stride n2 along the line) of the T threads, and
// the x lines' accesses (stride NY), onto T different bank groups.
template <int NX, int NY>
struct Plane1Lds {
    static constexpr int A2 = Shape<NX>::n2, B2 = Shape<NY>::n2;
    static_assert(Shape<NX>::t == A2 && Shape<NY>::t == B2, "a thread per column of the first factor");
    static_assert(NY % A2 == 0 && NY % B2 == 0, "the XORs stay inside a row");
    __device__ static __forceinline__ int at(int x, int y) {
        return x * NY + (y ^ ((y / B2) % B2) ^ (x % A2) ^ ((x / A2) % A2));
    }
};

constexpr int plane1_threads(int nx, int ny, int tx, int ty, int w) {
    const int s = (ny * tx > nx * ty ? ny * tx : nx * ty) * w;
    return ((s + 63) / 64) * 64;
}

// Columns per workgroup, and the grids whose step is two plane passes.  With four
// columns a wavefront's accesses are 64-byte (complex128) or 32-byte runs; measured
// per step against the three- or four-pass plan: 16x16 complex128 14.0 -> 8.9 us,
// 24x24 27.3 -> 21.2, 32x32 45.9 -> 34.5, 48x16 31.3 -> 23.4, 32x24 42.2 -> 25.4,
// complex64 33.1 -> 20.6 (launches and the latency of one short chain per kernel bound
// them; two columns 26.7 and eight 27.7 us at 32x24 complex128).  Past 1024 points a
// plane the runs cost more than the pass saved: 48x48 complex64 80.9 -> 83.7 us, 64x64
// complex128 (two columns, all that fit) 281 -> 304.
constexpr int kPlane1W = 4;
#define HOM4D_PAIR_SIZES                                                                                       \
    HOM4D_PLANE(8, 8) HOM4D_PLANE(8, 12) HOM4D_PLANE(8, 16) HOM4D_PLANE(8, 24) HOM4D_PLANE(8, 32)              \
    HOM4D_PLANE(8, 48) HOM4D_PLANE(8, 64)                                                                      \
    HOM4D_PLANE(12, 8) HOM4D_PLANE(12, 12) HOM4D_PLANE(12, 16) HOM4D_PLANE(12, 24) HOM4D_PLANE(12, 32)         \
    HOM4D_PLANE(12, 48) HOM4D_PLANE(12, 64)                                                                    \
    HOM4D_PLANE(16, 8) HOM4D_PLANE(16, 12) HOM4D_PLANE(16, 16) HOM4D_PLANE(16, 24) HOM4D_PLANE(16, 32)         \
    HOM4D_PLANE(16, 48) HOM4D_PLANE(16, 64)                                                                    \
    HOM4D_PLANE(24, 8) HOM4D_PLANE(24, 12) HOM4D_PLANE(24, 16) HOM4D_PLANE(24, 24) HOM4D_PLANE(24, 32)         \
    HOM4D_PLANE(32, 8) HOM4D_PLANE(32, 12) HOM4D_PLANE(32, 16) HOM4D_PLANE(32, 24) HOM4D_PLANE(32, 32)         \
    HOM4D_PLANE(48, 8) HOM4D_PLANE(48, 12) HOM4D_PLANE(48, 16) HOM4D_PLANE(64, 8) HOM4D_PLANE(64, 16)

template <class S, int NX, int NY, int W, int VK>
__global__ void __launch_bounds__(plane1_threads(NX, NY, Shape<NX>::t, Shape<NY>::t, W)) k_plane1(const PassArgs a) {
    using SX_ = Shape<NX>;
    using SY_ = Shape<NY>;
    using LY = Plane1Lds<NX, NY>;
    constexpr int NT = plane1_threads(NX, NY, SX_::t, SY_::t, W);
    constexpr int A1 = SX_::n1, A2 = SX_::n2, TX = SX_::t, B1 = SY_::n1, B2 = SY_::n2, TY = SY_::t;
    constexpr int EX = NX / TX, EY = NY / TY;
    static_assert(NT <= 1024 && 64 % (W * TX) == 0 && 64 % (W * TY) == 0, "lines inside a wavefront");
    using X = Xchg<S>;
    extern __shared__ double2 lds_raw[];
    typename X::T* L = reinterpret_cast<typename X::T*>(lds_raw);
    double2* TW = reinterpret_cast<double2*>(reinterpret_cast<char*>(lds_raw) + sizeof(typename X::T) * NX * NY * W);
    const double2* twx = TW;
    const double2* twy = TW + NX;
    const double2* ky = TW + NX + NY;

    const int tid = threadIdx.x, w = tid % W;
    constexpr int NXY = NX * NY;
    // Each of the 8 XCDs takes a run of neighbouring tiles: tiles narrower than a
    // 128-byte line then share it in that XCD's L2.
    const int ntiles = NXY / W, per = ntiles / 8;
    const int tile = (ntiles % 8 == 0) ? (blockIdx.x % 8) * per + blockIdx.x / 8 : blockIdx.x;
    const int r2 = tile * W + w, i2 = r2 / NY, j2 = r2 % NY;
    S* base = reinterpret_cast<S*>(a.psi) + r2;

    auto wave_sync = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    auto at = [&](int x, int y) { return LY::at(x, y) * W + w; };

    // ---------------- Y1 stage: line (x1, w), threads t along y1
    const int ty = (tid / W) % TY, x1 = tid / (W * TY);
    const bool on_y = x1 < NX;
    S raw[EY];
    if (on_y) {
#pragma unroll
        for (int e = 0; e < EY; ++e) raw[e] = ld_raw<S, false>(base + (int64_t)(x1 * NY + (e % B1) * B2 + ty + TY * (e / B1)) * NXY);
    }
    for (int i = tid; i < NX + 2 * NY; i += NT) TW[i] = i < NX ? a.tw[i] : i < NX + NY ? a.tw2[i - NX] : a.ktab2[i - NX - NY];
    __syncthreads();
    if (on_y) {
        double2 v[EY];
#pragma unroll
        for (int e = 0; e < EY; ++e) v[e] = widen(raw[e]);
        constexpr int JA = B2 / TY, IB = B1 / TY;
#pragma unroll
        for (int jj = 0; jj < JA; ++jj) {
            dft<B1, -1>(&v[jj * B1]);
            if constexpr (B2 > 1) {
                const int jc = ty + TY * jj;
#pragma unroll
                for (int k1 = 1; k1 < B1; ++k1) v[jj * B1 + k1] = cmul(v[jj * B1 + k1], twy[(jc * k1) % NY]);
#pragma unroll
                for (int k1 = 0; k1 < B1; ++k1) L[at(x1, k1 * B2 + jc)] = X::put(v[jj * B1 + k1]);
            }
        }
        if constexpr (B2 > 1) {
            wave_sync();
#pragma unroll
            for (int ii = 0; ii < IB; ++ii) {
#pragma unroll
                for (int j = 0; j < B2; ++j) v[ii * B2 + j] = X::get(L[at(x1, (ty + TY * ii) * B2 + j)]);
                dft<B2, -1>(&v[ii * B2]);
            }
        }
#pragma unroll
        for (int e = 0; e < EY; ++e) v[e] = cmul(v[e], ky[ty + TY * (e / B2) + B1 * (e % B2)]);
        if constexpr (B2 > 1) {
#pragma unroll
            for (int ii = 0; ii < IB; ++ii) {
                dft<B2, 1>(&v[ii * B2]);
#pragma unroll
                for (int j = 0; j < B2; ++j) L[at(x1, (ty + TY * ii) * B2 + j)] = X::put(v[ii * B2 + j]);
            }
            wave_sync();
#pragma unroll
            for (int jj = 0; jj < JA; ++jj)
#pragma unroll
                for (int k1 = 0; k1 < B1; ++k1) v[jj * B1 + k1] = X::get(L[at(x1, k1 * B2 + ty + TY * jj)]);
        }
#pragma unroll
        for (int jj = 0; jj < JA; ++jj) {
            if constexpr (B2 > 1) {
#pragma unroll
                for (int k1 = 1; k1 < B1; ++k1) v[jj * B1 + k1] = cmulc(v[jj * B1 + k1], twy[((ty + TY * jj) * k1) % NY]);
            }
            dft<B1, 1>(&v[jj * B1]);
        }
        // potential factor at (x1, y1 = (e % B1) B2 + t + TY (e / B1)), as the y1 line pass applies it
        if constexpr (VK == 1) {
            const double2 f2 = a.a1[r2];
            batched<EY, 4>(
                [&](int e) {
                    const int y = (e % B1) * B2 + ty + TY * (e / B1);
                    VLoad l;
                    l.p = a.a1[x1 * NY + y];
                    l.r = a.ac[(x1 - i2 + NX - 1) * (2 * NY - 1) + (y - j2 + NY - 1)];
                    return l;
                },
                [&](int e, const VLoad& l) { v[e] = cmul(v[e], cmul(cmul(l.p, f2), l.r)); });
        } else {
            batched<EY, 8>(
                [&](int e) { return vload<2>(a, x1, (e % B1) * B2 + ty + TY * (e / B1), i2, j2); },
                [&](int e, const VLoad& l) {
                    v[e] = cmul(v[e], vcombine<2, false>(a, l, x1, (e % B1) * B2 + ty + TY * (e / B1), i2, j2));
                });
        }
#pragma unroll
        for (int e = 0; e < EY; ++e) L[at(x1, (e % B1) * B2 + ty + TY * (e / B1))] = X::put(v[e]);
    }
    __syncthreads();

    // ---------------- X1 stage: line (y1, w), threads t along x1
    const int tx = (tid / W) % TX, y1 = tid / (W * TX);
    if (y1 < NY) {
        constexpr int JA = A2 / TX, IB = A1 / TX;
        double2 v[EX], kf[EX];
        const double2* kt = a.ktab + y1 * NX;  // y-major: the line's row of wave numbers
#pragma unroll
        for (int e = 0; e < EX; ++e) kf[e] = kt[tx + TX * (e / A2) + A1 * (e % A2)];
        // places of the thread's elements of stage A and of stage B
        auto at_a = [&](int e) { return at((e % A1) * A2 + tx + TX * (e / A1), y1); };
        auto at_b = [&](int e) { return at((tx + TX * (e / A2)) * A2 + e % A2, y1); };
        // Exchange of the line's elements, in FP64 for both storage types as in the x1 line
        // pass: complex64 moves the real parts, then the imaginary ones, through the line's own
        // 8-byte places, so that the LDS stays what the planes take.  (Complex64 elements
        // here round the state twice more a step: 32x24 over 20 steps 3.98e-7 off the
        // complex128 run against 3.62e-7 so and 3.60e-7 in four passes; 19.9 and 20.1 us a step.)
        auto exchange = [&](auto from, auto to) {
            if constexpr (std::is_same<S, double2>::value) {
#pragma unroll
                for (int e = 0; e < EX; ++e) L[from(e)] = v[e];
                wave_sync();
#pragma unroll
                for (int e = 0; e < EX; ++e) v[e] = L[to(e)];
            } else {
                double* D = reinterpret_cast<double*>(lds_raw);
                double re[EX];
                wave_sync();  // the places are read as complex64 before
#pragma unroll
                for (int e = 0; e < EX; ++e) D[from(e)] = v[e].x;
                wave_sync();
#pragma unroll
                for (int e = 0; e < EX; ++e) re[e] = D[to(e)];
                wave_sync();
#pragma unroll
                for (int e = 0; e < EX; ++e) D[from(e)] = v[e].y;
                wave_sync();
#pragma unroll
                for (int e = 0; e < EX; ++e) v[e] = make_double2(re[e], D[to(e)]);
            }
        };
#pragma unroll
        for (int jj = 0; jj < JA; ++jj) {
#pragma unroll
            for (int n1 = 0; n1 < A1; ++n1) v[jj * A1 + n1] = X::get(L[at_a(jj * A1 + n1)]);
            dft<A1, -1>(&v[jj * A1]);
            if constexpr (A2 > 1) {
#pragma unroll
                for (int k1 = 1; k1 < A1; ++k1) v[jj * A1 + k1] = cmul(v[jj * A1 + k1], twx[((tx + TX * jj) * k1) % NX]);
            }
        }
        if constexpr (A2 > 1) {
            exchange(at_a, at_b);
#pragma unroll
            for (int ii = 0; ii < IB; ++ii) dft<A2, -1>(&v[ii * A2]);
        }
#pragma unroll
        for (int e = 0; e < EX; ++e) v[e] = cmul(v[e], kf[e]);
        if constexpr (A2 > 1) {
#pragma unroll
            for (int ii = 0; ii < IB; ++ii) dft<A2, 1>(&v[ii * A2]);
            exchange(at_b, at_a);
        }
#pragma unroll
        for (int jj = 0; jj < JA; ++jj) {
            const int jc = tx + TX * jj;
            if constexpr (A2 > 1) {
#pragma unroll
                for (int k1 = 1; k1 < A1; ++k1) v[jj * A1 + k1] = cmulc(v[jj * A1 + k1], twx[(jc * k1) % NX]);
            }
            dft<A1, 1>(&v[jj * A1]);
#pragma unroll
            for (int n1 = 0; n1 < A1; ++n1) st<S>(base + (int64_t)((n1 * A2 + jc) * NY + y1) * NXY, v[jj * A1 + n1]);
        }
    }
}

// Threads per plane workgroup: enough for the larger of the two stages, at most 1024.
constexpr int plane_threads(int nx, int ny, int tx, int ty) {
    const int s = (ny * tx > nx * ty) ? ny * tx : nx * ty;
    const int r = ((s + 63) / 64) * 64;
    return r > 1024 ? 1024 : r;
}

}  // namespace dev
}  // namespace hom4d_impl

