// Per-axis pass for the long lines (n = 96, 128, 256) of the forward step:
// the same transform -> kinetic phase -> inverse round trip as k_axis
// (Sec. II.C Eq. (evoloperat); kinetic terms of Appendix A), with the line
// transform factored into three radix stages instead of two, so that every
// thread holds 8 (or 12) elements instead of 16 (or 24) and the kernels keep
// enough waves resident to stream HBM.  n = 256 takes 32 threads per line, so
// its blocks hold 16 lines in 512 threads (128-byte runs on the strided axes
// in complex64 storage), or 32 lines in 1024 threads on the complex64 x1
// pass.
//
// Line of n = R1 R2 R3 points, element m = n1 (R2 R3) + n2 R3 + j3, handled by T
// threads.  Forward:
//   stage A   DFT_R1 over n1 for each column jc = n2 R3 + j3, twiddle w_n^(jc k1);
//   stage B1  DFT_R2 over n2 for each (k1, j3), twiddle w_(R2 R3)^(j3 k2);
//   stage B2  DFT_R3 over j3 for each (k1, k2);
// giving wave number k = k1 + R1 (k2 + R2 k3).  The kinetic phase is applied
// there, and the transposed network (conjugate twiddles, inverse DFTs in the
// reverse order) brings every thread back to the elements it loaded.  Between
// stages the line is exchanged through LDS, each stage reading and writing its
// own disjoint set of positions.
//
// PERS (the forward complex64 x1 pass of 128- and 256-point lines): the kernel is
// persistent: a block walks tiles of W lines (tile = blockIdx.x, + gridDim.x, ...) and
// issues the loads of its next tile while it transforms the current one (in four parts,
// from its start and between its exchanges), so that the HBM reads of
// one tile overlap the arithmetic and LDS exchanges of the previous one inside the block,
// instead of relying on other resident blocks being out of phase.  Its exchanges
// synchronise the block on LDS alone (lds_barrier), leaving the prefetch loads and the
// stores in flight.  It pays where a pass has few resident blocks per CU: the 256-point x1
// pass, one 1024-thread block per CU, 5.87 ms without and 4.45 ms with it at 256x128; 128x64
// x1 237 and 228 us.  The y1 passes, and the reverse x1 pass with its two states, have
// enough wavefronts once they hold no addresses over the transform (axis_reads_apart):
// 256x128 y1 3.64 ms persistent, 3.25 so, 48x256 y1 590 and 530 us, reverse x1 12.1 and
// 11.0 ms at 256x128.  FP64 and n = 96 lines ran slower persistent as well (128x128 FP64 x1
// 1.62 -> 1.79 ms).  No global load is waited for inside a tile's transform (the kinetic
// factors come from LDS), and the first tile is peeled off the loop, so that the only wait
// for the prefetch, at the start of the next tile, leaves the stores in flight.
//
// The arithmetic is FP64 for both storage types.  With complex64 storage the
// exchange area holds complex64 too: each exchange then rounds like one more
// store of the state (random, not coherent, since the state changes every
// step), and the area takes half the LDS, so twice as many blocks fit a CU.
#pragma once

#include "axis_pass.hpp"

namespace hom4d_impl {
namespace dev {

template <int R1, int R2, int R3, int T>
struct Net3 {
    static constexpr int N = R1 * R2 * R3, N2 = R2 * R3;
    static constexpr int JA = N2 / T;        // stage-A columns per thread
    static constexpr int G1 = R1 * R3 / T;   // stage-B1 groups per thread
    static constexpr int G2 = R1 * R2 / T;   // stage-B2 groups per thread
    static constexpr int E = JA * R1;        // elements per thread
    static_assert(N2 % T == 0 && (R1 * R3) % T == 0 && (R1 * R2) % T == 0, "T must split every stage");
    static_assert(G1 * R2 == E && G2 * R3 == E, "every stage must give a thread E elements");
};

// Block-wide synchronisation on LDS only: wait for this wave's LDS accesses,
// then the barrier.  Global loads and stores stay in flight (a fence-carrying
// __syncthreads would wait for them); the memory clobber keeps the compiler
// from moving LDS accesses across it.  Exchanges along y2 with T | 64 stay
// wave-local as in line_sync.
template <int AXIS, int T>
__device__ __forceinline__ void lds_barrier() {
    if constexpr (AXIS == AX_Y2 && 64 % T == 0)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    else
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Elements per batch of the table-form potential loads: 2 on the complex64 y2
// pass of 128- and 256-point lines (90 instead of 116 VGPRs, five waves per
// SIMD instead of four: 256x128 y2+V 4.66 -> 4.48 ms), 4 elsewhere (the
// complex64 x2 pass measured slower with 2: 5.21 -> 5.36 ms, 128x96 0.674 ->
// 0.717 ms).
constexpr int potential_batch(int axis, int n, bool c64) { return (c64 && axis == AX_Y2 && n >= 128) ? 2 : 4; }

// Least wavefronts per SIMD the compiler plans for (0: its own choice): the complex64 reverse
// y1 pass of 128- and 256-point lines is 2 registers past 128, which its LDS would let four
// wavefronts use (64x128 y1 545 -> 510 us, for 5-10 spills).
constexpr int axis3_min_waves(int axis, int n, int nst, bool c64) {
    return c64 && nst == 2 && axis == AX_Y1 && n >= 128 ? 4 : 0;
}

// WC > 0: the block holds WC lines, a compile-time constant (the nominal width
// of the pass, axis3_nominal_w), so every LDS address is a per-thread base plus
// an immediate offset; WC = 0: a.W lines, for grids that allow fewer (never the persistent
// pass: its ny nx ny lines and nx ny are whole blocks of 32, nx being 128 or 256).
template <class S, int AXIS, int R1, int R2, int R3, int T, int NST, int VK, bool NT, bool PERS, int WC>
__global__ void __launch_bounds__(axis3_block_threads(AXIS, R1 * R2 * R3, NST, !std::is_same<S, double2>::value),
                                  axis3_min_waves(AXIS, R1 * R2 * R3, NST, !std::is_same<S, double2>::value)) k_axis3(const PassArgs a) {
    static_assert(!PERS || (NST == 1 && AXIS == AX_X1 && VK == 0 && WC > 0), "persistent: the forward x1 pass");
    // the reverse sweep (two states) applies every factor conjugated
    constexpr bool CONJ = NST == 2;
    constexpr bool SRC = axis_reads_apart(AXIS, R1 * R2 * R3, NST, VK, 0), LSRC = axis_reads_apart(AXIS, R1 * R2 * R3, NST, VK, 1);
    using NW = Net3<R1, R2, R3, T>;
    constexpr int N = NW::N, N2 = NW::N2, JA = NW::JA, G1 = NW::G1, G2 = NW::G2, E = NW::E;
    using X = Xchg<S>;
    extern __shared__ double2 lds_raw[];

    const int W = WC > 0 ? WC : a.W;
    const int tid = threadIdx.x;
    int t, cl;
    if constexpr (AXIS == AX_Y2) {
        t = tid % T;
        cl = tid / T;
    } else {
        cl = tid % W;
        t = tid / W;
    }

    // twiddles w_n^j (and, on y axes, the kinetic factor) staged after the exchange area
    constexpr bool KT_LDS = (AXIS == AX_Y1 || AXIS == AX_Y2);
    // persistent: the tile's kinetic row (its lines share y1) comes from
    // one of two LDS rows after the twiddles, written at the start of the tile
    // from a register loaded with the previous tile's prefetch, so that no
    // global load is issued inside the transform (a wait for one would also wait
    // for the next tile's loads and the previous tile's stores, issued earlier)
    constexpr bool KROW = PERS;
    const double2* krow = nullptr;
    const int LS = W + 1;  // padded LDS row: one line position across the block's W lines
    typename X::T* lds = reinterpret_cast<typename X::T*>(lds_raw);
    double2* twl = reinterpret_cast<double2*>(reinterpret_cast<char*>(lds_raw) +
                                              axis3_xchg_bytes(N, W, NST, sizeof(typename X::T) == 8));
    for (int i = tid; i < (KT_LDS ? 2 * N : N); i += T * W) {
        double2 w;
        if (i < N) {
            w = a.tw[i];
        } else {
            w = a.ktab[i - N];
            if constexpr (CONJ) w = conjd(w);
        }
        twl[i] = w;
    }
    __syncthreads();
    // state s, line position pos: s * N + pos rows of W + 1 slots
    auto Lw = [&](int st_, int pos, double2 v) { lds[(st_ * N + pos) * LS + cl] = X::put(v); };
    auto Lr = [&](int st_, int pos) -> double2 { return X::get(lds[(st_ * N + pos) * LS + cl]); };
    // the exchanges: LDS-only barriers in the persistent passes
    auto sync = [&]() {
        if constexpr (PERS)
            lds_barrier<AXIS, T>();
        else
            line_sync<AXIS, T>();
    };
    // element jj * R1 + n1 of a thread: line position n1 N2 + t + T jj
    // visit the thread's elements e = jj R1 + n1 of a line (line position
    // n1 N2 + t + T jj) with their addresses, stepping from one to the next by a
    // 64-bit add rather than forming each offset by multiplication
    auto walk = [&](const LineGeom<AXIS>& lg, auto* base, auto&& fn) {
        const int64_t step = (int64_t)N2 * lg.sN;
#pragma unroll
        for (int jj = 0; jj < JA; ++jj) {
            auto* p = base + (int64_t)(t + T * jj) * lg.sN;
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) {
                fn(jj * R1 + n1, p);
                p += step;
            }
        }
    };

    // elements e0 .. e1 - 1 of the walk above, each address formed directly
    auto walk_part = [&](const LineGeom<AXIS>& lg, auto* base, int e0, int e1, auto&& fn) {
#pragma unroll
        for (int e = e0; e < e1; ++e) {
            const int jj = e / R1, n1 = e % R1;
            fn(e, base + ((int64_t)(t + T * jj) + (int64_t)n1 * N2) * lg.sN);
        }
    };

    // Transform round trip of the block's tile held in v (loaded elements in,
    // the same elements out, stored in place), with the potential factor and
    // the reverse sweep's gradient terms.  between(k) runs after the k-th of the
    // four exchanges (k = 0..3).
    double2 v[NST][E];
    auto round_trip = [&](const LineGeom<AXIS>& lg, uint32_t line, uint32_t blk, S* const* ps, auto&& between) {
        // gradient accumulators of the reverse sweep: the potential marginal
        // Im(conj(lambda) psi) on the side of the potential factor the pass is told
        // to take it (before: G_MIN, after: G_MOUT), and the dL/dB term of the x
        // kinetic factor in reciprocal space
        double gm_acc = 0.0, gb_acc = 0.0;
        if constexpr (NST == 2) {
            if (a.gflags & G_MIN) {
#pragma unroll
                for (int e = 0; e < E; ++e) gm_acc += im_cl_p(v[1][e], v[0][e]);
            }
        }
        // the potential factor on the thread's elements (element e = jj R1 + n1 at
        // line position n1 N2 + t + T jj), its table entries loaded in batches
        auto potential = [&]() {
            if constexpr (VK == 1) {
                const LineTables<AXIS> tb(a, lg, t);
                const double2 f0 = tb.fixed();
                batched<E, potential_batch(AXIS, N, !std::is_same<S, double2>::value)>([&](int e) { return tb.load((e % R1) * N2 + T * (e / R1)); },
                              [&](int e, const VLoad& l) {
                                  const double2 f = tb.template combine<CONJ>(f0, l);
#pragma unroll
                                  for (int s = 0; s < NST; ++s) v[s][e] = cmul(v[s][e], f);
                              });
            } else {
                constexpr int VKF = VK == 0 ? 1 : VK;
                auto coords = [&](int e, int* c) {
                    elem_coord<AXIS>(lg.i1, lg.j1, lg.i2, lg.j2, (e % R1) * N2 + t + T * (e / R1), c);
                };
                batched<E, vbatch<VKF>()>(
                    [&](int e) {
                        int c[4];
                        coords(e, c);
                        return vload<VKF>(a, c[0], c[1], c[2], c[3]);
                    },
                    [&](int e, const VLoad& l) {
                        int c[4];
                        coords(e, c);
                        const double2 f = vcombine<VKF, CONJ>(a, l, c[0], c[1], c[2], c[3]);
#pragma unroll
                        for (int s = 0; s < NST; ++s) v[s][e] = cmul(v[s][e], f);
                    });
            }
        };
        if (VK != 0 && a.vmode == 1) potential();

        // ---- stage A (forward)
#pragma unroll
        for (int s = 0; s < NST; ++s)
#pragma unroll
            for (int jj = 0; jj < JA; ++jj) {
                const int jc = t + T * jj;
                dft<R1, -1>(&v[s][jj * R1]);
#pragma unroll
                for (int k1 = 1; k1 < R1; ++k1) v[s][jj * R1 + k1] = cmul(v[s][jj * R1 + k1], twl[(uint32_t)(jc * k1) % N]);
#pragma unroll
                for (int k1 = 0; k1 < R1; ++k1) Lw(s, k1 * N2 + jc, v[s][jj * R1 + k1]);
            }
        sync();
        between(0);

        // ---- stage B1 (forward), in place on its positions
#pragma unroll
        for (int s = 0; s < NST; ++s)
#pragma unroll
            for (int ii = 0; ii < G1; ++ii) {
                const int q = t + T * ii, k1 = q / R3, j3 = q % R3;
#pragma unroll
                for (int n2 = 0; n2 < R2; ++n2) v[s][ii * R2 + n2] = Lr(s, k1 * N2 + n2 * R3 + j3);
                dft<R2, -1>(&v[s][ii * R2]);
#pragma unroll
                for (int k2 = 1; k2 < R2; ++k2) v[s][ii * R2 + k2] = cmul(v[s][ii * R2 + k2], twl[(uint32_t)(R1 * j3 * k2) % N]);
#pragma unroll
                for (int k2 = 0; k2 < R2; ++k2) Lw(s, k1 * N2 + k2 * R3 + j3, v[s][ii * R2 + k2]);
            }
        sync();
        between(1);

        // ---- stage B2: forward, kinetic phase at k = k1 + R1 (k2 + R2 k3), inverse
        // x kinetic factor table: y-major [y][k] on the x1 pass, k-major [k][y] on the x2 pass
        const int yrow = (AXIS == AX_X1) ? lg.j1 : ((AXIS == AX_X2) ? lg.j2 : 0);
        const double2* kt = a.ktab + (AXIS == AX_X1 ? (int64_t)yrow * N : (int64_t)yrow);
        const int64_t kstride = AXIS == AX_X1 ? 1 : a.ny;
        constexpr bool GB = (NST == 2) && (AXIS == AX_X1 || AXIS == AX_X2);
        const bool gb_on = GB && (a.gflags & G_GB);
        const double yv = a.y0 + a.ystep * yrow;
        const double shift = yv * a.b_eoh;
#pragma unroll
        for (int ii = 0; ii < G2; ++ii) {
            const int q = t + T * ii, k1 = q / R2, k2 = q % R2;
            // x axes: the group's kinetic factors come from the L2-resident table;
            // their loads are issued ahead of the LDS reads and the DFT, which hide them
            double2 kf[R3];
            if constexpr (!KT_LDS) {
#pragma unroll
                for (int k3 = 0; k3 < R3; ++k3)
                    kf[k3] = KROW ? krow[k1 + R1 * (k2 + R2 * k3)] : kt[(k1 + R1 * (k2 + R2 * k3)) * kstride];
                if constexpr (!KROW) after_loads();
            }
#pragma unroll
            for (int s = 0; s < NST; ++s) {
#pragma unroll
                for (int j3 = 0; j3 < R3; ++j3) v[s][ii * R3 + j3] = Lr(s, k1 * N2 + k2 * R3 + j3);
                dft<R3, -1>(&v[s][ii * R3]);
            }
#pragma unroll
            for (int k3 = 0; k3 < R3; ++k3) {
                const int k = k1 + R1 * (k2 + R2 * k3);
                if constexpr (GB) {
                    if (gb_on) {
                        // d theta_X / dB at (k, y), on the values before the kinetic factor
                        const int m = (k < (N + 1) / 2) ? k : k - N;
                        const double dth = a.db_coef * (a.kstep * m - shift) * yv;
                        gb_acc += dth * im_cl_p(v[1][ii * R3 + k3], v[0][ii * R3 + k3]);
                    }
                }
                double2 f;
                if constexpr (KT_LDS) {
                    f = twl[N + k];
                } else {
                    f = kf[k3];
                    if constexpr (CONJ) f = conjd(f);
                }
#pragma unroll
                for (int s = 0; s < NST; ++s) v[s][ii * R3 + k3] = cmul(v[s][ii * R3 + k3], f);
            }
#pragma unroll
            for (int s = 0; s < NST; ++s) {
                dft<R3, 1>(&v[s][ii * R3]);
#pragma unroll
                for (int j3 = 0; j3 < R3; ++j3) Lw(s, k1 * N2 + k2 * R3 + j3, v[s][ii * R3 + j3]);
            }
        }
        sync();
        between(2);

        // ---- stage B1 (inverse)
#pragma unroll
        for (int s = 0; s < NST; ++s)
#pragma unroll
            for (int ii = 0; ii < G1; ++ii) {
                const int q = t + T * ii, k1 = q / R3, j3 = q % R3;
#pragma unroll
                for (int k2 = 0; k2 < R2; ++k2) v[s][ii * R2 + k2] = Lr(s, k1 * N2 + k2 * R3 + j3);
#pragma unroll
                for (int k2 = 1; k2 < R2; ++k2) v[s][ii * R2 + k2] = cmulc(v[s][ii * R2 + k2], twl[(uint32_t)(R1 * j3 * k2) % N]);
                dft<R2, 1>(&v[s][ii * R2]);
#pragma unroll
                for (int n2 = 0; n2 < R2; ++n2) Lw(s, k1 * N2 + n2 * R3 + j3, v[s][ii * R2 + n2]);
            }
        sync();
        between(3);

        // ---- stage A (inverse), back on the loaded elements
#pragma unroll
        for (int s = 0; s < NST; ++s)
#pragma unroll
            for (int jj = 0; jj < JA; ++jj) {
                const int jc = t + T * jj;
#pragma unroll
                for (int k1 = 0; k1 < R1; ++k1) v[s][jj * R1 + k1] = Lr(s, k1 * N2 + jc);
#pragma unroll
                for (int k1 = 1; k1 < R1; ++k1) v[s][jj * R1 + k1] = cmulc(v[s][jj * R1 + k1], twl[(uint32_t)(jc * k1) % N]);
                dft<R1, 1>(&v[s][jj * R1]);
            }

        if (VK != 0 && a.vmode == 2) potential();

        if constexpr (NST == 2) {
            if (a.gflags & G_MOUT) {
#pragma unroll
                for (int e = 0; e < E; ++e) gm_acc += im_cl_p(v[1][e], v[0][e]);
            }
        }

#pragma unroll
        for (int s = 0; s < NST; ++s) walk(lg, ps[s], [&](int e, S* p) { st<S, NT>(p, v[s][e]); });

        if constexpr (NST == 2) {
            // the same partial-sum layout as the two-stage pass: dL/dB per block; the
            // marginal per line on the x1 and y1 axes (the line's threads summed in
            // fixed order), per block on x2 and y2 (a block's lines share r1)
            double* red = reinterpret_cast<double*>(lds_raw);
            if (a.gflags & G_GB) {
                const double sum = block_sum(gb_acc, red);
                if (tid == 0) a.gb_part[blk] += sum;
            }
            if (a.gflags & (G_MIN | G_MOUT)) {
                if constexpr (AXIS == AX_X1 || AXIS == AX_Y1) {
                    __syncthreads();
                    red[t * W + cl] = gm_acc;
                    __syncthreads();
                    if (t == 0) {
                        double sum = 0.0;
                        for (int q = 0; q < T; ++q) sum += red[q * W + cl];
                        a.marg_part[line] += sum;
                    }
                } else {
                    const double sum = block_sum(gm_acc, red);
                    if (tid == 0) a.marg_part[blk] += sum;
                }
            }
        }
    };

    if constexpr (PERS) {
        // persistent: tiles blockIdx.x, + gridDim.x, ...; the next tile's
        // elements are loaded (as stored) before the current one is transformed
        const uint32_t ntiles = a.ntiles;
        S raw[E];
        S* const state = reinterpret_cast<S*>(a.psi);
        const S* const from = SRC ? reinterpret_cast<const S*>(a.src) : state;  // where the state is read
        double2 kreg = make_double2(0.0, 0.0);  // entry tid of the next tile's kinetic row
        // the kinetic row of tile tl: y1 of its lines (a tile's lines share y1)
        auto krow_of = [&](uint32_t tl) { return a.ktab + (int64_t)a.dnxy.div(tl * (uint32_t)W) * N; };
        uint32_t tile = blockIdx.x;
        if (tile < ntiles) {
            const LineGeom<AXIS> lg(a, tile * (uint32_t)W + (uint32_t)cl);
            walk(lg, from + lg.base, [&](int e, const S* p) { raw[e] = ld_raw<S, NT>(p); });
            if (tid < N) kreg = krow_of(tile)[tid];
        }
        uint32_t it = 0;  // the block's tile count: parity selects the kinetic row
        // The thread's tile-invariant addresses stay in registers (1024-thread blocks, one per CU
        // whatever their registers up to 128, at 256 points; 32-line 512-thread blocks, two per
        // CU at up to 128 registers, at 128), and the next tile's loads are issued in parts while
        // the current tile is transformed, instead of all at its start.  256x128 x1: hoisting
        // 5.25 -> 5.12 ms (about 8 fewer VALU instructions per point), spreading 5.10 -> 4.41 ms,
        // with fewer registers held over the tile; the 128-point pass, hoisted and spread:
        // 128x96 0.559 -> 0.526 ms, 128x64 0.279 -> 0.234 ms.
        auto one_tile = [&](uint32_t tl) {
            const uint32_t line = tl * (uint32_t)W + (uint32_t)cl;
            const LineGeom<AXIS> lg(a, line);
            S* const ps[1] = {state + lg.base};
#pragma unroll
            for (int e = 0; e < E; ++e) v[0][e] = widen(raw[e]);
            // visible to every thread after the first exchange barrier; the row
            // written two tiles ago was last read before this tile's barriers
            double2* row = twl + N * (1 + (it & 1));
            if (tid < N) row[tid] = kreg;
            krow = row;
            const uint32_t next = tl + gridDim.x;
            const bool has_next = next < ntiles;
            const LineGeom<AXIS> ln(a, (has_next ? next : tl) * (uint32_t)W + (uint32_t)cl);
            const S* nbase = from + ln.base;
            if (has_next && tid < N) kreg = krow_of(next)[tid];
            // NP parts of the E elements, part j issued at slot j - 1 (slot -1: before the first
            // stage, slot k >= 0: after exchange k), the fastest of the schedules measured
            // (after the four exchanges 4.56-4.65 ms at 256x128, three or two parts from the
            // start 4.62 and 4.76 ms)
            constexpr int NP = 4;
            constexpr int PART = (E + NP - 1) / NP;
            auto part = [&](int slot) {
                const int j = slot + 1;
                if (has_next && j >= 0 && j < NP)
                    walk_part(ln, nbase, j * PART, (j + 1) * PART < E ? (j + 1) * PART : E,
                              [&](int e, const S* p) { raw[e] = ld_raw<S, NT>(p); });
            };
            part(-1);
            round_trip(lg, line, tl, ps, part);
            ++it;
        };
        // The first tile is peeled off the loop, so that the loop is entered, like
        // its back edge, with the next tile's loads followed by this tile's stores
        // outstanding: the wait for those loads (the memory counter covers loads
        // and stores in issue order) then leaves the stores in flight, where a
        // loop entered with the loads alone outstanding waits for everything.
        if (tile < ntiles) {
            one_tile(tile);
            for (tile += gridDim.x; tile < ntiles; tile += gridDim.x) one_tile(tile);
        }
    } else {
        const uint32_t line = blockIdx.x * (uint32_t)W + (uint32_t)cl;
        const LineGeom<AXIS> lg(a, line);
        // the state, and in the reverse sweep the adjoint state beside it
        S* ps[NST];
        ps[0] = reinterpret_cast<S*>(a.psi) + lg.base;
        if constexpr (NST == 2) ps[1] = reinterpret_cast<S*>(a.lam) + lg.base;
        const S* from[NST];  // where the states are read
        from[0] = SRC ? reinterpret_cast<const S*>(a.src) + lg.base : ps[0];
        if constexpr (NST == 2) from[1] = LSRC ? reinterpret_cast<const S*>(a.lam_src) + lg.base : ps[1];
        S raw[NST][E];
#pragma unroll
        for (int s = 0; s < NST; ++s) walk(lg, from[s], [&](int e, const S* p) { raw[s][e] = ld_raw<S, NT>(p); });
        after_loads();
#pragma unroll
        for (int s = 0; s < NST; ++s)
#pragma unroll
            for (int e = 0; e < E; ++e) v[s][e] = widen(raw[s][e]);
        round_trip(lg, line, blockIdx.x, ps, [](int) {});
    }
}

// Three-stage factorisations: n = R1 R2 R3 on T threads per line.
// The compile-time-width form when the block takes the pass's nominal width w.
template <class S, int AXIS, int R1, int R2, int R3, int T, int NST, int VK, bool NT, bool PERS>
AxisKernel pick_w(int w) {
    constexpr int WN = axis3_nominal_w(AXIS, R1 * R2 * R3, T, NST, !std::is_same<S, double2>::value);
    if (w == WN) return k_axis3<S, AXIS, R1, R2, R3, T, NST, VK, NT, PERS, WN>;
    if constexpr (PERS)
        return nullptr;
    else
        return k_axis3<S, AXIS, R1, R2, R3, T, NST, VK, NT, PERS, 0>;
}

template <class S, int AXIS, int NST, int VK, bool NT, bool PERS = false>
AxisKernel pick3(int n, int w, int* t) {
    switch (n) {
        case 96:
            if constexpr (!PERS) {
                *t = 8;
                return pick_w<S, AXIS, 12, 4, 2, 8, NST, VK, NT, PERS>(w);
            }
            break;
        case 128: *t = 16; return pick_w<S, AXIS, 8, 4, 4, 16, NST, VK, NT, PERS>(w);
        case 256: *t = 32; return pick_w<S, AXIS, 8, 8, 4, 32, NST, VK, NT, PERS>(w);
        default: break;
    }
    *t = 0;
    return nullptr;
}

// Forward single-state passes: the x1 pass carries no potential factor, the
// y2 pass always carries it, x2 and y1 either.  Reverse dual-state passes: the
// x passes carry none, y1 (before its transform) and y2 (after) carry it.
// Persistent form: the complex64 x1 pass of 128- and 256-point lines.
template <class S, bool NT>
AxisKernel pick_axis3_nt(int axis, int n, int vk, int nst, bool pers, int w, int* t) {
    if (pers) {
        if constexpr (!std::is_same<S, double2>::value)
            if (nst == 1 && vk == 0 && axis == AX_X1) return pick3<S, AX_X1, 1, 0, NT, true>(n, w, t);
        *t = 0;
        return nullptr;
    }
    if (nst == 2) {
        switch (axis) {
            case AX_X1:
                if (vk == 0) return pick3<S, AX_X1, 2, 0, NT>(n, w, t);
                break;
            case AX_X2:
                if (vk == 0) return pick3<S, AX_X2, 2, 0, NT>(n, w, t);
                break;
            case AX_Y1:
                if (vk == 1) return pick3<S, AX_Y1, 2, 1, NT>(n, w, t);
                if (vk == 2) return pick3<S, AX_Y1, 2, 2, NT>(n, w, t);
                break;
            case AX_Y2:
                if (vk == 1) return pick3<S, AX_Y2, 2, 1, NT>(n, w, t);
                if (vk == 2) return pick3<S, AX_Y2, 2, 2, NT>(n, w, t);
                break;
            default: break;
        }
        *t = 0;
        return nullptr;
    }
    switch (axis) {
        case AX_X1:
            if (vk == 0) return pick3<S, AX_X1, 1, 0, NT>(n, w, t);
            break;
        case AX_X2:
            if (vk == 0) return pick3<S, AX_X2, 1, 0, NT>(n, w, t);
            if (vk == 1) return pick3<S, AX_X2, 1, 1, NT>(n, w, t);
            if (vk == 2) return pick3<S, AX_X2, 1, 2, NT>(n, w, t);
            break;
        case AX_Y1:
            if (vk == 0) return pick3<S, AX_Y1, 1, 0, NT>(n, w, t);
            if (vk == 1) return pick3<S, AX_Y1, 1, 1, NT>(n, w, t);
            if (vk == 2) return pick3<S, AX_Y1, 1, 2, NT>(n, w, t);
            break;
        case AX_Y2:
            if (vk == 1) return pick3<S, AX_Y2, 1, 1, NT>(n, w, t);
            if (vk == 2) return pick3<S, AX_Y2, 1, 2, NT>(n, w, t);
            break;
        default: break;
    }
    *t = 0;
    return nullptr;
}

template <class S>
AxisKernel pick_axis3(int axis, int n, int vk, int nst, bool nt, bool pers, int w, int* t) {
    return nt ? pick_axis3_nt<S, true>(axis, n, vk, nst, pers, w, t) : pick_axis3_nt<S, false>(axis, n, vk, nst, pers, w, t);
}

}  // namespace dev
}  // namespace hom4d_impl
