// The residual sweep P1 (see poisson_sweeps.hip): residual, weight, partial norms
// per tile, Hartley (or, between walls, cosine) transform along x.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "poisson_control.hpp"
#include "poisson_device.hpp"
#include "poisson_launch.hpp"
#include "poisson_rows.hpp"

namespace pois {

// The start of an evaluation: whether this launch of P1 has nothing to evaluate
// for the solve.  The phase of an FP32 step that was predicted to end after the
// update before it is closed here, by the last block (when every block has read
// the state that sent it here).
template <typename T>
__device__ __forceinline__ bool p1_idle(const Slot& s, int decide) {
    if (IterView<T>::skip_p1(s.st)) return true;
    if constexpr (sizeof(T) == 4) {
        if (s.st->stop_next != 0) {
            if (decide && last_block(s) && threadIdx.x == 0) close_inner(s.st);
            return true;
        }
    }
    return false;
}

// Sums of a unit: r^2, bt^2, and in FP64 p and p^2.
template <typename T>
constexpr int kSums = sizeof(T) == 8 ? 4 : 2;

// The end of an evaluation: the last block adds the units' sums and decides.
template <typename T, int NT>
__device__ __forceinline__ void p1_decide(const GridArgs& g, const Slot& s, unsigned units, int decide, double* red) {
    if (!decide || !last_block(s)) return;
    constexpr int K = kSums<T>;
    double sums[K];
    sum_units<NT, K>(s.partial, units, sums, red);
    if (threadIdx.x != 0) return;
    if constexpr (sizeof(T) == 4) decide_inner(s.st, sums, kMaxInnerPerStep);
    else decide_fp64(g, s.st, sums);
}

// ---- P1: residual, weight, Hartley along x --------------------------------------
// MODE 0: stencil residual of the iteration view; MODE 1: q = b (copy, for the
// stand-alone L^+ sweep).
template <typename T, int N, int MODE, int COEF, int WEIGHT>
__global__ void __launch_bounds__((LineCfg<T, N>::NT))
k_resid_dhtx(GridArgs g, const Slot* __restrict__ slots, Tables tb, int decide) {
    using C = LineCfg<T, N>;
    __shared__ cpx<T> lds[C::L * C::LS];
    __shared__ cpx<T> tw[N];
    __shared__ double red[(C::NT / 64) * kSums<T>];
    const Slot& s = slots[blockIdx.y];
    if (MODE == 0 && p1_idle<T>(s, decide)) return;
    const cpx<T>* twg = twiddles<T>(tb, 0);
    const cpx<T>* twc = dct_twiddles<T>(tb);
    for (int e = threadIdx.x; e < N; e += C::NT) tw[e] = twg[e];

    const unsigned nlines = (unsigned)(g.ny * g.nz / 2);
    const unsigned ngroups = (nlines + C::L - 1) / C::L;
    const IterView<T> v(s);
    POIS_GLOBAL T* W = (MODE == 0) ? v.W : (POIS_GLOBAL T*)gptr(s.W);
    double acc[kSums<T>] = {};

    // element `it` of this thread in a group: line (tid + it NT) / N, column (tid + it NT) % N
    auto fetch = [&](unsigned grp, int it, PairIn<T>& in) {
        const int e = threadIdx.x + it * C::NT;
        const unsigned P = grp * C::L + e / N;
        if (P < nlines) {
            const unsigned r0 = 2u * P;  // first row of the pair, k*ny + j
            pair_fetch<T>(g, v.p, v.rho, v.rhs, e % N, (int)(r0 % (unsigned)g.ny), (int)(r0 / (unsigned)g.ny), in);
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                in.r[k] = T(1);
                in.q[k] = T(0);
            }
            in.ba = in.bb = T(0);
        }
    };
    auto evaluate = [&](unsigned grp, int it, const PairIn<T>& in) {
        const int e = threadIdx.x + it * C::NT;
        const int l = e / N, i = e % N;
        cpx<T> qv = {T(0), T(0)};
        if (grp * C::L + l < nlines) {
            const PairOut<T> o = pair_eval<T, COEF, WEIGHT>(g, in, v.rhs_mean, v.rmax, v.rinv, x_walls(g, i));
            qv = {o.a.w * o.a.r, o.b.w * o.b.r};
            acc[0] += (double)o.a.r * o.a.r + (double)o.b.r * o.b.r;
            acc[1] += (double)o.a.bt * o.a.bt + (double)o.b.bt * o.b.bt;
            if constexpr (sizeof(T) == 8) {
                acc[2] += (double)o.a.pc + (double)o.b.pc;
                acc[3] += (double)o.a.pc * o.a.pc + (double)o.b.pc * o.b.pc;
            }
        }
        lds[l * C::LS + C::pos(x_slot(i, N, g.bcx))] = qv;
    };

    unsigned grp = blockIdx.x;
    PairIn<T> A, B;
    if (MODE == 0) fetch(grp, 0, A);
    while (true) {
        if (MODE == 0) {
            // two row pairs per step, each evaluated while the next one's loads fly
            for (int it = 0; it < C::IT; it += 2) {
                fetch(grp, it + 1, B);
                evaluate(grp, it, A);
                const bool last = it + 2 >= C::IT;
                const unsigned ng = last ? grp + gridDim.x : grp;
                if (ng < ngroups) fetch(ng, last ? 0 : it + 2, A);
                evaluate(grp, it + 1, B);
            }
        } else {
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                const int l = e / N, i = e % N;
                const unsigned P = grp * C::L + l;
                const POIS_GLOBAL double* q = gptr(s.b);
                lds[l * C::LS + C::pos(x_slot(i, N, g.bcx))] =
                    (P < nlines) ? cpx<T>{T(q[(2 * P) * N + i]), T(q[(2 * P + 1) * N + i])} : cpx<T>{T(0), T(0)};
            }
        }
        __syncthreads();
        fft_block_lines<T, N>(lds, tw);
#pragma unroll
        for (int it = 0; it < C::IT; ++it) {
            const int e = threadIdx.x + it * C::NT;
            const int l = e / N, k = e % N;
            const unsigned P = grp * C::L + l;
            if (P < nlines) {
                const cpx<T> h = x_forward_out<T, N>(lds + l * C::LS, k, g.bcx, twc);
                W[(2 * P) * N + k] = h.x;
                W[(2 * P + 1) * N + k] = h.y;
            }
        }
        if (MODE == 0) put_unit_sums<C::NT, kSums<T>>(acc, red, s.partial + (unsigned long long)grp * kPartialStride);
        grp += gridDim.x;
        if (grp >= ngroups) break;
        __syncthreads();  // the next group overwrites the lines
    }
    if (MODE == 0) p1_decide<T, C::NT>(g, s, ngroups, decide, red);
}

// In what an FP32 residual is squared and added up, over a flush, for the norms of the
// inner stopping test: FP32 on rows of whole waves, FP64 on the others (16 to 96
// cells, where it costs nothing that was measured: 96^3 632 us a solve with either).
template <int N>
using NormSum = std::conditional_t<N % 64 == 0, float, double>;

// P1 on rows of 16 and more: the residual of a tile of `nflush` KF planes x
// SUB row pairs is computed by z-marching columns (see ZMarch); every KF
// planes the tile's lines are transformed along x and written out.
// Bound by memory on large grids, by latency on small ones.  Measured (MI355X, the
// sweep back to back and without its decision, before -> now, us): FP64 at 64^3 33 ->
// 6.3 (small tiles), 128^3 34 -> 16.2 and 192^3 79 -> 61 (tiles of 8 planes: enough
// blocks, no short last round), 384^3 744 -> 456 (one column per thread instead of
// two), 96^3 32 -> 12.3 (marched, not gathered), 1024 x 512 x 512 2610 -> 2020 (two
// columns per thread, two waves per SIMD, instead of four in one); FP32 at 384^3 250
// -> 215, at 192^3 45 -> 27.  In a solve the launch also holds the hand-over of its
// sums and the decision, which were a kernel of 4-5 us: FP64 at 32^3 9.5 (the sweep
// 5.9), 64^3 11.9, 128^3 21.4, 192^3 68, 384^3 484; FP32 at 192^3 29.8, 384^3 237.
//
// Waves per SIMD the registers are sized for: FP32 rows of up to 512 within 128
// registers, the others within 256.
template <typename T, int N>
constexpr int resid_min_waves() {
    return sizeof(T) == 4 && N <= 512 ? 4 : 2;
}

template <typename T, int N, int COEF, int WEIGHT, int BCX>
__global__ void __launch_bounds__((RowTile<N, true>::NT), (resid_min_waves<T, N>()))
k_resid_dhtx_z(GridArgs g, const Slot* __restrict__ slots, Tables tb, int nflush, int decide) {
    using Z = RowTile<N, true>;
    using RF = RowFlush<T, N>;
    using LF = LineFft<T, N, true, RF::SET>;
    constexpr int KF = RF::KF;
    __shared__ cpx<T> lds[Z::SUB * KF * LF::LS];
    __shared__ cpx<T> tw[N];
    __shared__ double red[(Z::NT / 64) * kSums<T>];
    __shared__ PlaneRows<T> xb[2 * Z::SUB * Z::XV];  // x neighbours, double-buffered by step parity
    const Slot& s = slots[blockIdx.y];
    if (p1_idle<T>(s, decide)) return;
    const cpx<T>* twg = twiddles<T>(tb, 0);
    const cpx<T>* twc = dct_twiddles<T>(tb);
    for (int e = threadIdx.x; e < N; e += Z::NT) tw[e] = twg[e];
    const IterView<T> v(s);

    const unsigned nyh = (unsigned)g.ny / 2, nz = (unsigned)g.nz, km = (unsigned)(nflush * KF);
    const unsigned ngj = (nyh + Z::SUB - 1) / Z::SUB, ngk = (nz + km - 1) / km;
    const unsigned ntiles = ngj * ngk;
    const int sidx = (int)threadIdx.x / Z::MT;
    const unsigned col0 = threadIdx.x % Z::MT;
    ZMarch<T> zm;
    zm.p = (const T*)v.p;
    zm.rho = (const T*)v.rho;
    zm.rhs = (const T*)v.rhs;
    zm.nx = (unsigned)N;
    zm.nz = nz;
    zm.sz = (unsigned)N * (unsigned)g.ny;
    zm.lane = (int)(threadIdx.x & 63);
    double acc[kSums<T>] = {};

    for (unsigned tile = xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const unsigned tj = tile % ngj, tk = tile / ngj;
        const unsigned jp = tj * Z::SUB + sidx;
        const bool jvalid = jp < nyh;
        zm.rows_of(jvalid ? jp : 0u, (unsigned)g.ny);
        const int k0 = (int)(tk * km);
        PlaneRows<T> pl[Z::CPT][3];
        PlaneSide<T> sd[Z::CPT];
#pragma unroll
        for (int c = 0; c < Z::CPT; ++c) {
            const unsigned i = col0 + c * Z::MT;
            zm.load_rows(zm.plane(k0 - 1), i, pl[c][0]);
            zm.load_rows(zm.plane(k0), i, pl[c][1]);
            zm.load_rows(zm.plane(k0 + 1), i, pl[c][2]);
            zm.load_side(zm.plane(k0), i, sd[c]);
        }
        // the lower z faces of each column's pair, carried from plane to plane
        // (one marching column per thread: with more, the registers are spoken for)
        constexpr bool kZC = COEF == 0 && Z::CPT == 1;
        T zc[Z::CPT][2];
        for (int f = 0; f < nflush && k0 + f * KF < (int)nz; ++f) {
            NormSum<N> tacc[2] = {0, 0};
            // fully unrolled, so that the rotation of the plane registers below
            // is a renaming and not a copy that would wait for the prefetched loads
#pragma unroll
            for (int q = 0; q < KF; ++q) {
                const int k = k0 + f * KF + q;
                const bool valid = jvalid && k < (int)nz;
                // the next step's plane and side fly while this step computes (also
                // on the tile's last step, wrapped in z and unused, so that the wait
                // counts are the same every step)
                PlaneRows<T> nn[Z::CPT];
                PlaneSide<T> ns[Z::CPT];
                // waves issuing loads go first, so that the memory requests of
                // all resident waves are out before any spends its step computing
                __builtin_amdgcn_s_setprio(2);
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    const unsigned i = col0 + c * Z::MT;
                    zm.load_rows(zm.plane(k + 2), i, nn[c]);
                    zm.load_side(zm.plane(k + 1), i, ns[c]);
                }
                __builtin_amdgcn_s_setprio(0);
                PlaneRows<T>* eb = xb + ((q & 1) * Z::SUB + sidx) * Z::XV;
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) zm.template x_put<Z::DPP>(eb, col0 + c * Z::MT, pl[c][1]);
                __syncthreads();
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    const unsigned i = col0 + c * Z::MT;
                    PairIn<T> in;
                    PlaneRows<T> xm, xp;
                    zm.template x_get<Z::DPP>(eb, i, pl[c][1], xm, xp);
                    zm.pair(pl[c][0], pl[c][1], pl[c][2], sd[c], xm, xp, in);
                    cpx<T> qv = {T(0), T(0)};
                    if (valid) {
                        if constexpr (kZC)
                            if (q == 0 && f == 0) z_faces_below(in, v.rinv, zc[c]);
                        const PairOut<T> o = pair_eval<T, COEF, WEIGHT, kZC>(g, in, v.rhs_mean, v.rmax, v.rinv,
                                                                             BCX ? x_walls(g, i) : 0u, zc[c]);
                        qv = {o.a.w * o.a.r, o.b.w * o.b.r};
                        if constexpr (sizeof(T) == 8) {
                            acc[0] += o.a.r * o.a.r + o.b.r * o.b.r;
                            acc[1] += o.a.bt * o.a.bt + o.b.bt * o.b.bt;
                            acc[2] += o.a.pc + o.b.pc;
                            acc[3] += o.a.pc * o.a.pc + o.b.pc * o.b.pc;
                        } else {
                            // FP32 inner sweeps: only the two norms are used (the
                            // stopping test)
                            using S = NormSum<N>;
                            tacc[0] += (S)o.a.r * o.a.r + (S)o.b.r * o.b.r;
                            tacc[1] += (S)o.a.bt * o.a.bt + (S)o.b.bt * o.b.bt;
                        }
                    }
                    lds[(q * Z::SUB + sidx) * LF::LS + LF::pos((int)x_slot(i, N, BCX))] = qv;
                }
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    pl[c][0] = pl[c][1];
                    pl[c][1] = pl[c][2];
                    pl[c][2] = nn[c];
                    sd[c] = ns[c];
                }
            }
            if constexpr (sizeof(T) == 4) {
                acc[0] += (double)tacc[0];
                acc[1] += (double)tacc[1];
            }
            __syncthreads();
            const int kf = k0 + f * KF;
            transform_rows<T, N, RF::SET, Z::SUB, KF, Z::CPT>(lds, tw, BCX, twc, sidx, col0, [&](int q, int c, cpx<T> h) {
                if (jvalid && kf + q < (int)nz) {
                    // streaming stores: the transformed lines are not read
                    // again by this sweep, and left out of L2 they do not push
                    // out the rows that neighbouring tiles read as y halo
                    // (FP64 at 512^3: 1.09 -> 1.02 of the algorithmic bytes)
                    const unsigned at = (unsigned)(kf + q) * zm.sz + col0 + c * Z::MT;
                    __builtin_nontemporal_store(h.x, &v.W[at + zm.ra]);
                    __builtin_nontemporal_store(h.y, &v.W[at + zm.rb]);
                }
            });
            __syncthreads();  // the next flush overwrites the lines
        }
        put_unit_sums<Z::NT, kSums<T>>(acc, red, s.partial + (unsigned long long)tile * kPartialStride);
    }
    p1_decide<T, Z::NT>(g, s, ntiles, decide, red);
}

// P1 on small grids, rows of 16 to 512: a tile of KF planes x SUB row pairs whose
// loads are all issued at once, so that a block waits for memory once, and whose
// blocks are many: such a grid lies in the caches, and a marching tile would spend
// its time on one load latency per plane in a few blocks.
template <typename T, int N, int KF, int COEF, int WEIGHT>
__global__ void __launch_bounds__((RowTile<N, false>::NT))
k_resid_dhtx_s(GridArgs g, const Slot* __restrict__ slots, Tables tb, int decide) {
    using Z = RowTile<N, false>;
    using LF = LineFft<T, N, true, 1>;
    static_assert(Z::CPT == 1, "one column per thread");
    __shared__ cpx<T> lds[Z::SUB * KF * LF::LS];
    __shared__ cpx<T> tw[N];
    __shared__ double red[(Z::NT / 64) * kSums<T>];
    __shared__ PlaneRows<T> xb[KF * Z::SUB * Z::XV];
    const Slot& s = slots[blockIdx.y];
    if (p1_idle<T>(s, decide)) return;
    const cpx<T>* twg = twiddles<T>(tb, 0);
    const cpx<T>* twc = dct_twiddles<T>(tb);
    for (int e = threadIdx.x; e < N; e += Z::NT) tw[e] = twg[e];
    const IterView<T> v(s);

    const unsigned nyh = (unsigned)g.ny / 2, nz = (unsigned)g.nz;
    const unsigned ngj = (nyh + Z::SUB - 1) / Z::SUB, ngk = (nz + KF - 1) / KF;
    const unsigned ntiles = ngj * ngk;
    const int sidx = (int)threadIdx.x / N;
    const unsigned i = threadIdx.x % N;
    ZMarch<T> zm;
    zm.p = (const T*)v.p;
    zm.rho = (const T*)v.rho;
    zm.rhs = (const T*)v.rhs;
    zm.nx = (unsigned)N;
    zm.nz = nz;
    zm.sz = (unsigned)N * (unsigned)g.ny;
    zm.lane = (int)(threadIdx.x & 63);
    double acc[kSums<T>] = {};
    for (unsigned tile = xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const unsigned tj = tile % ngj, tk = tile / ngj;
        const unsigned jp = tj * Z::SUB + sidx;
        const bool jvalid = jp < nyh;
        zm.rows_of(jvalid ? jp : 0u, (unsigned)g.ny);
        const int k0 = (int)(tk * KF);
        PlaneRows<T> pl[KF + 2];
        PlaneSide<T> sd[KF];
#pragma unroll
        for (int q = 0; q < KF + 2; ++q) zm.load_rows(zm.plane(k0 + q - 1), i, pl[q]);
#pragma unroll
        for (int q = 0; q < KF; ++q) zm.load_side(zm.plane(k0 + q), i, sd[q]);
#pragma unroll
        for (int q = 0; q < KF; ++q)
            zm.template x_put<Z::DPP>(xb + (q * Z::SUB + sidx) * Z::XV, i, pl[q + 1]);
        __syncthreads();
        T zc[2];
        NormSum<N> tacc[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < KF; ++q) {
            const bool valid = jvalid && k0 + q < (int)nz;
            PairIn<T> in;
            PlaneRows<T> xm, xp;
            zm.template x_get<Z::DPP>(xb + (q * Z::SUB + sidx) * Z::XV, i, pl[q + 1], xm, xp);
            zm.pair(pl[q], pl[q + 1], pl[q + 2], sd[q], xm, xp, in);
            cpx<T> qv = {T(0), T(0)};
            if (valid) {
                if constexpr (COEF == 0)
                    if (q == 0) z_faces_below(in, v.rinv, zc);
                const PairOut<T> o =
                    pair_eval<T, COEF, WEIGHT, COEF == 0>(g, in, v.rhs_mean, v.rmax, v.rinv, x_walls(g, i), zc);
                qv = {o.a.w * o.a.r, o.b.w * o.b.r};
                if constexpr (sizeof(T) == 8) {
                    acc[0] += o.a.r * o.a.r + o.b.r * o.b.r;
                    acc[1] += o.a.bt * o.a.bt + o.b.bt * o.b.bt;
                    acc[2] += o.a.pc + o.b.pc;
                    acc[3] += o.a.pc * o.a.pc + o.b.pc * o.b.pc;
                } else {
                    using S = NormSum<N>;
                    tacc[0] += (S)o.a.r * o.a.r + (S)o.b.r * o.b.r;
                    tacc[1] += (S)o.a.bt * o.a.bt + (S)o.b.bt * o.b.bt;
                }
            }
            lds[(q * Z::SUB + sidx) * LF::LS + LF::pos((int)x_slot(i, N, g.bcx))] = qv;
        }
        if constexpr (sizeof(T) == 4) {
            acc[0] += (double)tacc[0];
            acc[1] += (double)tacc[1];
        }
        __syncthreads();
        transform_rows<T, N, 1, Z::SUB, KF, 1>(lds, tw, g.bcx, twc, sidx, i, [&](int q, int, cpx<T> h) {
            if (jvalid && k0 + q < (int)nz) {
                const unsigned at = (unsigned)(k0 + q) * zm.sz + i;
                v.W[at + zm.ra] = h.x;
                v.W[at + zm.rb] = h.y;
            }
        });
        put_unit_sums<Z::NT, kSums<T>>(acc, red, s.partial + (unsigned long long)tile * kPartialStride);  // ends on a barrier
    }
    p1_decide<T, Z::NT>(g, s, ntiles, decide, red);
}

// Gathered rows: `mode` 1 (any length), or rows shorter than 16.
template <typename T, int N, int MODE, int CO, int WE>
static hipError_t run_gather(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                             float share, int decide) {
    using C = LineCfg<T, N>;
    const unsigned ng = ((unsigned)(g.ny * g.nz / 2) + C::L - 1) / C::L;
    const void* k = (const void*)&k_resid_dhtx<T, N, MODE, CO, WE>;
    const int nb = persistent_grid(k, C::NT, ng, nslots, share);
    k_resid_dhtx<T, N, MODE, CO, WE><<<dim3(nb, nslots), C::NT, reserve_lds(k, share), s>>>(g, slots, t, decide);
    return hipGetLastError();
}

template <typename T, int N, int CO, int WE>
static hipError_t run_small(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                            float share, int decide, bool* fits) {
    using Z = RowTile<N, false>;
    const void* k = (const void*)&k_resid_dhtx_s<T, N, kSmallPlanes, CO, WE>;
    const unsigned nt =
        (((unsigned)g.ny / 2 + Z::SUB - 1) / Z::SUB) * (((unsigned)g.nz + kSmallPlanes - 1) / kSmallPlanes);
    *fits = small_tiles_fit(nt, (unsigned)persistent_grid(k, Z::NT, ~0u, 1, 1.0f));
    if (!*fits) return hipSuccess;
    const int nb = persistent_grid(k, Z::NT, nt, nslots, share);
    k_resid_dhtx_s<T, N, kSmallPlanes, CO, WE><<<dim3(nb, nslots), Z::NT, reserve_lds(k, share), s>>>(g, slots, t, decide);
    return hipGetLastError();
}

template <typename T, int N, int CO, int WE, int BC>
static hipError_t run_march(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                            float share, int decide) {
    using Z = RowTile<N, true>;
    constexpr int KF = RowFlush<T, N>::KF;
    const void* k = (const void*)&k_resid_dhtx_z<T, N, CO, WE, BC>;
    const unsigned strips = ((unsigned)g.ny / 2 + Z::SUB - 1) / Z::SUB;
    // long FP32 rows with many strips: shorter tiles keep neighbours closer in z,
    // so that more of the y halo rows they read from each other are still in L2
    // (512^3: 463 us, 32 planes 481; 512 x 256 x 256 the other way, 126 and 118)
    const int most = sizeof(T) == 4 && N >= 512 && strips >= 256 ? 16 : 32;
    const int nf = pick_flushes(KF, most, strips, (unsigned)g.nz, (unsigned)persistent_grid(k, Z::NT, ~0u, 1, 1.0f));
    const unsigned km = (unsigned)(nf * KF), nt = strips * (((unsigned)g.nz + km - 1) / km);
    const int nb = persistent_grid(k, Z::NT, nt, nslots, share);
    k_resid_dhtx_z<T, N, CO, WE, BC><<<dim3(nb, nslots), Z::NT, reserve_lds(k, share), s>>>(g, slots, t, nf, decide);
    return hipGetLastError();
}

// The tiles follow from the grid alone (and the chip's size), so that the units'
// sums are the same bits in every batch and share.
template <typename T>
hipError_t launch_resid(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                        float share, bool dec) {
    const int decide = dec ? 1 : 0;
    return dispatch_len(g.nx, [&]<int N>() {
        if (mode == 1) return run_gather<T, N, 1, 0, 0>(g, t, slots, nslots, s, share, decide);
        return dispatch_op(g.coef, g.weight, [&]<int CO, int WE>() {
            if constexpr (N < 16) {
                return run_gather<T, N, 0, CO, WE>(g, t, slots, nslots, s, share, decide);
            } else {
                if constexpr (N <= 512) {
                    bool fits = false;
                    const hipError_t e = run_small<T, N, CO, WE>(g, t, slots, nslots, s, share, decide, &fits);
                    if (fits) return e;
                }
                return dispatch_bc(g.bcx, [&]<int BC>() {
                    return run_march<T, N, CO, WE, BC>(g, t, slots, nslots, s, share, decide);
                });
            }
        });
    });
}

}  // namespace pois
