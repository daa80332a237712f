// The residual sweep P1 (see poisson_sweeps.hip): residual, weight, partial norms
// per tile, Hartley (or, between walls, cosine) transform along x.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_device.hpp"
#include "poisson_launch.hpp"

namespace pois {

// Rows that fill whole waves, and a register budget for CPT marching columns.
template <typename T, int N>
constexpr bool use_zmarch() {
    using C = LineCfg<T, N>;
    if constexpr (N % 64 != 0) return false;
    else return (N >= C::NT ? N / C::NT : 1) * (int)sizeof(T) <= 32;
}

// Minimum waves per SIMD the residual sweep's registers are sized for (the
// second __launch_bounds__ argument, which caps the registers per thread): one
// where four FP64 marching columns per thread need the accumulation registers
// too.  The FP32 sweep on 512-cell rows runs 512-thread blocks whose LDS leaves
// room for two per CU: asking for four waves per SIMD (128 registers) lets both
// be resident, 16 waves per CU instead of 8 (6% faster at 512^3; the FP32 y, z
// and x-update sweeps spill at 128 registers and lose 2x, so they keep one).
template <typename T, int N>
constexpr int p1_min_blocks() {
    using C = LineCfg<T, N>;
    if constexpr (sizeof(T) == 4 && N == 512 && C::NT == 512) return 4;
    return (N >= C::NT ? N / C::NT : 1) * (int)sizeof(T) > 16 ? 1 : C::MINB;
}

// ---- P1: residual, weight, Hartley along x --------------------------------------
// MODE 0: stencil residual of the iteration view; MODE 1: q = b (copy, for the
// stand-alone L^+ sweep).
template <typename T, int N, int MODE, int COEF, int WEIGHT>
__global__ void __launch_bounds__((LineCfg<T, N>::NT))
k_resid_dhtx(GridArgs g, const Slot* __restrict__ slots, Tables tb) {
    using C = LineCfg<T, N>;
    __shared__ cpx<T> lds[C::L * C::LS];
    __shared__ cpx<T> tw[N];
    __shared__ double red[(C::NT / 64) * 4];
    const Slot& s = slots[blockIdx.y];
    if (MODE == 0 && IterView<T>::skip_p1(s.st)) return;
    const cpx<T>* twg = twiddles<T>(tb, 0);
    const cpx<T>* twc = dct_twiddles<T>(tb);
    for (int e = threadIdx.x; e < N; e += C::NT) tw[e] = twg[e];

    const unsigned nlines = (unsigned)(g.ny * g.nz / 2);
    const unsigned ngroups = (nlines + C::L - 1) / C::L;
    const IterView<T> v(s);
    POIS_GLOBAL T* W = (MODE == 0) ? v.W : (POIS_GLOBAL T*)gptr(s.W);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};  // sum r^2, sum bt^2, sum p, sum p^2

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
            acc[2] += (double)o.a.pc + (double)o.b.pc;
            acc[3] += (double)o.a.pc * o.a.pc + (double)o.b.pc * o.b.pc;
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
        if (MODE == 0) put_unit_sums<C::NT, 4>(acc, red, s.partial + (unsigned long long)grp * kPartialStride);
        grp += gridDim.x;
        if (grp >= ngroups) break;
        __syncthreads();  // the next group overwrites the lines
    }
}

// P1 for rows whose length is a multiple of the wave size: the residual of a tile
// of KM planes x SUB row pairs is computed by z-marching columns (see ZMarch);
// every KF planes the tile's L lines are transformed along x and written out.
// Within a flush, line l = s KF + q is row pair jp = tj SUB + s of plane
// k = tk KM + f KF + q.
template <typename T, int N, int COEF, int WEIGHT, int BCX>
__global__ void __launch_bounds__((LineCfg<T, N>::NT), (p1_min_blocks<T, N>()))
k_resid_dhtx_z(GridArgs g, const Slot* __restrict__ slots, Tables tb) {
    using C = LineCfg<T, N>;
    using Z = P1Tile<T, N>;
    __shared__ cpx<T> lds[C::L * C::LS];
    __shared__ cpx<T> tw[N];
    __shared__ double red[(C::NT / 64) * 4];
    __shared__ T edge[2 * Z::SUB * Z::EDGE];  // wave-edge columns, double-buffered by step parity
    const Slot& s = slots[blockIdx.y];
    if (IterView<T>::skip_p1(s.st)) return;
    const cpx<T>* twg = twiddles<T>(tb, 0);
    const cpx<T>* twc = dct_twiddles<T>(tb);
    for (int e = threadIdx.x; e < N; e += C::NT) tw[e] = twg[e];
    const IterView<T> v(s);

    const unsigned nyh = (unsigned)g.ny / 2, nz = (unsigned)g.nz;
    const unsigned ngj = (nyh + Z::SUB - 1) / Z::SUB, ngk = (nz + Z::KM - 1) / Z::KM;
    const unsigned ntiles = ngj * ngk;
    const int sidx = (N >= C::NT) ? 0 : (int)threadIdx.x / N;
    const unsigned col0 = (N >= C::NT) ? threadIdx.x : threadIdx.x % N;
    ZMarch<T> zm;
    zm.p = (const T*)v.p;
    zm.rho = (const T*)v.rho;
    zm.rhs = (const T*)v.rhs;
    zm.nx = (unsigned)g.nx;
    zm.nz = nz;
    zm.sz = (unsigned)g.nx * (unsigned)g.ny;
    zm.lane = (int)(threadIdx.x & 63);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};  // sum r^2, sum bt^2, sum p, sum p^2

    for (unsigned tile = xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const unsigned tj = tile % ngj, tk = tile / ngj;
        const unsigned jp = tj * Z::SUB + sidx;
        const bool jvalid = jp < nyh;
        zm.rows_of(jvalid ? jp : 0u, (unsigned)g.ny);
        const int k0 = (int)(tk * Z::KM);
        PlaneRows<T> pl[Z::CPT][3];
        PlaneSide<T> sd[Z::CPT];
#pragma unroll
        for (int c = 0; c < Z::CPT; ++c) {
            const unsigned i = col0 + c * C::NT;
            zm.load_rows(zm.plane(k0 - 1), i, pl[c][0]);
            zm.load_rows(zm.plane(k0), i, pl[c][1]);
            zm.load_rows(zm.plane(k0 + 1), i, pl[c][2]);
            zm.load_side(zm.plane(k0), i, sd[c]);
        }
        // the lower z faces of each column's pair, carried from plane to plane
        // (one marching column per thread: with more, the registers are spoken for)
        constexpr bool kZC = COEF == 0 && Z::CPT == 1;
        T zc[Z::CPT][2];
        for (int f = 0; f < Z::KM / Z::KF; ++f) {
            T tacc[2] = {T(0), T(0)};
            // fully unrolled, so that the rotation of the plane registers below
            // is a renaming and not a copy that would wait for the prefetched loads
#pragma unroll
            for (int q = 0; q < Z::KF; ++q) {
                const int k = k0 + f * Z::KF + q;
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
                    const unsigned i = col0 + c * C::NT;
                    zm.load_rows(zm.plane(k + 2), i, nn[c]);
                    zm.load_side(zm.plane(k + 1), i, ns[c]);
                }
                __builtin_amdgcn_s_setprio(0);
                T* eb = edge + ((q & 1) * Z::SUB + sidx) * Z::EDGE;
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) zm.edge_put(eb, col0 + c * C::NT, pl[c][1]);
                __syncthreads();
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    const unsigned i = col0 + c * C::NT;
                    PairIn<T> in;
                    zm.pair(pl[c][0], pl[c][1], pl[c][2], sd[c], zm.edge_get(eb, i), in);
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
                            // stopping test), summed in FP32 over the flush
                            tacc[0] += o.a.r * o.a.r + o.b.r * o.b.r;
                            tacc[1] += o.a.bt * o.a.bt + o.b.bt * o.b.bt;
                        }
                    }
                    lds[(sidx * Z::KF + q) * C::LS + C::pos(x_slot(i, N, BCX))] = qv;
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
            fft_block_lines<T, N>(lds, tw);
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                const int l = e / N, k = e % N;
                const unsigned ljp = tj * Z::SUB + l / Z::KF;
                const unsigned lk = (unsigned)(k0 + f * Z::KF) + l % Z::KF;
                if (ljp < nyh && lk < nz) {
                    const unsigned P = lk * nyh + ljp;  // row pair index, rows 2P and 2P + 1
                    const cpx<T> h = x_forward_out<T, N>(lds + l * C::LS, k, BCX, twc);
                    // streaming stores: the transformed lines are not read
                    // again by this sweep, and left out of L2 they do not push
                    // out the rows that neighbouring tiles read as y halo
                    // (FP64 at 512^3: 1.09 -> 1.02 of the algorithmic bytes)
                    __builtin_nontemporal_store(h.x, &v.W[(2 * P) * N + k]);
                    __builtin_nontemporal_store(h.y, &v.W[(2 * P + 1) * N + k]);
                }
            }
            __syncthreads();  // the next flush overwrites the lines
        }
        put_unit_sums<C::NT, 4>(acc, red, s.partial + (unsigned long long)tile * kPartialStride);
    }
}

template <typename T, int MODE>
static hipError_t resid_t(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                          int* nunits, float share) {
    const unsigned rows = (unsigned)(g.ny * g.nz / 2);
    return dispatch_len(g.nx, [&]<int N>() {
        using C = LineCfg<T, N>;
        const unsigned ng = (rows + C::L - 1) / C::L;
        return dispatch_op(MODE == 1 ? 0 : g.coef, MODE == 1 ? 0 : g.weight, [&]<int CO, int WE>() {
            if constexpr (MODE == 0 && use_zmarch<T, N>()) {
                using Z = P1Tile<T, N>;
                const unsigned nt = (((unsigned)g.ny / 2 + Z::SUB - 1) / Z::SUB) *
                                    (((unsigned)g.nz + Z::KM - 1) / Z::KM);
                if (nunits) *nunits = (int)nt;
                return dispatch_bc(g.bcx, [&]<int BC>() {
                    const void* k = (const void*)&k_resid_dhtx_z<T, N, CO, WE, BC>;
                    const int nb = persistent_grid(k, C::NT, nt, nslots, share);
                    k_resid_dhtx_z<T, N, CO, WE, BC>
                        <<<dim3(nb, nslots), C::NT, reserve_lds(k, share), s>>>(g, slots, t);
                    return hipGetLastError();
                });
            } else {
                const void* k = (const void*)&k_resid_dhtx<T, N, MODE, CO, WE>;
                const int nb = persistent_grid(k, C::NT, ng, nslots, share);
                if (nunits) *nunits = (int)ng;
                k_resid_dhtx<T, N, MODE, CO, WE><<<dim3(nb, nslots), C::NT, reserve_lds(k, share), s>>>(g, slots, t);
            }
            return hipGetLastError();
        });
    });
}

template <typename T>
hipError_t launch_resid(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                        int* nunits, float share) {
    return mode == 1 ? resid_t<T, 1>(g, t, slots, nslots, s, nunits, share)
                     : resid_t<T, 0>(g, t, slots, nslots, s, nunits, share);
}

}  // namespace pois
