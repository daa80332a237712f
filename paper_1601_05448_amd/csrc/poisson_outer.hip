// The FP64 outer residual of a refinement step fused with the first FP32 inner
// sweep's residual (see poisson_sweeps.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_control.hpp"
#include "poisson_device.hpp"
#include "poisson_launch.hpp"
#include "poisson_rows.hpp"

namespace pois {

// The end of the sweep: the last block adds the units' sums and decides.
template <int NT>
__device__ __forceinline__ void outer_decide(const GridArgs& g, const Slot& s, unsigned units, int write, int decide,
                                             double* red) {
    if (!decide || !last_block(s)) return;
    double sums[5];
    sum_units<NT, 5>(s.partial, units, sums, red);
    if (threadIdx.x == 0) decide_outer(g, s.st, sums, write != 0, write == 0);
}

// FP32_REFINE: the FP64 outer residual of a refinement step fused with the
// residual half of its first FP32 inner sweep.  The inner correction starts at
// zero, so that sweep's weighted residual is q = w r32 with r32 = r s^-1 of the
// FP64 residual r = b~ - A p: the tile's FP64 residual (z-marching as in P1)
// gives r32 (stored for the later inner sweeps) and q, whose lines are
// transformed along x into W32 exactly as the FP32 P1 would.  The mean of r32,
// which the FP32 P1 removes, is FP64 rounding noise here and is not removed.
// Per tile: r^2, bt^2, p, p^2, r in FP64.  write = 0: the sums alone (the final
// check of a solve, which usually ends it: no r32, no transform, no W32).
template <int N, int COEF, int WEIGHT, int BCX>
__global__ void __launch_bounds__((RowTile<N, true>::NT), 2)
k_outer_resid_dhtx(GridArgs g, const Slot* __restrict__ slots, Tables tb, int write, int nflush, int decide) {
    using Z = RowTile<N, true>;
    using RF = RowFlush<double, N>;
    using LF = LineFft<float, N, true, RF::SET>;
    constexpr int KF = RF::KF;
    __shared__ cpx<float> lds[Z::SUB * KF * LF::LS];
    __shared__ cpx<float> tw[N];
    __shared__ double red[(Z::NT / 64) * 5];
    __shared__ PlaneRows<double> xb[2 * Z::SUB * Z::XV];
    const Slot& s = slots[blockIdx.y];
    SolveState* st = s.st;
    if (st->done || st->stage != 0) return;
    const cpx<float>* twg = twiddles<float>(tb, 0);
    const cpx<float>* twc = dct_twiddles<float>(tb);
    for (int e = threadIdx.x; e < N; e += Z::NT) tw[e] = twg[e];
    const double bm = st->b_mean, inv_s = st->inv_s, rmax = st->rho_max, rinv = recip(st->rho_max);

    const unsigned nyh = (unsigned)g.ny / 2, nz = (unsigned)g.nz, km = (unsigned)(nflush * KF);
    const unsigned ngj = (nyh + Z::SUB - 1) / Z::SUB, ngk = (nz + km - 1) / km;
    const unsigned ntiles = ngj * ngk;
    const int sidx = (int)threadIdx.x / Z::MT;
    const unsigned col0 = threadIdx.x % Z::MT;
    POIS_GLOBAL float* r32 = gptr(s.r32);
    POIS_GLOBAL float* W32 = gptr(s.W32);
    ZMarch<double> zm;
    zm.p = s.p;
    zm.rho = s.rho;
    zm.rhs = s.b;
    zm.nx = (unsigned)N;
    zm.nz = nz;
    zm.sz = (unsigned)N * (unsigned)g.ny;
    zm.lane = (int)(threadIdx.x & 63);
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};

    for (unsigned tile = xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const unsigned tj = tile % ngj, tk = tile / ngj;
        const unsigned jp = tj * Z::SUB + sidx;
        const bool jvalid = jp < nyh;
        zm.rows_of(jvalid ? jp : 0u, (unsigned)g.ny);
        const int k0 = (int)(tk * km);
        PlaneRows<double> pl[Z::CPT][3];
        PlaneSide<double> sd[Z::CPT];
#pragma unroll
        for (int c = 0; c < Z::CPT; ++c) {
            const unsigned i = col0 + c * Z::MT;
            zm.load_rows(zm.plane(k0 - 1), i, pl[c][0]);
            zm.load_rows(zm.plane(k0), i, pl[c][1]);
            zm.load_rows(zm.plane(k0 + 1), i, pl[c][2]);
            zm.load_side(zm.plane(k0), i, sd[c]);
        }
        // the lower z faces of the pair, carried from plane to plane (COEF 0)
        constexpr bool kZC = COEF == 0 && Z::CPT == 1;
        double zc[Z::CPT][2];
        for (int f = 0; f < nflush && k0 + f * KF < (int)nz; ++f) {
#pragma unroll
            for (int q = 0; q < KF; ++q) {
                const int k = k0 + f * KF + q;
                const bool valid = jvalid && k < (int)nz;
                PlaneRows<double> nn[Z::CPT];
                PlaneSide<double> ns[Z::CPT];
                __builtin_amdgcn_s_setprio(2);
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    const unsigned i = col0 + c * Z::MT;
                    zm.load_rows(zm.plane(k + 2), i, nn[c]);
                    zm.load_side(zm.plane(k + 1), i, ns[c]);
                }
                __builtin_amdgcn_s_setprio(0);
                PlaneRows<double>* eb = xb + ((q & 1) * Z::SUB + sidx) * Z::XV;
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) zm.template x_put<Z::DPP>(eb, col0 + c * Z::MT, pl[c][1]);
                __syncthreads();
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    const unsigned i = col0 + c * Z::MT;
                    PairIn<double> in;
                    PlaneRows<double> xm, xp;
                    zm.template x_get<Z::DPP>(eb, i, pl[c][1], xm, xp);
                    zm.pair(pl[c][0], pl[c][1], pl[c][2], sd[c], xm, xp, in);
                    cpx<float> qv = {0.0f, 0.0f};
                    if (valid) {
                        if constexpr (kZC)
                            if (q == 0 && f == 0) z_faces_below(in, rinv, zc[c]);
                        const PairOut<double> pr =
                            pair_eval<double, COEF, WEIGHT, kZC>(g, in, bm, rmax, rinv, BCX ? x_walls(g, i) : 0u, zc[c]);
                        acc[0] += pr.a.r * pr.a.r + pr.b.r * pr.b.r;
                        acc[1] += pr.a.bt * pr.a.bt + pr.b.bt * pr.b.bt;
                        acc[2] += pr.a.pc + pr.b.pc;
                        acc[3] += pr.a.pc * pr.a.pc + pr.b.pc * pr.b.pc;
                        acc[4] += pr.a.r + pr.b.r;
                        if (write) {
                            const float ra = (float)(pr.a.r * inv_s), rb = (float)(pr.b.r * inv_s);
                            const unsigned at = (unsigned)k * zm.sz + i;
                            __builtin_nontemporal_store(ra, &r32[at + zm.ra]);  // streaming (see k_resid_dhtx_z)
                            __builtin_nontemporal_store(rb, &r32[at + zm.rb]);
                            qv = {(float)pr.a.w * ra, (float)pr.b.w * rb};
                        }
                    }
                    if (write) lds[(q * Z::SUB + sidx) * LF::LS + LF::pos((int)x_slot(i, N, BCX))] = qv;
                }
#pragma unroll
                for (int c = 0; c < Z::CPT; ++c) {
                    pl[c][0] = pl[c][1];
                    pl[c][1] = pl[c][2];
                    pl[c][2] = nn[c];
                    sd[c] = ns[c];
                }
            }
            if (!write) continue;  // uniform
            __syncthreads();
            const int kf = k0 + f * KF;
            transform_rows<float, N, RF::SET, Z::SUB, KF, Z::CPT>(lds, tw, BCX, twc, sidx, col0,
                                                                   [&](int q, int c, cpx<float> h) {
                if (jvalid && kf + q < (int)nz) {
                    const unsigned at = (unsigned)(kf + q) * zm.sz + col0 + c * Z::MT;
                    __builtin_nontemporal_store(h.x, &W32[at + zm.ra]);
                    __builtin_nontemporal_store(h.y, &W32[at + zm.rb]);
                }
            });
            __syncthreads();  // the next flush overwrites the lines
        }
        put_unit_sums<Z::NT, 5>(acc, red, s.partial + (unsigned long long)tile * kPartialStride);
    }
    outer_decide<Z::NT>(g, s, ntiles, write, decide, red);
}

// The same on small grids, every load of a tile issued at once (see k_resid_dhtx_s).
template <int N, int KF, int COEF, int WEIGHT>
__global__ void __launch_bounds__((RowTile<N, false>::NT))
k_outer_resid_dhtx_s(GridArgs g, const Slot* __restrict__ slots, Tables tb, int write, int decide) {
    using Z = RowTile<N, false>;
    using LF = LineFft<float, N, true, 1>;
    static_assert(Z::CPT == 1, "one column per thread");
    __shared__ cpx<float> lds[Z::SUB * KF * LF::LS];
    __shared__ cpx<float> tw[N];
    __shared__ double red[(Z::NT / 64) * 5];
    __shared__ PlaneRows<double> xb[KF * Z::SUB * Z::XV];
    const Slot& s = slots[blockIdx.y];
    SolveState* st = s.st;
    if (st->done || st->stage != 0) return;
    const cpx<float>* twg = twiddles<float>(tb, 0);
    const cpx<float>* twc = dct_twiddles<float>(tb);
    for (int e = threadIdx.x; e < N; e += Z::NT) tw[e] = twg[e];
    const double bm = st->b_mean, inv_s = st->inv_s, rmax = st->rho_max, rinv = recip(st->rho_max);

    const unsigned nyh = (unsigned)g.ny / 2, nz = (unsigned)g.nz;
    const unsigned ngj = (nyh + Z::SUB - 1) / Z::SUB, ngk = (nz + KF - 1) / KF;
    const unsigned ntiles = ngj * ngk;
    const int sidx = (int)threadIdx.x / N;
    const unsigned i = threadIdx.x % N;
    POIS_GLOBAL float* r32 = gptr(s.r32);
    POIS_GLOBAL float* W32 = gptr(s.W32);
    ZMarch<double> zm;
    zm.p = s.p;
    zm.rho = s.rho;
    zm.rhs = s.b;
    zm.nx = (unsigned)N;
    zm.nz = nz;
    zm.sz = (unsigned)N * (unsigned)g.ny;
    zm.lane = (int)(threadIdx.x & 63);
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (unsigned tile = xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const unsigned tj = tile % ngj, tk = tile / ngj;
        const unsigned jp = tj * Z::SUB + sidx;
        const bool jvalid = jp < nyh;
        zm.rows_of(jvalid ? jp : 0u, (unsigned)g.ny);
        const int k0 = (int)(tk * KF);
        PlaneRows<double> pl[KF + 2];
        PlaneSide<double> sd[KF];
#pragma unroll
        for (int q = 0; q < KF + 2; ++q) zm.load_rows(zm.plane(k0 + q - 1), i, pl[q]);
#pragma unroll
        for (int q = 0; q < KF; ++q) zm.load_side(zm.plane(k0 + q), i, sd[q]);
#pragma unroll
        for (int q = 0; q < KF; ++q)
            zm.template x_put<Z::DPP>(xb + (q * Z::SUB + sidx) * Z::XV, i, pl[q + 1]);
        __syncthreads();
        double zc[2];
#pragma unroll
        for (int q = 0; q < KF; ++q) {
            const bool valid = jvalid && k0 + q < (int)nz;
            PairIn<double> in;
            PlaneRows<double> xm, xp;
            zm.template x_get<Z::DPP>(xb + (q * Z::SUB + sidx) * Z::XV, i, pl[q + 1], xm, xp);
            zm.pair(pl[q], pl[q + 1], pl[q + 2], sd[q], xm, xp, in);
            cpx<float> qv = {0.0f, 0.0f};
            if (valid) {
                if constexpr (COEF == 0)
                    if (q == 0) z_faces_below(in, rinv, zc);
                const PairOut<double> pr =
                    pair_eval<double, COEF, WEIGHT, COEF == 0>(g, in, bm, rmax, rinv, x_walls(g, i), zc);
                acc[0] += pr.a.r * pr.a.r + pr.b.r * pr.b.r;
                acc[1] += pr.a.bt * pr.a.bt + pr.b.bt * pr.b.bt;
                acc[2] += pr.a.pc + pr.b.pc;
                acc[3] += pr.a.pc * pr.a.pc + pr.b.pc * pr.b.pc;
                acc[4] += pr.a.r + pr.b.r;
                if (write) {
                    const float ra = (float)(pr.a.r * inv_s), rb = (float)(pr.b.r * inv_s);
                    const unsigned at = (unsigned)(k0 + q) * zm.sz + i;
                    r32[at + zm.ra] = ra;
                    r32[at + zm.rb] = rb;
                    qv = {(float)pr.a.w * ra, (float)pr.b.w * rb};
                }
            }
            if (write) lds[(q * Z::SUB + sidx) * LF::LS + LF::pos((int)x_slot(i, N, g.bcx))] = qv;
        }
        if (write) {
            __syncthreads();
            transform_rows<float, N, 1, Z::SUB, KF, 1>(lds, tw, g.bcx, twc, sidx, i, [&](int q, int, cpx<float> h) {
                if (jvalid && k0 + q < (int)nz) {
                    const unsigned at = (unsigned)(k0 + q) * zm.sz + i;
                    W32[at + zm.ra] = h.x;
                    W32[at + zm.rb] = h.y;
                }
            });
        }
        put_unit_sums<Z::NT, 5>(acc, red, s.partial + (unsigned long long)tile * kPartialStride);  // ends on a barrier
    }
    outer_decide<Z::NT>(g, s, ntiles, write, decide, red);
}

bool outer_fusable(const GridArgs& g) { return g.nx >= 16; }

hipError_t launch_outer_fused(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                              float share, bool write, bool decide) {
    const int wr = write ? 1 : 0, dec = decide ? 1 : 0;
    return dispatch_len(g.nx, [&]<int N>() {
        if constexpr (N < 16) {
            return hipErrorInvalidValue;
        } else {
            return dispatch_op(g.coef, g.weight, [&]<int CO, int WE>() {
                if constexpr (N <= 512) {
                    using Z = RowTile<N, false>;
                    const void* k = (const void*)&k_outer_resid_dhtx_s<N, kSmallPlanes, CO, WE>;
                    const unsigned nt = (((unsigned)g.ny / 2 + Z::SUB - 1) / Z::SUB) *
                                        (((unsigned)g.nz + kSmallPlanes - 1) / kSmallPlanes);
                    if (small_tiles_fit(nt, (unsigned)persistent_grid(k, Z::NT, ~0u, 1, 1.0f))) {
                        const int nb = persistent_grid(k, Z::NT, nt, nslots, share);
                        k_outer_resid_dhtx_s<N, kSmallPlanes, CO, WE>
                            <<<dim3(nb, nslots), Z::NT, reserve_lds(k, share), s>>>(g, slots, t, wr, dec);
                        return hipGetLastError();
                    }
                }
                return dispatch_bc(g.bcx, [&]<int BC>() {
                    using Z = RowTile<N, true>;
                    constexpr int KF = RowFlush<double, N>::KF;
                    const void* k = (const void*)&k_outer_resid_dhtx<N, CO, WE, BC>;
                    const unsigned strips = ((unsigned)g.ny / 2 + Z::SUB - 1) / Z::SUB;
                    const int nf = pick_flushes(KF, 32, strips, (unsigned)g.nz,
                                                (unsigned)persistent_grid(k, Z::NT, ~0u, 1, 1.0f));
                    const unsigned km = (unsigned)(nf * KF), nt = strips * (((unsigned)g.nz + km - 1) / km);
                    const int nb = persistent_grid(k, Z::NT, nt, nslots, share);
                    k_outer_resid_dhtx<N, CO, WE, BC>
                        <<<dim3(nb, nslots), Z::NT, reserve_lds(k, share), s>>>(g, slots, t, wr, nf, dec);
                    return hipGetLastError();
                });
            });
        }
    });
}

}  // namespace pois
