// The FP64 outer residual of a refinement step fused with the first FP32 inner
// sweep's residual (see poisson_sweeps.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_device.hpp"
#include "poisson_launch.hpp"

namespace pois {

// FP32_REFINE: the FP64 outer residual of a refinement step fused with the
// residual half of its first FP32 inner sweep.  The inner correction starts at
// zero, so that sweep's weighted residual is q = w r32 with r32 = r s^-1 of the
// FP64 residual r = b~ - A p: the tile's FP64 residual (z-marching as in P1)
// gives r32 (stored for the later inner sweeps) and q, whose lines are
// transformed along x into W32 exactly as the FP32 P1 would.  The mean of r32,
// which the FP32 P1 removes, is FP64 rounding noise here and is not removed.
// Per tile: r^2, bt^2, p, p^2, r in FP64.  One column per thread.  write = 0:
// the sums alone (the final check of a solve, which usually ends it: no r32,
// no transform, no W32).
template <int N, int COEF, int WEIGHT, int BCX>
__global__ void __launch_bounds__((LineCfg<float, N>::NT), (LineCfg<float, N>::MINB))
k_outer_resid_dhtx(GridArgs g, const Slot* __restrict__ slots, Tables tb, int write) {
    using C = LineCfg<float, N>;
    using Z = OuterTile<N>;
    static_assert(Z::CPT == 1, "one marching column per thread");
    __shared__ cpx<float> lds[C::L * C::LS];
    __shared__ cpx<float> tw[N];
    __shared__ double red[(C::NT / 64) * 5];
    __shared__ double edge[2 * Z::SUB * Z::EDGE];
    const Slot& s = slots[blockIdx.y];
    SolveState* st = s.st;
    if (st->done || st->stage != 0) return;
    const cpx<float>* twg = twiddles<float>(tb, 0);
    const cpx<float>* twc = dct_twiddles<float>(tb);
    for (int e = threadIdx.x; e < N; e += C::NT) tw[e] = twg[e];
    const double bm = st->b_mean, inv_s = st->inv_s, rmax = st->rho_max, rinv = recip(st->rho_max);

    const unsigned nyh = (unsigned)g.ny / 2, nz = (unsigned)g.nz;
    const unsigned ngj = (nyh + Z::SUB - 1) / Z::SUB, ngk = (nz + Z::KM - 1) / Z::KM;
    const unsigned ntiles = ngj * ngk;
    const int sidx = (N >= C::NT) ? 0 : (int)threadIdx.x / N;
    const unsigned i = (N >= C::NT) ? threadIdx.x : threadIdx.x % N;
    POIS_GLOBAL float* r32 = gptr(s.r32);
    POIS_GLOBAL float* W32 = gptr(s.W32);
    ZMarch<double> zm;
    zm.p = s.p;
    zm.rho = s.rho;
    zm.rhs = s.b;
    zm.nx = (unsigned)g.nx;
    zm.nz = nz;
    zm.sz = (unsigned)g.nx * (unsigned)g.ny;
    zm.lane = (int)(threadIdx.x & 63);
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};

    for (unsigned tile = xcd_block(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const unsigned tj = tile % ngj, tk = tile / ngj;
        const unsigned jp = tj * Z::SUB + sidx;
        const bool jvalid = jp < nyh;
        zm.rows_of(jvalid ? jp : 0u, (unsigned)g.ny);
        const int k0 = (int)(tk * Z::KM);
        PlaneRows<double> pl[3];
        PlaneSide<double> sd;
        zm.load_rows(zm.plane(k0 - 1), i, pl[0]);
        zm.load_rows(zm.plane(k0), i, pl[1]);
        zm.load_rows(zm.plane(k0 + 1), i, pl[2]);
        zm.load_side(zm.plane(k0), i, sd);
        double zc[2];  // the lower z faces of the pair, carried from plane to plane (COEF 0)
        for (int f = 0; f < Z::KM / Z::KF; ++f) {
#pragma unroll
            for (int q = 0; q < Z::KF; ++q) {
                const int k = k0 + f * Z::KF + q;
                const bool valid = jvalid && k < (int)nz;
                PlaneRows<double> nn;
                PlaneSide<double> ns;
                __builtin_amdgcn_s_setprio(2);
                zm.load_rows(zm.plane(k + 2), i, nn);
                zm.load_side(zm.plane(k + 1), i, ns);
                __builtin_amdgcn_s_setprio(0);
                double* eb = edge + ((q & 1) * Z::SUB + sidx) * Z::EDGE;
                zm.edge_put(eb, i, pl[1]);
                __syncthreads();
                PairIn<double> in;
                zm.pair(pl[0], pl[1], pl[2], sd, zm.edge_get(eb, i), in);
                cpx<float> qv = {0.0f, 0.0f};
                if (valid) {
                    if constexpr (COEF == 0)
                        if (q == 0 && f == 0) z_faces_below(in, rinv, zc);
                    const PairOut<double> pr =
                        pair_eval<double, COEF, WEIGHT, COEF == 0>(g, in, bm, rmax, rinv, BCX ? x_walls(g, i) : 0u, zc);
                    acc[0] += pr.a.r * pr.a.r + pr.b.r * pr.b.r;
                    acc[1] += pr.a.bt * pr.a.bt + pr.b.bt * pr.b.bt;
                    acc[2] += pr.a.pc + pr.b.pc;
                    acc[3] += pr.a.pc * pr.a.pc + pr.b.pc * pr.b.pc;
                    acc[4] += pr.a.r + pr.b.r;
                    if (write) {
                        const float ra = (float)(pr.a.r * inv_s), rb = (float)(pr.b.r * inv_s);
                        const unsigned a = (unsigned)k * zm.sz + zm.ra + i;
                        __builtin_nontemporal_store(ra, &r32[a]);  // streaming (see k_resid_dhtx_z)
                        __builtin_nontemporal_store(rb, &r32[a + (unsigned)g.nx]);
                        qv = {(float)pr.a.w * ra, (float)pr.b.w * rb};
                    }
                }
                if (write) lds[(sidx * Z::KF + q) * C::LS + C::pos(x_slot(i, N, BCX))] = qv;
                pl[0] = pl[1];
                pl[1] = pl[2];
                pl[2] = nn;
                sd = ns;
            }
            if (!write) continue;  // uniform
            __syncthreads();
            fft_block_lines<float, N>(lds, tw);
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                const int l = e / N, kx = e % N;
                const unsigned ljp = tj * Z::SUB + l / Z::KF;
                const unsigned lk = (unsigned)(k0 + f * Z::KF) + l % Z::KF;
                if (ljp < nyh && lk < nz) {
                    const unsigned P = lk * nyh + ljp;
                    const cpx<float> h = x_forward_out<float, N>(lds + l * C::LS, kx, BCX, twc);
                    __builtin_nontemporal_store(h.x, &W32[(2 * P) * N + kx]);
                    __builtin_nontemporal_store(h.y, &W32[(2 * P + 1) * N + kx]);
                }
            }
            __syncthreads();  // the next flush overwrites the lines
        }
        put_unit_sums<C::NT, 5>(acc, red, s.partial + (unsigned long long)tile * kPartialStride);
    }
}

template <int N>
constexpr bool outer_fusable_len() {
    if constexpr (N % 64 != 0) return false;
    else return OuterTile<N>::CPT == 1;
}

bool outer_fusable(const GridArgs& g) {
    bool ok = false;
    (void)dispatch_len(g.nx, [&]<int N>() {
        ok = outer_fusable_len<N>();
        return hipSuccess;
    });
    return ok;
}

hipError_t launch_outer_fused(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                              int* nunits, float share, bool write) {
    return dispatch_len(g.nx, [&]<int N>() {
        if constexpr (outer_fusable_len<N>()) {
            using C = LineCfg<float, N>;
            using Z = OuterTile<N>;
            const unsigned nt = (((unsigned)g.ny / 2 + Z::SUB - 1) / Z::SUB) * (((unsigned)g.nz + Z::KM - 1) / Z::KM);
            if (nunits) *nunits = (int)nt;
            return dispatch_op(g.coef, g.weight, [&]<int CO, int WE>() {
                return dispatch_bc(g.bcx, [&]<int BC>() {
                    const void* k = (const void*)&k_outer_resid_dhtx<N, CO, WE, BC>;
                    const int nb = persistent_grid(k, C::NT, nt, nslots, share);
                    k_outer_resid_dhtx<N, CO, WE, BC>
                        <<<dim3(nb, nslots), C::NT, reserve_lds(k, share), s>>>(g, slots, t, write ? 1 : 0);
                    return hipGetLastError();
                });
            });
        } else {
            return hipErrorInvalidValue;
        }
    });
}

}  // namespace pois
