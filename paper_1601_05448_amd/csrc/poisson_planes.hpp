// The y, z and y sweeps P2 - P3 - P4 of small grids as one launch (see
// poisson_sweeps.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_columns.hpp"

namespace pois {

// Between the two x transforms every complex column m is a problem of its own:
// Hartley along y, along z, the symbol, and back, on the NZ x NY plane of its
// values.  Small planes fit the LDS of one block (37 KB at 48 x 48 in FP64), which
// loads it, does all three sweeps there and stores it: the same transforms on the
// same lines as k_dht_cols and k_dht_z_solve, which give the same bits, with two
// launches and two round trips through memory fewer (32^3: 7.6 us; 3.3-4.0 each).
// What bounds it is the chain of one block - one load, five transforms and their
// barriers, one store - and the plane's column access (16 or 8 bytes per row of
// nxh): neighbouring columns, which share those cache lines, run on one XCD.
template <typename T, int NY, int NZ>
struct PlaneShape {
    using FY = LineFft<T, NY, false>;
    using FZ = LineFft<T, NZ, false>;
    static constexpr int USED = NZ * FY::TT > NY * FZ::TT ? NZ * FY::TT : NY * FZ::TT;
    static constexpr int NT = (USED + 63) / 64 * 64;
    static constexpr int LDS = NZ * FY::LS > NY * FZ::LS ? NZ * FY::LS : NY * FZ::LS;
};

template <typename T, int NY, int NZ>
__global__ void __launch_bounds__((PlaneShape<T, NY, NZ>::NT), 1)
k_dht_planes(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage, int mode) {
    using S = PlaneShape<T, NY, NZ>;
    using FY = typename S::FY;
    using FZ = typename S::FZ;
    constexpr int NT = S::NT;
    __shared__ cpx<T> lds[S::LDS];
    __shared__ cpx<T> twy[NY], twz[NZ];
    __shared__ T lzs[NZ / 2 + 1];  // the scaled z symbol, even in k
    const Slot& s = slots[blockIdx.y];
    TwiddleLoad<T, NY, NT> twly;
    TwiddleLoad<T, NZ, NT> twlz;
    twly.load(twiddles<T>(tb, 1));
    twlz.load(twiddles<T>(tb, 2));
    POIS_GLOBAL T* Wc = mode == 0 ? IterView<T>(s).W : (POIS_GLOBAL T*)gptr(s.W);  // complex-indexed
    const unsigned nxh = g.nxh;
    const T* lamx = symbol<T>(tb, 0);
    const T sc = symbol_scale<T>(g);
    const T kn = T(g.n) / sc;  // exact: sc is a power of two
    // y lines: one per z; z lines: one per y.  Threads without a line only take
    // part in the barriers (their loads are line 0's).
    const int zl = threadIdx.x % NZ, yl = threadIdx.x % NY;
    const bool ony = (int)threadIdx.x < NZ * FY::TT, onz = (int)threadIdx.x < NY * FZ::TT;
    const int ty = ony ? threadIdx.x / NZ : 0, tz = onz ? threadIdx.x / NY : 0;
    cpx<T>* lny = lds + zl * FY::LS;
    cpx<T>* lnz = lds + yl * FZ::LS;
    const unsigned off = ((unsigned)zl * NY + (unsigned)ty) * nxh;
    cpx<T> vy[FY::E];
    auto load = [&](unsigned m) {
#pragma unroll
        for (int a = 0; a < FY::E; ++a) vy[a] = gload_c(Wc, m + off + (unsigned)(a * FY::TT) * nxh);
    };
    unsigned m = xcd_block(blockIdx.x, gridDim.x);
    load(m);
    loads_issued();
    if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    twly.store(twy);
    twlz.store(twz);
    for (int e = threadIdx.x; e <= NZ / 2; e += NT) lzs[e] = symbol<T>(tb, 2)[e] * sc;
    const T lyj = symbol<T>(tb, 1)[yl];
    while (true) {
        const T lxe = lamx[2 * m], lxo = lamx[2 * m + 1];
        const T ta0 = (lxe + lyj) * sc, tb0 = (lxo + lyj) * sc;
        __syncthreads();  // twiddles, symbol; the last plane's reads
        typename FY::Out oy;
        typename FZ::Out oz;
        FY::forward(vy, lny, ty, twy, oy, ony);
        __syncthreads();  // the last stage's reads before its outputs
        if (ony) FY::put(oy, lny, ty);
        __syncthreads();
        // the z lines' inputs: Hartley along y of each row, from its outputs k and NY - k
        cpx<T> vz[FZ::E];
#pragma unroll
        for (int a = 0; a < FZ::E; ++a) {
            const cpx<T>* row = lds + (tz + a * FZ::TT) * FY::LS;
            vz[a] = hartley(row[FY::pos(yl)], row[FY::pos(NY - yl)]);
        }
        __syncthreads();
        FZ::forward(vz, lnz, tz, twz, oz, onz);
        __syncthreads();
        if (onz) FZ::put(oz, lnz, tz);
        __syncthreads();
        // scaled spectra of the pairs (k, NZ - k), conjugated (see k_dht_z_solve)
#pragma unroll
        for (int a = 0; a < FZ::E; ++a) {
            const int k = tz + a * FZ::TT;
            const T lzk = lzs[k <= NZ / 2 ? k : NZ - k];
            T hp, hm;
            if (a == 0) {
                pair_coefs0(ta0 + lzk, tb0 + lzk, kn, hp, hm);
            } else {
                const T sa = recip(kn * (ta0 + lzk)), sb = recip(kn * (tb0 + lzk));
                hp = T(0.5) * (sa + sb);
                hm = T(0.5) * (sa - sb);
            }
            vz[a] = scaled_conj_h(lnz[FZ::pos(k)], lnz[FZ::pos(NZ - k)], hp, hm);
        }
        __syncthreads();
        FZ::forward(vz, lnz, tz, twz, oz, onz);
        __syncthreads();
        if (onz)
            FZ::each(oz, tz, [&](int j, int dk, cpx<T> z) { lds[(j + dk) * FY::LS + yl] = cpx<T>{z.x, -z.y}; });
        __syncthreads();
        // the y lines' inputs, in natural order
#pragma unroll
        for (int a = 0; a < FY::E; ++a) vy[a] = lny[ty + a * FY::TT];
        __syncthreads();
        FY::forward(vy, lny, ty, twy, oy, ony);
        __syncthreads();
        if (ony) FY::put(oy, lny, ty);
        __syncthreads();
        if (ony) {
            const unsigned base = m + (unsigned)(zl * NY) * nxh;
            FY::each_pair(oy, lny, ty, [&](int j, int dk, cpx<T> z, cpx<T> zm) {
                gstore_c(Wc, base + (unsigned)(j + dk) * nxh, hartley(z, zm));
            });
        }
        m += gridDim.x;
        if (m >= nxh) break;
        load(m);
    }
}

template <class F>
static hipError_t plane_len(int n, F&& f) {
    switch (n) {
        case 16: return f.template operator()<16>();
        case 24: return f.template operator()<24>();
        case 32: return f.template operator()<32>();
        case 48: return f.template operator()<48>();
        case 64: return f.template operator()<64>();
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_planes(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage) {
    return plane_len(g.ny, [&]<int NY>() {
        return plane_len(g.nz, [&]<int NZ>() {
            if constexpr (NY * NZ > 48 * 48) {  // see planes_fusable
                return hipErrorInvalidValue;
            } else {
                const void* k = (const void*)&k_dht_planes<T, NY, NZ>;
                constexpr int nt = PlaneShape<T, NY, NZ>::NT;
                const int nb = persistent_grid(k, nt, (unsigned)g.nxh, nslots, share);
                k_dht_planes<T, NY, NZ><<<dim3(nb, nslots), nt, reserve_lds(k, share), s>>>(g, slots, t, stage, mode);
                return hipGetLastError();
            }
        });
    });
}

}  // namespace pois
