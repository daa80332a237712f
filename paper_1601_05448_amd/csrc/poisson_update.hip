// The x-update sweep P5 (see poisson_sweeps.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_device.hpp"
#include "poisson_launch.hpp"

namespace pois {

// ---- P5: Hartley along x, update -----------------------------------------------
// MODE 0: FP64 p += dp - mean(p) (or FP32 d32 += dp); MODE 1: assign to p (L^+
// sweep); MODE 2: FP32 d32 = dp, the first inner sweep after a fused outer
// residual (d32 holds nothing yet).
// The FP32 x-update sweep on periodic rows of 256 is sized for four blocks per
// CU (what its LDS allows; 128 registers, no spills): it then loads the values
// it updates after the transform, their latency covered by the other blocks
// instead of a second register buffer.
template <typename T, int N, int BCX>
constexpr int update_min_waves() {
    return (sizeof(T) == 4 && N == 256 && BCX == 0) ? 4 : 1;
}

template <typename T, int N, int MODE, int BCX>
__global__ void __launch_bounds__((LineCfg<T, N>::NT), (update_min_waves<T, N, BCX>()))
k_dhtx_update(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage) {
    using C = LineCfg<T, N>;
    __shared__ cpx<T> lds[C::L * C::LS];
    __shared__ cpx<T> tw[N];
    const Slot& s = slots[blockIdx.y];
    if (MODE != 1 && IterView<T>::skip(s.st, stage)) return;
    // the update of the last inner evaluation is applied here: the next inner
    // residual sweep may run (no other block of this launch reads the flag)
    if constexpr (MODE == 0 && sizeof(T) == 4)
        if (blockIdx.x == 0 && threadIdx.x == 0) s.st->upd_due = 0;
    const cpx<T>* twg = twiddles<T>(tb, 0);
    const cpx<T>* twc = dct_twiddles<T>(tb);
    for (int e = threadIdx.x; e < N; e += C::NT) tw[e] = twg[e];
    const POIS_GLOBAL T* W = (MODE != 1) ? IterView<T>(s).W : (const POIS_GLOBAL T*)gptr(s.W);
    POIS_GLOBAL T* out;
    if constexpr (sizeof(T) == 8) out = (POIS_GLOBAL T*)gptr(s.p);
    else out = (POIS_GLOBAL T*)gptr(s.d32);
    const T shift = (MODE == 0 && sizeof(T) == 8) ? T(s.st->p_shift) : T(0);
    const unsigned nlines = (unsigned)(g.ny * g.nz / 2);
    const unsigned ngroups = (nlines + C::L - 1) / C::L;

    cpx<T> wb[C::IT], pb[C::IT];
    auto load_w = [&](unsigned grp) {
#pragma unroll
        for (int it = 0; it < C::IT; ++it) {
            const int e = threadIdx.x + it * C::NT;
            const unsigned P = grp * C::L + e / N;
            const int i = e % N;
            wb[it] = (P < nlines) ? cpx<T>{W[(2 * P) * N + i], W[(2 * P + 1) * N + i]} : cpx<T>{T(0), T(0)};
        }
    };
    unsigned grp = blockIdx.x;
    load_w(grp);
    while (true) {
#pragma unroll
        for (int it = 0; it < C::IT; ++it) {
            const int e = threadIdx.x + it * C::NT;
            lds[(e / N) * C::LS + C::pos(e % N)] = wb[it];
        }
        if constexpr (BCX != 0) {
            // cosine transform between walls: the FFT input pairs coefficient k
            // with coefficient N - k of the same line
            __syncthreads();
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                const int l = e / N, k = e % N;
                const cpx<T> cm = (k == 0) ? cpx<T>{T(0), T(0)} : lds[l * C::LS + C::pos(N - k)];
                wb[it] = idct_in(wb[it], cm, twc[k]);
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                lds[(e / N) * C::LS + C::pos(e % N)] = wb[it];
            }
        }
        // FP32: the values to update are loaded now and are in flight during the
        // FFT; FP64 has no registers to spare for them and loads them after it
        constexpr bool kEarly = MODE == 0 && sizeof(T) == 4 && update_min_waves<T, N, BCX>() == 1;
        if (kEarly) {
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                const unsigned P = grp * C::L + e / N;
                const int k = e % N;
                pb[it] = (P < nlines) ? cpx<T>{out[(2 * P) * N + k], out[(2 * P + 1) * N + k]} : cpx<T>{T(0), T(0)};
            }
        }
        const unsigned ng = grp + gridDim.x;
        __builtin_amdgcn_s_setprio(2);
        if (ng < ngroups) load_w(ng);
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        fft_block_lines<T, N>(lds, tw);
        if (MODE == 0 && !kEarly) {
#pragma unroll
            for (int it = 0; it < C::IT; ++it) {
                const int e = threadIdx.x + it * C::NT;
                const unsigned P = grp * C::L + e / N;
                const int k = e % N;
                pb[it] = (P < nlines) ? cpx<T>{out[(2 * P) * N + k], out[(2 * P + 1) * N + k]} : cpx<T>{T(0), T(0)};
            }
        }
#pragma unroll
        for (int it = 0; it < C::IT; ++it) {
            const int e = threadIdx.x + it * C::NT;
            const int l = e / N, k = e % N;
            const unsigned P = grp * C::L + l;
            if (P < nlines) {
                cpx<T> h;
                if constexpr (BCX != 0) {
                    const cpx<T> r = lds[l * C::LS + C::pos(x_slot(k, N, 1))];
                    h = {r.x, -r.y};
                } else {
                    h = hartley(lds[l * C::LS + C::pos(k)], lds[l * C::LS + C::pos((k == 0 ? 0 : N - k))]);
                }
                const unsigned a = (2 * P) * N + k, b = a + N;
                if (MODE == 0) {
                    out[a] = pb[it].x + h.x - shift;
                    out[b] = pb[it].y + h.y - shift;
                } else {
                    out[a] = h.x;
                    out[b] = h.y;
                }
            }
        }
        grp = ng;
        if (grp >= ngroups) break;
        __syncthreads();
    }
}

template <typename T, int MODE>
static hipError_t update_t(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                           float share, int stage) {
    const unsigned rows = (unsigned)(g.ny * g.nz / 2);
    return dispatch_len(g.nx, [&]<int N>() {
        using C = LineCfg<T, N>;
        const unsigned ng = (rows + C::L - 1) / C::L;
        return dispatch_bc(g.bcx, [&]<int BC>() {
            const void* k = (const void*)&k_dhtx_update<T, N, MODE, BC>;
            const int nb = persistent_grid(k, C::NT, ng, nslots, share);
            k_dhtx_update<T, N, MODE, BC><<<dim3(nb, nslots), C::NT, reserve_lds(k, share), s>>>(g, slots, t, stage);
            return hipGetLastError();
        });
    });
}

template <typename T>
hipError_t launch_update(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage) {
    if (mode == 1) return update_t<T, 1>(g, t, slots, nslots, s, share, stage);
    if constexpr (sizeof(T) == 4)
        if (stage == kStageTail) return update_t<T, 2>(g, t, slots, nslots, s, share, stage);
    return update_t<T, 0>(g, t, slots, nslots, s, share, stage);
}

template hipError_t launch_update<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                          int);
template hipError_t launch_update<float>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, int);

}  // namespace pois
