// The x-update sweep P5 (see poisson_sweeps.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_device.hpp"
#include "poisson_launch.hpp"

namespace pois {

// ---- P5: Hartley along x, update -----------------------------------------------
// mode 0: FP64 p += dp - mean(p) (or FP32 d32 += dp); 1: assign to p or d32 (L^+
// sweep); 2: FP32 d32 = dp, the first inner sweep after a fused outer residual
// (d32 holds nothing yet).
//
// A block holds L row pairs.  Periodic rows start their transform from registers:
// thread t of a line loads the values t + a TT itself, so the rows pass LDS only
// between the stages and once at the end, where the threads change from the
// transform's order to whole rows for the (k, N - k) partners and the update.
// Between walls the input pairs coefficient k with N - k, so the rows come in
// through LDS.  The next group's rows and this group's values to update are in
// flight during the transform.
template <typename T, int N, int BCX, bool WIDE>
struct UpdateShape {
    using F = LineFft<T, N, true, 1>;
    // threads: about 256, or the fewest whole waves that whole lines fill; 512 on
    // periodic rows of 512 (512^3 FP64: 605 us, with 256 threads 625; between walls
    // the other way, 512 x 256 x 256: 182 and 150)
    static constexpr int WHOLE = N % 3 == 0 ? 192 : 64;
    static constexpr int NT = !WIDE || WHOLE == 192 ? WHOLE : N == 512 && !BCX ? 512 : 256;
    static constexpr int L = NT / F::TT;
    static constexpr int IT = L * N / NT;  // values per thread
    static constexpr bool EARLY = N < 256 || !WIDE;  // see loads_issued
    static_assert(NT % 64 == 0 && L * F::TT == NT && (NT % N == 0 || N % NT == 0), "whole lines and rows");
};

template <typename T, int N, int BCX, bool WIDE>
__global__ void __launch_bounds__((UpdateShape<T, N, BCX, WIDE>::NT), (sizeof(T) == 4 ? (BCX ? 3 : 4) : 2))
k_dhtx_update(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage, int mode) {
    using U = UpdateShape<T, N, BCX, WIDE>;
    using F = typename U::F;
    constexpr int NT = U::NT, L = U::L, IT = U::IT;
    __shared__ cpx<T> lds[L * F::LS];
    __shared__ cpx<T> tw[N];
    const Slot& s = slots[blockIdx.y];
    if constexpr (!U::EARLY)
        if (mode != 1 && IterView<T>::skip(s.st, stage)) return;
    const cpx<T>* twc = dct_twiddles<T>(tb);
    TwiddleLoad<T, N, NT> twl;
    twl.load(twiddles<T>(tb, 0));
    const POIS_GLOBAL T* W = (mode != 1) ? IterView<T>(s).W : (const POIS_GLOBAL T*)gptr(s.W);
    POIS_GLOBAL T* out;
    if constexpr (sizeof(T) == 8) out = (POIS_GLOBAL T*)gptr(s.p);
    else out = (POIS_GLOBAL T*)gptr(s.d32);
    const T shift = (mode == 0 && sizeof(T) == 8) ? T(s.st->p_shift) : T(0);
    const unsigned nlines = (unsigned)(g.ny * g.nz / 2);
    const unsigned ngroups = (nlines + L - 1) / L;

    // value `it` of this thread in whole rows: line row_l(it), column row_k(it)
    constexpr int RK = NT % N == 0 ? 1 : N / NT;
    const int tk = (int)threadIdx.x % N, tl = (int)threadIdx.x / N;
    auto row_l = [&](int it) { return RK == 1 ? tl + it * (NT / N) : it / RK; };
    auto row_k = [&](int it) { return RK == 1 ? tk : (int)threadIdx.x + (it % RK) * NT; };
    const int line = (int)threadIdx.x / F::TT, t = (int)threadIdx.x % F::TT;
    cpx<T>* ln = lds + line * F::LS;

    cpx<T> wb[BCX ? IT : F::E];
    // a line past the end loads line 0 and is not stored
    auto load_w = [&](unsigned grp) {
        if constexpr (BCX != 0) {
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const unsigned P = grp * L + row_l(it), at = (2 * (P < nlines ? P : 0u)) * N + row_k(it);
                wb[it] = cpx<T>{W[at], W[at + N]};
            }
        } else {
            const unsigned P = grp * L + line, at = (2 * (P < nlines ? P : 0u)) * N + t;
#pragma unroll
            for (int a = 0; a < F::E; ++a) wb[a] = cpx<T>{W[at + a * F::TT], W[at + N + a * F::TT]};
        }
    };
    unsigned grp = blockIdx.x;
    load_w(grp);
    if constexpr (U::EARLY) {
        loads_issued();
        if (mode != 1 && IterView<T>::skip(s.st, stage)) return;
    }
    // the update of the last inner evaluation is applied here: the next inner
    // residual sweep may run (no other block of this launch reads the flag)
    if constexpr (sizeof(T) == 4)
        if (mode == 0 && blockIdx.x == 0 && threadIdx.x == 0) s.st->upd_due = 0;
    twl.store(tw);
    __syncthreads();  // twiddles
    while (true) {
        cpx<T> v[F::E];
        if constexpr (BCX != 0) {
            // cosine transform between walls: the FFT input pairs coefficient k
            // with coefficient N - k of the same line
#pragma unroll
            for (int it = 0; it < IT; ++it) lds[row_l(it) * F::LS + F::pos(row_k(it))] = wb[it];
            __syncthreads();
#pragma unroll
            for (int a = 0; a < F::E; ++a) {
                const int k = t + a * F::TT;
                const cpx<T> c = ln[F::pos(k)], cm = (k == 0) ? cpx<T>{T(0), T(0)} : ln[F::pos(N - k)];
                v[a] = idct_in(c, cm, twc[k]);
            }
            __syncthreads();
        } else {
#pragma unroll
            for (int a = 0; a < F::E; ++a) v[a] = wb[a];
        }
        // the values to update and the next group's rows, in flight during the FFT
        cpx<T> pb[IT];
        __builtin_amdgcn_s_setprio(2);
        if (mode == 0) {
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const unsigned P = grp * L + row_l(it), at = (2 * (P < nlines ? P : 0u)) * N + row_k(it);
                pb[it] = cpx<T>{out[at], out[at + N]};
            }
        }
        const unsigned ng = grp + gridDim.x;
        if (ng < ngroups) load_w(ng);
        __builtin_amdgcn_s_setprio(0);
        typename F::Out o;
        F::forward(v, ln, t, tw, o);
        __syncthreads();  // the last stage's reads before its outputs
        F::put(o, ln, t);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const unsigned P = grp * L + row_l(it);
            if (P < nlines) {
                const cpx<T>* row = lds + row_l(it) * F::LS;
                const int k = row_k(it);
                cpx<T> h;
                if constexpr (BCX != 0) {
                    const cpx<T> r = row[F::pos((int)x_slot(k, N, 1))];
                    h = {r.x, -r.y};
                } else {
                    h = hartley(row[F::pos(k)], row[F::pos(N - k)]);
                }
                const unsigned a = (2 * P) * N + k, b = a + N;
                if (mode == 0) {
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
    // the rest of a fused first inner sweep ends here: the inner sweeps go on
    if constexpr (sizeof(T) == 4)
        if (mode == 2 && last_block(s) && threadIdx.x == 0) s.st->stage = 1;
}

template <typename T>
hipError_t launch_update(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage) {
    const unsigned rows = (unsigned)(g.ny * g.nz / 2);
    const int m = mode == 1 ? 1 : sizeof(T) == 4 && stage == kStageTail ? 2 : 0;
    return dispatch_len(g.nx, [&]<int N>() {
        auto run = [&](auto kernel, int nt, int lines) {
            const void* k = (const void*)kernel;
            const int nb = persistent_grid(k, nt, (rows + lines - 1) / lines, nslots, share);
            kernel<<<dim3(nb, nslots), nt, reserve_lds(k, share), s>>>(g, slots, t, stage, m);
            return hipGetLastError();
        };
        return dispatch_bc(g.bcx, [&]<int BC>() {
            using Wide = UpdateShape<T, N, BC, true>;
            using Narrow = UpdateShape<T, N, BC, false>;
            if constexpr (Wide::NT != Narrow::NT)
                if ((rows + Wide::L - 1) / Wide::L < kWideGroups)
                    return run(&k_dhtx_update<T, N, BC, false>, Narrow::NT, Narrow::L);
            return run(&k_dhtx_update<T, N, BC, true>, Wide::NT, Wide::L);
        });
    });
}

template hipError_t launch_update<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                          int);
template hipError_t launch_update<float>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, int);

}  // namespace pois
