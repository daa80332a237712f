// Tiles of rows marched along z, and the transform along x of the lines they
// fill: shared by the residual sweep P1 (poisson_resid.hpp) and the fused outer
// residual (poisson_outer.hip).
#pragma once

#include "poisson_device.hpp"

namespace pois {

// Thread layout of a tile for rows of length N (16 and longer): SUB strips (row
// pairs) of MT threads, each thread CPT columns of its strip's pair, MT apart.  About
// 256 threads; small tiles (not WIDE) of rows longer than 64 the fewest strips that fill
// whole waves.  (On shorter rows one wave alone had a quarter of its lanes busy in the
// transform of its two planes' lines, which a batch of solves pays for: 64 served FP32
// solves of 64^3 4.79 ms, with four waves of strips, whose lines fill one of them, 4.48.)
template <int N, bool WIDE>
struct RowTile {
    static_assert(N >= 16, "shorter rows are gathered");
    static constexpr int CPT = N > 512 ? 2 : 1;
    static constexpr int MT = N / CPT;
    static constexpr int WHOLE = N % 64 == 0 ? 1 : N % 32 == 0 ? 2 : N % 16 == 0 ? 4 : 8;  // strips of whole waves
    static constexpr int SUB = MT >= 192 || (!WIDE && N > 64) ? WHOLE : N == 96 ? 2 : N % 3 == 0 ? 192 / N : 256 / N;
    static constexpr int NT = SUB * MT;
    static constexpr bool DPP = N % 64 == 0;                  // x neighbours from the neighbouring lanes
    static constexpr int XV = DPP ? (N / 64) * 2 : N;         // exchanged PlaneRows per strip and plane
    static_assert(NT % 64 == 0 && NT <= 512, "whole waves");
};

// Transforms the L = SUB KF lines of a tile along x, line q SUB + s for strip s of
// plane q, in place in LDS (element i of a row written to pos(x_slot(i))), and
// hands out(q, c, h) the transformed pair of column c of the thread's own strip.
// NT threads; every thread calls it after a barrier; it ends on LDS reads.
template <typename F, int N, int SET, int SUB, int KF, int CPT, class Out>
__device__ __forceinline__ void transform_rows(cpx<F>* lds, const cpx<F>* tw, int bcx, const cpx<F>* twc, int sidx,
                                               unsigned col0, Out&& out_fn) {
    using LF = LineFft<F, N, true, SET>;
    constexpr int MT = N / CPT, NT = SUB * MT, L = SUB * KF, CL = NT / LF::TT;
    const int line0 = (int)threadIdx.x / LF::TT, t = (int)threadIdx.x % LF::TT;
#pragma unroll
    for (int r0 = 0; r0 < L; r0 += CL) {
        const bool on = (CL * LF::TT == NT || line0 < CL) && ((r0 + CL <= L) || r0 + line0 < L);
        cpx<F>* ln = lds + (on ? r0 + line0 : 0) * LF::LS;
        cpx<F> v[LF::E];
#pragma unroll
        for (int a = 0; a < LF::E; ++a) v[a] = ln[LF::pos(t + a * LF::TT)];
        __syncthreads();
        typename LF::Out o;
        LF::forward(v, ln, t, tw, o, on);
        __syncthreads();
        if (on) LF::put(o, ln, t);
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int k = (int)col0 + c * MT;
        const cpx<F>* zk = lds + sidx * LF::LS + LF::pos(k);
        const cpx<F>* zm = lds + sidx * LF::LS + LF::pos(N - k);
        const cpx<F> w = bcx ? twc[k] : cpx<F>{F(1), F(0)};
#pragma unroll
        for (int q = 0; q < KF; ++q) {
            const cpx<F> a = zk[q * SUB * LF::LS], b = zm[q * SUB * LF::LS];
            out_fn(q, c, bcx ? dct_out(a, b, w) : hartley(a, b));
        }
    }
}

// Planes per flush of a wide tile of a T residual, and the plan of its lines: as
// many lines as the threads transform at once, 16 planes of FP64 rows of 256 and
// 512 (512^3: 934 us; 8 planes and eight values per thread 990), else 8 (FP32 at
// 512^3: 463 us against 520, on 512 x 256 x 256 118 against 140).
template <typename T, int N>
struct RowFlush {
    static constexpr bool BIG = sizeof(T) == 8 && (N == 256 || N == 512);
    static constexpr int KF = BIG ? 16 : 8, SET = BIG ? 2 : 1;
};

// Flushes of `kf` planes per wide tile (so that the two halo planes are shared by
// more planes), up to `most` planes, that give the fewest plane steps over the
// rounds of tiles the resident blocks take: 192^3 in FP64 takes 8 planes (61 us),
// not 32 (80 us: 512 of 576 tiles in a first round).
inline int pick_flushes(int kf, int most, unsigned strips, unsigned nz, unsigned resident) {
    const unsigned all = (nz + (unsigned)kf - 1) / (unsigned)kf;
    int best = 1;
    double cost = 0.0;
    for (unsigned f = 1; (int)f * kf <= most && f <= all; f *= 2) {
        const unsigned tiles = strips * ((all + f - 1) / f), rounds = (tiles + resident - 1) / resident;
        const double c = (double)rounds * (f * (unsigned)kf + 3.0);  // three more plane loads open a tile
        if (f == 1 || c < cost) {
            cost = c;
            best = (int)f;
        }
    }
    return best;
}

// Planes of a small tile.
constexpr int kSmallPlanes = 2;

// Whether a sweep takes its small tiles (all loads at once): where they all fit on
// the chip at once, so that the sweep lasts one block's chain (the sweep alone, 64^3
// in FP64: 6.3 us, marching 11.0; 96^3, more than one round: 17.5 against 12.3).
inline bool small_tiles_fit(unsigned tiles, unsigned resident) { return tiles <= resident; }

}  // namespace pois
