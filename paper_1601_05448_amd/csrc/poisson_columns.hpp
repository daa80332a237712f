// The y and z sweeps P2 (= P4) and P3 (see poisson_sweeps.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "poisson_device.hpp"
#include "poisson_launch.hpp"

namespace pois {

// ---- P2 / P4: Hartley along y of the pair-packed columns ------------------------
// Line = (o, m): complex column m (real columns 2m, 2m+1) at outer index o;
// element e along the axis.  y: address (o*ny + e)*nxh + m; z: (e*ny + o)*nxh + m.
// Thread t of a block always works on line t % L of the group.
template <int AX>
__device__ __forceinline__ unsigned col_base(const GridArgs& g, unsigned line) {
    const unsigned nxh = g.nxh, o = line / nxh, m = line - o * nxh;
    return (AX == 1) ? o * (unsigned)g.ny * nxh + m : o * nxh + m;
}

// Lines of 256 and 512 whose groups fill the chip run in the register kernels
// (k_dht_cols_regs, k_dht_z_solve_regs); every other line in the kernels on
// FftPlan lines below.  Both are bound by memory on large grids and by the chain
// of loads, LDS passes and barriers of one line group on small ones.  Against
// stages that start and end in LDS (MI355X, start -> now, us): FP32 y / z sweep
// of 384^3 108 -> 61 / 162 -> 91 (7.5 / 5.0 TB/s), of 192^3 13.2 -> 10.1 / 19.4 -> 14.3; FP64
// z sweep of 192^3 36 -> 25, of 32^3 8.4 -> 4.2; FP64 y sweep of 768 x 768 x 256
// 813 -> 502.  (On 512 lines the FftPlan form is slower than the register
// kernels: FP64 y 488 us against 421 at 512^3; at 256 it is within 5%.)
//
// Lines per block of the column sweeps on FftPlan lines.  Wide: about 256
// threads and runs of at least 128 bytes per row (8 FP64 or 16 FP32 complex
// values; 8 on FP32 lines of 768 and 1024, whose 1024-thread blocks would spill).
// Narrow: one to four waves, for grids whose wide line groups would not give every CU
// two blocks (kWideGroups): such sweeps are bound by the
// latency of one block's chain of loads, transposes and stores, and more, smaller
// blocks spread the same lines over more CUs.
template <typename T, int N>
constexpr int wide_lines() {
    constexpr int tt = FftPlan<N>::TT, run = sizeof(T) == 8 || tt >= 64 ? 8 : 16;
    return 256 / tt > run ? 256 / tt : run;
}
template <typename T, int N>
constexpr int narrow_lines() {
    constexpr int tt = FftPlan<N>::TT, run = sizeof(T) == 8 || tt >= 64 ? 8 : 16;
    return 64 / tt > run ? 64 / tt : run;
}

template <typename T, int N, int L>
struct ColShape {
    using F = LineFft<T, N, false>;
    static constexpr int NT = L * F::TT;
    // waves per SIMD the registers are sized for: two, or what the LDS of a CU
    // (163840 bytes; lines, twiddles, half a symbol table) has room for
    static constexpr int LDS = L * F::LS * (int)sizeof(cpx<T>) + N * (int)sizeof(cpx<T>) + (N / 2 + 1) * (int)sizeof(T);
    static constexpr int FIT = 163840 / LDS * NT / 256;
    // Groups narrower than a 128-byte cache line: neighbouring groups, which share
    // the lines, go to one XCD's L2 (FP32 y sweep of 1024 x 1024 x 64: 133 -> 102 us).
    // Wider groups stay dealt round-robin (192^3, FP32 y: 10.2 us, renumbered 14.5).
    static __device__ __forceinline__ unsigned first_group(unsigned b, unsigned nb) {
        return L * (int)sizeof(cpx<T>) < 128 ? xcd_block(b, nb) : b;
    }
    static constexpr int MINW = NT > 512 ? NT / 256 : FIT < 1 ? 1 : FIT > 2 ? 2 : FIT;
    static constexpr bool EARLY = N < 256 || L == narrow_lines<T, N>();  // see loads_issued
};

template <typename T, int N, int L>
__global__ void __launch_bounds__((ColShape<T, N, L>::NT), (ColShape<T, N, L>::MINW))
k_dht_cols(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage, int mode) {
    using F = LineFft<T, N, false>;
    constexpr int NT = ColShape<T, N, L>::NT;
    __shared__ cpx<T> lds[L * F::LS];
    __shared__ cpx<T> tw[N];
    const Slot& s = slots[blockIdx.y];
    if constexpr (!ColShape<T, N, L>::EARLY)
        if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    TwiddleLoad<T, N, NT> twl;
    twl.load(twiddles<T>(tb, 1));
    POIS_GLOBAL T* Wc = mode == 0 ? IterView<T>(s).W : (POIS_GLOBAL T*)gptr(s.W);  // complex-indexed
    const unsigned nlines = (unsigned)(g.nxh * g.nz), ngroups = (nlines + L - 1) / L;
    const unsigned se = (unsigned)g.nxh;
    const int l = threadIdx.x % L, t = threadIdx.x / L;
    const unsigned lane_off = (unsigned)t * se;
    cpx<T>* ln = lds + l * F::LS;
    cpx<T> buf[F::E];
    // a line past the end (in the last group) loads line 0 and is not stored
    auto load = [&](unsigned grp, bool& valid, unsigned& base) {
        const unsigned line = grp * L + l;
        valid = line < nlines;
        base = valid ? col_base<1>(g, line) : 0u;
#pragma unroll
        for (int a = 0; a < F::E; ++a) buf[a] = gload_c(Wc, base + lane_off + (unsigned)(a * F::TT) * se);
    };
    unsigned grp = ColShape<T, N, L>::first_group(blockIdx.x, gridDim.x), base;
    bool valid;
    load(grp, valid, base);
    if constexpr (ColShape<T, N, L>::EARLY) {
        loads_issued();
        if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    }
    twl.store(tw);
    __syncthreads();  // twiddles
    while (true) {
        cpx<T> v[F::E];
#pragma unroll
        for (int a = 0; a < F::E; ++a) v[a] = buf[a];
        const bool cur_valid = valid;
        const unsigned cur_base = base;
        const unsigned ng = grp + gridDim.x;
        __builtin_amdgcn_s_setprio(2);
        if (ng < ngroups) load(ng, valid, base);  // in flight during the FFT
        __builtin_amdgcn_s_setprio(0);
        typename F::Out out;
        F::forward(v, ln, t, tw, out);
        __syncthreads();  // the last stage's reads before its outputs
        F::put(out, ln, t);
        __syncthreads();
        if (cur_valid) {
            F::each_pair(out, ln, t, [&](int j, int dk, cpx<T> z, cpx<T> zm) {
                gstore_c(Wc, cur_base + (unsigned)j * se + (unsigned)dk * se, hartley(z, zm));
            });
        }
        grp = ng;
        if (grp >= ngroups) break;
        __syncthreads();
    }
}

// Lines of 256 and 512 held in registers (fft256_regs, fft512_regs).
template <typename T, int N>
__global__ void __launch_bounds__((LineCfg<T, N>::NT), (LineCfg<T, N>::MINB))
k_dht_cols_regs(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage, int mode) {
    using C = LineCfg<T, N>;
    __shared__ cpx<T> lds[C::L * C::LS];
    __shared__ cpx<T> tw[N];
    const Slot& s = slots[blockIdx.y];
    if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    TwiddleLoad<T, N, C::NT> twl;
    twl.load(twiddles<T>(tb, 1));
    POIS_GLOBAL T* Wc = mode == 0 ? IterView<T>(s).W : (POIS_GLOBAL T*)gptr(s.W);  // complex-indexed
    const unsigned nlines = (unsigned)(g.nxh * g.nz);
    const unsigned ngroups = (nlines + C::L - 1) / C::L;
    const unsigned se = (unsigned)g.nxh;
    static_assert(C::L == 16, "16 lines per block (reg_col)");
    const int l = threadIdx.x % C::L;
    const int e0 = reg_col<N>((int)threadIdx.x / 16);

    // element e0 + it TT of a line at base + e0 se + (it TT) se: the lane's part
    // in one register, the rest wave-uniform (no per-element address registers
    // live across the transform).  A line past the end (in the last group)
    // loads line 0 and is not stored: no branch per element.
    const unsigned lane_off = (unsigned)e0 * se;
    cpx<T> buf[C::IT];
    auto load = [&](unsigned grp, bool& valid, unsigned& base) {
        const unsigned line = grp * C::L + l;
        valid = line < nlines;
        base = valid ? col_base<1>(g, line) : 0u;
#pragma unroll
        for (int it = 0; it < C::IT; ++it) buf[it] = gload_c(Wc, base + lane_off + (unsigned)(it * C::TT) * se);
    };
    unsigned grp = blockIdx.x, base;
    bool valid;
    load(grp, valid, base);
    twl.store(tw);
    // the line stays in registers; LDS only for the transpose of the
    // transform and the exchange of the (k, N-k) partners, which stays
    // within the wave (reg_col, exchange_write)
    __syncthreads();  // twiddles
    cpx<T>* ln = lds + l * C::LS;
    while (true) {
        cpx<T> v[16];
#pragma unroll
        for (int a = 0; a < 16; ++a) v[a] = buf[a];
        const bool cur_valid = valid;
        const unsigned cur_base = base;
        const unsigned ng = grp + gridDim.x;
        __builtin_amdgcn_s_setprio(2);
        if (ng < ngroups) load(ng, valid, base);  // in flight during the FFT
        __builtin_amdgcn_s_setprio(0);
        // the column, opaque within each group: the lane-dependent
        // addresses derived from it are formed here rather than held in
        // registers across the loop
        int c = e0;
        asm volatile("" : "+v"(c));
        if constexpr (N == 256) fft256_regs<T>(v, ln, c, tw);
        else fft512_regs<T>(v, ln, c, tw);
        exchange_write<T, N>(ln, c, v);
        wave_lds_sync();
        if (cur_valid) {
            const cpx<T>* pp = exchange_partner<T, N>(ln, c);
            // k = kb + 16 b
            const unsigned kb = N == 256 ? (unsigned)c : (unsigned)((c >> 1) + 256 * (c & 1));
            const unsigned st_base = cur_base + kb * se;
#pragma unroll
            for (int b = 0; b < 16; ++b)
                gstore_c(Wc, st_base + (unsigned)(16 * b) * se, hartley(v[b], pp[17 * (15 - b)]));
        }
        grp = ng;
        if (grp >= ngroups) break;
        // N = 256: the next transpose writes this thread's own column, read
        // only by its wave; N = 512: it writes every wave's positions
        if constexpr (N == 256) wave_lds_sync();
        else __syncthreads();
    }
}

// ---- P3: Hartley along z, divide by n * symbol, Hartley along z ----------------
// The z symbol is even in k_z, so Hartley-scale-Hartley equals an FFT, a scaling
// of each packed row's spectrum, and an inverse FFT: the two rows of a pair
// (x wavenumbers 2m and 2m+1, symbols s_a and s_b) are separated as
// A_k = (Z_k + conj Z_{N-k})/2 and i B_k = (Z_k - conj Z_{N-k})/2, so the scaled
// spectrum is Z'_k = (s_a + s_b)/2 Z_k + (s_a - s_b)/2 conj Z_{N-k}; the inverse is
// taken as conj(FFT(conj Z')), which needs no exchange of (k, N-k) partners.
template <typename T>
__device__ __forceinline__ cpx<T> scaled_conj_h(cpx<T> zk, cpx<T> zm, T hp, T hm) {
    return {hp * zk.x + hm * zm.x, hm * zm.y - hp * zk.y};  // conj(hp Z_k + hm conj Z_{N-k})
}

// The register paths take hp = (s_a + s_b)/2 and hm = (s_a - s_b)/2 with one
// reciprocal per wavenumber instead of two.  The symbols are scaled by a power
// of two sc (exact, and the product of two of them then stays in range): with
// ta = sc lam_a, tb = sc lam_b and kn = n / sc, s_a = 1 / (n lam_a) = 1 / (kn ta)
// and
//     hp = (ta + tb) / (2 kn ta tb),   hm = (tb - ta) / (2 kn ta tb).
// Only the constant mode has a zero symbol; the one value per thread that may
// hold it takes pair_coefs0, which inverts each symbol on its own (0 for 0).
template <typename T>
__device__ __forceinline__ void pair_coefs(T ta, T tb, T dt, T kn2, T& hp, T& hm) {
    const T r = recip(ta * tb * kn2);
    hp = (ta + tb) * r;
    hm = dt * r;
}
template <typename T>
__device__ __forceinline__ void pair_coefs0(T ta, T tb, T kn, T& hp, T& hm) {
    const T sa = ta == T(0) ? T(0) : recip(kn * ta), sb = tb == T(0) ? T(0) : recip(kn * tb);
    hp = T(0.5) * (sa + sb);
    hm = T(0.5) * (sa - sb);
}
// sc = 2^-e, with every symbol's magnitude (at most 4 (1/hx^2 + 1/hy^2 + 1/hz^2))
// below 2^e
template <typename T>
__device__ __forceinline__ T symbol_scale(const GridArgs& g) {
    int e;
    (void)frexp(4.0 * (g.ihx2 + g.ihy2 + g.ihz2), &e);
    e = e < -120 ? -120 : (e > 120 ? 120 : e);
    return T(ldexp(1.0, -e));
}

// Launch shape of the z sweep's register paths: PF whether the next line group
// is loaded during this one's transforms, MINW the waves per SIMD its registers
// are sized for (the second __launch_bounds__ argument).  Measured (MI355X): the
// FP32 256-point path runs four blocks per CU with the prefetch (111 registers);
// the FP32 512-point path runs two 512-thread blocks per CU without it (no
// spills; 14% faster than one block with it); the FP64 paths prefetch (no spills
// at 2 and 1 blocks per CU).
template <typename T, int N>
struct ZRegsCfg {
    static constexpr bool PF = !(sizeof(T) == 4 && N == 512);
    static constexpr int MINW = sizeof(T) == 4 ? 4 : LineCfg<T, N>::MINB;
};

template <typename T, int N, bool PF, int MINW>
__global__ void __launch_bounds__((LineCfg<T, N>::NT), (MINW))
k_dht_z_solve_regs(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage, int mode) {
    using C = LineCfg<T, N>;
    __shared__ cpx<T> lds[C::L * C::LS];
    __shared__ cpx<T> tw[N];
    // the z symbol of the register path, in LDS: a global load of it after the
    // next group's prefetch would make the wait for it a wait for the prefetch
    __shared__ T lzs[N];
    const Slot& s = slots[blockIdx.y];
    if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    const cpx<T>* twg = twiddles<T>(tb, 2);
    for (int e = threadIdx.x; e < N; e += C::NT) tw[e] = twg[e];
    const T sc = symbol_scale<T>(g);
    for (int e = threadIdx.x; e < N; e += C::NT) lzs[e] = symbol<T>(tb, 2)[e] * sc;
    POIS_GLOBAL T* Wc = mode == 0 ? IterView<T>(s).W : (POIS_GLOBAL T*)gptr(s.W);  // complex-indexed
    const unsigned nlines = (unsigned)(g.nxh * g.ny);
    const unsigned ngroups = (nlines + C::L - 1) / C::L;
    const unsigned se = (unsigned)(g.nxh * g.ny);
    static_assert(C::L == 16, "16 lines per block (reg_col)");
    const int l = threadIdx.x % C::L;
    const int e0 = reg_col<N>((int)threadIdx.x / 16);
    const T* lamx = symbol<T>(tb, 0);
    const T* lamy = symbol<T>(tb, 1);
    const T nn = T(g.n);
    const T kn = nn / sc, kn2 = T(2) * kn;  // exact: sc is a power of two

    // element e0 + it TT of a line at base + e0 se + (it TT) se; a line past
    // the end loads line 0 and is not stored (see k_dht_cols)
    const unsigned lane_off = (unsigned)e0 * se;
    cpx<T> buf[C::IT];
    auto load = [&](unsigned grp, bool& valid, unsigned& base) {
        const unsigned line = grp * C::L + l;
        valid = line < nlines;
        base = valid ? col_base<2>(g, line) : 0u;
#pragma unroll
        for (int it = 0; it < C::IT; ++it) buf[it] = gload_c(Wc, base + lane_off + (unsigned)(it * C::TT) * se);
    };
    unsigned grp = blockIdx.x, base;
    bool valid;
    if constexpr (PF) load(grp, valid, base);
    if constexpr (N == 256) {
        // the line stays in registers (see fft256_regs); LDS only for the
        // transposes and the exchange of the (k, N-k) partners, which stays
        // within the wave (reg_col): 4 block barriers per line group
        __syncthreads();  // twiddles
        cpx<T>* ln = lds + l * C::LS;
        while (true) {
            if constexpr (!PF) load(grp, valid, base);
            cpx<T> v[16];
#pragma unroll
            for (int a = 0; a < 16; ++a) v[a] = buf[a];
            const bool cur_valid = valid;
            const unsigned cur_base = base;
            const unsigned line = grp * C::L + l;
            const unsigned j = cur_valid ? line / (unsigned)g.nxh : 0u, m = cur_valid ? line - j * (unsigned)g.nxh : 0u;
            const T lxe = lamx[2 * m], lxo = lamx[2 * m + 1], lyj = lamy[j];
            const T ta0 = (lxe + lyj) * sc, tb0 = (lxo + lyj) * sc, dt = (lxo - lxe) * sc;
            const unsigned ng = grp + gridDim.x;
            if constexpr (PF) {
                __builtin_amdgcn_s_setprio(2);
                if (ng < ngroups) load(ng, valid, base);  // in flight during the two FFTs
                __builtin_amdgcn_s_setprio(0);
            }
            int c = e0;  // opaque within each group (see k_dht_cols)
            asm volatile("" : "+v"(c));
            fft256_regs<T>(v, ln, c, tw);  // v[b] = X[c + 16 b]
            exchange_write<T, N>(ln, c, v);
            wave_lds_sync();
            {
                const cpx<T>* pp = exchange_partner<T, N>(ln, c);
                const T* lz = lzs + c;  // sc times the z symbol at k = c + 16 b (zero only for k = 0)
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    const T lzk = lz[16 * b];
                    T hp, hm;
                    if (b == 0) pair_coefs0(ta0 + lzk, tb0 + lzk, kn, hp, hm);
                    else pair_coefs(ta0 + lzk, tb0 + lzk, dt, kn2, hp, hm);
                    // the second transform's input x[c + 16 b]
                    v[b] = scaled_conj_h(v[b], pp[17 * (15 - b)], hp, hm);
                }
            }
            wave_lds_sync();  // the partner lanes' reads before this wave's transpose writes
            fft256_regs<T>(v, ln, c, tw);
            if (cur_valid) {
                const unsigned st_base = cur_base + (unsigned)c * se;
#pragma unroll
                for (int b = 0; b < 16; ++b)
                    gstore_c(Wc, st_base + (unsigned)(16 * b) * se, cpx<T>{v[b].x, -v[b].y});
            }
            grp = ng;
            if (grp >= ngroups) break;
        }
        return;
    }
    if constexpr (N == 512) {
        // the line stays in registers: thread e0 of a line holds x[e0 + 32 a];
        // after fft512_regs it holds X[k] for k = k1 + 16 b + 256 h (k1 = e0 / 2,
        // h = e0 % 2).  The spectrum goes through the line's LDS row once, which
        // hands each thread its natural-order input of the second transform and
        // the (k, N-k) partners: 6 block barriers per line group, with the fewest
        // registers (two 512-thread FP32 blocks per CU).
        static_assert(C::TT == 32 && C::IT == 16, "512-point lines: 32 threads of 16 values");
        __syncthreads();  // twiddles, symbol
        cpx<T>* ln = lds + l * C::LS;
        while (true) {
            if constexpr (!PF) load(grp, valid, base);
            cpx<T> v[16];
#pragma unroll
            for (int a = 0; a < 16; ++a) v[a] = buf[a];
            const bool cur_valid = valid;
            const unsigned cur_base = base;
            const unsigned line = grp * C::L + l;
            const unsigned j = cur_valid ? line / (unsigned)g.nxh : 0u, m = cur_valid ? line - j * (unsigned)g.nxh : 0u;
            const T lxe = lamx[2 * m], lxo = lamx[2 * m + 1], lyj = lamy[j];
            const T ta0 = (lxe + lyj) * sc, tb0 = (lxo + lyj) * sc, dt = (lxo - lxe) * sc;
            const unsigned ng = grp + gridDim.x;
            if constexpr (PF) {
                __builtin_amdgcn_s_setprio(2);
                if (ng < ngroups) load(ng, valid, base);  // in flight during the two FFTs
                __builtin_amdgcn_s_setprio(0);
            }
            int c = e0;  // opaque within each group (see k_dht_cols)
            asm volatile("" : "+v"(c));
            fft512_regs<T>(v, ln, c, tw);  // v[b] = X[c/2 + 16 b + 256 (c mod 2)]
            exchange_write<T, N>(ln, c, v);
            // the whole spectrum through LDS: the second forward transform
            // takes its input x[c + 32 a] in natural order, at pos(c + 32 a) =
            // c + c/16 + 34 a, its partner at pos(N - c - 32 a) = p2 - 34 a
            // (for c = 0 the padding slot holding X[0] at a = 0)
            __syncthreads();
            {
                const cpx<T>* pk = ln + c + (c >> 4);
                const int p2 = c == 0 ? 544 : (512 - c) + ((512 - c) >> 4);
                const cpx<T>* pm = ln + (p2 - 510);
                const T* lz = lzs + c;  // sc times the z symbol at k = c + 32 a (zero only for k = 0)
#pragma unroll
                for (int a = 0; a < 16; ++a) {
                    const T lzk = lz[32 * a];
                    T hp, hm;
                    if (a == 0) pair_coefs0(ta0 + lzk, tb0 + lzk, kn, hp, hm);
                    else pair_coefs(ta0 + lzk, tb0 + lzk, dt, kn2, hp, hm);
                    v[a] = scaled_conj_h(pk[34 * a], pm[34 * (15 - a)], hp, hm);
                }
            }
            __syncthreads();
            fft512_regs<T>(v, ln, c, tw);  // v[b] = conj(x'[c/2 + 16 b + 256 (c mod 2)])
            if (cur_valid) {
                const unsigned st_base = cur_base + (unsigned)((c >> 1) + 256 * (c & 1)) * se;
#pragma unroll
                for (int b = 0; b < 16; ++b)
                    gstore_c(Wc, st_base + (unsigned)(16 * b) * se, cpx<T>{v[b].x, -v[b].y});
            }
            // fft512_regs ends on a barrier: the next group's writes are safe
            grp = ng;
            if (grp >= ngroups) break;
        }
        return;
    }
}

template <typename T, int N, int L>
__global__ void __launch_bounds__((ColShape<T, N, L>::NT), (ColShape<T, N, L>::MINW))
k_dht_z_solve(GridArgs g, const Slot* __restrict__ slots, Tables tb, int stage, int mode) {
    using F = LineFft<T, N, false>;
    constexpr int NT = ColShape<T, N, L>::NT;
    __shared__ cpx<T> lds[L * F::LS];
    __shared__ cpx<T> tw[N];
    __shared__ T lzs[N / 2 + 1];  // the scaled z symbol, even in k (see k_dht_z_solve_regs)
    const Slot& s = slots[blockIdx.y];
    if constexpr (!ColShape<T, N, L>::EARLY)
        if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    TwiddleLoad<T, N, NT> twl;
    twl.load(twiddles<T>(tb, 2));
    POIS_GLOBAL T* Wc = mode == 0 ? IterView<T>(s).W : (POIS_GLOBAL T*)gptr(s.W);  // complex-indexed
    const unsigned nlines = (unsigned)(g.nxh * g.ny), ngroups = (nlines + L - 1) / L;
    const unsigned se = (unsigned)(g.nxh * g.ny);
    const int l = threadIdx.x % L, t = threadIdx.x / L;
    const T* lamx = symbol<T>(tb, 0);
    const T* lamy = symbol<T>(tb, 1);
    const T sc = symbol_scale<T>(g);
    const T kn = T(g.n) / sc;  // exact: sc is a power of two
    const unsigned lane_off = (unsigned)t * se;
    cpx<T>* ln = lds + l * F::LS;
    cpx<T> buf[F::E];
    auto load = [&](unsigned grp, bool& valid, unsigned& base) {
        const unsigned line = grp * L + l;
        valid = line < nlines;
        base = valid ? col_base<2>(g, line) : 0u;
#pragma unroll
        for (int a = 0; a < F::E; ++a) buf[a] = gload_c(Wc, base + lane_off + (unsigned)(a * F::TT) * se);
    };
    unsigned grp = ColShape<T, N, L>::first_group(blockIdx.x, gridDim.x), base;
    bool valid;
    load(grp, valid, base);
    if constexpr (ColShape<T, N, L>::EARLY) {
        loads_issued();
        if (mode == 0 && IterView<T>::skip(s.st, stage)) return;
    }
    twl.store(tw);
    for (int e = threadIdx.x; e <= N / 2; e += NT) lzs[e] = symbol<T>(tb, 2)[e] * sc;
    __syncthreads();  // twiddles, symbol
    while (true) {
        cpx<T> v[F::E];
#pragma unroll
        for (int a = 0; a < F::E; ++a) v[a] = buf[a];
        const bool cur_valid = valid;
        const unsigned cur_base = base;
        // symbol of this thread's line: x wavenumbers 2m, 2m+1 (the pair), y wavenumber j
        const unsigned line = grp * L + l;
        const unsigned j = cur_valid ? line / (unsigned)g.nxh : 0u, m = cur_valid ? line - j * (unsigned)g.nxh : 0u;
        const T lxe = lamx[2 * m], lxo = lamx[2 * m + 1], lyj = lamy[j];
        const T ta0 = (lxe + lyj) * sc, tb0 = (lxo + lyj) * sc;
        const unsigned ng = grp + gridDim.x;
        __builtin_amdgcn_s_setprio(2);
        if (ng < ngroups) load(ng, valid, base);  // in flight during the two FFTs
        __builtin_amdgcn_s_setprio(0);
        typename F::Out out;
        F::forward(v, ln, t, tw, out);
        __syncthreads();  // the last stage's reads before its outputs
        F::put(out, ln, t);
        __syncthreads();
        // scaled spectra of the pairs (k, N-k), conjugated: the second
        // transform's input x[t + a TT]
#pragma unroll
        for (int a = 0; a < F::E; ++a) {
            const int k = t + a * F::TT;  // the two positions: a base plus, a base minus immediate offsets
            const T lzk = lzs[k <= N / 2 ? k : N - k];
            T hp, hm;
            if (a == 0) {
                pair_coefs0(ta0 + lzk, tb0 + lzk, kn, hp, hm);
            } else {
                // each symbol inverted on its own: no bound on the ratio of the cell sizes
                const T sa = recip(kn * (ta0 + lzk)), sb = recip(kn * (tb0 + lzk));
                hp = T(0.5) * (sa + sb);
                hm = T(0.5) * (sa - sb);
            }
            v[a] = scaled_conj_h(ln[F::pos(k)], ln[F::pos(N - k)], hp, hm);
        }
        __syncthreads();
        F::forward(v, ln, t, tw, out);
        if (cur_valid) {
            F::each(out, t, [&](int j, int dk, cpx<T> z) {
                gstore_c(Wc, cur_base + (unsigned)j * se + (unsigned)dk * se, cpx<T>{z.x, -z.y});
            });
        }
        grp = ng;
        if (grp >= ngroups) break;
        __syncthreads();
    }
}

// ---- launch ---------------------------------------------------------------------
// Lines of 256 and 512 whose groups fill the chip take the register kernels;
// every other line the FftPlan kernels, wide or narrow.
template <typename T, int N, class Go>
static hipError_t col_shape(unsigned nlines, Go&& go) {
    if ((nlines + wide_lines<T, N>() - 1) / wide_lines<T, N>() >= kWideGroups)
        return go.template operator()<wide_lines<T, N>()>();
    return go.template operator()<narrow_lines<T, N>()>();
}

template <typename T, bool SHORT>
hipError_t launch_cols_y(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage) {
    return dispatch_len(g.ny, [&]<int N>() {
        if constexpr ((N <= kShortLine) != SHORT) {
            return hipErrorInvalidValue;
        } else {
            const unsigned nlines = (unsigned)(g.nxh * g.nz);
            auto run = [&](auto kernel, int nt, int lines) {
                const void* k = (const void*)kernel;
                const int nb = persistent_grid(k, nt, (nlines + lines - 1) / lines, nslots, share);
                kernel<<<dim3(nb, nslots), nt, reserve_lds(k, share), s>>>(g, slots, t, stage, mode);
                return hipGetLastError();
            };
            if constexpr (N == 256 || N == 512)
                if (nlines / 16 >= kWideGroups) return run(&k_dht_cols_regs<T, N>, LineCfg<T, N>::NT, 16);
            return col_shape<T, N>(nlines, [&]<int L>() {
                return run(&k_dht_cols<T, N, L>, ColShape<T, N, L>::NT, L);
            });
        }
    });
}

template <typename T, bool SHORT>
hipError_t launch_z_solve(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                          float share, int stage) {
    return dispatch_len(g.nz, [&]<int N>() {
        if constexpr ((N <= kShortLine) != SHORT) {
            return hipErrorInvalidValue;
        } else {
            const unsigned nlines = (unsigned)(g.nxh * g.ny);
            auto run = [&](auto kernel, int nt, int lines) {
                const void* k = (const void*)kernel;
                const int nb = persistent_grid(k, nt, (nlines + lines - 1) / lines, nslots, share);
                kernel<<<dim3(nb, nslots), nt, reserve_lds(k, share), s>>>(g, slots, t, stage, mode);
                return hipGetLastError();
            };
            if constexpr (N == 256 || N == 512)
                if (nlines / 16 >= kWideGroups) {
                    using Z = ZRegsCfg<T, N>;
                    return run(&k_dht_z_solve_regs<T, N, Z::PF, Z::MINW>, LineCfg<T, N>::NT, 16);
                }
            return col_shape<T, N>(nlines, [&]<int L>() {
                return run(&k_dht_z_solve<T, N, L>, ColShape<T, N, L>::NT, L);
            });
        }
    });
}

}  // namespace pois
