// Particles and the grid (section "Physical model" of the paper): the linear
// projection P of particle values to the grid, per unit volume, and the linear
// interpolation I of a grid field at the particle positions, periodic.  A
// particle at x has, per direction, s = x/h - 1/2, i0 = floor(s), f = s - i0 and
// gives weight 1 - f to cell i0 and f to cell i0 + 1; its eight cells get the
// products of the three directions' weights.
//
// P without floating-point atomics, deterministic: every particle gets the key
// of its lower corner cell (i0, j0, k0); a stable radix sort (least significant
// digit first; the rank of a key among equal digits comes from wave ballots, so
// equal keys keep their index order) orders the particles by key and, within a
// key, by index; the run of each occupied cell is summed in pieces of at most
// kPiece sorted particles (so a cell holding many particles costs a few piece
// sums, not a long serial loop), and the pieces of a run are added in order into
// its eight corner sums sum_p q_p W_a W_b W_e (a, b, e the offsets 0/1 of the
// corner cell in x, y, z).  The runs are listed in the order of their cells.  Then
// every block owns a few tiles of rows of the grid, adds the runs' corner sums that
// fall on them in LDS in a fixed order, and writes each of its cells once
// (k_part_cells).  I is a plain gather, one thread per particle.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "poisson_device.hpp"
#include "poisson_particle_tiles.hpp"

namespace pois {

constexpr int kPartThreads = 256;
constexpr int kGroupStep = 32;  // words from one group's run count to the next

// lower cell index and fraction of a coordinate along one direction; false if
// the position is not finite or more than 2^30 cells away
__device__ __forceinline__ bool cell_frac(double x, double inv_h, int n, int& i0, double& f) {
    const double s = x * inv_h - 0.5;
    if (!(fabs(s) < 1073741824.0)) return false;
    const double fl = floor(s);
    f = s - fl;
    int a = (int)fl;
    if ((unsigned)a >= (unsigned)n) {  // outside the box: wrapped
        a %= n;
        if (a < 0) a += n;
    }
    i0 = a;
    return true;
}

struct PartGeom {
    int nx, ny, nz;
    double inv_hx, inv_hy, inv_hz, inv_v;
};

// The key of a particle: its lower corner cell (k ny + j) nx + i.  Sorted, the
// particles of any rows of one plane are one contiguous range.
__global__ void __launch_bounds__(kPartThreads)
k_part_keys(PartGeom pg, int np, const double* __restrict__ pos, uint2* __restrict__ pair, int* __restrict__ bad) {
    const int p = blockIdx.x * kPartThreads + threadIdx.x;
    if (p >= np) return;
    int i, j, k;
    double fx, fy, fz;
    const bool ok = cell_frac(pos[3 * (size_t)p], pg.inv_hx, pg.nx, i, fx) &&
                    cell_frac(pos[3 * (size_t)p + 1], pg.inv_hy, pg.ny, j, fy) &&
                    cell_frac(pos[3 * (size_t)p + 2], pg.inv_hz, pg.nz, k, fz);
    if (!ok) {
        bad[0] = 1;  // plain vector store: every writer writes the same value
        i = j = k = 0;
    }
    const unsigned cell = ((unsigned)k * (unsigned)pg.ny + (unsigned)j) * (unsigned)pg.nx + (unsigned)i;
    pair[p] = make_uint2(cell, (unsigned)p);
}

// Clears the bad-position flag and the run counts of the groups (none for the
// interpolation).
__global__ void __launch_bounds__(kPartThreads)
k_part_clear(int* __restrict__ bad, unsigned* __restrict__ group_runs, int groups) {
    if (threadIdx.x == 0) bad[0] = 0;
    for (int q = threadIdx.x; q < groups; q += kPartThreads) group_runs[q * (size_t)kGroupStep] = 0u;
}

// ---- stable LSD radix sort of (key, index) pairs ----------------------------------
// One pass orders by the digit (key >> shift) & (2^db - 1), keeping the order of
// equal digits: per tile of kSortTile pairs a block counts its digits
// (k_rs_count), the counts become each (tile, digit)'s first position among its
// digit (k_rs_scan), and every block writes its pairs there in tile order
// (k_rs_scatter).  The digits are as narrow as the number of passes allows (27
// bits: three of 9).  Latency bounds it, not traffic (8 MB of pairs per pass at
// 10^6), so the loads of a tile are all issued at once, the counts lie tile-major
// (every access of them is coalesced; digit-major they were 10^6 four-byte
// stores), and a wave ranks its pairs without a barrier.  10^6 pairs: 24 us per pass
// (count 4, scan 5, scatter 15), where it was 98 us (35, 23 and 5, 35).
constexpr int kDigitBits = 10;
constexpr int kDigits = 1 << kDigitBits;
constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;

__global__ void __launch_bounds__(kSortThreads)
k_rs_count(int np, const uint2* __restrict__ pair, int shift, int db, unsigned* __restrict__ counts) {
    __shared__ unsigned hist[kDigits];
    const unsigned nd = 1u << db;
    const long long base = (long long)blockIdx.x * kSortTile + threadIdx.x;
    unsigned k[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
        k[it] = base + it * kSortThreads < np ? pair[base + it * kSortThreads].x : 0u;
    for (unsigned d = threadIdx.x; d < nd; d += kSortThreads) hist[d] = 0u;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)  // integer: exact in any order
        if (base + it * kSortThreads < np) atomicAdd(&hist[(k[it] >> shift) & (nd - 1)], 1u);
    __syncthreads();
    for (unsigned d = threadIdx.x; d < nd; d += kSortThreads) counts[(size_t)blockIdx.x * nd + d] = hist[d];
}

// Exclusive prefix sums of every digit's counts over the tiles, in place, and the
// digits' totals.  A block takes kScanDigits digits (a 128-byte line of the
// counts) and its kScanGroups thread groups equal shares of the tiles.
constexpr int kScanDigits = 32;
constexpr int kScanGroups = 32;

__global__ void __launch_bounds__(kScanDigits * kScanGroups)
k_rs_scan(unsigned* __restrict__ counts, int tiles, int db, unsigned* __restrict__ digit_tot) {
    __shared__ unsigned part[kScanGroups][kScanDigits];
    const unsigned nd = 1u << db, dl = threadIdx.x % kScanDigits, grp = threadIdx.x / kScanDigits;
    const unsigned d = blockIdx.x * kScanDigits + dl;
    const int share = (tiles + kScanGroups - 1) / kScanGroups;
    const long long t0 = (long long)grp * share;
    const int t1 = (int)min((long long)tiles, t0 + share);
    unsigned sum = 0u;
#pragma unroll 8
    for (int t = (int)min(t0, (long long)tiles); t < t1; ++t) sum += counts[(size_t)t * nd + d];
    part[grp][dl] = sum;
    __syncthreads();
    unsigned at = 0u;
    for (unsigned q = 0; q < grp; ++q) at += part[q][dl];
    if (grp + 1 == kScanGroups) digit_tot[d] = at + sum;
#pragma unroll 8
    for (int t = (int)min(t0, (long long)tiles); t < t1; ++t) {
        const unsigned v = counts[(size_t)t * nd + d];
        counts[(size_t)t * nd + d] = at;
        at += v;
    }
}

__global__ void __launch_bounds__(kSortThreads)
k_rs_scatter(int np, const uint2* __restrict__ pair, int shift, int db, const unsigned* __restrict__ start,
             const unsigned* __restrict__ digit_tot, uint2* __restrict__ pair_out) {
    constexpr int kPer = kDigits / kSortThreads;
    __shared__ unsigned cnt[kSortWaves][kDigits];  // a wave's pairs of each digit, then their first position
    __shared__ unsigned wsum[kSortWaves];
    const unsigned nd = 1u << db;
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const long long base = (long long)blockIdx.x * kSortTile + wave * (64 * kSortItems) + lane;
    uint2 pr[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
        pr[it] = base + it * 64 < np ? pair[base + it * 64] : make_uint2(0u, 0u);
    // thread t holds the digits kPer t ..
    unsigned tot[kPer], mine = 0u;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const unsigned d = threadIdx.x * kPer + q;
        tot[q] = d < nd ? digit_tot[d] : 0u;
        mine += tot[q];
    }
    for (unsigned d = lane; d < nd; d += 64) cnt[wave][d] = 0u;
    unsigned incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned u = __shfl_up(incl, off);
        if (lane >= off) incl += u;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    unsigned rank[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const unsigned d = (pr[it].x >> shift) & (nd - 1);
        // lanes of this wave with the same digit: the AND over the digit's bits
        const bool valid = base + it * 64 < np;
        unsigned long long same = __ballot(valid);
        for (int bit = 0; bit < db; ++bit) {
            const unsigned long long on = __ballot((d >> bit) & 1u);
            same &= ((d >> bit) & 1u) ? on : ~on;
        }
        const unsigned ahead = (unsigned)__popcll(same & below);
        unsigned before = 0u;
        if (valid) before = __hip_atomic_load(&cnt[wave][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the lowest lane of each digit adds its group
        if (valid && ahead == 0u)
            __hip_atomic_store(&cnt[wave][d], before + (unsigned)__popcll(same), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WAVEFRONT);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        rank[it] = before + ahead;
    }
    __syncthreads();
    unsigned first = incl - mine;
    for (int w = 0; w < wave; ++w) first += wsum[w];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const unsigned d = threadIdx.x * kPer + q;
        if (d < nd) {
            unsigned at = first + start[(size_t)blockIdx.x * nd + d];
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const unsigned c = cnt[w][d];
                cnt[w][d] = at;
                at += c;
            }
        }
        first += tot[q];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
        if (base + it * 64 < np) pair_out[cnt[wave][(pr[it].x >> shift) & (nd - 1)] + rank[it]] = pr[it];
}

// ---- run sums --------------------------------------------------------------------------
// Pieces: runs cut at every multiple of kPiece sorted positions.  Each piece is
// summed in sorted order and its eight sums stored at its first position; then
// the thread at each run start adds the run's pieces in order (its own, then
// those at the following multiples of kPiece).
constexpr int kPiece = 8;

// The list of the runs, (cell, first position) in the order of the cells: the blocks
// of k_part_pieces count the runs that start in their kPartThreads positions, for
// themselves and for their group of blocks, and each block of k_part_runs adds the
// counts before its own: of whole groups, and of blocks of its own group.  A group is
// about the square root of the number of blocks, which keeps both short, and at least
// 64; its counter has a cache line to itself (an atomic on a line takes some 10 ns:
// 10^6 particles' 3907 blocks on four counters of one line cost 25 us, on 61 of four
// lines 9).
static int position_blocks(int np) { return (int)(((long long)np + kPartThreads - 1) / kPartThreads); }
static int group_blocks(int np) {
    int b = 64;
    while ((long long)b * b < position_blocks(np)) b *= 2;
    return b;
}
static int run_groups(int np) { return (position_blocks(np) + group_blocks(np) - 1) / group_blocks(np); }

// The particles lie anywhere in memory: each thread gathers one (64 B, or two
// lines of it), so that all of a block's loads are in flight together; then
// eight threads sum each kPiece positions, one per corner, and store the eight
// sums of a piece side by side.  (10^6 particles on 512^3: 32 us; one
// thread per kPiece particles and all corners took 64.)
__global__ void __launch_bounds__(kPartThreads)
k_part_pieces(PartGeom pg, int np, const double* __restrict__ pos, const double* __restrict__ q,
              const uint2* __restrict__ pair, double* __restrict__ psum, const int* __restrict__ bad,
              unsigned* __restrict__ block_runs, unsigned* __restrict__ group_runs, int group_size) {
    static_assert(kPartThreads % kPiece == 0, "a block's positions start at a multiple of kPiece");
    __shared__ double f[4][kPartThreads];
    __shared__ unsigned key[kPartThreads], wave_runs[kPartThreads / 64];
    const int t = (int)threadIdx.x;
    const long long base = (long long)blockIdx.x * kPartThreads;
    const int n = (int)min((long long)kPartThreads, np - base);
    const uint2 pr = pair[base + min(t, n - 1)];
    const unsigned before = pair[max(base - 1, 0ll)].x;
    if (bad[0]) return;  // a bad position: nothing is summed
    if (t < n) {
        const double* x = pos + 3 * (size_t)pr.y;
        int i;
        double fx = 0.0, fy = 0.0, fz = 0.0;
        const double x0 = x[0], x1 = x[1], x2 = x[2], qp = q ? q[pr.y] : 1.0;
        (void)cell_frac(x0, pg.inv_hx, pg.nx, i, fx);
        (void)cell_frac(x1, pg.inv_hy, pg.ny, i, fy);
        (void)cell_frac(x2, pg.inv_hz, pg.nz, i, fz);
        f[0][t] = fx;
        f[1][t] = fy;
        f[2][t] = fz;
        f[3][t] = qp;
        key[t] = pr.x;
    }
    __syncthreads();
    const bool starts = t < n && ((t == 0 && base == 0) || (t > 0 ? key[t - 1] : before) != pr.x);
    const unsigned long long started = __ballot(starts);
    if ((t & 63) == 0) wave_runs[t >> 6] = (unsigned)__popcll(started);
    const int c = t & 7, p0 = (t >> 3) * kPiece, p1 = min(p0 + kPiece, n);
    double acc = 0.0;
    int at = p0;
    for (int p = p0; p < p1; ++p) {
        if (p > p0 && key[p] != key[p - 1]) {
            psum[8 * (size_t)(base + at) + c] = acc;
            acc = 0.0;
            at = p;
        }
        const double fx = f[0][p], fy = f[1][p], fz = f[2][p];
        acc += f[3][p] * ((c & 1) ? fx : 1.0 - fx) * ((c & 2) ? fy : 1.0 - fy) * ((c & 4) ? fz : 1.0 - fz);
    }
    if (p0 < n) psum[8 * (size_t)(base + at) + c] = acc;
    __syncthreads();
    if (t == 0) {
        unsigned runs = 0u;
#pragma unroll
        for (int w = 0; w < kPartThreads / 64; ++w) runs += wave_runs[w];
        block_runs[blockIdx.x] = runs;
        atomicAdd(&group_runs[blockIdx.x / (unsigned)group_size * (size_t)kGroupStep], runs);  // integer: exact in any order
    }
}

// edge[from, to) = value of every lane: by the lane where they are few, by the whole
// wave, lane after lane, where they are many (few particles on a large grid).  Every
// lane of the wave calls it.
__device__ __forceinline__ void put_edges(int* __restrict__ edge, unsigned from, unsigned to, int value) {
    constexpr unsigned kFew = 4;
    const bool many = to - from > kFew;
    if (!many)
        for (unsigned e = from; e < to; ++e) edge[e] = value;
    for (unsigned long long left = __ballot(many); left; left &= left - 1) {
        const int src = __builtin_ctzll(left);
        const unsigned f = (unsigned)__builtin_amdgcn_readlane((int)from, src);
        const unsigned l = (unsigned)__builtin_amdgcn_readlane((int)to, src);
        const int v = __builtin_amdgcn_readlane(value, src);
        for (unsigned e = f + (threadIdx.x & 63u); e < l; e += 64u) edge[e] = v;
    }
}

// No particles: every edge is the end of an empty list.
__global__ void __launch_bounds__(kPartThreads) k_part_no_edges(unsigned n, int* __restrict__ edge) {
    const unsigned e = blockIdx.x * kPartThreads + threadIdx.x;
    if (e < n) edge[e] = 0;
}

// Adds the pieces of the runs that start in a block's positions, lists the runs and
// puts the edges that lie between a run and the one before it, and after the last
// run.  (A run's later pieces are read kAhead at a time, so that one long run does not
// wait for memory at every piece.)
__global__ void __launch_bounds__(kPartThreads)
k_part_runs(int np, const uint2* __restrict__ pair, double* __restrict__ psum, const int* __restrict__ bad,
            const unsigned* __restrict__ block_runs, const unsigned* __restrict__ group_runs, int group_size,
            TileGeom tg, uint2* __restrict__ run, int* __restrict__ edge) {
    constexpr int kAhead = 4;
    __shared__ unsigned wave_first[kPartThreads / 64], wave_before[kPartThreads / 64];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    const long long s = (long long)blockIdx.x * kPartThreads + t;
    const unsigned k = pair[min(s, (long long)np - 1)].x;
    const unsigned prev = pair[min(max(s - 1, 0ll), (long long)np - 1)].x;
    // runs that start before this block: whole groups, then the blocks of its own
    const unsigned group = blockIdx.x / (unsigned)group_size;
    unsigned before = 0u;
    for (unsigned q = t; q < group; q += kPartThreads) before += group_runs[q * (size_t)kGroupStep];
    for (unsigned b = group * (unsigned)group_size + t; b < blockIdx.x; b += kPartThreads) before += block_runs[b];
    // a bad position: nothing is summed (all of them bad are one run, 22 ms of 10^6)
    if (bad[0]) return;
    const bool starts = s < np && (s == 0 || prev != k);
    const unsigned long long started = __ballot(starts);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
    if (lane == 0) {
        wave_before[wave] = before;
        wave_first[wave] = (unsigned)__popcll(started);
    }
    __syncthreads();
    unsigned at = 0u;
#pragma unroll
    for (int w = 0; w < kPartThreads / 64; ++w) at += wave_before[w] + (w < wave ? wave_first[w] : 0u);
    at += (unsigned)__popcll(started & (lane == 0 ? 0ull : ~0ull >> (64 - lane)));
    const unsigned here = tg.edges_to(k);
    put_edges(edge, starts && s > 0 ? tg.edges_to(prev) : 0u, starts ? here : 0u, (int)at);
    if (blockIdx.x + 1 == gridDim.x) {
        const bool last = s + 1 == np;
        put_edges(edge, last ? here : 0u, last ? tg.edges() + 1u : 0u, (int)at + (starts ? 1 : 0));
    }
    if (!starts) return;
    run[at] = make_uint2(k, (unsigned)s);
    long long nxt = (s / kPiece + 1) * kPiece;
    if (nxt >= np || pair[nxt].x != k) return;  // a single piece: its sums are the run's
    double acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = psum[8 * (size_t)s + c];
    for (bool more = true; more; nxt += kAhead * kPiece) {
        unsigned kk[kAhead];
        double v[kAhead][8];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const long long a = min(nxt + u * kPiece, (long long)np - 1);
            kk[u] = pair[a].x;
#pragma unroll
            for (int c = 0; c < 8; ++c) v[u][c] = psum[8 * (size_t)a + c];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            more = more && nxt + u * kPiece < np && kk[u] == k;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = more ? acc[c] + v[u][c] : acc[c];
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) psum[8 * (size_t)s + c] = acc[c];
}

// The deposit itself: a block owns up to kSpanMax tiles of `rows` rows of one plane, a
// few neighbours and then others far away, one after the other, and gathers the corner
// sums that fall on each tile [j0, j1) x nx in LDS.  They come from the runs of plane k - 1 (their upper half,
// e = 1) and of plane k (e = 0), rows j0 - 1 to j1 - 1: two contiguous ranges of the
// list of runs, and two more for the row below row 0, ny - 1.  Half of the block's
// threads take each plane's range, kRuns runs each at a time.  Runs are distinct cells,
// so for one corner (a, b) of one plane no two threads add to one cell; barriers
// separate the corners, and every cell receives its contributions in the same order
// in every call.
//
// What bounds it is the grid's one write, and, per tile, the chain runs - sums -
// LDS.  Filling the grid with zeros and adding the runs in eight passes (one per
// parity class of the run's cell) moved whole lines both ways for 8-byte updates:
// 172 us of filling beside the sort and 267 us of passes after it, for 10^6 particles
// on 512^3, now 252-265 us in all (4.1-4.3 TB/s of the grid's 1.07 GB).
// A tile's work is bounded by its cells, however many particles they hold, because
// it walks runs, and particles that crowd some planes or rows crowd tiles of many
// blocks, because most of a block's tiles lie far apart.  (Walking the particles, in
// tiles that were all neighbours, was 10 us faster on uniform particles and took 3870
// us for 10^6 of them in one plane of 512^3, 6850 in 16 rows of it.)  Deposits, passes
// by class / now, us: 10^6 on 512^3 uniform 732 / 427, one plane 490 / 470, 16 rows 500 /
// 430, a ball of 16^3 cells 490 / 398, one cell 53500 / 22100; 2 10^6 on 256^3 639 / 306,
// 2000 on 32^3 152 / 75.
// runs of a thread at a time (10^6 uniform particles on 64 x 512 x 512, x first: 213 us;
// with four 235)
constexpr int kRuns = 2;

__global__ void __launch_bounds__(kPartThreads)
k_part_cells(PartGeom pg, TileGeom tg, const uint2* __restrict__ run, const int* __restrict__ edge,
             const double* __restrict__ psum, const int* __restrict__ bad, double* __restrict__ out) {
    constexpr int kHalf = kPartThreads / 2;
    static_assert(8 * kSpanMax == kPartThreads, "one thread per bound");
    extern __shared__ double acc[];
    __shared__ int bound[kSpanMax][2][4];  // [tile][plane k - 1, k]: its rows' first run and end; row ny - 1's
    __shared__ int2 place[kSpanMax];       // its plane and first row, plane -1 after the block's last tile
    const int nx = pg.nx, ny = pg.ny, nz = pg.nz, rows = tg.rows, t = (int)threadIdx.x;
    const unsigned tiles_y = (unsigned)tg.tiles_y, tiles = tg.tiles;
    const int flag = bad[0];
    if (const unsigned tile = block_tile((unsigned)t >> 3, tg.group, blockIdx.x, gridDim.x); tile < tiles) {
        const unsigned k = tile / tiles_y, jt = tile - k * tiles_y;
        const unsigned kp = (t & 4) ? k : k == 0 ? (unsigned)nz - 1 : k - 1;
        if ((t & 7) == 0) place[t >> 3] = make_int2((int)k, (int)jt * rows);
        const int which = t & 3;  // row max(j0 - 1, 0); row j1; row ny - 1; the plane's end
        const unsigned e = which == 0 ? (jt == 0 ? 0u : 2 * jt - 1)
                           : which == 1 ? 2 * jt + 2
                                        : 2 * tiles_y - (which == 2 ? 1u : 0u);
        bound[t >> 3][(t >> 2) & 1][which] = edge[kp * 2 * tiles_y + e];
    } else if ((t & 7) == 0) {
        place[t >> 3].x = -1;
    }
    if (flag) return;  // a bad position: the output stays as it is
    __syncthreads();
    const int pl = __builtin_amdgcn_readfirstlane(t / kHalf);  // the plane whose runs this wave takes
    const int wave0 = __builtin_amdgcn_readfirstlane(t & (kHalf - 64)), lane = t & 63;
    for (unsigned m = 0; m < kSpanMax; ++m) {
        const int k = __builtin_amdgcn_readfirstlane(place[m].x), j0 = __builtin_amdgcn_readfirstlane(place[m].y);
        if (k < 0) break;
        const int j1 = min(j0 + rows, ny), cells = (j1 - j0) * nx;
        const unsigned row0 = (unsigned)(pl ? k : k == 0 ? nz - 1 : k - 1) * (unsigned)ny;
        for (int c = t; c < cells; c += kPartThreads) acc[c] = 0.0;
        __syncthreads();
        for (int wrap = j0 == 0 ? 1 : 0; wrap >= 0; --wrap) {
            int lo[2], hi[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                lo[u] = __builtin_amdgcn_readfirstlane(bound[m][u][2 * wrap]);
                hi[u] = __builtin_amdgcn_readfirstlane(bound[m][u][2 * wrap + 1]);
            }
            const int most = max(hi[0] - lo[0], hi[1] - lo[1]), end = pl ? hi[1] : hi[0];
            const auto add = [&]<int R>(int first) {
                // all the runs' loads, then all their sums', then the cells: lanes past
                // the end take the last run and add nothing
                const int at0 = (pl ? lo[1] : lo[0]) + first + wave0;
                uint2 rn[R];
                double w[R][4];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (at0 + r * kHalf < end) rn[r] = run[min(at0 + r * kHalf + lane, end - 1)];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (at0 + r * kHalf < end) {
                        const double* sums = psum + 8 * (size_t)rn[r].y + (pl ? 0 : 4);
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[r][q] = sums[q];
                    }
                int c0[R], c1[R], dx[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    c0[r] = c1[r] = -1;
                    if (at0 + r * kHalf < end) {
                        const unsigned row = tg.by_nx(rn[r].x);
                        const int i = (int)(rn[r].x - row * (unsigned)nx), j = (int)(row - row0);
                        const bool in = at0 + r * kHalf + lane < end;
                        dx[r] = i + 1 == nx ? -i : 1;
                        if (in && !wrap && j >= j0) c0[r] = (j - j0) * nx + i;
                        if (in && wrap) c1[r] = i;
                        else if (in && j + 1 < j1) c1[r] = (j + 1 - j0) * nx + i;
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[r][q] *= pg.inv_v;
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (lo[u] + first >= hi[u]) continue;  // the same in every thread
                    const bool mine = pl == u;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            if (mine && at0 + r * kHalf < end) {
                                const int c = q < 2 ? c0[r] : c1[r];
                                if (c >= 0) acc[c + ((q & 1) ? dx[r] : 0)] += w[r][q];
                            }
                        __syncthreads();
                    }
                }
            };
            if (most <= kHalf) {
                if (most > 0) add.template operator()<1>(0);
            } else {
                for (int first = 0; first < most; first += kRuns * kHalf) add.template operator()<kRuns>(first);
            }
        }
        // (a thread writes and clears the same cells of LDS: no barrier between the two)
        double* o = out + ((size_t)k * ny + j0) * nx;
        for (int c = t; c < cells; c += kPartThreads) o[c] = acc[c];
    }
}

__global__ void __launch_bounds__(kPartThreads)
k_part_interp(PartGeom pg, int np, const double* __restrict__ pos, const double* __restrict__ field,
              double* __restrict__ out, int* __restrict__ bad) {
    const int p = blockIdx.x * kPartThreads + threadIdx.x;
    if (p >= np) return;
    int i, j, k;
    double fx, fy, fz;
    const bool ok = cell_frac(pos[3 * (size_t)p], pg.inv_hx, pg.nx, i, fx) &&
                    cell_frac(pos[3 * (size_t)p + 1], pg.inv_hy, pg.ny, j, fy) &&
                    cell_frac(pos[3 * (size_t)p + 2], pg.inv_hz, pg.nz, k, fz);
    if (!ok) {
        bad[0] = 1;
        out[p] = 0.0;
        return;
    }
    const unsigned nx = pg.nx, ny = pg.ny, nz = pg.nz;
    const unsigned ix[2] = {(unsigned)i, (unsigned)i + 1 == nx ? 0u : (unsigned)i + 1};
    const unsigned iy[2] = {(unsigned)j, (unsigned)j + 1 == ny ? 0u : (unsigned)j + 1};
    const unsigned iz[2] = {(unsigned)k, (unsigned)k + 1 == nz ? 0u : (unsigned)k + 1};
    const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a)
                acc += wx[a] * wy[b] * wz[e] * field[((size_t)iz[e] * ny + iy[b]) * nx + ix[a]];
    out[p] = acc;
}

static PartGeom part_geom(const GridArgs& g) {
    PartGeom pg;
    pg.nx = g.nx;
    pg.ny = g.ny;
    pg.nz = g.nz;
    pg.inv_hx = std::sqrt(g.ihx2);
    pg.inv_hy = std::sqrt(g.ihy2);
    pg.inv_hz = std::sqrt(g.ihz2);
    pg.inv_v = pg.inv_hx * pg.inv_hy * pg.inv_hz;
    return pg;
}

static int key_bits(long long n) {
    int b = 1;
    while ((1ll << b) < n) ++b;
    return b;
}

static size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }

static int sort_tiles(int np) { return (int)(((long long)np + kSortTile - 1) / kSortTile); }

// The pairs (two copies for the sort passes; the list of runs takes the one that the
// last pass leaves), the piece and run sums, the digit totals, the run counts, the
// tiles' edges, the bad-position flag.  The (tile, digit) counts of the sort
// lie where the sums come later.
size_t particle_workspace_bytes(const GridArgs& g, int np) {
    return 2 * up256((size_t)np * 8) +
           std::max(up256((size_t)np * 64), up256((size_t)kDigits * std::max(1, sort_tiles(np)) * 4)) +
           up256((size_t)kDigits * 4) + up256((size_t)position_blocks(np) * 4) + up256((size_t)run_groups(np) * kGroupStep * 4) +
           up256(((size_t)tile_geom(g).edges() + 1) * 4) + 256;
}

hipError_t launch_deposit(const GridArgs& g, int np, const double* pos, const double* q, double* out, void* ws,
                          size_t ws_bytes, int* bad_host, hipStream_t s) {
    if (ws_bytes < particle_workspace_bytes(g, np)) return hipErrorInvalidValue;
    const PartGeom pg = part_geom(g);
    char* w = static_cast<char*>(ws);
    const size_t kb = up256((size_t)np * 8);
    int* bad = reinterpret_cast<int*>(w);
    unsigned* digit_tot = reinterpret_cast<unsigned*>(w + 256);
    w += 256 + up256((size_t)kDigits * 4);
    unsigned* block_runs = reinterpret_cast<unsigned*>(w);
    w += up256((size_t)position_blocks(np) * 4);
    unsigned* group_runs = reinterpret_cast<unsigned*>(w);
    w += up256((size_t)run_groups(np) * kGroupStep * 4);
    const TileGeom tg = tile_geom(g);
    int* edge = reinterpret_cast<int*>(w);
    w += up256(((size_t)tg.edges() + 1) * 4);
    uint2* pair = reinterpret_cast<uint2*>(w);
    uint2* pair2 = reinterpret_cast<uint2*>(w + kb);
    double* psum = reinterpret_cast<double*>(w + 2 * kb);
    unsigned* counts = reinterpret_cast<unsigned*>(psum);
    hipError_t e;
    k_part_clear<<<1, kPartThreads, 0, s>>>(bad, group_runs, run_groups(np));
    if (np > 0) {
        const unsigned pb = (unsigned)position_blocks(np);
        k_part_keys<<<pb, kPartThreads, 0, s>>>(pg, np, pos, pair, bad);
        const int tiles = sort_tiles(np), bits = key_bits(g.n);
        const int passes = (bits + kDigitBits - 1) / kDigitBits;
        // at least 5 bits: k_rs_scan's blocks take 32 digits each
        const int db = std::max(5, (bits + passes - 1) / passes);
        for (int shift = 0; shift < bits; shift += db) {
            k_rs_count<<<tiles, kSortThreads, 0, s>>>(np, pair, shift, db, counts);
            k_rs_scan<<<(1 << db) / kScanDigits, kScanDigits * kScanGroups, 0, s>>>(counts, tiles, db, digit_tot);
            k_rs_scatter<<<tiles, kSortThreads, 0, s>>>(np, pair, shift, db, counts, digit_tot, pair2);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            std::swap(pair, pair2);
        }
        k_part_pieces<<<pb, kPartThreads, 0, s>>>(pg, np, pos, q, pair, psum, bad, block_runs, group_runs,
                                                       group_blocks(np));
        k_part_runs<<<pb, kPartThreads, 0, s>>>(np, pair, psum, bad, block_runs, group_runs, group_blocks(np), tg,
                                                     pair2, edge);
    } else {
        k_part_no_edges<<<(tg.edges() + kPartThreads) / kPartThreads, kPartThreads, 0, s>>>(tg.edges() + 1, edge);
    }
    k_part_cells<<<tile_blocks(tg), kPartThreads, (size_t)tg.rows * g.nx * sizeof(double), s>>>(
        pg, tg, pair2, edge, psum, bad, out);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int flag = 0;
    if ((e = hipMemcpyAsync(&flag, bad, sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    *bad_host = flag;
    return hipSuccess;
}

hipError_t launch_interpolate(const GridArgs& g, int np, const double* pos, const double* field, double* out,
                              int* bad_dev, int* bad_host, hipStream_t s) {
    const PartGeom pg = part_geom(g);
    k_part_clear<<<1, kPartThreads, 0, s>>>(bad_dev, nullptr, 0);
    if (np > 0) k_part_interp<<<(np + kPartThreads - 1) / kPartThreads, kPartThreads, 0, s>>>(pg, np, pos, field,
                                                                                               out, bad_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int flag = 0;
    if ((e = hipMemcpyAsync(&flag, bad_dev, sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    *bad_host = flag;
    return hipSuccess;
}

}  // namespace pois
