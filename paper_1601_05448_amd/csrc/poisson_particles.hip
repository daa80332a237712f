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
// corner cell in x, y, z).  Then every block owns a few rows of the grid, adds
// the corner sums that fall on them in LDS in a fixed order, and writes each of
// its cells once (k_part_cells).  I is a plain gather, one thread per particle.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "poisson_device.hpp"

namespace pois {

constexpr int kPartThreads = 256;

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

__global__ void __launch_bounds__(kPartThreads) k_part_flag_clear(int* __restrict__ bad) {
    if (threadIdx.x == 0) bad[0] = 0;
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

// The particles lie anywhere in memory: each thread gathers one (64 B, or two
// lines of it), so that all of a block's loads are in flight together; then
// eight threads sum each kPiece positions, one per corner, and store the eight
// sums of a piece side by side.  (10^6 particles on 512^3: 47 us; one
// thread per kPiece particles and all corners took 64.)
__global__ void __launch_bounds__(kPartThreads)
k_part_pieces(PartGeom pg, int np, const double* __restrict__ pos, const double* __restrict__ q,
              const uint2* __restrict__ pair, double* __restrict__ psum) {
    static_assert(kPartThreads % kPiece == 0, "a block's positions start at a multiple of kPiece");
    __shared__ double f[4][kPartThreads];
    __shared__ unsigned key[kPartThreads];
    const int t = (int)threadIdx.x;
    const long long base = (long long)blockIdx.x * kPartThreads;
    const int n = (int)min((long long)kPartThreads, np - base);
    if (t < n) {
        const uint2 pr = pair[base + t];
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
}

// (A run's later pieces are read kAhead at a time, so that one long run does not
// wait for memory at every piece.)
__global__ void __launch_bounds__(kPartThreads)
k_part_runs(int np, const uint2* __restrict__ pair, double* __restrict__ psum) {
    constexpr int kAhead = 4;
    const long long s = (long long)blockIdx.x * kPartThreads + threadIdx.x;
    if (s >= np) return;
    const unsigned k = pair[s].x;
    if (s > 0 && pair[s - 1].x == k) return;
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
            const long long at = min(nxt + u * kPiece, (long long)np - 1);
            kk[u] = pair[at].x;
#pragma unroll
            for (int c = 0; c < 8; ++c) v[u][c] = psum[8 * (size_t)at + c];
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

// First sorted position with a key of at least `key`: a wave narrows the range
// 64-fold per step (10^6 pairs: four dependent loads, where halving takes 20).
__device__ __forceinline__ int first_at_least(const uint2* __restrict__ pair, int np, unsigned long long key) {
    const long long lane = threadIdx.x & 63;
    long long lo = 0, len = np;  // the answer is in [lo, lo + len]
    while (len > 0) {
        const long long step = (len + 63) / 64, at = lane * step;
        const bool less = at < len && (unsigned long long)pair[lo + at].x < key;
        const long long nless = __popcll(__ballot(less));
        if (nless == 0) return (int)lo;
        lo += (nless - 1) * step + 1;
        len = min(step - 1, len - ((nless - 1) * step + 1));
    }
    return (int)lo;
}

// The same within [lo, hi], by one thread.
__device__ __forceinline__ int first_between(const uint2* __restrict__ pair, int lo, int hi, unsigned long long key) {
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (pair[mid].x < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The deposit itself: a block owns `span` tiles of `rows` rows of one plane, one
// after the other, and gathers the corner sums that fall on each tile [j0, j1) x
// nx in LDS.  They come from the runs of plane k - 1 (their upper half, e = 1) and
// of plane k (e = 0), rows j0 - 1 to j1 - 1: two contiguous ranges of the sorted
// pairs, and two more for the row below row 0, ny - 1.  Half of the block's
// threads walk each plane's range.  Runs are distinct cells, so for one corner
// (a, b) of one plane no two threads add to one cell; barriers separate the
// corners, and every cell receives its contributions in the same order in every
// call.  A run longer than a chunk of the walk is skipped by a search for its end.
//
// What bounds it is the grid's one write, and, per tile, the chain bounds - pairs
// - sums - LDS: the bounds of all the block's tiles are found at once (one tile
// per block and the planes in turn: 381 us for 10^6 particles on 512^3).  Filling
// the grid with zeros and adding the runs in eight passes (one per parity class
// of the run's cell) moved whole lines both ways for 8-byte updates: 172 us of
// filling beside the sort and 267 us of passes after it, now 255 us in all (4.2
// TB/s of the grid's 1.07 GB).  Deposits, before and after: 10^6 particles on
// 512^3 746 -> 416 us (10^4 of them in one cell 1264 -> 634, all of them 53.5 ->
// 22.1 ms), 2 10^6 on 256^3 647 -> 310, 2000 on 32^3 160 -> 80.
constexpr int kSpanMax = 32;  // tiles of a block at most (their bounds: 512 bytes of LDS)

__global__ void __launch_bounds__(kPartThreads)
k_part_cells(PartGeom pg, int np, const uint2* __restrict__ pair, const double* __restrict__ psum,
             const int* __restrict__ bad, int rows, int span, int spans, double* __restrict__ out) {
    constexpr int kHalf = kPartThreads / 2;
    extern __shared__ double acc[];
    __shared__ int edge[2][2], wrap_edge[2][2];   // [plane k - 1, k][first, end]: the block's rows; row ny - 1
    __shared__ int bound[kSpanMax][2][2];
    if (bad[0]) return;  // a bad position: the output stays as it is
    const int nx = pg.nx, ny = pg.ny, nz = pg.nz, t = (int)threadIdx.x;
    const int k = (int)(blockIdx.x / (unsigned)spans);
    const int jb0 = (int)(blockIdx.x - (unsigned)k * (unsigned)spans) * rows * span, jb1 = min(jb0 + rows * span, ny);
    const int tiles = (jb1 - jb0 + rows - 1) / rows;
    const unsigned row0[2] = {(unsigned)(k == 0 ? nz - 1 : k - 1) * (unsigned)ny, (unsigned)k * (unsigned)ny};
    const auto row_key = [&](int pl, int row) {
        return (unsigned long long)(row0[pl] + (unsigned)row) * (unsigned)nx;
    };
    {
        const int w = __builtin_amdgcn_readfirstlane(t >> 6), pl = w >> 1, end = w & 1;
        const int a = first_at_least(pair, np, row_key(pl, end ? jb1 : max(jb0 - 1, 0)));
        const int b = jb0 == 0 ? first_at_least(pair, np, row_key(pl, ny - 1 + end)) : 0;
        if ((t & 63) == 0) {
            edge[pl][end] = a;
            wrap_edge[pl][end] = b;
        }
    }
    __syncthreads();
    for (int q = t; q < 4 * tiles; q += kPartThreads) {
        const int m = q >> 2, pl = (q >> 1) & 1, end = q & 1, j0 = jb0 + m * rows;
        int at;
        if (end == 0 && m == 0) at = edge[pl][0];
        else if (end == 1 && m == tiles - 1) at = edge[pl][1];
        else at = first_between(pair, edge[pl][0], edge[pl][1], row_key(pl, end ? j0 + rows : j0 - 1));
        bound[m][pl][end] = at;
    }
    const int pl = t / kHalf;  // the plane this thread walks
    for (int m = 0; m < tiles; ++m) {
        const int j0 = jb0 + m * rows, j1 = min(j0 + rows, ny), cells = (j1 - j0) * nx;
        for (int c = t; c < cells; c += kPartThreads) acc[c] = 0.0;
        __syncthreads();
        for (int wrap = j0 == 0 ? 1 : 0; wrap >= 0; --wrap) {
            long long at[2], hi[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                at[u] = wrap ? wrap_edge[u][0] : bound[m][u][0];
                hi[u] = wrap ? wrap_edge[u][1] : bound[m][u][1];
            }
            while (at[0] < hi[0] || at[1] < hi[1]) {
                const long long s = (pl ? at[1] : at[0]) + (t & (kHalf - 1));
                double w[4] = {0.0, 0.0, 0.0, 0.0};
                int c0 = -1, c1 = -1, dx = 0;
                if (s < (pl ? hi[1] : hi[0])) {
                    const unsigned key = pair[s].x;
                    if (s == 0 || pair[s - 1].x != key) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) w[q] = psum[8 * (size_t)s + (pl ? 0 : 4) + q] * pg.inv_v;
                        const unsigned row = key / (unsigned)nx;
                        const int i = (int)(key - row * (unsigned)nx), j = (int)(row - (pl ? row0[1] : row0[0]));
                        dx = i + 1 == nx ? -i : 1;
                        if (!wrap && j >= j0) c0 = (j - j0) * nx + i;
                        if (wrap) c1 = i;
                        else if (j + 1 < j1) c1 = (j + 1 - j0) * nx + i;
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (at[u] >= hi[u]) continue;
                    const bool mine = pl == u;
                    if (mine && c0 >= 0) acc[c0] += w[0];
                    __syncthreads();
                    if (mine && c0 >= 0) acc[c0 + dx] += w[1];
                    __syncthreads();
                    if (mine && c1 >= 0) acc[c1] += w[2];
                    __syncthreads();
                    if (mine && c1 >= 0) acc[c1 + dx] += w[3];
                    __syncthreads();
                    at[u] += kHalf;
                    if (at[u] < hi[u]) {
                        const unsigned last = pair[at[u] - 1].x;
                        if (pair[min(at[u] + kHalf, hi[u]) - 1].x == last)
                            at[u] = first_at_least(pair, np, (unsigned long long)last + 1u);
                    }
                }
            }
        }
        // (a thread writes and clears the same cells of LDS: no barrier between the two)
        double* o = out + ((size_t)k * ny + j0) * nx;
        for (int c = t; c < cells; c += kPartThreads) o[c] = acc[c];
    }
}

// Rows of a tile of k_part_cells: eight, or what fits 32 KB of LDS (five blocks per
// CU), fewer where that leaves the chip without four blocks per CU.  More rows
// share the search and the row below the tile (10^6 particles on 512^3: 491, 433
// and 416 us with 2, 4 and 8 rows; 3 10^5 on 384 x 192 x 768: 240 with 2, 221 with
// 5), more than eight leave too little work in flight (2 10^6 on 256^3: 317 with 8,
// 334 with 16).  Then as many tiles per block as leave eight blocks per CU (fewer
// would not fill it, more repeat the search for the rows' bounds: with 32 blocks
// per CU 460 us on 512^3 and 337 on 256^3 where it was 444 and 317).
static int tile_rows(const GridArgs& g) {
    int rows = std::max(1, std::min({g.ny, 8, 4096 / g.nx}));
    while (rows > 1 && (long long)g.nz * ((g.ny + rows - 1) / rows) < 1024) rows = (rows + 1) / 2;
    return rows;
}

static int tile_span(const GridArgs& g, int rows) {
    const int tiles = (g.ny + rows - 1) / rows;
    return std::max(1, std::min({tiles, kSpanMax, (int)((long long)tiles * g.nz / 2048)}));
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

// The pairs (two copies for the sort passes), the piece and run sums, the digit
// totals, the bad-position flag.  The (tile, digit) counts of the sort lie where
// the sums come later.
size_t particle_workspace_bytes(const GridArgs& g, int np) {
    (void)g;
    return 2 * up256((size_t)np * 8) +
           std::max(up256((size_t)np * 64), up256((size_t)kDigits * std::max(1, sort_tiles(np)) * 4)) +
           up256((size_t)kDigits * 4) + 256;
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
    uint2* pair = reinterpret_cast<uint2*>(w);
    uint2* pair2 = reinterpret_cast<uint2*>(w + kb);
    double* psum = reinterpret_cast<double*>(w + 2 * kb);
    unsigned* counts = reinterpret_cast<unsigned*>(psum);
    hipError_t e;
    k_part_flag_clear<<<1, 64, 0, s>>>(bad);
    if (np > 0) {
        const unsigned pb = ((unsigned)np + kPartThreads - 1) / kPartThreads;
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
        k_part_pieces<<<pb, kPartThreads, 0, s>>>(pg, np, pos, q, pair, psum);
        k_part_runs<<<pb, kPartThreads, 0, s>>>(np, pair, psum);
    }
    const int rows = tile_rows(g), span = tile_span(g, rows), spans = (g.ny + rows * span - 1) / (rows * span);
    k_part_cells<<<(unsigned)g.nz * (unsigned)spans, kPartThreads, (size_t)rows * g.nx * sizeof(double), s>>>(
        pg, np, pair, psum, bad, rows, span, spans, out);
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
    k_part_flag_clear<<<1, 64, 0, s>>>(bad_dev);
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
