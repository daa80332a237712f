// The four field sweeps of one iteration of the paper's method (section
// "Poisson equation", eq. (Pois)), written for gfx950:
//   P1 k_resid_dhtx_z r = b~ - A p, q = w r, partial norms per tile, Hartley
//                     along x -> W (z-marching stencil; k_resid_dhtx_s, tiles whose
//                     loads are issued at once, on small grids; k_resid_dhtx, a
//                     row-pair gather, for rows shorter than 16)
//   P2 k_dht_cols     Hartley along y of W (also P4: the transform is self-inverse)
//   P3 k_dht_z_solve  Hartley along z, divide by n * symbol, Hartley along z
//                     (taken as FFT, scaling of the separated spectra, inverse FFT)
//   (P2, P3 and P4 of small grids as one launch: k_dht_planes)
//   P5 k_dhtx_update  Hartley along x, p += dp (minus the mean of p)
// With walls in x (GridArgs::bcx) P1 and P5 take the cosine transform along x
// instead of the Hartley transform; P2-P4 are the same.
// and, for the FP32 refinement, k_outer_resid_dhtx: the FP64 outer residual
// fused with the first inner sweep's residual.
//
// Each block holds whole lines of its transform direction.  The registers and the
// LDS of a line group leave a sweep two to four waves per SIMD on large grids, too
// few to hide memory latency by occupancy alone, so the blocks are persistent and
// software-pipelined: a block loops over line groups, and the global loads of the
// next group are issued before the FFT of the current group, so that they are in
// flight while the block works in LDS.  The stencil sweeps keep the next plane's
// loads in flight while they evaluate the current one, for the same reason.
//
// blockIdx.y selects the solve (slot) of a batch of equal-size grids; every sweep
// returns at once for solves that are done or, on the FP32 path, not in the
// stage the sweep serves.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <cstdint>

#include "poisson_device.hpp"
#include "poisson_launch.hpp"

namespace pois {
// ---- launch ---------------------------------------------------------------------

// Blocks of a persistent sweep: every resident block of the device, shared by
// the slots of the batch, never more than there are line groups.
// The occupancy of each kernel is asked once and kept in a fixed table (no
// host allocation on the launch path; a kernel beyond the table's capacity is
// asked every time).
static int device_cus() {
    static std::once_flag once;
    static int cus = 256;
    std::call_once(once, [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n >= 1)
            cus = n;
    });
    return cus;
}

static int resident_blocks(const void* kernel, int threads) {
    constexpr int kCap = 4096;  // a power of two, above the number of kernels
    static std::mutex mu;
    static const void* keys[kCap] = {};
    static int vals[kCap] = {};
    const int cus = device_cus();
    std::lock_guard<std::mutex> lock(mu);
    const uintptr_t hsh = (reinterpret_cast<uintptr_t>(kernel) >> 4) * 0x9E3779B97F4A7C15ull;
    for (int probe = 0; probe < kCap; ++probe) {
        const int at = (int)((hsh + (uintptr_t)probe) & (kCap - 1));
        if (keys[at] == kernel) return vals[at] * cus;
        if (keys[at] == nullptr) {
            int nb = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1) nb = 1;
            keys[at] = kernel;
            vals[at] = nb;
            return nb * cus;
        }
    }
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1) nb = 1;
    return nb * cus;
}

// A share of at most one half (a very large size class served beside small
// ones) is a share of the CUs: one block per CU over that share, each block
// reserving the rest of its CU's LDS (reserve_lds), so that no block of
// another kernel shares a CU with it and the dispatcher, which spreads blocks
// over the CUs, leaves the other CUs whole to the small classes.  A larger
// partial share is a share of the resident blocks on every CU.
unsigned reserve_lds(const void* kernel, float share) {
    if (share > 0.5f) return 0;
    static std::once_flag once;
    static int lds_cu = 0, lds_block = 0;
    std::call_once(once, [] {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return;
        if (hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess)
            lds_cu = 0;
        if (hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
            lds_block = 0;
    });
    constexpr int kCap = 1024;  // a power of two, above the number of kernels launched with a half share
    static std::mutex mu;
    static const void* keys[kCap] = {};
    static unsigned vals[kCap] = {};
    std::lock_guard<std::mutex> lock(mu);
    const uintptr_t hsh = (reinterpret_cast<uintptr_t>(kernel) >> 4) * 0x9E3779B97F4A7C15ull;
    int at = -1;
    for (int probe = 0; probe < kCap; ++probe) {
        at = (int)((hsh + (uintptr_t)probe) & (kCap - 1));
        if (keys[at] == kernel) return vals[at];
        if (keys[at] == nullptr) break;
        at = -1;
    }
    unsigned pad = 0;
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, kernel) == hipSuccess) {
        const long long total = std::min(lds_cu, lds_block), own = (long long)fa.sharedSizeBytes;
        if (total > own) {
            if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(total - own)) ==
                hipSuccess)
                pad = (unsigned)(total - own);
            else
                (void)hipGetLastError();  // a refused reservation is not an error of the launch
        }
    } else {
        (void)hipGetLastError();
    }
    if (at >= 0) {
        keys[at] = kernel;
        vals[at] = pad;
    }
    return pad;
}

int persistent_grid(const void* kernel, int threads, unsigned ngroups, int nslots, float share) {
    int blocks = resident_blocks(kernel, threads);
    if (share <= 0.5f) blocks = std::min(blocks, device_cus());
    const int cap = std::max(1, (int)(blocks * share) / std::max(1, nslots));
    return (int)std::min<unsigned>(ngroups, (unsigned)cap);
}

template <typename T>
static hipError_t sweep_t(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int which, int mode,
                          hipStream_t s, float share, int stage, bool decide) {
    switch (which) {
        case 1: return launch_resid<T>(g, t, slots, nslots, mode, s, share, decide);
        case 2:
            return g.ny <= kShortLine ? launch_cols_y<T, true>(g, t, slots, nslots, mode, s, share, stage)
                                      : launch_cols_y<T, false>(g, t, slots, nslots, mode, s, share, stage);
        case 3:
            return g.nz <= kShortLine ? launch_z_solve<T, true>(g, t, slots, nslots, mode, s, share, stage)
                                      : launch_z_solve<T, false>(g, t, slots, nslots, mode, s, share, stage);
        case kSweepPlanes: return launch_planes<T>(g, t, slots, nslots, mode, s, share, stage);
        case 5: return launch_update<T>(g, t, slots, nslots, mode, s, share, stage);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sweep_mode(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, bool fp32, int which,
                             int mode, hipStream_t s, float share, int stage, bool decide) {
    if (mode == 1) stage = 1;
    return fp32 ? sweep_t<float>(g, t, slots, nslots, which, mode, s, share, stage, decide)
                : sweep_t<double>(g, t, slots, nslots, which, mode, s, share, 1, decide);
}

// Planes of up to 48 x 48 values while the launch's columns are few: a larger
// plane's chain of transforms, or many columns' access (16 or 8 bytes per row),
// takes longer than the sweeps it replaces.  The bits are the same either way, so
// the batch may decide.  Whole solves, three launches / one, us: FP64 32^3
// 411 / 358, 24 x 48 x 64 430 / 381, 48^3 429 / 417, 32 x 64 x 64 426 / 400, 48 x 48 x
// 512 741 / 725 (but x 1024 944 / 981, and 64^3 403 / 426); FP32 + refinement 434 /
// 386, 457 / 405, 449 / 432, 453 / 416, 619 / 618 (but 64^3 465 / 480, and 40 served
// ones 4861 / 6560).
bool planes_fusable(const GridArgs& g, int nslots) {
    if (g.ny < 16 || g.ny > 64 || g.nz < 16 || g.nz > 64) return false;
    return g.ny * g.nz <= 48 * 48 && (long long)g.ny * g.nz * g.nxh * nslots <= 48 * 48 * 256;
}

unsigned sweep_groups_x(const GridArgs& g) {
    // line groups of P1 at the FP64 and FP32 configurations (the larger)
    unsigned out = 0;
    (void)dispatch_len(g.nx, [&]<int N>() {
        const unsigned rows = (unsigned)(g.ny * g.nz / 2);
        out = std::max((rows + LineCfg<double, N>::L - 1) / LineCfg<double, N>::L,
                       (rows + LineCfg<float, N>::L - 1) / LineCfg<float, N>::L);
        return hipSuccess;
    });
    return out;
}

}  // namespace pois
