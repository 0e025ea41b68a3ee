// Several Monte Carlo sweeps of a small lattice (Sec. II, Eq. (1)) in one launch
// on gfx950.
//
// A lattice whose blocks fit one workgroup (at most 1024 cells: one 256 x 256
// block, or up to 64 smaller ones) needs no other workgroup between sweeps, so
// one workgroup runs them in a row, handing the lattice from sweep to sweep
// through its own CU's caches.  What bounds such a lattice is the chain of one
// sweep's 64 barriered steps; a launch of its own per sweep adds about a
// microsecond to it (256 x 256, p = 1, q = 0: 17.9 us per sweep in launches of
// one, 16.9 us in launches of ten).
//
// Unlike the other 1024-thread kernels these may take more than 80 scalar registers, which
// leaves them one workgroup per CU: a launch is one workgroup, and the four hardware queues
// of a process run four such launches at a time (64 to 512 lattices of 256 x 256 on
// streams of their own: 4.26 us per sweep and lattice, a quarter of one lattice's
// 16.9).  Capped at 80 they spill scalar registers and a sweep is 1 to 4 % slower.
#include "sweep_core.h"

namespace okpz {
namespace {

template <int kMode, int kFixedB, bool kLaneOrg>
__global__ __launch_bounds__(1024) void sweep_chain_kernel(SweepLaunch a, int n)
{
    __shared__ __align__(16) uint8_t tile[kFixedB ? core::kPitch + kFixedB * core::kPitch : core::kGroupLds];
    __shared__ uint32_t opk_fix[kFixedB ? 32 : 1];
    const int G = a.ncol * a.nby;
    uint32_t *const opk = kFixedB ? opk_fix : reinterpret_cast<uint32_t *>(tile + core::tile_bytes(a.Bx, a.By, G));
    uint32_t *const copy0 = const_cast<uint32_t *>(a.src), *const copy1 = a.dst;
    for (int i = 0; i < n; ++i) {
        const Ctr4 r = philox10(Ctr4{a.s, 0, 0, kTagShift}, a.k0, a.k1);
        a.sx = (int32_t)below(r.x, (uint32_t)a.Bx);
        a.sy = (int32_t)below(r.y, (uint32_t)a.By);
        const int x00 = a.sx ? a.Lx - a.sx : 0, y00 = a.sy ? a.Ly - a.sy : 0;
        a.blk00 = (y00 / a.By) * a.nbx + x00 / a.Bx;
        a.u00 = x00 & (a.Bx - 1);
        a.v00 = y00 & (a.By - 1);
        a.src = (i & 1) ? copy1 : copy0;
        a.dst = (i & 1) ? copy0 : copy1;
        core::sweep_group<1024, kMode | core::kEagerReads, kFixedB, false, kLaneOrg>(a, 0, G, tile, opk);
        a.ox_src = a.sx;
        a.s += 1;
        // the stored words reach the workgroup's other waves, and the tile is free
        __syncthreads();
    }
}

template <int kMode>
hipError_t launch_m(const SweepLaunch &a, int n, hipStream_t st)
{
    const dim3 one(1), threads(1024);
    if (a.Bx == core::kMaxB && a.By == core::kMaxB)
        hipLaunchKernelGGL((sweep_chain_kernel<kMode, core::kMaxB, false>), one, threads, 0, st, a, n);
    else if (a.Bx * a.By >= 128 * 128)
        hipLaunchKernelGGL((sweep_chain_kernel<kMode, 0, false>), one, threads, 0, st, a, n);
    else
        hipLaunchKernelGGL((sweep_chain_kernel<kMode, 0, true>), one, threads, 0, st, a, n);
    return hipGetLastError();
}

template <int kCells>
hipError_t launch_c(const SweepLaunch &a, int n, hipStream_t st)
{
    if (a.need_accept_draws) return launch_m<core::kDraw | kCells>(a, n, st);
    if (a.Tp == uint64_t(1) << 32 && a.Tq == 0) return launch_m<core::kGrowth | kCells>(a, n, st);
    return launch_m<core::kFixed | kCells>(a, n, st);
}

}  // namespace

bool sweep_chain_ok(const SweepLaunch &a, int threads)
{
    const int nblk = a.nbx * a.nby;
    return threads == 1024 && !a.in_place && core::group_size(a.Bx, a.By, nblk) >= nblk;
}

hipError_t launch_sweep_chain(const SweepLaunch &a, int n, hipStream_t st)
{
    SweepLaunch b = a;
    b.col0 = 0;
    b.col_step = 1;
    b.ncol = a.nbx;
    return a.delayed_cells ? launch_c<core::kDelayedCells>(b, n, st) : launch_c<0>(b, n, st);
}

}  // namespace okpz
