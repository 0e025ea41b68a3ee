// Lattice transfers between the packed bit planes and the canonical host layout
// (one byte per site) on gfx950: rotation, bits <-> bytes and the slope field test
// run on the device, the host only copies.
//
// What bounds them: the copy of one byte per site over PCIe (18 GB/s from pageable
// memory to the host, 31 GB/s to the device, measured at 256 MiB); the kernels move
// 1.25 bytes per site at HBM rate.  A 4096 x 4096 lattice set, saved, restored and
// read back took 230 ms with per-site loops on the host.
#include "state_io.h"

namespace okpz {
namespace {

constexpr int kThreads = 256;

// 4 bits -> bit 0 of 4 bytes: nib * (1 + 2^7 + 2^14 + 2^21) puts bit j at j + 7 i,
// all distinct; byte j keeps i = j
__device__ __forceinline__ uint32_t bytes_of(uint32_t nib) { return __umul24(nib, 0x204081u) & 0x01010101u; }

// Thread: 16 sites of a row (one 16-byte store), x0 = 16 i.
__global__ __launch_bounds__(kThreads) void unpack_rows_kernel(LatticeView v, int32_t y0, int32_t n, uint8_t *bytes)
{
    const int per = v.Lx >> 4;
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= (int64_t)n * per) return;
    const int r = (int)(e / per), x0 = (int)(e - (int64_t)r * per) << 4;
    int c = x0 - v.ox;
    if (c < 0) c += v.Lx;
    const int w = c >> 5;
    const uint32_t sh = (uint32_t)(c & 31);
    const int w1 = w + 1 == v.W ? 0 : w + 1;
    const uint32_t *rx = v.planes + (size_t)(y0 + r) * v.W, *ry = rx + (size_t)v.Ly * v.W;
    const uint32_t bx = __builtin_amdgcn_alignbit(rx[w1], rx[w], sh);
    const uint32_t by = __builtin_amdgcn_alignbit(ry[w1], ry[w], sh);
    uint32_t d[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        d[k] = bytes_of((bx >> (4 * k)) & 15u) | (bytes_of((by >> (4 * k)) & 15u) << 1);
    *reinterpret_cast<uint4 *>(bytes + (size_t)r * v.Lx + x0) = uint4{d[0], d[1], d[2], d[3]};
}

// Thread: one word of each plane (32 sites, two 16-byte loads).
__global__ __launch_bounds__(kThreads) void pack_rows_kernel(LatticeView v, int32_t y0, int32_t n,
                                                             const uint8_t *bytes, int64_t *state)
{
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= (int64_t)n * v.W) return;
    const int r = (int)(e / v.W), w = (int)(e - (int64_t)r * v.W);
    const uint4 *src = reinterpret_cast<const uint4 *>(bytes + (size_t)r * v.Lx + 32 * (size_t)w);
    const uint4 a = src[0], b = src[1];
    const uint32_t d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t bx = 0, by = 0, high = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        high |= d[k] & 0xFCFCFCFCu;
        // byte weights 1, 2, 4, 8: four sites' bits as one nibble
        bx |= __builtin_amdgcn_udot4(d[k] & 0x01010101u, 0x08040201u, 0u, false) << (4 * k);
        by |= __builtin_amdgcn_udot4((d[k] >> 1) & 0x01010101u, 0x08040201u, 0u, false) << (4 * k);
    }
    uint32_t *rx = v.planes + (size_t)(y0 + r) * v.W;
    rx[w] = bx;
    rx[(size_t)v.Ly * v.W + w] = by;
    if (high) state[0] = 1;
}

__global__ void clear_check_state_kernel(int64_t *state)
{
    if (threadIdx.x < 3) state[threadIdx.x] = 0;
}

// Thread: one word; plaquettes a = sx(x,y), b = sy(x+1,y), c = sx(x,y+1),
// d = sy(x,y) close iff a + b = c + d, that is (a ^ b) == (c ^ d) and
// (a & b) == (c & d).  With all closed, row 0 and column 0 stand for the rest.
__global__ __launch_bounds__(kThreads) void check_planes_kernel(LatticeView v, int64_t *state)
{
    const int64_t total = (int64_t)v.Ly * v.W;
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < total; e += (int64_t)gridDim.x * kThreads) {
        const int y = (int)(e / v.W), w = (int)(e - (int64_t)y * v.W);
        const uint32_t *rx = v.planes + (size_t)y * v.W, *ry = rx + (size_t)v.Ly * v.W;
        const uint32_t *rx1 = y + 1 == v.Ly ? v.planes : rx + v.W;
        const uint32_t a = rx[w], d = ry[w], c = rx1[w];
        const uint32_t b = (d >> 1) | (ry[w + 1 == v.W ? 0 : w + 1] << 31);
        if (((a ^ b) != (c ^ d)) | ((a & b) != (c & d))) state[0] = 1;
        unsigned long long *count = reinterpret_cast<unsigned long long *>(state);
        if (y == 0) atomicAdd(count + 1, (unsigned long long)__popc(a));
        if (w == 0) atomicAdd(count + 2, (unsigned long long)(d & 1u));
    }
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

hipError_t launch_unpack_rows(const LatticeView &v, int32_t y0, int32_t n, uint8_t *bytes, hipStream_t st)
{
    hipLaunchKernelGGL(unpack_rows_kernel, dim3(blocks_for((int64_t)n * (v.Lx >> 4))), dim3(kThreads), 0, st, v, y0,
                       n, bytes);
    return hipGetLastError();
}

hipError_t launch_pack_rows(const LatticeView &v, int32_t y0, int32_t n, const uint8_t *bytes, int64_t *state,
                            hipStream_t st)
{
    hipLaunchKernelGGL(pack_rows_kernel, dim3(blocks_for((int64_t)n * v.W)), dim3(kThreads), 0, st, v, y0, n, bytes,
                       state);
    return hipGetLastError();
}

hipError_t launch_clear_check_state(int64_t *state, hipStream_t st)
{
    hipLaunchKernelGGL(clear_check_state_kernel, dim3(1), dim3(64), 0, st, state);
    return hipGetLastError();
}

hipError_t launch_check_planes(const LatticeView &v, int64_t *state, hipStream_t st)
{
    const int64_t n = (int64_t)v.Ly * v.W;
    const unsigned blocks = n > (int64_t)65536 * kThreads ? 65536u : blocks_for(n);
    hipLaunchKernelGGL(check_planes_kernel, dim3(blocks), dim3(kThreads), 0, st, v, state);
    return hipGetLastError();
}

hipError_t download_rows(const LatticeView &v, int64_t y0, int64_t n, uint8_t *host, void *io, size_t io_size,
                         hipStream_t st)
{
    const int64_t most = (int64_t)(io_size / (size_t)v.Lx);
    hipError_t e = hipSuccess;
    for (int64_t done = 0; done < n && e == hipSuccess;) {
        const int64_t y = (y0 + done) % v.Ly;
        int64_t run = n - done < v.Ly - y ? n - done : v.Ly - y;
        if (run > most) run = most;
        e = launch_unpack_rows(v, (int32_t)y, (int32_t)run, static_cast<uint8_t *>(io), st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(host + (size_t)done * v.Lx, io, (size_t)run * v.Lx, hipMemcpyDeviceToHost, st);
        done += run;
    }
    const hipError_t s = hipStreamSynchronize(st);
    return e != hipSuccess ? e : s;
}

}  // namespace okpz
