// Scratch layout and split of the spectrum pass.  Plain C++, so that its bounds can
// be checked on the CPU for every size.
#pragma once

#include <cstddef>
#include <cstdint>

namespace okpz {

constexpr int kPlaneThreads = 512;
constexpr int kPlaneWaves = kPlaneThreads / 64;
constexpr int kStripWords = 256;          // words of a row a wavefront takes: four per lane
constexpr int kStripCols = 32 * kStripWords;
constexpr int kGroupRows = 8;             // rows per carry-save group
constexpr int kMaxWaveRows = 255 * kGroupRows;  // byte lanes count up to 255 groups
constexpr int kPlaneTarget = 512;         // workgroups of the plane pass
constexpr int kProfThreads = 256;

// Power spectrum along the lattice axes: scratch layout (byte offsets into one
// device allocation of `bytes`).  S along x (Lx/2+1 doubles) followed by S along y
// (Ly/2+1 doubles) end up at off_spec.
struct PsdPlan {
    int32_t R, nch;  // rows per workgroup of the plane pass, number of such chunks
    size_t off_rowpart, off_zx, off_zy, off_conv, off_spec, off_prefix, off_blk, bytes;
    bool together;  // both axes' transforms in the same launches
    // Row sums added up in the rows scratch instead of kept per strip, and column
    // counters added up every kMaxWaveRows rows, so that neither grows with the lattice.
    bool tall;
};

PsdPlan psd_plan(int64_t Lx, int64_t Ly);
// The same with taller chunks and the axes one after the other, as far as needed to
// bring the scratch down to max_bytes if possible (check .bytes against the cap).
PsdPlan psd_plan_capped(int64_t Lx, int64_t Ly, size_t max_bytes);

// What okpz_psd may allocate (okpz.h): min(32 MiB, Lx Ly / 4) + 40 max(Lx, Ly) bytes,
// 128 max(Lx, Ly) more when a side is not a power of two, and 2 KiB for the pieces'
// alignment.
size_t psd_scratch_bound(int64_t Lx, int64_t Ly);

// Bluestein length for a side n: the power of two M >= 2n - 1.
inline int64_t conv_len(int64_t n)
{
    int64_t M = 1;
    while (M < 2 * n - 1) M <<= 1;
    return M;
}

inline bool pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }

// Blocks of kProfThreads values of a profile.
inline int32_t blocks_of(int64_t n) { return (int32_t)((n + kProfThreads - 1) / kProfThreads); }

}  // namespace okpz
