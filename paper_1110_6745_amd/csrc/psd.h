// Internal declarations of the spectrum pass (not part of the C ABI).
#pragma once

#include "okpz_internal.h"

namespace okpz {

// Power spectrum along the lattice axes: scratch layout (byte offsets into one
// device allocation of `bytes`) and launch.  Also needs the width's rows scratch
// (2 Ly words of it).  Leaves S along x (Lx/2+1 doubles) followed by S along y
// (Ly/2+1 doubles) at off_spec.
struct PsdPlan {
    int32_t R, nch;  // rows per workgroup of the plane pass, number of such chunks
    size_t off_rowpart, off_zx, off_zy, off_conv, off_spec, off_prefix, off_blk, bytes;
    bool together;  // both axes' transforms in the same launches
};
PsdPlan psd_plan(int64_t Lx, int64_t Ly);
// The same with taller chunks and the axes one after the other, as far as needed to
// bring the scratch down to max_bytes if possible (check .bytes against the cap).
PsdPlan psd_plan_capped(int64_t Lx, int64_t Ly, size_t max_bytes);
hipError_t launch_psd(const LatticeView &v, const PsdPlan &p, int64_t *rows, void *scratch, hipStream_t st);

}  // namespace okpz
