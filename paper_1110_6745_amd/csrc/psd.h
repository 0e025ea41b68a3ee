// Internal declarations of the spectrum pass (not part of the C ABI).
#pragma once

#include "okpz_internal.h"
#include "psd_plan.h"

namespace okpz {

// The spectra, by plan p in scratch of p.bytes (psd_plan.h).  Also needs the width's rows
// scratch (1.5 Ly words of it; 3 Ly if p.tall).
hipError_t launch_psd(const LatticeView &v, const PsdPlan &p, int64_t *rows, void *scratch, hipStream_t st);

}  // namespace okpz
