// Internal declarations of the lattice transfer kernels (not part of the C ABI).
#pragma once

#include "okpz_internal.h"

namespace okpz {

// Canonical bytes (one per site, physical columns) of rows [y0, y0 + n) of
// lattice view v into the device buffer bytes (n * Lx); y0 + n <= Ly.
hipError_t launch_unpack_rows(const LatticeView &v, int32_t y0, int32_t n, uint8_t *bytes, hipStream_t st);

// The inverse for an unrotated copy (v.ox = 0): rows [y0, y0 + n) of v from
// canonical bytes.  Sets state[0] to 1 if a byte is above 3.
hipError_t launch_pack_rows(const LatticeView &v, int32_t y0, int32_t n, const uint8_t *bytes, int64_t *state,
                            hipStream_t st);

// Slope field test of a whole copy, any rotation.  state[0]: not zero if some
// plaquette is open (or a byte was bad, above); state[1]: sigma_x = +1 bonds of
// row 0; state[2]: sigma_y = +1 bonds of stored column 0.  clear_check_state
// first zeroes the three words.
hipError_t launch_clear_check_state(int64_t *state, hipStream_t st);
hipError_t launch_check_planes(const LatticeView &v, int64_t *state, hipStream_t st);

// Bytes of a staging buffer for transfers in chunks of whole rows: the whole
// lattice up to 16 MiB.
inline size_t io_bytes(int64_t Lx, int64_t Ly)
{
    const int64_t most = (int64_t(16) << 20) / Lx;  // rows, at least 16 (Lx <= 2^20)
    return (size_t)(Lx * (Ly < most ? Ly : most));
}

// Rows [y0, y0 + n) (mod Ly) of v as canonical bytes in host memory, through
// the device staging buffer io of io_size >= Lx bytes.  Returns when they are
// there.
hipError_t download_rows(const LatticeView &v, int64_t y0, int64_t n, uint8_t *host, void *io, size_t io_size,
                         hipStream_t st);

}  // namespace okpz
