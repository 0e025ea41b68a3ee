// The fixed device scratch of a GPU (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <mutex>

namespace okpz {

// One array per GPU, held until the process ends, never allocated or freed by a call:
// the scratch of okpz_psd_noalloc and the staging of lattice transfers.  An object is
// one turn at it: made once `stream` has no earlier work left to do (a turn should
// not wait for that), and over when it is destroyed, which first waits for the turn's own
// work on the stream.  Turns of all threads follow one another.
class StaticScratch {
public:
    static constexpr size_t kBytes = size_t(24) << 20;
    StaticScratch(int device, hipStream_t stream);
    ~StaticScratch();
    StaticScratch(const StaticScratch &) = delete;
    StaticScratch &operator=(const StaticScratch &) = delete;
    void *mem() const { return mem_; }  // nullptr: error()
    hipError_t error() const { return err_; }

private:
    std::unique_lock<std::mutex> turn_;
    hipStream_t stream_;
    void *mem_;
    hipError_t err_;
};

}  // namespace okpz
