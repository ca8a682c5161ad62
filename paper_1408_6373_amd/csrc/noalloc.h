// noalloc.h -- the device scratch of the allocation-free DoSample entry point
// (ccuba_vegas_dosample_raw_noalloc).
#pragma once
#include <hip/hip_runtime.h>

#include "engine.h"

namespace ccuba {

// Size of the scratch array every device holds for the process's lifetime.
constexpr size_t kNoallocScratchBytes = (size_t)16 << 20;

// Records, once per device and with that device current, the device address
// of the scratch array.  Returns CCUBA_OK, CCUBA_EINVAL (device index beyond
// the table) or CCUBA_EHIP (the runtime could not give the address).
int noalloc_init(int device);
// The recorded address of the device's scratch array, or nullptr.
void *noalloc_scratch(int device);

// The descriptors of one integral, passed by value to a kernel that writes
// them to device memory (kernel arguments need no host buffer that must
// outlive the call, nor a copy to wait for).
struct JobSetup {
  VJob job;
  VState st;
  double p64[2][kParamRow];
  float p32[2][kParamRow];
  long long end;  // the fold tasks of the one job
  VJob *job_dst;        // (null: the descriptor is not wanted)
  VState *st_dst;
  double *p64_dst;      // (null: not wanted)
  float *p32_dst;       // (null: not wanted)
  long long *end_dst;   // (null: not wanted)
  double *grid_dst;     // the uniform starting grid goes here (null: none)
};
hipError_t launch_job_setup(const JobSetup &S, hipStream_t s);

}  // namespace ccuba
