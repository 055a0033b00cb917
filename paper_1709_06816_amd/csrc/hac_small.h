// Internal interface of the small-instance kernel (hac_small.hip): a whole run
// in one workgroup's LDS.  Not installed; the public interface is hac.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hac_engine.h"

namespace hac {

constexpr int kSmallMaxN = 192;  // 192 x 193 floats of LDS
// Row pitch of the matrix in LDS: odd, so that a column's entries fall into banks of
// their own as a row's do.
__host__ __device__ constexpr int small_pitch(int n) { return n | 1; }

// LDS limit of the kernel; call once per device.
hipError_t small_setup();

// Cluster the n-item instance whose strict upper triangle is at `src`
// (row-major, leading dimension n; only read).  Writes the records to `out`,
// and the control block and the status word whole (nothing to clear before).
hipError_t launch_small(const float *src, int n, int link, hac_merge *out, uint32_t *status, Control *ctl,
                        hipStream_t stream);

}  // namespace hac
