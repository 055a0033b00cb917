// What the serving layer and the other entry points need to know about each
// other (internal).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "hac.h"

namespace hac {

struct CtxInfo {
    int device;
    int cus;
    int wallclock_khz;
    size_t lds_max;      // dynamic LDS a launch may request
    int64_t timeout_ms;  // 0 = default
    bool lazy;           // HAC_OPT_LAZY_MIRROR
};
void ctx_info(const hac_ctx *c, CtxInfo *out);

// Compute units of a device that this process's serving kernels hold at the moment.
int serving_cus(int device);

}  // namespace hac
