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

// Tests: single and complete linkage by rounds of this context in place at every size
// (on = 1), not only above kContractMaxN (0, the default).  Not part of hac.h.
extern "C" int hac_internal_rounds_in_place(hac_ctx *c, int on);

// Tests and measurements: exchanges of the context's last completed hac_run if it went
// through the ordered-round engine (0 otherwise), and whether that handed over.
// hac_stats.rounds and handed_over stay 0 for it.  Not part of hac.h.
extern "C" int hac_internal_ordered_rounds(const hac_ctx *c, int32_t *rounds, int32_t *handed_over);

// Compute units of a device that this process's serving kernels hold at the moment.
int serving_cus(int device);

}  // namespace hac
