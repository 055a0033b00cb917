// Internal interface of the ordered-round engine (hac_order.hip): group
// average, weighted average and Ward linkage, several merges per exchange in
// the sequential order.  Not installed; the public interface is hac.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hac_engine.h"

namespace hac {

constexpr int kOrderBlock = 1024;    // threads per workgroup
constexpr int kOrderMaxPairs = 64;   // merges per round at most
constexpr int kOrderMaxGroup = 256;  // workgroups at most
constexpr int kOrderAllToAll = 128;  // up to here every workgroup reads every slot; above, workgroup 0 does
// Exchange slot of one workgroup: header, smallest pair, other pairs and one
// partial row minimum per merge of the previous round, 16 bytes each.
constexpr int kOrderUnits = 2 + 2 * kOrderMaxPairs;
constexpr int kOrderSlotWords = (2 * kOrderUnits + 15) / 16 * 16;

// Device workspace; offsets in bytes from the workspace base.
struct OrderLayout {
    size_t rk, m2, size, vsize, live, state, slots, bytes;
};
OrderLayout order_layout(int n, int G);

// Columns (= rows) per workgroup for n items: the smallest power of two from
// 64 to 1024 that needs at most `want` workgroups; 0 if even 1024 needs more.
int order_columns(int n, int want);
// Workgroups of the kernel for `columns` that fit on one CU; also sets its LDS limit.
int order_occupancy(int n, int columns, int link);

// Row minima of the symmetric matrix, then the merge kernel on
// ceil(n / columns) co-resident workgroups.  Records go to `out` in merge
// order.  With kFlagNoHandover in `flags` it makes every merge; otherwise it
// leaves the rest to a k_run launch queued behind it (kHandover in `status`,
// state from order_resume, the live rows' minima in `rowkey`) when rounds make
// few merges each.
// The workspace must be zero from `state` on.
hipError_t launch_order(float *D, int n, int link, hac_merge *out, uint32_t *status, Control *ctl, uint64_t *rowkey,
                        void *ws, int columns, uint64_t timeout_ticks, int flags, hipStream_t stream);
Resume order_resume(int n, int G, void *ws);

}  // namespace hac
