// Internal interface of the contraction engine (hac_contract.hip): single and
// complete linkage by rounds of merges on a shrinking matrix.  Not installed;
// the public interface is hac.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hac_engine.h"
#include "hac_rounds.h"

namespace hac {

constexpr int kContractBlock = 1024;   // threads per workgroup
constexpr int kContractMaxN = 32768;   // a row fits one workgroup's registers and LDS

// Workgroups that m clusters keep busy, of at most G: the barriers of fewer cost
// less (n = 512: 327 us for the call on 256, 330 on 64, 340 on 16, 365 on 8; n = 1500: 423 on
// 256, 428 on 128, 437 on 64; n = 150: 257 on 256, 249 on 16).
__host__ __device__ constexpr int contract_workgroups(int m, int G) {
    const int k = m > 4096 ? G : m > 1024 ? 128 : m > 256 ? 64 : m > 64 ? 16 : 4;
    return k < G ? k : G;
}

struct ContractCtl {
    uint32_t bar;                      // grid barrier arrivals (monotonic)
    uint32_t abort;                    // set by a workgroup that gives up
    uint32_t merges;                   // at a hand-over: merges done (read as Resume::state[0])
    uint32_t round;                    //   and rounds run (Resume::state[1])
};

// Device workspace; offsets in bytes from the workspace base.
struct ContractLayout {
    size_t ctl, rank;       // cleared before a launch: zero_bytes from the start
    size_t zero_bytes;
    size_t nn[2], ties[2], val[2], slot[2], size[2], part, pcnt, rec, key, live, hsize, bytes;
};
ContractLayout contract_layout(int n);

// Workgroups of the kernel that fit on one CU; also sets its LDS limit.
int contract_occupancy(int link);

// The rounds of HAC_SINGLE or HAC_COMPLETE on G co-resident workgroups, from
// the symmetric matrix written by the set-up kernel.  Records (claim order,
// with sort keys) stay in the workspace until launch_rank writes them in merge
// order.  Hands over as launch_rounds does (kHandover, contract_resume), and with
// kFlagInplaceNext in `flags` (complete linkage) leaves the rest to a launch_rounds
// queued behind it on the layout contract_rounds_layout (kInplace in `status`) when
// rounds have too few pairs to stream the matrix for them.
// At a hand-over the live rows' minima go to `rowkey` (Instance::rowkey).
hipError_t launch_contract(float *D, int n, int link, uint32_t *status, Control *ctl, uint64_t *rowkey, void *ws, int G,
                           uint64_t timeout_ticks, int flags, hipStream_t stream);
Resume contract_resume(int n, void *ws);
// Workspace of that launch_rounds, on the same base: its own words follow the
// contraction engine's (ctl: to be cleared, sizeof(RoundsCtl)); records, keys, live
// mask, sizes and hand-over state are the same, so that contract_resume serves both.
RoundsLayout contract_rounds_layout(int n, int G);

}  // namespace hac
