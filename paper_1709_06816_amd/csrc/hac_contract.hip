// Contraction engine: single and complete linkage by rounds of merges on a
// matrix that shrinks with every round (n <= 32768).
//
// Which pairs a round merges, and why sorting the records by (height, i,
// round) gives the sequential list of Section 4, is stated in hac_rounds.hip:
// complete linkage merges every reciprocal nearest-neighbour pair, single
// linkage the globally closest pair and every reciprocal pair whose distance is
// the only minimum of both rows.  This engine differs in how a round is applied.
// Updating the merged rows and columns in place costs one 4-byte store per
// entry of a column, each a read-modify-write of a memory sector, and
// rescans that read retired columns.  On clustered points 8 to 16 percent of
// the clusters merge in a round, so that nearly every cache line of the matrix
// holds a changed entry anyway: here a round streams the whole matrix once
// instead, D' = D with rows and columns i and j of every pair replaced by their
// minimum / maximum and retired columns closed up, and takes every row's next
// minimum from the values on their way out.
//
// Layout: live clusters are numbered 0 .. m-1 in slot order (so that ties
// resolve as on the slots); row r starts at D + slot[r] * n and holds its m
// entries contiguously.  A merged pair's row is written where the survivor's
// was, so the contraction is in place: a row (and its partner's) is read and
// written by one workgroup only, whole before the first store.
//
// A round, on G co-resident workgroups, one grid barrier each:
//   every workgroup reads the nearest neighbour of every row (2 bytes each),
//   finds the pairs, and derives from the retired columns' bit mask and its
//   prefix counts where every column goes; then it contracts its share of the
//   rows: T threads per row load it (and the partner's), fold every column
//   into its new place in LDS (LDS minimum / maximum: a survivor's place gets
//   both), and store the row from LDS with its minimum taken on the way.
//   The next row's first loads are in flight meanwhile.
//
// A round streams the matrix however few its pairs are.  Single linkage, which
// has few, updates their rows and columns in place in between (kRetired); complete
// linkage leaves such runs to the in-place engine (cheaper_in_place), and both leave
// the last merges, or all of a run on tied input, to the one-merge-per-step kernel.
//
// What bounds it: memory bandwidth while m is large (read m^2, write m'^2
// entries per round), the chain barrier -> nearest neighbours -> row ->
// barrier below a few thousand clusters.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hac_contract.h"
#include "hac_dev.h"

namespace hac {
namespace {

constexpr int B = kContractBlock, W = B / 64;
constexpr int KE = 32;                       // columns per thread and row at most
constexpr int U = 8;                         // columns per thread loaded at once
constexpr int V = 4;                         // the same for in-place updates
constexpr int kMaxM = kContractMaxN;
constexpr int kWords = kMaxM / 64;
constexpr uint64_t kNone = ~0ull;
constexpr uint32_t kNowhere = 0xFFFFu;       // no column's place
constexpr uint32_t kIndex = 0x7FFFu;
constexpr uint32_t kTied = 0x8000u;          // nearest-neighbour entry: the minimum is attained more than once
constexpr int kWindow = 8;                   // hand-over, as in hac_rounds.hip
constexpr int kMinPerRound = 12;
constexpr int kHandoverLeft = 96;            // the last merges are made here: they cost little
// Up to this size the kernel behind is one workgroup, a merge there cheaper, and the
// hand-over (its start, the rows back to their slots) dear: from the second round on
// what is left is priced both ways, at the last rounds' pace (eight rounds below 12
// pairs and 96 merges left / this rule / one merge per step alone: single linkage,
// uniform values, n = 208 1.12 / 0.49 / 0.62 ms, RMSD-like n = 320 0.82 / 0.45 / 0.99, 50
// distinct values n = 320 1.04 / 0.87 / 0.75).
constexpr int kSmallN = 1536;
__device__ __forceinline__ bool cheaper_behind(int recent, int rounds, int left, int n) {
    const float merge_us = fminf(4.5f, 1.3f + 0.004f * (float)n), round_us = 12.0f, start_us = 150.0f;
    return (float)left * (round_us * (float)rounds - merge_us * (float)recent) > start_us * (float)recent;
}

constexpr int kWideMin = 4096;
constexpr int kInplaceMin = 1024;            // smaller matrices are contracted every round
// Columns per retired column at which single linkage contracts.  A contraction streams
// the matrix, in between every row carries the retired columns along.  12 / 6 / 4 / 3: points
// growing in 150 chains, n = 32768, 43.2 / 38.6 / 37.2 / 37.3 ms; mixture of 32 clusters
// in 3 dimensions 28.0 / 28.1 / 28.7 / 32.0, in 16 dimensions 50.0 / 48.3 / 47.4 / 48.4, and
// at n = 8192 6.16 / 5.92 / 5.97 / 5.92.
constexpr int kRetired = 6;
// Complete linkage leaves the rest to the in-place round engine when two rounds
// running, or the first, have fewer pairs than this.  With p pairs in every round that is left, m
// clusters cost m / p rounds here of 0.63e-6 m^2 us on average (a third of the
// first one's 8 m^2 bytes at 4.2 TB/s), there of 40 us more than here for the
// barriers and about 3.5e-5 n us a pair (column stores, rescans of full rows).
// Points on C lines, which merge about 2 C pairs a round; streamed / in place from the
// start / this rule: n = 32768, C = 16: 650 / 82 / 81 ms, C = 150: 78 / 37 / 38, C = 400:
// 34 / 32 / 32, C = 1000: 17 / 26 / 17; n = 16000, C = 16: 91 / 33 / 33, C = 250: 7.9 /
// 8.6 / 7.9.  Up to 8192 items rounds here are never the dearer ones (n = 8192, C = 16:
// 15.3 / 15.4, C = 40: 6.7 / 9.1), and no engine is queued behind.
__device__ __forceinline__ bool cheaper_in_place(int np, int m, int n) {
    return (float)np * (3.5e-5f * (float)n) < 0.63e-6f * (float)m * (float)m - 40.0f;
}
static_assert(KE * B == kMaxM && KE == 4 * U, "a row takes one workgroup, four chunks");

// LDS (dynamic), byte offsets.  The row area holds the rows on their way;
// before the first of a round, the nearest neighbours and the columns' places
// (2 bytes each).
constexpr uint32_t kRowArea = (kMaxM + 64) * 4;
constexpr uint32_t oRow = 0;
constexpr uint32_t oRet = oRow + kRowArea;   // u64 per 64 columns: retired this round
constexpr uint32_t oSur = oRet + kWords * 8; // u64: survivors of a merge
constexpr uint32_t oDead = oSur + kWords * 8;  // u64: retired in earlier rounds, columns still there (single)
constexpr uint32_t oPre = oDead + kWords * 8;  // u16: kept columns before each word
constexpr uint32_t oPrs = oPre + (kWords + 8) * 2;  // u16: survivors before each word
constexpr uint32_t kLdsBytes = oPrs + (kWords + 8) * 2;

extern __shared__ __align__(16) uint8_t smem[];
template <class T> __device__ __forceinline__ T *lds(uint32_t off) { return reinterpret_cast<T *>(smem + off); }

struct Args {
    float *D;
    uint32_t *status;
    Control *ctl;
    ContractCtl *cc;
    uint16_t *nn[2];      // complete: nearest neighbour (smallest index among equals)
    uint32_t *ns[2];      // single: the same, a word each, and how many columns attain the minimum
    uint32_t *ties[2];
    uint64_t *part;       // single, in place: smallest entry (ord:32 | column) of every part of a row
    uint32_t *pcnt;       // and how many columns attain it
    uint32_t *val[2];     // its distance (ord)
    int32_t *slot[2];
    int32_t *size[2];
    int4 *rec;            // records in claim order, with their sort keys
    uint64_t *key;
    uint32_t *live;       // hand-over: live mask and sizes by slot
    int32_t *hsize;
    uint64_t *rowkey;     //   and the live rows' minima over the live columns to their right
    uint64_t timeout;
    int n, flags;
};

__device__ __forceinline__ void st32(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st64(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st16(uint16_t *p, uint16_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Start of the row kept at slot s: once it is at least three entries shorter
// than its storage, at the first 16-byte boundary there.
__device__ __forceinline__ float *row_at(float *D, int n, int s, bool aligned) {
    float *p = D + (size_t)s * n;
    return aligned ? reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(p) + 15) & ~(uintptr_t)15) : p;
}

// Grid barrier.  Agent-scope stores are at the device's point of coherence once
// complete; `writeback` writes this XCD's L2 back first (after plain stores).
__device__ bool arrive_and_wait(const Args &A, uint32_t &target, uint32_t G, bool stall, bool writeback = false) {
    __shared__ uint32_t s_stop;
    barrier_stores_done();
    if (threadIdx.x == 0) {
        if (writeback) release_agent();
        target += G;
        if (!stall) __hip_atomic_fetch_add(&A.cc->bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t stop = 0;
        const uint64_t t0 = wall_clock64();
        for (uint32_t it = 1;; ++it) {
            if (__hip_atomic_load(&A.cc->bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target) break;
            if ((it & 63u) == 0) {
                if (__hip_atomic_load(&A.cc->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    stop = 1;
                    break;
                }
                if (wall_clock64() - t0 > A.timeout) {
                    atomicOr(&A.ctl->error, kErrTimeout);
                    __hip_atomic_store(&A.cc->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    stop = 1;
                    break;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        s_stop = stop;
    }
    __syncthreads();
    return s_stop == 0;
}

// Smallest entry of a row as its threads see it: value, smallest column
// attaining it, number of columns attaining it.
struct Low {
    uint32_t o = 0xFFFFFFFFu;
    int c = 0, cnt = 0;
    template <bool kCount> __device__ __forceinline__ void take(uint32_t v, int col) {
        if (v < o) {
            o = v;
            c = col;
            cnt = 1;
        } else if (kCount && v == o) {
            ++cnt;  // columns arrive in increasing order
        }
    }
};

struct Chunk {
    float x[U];
};

// Set bits of `kept` below this lane's.
__device__ __forceinline__ int below(uint64_t kept) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
}

// Inclusive prefix sum over the wave (DPP: shifts within rows, then row ends).
template <int CTRL, int ROW_MASK> __device__ __forceinline__ int prefix_step(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ int wave_prefix(int v) {
    v = prefix_step<0x111, 0xF>(v);
    v = prefix_step<0x112, 0xF>(v);
    v = prefix_step<0x114, 0xF>(v);
    v = prefix_step<0x118, 0xF>(v);
    v = prefix_step<0x142, 0xA>(v);
    return prefix_step<0x143, 0xC>(v);
}

struct Clock {
    bool on;
    uint64_t mark;
    unsigned long long *t;
    __device__ __forceinline__ void lap(int p) {
        if (on && threadIdx.x == 0) {
            const uint64_t now = wall_clock64();
            t[p] += now - mark;
            mark = now;
        }
    }
};

template <int link>
__global__ __launch_bounds__(B) void k_contract(Args A) {
    // Per wave: its part of a row's smallest entry.  Two sets, taken in turn: a
    // row's words are read after its one barrier, when other waves may already
    // be writing the next row's (the first pass has no second barrier per row).
    __shared__ uint64_t s_key[2][W];
    __shared__ uint32_t s_cnt[2][W];
    __shared__ uint64_t s_k1;
    __shared__ unsigned long long s_prof[kPhases];
    constexpr bool kCount = link == HAC_SINGLE;
    // Rows in LDS hold order-preserving integers, so that the LDS minimum and
    // maximum are exact for subnormal values too.
    constexpr uint32_t kInit = link == HAC_SINGLE ? 0xFFFFFFFFu : 0u;
    const int n = A.n;
    int G = (int)gridDim.x;  // workgroups still at work
    const int w = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (__hip_atomic_load(A.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrInput) return;
    Clock clk{(A.flags & kFlagProfile) != 0, 0, s_prof};
    if (clk.on && tid == 0) {
        for (int q = 0; q < kPhases; ++q) s_prof[q] = 0;
        clk.mark = wall_clock64();
    }
    uint32_t *const row = lds<uint32_t>(oRow);
    uint16_t *const near = lds<uint16_t>(oRow);
    uint16_t *const goes = lds<uint16_t>(oRow + kMaxM * 2);
    uint64_t *const ret = lds<uint64_t>(oRet), *const sur = lds<uint64_t>(oSur), *const dead = lds<uint64_t>(oDead);
    uint16_t *const pre = lds<uint16_t>(oPre), *const prs = lds<uint16_t>(oPrs);
    float *D = A.D;
    uint32_t arrivals = 0;  // of all workgroups at the next barrier (thread 0)
    unsigned long long st_resc = 0, st_upd = 0, st_rows = 0;  // workgroup 0
    if (tid == 0) s_k1 = kNone;
    for (int c = w * B + tid; c < n; c += G * B) {
        st32(reinterpret_cast<uint32_t *>(A.slot[0] + c), (uint32_t)c);
        st32(reinterpret_cast<uint32_t *>(A.size[0] + c), 1u);
    }
    // No merge before the first pass, which only takes the rows' minima.
    for (int q = tid; q <= kWords; q += B) {
        if (q < kWords) ret[q] = sur[q] = dead[q] = 0;
        pre[q] = (uint16_t)min(n, q * 64);
    }
    __syncthreads();

    int m = n, merges = 0, round = 0, par = 0;
    int parts = 0;  // single: parts that the last round's rows were updated in, if in place
    auto survivors_before = [&](int c) {
        return (int)prs[c >> 6] + __popcll(sur[c >> 6] & ((1ull << (c & 63)) - 1ull));
    };
    uint64_t window = 0;  // merges of the last 8 rounds, at most 255 each, a byte each
    int recent = 0;       // their sum
    int sparse = 0;       // complete: rounds running that would have been cheaper in place
    uint32_t leave = 0;   // the kernel that makes the remaining merges (kHandover, kInplace)
    const bool may_hand_over = !(A.flags & kFlagNoHandover);
    bool aligned = false;  // the rows' storage as it is now (row_at)
    bool first = true, stall = (A.flags & kFlagStall) && w == 0;
    for (;;) {
        int mk = m, np = 0, out = par;  // clusters after this round's merges; where the next numbering goes
        int lt = 10;                    // log2 of the threads per row
        // ---- pairs, and where every column goes ---------------------------
        if (!first) {
            out = par ^ 1;
            if (kCount) {
                // The globally closest pair, and what nearest neighbours are tied.
                uint64_t k1 = kNone;
                for (int c = tid; c < m; c += B) {
                    uint32_t b = A.ns[par][c], v = A.val[par][c], ties = A.ties[par][c];
                    const bool gone = (dead[c >> 6] >> (c & 63)) & 1ull;
                    if (parts && ((sur[c >> 6] >> (c & 63)) & 1ull)) {
                        // A survivor of the last round, in place: join the parts of
                        // its row.  The first to read it by that rule also keeps
                        // the result (nobody reads the row's words themselves).
                        const int r = survivors_before(c);
                        uint64_t best = kNone;
                        for (int q = 0; q < parts; ++q) best = umin64(best, A.part[r * parts + q]);
                        ties = 0;
                        for (int q = 0; q < parts; ++q)
                            if ((A.part[r * parts + q] >> 32) == (best >> 32)) ties += A.pcnt[r * parts + q];
                        b = (uint32_t)best;
                        v = (uint32_t)(best >> 32);
                        if (r % G == w) {
                            st32(A.ns[par] + c, b);
                            st32(A.ties[par] + c, ties);
                            st32(A.val[par] + c, v);
                        }
                    }
                    near[c] = (uint16_t)(b | (ties > 1 ? kTied : 0u));
                    if (!gone)
                        k1 = umin64(k1, ((uint64_t)v << 32) | ((uint64_t)min((uint32_t)c, b) << 16) |
                                            (uint64_t)max((uint32_t)c, b));
                }
                k1 = last_min64(k1);
                if (lane == 63) atomicMin(reinterpret_cast<unsigned long long *>(&s_k1), (unsigned long long)k1);
            } else {
                const uint32_t *nsrc = reinterpret_cast<const uint32_t *>(A.nn[par]);
                for (int q = tid; q < (m + 1) / 2; q += B) lds<uint32_t>(oRow)[q] = nsrc[q];
            }
            __syncthreads();
            const int ka = kCount ? (int)((s_k1 >> 16) & 0xFFFFull) : -1, kb = kCount ? (int)(s_k1 & 0xFFFFull) : -1;
            const int words = (m + 63) >> 6;
            for (int q = wv; q < words; q += W) {
                const int c = q * 64 + lane;
                bool pair = false;
                int b = 0;
                if (c < m && !(kCount && ((dead[q] >> lane) & 1ull))) {
                    const uint32_t e = near[c];
                    b = (int)(e & kIndex);
                    const uint32_t f = near[b];
                    pair = (int)(f & kIndex) == c;
                    if (kCount && ((e | f) & kTied) && c != ka && c != kb) pair = false;
                }
                const uint64_t r = __ballot(pair && c > b), s = __ballot(pair && c < b);
                if (lane == 0) {
                    ret[q] = r;
                    sur[q] = s;
                }
            }
            __syncthreads();
            // Kept columns before each word: wave 0, eight words per lane.
            if (wv == 0) {
                int cnt[8], scn[8], sum = 0, ssum = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int q = lane * 8 + k;
                    cnt[k] = q < words ? min(64, m - q * 64) - __popcll(kCount ? ret[q] | dead[q] : ret[q]) : 0;
                    scn[k] = q < words ? __popcll(sur[q]) : 0;
                    sum += cnt[k];
                    ssum += scn[k];
                }
                const int run = wave_prefix(sum), srun = wave_prefix(ssum);
                int at = run - sum, sat = srun - ssum;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    pre[lane * 8 + k] = (uint16_t)at;
                    prs[lane * 8 + k] = (uint16_t)sat;
                    at += cnt[k];
                    sat += scn[k];
                }
                if (lane == 63) {
                    pre[kWords] = (uint16_t)at;
                    prs[kWords] = (uint16_t)sat;
                }
            }
            if (tid == 0) s_k1 = kNone;
            __syncthreads();
            mk = (int)pre[kWords];
            np = (int)prs[kWords];
            if (np == 0) {  // no pair although clusters remain
                if (tid == 0) {
                    atomicOr(&A.ctl->error, kErrInternal);
                    atomicOr(A.status, kErrInternal);
                    __hip_atomic_store(&A.cc->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                return;
            }
        }
        if (link == HAC_COMPLETE && (A.flags & kFlagInplaceNext) && !first) {
            sparse = cheaper_in_place(np, m, n) ? sparse + 1 : 0;
            if (sparse == 2 || (sparse && round == 0)) {  // nothing of this round has been applied
                leave = kInplace;
                break;
            }
        }
        // Single linkage with few pairs: their rows and columns in place, the
        // retired columns stay until they are kRetired of the whole.
        const bool inplace = kCount && !first && m > kInplaceMin && (m - mk) * kRetired < m && mk > 1;
        // Every workgroup has read the nearest neighbours before one changes, and
        // the joined rows of an update in place are kept.
        if (kCount && (inplace || parts) && !arrive_and_wait(A, arrivals, (uint32_t)G, false)) return;
        parts = 0;
        if (inplace) {
            // A row in as many parts as give every workgroup one.
            parts = max(1, min(G / np, (m + V * B - 1) / (V * B)));
            const int len = ((m + parts - 1) / parts + 63) & ~63;
            for (int unit = w; unit < np * parts; unit += G) {
                const int r = unit / parts, at = (unit - r * parts) * len, end = min(m, at + len);
                int i = 0;
                {
                    const int big = 63 - __clzll((long long)__ballot((int)prs[lane * 8] <= r));
                    const int q = big * 8 + 31 - __clz((int)(uint32_t)(__ballot((int)prs[big * 8 + (lane & 7)] <= r) & 0xFFull));
                    const uint64_t set = sur[q];
                    const uint64_t hit = __ballot(((set >> lane) & 1ull) && below(set) == r - (int)prs[q]);
                    i = __builtin_amdgcn_readfirstlane(q * 64 + __ffsll((unsigned long long)hit) - 1);
                }
                const int j = __builtin_amdgcn_readfirstlane((int)(near[i] & kIndex));
                const int si = A.slot[par][i], sj = A.slot[par][j];
                float *Di = row_at(D, n, si, aligned);
                const float *Dj = row_at(D, n, sj, aligned);
                Low low;
                for (int c0 = at + tid; c0 < end; c0 += V * B) {
                    float xi[V], xj[V], xk[V], xl[V];
                    uint32_t best[V];
                    int sl[V], kind[V];  // 0: not a live column, 1: unmerged, 2: survivor of another pair
#pragma unroll
                    for (int u = 0; u < V; ++u) {
                        const int c = c0 + u * B;
                        kind[u] = 0;
                        if (c < end && c != i && c != j) {
                            const uint64_t bit = 1ull << (c & 63);
                            if (!((ret[c >> 6] | dead[c >> 6]) & bit)) kind[u] = (sur[c >> 6] & bit) ? 2 : 1;
                        }
                        if (kind[u]) {
                            xi[u] = Di[c];
                            xj[u] = Dj[c];
                        }
                        if (kind[u] == 1) {
                            best[u] = A.val[par][c];
                            sl[u] = A.slot[par][c];
                        }
                        if (kind[u] == 2) {
                            const int cj = (int)(near[c] & kIndex);
                            xk[u] = Di[cj];
                            xl[u] = Dj[cj];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < V; ++u) {
                        const int c = c0 + u * B;
                        if (!kind[u]) continue;
                        float v = fminf(xi[u], xj[u]);
                        if (kind[u] == 2) {
                            // Two clusters merged in this round: the smallest of the
                            // four entries; the other one's row is written by its owner.
                            v = fminf(v, fminf(xk[u], xl[u]));
                        } else {
                            if (ord32(v) == best[u]) {
                                // The row's smallest entry moves to column i; one column
                                // less attains it if both did.
                                if (ord32(xi[u]) == best[u] && ord32(xj[u]) == best[u])
                                    __hip_atomic_fetch_sub(A.ties[par] + c, 1u, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT);
                                __hip_atomic_fetch_min(A.ns[par] + c, (uint32_t)i, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
                            }
                            st32(reinterpret_cast<uint32_t *>(row_at(D, n, sl[u], aligned) + i), __float_as_uint(v));
                        }
                        st32(reinterpret_cast<uint32_t *>(Di + c), __float_as_uint(v));
                        low.take<true>(ord32(v), c);
                    }
                }
                const uint64_t mine = low.o == 0xFFFFFFFFu ? kNone : ((uint64_t)low.o << 32) | (uint64_t)low.c;
                const uint64_t best = wave_min64(mine);
                const uint32_t ties =
                    (uint32_t)wave_sum(low.o == (uint32_t)(best >> 32) ? (unsigned long long)low.cnt : 0ull);
                __syncthreads();
                if (lane == 0) {
                    s_key[0][wv] = best;
                    s_cnt[0][wv] = ties;
                }
                __syncthreads();
                if (tid == 0) {
                    uint64_t b = kNone;
                    for (int q = 0; q < W; ++q) b = umin64(b, s_key[0][q]);
                    uint32_t t = 0;
                    for (int q = 0; q < W; ++q)
                        if ((uint32_t)(s_key[0][q] >> 32) == (uint32_t)(b >> 32)) t += s_cnt[0][q];
                    st64(A.part + unit, b);
                    st32(A.pcnt + unit, t);
                    if (at == 0) {
                        const uint32_t h = A.val[par][i];
                        const int sz = A.size[par][i] + A.size[par][j];
                        A.rec[merges + r] = make_int4(si, sj, __float_as_int(unord32(h)), sz);
                        A.key[merges + r] = ((uint64_t)h << 32) | ((uint64_t)si << 16) | (uint64_t)round;
                        st32(reinterpret_cast<uint32_t *>(A.size[par] + i), (uint32_t)sz);
                    }
                }
            }
            merges += np;
            const int capped = min(np, 255);
            recent += capped - (int)(window >> 56);
            window = (window << 8) | (uint64_t)capped;
            ++round;
            if (w == 0 && tid == 0) {
                st_rows += (unsigned)np;
                st_upd += (unsigned long long)np * (unsigned long long)(mk - 1) -
                          (unsigned long long)np * (unsigned long long)(np - 1) / 2;
            }
            clk.lap(kPhRescan);
            if (!arrive_and_wait(A, arrivals, (uint32_t)G, false)) return;
            clk.lap(kPhWait);
            for (int q = tid; q < (m + 63) >> 6; q += B) dead[q] |= ret[q];
            __syncthreads();
        } else {
        // Threads per row: as few as let every row be under way at once, at
        // least one per KE columns.
        while (lt > 6 && m <= (KE << (lt - 1)) && ((int64_t)mk << lt) > (int64_t)G * B) --lt;
        const int T = 1 << lt, NG = B >> lt, grp = tid >> lt;
        int t = tid & (T - 1);
        const int stride = (mk + 3) & ~3;
        const bool shorter = !first && mk <= n - 3;
        // Large matrices leave by ordinary 16-byte stores and an L2 write back at
        // the barrier, small ones by write-through stores (n=32768: 8.8 against
        // 10.4 ms for the whole kernel; n=2000: 0.43 against 0.41 ms).
        const bool wide = mk > kWideMin;
        uint32_t *const buf = row + grp * stride;
        const int iters = (mk + G * NG - 1) / (G * NG);

        // Row r of the new matrix: old row a, and its partner's if it survives
        // a merge.  Its columns come in chunks of U per thread: t, t + T, ...
        Chunk even, odd;
        uint32_t place[KE / 2];
#pragma unroll
        for (int k = 0; k < KE / 2; ++k) place[k] = 0;
        bool merged = false;
        int sa = 0;
        const float *pa = nullptr, *pb = nullptr;
        auto find = [&](int r) {
            int a = r;
            merged = false;
            if (!first) {
                // The word by its prefix count, then the bit.
                const int big = 63 - __clzll((long long)__ballot((int)pre[lane * 8] <= r));
                const int q = big * 8 + 31 - __clz((int)(uint32_t)(__ballot((int)pre[big * 8 + (lane & 7)] <= r) & 0xFFull));
                const uint64_t kept = kCount ? ~(ret[q] | dead[q]) : ~ret[q];
                const uint64_t hit = __ballot(((kept >> lane) & 1ull) && below(kept) == r - (int)pre[q]);
                const int bit = __ffsll((unsigned long long)hit) - 1;
                a = __builtin_amdgcn_readfirstlane(q * 64 + bit);
                merged = __builtin_amdgcn_readfirstlane((int)((sur[q] >> bit) & 1ull)) != 0;
            }
            sa = first ? r : __builtin_amdgcn_readfirstlane(A.slot[par][a]);
            pa = row_at(D, n, sa, aligned);
            if (merged) {
                const int b = kCount ? (int)A.ns[par][a] : (int)A.nn[par][a];
                pb = row_at(D, n, __builtin_amdgcn_readfirstlane(A.slot[par][b]), aligned);
            }
        };
        auto load = [&](Chunk &q, int k0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t c = (uint32_t)(((k0 + u) << lt) + t);
                q.x[u] = 0.0f;
                if ((int)c < m) q.x[u] = pa[c];
            }
        };
        int r = grp * G + w;
        if (mk > 1 && r < mk) {
            find(r);
            load(even, 0);
        }
        // ---- records, the new numbering (a share each), the retired columns' targets
        if (!first) {
            auto kept_before = [&](int c) {
                const uint64_t gone = kCount ? ret[c >> 6] | dead[c >> 6] : ret[c >> 6];
                return (int)pre[c >> 6] + __popcll(~gone & ((1ull << (c & 63)) - 1ull));
            };
            for (int c = w * B + tid; c < m; c += G * B) {
                if (kCount && ((dead[c >> 6] >> (c & 63)) & 1ull)) continue;
                const int kept = kept_before(c);
                const int sl = A.slot[par][c], sz = A.size[par][c];
                const int b = (int)(near[c] & kIndex);
                if ((ret[c >> 6] >> (c & 63)) & 1ull) {
                    const int q = merges + survivors_before(b), si = A.slot[par][b];
                    const uint32_t v = A.val[par][c];
                    A.rec[q] = make_int4(si, sl, __float_as_int(unord32(v)), A.size[par][b] + sz);
                    A.key[q] = ((uint64_t)v << 32) | ((uint64_t)si << 16) | (uint64_t)round;
                } else {
                    const bool mg = (sur[c >> 6] >> (c & 63)) & 1ull;
                    st32(reinterpret_cast<uint32_t *>(A.slot[out] + kept), (uint32_t)sl);
                    st32(reinterpret_cast<uint32_t *>(A.size[out] + kept), (uint32_t)(mg ? sz + A.size[par][b] : sz));
                }
            }
            // Where every column goes, the same for every row: kept columns to
            // their new places, retired ones to their survivors'; columns retired
            // before go to a word that nothing reads.  A table beside the nearest
            // neighbours, from which each thread takes its columns'.
            for (int c = tid; c < m; c += B) {
                const uint64_t bit = 1ull << (c & 63), r0 = ret[c >> 6];
                const int to = (r0 & bit) ? (int)(near[c] & kIndex) : c;
                goes[c] = (uint16_t)(kCount && (dead[c >> 6] & bit) ? kNowhere : kept_before(to));
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KE; ++k) {
                const int c = (k << lt) + t;
                uint32_t at = kNowhere;
                if ((k << lt) < m && c < m) at = goes[c];
                if (kCount && at == kNowhere) at = (uint32_t)(kMaxM + 32 - grp * stride);
                if (k & 1)
                    place[k / 2] |= at << 16;
                else
                    place[k / 2] = at;
            }
            merges += np;
            const int capped = min(np, 255);
            recent += capped - (int)(window >> 56);
            window = (window << 8) | (uint64_t)capped;
            ++round;
        }
        if (w == 0 && tid == 0) {
            st_rows += (unsigned)mk;
            // Entries streamed through: read, and but for the first pass written.
            st_resc += (unsigned long long)m * (unsigned long long)(mk + np) +
                       (first ? 0ull : (unsigned long long)mk * (unsigned long long)mk);
            st_upd += (unsigned long long)np * (unsigned long long)(mk - 1) -
                      (unsigned long long)np * (unsigned long long)(np > 0 ? np - 1 : 0) / 2;
        }
        if (mk == 1) break;
        __syncthreads();  // the nearest neighbours have been read: the row area is free
        if (!first) {
            for (int q = tid; q < NG * stride; q += B) row[q] = kInit;
            __syncthreads();
        }
        clk.lap(kPhCand);
        // ---- rows ------------------------------------------------------------
        for (int it = 0; it < iters; ++it) {
            const bool valid = r < mk;
            // Column numbers and places are worked out anew for every row: kept
            // across rows, unpacked, they would take more registers than there are.
            asm volatile("" : "+v"(t));
#pragma unroll
            for (int k = 0; k < KE / 2; ++k) asm volatile("" : "+v"(place[k]));
            Low low;
            if (valid) {
                auto use = [&](Chunk &q, auto first_column) {
                    constexpr int k0 = decltype(first_column)::value;
                    __builtin_amdgcn_sched_barrier(0);
                    if (merged) {
                        float y[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint32_t c = (uint32_t)(((k0 + u) << lt) + t);
                            y[u] = 0.0f;
                            if ((int)c < m) y[u] = pb[c];
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) q.x[u] = link == HAC_SINGLE ? fminf(q.x[u], y[u]) : fmaxf(q.x[u], y[u]);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int c = ((k0 + u) << lt) + t;
                        if (c >= m) continue;
                        if (first) {
                            if (c != r) low.take<kCount>(ord32(q.x[u]), c);
                            continue;
                        }
                        const float v = q.x[u];
                        const uint32_t at = ((k0 + u) & 1) ? place[(k0 + u) / 2] >> 16 : place[(k0 + u) / 2] & 0xFFFFu;
                        if (link == HAC_SINGLE)
                            __hip_atomic_fetch_min(buf + at, ord32(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        else
                            __hip_atomic_fetch_max(buf + at, ord32(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                };
                // Two chunks in turn: one's loads are in flight while the
                // other is used.
                const bool m1 = (U << lt) < m, m2 = ((2 * U) << lt) < m, m3 = ((3 * U) << lt) < m;
                if (m1) load(odd, U);
                use(even, std::integral_constant<int, 0>{});
                if (m2) load(even, 2 * U);
                if (m1) use(odd, std::integral_constant<int, U>{});
                if (m3) load(odd, 3 * U);
                if (m2) use(even, std::integral_constant<int, 2 * U>{});
                if (m3) use(odd, std::integral_constant<int, 3 * U>{});
            }
            if (!first) __syncthreads();
            const int rn = r + NG * G, so = sa;
            if (it + 1 < iters && rn < mk) {  // in flight while this row leaves
                find(rn);
                load(even, 0);
            }
            if (!first && valid) {
                float *dst = row_at(D, n, so, shorter);
                for (int c = 4 * t; c < mk; c += 4 * T) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(buf + c);
                    *reinterpret_cast<uint4 *>(buf + c) = make_uint4(kInit, kInit, kInit, kInit);  // for the next row
                    if (c != r) low.take<kCount>(v.x, c);
                    if (c + 1 < mk && c + 1 != r) low.take<kCount>(v.y, c + 1);
                    if (c + 2 < mk && c + 2 != r) low.take<kCount>(v.z, c + 2);
                    if (c + 3 < mk && c + 3 != r) low.take<kCount>(v.w, c + 3);
                    const uint32_t u[4] = {__float_as_uint(unord32(v.x)), __float_as_uint(unord32(v.y)),
                                           __float_as_uint(unord32(v.z)), __float_as_uint(unord32(v.w))};
                    if (shorter && c + 3 < mk) {
                        if (wide) {
                            *reinterpret_cast<uint4 *>(dst + c) = make_uint4(u[0], u[1], u[2], u[3]);
                        } else {
                            st64(reinterpret_cast<uint64_t *>(dst + c), ((uint64_t)u[1] << 32) | u[0]);
                            st64(reinterpret_cast<uint64_t *>(dst + c + 2), ((uint64_t)u[3] << 32) | u[2]);
                        }
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (c + q < mk) st32(reinterpret_cast<uint32_t *>(dst + c + q), u[q]);
                    }
                }
            }
            if (valid) {
                const uint64_t mine = low.o == 0xFFFFFFFFu ? kNone : ((uint64_t)low.o << 32) | (uint64_t)low.c;
                const uint64_t best = wave_min64(mine);
                uint32_t ties = 0;
                if (kCount)
                    ties = (uint32_t)wave_sum(low.o == (uint32_t)(best >> 32) ? (unsigned long long)low.cnt : 0ull);
                if (lane == 0) {
                    s_key[it & 1][wv] = best;
                    if (kCount) s_cnt[it & 1][wv] = ties;
                }
            }
            __syncthreads();
            if (valid && t == 0) {
                uint64_t best = kNone;
                const uint64_t *keys = s_key[it & 1] + wv;
                for (int q = 0; q < T / 64; ++q) best = umin64(best, keys[q]);
                if (kCount) {
                    uint32_t ties = 0;
                    for (int q = 0; q < T / 64; ++q)
                        if ((uint32_t)(keys[q] >> 32) == (uint32_t)(best >> 32)) ties += s_cnt[it & 1][wv + q];
                    st32(A.ns[out] + r, (uint32_t)best);
                    st32(A.ties[out] + r, ties);
                } else {
                    st16(A.nn[out] + r, (uint16_t)best);
                }
                st32(A.val[out] + r, (uint32_t)(best >> 32));
            }
            r = rn;
        }
        clk.lap(kPhUpdate);
        if (!arrive_and_wait(A, arrivals, (uint32_t)G, stall, wide)) return;
        clk.lap(kPhWait);
        m = mk;
        par = out;
        aligned = shorter;
        first = false;
        if (kCount) {
            for (int q = tid; q < kWords; q += B) dead[q] = 0;
            __syncthreads();  // every wave reads the whole mask next
        }
        }
        const int keep = contract_workgroups(m, G);  // the others leave
        if (w >= keep) return;
        G = keep;
        const bool few = n <= kSmallN ? round >= 2 && cheaper_behind(recent, min(round, kWindow), n - merges, n)
                                      : round >= kWindow && n - merges > kHandoverLeft &&
                                            recent < kWindow * kMinPerRound;
        if (may_hand_over && few) {
            leave = kHandover;
            break;
        }
    }
    if (leave) {
        __syncthreads();
        // Rows back to their columns' slots for the kernel that goes on (they are
        // still there before the first contraction), and their minima for k_run.
        const bool moved = m < n;
        for (int q = w; q < m && (moved || leave == kHandover); q += G) {
            if ((dead[q >> 6] >> (q & 63)) & 1ull) continue;
            const int s = A.slot[par][q];
            const float *from = row_at(D, n, s, aligned);
            float *p = D + (size_t)s * n;
            uint64_t best = kNone;
            for (int c = tid; c < m; c += B) {
                const float x = from[c];
                row[c] = __float_as_uint(x);
                if (c > q && !((dead[c >> 6] >> (c & 63)) & 1ull))
                    best = umin64(best, ((uint64_t)ord32(x) << 32) | ((uint64_t)A.slot[par][c] << 16));
            }
            best = wave_min64(best);
            if (lane == 0) s_key[0][wv] = best;
            __syncthreads();
            if (moved)
                for (int c = tid; c < m; c += B) p[A.slot[par][c]] = __uint_as_float(row[c]);
            if (tid == 0) {
                for (int k = 1; k < W; ++k) best = umin64(best, s_key[0][k]);
                A.rowkey[s] = best;
            }
            __syncthreads();
        }
        __syncthreads();
        for (int c = w * B + tid; c < m; c += G * B)
            if (!((dead[c >> 6] >> (c & 63)) & 1ull)) A.hsize[A.slot[par][c]] = A.size[par][c];
        if (w == 0) {
            uint32_t *bits = lds<uint32_t>(oRow);
            const int words = (n + 31) >> 5;
            for (int q = tid; q < words; q += B) bits[q] = 0;
            __syncthreads();
            for (int c = tid; c < m; c += B) {
                if ((dead[c >> 6] >> (c & 63)) & 1ull) continue;
                const int s = A.slot[par][c];
                atomicOr(&bits[s >> 5], 1u << (s & 31));
            }
            __syncthreads();
            for (int q = tid; q < words; q += B) A.live[q] = bits[q];
            if (tid == 0) {
                A.cc->merges = (uint32_t)merges;
                A.cc->round = (uint32_t)round;
                if (leave == kHandover) {
                    const unsigned long long left = (unsigned long long)(n - merges);
                    atomicAdd(&A.ctl->rescans, left);
                    atomicAdd(&A.ctl->rescan_elems, left * (left - 1) / 2);
                }
                atomicOr(A.status, leave);
            }
        }
    }
    if (w == 0 && tid == 0) {
        atomicAdd(&A.ctl->rescans, st_rows);
        atomicAdd(&A.ctl->rescan_elems, st_resc);
        atomicAdd(&A.ctl->update_elems, st_upd);
        atomicAdd(&A.ctl->rounds_rescans, st_rows);
        atomicAdd(&A.ctl->rounds_rescan_elems, st_resc);
        atomicAdd(&A.ctl->rounds_update_elems, st_upd);
        A.ctl->rounds = (uint32_t)round;
    }
    if (clk.on && tid == 0) {
        for (int p = 0; p < kPhases; ++p) {
            atomicAdd(&A.ctl->prof_sum[p], s_prof[p]);
            atomicMax(&A.ctl->prof_max[p], s_prof[p]);
        }
    }
}

const void *contract_kernel(int link) {
    return link == HAC_SINGLE ? reinterpret_cast<const void *>(&k_contract<HAC_SINGLE>)
                              : reinterpret_cast<const void *>(&k_contract<HAC_COMPLETE>);
}

}  // namespace

ContractLayout contract_layout(int n) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    ContractLayout L{};
    const size_t m = (size_t)(n > 1 ? n - 1 : 1);
    size_t off = 0;
    L.ctl = off;  off += al(sizeof(ContractCtl));
    L.rank = off; off += al((size_t)n * 4);
    L.zero_bytes = off;
    for (int q = 0; q < 2; ++q) {
        L.nn[q] = off;   off += al((size_t)(n + 2) * 4);
        L.ties[q] = off; off += al((size_t)n * 4);
        L.val[q] = off;  off += al((size_t)n * 4);
        L.slot[q] = off; off += al((size_t)n * 4);
        L.size[q] = off; off += al((size_t)n * 4);
    }
    L.part = off;  off += al((size_t)(n + 256) * 8);  // max(pairs, workgroups)
    L.pcnt = off;  off += al((size_t)(n + 256) * 4);
    L.rec = off;   off += al(m * 16);
    L.key = off;   off += al(m * 8);
    L.live = off;  off += al((size_t)((n + 31) / 32) * 4);
    L.hsize = off; off += al((size_t)n * 4);
    L.bytes = off;
    return L;
}

int contract_occupancy(int link) {
    const void *fn = contract_kernel(link);
    int blocks = 0;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, B, kLdsBytes) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return blocks;
}

hipError_t launch_contract(float *D, int n, int link, uint32_t *status, Control *ctl, uint64_t *rowkey, void *ws, int G,
                           uint64_t timeout_ticks, int flags, hipStream_t stream) {
    const ContractLayout Lo = contract_layout(n);
    char *b = static_cast<char *>(ws);
    Args a;
    a.D = D;
    a.status = status;
    a.ctl = ctl;
    a.cc = reinterpret_cast<ContractCtl *>(b + Lo.ctl);
    for (int q = 0; q < 2; ++q) {
        a.nn[q] = reinterpret_cast<uint16_t *>(b + Lo.nn[q]);
        a.ns[q] = reinterpret_cast<uint32_t *>(b + Lo.nn[q]);
        a.ties[q] = reinterpret_cast<uint32_t *>(b + Lo.ties[q]);
        a.val[q] = reinterpret_cast<uint32_t *>(b + Lo.val[q]);
        a.slot[q] = reinterpret_cast<int32_t *>(b + Lo.slot[q]);
        a.size[q] = reinterpret_cast<int32_t *>(b + Lo.size[q]);
    }
    a.part = reinterpret_cast<uint64_t *>(b + Lo.part);
    a.pcnt = reinterpret_cast<uint32_t *>(b + Lo.pcnt);
    a.rec = reinterpret_cast<int4 *>(b + Lo.rec);
    a.key = reinterpret_cast<uint64_t *>(b + Lo.key);
    a.live = reinterpret_cast<uint32_t *>(b + Lo.live);
    a.hsize = reinterpret_cast<int32_t *>(b + Lo.hsize);
    a.rowkey = rowkey;
    a.timeout = timeout_ticks;
    a.n = n;
    a.flags = flags;
    void *args[] = {&a};
    return hipLaunchCooperativeKernel(contract_kernel(link), dim3(G), dim3(B), args, kLdsBytes, stream);
}

RoundsLayout contract_rounds_layout(int n, int G) {
    const ContractLayout Lc = contract_layout(n);
    RoundsLayout L = rounds_layout(n, G, Lc.bytes);
    L.rec = Lc.rec;
    L.key = Lc.key;
    L.live = Lc.live;
    L.size = Lc.hsize;
    L.state = Lc.ctl + offsetof(ContractCtl, merges);
    return L;
}

Resume contract_resume(int n, void *ws) {
    const ContractLayout Lo = contract_layout(n);
    char *b = static_cast<char *>(ws);
    Resume r;
    r.live = reinterpret_cast<const uint32_t *>(b + Lo.live);
    r.size = reinterpret_cast<const int32_t *>(b + Lo.hsize);
    r.keys = reinterpret_cast<uint64_t *>(b + Lo.key);
    r.state = reinterpret_cast<const uint32_t *>(b + Lo.ctl + offsetof(ContractCtl, merges));
    return r;
}

}  // namespace hac
