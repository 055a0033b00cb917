// Ordered-round engine: group average, weighted average and Ward linkage,
// several merges per exchange, byte for byte the sequential merge list.
//
// The fp32 updates of these linkages depend on the order in which merges are
// applied, so a round may only make merges that the one-merge-per-step loop
// (Section 4, steps 1-4) would make next, in its order.  Which ones those
// are follows from the rows' two smallest entries.  Let m1(a), n1(a) be the
// smallest entry of row a over all live columns and its column, m2(a) the
// second smallest entry, and T the smallest m2 over the live rows.
//
//   Every row with m1(a) < T is half of a reciprocal nearest-neighbour pair:
//   if the partner's nearest were another row x, the partner's row would
//   hold two entries <= m1(a) < T, so its m2 would be below T.  Sorted by
//   (D, i, j) these pairs are the next merges of the sequential loop:
//   Table 1's rows are averages of D_ki and D_kj (Ward: after subtracting
//   D_ij, which is not above them), so the entry of a merged cluster with any
//   other is at least the smaller of its members' entries with that other,
//   which is at least T (both members of the pair have their single smaller
//   entry with each other).  So until the last of these pairs has merged,
//   every new entry, and every old entry between two clusters outside them,
//   stays at T or above, and the smallest key is the next pair of the list.
//
// In fp32 a new entry can come out below that bound by a few units in the
// last place (weighted average: 1, group average: 4, Ward: 12, entries not
// negative), so pairs are taken only below T (1 - 2^-18), with T >= 2^-100
// so that subnormal rounding cannot matter.  If no pair qualifies (ties,
// zeros, negative entries) the round makes the one smallest merge, which
// needs no bound.
//
// m2 may be a lower bound: when the column that held it merges, its value is
// kept and the row is marked; T computed from it is only smaller, so fewer
// merges qualify.  Rows whose mark holds T back are rescanned beside the
// rows whose partner merged.
//
// Work split: workgroup w of G owns the columns (and rows) w*C .. w*C+C-1, one
// thread each keeping its row's two smallest entries in registers.  A round is
// one exchange: every workgroup publishes the smallest m2 of its rows, its
// pairs below it, and its part of the row minima of the clusters merged in
// the previous round; every workgroup reads all slots and derives the same
// list of merges, then updates its own columns: D[i][c] and D[c][i] for every
// merge (i, j) of the list, and rescans its own rows whose partner merged.
// An entry between two clusters merged in the same round is computed from
// the four entries between their members, the earlier merge first, by the
// owner of the column, from the copies only that owner writes.
//
// What bounds it: the chain exchange -> loads of rows i, j -> stores
// complete, once per round instead of once per merge (about sqrt(n) rounds
// per factor of two in live clusters on clustered points).
#include <hip/hip_runtime.h>

#include "hac_dev.h"
#include "hac_order.h"
#include "hac_slots.h"

namespace hac {
namespace {

constexpr uint64_t kNoKey = ~0ull;
constexpr uint32_t kNoOrd = 0xFFFFFFFFu;
constexpr int B = kOrderBlock, W = B / 64;
constexpr int KP = kOrderMaxPairs;
// Instances up to this size keep the cluster sizes in every workgroup's LDS
// (2 bytes each); above, they are read from memory each round.
constexpr int kOrderSizesN = 32768;
constexpr int kSegCols = 1024;       // columns one wave rescans at a time

struct OrderArgs {
    float *D;
    hac_merge *out;
    uint32_t *status;
    Control *ctl;
    uint64_t *rk;      // n first row minima: ord:32 | column:16 | 0
    uint32_t *m2;      // n second smallest entries (ord)
    uint64_t *vsize;   // n cluster sizes with the round that last changed them (size_word)
    int32_t *size;     // n cluster sizes left at a hand-over
    uint32_t *live;    // live mask left at a hand-over
    uint32_t *state;   // [0] merges, [1] rounds at a hand-over; [2] workgroups arrived there
    uint64_t *rowkey;  // the live rows' minima over the columns to their right, left at a hand-over
    uint64_t *slots;   // 2 * (G + 2) * kOrderSlotWords: G slots, then workgroup 0's list (two slots' room)
    uint64_t timeout;
    int n, flags;
};

// A cluster's size in memory, with the round that last changed it and the
// size before: its owner writes it at the end of a round that another
// workgroup may still be beginning, and no other round can be mixed up,
// because an exchange lies between.
__device__ __forceinline__ uint64_t size_word(int round, int before, int now) {
    return ((uint64_t)(round + 1) << 40) | ((uint64_t)before << 20) | (uint64_t)now;
}
__device__ __forceinline__ int size_before(uint64_t v, int round) {
    return (int)((int)(v >> 40) == round + 1 ? (v >> 20) & 0xFFFFFu : v & 0xFFFFFu);
}

// Running two smallest entries of one lane: keys arrive in increasing column
// order, so the first of equal entries keeps the smallest column.
struct Two {
    uint32_t m1 = kNoOrd, m2 = kNoOrd;
    int c = 0;
    __device__ __forceinline__ void take(uint32_t o, int col) {
        if (o < m1) {
            m2 = m1;
            m1 = o;
            c = col;
        } else {
            m2 = o < m2 ? o : m2;
        }
    }
};
// The same over the wave, valid in lane 63: (ord:32 | column:16 | 0) and the
// second ord.  Each step joins two disjoint parts: the smaller key stays, the
// larger one competes for second.  (Rows left out by a step's mask join with
// themselves and spoil their second word; no later step reads them.)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void join_two(uint64_t &k, uint32_t &s) {
    const uint64_t ok = dpp64<CTRL, ROW_MASK>(k);
    const uint32_t os = dpp32<CTRL, ROW_MASK>(s);
    const uint32_t loser = (uint32_t)((ok < k ? k : ok) >> 32);
    s = min(min(s, os), loser);
    k = umin64(k, ok);
}
__device__ __forceinline__ uint64_t last_two(const Two &t, uint32_t &second) {
    uint64_t k = t.m1 == kNoOrd ? kNoKey : ((uint64_t)t.m1 << 32) | ((uint64_t)t.c << 16);
    second = t.m2;
    join_two<0xB1, 0xF>(k, second);
    join_two<0x4E, 0xF>(k, second);
    join_two<0x141, 0xF>(k, second);
    join_two<0x140, 0xF>(k, second);
    join_two<0x142, 0xA>(k, second);
    join_two<0x143, 0xC>(k, second);
    return k;
}

// Fold one part's (smallest, second) into LDS words: every smallest but the
// final one ends up in the second word, either on arrival or when displaced.
__device__ __forceinline__ void lds_two(uint64_t *w1, uint32_t *w2, uint64_t b1, uint32_t b2) {
    if (b1 == kNoKey) return;
    const uint64_t old = atomicMin(reinterpret_cast<unsigned long long *>(w1), (unsigned long long)b1);
    const uint64_t loser = old > b1 ? old : b1;
    const uint32_t l = (uint32_t)(loser >> 32);
    atomicMin(w2, l < b2 ? l : b2);
}

// Two smallest entries of every row over all other columns; one wave per row.
__global__ __launch_bounds__(256) void k_row_two(const float *__restrict__ D, int n, const uint32_t *status,
                                                 uint64_t *__restrict__ rk, uint32_t *__restrict__ m2,
                                                 uint64_t *__restrict__ vsize) {
    if (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrInput) return;
    const int lane = threadIdx.x & 63;
    const int r = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (r >= n) return;
    const float *row = D + (size_t)r * n;
    Two t;
    if ((n & 3) == 0) {
        constexpr int U = 8;
        for (int c0 = 0; c0 < n; c0 += 256 * U) {
            float4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + 4 * (u * 64 + lane);
                x[u] = c < n ? *reinterpret_cast<const float4 *>(row + c) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + 4 * (u * 64 + lane);
                if (c >= n) continue;
                const float v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (c + q != r) t.take(ord32(v[q]), c + q);
            }
        }
    } else {
        constexpr int U = 16;
        for (int c0 = 0; c0 < n; c0 += 64 * U) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * 64 + lane;
                x[u] = c < n ? row[c] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * 64 + lane;
                if (c < n && c != r) t.take(ord32(x[u]), c);
            }
        }
    }
    uint32_t second;
    const uint64_t best = last_two(t, second);
    if (lane == 63) {
        rk[r] = best;
        m2[r] = second;
        vsize[r] = 1;  // size_word of a cluster never merged
    }
}

// Merges applied together: eight per thread (16 loads in flight per lane), at most
// KP.  The variants of 128 to 512 columns spill 18 to 23 registers for it at 1024
// threads, those of 1024 columns 9 to 11, of 64 columns 2.
__host__ __device__ constexpr int group_pairs(int LC) { return ((8 * B) >> LC) < KP ? ((8 * B) >> LC) : KP; }

// LDS of one workgroup: byte offsets into its dynamic LDS, constants so that
// every access is an LDS instruction at an immediate offset.
constexpr int kMaskWords = (HAC_MAX_N + 31) / 32;
// Pairs a workgroup offers per round beside its smallest: all it may merge
// when there are few workgroups, fewer when many share them.
__host__ __device__ constexpr int cands(int G) { return G <= 2 ? KP : G <= 8 ? KP / 2 : G <= 16 ? KP / 4 : KP / 8; }
constexpr int kCandMax = kOrderMaxGroup * (cands(kOrderMaxGroup) + 1) + KP;
static_assert(cands(1) + 2 + KP <= kOrderUnits && kCandMax >= 16 * (cands(16) + 1) + KP, "slots and lists hold every split");
static_assert(2 * (1 + 2 * KP) <= 2 * kOrderSlotWords, "workgroup 0's list fits two slots' room");
template <int LC> struct Map {
    static constexpr uint32_t C = 1u << LC;
    static constexpr uint32_t v = 0;                            // u32: this group's new entries (ord), [merge][own column]
    static constexpr uint32_t cand = v + group_pairs(LC) * C * 4;  // u64: pairs offered by the workgroups and the previous survivors
    static constexpr uint32_t sel = cand + kCandMax * 8;        // u64: those below the bound
    static constexpr uint32_t rq1 = sel + kCandMax * 8;         // u64: rescanned rows: smallest
    static constexpr uint32_t r1 = rq1 + C * 8;                 // u64: merged rows: smallest over all columns
    static constexpr uint32_t p1 = r1 + KP * 8;                 // u64: the same over this workgroup's columns
    static constexpr uint32_t scand = p1 + KP * 8;              // u64: this workgroup's pairs
    static constexpr uint32_t pair = scand + KP * 8;            // int2: this round's merges
    static constexpr uint32_t nij = pair + KP * 8;              // int2: their sizes
    static constexpr uint32_t h = nij + KP * 8;                 // float
    static constexpr uint32_t ai = h + KP * 4;                  // float
    static constexpr uint32_t aj = ai + KP * 4;                 // float
    static constexpr uint32_t r2 = aj + KP * 4;                 // u32: second entries of r1, p1, rq1
    static constexpr uint32_t p2 = r2 + KP * 4;
    static constexpr uint32_t rq2 = p2 + KP * 4;
    static constexpr uint32_t m2 = rq2 + C * 4;                 // u32: own rows' second entries before the round
    static constexpr uint32_t mark = m2 + C * 4;                // u32: own rows whose second entry's column merged
    static constexpr uint32_t role = mark + C * 4;              // i32: own columns: +(q+1) survivor, -(q+1) retired, 0
    static constexpr uint32_t csize = role + C * 4;             // i32: own columns: cluster size
    static constexpr uint32_t amask = csize + C * 4;            // u32: live clusters
    static constexpr uint32_t tmask = amask + kMaskWords * 4;   // u32: clusters merging this round
    static constexpr uint32_t queue = tmask + kMaskWords * 4;   // u16: own rows to rescan
    static constexpr uint32_t surv = queue + C * 2;             // u16: own columns that survive a merge of this round
    static constexpr uint32_t bytes = surv + KP * 2;
};

extern __shared__ __align__(16) uint8_t smem[];
template <class T> __device__ __forceinline__ T *lds(uint32_t off) { return reinterpret_cast<T *>(smem + off); }

__device__ __forceinline__ bool bit(const uint32_t *m, int c) { return (m[c >> 5] >> (c & 31)) & 1u; }

__device__ __forceinline__ uint64_t pair_key(uint32_t o, int i, int j) {
    return ((uint64_t)o << 32) | ((uint64_t)i << 16) | (uint64_t)j;
}

__device__ __forceinline__ uint64_t ld64(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st64(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Read this thread's units u = tid, tid + STEP, ... below `total` (unit u's
// words are at at(u)) and hand each to take(u, word0, word1) once both words
// carry generation `gen`; U units' loads are in flight at a time.  False if the
// launch was aborted or the watchdog expired.
template <int U, int STEP, class At, class Take>
__device__ __forceinline__ bool get_units(int total, uint64_t gen, const OrderArgs &A, At at, Take take) {
    const uint64_t t0 = wall_clock64();
    for (int u0 = (int)threadIdx.x; u0 < total; u0 += U * STEP) {
        uint32_t left = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) left |= u0 + k * STEP < total ? 1u << k : 0u;
        for (uint32_t it = 1; left; ++it) {
            uint64_t a[U], b[U];
#pragma unroll
            for (int k = 0; k < U; ++k)
                if ((left >> k) & 1u) {
                    const uint64_t *p = at(u0 + k * STEP);
                    a[k] = ld64(p);
                    b[k] = ld64(p + 1);
                }
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (((left >> k) & 1u) && (a[k] & 0xFFFFull) == gen && (b[k] & 0xFFFFull) == gen) {
                    take(u0 + k * STEP, a[k], b[k]);
                    left &= ~(1u << k);
                }
            if ((it & 63u) == 0 && left) {
                if (__hip_atomic_load(&A.ctl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
                if (wall_clock64() - t0 > A.timeout) {
                    atomicOr(&A.ctl->error, kErrTimeout);
                    atomicOr(A.status, kErrTimeout);
                    __hip_atomic_store(&A.ctl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return false;
                }
            }
        }
    }
    return true;
}

// One wave: fold the two smallest entries of columns seg*kSegCols .. of row r
// over the live columns that do not merge this round into (*w1, *w2).
template <int LC>
__device__ __forceinline__ void rescan_part(const float *__restrict__ D, int n, int r, int seg, uint64_t *w1,
                                            uint32_t *w2, uint32_t &elems) {
    const uint32_t *amask = lds<uint32_t>(Map<LC>::amask), *tmask = lds<uint32_t>(Map<LC>::tmask);
    const int lane = threadIdx.x & 63;
    const float *row = D + (size_t)r * n;
    const int c0 = seg * kSegCols, c1 = min(n, c0 + kSegCols);
    Two t;
    if ((n & 3) == 0) {
        constexpr int U = kSegCols / 256;
        float4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + 4 * (u * 64 + lane);
            x[u] = c < c1 ? *reinterpret_cast<const float4 *>(row + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + 4 * (u * 64 + lane);
            if (c >= c1) continue;
            const int q = c >> 2;
            uint32_t m = ((amask[q >> 3] & ~tmask[q >> 3]) >> ((q & 7) * 4)) & 0xFu;
            if ((r >> 2) == q) m &= ~(1u << (r & 3));
            elems += __popc(m);
            const float v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((m >> k) & 1u) t.take(ord32(v[k]), c + k);
        }
    } else {
        constexpr int U = 16;
        for (int b0 = c0; b0 < c1; b0 += 64 * U) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = b0 + u * 64 + lane;
                x[u] = c < c1 ? row[c] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = b0 + u * 64 + lane;
                if (c < c1 && c != r && bit(amask, c) && !bit(tmask, c)) {
                    t.take(ord32(x[u]), c);
                    ++elems;
                }
            }
        }
    }
    uint32_t second;
    const uint64_t best = last_two(t, second);
    if (lane == 63) lds_two(w1, w2, best, second);
}

// Wall clock of thread 0 charged to phases (kFlagProfile).
__shared__ unsigned long long s_prof[kPhases];
struct Clock {
    bool on;
    uint64_t mark;
    __device__ __forceinline__ void lap(int p) {
        if (on && threadIdx.x == 0) {
            const uint64_t now = wall_clock64();
            s_prof[p] += now - mark;
            mark = now;
        }
    }
};

// Hand over when rounds have come down to two merges each (a round costs two
// to three of the one-merge-per-step kernel's exchanges) and enough merges are
// left to pay for that kernel's start.
constexpr int kHandoverPace = 2 << 8;
constexpr int kHandoverLeft = 128;
// A row known only by a bound is rescanned when the bound comes below this
// multiple of the smallest exact second entry, early enough that the bound does
// not hold back the rounds that follow: the closer entries lie (many items),
// the smaller the margin may be.  Measured at 1.02 / 1.05 / 1.1: n=512
// 0.87 / 0.82 / 0.80 ms, n=3001 4.1 / 3.6 / 3.6, n=8192 8.5 / 8.7 / 9.1,
// n=65536 193 / 211 / 220.
__device__ __forceinline__ float mark_factor(int n) { return 1.0f + fminf(0.15f, fmaxf(0.02f, 160.0f / (float)n)); }

template <int LC, int link>
__global__ __launch_bounds__(B) void k_order(OrderArgs A) {
    __shared__ uint64_t s_min, s_pmin;                                  // smallest offered pair: all, own
    __shared__ uint32_t s_T, s_TE, s_TI, s_pT, s_pTE, s_pTI, s_pT2;     // bounds: all, own
    __shared__ uint32_t s_cnt, s_pcnt, s_nq, s_ns, s_fail, s_p, s_smin;
    constexpr int C = 1 << LC, QG = group_pairs(LC), QS = B / C, K = QG / QS;  // K merges per thread and group
    const int n = A.n;
    const int KC = cands((int)gridDim.x);
    const int G = (int)gridDim.x, w = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (__hip_atomic_load(A.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrInput) return;
    using M = Map<LC>;
    struct {
        uint32_t *v = lds<uint32_t>(M::v), *rq2 = lds<uint32_t>(M::rq2), *r2 = lds<uint32_t>(M::r2),
                 *p2 = lds<uint32_t>(M::p2), *m2 = lds<uint32_t>(M::m2), *mark = lds<uint32_t>(M::mark),
                 *amask = lds<uint32_t>(M::amask), *tmask = lds<uint32_t>(M::tmask);
        uint64_t *cand = lds<uint64_t>(M::cand), *sel = lds<uint64_t>(M::sel), *rq1 = lds<uint64_t>(M::rq1),
                 *r1 = lds<uint64_t>(M::r1), *p1 = lds<uint64_t>(M::p1), *scand = lds<uint64_t>(M::scand);
        int32_t *role = lds<int32_t>(M::role), *csize = lds<int32_t>(M::csize);
        uint16_t *queue = lds<uint16_t>(M::queue), *surv = lds<uint16_t>(M::surv);
        int2 *pair = lds<int2>(M::pair), *nij = lds<int2>(M::nij);
        float *h = lds<float>(M::h), *ai = lds<float>(M::ai), *aj = lds<float>(M::aj);
    } const L;
    // Every workgroup's copy of the cluster sizes (less 1), where it fits.
    const bool lsize = n <= kOrderSizesN;
    uint16_t *const Lsize = lds<uint16_t>(M::bytes);
    float *D = A.D;
    Clock clk{(A.flags & kFlagProfile) != 0, 0};
    if (clk.on && tid == 0) {
        for (int q = 0; q < kPhases; ++q) s_prof[q] = 0;
        clk.mark = wall_clock64();
    }
    uint32_t st_upd = 0, st_elems = 0, st_rows = 0;  // a lane's counts stay below 2^32 (n^2 / 64 at most)

    // This thread's own row (threads below C).
    const int c = w * C + tid;
    bool alive = tid < C && c < n, marked = false;
    uint32_t m1 = kNoOrd, m2 = kNoOrd;
    int n1 = 0, myq = -1;
    if (alive) {
        const uint64_t k = A.rk[c];
        m1 = (uint32_t)(k >> 32);
        n1 = (int)((k >> 16) & 0xFFFFull);
        m2 = A.m2[c];
    }
    const int words = (n + 31) >> 5;
    for (int q = tid; q < words; q += B) {
        const int rem = n - q * 32;
        L.amask[q] = rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
        L.tmask[q] = 0;
    }
    if (lsize)
        for (int q = tid; q < n; q += B) Lsize[q] = 0;
    if (tid < C) {
        L.role[tid] = 0;
        L.csize[tid] = 1;
    }
    if (tid == 0) {
        s_pT = s_pTE = s_pTI = s_pT2 = kNoOrd;
        s_pmin = kNoKey;
        s_pcnt = 0;
        s_nq = 0;
        s_fail = 0;
    }
    __syncthreads();

    int merges = 0, round = 0, p = 0, qidx = -1;
    uint32_t TE = 0, smin = 0;  // of the last exchange: smallest exact second entry, smallest pair's value
    bool stuck = false;         // it found no merge
    // Merges per round, running mean over about 16 rounds (8 fractional bits), from
    // what clustered points of this many items make (from 16 always: constant matrix,
    // n = 300, 1.04 ms instead of 0.85, uniform values 0.90 and 0.89).  A mean that falls
    // faster when a round of ties makes no merge hands uniform values over too, which
    // are better off here (n = 5000: 13.7 ms instead of 5.8).
    int pace = (int)(256.0f * fminf(16.0f, fmaxf(3.0f, 0.2f * sqrtf((float)n))));
    bool negative = false;
    const bool may_hand_over = !(A.flags & kFlagNoHandover);
    const int nseg = (n + kSegCols - 1) / kSegCols;
    const float factor = mark_factor(n);
    for (;;) {
        // ---- publish: bounds, pairs, parts of the merged rows' minima ----
        const uint32_t e = (uint32_t)round + 1u;
        {
            const bool mine = alive && myq < 0;
            qidx = -1;
            if (tid < C) {
                const uint32_t a = last_min32(mine ? m2 : kNoOrd);
                const uint32_t b = last_min32(mine && !marked ? m2 : kNoOrd);
                const uint32_t f = last_min32(mine && m1 == kNoOrd ? m2 : kNoOrd);
                const uint64_t k = last_min64(mine && m1 != kNoOrd && c < n1 ? pair_key(m1, c, n1) : kNoKey);
                if (lane == 63) {
                    atomicMin(&s_pT, a);
                    atomicMin(&s_pTE, b);
                    atomicMin(&s_pTI, f);
                    atomicMin(reinterpret_cast<unsigned long long *>(&s_pmin), (unsigned long long)k);
                }
            }
            if (tid == 0) {
                s_T = s_TE = s_TI = kNoOrd;
                s_min = kNoKey;
                s_cnt = s_ns = 0;
            }
            if (tid < KP) {
                L.r1[tid] = kNoKey;
                L.r2[tid] = kNoOrd;
            }
            __syncthreads();
            // Rows known by a bound that may hold the next rounds back: rescanned
            // while the exchange is under way, so exact from the next round on.
            if (mine && marked && m2 != kNoOrd &&
                (TE == kNoOrd || unord32(m2) < unord32(TE) * factor || (stuck && m2 <= smin))) {
                qidx = (int)atomicAdd(&s_nq, 1u);
                L.queue[qidx] = (uint16_t)tid;
                L.rq1[qidx] = kNoKey;
                L.rq2[qidx] = kNoOrd;
            }
            if (mine && m1 < s_pT && c < n1) {
                const uint64_t k = pair_key(m1, c, n1);
                if (k != s_pmin) {
                    const uint32_t at = atomicAdd(&s_pcnt, 1u);
                    if (at < (uint32_t)KC)
                        L.scand[at] = k;
                    else
                        atomicMin(&s_pT2, m1);  // not offered: nothing from here on may merge past it
                }
            }
            barrier_stores_done();  // this round's updates are complete before the slot says so
        }
        const int units = 2 + KC + p;
        const uint32_t pT = s_pT < s_pT2 ? s_pT : s_pT2;
        const int pcnt = min((int)s_pcnt, KC);
        const int ncand = G * (KC + 1) + p;
        const uint64_t gen = e & 0xFFFFu;
        uint64_t *base = A.slots + (size_t)(e & 1u) * (G + 2) * kOrderSlotWords;
        uint64_t *cast = base + (size_t)G * kOrderSlotWords;
        clk.lap(kPhCand);
        if (G > 1 && tid < (writes_whole_slot(e) ? kOrderUnits : units) && !((A.flags & kFlagStall) && w == 0)) {
            uint64_t a, b;
            if (tid >= units) {
                a = b = gen;  // read by nobody
            } else if (tid == 0) {
                a = ((uint64_t)pT << 32) | gen;
                b = ((uint64_t)s_pTE << 32) | gen;
            } else if (tid < 2 + KC) {
                const uint64_t k = tid == 1 ? s_pmin : tid - 2 < pcnt ? L.scand[tid - 2] : kNoKey;
                a = (k & ~0xFFFFull) | gen;
                b = ((uint64_t)(tid == 1 ? s_pTI : 0u) << 32) | ((k & 0xFFFFull) << 16) | gen;
            } else {
                a = (L.p1[tid - 2 - KC] & ~0xFFFFull) | gen;
                b = ((uint64_t)L.p2[tid - 2 - KC] << 32) | gen;
            }
            uint64_t *s = base + (size_t)w * kOrderSlotWords + 2 * tid;
            st64(s, a);
            st64(s + 1, b);
        }
        // ---- rescans of own rows, whose entries no other workgroup writes
        // before this exchange completes
        const int nq = (int)s_nq;
        for (int t = wv; t < nq * nseg; t += W) {
            const int r = t / nseg;
            rescan_part<LC>(D, n, w * C + L.queue[r], t - r * nseg, &L.rq1[r], &L.rq2[r], st_elems);
        }
        if (tid == 0) st_rows += (unsigned)nq;
        clk.lap(kPhRescan);
        const bool select = G <= kOrderAllToAll || w == 0;
        const int pprev = p;
        auto enter = [&](int q, int i, int j) {  // merge q of this round
            L.pair[q] = make_int2(i, j);
            atomicOr(&L.tmask[i >> 5], 1u << (i & 31));
            atomicOr(&L.tmask[j >> 5], 1u << (j & 31));
            if (i / C == w) L.role[i & (C - 1)] = q + 1;
            if (j / C == w) L.role[j & (C - 1)] = -(q + 1);
        };
        if (select) {
            // ---- read every slot ----------------------------------------
            if (G > 1) {
                const bool ok = get_units<4, B>(
                    G * units, gen, A,
                    [&](int u) {
                        const int g = u / units;
                        return base + (size_t)g * kOrderSlotWords + 2 * (u - g * units);
                    },
                    [&](int u, uint64_t a, uint64_t b) {
                        const int g = u / units, k = u - g * units;
                        if (k == 0) {
                            atomicMin(&s_T, (uint32_t)(a >> 32));
                            atomicMin(&s_TE, (uint32_t)(b >> 32));
                        } else if (k < 2 + KC) {
                            if (k == 1) atomicMin(&s_TI, (uint32_t)(b >> 32));
                            L.cand[g * (KC + 1) + k - 1] =
                                (uint32_t)(a >> 32) == kNoOrd ? kNoKey : (a & ~0xFFFFull) | ((b >> 16) & 0xFFFFull);
                        } else if ((uint32_t)(a >> 32) != kNoOrd) {
                            lds_two(&L.r1[k - 2 - KC], &L.r2[k - 2 - KC], a & ~0xFFFFull, (uint32_t)(b >> 32));
                        }
                    });
                if (!ok) atomicOr(&s_fail, 1u);
            } else {
                if (tid == 0) {
                    s_T = pT;
                    s_TE = s_pTE;
                    s_TI = s_pTI;
                }
                if (tid < KC + 1) L.cand[tid] = tid == 0 ? s_pmin : tid - 1 < pcnt ? L.scand[tid - 1] : kNoKey;
                if (tid < pprev) {
                    L.r1[tid] = L.p1[tid];
                    L.r2[tid] = L.p2[tid];
                }
            }
            __syncthreads();
            if (s_fail) return;
            clk.lap(kPhWait);
            // ---- this round's merges; the previous survivors' rows are known now
            // Every wave folds the survivors' second entries into the bounds.
            const uint32_t sm = wave_min32(lane < pprev ? L.r2[lane] : kNoOrd);
            const uint32_t T = s_T < sm ? s_T : sm;
            TE = s_TE < sm ? s_TE : sm;
            uint32_t lim = 0;
            {
                const float t = T == kNoOrd ? __uint_as_float(0x7F800000u) : unord32(T);
                if (round > 0 && !negative && t >= 0x1p-100f)
                    lim = T == kNoOrd ? kNoOrd : ord32(t * (1.0f - 0x1p-18f));
            }
            {
                uint64_t best = kNoKey;
                for (int q = tid; q < ncand; q += B) {
                    uint64_t k;
                    if (q < G * (KC + 1)) {
                        k = L.cand[q];
                    } else {
                        const uint64_t r = L.r1[q - G * (KC + 1)];
                        const int i = L.pair[q - G * (KC + 1)].x, b = (int)((r >> 16) & 0xFFFFull);
                        k = r != kNoKey && i < b ? pair_key((uint32_t)(r >> 32), i, b) : kNoKey;
                    }
                    best = umin64(best, k);
                    if ((uint32_t)(k >> 32) < lim) L.sel[atomicAdd(&s_cnt, 1u)] = k;
                }
                if (wv * 64 < ncand) {
                    best = last_min64(best);
                    if (lane == 63 && best != kNoKey)
                        atomicMin(reinterpret_cast<unsigned long long *>(&s_min), (unsigned long long)best);
                }
            }
            if (G > 1 && wv == W - 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the barrier orders the other waves' loads after it
            __syncthreads();
            const int cnt = (int)s_cnt;
            if (s_min == kNoKey && s_TI == kNoOrd) {  // no pair although clusters remain
                if (tid == 0) {
                    atomicOr(&A.ctl->error, kErrInternal);
                    atomicOr(A.status, kErrInternal);
                    __hip_atomic_store(&A.ctl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                return;
            }
            if (round == 0) negative = (uint32_t)(s_min >> 32) < 0x80000000u;
            // No pair below the bound: the smallest pair alone, if no row
            // known only by a bound could hold a smaller one; else none, and
            // those rows are rescanned.
            p = cnt ? min(cnt, KP) : (uint32_t)(s_min >> 32) < s_TI ? 1 : 0;
            smin = (uint32_t)(s_min >> 32);
            // Rank of each selected pair: 16 threads per pair share the comparisons.
            for (int q0 = 0; q0 < (cnt ? cnt : p); q0 += B / 16) {
                const int q = q0 + tid / 16;
                const uint64_t k = q < (cnt ? cnt : p) ? (cnt ? L.sel[q] : s_min) : kNoKey;
                int rank = 0;
                for (int z = tid & 15; z < cnt; z += 16) rank += L.sel[z] < k;
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) rank += __shfl_xor(rank, o, 16);
                if ((tid & 15) == 0 && k != kNoKey && rank < KP) {
                    L.h[rank] = unord32((uint32_t)(k >> 32));
                    enter(rank, (int)((k >> 16) & 0xFFFFull), (int)(k & 0xFFFFull));
                }
            }
            if (G > kOrderAllToAll) __syncthreads();
            if (G > kOrderAllToAll && tid < 1 + KP + (writes_whole_slot(e) ? KP : pprev)) {
                uint64_t a, b;
                if (tid >= 1 + KP + pprev) {
                    a = b = gen;
                } else if (tid == 0) {
                    a = ((uint64_t)TE << 32) | ((uint64_t)p << 16) | gen;
                    b = ((uint64_t)smin << 32) | gen;
                } else if (tid < 1 + KP) {
                    const int2 ij = tid <= p ? L.pair[tid - 1] : make_int2(0, 0);
                    a = ((uint64_t)(tid <= p ? __float_as_uint(L.h[tid - 1]) : 0u) << 32) | ((uint64_t)ij.x << 16) | gen;
                    b = ((uint64_t)ij.y << 16) | gen;
                } else {
                    a = (L.r1[tid - 1 - KP] & ~0xFFFFull) | gen;
                    b = ((uint64_t)L.r2[tid - 1 - KP] << 32) | gen;
                }
                st64(cast + 2 * tid, a);
                st64(cast + 2 * tid + 1, b);
            }
        } else {
            // ---- many workgroups: workgroup 0 has read the slots ------------
            const bool ok = get_units<1, B>(
                1 + KP + pprev, gen, A, [&](int u) { return cast + 2 * u; },
                [&](int u, uint64_t a, uint64_t b) {
                    if (u == 0) {
                        s_TE = (uint32_t)(a >> 32);
                        s_p = (uint32_t)(a >> 16) & 0xFFFFu;
                        s_smin = (uint32_t)(b >> 32);
                    } else if (u < 1 + KP) {
                        const int i = (int)((a >> 16) & 0xFFFFull), j = (int)((b >> 16) & 0xFFFFull);
                        L.h[u - 1] = __uint_as_float((uint32_t)(a >> 32));
                        L.pair[u - 1] = make_int2(i, j);
                    } else {
                        L.r1[u - 1 - KP] = (uint32_t)(a >> 32) == kNoOrd ? kNoKey : a & ~0xFFFFull;
                        L.r2[u - 1 - KP] = (uint32_t)(b >> 32);
                    }
                });
            if (!ok) atomicOr(&s_fail, 1u);
            __syncthreads();
            if (s_fail) return;
            p = (int)s_p;
            TE = s_TE;
            smin = s_smin;
            if (wv == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // ordered before the other waves' loads by the barrier below
            clk.lap(kPhWait);
            if (tid < p) enter(tid, L.pair[tid].x, L.pair[tid].y);  // no rescan reads the masks any more
        }
        if (myq >= 0) {
            const uint64_t k = L.r1[myq];
            m1 = (uint32_t)(k >> 32);
            n1 = (int)((k >> 16) & 0xFFFFull);
            m2 = L.r2[myq];
            marked = false;
            myq = -1;
        }
        if (tid == 0) {
            s_pT = s_pTE = s_pTI = s_pT2 = kNoOrd;
            s_pmin = kNoKey;
            s_pcnt = 0;
            s_nq = 0;
        }
        stuck = p == 0;
        __syncthreads();
        // ---- sizes, queue of rows to rescan, loads of the first group --------
        int ni = 0, nj = 0;
        const int pt = B - 1 - tid;  // the last wave looks after the merges themselves
        if (pt < p) {
            const int2 ij = L.pair[pt];
            if (lsize) {
                ni = (int)Lsize[ij.x] + 1;
                nj = (int)Lsize[ij.y] + 1;
            } else {
                ni = size_before(ld64(A.vsize + ij.x), round);
                nj = size_before(ld64(A.vsize + ij.y), round);
            }
        }
        int myrole = 0;
        if (alive) {
            if (qidx >= 0) {  // rescanned
                const uint64_t k = L.rq1[qidx];
                m1 = (uint32_t)(k >> 32);
                n1 = (int)((k >> 16) & 0xFFFFull);
                m2 = L.rq2[qidx];
                marked = false;
            }
            myrole = L.role[tid];
            if (myrole > 0) L.surv[atomicAdd(&s_ns, 1u)] = (uint16_t)tid;
            if (myrole == 0) {
                if (m1 != kNoOrd && bit(L.tmask, n1)) {  // the smallest entry goes: the others are not below the second
                    m1 = kNoOrd;
                    marked = true;
                }
            }
        }
        if (tid < C) {
            L.m2[tid] = m2;
            L.mark[tid] = 0;
        }
        const int cl = tid & (C - 1), col = w * C + cl;
        const bool plain = col < n && bit(L.amask, col) && !bit(L.tmask, col);
        float x[K], y[K];
        auto load_group = [&](int qb) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = qb + tid / C + k * QS;
                x[k] = y[k] = 0.0f;
                if (q < p && plain) {
                    const int2 ij = L.pair[q];
                    x[k] = D[(size_t)ij.x * n + col];
                    y[k] = D[(size_t)ij.y * n + col];
                }
            }
        };
        load_group(0);
        if (pt < p) {
            L.nij[pt] = make_int2(ni, nj);
            if (link == HAC_AVERAGE) {
                const double sum = (double)(ni + nj);
                L.ai[pt] = (float)((double)ni / sum);
                L.aj[pt] = (float)((double)nj / sum);
            }
            if (w == 0) {
                const int2 ij = L.pair[pt];
                reinterpret_cast<int4 *>(A.out)[merges + pt] =
                    make_int4(ij.x, ij.y, __float_as_int(L.h[pt]), ni + nj);
            }
        }
        __syncthreads();
        clk.lap(kPhSetup);
        const int ns = (int)s_ns;
        const bool last = merges + p >= n - 1;
        if (last) {
            merges += p;
            ++round;
            break;
        }
        // Entries with clusters that survive a merge of this round, for own
        // columns: task t is merge R of the group and own survivor sc (of
        // merge S).  D between members, read in rows r (in which only this
        // workgroup, the owner of column s.x, writes these entries).
        float ii = 0.0f, ji = 0.0f, ij4 = 0.0f, jj = 0.0f;
        auto load_cross = [&](int t, int qb, int gq) {
            const int sidx = t / gq, R = qb + t - sidx * gq, S = L.role[L.surv[sidx]] - 1;
            const int2 r = L.pair[R], z = L.pair[S];
            ii = D[(size_t)r.x * n + z.x];
            ji = D[(size_t)r.y * n + z.x];
            ij4 = D[(size_t)r.x * n + z.y];
            jj = D[(size_t)r.y * n + z.y];
        };
        if (tid < ns * min(p, QG)) load_cross(tid, 0, min(p, QG));
        int qb = 0;
        do {
            const int qe = min(p, qb + QG), gq = qe - qb;
            if (qb) {
                __syncthreads();  // the previous group's entries have been read
                load_group(qb);
                if (tid < ns * gq) load_cross(tid, qb, gq);
            }
            // The earlier of the two merges first.
            for (int t = tid; t < ns * gq; t += B) {
                const int sidx = t / gq, R = qb + t - sidx * gq;
                const int sc = L.surv[sidx], S = L.role[sc] - 1;
                uint32_t o = kNoOrd;
                if (t != tid) load_cross(t, qb, gq);
                if (R != S) {
                    const int2 r = L.pair[R], s = L.pair[S];
                    const float ij = ij4;
                    const int2 nr = L.nij[R], nsz = L.nij[S];
                    float v;
                    if (R < S) {
                        const float u0 = lw_update(link, ii, ji, L.h[R], nr.x, nr.y, nsz.x, L.ai[R], L.aj[R], 0.0f);
                        const float u1 = lw_update(link, ij, jj, L.h[R], nr.x, nr.y, nsz.y, L.ai[R], L.aj[R], 0.0f);
                        v = lw_update(link, u0, u1, L.h[S], nsz.x, nsz.y, nr.x + nr.y, L.ai[S], L.aj[S], 0.0f);
                    } else {
                        const float u0 = lw_update(link, ii, ij, L.h[S], nsz.x, nsz.y, nr.x, L.ai[S], L.aj[S], 0.0f);
                        const float u1 = lw_update(link, ji, jj, L.h[S], nsz.x, nsz.y, nr.y, L.ai[S], L.aj[S], 0.0f);
                        v = lw_update(link, u0, u1, L.h[R], nr.x, nr.y, nsz.x + nsz.y, L.ai[R], L.aj[R], 0.0f);
                    }
                    o = ord32(v);
                    if (G > 1)
                        __hip_atomic_store(reinterpret_cast<uint32_t *>(D + (size_t)r.x * n + s.x), __float_as_uint(v),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else
                        D[(size_t)r.x * n + s.x] = v;
                    ++st_upd;
                }
                L.v[(R - qb) * C + sc] = o;
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = qb + tid / C + k * QS;
                if (q >= qe) continue;
                if (plain) {
                    const int2 ij = L.pair[q], sz = L.nij[q];
                    const int nk = link == HAC_WARD ? L.csize[cl] : 1;
                    const float v = lw_update(link, x[k], y[k], L.h[q], sz.x, sz.y, nk, L.ai[q], L.aj[q], 0.0f);
                    if (G > 1) {
                        __hip_atomic_store(reinterpret_cast<uint32_t *>(D + (size_t)ij.x * n + col), __float_as_uint(v),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_store(reinterpret_cast<uint32_t *>(D + (size_t)col * n + ij.x), __float_as_uint(v),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    } else {
                        D[(size_t)ij.x * n + col] = v;
                        D[(size_t)col * n + ij.x] = v;
                    }
                    ++st_upd;
                    const uint32_t om = L.m2[cl];
                    if (ord32(x[k]) == om || ord32(y[k]) == om) L.mark[cl] = 1u;
                    L.v[(q - qb) * C + cl] = ord32(v);
                } else if (!(col < n && L.role[cl] > 0)) {
                    L.v[(q - qb) * C + cl] = kNoOrd;
                }
            }
            __syncthreads();
            // This workgroup's part of each merged row's two smallest entries.
            // From the last wave down: the first waves fold their own rows below.
            for (int q = qb + W - 1 - wv; q < qe; q += W) {
                Two t;
#pragma unroll
                for (int k = 0; k < C / 64; ++k) {
                    const uint32_t o = L.v[(q - qb) * C + k * 64 + lane];
                    if (o != kNoOrd) t.take(o, w * C + k * 64 + lane);
                }
                uint32_t second;
                const uint64_t best = last_two(t, second);
                if (lane == 63) {
                    L.p1[q] = best;
                    L.p2[q] = second;
                }
            }
            // Own rows: the new entries.
            if (alive && myrole == 0) {
                if (L.mark[tid]) marked = true;
                // The group's two smallest new entries, then the row's.
                uint64_t k1 = kNoKey;
                uint32_t k2 = kNoOrd;
#pragma unroll 4
                for (int q = qb; q < qe; ++q) {
                    const uint64_t k = ((uint64_t)L.v[(q - qb) * C + tid] << 32) | ((uint64_t)L.pair[q].x << 16);
                    k2 = min(k2, (uint32_t)((k < k1 ? k1 : k) >> 32));
                    k1 = umin64(k1, k);
                }
                const uint32_t o = (uint32_t)(k1 >> 32);
                const int i = (int)((k1 >> 16) & 0xFFFFull);
                if (m1 == kNoOrd && marked) {
                    // Only a bound is known: an entry below it is the smallest.
                    if (o < m2) {
                        m1 = o;
                        n1 = i;
                        if (k2 <= m2) {
                            m2 = k2;
                            marked = false;
                        }
                    }
                } else {
                    uint32_t second;  // of the old smallest and the new entries
                    if (o < m1 || (o == m1 && i < n1)) {
                        second = min(m1, k2);
                        m1 = o;
                        n1 = i;
                    } else {
                        second = o;
                    }
                    if (second <= m2) {
                        m2 = second;
                        marked = false;
                    }
                }
            }
            qb += QG;
        } while (qb < p);
        // ---- retire, new sizes ---------------------------------------------
        if (alive && myrole != 0) {
            if (myrole < 0) {
                alive = false;
            } else {
                myq = myrole - 1;
                const int2 sz = L.nij[myq];
                L.csize[tid] = sz.x + sz.y;
                if (!lsize) st64(A.vsize + c, size_word(round, sz.x, sz.x + sz.y));
            }
            L.role[tid] = 0;
        }
        __syncthreads();
        if (tid < p) {
            const int2 ij = L.pair[tid];
            if (lsize) Lsize[ij.x] = (uint16_t)(L.nij[tid].x + L.nij[tid].y - 1);
            atomicAnd(&L.amask[ij.y >> 5], ~(1u << (ij.y & 31)));
            atomicAnd(&L.tmask[ij.x >> 5], ~(1u << (ij.x & 31)));
            atomicAnd(&L.tmask[ij.y >> 5], ~(1u << (ij.y & 31)));
        }
        clk.lap(kPhUpdate);
        merges += p;
        pace += ((p << 8) - pace) / 16;
        ++round;
        if (may_hand_over && n - 1 - merges > kHandoverLeft) {
            if (pace < kHandoverPace) {
                // Own rows' minima, once every workgroup's entries are written.
                uint32_t arrived = 0;
                if (!grid_sync(A.state + 2, &A.ctl->abort, &A.ctl->error, kErrTimeout, arrived, (uint32_t)G, A.timeout))
                    return;
                if (tid < C && c < n) A.size[c] = L.csize[tid];
                for (int r = w * C + wv; r < min(n, (w + 1) * C); r += W) {
                    if (!bit(L.amask, r)) continue;
                    const uint64_t v = upper_row_min(D, n, r, L.amask);
                    if (lane == 0) A.rowkey[r] = v;
                }
                if (w == 0) {
                    for (int q = tid; q < words; q += B) A.live[q] = L.amask[q];
                    if (tid == 0) {
                        A.state[0] = (uint32_t)merges;
                        A.state[1] = (uint32_t)round;
                        const unsigned long long left = (unsigned long long)(n - merges);
                        atomicAdd(&A.ctl->rescans, left);
                        atomicAdd(&A.ctl->rescan_elems, left * (left - 1) / 2);
                        atomicOr(A.status, kHandover);
                    }
                }
                break;
            }
        }
    }
    // Statistics.
    const unsigned long long re = wave_sum((unsigned long long)st_elems);
    const unsigned long long up = wave_sum((unsigned long long)st_upd);
    if (lane == 0) {
        atomicAdd(&A.ctl->rescan_elems, re);
        atomicAdd(&A.ctl->update_elems, up);
    }
    if (tid == 0) atomicAdd(&A.ctl->rescans, (unsigned long long)st_rows);
    if (w == 0 && tid == 0) A.ctl->rounds = (uint32_t)round;
    if (clk.on && tid == 0) {
        for (int q = 0; q < kPhases; ++q) {
            atomicAdd(&A.ctl->prof_sum[q], s_prof[q]);
            atomicMax(&A.ctl->prof_max[q], s_prof[q]);
        }
    }
}

template <int link>
const void *order_kernel_l(int columns) {
    switch (columns) {
    case 64: return reinterpret_cast<const void *>(&k_order<6, link>);
    case 128: return reinterpret_cast<const void *>(&k_order<7, link>);
    case 256: return reinterpret_cast<const void *>(&k_order<8, link>);
    case 512: return reinterpret_cast<const void *>(&k_order<9, link>);
    default: return reinterpret_cast<const void *>(&k_order<10, link>);
    }
}

const void *order_kernel(int columns, int link) {
    switch (link) {
    case HAC_AVERAGE: return order_kernel_l<HAC_AVERAGE>(columns);
    case HAC_WEIGHTED: return order_kernel_l<HAC_WEIGHTED>(columns);
    default: return order_kernel_l<HAC_WARD>(columns);
    }
}

}  // namespace

OrderLayout order_layout(int n, int G) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    OrderLayout L{};
    size_t off = 0;
    L.rk = off;    off += al((size_t)n * 8);
    L.m2 = off;    off += al((size_t)n * 4);
    L.size = off;  off += al((size_t)n * 4);
    L.vsize = off; off += al((size_t)n * 8);
    L.live = off;  off += al((size_t)((n + 31) / 32) * 4);
    L.state = off; off += 256;
    L.slots = off; off += al((size_t)2 * (G + 2) * kOrderSlotWords * 8);
    L.bytes = off;
    return L;
}

int order_columns(int n, int want) {
    for (int c = 64; c <= 1024; c *= 2)
        if ((n + c - 1) / c <= want) return c;
    return 0;
}

static size_t order_lds_bytes(int n, int columns) {
    const size_t sizes = n <= kOrderSizesN ? ((size_t)n * 2 + 15) / 16 * 16 : 0;
    switch (columns) {
    case 64: return Map<6>::bytes + sizes;
    case 128: return Map<7>::bytes + sizes;
    case 256: return Map<8>::bytes + sizes;
    case 512: return Map<9>::bytes + sizes;
    default: return Map<10>::bytes + sizes;
    }
}

int order_occupancy(int n, int columns, int link) {
    const size_t lds = order_lds_bytes(n, columns);
    const void *fn = order_kernel(columns, link);
    int blocks = 0;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, kOrderBlock, lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return blocks;
}

hipError_t launch_order(float *D, int n, int link, hac_merge *out, uint32_t *status, Control *ctl, uint64_t *rowkey,
                        void *ws, int columns, uint64_t timeout_ticks, int flags, hipStream_t stream) {
    const int G = (n + columns - 1) / columns;
    const OrderLayout Lo = order_layout(n, G);
    char *b = static_cast<char *>(ws);
    OrderArgs a;
    a.D = D;
    a.out = out;
    a.status = status;
    a.ctl = ctl;
    a.rk = reinterpret_cast<uint64_t *>(b + Lo.rk);
    a.m2 = reinterpret_cast<uint32_t *>(b + Lo.m2);
    a.size = reinterpret_cast<int32_t *>(b + Lo.size);
    a.vsize = reinterpret_cast<uint64_t *>(b + Lo.vsize);
    a.live = reinterpret_cast<uint32_t *>(b + Lo.live);
    a.state = reinterpret_cast<uint32_t *>(b + Lo.state);
    a.slots = reinterpret_cast<uint64_t *>(b + Lo.slots);
    a.rowkey = rowkey;
    a.timeout = timeout_ticks;
    a.n = n;
    a.flags = flags;
    hipLaunchKernelGGL(k_row_two, dim3((n + 3) / 4), dim3(256), 0, stream, D, n, status, a.rk, a.m2, a.vsize);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    const size_t lds = order_lds_bytes(n, columns);
    if (G == 1) return hipLaunchKernel(order_kernel(columns, link), dim3(1), dim3(kOrderBlock), args, lds, stream);
    return hipLaunchCooperativeKernel(order_kernel(columns, link), dim3(G), dim3(kOrderBlock), args, (unsigned)lds, stream);
}

Resume order_resume(int n, int G, void *ws) {
    const OrderLayout Lo = order_layout(n, G);
    char *b = static_cast<char *>(ws);
    Resume r;
    r.live = reinterpret_cast<const uint32_t *>(b + Lo.live);
    r.size = reinterpret_cast<const int32_t *>(b + Lo.size);
    r.keys = nullptr;
    r.state = reinterpret_cast<const uint32_t *>(b + Lo.state);
    return r;
}

}  // namespace hac
