// Small instances (2 <= n <= 192): the whole run in one workgroup, the matrix
// in its LDS, the merges made by one wave without a barrier.
//
// At these sizes a merge is a chain of dependent steps over a few hundred
// values, so what counts is the latency of each step: the matrix in LDS
// (odd row pitch: rows and columns are both free of bank conflicts) saves the
// trips to L2, one wave saves the barriers, and one launch does what five did.
// Sixteen waves load and check the input; then wave 0 goes on alone, each of
// its lanes keeping up to three rows' minima in registers.
//
// Row k's entry is the smallest (value, l) over live l > k.  A row whose
// partner merged keeps its old value as a lower bound (lowered by every new
// entry), and is rescanned, by the whole wave, only when that bound wins the
// minimum: the rule of the engines' deferred rescans.  Ties resolve to the
// smallest (i, j) as everywhere: bounds before exact entries, then i, then j.
//
// What bounds it: one wave's instruction chain, 0.9 us a merge at n=50 and 1.2 at
// n=100 (two wave minima, an LDS round trip, 0.65 rescans a merge), against 1.6
// with the matrix in L2 and 16 waves.  The two wave minima taken in interleaved
// steps measured slower (n=100: 139 against 125 us): it issues more instructions.
#include <hip/hip_runtime.h>

#include "hac_dev.h"
#include "hac_small.h"

namespace hac {
namespace {

constexpr int B = 1024;
constexpr uint32_t kNoOrd = 0xFFFFFFFFu;

extern __shared__ __align__(16) float s_d[];
__shared__ uint32_t s_bad, s_m[kSmallMaxN];
__shared__ int s_p[kSmallMaxN];

// Order within the wave: LDS accesses of one wave complete in order; the
// compiler is kept from moving them across.
__device__ __forceinline__ void in_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Lane that holds (o, smallest tie), given the wave's minimum o of `mine`.
__device__ __forceinline__ int holder(uint32_t mine, uint32_t tie, uint32_t o) {
    uint64_t at = __ballot(mine == o);
    if (__popcll(at) > 1 && o != kNoOrd) {
        const uint32_t t = mine == o ? tie : kNoOrd;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)last_min32(t), 63);
        at = __ballot(t == first);
    }
    return __ffsll((unsigned long long)at) - 1;
}
__device__ __forceinline__ int winner(uint32_t mine, uint32_t tie, uint32_t &o) {
    o = (uint32_t)__builtin_amdgcn_readlane((int)last_min32(mine), 63);
    return holder(mine, tie, o);
}

// R: rows per lane of wave 0 (n <= 64 R).
template <int link, int R>
__global__ __launch_bounds__(B) void k_small(const float *__restrict__ src, int n, hac_merge *__restrict__ out,
                                             uint32_t *status, Control *ctl) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6, P = small_pitch(n);
    if (tid == 0) s_bad = 0;
    __syncthreads();
    // ---- load, check and mirror the strict upper triangle --------------------
    // Wave w takes rows w, w + 16, ...; four rows' loads at a time.
    constexpr int U = 4;
    for (int r0 = wv; r0 < n; r0 += 16 * U) {
        float x[U][R];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + 16 * u;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int c = lane + 64 * k;
                x[u][k] = r < n && c < n && c > r ? src[r * n + c] : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + 16 * u;
            if (r >= n) break;
            // On the way: the row's first minimum.
            uint32_t best = kNoOrd;
            int col = 1;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int c = lane + 64 * k;
                if (c < n && c > r) {
                    if (!(fabsf(x[u][k]) <= 0x1p100f)) s_bad = 1;
                    const float v = x[u][k] == 0.0f ? 0.0f : x[u][k];
                    s_d[r * P + c] = v;
                    s_d[c * P + r] = v;
                    const uint32_t o = ord32(v);
                    if (o < best) {
                        best = o;
                        col = c;
                    }
                }
            }
            uint32_t low;
            const int from = winner(best, (uint32_t)col, low);
            const int partner = __builtin_amdgcn_readlane(col, from);
            if (lane == 0) {
                s_m[r] = low;
                s_p[r] = partner;
            }
        }
    }
    __syncthreads();
    if (wv != 0) return;
    if (lane == 0) {
        Control z{};
        z.rescans = (unsigned long long)n;
        *ctl = z;
        *status = s_bad ? kErrInput : 0u;
    }
    if (s_bad) return;

    uint32_t m[R], live = 0;  // minima (ord) or bounds; bit k: row lane + 64 k is live
    int p[R], size[R];        // partner (0: the minimum is only a bound); cluster size
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int row = lane + 64 * k;
        m[k] = row < n ? s_m[row] : kNoOrd;
        p[k] = row < n ? s_p[row] : 1;
        size[k] = 1;
        if (row < n) live |= 1u << k;
    }
    uint32_t updates = 0, rescans = 0, forced = 0, elems = 0;
for (int s = 0; s < n - 1; ++s) {
        // ---- the closest pair ------------------------------------------------
        int i, j;
        uint32_t o;
        for (;;) {
            // The lane's smallest (value, row, partner): a bound's partner 0
            // sorts before any the row can really have.
            uint32_t mine = m[0], tie = ((uint32_t)lane << 8) | (uint32_t)p[0];
#pragma unroll
            for (int k = 1; k < R; ++k)
                if (m[k] < mine) {
                    mine = m[k];
                    tie = ((uint32_t)(lane + 64 * k) << 8) | (uint32_t)p[k];
                }
            const int at = winner(mine, tie, o);
            const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)tie, at);
            i = (int)(t >> 8);
            j = (int)(t & 0xFFu);
            if (j != 0 || o == kNoOrd) break;
            // A bound won: rescan that row and look again.
            uint32_t best = kNoOrd;
            int col = 0;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int c = lane + 64 * k;
                if (((live >> k) & 1u) && c > i) {
                    const uint32_t v = ord32(s_d[i * P + c]);
                    ++elems;
                    if (v < best) {
                        best = v;
                        col = c;
                    }
                }
            }
            uint32_t low;
            const int from = winner(best, (uint32_t)col, low);
            const int partner = __builtin_amdgcn_readlane(col, from);
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (lane + 64 * k == i) {
                    m[k] = low;
                    p[k] = low == kNoOrd ? 1 : partner;
                }
            ++rescans;
            ++forced;
        }
        if (o == kNoOrd) {
            if (lane == 0) {
                ctl->error = kErrInternal;
                *status = kErrInternal;
            }
            return;
        }
        const float h = unord32(o);
        // Cluster sizes of i and j.
        int ni = size[0], nj = size[0];
#pragma unroll
        for (int k = 1; k < R; ++k) {
            ni = (i >> 6) == k ? size[k] : ni;
            nj = (j >> 6) == k ? size[k] : nj;
        }
        ni = __builtin_amdgcn_readlane(ni, i & 63);
        nj = __builtin_amdgcn_readlane(nj, j & 63);
        if (lane == 0)
            reinterpret_cast<int4 *>(out)[s] = make_int4(i, j, __float_as_int(h), ni + nj);
        if (s == n - 2) break;
        // ---- update of row and column i (Section 4 step 3) ----------------------
        float a[R], b[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int c = lane + 64 * k;
            a[k] = b[k] = 0.0f;
            if (c < n) {
                a[k] = s_d[i * P + c];
                b[k] = s_d[j * P + c];
            }
        }
        float ai = 0.0f, aj = 0.0f, bij = 0.0f;
        if (link == HAC_AVERAGE || link == HAC_CENTROID) {
            // One division for both quotients (and centroid's third): lanes 0-2.
            const double sum = (double)(ni + nj);
            const double num = lane == 0 ? (double)ni : lane == 1 ? (double)nj : -((double)ni * (double)nj);
            const float q = (float)(num / (lane == 2 ? sum * sum : sum));
            ai = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q), 0));
            aj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q), 1));
            if (link == HAC_CENTROID) bij = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q), 2));
        }
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (lane + 64 * k == j) {
                live &= ~(1u << k);
                m[k] = kNoOrd;
                p[k] = 1;
            }
        uint32_t best = kNoOrd;  // row i's new minimum over columns to its right
        int col = 0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int c = lane + 64 * k;
            if (!((live >> k) & 1u) || c == i) continue;
            const float v = lw_update(link, a[k], b[k], h, ni, nj, size[k], ai, aj, bij);
            s_d[i * P + c] = v;
            s_d[c * P + i] = v;
            ++updates;
            const uint32_t q = ord32(v);
            if (c > i) {
                if (q < best) {
                    best = q;
                    col = c;
                }
                if (c < j && p[k] == j) p[k] = 0;  // its partner is gone
            } else {
                if (p[k] == i || p[k] == j) p[k] = 0;
                // The row's new entry at column i.
                if (p[k] == 0)
                    m[k] = q < m[k] ? q : m[k];
                else if (q < m[k] || (q == m[k] && i < p[k])) {
                    m[k] = q;
                    p[k] = i;
                }
            }
        }
        uint32_t low;
        const int from = winner(best, (uint32_t)col, low);
        const int partner = __builtin_amdgcn_readlane(col, from);
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (lane + 64 * k == i) {
                m[k] = low;
                p[k] = low == kNoOrd ? 1 : partner;
                size[k] = ni + nj;
            }
        in_order();
    }
    const unsigned long long up = wave_sum((unsigned long long)updates), el = wave_sum((unsigned long long)elems);
    if (lane == 0) {
        ctl->rescans = rescans;
        ctl->rescan_elems = el;
        ctl->update_elems = up;
        ctl->forced = forced;
    }
}

template <int link>
const void *small_kernel_l(int rows) {
    switch (rows) {
    case 1: return reinterpret_cast<const void *>(&k_small<link, 1>);
    case 2: return reinterpret_cast<const void *>(&k_small<link, 2>);
    default: return reinterpret_cast<const void *>(&k_small<link, 3>);
    }
}

const void *small_kernel(int link, int rows) {
    switch (link) {
    case HAC_SINGLE: return small_kernel_l<HAC_SINGLE>(rows);
    case HAC_COMPLETE: return small_kernel_l<HAC_COMPLETE>(rows);
    case HAC_AVERAGE: return small_kernel_l<HAC_AVERAGE>(rows);
    case HAC_WARD: return small_kernel_l<HAC_WARD>(rows);
    case HAC_WEIGHTED: return small_kernel_l<HAC_WEIGHTED>(rows);
    default: return small_kernel_l<HAC_CENTROID>(rows);
    }
}

constexpr size_t small_lds(int n) { return (size_t)n * small_pitch(n) * 4; }

}  // namespace

hipError_t small_setup() {
    for (int link = 0; link <= HAC_CENTROID; ++link)
        for (int rows = 1; rows <= kSmallMaxN / 64; ++rows) {
            hipError_t e = hipFuncSetAttribute(small_kernel(link, rows), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)small_lds(kSmallMaxN));
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t launch_small(const float *src, int n, int link, hac_merge *out, uint32_t *status, Control *ctl,
                        hipStream_t stream) {
    const float *a0 = src;
    int a1 = n;
    hac_merge *a2 = out;
    uint32_t *a3 = status;
    Control *a4 = ctl;
    void *args[] = {&a0, &a1, &a2, &a3, &a4};
    return hipLaunchKernel(small_kernel(link, (n + 63) / 64), dim3(1), dim3(B), args, small_lds(n), stream);
}

}  // namespace hac
