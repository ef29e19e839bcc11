// Distance queries by merge of two sorted label lists (Section 5, labels of
// every vertex held by one device): d(u, v) = min over hubs common to L_u
// and L_v of d_u + d_v, -1 when they share none (for a directed graph L_u is
// u's out-list and L_v v's in-list, footnote of Section 1). A group of G
// lanes answers one query: each lane takes every G-th hub of the shorter
// list and looks it up by binary search in the longer one (both lists are
// sorted by hub rank position), then the group reduces the minimum. Large
// batches over short lists first give each query one lane (k_query_tier);
// long lists meet in an LDS hash table (k_query_hash).
#include "internal.h"

#include <algorithm>

namespace chl {

namespace {

// Two tiers in one pass. Every lane first takes one query of its wave's 64:
// when the shorter list has at most SMALL entries (a vertex with only its
// own label, frequent in scale-free graphs, or very few), the lane answers
// it alone. The other queries of the 64 are then answered by groups of G
// lanes of the same wave, a few at a time, their list bounds passed between
// lanes by shuffles: every lane of a group takes every G-th hub of the
// shorter list, searches it in the longer one, and the group reduces.
constexpr int SMALL = 2;

template <int G>
__global__ __launch_bounds__(256) void k_query_tier(int32_t n, const int64_t* __restrict__ off_u,
                                               const int32_t* __restrict__ hub_u,
                                               const int32_t* __restrict__ dist_u,
                                               const int64_t* __restrict__ off_v,
                                               const int32_t* __restrict__ hub_v,
                                               const int32_t* __restrict__ dist_v,
                                               const int32_t* __restrict__ pairs, int64_t q,
                                               int64_t* __restrict__ out, int32_t* err) {
    constexpr int NSUB = 64 / G;
    const int lane = threadIdx.x & 63, sub = lane / G, gl = lane & (G - 1);
    const int64_t wave = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * 256) >> 6;
    for (int64_t base = wave * 64; base < q; base += nwaves * 64) {
        const int64_t k = base + lane;
        bool big = false;
        int64_t ab = 0, ae = 0, bb = 0, be = 0;
        int swapped = 0;
        if (k < q) {
            const int32_t u = pairs[2 * k], v = pairs[2 * k + 1];
            if (u >= 0 && u < n && v >= 0 && v < n) {
                ab = off_u[u]; ae = off_u[u + 1]; bb = off_v[v]; be = off_v[v + 1];
                if (ae - ab > be - bb) {
                    int64_t t = ab; ab = bb; bb = t;
                    t = ae; ae = be; be = t;
                    swapped = 1;
                }
                if (ae - ab <= SMALL) {
                    const int32_t *ha = swapped ? hub_v : hub_u, *da = swapped ? dist_v : dist_u;
                    const int32_t *hb = swapped ? hub_u : hub_v, *db = swapped ? dist_u : dist_v;
                    int64_t best = INT64_MAX;
                    for (int64_t i = ab; i < ae; i++) {
                        const int32_t x = ha[i];
                        const int64_t lo = lower_hub(hb, bb, be, x);
                        if (lo < be && hb[lo] == x) {
                            const int64_t sum = (int64_t)da[i] + (int64_t)db[lo];
                            best = sum < best ? sum : best;
                        }
                    }
                    out[k] = best == INT64_MAX ? -1 : best;
                } else {
                    big = true;
                }
            } else {
                set_invalid(err);
                out[k] = -2;
            }
        }
        // the remaining queries of the wave, NSUB at a time, one per group
        unsigned long long mask = __ballot(big);
        while (mask) {
            unsigned long long m = mask;
            for (int j = 0; j < sub && m; j++) m &= m - 1;
            const int src = m ? __ffsll((long long)m) - 1 : 0;
            const bool has = m != 0;
            const int64_t gab = __shfl(ab, src), gae = __shfl(ae, src);
            const int64_t gbb = __shfl(bb, src), gbe = __shfl(be, src);
            const int gsw = __shfl(swapped, src);
            int64_t best = INT64_MAX;
            if (has) {
                const int32_t *ha = gsw ? hub_v : hub_u, *da = gsw ? dist_v : dist_u;
                const int32_t *hb = gsw ? hub_u : hub_v, *db = gsw ? dist_u : dist_v;
                for (int64_t i = gab + gl; i < gae; i += G) {
                    const int32_t x = ha[i];
                    const int64_t lo = lower_hub(hb, gbb, gbe, x);
                    if (lo < gbe && hb[lo] == x) {
                        const int64_t sum = (int64_t)da[i] + (int64_t)db[lo];
                        best = sum < best ? sum : best;
                    }
                }
            }
#pragma unroll
            for (int d = G / 2; d >= 1; d >>= 1) {
                const int64_t o = __shfl_xor(best, d, G);
                best = o < best ? o : best;
            }
            if (has && gl == 0) out[base + src] = best == INT64_MAX ? -1 : best;
            for (int j = 0; j < NSUB && mask; j++) mask &= mask - 1;
        }
    }
}

// Long lists (hundreds to thousands of labels, road-like graphs). The shorter
// list goes into an LDS hash table (hub -> distance), the longer one is read
// once, in order, and each of its hubs looked up: one or two LDS accesses per
// hub, where a binary search of the sorted list in LDS takes eleven, each
// waiting for the one before. NWV waves share a query, so that a list of a
// thousand hubs is a handful of coalesced loads per lane, and enough queries
// are in flight although each needs a table. The next query's list bounds are
// loaded while this one runs. A distance of the longer list is read only
// where a hub matches. A list too long for the table (over 3/4 of its
// entries) is searched in global memory instead. 10^6 uniform queries on a
// 512x512 grid: 6.4 ms with the binary search,
// 3.3 ms so (705 labels on average there); 200x200 (290): 2.6 -> 1.4 ms;
// 64x64 (104): 1.05 -> 0.47 ms.
constexpr int QILP = 4;      // loads in flight per lane
constexpr int64_t QUERY_FEW = 1 << 14;    // queries that do not fill the device
constexpr double QUERY_FEW_LEN = 160;
constexpr double QUERY_WAVE_LEN = 400;   // average list up to which a wave takes a query

__device__ __forceinline__ uint32_t qslot(int32_t x, int tbits) { return ((uint32_t)x * 2654435761u) >> (32 - tbits); }

template <int NWV>
__global__ __launch_bounds__(256) void k_query_hash(int32_t n, const int64_t* __restrict__ off_u,
                                                    const int32_t* __restrict__ hub_u,
                                                    const int32_t* __restrict__ dist_u,
                                                    const int64_t* __restrict__ off_v,
                                                    const int32_t* __restrict__ hub_v,
                                                    const int32_t* __restrict__ dist_v,
                                                    const int32_t* __restrict__ pairs, int64_t q,
                                                    int64_t* __restrict__ out, int32_t* err, int tbits) {
    constexpr int GS = 64 * NWV;          // lanes of a query
    constexpr int GROUPS = 256 / GS;
    static_assert(NWV == 1 || GROUPS == 1, "a query is one wave or the whole workgroup");
    extern __shared__ int4 lds4[];
    __shared__ long long red[4];
    const int gl = threadIdx.x & (GS - 1);
    const int T = 1 << tbits, cap = T / 4 * 3;
    int32_t* hk = (int32_t*)lds4 + (threadIdx.x / GS) * 2 * T;   // hubs (-1: free), then distances
    int32_t* hd = hk + T;
    auto sync = [&]() {
        if (NWV > 1) __syncthreads(); else wave_sync();
    };
    const int64_t ngrp = (int64_t)gridDim.x * GROUPS;
    int64_t k = (int64_t)blockIdx.x * GROUPS + threadIdx.x / GS;
    int64_t nab = 0, nae = 0, nbb = 0, nbe = 0;
    bool nok = false;
    auto fetch = [&](int64_t i) {
        nok = false;
        if (i >= q) return;
        const int32_t u = pairs[2 * i], v = pairs[2 * i + 1];
        nok = u >= 0 && u < n && v >= 0 && v < n;
        if (nok) { nab = off_u[u]; nae = off_u[u + 1]; nbb = off_v[v]; nbe = off_v[v + 1]; }
    };
    fetch(k);
    for (; k < q; k += ngrp) {
        const bool ok = nok;
        int64_t ab = nab, ae = nae, bb = nbb, be = nbe;
        fetch(k + ngrp);
        const int32_t *ha = hub_u, *da = dist_u, *hb = hub_v, *db = dist_v;
        int64_t best = INT64_MAX;
        if (ok) {
            if (ae - ab > be - bb) {
                int64_t t = ab; ab = bb; bb = t;
                t = ae; ae = be; be = t;
                ha = hub_v; da = dist_v; hb = hub_u; db = dist_u;
            }
            const int64_t la = ae - ab, lb = be - bb;
            if (la <= cap) {
                for (int i = gl; i < T / 4; i += GS) ((int4*)hk)[i] = make_int4(-1, -1, -1, -1);
                sync();
                for (int64_t t0 = gl; t0 < la; t0 += GS * QILP) {
                    int32_t x[QILP], d[QILP];
#pragma unroll
                    for (int r = 0; r < QILP; r++) {
                        const bool in = t0 + r * GS < la;
                        x[r] = in ? ha[ab + t0 + r * GS] : -1;
                        d[r] = in ? da[ab + t0 + r * GS] : 0;
                    }
#pragma unroll
                    for (int r = 0; r < QILP; r++)
                        if (x[r] >= 0) {
                            uint32_t s = qslot(x[r], tbits);
                            while (atomicCAS(&hk[s], -1, x[r]) != -1) s = (s + 1) & (T - 1);
                            hd[s] = d[r];
                        }
                }
                sync();
                for (int64_t t0 = gl; t0 < lb; t0 += GS * QILP) {
                    int32_t x[QILP], d[QILP];
#pragma unroll
                    for (int r = 0; r < QILP; r++) x[r] = t0 + r * GS < lb ? hb[bb + t0 + r * GS] : -2;
#pragma unroll
                    for (int r = 0; r < QILP; r++) {
                        d[r] = -1;
                        if (x[r] < 0) continue;
                        uint32_t s = qslot(x[r], tbits);
                        int32_t y = hk[s];
                        while (y != x[r] && y != -1) { s = (s + 1) & (T - 1); y = hk[s]; }
                        if (y == x[r]) d[r] = hd[s];
                    }
#pragma unroll
                    for (int r = 0; r < QILP; r++)
                        if (d[r] >= 0) {
                            const int64_t sum = (int64_t)d[r] + (int64_t)db[bb + t0 + r * GS];
                            best = sum < best ? sum : best;
                        }
                }
                // every lookup is done before the table is cleared again (with
                // four waves the barriers of the reduction see to that)
                if (NWV == 1) sync();
            } else {
                for (int64_t i = ab + gl; i < ae; i += GS) {
                    const int32_t x = ha[i];
                    const int64_t lo = lower_hub(hb, bb, be, x);
                    if (lo < be && hb[lo] == x) {
                        const int64_t sum = (int64_t)da[i] + (int64_t)db[lo];
                        best = sum < best ? sum : best;
                    }
                }
            }
        } else if (gl == 0) {
            set_invalid(err);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const int64_t o = __shfl_xor(best, d);
            best = o < best ? o : best;
        }
        if (NWV > 1) {
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NWV; w++) best = red[w] < best ? red[w] : best;
            __syncthreads();
        }
        if (gl == 0) out[k] = ok ? (best == INT64_MAX ? -1 : best) : -2;
    }
}

// One group of G lanes per query (short lists, few queries).
template <int G>
__global__ __launch_bounds__(256) void k_query_group(int32_t n, const int64_t* __restrict__ off_u,
                                               const int32_t* __restrict__ hub_u,
                                               const int32_t* __restrict__ dist_u,
                                               const int64_t* __restrict__ off_v,
                                               const int32_t* __restrict__ hub_v,
                                               const int32_t* __restrict__ dist_v,
                                               const int32_t* __restrict__ pairs, int64_t q,
                                               int64_t* __restrict__ out, int32_t* err) {
    const int gl = threadIdx.x & (G - 1);
    const int64_t grp = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
    const int64_t ngrp = ((int64_t)gridDim.x * 256) / G;
    for (int64_t k = grp; k < q; k += ngrp) {
        const int32_t u = pairs[2 * k], v = pairs[2 * k + 1];
        const bool ok = u >= 0 && u < n && v >= 0 && v < n;
        int64_t best = INT64_MAX;
        if (ok) {
            int64_t ab = off_u[u], ae = off_u[u + 1], bb = off_v[v], be = off_v[v + 1];
            const int32_t *ha = hub_u, *da = dist_u, *hb = hub_v, *db = dist_v;
            if (ae - ab > be - bb) {
                int64_t t = ab; ab = bb; bb = t;
                t = ae; ae = be; be = t;
                ha = hub_v; da = dist_v; hb = hub_u; db = dist_u;
            }
            for (int64_t i = ab + gl; i < ae; i += G) {
                const int32_t x = ha[i];
                const int64_t lo = lower_hub(hb, bb, be, x);
                if (lo < be && hb[lo] == x) {
                    int64_t s = (int64_t)da[i] + (int64_t)db[lo];
                    best = s < best ? s : best;
                }
            }
        } else if (gl == 0) {
            set_invalid(err);
        }
#pragma unroll
        for (int d = G / 2; d >= 1; d >>= 1) {
            int64_t o = __shfl_xor(best, d, G);
            best = o < best ? o : best;
        }
        if (gl == 0) out[k] = ok ? (best == INT64_MAX ? -1 : best) : -2;
    }
}

}  // namespace

int launch_query(int32_t n, const int64_t* off_u, const int32_t* hub_u, const int32_t* dist_u,
                 const int64_t* off_v, const int32_t* hub_v, const int32_t* dist_v,
                 const int32_t* pairs, int64_t q, int64_t* out, int32_t* err, double avg_len,
                 hipStream_t st) {
    if (q <= 0) return 0;
    const int G = avg_len <= 24 ? 8 : avg_len <= 96 ? 16 : avg_len <= 256 ? 32 : 64;
    // the two-tier kernel for short lists and batches that fill the device
    // with one wave per 64 queries (its groups then only take the longer
    // lists: 16 lanes up to an average of 32 labels, else 32, measured on
    // R-MAT 16, directed R-MAT 16 and R-MAT 20); else one group per query
    const bool tier = G <= 16 && q >= (1 << 16);
    const int GT = avg_len <= 32 ? 16 : 32;
    int64_t blocks = tier ? (q + 255) / 256 : (q * G + 255) / 256;
    if (blocks > 1 << 20) blocks = 1 << 20;
    if (blocks < 1) blocks = 1;
#define CHL_QUERY(KER, GG)                                                                                  \
    hipLaunchKernelGGL(KER<GG>, dim3(blocks), dim3(256), 0, st, n, off_u, hub_u, dist_u, off_v, hub_v, dist_v, \
                       pairs, q, out, err)
    if (G >= 32) {
        // a table of at least 1.7 times the average list, 512 to 4096 entries:
        // a larger one leaves fewer queries in flight, a smaller one more
        // lists to the search (705 labels on average, 10^6 queries: 1024
        // entries 5.6 ms, 2048 3.3, 4096 5.2; 290 labels: 256 entries 2.2,
        // 512 1.4, 1024 1.5). A wave per query while the average list is a
        // few loads per lane (290 labels: 1.4 ms against 1.8 with four), else
        // four waves (705 labels: 3.3 against 6.9 with one).
        // A batch that does not fill the device takes four waves per query
        // and a table that nearly every list fits: its time is that of its
        // longest query (290 labels, 1000 queries: 55 us with the small table
        // and one wave, 34 with four; 104 labels, 10^4 queries: 37 with one
        // wave, 44 with four).
        const bool few = q <= QUERY_FEW && avg_len > QUERY_FEW_LEN;
        int tbits = 9;
        while (tbits < 12 && (double)(1 << tbits) < (few ? 3.0 : 1.7) * avg_len) tbits++;
        const bool one = !few && avg_len <= QUERY_WAVE_LEN;
        const size_t lds = (size_t)(one ? 4 : 1) * 8 << tbits;
        int64_t wb = one ? (q + 3) / 4 : q;
        wb = std::min<int64_t>(wb, 256 * 16);
        if (one)
            hipLaunchKernelGGL(k_query_hash<1>, dim3(wb), dim3(256), lds, st, n, off_u, hub_u, dist_u, off_v, hub_v,
                               dist_v, pairs, q, out, err, tbits);
        else
            hipLaunchKernelGGL(k_query_hash<4>, dim3(wb), dim3(256), lds, st, n, off_u, hub_u, dist_u, off_v, hub_v,
                               dist_v, pairs, q, out, err, tbits);
    } else if (tier) {
        if (GT == 16) CHL_QUERY(k_query_tier, 16);
        else CHL_QUERY(k_query_tier, 32);
    } else {
        if (G == 8) CHL_QUERY(k_query_group, 8);
        else CHL_QUERY(k_query_group, 16);
    }
#undef CHL_QUERY
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace chl
