// Query order of the traversal kernels: which particle each lane of a
// workgroup takes (shared by the exact and the paper-mode traversal).
#pragma once

#include "qbvh_internal.h"

namespace qbi {

// Workgroups are dealt round-robin to the 8 XCDs; each XCD gets one
// contiguous stretch of the Z-ordered queries so its L2 holds one region.
__device__ __forceinline__ int32_t xcd_logical_block() {
    const uint32_t nb = gridDim.x, b = blockIdx.x;
    const uint32_t xcd = b & 7u, qq = nb >> 3, rr = nb & 7u;
    return (int32_t)(xcd * qq + (xcd < rr ? xcd : rr) + (b >> 3));
}

// Query order.  A system of one type takes its queries in sorted (Z) order,
// a.qpw per wavefront.  In a system of several types, the workgroups form
// eight equal stretches (one per XCD when the system covers the whole
// launch); stretch x takes the x-th eighth of every type's queries, smallest
// type first, in wavefronts of type_qpw queries of one type.  A sparse type's
// wavefronts span the widest regions and run longest: this way they start
// first, are spread over the stretches, and each takes few queries, instead
// of closing the launch on one XCD.  `wg` is the system's workgroup in
// dispatch order and `nwg` its workgroup count (trav_blocks, an upper bound
// for several types); returns the lane's position in the system, or a.n for
// an idle lane.
template <int kBlock, class Args>
__device__ __forceinline__ int32_t query_position(Args &a, const TreeMeta *__restrict__ meta, int32_t wg,
                                                  int32_t nwg) {
    const int32_t lane = (int32_t)(threadIdx.x & 63u), wave = (int32_t)(threadIdx.x >> 6);
    if (a.ntypes <= 1) {
        // wavefronts of a.qpw queries: lanes past a.qpw idle
        const int32_t qpw = a.qpw;
        if (lane >= qpw) return a.n;
        return (wg * (kBlock / 64) + wave) * qpw + lane;
    }
    const int32_t per = nwg / 8;
    const int64_t part = wg / per;
    int32_t wi = (wg % per) * (kBlock / 64) + wave;  // wavefront of the stretch
    for (int r = 0; r < a.ntypes; ++r) {
        // the type of rank r by (count, type index)
        int t = 0;
        for (int u = 0; u < a.ntypes; ++u) {
            int rank = 0;
            for (int w = 0; w < a.ntypes; ++w)
                rank += (meta[w].count < meta[u].count || (meta[w].count == meta[u].count && w < u)) ? 1 : 0;
            if (rank == r) t = u;
        }
        const int64_t len = meta[t].count;
        const int32_t lo = stretch_lo(len, part), hi = stretch_lo(len, part + 1);
        const int32_t qt = type_qpw(len, a.n, a.qpw);
        const int32_t nw = type_waves(len, a.n, a.qpw, part);
        if (wi < nw) {
            const int32_t j = wi * qt + lane;
            return (lane < qt && j < hi - lo) ? meta[t].start - a.start + lo + j : a.n;
        }
        wi -= nw;
    }
    return a.n;
}

}  // namespace qbi
