// Traversal launch geometry shared by the host (workgroup counts) and the
// device (which queries a wavefront takes).  Plain C++ apart from the
// host/device qualifiers, so that a CPU test can check the host's bound
// against the device's mapping (tests/launch_geometry_test.cpp).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define QBVH_HD __host__ __device__
#else
#define QBVH_HD
#endif

namespace qbi {

// Queries per wavefront of one type of a system of several types.  A type
// with fewer than an eighth of the system's particles is sparse: its
// Z-consecutive queries lie far apart, so a wavefront of many of them walks a
// very wide union and runs far longer than the others; such a type takes at
// most kSparseQpw queries per wavefront.
constexpr int32_t kSparseQpw = 16;
QBVH_HD inline int32_t type_qpw(int64_t count, int64_t n, int32_t qpw) {
    return (count * 8 < n && qpw > kSparseQpw) ? kSparseQpw : qpw;
}

// A system of several types is traversed in eight stretches; stretch `part`
// takes queries [stretch_lo(count, part), stretch_lo(count, part + 1)) of a
// type of `count` particles, in type_waves(...) wavefronts.
QBVH_HD inline int32_t stretch_lo(int64_t count, int64_t part) { return (int32_t)(count * part / 8); }
QBVH_HD inline int32_t type_waves(int64_t count, int64_t n, int32_t qpw, int64_t part) {
    const int32_t len = stretch_lo(count, part + 1) - stretch_lo(count, part);
    const int32_t qt = type_qpw(count, n, qpw);
    return (len + qt - 1) / qt;
}

// Traversal workgroups of a system whose wavefronts take `qpw` queries each.
// A system of several types gets eight equal stretches, each with room for
// an eighth of every type (see the traversal's query order); the count is an
// upper bound there (the device knows the type sizes, the host does not), and
// wavefronts past a stretch's share exit at once.  Per stretch a type t takes
// len_t <= ceil(count_t / 8) queries in ceil(len_t / qpw_t) wavefronts, so
//   waves <= sum_t (len_t / qpw_t + 1)
//         <= (ceil(n/8) + ntypes) / qpw + (ntypes - 1) (ceil(n/64) + 1) / min(qpw, kSparseQpw) + ntypes,
// the second term bounding the sparse types (each has len_t <= ceil(n/64)).
// An empty system gets none, whatever its types: nothing writes the tree
// descriptions its workgroups would size their queries from.
inline int64_t trav_blocks(int64_t n, int32_t ntypes, int32_t block, int32_t qpw = 64) {
    if (n <= 0) return 0;
    const int64_t per_wg = (int64_t)(block / 64) * qpw;
    if (ntypes <= 1) return (n + per_wg - 1) / per_wg;
    const int64_t sq = qpw > kSparseQpw ? kSparseQpw : qpw;
    const int64_t dense = ((n + 7) / 8 + ntypes + qpw - 1) / qpw;
    const int64_t sparse = (int64_t)(ntypes - 1) * (((n + 63) / 64 + 1 + sq - 1) / sq);
    const int64_t waves = dense + sparse + ntypes;
    return 8 * ((waves + block / 64 - 1) / (block / 64));
}

// Query order.  A system of one type takes its queries in sorted (Z) order,
// qpw per wavefront.  In a system of several types, the workgroups form
// eight equal stretches (one per XCD when the system covers the whole
// launch); stretch x takes the x-th eighth of every type's queries, smallest
// type first, in wavefronts of type_qpw queries of one type.  A sparse type's
// wavefronts span the widest regions and run longest: this way they start
// first, are spread over the stretches, and each takes few queries, instead
// of closing the launch on one XCD.  `wg` is the system's workgroup in
// dispatch order, `nwg` its workgroup count (trav_blocks, an upper bound
// for several types), `wave` and `lane` the place in it, `start` the system's
// first sorted position and meta[t] the start and count of type t; returns the
// lane's position in the system, or n for an idle lane (every lane of an empty
// system, whatever its descriptions hold).
template <class Meta>
QBVH_HD inline int32_t query_position(const Meta *meta, int32_t n, int32_t ntypes, int32_t qpw, int32_t start,
                                      int32_t waves_per_wg, int32_t wg, int32_t nwg, int32_t wave, int32_t lane) {
    if (n <= 0) return n;
    if (ntypes <= 1) {
        // wavefronts of qpw queries: lanes past qpw idle
        if (lane >= qpw) return n;
        return (wg * waves_per_wg + wave) * qpw + lane;
    }
    const int32_t per = nwg / 8;
    const int64_t part = wg / per;
    int32_t wi = (wg % per) * waves_per_wg + wave;  // wavefront of the stretch
    for (int r = 0; r < ntypes; ++r) {
        // the type of rank r by (count, type index)
        int t = 0;
        for (int u = 0; u < ntypes; ++u) {
            int rank = 0;
            for (int w = 0; w < ntypes; ++w)
                rank += (meta[w].count < meta[u].count || (meta[w].count == meta[u].count && w < u)) ? 1 : 0;
            if (rank == r) t = u;
        }
        const int64_t len = meta[t].count;
        const int32_t lo = stretch_lo(len, part), hi = stretch_lo(len, part + 1);
        const int32_t qt = type_qpw(len, n, qpw);
        const int32_t nw = type_waves(len, n, qpw, part);
        if (wi < nw) {
            const int32_t j = wi * qt + lane;
            return (lane < qt && j < hi - lo) ? meta[t].start - start + lo + j : n;
        }
        wi -= nw;
    }
    return n;
}

}  // namespace qbi
