// Paper-mode lists (Section 2.3, nlist_build_ex with QBVH_LIST_PAPER): one lane
// per Z-ordered particle, the lanes of a wavefront walking the rope-linked
// quantized tree together (Algorithm 1).
//
// Per wavefront and per type tree:
//   1. image mask per lane: which of the 27 periodic images of its search
//      sphere touch the tree's root box (the image test of Algorithm 1); the wavefront
//      visits the union of its lanes' images;
//   2. per image, one stackless walk over the two-wide records, shared by the
//      wavefront.  A step loads one record (both child boxes and references)
//      and its rope with uniform (scalar) loads; every lane tests its own
//      sphere against both boxes in grid units (nearest point by a clamp per
//      axis, eq. (2)); a ballot over the lanes decides the step: the left
//      child's record if any lane hit that box, else the right child's record
//      if any lane hit that one, else the rope.  A lane whose sphere misses a
//      node misses everything below it, so the wavefront walks exactly the
//      union of the lanes' own walks;
//   3. a hit particle run is fetched once (uniform loads) and each particle's
//      cell box tested by the lanes that hit the run.
//
// Grid-unit test.  With h the tree's bin width and g(x) = (x - root_lo) / h,
// a quantized bound q decodes exactly to the float 2^23 + q (bit trick: OR
// with 0x4B000000), and the query image is placed at 2^23 + g(x) rounded to
// fp32.  Rounding of the query position, of the differences and of the sum of
// squares is covered by comparing against
//   ((R / h) * (1 + 2^-20) + 2)^2 * (1 + 2^-20),
// a pad of two bins plus a relative 2^-20, so no listed pair is lost.
#include "build_common.h"
#include "query_order.h"

namespace qbi {
namespace {

// Decoding a 16-bit bound q of a record word held in a scalar register: the
// float with bits 0x4B000000 | q is exactly 2^23 + q.  The lower bound is
// decoded by the scalar unit (s_pack_ll_b32_b16 puts 0x4B00 above the low half
// word), the upper one by the VALU (v_or_b32 with a 16-bit source select of
// the scalar word against the bias held in a VGPR).  Splitting the decodes
// balances the two issue slots of the shared walk, and leaves the clamp with
// one scalar and one vector bound (a VALU op may read one scalar operand).
__device__ __forceinline__ uint32_t vgpr_bias() {
    uint32_t v;
    asm volatile("v_mov_b32 %0, 0x4b000000" : "=v"(v));
    return v;
}

__device__ __forceinline__ float lo_bound(uint32_t w) {
    float r;
    asm("s_pack_ll_b32_b16 %0, %1, 0x4b00" : "=s"(r) : "s"(w));
    return r;
}

__device__ __forceinline__ float hi_bound(uint32_t w, uint32_t bias) {
    float r;
    asm("v_or_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD"
        : "=v"(r)
        : "s"(w), "v"(bias));
    return r;
}

// Squared grid-unit distance from the query (ux, uy, uz) to a packed box.
__device__ __forceinline__ float box_d2(uint32_t wx, uint32_t wy, uint32_t wz, float ux, float uy, float uz,
                                        uint32_t bias) {
    const float cx = __builtin_amdgcn_fmed3f(ux, lo_bound(wx), hi_bound(wx, bias)) - ux;
    const float cy = __builtin_amdgcn_fmed3f(uy, lo_bound(wy), hi_bound(wy, bias)) - uy;
    const float cz = __builtin_amdgcn_fmed3f(uz, lo_bound(wz), hi_bound(wz, bias)) - uz;
    return __builtin_fmaf(cz, cz, __builtin_fmaf(cy, cy, cx * cx));
}

__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// Row staging.  Each lane keeps its newest list entries in a ring of kRing
// LDS slots (its own column, so lanes never share a bank row) and writes them
// to its row kFlush at a time: with 16-byte aligned rows as two 16-byte
// stores.  A candidate's index is written to the lane's next free slot
// whether or not it is accepted, and the count advances only on acceptance,
// so the per-candidate path has no branch.  Runs are taken 8 particles at a
// time and the ring is flushed after each such part once kFlush entries wait,
// so no more than 15 entries are ever pending.
constexpr int kRing = 16;
constexpr int kFlush = 8;

struct Lane {
    float x, y, z;         // query position
    float ux, uy, uz;      // query image in grid units (2^23 offset form)
    float r2g;             // padded squared radius in grid units (negative: lane idle)
    int32_t k, orig;
    int32_t cnt;           // entries of the list so far
    int32_t flushed;       // entries already written to the row (a multiple of kFlush)
    float px, py, pz;      // query image in per-axis grid units (plain, not offset)
    float phx, phy, phz;   // bin width of each axis
    float rp2;             // squared tight radius (world units)
};

template <bool kVec4, int kBlock>
__device__ __forceinline__ void flush_ring(Lane &q, int32_t (*s_out)[kBlock], int32_t *nbr, int32_t max_nbr) {
    const int32_t f = q.flushed;
    const int s0 = f & (kRing - 1);
    int32_t *row = nbr + ((int64_t)q.orig * max_nbr + f);
    if (kVec4) {
        // f and max_nbr are multiples of 4 here; one compare covers the usual
        // case of a row with room for all eight
        const int4 lo = make_int4(s_out[s0][threadIdx.x], s_out[s0 + 1][threadIdx.x], s_out[s0 + 2][threadIdx.x],
                                  s_out[s0 + 3][threadIdx.x]);
        if (f <= max_nbr - 8) {
            *reinterpret_cast<int4 *>(row) = lo;
            *reinterpret_cast<int4 *>(row + 4) = make_int4(s_out[s0 + 4][threadIdx.x], s_out[s0 + 5][threadIdx.x],
                                                           s_out[s0 + 6][threadIdx.x], s_out[s0 + 7][threadIdx.x]);
        } else if (f <= max_nbr - 4) {
            *reinterpret_cast<int4 *>(row) = lo;
        }
    } else {
#pragma unroll
        for (int e = 0; e < kFlush; ++e)
            if (f + e < max_nbr) row[e] = s_out[s0 + e][threadIdx.x];
    }
    q.flushed = f + kFlush;
}

// 16-bit bound of a record-style word held in a scalar register, as a float.
__device__ __forceinline__ float cvt_lo(uint32_t w) {
    float r;
    asm("v_cvt_f32_u32_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0" : "=v"(r) : "s"(w));
    return r;
}

__device__ __forceinline__ float cvt_hi(uint32_t w) {
    float r;
    asm("v_cvt_f32_u32_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1" : "=v"(r) : "s"(w));
    return r;
}

// Paper-mode pass (Section 2.3): a particle of the run is listed when the
// lane's sphere overlaps the particle's own cell box (its leaf box in the
// quantized tree, on the paper's per-axis grid), with no distance check.  The
// nearest point is found in each axis's grid units and scaled to world units
// by that axis's bin width; the test is against the tight radius
// R (1 + 2^-20) + 0.02 max_d h_d.
template <bool kSelf, int kBlock>
__device__ __forceinline__ void run_paper(const uint4 *__restrict__ qrun, uint32_t count, uint32_t rel, bool hit,
                                          Lane &q, int32_t (*s_out)[kBlock]) {
    uint4 b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) b[u] = qrun[u];
    asm volatile("" ::"s"(b[0].x), "s"(b[4].x));
    const float r2 = hit ? q.rp2 : -1.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if ((uint32_t)u >= count) break;
        const float cx = (__builtin_amdgcn_fmed3f(q.px, cvt_lo(b[u].x), cvt_hi(b[u].x)) - q.px) * q.phx;
        const float cy = (__builtin_amdgcn_fmed3f(q.py, cvt_lo(b[u].y), cvt_hi(b[u].y)) - q.py) * q.phy;
        const float cz = (__builtin_amdgcn_fmed3f(q.pz, cvt_lo(b[u].z), cvt_hi(b[u].z)) - q.pz) * q.phz;
        const float d2 = __builtin_fmaf(cz, cz, __builtin_fmaf(cy, cy, cx * cx));
        const bool other = !kSelf || (uint32_t)u != rel;
        s_out[q.cnt & (kRing - 1)][threadIdx.x] = (int32_t)b[u].w;
        q.cnt += (d2 <= r2 && other) ? 1 : 0;
    }
}

// The particles of one hit run for the lanes with `hit` set.  A run
// of up to 16 particles is taken in halves of at most 8: each half adds at
// most 8 entries to a ring holding fewer than kFlush, and the ring is
// flushed after every half.
template <bool kVec4, int kBlock>
__device__ __forceinline__ void take_run(int32_t ref, bool hit, Lane &q, int img, const uint4 *__restrict__ qpoint,
                                         uint32_t nend, int32_t (*s_out)[kBlock], int32_t *nbr, int32_t max_nbr) {
    const int32_t v = ~ref;
    const uint32_t first = (uint32_t)uniform(v >> kRunCountBits);
    const uint32_t count = (uint32_t)uniform((v & kRunCountMask) + 1);
    // a well-formed tree never fails this; it keeps a corrupt reference from
    // reading outside the particle array
    if (first + count > nend) return;
    for (uint32_t h0 = 0; h0 < count; h0 += 8) {
        const uint32_t c8 = count - h0 < 8u ? count - h0 : 8u;
        // the lane's own particle can only be accepted through the unshifted image
        const uint32_t rel = (uint32_t)(q.k - (int32_t)(first + h0));
        const bool self = img == 13 && __any(hit && rel < c8);
        if (self)
            run_paper<true, kBlock>(qpoint + first + h0, c8, rel, hit, q, s_out);
        else
            run_paper<false, kBlock>(qpoint + first + h0, c8, rel, hit, q, s_out);
        // a plain per-lane branch: the wavefront skips it when no lane's
        // condition holds, with one compare instead of a ballot and a test
        if (q.cnt - q.flushed >= kFlush)
            flush_ring<kVec4, kBlock>(q, s_out, nbr, max_nbr);
    }
}

// One workgroup of queries; li >= a.n is an idle lane.
template <bool kVec4, int kBlock>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) void k_traverse_paper(
    TravArgs a, const uint4 *__restrict__ records, const int32_t *__restrict__ ropes,
    const float4 *__restrict__ sorted, const uint4 *__restrict__ qpoint, const TreeMeta *__restrict__ meta) {
    __shared__ int32_t s_out[kRing][kBlock];
    const int32_t li = query_position<kBlock>(a, meta, xcd_logical_block(), (int32_t)gridDim.x);
    const bool valid = li < a.n;  // idle lanes still take part in the shared walk
    const int32_t k = a.start + li;
    const uint32_t nend = (uint32_t)(a.start + a.n);

    Lane q;
    const float4 qp = sorted[valid ? k : a.start];
    q.x = qp.x;
    q.y = qp.y;
    q.z = qp.z;
    q.k = k;
    q.orig = ~__float_as_int(qp.w);
    int ta = 0;
    for (int t = 1; t < a.ntypes; ++t)
        if (k >= meta[t].start) ta = t;

    q.cnt = 0;
    q.flushed = 0;
    const uint32_t bias = vgpr_bias();
    for (int tb = 0; tb < a.ntypes; ++tb) {
        const TreeMeta &m = meta[tb];
        if (m.count == 0) continue;
        double r2 = a.rlist2[tb];
        for (int t = 1; t < a.ntypes; ++t)
            if (ta == t) r2 = a.rlist2[t * QBVH_MAX_TYPES + tb];
        const bool lane_on = valid && r2 >= 0.0;
        const double R = lane_on ? sqrt(r2) : 0.0;

        // (1) image mask against the root box (the image test of Algorithm 1), in fp32
        // with an outward pad of 2^-18 of the largest box edge (far above the
        // fp32 rounding of the shifted coordinates) plus 2^-20 relative.
        uint32_t bits = 0;
        if (lane_on) {
            const float pad = (float)(a.lmax * 0x1p-18);
            const float rimg = (float)R * (1.0f + 0x1p-20f) + pad;
            const float rimg2 = rimg * rimg;
            float e2[3][3];
            const float xq[3] = {q.x, q.y, q.z};
#pragma unroll
            for (int dd = 0; dd < 3; ++dd) {
#pragma unroll
                for (int sh = 0; sh < 3; ++sh) {
                    const float p = xq[dd] + (float)(sh - 1) * a.Lf[dd];
                    const float e = fmaxf(fmaxf(m.lo[dd] - p, p - m.hi[dd]), 0.0f);
                    e2[dd][sh] = e * e;
                }
            }
#pragma unroll
            for (int img = 0; img < 27; ++img) {
                const float sum = (e2[0][img % 3] + e2[1][(img / 3) % 3]) + e2[2][img / 9];
                if (sum <= rimg2) bits |= 1u << img;
            }
        }
        uint32_t wave_bits = bits;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) wave_bits |= (uint32_t)__shfl_xor((int)wave_bits, o, 64);
        wave_bits = (uint32_t)uniform((int32_t)wave_bits);

        const double rg = R * m.inv_h;
        const double rgp = rg * (1.0 + 0x1p-20) + 2.0;
        const float r2g = lane_on ? (float)(rgp * rgp * (1.0 + 0x1p-20)) : -1.0f;
        const int32_t root = m.root, end = m.end;
        double ph[3];
        // the paper's per-axis bins (as the cell boxes were quantized); the
        // pad covers the rounding of the query's grid position (at most
        // 2^-24 of 65535 bins per axis) and of the fp32 distance
        double hmax = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            ph[d] = axis_spacing(m.lo[d], m.hi[d], a.lmax * 0x1p-24, a.qbits);
            hmax = ph[d] > hmax ? ph[d] : hmax;
        }
        q.phx = (float)ph[0];
        q.phy = (float)ph[1];
        q.phz = (float)ph[2];
        const double rp = R * (1.0 + 0x1p-20) + 0.02 * hmax;
        q.rp2 = (float)(rp * rp * (1.0 + 0x1p-20));

        // (2) one shared stackless walk per image in the union (the walk of Algorithm 1)
        while (wave_bits) {
            const int img = __builtin_ctz(wave_bits);
            wave_bits &= wave_bits - 1u;
            const bool on = (bits >> img) & 1u;
            q.r2g = on ? r2g : -1.0f;
            const double sx = (double)(img % 3 - 1) * a.L[0];
            const double sy = (double)((img / 3) % 3 - 1) * a.L[1];
            const double sz = (double)(img / 9 - 1) * a.L[2];
            q.ux = (float)((((double)q.x + sx) - (double)m.lo[0]) * m.inv_h + 8388608.0);
            q.uy = (float)((((double)q.y + sy) - (double)m.lo[1]) * m.inv_h + 8388608.0);
            q.uz = (float)((((double)q.z + sz) - (double)m.lo[2]) * m.inv_h + 8388608.0);
            q.px = (float)((((double)q.x + sx) - (double)m.lo[0]) / ph[0]);
            q.py = (float)((((double)q.y + sy) - (double)m.lo[1]) / ph[1]);
            q.pz = (float)((((double)q.z + sz) - (double)m.lo[2]) / ph[2]);
            if (root < 0) {  // a tree of at most leaf_size particles is one run
                take_run<kVec4, kBlock>(root, on, q, img, qpoint, nend, s_out, a.nbr, a.max_nbr);
                continue;
            }
            int32_t v = root;
            while (v < end) {
                // 32-bit byte offsets keep the address arithmetic to one scalar op
                const uint32_t off = (uint32_t)v << 5;
                const uint4 r0 = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(records) + off);
                const uint4 r1 = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(records) + off + 16u);
                const int32_t rope =
                    *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(ropes) + ((uint32_t)v << 2));
                const bool hl = box_d2(r0.x, r0.y, r0.z, q.ux, q.uy, q.uz, bias) <= q.r2g;
                const uint64_t ml = __ballot(hl);
                const bool anyl = ml != 0;
                const int32_t cl = (int32_t)r1.z, cr = (int32_t)r1.w;
                if (cl < 0 && anyl)
                    take_run<kVec4, kBlock>(cl, hl, q, img, qpoint, nend, s_out, a.nbr, a.max_nbr);
                // Descending into an internal left child with an internal right
                // child, the right box is not needed: the walk reaches the right
                // child's record by the left subtree's rope and tests its
                // children there (they lie inside its box).
                int32_t next = cl;
                if (!(anyl && cl >= 0 && cr >= 0)) {
                    const bool hr = box_d2(r0.w, r1.x, r1.y, q.ux, q.uy, q.uz, bias) <= q.r2g;
                    const uint64_t mr = __ballot(hr);
                    const bool anyr = mr != 0;
                    if (cr < 0 && anyr)
                        take_run<kVec4, kBlock>(cr, hr, q, img, qpoint, nend, s_out, a.nbr, a.max_nbr);
                    next = (anyl && cl >= 0) ? cl : ((anyr && cr >= 0) ? cr : rope);
                }
                // references always point forward; max() makes progress unconditional
                v = uniform(max(next, v + 1));
            }
        }
    }

    if (!valid) return;
    a.count[q.orig] = q.cnt;
    // the last (fewer than kFlush) entries
    const int32_t f = q.flushed, s0 = f & (kRing - 1);
    int32_t *row = a.nbr + ((int64_t)q.orig * a.max_nbr + f);
    for (int32_t e = 0; e < q.cnt - f; ++e)
        if (f + e < a.max_nbr) row[e] = s_out[(s0 + e) & (kRing - 1)][threadIdx.x];
    if (q.cnt > a.max_nbr) atomicOr(a.overflow, 1);
}

template <bool kVec4, int kBlock>
void launch_one(const TravArgs &a, const uint4 *qpoint, hipStream_t s) {
    const unsigned grid = (unsigned)trav_blocks(a.n, a.ntypes, kBlock, a.qpw);
    hipLaunchKernelGGL((k_traverse_paper<kVec4, kBlock>), dim3(grid), dim3(kBlock), 0, s, a, a.records, a.ropes,
                       a.sorted, qpoint, a.meta);
}

template <bool kVec4>
void launch_block(const TravArgs &a, int32_t block, const uint4 *qpoint, hipStream_t s) {
    switch (block) {
    case 64: launch_one<kVec4, 64>(a, qpoint, s); break;
    case 128: launch_one<kVec4, 128>(a, qpoint, s); break;
    case 192: launch_one<kVec4, 192>(a, qpoint, s); break;
    default: launch_one<kVec4, 256>(a, qpoint, s); break;
    }
}

}  // namespace

hipError_t launch_traverse_paper(const TravArgs &a, int32_t block, bool vec4, const uint4 *qpoint, hipStream_t s) {
    if (vec4)
        launch_block<true>(a, block, qpoint, s);
    else
        launch_block<false>(a, block, qpoint, s);
    return hipGetLastError();
}

}  // namespace qbi
