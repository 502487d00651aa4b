// Neighbor-list traversal (Algorithm 1; Section 2.3; Section 3 runs the
// queries in Z order so that the queries of a wavefront need similar
// subtrees).  A wavefront takes up to 64 Z-consecutive queries
// of one type and does two things in turn:
//
//   walk      lanes are tree nodes.  A stack in LDS holds the nodes still to
//             open, in preorder, of all periodic images together.  A round
//             takes the 32 next ones, two lanes each: a lane loads one child
//             box and reference of its record and tests the box against the
//             queries' search region (the image test and the node test of
//             Algorithm 1, eq. (2)).  Hit runs that precede every hit internal
//             node go to a queue of run parts of at most 8 particles; the
//             rest goes back on the stack, in order, so candidates come out
//             in exactly the order of a depth-first walk (a record's runs
//             before its internal child).
//   test      lanes are candidates, then queries.  Eight parts (64 candidates)
//             are loaded, one per lane, and tested against all 64 queries on
//             the matrix cores: with c and q relative to the wavefront's own
//             origin, d^2 - R^2 = (|q|^2 - R^2) + |c|^2 - 2 q.c is one
//             16x16x4 fp32 product per 16 candidates and 16 queries.  The
//             signs of the results are the accept mask of each query.
//
// The search region is the union of kSegs boxes around consecutive queries,
// cut where neighbouring queries lie farthest apart (Z order jumps), grown by
// R, or the queries' own spheres where these are much less (see kSphereCost).
// For 64 queries of an LJ fluid at R = 3.4 four boxes meet 3% more candidates
// than the 64 spheres themselves do, and two boxes, which take half the
// instructions per node, measured faster on every workload (N = 1M: LJ 565 ->
// 560 us, WCA 268 -> 257 us).
//
// Exactness.  |v| <= band (v the product's d^2 - R^2) marks the pairs that
// need more: they are decided, one by one, by an fp32 distance with a proven
// error band (see decide_pair) and inside that by the fp64 arithmetic of the
// list definition, so the lists are exact.  The band is derived at
// pair_band().
//
// Cost.  At N = 8M (LJ, R = 3.4) a wavefront issues 13.2k VALU instructions
// and 436 matrix products (26 batches, 25 rounds) and the VALU is busy 65% of
// the time; of 4.12 ms the walk takes 1.0, the tests 1.8, taking the rows'
// entries from the masks 0.8 and storing the rows 0.65 (4.5 GB).  With one lane
// per query walking and testing every candidate itself a wavefront issued
// 26.1k VALU and 21.1k scalar instructions.  Traversal before and now: LJ 8M
// 6.09 -> 4.12 ms, 1M 942 -> 509 us, 4000 102 -> 33 us, WCA 1M 533 -> 230 us,
// two-type mixture 1M 523 -> 274 us.
//
// Paper-mode lists (Section 2.3: a particle is listed when the query's sphere
// overlaps the particle's own cell box, with no distance check) take the same
// walk and the same products, with the middle of the cell box for the particle:
// within R and the cell's inscribed radius a pair is listed, beyond the tight
// radius and half the cell's diagonal it is not; the pairs between are decided
// one by one by the cell box (see decide_cell).  With the particle itself the
// pairs between span a whole diagonal, five times as many.
//
// Row order.  A row lists, image by image and tree order within an image, the
// candidates of each run part that the fp32 distance accepts, then those of
// the part that the fp64 arithmetic accepts.
#include "build_common.h"

namespace qbi {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)x);
}
__device__ __forceinline__ float uniform(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ float lane_value(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// A lane's bit of a wave-uniform mask.
__device__ __forceinline__ bool lane_bit(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// LDS written by some lanes of the wavefront is read by others after this
// (a wavefront's LDS operations complete in order; this keeps the compiler
// from reordering them).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Search-region boxes per wavefront.
constexpr int kSegs = 2;
// Scattered queries.  Where a wavefront's queries lie far apart (a type with few
// particles, the vapour around a droplet), two boxes around them may hold half
// the system: then nodes are tested against each query's own sphere instead.
// With V the boxes' volume grown by R, U the spheres' union and rho the tree's
// density, boxes meet rho (V - U) more candidates, 64 to a batch of about 500
// instructions; the spheres cost 13 instructions per query and round, in
// rho U / 64 rounds and those at the top of the tree, where few nodes are on the
// stack, and in any case some latency per round.  So spheres are taken when
//   rho (V - U (1 + nq / 40)) > 8 (nq + 8).
// Measured, boxes only and with this rule (whole call): 60 particles of a second
// type among 1M 6340 -> 710 us, among 4M 29.1 -> 2.87 ms, 300 among 100k 613 ->
// 339 us; 1M particles of a droplet with 1% vapour 5.18 -> 0.67 ms; a gas of
// density 0.001, where V / U is large and rho V small, 320 -> 321 us (682 when
// the volumes alone decide).  2 (nq + 8) in place of 8 takes spheres too often
// (two types of 20k and 980k 458 -> 482 us), 16 too rarely (droplet of 100k with
// 1% vapour 199 -> 294 us).
constexpr float kSphereCost = 1.0f / 40.0f;
constexpr float kSphereRounds = 8.0f;
// A tree that cannot tell its particles apart (many more of them in a Morton bin
// than the spheres hold) is searched whole by spheres too, so they are given up
// for it after this many rounds in a row in which they miss no more than an eighth
// of the nodes: 500k particles, most of them outside the box and so in its first
// bin, 60 -> 12 ms (boxes only 11.6).  12 rounds give them up too early (1M
// particles in 40 clusters 2.74 -> 3.09 ms).
constexpr int32_t kPatience = 16;
// Queries in places far apart.  The band of pairs that the products leave to the
// exact test grows with the square of the wavefront's extent (see pair_band): at
// a gap of 512 R between two queries it holds 37% of R^2, from about 850 R all.
// So a wavefront with up to kWideGaps gaps wider than kWideGap R (it spans
// clusters in a wide box) takes its queries up to the first gap, then the rest,
// each part with its own origin and boxes.  (More gaps: a thin gas, with few
// pairs to test.)  100 clusters of 2000 particles at R = 2.8 in a box of edge
// 10^4 1400 -> 414 us, of edge 10^5 1619 -> 508, 8 of 25000 in 10^4 2.61 -> 0.92
// ms (whole calls).  The parts take 8 more registers from the walk, which costs 2%
// of LJ 1M, so only boxes with room for such a gap get the kernels with them.  A
// line at 256 R would give those clusters another 2% to 20% and takes 3% from 1M
// particles of a gas of density 0.001.
constexpr float kWideGap = 512.0f;
constexpr int kWideGaps = 3;
// Nodes opened per round (two lanes each).
constexpr int kOpen = 32;
// Stack entries.  A round that opens p nodes adds at most p entries; p is held
// to the room left below kStack - kDepthMax, and to one node when there is
// none: from then on the walk is depth first and one node deep per level, so
// it adds at most the depth of the record tree, kDepthMax (a radix tree over
// 32-bit keys and 32-bit positions has at most 64 internal levels), before it
// comes back to where it was.
constexpr int kDepthMax = 64;
constexpr int kStack = 160;
static_assert(kStack - kDepthMax >= 27 + kOpen, "room for every image's root");
// The square of a distance that nothing listed has: what an empty slot's or an
// idle lane's products start from.  Above every |q|^2, R^2 and band of boxes whose
// edges are below 1e17 (to larger ones, and to wavefronts as wide, the products do
// not apply), and low enough that its sum with any |c|^2 below 1e37 is finite.
constexpr float kFar = 1e36f;
// Queue of run parts: parts of fewer than 64 particles in all wait when a
// round adds those of at most 2 kOpen runs, two parts each.
constexpr int kParts = 64 + 4 * kOpen;
// Rows.  A batch leaves each query up to four words (16 candidates each) of
// accepted candidates; empty ones are not kept.  They wait in LDS, with the
// candidates' original indices, until a query's words or the index tables
// might not hold another batch; then every lane writes its row from its words,
// four entries (16 bytes) at a time.  Waiting pays twice: the lanes of a
// wavefront step together, and over several batches their entries are of more
// nearly equal number (one batch gives 0 to 16 entries a lane, five give 33 +- 7);
// and a row's 128-byte lines are filled in one go instead of being written
// back in parts.  Fewer than four entries are carried over in LDS.
constexpr int kWords = 16;
constexpr int kTables = 8;

// Few queries.  With at most 16 queries per wavefront (small systems) a query's
// four lanes, one per row of 16 lanes, each hold the mask of a quarter of the
// batch as the products leave it.  They write their entries straight to the
// row, each from its own place in it, and nothing is queued: serial steps
// count there, not stores (traversal of 1000 particles 32 -> 23 us, 30k 69 -> 59).
constexpr int kFewQueries = 16;

// One wavefront's LDS: 9.6 KB, so four wavefronts per SIMD fit a compute unit.
template <bool kFew>
struct WaveLds {
    uint32_t word[kFew ? 1 : kWords + 1][64];  // per query: candidate mask (16 bits, first highest), byte
                                               // offset into index
    int32_t index[kFew ? 64 : kTables * 64 + 64 * 4];  // original indices of each batch's candidates; the
                                                       // entries carried over
    int32_t sref[kStack];           // stack: record index, or run reference (< 0)
    uint2 part[kParts];             // queue: first sorted position, length - 1 from bit 27; particles
                                    // queued before the part, image code from bit 16
    uint8_t simg[kStack];           // image codes
    uint8_t map[64];                // scratch: part starts by slot; candidate slot of each query's own particle
};
static_assert(sizeof(WaveLds<false>) <= 10240, "four wavefronts per SIMD");

// Periodic image m in {-1, 0, 1}^3 as three 2-bit fields m + 1; kHome is m = 0.
constexpr uint32_t kHome = 1u | (1u << 2) | (1u << 4);

// List semantics: exact lists of fp32 or of fp64 data, paper-mode lists.
enum Mode { kExact, kExact64, kPaper };

// Paper mode: an image of a query in a tree's grid.
struct CellQuery {
    float p[3];  // position in bins
    bool in;     // the sphere touches the tree's root box
};

// Per-query state of a lane.
struct Query {
    int32_t k, orig;
    int32_t cnt;      // entries of the row so far
    int32_t done;     // entries written to the row (a multiple of 4)
    uint32_t words;   // words waiting
    uint32_t carry;   // entries carried over (fewer than 4)
    bool valid;
    CellQuery home;   // paper mode: itself, unshifted, as the present tree sees it
};

// A type tree as the test sees it (wave-uniform).
struct TreeTest {
    float r2in, r2out;   // accept and reject thresholds of the fp32 distance
    double r2;           // exact squared list radius
    // |v| that needs the fp32 distance: home image, other images (paper mode:
    // that needs the cell box; batches with a cell of no width on some axis)
    float band, band_img;
    bool force;          // coordinates too large for the product: every pair needs it
    // paper mode: bin width of each axis, squared tight radius, squared radius
    // of the image test
    double h[3];
    float hf[3];
    float rp2, rimg2;
};

// ------------------------------------------------------------------ rows

// Writes the rows' waiting entries, all but the last (fewer than 4) of each.
template <bool kVec4>
__device__ __forceinline__ void write_rows(Query &q, WaveLds<false> &w, int32_t *nbr, int32_t max_nbr, uint32_t lane) {
    const uint32_t mine = kTables * 64 + lane * 4;  // the lane's carried entries
    w.word[q.words][lane] = 0;
    // the word in hand and the next one
    uint32_t cur = ~(0xFFFFFFFFu >> q.carry) | (mine * 4u);
    uint32_t nxt = w.word[0][lane];
    uint32_t at = 0;
    auto next = [&]() {
        const bool empty = cur < 0x10000u;
        cur = empty ? nxt : cur;
        at += empty ? 1u : 0u;
        nxt = w.word[at][lane];
        const uint32_t b = (uint32_t)__builtin_clz(cur);
        cur ^= 0x80000000u >> b;
        return *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(w.index) + ((cur & 0xFFFFu) + (b << 2)));
    };
    int32_t left = q.cnt - q.done;
    int32_t *row = nbr + ((int64_t)q.orig * max_nbr + q.done);
    while (left >= 4) {
        int4 e;
        e.x = next();
        e.y = next();
        e.z = next();
        e.w = next();
        if (kVec4) {
            // done and max_nbr are multiples of 4 here
            if (q.done < max_nbr) *reinterpret_cast<int4 *>(row) = e;
        } else {
            if (q.done + 0 < max_nbr) row[0] = e.x;
            if (q.done + 1 < max_nbr) row[1] = e.y;
            if (q.done + 2 < max_nbr) row[2] = e.z;
            if (q.done + 3 < max_nbr) row[3] = e.w;
        }
        row += 4;
        q.done += 4;
        left -= 4;
    }
    // (a step never reads a carried entry that an earlier one has replaced)
    for (int32_t i = 0; i < left; ++i) w.index[mine + i] = next();
    q.carry = (uint32_t)left;
    q.words = 0;
    wave_lds_sync();
}

// Queues the candidates `m` (first of 32 slots highest) of a batch; `base` is
// the byte offset of their indices.
__device__ __forceinline__ void add_words(uint32_t m, uint32_t base, Query &q, WaveLds<false> &w, uint32_t lane) {
    const uint32_t a = (m & 0xFFFF0000u) | base, b = (m << 16) | (base + 64u);
    w.word[q.words][lane] = a;
    q.words += a >= 0x10000u ? 1u : 0u;
    w.word[q.words][lane] = b;
    q.words += b >= 0x10000u ? 1u : 0u;
}

// ------------------------------------------------------------------ pairs

// Exchanges rows and registers: with rows the four groups of 16 lanes, on
// return register t's row c holds what register c's row t held.
__device__ __forceinline__ void transpose4(uint32_t &a, uint32_t &b, uint32_t &c, uint32_t &d) {
    auto p = __builtin_amdgcn_permlane32_swap(a, c, false, false);
    auto q = __builtin_amdgcn_permlane32_swap(b, d, false, false);
    auto r = __builtin_amdgcn_permlane16_swap(p[0], q[0], false, false);
    auto s = __builtin_amdgcn_permlane16_swap(p[1], q[1], false, false);
    a = r[0];
    b = r[1];
    c = s[0];
    d = s[1];
}

__device__ __forceinline__ void transpose4(float &a, float &b, float &c, float &d) {
    uint32_t x = __float_as_uint(a), y = __float_as_uint(b), z = __float_as_uint(c), u = __float_as_uint(d);
    transpose4(x, y, z, u);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
    c = __uint_as_float(z);
    d = __uint_as_float(u);
}

// Batch slot of lane l's candidate (and lane of slot l's: the map is its own
// inverse).  The product of candidate group t leaves candidate row 4 k + i in
// register i of lane row k; with this order the (4 t + i)-th sign shifted into
// the mask there is slot 16 k + 4 t + i, so the four rows' masks concatenate
// to one mask in slot order, first slot highest.
__device__ __forceinline__ uint32_t slot_of(uint32_t l) {
    return (((l >> 2) & 3u) << 4) | (((l >> 4) & 3u) << 2) | (l & 3u);
}

__device__ __forceinline__ uint32_t shift_in_sign(uint32_t mask, float v) {
    return __builtin_amdgcn_alignbit(mask, __float_as_uint(v), 31);
}

// 64 candidates against query group g: accept mask of the lane's 16
// candidates and the smallest |v|.
__device__ __forceinline__ void test_group(const float a[4], float b, float c, uint32_t &mask, float &near) {
    const v4f cc = {c, c, c, c};
    v4f d[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b, cc, 0, 0, 0);
    uint32_t m = 0;
    float nr = __builtin_inff();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) m = shift_in_sign(m, d[t][i]);
        nr = fminf(fminf(nr, fabsf(d[t][0])), fabsf(d[t][1]));
        nr = fminf(fminf(nr, fabsf(d[t][2])), fabsf(d[t][3]));
    }
    mask = m;
    near = nr;
}

// The same products, as the mask of the pairs with |v| < band.
__device__ __forceinline__ uint32_t near_group(const float a[4], float b, float c, float band) {
    const v4f cc = {c, c, c, c};
    uint32_t m = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const v4f d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b, cc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) m = shift_in_sign(m, fabsf(d[i]) - band);
    }
    return m;
}

// fp32 pair test.  With qs = fl(x_i + m L) per axis and a = fl(x_j - qs), each
// |a - dx| <= 2^-24 (2 L + |a|), so the computed distance differs from the
// definition's by at most eta = sqrt(3) 2^-22 (2 L_max + 2 R) while the pair
// is near the cutoff.  Pairs with d32^2 <= ((R - eta)(1 - 2^-20))^2 are in,
// pairs with d32^2 > ((R + eta)(1 + 2^-20))^2 are out, the rest (a shell a few
// 1e-4 wide) take the fp64 arithmetic of the definition.
// Returns 0: out, 1: in, 2: in by the fp64 arithmetic.
template <bool kF64, class LArr>
__device__ __forceinline__ int decide_pair(const float4 &qp, int32_t k, const float4 &p, int32_t idx, uint32_t img,
                                           const TreeTest &tt, const LArr &L, const double *__restrict__ sorted64) {
    const double sx = (double)((int)(img & 3u) - 1) * L[0];
    const double sy = (double)((int)((img >> 2) & 3u) - 1) * L[1];
    const double sz = (double)((int)((img >> 4) & 3u) - 1) * L[2];
    const float ax = p.x - (float)((double)qp.x + sx), ay = p.y - (float)((double)qp.y + sy),
                az = p.z - (float)((double)qp.z + sz);
    const float d2 = __builtin_fmaf(az, az, __builtin_fmaf(ay, ay, ax * ax));
    if (d2 <= tt.r2in) return 1;
    if (!(d2 <= tt.r2out)) return 0;
    double dx, dy, dz;
    if (kF64) {
        // fp64 data: the pair's own fp64 positions
        const double *q64 = sorted64 + 4 * (int64_t)k, *p64 = sorted64 + 4 * (int64_t)idx;
        dx = (p64[0] - q64[0]) - sx;
        dy = (p64[1] - q64[1]) - sy;
        dz = (p64[2] - q64[2]) - sz;
    } else {
        dx = ((double)p.x - (double)qp.x) - sx;
        dy = ((double)p.y - (double)qp.y) - sy;
        dz = ((double)p.z - (double)qp.z) - sz;
    }
    return (dx * dx + dy * dy) + dz * dz <= tt.r2 ? 2 : 0;
}

// Paper mode: whether the query's sphere (tight radius R (1 + 2^-20) +
// 0.02 max_d h_d) overlaps the candidate's cell box `b`.  The nearest point is
// found in each axis's grid units and scaled to world units by that axis's bin
// width; the pad covers the rounding of the query's grid position (at most
// 2^-24 of 65535 bins per axis) and of the fp32 distance.  A periodic image
// counts when the sphere touches the tree's root box, in fp32 with an outward
// pad of 2^-18 of the largest box edge plus 2^-20 relative.
// The query's side of this takes three fp64 divisions, so the unshifted image's
// is kept for a whole tree.  LJ 8M on a 10-bit grid: 12.66 -> 11.99 ms, and 8.53
// with v taken to the cells' middles (100k 310 -> 296 -> 265 us for build and
// list; a lane per query testing every cell box took 10.8 ms and 489 us).
template <class LArr, class FArr>
__device__ __forceinline__ CellQuery cell_query(const float4 &qp, uint32_t img, const TreeTest &tt, const TreeMeta &m,
                                                const LArr &L, const FArr &Lf) {
    const float x[3] = {qp.x, qp.y, qp.z};
    CellQuery q;
    float e2[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int sh = (int)((img >> (2 * d)) & 3u) - 1;
        q.p[d] = (float)((((double)x[d] + (double)sh * L[d]) - (double)m.lo[d]) / tt.h[d]);
        const float y = x[d] + (float)sh * Lf[d];
        const float e = fmaxf(fmaxf(m.lo[d] - y, y - m.hi[d]), 0.0f);
        e2[d] = e * e;
    }
    q.in = (e2[0] + e2[1]) + e2[2] <= tt.rimg2;
    return q;
}

__device__ __forceinline__ bool decide_cell(const CellQuery &q, const uint4 &b, const TreeTest &tt) {
    const uint32_t w[3] = {b.x, b.y, b.z};
    float c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
        c[d] = (__builtin_amdgcn_fmed3f(q.p[d], (float)(w[d] & 0xFFFFu), (float)(w[d] >> 16)) - q.p[d]) * tt.hf[d];
    const float d2 = __builtin_fmaf(c[2], c[2], __builtin_fmaf(c[1], c[1], c[0] * c[0]));
    return d2 <= tt.rp2 && q.in;
}

// Band of the matrix-core test.  Let T be a pair's squared distance as the
// fp32 positions and the exact image shift give it, and e_s the fp32
// distance's own error near the cutoff (eta above for a shifted image; the
// unshifted one has no rounded shift: 2^-21 R).  A pair outside the band must
// be one that the fp32 distance certainly accepts (d32 <= sqrt(r2in) whenever
// T <= (sqrt(r2in) - e_s)^2) or certainly rejects, so the band is
//   max(R^2 - (sqrt(r2in) - e_s)^2, (sqrt(r2out) + e_s)^2 - R^2) + E
// with E the error of v.  With u = 2^-24, S = 2 M + R (M the largest |q|, so
// |q| + |c| <= S for a pair near the cutoff) the products and their sum cost
// at most 12 u (S^2 + R^2) (five terms, two roundings' worth each), |c|^2 and
// |q|^2 - R^2 at most 5 u (S^2 + R^2); rounding c and q moves the distance by
// at most u S, a rounded image origin by sqrt(3) u 2 L_max.  E = 24 u (S^2 +
// R^2) + 2.5 R (u S + 3.5 u L_max) covers them with room, which also keeps
// candidates far from the cutoff (their error grows with |c|^2 2^-20, their
// distance with |c|^2) from ever falling below -band.  In paper mode v is
// taken against the middle of the squared acceptance and rejection radii, and
// the band is half their difference and E.
__device__ __forceinline__ double product_error(double R, double e_o, double M) {
    const double u = 0x1p-24, S = 2.0 * M + R;
    return 24.0 * u * (S * S + R * R) + 2.5 * R * (u * S + e_o);
}

__device__ __forceinline__ float round_band(double b) { return (float)(b * (1.0 + 0x1p-20) + 1e-30); }

__device__ __forceinline__ float pair_band(double R, double rin, double rout, double e_s, double e_o, double M) {
    // r2in and r2out are rin^2 and rout^2 up to less than 2^-19 of themselves
    const double in = fmax(rin * (1.0 - 0x1p-20) - e_s, 0.0), out = rout * (1.0 + 0x1p-20) + e_s;
    return round_band(fmax(R * R - in * in, out * out - R * R) + product_error(R, e_o, M));
}

// A batch: the queue's next parts, as many whole ones as 64 slots hold; this
// lane's candidate is that of slot slot_of(lane).
struct Batch {
    uint64_t starts;   // slots at which a part starts
    uint32_t parts, slots;
    float4 p;          // (paper mode: the middle of its cell box)
    int32_t idx;       // sorted position, -1: an empty slot
    uint32_t img;
    bool flat;         // paper mode: some candidate's cell box has no width on some axis
};

template <Mode kMode, bool kFew>
__device__ __forceinline__ Batch take_batch(uint32_t at, uint32_t parts, WaveLds<kFew> &w,
                                            const float4 *__restrict__ sorted, const uint4 *__restrict__ qpoint,
                                            const TreeTest &tt, const TreeMeta &m, uint32_t lane) {
    Batch b;
    const uint2 mine = w.part[min(at + lane, parts - 1u)];
    const uint32_t base = uniform(mine.y & 0xFFFFu);
    const uint32_t s0 = (mine.y & 0xFFFFu) - base, s1 = s0 + (mine.x >> 27) + 1u;
    const uint64_t take = __ballot(at + lane < parts) & __ballot(s1 <= 64u);
    b.parts = (uint32_t)__popcll(take);
    b.slots = (uint32_t)__builtin_amdgcn_readlane((int32_t)s1, (int32_t)b.parts - 1);
    w.map[lane] = 0;
    wave_lds_sync();
    if (lane_bit(take)) w.map[s0] = 1;
    wave_lds_sync();
    b.starts = __ballot(w.map[lane] != 0);
    wave_lds_sync();
    const uint32_t slot = slot_of(lane);
    const uint64_t upto = b.starts & (~0ull >> (63u - slot));
    const uint2 part = w.part[at + (uint32_t)__popcll(upto) - 1u];
    const bool on = slot < b.slots;
    b.img = part.y >> 16;
    b.idx = (int32_t)((part.x & 0x7FFFFFFu) + (on ? slot - ((part.y & 0xFFFFu) - base) : 0u));
    b.flat = false;
    if constexpr (kMode == kPaper) {
        const uint4 c = qpoint[b.idx];
        auto middle = [&](uint32_t x, int d) {
            return __builtin_fmaf(tt.hf[d], 0.5f * (float)((x & 0xFFFFu) + (x >> 16)), m.lo[d]);
        };
        auto width0 = [](uint32_t x) { return (x & 0xFFFFu) == (x >> 16); };
        b.p = make_float4(middle(c.x, 0), middle(c.y, 1), middle(c.z, 2), __int_as_float(~(int32_t)c.w));
        b.flat = __any(on && (width0(c.x) || width0(c.y) || width0(c.z)));
    } else {
        b.p = sorted[b.idx];
    }
    if (!on) b.idx = -1;
    return b;
}

// A pair too near the cutoff for the product: 0 out, 1 in, 2 in by the fp64
// arithmetic.  ci < 0: an empty slot.
template <Mode kMode, class Args>
__device__ __forceinline__ int decide(const float4 &qp, const Query &q, int32_t ci, uint32_t img, const TreeTest &tt,
                                      Args &a, const TreeMeta &tree, const float4 *__restrict__ sorted,
                                      const double *__restrict__ sorted64, const uint4 *__restrict__ qpoint) {
    if (ci < 0) return 0;
    if constexpr (kMode == kPaper) {
        CellQuery c = q.home;
        if (img != kHome) c = cell_query(qp, img, tt, tree, a.L, a.Lf);
        return decide_cell(c, qpoint[ci], tt) ? 1 : 0;
    } else
        return decide_pair<kMode == kExact64>(qp, q.k, sorted[ci], ci, img, tt, a.L, sorted64);
}

// Slots [from, to) of a half batch as a mask, first slot highest.
__device__ __forceinline__ uint32_t slot_range(uint32_t from, uint32_t to, uint32_t half) {
    const uint32_t lo = half * 32u, a = from > lo ? min(from - lo, 32u) : 0u, b = to > lo ? min(to - lo, 32u) : 0u;
    const uint64_t ones = 0xFFFFFFFF00000000ull;
    return b > a ? (uint32_t)((ones >> b) & ~(ones >> a)) : 0u;
}

// The batch's candidates as matrix rows (c), their original indices in the
// given index table, and which of them are queries of this wavefront.  Returns
// whether some candidate comes through a shifted image.
template <bool kFew, class Args>
__device__ __forceinline__ bool stage_batch(Args &a, const Batch &t, uint32_t table, float ox, float oy, float oz,
                                            int32_t kw0, WaveLds<kFew> &w, float (&c)[4], uint64_t &mine,
                                            uint32_t lane) {
    const uint32_t slot = slot_of(lane);
    const bool on = t.idx >= 0;
    float osx = ox, osy = oy, osz = oz;
    const bool shifted = __any(on && t.img != kHome);
    if (shifted) {
        osx = (float)((double)ox + (double)((int)(t.img & 3u) - 1) * a.L[0]);
        osy = (float)((double)oy + (double)((int)((t.img >> 2) & 3u) - 1) * a.L[1]);
        osz = (float)((double)oz + (double)((int)((t.img >> 4) & 3u) - 1) * a.L[2]);
    }
    c[0] = t.p.x - osx;
    c[1] = t.p.y - osy;
    c[2] = t.p.z - osz;
    c[3] = __builtin_fmaf(c[2], c[2], __builtin_fmaf(c[1], c[1], c[0] * c[0]));
    if (!on || !(c[3] < 1e37f)) {  // (not a number: the sign of such a product would mean nothing)
        c[0] = c[1] = c[2] = 0.0f;
        c[3] = kFar;
    }
    w.index[table * 64u + slot] = ~__float_as_int(t.p.w);
    // a query's own particle is never listed: it can only come up unshifted
    mine = __ballot(on && t.img == kHome && (uint32_t)(t.idx - kw0) < 64u);
    if (mine) {
        w.map[lane] = 64;
        wave_lds_sync();
        if (lane_bit(mine)) w.map[t.idx - kw0] = (uint8_t)slot;
    }
    wave_lds_sync();
    transpose4(c[0], c[1], c[2], c[3]);
    return shifted;
}

// The batch against the wavefront's queries; accepted candidates are queued
// for the rows.  `table` is the index table it uses.
template <bool kVec4, Mode kMode, class Args>
__device__ __forceinline__ void test_batch(Args &a, const TreeTest &tt, const Batch &t, uint32_t table, int groups,
                                           const float *bq, const float *cq, float ox, float oy, float oz,
                                           int32_t kw0, Query &q, WaveLds<false> &w,
                                           const float4 *__restrict__ sorted, const double *__restrict__ sorted64,
                                           const uint4 *__restrict__ qpoint, const TreeMeta &tree, uint32_t lane) {
    float c[4];
    uint64_t mine;
    const bool shifted = stage_batch<false>(a, t, table, ox, oy, oz, kw0, w, c, mine, lane);
    uint32_t self_lo = 0, self_hi = 0;
    if (mine) {
        const uint32_t s = w.map[lane];
        self_lo = s < 32u ? 0x80000000u >> s : 0u;
        self_hi = s >= 32u && s < 64u ? 0x80000000u >> (s - 32u) : 0u;
        wave_lds_sync();
    }

    uint32_t m[4] = {0u, 0u, 0u, 0u};
    float nr[4] = {__builtin_inff(), __builtin_inff(), __builtin_inff(), __builtin_inff()};
    if (groups == 4) {
#pragma unroll
        for (int g = 0; g < 4; ++g) test_group(c, bq[g], cq[g], m[g], nr[g]);
    } else {
        test_group(c, bq[0], cq[0], m[0], nr[0]);
        if (groups > 1) test_group(c, bq[1], cq[1], m[1], nr[1]);
        if (groups > 2) test_group(c, bq[2], cq[2], m[2], nr[2]);
    }
    const float band = (kMode == kPaper ? t.flat : shifted) ? tt.band_img : tt.band;
    const bool near_any = __any(fminf(fminf(nr[0], nr[1]), fminf(nr[2], nr[3])) <= band) || tt.force;
    transpose4(m[0], m[1], m[2], m[3]);
    uint32_t lo = ((m[0] << 16) | m[1]) & ~self_lo, hi = ((m[2] << 16) | m[3]) & ~self_hi;
    const uint32_t base = table * 256u;
    if (near_any) {
        // some pair lies too near the cutoff for the product to decide
        uint32_t e[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) e[g] = __any(nr[g] <= band) ? near_group(c, bq[g], cq[g], band) : 0u;
        transpose4(e[0], e[1], e[2], e[3]);
        uint32_t nlo = (e[0] << 16) | e[1], nhi = (e[2] << 16) | e[3];
        if (tt.force) nlo = nhi = 0xFFFFFFFFu;
        nlo = q.valid ? nlo & ~self_lo : 0u;
        nhi = q.valid ? nhi & ~self_hi : 0u;
        lo &= ~nlo;
        hi &= ~nhi;
        uint32_t xlo = 0, xhi = 0;  // accepted by the fp64 arithmetic
        const float4 qp = sorted[q.k];
        while (__any((nlo | nhi) != 0u)) {
            const uint32_t b = nlo ? (uint32_t)__builtin_clz(nlo) : 32u + (uint32_t)__builtin_clz(nhi | 1u);
            const uint32_t bit = 0x80000000u >> (b & 31u);
            const int from = (int)slot_of(b);
            const int32_t ci = __shfl(t.idx, from);
            const uint32_t im = (uint32_t)__shfl((int32_t)t.img, from);
            if ((nlo | nhi) != 0u) {
                const int r = decide<kMode>(qp, q, ci, im, tt, a, tree, sorted, sorted64, qpoint);
                if (b < 32u) {
                    nlo ^= bit;
                    lo |= r == 1 ? bit : 0u;
                    xlo |= r == 2 ? bit : 0u;
                } else {
                    nhi ^= bit;
                    hi |= r == 1 ? bit : 0u;
                    xhi |= r == 2 ? bit : 0u;
                }
            }
        }
        if (kMode != kPaper && __any((xlo | xhi) != 0u)) {
            // a part's candidates that the fp64 arithmetic accepted follow
            // those the fp32 distance accepted
            auto room = [&]() {
                if (__any(q.words > (uint32_t)kWords - 4u)) {
                    wave_lds_sync();
                    write_rows<kVec4>(q, w, a.nbr, a.max_nbr, lane);
                }
            };
            uint32_t from = 0;
            for (uint64_t st = t.starts; st; st &= st - 1u) {
                const uint32_t p0 = (uint32_t)__builtin_ctzll(st);
                const uint64_t more = st & (st - 1u);
                const uint32_t p1 = more ? (uint32_t)__builtin_ctzll(more) : t.slots;
                const uint32_t x0 = xlo & slot_range(p0, p1, 0), x1 = xhi & slot_range(p0, p1, 1);
                if (!__any((x0 | x1) != 0u)) continue;
                const uint32_t y0 = lo & slot_range(from, p1, 0), y1 = hi & slot_range(from, p1, 1);
                room();
                add_words(y0, base, q, w, lane);
                add_words(y1, base + 128u, q, w, lane);
                q.cnt += (int32_t)(__popc(y0) + __popc(y1));
                room();
                add_words(x0, base, q, w, lane);
                add_words(x1, base + 128u, q, w, lane);
                q.cnt += (int32_t)(__popc(x0) + __popc(x1));
                from = p1;
            }
            lo &= slot_range(from, 64u, 0);
            hi &= slot_range(from, 64u, 1);
            room();
        }
    }
    add_words(lo, base, q, w, lane);
    add_words(hi, base + 128u, q, w, lane);
    q.cnt += (int32_t)(__popc(lo) + __popc(hi));
    wave_lds_sync();
}

// How many of a 64-slot mask's first p slots are set (first slot highest).
__device__ __forceinline__ int32_t set_before(uint64_t m, uint32_t p) {
    return p == 0u ? 0 : __popcll(m >> (64u - p));
}

// The batch against at most kFewQueries queries: lane l has query l % 16 and
// slots 16 (l / 16) .. + 15.
template <Mode kMode, class Args>
__device__ __forceinline__ void test_batch_few(Args &a, const TreeTest &tt, const Batch &t, float bq, float cq,
                                               float ox, float oy, float oz, int32_t kw0, Query &q,
                                               WaveLds<true> &w, const float4 *__restrict__ sorted,
                                               const double *__restrict__ sorted64,
                                               const uint4 *__restrict__ qpoint, const TreeMeta &tree,
                                               uint32_t lane) {
    float c[4];
    uint64_t mine;
    const bool shifted = stage_batch<true>(a, t, 0, ox, oy, oz, kw0, w, c, mine, lane);
    const uint32_t row = lane >> 4;
    const int qi = (int)(lane & 15u);
    uint32_t self = 0;
    if (mine) {
        const uint32_t s = w.map[qi];
        self = (s >> 4) == row ? 0x80000000u >> (s & 15u) : 0u;
        wave_lds_sync();
    }
    uint32_t m;
    float nr;
    test_group(c, bq, cq, m, nr);
    m = (m << 16) & ~self;
    const float band = (kMode == kPaper ? t.flat : shifted) ? tt.band_img : tt.band;
    uint32_t x = 0;  // accepted by the fp64 arithmetic
    if (__any(nr <= band) || tt.force) {
        // some pair lies too near the cutoff for the product to decide
        uint32_t near = tt.force ? 0xFFFF0000u : near_group(c, bq, cq, band) << 16;
        near = q.valid ? near & ~self : 0u;
        m &= ~near;
        const float4 qp = sorted[q.k];
        while (__any(near != 0u)) {
            const uint32_t b = (uint32_t)__builtin_clz(near | 1u) & 15u, bit = 0x80000000u >> b;
            const int from = (int)slot_of(row * 16u + b);
            const int32_t ci = __shfl(t.idx, from);
            const uint32_t im = (uint32_t)__shfl((int32_t)t.img, from);
            if (near != 0u) {
                const int r = decide<kMode>(qp, q, ci, im, tt, a, tree, sorted, sorted64, qpoint);
                near ^= bit;
                m |= r == 1 ? bit : 0u;
                x |= r == 2 ? bit : 0u;
            }
        }
    }
    int32_t *out = a.nbr + (int64_t)q.orig * a.max_nbr;
    if (kMode != kPaper && __any(x != 0u)) {
        // a part's candidates that the fp64 arithmetic accepted follow those
        // the fp32 distance accepted: each entry's place from the whole masks
        uint64_t M = 0, X = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            M = (M << 16) | ((uint32_t)__shfl((int32_t)m, qi + 16 * r) >> 16);
            X = (X << 16) | ((uint32_t)__shfl((int32_t)x, qi + 16 * r) >> 16);
        }
        uint32_t all = m | x;
        while (all) {
            const uint32_t b = (uint32_t)__builtin_clz(all), bit = 0x80000000u >> b, s = row * 16u + b;
            all ^= bit;
            const uint64_t upto = t.starts & (~0ull >> (63u - s)), after = t.starts & ~(~0ull >> (63u - s));
            const uint32_t p0 = 63u - (uint32_t)__builtin_clzll(upto),
                           p1 = after ? (uint32_t)__builtin_ctzll(after) : t.slots;
            int32_t at = q.cnt + set_before(M | X, p0);
            if (m & bit)
                at += set_before(M, s) - set_before(M, p0);
            else
                at += set_before(M, p1) - set_before(M, p0) + set_before(X, s) - set_before(X, p0);
            if (at < a.max_nbr) out[at] = w.index[s];
        }
        q.cnt += __popcll(M | X);
    } else {
        const int32_t n = __popc(m);
        const int32_t n0 = __shfl(n, qi), n1 = __shfl(n, qi + 16), n2 = __shfl(n, qi + 32), n3 = __shfl(n, qi + 48);
        int32_t at = q.cnt + (row > 0u ? n0 : 0) + (row > 1u ? n1 : 0) + (row > 2u ? n2 : 0);
        const int32_t *idx = &w.index[row * 16u];
        while (m) {
            const uint32_t b = (uint32_t)__builtin_clz(m);
            m ^= 0x80000000u >> b;
            const int32_t e = idx[b];
            if (at < a.max_nbr) out[at] = e;
            ++at;
        }
        q.cnt += (n0 + n1) + (n2 + n3);
    }
    wave_lds_sync();
}

// ------------------------------------------------------------------ walk

// An integer that orders like the float (and back).
__device__ __forceinline__ int32_t order_key(float x) {
    const int32_t i = __float_as_int(x);
    return i ^ ((i >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float from_key(int32_t k) { return __int_as_float(k ^ ((k >> 31) & 0x7FFFFFFF)); }

// Largest and smallest of the wavefront's keys.
__device__ __forceinline__ int32_t wave_max(int32_t x) {
    constexpr int32_t none = INT32_MIN;
    x = max(x, __builtin_amdgcn_update_dpp(none, x, 0x111, 0xF, 0xF, false));  // row_shr:1
    x = max(x, __builtin_amdgcn_update_dpp(none, x, 0x112, 0xF, 0xF, false));  // row_shr:2
    x = max(x, __builtin_amdgcn_update_dpp(none, x, 0x114, 0xF, 0xF, false));  // row_shr:4
    x = max(x, __builtin_amdgcn_update_dpp(none, x, 0x118, 0xF, 0xF, false));  // row_shr:8
    x = max(x, __builtin_amdgcn_update_dpp(none, x, 0x142, 0xA, 0xF, false));  // row_bcast:15 into rows 1 and 3
    x = max(x, __builtin_amdgcn_update_dpp(none, x, 0x143, 0xC, 0xF, false));  // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(x, 63);
}
__device__ __forceinline__ int32_t wave_min(int32_t x) {
    constexpr int32_t none = INT32_MAX;
    x = min(x, __builtin_amdgcn_update_dpp(none, x, 0x111, 0xF, 0xF, false));
    x = min(x, __builtin_amdgcn_update_dpp(none, x, 0x112, 0xF, 0xF, false));
    x = min(x, __builtin_amdgcn_update_dpp(none, x, 0x114, 0xF, 0xF, false));
    x = min(x, __builtin_amdgcn_update_dpp(none, x, 0x118, 0xF, 0xF, false));
    x = min(x, __builtin_amdgcn_update_dpp(none, x, 0x142, 0xA, 0xF, false));
    x = min(x, __builtin_amdgcn_update_dpp(none, x, 0x143, 0xC, 0xF, false));
    return __builtin_amdgcn_readlane(x, 63);
}

// Sum over the lanes up to and with this one.
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x) {
    int32_t v = (int32_t)x;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
    return (uint32_t)v;
}

// One wavefront of queries; this lane's query is position `li` of the system
// `a` (li >= a.n: an idle lane; the valid lanes come first).
template <bool kVec4, Mode kMode, bool kFew, class Args>
__device__ __forceinline__ void traverse_wave(Args &a, int32_t li, const uint4 *__restrict__ records,
                                              const float4 *__restrict__ sorted, const double *__restrict__ sorted64,
                                              const uint4 *__restrict__ qpoint, const TreeMeta *__restrict__ meta,
                                              WaveLds<kFew> &w) {
    const uint32_t lane = (uint32_t)(threadIdx.x & 63u);
    Query q;
    bool valid = li < a.n;
    const int32_t nq = (int32_t)__popcll(__ballot(valid));
    if (nq == 0) return;
    const int32_t kw0 = uniform(a.start + li);  // lane 0 is valid
    const uint32_t nend = (uint32_t)(a.start + a.n);
    q.k = kw0 + min((int32_t)lane, nq - 1);  // idle lanes repeat the last query
    float4 qp = sorted[q.k];
    q.orig = ~__float_as_int(qp.w);
    // A query without finite coordinates lists nobody.  Its lane goes idle where
    // the first finite one stands, so that the search and the products are those
    // of the others (with 6 such particles among 20k the traversal took 64.6 ms
    // instead of 0.04: their boxes are the whole system).
    const uint64_t finite = __ballot(__builtin_isfinite(qp.x) && __builtin_isfinite(qp.y) && __builtin_isfinite(qp.z));
    if (~finite) {
        valid = valid && lane_bit(finite);
        if (finite == 0) {
            if ((int32_t)lane < nq) a.count[q.orig] = 0;
            return;
        }
        const int from = (int)__builtin_ctzll(finite);
        const float x = lane_value(qp.x, from), y = lane_value(qp.y, from), z = lane_value(qp.z, from);
        qp.x = lane_bit(finite) ? qp.x : x;
        qp.y = lane_bit(finite) ? qp.y : y;
        qp.z = lane_bit(finite) ? qp.z : z;
    }
    q.valid = valid;
    if (kFew) {  // the queries' four lanes each
        const int own = min((int)(lane & 15u), nq - 1);
        q.k = kw0 + own;
        q.orig = __shfl(q.orig, own);
        q.valid = (int32_t)(lane & 15u) < nq && ((finite >> own) & 1u) != 0u;
    }
    q.cnt = 0;
    q.done = 0;
    q.words = 0;
    q.carry = 0;
    int ta = 0;
    for (int t = 1; t < a.ntypes; ++t)
        if (kw0 >= meta[t].start && meta[t].count > 0) ta = t;
    ta = uniform(ta);
    const int groups = (nq + 15) >> 4;

    // cut the queries where neighbours lie farthest apart
    const float gx = qp.x - __shfl_up(qp.x, 1), gy = qp.y - __shfl_up(qp.y, 1), gz = qp.z - __shfl_up(qp.z, 1);
    const int32_t gap = lane == 0 ? -1 : __float_as_int(__builtin_fmaf(gz, gz, __builtin_fmaf(gy, gy, gx * gx)));
    const uint64_t widest = __ballot(gap == wave_max(gap) && gap > 0);
    const uint32_t half = widest ? (uint32_t)__builtin_ctzll(widest) : 64u;  // first lane of the second half
    // bounds of each half (of the whole, twice, when there is one point only)
    const int32_t key[3] = {order_key(qp.x), order_key(qp.y), order_key(qp.z)};
    float wlo[kSegs][3], whi[kSegs][3];
#pragma unroll
    for (int s = 0; s < kSegs; ++s) {
        const bool in = half == 64u || (lane >= half) == (s == 1);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            wlo[s][d] = from_key(wave_min(in ? key[d] : INT32_MAX));
            whi[s][d] = from_key(wave_max(in ? key[d] : INT32_MIN));
        }
    }
    // the wavefront's origin: the middle of its queries
    const float ox = uniform(0.5f * (fminf(wlo[0][0], wlo[1][0]) + fmaxf(whi[0][0], whi[1][0]))),
                oy = uniform(0.5f * (fminf(wlo[0][1], wlo[1][1]) + fmaxf(whi[0][1], whi[1][1]))),
                oz = uniform(0.5f * (fminf(wlo[0][2], wlo[1][2]) + fmaxf(whi[0][2], whi[1][2])));
    // Idle lanes take the origin itself: with their constant (c0 below) every
    // product of theirs is kFar + |c|^2, positive whatever the coordinates (the
    // candidates' are finite), so none of their bits is ever set and the row
    // that they share with the last query is its own.
    const float rx = valid ? qp.x - ox : 0.0f, ry = valid ? qp.y - oy : 0.0f, rz = valid ? qp.z - oz : 0.0f;
    const float q2 = __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
    const float M2 = from_key(wave_max(order_key(q2)));  // (rounded: the bands below leave room for it)
    float bq[4] = {-2.0f * rx, -2.0f * ry, -2.0f * rz, 1.0f};
    transpose4(bq[0], bq[1], bq[2], bq[3]);

    // Trees that the queries lie too far apart for (see kSphereCost), in volumes
    // in units of R^3.  Most wavefronts are done with the first, rougher test (a
    // single query's box is its sphere's).
    uint32_t scattered = 0;
    for (int tb = 0; tb < (nq > 1 ? a.ntypes : 0); ++tb) {
        const TreeMeta &m = meta[tb];
        const double r2 = a.rlist2[ta * QBVH_MAX_TYPES + tb];
        if (m.count == 0 || !(r2 >= 0.0)) continue;
        constexpr float kBall = 4.1887902f;
        const float iR = __builtin_amdgcn_rsqf((float)r2);
        // a box grown by R (Steiner's formula)
        auto grown = [&](float x, float y, float z) {
            return ((x * y * z + 2.0f * (x * y + y * z + z * x)) + 3.1415927f * (x + y + z)) + kBall;
        };
        float all[3], room = 1.0f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            all[d] = (fmaxf(whi[0][d], whi[1][d]) - fminf(wlo[0][d], wlo[1][d])) * iR;
            room *= (m.hi[d] - m.lo[d]) * iR + 2.0f;
        }
        const float boxes = grown(all[0], all[1], all[2]);
        const float cost = 1.0f + kSphereCost * (float)nq, rounds = kSphereRounds * (float)(nq + 8) * room;
        const float count = (float)m.count;
        if (uniform(count * (boxes - kBall * cost) > rounds ? 1 : 0)) {
            float each = 0.0f;
#pragma unroll
            for (int s = 0; s < kSegs; ++s)
                each += grown((whi[s][0] - wlo[s][0]) * iR, (whi[s][1] - wlo[s][1]) * iR, (whi[s][2] - wlo[s][2]) * iR);
            // the spheres' union: at most one sphere and, for each further query
            // at distance g from the one before, the share 3/4 g / R of a sphere
            const float share = fminf(0.75f * iR * __builtin_amdgcn_sqrtf(__int_as_float(max(gap, 0))), 1.0f);
            const uint32_t sum = wave_prefix_sum((uint32_t)(share * 1024.0f));
            const float spheres = kBall * (1.0f + (float)__builtin_amdgcn_readlane((int32_t)sum, 63) * 0x1p-10f);
            const bool far = count * (fminf(boxes, each) - spheres * cost) > rounds;
            scattered |= uniform(far ? 1u << tb : 0u);
        }
    }

    uint32_t table = 0;  // index tables in use
    for (int tb = 0; tb < a.ntypes; ++tb) {
        const TreeMeta &m = meta[tb];
        const double r2 = a.rlist2[ta * QBVH_MAX_TYPES + tb];
        if (m.count == 0 || !(r2 >= 0.0)) continue;
        const double R = sqrt(r2);
        // fp64 data: the tree and the queries are the data rounded to fp32,
        // which moves each point by up to 2^-24 L_max per axis, so a pair's
        // distance by up to sqrt(3) 2^-23 L_max: the node test widens the
        // search by that much, and the fp32 pair band is doubled
        const double rshift = kMode == kExact64 ? 1.7320508075688772 * 0x1p-23 * a.lmax : 0.0;
        const double eta = (kMode == kExact64 ? 2.0 : 1.0) * 1.7320508075688772 * 0x1p-22 * (2.0 * a.lmax + 2.0 * R);
        const double rin = fmax(R - eta, 0.0) * (1.0 - 0x1p-20);
        const double rout = (R + eta) * (1.0 + 0x1p-20);
        TreeTest tt;
        tt.r2 = r2;
        tt.r2in = (float)(rin * rin * (1.0 - 0x1p-20));
        tt.r2out = (float)(rout * rout * (1.0 + 0x1p-20));
        const double M = (double)(sqrtf(M2) * (1.0f + 0x1p-20f));
        const double e_o = 3.5 * 0x1p-24 * a.lmax;  // of a shifted origin
        double mid = r2;                            // v is the squared distance less this
        if constexpr (kMode == kPaper) {
            // v is the distance to the middle of the candidate's cell box:
            // listed surely within R and the cell's inscribed radius, surely
            // not beyond the tight radius and half its diagonal (with room for
            // the rounding of the cell test)
            double hmax = 0.0, hmin = INFINITY, diag = 0.0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                tt.h[d] = axis_spacing(m.lo[d], m.hi[d], a.lmax * 0x1p-24, a.qbits);
                hmax = fmax(hmax, tt.h[d]);
                hmin = fmin(hmin, tt.h[d]);
                diag += tt.h[d] * tt.h[d];
                tt.hf[d] = (float)tt.h[d];
            }
            const double rp = R * (1.0 + 0x1p-20) + 0.02 * hmax;
            tt.rp2 = (float)(rp * rp * (1.0 + 0x1p-20));
            const float rimg = (float)R * (1.0f + 0x1p-20f) + (float)(a.lmax * 0x1p-18);
            tt.rimg2 = rimg * rimg;
            q.home = cell_query(sorted[q.k], kHome, tt, m, a.L, a.Lf);
            const double far = rp * (1.0 + 0x1p-18) + 0.5 * sqrt(diag) + 0.05 * hmax;
            const double in = R + 0.5 * hmin * (1.0 - 0x1p-10);
            mid = 0.5 * (in * in + far * far);
            // (the middle is rounded by at most 6 2^-24 L_max)
            const double e = product_error(far, e_o + 6.0 * 0x1p-24 * a.lmax, M);
            tt.band = uniform(round_band(0.5 * (far * far - in * in) + e));
            tt.band_img = uniform(round_band(mid - r2 + e));
        } else {
            tt.band = uniform(pair_band(R, rin, rout, R * 0x1p-21, 0.0, M));
            tt.band_img =
                uniform(pair_band(R, rin, rout, 1.7320508075688772 * 0x1p-22 * (2.0 * a.lmax + 2.0 * R), e_o, M));
        }
        // (squares of such coordinates come near kFar or overflow)
        tt.force = !(M2 < kFar * 1e-2f) || !(a.lmax < 1e17);
        const float c0 = valid ? q2 - (float)mid : kFar;
        float cq[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) cq[g] = __shfl(c0, 16 * g + (int)(lane & 15u));

        // Node test in grid units.  A quantized bound is an exact float; a
        // search box bound and an image shift are rounded once each, the
        // radius is padded by two bins, 2^-20 of itself and 2^-21 of the
        // largest box edge in bins (far above those roundings; for the spheres,
        // whose centres paper mode rounds three times, twice that).
        const double ih = m.inv_h;
        // (grid positions in a root box without bounds are not numbers: there
        // the boxes, which such a bound opens, are searched)
        const bool by_sphere = ((scattered >> tb) & 1u) != 0u && ih > 0.0;
        const double rgp = (R + rshift) * ih * (1.0 + 0x1p-20) + 2.0 + (by_sphere ? 0x1p-20 : 0x1p-21) * (a.lmax * ih);
        const float r2g = uniform((float)(rgp * rgp * (1.0 + 0x1p-20)));
        float sl[kSegs][3], sh[kSegs][3];
#pragma unroll
        for (int s = 0; s < kSegs; ++s) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                sl[s][d] = uniform((float)(((double)wlo[s][d] - (double)m.lo[d]) * ih));
                sh[s][d] = uniform((float)(((double)whi[s][d] - (double)m.lo[d]) * ih));
            }
        }
        const float gLx = uniform((float)(a.L[0] * ih)), gLy = uniform((float)(a.L[1] * ih)),
                    gLz = uniform((float)(a.L[2] * ih));
        const int32_t end = m.end;
        // rounds that the spheres may go without a gain (see kPatience)
        int32_t patience = by_sphere ? kPatience : 0;

        // every image's root, the first image on top
        if (lane < 27u) {
            const uint32_t img = lane % 3u | ((lane / 3u) % 3u) << 2 | (lane / 9u) << 4;
            w.sref[26u - lane] = m.root;
            w.simg[26u - lane] = (uint8_t)img;
        }
        uint32_t size = 27, parts = 0, queued = 0;  // nodes to open; parts and particles queued
        wave_lds_sync();
        while (size) {
            // (1) open the next nodes.  A walking wavefront issues little and
            // waits for memory: it goes first on its SIMD, fetching candidates
            // second, those that test and write rows last (N = 8M 4.19 -> 4.13
            // ms, 1M LJ 515 -> 508 us, WCA 234 -> 230; with few queries, hardly
            // more than a wavefront per SIMD, it costs 2%).
            if constexpr (!kFew) __builtin_amdgcn_s_setprio(3);
            const uint32_t room = size < (uint32_t)(kStack - kDepthMax) ? (uint32_t)(kStack - kDepthMax) - size : 1u;
            const uint32_t p = min(min(size, (uint32_t)kOpen), room);
            // (the lanes past the opened nodes read other live entries)
            const int32_t at = max((int32_t)(size - 1u - (lane >> 1)), 0);
            const int32_t ref = w.sref[at];
            const uint32_t img = w.simg[at];
            wave_lds_sync();
            size -= p;
            const uint64_t A = p == 32u ? ~0ull : (1ull << (2u * p)) - 1ull, R0 = __ballot(ref < 0);
            const char *rec = reinterpret_cast<const char *>(records) + ((uint64_t)(uint32_t)max(ref, 0) << 5);
            const uint32_t *box = reinterpret_cast<const uint32_t *>(rec + (lane & 1u) * 12u);
            const int2 child = *reinterpret_cast<const int2 *>(rec + 24);
            const uint32_t wx = box[0], wy = box[1], wz = box[2];
            // a run on the right of an internal child comes before it: the two
            // lanes then exchange their children (and, below, their hits)
            const bool swap = child.x >= 0 && child.y < 0;
            const int32_t nref = ref < 0 ? ref : (((lane & 1u) != 0u) != swap ? child.y : child.x);
            float lx = (float)(wx & 0xFFFFu), ly = (float)(wy & 0xFFFFu), lz = (float)(wz & 0xFFFFu);
            float hx = (float)(wx >> 16), hy = (float)(wy >> 16), hz = (float)(wz >> 16);
            if (__any(img != kHome)) {
                // the search box of the shifted queries against the node is the
                // unshifted one against the node shifted back
                const float tx = (float)((int)(img & 3u) - 1) * gLx, ty = (float)((int)((img >> 2) & 3u) - 1) * gLy,
                            tz = (float)((int)((img >> 4) & 3u) - 1) * gLz;
                lx -= tx;
                hx -= tx;
                ly -= ty;
                hy -= ty;
                lz -= tz;
                hz -= tz;
            }
            float best = __builtin_inff();
            // (out of the way of the usual round: few wavefronts wait for the jump over
            // it, 12000 particles 141.8 -> 140.1 us)
            if (__builtin_expect(patience > 0, 0)) {
                // (the lanes past the queries repeat the last one)
                const float4 own = sorted[q.k];
                float ux, uy, uz;
                if constexpr (kMode == kPaper) {  // (fewer registers to spare)
                    const float ihf = (float)ih;
                    ux = (own.x - m.lo[0]) * ihf, uy = (own.y - m.lo[1]) * ihf, uz = (own.z - m.lo[2]) * ihf;
                } else {
                    ux = (float)(((double)own.x - (double)m.lo[0]) * ih);
                    uy = (float)(((double)own.y - (double)m.lo[1]) * ih);
                    uz = (float)(((double)own.z - (double)m.lo[2]) * ih);
                }
                for (int i = 0; i < nq; i += 4) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float x = lane_value(ux, i + j), y = lane_value(uy, i + j), z = lane_value(uz, i + j);
                        const float cx = __builtin_amdgcn_fmed3f(x, lx, hx) - x;
                        const float cy = __builtin_amdgcn_fmed3f(y, ly, hy) - y;
                        const float cz = __builtin_amdgcn_fmed3f(z, lz, hz) - z;
                        best = fminf(best, __builtin_fmaf(cz, cz, __builtin_fmaf(cy, cy, cx * cx)));
                    }
                }
                const uint64_t opened = A & ~R0, missed = opened & __ballot(!(best <= r2g));
                patience = 8 * __popcll(missed) > __popcll(opened) ? kPatience : patience - 1;
            } else {
#pragma unroll
                for (int s = 0; s < kSegs; ++s) {
                    const float cx = fmaxf(fmaxf(lx - sh[s][0], sl[s][0] - hx), 0.0f);
                    const float cy = fmaxf(fmaxf(ly - sh[s][1], sl[s][1] - hy), 0.0f);
                    const float cz = fmaxf(fmaxf(lz - sh[s][2], sl[s][2] - hz), 0.0f);
                    best = fminf(best, __builtin_fmaf(cz, cz, __builtin_fmaf(cy, cy, cx * cx)));
                }
            }
            const uint32_t v = (uint32_t)~nref;
            const uint32_t first = v >> kRunCountBits, count = (v & (uint32_t)kRunCountMask) + 1u;
            constexpr uint64_t kEven = 0x5555555555555555ull;
            uint64_t H = __ballot(best <= r2g);
            const uint64_t S = __ballot(swap);
            H = (H & ~S) | (((H & kEven) << 1 | (H >> 1 & kEven)) & S);
            // a run on the stack was hit already (its even lane stands for it)
            H = A & ((H & ~R0) | (R0 & kEven));
            // (a well-formed tree's references point forward and its runs end
            // inside the system: this only keeps a corrupt one from running on)
            const uint64_t N = __ballot(nref >= 0);
            H &= (N & __ballot(nref > ref) & __ballot(nref < end)) | (~N & __ballot(first + count <= nend));
            // runs before the first internal node are next in order
            const uint64_t I = H & N;
            const uint64_t E = I ? H & ((I & (~I + 1ull)) - 1ull) : H;
            const uint64_t P = H & ~E;
            const uint32_t np = (uint32_t)__popcll(P);
            if (lane_bit(P)) {
                const uint32_t to = size + np - 1u - mbcnt(P);
                w.sref[to] = nref;
                w.simg[to] = (uint8_t)img;
            }
            size += np;
            // (2) queue their parts
            if (E) {
                const bool run = lane_bit(E);
                const uint64_t two = E & __ballot(count > 8u);
                const uint32_t sum = wave_prefix_sum(run ? count : 0u);
                if (run) {
                    const uint32_t to = parts + mbcnt(E) + mbcnt(two), off = (queued + sum - count) | img << 16;
                    w.part[to] = make_uint2(first | ((count > 8u ? 7u : count - 1u) << 27), off);
                    if (count > 8u) w.part[to + 1u] = make_uint2((first + 8u) | ((count - 9u) << 27), off + 8u);
                }
                parts += (uint32_t)__popcll(E) + (uint32_t)__popcll(two);
                queued += (uint32_t)__builtin_amdgcn_readlane((int32_t)sum, 63);
            }
            wave_lds_sync();
            // (3) test full batches; what the walk's end leaves is tested too
            if (queued >= 64u || size == 0u) {
                uint32_t done = 0, rest = queued;
                while (rest >= 64u || (size == 0u && rest > 0u)) {
                    if constexpr (!kFew) {
                        if (table == (uint32_t)kTables || __any(q.words > (uint32_t)kWords - 4u)) {
                            write_rows<kVec4>(q, w, a.nbr, a.max_nbr, lane);
                            table = 0;
                        }
                    }
                    if constexpr (!kFew) __builtin_amdgcn_s_setprio(2);
                    const Batch t = take_batch<kMode>(done, parts, w, sorted, qpoint, tt, m, lane);
                    if constexpr (!kFew) __builtin_amdgcn_s_setprio(0);
                    if constexpr (kFew)
                        test_batch_few<kMode>(a, tt, t, bq[0], cq[0], ox, oy, oz, kw0, q, w, sorted, sorted64, qpoint,
                                              m, lane);
                    else
                        test_batch<kVec4, kMode>(a, tt, t, table, groups, bq, cq, ox, oy, oz, kw0, q, w, sorted,
                                                 sorted64, qpoint, m, lane);
                    ++table;
                    done += t.parts;
                    rest -= t.slots;
                }
                const uint32_t left = parts - done, gone = queued - rest;
                uint2 keep = make_uint2(0u, 0u);
                if (lane < left) keep = w.part[done + lane];
                wave_lds_sync();
                if (lane < left) w.part[lane] = make_uint2(keep.x, keep.y - gone);
                parts = left;
                queued = rest;
                wave_lds_sync();
            }
        }
    }

    if constexpr (!kFew) write_rows<kVec4>(q, w, a.nbr, a.max_nbr, lane);
    if ((int32_t)lane >= nq) return;
    a.count[q.orig] = q.cnt;
    if (q.cnt > a.max_nbr) atomicOr(a.overflow, 1);
    if (kFew) return;
    int32_t *row = a.nbr + ((int64_t)q.orig * a.max_nbr + q.done);
    for (uint32_t e = 0; e < q.carry; ++e)
        if (q.done + (int32_t)e < a.max_nbr) row[e] = w.index[kTables * 64 + lane * 4 + e];
}

// How many of the `rest` queries from position `first` on a wavefront takes at
// once: those before a wide gap.
template <class Args>
__device__ __forceinline__ int32_t part_size(Args &a, int32_t first, int32_t rest, const float4 *__restrict__ sorted,
                                             const TreeMeta *__restrict__ meta) {
    const int32_t lane = (int32_t)(threadIdx.x & 63u), k0 = a.start + first;
    const float4 p = sorted[k0 + min(lane, rest - 1)];
    const float x = p.x - __shfl_up(p.x, 1), y = p.y - __shfl_up(p.y, 1), z = p.z - __shfl_up(p.z, 1);
    const float gap2 = __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x));
    int ta = 0;
    for (int t = 1; t < a.ntypes; ++t)
        if (k0 >= meta[t].start && meta[t].count > 0) ta = t;
    ta = uniform(ta);
    double r2 = INFINITY;
    for (int t = 0; t < a.ntypes; ++t) {
        const double q = a.rlist2[ta * QBVH_MAX_TYPES + t];
        if (q >= 0.0) r2 = fmin(r2, q);
    }
    const uint64_t wide = __ballot(lane > 0 && gap2 > (float)r2 * (kWideGap * kWideGap));
    return wide != 0 && __popcll(wide) <= kWideGaps ? (int32_t)__builtin_ctzll(wide) : rest;
}

// A wavefront of queries in as many parts as its wide gaps ask for.
template <bool kVec4, Mode kMode, bool kFew, class Args>
__device__ __forceinline__ void traverse_parts(Args &a, int32_t li, const uint4 *__restrict__ records,
                                               const float4 *__restrict__ sorted, const double *__restrict__ sorted64,
                                               const uint4 *__restrict__ qpoint, const TreeMeta *__restrict__ meta,
                                               WaveLds<kFew> &w) {
    const int32_t lane = (int32_t)(threadIdx.x & 63u);
    int32_t rest = (int32_t)__popcll(__ballot(li < a.n)), first = uniform(li);
    while (rest > 0) {
        const int32_t part = part_size(a, first, rest, sorted, meta);
        traverse_wave<kVec4, kMode, kFew, Args>(a, lane < part ? first + lane : a.n, records, sorted, sorted64, qpoint,
                                                meta, w);
        rest -= part;
        first += part;
        wave_lds_sync();
    }
}

// Workgroups are dealt round-robin to the 8 XCDs; each XCD gets one
// contiguous stretch of the Z-ordered queries so its L2 holds one region.
__device__ __forceinline__ int32_t xcd_logical_block() {
    const uint32_t nb = gridDim.x, b = blockIdx.x;
    const uint32_t xcd = b & 7u, qq = nb >> 3, rr = nb & 7u;
    return (int32_t)(xcd * qq + (xcd < rr ? xcd : rr) + (b >> 3));
}

// This lane's query (a position in the system; a.n: an idle lane).
template <int kBlock, class Args>
__device__ __forceinline__ int32_t lane_query(Args &a, const TreeMeta *__restrict__ meta, int32_t wg, int32_t nwg) {
    return query_position(meta, a.n, a.ntypes, a.qpw, a.start, kBlock / 64, wg, nwg, (int32_t)(threadIdx.x >> 6),
                          (int32_t)(threadIdx.x & 63u));
}

template <bool kVec4, int kBlock, Mode kMode, bool kFew, bool kWide>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_traverse(
    TravArgs a, const uint4 *__restrict__ records, const float4 *__restrict__ sorted,
    const uint4 *__restrict__ qpoint, const TreeMeta *__restrict__ meta) {
    __shared__ WaveLds<kFew> s_wave[kBlock / 64];
    const int32_t li = lane_query<kBlock>(a, meta, xcd_logical_block(), (int32_t)gridDim.x);
    if constexpr (kWide)
        traverse_parts<kVec4, kMode, kFew, const TravArgs>(a, li, records, sorted, a.sorted64, qpoint, meta,
                                                           s_wave[threadIdx.x >> 6]);
    else
        traverse_wave<kVec4, kMode, kFew, const TravArgs>(a, li, records, sorted, a.sorted64, qpoint, meta,
                                                          s_wave[threadIdx.x >> 6]);
}

// Batched form: the workgroups of all systems form one grid; each workgroup
// belongs to one system (found from the per-system first-workgroup table) and
// reads that system's arguments from the device table, so every per-system
// value stays wave-uniform.
template <bool kVec4, int kBlock, bool kFew, bool kWide>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_traverse_batch(
    const TravArgs *__restrict__ table, const int32_t *__restrict__ tblk_first, int32_t nsys,
    const uint4 *__restrict__ records, const float4 *__restrict__ sorted, const TreeMeta *__restrict__ meta_all) {
    __shared__ WaveLds<kFew> s_wave[kBlock / 64];
    const int32_t logical = xcd_logical_block();
    const int32_t sys = find_seg(tblk_first, nsys, logical);
    // the system's arguments are read through the constant address space, as
    // kernel arguments are: the compiler may then fetch a field again where it
    // is needed instead of holding it in registers through the walk
    using ConstArgs = const TravArgs __attribute__((address_space(4)));
    ConstArgs *args = reinterpret_cast<ConstArgs *>(reinterpret_cast<uintptr_t>(table + sys));
    const TreeMeta *meta = meta_all + sys * QBVH_MAX_TYPES;
    const int32_t li = lane_query<kBlock>(*args, meta, logical - tblk_first[sys], tblk_first[sys + 1] - tblk_first[sys]);
    if constexpr (kWide)
        traverse_parts<kVec4, kExact, kFew, ConstArgs>(*args, li, records, sorted, nullptr, nullptr, meta,
                                                       s_wave[threadIdx.x >> 6]);
    else
        traverse_wave<kVec4, kExact, kFew, ConstArgs>(*args, li, records, sorted, nullptr, nullptr, meta,
                                                      s_wave[threadIdx.x >> 6]);
}

__global__ void k_clear_flag(int32_t *f) {
    if (threadIdx.x == 0) *f = 0;
}

// (few queries per wavefront: small systems, which gain nothing from parts)
template <bool kVec4, int kBlock, Mode kMode>
void launch_one(const TravArgs &a, const uint4 *qpoint, hipStream_t s) {
    const unsigned grid = (unsigned)trav_blocks(a.n, a.ntypes, kBlock, a.qpw);
    // (rows of few queries are written entry by entry, whatever their alignment)
    if (a.qpw <= kFewQueries)
        hipLaunchKernelGGL((k_traverse<false, kBlock, kMode, true, false>), dim3(grid), dim3(kBlock), 0, s, a,
                           a.records, a.sorted, qpoint, a.meta);
    else if (wide_box(a))
        hipLaunchKernelGGL((k_traverse<kVec4, kBlock, kMode, false, true>), dim3(grid), dim3(kBlock), 0, s, a,
                           a.records, a.sorted, qpoint, a.meta);
    else
        hipLaunchKernelGGL((k_traverse<kVec4, kBlock, kMode, false, false>), dim3(grid), dim3(kBlock), 0, s, a,
                           a.records, a.sorted, qpoint, a.meta);
}

template <bool kVec4, int kBlock>
void launch_one_batch(const BatchLaunch &b, hipStream_t s) {
    if (b.qpw <= kFewQueries)
        hipLaunchKernelGGL((k_traverse_batch<false, kBlock, true, false>), dim3((unsigned)b.tblocks), dim3(kBlock), 0,
                           s, b.trav, b.tblk_first, b.nsys, b.ws.records, b.ws.sorted, b.meta);
    else if (b.wide)
        hipLaunchKernelGGL((k_traverse_batch<kVec4, kBlock, false, true>), dim3((unsigned)b.tblocks), dim3(kBlock), 0,
                           s, b.trav, b.tblk_first, b.nsys, b.ws.records, b.ws.sorted, b.meta);
    else
        hipLaunchKernelGGL((k_traverse_batch<kVec4, kBlock, false, false>), dim3((unsigned)b.tblocks), dim3(kBlock), 0,
                           s, b.trav, b.tblk_first, b.nsys, b.ws.records, b.ws.sorted, b.meta);
}

template <Mode kMode, bool kVec4>
void launch_block(const TravArgs &a, int32_t block, const uint4 *qpoint, hipStream_t s) {
    switch (block) {
    case 64: launch_one<kVec4, 64, kMode>(a, qpoint, s); break;
    case 128: launch_one<kVec4, 128, kMode>(a, qpoint, s); break;
    case 192: launch_one<kVec4, 192, kMode>(a, qpoint, s); break;
    default: launch_one<kVec4, 256, kMode>(a, qpoint, s); break;
    }
}

template <Mode kMode>
void launch_mode(const TravArgs &a, int32_t block, bool vec4, const uint4 *qpoint, hipStream_t s) {
    if (vec4)
        launch_block<kMode, true>(a, block, qpoint, s);
    else
        launch_block<kMode, false>(a, block, qpoint, s);
}

template <bool kVec4>
void launch_block_batch(const BatchLaunch &b, hipStream_t s) {
    switch (b.block_size) {
    case 64: launch_one_batch<kVec4, 64>(b, s); break;
    case 128: launch_one_batch<kVec4, 128>(b, s); break;
    case 192: launch_one_batch<kVec4, 192>(b, s); break;
    default: launch_one_batch<kVec4, 256>(b, s); break;
    }
}

}  // namespace

bool wide_box(const TravArgs &a) {
    double r2 = INFINITY;
    for (int t = 0; t < a.ntypes; ++t)
        for (int u = 0; u < a.ntypes; ++u) {
            const double x = a.rlist2[t * QBVH_MAX_TYPES + u];
            if (x >= 0.0) r2 = fmin(r2, x);
        }
    // (no two particles are farther apart than the box's diagonal; with one in
    // every R^3 there is no room for such gaps)
    double d2 = 0.0, volume = 1.0;
    for (int d = 0; d < 3; ++d) {
        d2 += a.L[d] * a.L[d];
        volume *= a.L[d];
    }
    return d2 > r2 * ((double)kWideGap * kWideGap) && (double)a.n * r2 * sqrt(r2) < volume;
}

hipError_t launch_traverse(const TravArgs &a, int32_t block, bool vec4, bool paper, const uint4 *qpoint, bool cleared,
                           hipStream_t s) {
    if (!cleared) hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(64), 0, s, a.overflow);
    if (a.n > 0) {
        if (paper)  // fp32 data only
            launch_mode<kPaper>(a, block, vec4, qpoint, s);
        else if (a.sorted64)
            launch_mode<kExact64>(a, block, vec4, nullptr, s);
        else
            launch_mode<kExact>(a, block, vec4, nullptr, s);
    }
    return hipGetLastError();
}

// The overflow flags of a batch are cleared by the batch's first kernel.
hipError_t launch_traverse_batch(const BatchLaunch &b, hipStream_t s) {
    if (b.tblocks > 0) {
        if (b.vec4)
            launch_block_batch<true>(b, s);
        else
            launch_block_batch<false>(b, s);
    }
    return hipGetLastError();
}

}  // namespace qbi
