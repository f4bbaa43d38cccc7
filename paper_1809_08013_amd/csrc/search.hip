// Algorithm 1, step 2 on the GPU: the neighbour search.
//
// The particles are taken in tiles of 64 consecutive ones (cell order). A
// tile's wave or waves build the union of the 27-cell stencils of the cells its
// particles live in: the non-empty cells, each cut to the part within reach
// of the tile, sorted by first particle, so that walking them visits
// candidates in ascending index order. The union is walked in blocks of 64
// candidates.
//
// The relation of a block, 64 candidates x 64 particles, is a contraction:
//   d_ji = |x_j|^2 - 2 x_j . x_i + (|x_i|^2 - s_i^2),  s = 2h,
// in coordinates relative to the tile's centre and scaled by the largest
// reach, so sixteen FP32 matrix products of 16 x 16 x 4 give it, and the sign
// bits are shifted out of the accumulators, one vector instruction per 64
// pairs. The relation itself is FP64 (r^2 < s^2, strictly, with r^2 =
// fma(dz, dz, fma(dy, dy, dx dx))): the FP32 value only has to tell on which
// side of zero d lies, and a pair with |d| under a bound eps on its error is
// settled by the FP64 relation on its own. With u = 2^-24 and t = |x_i| + |x_j|, a
// pair at the reach (at most 1, so |x_i| and |x_j| differ by no more):
//   coordinates rounded to FP32: 2 u t;
//   |x_j|^2, three roundings: 3 u |x_j|^2;
//   the start value and the first three partial sums of the product, each below
//   max(|x_i|^2, 1) + 2 |x_i| |x_j| (the fourth is d itself);
// together u (3.25 t^2 + 2.5 t + 4.25). With varying h a second product forms d -
// s_j^2 + s_i^2, where the roundings of d (at most 1 there), of the first sum, of
// s_i^2 and of s_j^2 add 4 u. eps = u (6 t^2 + 2.4 t + 9.6) with t = 2 max|x_i| + 1 is
// above both. (Measured on 6 million pairs each within 1e-5 of the reach, tiles of 0 to
// 1,000 reaches: uniform h at most 0.35 of eps, varying h 0.29.) For a pair farther
// away the error grows as t^2 but d as the square of its distance. On a
// 1%-jittered lattice, where 30 pairs of every particle lie within 1% of the
// reach, one block in ten holds such a pair; lattice points exactly on the
// shell are such pairs. So the lists are exactly those of the FP64 relation.
//
// The bits (two 32-bit words a lane and block) stay in LDS, and each lane then
// walks its own words and writes its list, row k of all lanes together. A
// union of more candidates than LDS has bits for is taken in several chunks.
// One wave does a tile; small runs put four on each, the smallest sixteen, every
// wave taking its share of the candidates.
//
// Periodic axes: every position is taken as its image nearest to the tile's
// centre. Where the tile's extent from its centre plus the reach stays below
// half the box, the difference of two such images is the minimum image for
// every true neighbour (both lie within that distance of the centre) and
// larger than the reach for every other pair. On a shorter axis a neighbour may
// be the candidate's other image: a block with candidates so far out is tested
// with both (no particle is within reach of two images, the axis being longer
// than twice the reach). Blocks with a coordinate that FP32 cannot hold take
// the FP64 relation with the minimum image for every pair.
//
// A tile with more distinct cells than its union build holds (9 or 18) takes the
// per-lane path: each lane walks its own stencil (sorted by Morton key) and
// writes its entries directly. Both paths produce the same set
// in the same (ascending) order, so the sums over a list do not depend on the
// path or on where the tile boundaries fall.
#include <algorithm>
#include <climits>

#include "sph_internal.h"

namespace sph {
namespace {

constexpr int kWave = 64;
// Shape of the search for W waves per tile. kMaxDist: distinct cells of a
// tile that the union build takes (27 stencil entries each), kCells: cells of
// the union after the cells out of reach are dropped; kBlocks: blocks of 64
// candidates whose relation bits LDS holds at a time (a larger union is
// taken in several chunks).
//   W = 1: one wave does a tile. 16 blocks = 1,024 candidates (the mean union
//          of the 1M patch is 1,395) leave four waves to a SIMD; 22 leave three.
//          104 cells are what then fits (10,212 of 10,240 B of LDS): a cloud of 52
//          neighbours on average has a few tiles of 93 to 104, and one tile on the
//          per-lane path ends 100 us after the others (180,000 particles: 176 us
//          with 92 cells, 80 with 104; 300,000 of 25 in varying h: 182 and 162).
//   W = 4: four waves share one, for runs too small to fill the chip.
//   W = 16: sixteen, for the smallest.
template <int W>
struct SearchShape;
template <>
struct SearchShape<1> {
    static constexpr int kMaxDist = 9, kEntries = 256, kCells = 104, kBlocks = 16;
    typedef uint8_t Cell;
};
template <>
struct SearchShape<4> {
    static constexpr int kMaxDist = 18, kEntries = 512, kCells = 486, kBlocks = 28;
    typedef uint16_t Cell;
};
template <>
struct SearchShape<16> : SearchShape<4> {
    static constexpr int kEntries = 1024;
};

__device__ __forceinline__ uint32_t spread3(uint32_t v)
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t compact3(uint32_t v)
{
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030C30C3u;
    v = (v | (v >> 4)) & 0x0300F00Fu;
    v = (v | (v >> 8)) & 0x030000FFu;
    v = (v | (v >> 16)) & 0x000003FFu;
    return v;
}

// LDS operations of one wave complete in order; this only keeps the
// compiler from moving them across the point (the wave's regions are its own).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Minimum image as a select chain: identical results to
// "if (d > half) d -= len; else if (d < -half) d += len;".
__device__ __forceinline__ double min_image_sel(double d, double len, double half)
{
    d = d > half ? d - len : d;
    return d < -half ? d + len : d;
}

__device__ __forceinline__ int wrap_or_clip(int c, int nc, int periodic, bool &ok)
{
    if (periodic) {
        ok = true;
        return c < 0 ? c + nc : (c >= nc ? c - nc : c);
    }
    ok = c >= 0 && c < nc;
    return c;
}

// A double that is the same in every lane, as a wave-uniform value.
__device__ __forceinline__ double uniform_f64(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Relation test: r2 < (2h_i)^2 or r2 < (2h_j)^2, i.e. r2 < (2 max(h_i,h_j))^2, with
// the minimum image on periodic axes.
__device__ __forceinline__ bool related(const SearchRec &me, const SearchRec &o, const Grid &g)
{
    double dx = me.x - o.x, dy = me.y - o.y, dz = me.z - o.z;
    if (g.periodic[0]) dx = min_image_sel(dx, g.len[0], g.half[0]);
    if (g.periodic[1]) dy = min_image_sel(dy, g.len[1], g.half[1]);
    if (g.periodic[2]) dz = min_image_sel(dz, g.len[2], g.half[2]);
    const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
    return (r2 < me.s2) | (r2 < o.s2);
}

// Window of cell (cx, cy, cz) for the sphere of radius r around pt (no periodic
// image in play): the sub-range of the cell's particles that can hold a point
// within r. The cell's x and y ranges leave sqrt(r^2 - dx^2 - dy^2) of the radius
// along z, dx and dy being the distances to them less a millionth of a cell (a
// particle's cell index comes from the same arithmetic, whose rounding is some
// 1e-13 of a cell); without any left the cell is skipped, else only the z slices
// within that + (one slice) are kept. A cell's keys are ordered by slice, so the
// window is found by binary search.
// The first and last cell of an axis also hold the particles clamped into
// them from outside the box, so their range is taken as unbounded on the
// outer side, and their outer slice is always kept.
__device__ __forceinline__ int2 sphere_window(int2 cr, int cx, int cy, int cz, const Grid &g,
                                              const double (&pt)[3], double r,
                                              const uint32_t *__restrict__ keys)
{
    if (cr.x >= cr.y) return cr;
    const int cxy[2] = {cx, cy};
    double left = r * r;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const double f = (pt[a] - g.lo[a]) * g.inv_s[a] - (double)cxy[a];
        const double below = cxy[a] > 0 ? -f : 0.0;
        const double above = cxy[a] < g.nc[a] - 1 ? f - 1.0 : 0.0;
        const double d = fmax(fmax(below, above) - 1e-6, 0.0) / g.inv_s[a];
        left -= d * d;
    }
    if (left < 0.0) return make_int2(cr.x, cr.x);
    const double rz = sqrt(left) * (1.0 + 1e-6);
    const double ns = (double)(1 << g.zbits);
    const double fl = ((pt[2] - rz) - g.lo[2]) * g.inv_s[2] - (double)cz;
    const double fh = ((pt[2] + rz) - g.lo[2]) * g.inv_s[2] - (double)cz;
    double ql = fmax(floor(fl * ns) - 1.0, 0.0);
    double qh = fmin(floor(fh * ns) + 1.0, ns - 1.0);
    if (cz == 0) qh = fmax(qh, 0.0);
    if (cz == g.nc[2] - 1) ql = fmin(ql, ns - 1.0);
    if (ql > qh) return make_int2(cr.x, cr.x);
    if (ql == 0.0 && qh == ns - 1.0) return cr;
    const uint32_t base = keys[cr.x] & ~((1u << g.zbits) - 1u);
    const uint32_t klo = base | (uint32_t)ql, khi = base | (uint32_t)qh;
    // first key >= klo and first key > khi, side by side
    int a = cr.x, e = cr.y, p = cr.x, q = cr.y;
    while (a < e || p < q) {
        const int m = (a + e) >> 1, n = (p + q) >> 1;
        const uint32_t km = keys[min(m, cr.y - 1)], kn = keys[min(n, cr.y - 1)];
        if (a < e) {
            if (km < klo) a = m + 1; else e = m;
        }
        if (p < q) {
            if (kn <= khi) p = n + 1; else q = n;
        }
    }
    return make_int2(a, p);
}

// Window of a union cell (coordinates cc) for a tile of the given centre and
// half extents and a reach r, on images nearest to the centre: an empty range
// when the cell lies more than r + a millionth of a cell beyond the tile on
// some axis, else the z slices within r + (one slice) of the tile's z extent.
// As in sphere_window, the outer side of an open axis'
// border cells is unbounded. Only a cell of kWindowMin particles or more is
// searched for its slices: a shorter one costs less tested whole.
constexpr int kWindowMin = 48;
__device__ __forceinline__ int2 tile_window(int2 cr, const int (&cc)[3], const Grid &g,
                                            const double (&ctr)[3], const double (&ext)[3],
                                            double r, const uint32_t *__restrict__ keys)
{
    double fl = 0.0, fh = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // low face of the cell from the centre, in cells
        double d = (double)cc[a] - (ctr[a] - g.lo[a]) * g.inv_s[a];
        if (g.periodic[a]) {
            const double half = 0.5 * g.nc[a];
            if (d + 0.5 > half) d -= g.nc[a];
            else if (d + 0.5 < -half) d += g.nc[a];
        }
        const double e = (ext[a] + r) * g.inv_s[a] + 1e-6;
        const bool above = d > e && (g.periodic[a] || cc[a] > 0);
        const bool below = d + 1.0 < -e && (g.periodic[a] || cc[a] < g.nc[a] - 1);
        if (above || below) return make_int2(cr.x, cr.x);
        fl = -e - d;
        fh = e - d;
    }
    if (cr.y - cr.x < kWindowMin) return cr;
    const double ns = (double)(1 << g.zbits);
    double ql = fmax(floor(fl * ns) - 1.0, 0.0);
    double qh = fmin(floor(fh * ns) + 1.0, ns - 1.0);
    if (!g.periodic[2] && cc[2] == 0) qh = fmax(qh, 0.0);
    if (!g.periodic[2] && cc[2] == g.nc[2] - 1) ql = fmin(ql, ns - 1.0);
    if (ql > qh) return make_int2(cr.x, cr.x);
    if (ql == 0.0 && qh == ns - 1.0) return cr;
    const uint32_t base = keys[cr.x] & ~((1u << g.zbits) - 1u);
    const uint32_t klo = base | (uint32_t)ql, khi = base | (uint32_t)qh;
    // first key >= klo and first key > khi, side by side
    int a = cr.x, e = cr.y, p = cr.x, q = cr.y;
    while (a < e || p < q) {
        const int m = (a + e) >> 1, r = (p + q) >> 1;
        const uint32_t km = keys[min(m, cr.y - 1)], kr = keys[min(r, cr.y - 1)];
        if (a < e) {
            if (km < klo) a = m + 1; else e = m;
        }
        if (p < q) {
            if (kr <= khi) p = r + 1; else q = r;
        }
    }
    return make_int2(a, p);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));

// 4 x 4 transpose of registers against groups of 16 lanes: out[q] holds, in
// lane group k, what in[k] held in lane group q.
__device__ __forceinline__ void transpose4(uint32_t (&v)[4])
{
    auto s32 = [](uint32_t &x, uint32_t &y) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    };
    auto s16 = [](uint32_t &x, uint32_t &y) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    };
    s32(v[0], v[2]);
    s32(v[1], v[3]);
    s16(v[0], v[1]);
    s16(v[2], v[3]);
}
__device__ __forceinline__ void transpose4(float a, float b, float c, float d, float (&out)[4])
{
    uint32_t v[4] = {__float_as_uint(a), __float_as_uint(b), __float_as_uint(c),
                     __float_as_uint(d)};
    transpose4(v);
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = __uint_as_float(v[q]);
}

// LDS of a tile. The union build's arrays are dead when the first relation
// bits are written.
template <int W>
struct SearchLds {
    typedef SearchShape<W> S;
    static constexpr int E = S::kCells + 4;  // (whole groups of four)
    static constexpr int kChunk = S::kBlocks * kWave;
    union {
        struct {
            int ukey[S::kEntries + 4];   // first particle of each distinct non-empty cell
            int2 urange[S::kEntries];    // the part of it within reach
        };
        uint32_t mask[2 * S::kBlocks][kWave];  // relation bits, [word of 32 candidates][lane]
    };
    int u0[E];                  // union position of each cell's first candidate
    int base[E];                // first candidate minus union position
    typename S::Cell cellof[kChunk];  // cell at each position of the chunk
    int cnt[W][W > 1 ? kWave : 1];  // entries of each wave's share of the chunk
    double red[6];              // extents x, y, z of the tile (low, high)
    uint32_t dkeys[S::kMaxDist];
    int wsum[W];
};

static_assert(sizeof(SearchLds<1>) <= 160 * 1024 / 16, "four waves per SIMD");

// A position relative to the tile's centre, as its nearest image on periodic
// axes.
__device__ __forceinline__ double rel(double v, double c, const Grid &g, int a)
{
    const double d = v - c;
    return g.periodic[a] ? min_image_sel(d, g.len[a], g.half[a]) : d;
}

// What the relation of a tile's blocks needs of the tile's particles, in four
// groups of 16: the matrix operands (-2x, -2y, -2z, 1), for varying h also
// (-1, s_i^2, 0, 0), and the accumulators' start |x_i|^2 - s_i^2.
struct TileOps {
    float b[4], b3[4], c[4];
    float eps;  // |d| below this: the FP64 relation decides
};

// Relation bits of 64 candidates (one per lane: x, y, z, |x|^2, s^2) with the
// lane's particle: w[0] candidates 0..31, w[1] 32..63, the first at bit 31,
// given the lanes hold the candidates in the order of cand_of_lane. Close:
// the pairs too close to call instead. Returns the smallest |d| the lane saw.
template <bool UniformH, bool Close>
__device__ __forceinline__ float block_bits(float x, float y, float z, float n, float s,
                                            const TileOps &T, uint32_t (&w)[2])
{
    // operands of the four 16-candidate groups, one component per lane group
    float a[4], a3[4];
    transpose4(x, y, z, n, a);
    if (!UniformH) transpose4(s, 1.0f, 0.0f, 0.0f, a3);
    uint32_t bit[4];
    float m = 3e38f;
    auto products = [&](int h, floatx4 (&d)[4]) {
        const floatx4 c = {T.c[h], T.c[h], T.c[h], T.c[h]};
#pragma unroll
        for (int r = 0; r < 4; ++r)
            d[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], T.b[h], c, 0, 0, 0);
        if (!UniformH) {
            // r^2 - s_j^2 beside r^2 - s_i^2: the smaller one decides
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const floatx4 e =
                    __builtin_amdgcn_mfma_f32_16x16x4f32(a3[r], T.b3[h], d[r], 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) d[r][q] = fminf(d[r][q], e[q]);
            }
        }
    };
    auto collect = [&](int h, const floatx4 (&d)[4]) {
        uint32_t b = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float t = Close ? fabsf(d[r][q]) - T.eps : d[r][q];
                b = __builtin_amdgcn_alignbit(b, __float_as_uint(t), 31);
            }
            if (!Close) {
                m = fminf(fminf(m, fabsf(d[r][0])), fabsf(d[r][1]));
                m = fminf(fminf(m, fabsf(d[r][2])), fabsf(d[r][3]));
            }
        }
        bit[h] = b;
    };
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        floatx4 d[4];
        products(h, d);
        collect(h, d);
    }
    // Accumulator q of a lane is row 4 (lane / 16) + q of a product, column
    // lane % 16; after the transpose each lane has all four lane groups' bits
    // of its own particle.
    transpose4(bit);
    w[0] = (bit[0] << 16) | (bit[1] & 0xffffu);
    w[1] = (bit[2] << 16) | (bit[3] & 0xffffu);
    return m;
}

// Candidate (of a block's 64) that a lane holds as a matrix row, so that the
// bits of block_bits come out in candidate order: row 4 g + q of group r is
// candidate 16 g + 4 r + q.
__device__ __forceinline__ int cand_of_lane(int lane)
{
    return ((lane & 12) << 2) | ((lane & 48) >> 2) | (lane & 3);
}

// Barrier of the tile's waves.
template <int W>
__device__ __forceinline__ void tile_sync()
{
    if constexpr (W == 1) wave_sync(); else __syncthreads();
}

// One tile of 64 particles by the whole block of W waves. Multi: the
// particles belong to one run of an ensemble (slot in the high key bits), and
// the tile uses that run's grid and cell range.
// Returns false, with nothing written, for a tile with more distinct cells or
// union cells than the shape holds (the same for every thread).
template <bool Multi, int W>
__device__ __forceinline__ bool search_tile(
    int64_t tile, int64_t n, int64_t ld, const SearchRec *__restrict__ srec,
    const uint32_t *__restrict__ keys, const int32_t *__restrict__ cstart,
    const int32_t *__restrict__ cend, const Grid &g0, int max_nb, int32_t *__restrict__ count,
    int32_t *__restrict__ idx, const uint32_t *__restrict__ hflag, uint32_t *status0,
    const BatchDev &b, SearchLds<W> &L, const unsigned long long *__restrict__ s2max)
{
    typedef SearchShape<W> Shape;
    constexpr int kThreadsT = W * kWave;
    constexpr int kQ = Shape::kEntries / kThreadsT;  // stencil entries per thread, at most
    constexpr int kChunk = SearchLds<W>::kChunk;
    static_assert(Shape::kMaxDist * kStencil <= Shape::kEntries, "entries");
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / kWave);
    int64_t t0, tend;
    tile_span<Multi>(tile, n, b, t0, tend);
    const int64_t i = t0 + lane;
    const bool active = i < tend;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));

    // Every wave holds the tile's 64 particles, one per lane.
    const uint32_t key = keys[active ? i : t0];
    const SearchRec me = srec[active ? i : t0];  // (idle lanes: the first particle's)
    int slot0 = 0;
    if constexpr (Multi) slot0 = __builtin_amdgcn_readfirstlane((int)(key >> kEnsSlotShift));
    // the run's grid, read once into wave-uniform registers
    Grid gm;
    if constexpr (Multi) {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(&b.runs[slot0].grid);
        uint32_t *dst = reinterpret_cast<uint32_t *>(&gm);
#pragma unroll
        for (int k = 0; k < (int)(sizeof(Grid) / 4); ++k)
            dst[k] = __builtin_amdgcn_readfirstlane(src[k]);
    }
    const Grid &g = Multi ? gm : g0;
    const int64_t cbase = Multi ? (int64_t)b.runs[slot0].cell_base : 0;
    // cell part of the key (run and Morton code, without the z slice)
    const uint32_t ckey = key >> (Multi ? kSliceBits : g0.zbits);
    const uint32_t mkey = Multi ? (ckey & kEnsMortonMask) : ckey;
    const uint32_t prev = __shfl_up(ckey, 1, kWave);
    const bool first = active && (lane == 0 || ckey != prev);
    const uint64_t fm = __ballot(first);
    const int ndist = __popcll(fm);
    if (ndist > Shape::kMaxDist) return false;
    if (w == 0 && first) L.dkeys[__popcll(fm & lt)] = mkey;

    // Extents of the tile around its first particle (nearest images), the
    // axes dealt to the waves; the centre is taken from them.
    const double ref[3] = {uniform_f64(me.x), uniform_f64(me.y), uniform_f64(me.z)};
    const double mc[3] = {me.x, me.y, me.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (a % W != w) continue;
        double lo = rel(mc[a], ref[a], g, a), hi = lo;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o, kWave));
            hi = fmax(hi, __shfl_xor(hi, o, kWave));
        }
        if (lane == 0) {
            L.red[2 * a] = lo;
            L.red[2 * a + 1] = hi;
        }
    }
    double s2t = me.s2;
    const bool uniform_h = Multi ? b.runs[slot0].uniform_h != 0 : hflag[0] == 0;
    if (!uniform_h) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s2t = fmax(s2t, __shfl_xor(s2t, o, kWave));
    }
    tile_sync<W>();

    // Centre and half extents; the periodic axes (bits of both) on which the
    // image nearest to the centre does not do for every pair, a candidate's
    // other image being within reach too; and whether whole cells can be placed
    // by their nearest image (a cell to spare).
    double ctr[3], ext[3];
    int both = 0;
    bool cull = g.zbits > 0, plain = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double lo = uniform_f64(L.red[2 * a]), hi = uniform_f64(L.red[2 * a + 1]);
        ctr[a] = ref[a] + 0.5 * (lo + hi);
        ext[a] = 0.5 * (hi - lo) * (1.0 + 1e-9);
        if (g.periodic[a]) {
            const double far = ext[a] + g.reach * (1.0 + 1e-6);
            if (!(far + 1.001 / g.inv_s[a] < g.half[a])) cull = false;
            if (!(far < g.half[a])) {
                both |= 1 << a;
                ext[a] = g.half[a];
            }
            // no cell of the stencils across a boundary: raw differences
            const double cw = 1.0 / g.inv_s[a];
            plain = plain && ctr[a] - ext[a] > g.lo[a] + 1.001 * cw &&
                    ctr[a] + ext[a] < g.hi[a] - 1.001 * cw &&
                    ext[a] + 2.001 * cw < g.half[a];
        }
    }
    both = __builtin_amdgcn_readfirstlane(both);
    plain = __builtin_amdgcn_readfirstlane((int)plain) != 0;

    // The union: stencil entries of the distinct cells, without those that an
    // earlier distinct cell's stencil holds too (and without the second copy of
    // a cell on a periodic axis of two cells), cut to what is within reach.
    int nu = 0;
#pragma unroll 1
    for (int q = 0; q < kQ; ++q) {
        if (q * kThreadsT >= ndist * kStencil) break;
        const int e = tid + q * kThreadsT;
        const int c = e / kStencil, st = e - c * kStencil;
        int ekey = INT_MAX;
        int2 er = make_int2(0, 0);
        if (c < ndist) {
            const uint32_t k = L.dkeys[c];
            const int oz = st / 9, oy = (st - oz * 9) / 3, ox = st - oz * 9 - oy * 3;
            const int off[3] = {ox - 1, oy - 1, oz - 1};
            const int own[3] = {(int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2)};
            int cc[3];
            bool ok = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                bool oka;
                cc[a] = wrap_or_clip(own[a] + off[a], g.nc[a], g.periodic[a], oka);
                ok = ok && oka;
                if (g.periodic[a] &&
                    ((g.nc[a] == 2 && off[a] > 0) || (g.nc[a] == 1 && off[a] != 0)))
                    ok = false;
            }
            for (int p = 0; p < c; ++p) {
                const uint32_t kp = L.dkeys[p];
                const int po[3] = {(int)compact3(kp), (int)compact3(kp >> 1),
                                   (int)compact3(kp >> 2)};
                bool near = true;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int d = abs(cc[a] - po[a]);
                    near = near && (d <= 1 || (g.periodic[a] && d >= g.nc[a] - 1));
                }
                ok = ok && !near;
            }
            if (ok) {
                const int64_t cell =
                    cbase + ((int64_t)cc[2] * g.nc[1] + cc[1]) * g.nc[0] + cc[0];
                er = make_int2(cstart[cell], cend[cell]);
                if (er.x < er.y) {
                    ekey = er.x;
                    if (cull) {
                        const double s2c =
                            Multi ? g.reach * g.reach
                                  : (uniform_h ? s2t
                                               : __longlong_as_double((long long)s2max[cell]));
                        er = tile_window(er, cc, g, ctr, ext, sqrt(fmax(s2t, s2c)), keys);
                        if (er.x >= er.y) ekey = INT_MAX;
                    }
                }
            }
        }
        // append the kept entries
        const uint64_t m = __ballot(ekey != INT_MAX);
        int at = nu;
        if constexpr (W == 1) {
            nu += __popcll(m);
        } else {
            if (lane == 0) L.wsum[w] = __popcll(m);
            tile_sync<W>();
#pragma unroll
            for (int v = 0; v < W; ++v) {
                const int cv = L.wsum[v];
                if (v < w) at += cv;
                nu += cv;
            }
            tile_sync<W>();
        }
        if (ekey != INT_MAX) {
            at += __popcll(m & lt);
            L.ukey[at] = ekey;
            L.urange[at] = er;
        }
    }
    nu = __builtin_amdgcn_readfirstlane(nu);
    if (nu > Shape::kCells) return false;
    if (tid < 4) L.ukey[nu + tid] = INT_MAX;  // (read in groups of four)
    tile_sync<W>();
    // place in the order of first particles: the number of smaller keys
    for (int e = tid; e < nu; e += kThreadsT) {
        const int k = L.ukey[e];
        const int2 r = L.urange[e];
        int rank = 0;
        for (int q = 0; q < nu; q += 4) {
            const int4 o = *reinterpret_cast<const int4 *>(&L.ukey[q]);
            rank += (o.x < k) + (o.y < k) + (o.z < k) + (o.w < k);
        }
        L.base[rank] = r.x;          // (first candidate; the position is taken off below)
        L.u0[rank] = r.y - r.x;      // (length)
    }
    tile_sync<W>();
    // union positions: exclusive prefix of the lengths
    int total = 0;
    if (w == 0) {
        for (int c0 = 0; c0 < nu; c0 += kWave) {
            const int c = c0 + lane;
            const int l = c < nu ? L.u0[c] : 0;
            int sc = l;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int t = __shfl_up(sc, o, kWave);
                if (lane >= o) sc += t;
            }
            if (c < nu) {
                L.u0[c] = total + sc - l;
                L.base[c] -= total + sc - l;
            }
            total += __shfl(sc, kWave - 1, kWave);
        }
        if (W > 1 && lane == 0) L.wsum[0] = total;
    }
    tile_sync<W>();
    if (W > 1) total = L.wsum[0];
    total = __builtin_amdgcn_readfirstlane(total);
    // union position of the lane's own particle (its cell's part holds it)
    int u_self = -1;
    {
        int lo = 0, hi = nu - 1;
        while (lo < hi) {  // last cell with first candidate <= i
            const int mid = (lo + hi + 1) >> 1;
            if (L.base[mid] + L.u0[mid] <= (int)i) lo = mid; else hi = mid - 1;
        }
        if (active) u_self = (int)i - L.base[lo];
    }

    // The tile's matrix operands.
    const double scale = 1.0 / g.reach;
    // coordinates from the centre; axes of `far`: on the other side of the box
    auto scaled = [&](const SearchRec &o, int far, float (&v)[3]) {
        const double p[3] = {o.x, o.y, o.z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double d = p[a] - ctr[a];
            if (!plain) {
                d = rel(p[a], ctr[a], g, a);
                if ((far >> a) & 1) d -= __builtin_copysign(g.len[a], d);
            }
            v[a] = (float)(d * scale);
        }
    };
    // coordinates whose squares FP32 does not hold, or an s above the reach
    // the grid was built for: FP64 for every pair
    auto odd = [](float nn, float s) { return !(nn < 1.2e24f && s <= 1.0001f); };
    TileOps T;
    bool exact = false;
    {
        float v[3];
        scaled(me, 0, v);
        const double s2 = me.s2 * (scale * scale);
        const double nd = ((double)v[0] * v[0] + (double)v[1] * v[1]) + (double)v[2] * v[2];
        const float cc = (float)(nd - s2), ss = (float)s2, nn = (float)nd;
        transpose4(-2.0f * v[0], -2.0f * v[1], -2.0f * v[2], 1.0f, T.b);
        transpose4(-1.0f, ss, 0.0f, 0.0f, T.b3);
        transpose4(cc, cc, cc, cc, T.c);
        float most = nn;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) most = fmaxf(most, __shfl_xor(most, o, kWave));
        const float t1 = 2.0f * sqrtf(most) * 1.00001f + 1.0f;
        T.eps = 5.9604645e-8f * ((6.0f * t1 + 2.4f) * t1 + 9.6f);
        if (__ballot(odd(nn, ss)) != 0ull || !(T.eps < 1e30f)) exact = true;
    }
    exact = __ballot(exact) != 0ull;
    const bool full = tend - t0 == kWave;

    int carry = 0;  // the lane's entries in earlier chunks
    const int cand = cand_of_lane(lane);
    for (int c0 = 0; c0 < total; c0 += kChunk) {
        const int len = min(total - c0, kChunk);
        // ---- cell of each position of the chunk: a lane per cell; long cells
        // by the whole wave
        for (int cb = w * kWave; cb < nu; cb += W * kWave) {
            const int c = cb + lane;
            int a = 0, e = 0;
            if (c < nu) {
                a = max(L.u0[c] - c0, 0);
                e = min((c + 1 < nu ? L.u0[c + 1] : total) - c0, len);
            }
            const uint64_t big = __ballot(e - a > kWave);
            if (e - a <= kWave)
                for (int u = a; u < e; ++u) L.cellof[u] = (typename Shape::Cell)c;
            for (uint64_t m = big; m != 0ull; m &= m - 1) {
                const int q = __builtin_ctzll(m);
                const int qa = __builtin_amdgcn_readlane(a, q), qe = __builtin_amdgcn_readlane(e, q);
                for (int u = qa + lane; u < qe; u += kWave)
                    L.cellof[u] = (typename Shape::Cell)(cb + q);
            }
        }
        tile_sync<W>();
        auto candidate_at = [&](int u) -> int { return L.base[L.cellof[u]] + c0 + u; };
        // ---- relation bits of the wave's blocks [b0, b1)
        const int nblk = (len + kWave - 1) / kWave;
        const int per = W == 1 ? nblk : (nblk + W - 1) / W;
        const int b0 = min(w * per, nblk), b1 = min(b0 + per, nblk);
        int cnt = 0;
        uint32_t occ = 0u;  // words 2 b0 + k that hold a neighbour
        auto load = [&](int blk) -> SearchRec {
            return srec[candidate_at(min(blk * kWave + cand, len - 1))];
        };
        SearchRec nx = me;
        if (b0 < b1) nx = load(b0);
        for (int blk = b0; blk < b1; ++blk) {
            const SearchRec o = nx;
            if (blk + 1 < b1) nx = load(blk + 1);
            const int ub = blk * kWave;
            float v[3];
            scaled(o, 0, v);
            auto norm = [&]() {
                return __builtin_fmaf(v[2], v[2], __builtin_fmaf(v[1], v[1], v[0] * v[0]));
            };
            const float sj = uniform_h ? 0.0f : (float)(o.s2 * (scale * scale));
            uint32_t bits[2] = {0u, 0u};
            // both images of the candidates, on the axes where some of them
            // may be within reach on the other side
            int other = 0;
            if (both) {
                const double p[3] = {o.x, o.y, o.z};
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double lim = g.half[a] - g.reach * (1.0 + 1e-6);
                    if (((both >> a) & 1) &&
                        __ballot(!(fabs(rel(p[a], ctr[a], g, a)) < lim)) != 0ull)
                        other |= 1 << a;
                }
            }
            auto images = [&](auto &&each) {
                for (int far = other;; far = (far - 1) & other) {
                    if (other) scaled(o, far, v);
                    each(norm());
                    if (far == 0) break;
                }
            };
            bool close = false;
            if (!exact && __ballot(odd(norm(), sj)) == 0ull) {
                float m = 3e38f;
                images([&](float nn) {
                    uint32_t t[2];
                    m = fminf(m, uniform_h
                                     ? block_bits<true, false>(v[0], v[1], v[2], nn, sj, T, t)
                                     : block_bits<false, false>(v[0], v[1], v[2], nn, sj, T, t));
                    bits[0] |= t[0];
                    bits[1] |= t[1];
                });
                close = __ballot(m < T.eps) != 0ull;
            } else {
                const SearchRec mine = srec[active ? i : t0];
                uint32_t acc = 0u;
#pragma unroll 1
                for (int c = 0; c < kWave; ++c) {
                    const int j = __builtin_amdgcn_readfirstlane(candidate_at(min(ub + c, len - 1)));
                    acc = (acc << 1) | (related(mine, srec[j], g) ? 1u : 0u);
                    if (c == 31) bits[0] = acc;
                }
                bits[1] = acc;
            }
            // positions past the end, idle lanes
            const int nv = len - ub;
            auto cut = [&](uint32_t (&q)[2]) {
                if (nv < kWave) {
                    q[0] &= nv >= 32 ? 0xffffffffu : ~(0xffffffffu >> nv);
                    q[1] &= nv <= 32 ? 0u : ~(0xffffffffu >> (nv - 32));
                }
                if (!full) {
                    q[0] = active ? q[0] : 0u;
                    q[1] = active ? q[1] : 0u;
                }
            };
            cut(bits);
            if (close) {
                // pairs too close to call: the FP64 relation, one pair of
                // every lane at a time
                uint32_t amb[2] = {0u, 0u};
                images([&](float nn) {
                    uint32_t t[2];
                    if (uniform_h) block_bits<true, true>(v[0], v[1], v[2], nn, sj, T, t);
                    else block_bits<false, true>(v[0], v[1], v[2], nn, sj, T, t);
                    amb[0] |= t[0];
                    amb[1] |= t[1];
                });
                cut(amb);
                const SearchRec mine = srec[active ? i : t0];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    uint32_t a = amb[r];
                    while (__ballot(a != 0u) != 0ull) {
                        if (a != 0u) {
                            const int t = __builtin_clz(a);
                            const uint32_t bt = 0x80000000u >> t;
                            a &= ~bt;
                            const SearchRec oj = srec[candidate_at(ub + 32 * r + t)];
                            bits[r] = related(mine, oj, g) ? bits[r] | bt : bits[r] & ~bt;
                        }
                    }
                }
            }
            L.mask[2 * blk][lane] = bits[0];
            L.mask[2 * blk + 1][lane] = bits[1];
            cnt += __popc(bits[0]) + __popc(bits[1]);
            occ |= ((bits[0] ? 1u : 0u) | (bits[1] ? 2u : 0u)) << (2 * (blk - b0));
        }
        // the lane's own particle
        const int us = u_self - c0;
        if (us >= b0 * kWave && us < min(b1 * kWave, len)) {
            const uint32_t word = L.mask[us >> 5][lane], bt = 0x80000000u >> (us & 31);
            if (word & bt) {
                L.mask[us >> 5][lane] = word & ~bt;
                --cnt;
                if (word == bt) occ &= ~(1u << ((us >> 5) - 2 * b0));
            }
        }
        // ---- rows of the wave's entries: after those of the waves before it
        int row0 = carry, tot = cnt;
        if constexpr (W > 1) {
            L.cnt[w][lane] = cnt;
            tile_sync<W>();
            tot = 0;
#pragma unroll
            for (int v = 0; v < W; ++v) {
                const int cv = L.cnt[v][lane];
                if (v < w) row0 += cv;
                tot += cv;
            }
        } else {
            wave_sync();
        }
        const int mine = max(0, min(cnt, max_nb - row0));
        int rows = mine;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) rows = max(rows, __shfl_xor(rows, o, kWave));
        rows = __builtin_amdgcn_readfirstlane(rows);
        // Each lane walks its non-empty words with the next one already in
        // flight; the entries of 16 rows are formed, looked up and stored
        // together. One wave and one chunk: row k of every lane at once, whole
        // lines, stored non-temporally, so that the list (read back only by the
        // next calls) does not evict the records from L2. Rows that start at
        // different places are ordinary stores (partial lines written
        // non-temporally double their time).
        const bool whole = W == 1 && c0 == 0;
        uint32_t cur = 0u, nxt = 0u;
        int ucur = 0, unxt = 0;
        auto pop = [&]() {
            // (no word left: any in bounds, its entries are past the lane's)
            const int k = min(2 * b0 + __builtin_ctz(occ | 0x80000000u), 2 * Shape::kBlocks - 1);
            occ &= occ - 1u;
            unxt = 32 * k;
            nxt = L.mask[k][lane];
        };
        pop();
        constexpr int kRows = 16;
        for (int k0 = 0; k0 < rows; k0 += kRows) {
            int val[kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                if (cur == 0u) {
                    cur = nxt;
                    ucur = unxt;
                    pop();
                }
                const int t = __builtin_clz(cur | 1u);
                val[r] = min(ucur + t, len - 1);
                cur &= ~(0x80000000u >> t);
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) val[r] = candidate_at(val[r]);
            if (whole) {
                int32_t *at = idx + (int64_t)k0 * ld + t0;
#pragma unroll
                for (int r = 0; r < kRows; ++r)
                    if (k0 + r < mine)
                        __builtin_nontemporal_store(val[r], &at[(int64_t)r * ld + lane]);
            } else {
                int32_t *at = idx + (int64_t)(row0 + k0) * ld + i;
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    if (k0 + r < mine) *at = val[r];
                    at += ld;
                }
            }
        }
        carry += tot;
        if (c0 + kChunk < total) tile_sync<W>();  // the chunk's arrays are written again
    }
    if (w == 0 && active) {
        count[i] = carry;
        if (carry > max_nb) atomicOr(Multi ? &b.status[slot0] : status0, ST_CAPACITY);
    }
    return true;
}

// Per-lane path, one wave for a tile whose union is not taken: each lane visits
// its own stencil's cells in ascending Morton order (= ascending order of their
// particles): the 27 keys are sorted in registers, then each cell is walked
// once with the next record already in flight, so the lane's list is
// ascending too.
template <bool Multi>
__device__ __forceinline__ void lane_lists(
    int64_t tile, int64_t n, int64_t ld, const SearchRec *__restrict__ srec,
    const uint32_t *__restrict__ keys, const int32_t *__restrict__ cstart,
    const int32_t *__restrict__ cend, const Grid &g0, int max_nb, int32_t *__restrict__ count,
    int32_t *__restrict__ idx, uint32_t *status0, const BatchDev &b)
{
    int64_t t0, tend;
    tile_span<Multi>(tile, n, b, t0, tend);
    const int64_t i = t0 + (threadIdx.x & (kWave - 1));
    if (i >= tend) return;
    const uint32_t key = keys[i];
    const SearchRec me = srec[i];
    const int my_slot = Multi ? (int)(key >> kEnsSlotShift) : 0;
    const uint32_t mkey = Multi ? ((key >> kSliceBits) & kEnsMortonMask) : (key >> g0.zbits);
    const int myc[3] = {(int)compact3(mkey), (int)compact3(mkey >> 1),
                        (int)compact3(mkey >> 2)};
    const Grid &gl = Multi ? b.runs[my_slot].grid : g0;
    const int64_t cbl = Multi ? (int64_t)b.runs[my_slot].cell_base : 0;
    uint32_t ks[32];
#pragma unroll
    for (int s = 0; s < 32; ++s) {
        ks[s] = 0xFFFFFFFFu;
        if (s < kStencil) {
            bool okx, oky, okz;
            const int x = wrap_or_clip(myc[0] + s % 3 - 1, gl.nc[0], gl.periodic[0], okx);
            const int y = wrap_or_clip(myc[1] + (s / 3) % 3 - 1, gl.nc[1], gl.periodic[1], oky);
            const int z = wrap_or_clip(myc[2] + s / 9 - 1, gl.nc[2], gl.periodic[2], okz);
            if (okx && oky && okz)
                ks[s] = spread3((uint32_t)x) | (spread3((uint32_t)y) << 1) |
                        (spread3((uint32_t)z) << 2);
        }
    }
    // bitonic sorting network over the 32 registers (indices are constants)
#pragma unroll
    for (int k = 2; k <= 32; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int t = 0; t < 32; ++t) {
                const int p = t ^ j;
                if (p > t) {
                    const uint32_t lo = min(ks[t], ks[p]), hi = max(ks[t], ks[p]);
                    const bool up = (t & k) == 0;
                    ks[t] = up ? lo : hi;
                    ks[p] = up ? hi : lo;
                }
            }
        }
    }
    int cnt = 0;
    const int32_t ii = (int32_t)i;
    uint32_t prev_key = 0xFFFFFFFFu;
#pragma unroll 1
    for (int s = 0; s < kStencil; ++s) {
        const uint32_t kc = ks[s];
        if (kc == 0xFFFFFFFFu) break;
        if (kc == prev_key) continue;  // a short periodic axis lists a cell twice
        prev_key = kc;
        const int x = (int)compact3(kc), y = (int)compact3(kc >> 1), z = (int)compact3(kc >> 2);
        const int64_t cell = cbl + ((int64_t)z * gl.nc[1] + y) * gl.nc[0] + x;
        const int a = cstart[cell], e = cend[cell];
        if (a >= e) continue;
        SearchRec nx = srec[a];
        for (int32_t j = a; j < e; ++j) {
            const SearchRec o = nx;
            if (j + 1 < e) nx = srec[j + 1];
            if (related(me, o, gl) && j != ii) {
                if (cnt < max_nb) idx[(int64_t)cnt * ld + i] = j;
                ++cnt;
            }
        }
    }
    count[i] = cnt;
    if (cnt > max_nb) atomicOr(Multi ? &b.status[my_slot] : status0, ST_CAPACITY);
}

// What bounds it (1M patch, one wave per tile): vector issue, 11,400
// instructions a tile (3,800 for the 21.8 blocks of candidates, 3,600 for the
// 124 list rows), 60% of the chip's rate at four waves per SIMD; the matrix
// pipe is busy 17% of the time. Before, each candidate was tested in FP64 by
// every lane (8 instructions a pair row) and the bits went through HBM: the 1M
// patch took 715 us, now 480; the 1M Evrard sphere 2,700 us, now 1,990; 104k
// particles 229 us, now 103; 8,000 particles 188 us, now 36 (one wave did a
// tile however few there were, now sixteen).
template <bool Multi, int W>
__global__ void __launch_bounds__(W * kWave, 4)
find_neighbors_kernel(int64_t n, int64_t ld, const SearchRec *__restrict__ srec,
                      const uint32_t *__restrict__ keys, const int32_t *__restrict__ cstart,
                      const int32_t *__restrict__ cend, Grid g, int max_nb,
                      int32_t *__restrict__ count, int32_t *__restrict__ idx,
                      const uint32_t *__restrict__ hflag, uint32_t *status, BatchDev b,
                      StepMask mask, const unsigned long long *__restrict__ s2max)
{
    __shared__ __attribute__((aligned(16))) SearchLds<W> L;
    const int64_t nn = Multi ? b.hdr->n_out : n;
    int64_t tile;
    if constexpr (Multi) {
        // The grid covers the capacity's tiles, the step uses the first
        // ntile: their blocks are spread over the eight XCDs, the rest exit.
        tile = xcd_used_block(b.hdr->ntile);
        if (tile < 0) return;
    } else {
        tile = xcd_block();
        if (mask.bin) {
            // individual time steps: only tiles holding a particle whose step
            // closes need lists (the others keep their stale ones, unread)
            const int64_t i = tile * kWave + (threadIdx.x & (kWave - 1));
            if (__ballot(i < nn && step_closes(mask, i)) == 0ull) return;
        }
    }
    if (!search_tile<Multi, W>(tile, nn, ld, srec, keys, cstart, cend, g, max_nb, count, idx, hflag,
                               status, b, L, s2max) &&
        threadIdx.x < kWave)
        lane_lists<Multi>(tile, nn, ld, srec, keys, cstart, cend, g, max_nb, count, idx, status, b);
}

// ---------------------------------------------------------------------------
// Smoothing-length iteration (Algorithm 1, step 2, "neighbours and smoothing
// length"; Sec. 3, target neighbour count): gather counts
// N_i = #{j != i : r^2 < (2 h_i)^2}, the number of particles outside the
// accepted band, and the update of h with a cube root computed by a fixed
// rule of IEEE operations (cbrt_newton), so that any implementation of the
// same rule gets the same h.

// Cells walked on one axis for a reach of r: those the sphere meets, on a periodic
// axis of the own one and k (1 or 2) to either side, or every cell once where it has
// fewer than that (all). (A position outside a periodic axis's range: all of the own
// one and k.)
struct AxisCells {
    int first, n;
    bool all;
};
__device__ __forceinline__ AxisCells axis_cells(const Grid &g, int a, int own, double x, double r)
{
    if (!g.periodic[a]) {
        const double f = (x - g.lo[a]) * g.inv_s[a], fr = r * g.inv_s[a] + 1e-6;
        const double top = (double)(g.nc[a] - 1);
        const int lo = (int)fmin(fmax(floor(f - fr), 0.0), top);
        const int hi = (int)fmin(fmax(floor(f + fr), 0.0), top);
        return AxisCells{lo, hi - lo + 1, false};
    }
    const int k = r * g.inv_s[a] * (1.0 + 1e-12) <= 1.0 ? 1 : 2;
    if (g.nc[a] < 2 * k + 1) return AxisCells{0, g.nc[a], true};
    const double f = (x - g.lo[a]) * g.inv_s[a], fr = r * g.inv_s[a] + 1e-6;
    int lo = own - k, hi = own + k;
    if (f >= 0.0 && f <= (double)g.nc[a]) {
        lo = max(lo, (int)floor(f - fr));
        hi = min(hi, (int)floor(f + fr));
    }
    return AxisCells{lo, hi - lo + 1, false};
}

__global__ void h_begin_kernel(uint32_t *words, int32_t first)
{
    words[IT_DONE] = words[IT_REACH] = 0u;
    words[IT_STOP] = 0x7FFFFFFFu;
    words[IT_SWEEP] = (uint32_t)first;
}

__global__ void h_end_kernel(uint32_t *words)
{
    if (words[IT_REACH]) words[IT_SWEEP] = words[IT_STOP];
    else words[IT_DONE] = 1u;
}

// Cube root of a > 0 by Newton's iteration for y^3 = a in correctly rounded
// IEEE operations only, so that every implementation that performs the same
// operations gets the same number: a is brought into [1, 8) by exact
// factors of 8, y starts at 3/2 and takes seven steps y <- (2 y + a / y^2) / 3
// (the relative error 1/2 of the start squares at each step), and the
// result is scaled back by the matching power of 2. (A quotient that has underflowed
// to 0, which no factor of 8 would bring up, has the root 0.)
__device__ __forceinline__ double cbrt_newton(double a)
{
    if (!(a > 0.0)) return 0.0;
    int k = 0;
    while (a >= 8.0) {
        a *= 0.125;
        ++k;
    }
    while (a < 1.0) {
        a *= 8.0;
        --k;
    }
    double y = 1.5;
    for (int t = 0; t < 7; ++t) y = (2.0 * y + a / (y * y)) / 3.0;
    return ldexp(y, k);
}

// All sweeps of a particle in one go: kHLanes lanes per particle. The sweeps of
// the definition - count every particle's neighbours, change the h of those
// outside the band, until none is (or sweep max_iter) - only meet in the number
// of the last one, as a count depends on the particle's own h alone.
//
// The lanes gather the squares of the distances within kHMargin times the
// particle's reach into LDS, and count from there for as long as h stays within
// it and they fit; else they gather again. (For a target whose list would not fit
// they gather without the margin: 300,000 particles, target 150, 2.29 -> 1.37 ms,
// periodic 3.52 -> 1.40; 200, 2.54 -> 2.22 and 4.35 -> 3.62.) The cells were built for a largest h
// that the sweeps may outgrow: a particle with 2 h_i up to two cells walks the
// cells its sphere meets, beyond that it raises IT_REACH and stops. Each cell
// reached without a periodic image is walked only in its window for the sphere.
// Periodic: some axis of the box is periodic (then each pair takes the minimum image;
// else the separation is used as it is).
//
// redo = 0: h goes to `tmp`. redo = 1: to `h`; from tmp, unless a particle
// outgrew the reach at some sweep: then every particle stops before that sweep,
// as the sweeps in order do, and h is what the updates until then made of it.
//
// Bound by the latency of the first gather (table, window searches and records
// one after the other), so six waves per SIMD. 300,000 particles of the Evrard
// sphere, 11 sweeps: 0.7 ms, where a counting and an update kernel per sweep took
// 3.5 (and 32 kernels). Lanes per particle 8, 16, 32: 1790, 1503, 1476 us a call
// before the windows took the sphere's shape (1180 then, 1185 with 32); margins
// 1.06 and 1.3 against 1.15: 4% more each; at six waves 1.1 against 1.15: 3% less.
constexpr int kHLanes = 16;
constexpr int kHList = 192;
constexpr double kHMargin = 1.1;
template <bool Periodic>
__global__ void __launch_bounds__(256, 6)
h_iteration_kernel(int64_t n, const SearchRec *__restrict__ srec,
                   const uint32_t *__restrict__ keys, const int32_t *__restrict__ cstart,
                   const int32_t *__restrict__ cend, Grid g, double *__restrict__ h,
                   double *__restrict__ tmp, int32_t *__restrict__ count, int32_t lo_count,
                   int32_t hi_count, double n_target, int32_t first, int32_t max_iter,
                   uint32_t *words, int redo)
{
    __shared__ double list_all[256 / kHLanes][kHList + kHLanes];  // (padded for the banks)
    const int sub = threadIdx.x % kHLanes, grp = threadIdx.x / kHLanes;
    double *list = list_all[grp];
    const int64_t i = xcd_block() * (256 / kHLanes) + grp;
    const bool active = i < n;
    if (redo && !words[IT_REACH]) {
        if (active && sub == 0) h[i] = tmp[i];
        return;
    }
    const int32_t stop = redo ? (int32_t)words[IT_STOP] : 0x7FFFFFFF;
    const int64_t ii = active ? i : n - 1;
    const SearchRec me = srec[ii];
    double hh = h[ii];
    const uint32_t key = keys[ii] >> g.zbits;
    const int myc[3] = {(int)compact3(key), (int)compact3(key >> 1), (int)compact3(key >> 2)};
    const double pt[3] = {me.x, me.y, me.z};
    // the particle's lanes in a ballot
    const int gshift = threadIdx.x & 63 & ~(kHLanes - 1);
    const uint32_t lt = (1u << sub) - 1u;
    int32_t sweep = first;
    int cnt = 0, nlist = 0;
    double rc2 = -1.0;  // the list holds every r^2 below this
    // a list of the target's neighbours with the margin would not fit
    const bool margin = n_target * (kHMargin * kHMargin * kHMargin) <= kHList;
    bool run = active && sweep < stop;
    while (run) {
        const double s = 2.0 * hh, s2 = s * s;
        const double R = sqrt(s2);
        cnt = 0;
        if (s2 <= rc2) {
            for (int q = sub; q < nlist; q += kHLanes) cnt += list[q] < s2 ? 1 : 0;
        } else {
            double Rc = margin ? kHMargin * R : R;
            bool outgrown = false;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double c = g.inv_s[a] * (1.0 + 1e-12);
                // (an open axis of one cell holds every finite h, also one whose
                // square is not: no rebuild would give it a larger cell)
                const bool holds = g.nc[a] == 1 && !g.periodic[a] ? hh < INFINITY : R * c <= 2.0;
                outgrown = outgrown || !holds;
                if (!(Rc * c <= 2.0)) Rc = R;
            }
            if (outgrown) {
                if (sub == 0) {
                    atomicMin(&words[IT_STOP], (uint32_t)sweep);
                    atomicOr(&words[IT_REACH], 1u);
                }
                break;
            }
            rc2 = Rc == R ? s2 : Rc * Rc;
            const AxisCells X = axis_cells(g, 0, myc[0], me.x, Rc);
            const AxisCells Y = axis_cells(g, 1, myc[1], me.y, Rc);
            const AxisCells Z = axis_cells(g, 2, myc[2], me.z, Rc);
            nlist = 0;
            const int ncell = X.n * Y.n * Z.n;
            for (int f0 = 0; f0 < ncell; f0 += kHLanes) {
                // a cell's window per lane
                const int f = f0 + sub;
                int2 w = make_int2(0, 0);
                if (f < ncell) {
                    const int c = f / (X.n * Y.n), r = f - c * (X.n * Y.n), b = r / X.n;
                    const int raw[3] = {X.first + r - b * X.n, Y.first + b, Z.first + c};
                    bool ok[3] = {true, true, true};
                    const int x = wrap_or_clip(raw[0], g.nc[0], g.periodic[0], ok[0]);
                    const int y = wrap_or_clip(raw[1], g.nc[1], g.periodic[1], ok[1]);
                    const int z = wrap_or_clip(raw[2], g.nc[2], g.periodic[2], ok[2]);
                    if (ok[0] && ok[1] && ok[2]) {
                        const int64_t cell = ((int64_t)z * g.nc[1] + y) * g.nc[0] + x;
                        w = make_int2(cstart[cell], cend[cell]);
                        const bool direct = !X.all && !Y.all && !Z.all && x == raw[0] &&
                                            y == raw[1] && z == raw[2];
                        if (direct && g.zbits > 0)
                            w = sphere_window(w, x, y, z, g, pt, Rc, keys);
                    }
                }
                uint32_t some = (uint32_t)(__ballot(w.x < w.y) >> gshift) & ((1u << kHLanes) - 1u);
                while (some) {
                    const int t = __builtin_ctz(some);
                    some &= some - 1u;
                    const int j1 = __shfl(w.y, t, kHLanes);
                    for (int j0 = __shfl(w.x, t, kHLanes); j0 < j1; j0 += kHLanes) {
                        const int j = j0 + sub;
                        const SearchRec o = srec[j < j1 ? j : j0];
                        double dx = me.x - o.x, dy = me.y - o.y, dz = me.z - o.z;
                        if (Periodic) {
                            if (g.periodic[0]) dx = min_image_sel(dx, g.len[0], g.half[0]);
                            if (g.periodic[1]) dy = min_image_sel(dy, g.len[1], g.half[1]);
                            if (g.periodic[2]) dz = min_image_sel(dz, g.len[2], g.half[2]);
                        }
                        const double r2 =
                            __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
                        const bool other = j < j1 && j != (int)i;
                        cnt += other && r2 < s2 ? 1 : 0;
                        const bool near = other && r2 < rc2;
                        const uint32_t m =
                            (uint32_t)(__ballot(near) >> gshift) & ((1u << kHLanes) - 1u);
                        const int at = nlist + __popc(m & lt);
                        if (near && at < kHList) list[at] = r2;
                        nlist += __popc(m);
                    }
                }
            }
            if (nlist > kHList) rc2 = -1.0;  // did not fit: gather again next time
            wave_sync();
        }
#pragma unroll
        for (int o = kHLanes / 2; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, kHLanes);
        if ((cnt >= lo_count && cnt <= hi_count) || sweep == max_iter) break;
        hh = cnt == 0 ? 2.0 * hh : (hh * 0.5) * (1.0 + cbrt_newton(n_target / (double)cnt));
        ++sweep;
        run = sweep < stop;
    }
    if (active && sub == 0) {
        if (redo) {
            h[i] = hh;
        } else {
            tmp[i] = hh;
            count[i] = cnt;
            // (atomics on one word serialise in its L2 channel: only where it
            // would grow)
            if ((uint32_t)sweep >
                __hip_atomic_load(&words[IT_SWEEP], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&words[IT_SWEEP], (uint32_t)sweep);
        }
    }
}

// Largest h, as the ordered bit patterns of positive doubles.
__global__ void __launch_bounds__(256)
max_h_kernel(int64_t n, const double *__restrict__ h, unsigned long long *out)
{
    unsigned long long m = 0;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
        const unsigned long long v = (unsigned long long)__double_as_longlong(h[i]);
        m = v > m ? v : m;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long t = __shfl_xor(m, o, 64);
        m = t > m ? t : m;
    }
    // one atomic per block, and none when the word already holds as much
    // (atomics on one word serialise in its L2 channel)
    __shared__ unsigned long long wmax[4];
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) m = wmax[w] > m ? wmax[w] : m;
        if (m > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(out, m);
    }
}

__global__ void clear_words_kernel(uint32_t *a, int k)
{
    if ((int)threadIdx.x < k) a[threadIdx.x] = 0u;
}

}  // namespace

// Waves per tile of the search: four while the tiles would leave most of the
// chip's 1,024 SIMDs with less than two waves each, sixteen while they would leave
// most of the CUs without one. 4, 8 and 16 waves: 8,000 particles 40.4, 37.1, 36.4
// us, 15,600: 42.7, 41.8, 41.6, 32,800: 53, 54, 75. (A tile's union and the first
// load of its candidates come one after the other whatever the waves.)
// 1 and 4 waves: patch of 91,125 particles 117, 90 us, 132,651: 124, 118, 157,464:
// 135, 128, 195,112: 133, 146; clouds of 60 neighbours in varying h 90,000: 148,
// 105, 131,072: 147, 135, 200,000: 213, 204, 260,000: 238, 249, of 110 in uniform h
// 110,000: 97, 90, 131,072: 100, 102, 160,000: 115, 121. With fewer than 4.5
// particles per cell nearly every tile takes the per-lane path, where three of four
// waves only hold their place: 5 neighbours 55,000: 54, 54, 70,000: 62, 61, 110,000:
// 81, 83, 131,072: 81, 119; 16 neighbours 55,000: 84, 86, 70,000: 95, 108, 131,072:
// 100, 131.
constexpr int64_t kCuTiles = 256, kSharedTiles = 2048;
constexpr int64_t kThinTiles = 1024;
constexpr double kThinCell = 4.5;

hipError_t launch_find_neighbors(sph_ctx ctx, const sph_particles &p, const sph_nbrs &nb,
                                 const StepMask &mask)
{
    const int64_t tiles = (p.n + kWave - 1) / kWave;
    const int tk = ktime_begin(ctx, TK_FIND_NEIGHBORS);
    const unsigned long long *s2max =
        reinterpret_cast<const unsigned long long *>(ctx->cell_s2max);
#define SPH_SEARCH(W)                                                                      \
    find_neighbors_kernel<false, W><<<(unsigned)tiles, W * kWave, 0, ctx->stream>>>(       \
        p.n, p.n, ctx->srec, ctx->sorted_keys, ctx->cell_start, ctx->cell_end, ctx->grid,  \
        nb.max_nb, nb.count, nb.idx, ctx->hflag_dev, ctx->status_dev, BatchDev{},          \
        mask, s2max)
    // (tiles without a particle whose step closes exit at once)
    const int64_t live = mask.bin ? std::min(tiles, mask.active) : tiles;
    const Grid &g = ctx->grid;
    const bool thin = (double)p.n < kThinCell * g.nc[0] * g.nc[1] * g.nc[2];
    if (live <= kCuTiles && tiles <= 32 * kCuTiles) SPH_SEARCH(16);
    else if (tiles <= (thin ? kThinTiles : kSharedTiles)) SPH_SEARCH(4);
    else SPH_SEARCH(1);
#undef SPH_SEARCH
    ktime_end(ctx, tk);
    return hipGetLastError();
}

hipError_t launch_find_neighbors_batch(sph_ctx ctx, const BatchDev &b, int max_nb,
                                       int32_t *count, int32_t *idx)
{
    // the capacity's tiles, plus at most one partial tile per run (each run
    // is cut into its own tiles)
    const int64_t tiles = (b.cap + kWave - 1) / kWave + kEnsMaxSlots;
#define SPH_SEARCH(W)                                                                      \
    find_neighbors_kernel<true, W><<<(unsigned)tiles, W * kWave, 0, ctx->stream>>>(        \
        0, b.cap, ctx->srec, ctx->sorted_keys, ctx->cell_start, ctx->cell_end, Grid{},     \
        max_nb, count, idx, nullptr, nullptr, b, StepMask{}, nullptr)
    if (tiles <= kSharedTiles + kEnsMaxSlots) SPH_SEARCH(4);
    else SPH_SEARCH(1);
#undef SPH_SEARCH
    return hipGetLastError();
}

hipError_t launch_max_h(sph_ctx ctx, const sph_particles &p, unsigned long long *out)
{
    clear_words_kernel<<<1, 64, 0, ctx->stream>>>(reinterpret_cast<uint32_t *>(out), 2);
    const unsigned blocks = (unsigned)std::min<int64_t>((p.n + 255) / 256, 512);
    max_h_kernel<<<blocks, 256, 0, ctx->stream>>>(p.n, p.h, out);
    return hipGetLastError();
}

hipError_t launch_h_iteration(sph_ctx ctx, const sph_particles &p, int32_t *count,
                              int32_t lo_count, int32_t hi_count, double n_target,
                              int32_t first_sweep, int32_t max_iter, uint32_t *words)
{
    // The new h wait in the reorder scratch, which no kernel uses between two cell builds.
    const Grid &g = ctx->grid;
    const unsigned blocks = (unsigned)((p.n + 256 / kHLanes - 1) / (256 / kHLanes));
    h_begin_kernel<<<1, 1, 0, ctx->stream>>>(words, first_sweep);
    for (int redo = 0; redo < 2; ++redo) {
        if (g.periodic[0] || g.periodic[1] || g.periodic[2])
            h_iteration_kernel<true><<<blocks, 256, 0, ctx->stream>>>(
                p.n, ctx->srec, ctx->sorted_keys, ctx->cell_start, ctx->cell_end, g, p.h,
                ctx->perm_tmp, count, lo_count, hi_count, n_target, first_sweep, max_iter, words,
                redo);
        else
            h_iteration_kernel<false><<<blocks, 256, 0, ctx->stream>>>(
                p.n, ctx->srec, ctx->sorted_keys, ctx->cell_start, ctx->cell_end, g, p.h,
                ctx->perm_tmp, count, lo_count, hi_count, n_target, first_sweep, max_iter, words,
                redo);
    }
    h_end_kernel<<<1, 1, 0, ctx->stream>>>(words);
    return hipGetLastError();
}

}  // namespace sph
