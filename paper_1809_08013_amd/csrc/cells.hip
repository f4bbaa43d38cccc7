// Algorithm 1, step 1 on the GPU: cell assignment, Morton keys, stable LSD
// radix sort, in-place reorder of the particle arrays and the cell table.
//
// The paper's parent codes build an octree here (Sec. 5.2.5, phase A). A
// uniform grid of cells of side >= 2 h_max sorted along a Morton curve gives
// the same exact candidate set for a fixed-radius search and keeps the
// particles of a cell, and of neighbouring cells, contiguous in memory.
#include <algorithm>

#include "sph_internal.h"

namespace sph {
namespace {

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

__device__ __forceinline__ int cell_of(double v, double lo, double inv_s, int nc)
{
    double f = floor((v - lo) * inv_s);
    f = fmin(fmax(f, 0.0), (double)(nc - 1));
    return (int)f;
}

// z slice of a point in its cell (zbits bits): the fractional part of its
// cell coordinate, scaled by 2^zbits, with points outside the box clamped
// to the first or last slice.
__device__ __forceinline__ uint32_t slice_of(double v, double lo, double inv_s, int cz, int zbits)
{
    const double f = (v - lo) * inv_s;
    double q = floor((f - (double)cz) * (double)(1 << zbits));
    q = fmin(fmax(q, 0.0), (double)((1 << zbits) - 1));
    return (uint32_t)q;
}

// Place of a tile's count of a digit: digit-major where a scan turns the counts
// into offsets; tile-major where the scatter adds them up itself, so that a wave
// reads a tile's 256 counts as one row.
struct HistAt {
    int64_t digit, tile;
    __device__ int64_t operator()(int64_t d, int64_t t) const { return d * digit + t * tile; }
};

// The arrays of one build: the fields present (x, y, z first, then vx .. p_bg,
// gx .. xw and the extra ones), where h and v stand among them, and the scratch
// copies.
struct BuildArrays {
    PermFields f;
    int h, g;               // index of h, and of gx (-1: absent)
    int w;                  // index of the density records' weight (-1: no records)
    double *tmp;            // rows of `stride`
    int64_t stride;
    int32_t *tmp_id;
};

// First kernel of a build, one block per sort tile: copies every field to the
// scratch rows (the last kernel gathers them back in cell order), forms each
// particle's sort key (the Morton key of its cell, then its z slice in the
// cell) and the tile's digit counts for the first sort pass, clears the cell
// table, flags h > h_max and notes whether some h differs from h[0]. Drift: the
// particles take their kick-drift on the way, which saves a pass over the
// state.
template <bool Drift, int Threads, int Items, int Bits>
__global__ void __launch_bounds__(Threads)
build_head_kernel(int64_t n, BuildArrays A, Grid g, double h_max, BuildWith kd,
                  uint32_t *__restrict__ keys, uint32_t *__restrict__ hist, HistAt at,
                  uint32_t *__restrict__ flag_part, uint32_t *status, int64_t ncell,
                  int32_t *__restrict__ cstart, int32_t *__restrict__ cend,
                  unsigned long long *__restrict__ s2max)
{
    constexpr int kFirst = 11;  // fields in flight together: x .. p_bg
    constexpr int kBins = 1 << Bits;
    __shared__ uint32_t cnt[kBins];
    const int tid = threadIdx.x;
    if (tid < kBins) cnt[tid] = 0;
    for (int64_t c = (int64_t)blockIdx.x * Threads + tid; c < ncell;
         c += (int64_t)gridDim.x * Threads) {
        cstart[c] = 0;
        cend[c] = 0;
        s2max[c] = 0ull;
    }
    const double *hp = A.f.f[A.h];
    const double h0 = hp[0];
    double dt = 0.0;
    if (Drift) dt = kd.dt_dev[0];
    bool differs = false, above = false;
    __syncthreads();
#pragma unroll 1
    for (int it = 0; it < Items; ++it) {
        const int64_t i = (int64_t)blockIdx.x * (Threads * Items) + it * Threads + tid;
        if (i >= n) break;
        double w[kFirst];
#pragma unroll
        for (int k = 0; k < kFirst; ++k)
            if (k < A.f.nf) w[k] = A.f.f[k][i];
        const double hi = hp[i];
        const int32_t id = A.f.id[i];
        if (Drift) {
            // (the state of a step has x .. m, so v and u are 3 .. 6)
            double t[3] = {kd.ax[i], kd.ay[i], kd.az[i]};
            if (A.g >= 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) t[a] += A.f.f[A.g + a][i];
            }
            double p[3] = {w[0], w[1], w[2]}, v[3] = {w[3], w[4], w[5]};
            half_kick(0.5 * dt, t, kd.dudt[i], v, w[6]);
            drift(dt, g, v, p);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                w[a] = p[a];
                w[3 + a] = v[a];
            }
        }
#pragma unroll
        for (int k = 0; k < kFirst; ++k)
            if (k < A.f.nf) A.tmp[k * A.stride + i] = w[k];
        A.tmp_id[i] = id;
        differs |= hi != h0;
        above |= !(hi <= h_max);
        const uint32_t cx = (uint32_t)cell_of(w[0], g.lo[0], g.inv_s[0], g.nc[0]);
        const uint32_t cy = (uint32_t)cell_of(w[1], g.lo[1], g.inv_s[1], g.nc[1]);
        const uint32_t cz = (uint32_t)cell_of(w[2], g.lo[2], g.inv_s[2], g.nc[2]);
        const uint32_t zq = slice_of(w[2], g.lo[2], g.inv_s[2], (int)cz, g.zbits);
        const uint32_t key =
            ((spread3(cx) | (spread3(cy) << 1) | (spread3(cz) << 2)) << g.zbits) | zq;
        keys[i] = key;
        atomicAdd(&cnt[key & (kBins - 1)], 1u);
#pragma unroll 4
        for (int k = kFirst; k < A.f.nf; ++k) A.tmp[k * A.stride + i] = A.f.f[k][i];
    }
    const int any_differs = __syncthreads_or(differs);
    const int any_above = __syncthreads_or(above);
    if (tid == 0) {
        flag_part[blockIdx.x] = any_differs ? 1u : 0u;
        if (any_above) atomicOr(status, ST_DOMAIN);
    }
    if (tid < kBins) hist[at(tid, blockIdx.x)] = cnt[tid];
}

// Per-tile digit histogram.
template <int Threads, int Items, int Bits>
__global__ void __launch_bounds__(Threads)
radix_hist_kernel(const uint32_t *__restrict__ keys, int64_t n, const int64_t *n_dev, int shift,
                  uint32_t *__restrict__ hist, HistAt at)
{
    constexpr int kBins = 1 << Bits;
    __shared__ uint32_t cnt[kBins];
    if (n_dev) n = *n_dev;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * (Threads * Items);
    if (base >= n && at.digit == 1) return;  // (the scatter skips these tiles)
    if (tid < kBins) cnt[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < Items; ++it) {
        const int64_t i = base + it * Threads + tid;
        if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & (kBins - 1)], 1u);
    }
    __syncthreads();
    if (tid < kBins) hist[at(tid, blockIdx.x)] = cnt[tid];
}

// Block-wide exclusive scan of one value per thread (256 threads, wave64).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *total,
                                                         uint32_t *lds /*[4]*/)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
        uint32_t s = lds[w];
        if (w < wave) before += s;
        all += s;
    }
    __syncthreads();
    *total = all;
    return before + incl - v;
}

// Scan phase 1: per-chunk sums.
__global__ void __launch_bounds__(kScanThreads)
scan_reduce_kernel(const uint32_t *__restrict__ a, int64_t len,
                   uint32_t *__restrict__ part)
{
    __shared__ uint32_t lds[4];
    int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < len) s += a[base + k];
    uint32_t total;
    block_exclusive_scan(s, &total, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Scan phase 2: exclusive scan of the chunk sums in one block.
__global__ void __launch_bounds__(kScanThreads)
scan_partials_kernel(uint32_t *__restrict__ part, int64_t nparts)
{
    __shared__ uint32_t lds[4];
    uint32_t carry = 0;
    for (int64_t base = 0; base < nparts; base += kScanThreads) {
        int64_t i = base + threadIdx.x;
        uint32_t v = i < nparts ? part[i] : 0u;
        uint32_t total;
        uint32_t ex = block_exclusive_scan(v, &total, lds);
        if (i < nparts) part[i] = carry + ex;
        carry += total;
    }
}

// Scan phase 3: exclusive scan inside each chunk plus the chunk offset.
__global__ void __launch_bounds__(kScanThreads)
scan_down_kernel(uint32_t *__restrict__ a, int64_t len,
                 const uint32_t *__restrict__ part)
{
    __shared__ uint32_t lds[4];
    int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < len) ? a[base + k] : 0u;
        s += v[k];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, &total, lds) + part[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < len) a[base + k] = run;
        run += v[k];
    }
}

// Stable scatter of one radix pass. Each wave takes a contiguous run of the
// tile's keys and ranks it 64 at a time (lanes holding the same digit are
// matched with one ballot per digit bit) against its own digit counts, so the
// index order within a digit is kept and the block meets only three times. The last
// pass's digit has fewer bits: the keys have none above them, so the counts, which
// take the digit at its full width, see the same digits as the ballots.
// Self: hist holds the tiles' digit counts (tile-major), and the block adds them
// up into the offsets it needs; else they have been scanned (digit-major). vin
// null: the values are the indices. flag_part (not null): block 0 also reduces
// the build's h flags into hflag.
// A pass over 1M keys takes 18.7 us in 2 launches (33 in 5 with the scan), over
// 104,000 10.4 us (28), of which the scatter 5.9; blocks of 256 threads, with four
// waves to add up the counts, took 7.7.
template <int Threads, int Items, bool Self, int Bits>
__global__ void __launch_bounds__(Threads)
radix_scatter_kernel(const uint32_t *__restrict__ kin, const int32_t *__restrict__ vin,
                     int64_t n, const int64_t *n_dev, int shift, int bits,
                     const uint32_t *__restrict__ hist, int64_t tiles,
                     uint32_t *__restrict__ kout, int32_t *__restrict__ vout,
                     const uint32_t *__restrict__ flag_part, uint32_t *__restrict__ hflag)
{
    if (n_dev) n = *n_dev;
    const int64_t tile0 = (int64_t)blockIdx.x * (Threads * Items);
    if (tile0 >= n) return;
    constexpr int kWaves = Threads / 64, kBins = 1 << Bits, kQuads = kBins / 256;
    __shared__ __attribute__((aligned(16))) uint32_t wcnt[kWaves][kBins];  // (written as uint4)
    __shared__ uint32_t base[kBins];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (flag_part && blockIdx.x == 0) {
        bool f = false;
        for (unsigned q = tid; q < gridDim.x; q += Threads) f |= flag_part[q] != 0u;
        const int any = __syncthreads_or(f);
        if (tid == 0) hflag[0] = any ? 1u : 0u;
    }
    // the keys and the offsets are under way together
    const int64_t first = tile0 + (int64_t)wave * (64 * Items) + lane;
    uint32_t key[Items];
    int32_t val[Items];
#pragma unroll
    for (int it = 0; it < Items; ++it) {
        const int64_t i = first + it * 64;
        key[it] = i < n ? kin[i] : 0u;
        val[it] = i < n ? (vin ? vin[i] : (int32_t)i) : 0;
    }
    if constexpr (Self) {
        // every wave adds up its share of the tiles, four digits a lane
        __shared__ __attribute__((aligned(16))) uint32_t wbefore[kWaves][kBins];
        __shared__ uint32_t wsum[kBins / 64];
        const int live = (int)((n + Threads * Items - 1) / (Threads * Items));
#pragma unroll
        for (int k = 0; k < kQuads; ++k) {
            const uint4 *row = reinterpret_cast<const uint4 *>(hist) + 64 * k + lane;
            uint4 total = {0, 0, 0, 0}, before = {0, 0, 0, 0};
#pragma unroll 8
            for (int t = wave; t < live; t += kWaves) {
                const uint4 c = row[t * (kBins / 4)];
                const uint32_t m = t < (int)blockIdx.x ? ~0u : 0u;
                total.x += c.x;
                total.y += c.y;
                total.z += c.z;
                total.w += c.w;
                before.x += c.x & m;
                before.y += c.y & m;
                before.z += c.z & m;
                before.w += c.w & m;
            }
            reinterpret_cast<uint4 *>(wcnt[wave])[64 * k + lane] = total;
            reinterpret_cast<uint4 *>(wbefore[wave])[64 * k + lane] = before;
        }
        __syncthreads();
        uint32_t sum = 0, off = 0, run = 0;
        if (tid < kBins) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                sum += wcnt[w][tid];
                off += wbefore[w][tid];
                wcnt[w][tid] = 0;
            }
            run = sum;  // inclusive sum over the digits
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t v = __shfl_up(run, o, 64);
                if (lane >= o) run += v;
            }
            if (lane == 63) wsum[wave] = run;
        }
        __syncthreads();
        if (tid < kBins) {
            off += run - sum;
            for (int w = 0; w < wave; ++w) off += wsum[w];
            base[tid] = off;
        }
    } else {
        for (int d = lane; d < kBins; d += 64) wcnt[wave][d] = 0;
        if (tid < kBins) base[tid] = hist[(int64_t)tid * tiles + blockIdx.x];
    }
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint32_t at[Items];  // rank within the wave's keys of the same digit
#pragma unroll
    for (int it = 0; it < Items; ++it) {
        const bool valid = first + it * 64 < n;
        const uint32_t d = (key[it] >> shift) & (kBins - 1);
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t ones = __ballot(bit);
            same &= bit ? ones : ~ones;
        }
        const uint32_t rank = __popcll(same & lt_mask);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t before = wcnt[wave][d];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid && rank == 0) wcnt[wave][d] = before + __popcll(same);
        at[it] = before + rank;
    }
    __syncthreads();
    // first position of each (digit, wave)
    if (tid < kBins) {
        uint32_t run = base[tid];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = wcnt[w][tid];
            wcnt[w][tid] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < Items; ++it) {
        if (first + it * 64 < n) {
            const uint32_t pos = wcnt[wave][(key[it] >> shift) & (kBins - 1)] + at[it];
            kout[pos] = key[it];
            vout[pos] = val[it];
        }
    }
}

// Gather every particle array into scratch in sorted order.
__global__ void __launch_bounds__(256)
permute_gather_kernel(int64_t n, const int64_t *n_dev, int64_t stride,
                      const int32_t *__restrict__ perm, PermFields f,
                      double *__restrict__ tmp, int32_t *__restrict__ tmp_id,
                      int32_t *__restrict__ tmp_slot)
{
    if (n_dev) n = *n_dev;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
        const int64_t j = perm[i];
        for (int k = 0; k < f.nf; ++k) tmp[k * stride + i] = f.f[k][j];
        tmp_id[i] = f.id[j];
        if (f.slot) tmp_slot[i] = f.slot[j];
    }
}

// Copy the sorted arrays back into the caller's storage and write the
// search records (position and (2h)^2). Fields 0..2 are x, y, z (always
// present).
__global__ void __launch_bounds__(256)
permute_store_kernel(int64_t n, const int64_t *n_dev, int64_t stride, PermFields f,
                     const double *__restrict__ tmp, const int32_t *__restrict__ tmp_id,
                     const int32_t *__restrict__ tmp_slot, int h_field, int m_field,
                     SearchRec *__restrict__ srec, DensRec *__restrict__ drec)
{
    if (n_dev) n = *n_dev;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
        for (int k = 0; k < f.nf; ++k) f.f[k][i] = tmp[k * stride + i];
        f.id[i] = tmp_id[i];
        if (f.slot) f.slot[i] = tmp_slot[i];
        const double x = tmp[i], y = tmp[stride + i], z = tmp[2 * stride + i];
        const double s = 2.0 * tmp[h_field * stride + i];
        srec[i] = SearchRec{x, y, z, s * s};
        drec[i] = DensRec{x, y, z, tmp[m_field * stride + i]};
    }
}

// Last kernel of a build: gathers every field from the scratch rows into the
// caller's arrays in cell order, writes the search records (position and
// (2h)^2), the density records if asked for and the cell table (a particle whose
// predecessor lies in another cell ends that one and starts its own; cells without
// particles stay empty). With varying h also each cell's largest (2h)^2, as the
// ordered bit pattern of a positive double: a segmented maximum over the wave's lanes
// (a cell's particles are consecutive), then one atomic per cell and wave.
__global__ void __launch_bounds__(256)
build_tail_kernel(int64_t n, const int32_t *__restrict__ perm, const uint32_t *__restrict__ keys,
                  BuildArrays A, Grid g, SearchRec *__restrict__ srec,
                  DensRec *__restrict__ drec, int32_t *__restrict__ cstart, int32_t *__restrict__ cend,
                  const uint32_t *__restrict__ hflag, unsigned long long *__restrict__ s2max)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool active = i < n;
    const int64_t at = active ? i : n - 1;
    const int64_t j = perm[at];
    const uint32_t ck = keys[at] >> g.zbits;
    double w[kPermFields];
#pragma unroll
    for (int k = 0; k < kPermFields; ++k)
        if (k < A.f.nf) w[k] = A.tmp[k * A.stride + j];
    const int32_t id = A.tmp_id[j];
    const double s = 2.0 * A.tmp[A.h * A.stride + j];
    const double s2 = s * s;
    const double dw = A.w >= 0 ? A.tmp[A.w * A.stride + j] : 0.0;
    auto cell = [&](uint32_t c) -> int64_t {
        return ((int64_t)compact3(c >> 2) * g.nc[1] + compact3(c >> 1)) * g.nc[0] + compact3(c);
    };
    if (active) {
#pragma unroll
        for (int k = 0; k < kPermFields; ++k)
            if (k < A.f.nf) A.f.f[k][i] = w[k];
        A.f.id[i] = id;
        srec[i] = SearchRec{w[0], w[1], w[2], s2};
        if (A.w >= 0) drec[i] = DensRec{w[0], w[1], w[2], dw};
        const uint32_t pk = i > 0 ? keys[i - 1] >> g.zbits : 0u;
        if (i == 0 || pk != ck) {
            cstart[cell(ck)] = (int32_t)i;
            if (i > 0) cend[cell(pk)] = (int32_t)i;
        }
        if (i == n - 1) cend[cell(ck)] = (int32_t)n;
    }
    if (hflag[0] == 0u) return;  // uniform h: not read
    const uint32_t gk = active ? ck : 0xFFFFFFFFu;
    unsigned long long v = active ? (unsigned long long)__double_as_longlong(s2) : 0ull;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_down(v, o, 64);
        const uint32_t tk = __shfl_down(gk, o, 64);
        if (lane + o < 64 && tk == gk) v = t > v ? t : v;
    }
    const uint32_t pk = __shfl_up(gk, 1, 64);
    if (active && (lane == 0 || pk != gk)) atomicMax(&s2max[cell(ck)], v);
}

// ---------------------------------------------------------------------------
// Ensemble kernels: the same cell assignment and table per run, with the
// run's slot in the high key bits. Counts come from the step header, so one
// captured launch sequence serves every batch composition.

// Runs admitted before this step: tag their particles with the slot and
// clear the slot's status word.
__global__ void __launch_bounds__(256)
admit_kernel(BatchDev b)
{
    const BatchHdr *hd = b.hdr;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int r = 0; r < hd->nnew; ++r) {
        const int s = hd->new_slot[r];
        const int64_t off = hd->new_off[r], nr = hd->new_n[r];
        for (int64_t i = t0; i < nr; i += step) b.slot[off + i] = s;
        if (t0 == 0) b.status[s] = 0u;
    }
}

// Kick-drift of the particles of stepping runs (not at a run's t = 0 evaluation,
// not when it is being dropped) with their run's dt and box, and the keys.
__global__ void __launch_bounds__(256)
keys_batch_kernel(BatchDev b, double *__restrict__ F, const double *__restrict__ ax,
                  const double *__restrict__ ay, const double *__restrict__ az,
                  const double *__restrict__ dudt, uint32_t *__restrict__ keys)
{
    const int64_t n = b.hdr->n_in, cap = b.cap;
    const double *h = F + 7 * cap;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
        const int s = b.slot[i];
        const RunDev &r = b.runs[s];
        uint32_t key = kEnsDropKey;
        if (r.phase == RUN_INIT || r.phase == RUN_STEP) {
            const Grid &g = r.grid;
            double p[3] = {F[i], F[cap + i], F[2 * cap + i]};
            if (r.phase == RUN_STEP) {
                const double dt = b.dt[s];
                const double t[3] = {ax[i], ay[i], az[i]};
                double v[3] = {F[3 * cap + i], F[4 * cap + i], F[5 * cap + i]}, u = F[6 * cap + i];
                half_kick(0.5 * dt, t, dudt[i], v, u);
                drift(dt, g, v, p);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    F[a * cap + i] = p[a];
                    F[(3 + a) * cap + i] = v[a];
                }
                F[6 * cap + i] = u;
            }
            const uint32_t cx = (uint32_t)cell_of(p[0], g.lo[0], g.inv_s[0], g.nc[0]);
            const uint32_t cy = (uint32_t)cell_of(p[1], g.lo[1], g.inv_s[1], g.nc[1]);
            const uint32_t cz = (uint32_t)cell_of(p[2], g.lo[2], g.inv_s[2], g.nc[2]);
            const uint32_t zq = slice_of(p[2], g.lo[2], g.inv_s[2], (int)cz, g.zbits);
            key = ((uint32_t)s << kEnsSlotShift) |
                  ((spread3(cx) | (spread3(cy) << 1) | (spread3(cz) << 2)) << kSliceBits) |
                  (zq << (kSliceBits - g.zbits));
            if (!(h[i] <= r.h_max)) atomicOr(&b.status[s], ST_DOMAIN);
        }
        keys[i] = key;
    }
}

// Cell table of every live run: global cell c belongs to the live run whose
// cell range holds it; its particles are found by binary search inside the
// run's sorted range.
__global__ void __launch_bounds__(256)
cell_table_batch_kernel(BatchDev b, const uint32_t *__restrict__ keys,
                        int32_t *__restrict__ cstart, int32_t *__restrict__ cend)
{
    const BatchHdr *hd = b.hdr;
    const int64_t ncell = hd->ncell;
    const int nlive = hd->nlive;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < ncell; c += step) {
        int lo = 0, hi = nlive - 1;
        while (lo < hi) {  // last live run with cell_base <= c
            const int mid = (lo + hi + 1) >> 1;
            if (hd->live_cell_base[mid] <= c) lo = mid; else hi = mid - 1;
        }
        const int s = hd->live_slot[lo];
        const RunDev &r = b.runs[s];
        const Grid &g = r.grid;
        const int64_t lc = c - r.cell_base;
        const uint32_t cx = (uint32_t)(lc % g.nc[0]);
        const uint32_t cy = (uint32_t)((lc / g.nc[0]) % g.nc[1]);
        const uint32_t cz = (uint32_t)(lc / ((int64_t)g.nc[0] * g.nc[1]));
        const uint32_t key = ((uint32_t)s << kEnsSlotShift) |
                             ((spread3(cx) | (spread3(cy) << 1) | (spread3(cz) << 2)) << kSliceBits);
        const uint32_t last = key | ((1u << kSliceBits) - 1u);
        int64_t a = r.start, e = (int64_t)r.start + r.n;
        while (a < e) {
            const int64_t mid = (a + e) >> 1;
            if (keys[mid] < key) a = mid + 1; else e = mid;
        }
        const int64_t first = a;
        e = (int64_t)r.start + r.n;
        while (a < e) {
            const int64_t mid = (a + e) >> 1;
            if (keys[mid] <= last) a = mid + 1; else e = mid;
        }
        cstart[c] = (int32_t)first;
        cend[c] = (int32_t)a;
    }
}

inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

hipError_t exclusive_scan(sph_ctx ctx, uint32_t *a, int64_t len)
{
    const int64_t nparts = (len + kScanChunk - 1) / kScanChunk;
    scan_reduce_kernel<<<(unsigned)nparts, kScanThreads, 0, ctx->stream>>>(a, len, ctx->scan_part);
    scan_partials_kernel<<<1, kScanThreads, 0, ctx->stream>>>(ctx->scan_part, nparts);
    scan_down_kernel<<<(unsigned)nparts, kScanThreads, 0, ctx->stream>>>(a, len, ctx->scan_part);
    return hipGetLastError();
}

// Tiles of a sort of up to n keys: the smallest of 512 x 1, 1024 x 1, 1024 x 2 and
// 1024 x 4 keys (threads x keys of one) that give at most kSortSelfTiles of
// them, as small tiles keep more of the chip busy; the largest beyond. Digits of 9
// bits where they save a pass of 8 and the tiles are few: a block then reads at
// most 128 KB of counts (a pass of 8,000 keys takes two launches, 7 us).
struct SortPlan {
    int tile, bits;
    int64_t tiles;
    bool self;
    HistAt at() const { return self ? HistAt{1, 1 << bits} : HistAt{tiles, 1}; }
};

SortPlan sort_plan(int64_t n, int key_bits)
{
    SortPlan p{kSortTileMin, kRadixBits, 0, true};
    while ((p.tiles = (n + p.tile - 1) / p.tile) > kSortSelfTiles && p.tile < kSortTile)
        p.tile *= 2;
    p.self = p.tiles <= kSortSelfTiles;
    if (p.tiles <= kSortWideTiles && (key_bits + 8) / 9 < (key_bits + 7) / 8) p.bits = 9;
    return p;
}

// CALL(threads, items, bits) for a plan
#define SPH_SORT_TILE(sp, CALL)                                                            \
    do {                                                                                   \
        switch ((sp).tile) {                                                               \
        case 512:                                                                          \
            if ((sp).bits == 9) CALL(512, 1, 9);                                           \
            else CALL(512, 1, 8);                                                          \
            break;                                                                         \
        case 1024: CALL(1024, 1, 8); break;                                                \
        case 2048: CALL(1024, 2, 8); break;                                                \
        default: CALL(1024, 4, 8); break;                                                  \
        }                                                                                  \
    } while (0)

// The passes over key_bits bits, from k[*cur], v[*cur]. identity: the first
// pass's values are the indices; counted: its digit counts are in the
// histogram already; flags: it also reduces the build's h flags.
hipError_t sort_passes(sph_ctx ctx, uint32_t *const k[2], int32_t *const v[2], int64_t n,
                       const int64_t *n_dev, int key_bits, const SortPlan &sp, bool identity,
                       bool counted, bool flags, int *cur)
{
    hipStream_t s = ctx->stream;
    const unsigned nb = (unsigned)sp.tiles;
    hipError_t e;
    for (int shift = 0; shift < key_bits; shift += sp.bits) {
        const bool head = shift == 0;
        const int bits = std::min(sp.bits, key_bits - shift);
        if (!(head && counted)) {
#define SPH_HIST(T, I, B)                                                                  \
    radix_hist_kernel<T, I, B><<<nb, T, 0, s>>>(k[*cur], n, n_dev, shift, ctx->hist, sp.at())
            SPH_SORT_TILE(sp, SPH_HIST);
#undef SPH_HIST
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        const int32_t *vin = head && identity ? nullptr : v[*cur];
        const uint32_t *fp = head && flags ? ctx->flag_part : nullptr;
        if (sp.self) {
#define SPH_SCATTER(T, I, B)                                                               \
    radix_scatter_kernel<T, I, true, B><<<nb, T, 0, s>>>(                                  \
        k[*cur], vin, n, n_dev, shift, bits, ctx->hist, sp.tiles, k[*cur ^ 1],             \
        v[*cur ^ 1], fp, ctx->hflag_dev)
            SPH_SORT_TILE(sp, SPH_SCATTER);
#undef SPH_SCATTER
        } else {
            if ((e = exclusive_scan(ctx, ctx->hist, sp.tiles * kRadixBins)) != hipSuccess)
                return e;
            radix_scatter_kernel<1024, 4, false, 8><<<nb, 1024, 0, s>>>(
                k[*cur], vin, n, n_dev, shift, bits, ctx->hist, sp.tiles, k[*cur ^ 1],
                v[*cur ^ 1], fp, ctx->hflag_dev);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        *cur ^= 1;
    }
    return hipSuccess;
}

}  // namespace

hipError_t radix_sort_pairs(sph_ctx ctx, uint32_t *k[2], int32_t *v[2], int64_t n,
                            int key_bits, int *cur)
{
    return sort_passes(ctx, k, v, n, nullptr, key_bits, sort_plan(n, key_bits), false, false, false, cur);
}

// A build is: the head kernel (scratch copies, keys, first digit counts), the
// sort's passes (count and scatter, the first without its count), and the tail
// kernel (gather, search records, cell table). Bound by launches up to 100,000
// particles (no kernel is under 2 to 4.5 us here) and by the two passes over the
// state, 92 B each way a particle, beyond. With the drift (and the density
// records) a build of 8,000 particles takes 26 us in 5 launches, of 104,000 45 us
// and of 1M 154 us in 7; in the 21 launches of one kernel per job 101, 127 and 234.
// A sort of up to 12,288 keys in one block's LDS took 20 us (bound by its one CU).
hipError_t launch_build_cells(sph_ctx ctx, const sph_particles &p, const Grid &g,
                              double h_max, double *const *extra, int n_extra,
                              const BuildWith &with)
{
    const int64_t n = p.n;
    hipStream_t s = ctx->stream;
    const int64_t ncell = (int64_t)g.nc[0] * g.nc[1] * g.nc[2];
    BuildArrays A{};
    double *fields[kPermFields] = {p.x, p.y, p.z, p.vx, p.vy, p.vz, p.u, p.h, p.m,
                                   p.rho_ref, p.p_bg, p.gx, p.gy, p.gz, p.xw};
    for (int k = 0; k < n_extra && 15 + k < kPermFields; ++k) fields[15 + k] = extra[k];
    A.h = A.g = A.w = -1;
    for (int k = 0; k < kPermFields; ++k) {
        if (!fields[k]) continue;
        if (k == 7) A.h = A.f.nf;
        if (k == 11) A.g = A.f.nf;
        if ((k == 8 && with.dens == BuildWith::MASS) || (k == 14 && with.dens == BuildWith::WEIGHT))
            A.w = A.f.nf;
        A.f.f[A.f.nf++] = fields[k];
    }
    A.f.id = p.id;
    A.tmp = ctx->perm_tmp;
    A.stride = ctx->n_max;
    A.tmp_id = ctx->perm_tmp_id;
    unsigned long long *s2max = reinterpret_cast<unsigned long long *>(ctx->cell_s2max);
    const int key_bits = std::max(1, 3 * g.bits + g.zbits);
    const SortPlan sp = sort_plan(n, key_bits);
#define SPH_HEAD_D(D, T, I, B)                                                             \
    build_head_kernel<D, T, I, B><<<(unsigned)sp.tiles, T, 0, s>>>(                        \
        n, A, g, h_max, with, ctx->keys[0], ctx->hist, sp.at(), ctx->flag_part,            \
        ctx->status_dev, ncell, ctx->cell_start, ctx->cell_end, s2max)
#define SPH_HEAD(T, I, B)                                                                  \
    do {                                                                                   \
        if (with.dt_dev) SPH_HEAD_D(true, T, I, B);                                        \
        else SPH_HEAD_D(false, T, I, B);                                                   \
    } while (0)
    SPH_SORT_TILE(sp, SPH_HEAD);
#undef SPH_HEAD_D
#undef SPH_HEAD
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int cur = 0;
    if ((e = sort_passes(ctx, ctx->keys, ctx->vals, n, nullptr, key_bits, sp, true, true, true,
                         &cur)) != hipSuccess)
        return e;
    ctx->sorted_keys = ctx->keys[cur];
    build_tail_kernel<<<blocks_for(n, 256), 256, 0, s>>>(n, ctx->vals[cur], ctx->sorted_keys, A, g,
                                                         ctx->srec, ctx->drec, ctx->cell_start,
                                                         ctx->cell_end, ctx->hflag_dev, s2max);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256)
gather_i32_kernel(int64_t n, const int32_t *__restrict__ perm, const int32_t *__restrict__ src,
                  int32_t *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[perm[i]];
}

__global__ void __launch_bounds__(256)
copy_i32_kernel(int64_t n, const int32_t *__restrict__ src, int32_t *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_permute_like_build(sph_ctx ctx, int32_t *a, int64_t n)
{
    // the sort's values are the particles' indices before the build, in
    // sorted order, next to the sorted keys
    const int32_t *perm = ctx->sorted_keys == ctx->keys[0] ? ctx->vals[0] : ctx->vals[1];
    gather_i32_kernel<<<blocks_for(n, 256), 256, 0, ctx->stream>>>(n, perm, a, ctx->perm_tmp_id);
    copy_i32_kernel<<<blocks_for(n, 256), 256, 0, ctx->stream>>>(n, ctx->perm_tmp_id, a);
    return hipGetLastError();
}

hipError_t launch_admit_batch(sph_ctx ctx, const BatchDev &b)
{
    admit_kernel<<<256, 256, 0, ctx->stream>>>(b);
    return hipGetLastError();
}

hipError_t launch_build_cells_batch(sph_ctx ctx, const BatchDev &b, double *F, int32_t *id,
                                    int32_t *slot_tmp, const double *ax, const double *ay,
                                    const double *az, const double *dudt)
{
    hipStream_t s = ctx->stream;
    const int64_t cap = b.cap;
    const unsigned grid = std::min<unsigned>(blocks_for(cap, 256), 4096u);
    const int64_t *n_in = &b.hdr->n_in;
    keys_batch_kernel<<<grid, 256, 0, s>>>(b, F, ax, ay, az, dudt, ctx->keys[0]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int cur = 0;
    if ((e = sort_passes(ctx, ctx->keys, ctx->vals, cap, n_in, kEnsKeyBits, sort_plan(cap, kEnsKeyBits), true,
                         false, false, &cur)) != hipSuccess)
        return e;
    ctx->sorted_keys = ctx->keys[cur];
    PermFields f{};
    for (int k = 0; k < kEnsFields; ++k) f.f[f.nf++] = F + k * cap;
    f.id = id;
    f.slot = b.slot;
    permute_gather_kernel<<<grid, 256, 0, s>>>(cap, n_in, ctx->n_max, ctx->vals[cur], f,
                                               ctx->perm_tmp, ctx->perm_tmp_id, slot_tmp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    permute_store_kernel<<<grid, 256, 0, s>>>(cap, n_in, ctx->n_max, f, ctx->perm_tmp,
                                              ctx->perm_tmp_id, slot_tmp, 7, 8, ctx->srec, ctx->drec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const unsigned cgrid = std::min<unsigned>(blocks_for(b.cell_cap, 256), 4096u);
    cell_table_batch_kernel<<<cgrid, 256, 0, s>>>(b, ctx->sorted_keys, ctx->cell_start,
                                                  ctx->cell_end);
    return hipGetLastError();
}

}  // namespace sph
