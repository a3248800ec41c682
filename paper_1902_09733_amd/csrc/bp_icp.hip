// Point-to-point ICP fine registration of two clouds (Sec. 2.3: the clouds
// computed with Eq. 3 are registered by ICP starting from the estimated
// poses).
//
// Both clouds are counting-sorted by the cell (edge dmax / 0.99) they fall
// in, into float4 records {x, y, z, index}, so every target within dmax of a
// query lies in the 27 cells around the query's cell.  Buckets are cell
// coordinates relative to the target's bounding box, wrapped to the bits a
// table of T buckets allows, with z fastest, then x, then y: the three
// z-neighbours of a column are adjacent buckets (for terrain, a column holds
// all its points) and queries taken in bucket order sweep the surface in
// raster order, so neighbouring wavefronts share cells in cache.  Cells that
// wrap onto the same bucket only add candidates.  Per iteration:
//   1. correspondences (queries in sorted order): p' = R p + T and its
//      nearest target within dmax in FP32, every operation rounded on its own
//      in a fixed order (ties to the lowest target index).  The target paired
//      in the previous iteration is looked at first: whatever it is, it only
//      shrinks the radius to search.  A neighbour cell is skipped when a lower
//      bound of its distance, reduced by a margin that covers every rounding
//      involved, already exceeds the best squared distance found (or dmax^2),
//      so the pairing equals the exhaustive one;
//   2. in the same kernel, FP64 sums over the accepted pairs (count, sums of p'
//      and q, sum of p' q^T, sum of squared distances), per block and then over
//      the blocks in fixed orders; the queries' order (by bucket, then by
//      source index; sources that can pair with nothing last) does not depend
//      on the atomics of the sort where it matters to the sums;
//   3. one thread: centroids and cross-covariance H, the optimal rotation by
//      Horn's quaternion method (largest eigenvector of the symmetric 4 x 4
//      matrix built from H, cyclic Jacobi in FP64), translation, composed
//      onto the pose (FP64), rounded to FP32 for the next correspondences.
// An iteration with fewer than 3 pairs leaves the pose unchanged.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "bp_internal.h"

namespace bpk {

constexpr int kIcpBlock = 256;
constexpr int kIcpSums = 17;     // n, sum p'(3), sum q(3), sum p' q^T (9), sum d2

// Bucket of a cell: ((z - oz) & mz) | ((x - ox) & mx) << sx | ((y - oy) & my) << sy.
struct IcpHash {
    int ox, oy, oz;
    uint32_t mx, my, mz, sx, sy;
};

struct IcpGrid {
    const uint32_t *start;       // [T + 1] first record of each bucket
    const float4 *rec;           // [m] targets {x, y, z, index bits} sorted by bucket
    const IcpHash *hash;
    float inv_cell;              // 0.99 / dmax
    float cell;                  // 1 / inv_cell
};

__device__ __forceinline__ uint32_t cell_bucket(const IcpHash &h, int ix, int iy, int iz)
{
    return (((uint32_t)iz - (uint32_t)h.oz) & h.mz) | ((((uint32_t)ix - (uint32_t)h.ox) & h.mx) << h.sx) |
           ((((uint32_t)iy - (uint32_t)h.oy) & h.my) << h.sy);
}

// Integer cell of a floored coordinate, clamped to +-2^30 so that huge or
// non-finite coordinates (NaN clamps to -2^30) still convert to a defined
// integer; such points never pair anyway (their distances are not <= dmax^2).
__device__ __forceinline__ int cell_index(float fl)
{
    return (int)__builtin_fminf(__builtin_fmaxf(fl, -0x1p30f), 0x1p30f);
}

__device__ __forceinline__ int cell_of(float v, float inv_cell) { return cell_index(__builtin_floorf(v * inv_cell)); }

__device__ __forceinline__ uint32_t bucket_of(const IcpHash &h, float x, float y, float z, float inv_cell)
{
    return cell_bucket(h, cell_of(x, inv_cell), cell_of(y, inv_cell), cell_of(z, inv_cell));
}

// p' = R p + T in FP32, each product and sum rounded on its own, in row order.
__device__ __forceinline__ void icp_move(const float *__restrict__ P, float x, float y, float z, float q[3])
{
#pragma clang fp contract(off)
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        float a = P[r * 3 + 0] * x;
        a = a + P[r * 3 + 1] * y;
        a = a + P[r * 3 + 2] * z;
        q[r] = a + P[9 + r];
    }
}

__device__ __forceinline__ float icp_dist2(const float q[3], float tx, float ty, float tz)
{
#pragma clang fp contract(off)
    const float ex = q[0] - tx, ey = q[1] - ty, ez = q[2] - tz;
    float d = ex * ex;
    d = d + ey * ey;
    return d + ez * ez;
}

// The counting sorts of the two clouds, source and target, which share every
// launch (blockIdx.y): a launch costs about 4.5 us whatever it does.  Bound by
// the counting's atomics, whose results are each point's place in its bucket, so
// that the records need none.  Two clouds of 256 880 points: 16 launches with
// atomics in both passes 109 us, these 8 64 us.

// Source points of a bucket up to which all are compared with all to order
// them; a block of its own orders a larger bucket.  256 000 points, k_icp_order:
// in buckets of 250 / 500 points 25 / 45 us, of 530 / 1000 / 4000 22 / 21 / 90.
constexpr uint32_t kCrowd = 512;

struct IcpSort {
    const float *pts;
    int n;
    uint32_t *count, *start;     // [T + 1]
    uint32_t *tile;              // [T / kCrowd], T / 1024 used
    uint32_t *rank;              // [n] each point's place in its bucket
    float4 *rec;
};
struct IcpSorts {
    IcpSort c[2];
    // Sources that can pair with nothing whatever the pose: a coordinate that is
    // NaN, or infinite where dmax^2 is finite (every coordinate of the moved
    // point is then NaN or infinite).  A triangulated cloud has one per hole.
    // They take the records after all others', in any order, since they add
    // nothing to any sum.
    bool inf_pairs;              // dmax^2 overflows: infinite distances are accepted
    uint32_t *gone;              // how many there are
    // Source buckets of more than kCrowd points, in any order.
    uint32_t *crowded, *ncrowded;
};

__device__ __forceinline__ bool never_pairs(const IcpSorts &so, const float *q)
{
    bool nan = false, inf = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        nan |= __builtin_isnan(q[a]);
        inf |= __builtin_isinf(q[a]);
    }
    return nan || (inf && !so.inf_pairs);
}

// Bounding box of the target's cells, per block: part[block][0..2] min,
// part[block][3..5] max (INT_MAX / INT_MIN for a block without points).  The
// blocks from nparts on clear both clouds' T counts.
constexpr int kBoxBlocks = 256;

__global__ void __launch_bounds__(256) k_icp_bbox(const IcpSorts so, int nparts, uint32_t T, float inv_cell,
                                                 int *__restrict__ part)
{
    __shared__ int s_box[4][6];
    if ((int)blockIdx.x >= nparts) {
        const size_t i = ((size_t)(blockIdx.x - (unsigned)nparts) * 256 + threadIdx.x) * 4;   // T is a multiple of 4
        if (i < T) *(uint4 *)(so.c[0].count + i) = *(uint4 *)(so.c[1].count + i) = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    const float *pts = so.c[1].pts;
    const int m = so.c[1].n;
    int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
    for (int j = blockIdx.x * 256 + threadIdx.x; j < m; j += nparts * 256) {
        const float *q = pts + (int64_t)j * 3;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int v = cell_of(q[a], inv_cell);
            lo[a] = min(lo[a], v);
            hi[a] = max(hi[a], v);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = max(hi[a], __shfl_xor(hi[a], o, 64));
        }
    const int w = threadIdx.x / 64;
    if (threadIdx.x % 64 == 0)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            s_box[w][a] = lo[a];
            s_box[w][3 + a] = hi[a];
        }
    __syncthreads();
    if (threadIdx.x < 6) {
        int v = s_box[0][threadIdx.x];
        for (int k = 1; k < 4; ++k) v = threadIdx.x < 3 ? min(v, s_box[k][threadIdx.x]) : max(v, s_box[k][threadIdx.x]);
        part[blockIdx.x * 6 + threadIdx.x] = v;
    }
}

__host__ __device__ static inline uint32_t ceil_log2(uint64_t v)
{
    uint32_t b = 0;
    while (((uint64_t)1 << b) < v) ++b;
    return b;
}

// Bucket mapping from the bounding box: one cell of margin on each side, as
// many bits per axis as the extent needs while they fit in log2(T), the
// widest axes cut first when they do not.
// The lanes also set the pose and its FP32 copy, and clear the sorts' counters.
__global__ void __launch_bounds__(64) k_icp_hash(const IcpSorts so, const int *__restrict__ part, int nparts,
                                                uint32_t log2T, IcpHash *__restrict__ h,
                                                const double *__restrict__ pose_in, double *__restrict__ pose,
                                                float *__restrict__ pose_f)
{
    if (threadIdx.x == 0) *so.gone = *so.ncrowded = 0u;
    if (threadIdx.x < 12) {
        pose[threadIdx.x] = pose_in[threadIdx.x];
        pose_f[threadIdx.x] = (float)pose_in[threadIdx.x];
    }
    int box[6];
    for (int a = 0; a < 6; ++a) {
        int v = a < 3 ? INT_MAX : INT_MIN;
        for (int b = threadIdx.x; b < nparts; b += 64) v = a < 3 ? min(v, part[b * 6 + a]) : max(v, part[b * 6 + a]);
        for (int o = 32; o >= 1; o >>= 1) v = a < 3 ? min(v, __shfl_xor(v, o, 64)) : max(v, __shfl_xor(v, o, 64));
        box[a] = v;
    }
    if (threadIdx.x != 0) return;
    int64_t org[3] = {0, 0, 0};
    uint32_t bits[3] = {log2T / 2, log2T - log2T / 2, 0};          // x, y, z for an empty cloud
    if (box[0] <= box[3]) {
        for (int a = 0; a < 3; ++a) {
            org[a] = (int64_t)box[a] - 1;
            bits[a] = ceil_log2((uint64_t)((int64_t)box[3 + a] - (int64_t)box[a] + 3));
        }
        while (bits[0] + bits[1] + bits[2] > log2T) {
            int w = 2;
            if (bits[0] > bits[w]) w = 0;
            if (bits[1] > bits[w]) w = 1;
            --bits[w];
        }
    }
    IcpHash r;
    r.ox = (int)(uint32_t)org[0];
    r.oy = (int)(uint32_t)org[1];
    r.oz = (int)(uint32_t)org[2];
    r.mx = (1u << bits[0]) - 1u;
    r.my = (1u << bits[1]) - 1u;
    r.mz = (1u << bits[2]) - 1u;
    r.sx = bits[2];
    r.sy = bits[2] + bits[0];
    *h = r;
}

__global__ void __launch_bounds__(256) k_icp_hist(const IcpSorts so, float inv_cell, const IcpHash *__restrict__ hp)
{
    const IcpSort &c = so.c[blockIdx.y];
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= c.n) return;
    const IcpHash h = *hp;
    const float *q = c.pts + (int64_t)j * 3;
    if (blockIdx.y == 0 && never_pairs(so, q)) {
        // One atomic per wavefront: the counter is the same for all.
        const uint64_t m = __ballot(true);
        const int lane = (int)threadIdx.x & 63, first = __builtin_ctzll(m);
        uint32_t at = 0;
        if (lane == first) at = atomicAdd(so.gone, (uint32_t)__builtin_popcountll(m));
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, first);
        c.rank[j] = at + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
        return;
    }
    c.rank[j] = atomicAdd(&c.count[bucket_of(h, q[0], q[1], q[2], inv_cell)], 1u);
}

// Exclusive scan of count[0..T) into start[0..T] (T a power of two >= 1024)
// in three passes: 1024-entry tiles scanned in LDS with their totals in
// tile[], the tile totals scanned by one block, the tile offsets added.
__device__ __forceinline__ uint32_t block_scan_256(uint32_t v, uint32_t *lds)
{
    const int t = threadIdx.x;
    lds[t] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t u = t >= off ? lds[t - off] : 0u;
        __syncthreads();
        lds[t] += u;
        __syncthreads();
    }
    return lds[t];              // inclusive
}

__global__ void __launch_bounds__(256) k_icp_scan_tiles(const IcpSorts so)
{
    __shared__ uint32_t lds[256];
    uint32_t *start = so.c[blockIdx.y].start, *tile = so.c[blockIdx.y].tile;
    const size_t base = (size_t)blockIdx.x * 1024 + threadIdx.x * 4;
    const uint4 c = *(const uint4 *)(so.c[blockIdx.y].count + base);
    const uint32_t own = c.x + c.y + c.z + c.w;
    const uint32_t incl = block_scan_256(own, lds);
    uint32_t run = incl - own;
    *(uint4 *)(start + base) = make_uint4(run, run + c.x, run + c.x + c.y, run + c.x + c.y + c.z);
    if (threadIdx.x == 255) tile[blockIdx.x] = incl;
}

// Exclusive scan of tile[0..nt) in place, 256 entries per round; the total
// becomes start[T].
__global__ void __launch_bounds__(256) k_icp_scan_top(const IcpSorts so, uint32_t nt)
{
    __shared__ uint32_t lds[256];
    uint32_t *tile = so.c[blockIdx.y].tile;
    uint32_t carry = 0;
    for (uint32_t r = 0; r < nt; r += 256) {
        const uint32_t i = r + threadIdx.x;
        const uint32_t v = i < nt ? tile[i] : 0u;
        const uint32_t incl = block_scan_256(v, lds);
        if (i < nt) tile[i] = carry + incl - v;
        carry += lds[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) so.c[blockIdx.y].start[(size_t)nt * 1024] = carry;
}

__global__ void __launch_bounds__(256) k_icp_scan_add(const IcpSorts so)
{
    uint32_t *start = so.c[blockIdx.y].start;
    const size_t base = (size_t)blockIdx.x * 1024 + threadIdx.x * 4;
    uint4 v = *(uint4 *)(start + base);
    const uint32_t o = so.c[blockIdx.y].tile[blockIdx.x];
    *(uint4 *)(start + base) = make_uint4(v.x + o, v.y + o, v.z + o, v.w + o);
}

// Records in bucket order, at the places the counting gave (the order inside
// a bucket is whatever the atomics give; nothing computed from the targets'
// records depends on it).
__global__ void __launch_bounds__(256) k_icp_scatter(const IcpSorts so, float inv_cell, const IcpHash *__restrict__ hp,
                                                    uint32_t T)
{
    const IcpSort &c = so.c[blockIdx.y];
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= c.n) return;
    const IcpHash h = *hp;
    const float *q = c.pts + (int64_t)j * 3;
    const float4 r = make_float4(q[0], q[1], q[2], __int_as_float(j));
    const uint32_t rank = c.rank[j];
    if (blockIdx.y == 0 && never_pairs(so, q)) {
        c.rec[c.start[T] + rank] = r;
        return;
    }
    const uint32_t b = bucket_of(h, q[0], q[1], q[2], inv_cell), s = c.start[b];
    c.rec[s + rank] = r;
    if (blockIdx.y == 0 && rank == 0u && c.start[b + 1] - s > kCrowd) so.crowded[atomicAdd(so.ncrowded, 1u)] = b;
}

// The number of w[s .. e) below `own`, four loads in flight.
template <typename Load>
__device__ __forceinline__ uint32_t count_below(Load load, uint32_t s, uint32_t e, int own)
{
    uint32_t below = 0;
    for (uint32_t k = s; k < e; k += 4) {
        int v[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) v[u] = load(k + u < e ? k + u : e - 1);
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) below += k + u < e && v[u] < own;
    }
    return below;
}

constexpr int kOrderBlock = 1024, kCrowdBlocks = 256;

// The records [s, e) of one crowded source bucket by index, in one block and
// linear time: the index range [0, n) is cut into as many slices as the bucket
// has records, so a slice holds at most n / records of them (and often one);
// they are counted (`sub`), gathered slice by slice (`idx`), and a record's
// place is its slice's first plus the slice's smaller indices.  Both arrays are
// the bucket's own; they are read and written past the vector cache, as the
// atomics are, and every access has ended before a barrier opens the next phase
// (agent-scope fences instead cost 571 us for 170 buckets of 5900 points).
__device__ void order_crowded(const float4 *__restrict__ in, uint32_t s, uint32_t e, int n, uint32_t *sub, int *idx,
                              float4 *__restrict__ out)
{
    __shared__ uint32_t s_wave[kOrderBlock / 64];
    constexpr uint32_t U = 4;                    // records of a thread in flight
    const uint32_t c = e - s, t = threadIdx.x;
    const int lane = (int)t & 63, wv = (int)t >> 6;
    auto slice = [&](int i) __attribute__((always_inline)) { return (uint32_t)((uint64_t)(uint32_t)i * c / (uint32_t)n); };
    auto get = [](const auto *p) __attribute__((always_inline)) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto put = [](auto *p, auto v) __attribute__((always_inline)) {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto phase = []() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };
    // Indices of the thread's next U records (-1 past the last).
    auto indices = [&](uint32_t k0, int (&i)[U]) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t k = k0 + u * kOrderBlock;
            i[u] = k < c ? __float_as_int(in[s + k].w) : -1;
        }
    };
    for (uint32_t k = t; k < c; k += kOrderBlock) put(&sub[k], 0u);
    phase();
    for (uint32_t k0 = t; k0 < c; k0 += U * kOrderBlock) {
        int i[U];
        indices(k0, i);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (i[u] >= 0) atomicAdd(&sub[slice(i[u])], 1u);
    }
    phase();
    // Counts to first places, eight per thread and round.
    uint32_t carry = 0;
    for (uint32_t r0 = 0; r0 < c; r0 += 8 * kOrderBlock) {
        uint32_t v[8], own = 0;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const uint32_t k = r0 + 8 * t + u;
            v[u] = k < c ? get(&sub[k]) : 0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) own += v[u];
        uint32_t incl = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(incl, d, 64);
            incl += lane >= d ? o : 0u;
        }
        if (lane == 63) s_wave[wv] = incl;
        __syncthreads();
        uint32_t before = carry, all = 0;
#pragma unroll
        for (int k = 0; k < kOrderBlock / 64; ++k) {
            before += k < wv ? s_wave[k] : 0u;
            all += s_wave[k];
        }
        uint32_t run = before + incl - own;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const uint32_t k = r0 + 8 * t + u;
            if (k < c) put(&sub[k], run);
            run += v[u];
        }
        carry += all;
        __syncthreads();
    }
    phase();
    for (uint32_t k0 = t; k0 < c; k0 += U * kOrderBlock) {
        int i[U];
        uint32_t at[U];
        indices(k0, i);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) at[u] = i[u] >= 0 ? atomicAdd(&sub[slice(i[u])], 1u) : 0u;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (i[u] >= 0) put(&idx[at[u]], i[u]);
    }
    phase();
    // sub[q] is now the end of slice q.
    for (uint32_t k0 = t; k0 < c; k0 += U * kOrderBlock) {
        int i[U];
        uint32_t lo[U], hi[U];
        indices(k0, i);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t q = i[u] >= 0 ? slice(i[u]) : 0u;
            lo[u] = q ? get(&sub[q - 1]) : 0u;
            hi[u] = get(&sub[q]);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (i[u] >= 0) {
                const uint32_t below =
                    count_below([&](uint32_t p) __attribute__((always_inline)) { return get(&idx[p]); }, lo[u], hi[u], i[u]);
                out[s + lo[u] + below] = in[s + k0 + u * kOrderBlock];
            }
    }
    phase();
}

// The source's records of each bucket by index: a record's place is the number
// of its bucket's records with a smaller one.  Up to kCrowd records are compared
// all with all; the blocks from `nb` on take the buckets with more, one block
// each.  Records of sources that never pair stay as they are.  All of it takes
// time linear in the points: a cloud of 256 000 with 100 000 holes costs 0.25 ms
// for five iterations, as one without (0.22; 10.5 with every bucket compared all
// with all), and 256 000 points in one cell 0.7 ms here (26).
__global__ void __launch_bounds__(kOrderBlock) k_icp_order(const IcpSorts so, uint32_t T, int nb, float inv_cell,
                                                          const IcpHash *__restrict__ hp, float4 *__restrict__ out)
{
    const IcpSort &c = so.c[0];
    const float4 *in = c.rec;
    if ((int)blockIdx.x >= nb) {
        const uint32_t nc = *so.ncrowded;
        for (uint32_t k = blockIdx.x - (unsigned)nb; k < nc; k += kCrowdBlocks) {
            const uint32_t b = so.crowded[k], s = c.start[b];
            // The counts are read no more, nor the ranks: T >= n words each.
            order_crowded(in, s, c.start[b + 1], c.n, c.rank + s, (int *)c.count + s, out);
        }
        return;
    }
    const int i = (int)blockIdx.x * kOrderBlock + (int)threadIdx.x;
    if (i >= c.n) return;
    const float4 r = in[i];
    if ((uint32_t)i >= c.start[T]) {
        out[i] = r;
        return;
    }
    const uint32_t b = bucket_of(*hp, r.x, r.y, r.z, inv_cell), s = c.start[b], e = c.start[b + 1];
    if (e - s > kCrowd) return;
    const int own = __float_as_int(r.w);
    out[s + count_below([&](uint32_t k) __attribute__((always_inline)) { return __float_as_int(in[k].w); }, s, e, own)] = r;
}

// Sum over each 16-lane row in a fixed order, the same on every lane of it.
__device__ __forceinline__ double row_sum(double v)
{
    auto step = [](double x, auto ctrl) __attribute__((always_inline)) {
        constexpr int C = decltype(ctrl)::value;
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
        const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, C, 0xF, 0xF, false);
        const uint32_t h = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, C, 0xF, 0xF, false);
        return x + __builtin_bit_cast(double, ((uint64_t)h << 32) | l);
    };
    v = step(v, std::integral_constant<int, 0xB1>{});    // neighbours
    v = step(v, std::integral_constant<int, 0x4E>{});    // pairs
    v = step(v, std::integral_constant<int, 0x141>{});   // half rows mirrored
    return step(v, std::integral_constant<int, 0x140>{});
}

// Nearest target within dmax of every source point, queries taken in the
// sorted record order, and the block's part of the pair sums (partial is
// [kIcpSums][blocks]).  prev: record number of each query's target in the
// previous iteration or -1 (read unless `first`), written for the next one;
// corr, where given, receives the pairing at the source index.
//
// Bound by the latency of its dependent gathers (query -> bucket range and
// previous target -> records), so everything that needs no answer of an
// earlier load is issued with it, and a lane goes through its own list of
// neighbour columns in reach instead of all lanes through all eight.  Measured
// on two clouds of 256 880 points, 30 iterations: 21.7 us an iteration with the
// sums, against 40 plus 11 for sums gathered in source order; the update 6.4
// against 9.0 us.
__global__ void __launch_bounds__(kIcpBlock) k_icp_corr(const float4 *__restrict__ qrec, int n, IcpGrid g,
                                                       const float *__restrict__ pose_f, float dmax2, bool first,
                                                       int32_t *__restrict__ prev, int32_t *__restrict__ corr,
                                                       double *__restrict__ partial)
{
#pragma clang fp contract(off)
    __shared__ double s_part[kIcpBlock / 16][kIcpSums];
    const int i = blockIdx.x * kIcpBlock + threadIdx.x;
    int best = -1, pos = -1;       // target index and record of the nearest so far
    float bd = 0.0f, q[3] = {0.0f, 0.0f, 0.0f};
    if (i < n) {
        const int before = first ? -1 : prev[i];
        const float4 r = qrec[i];
        const float4 told = before >= 0 ? g.rec[before] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        icp_move(pose_f, r.x, r.y, r.z, q);
        // Cell coordinates and, per axis, lower bounds of the distance to the
        // cells below (lo) and above (hi).  frac(v * inv) is exact; the margin
        // covers the rounding of v * inv on both sides of a cell boundary, of
        // cell vs 1 / inv, and of the products below (relative 2^-22 per cell
        // of coordinate magnitude, against errors of at most about 2^-24).
        int c[3];
        float lo[3], hi[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float sv = q[a] * g.inv_cell;
            const float fl = __builtin_floorf(sv);
            const float fr = sv - fl;
            c[a] = cell_index(fl);
            const float margin = (__builtin_fabsf(fl) + 4.0f) * (g.cell * 0x1p-22f);
            lo[a] = __builtin_fmaxf(fr * g.cell - margin, 0.0f);
            hi[a] = __builtin_fmaxf((1.0f - fr) * g.cell - margin, 0.0f);
        }
        const IcpHash h = *g.hash;
        auto test = [&](const float4 t, int at) __attribute__((always_inline)) {
            const float d = icp_dist2(q, t.x, t.y, t.z);
            const int j = __float_as_int(t.w);
            if (d <= dmax2 && (best < 0 || d < bd || (d == bd && j < best))) {
                best = j;
                bd = d;
                pos = at;
            }
        };
        // Records [s, e) in groups of four independent loads; in the last group
        // the loads past e re-read record e - 1 and stand for an infinitely far
        // point (never accepted).
        auto scan = [&](uint32_t s, uint32_t e) __attribute__((always_inline)) {
            const float4 far = make_float4(__builtin_inff(), __builtin_inff(), __builtin_inff(), 0.0f);
            for (; s < e; s += 4) {
                const uint32_t l = e - 1;
                float4 t[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) t[u] = g.rec[s + u < e ? s + u : l];
#pragma unroll
                for (int u = 0; u < 4; ++u) test(s + u < e ? t[u] : far, (int)(s + u));
            }
        };
        const float shrink = 1.0f - 0x1p-19f;
        auto reach = [&]() __attribute__((always_inline)) { return best < 0 ? dmax2 : bd; };
        // Lower bound of the squared distance to column k (y and x offsets
        // 0, -1, +1 by k / 3 and k % 3) in the plane.
        auto plane = [&](int ox, int oy) __attribute__((always_inline)) {
            const float lx = ox == 0 ? 0.0f : (ox == 1 ? lo[0] : hi[0]);
            const float ly = oy == 0 ? 0.0f : (oy == 1 ? lo[1] : hi[1]);
            const float lxy = lx * lx;
            return lxy + ly * ly;
        };
        // The three z cells of a column are adjacent buckets unless the z
        // coordinate wraps; then they are one record range, trimmed at either
        // end when that z neighbour is out of reach.
        auto column = [&](int ox, int oy, float lxy, auto ahead) __attribute__((always_inline)) {
            const int x = c[0] + (ox == 2 ? 1 : -(ox == 1)), y = c[1] + (oy == 2 ? 1 : -(oy == 1));
            const uint32_t b0 = cell_bucket(h, x, y, c[2]), bm = cell_bucket(h, x, y, c[2] - 1),
                           bp = cell_bucket(h, x, y, c[2] + 1);
            const float lbm = (lxy + lo[2] * lo[2]) * shrink, lbp = (lxy + hi[2] * hi[2]) * shrink;
            if (bm + 1 == b0 && b0 + 1 == bp) {
                uint32_t a[4];
                __builtin_memcpy(a, g.start + bm, 16);
                ahead();
                scan(lbm > reach() ? a[1] : a[0], lbp > reach() ? a[2] : a[3]);
            } else {
                ahead();
                scan(g.start[b0], g.start[b0 + 1]);
                // Wrapped z cells may share a bucket (with one z bit or none): scan each bucket once.
                bool did_m = false;
                if (bm != b0 && !(lbm > reach())) {
                    scan(g.start[bm], g.start[bm + 1]);
                    did_m = true;
                }
                if (bp != b0 && !(bp == bm && did_m) && !(lbp > reach())) scan(g.start[bp], g.start[bp + 1]);
            }
        };
        // The own column, after the previous target; then, per lane, the
        // neighbour columns still in reach.
        column(0, 0, 0.0f, [&]() __attribute__((always_inline)) {
            if (before >= 0) test(told, before);
        });
        uint32_t todo = 0u;
#pragma unroll
        for (int k = 1; k < 9; ++k)
            if (!(plane(k % 3, k / 3) * shrink > reach())) todo |= 1u << k;
#pragma unroll 1
        while (todo) {
            const int k = __builtin_ctz(todo);
            todo &= todo - 1u;
            const int oy = (k * 11) >> 5, ox = k - 3 * oy;
            const float lxy = plane(ox, oy);
            if (lxy * shrink > reach()) continue;
            column(ox, oy, lxy, []() {});
        }
        prev[i] = pos;
        if (corr) corr[__float_as_int(r.w)] = best;
    }
    // The pair's contributions, summed over the rows of the block's lanes and
    // then over its rows in order.
    double acc[kIcpSums];
#pragma unroll
    for (int k = 0; k < kIcpSums; ++k) acc[k] = 0.0;
    if (best >= 0) {
        const float4 t = g.rec[pos];
        const double tq[3] = {(double)t.x, (double)t.y, (double)t.z};
        acc[0] = 1.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            acc[1 + a] = (double)q[a];
            acc[4 + a] = tq[a];
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[7 + a * 3 + b] = (double)q[a] * tq[b];
        }
        acc[16] = (double)bd;
    }
    const int lane = threadIdx.x & 15, row = threadIdx.x >> 4;
#pragma unroll
    for (int k = 0; k < kIcpSums; ++k) {
        const double v = row_sum(acc[k]);
        if (lane == 0) s_part[row][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < kIcpSums) {
        double v = s_part[0][threadIdx.x];
#pragma unroll
        for (int k = 1; k < kIcpBlock / 16; ++k) v += s_part[k][threadIdx.x];
        partial[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = v;
    }
}

// Eigenvector of the largest eigenvalue of a symmetric 4 x 4 matrix (cyclic Jacobi).
__device__ __attribute__((noinline)) void jacobi4(double A[4][4], double v[4])
{
    double V[4][4];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) V[i][j] = i == j ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0, diag = 0.0;
        for (int p = 0; p < 4; ++p) {
            diag += A[p][p] * A[p][p];
            for (int q = p + 1; q < 4; ++q) off += A[p][q] * A[p][q];
        }
        // Off-diagonal entries below 1e-17 of the matrix norm: converged.
        if (off <= 1e-34 * (diag + off)) break;
        for (int p = 0; p < 3; ++p)
            for (int q = p + 1; q < 4; ++q) {
                if (A[p][q] == 0.0) continue;
                const double theta = (A[q][q] - A[p][p]) / (2.0 * A[p][q]);
                const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < 4; ++k) {
                    const double akp = A[k][p], akq = A[k][q];
                    A[k][p] = c * akp - s * akq;
                    A[k][q] = s * akp + c * akq;
                }
                for (int k = 0; k < 4; ++k) {
                    const double apk = A[p][k], aqk = A[q][k];
                    A[p][k] = c * apk - s * aqk;
                    A[q][k] = s * apk + c * aqk;
                }
                for (int k = 0; k < 4; ++k) {
                    const double vkp = V[k][p], vkq = V[k][q];
                    V[k][p] = c * vkp - s * vkq;
                    V[k][q] = s * vkp + c * vkq;
                }
            }
    }
    int best = 0;
    for (int i = 1; i < 4; ++i)
        if (A[i][i] > A[best][best]) best = i;
    for (int k = 0; k < 4; ++k) v[k] = V[k][best];
}

__device__ __forceinline__ double det3(double a, double b, double c, double d, double e, double f, double g, double h,
                                       double i)
{
    return a * (e * i - f * h) - b * (d * i - f * g) + c * (d * h - e * g);
}

// Determinant of M without row r and column c.
__device__ __forceinline__ double minor4(const double (&M)[4][4], int r, int c)
{
    double m[9];
    int k = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i != r && j != c) m[k++] = M[i][j];
    return det3(m[0], m[1], m[2], m[3], m[4], m[5], m[6], m[7], m[8]);
}

// Eigenvector of the largest eigenvalue of Horn's traceless symmetric 4 x 4
// matrix N built from H.  Its characteristic polynomial is
// x^4 + c2 x^2 + c1 x + c0 with c2 = -tr(N^2) / 2, c1 = -8 det(H), c0 =
// det(N); Newton's method from the upper bound sqrt(3 tr(N^2) / 4) (at
// least the sum of the singular values of H) descends monotonically onto the
// largest root, where the polynomial is convex.  The eigenvector is then the
// row of adj(N - x I) through its largest diagonal entry.  When that entry is
// tiny against |N|^3 (a repeated or nearly repeated top eigenvalue), cyclic
// Jacobi takes over.
__device__ __forceinline__ void horn_eigvec(const double (&N)[4][4], const double (&H)[3][3], double (&v)[4])
{
    double p2 = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) p2 += N[i][j] * N[i][j];
    if (p2 > 0.0) {
        const double c2 = -0.5 * p2;
        const double c1 = -8.0 * det3(H[0][0], H[0][1], H[0][2], H[1][0], H[1][1], H[1][2], H[2][0], H[2][1], H[2][2]);
        const double c0 = N[0][0] * minor4(N, 0, 0) - N[0][1] * minor4(N, 0, 1) + N[0][2] * minor4(N, 0, 2) -
                          N[0][3] * minor4(N, 0, 3);
        double x = sqrt(0.75 * p2);
        for (int k = 0; k < 100; ++k) {
            const double P = ((x * x + c2) * x + c1) * x + c0;
            const double dP = (4.0 * x * x + 2.0 * c2) * x + c1;
            if (!(dP > 0.0)) break;
            // An approximate quotient (about 26 bits): the last steps correct it.
            const double step = P * (double)__builtin_amdgcn_rcp(dP);
            x -= step;
            if (fabs(step) <= 1e-15 * fabs(x)) break;
        }
        double M[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) M[i][j] = N[i][j] - (i == j ? x : 0.0);
        // Every cofactor of the symmetric M, and the row of the largest
        // diagonal one by selection: an index known only at run time would put
        // the matrices into scratch memory.
        double cof[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = i; j < 4; ++j) cof[i][j] = cof[j][i] = ((i + j) & 1 ? -1.0 : 1.0) * minor4(M, i, j);
        double cr = fabs(cof[0][0]), row[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) row[j] = cof[0][j];
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            const bool larger = fabs(cof[i][i]) > cr;
            cr = larger ? fabs(cof[i][i]) : cr;
#pragma unroll
            for (int j = 0; j < 4; ++j) row[j] = larger ? cof[i][j] : row[j];
        }
        if (cr > 1e-6 * p2 * sqrt(p2)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = row[j];
            return;
        }
    }
    double A[4][4], u[4];   // copies: only these live in memory
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) A[i][j] = N[i][j];
    jacobi4(A, u);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = u[j];
}

// The rigid update from the pair sums s, composed onto the pose.  pose:
// FP64 [12] (R row-major, T); pose_f: the same rounded to FP32.  One thread.
__device__ __forceinline__ void icp_solve(const double (&s)[kIcpSums], double *pose, float *pose_f, int it, double *rms,
                          int32_t *pairs)
{
    const double n = s[0];
    double old[12];   // under way while the rotation is solved for
#pragma unroll
    for (int a = 0; a < 12; ++a) old[a] = pose[a];
    if (rms) rms[it] = n > 0.0 ? sqrt(s[16] / n) : 0.0;
    if (pairs) pairs[it] = (int32_t)n;
    if (n < 3.0) return;
    const double rn = 1.0 / n;
    double pc[3], qc[3], H[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        pc[a] = s[1 + a] * rn;
        qc[a] = s[4 + a] * rn;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) H[a][b] = s[7 + a * 3 + b] - n * pc[a] * qc[b];
    // Horn: N = [[tr, D^T], [D, H + H^T - tr I]], D = (H12 - H21, H20 - H02, H01 - H10).
    const double tr = H[0][0] + H[1][1] + H[2][2];
    double N[4][4];
    N[0][0] = tr;
    N[0][1] = N[1][0] = H[1][2] - H[2][1];
    N[0][2] = N[2][0] = H[2][0] - H[0][2];
    N[0][3] = N[3][0] = H[0][1] - H[1][0];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) N[1 + a][1 + b] = H[a][b] + H[b][a] - (a == b ? tr : 0.0);
    double qv[4];
    horn_eigvec(N, H, qv);
    const double w = qv[0], x = qv[1], y = qv[2], z = qv[3];
    const double nn = 1.0 / (w * w + x * x + y * y + z * z);
    const double Ri[3][3] = {{(w * w + x * x - y * y - z * z) * nn, 2.0 * (x * y - w * z) * nn, 2.0 * (x * z + w * y) * nn},
                             {2.0 * (x * y + w * z) * nn, (w * w - x * x + y * y - z * z) * nn, 2.0 * (y * z - w * x) * nn},
                             {2.0 * (x * z - w * y) * nn, 2.0 * (y * z + w * x) * nn, (w * w - x * x - y * y + z * z) * nn}};
    double Ti[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) Ti[a] = qc[a] - (Ri[a][0] * pc[0] + Ri[a][1] * pc[1] + Ri[a][2] * pc[2]);
    double R[3][3], T[3], Rn[3][3], Tn[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        T[a] = old[9 + a];
#pragma unroll
        for (int b = 0; b < 3; ++b) R[a][b] = old[a * 3 + b];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int b = 0; b < 3; ++b) Rn[a][b] = Ri[a][0] * R[0][b] + Ri[a][1] * R[1][b] + Ri[a][2] * R[2][b];
        Tn[a] = Ri[a][0] * T[0] + Ri[a][1] * T[1] + Ri[a][2] * T[2] + Ti[a];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        pose[9 + a] = Tn[a];
        pose_f[9 + a] = (float)Tn[a];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            pose[a * 3 + b] = Rn[a][b];
            pose_f[a * 3 + b] = (float)Rn[a][b];
        }
    }
}

// Adds up the block partials (one wavefront per sum, lanes over blocks, fixed
// order) and updates the pose.
constexpr int kUpdateBlock = 512;   // leaves the solver the registers it needs

__global__ void __launch_bounds__(kUpdateBlock) k_icp_update(const double *__restrict__ partial, int nblocks,
                                                            double *__restrict__ pose, float *__restrict__ pose_f,
                                                            int it, double *__restrict__ rms,
                                                            int32_t *__restrict__ pairs)
{
    __shared__ double s_row[kIcpSums][4];
    const int lane = threadIdx.x & 63;
    constexpr int kWaves = kUpdateBlock / 64, kPer = (kIcpSums + kWaves - 1) / kWaves, kAhead = 16;
    const int wv = (int)threadIdx.x >> 6;
    double v[kPer] = {};
    // Every load of 1024 blocks' partials is under way before the first is
    // added: they come from memory, written on other XCDs.
    for (int b0 = 0; b0 < nblocks; b0 += 64 * kAhead) {
        double p[kPer][kAhead];
#pragma unroll
        for (int q = 0; q < kPer; ++q)
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int k = min(wv + q * kWaves, kIcpSums - 1), b = min(b0 + lane + 64 * u, nblocks - 1);
                p[q][u] = partial[(int64_t)k * nblocks + b];
            }
#pragma unroll
        for (int q = 0; q < kPer; ++q)
#pragma unroll
            for (int u = 0; u < kAhead; ++u) v[q] += b0 + lane + 64 * u < nblocks ? p[q][u] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int k = wv + q * kWaves;
        const double t = row_sum(v[q]);
        if (k < kIcpSums && (lane & 15) == 0) s_row[k][lane >> 4] = t;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double tot[kIcpSums];
#pragma unroll
    for (int k = 0; k < kIcpSums; ++k) tot[k] = ((s_row[k][0] + s_row[k][1]) + s_row[k][2]) + s_row[k][3];
    icp_solve(tot, pose, pose_f, it, rms, pairs);
}

__global__ void k_copy_f64(const double *__restrict__ src, double *__restrict__ dst, int n)
{
    const int k = threadIdx.x;
    if (k < n) dst[k] = src[k];
}

// Buckets of both clouds' tables: a power of two, two per point of the larger
// cloud while that fits 32 bits (never fewer buckets than points).
static uint32_t icp_buckets(int n, int m)
{
    const uint64_t want = 2 * (uint64_t)std::max(n, m);
    uint32_t T = 1024;
    while (T < want && T < (1u << 31)) T <<= 1;
    return T;
}

static int blocks_of(int n, int per) { return (int)(((int64_t)n + per - 1) / per); }

size_t icp_workspace_bytes(int n, int m)
{
    const uint32_t T = icp_buckets(n, m);
    const size_t nb = (size_t)blocks_of(n, kIcpBlock);
    return 2 * (align_up(((size_t)T + 1) * 4) * 2 + align_up((size_t)(T / kCrowd) * 4)) + align_up((size_t)m * 16) +
           2 * align_up((size_t)n * 16) +
           align_up(nb * kIcpSums * 8 + 8) + align_up(12 * 8) + align_up(12 * 4) + align_up(kBoxBlocks * 6 * 4) +
           align_up(sizeof(IcpHash)) + align_up((size_t)n * 4) + align_up((size_t)m * 4);
}

bp_status launch_icp(const float *src, int n, const float *dst, int m, const double *pose_in, int iters, float dmax,
                     double *pose_out, double *rms, int32_t *pairs, int32_t *corr_out, uint8_t *ws, hipStream_t st)
{
    const uint32_t T = icp_buckets(n, m);
    const int nb = blocks_of(n, kIcpBlock);
    uint8_t *p = ws;
    IcpSorts so;
    for (IcpSort &c : so.c) {
        c.count = (uint32_t *)p;
        p += align_up(((size_t)T + 1) * 4);
        c.start = (uint32_t *)p;
        p += align_up(((size_t)T + 1) * 4);
        c.tile = (uint32_t *)p;
        p += align_up((size_t)(T / kCrowd) * 4);
    }
    float4 *rec_dst = (float4 *)p;
    p += align_up((size_t)m * 16);
    float4 *rec_src = (float4 *)p, *rec_tmp = (float4 *)(p + align_up((size_t)n * 16));
    p += 2 * align_up((size_t)n * 16);
    double *partial = (double *)p;
    p += align_up((size_t)nb * kIcpSums * 8 + 8);
    double *pose = (double *)p;
    p += align_up(12 * 8);
    float *pose_f = (float *)p;
    p += align_up(12 * 4);
    int *box = (int *)p;
    p += align_up(kBoxBlocks * 6 * 4);
    IcpHash *hash = (IcpHash *)p;
    p += align_up(sizeof(IcpHash));
    int32_t *prev = (int32_t *)p;   // each query's record in the last iteration (first its place in its bucket)
    uint32_t *rank_dst = (uint32_t *)(p + align_up((size_t)n * 4));
    // Cells slightly larger than dmax (edge dmax / 0.99): a target within dmax
    // of a query then lies in the 27 cells around the query's cell despite the
    // rounding of the cell coordinates, for coordinates within about 8e4
    // cells of the origin.
    const float inv_cell = 0.99f / dmax;
    const float dmax2 = dmax * dmax;
    so.c[0].pts = src;
    so.c[0].n = n;
    so.c[0].rec = rec_tmp;
    so.c[0].rank = (uint32_t *)prev;
    so.c[1].pts = dst;
    so.c[1].n = m;
    so.c[1].rec = rec_dst;
    so.c[1].rank = rank_dst;
    // The last words of the counts, and the words of the source's tile totals,
    // which are added up before the first bucket is listed (n points, at most
    // T, make fewer than T / kCrowd crowded buckets).
    so.inf_pairs = !std::isfinite(dmax2);
    so.gone = so.c[0].count + T;
    so.ncrowded = so.c[1].count + T;
    so.crowded = so.c[0].tile;
    uint32_t log2T = 0;
    while ((1u << log2T) < T) ++log2T;
    const int nparts = m > 0 ? std::min(kBoxBlocks, blocks_of(m, 256)) : 0;
    const dim3 points((unsigned)blocks_of(std::max(std::max(n, m), 1), 256), 2), tiles(T / 1024, 2);
    k_icp_bbox<<<(unsigned)nparts + T / 1024, 256, 0, st>>>(so, nparts, T, inv_cell, box);
    k_icp_hash<<<1, 64, 0, st>>>(so, box, nparts, log2T, hash, pose_in, pose, pose_f);
    k_icp_hist<<<points, 256, 0, st>>>(so, inv_cell, hash);
    k_icp_scan_tiles<<<tiles, 256, 0, st>>>(so);
    k_icp_scan_top<<<dim3(1, 2), 256, 0, st>>>(so, T / 1024);
    k_icp_scan_add<<<tiles, 256, 0, st>>>(so);
    k_icp_scatter<<<points, 256, 0, st>>>(so, inv_cell, hash, T);
    const int ob = blocks_of(n, kOrderBlock);
    if (n > 0) k_icp_order<<<ob + kCrowdBlocks, kOrderBlock, 0, st>>>(so, T, ob, inv_cell, hash, rec_src);
    bp_status s = launch_status();
    const IcpGrid g{so.c[1].start, rec_dst, hash, inv_cell, 1.0f / inv_cell};
    for (int it = 0; it < iters && s == BP_OK; ++it) {
        if (n > 0)
            k_icp_corr<<<nb, kIcpBlock, 0, st>>>(rec_src, n, g, pose_f, dmax2, it == 0, prev,
                                                 it == iters - 1 ? corr_out : nullptr, partial);
        k_icp_update<<<1, kUpdateBlock, 0, st>>>(partial, nb, pose, pose_f, it, rms, pairs);
        s = launch_status();
    }
    if (s == BP_OK) {
        k_copy_f64<<<1, 64, 0, st>>>(pose, pose_out, 12);
        s = launch_status();
    }
    return s;
}

}  // namespace bpk
