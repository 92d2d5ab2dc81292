// build.hip -- bounding volume hierarchy construction on gfx950.
//
// Steps (paper: Background -- Morton codes, spatial sort, binary radix tree of
// Karras 2012; Specific changes -- Morton kernel, 64-bit codes; Case Studies
// 1-2 -- sorted int32 triangle ids, bottom-up node filling with one atomic
// counter per internal node, N_t - 1 internal nodes, a launch sized by N_t):
//   1. mesh extent            min / max over all vertices
//   2. Morton keys            one lane per triangle, first digit counted
//   3. LDS radix sort         stable LSD, 8-bit digits: tile histograms,
//                             one device-wide scan, stable tile scatter
//   4. radix tree             one lane per internal node (Karras section 3)
//   5. leaves + bottom-up     one lane per leaf, arrival counters in LDS
//                             inside subtrees of <= 1024 leaves; one
//                             workgroup finishes the nodes above them
#include "rsi_internal.h"

namespace rsi {
namespace {

constexpr int kSortThreads = 1024;
constexpr int kSortItems = 2;
constexpr int kSortTile = kSortThreads * kSortItems;  // 2048 keys per tile
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kRadix = 256;
// Up to this many tiles (131,072 keys) a pass is one launch: every scatter
// workgroup derives its own offsets from the whole (small) histogram and adds
// its keys to the next pass's histogram as it places them.
constexpr int kSmallSortTiles = 64;
constexpr int kBoxTile = kTileLeaves;  // leaves per bottom-up workgroup (one per lane)
constexpr int kNoTile = INT32_MIN;  // never a child reference (leaves are ~k with k < 2^30)
constexpr int kRestructureRounds = 2;  // treelet restructuring passes of algorithm 2

// ---------------------------------------------------------------- 1. extent
// Min / max are exact in any order, so the extent is reduced in two steps:
// up to kBoundsParts workgroups each reduce a strided share of the vertices;
// every workgroup of the Morton kernel combines their partial boxes (6 KB from
// L2), which costs less than a launch of its own (about 4.6 us).

// Block-wide min / max of six values (lo xyz, hi xyz); the result is valid in
// thread 0.
__device__ __forceinline__ void block_minmax(float lo[3], float hi[3]) {
    for (int off = 32; off > 0; off >>= 1)
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], off));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off));
        }
    __shared__ float red[16][6];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0)
        for (int a = 0; a < 3; ++a) {
            red[w][a] = lo[a];
            red[w][3 + a] = hi[a];
        }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        for (int k = 1; k < nw; ++k)
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], red[k][a]);
                hi[a] = fmaxf(hi[a], red[k][3 + a]);
            }
    }
}

// The same over the first WAVES waves, valid in every thread.
template <int WAVES>
__device__ __forceinline__ void block_minmax_all(float lo[3], float hi[3]) {
    __shared__ float red[WAVES][6];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (w < WAVES) {
        for (int off = 32; off > 0; off >>= 1)
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], __shfl_xor(lo[a], off));
                hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off));
            }
        if (lane == 0)
            for (int a = 0; a < 3; ++a) {
                red[w][a] = lo[a];
                red[w][3 + a] = hi[a];
            }
    }
    __syncthreads();
    for (int a = 0; a < 3; ++a) {
        lo[a] = red[0][a];
        hi[a] = red[0][3 + a];
#pragma unroll
        for (int k = 1; k < WAVES; ++k) {
            lo[a] = fminf(lo[a], red[k][a]);
            hi[a] = fmaxf(hi[a], red[k][3 + a]);
        }
    }
}

// (also copies the caller's vertices into the mesh's own array, and clears
// the build flags)
__global__ __launch_bounds__(1024) void k_mesh_bounds_part(const float *__restrict__ V, int64_t nv,
                                                           float *__restrict__ partial, float *__restrict__ V_copy,
                                                           int32_t *__restrict__ flags) {
    if (blockIdx.x == 0 && threadIdx.x < 4)
        flags[threadIdx.x] = 0;  // (flags[2]: the number of tiles the radix-tree kernel lists)
    float lo[3] = {INFINITY, INFINITY, INFINITY};
    float hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += (int64_t)gridDim.x * blockDim.x)
        for (int a = 0; a < 3; ++a) {
            const float x = V[3 * i + a];
            V_copy[3 * i + a] = x;
            lo[a] = fminf(lo[a], x);
            hi[a] = fmaxf(hi[a], x);
        }
    block_minmax(lo, hi);
    if (threadIdx.x == 0)
        for (int a = 0; a < 3; ++a) {
            partial[6 * blockIdx.x + a] = lo[a];
            partial[6 * blockIdx.x + 3 + a] = hi[a];
        }
}

// ---------------------------------------------------------- 2. Morton keys
// Spread the low 10 (or 21) bits of x so that bit k lands on bit 3k.
__device__ __forceinline__ uint32_t spread3(uint32_t x) {
    x &= 0x3ffu;
    x = (x | (x << 16)) & 0x030000ffu;
    x = (x | (x << 8)) & 0x0300f00fu;
    x = (x | (x << 4)) & 0x030c30c3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}
__device__ __forceinline__ uint64_t spread3(uint64_t x) {
    x &= 0x1fffffull;
    x = (x | (x << 32)) & 0x001f00000000ffffull;
    x = (x | (x << 16)) & 0x001f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Quantise one centroid coordinate: n = (c - lo) / ext (0 for a flat axis),
// q = floor(min(n 2^b, 2^b - 1)), 0 for n <= 0 or NaN.  Single float32 ops,
// no contraction.
__device__ __forceinline__ uint32_t quantise(float c, float lo, float ext, float two_b, float top) {
#pragma clang fp contract(off)
    float n = ext > 0.0f ? (c - lo) / ext : 0.0f;
    float x = n * two_b;
    return x > 0.0f ? (uint32_t)floorf(fminf(x, top)) : 0u;
}

// The digit counts of one sort tile in LDS: a lane per digit clears h before
// and writes it after (a workgroup of kSortThreads lanes).
__device__ __forceinline__ void put_hist(const uint32_t *h, int tile, int ntiles, uint32_t *__restrict__ hist,
                                         uint32_t *__restrict__ clear) {
    if (threadIdx.x < kRadix) {
        hist[(int64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
        if (clear)  // one-launch passes: the histogram the first pass adds to
            clear[(int64_t)threadIdx.x * ntiles + tile] = 0u;
    }
}

// One workgroup per sort tile: the mesh extent from its partial boxes, the
// keys, and the counts of their lowest digit for the sort's first pass.
// (Also copies the caller's triangles into the mesh's own array.)
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_morton(const float *__restrict__ V, int64_t nv,
                                                         const int32_t *__restrict__ F, int64_t nt,
                                                         const float *__restrict__ partial, int parts,
                                                         float *__restrict__ bounds, K *__restrict__ keys,
                                                         int32_t *__restrict__ ids, int32_t *__restrict__ flags,
                                                         int32_t *__restrict__ F_copy, int ntiles,
                                                         uint32_t *__restrict__ hist, uint32_t *__restrict__ clear) {
#pragma clang fp contract(off)
    __shared__ uint32_t h[kRadix];
    const int tid = threadIdx.x;
    if (tid < kRadix)
        h[tid] = 0;
    float lo[3] = {INFINITY, INFINITY, INFINITY};
    float hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (tid < parts)
        for (int a = 0; a < 3; ++a) {
            lo[a] = partial[6 * tid + a];
            hi[a] = partial[6 * tid + 3 + a];
        }
    block_minmax_all<kBoundsParts / 64>(lo, hi);  // (also orders the clearing of h)
    if (blockIdx.x == 0 && tid == 0) {
        float scale = 0.0f;
        for (int a = 0; a < 3; ++a) {
            bounds[a] = lo[a];
            bounds[3 + a] = hi[a];
            if (lo[a] <= hi[a])  // no vertices: no scale
                scale = fmaxf(scale, fmaxf(fabsf(lo[a]), fabsf(hi[a])));
        }
        bounds[6] = scale;
        bounds[7] = 0.0f;
    }
    constexpr int b = sizeof(K) == 4 ? 10 : 21;
    const float two_b = (float)(1u << b), top = (float)((1u << b) - 1u);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t t = (int64_t)blockIdx.x * kSortTile + r * kSortThreads + tid;
        if (t >= nt)
            break;
        const int32_t i0 = F[3 * t], i1 = F[3 * t + 1], i2 = F[3 * t + 2];
        F_copy[3 * t] = i0;
        F_copy[3 * t + 1] = i1;
        F_copy[3 * t + 2] = i2;
        ids[t] = (int32_t)t;
        K key = 0;
        if (i0 < 0 || i1 < 0 || i2 < 0 || i0 >= nv || i1 >= nv || i2 >= nv) {
            atomicOr(flags, 1);
        } else {
            float c[3];
            for (int a = 0; a < 3; ++a)
                c[a] = ((V[3 * (int64_t)i0 + a] + V[3 * (int64_t)i1 + a]) + V[3 * (int64_t)i2 + a]) / 3.0f;
            for (int a = 2; a >= 0; --a)  // z, then y, then x: z lands on the top bit of each triple
                key = (K)(key << 1) | spread3((K)quantise(c[a], lo[a], hi[a] - lo[a], two_b, top));
        }
        keys[t] = key;
        atomicAdd(&h[(uint32_t)key & 0xffu], 1u);
    }
    __syncthreads();
    put_hist(h, blockIdx.x, ntiles, hist, clear);
}

// Batched form: the key of a triangle of mesh m is m (6 bits) above a 30-bit
// Morton code (10 bits per axis) of its centroid normalised to mesh m's box,
// so each mesh's triangles are contiguous after the sort and form one subtree.
// One workgroup per sort tile, as k_morton.  The meshes' extents come as
// order-preserving integers; the first workgroup also writes them as floats,
// with their union and the largest coordinate magnitude (the traversal widens
// boxes relative to it).
__global__ __launch_bounds__(kSortThreads) void k_morton_batch(
    const float *__restrict__ V, const int32_t *__restrict__ F, const int32_t *__restrict__ tri_mesh, int64_t nt,
    const uint32_t *__restrict__ key_bounds, int M, float *__restrict__ mesh_bounds, float *__restrict__ bounds,
    uint64_t *__restrict__ keys, int32_t *__restrict__ ids, int ntiles, uint32_t *__restrict__ hist,
    uint32_t *__restrict__ clear) {
#pragma clang fp contract(off)
    __shared__ uint32_t h[kRadix];
    __shared__ float bb[64][6];
    const int tid = threadIdx.x;
    if (tid < kRadix)
        h[tid] = 0;
    for (int k = tid; k < 6 * M; k += kSortThreads)
        bb[k / 6][k % 6] = order_value(key_bounds[8 * (k / 6) + k % 6]);
    __syncthreads();
    if (blockIdx.x == 0 && tid < 64) {
        float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY}, scale = 0.0f;
        if (tid < M) {
            for (int a = 0; a < 3; ++a) {
                lo[a] = bb[tid][a];
                hi[a] = bb[tid][3 + a];
                mesh_bounds[8 * tid + a] = lo[a];
                mesh_bounds[8 * tid + 3 + a] = hi[a];
                if (lo[a] <= hi[a])  // an empty mesh (lo = +inf, hi = -inf) adds no scale
                    scale = fmaxf(scale, fmaxf(fabsf(lo[a]), fabsf(hi[a])));
            }
            mesh_bounds[8 * tid + 6] = scale;
            mesh_bounds[8 * tid + 7] = 0.0f;
        }
        for (int off = 32; off > 0; off >>= 1) {
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], __shfl_xor(lo[a], off));
                hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off));
            }
            scale = fmaxf(scale, __shfl_xor(scale, off));
        }
        if (tid == 0) {
            for (int a = 0; a < 3; ++a) {
                bounds[a] = lo[a];
                bounds[3 + a] = hi[a];
            }
            bounds[6] = scale;
            bounds[7] = 0.0f;
        }
    }
    // 10 bits per axis of the mesh's own box, as the single-mesh 30-bit codes
    const float two_b = (float)(1u << 10), top = (float)((1u << 10) - 1u);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t t = (int64_t)blockIdx.x * kSortTile + r * kSortThreads + tid;
        if (t >= nt)
            break;
        ids[t] = (int32_t)t;
        const int m = tri_mesh[t];
        const int32_t i0 = F[3 * t], i1 = F[3 * t + 1], i2 = F[3 * t + 2];
        uint64_t key = 0;
        if (i0 >= 0 && i1 >= 0 && i2 >= 0)  // (-1: marked invalid while copying)
            for (int a = 2; a >= 0; --a) {
                const float c =
                    ((V[3 * (int64_t)i0 + a] + V[3 * (int64_t)i1 + a]) + V[3 * (int64_t)i2 + a]) / 3.0f;
                key = (key << 1) | spread3((uint64_t)quantise(c, bb[m][a], bb[m][3 + a] - bb[m][a], two_b, top));
            }
        keys[t] = ((uint64_t)m << kBatchMortonBits) | key;
        atomicAdd(&h[(uint32_t)key & 0xffu], 1u);
    }
    __syncthreads();
    put_hist(h, blockIdx.x, ntiles, hist, clear);
}

// ---------------------------------------------------------- 3. radix sort
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const K *__restrict__ keys, int64_t n, int shift,
                                                            int ntiles, uint32_t *__restrict__ hist,
                                                            uint32_t *__restrict__ clear) {
    __shared__ uint32_t h[kRadix];
    const int tid = threadIdx.x, tile = blockIdx.x;
    if (tid < kRadix)
        h[tid] = 0;
    __syncthreads();
    const int64_t base = (int64_t)tile * kSortTile;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t idx = base + r * kSortThreads + tid;
        if (idx < n)
            atomicAdd(&h[(uint32_t)(keys[idx] >> shift) & 0xffu], 1u);
    }
    __syncthreads();
    put_hist(h, tile, ntiles, hist, clear);
}

// Exclusive scan of hist[0..len) in place, one workgroup of 1024 lanes.
__global__ __launch_bounds__(1024) void k_sort_scan(uint32_t *__restrict__ hist, int64_t len) {
    __shared__ uint32_t part[1024];
    const int tid = threadIdx.x;
    const int64_t chunk = (len + 1023) / 1024;
    const int64_t beg = tid * chunk, end = beg + chunk < len ? beg + chunk : len;
    uint32_t s = 0;
    for (int64_t i = beg; i < end; ++i)
        s += hist[i];
    part[tid] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        uint32_t v = tid >= off ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    uint32_t run = part[tid] - s;  // exclusive prefix of this chunk
    for (int64_t i = beg; i < end; ++i) {
        uint32_t v = hist[i];
        hist[i] = run;
        run += v;
    }
}

// Large histograms: per-block sums, a scan of those (k_sort_scan), then each
// block scans its own segment from its offset.  Reads are coalesced rounds of
// 1024 entries; seg is a multiple of 1024.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *wsum, uint32_t &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off)
            x += y;
    }
    if (lane == 63)
        wsum[w] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int k = 0; k < nw; ++k) {
        const uint32_t t = wsum[k];
        before += k < w ? t : 0u;
        all += t;
    }
    __syncthreads();  // wsum is reused by the next round
    total = all;
    return before + x - v;
}

__global__ __launch_bounds__(1024) void k_scan_partials(const uint32_t *__restrict__ hist, int64_t len, int64_t seg,
                                                        uint32_t *__restrict__ partial) {
    __shared__ uint32_t wsum[16];
    const int64_t beg = (int64_t)blockIdx.x * seg, end = beg + seg < len ? beg + seg : len;
    uint32_t s = 0;
    for (int64_t i = beg + threadIdx.x; i < end; i += blockDim.x)
        s += hist[i];
    uint32_t total;
    (void)block_excl_scan(s, wsum, total);
    if (threadIdx.x == 0)
        partial[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan_apply(uint32_t *__restrict__ hist, int64_t len, int64_t seg,
                                                     const uint32_t *__restrict__ partial) {
    __shared__ uint32_t wsum[16];
    const int64_t beg = (int64_t)blockIdx.x * seg, end = beg + seg < len ? beg + seg : len;
    uint32_t run = partial[blockIdx.x];
    for (int64_t r = beg; r < end; r += blockDim.x) {
        const int64_t i = r + threadIdx.x;
        const uint32_t v = i < end ? hist[i] : 0u;
        uint32_t total;
        const uint32_t ex = block_excl_scan(v, wsum, total);
        if (i < end)
            hist[i] = run + ex;
        run += total;
    }
}

// The tile histograms of a large sort, one row of ntiles per digit: workgroup
// d scans row d in place (exclusive) and writes its total to totals[d]; the
// scatter adds the digits below from those totals.  One launch instead of
// a three-step scan of the whole histogram.
__global__ __launch_bounds__(1024) void k_scan_rows(uint32_t *__restrict__ hist, int64_t ntiles,
                                                    uint32_t *__restrict__ totals) {
    __shared__ uint32_t wsum[16];
    uint32_t *row = hist + (int64_t)blockIdx.x * ntiles;
    uint32_t run = 0;
    for (int64_t r = 0; r < ntiles; r += blockDim.x) {
        const int64_t i = r + threadIdx.x;
        const uint32_t v = i < ntiles ? row[i] : 0u;
        uint32_t total;
        const uint32_t ex = block_excl_scan(v, wsum, total);
        if (i < ntiles)
            row[i] = run + ex;
        run += total;
    }
    if (threadIdx.x == 0)
        totals[blockIdx.x] = run;
}

// Exclusive scan of hist[0..len); partial holds 1024 entries.
void scan_hist(uint32_t *hist, int64_t len, uint32_t *partial, hipStream_t s) {
    if (len <= 32768) {
        k_sort_scan<<<1, 1024, 0, s>>>(hist, len);
        return;
    }
    const int64_t per = (len + 1023) / 1024;
    const int64_t seg = (per + 1023) / 1024 * 1024;
    const int g = (int)((len + seg - 1) / seg);
    k_scan_partials<<<g, 1024, 0, s>>>(hist, len, seg, partial);
    k_sort_scan<<<1, 1024, 0, s>>>(partial, g);
    k_scan_apply<<<g, 1024, 0, s>>>(hist, len, seg, partial);
}

// Stable scatter of one tile of 2048 keys by a workgroup of 16 waves, two
// keys a lane.  A key's rank inside its wave's 64 consecutive keys comes from
// matching the 8 digit bits with ballots; the counts of all 32 groups of 64
// are scanned per digit in one step (four lanes a digit), so the tile takes
// three barriers.  (Eight keys a lane of four waves, ranked in eight rounds of
// three barriers each, took 11.5 us a pass at 32,258 keys and 22 us at 11,000
// 64-bit ones, against 8.1 and 7.9.)  base[d] is where the tile's keys of
// digit d start.  With hist_next, each placed key's next digit is counted at
// the tile its new position falls in.
template <typename K>
__device__ __forceinline__ void scatter_tile(const K *__restrict__ kin, const int32_t *__restrict__ iin,
                                             K *__restrict__ kout, int32_t *__restrict__ iout, int64_t n,
                                             int shift, int tile, const uint32_t *base,
                                             uint32_t (*cnt)[kRadix], uint32_t *__restrict__ hist_next,
                                             int ntiles) {
    const int tid = threadIdx.x, wave = tid >> 6;
    const int64_t t0 = (int64_t)tile * kSortTile;
    K key[kSortItems];
    int32_t id[kSortItems];
    uint32_t rank[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t idx = t0 + r * kSortThreads + tid;
        key[r] = idx < n ? kin[idx] : K(0);
        id[r] = idx < n ? iin[idx] : 0;
    }
    uint32_t *flat = &cnt[0][0];
#pragma unroll
    for (int k = 0; k < kSortItems * kSortWaves * kRadix / kSortThreads; ++k)
        flat[k * kSortThreads + tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const bool valid = t0 + r * kSortThreads + tid < n;
        const uint32_t digit = (uint32_t)(key[r] >> shift) & 0xffu;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool set = (digit >> bit) & 1u;
            const uint64_t m = __ballot(set);
            peers &= set ? m : ~m;
        }
        rank[r] = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
        if (valid && rank[r] == 0)
            cnt[r * kSortWaves + wave][digit] = __popcll(peers);
    }
    __syncthreads();
    {
        // four lanes a digit, eight groups of 64 each: where each group's keys
        // of the digit start
        constexpr int kGroups = kSortItems * kSortWaves / 4;
        const int d = tid >> 2, q = tid & 3;
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kGroups; ++k)
            sum += cnt[q * kGroups + k][d];
        uint32_t before = 0;  // the sums of the lower lanes of the four
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            const uint32_t o = __shfl(sum, (threadIdx.x & 63 & ~3) | ((q - k) & 3));
            before += q >= k ? o : 0u;
        }
        before += base[d];
#pragma unroll
        for (int k = 0; k < kGroups; ++k) {
            const uint32_t c = cnt[q * kGroups + k][d];
            cnt[q * kGroups + k][d] = before;
            before += c;
        }
    }
    __syncthreads();
    uint32_t pos[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t digit = (uint32_t)(key[r] >> shift) & 0xffu;
        pos[r] = cnt[r * kSortWaves + wave][digit] + rank[r];
        if (t0 + r * kSortThreads + tid < n) {
            kout[pos[r]] = key[r];
            iout[pos[r]] = id[r];
        }
    }
    if (!hist_next)
        return;
    // the tile's next digits by destination tile, counted in the LDS that held
    // the groups' counts (two 16-bit counts a word), then added to the next
    // pass's histogram: a global atomic per key took most of a pass where few
    // digits occur (22 us for 11,000 keys)
    const int words = kRadix * ntiles / 2;
    __syncthreads();
    for (int k = tid; k < words; k += kSortThreads)
        flat[k] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
        if (t0 + r * kSortThreads + tid < n) {
            const uint32_t at = ((uint32_t)(key[r] >> (shift + 8)) & 0xffu) * ntiles + pos[r] / kSortTile;
            atomicAdd(flat + (at >> 1), 1u << (16 * (at & 1)));
        }
    __syncthreads();
    for (int k = tid; k < words; k += kSortThreads) {
        const uint32_t c = flat[k];
        if (c & 0xffffu)
            atomicAdd(hist_next + 2 * k, c & 0xffffu);
        if (c >> 16)
            atomicAdd(hist_next + 2 * k + 1, c >> 16);
    }
}
static_assert(kRadix * kSmallSortTiles / 2 <= kSortItems * kSortWaves * kRadix, "the counts fit");

// One scatter pass over tile histograms scanned per digit (offs: digit-major,
// exclusive within each digit's row; totals: each digit's count).
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const K *__restrict__ kin,
                                                               const int32_t *__restrict__ iin,
                                                               K *__restrict__ kout, int32_t *__restrict__ iout,
                                                               int64_t n, int shift, int ntiles,
                                                               const uint32_t *__restrict__ offs,
                                                               const uint32_t *__restrict__ totals) {
    __shared__ uint32_t base[kRadix];
    __shared__ uint32_t cnt[kSortItems * kSortWaves][kRadix];
    __shared__ uint32_t wsum[kSortWaves];
    const int tid = threadIdx.x, tile = blockIdx.x;
    uint32_t all;
    const uint32_t below = block_excl_scan(tid < kRadix ? totals[tid] : 0u, wsum, all);  // keys of the digits below
    if (tid < kRadix)
        base[tid] = below + offs[(int64_t)tid * ntiles + tile];
    scatter_tile<K>(kin, iin, kout, iout, n, shift, tile, base, cnt, nullptr, ntiles);
}

// One pass of a small sort in one launch.  hist holds this pass's per-tile
// digit counts (digit-major); each workgroup sums them into its own offsets
// (digits below, then earlier tiles of its digit; four lanes a digit) and
// scatters its tile, counting the next digit into hist_next (null after the
// last pass).  hist_clear (the histogram two passes on) is zeroed here: nothing
// reads or adds to it during this pass.
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_sort_pass_small(const K *__restrict__ kin,
                                                                  const int32_t *__restrict__ iin,
                                                                  K *__restrict__ kout, int32_t *__restrict__ iout,
                                                                  int64_t n, int shift, int ntiles,
                                                                  const uint32_t *__restrict__ hist,
                                                                  uint32_t *__restrict__ hist_next,
                                                                  uint32_t *__restrict__ hist_clear) {
    __shared__ uint32_t base[kRadix];
    __shared__ uint32_t total[kRadix];
    __shared__ uint32_t cnt[kSortItems * kSortWaves][kRadix];
    __shared__ uint32_t wsum[kSortWaves];
    const int tid = threadIdx.x, tile = blockIdx.x;
    uint32_t earlier = 0, sum = 0;
    const uint32_t *h = hist + (int64_t)(tid >> 2) * ntiles;
    for (int t = tid & 3; t < ntiles; t += 4) {
        const uint32_t v = h[t];
        earlier += t < tile ? v : 0u;
        sum += v;
    }
#pragma unroll
    for (int off = 1; off < 4; off <<= 1) {
        earlier += __shfl_xor(earlier, off);
        sum += __shfl_xor(sum, off);
    }
    if ((tid & 3) == 0) {
        base[tid >> 2] = earlier;
        total[tid >> 2] = sum;
    }
    __syncthreads();
    uint32_t all;
    const uint32_t below = block_excl_scan(tid < kRadix ? total[tid] : 0u, wsum, all);
    if (tid < kRadix) {
        base[tid] += below;
        hist_clear[(int64_t)tid * ntiles + tile] = 0u;
    }
    scatter_tile<K>(kin, iin, kout, iout, n, shift, tile, base, cnt, hist_next, ntiles);
}

// ---------------------------------------------------------- 4. radix tree
// Length of the common prefix of key_i || i and key_j || j; -1 outside [0, n).
template <typename K>
__device__ __forceinline__ int prefix(const K *__restrict__ k, int n, int i, K ki, int j) {
    if (j < 0 || j >= n)
        return -1;
    const K kj = k[j];
    if (ki != kj) {
        if constexpr (sizeof(K) == 8)
            return __builtin_clzll((unsigned long long)(ki ^ kj));
        else
            return __builtin_clz((unsigned)(ki ^ kj));
    }
    return (int)(8 * sizeof(K)) + __builtin_clz((unsigned)(i ^ j));
}

// Also lists the bottom-up tiles: the largest subtrees with at most kBoxTile
// leaves (children of larger nodes, or the root itself), wave-aggregated into
// tiles[0 .. *n_tiles).  In the batched form (roots not NULL) it also finds
// each mesh's subtree root and flags it for the 4-wide collapse.
template <typename K>
__global__ __launch_bounds__(256) void k_radix_tree(const K *__restrict__ keys, int n, Node *__restrict__ nodes,
                                                    int32_t *__restrict__ parent, int32_t *__restrict__ counters,
                                                    int32_t *__restrict__ tiles, int32_t *__restrict__ n_tiles,
                                                    int32_t *__restrict__ flag, int32_t *__restrict__ roots) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1)
        return;
    // the root of a mesh of one triangle is its leaf
    auto mesh = [&](int k) { return (int)((uint64_t)keys[k] >> kBatchMortonBits); };
    auto leaf_root = [&](int k) {
        const int m = mesh(k);
        if ((k == 0 || mesh(k - 1) != m) && (k == n - 1 || mesh(k + 1) != m))
            roots[m] = ~k;
    };
    if (roots) {
        leaf_root(i);
        if (i == n - 2)
            leaf_root(n - 1);
    }
    const K ki = keys[i];
    const int d = prefix(keys, n, i, ki, i + 1) > prefix(keys, n, i, ki, i - 1) ? 1 : -1;
    const int below = prefix(keys, n, i, ki, i - d);
    int len_max = 2;
    while (prefix(keys, n, i, ki, i + len_max * d) > below)
        len_max <<= 1;
    int len = 0;
    for (int step = len_max >> 1; step >= 1; step >>= 1)
        if (prefix(keys, n, i, ki, i + (len + step) * d) > below)
            len += step;
    const int j = i + len * d;
    const int node_prefix = prefix(keys, n, i, ki, j);
    int s = 0;
    for (int div = 2;; div <<= 1) {
        const int step = (len + div - 1) / div;
        if (prefix(keys, n, i, ki, i + (s + step) * d) > node_prefix)
            s += step;
        if (step <= 1)
            break;
    }
    const int split = i + s * d + (d < 0 ? -1 : 0);
    const int lo = min(i, j), hi = max(i, j);
    const int left = (lo == split) ? ~split : split;
    const int right = (hi == split + 1) ? ~(split + 1) : split + 1;
    nodes[i].refs = make_int4(left, right, lo, hi);
    parent[left >= 0 ? left : (n - 1) + ~left] = i;
    parent[right >= 0 ? right : (n - 1) + ~right] = i;
    counters[i] = 0;
    // the internal node whose key range is exactly a mesh's keys is its root
    if (roots) {
        const int m = mesh(lo);
        const bool is_root = mesh(hi) == m && (lo == 0 || mesh(lo - 1) != m) && (hi == n - 1 || mesh(hi + 1) != m);
        if (is_root)
            roots[m] = i;
        flag[i] = is_root ? kMeshRootFlag : 0;
    }
    if (i == 0)
        parent[0] = -1;

    int emit0 = kNoTile, emit1 = kNoTile;
    if (hi - lo + 1 > kBoxTile) {
        if (split - lo + 1 <= kBoxTile)
            emit0 = left;
        if (hi - split <= kBoxTile)
            emit1 = right;
    } else if (i == 0) {
        emit0 = 0;  // the whole tree is one tile
    }
    const uint64_t m1 = __ballot(emit0 != kNoTile || emit1 != kNoTile);
    const uint64_t m2 = __ballot(emit0 != kNoTile && emit1 != kNoTile);
    if (m1) {
        const int lane = threadIdx.x & 63;
        const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
        const int leader = __ffsll((unsigned long long)m1) - 1;
        int base = 0;
        if (lane == leader)
            base = atomicAdd(n_tiles, __popcll(m1) + __popcll(m2));
        base = __shfl(base, leader);
        int o = base + __popcll(m1 & lt) + __popcll(m2 & lt);
        if (emit0 != kNoTile)
            tiles[o++] = emit0;
        if (emit1 != kNoTile)
            tiles[o] = emit1;
    }
}

// one triangle: the leaf is the whole tree (batched form: of its mesh)
template <typename K>
__global__ void k_single_tile(int32_t *tiles, int32_t *n_tiles, const K *keys, int32_t *roots) {
    tiles[0] = ~0;
    *n_tiles = 1;
    if (roots)
        roots[(uint64_t)keys[0] >> kBatchMortonBits] = ~0;
}

// ------------------------------------------------- 5. leaves and bottom-up
// Boxes are merged bottom-up, each internal node by the second of its two
// children to finish (the paper's Case Study 2: one arrival counter per
// internal node).  The tree is cut into tiles, the largest subtrees with at
// most kBoxTile leaves (listed by k_radix_tree), and nodes above them:
//   k_leaves_subtree  one workgroup per tile: counters and child boxes in LDS,
//                     no cross-workgroup synchronisation at all;
//   k_boxes_top       one workgroup climbs the nodes above the tiles with
//                     workgroup-scope atomics.
// Cross-XCD agent-scope atomics, which cost an L2 write-back each on gfx950,
// are not needed.  Every child box lands in its parent node in HBM; a
// finished internal node's counter reads 2.
// Leaf k (sorted position): write its triangle (A, B - A, C - A, input index)
// and return its box.  An invalid triangle is never hit and widens no box.
__device__ __forceinline__ void make_leaf(const float *__restrict__ V, int64_t nv, const int32_t *__restrict__ F,
                                          const int32_t *__restrict__ ids, int n, int k, Tri *__restrict__ tris,
                                          float *lo, float *hi) {
    int t = ids[k];
    const bool t_ok = t >= 0 && t < n;  // always true for a correct sort; guards the loads below
    if (!t_ok)
        t = 0;
    const int32_t i0 = F[3 * (int64_t)t], i1 = F[3 * (int64_t)t + 1], i2 = F[3 * (int64_t)t + 2];
    Tri tri;
    if (!t_ok || i0 < 0 || i1 < 0 || i2 < 0 || i0 >= nv || i1 >= nv || i2 >= nv) {
        tri.a = make_float4(NAN, NAN, NAN, __int_as_float(t));
        tri.e1 = make_float4(NAN, NAN, NAN, 0.0f);
        tri.e2 = make_float4(NAN, NAN, NAN, 0.0f);
        for (int d = 0; d < 3; ++d) {
            lo[d] = INFINITY;
            hi[d] = -INFINITY;
        }
    } else {
        float A[3], B[3], C[3];
        for (int d = 0; d < 3; ++d) {
            A[d] = V[3 * (int64_t)i0 + d];
            B[d] = V[3 * (int64_t)i1 + d];
            C[d] = V[3 * (int64_t)i2 + d];
            lo[d] = fminf(A[d], fminf(B[d], C[d]));
            hi[d] = fmaxf(A[d], fmaxf(B[d], C[d]));
        }
        tri.a = make_float4(A[0], A[1], A[2], __int_as_float(t));
        tri.e1 = make_float4(B[0] - A[0], B[1] - A[1], B[2] - A[2], 0.0f);
        tri.e2 = make_float4(C[0] - A[0], C[1] - A[1], C[2] - A[2], 0.0f);
    }
    tris[k] = tri;
}

// A tile in LDS: its internal nodes at their index minus the first leaf's.
// Child references: a local node, or kLeafBit and a local leaf; parents: a
// local node, kOutside for the tile root's.
constexpr int kLeafBit = 0x8000, kOutside = 0xffff;
struct BoxTile {
    float box[kBoxTile][2][6];  // both children's boxes: lo xyz, hi xyz
    int arrived[kBoxTile];
    uint16_t left[kBoxTile], parent[kBoxTile];
};

// One workgroup per listed tile (a subtree of at most kBoxTile leaves, sorted
// positions [a, b]).  Every internal node of the tile lies in [a, b], so the
// whole tile is in LDS: its references are loaded in one step, lane j then
// takes leaf a + j, writes its triangle and climbs with arrival counters and
// child boxes in LDS; the lane completing the tile root hands its box to the
// root's parent.  (Parents and references read from L2 at every level of the
// climb: 19.7 us at 32,258 triangles, against 16.6.)
__global__ __launch_bounds__(kBoxTile) void k_leaves_subtree(const float *__restrict__ V, int64_t nv,
                                                            const int32_t *__restrict__ F,
                                                            const int32_t *__restrict__ ids, int n,
                                                            Tri *__restrict__ tris, Node *nodes,
                                                            const int32_t *__restrict__ parent, int32_t *counters,
                                                            const int32_t *__restrict__ tiles,
                                                            const int32_t *__restrict__ n_tiles) {
    __shared__ BoxTile T;
    const int tid = threadIdx.x;
    const int total = *n_tiles;
    for (int e = blockIdx.x; e < total; e += gridDim.x) {
        const int c = tiles[e];
        int a, b;
        if (c < 0) {
            a = b = ~c;
        } else {
            const int4 r = nodes[c].refs;
            a = r.z;
            b = r.w;
        }
        const bool ok = a >= 0 && b < n && b - a < kBoxTile;  // always, for a tile the radix-tree kernel listed
        // a subtree over [a, b] rooted at a holds the internal nodes [a, b - 1],
        // rooted at b those of [a + 1, b]
        const int base = c == a ? a : a + 1, g = a + tid;
        T.arrived[tid] = 0;
        if (ok && c >= 0 && g >= base && g < base + b - a) {
            const int l = nodes[g].refs.x;
            T.left[tid] = (uint16_t)(l >= 0 ? l - a : kLeafBit | (~l - a));
            T.parent[tid] = (uint16_t)(g == c ? kOutside : parent[g] - a);
        }
        const int k = a + tid;
        const bool mine = ok && k <= b;
        float lo[3], hi[3];
        if (mine)
            make_leaf(V, nv, F, ids, n, k, tris, lo, hi);
        int p = mine && n >= 2 ? parent[(n - 1) + k] : -1;
        __syncthreads();
        if (mine && c < 0) {
            // a one-leaf tile: its box goes straight to the parent
            if (p >= 0 && p < n - 1)
                store_child_box(nodes + p, nodes[p].refs.x == ~k, lo, hi);
        } else if (mine) {
            int self = kLeafBit | tid, j = p - a;
            // a radix tree is at most 97 levels deep; the bound only guards the loop
            for (int level = 0; j >= 0 && j < kBoxTile && level < kDeepStack; ++level) {
                const int side = T.left[j] == self ? 0 : 1;
                store_child_box(nodes + a + j, side == 0, lo, hi);
                float *own = T.box[j][side];
                for (int d = 0; d < 3; ++d) {
                    own[d] = lo[d];
                    own[3 + d] = hi[d];
                }
                __threadfence_block();
                if (atomicAdd(&T.arrived[j], 1) == 0)
                    break;  // the sibling subtree is not finished; its last lane continues
                __threadfence_block();
                const float *other = T.box[j][side ^ 1];
                for (int d = 0; d < 3; ++d) {
                    lo[d] = fminf(lo[d], other[d]);
                    hi[d] = fmaxf(hi[d], other[3 + d]);
                }
                counters[a + j] = 2;
                const int up = T.parent[j];
                if (up == kOutside) {
                    const int q = parent[c];
                    if (q >= 0 && q < n - 1)
                        store_child_box(nodes + q, nodes[q].refs.x == c, lo, hi);
                    break;
                }
                self = j;
                j = up;
            }
        }
        __syncthreads();  // LDS is reused by the next tile
    }
}

// One workgroup finishes the nodes above the tiles (every node with more than
// kBoxTile leaves).  Each listed tile is an arrival at its parent; the second
// arrival merges the two child boxes (written by the tile's workgroup, or by
// this one before its release) and climbs on: about log2(N_t / kBoxTile) levels.
// (A build that restructures its tiles has a workgroup of that launch do it.)
__global__ __launch_bounds__(1024) void k_boxes_top(Node *nodes, const int32_t *__restrict__ parent,
                                                    int32_t *counters, const int32_t *__restrict__ tiles,
                                                    const int32_t *__restrict__ n_tiles, int n) {
    boxes_above_tiles(nodes, parent, counters, tiles, *n_tiles, n);
}

// ------------------------------------------ 5'. agglomerative single pass
// The same binary radix tree, built bottom-up in one pass (Apetrei 2014,
// "Fast and simple agglomerative LBVH construction"; the numbering the paper's
// Case Study 1 dump shows): a lane per leaf climbs; a node covering [l, r]
// joins the neighbour across the boundary with the longer common prefix, so
// its parent is internal node r (it is the left child) or l - 1 (the right
// child) -- internal nodes are numbered by their split position.  The first
// child to reach a parent leaves its far bound in other[p] and stops; the
// second learns the parent's range from the exchange, merges the boxes and
// climbs on.  Every step is a cross-workgroup exchange at agent scope.
template <typename K>
__global__ __launch_bounds__(256) void k_agglomerate(const K *__restrict__ keys, const float *__restrict__ V,
                                                     int64_t nv, const int32_t *__restrict__ F,
                                                     const int32_t *__restrict__ ids, int n, Tri *__restrict__ tris,
                                                     Node *nodes, int32_t *__restrict__ parent, int32_t *counters,
                                                     int32_t *other, int32_t *__restrict__ root_out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n)
        return;
    float lo[3], hi[3];
    make_leaf(V, nv, F, ids, n, k, tris, lo, hi);
    if (n < 2) {
        *root_out = ~0;
        return;
    }
    auto delta = [&](int i) { return prefix(keys, n, i, keys[i], i + 1); };  // boundary between i and i + 1
    int l = k, r = k, self = ~k;
    for (int level = 0; level < kDeepStack; ++level) {
        const bool left_child = l == 0 || (r != n - 1 && delta(r) > delta(l - 1));
        const int p = left_child ? r : l - 1;
        Node *node = nodes + p;
        store_child_box(node, left_child, lo, hi);
        if (left_child)
            node->refs.x = self;
        else
            node->refs.y = self;
        parent[self >= 0 ? self : (n - 1) + ~self] = p;
        const int prev = __hip_atomic_exchange(other + p, left_child ? l : r, __ATOMIC_ACQ_REL,
                                               __HIP_MEMORY_SCOPE_AGENT);
        if (prev < 0)
            return;  // the sibling is not finished; its lane continues
        const int pl = left_child ? l : prev, pr = left_child ? prev : r;
        const float4 xy = left_child ? node->xy_right : node->xy_left;
        const float2 z = left_child ? *reinterpret_cast<const float2 *>(&node->z_both.z)
                                    : *reinterpret_cast<const float2 *>(&node->z_both.x);
        lo[0] = fminf(lo[0], xy.x);
        hi[0] = fmaxf(hi[0], xy.y);
        lo[1] = fminf(lo[1], xy.z);
        hi[1] = fmaxf(hi[1], xy.w);
        lo[2] = fminf(lo[2], z.x);
        hi[2] = fmaxf(hi[2], z.y);
        node->refs.z = pl;
        node->refs.w = pr;
        counters[p] = 2;
        l = pl;
        r = pr;
        self = p;
        if (l == 0 && r == n - 1) {
            parent[p] = -1;
            *root_out = p;
            return;
        }
    }
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = v;
}

__global__ void k_zero_i32(int32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = 0;
}

inline int blocks_for(int64_t n, int threads) { return (int)((n + threads - 1) / threads); }

// Where a sort of n pairs keeps what (in its scratch).
template <typename K>
struct SortArea {
    K *keys;        // ping-pong copies
    int32_t *ids;
    int ntiles;
    uint32_t *hist;     // digit-major, three histograms in turn for one-launch passes
    uint32_t *partial;  // digit totals of a large sort
    SortArea(void *tmp, int64_t n)
        : keys(static_cast<K *>(tmp)), ids(reinterpret_cast<int32_t *>(keys + n)), ntiles(blocks_for(n, kSortTile)),
          hist(reinterpret_cast<uint32_t *>(ids + n)), partial(hist + (int64_t)kRadix * ntiles) {}
    bool small() const { return ntiles <= kSmallSortTiles; }
    uint32_t *clear() const { return small() ? hist + (int64_t)kRadix * ntiles : nullptr; }
};

// Stable LSD passes over the pairs, with 8-bit digits.  An even number of
// passes sorts (keys, ids) in place; with an odd one (the batched form's 36-bit
// keys) the pairs start in the scratch copies.  The first pass's tile counts
// are in the scratch already (put_hist).  Up to kSmallSortTiles tiles a pass is
// one launch; above that, a histogram, a scan of each digit's row and a
// scatter.
template <typename K>
void sort_passes(K *keys, int32_t *ids, void *tmp, int64_t n, int key_bits, hipStream_t s) {
    if (n <= 1)
        return;  // nothing to order
    const SortArea<K> A(tmp, n);
    const bool odd = ((key_bits + 7) / 8) & 1;
    K *src_k = odd ? A.keys : keys, *dst_k = odd ? keys : A.keys;
    int32_t *src_i = odd ? A.ids : ids, *dst_i = odd ? ids : A.ids;
    const int64_t hl = (int64_t)kRadix * A.ntiles;
    // three histograms in turn: read by this pass, added to for the next,
    // cleared for the one after
    uint32_t *H[3] = {A.hist, A.hist + hl, A.hist + 2 * hl};
    for (int shift = 0, pass = 0; shift < key_bits; shift += 8, ++pass) {
        if (A.small()) {
            k_sort_pass_small<K><<<A.ntiles, kSortThreads, 0, s>>>(
                src_k, src_i, dst_k, dst_i, n, shift, A.ntiles, H[pass % 3],
                shift + 8 < key_bits ? H[(pass + 1) % 3] : nullptr, H[(pass + 2) % 3]);
        } else {
            if (pass > 0)
                k_sort_hist<K><<<A.ntiles, kSortThreads, 0, s>>>(src_k, n, shift, A.ntiles, A.hist, nullptr);
            k_scan_rows<<<kRadix, 1024, 0, s>>>(A.hist, A.ntiles, A.partial);
            k_sort_scatter<K><<<A.ntiles, kSortThreads, 0, s>>>(src_k, src_i, dst_k, dst_i, n, shift, A.ntiles, A.hist,
                                                                 A.partial);
        }
        K *tk = src_k; src_k = dst_k; dst_k = tk;
        int32_t *ti = src_i; src_i = dst_i; dst_i = ti;
    }
}

size_t pass_tmp_bytes(int64_t n, size_t key_bytes) {
    const int64_t ntiles = (n + kSortTile - 1) / kSortTile;
    const int64_t hists = ntiles <= kSmallSortTiles ? 3 : 1;  // one-launch passes keep three
    return key_bytes * n + 4 * n + 4 * (size_t)kRadix * ntiles * hists + 4 * 1024 + 256;
}

// Sort (key, id), build the radix tree and fill the boxes bottom-up, for keys
// and ids where sort_passes takes them and their first digit counted.  roots
// (NULL for one mesh) receives each mesh's subtree root.
template <typename K>
hipError_t build_from_keys(MeshDev &m, int key_bits, int32_t *roots, hipStream_t s) {
    const int64_t nt = m.nt;
    K *keys = static_cast<K *>(m.keys);
    sort_passes<K>(keys, m.ids, m.sort_tmp, nt, key_bits, s);  // sorted pairs back in (keys, ids)
    if (m.algorithm == 1) {
        // the sort's scratch is free again: the exchange slots
        int32_t *other = static_cast<int32_t *>(m.sort_tmp);
        if (nt >= 2) {
            k_fill_i32<<<blocks_for(nt - 1, 256), 256, 0, s>>>(other, nt - 1, -1);
            k_zero_i32<<<blocks_for(nt - 1, 256), 256, 0, s>>>(m.counters, (int)(nt - 1));
        }
        k_agglomerate<K><<<blocks_for(nt, 256), 256, 0, s>>>(keys, m.V, m.nv, m.F, m.ids, (int)nt, m.tris, m.nodes,
                                                            m.parent, m.counters, other, m.flags + 1);
        return hipGetLastError();
    }
    // the sort's scratch is free again: the list of bottom-up tiles
    const BuildLists L = build_lists(m);
    int32_t *n_tiles = L.n_tiles;
    int32_t *tiles = L.tiles;
    if (nt >= 2)
        k_radix_tree<K><<<blocks_for(nt - 1, 256), 256, 0, s>>>(keys, (int)nt, m.nodes, m.parent, m.counters, tiles,
                                                                n_tiles, L.flag, roots);
    else
        k_single_tile<K><<<1, 1, 0, s>>>(tiles, n_tiles, keys, roots);
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t grid = nt < 2 * (int64_t)cus ? nt : 2 * (int64_t)cus;  // tiles are taken in a loop
    k_leaves_subtree<<<(int)grid, kBoxTile, 0, s>>>(m.V, m.nv, m.F, m.ids, (int)nt, m.tris, m.nodes, m.parent,
                                                    m.counters, tiles, n_tiles);
    if (nt > kBoxTile && m.algorithm != 2)
        k_boxes_top<<<1, 1024, 0, s>>>(m.nodes, m.parent, m.counters, tiles, n_tiles, (int)nt);
    return hipGetLastError();
}

template <typename K>
hipError_t build_typed(MeshDev &m, const int32_t *F_in, int parts, hipStream_t s) {
    const int64_t nt = m.nt;
    const SortArea<K> A(m.sort_tmp, nt);
    k_morton<K><<<A.ntiles, kSortThreads, 0, s>>>(m.V, m.nv, F_in, nt, m.partial, parts, m.bounds,
                                                  static_cast<K *>(m.keys), m.ids, m.flags, m.F, A.ntiles, A.hist,
                                                  A.clear());
    return build_from_keys<K>(m, m.morton_bits, nullptr, s);
}

}  // namespace

hipError_t launch_build_batch(MeshDev &m, const BatchDev &b, hipStream_t s) {
    // five 8-bit passes: the pairs start in the sort's scratch (a single pair
    // is not sorted and starts in place)
    constexpr int key_bits = kBatchMortonBits + 6;
    const SortArea<uint64_t> A(m.sort_tmp, m.nt);
    uint64_t *keys = m.nt > 1 ? A.keys : static_cast<uint64_t *>(m.keys);
    int32_t *ids = m.nt > 1 ? A.ids : m.ids;
    k_morton_batch<<<A.ntiles, kSortThreads, 0, s>>>(m.V, m.F, b.tri_mesh, m.nt, b.key_bounds, b.M, b.mesh_bounds,
                                                     m.bounds, keys, ids, A.ntiles, A.hist, A.clear());
    return build_from_keys<uint64_t>(m, key_bits, b.roots, s);
}

size_t sort_tmp_bytes(int64_t nt, int morton_bits) {
    const size_t kb = morton_bits > 32 ? 8 : 4;
    const size_t sort = pass_tmp_bytes(nt, kb);
    const size_t lists = build_lists_bytes(nt);  // lists kept after the sort
    return sort > lists ? sort : lists;
}

size_t sort_u32_tmp_bytes(int64_t n) { return pass_tmp_bytes(n, 4); }

hipError_t scan_u32_exclusive(uint32_t *a, int64_t len, uint32_t *partial, hipStream_t s) {
    if (len > 0)
        scan_hist(a, len, partial, s);
    return hipGetLastError();
}

hipError_t sort_u32_pairs(uint32_t *keys, int32_t *ids, void *tmp, int64_t n, hipStream_t s) {
    if (n > 1) {
        const SortArea<uint32_t> A(tmp, n);
        k_sort_hist<uint32_t><<<A.ntiles, kSortThreads, 0, s>>>(keys, n, 0, A.ntiles, A.hist, A.clear());
        sort_passes<uint32_t>(keys, ids, tmp, n, 32, s);  // four passes
    }
    return hipGetLastError();
}

hipError_t launch_build(MeshDev &m, const float *V_in, const int32_t *F_in, hipStream_t s, size_t) {
    // the first kernels also copy the caller's vertices and triangles into the mesh
    const int64_t want = (m.nv + 1023) / 1024;
    const int parts = (int)(want < 1 ? 1 : (want < kBoundsParts ? want : kBoundsParts));
    k_mesh_bounds_part<<<parts, 1024, 0, s>>>(V_in, m.nv, m.partial, m.V, m.flags);
    hipError_t e = m.morton_bits > 32 ? build_typed<uint64_t>(m, F_in, parts, s)
                                      : build_typed<uint32_t>(m, F_in, parts, s);
    if (e == hipSuccess && m.algorithm == 2 && m.nt >= kRestructureMin)
        e = launch_restructure(m, kRestructureRounds, s);
    if (e == hipSuccess && m.algorithm != 1 && m.nodes4)
        e = launch_collapse(m, s);
    return e;
}

}  // namespace rsi
