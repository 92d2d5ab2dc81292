// wide.hip -- collapse of the binary BVH into a 4-wide one on gfx950.
//
// The traversal's cost per node is one dependent fetch from L2 plus the box
// arithmetic; a 4-wide node halves the number of dependent fetches per
// segment (each tests four children at once) and fits one 128-byte L2 line.
// The collapse keeps the binary tree's boxes and leaves: a 4-wide node starts
// at a binary internal node r and takes its two children, then opens the
// child of largest surface area twice (greedy, as in the usual collapse of
// binary BVHs into wide ones), so it covers exactly the leaves of r.  It is
// stored at index r of the 4-wide array, so no renumbering is needed.
//
// Every binary node gets its 4-wide node, a lane each, whether or not a
// 4-wide path from the root leads to it (about half are reached).  Following
// the paths instead, breadth-first per tile and above the tiles, writes half
// as much but pays one node's latency per level: 16 us at 32,258 triangles, 42
// at 522,242 and 120 at 1.81 million, against 6, 21 and 79.  It
// also made every tile root start a 4-wide node; now only the nodes flagged by
// the caller do (mesh roots, the proposal's frontier).
#include <cstddef>

#include "rsi_internal.h"

namespace rsi {
namespace {

constexpr int kFrontierFlag = 2;

__global__ void k_clear_flags(int32_t *flag, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        flag[i] = 0;
}

__device__ __forceinline__ float half_area6(const float *b) {
    const float dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
    return dx * dy + dy * dz + dz * dx;
}

// Reference and box (lo xyz, hi xyz) of one child (side 0 or 1) of a node.
__device__ __forceinline__ int child_ref(const Node *__restrict__ nodes, int r, int side) {
    return (&nodes[r].refs.x)[side];
}
__device__ __forceinline__ void child_box(const Node *__restrict__ nodes, int r, int side, float b[6]) {
    const float4 xy = (&nodes[r].xy_left)[side];
    const float2 z = reinterpret_cast<const float2 *>(&nodes[r].z_both)[side];
    b[0] = xy.x, b[1] = xy.z, b[2] = z.x, b[3] = xy.y, b[4] = xy.w, b[5] = z.y;
}

// The 4-wide node at each binary internal node.  A child whose flags share a
// bit with no_open (flag may be NULL for no_open = 0) is not opened: it starts
// a 4-wide node of its own.  Where each child's box lies (a node and a side) is
// kept through the two openings, and the boxes are fetched at the end.  A
// wave's 64 nodes go out through LDS, 1 KB a store (swizzled, so that neither
// side conflicts).
__global__ __launch_bounds__(256) void k_collapse(const Node *__restrict__ nodes, int n_internal,
                                                  const int32_t *__restrict__ flag, int no_open,
                                                  Node4 *__restrict__ nodes4) {
    __shared__ float4 out[256 / 64][64 * 8];
    const int lane = threadIdx.x & 63;
    float4 *const mine = out[threadIdx.x >> 6];
    const int r_own = blockIdx.x * blockDim.x + threadIdx.x;
    const int r = r_own < n_internal ? r_own : n_internal - 1;
    auto area_of = [&](int n, int s) {
        float b[6];
        child_box(nodes, n, s, b);
        return half_area6(b);
    };
    int at[4] = {r, r, r, r}, side[4] = {0, 1, 0, 0};
    int ref[4] = {child_ref(nodes, r, 0), child_ref(nodes, r, 1), kEmptyChild, kEmptyChild};
    float area[4] = {area_of(r, 0), area_of(r, 1), -1.0f, -1.0f};
    int m = 2;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        int best = -1, c = 0;
        float best_a = -1.0f;
#pragma unroll
        for (int i = 0; i < 2 + e; ++i) {
            const bool open = i < m && ref[i] >= 0 && ref[i] < n_internal && !(no_open && (flag[ref[i]] & no_open));
            if (open && area[i] > best_a) {
                best_a = area[i];
                best = i;
                c = ref[i];
            }
        }
        if (best < 0)
            break;
        const int l = child_ref(nodes, c, 0), rr = child_ref(nodes, c, 1);
        const float la = area_of(c, 0), ra = area_of(c, 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool first = i == best, second = i == m;
            at[i] = first || second ? c : at[i];
            side[i] = first ? 0 : (second ? 1 : side[i]);
            ref[i] = first ? l : (second ? rr : ref[i]);
            area[i] = first ? la : (second ? ra : area[i]);
        }
        ++m;
    }
    float b[4][6];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        child_box(nodes, at[i], side[i], b[i]);
#pragma unroll
        for (int a = 0; a < 6; ++a)
            b[i][a] = i < m ? b[i][a] : INFINITY;
    }
    // the node's eight 16-byte words in the order of Node4
    auto put = [&](int k, float4 v) { mine[8 * lane + (k ^ (lane & 7))] = v; };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        put(2 * a, make_float4(b[0][a], b[1][a], b[2][a], b[3][a]));
        put(2 * a + 1, make_float4(b[0][3 + a], b[1][3 + a], b[2][3 + a], b[3][3 + a]));
    }
    // internal children are named by binary index + kTopSlots (the top slots
    // are assigned afterwards)
    auto enc = [](int c) { return __int_as_float(c >= 0 ? c + kTopSlots : c); };
    put(6, make_float4(enc(ref[0]), enc(ref[1]), enc(ref[2]), enc(ref[3])));
    put(7, make_float4(__int_as_float(m), 0.0f, 0.0f, 0.0f));
    __syncthreads();
    const int first = r_own - lane;  // the wave's first node
    float4 *dst = reinterpret_cast<float4 *>(nodes4 + first);
    const int words = 8 * (n_internal - first < 64 ? n_internal - first : 64);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int w = 64 * k + lane, n = w >> 3;
        if (w < words)
            dst[w] = mine[8 * n + ((w & 7) ^ (n & 7))];
    }
}
static_assert(offsetof(Node4, hix) == 16 && offsetof(Node4, loy) == 32 && offsetof(Node4, loz) == 64 &&
                  offsetof(Node4, child) == 96,
              "the words' order");

// One workgroup of kTopSlots lanes: the first kTopSlots 4-wide nodes in
// breadth-first order from the nodes in bidx[0 .. n_roots), copied into top4
// with the references of children that also got a slot rewritten to that slot.
// Slots follow a block-wide prefix sum over each level, so the layout does not
// depend on thread timing.  A level costs one fetch of its nodes' references
// and two barriers; the boxes are copied at the end.  Returns the number of
// slots in use; bidx then holds the binary index of each slot's node.
struct TopLds {
    int bidx[kTopSlots];
    int4 child[kTopSlots];
    int wave_sum[kTopSlots / 64];
};
__device__ __forceinline__ int lay_out_top(TopLds &T, int n_roots, const Node4 *__restrict__ nodes4,
                                           Node4 *__restrict__ top4) {
    constexpr int kWaves = kTopSlots / 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int b0 = 0, b1 = n_roots;
    while (b0 < b1) {
        const int i = b0 + tid;  // a level has at most kTopSlots = blockDim nodes
        int4 child = make_int4(-1, -1, -1, -1);
        if (i < b1)
            child = nodes4[T.bidx[i]].child;
        const int cnt = (child.x >= 0) + (child.y >= 0) + (child.z >= 0) + (child.w >= 0);
        // inclusive prefix sum of cnt: within the wave by shuffles, then across waves
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off);
            incl += lane >= off ? t : 0;
        }
        if (lane == 63)
            T.wave_sum[w] = incl;
        __syncthreads();
        int total = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            const int x = T.wave_sum[k];
            incl += k < w ? x : 0;
            total += x;
        }
        if (i < b1) {
            int slot = b1 + incl - cnt;
            auto take = [&](int c) {
                if (c < 0)
                    return c;
                const int s = slot++;
                if (s < kTopSlots)
                    T.bidx[s] = c - kTopSlots;
                return s < kTopSlots ? s : c;
            };
            const int x = take(child.x), y = take(child.y), z = take(child.z), v = take(child.w);
            T.child[i] = make_int4(x, y, z, v);
        }
        __syncthreads();  // bidx of the next level written, wave_sum read
        b0 = b1;
        b1 = b1 + total < kTopSlots ? b1 + total : kTopSlots;
    }
    if (tid < b1) {
        const Node4 *nd = nodes4 + T.bidx[tid];
        Node4 *o = top4 + tid;
        o->lox = nd->lox;
        o->hix = nd->hix;
        o->loy = nd->loy;
        o->hiy = nd->hiy;
        o->loz = nd->loz;
        o->hiz = nd->hiz;
        o->child = T.child[tid];
        o->spare = nd->spare;
    }
    return b1;
}

// The whole tree's top, from node 0.  slot_bin (may be NULL) receives the
// binary index of the node in each slot, -1 for unused slots.
__device__ __forceinline__ void top_of_tree(TopLds &T, const Node4 *__restrict__ nodes4, Node4 *__restrict__ top4,
                                            int32_t *slot_bin) {
    const int tid = threadIdx.x;
    if (tid == 0)
        T.bidx[0] = 0;
    __syncthreads();
    const int used = lay_out_top(T, 1, nodes4, top4);
    if (slot_bin)
        slot_bin[tid] = tid < used ? T.bidx[tid] : -1;
}

__global__ __launch_bounds__(kTopSlots) void k_top_cache(const Node4 *__restrict__ nodes4, Node4 *__restrict__ top4,
                                                         int32_t *slot_bin) {
    __shared__ TopLds T;
    top_of_tree(T, nodes4, top4, slot_bin);
}

// The reference under which each bucket's frontier node appears in the
// 4-wide tree: its top slot if it has one, else binary index + kTopSlots;
// a leaf keeps its leaf reference.
// (The same for each mesh root of the batched form.)
// One workgroup of kTopSlots threads: the buckets' references are staged in
// LDS, then each slot claims the buckets whose node it holds (at most
// kTopSlots buckets or meshes).
__device__ __forceinline__ void bucket_refs(const int32_t *__restrict__ bucket_ref, int n_raw, const int32_t *slot_bin,
                                            int32_t *__restrict__ ref4) {
    __shared__ int ref[kTopSlots];  // each bucket's binary reference
    const int t = threadIdx.x;
    const int n = n_raw < kTopSlots ? n_raw : kTopSlots;
    const int c = t < n ? bucket_ref[t] : -1;
    ref[t] = c;
    if (t < n)
        ref4[t] = c >= 0 ? c + kTopSlots : c;  // by default the node itself (not in the top)
    __syncthreads();  // the defaults are written before any slot claims a bucket
    // slot t claims the buckets whose node it holds (each slot holds one node)
    const int mine = slot_bin[t];
    if (mine >= 0)
        for (int b = 0; b < n; ++b)
            if (ref[b] == mine)
                ref4[b] = t;
}

__global__ __launch_bounds__(kTopSlots) void k_bucket_ref4(const int32_t *__restrict__ bucket_ref,
                                                           const int32_t *__restrict__ n_buckets,
                                                           const int32_t *__restrict__ slot_bin,
                                                           int32_t *__restrict__ ref4) {
    bucket_refs(bucket_ref, *n_buckets, slot_bin, ref4);
}

// Batched form: the top of each item group's meshes, breadth-first from their
// roots (group g = blockIdx.x), and each mesh's root as a reference in it (a
// slot for the group's own meshes, the node index + kTopSlots or a leaf
// reference for the others).  The last workgroup does the same for the combined
// tree.
__global__ __launch_bounds__(kTopSlots) void k_top_cache_group(const Node4 *__restrict__ nodes4,
                                                               const int32_t *__restrict__ roots,
                                                               const uint64_t *__restrict__ group_meshes, int M,
                                                               Node4 *__restrict__ top4g,
                                                               int32_t *__restrict__ roots4g,
                                                               Node4 *__restrict__ combined, int32_t *slot_bin,
                                                               int32_t *roots4) {
    __shared__ TopLds T;
    __shared__ int root_slot[64];
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    if (g == (int)gridDim.x - 1) {
        top_of_tree(T, nodes4, combined, slot_bin);
        __threadfence_block();
        __syncthreads();
        bucket_refs(roots, M, slot_bin, roots4);
        return;
    }
    // the group's internal roots in mesh order take the first slots
    if (tid < 64) {
        const bool mine = tid < M && (group_meshes[g] >> tid & 1u) && roots[tid] >= 0;
        const uint64_t all = __ballot(mine);  // the whole wave votes: not inside a lane branch
        const int k = __popcll(all & (lane ? (~0ull >> (64 - lane)) : 0ull));
        root_slot[tid] = mine ? k : -1;
        if (mine)
            T.bidx[k] = roots[tid];
        if (lane == 0)
            T.wave_sum[0] = __popcll(all);
    }
    __syncthreads();
    const int n_roots = T.wave_sum[0];
    __syncthreads();
    lay_out_top(T, n_roots, nodes4, top4g + (int64_t)g * kTopSlots);
    if (tid < M) {
        const int r = roots[tid];
        const int sl = root_slot[tid];  // (at most 64 meshes)
        roots4g[(int64_t)g * 64 + tid] = sl >= 0 ? sl : (r >= 0 ? r + kTopSlots : r);
    }
}

__global__ void k_mark_frontier(const int32_t *__restrict__ bucket_ref, const int32_t *__restrict__ n_buckets,
                                int32_t *flag, int64_t n_internal) {
    const int b = threadIdx.x;
    if (b < *n_buckets) {
        const int c = bucket_ref[b];
        if (c >= 0 && c < n_internal)
            flag[c] |= kFrontierFlag;
    }
}

}  // namespace

static void collapse(const MeshDev &m, Node4 *nodes4, const int32_t *flag, int no_open, hipStream_t s) {
    const int n_internal = (int)(m.nt - 1);
    k_collapse<<<(n_internal + 255) / 256, 256, 0, s>>>(m.nodes, n_internal, flag, no_open, nodes4);
}

hipError_t launch_collapse(MeshDev &m, hipStream_t s) {
    if (m.nt < 2)
        return hipSuccess;  // one leaf: nothing to collapse
    collapse(m, m.nodes4, nullptr, 0, s);
    k_top_cache<<<1, kTopSlots, 0, s>>>(m.nodes4, m.top4, nullptr);
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        m.node_width = 4;
    return e;
}

hipError_t launch_collapse_proposal(const MeshDev &m, Proposal &pr, hipStream_t s) {
    if (m.nt < 2 || m.node_width != 4 || !pr.top4)
        return hipSuccess;
    const int64_t n_internal = m.nt - 1;
    const int blocks = (int)((n_internal + 255) / 256);
    k_clear_flags<<<blocks, 256, 0, s>>>(pr.wide_flag, n_internal);
    k_mark_frontier<<<1, kMlpOut, 0, s>>>(pr.bucket_ref, pr.dev_n_buckets, pr.wide_flag, n_internal);
    collapse(m, pr.top4 + kTopSlots, pr.wide_flag, kFrontierFlag, s);
    k_top_cache<<<1, kTopSlots, 0, s>>>(pr.top4 + kTopSlots, pr.top4, pr.slot_bin);
    k_bucket_ref4<<<1, kTopSlots, 0, s>>>(pr.bucket_ref, pr.dev_n_buckets, pr.slot_bin, pr.bucket_ref4);
    return hipGetLastError();
}

// Batched form: every mesh's subtree root starts a 4-wide node (never opened
// from above), so a segment starts at its mesh root's 4-wide node.
hipError_t launch_collapse_batch(MeshDev &m, BatchDev &b, hipStream_t s) {
    if (m.nt < 2) {
        m.node_width = 2;
        return hipSuccess;
    }
    collapse(m, m.nodes4, build_lists(m).flag, kMeshRootFlag, s);
    k_top_cache_group<<<kItemGroups + 1, kTopSlots, 0, s>>>(m.nodes4, b.roots, b.group_meshes, b.M, b.top4g, b.roots4g,
                                                            m.top4, b.slot_bin, b.roots4);
    const hipError_t e = hipGetLastError();
    m.node_width = e == hipSuccess ? 4 : 2;
    return e;
}

}  // namespace rsi
