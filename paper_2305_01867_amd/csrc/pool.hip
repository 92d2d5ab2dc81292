// pool.hip -- the first pass in pool form (pool.h): calls with too few
// segments to fill the GPU with a lane each, and the count mode.
#include "pool.h"

namespace rsi {
namespace {

// A launch's shape: segments in flight per wave, node entries per wave, leaves
// tested at a time.
struct PoolShape {
    int slots, cap, leaves;
};
// Node entries per wave (64 segments in flight keep a few hundred).  Count
// mode, whose lists of hits take 5.9 KB a wave: 384, so that 16 waves and part
// of the tree's top fit (4e6 segments at the paper's scale: 12 waves of 1024
// entries 1,990 us, 16 of 512 1,890; with the top 12 / 512 1,935, 16 / 512
// 1,765, 16 / 384 1,741, 16 / 256, which run out of entries, 2,145).
template <int MODE>
constexpr int kPoolNodes = MODE == MODE_COUNT ? 384 : 1024;
// Resident waves per CU, what the registers allow.
constexpr int kPoolWavesPerCU = 16;
// From this many segments per CU on the tree's top is kept in LDS: at least
// twelve for each wave, whose steps then spend less on fetches than the copy of
// 20 to 64 KB costs (522,242 triangles, nearest hit: 1e5 segments 136 -> 112 us,
// 3.9e5 357 -> 277; 7,938 triangles: 5e4 56 -> 53, 3.9e5 186 -> 171, but 1e4 39 -> 41).
constexpr int kPoolTopMin = 192;

// Threads of a workgroup.  With the tree's top in LDS (TOP) one workgroup has
// all of a CU's waves, so there is one copy of it.
template <bool TOP>
constexpr int kPoolBlock = TOP ? 64 * kPoolWavesPerCU : 256;

// Each wave owns a contiguous range of segments; with more than twice as many
// as are in flight at once the last 1/kPoolTailDiv of them is a pool of
// kPoolChunk-segment chunks that waves take in turn once their own share is
// handed out.  (With fewer, a chunk would be a second full round for the waves
// that get one: 3e5 segments at the paper's scale 142 us so, 104 without.  At
// 4e6 the count mode takes 1,877 us without chunks, 1,895 with chunks of 16 and
// 1,750 with these.)
constexpr int64_t kPoolTailDiv = 6;
constexpr int kPoolChunk = 64;

// The root and first triangle of a segment's mesh (batched form).
__device__ __forceinline__ void mesh_of(const TravParams &p, int64_t ray, int &root, int &toff) {
    root = 0;
    toff = 0;
    if (p.items) {
        const int m = mesh_of_segment(p.ray_off, p.n_meshes, ray);
        root = p.mesh_root4[m];
        toff = p.mesh_toff[m];
    }
}

template <int MODE, bool CERT, bool TOP>
__global__ __launch_bounds__(kPoolBlock<TOP>, kPoolWavesPerCU / 4) void k_pool(TravParams p, PoolShape sh) {
    constexpr int kWords = pool_words<MODE, CERT>(64, kPoolNodes<MODE>);
    constexpr int kBlock = kPoolBlock<TOP>;
    uint32_t *words;
    int top_n = 0;
    if constexpr (TOP) {
        extern __shared__ float4 lds_dyn[];  // the tree's top, then the waves' words
        if ((uint32_t)(uintptr_t)(LdsInt)(int *)lds_dyn == 0)  // (no static LDS: so it is)
            top_n = p.top_lds;
        const float4 *src = reinterpret_cast<const float4 *>(p.top4);
        for (int i = threadIdx.x; i < 8 * top_n; i += kBlock)
            lds_dyn[i] = src[i];
        __syncthreads();
        words = reinterpret_cast<uint32_t *>(lds_dyn + 8 * p.top_lds);
    } else {
        __shared__ uint32_t fixed[kWords * (kBlock / 64)];
        words = fixed;
    }
    const int lane = threadIdx.x & 63;
    const float scale = p.bounds[6];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    const int64_t wave_id = (int64_t)blockIdx.x * (kBlock / 64) + wave;
    const int64_t n_static = p.n <= 2 * waves * sh.slots ? p.n : p.n - p.n / kPoolTailDiv;
    int64_t cursor = n_static * wave_id / waves;
    int64_t range_end = n_static * (wave_id + 1) / waves;
    bool chunks_left = n_static < p.n;

    Pool<MODE, CERT, false> pool;
    pool.init(p, words + wave * kWords, sh.slots, sh.cap);
    pool.top_lds = top_n;
    PoolSegment<MODE, CERT> s;
    s.ray = -1;
    s.toff = 0;
    s.reset();
    s.o = s.d = s.inv = s.nn = s.nf = make_float3(0.0f, 0.0f, 0.0f);
    uint32_t redecided = 0;

    for (;;) {
        // ---- new segments for the slots without one
        const bool idle = s.ray < 0 && lane < sh.slots;
        const uint64_t idle_m = __ballot(idle);
        if (chunks_left && cursor >= range_end && idle_m) {
            uint32_t k = 0;
            if (lane == 0)
                k = atomicAdd(p.next_ray, 1u);
            k = __builtin_amdgcn_readfirstlane(k);
            const int64_t start = n_static + (int64_t)k * kPoolChunk;
            if (start < p.n) {
                cursor = start;
                range_end = start + kPoolChunk < p.n ? start + kPoolChunk : p.n;
            } else {
                chunks_left = false;
            }
        }
        if (cursor < range_end && idle_m) {
            const int64_t at = cursor + lane_rank(idle_m);
            bool fresh = idle && at < range_end;
            int root = 0;
            if (fresh) {
                s.ray = p.order ? p.order[at] : (int)at;
                s.reset();
                mesh_of(p, s.ray, root, s.toff);
                Ray r;
                if (!setup_ray(p.from, p.to, s.ray, scale, r)) {
                    if (CERT)
                        enqueue(p, s.ray, 0);  // finished by the second pass
                    else
                        write_out(p.out, s.ray, MODE, -1, 0.0f, 0.0f, 0.0f);
                    s.ray = -1;
                    fresh = false;
                } else {
                    s.set(r);
                    if (MODE == MODE_COUNT)
                        pool.mail[lane] = 0;
                }
            }
            cursor += __popcll(idle_m);
            cursor = cursor < range_end ? cursor : range_end;
            pool.push(fresh && root != kEmptyChild, root, (uint32_t)lane << kPoolRefBits);
            wave_lds_fence();
        }
        const bool more = cursor < range_end || chunks_left;
        if (!__ballot(s.ray >= 0)) {
            if (!more)
                break;
            continue;
        }

        // while there are more segments, down to half as many entries as slots
        pool.run(p, s, more ? sh.slots / 2 : 0, sh.leaves);

        // ---- results of the segments with nothing left
        const bool pending = pool.pending();
        const bool done = s.ray >= 0 && !pending;
        const uint64_t done_m = __ballot(done);
        if (done) {
            const bool lost = (pool.lost >> lane) & 1ull;
            if (lost && !(MODE == MODE_BOOL && s.best_id >= 0)) {
                enqueue(p, s.ray, 1);
            } else if (MODE == MODE_COUNT) {
                const int total = pool.mail[lane];
                const bool full = total >= kPoolFull;
                const int kept = full ? kCountSlots<CERT> : total;
                const float *l = pool.list(lane);
                // plain: distinct values; certified: disjoint intervals hold
                // distinct values, intervals that meet are counted exactly by
                // the second pass
                int distinct = 0;
                bool meet = (total & kPoolMeet) != 0;
                for (int a = 0; a < kept; ++a) {
                    bool first = true;
                    for (int b = 0; b < a; ++b)
                        if (CERT ? !(l[kCountSlots<CERT> + a] < l[b] || l[a] > l[kCountSlots<CERT> + b])
                                 : l[a] == l[b])
                            first = false;
                    distinct += first ? 1 : 0;
                    meet = meet || !first;
                }
                if (CERT && meet)
                    enqueue(p, s.ray, 0);
                else if (full)
                    enqueue(p, s.ray, 3);
                else
                    write_count(p.out, s.ray, distinct);
            } else {
                if (CERT && s.redecided > 0)
                    ++redecided;
                const int id = MODE == MODE_BOOL ? s.best_id : (s.best_id >= 0 ? s.best_id - s.toff : -1);
                if (CERT && MODE == MODE_BARY && s.best_id >= 0) {
                    if (p.bary_after) {  // (u, v, t) after both passes, a lane per segment
                        if (p.out.hit)
                            p.out.hit[s.ray] = 1;
                        p.out.id[s.ray] = id;
                    } else {
                        const float *o = p.from + 3 * (int64_t)s.ray, *e = p.to + 3 * (int64_t)s.ray;
                        const MT64 h = mt64(o[0], o[1], o[2], e[0], e[1], e[2], p.V, p.F, s.best_id);
                        write_out(p.out, s.ray, MODE, id, (float)h.u, (float)h.v, (float)h.t);
                    }
                } else {
                    write_out(p.out, s.ray, MODE, id, s.best_u, s.best_v, s.best_t);
                }
            }
            s.ray = -1;
        }
        pool.lost &= ~done_m;
        if (more && !__ballot(s.ray < 0 && lane < sh.slots)) {
            // every slot waits on its last entries: go on with those
            if (pool.ls > 0)
                pool.leaf_step(p, s);
            else
                pool.node_step(p, s);
        }
    }
    if (MODE != MODE_COUNT && CERT) {
        // segments with a pair decided in binary64, one atomic per wave
        for (int off = 32; off > 0; off >>= 1)
            redecided += __shfl_xor(redecided, off);
        if (lane == 0 && redecided)
            atomicAdd(p.counters, (unsigned long long)redecided);
    }
}

template <int MODE, bool CERT, bool TOP>
void launch_shape(const TravParams &p, int cus, hipStream_t s) {
    constexpr int kBlock = kPoolBlock<TOP>, kWaves = kBlock / 64;
    constexpr size_t kBytes = TOP ? (size_t)pool_words<MODE, CERT>(64, kPoolNodes<MODE>) * 4 * kWaves : 0;
    TravParams q = p;
    q.top_lds = 0;
    size_t lds = 0;
    if constexpr (TOP) {
        static_assert(kBytes + sizeof(Node4) < 160 * 1024, "the waves' words leave room for nodes");
        constexpr int kRoom = (int)((160 * 1024 - kBytes) / sizeof(Node4));
        q.top_lds = kRoom < kTopSlots ? kRoom : kTopSlots;
        lds = kBytes + (size_t)q.top_lds * sizeof(Node4);
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_pool<MODE, CERT, TOP>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    }
    int per_cu = 0;
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(&k_pool<MODE, CERT, TOP>), kBlock, lds);
    per_cu = per_cu < kPoolWavesPerCU / kWaves ? per_cu : kPoolWavesPerCU / kWaves;
    per_cu = per_cu < 1 ? 1 : per_cu;
    const int64_t resident = (int64_t)cus * per_cu;
    // few segments: as few per wave as fill the resident waves (so the lanes
    // of a wave share them), and leaves tested earlier, as fewer come up
    const int64_t share = (p.n + resident * kWaves - 1) / (resident * kWaves);
    PoolShape sh;
    sh.slots = (int)(share < 64 ? share : 64);
    sh.cap = p.pool_cap < kPoolNodes<MODE> ? p.pool_cap : kPoolNodes<MODE>;
    sh.leaves = sh.slots <= 32 ? 32 : 64;
    const int64_t per_block = (int64_t)sh.slots * kWaves;
    const int64_t want = (p.n + per_block - 1) / per_block;
    k_pool<MODE, CERT, TOP><<<(int)(want < resident ? want : resident), kBlock, lds, s>>>(q, sh);
}

template <int MODE, bool CERT>
void launch(const TravParams &p, hipStream_t s) {
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (p.n >= (int64_t)cus * kPoolTopMin)
        launch_shape<MODE, CERT, true>(p, cus, s);
    else
        launch_shape<MODE, CERT, false>(p, cus, s);
}

}  // namespace

void launch_pool(const TravParams &p, int mode, bool cert, hipStream_t s) {
    if (mode == MODE_BOOL)
        cert ? launch<MODE_BOOL, true>(p, s) : launch<MODE_BOOL, false>(p, s);
    else if (mode == MODE_FIRST)
        cert ? launch<MODE_FIRST, true>(p, s) : launch<MODE_FIRST, false>(p, s);
    else if (mode == MODE_BARY)
        cert ? launch<MODE_BARY, true>(p, s) : launch<MODE_BARY, false>(p, s);
    else
        cert ? launch<MODE_COUNT, true>(p, s) : launch<MODE_COUNT, false>(p, s);
}

}  // namespace rsi
