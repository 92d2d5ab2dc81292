// traverse.hip -- tree search and Moller-Trumbore leaf tests on gfx950.
//
// Paper: Background -- a tree search gathers the candidate triangles of each
// segment and the Moller-Trumbore test (Moller & Trumbore 1997) decides; the
// operating modes boolean / barycentric; Epilogue -- binary32 can misjudge
// near-parallel rays, binary64 intermediates fix it.
//
// Pass 1 (k_traverse; calls with few segments and the intercept count: k_pool in
// pool.hip): one lane per segment, stack of pending subtrees in LDS (stack_depth
// entries per lane), binary32 arithmetic.  Of a node's children the nearer first;
// in boolean mode the one with the longer way through its box.
//   PLAIN      the binary32 predicates decide.
//   CERTIFIED  each predicate X comes with a proven bound B(X) on its distance
//              from the exact value and from the binary64 value; |X| > B(X)
//              fixes the sign of the binary64 result, so the pair is a sure
//              hit or a sure miss.  Otherwise the pair is "unsure" and the
//              lane decides it at once with the binary64 test in the
//              oracle's operation order (no contraction, correctly rounded
//              division).  Nearest-hit choice uses proven intervals around
//              the binary64 t, and the binary64 t themselves where two
//              intervals overlap.
// A segment whose path outgrows the LDS stack waits for its wave's end, where the
// wave's lanes share such segments (pool.h).  What finds no room there either, or
// outgrows a stack too small for that pool or over binary nodes, and in count
// mode a segment whose list of distinct t overflows or holds nearly equal ones,
// is appended to a queue and finished by pass 2 (k_finish): a deep private stack
// and, in CERTIFIED precision, the binary64 test on every candidate.
//
// Box test: the slab test on each child box widened by eta = 2^-20 max(|coord|)
// of the segment and mesh.  That margin exceeds every rounding of the slab
// arithmetic, so a point within eta/4 of a box is never culled -- in
// particular any binary64 hit of a non-grazing segment.
#include "pool.h"

#include <cstdlib>
#include <type_traits>

namespace rsi {
namespace {

// ------------------------------------------------------------------ pass 1
// Persistent waves.  Each wave owns a contiguous range of segments; a lane
// whose segment is finished is refilled from that range while the others go
// on, so a wave's time follows the mean cost of a segment instead of the
// slowest of its 64 (no atomics: a shared counter across eight XCDs costs more
// than the imbalance of ~1e3 segments per wave).  Leaf tests are postponed: a lane holds up to
// kPend leaves aside and continues with internal nodes; the leaf phase runs
// once a set share of the wave is waiting (on a further leaf, or done), so the
// leaf code runs for many lanes at once.
constexpr int kRefillMin = 8;     // refill when at least this many lanes idle
// The node phase hands over to the leaf phase once more than 1/kLeafShare of
// the active lanes wait on a leaf: at a third where a leaf test is cheap or ends
// the search (node steps keep more lanes busy), at half where it costs as much as
// a node step or more and more lanes should share it: certified nearest hits
// (3e6 segments of the precision form 1,022 us at a third, 957 at half, 967 at
// two thirds; the paper's scale 787 / 777 / 820; plain 619 / 620 / 651, boolean
// 1e7 1,625 / 1,637) and the count mode, which tests every leaf it reaches.
template <int MODE, bool CERT>
constexpr int kLeafShare = MODE == MODE_COUNT || (CERT && MODE != MODE_BOOL) ? 2 : 3;
// Leaves a lane may hold aside while it goes on with internal nodes: two
// keep more lanes in the node phase (boolean -2%, intercept count -5% at the
// paper's scale against one; three gain nothing more).
template <int MODE>
constexpr int kPend = 2;
// Resident waves per CU of the persistent traversal unless asked otherwise:
// fewer waves than registers allow share the CU's L1 among fewer tree paths.
constexpr int kDefaultWavesPerCU = 16;
constexpr int kDone = INT32_MIN;  // nothing left for the lane's segment
// One mesh: the share of the segments handed out in chunks at the end of the
// launch (1/kTailDiv of them), and the chunk size.  At the paper's scale a
// sixth measured best (a quarter, an eighth, a tenth, a twelfth and a
// sixteenth all ended later).
constexpr int64_t kTailDiv = 6;
constexpr int kTailChunk = 64;

// Once a wave has no new segments and at most this many in flight, its lanes
// share them (16 to 64 measure the same within 1%, 8 less: 1e6 boolean
// segments 351 us without, 243 at 8, 230 at 24; 1e7 1631 / 1538 / 1527).
constexpr int kTailLanes = 24;

// Boolean results of one mesh in input order are staged per wave in LDS and
// written out a window of kStageWin segments at a time (whole lines instead
// of single bytes as segments finish): two windows per wave, each a value
// and a done bitmap and a count of finished segments.  A wave's range starts
// at a multiple of 4, so a window's groups of four are 4-byte aligned (a
// coarser alignment would unbalance the waves' ranges).
constexpr int kStageWin = 256;
constexpr int kStageWords = 2 * kStageWin / 32 + 1;  // value bits, done bits, count
constexpr int kStageWaveWords = 2 * kStageWords + 2;  // two windows, padded to 16 bytes

// PROP: proposal-first order.  Phase 0 traverses the predicted frontier
// subtree; phase 1 the whole tree with that subtree left out.  Together they
// visit exactly what the plain order visits, so results do not change.
template <int MODE, bool CERT, bool STATS, bool PROP, bool WIDE>
__device__ __forceinline__ void traverse_pass1(TravParams p, int *lds_stack) {
    const int lane = threadIdx.x & 63;
    // LDS: the top of the 4-wide tree (read-only once filled) from address 0,
    // so that a node's byte offset is its address there too; one spare row of
    // 64 entries; the waves' stacks, each a block of its own, an entry of all 64
    // lanes after the other; the staging windows.  Stack positions are LDS byte
    // addresses of the top entry (one row below the block: empty), so a step
    // needs no address arithmetic: reads and pushes are at fixed offsets.
    constexpr int stride = 64;
    constexpr int kRow = stride * (int)sizeof(int);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LdsInt)lds_stack;
    const int top_n = WIDE && lds0 == 0 ? p.top_lds : 0;  // (no static LDS: lds0 is 0)
    const bool top_group = WIDE && p.top_group && lds0 == 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_stack = (p.stack_depth + (WIDE ? 3 : 1)) * stride;
    int *stk = lds_stack + 32 * p.top_lds + stride + wave * wave_stack;  // the wave's block
    const int sp_base = (int)lds0 + 4 * (32 * p.top_lds + stride + wave * wave_stack);
    const int sp_empty = sp_base - kRow + 4 * lane;  // stack positions at or above sp_base hold something
    const int sp_lim = sp_base + p.stack_depth * kRow;  // at or above: more than stack_depth entries
    const float scale = p.bounds[6];
    const int n_internal = (int)p.nt - 1;
    const int max_steps = 2 * (int)p.nt + 8;  // N_t < 2^30
    const bool far = far_nodes(p.nt);
    const int ref_lim = WIDE ? n_internal + kTopSlots : n_internal;
    float4 *top_cache = reinterpret_cast<float4 *>(lds_stack);
    const int group = p.n_groups > 0 ? (int)(blockIdx.x % p.n_groups) : 0;
    if (WIDE) {
        const Node4 *top = top_group ? p.top4g + (int64_t)group * kTopSlots : p.top4;
        const float4 *src = reinterpret_cast<const float4 *>(top);
        for (int i = threadIdx.x; i < 8 * top_n; i += blockDim.x)
            top_cache[i] = src[i];
        __syncthreads();
    }
    const int32_t *roots4 = top_group ? p.roots4g + (int64_t)group * 64 : p.mesh_root4;

    // One mesh: each wave owns a contiguous range of segments and its lanes
    // draw from it.  Batched form: waves take (mesh, segment range) items from
    // a shared queue, one atomic per item.  Wave-uniform state.
    const bool batch = p.items != nullptr;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t wave_id = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    // boolean results staged in LDS (one mesh, input order, 4-byte aligned output)
    const bool stage = MODE == MODE_BOOL && !STATS && !batch && p.order == nullptr && p.stage_ok;
    // One mesh: the first segments are split evenly over the waves; the rest
    // (1/kTailDiv, from a multiple of 4) is a pool of kTailChunk-segment chunks
    // that waves take in turn once their own share is handed out, so the waves
    // whose shares cost more do not hold up the end of the launch.
    const int64_t n_static = batch ? 0 : (p.n - p.n / kTailDiv) & ~int64_t(3);
    int64_t cursor = batch ? 0 : n_static * wave_id / waves;
    int64_t range_end = batch ? 0 : n_static * (wave_id + 1) / waves;
    if (stage) {  // ranges start at multiples of 4
        cursor &= ~int64_t(3);
        range_end = wave_id + 1 == waves ? n_static : (range_end & ~int64_t(3));
    }
    uint32_t *stage_w = nullptr;  // this wave's two windows
    int64_t win_base = cursor;    // first segment of the older window
    int win_old = 0;              // which of the two holds the older window
    if (stage) {
        // after the stacks (stack_depth + 3 entries per lane with 4-wide nodes,
        // + 1 with binary ones)
        stage_w = reinterpret_cast<uint32_t *>(lds_stack + 32 * p.top_lds + stride +
                                               (p.stack_depth + (WIDE ? 3 : 1)) * blockDim.x) +
                  wave * kStageWaveWords;
        if (lane < kStageWaveWords)
            stage_w[lane] = 0u;
    }
    // write the finished entries of the older window (all of them once its
    // count is complete) and make the newer one the older
    auto stage_flush = [&]() {
        const uint32_t *W = stage_w + win_old * kStageWords;
        const int j = 4 * lane;
        const uint32_t v = (W[j >> 5] >> (j & 31)) & 0xfu, d = (W[8 + (j >> 5)] >> (j & 31)) & 0xfu;
        const int64_t i = win_base + j;
        if (d == 0xfu && i + 3 < range_end) {
            const uint32_t word = (v & 1u) | ((v >> 1) & 1u) << 8 | ((v >> 2) & 1u) << 16 | ((v >> 3) & 1u) << 24;
            *reinterpret_cast<uint32_t *>(p.out.hit + i) = word;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (((d >> k) & 1u) && i + k < range_end)
                    p.out.hit[i + k] = (uint8_t)((v >> k) & 1u);
        }
        if (lane < kStageWords)
            stage_w[win_old * kStageWords + lane] = 0u;  // read above by every lane first (in wave order)
        win_base += kStageWin;
        win_old ^= 1;
    };
    // a finished boolean segment: into its window, or straight out if its
    // window has been written already (a segment that outlasted it)
    auto put_hit = [&](int64_t i, uint32_t v) {
        const int64_t off = i - win_base;
        if (stage && off >= 0 && off < 2 * kStageWin) {
            uint32_t *W = stage_w + ((win_old + (int)(off >> 8)) & 1) * kStageWords;
            const int j = (int)(off & (kStageWin - 1));
            if (v)
                atomicOr(W + (j >> 5), 1u << (j & 31));
            atomicOr(W + 8 + (j >> 5), 1u << (j & 31));
            atomicAdd(W + 16, 1u);
        } else {
            p.out.hit[i] = (uint8_t)v;
        }
    };
    bool items_left = batch || n_static < p.n;  // batch items, or the pool's chunks
    bool own_done = false;  // nothing left in this workgroup's item group (wave-uniform)
    int cur_root = p.root, cur_toff = 0;
    int lane_root = p.root, lane_toff = 0;  // of the lane's current segment

    // (fewer than 2^31 segments: 32 bits would do, and give certified nearest hits a
    // register back, 0.7%; plain ones lose 1% with the conversions)
    using RayId = std::conditional_t<CERT && MODE != MODE_BOOL, int, int64_t>;
    RayId ray = -1;
    // the last segments shared by the wave's lanes: where a pool of at least
    // 512 node entries fits in the wave's stacks
    constexpr bool kTail = WIDE && !STATS && MODE != MODE_COUNT;
    int later = -1, later_root = 0, later_toff = 0, n_later = 0;  // segments put off to the wave's end
    const bool tail = kTail && wave_stack >= 512 + kPoolLeafCap + 64 && p.nt <= kMaxPoolTris;
    Ray r;
    // 4-wide: byte offsets in a node of the near-face rows (x lo or hi at 0 /
    // 16, y at 32 / 48, z at 64 / 80; the far row is the other of each pair)
    // and the matching slab offsets, fixed per segment by the direction signs
    int offx = 0, offy = 32, offz = 64;
    float3 nn = make_float3(0.0f, 0.0f, 0.0f), nf = nn;
    int ref = kDone, sp = sp_empty;  // idle lanes have ref == kDone
    int held[kPend<MODE>];    // leaves held aside (-1: free), tested in this order
#pragma unroll
    for (int k = 0; k < kPend<MODE>; ++k)
        held[k] = -1;
    auto none_held = [&]() {
        bool none = true;
#pragma unroll
        for (int k = 0; k < kPend<MODE>; ++k)
            none = none && held[k] < 0;
        return none;
    };
    auto drop_held = [&]() {
#pragma unroll
        for (int k = 0; k < kPend<MODE>; ++k)
            held[k] = -1;
    };
    float tlimit = 1.0f;
    int best_id = -1;
    float best_t = INFINITY, best_lo = INFINITY, best_hi = INFINITY, best_u = 0.0f, best_v = 0.0f;
    // certified nearest hit: its binary64 t when computed (it decided a tie)
    bool best_exact = false;
    double best_t64 = 0.0;
    bool found = false, flagged = false, overflow = false;
    uint32_t n_nodes = 0, n_tests = 0;
    int steps = 0;
    int phase = 1, skip = kDone;  // kDone never equals a child reference
    bool best_late = false;       // best hit found in phase 1 (a proposal miss)
    uint32_t n_late = 0;          // this lane's proposal misses, summed per wave at exit
    uint32_t n_redecided = 0;     // boolean, certified: pairs of this segment decided in binary64
    uint32_t seg_redecided = 0;   // this lane's segments with such a pair, summed per wave at exit
    // count mode: the distinct t found so far -- binary32 values (plain), or
    // intervals that each hold one hit's binary64 t (certified): disjoint
    // intervals hold distinct values, so only overlapping ones need the exact
    // second pass
    float tk[kCountSlots<CERT>], tk_hi[kCountSlots<CERT>];
    int nk = 0;
    bool list_full = false;

    // (popping an empty stack reads the row below it and leaves sp below
    // sp_empty: the segment, or its proposed subtree, is done then)
    auto entry = [](int at) -> int { return *(LdsInt)(uint32_t)at; };
    auto put_entry = [](int at, int x) { *(LdsInt)(uint32_t)at = x; };
    auto pop = [&]() -> int {
        const int x = entry(sp);
        const int r = sp >= sp_base ? x : kDone;
        sp -= kRow;
        return r;
    };

    // the lane's segment is decided: its result goes out
    auto finish = [&]() {
        if (PROP && !STATS && best_late && (found || (MODE != MODE_BOOL && best_id >= 0 && !flagged && !overflow)))
            ++n_late;  // the proposal did not hold the answer
        if (STATS) {
            p.visits[ray] = n_nodes;
            p.tests[ray] = n_tests;
        } else if (MODE == MODE_COUNT) {
            if (overflow)
                enqueue(p, ray, 1);
            else if (list_full)
                enqueue(p, ray, 3);
            else if (CERT && flagged)
                enqueue(p, ray, 0);
            else
                write_count(p.out, ray, nk);
        } else if (MODE == MODE_BOOL) {
            // a queued segment counts as finished here (0); the second
            // pass writes its result after this kernel
            if (!found && overflow)
                enqueue(p, ray, 1);
            seg_redecided += n_redecided > 0 ? 1u : 0u;
            put_hit(ray, found ? 1u : 0u);
        } else {
            if (CERT && n_redecided > 0 && !flagged)
                ++seg_redecided;  // (a flagged segment is counted when queued)
            if (overflow) {
                enqueue(p, ray, 1);
            } else if (CERT && flagged) {
                enqueue(p, ray, 0);
            } else if (CERT && MODE == MODE_BARY && best_id >= 0) {
                // (u, v, t) after both passes, a lane per segment (k_bary64):
                // with the binary64 test here these kernels spilled, or ran
                // three waves a SIMD instead of four (129 registers)
                if (p.out.hit)
                    p.out.hit[ray] = 1;
                p.out.id[ray] = best_id - lane_toff;
            } else {
                write_out(p.out, ray, MODE, best_id >= 0 ? best_id - lane_toff : -1, CERT ? 0.0f : best_u,
                          CERT ? 0.0f : best_v, CERT ? 0.0f : best_t);
            }
        }
        ray = -1;
    };

    for (;;) {
        // ---- refill idle lanes
        const uint64_t idle = __ballot(ray < 0);
        if (!batch && items_left && cursor >= range_end && idle) {
            uint32_t k = 0;
            if (lane == 0)
                k = atomicAdd(p.next_ray, 1u);
            k = __shfl(k, 0);
            const int64_t start = n_static + (int64_t)k * kTailChunk;
            if (start < p.n) {
                if (stage) {
                    // what the old range left in its windows goes out (against
                    // the old range end); then the windows start at the chunk.
                    // Segments of the old range still in flight come before
                    // it, so they are written straight out when they finish.
                    if (win_base < range_end)
                        stage_flush();
                    if (win_base < range_end)
                        stage_flush();
                    win_base = start;
                    win_old = 0;
                }
                cursor = start;
                range_end = start + kTailChunk < p.n ? start + kTailChunk : p.n;
            } else {
                items_left = false;
            }
        }
        if (batch && items_left && cursor >= range_end && idle) {
            int item = -1;
            if (p.group_start) {
                // workgroups are spread over the eight XCDs in turn: this
                // workgroup's group first, whose meshes' tops are in its LDS,
                // then those on the same XCD, whose trees are in its L2, then
                // the others, so no XCD idles while work is left.  Where work
                // is left is read, a lane per group in that order, before an
                // item is asked for: at the end thousands of waves would queue
                // up at each counter in turn.
                int own_group = group;
                if (MODE == MODE_COUNT)  // worked out here: outside the loop it holds registers that the list needs
                    asm volatile("" : "+s"(own_group));
                const int per = p.n_groups / kXcds;
                const int mine = (own_group + lane / per) % kXcds + (own_group / kXcds + lane % per) % per * kXcds;
                for (bool own = true;; own = false) {
                    uint64_t left = own && !own_done ? 1ull : 0ull;
                    if (!left) {
                        bool some = false;
                        if (lane < p.n_groups) {
                            const uint32_t next = __hip_atomic_load(p.queue_len + kGroupNext + mine, __ATOMIC_RELAXED,
                                                                    __HIP_MEMORY_SCOPE_AGENT);
                            some = next < (uint32_t)(p.group_start[mine + 1] - p.group_start[mine]);
                        }
                        left = __ballot(some);
                        if (!left)
                            break;
                    }
                    const int g = __builtin_amdgcn_readlane(mine, __builtin_ctzll(left));
                    uint32_t k = 0;
                    if (lane == 0)
                        k = atomicAdd(p.queue_len + kGroupNext + g, 1u);
                    k = __shfl(k, 0);
                    const int first = p.group_start[g], count = p.group_start[g + 1] - first;
                    if (k < (uint32_t)count) {
                        item = first + (int)k;
                        break;
                    }
                    own_done = own_done || g == group;  // (a group found empty stays so: the loop ends)
                }
            } else {
                uint32_t k = 0;
                if (lane == 0)
                    k = atomicAdd(p.next_ray, 1u);
                k = __shfl(k, 0);
                item = k < (uint32_t)p.n_items ? (int)k : -1;
            }
            if (item >= 0) {
                const int4 it = p.items[item];
                cursor = it.y;
                range_end = it.z;
                cur_root = WIDE ? roots4[it.x] : p.mesh_root[it.x];
                cur_toff = p.mesh_toff[it.x];
            } else {
                items_left = false;
            }
        }
        if (cursor < range_end && idle && (__popcll(idle) >= kRefillMin || idle == ~0ull)) {
            const int cnt = __popcll(idle);
            if (stage && cursor + cnt > win_base + 2 * kStageWin)
                stage_flush();  // the older window waits on a slow segment: write what is done
            const int64_t base = cursor;
            cursor = base + cnt < range_end ? base + cnt : range_end;
            if (ray < 0) {
                const int64_t idx = base + lane_rank(idle);
                if (idx < range_end) {
                    ray = p.order ? p.order[idx] : (RayId)idx;
                    lane_root = cur_root;
                    lane_toff = cur_toff;
                    ref = lane_root;
                    drop_held();
                    sp = sp_empty;
                    tlimit = 1.0f;
                    best_id = -1;
                    best_t = best_lo = best_hi = INFINITY;
                    best_exact = false;
                    best_u = best_v = 0.0f;
                    found = flagged = overflow = false;
                    n_redecided = 0;
                    n_nodes = n_tests = 0;
                    nk = 0;
                    list_full = false;
                    steps = 0;
                    best_late = false;
                    if (PROP) {
                        skip = p.bucket_ref[p.bucket[ray]];
                        ref = skip;
                        phase = 0;
                    }
                    if (!setup_ray(p.from, p.to, ray, scale, r)) {
                        if (STATS) {
                            p.visits[ray] = 0;
                            p.tests[ray] = 0;
                        } else if (CERT) {
                            enqueue(p, ray, 0);
                            if (MODE == MODE_BOOL)
                                put_hit(ray, 0u);  // written again by the second pass
                        } else if (MODE == MODE_BOOL) {
                            put_hit(ray, 0u);
                        } else {
                            write_out(p.out, ray, MODE, -1, 0.0f, 0.0f, 0.0f);
                        }
                        ray = -1;
                        ref = kDone;
                    } else if (WIDE) {
                        const bool sx = r.inv.x < 0.0f, sy = r.inv.y < 0.0f, sz = r.inv.z < 0.0f;
                        offx = sx ? 16 : 0;
                        offy = sy ? 48 : 32;
                        offz = sz ? 80 : 64;
                        nn = make_float3(sx ? r.nrb.x : r.nra.x, sy ? r.nrb.y : r.nra.y, sz ? r.nrb.z : r.nra.z);
                        nf = make_float3(sx ? r.nra.x : r.nrb.x, sy ? r.nra.y : r.nrb.y, sz ? r.nra.z : r.nrb.z);
                    }
                }
            }
        }
        const uint64_t active = __ballot(ray >= 0);
        if (!active) {
            if (cursor >= range_end && !items_left)
                break;
            continue;
        }

        // the wave's last segments, once no new ones are left: see after the loop
        if (kTail && tail && !items_left && cursor >= range_end && __popcll(active) <= kTailLanes)
            break;

        // ---- node phase
        // Push and pop are branch-free: every lane has spare LDS slots past its
        // stack_depth entries, so the push slots are written unconditionally (a
        // slot above sp holds nothing live), and the top of stack is read ahead
        // of the node fetch and used only if the node yields nothing.  The step
        // count is checked after the phase, which is bounded itself.
        for (int turn = 0; turn <= max_steps; ++turn) {
            if ((uint32_t)ref > (uint32_t)kDone) {  // a leaf: hold it aside if a slot is free
                bool put = false;
#pragma unroll
                for (int k = 0; k < kPend<MODE>; ++k)
                    if (!put && held[k] < 0) {
                        held[k] = ~ref;
                        put = true;
                    }
                if (put)
                    ref = pop();
            }
            const bool want = ref >= 0;
            const uint64_t w = __builtin_amdgcn_ballot_w64(want);
            if (!w)
                break;
            const uint64_t waiting = active & ~w;
            if (kLeafShare<MODE, CERT> * __popcll(waiting) > __popcll(active))
                break;
            if (want) {
                ++steps;
                if (ref >= ref_lim) {
                    overflow = true;  // cannot happen for a well-formed tree
                    ref = kDone;
                    drop_held();
                } else {
                    const int top = entry(sp);  // an empty stack: the row below, not used
                    if (STATS)
                        ++n_nodes;
                    if (WIDE) {
                        // four children per fetch; the hits after the next one
                        // go on the stack, at most three slots past sp (the
                        // lane has three spare slots past stack_depth)
                        const NodeRows c = fetch_node(p.top4, ref, top_n, far, offx, offy, offz);
                        float k0, k1, k2, k3;
                        bool h0 = slab_nf<MODE == MODE_BOOL>(c.nx.x, c.fx.x, c.ny.x, c.fy.x, c.nz.x, c.fz.x, r.inv, nn, nf, tlimit, k0);
                        bool h1 = slab_nf<MODE == MODE_BOOL>(c.nx.y, c.fx.y, c.ny.y, c.fy.y, c.nz.y, c.fz.y, r.inv, nn, nf, tlimit, k1);
                        bool h2 = slab_nf<MODE == MODE_BOOL>(c.nx.z, c.fx.z, c.ny.z, c.fy.z, c.nz.z, c.fz.z, r.inv, nn, nf, tlimit, k2);
                        bool h3 = slab_nf<MODE == MODE_BOOL>(c.nx.w, c.fx.w, c.ny.w, c.fy.w, c.nz.w, c.fz.w, r.inv, nn, nf, tlimit, k3);
                        int c0 = c.ch.x, c1 = c.ch.y, c2 = c.ch.z, c3 = c.ch.w;
                        if (PROP) {  // in phase 1 the proposed subtree is done already
                            h0 = h0 && c0 != skip;
                            h1 = h1 && c1 != skip;
                            h2 = h2 && c2 != skip;
                            h3 = h3 && c3 != skip;
                        }
                        const int nh = (int)h0 + (int)h1 + (int)h2 + (int)h3;
                        if (MODE != MODE_COUNT) {
                            // in the mode's order (slab_nf)
                            double s0 = sort_key(h0, k0, c0), s1 = sort_key(h1, k1, c1);
                            double s2 = sort_key(h2, k2, c2), s3 = sort_key(h3, k3, c3);
                            order2(s0, s1);
                            order2(s2, s3);
                            order2(s0, s2);
                            order2(s1, s3);
                            order2(s1, s2);
                            c0 = key_child(s0);
                            c1 = key_child(s1);
                            c2 = key_child(s2);
                            c3 = key_child(s3);
                            put_entry(sp + kRow, nh == 4 ? c3 : (nh == 3 ? c2 : c1));
                            put_entry(sp + 2 * kRow, nh == 4 ? c2 : c1);
                            put_entry(sp + 3 * kRow, c1);
                        } else {
                            // count mode visits every candidate whatever the
                            // order: the first hit child is next, the others go
                            // on the stack in child order
                            const int p1 = h0, p2 = p1 + h1, p3 = p2 + h2;
                            if (h1 && p1)
                                put_entry(sp + kRow, c1);
                            if (h2 && p2)
                                put_entry(sp + p2 * kRow, c2);
                            if (h3 && p3)
                                put_entry(sp + p3 * kRow, c3);
                            c0 = h0 ? c0 : (h1 ? c1 : (h2 ? c2 : c3));
                        }
                        ref = nh ? c0 : (sp >= sp_base ? top : kDone);
                        sp += (nh - 1) * kRow;
                        if (sp >= sp_lim) {
                            overflow = true;  // the segment goes to the deep-stack pass
                            ref = kDone;
                            drop_held();
                        }
                    } else {
                        const Node *nd = p.nodes + ref;
                        const float4 L = nd->xy_left, R = nd->xy_right, Z = nd->z_both;
                        const int4 refs = nd->refs;
                        float tl, tr;
                        bool hl = slab(L.x, L.y, L.z, L.w, Z.x, Z.y, r, tlimit, tl);
                        bool hr = slab(R.x, R.y, R.z, R.w, Z.z, Z.w, r, tlimit, tr);
                        if (PROP) {  // in phase 1 the proposed subtree is done already
                            hl = hl && refs.x != skip;
                            hr = hr && refs.y != skip;
                        }
                        const bool both = hl && hr, any = hl || hr;
                        const bool left_first = both ? tl <= tr : hl;
                        put_entry(sp + kRow, left_first ? refs.y : refs.x);
                        const int next = left_first ? refs.x : refs.y;
                        ref = any ? next : (sp >= sp_base ? top : kDone);
                        sp += both ? kRow : (any ? 0 : -kRow);
                        if (sp >= sp_lim) {
                            overflow = true;  // the segment goes to the deep-stack pass
                            ref = kDone;
                            drop_held();
                        }
                    }
                }
            }
        }

        if (ray >= 0 && steps > max_steps) {  // cannot happen for a well-formed tree
            overflow = true;
            ref = kDone;
            drop_held();
        }

        // ---- leaf phase: the leaves held aside, in the order they were met;
        // a decided segment drops the rest
        auto test_leaf = [&](const int leaf) {
            if (leaf >= p.nt) {
                overflow = true;  // cannot happen for a well-formed tree
                ref = kDone;
            } else {
                const Tri tri = p.tris[leaf];
                if (STATS)
                    ++n_tests;
                const MT32 m = mt32(tri, r);
                const int id = __float_as_int(tri.a.w);
                if (MODE == MODE_COUNT) {
                    // every hit counts once per distinct t; no early exit, no pruning
                    if (!CERT) {
                        if (decide32(m)) {
                            const float t = m.T / m.det;
                            bool dup = false;
#pragma unroll
                            for (int k = 0; k < kCountSlots<CERT>; ++k)
                                dup = dup || (k < nk && tk[k] == t);
                            if (!dup) {
                                if (nk == kCountSlots<CERT>) {
                                    list_full = true;  // finished by the second pass
                                    ref = kDone;
                                } else {
#pragma unroll
                                    for (int k = 0; k < kCountSlots<CERT>; ++k)
                                        if (k == nk)
                                            tk[k] = t;
                                    ++nk;
                                }
                            }
                        }
                    } else {
                        // a sure hit brings an interval holding its binary64 t;
                        // an unsure pair is decided in binary64 here
                        float lo = 0.0f, hi = 0.0f;
                        const int c = classify(m, tri, r, lo, hi);
                        bool take = c == kHit;
                        if (c == kUnsure && valid_tri(p.F, p.nv, id)) {
                            const float *e = p.to + 3 * (int64_t)ray;
                            const MT64 h = mt64(r.o.x, r.o.y, r.o.z, e[0], e[1], e[2], p.V, p.F, id);
                            take = h.hit;
                            lo = __double2float_rd(h.t);
                            hi = __double2float_ru(h.t);
                        }
                        if (take) {
                            bool meet = false;
#pragma unroll
                            for (int k = 0; k < kCountSlots<CERT>; ++k)
                                meet = meet || (k < nk && !(hi < tk[k] || lo > tk_hi[k]));
                            if (meet) {
                                flagged = true;  // equal or nearly equal t: counted exactly by the second pass
                                ref = kDone;
                            } else if (nk == kCountSlots<CERT>) {
                                list_full = true;
                                ref = kDone;
                            } else {
#pragma unroll
                                for (int k = 0; k < kCountSlots<CERT>; ++k)
                                    if (k == nk) {
                                        tk[k] = lo;
                                        tk_hi[k] = hi;
                                    }
                                ++nk;
                            }
                        }
                    }
                } else if (!CERT) {
                    if (decide32(m)) {
                        if (MODE == MODE_BOOL) {
                            found = true;
                            best_late = phase == 1;
                            ref = kDone;
                        } else {
                            const float t = m.T / m.det;
                            if (t < best_t || (t == best_t && id < best_id)) {
                                best_t = t;
                                best_id = id;
                                best_late = phase == 1;
                                if (MODE == MODE_BARY) {
                                    best_u = m.U / m.det;
                                    best_v = m.W / m.det;
                                }
                                tlimit = best_t;
                            }
                        }
                    }
                } else {
                    float lo = 0.0f, hi = 0.0f;
                    const int c = classify(m, tri, r, lo, hi);
                    if (MODE == MODE_BOOL) {
                        bool hit = c == kHit;
                        if (c == kUnsure) {
                            // decided here in binary64, in the oracle's
                            // operation order: a segment aimed at an edge or a
                            // vertex would otherwise search on for a sure hit
                            // through everything its box overlaps
                            ++n_redecided;
                            if (valid_tri(p.F, p.nv, id)) {
                                const float *o = p.from + 3 * (int64_t)ray, *e = p.to + 3 * (int64_t)ray;
                                hit = mt64(o[0], o[1], o[2], e[0], e[1], e[2], p.V, p.F, id).hit;
                            }
                        }
                        if (hit) {
                            found = true;
                            best_late = phase == 1;
                            ref = kDone;
                        }
                    } else {
                        // an unsure pair is decided here in binary64, in the
                        // oracle's operation order; a hit then takes part
                        // like a sure one, its interval holding the exact t
                        bool hit = c == kHit, exact = false;
                        double t64 = 0.0;
                        const float *o = p.from + 3 * (int64_t)ray, *e = p.to + 3 * (int64_t)ray;
                        if (c == kUnsure) {
                            ++n_redecided;
                            hit = false;
                            if (valid_tri(p.F, p.nv, id)) {
                                const MT64 h = mt64(o[0], o[1], o[2], e[0], e[1], e[2], p.V, p.F, id);
                                hit = h.hit;
                                exact = true;
                                t64 = h.t;
                                lo = __double2float_rd(h.t);
                                hi = __double2float_ru(h.t);
                            }
                        }
                        if (hit && !(best_id < 0 || hi < best_lo) && !(lo > best_hi)) {
                            // the intervals overlap: compare the binary64 t
                            // themselves (both pairs are binary64 hits), ties
                            // to the smaller triangle id, as the oracle
                            if (!exact) {
                                t64 = mt64(o[0], o[1], o[2], e[0], e[1], e[2], p.V, p.F, id).t;
                                exact = true;
                            }
                            if (!best_exact) {
                                best_t64 = mt64(o[0], o[1], o[2], e[0], e[1], e[2], p.V, p.F, best_id).t;
                                best_exact = true;
                            }
                            ++n_redecided;
                            hit = t64 < best_t64 || (t64 == best_t64 && id < best_id);
                            lo = __double2float_rd(t64);
                            hi = __double2float_ru(t64);
                        } else if (hit && best_id >= 0 && !(hi < best_lo)) {
                            hit = false;  // beyond the best hit
                        }
                        if (hit) {
                            best_lo = lo;
                            best_hi = hi;
                            best_id = id;
                            best_exact = exact;
                            best_t64 = t64;
                            best_late = phase == 1;
                            tlimit = fminf(tlimit, hi * (1.0f + 0x1p-20f));
                        }
                    }
                }
            }
        };
#pragma unroll
        for (int k = 0; k < kPend<MODE>; ++k)
            if (ray >= 0 && held[k] >= 0) {
                const int leaf = held[k];
                held[k] = -1;
                if (!(found || flagged || list_full || overflow))
                    test_leaf(leaf);
            }

        // ---- proposal: the predicted subtree is exhausted, go on with the rest
        if (PROP && ray >= 0 && ref == kDone && none_held() && phase == 0 && !found && !flagged && !overflow) {
            phase = 1;
            ref = lane_root == skip ? kDone : lane_root;
            sp = sp_empty;
        }

        // ---- finish lanes whose segment is decided; one whose path outgrew the
        // stack waits for the wave's end (lane k keeps the k-th of them)
        if constexpr (kTail) {
            const bool out = tail && ray >= 0 && ref == kDone && none_held() && overflow && !found;
            for (uint64_t m = __ballot(out); m && n_later < 64; m &= m - 1) {
                const int l = __builtin_ctzll(m);
                const int who = __builtin_amdgcn_readlane((int)ray, l);
                const int root = __builtin_amdgcn_readlane(lane_root, l);
                const int toff = __builtin_amdgcn_readlane(lane_toff, l);
                if (lane == n_later) {
                    later = who;
                    later_root = root;
                    later_toff = toff;
                }
                ++n_later;
                if (lane == l) {
                    if (MODE == MODE_BOOL)
                        put_hit(ray, 0u);  // written again then
                    atomicAdd(p.counters + 1, 1ull);
                    ray = -1;
                }
            }
        }
        if (ray >= 0 && ref == kDone && none_held())
            finish();
        if (stage) {  // a complete older window goes out whole (then perhaps the next one)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t need = range_end - win_base < kStageWin ? range_end - win_base : kStageWin;
                if (need > 0 && stage_w[win_old * kStageWords + 16] == (uint32_t)need)
                    stage_flush();
            }
        }
    }
    if constexpr (kTail) {
        // The wave's last segments: all lanes share them through a pool in the
        // wave's stack memory (pool.h).  They start again from the root,
        // keeping the limit found so far.  Then those that outgrew their stack,
        // from the beginning (the second pass takes 12 to 20 us for a queue of
        // one segment).
        Pool<MODE, CERT, PROP> pool;
        const int room = wave_stack - kPoolLeafCap - 64;
        pool.init(p, reinterpret_cast<uint32_t *>(stk), 64, room < p.pool_cap ? room : p.pool_cap);
        pool.top_lds = top_n;
        PoolSegment<MODE, CERT> s;
        s.reset();
        s.ray = (int)ray;
        s.toff = 0;
        s.o = r.o;
        s.d = r.d;
        s.inv = r.inv;
        s.nn = nn;
        s.nf = nf;
        s.tlimit = tlimit;
        s.best_id = best_id;
        s.best_t = best_t;
        s.best_u = best_u;
        s.best_v = best_v;
        s.best_lo = best_lo;
        s.best_hi = best_hi;
        s.best_exact = best_exact;
        s.best_t64 = best_t64;
        s.best_late = best_late;
#pragma unroll 1
        for (int turn = 0; turn < (n_later ? 2 : 1); ++turn) {
            if (turn == 1) {
                ray = lane < n_later ? later : -1;
                s.reset();
                s.ray = (int)ray;
                n_redecided = 0;
                if (ray >= 0) {
                    if (!PROP) {
                        lane_root = later_root;
                        lane_toff = later_toff;
                    }
                    (void)setup_ray(p.from, p.to, ray, scale, r);  // (finite: it was in flight before)
                    s.set(r);
                    if (PROP) {
                        skip = p.bucket_ref[p.bucket[ray]];
                        phase = 0;
                    }
                }
            }
            if (!__ballot(ray >= 0))
                continue;
            const uint32_t tag = (uint32_t)lane << kPoolRefBits;
            bool rest = ray >= 0;
            wave_lds_fence();
            if (PROP) {  // the proposed subtree first, then what is left without it
                s.late = phase == 1;
                pool.push(ray >= 0 && phase == 0, skip, tag);
                wave_lds_fence();
                pool.run(p, s, 0, 64);
                s.late = true;
                s.skip = skip;
                rest = ray >= 0 && s.tlimit >= 0.0f && lane_root != skip;
            }
            pool.push(rest, lane_root, tag);
            wave_lds_fence();
            pool.run(p, s, 0, 64);
            if (ray >= 0) {
                best_late = s.best_late;
                found = MODE == MODE_BOOL && s.best_id >= 0;
                flagged = false;
                overflow = (pool.lost >> lane) & 1ull;
                best_id = s.best_id;
                if (!CERT) {
                    best_t = s.best_t;
                    best_u = s.best_u;
                    best_v = s.best_v;
                }
                n_redecided += s.redecided;
                if (turn == 1 && overflow && !found)
                    atomicAdd(p.counters + 1, ~0ull);  // counted when put off, and again as it is queued now
                finish();
            }
            pool.lost = 0;
        }
    }
    if (stage) {  // every segment is finished: whatever is left in the windows
        if (win_base < range_end)
            stage_flush();
        if (win_base < range_end)
            stage_flush();
    }
    if (MODE != MODE_COUNT && CERT && !STATS) {
        // segments with a pair decided in binary64 in this pass, one atomic per wave
        uint32_t w = seg_redecided;
        for (int off = 32; off > 0; off >>= 1)
            w += __shfl_xor(w, off);
        if (lane == 0 && w)
            atomicAdd(p.counters, (unsigned long long)w);
    }
    if (PROP && !STATS) {
        // one atomic per wave: a shared counter across eight XCDs is costly
        uint32_t w = n_late;
        for (int off = 32; off > 0; off >>= 1)
            w += __shfl_xor(w, off);
        if (lane == 0 && w)
            atomicAdd(p.counters + 2, (unsigned long long)w);
    }
}

// Workgroup bound per node width: the binary kernels keep 256 (a larger
// bound changed their code and cost the batched form 18%); the 4-wide ones
// take up to 1024 threads, whose workgroups keep more of the tree's top.
template <bool WIDE>
constexpr int kMaxBlock = WIDE ? 1024 : 256;

template <int MODE, bool CERT, bool STATS, bool PROP, bool WIDE>
__global__ __attribute__((amdgpu_flat_work_group_size(1, kMaxBlock<WIDE>))) void k_traverse(TravParams p) {
    extern __shared__ float4 lds_dyn[];  // 16-byte aligned: the 4-wide top nodes follow the stacks
    traverse_pass1<MODE, CERT, STATS, PROP, WIDE>(p, reinterpret_cast<int *>(lds_dyn));
}

// Count mode over binary nodes, or with a launch shape the caller chose (others
// take k_pool), holds its list of distinct t in registers; the register budget
// is fixed at four waves per SIMD (the default resident count) so the list
// cannot lower occupancy.
template <bool CERT, bool STATS, bool WIDE>
__global__ __attribute__((amdgpu_flat_work_group_size(1, kMaxBlock<WIDE>), amdgpu_waves_per_eu(4))) void k_traverse_count(
    TravParams p) {
    extern __shared__ float4 lds_dyn[];
    traverse_pass1<MODE_COUNT, CERT, STATS, false, WIDE>(p, reinterpret_cast<int *>(lds_dyn));
}

// ------------------------------------------------------------------ pass 2
// Queued segments are finished exactly: a stack deep enough for any radix
// tree, and in CERTIFIED precision every candidate not already a proven
// binary32 miss decided in binary64 with the oracle's operation order.  A
// segment whose binary32 setup is not finite is tested against every
// triangle under its root.
//
// Two shapes, chosen per launch from the queue length (uniform per block):
//   short queue: one wave per segment.  The wave shares an LDS stack and pops
//     up to 64 subtrees per step, one per lane, so a segment takes about
//     (tree depth + candidates / 64) steps instead of one dependent load per
//     visited node.
//   long queue: one lane per segment with a private deep stack (throughput).
constexpr int kFinishThreads = 64;
constexpr int kCountList = 256;  // hits a wave collects per segment in count mode (more: rounds)
constexpr int kWaveFinishMax = 8192;                      // queue length up to which a wave takes a segment
constexpr int kWaveStack = kDeepStack * kFinishThreads;  // shared entries (same LDS as the private stacks)
// Steps that pop k entries push at most 2k; popping at most (soft - size),
// soft = capacity - kDeepStack, keeps the stack at or below soft, and above it
// single pops (a plain depth-first walk) add at most one entry per tree level.
// Count mode always takes the wave shape, so its blocks need only the shared
// stack (a soft limit of 1024 entries plus the depth-first headroom) and a
// short hit list: about 7 KB of LDS instead of 48, so eight times as many
// segments are in flight (its queue holds every segment with more distinct
// hits than the first pass keeps, ~14k of 1e7 at the paper's scale).
template <int MODE>
constexpr int kWaveCap = MODE == MODE_COUNT ? 1024 + kDeepStack : kWaveStack;

template <int MODE, bool CERT>
struct Finish {
    Ray r;
    double ox, oy, oz, ex, ey, ez;
    int best_id;
    double bu, bv, bt;
    float t32, u32, v32;
    float tlimit;
    bool done;
    // count mode: only hits beyond the last counted t take part; with
    // `list` set, every such hit's t is appended there instead
    double floor64;
    float floor32;
    double *list;
    int *list_len;

    __device__ void reset_best() {
        best_id = -1;
        bu = bv = bt = 0.0;
        t32 = INFINITY;
        u32 = v32 = 0.0f;
        tlimit = 1.0f;
        done = false;
    }

    __device__ bool init(const TravParams &p, int64_t i) {
        reset_best();
        floor64 = -INFINITY;
        floor32 = -INFINITY;
        list = nullptr;
        list_len = nullptr;
        const float *o = p.from + 3 * i, *e = p.to + 3 * i;
        ox = o[0]; oy = o[1]; oz = o[2];
        ex = e[0]; ey = e[1]; ez = e[2];
        return setup_ray(p.from, p.to, i, p.bounds[6], r);
    }

    __device__ void test_leaf(const TravParams &p, int leaf) {
        const Tri tri = p.tris[leaf];
        const int id = __float_as_int(tri.a.w);
        const MT32 m = mt32(tri, r);
        if (CERT) {
            float lo, hi;
            if (classify(m, tri, r, lo, hi) == kMiss)
                return;  // the bound proves the binary64 test misses too
            MT64 h{false, 0.0, 0.0, 0.0};
            if (valid_tri(p.F, p.nv, id))
                h = mt64(ox, oy, oz, ex, ey, ez, p.V, p.F, id);
            if (!h.hit || !(h.t > floor64))
                return;
            if (MODE == MODE_COUNT && list) {
                append(h.t);
                return;
            }
            if (MODE == MODE_BOOL) {
                best_id = id;
                done = true;
                return;
            }
            if (best_id < 0 || h.t < bt || (h.t == bt && id < best_id)) {
                best_id = id;
                bu = h.u;
                bv = h.v;
                bt = h.t;
                // round up, then widen: no box holding a hit at t <= bt is culled
                tlimit = fminf(tlimit, __double2float_ru(h.t) * (1.0f + 0x1p-20f));
            }
        } else if (decide32(m)) {
            if (MODE == MODE_BOOL) {
                best_id = id;
                done = true;
                return;
            }
            const float t = m.T / m.det;
            if (!(t > floor32))
                return;
            if (MODE == MODE_COUNT && list) {
                append((double)t);
                return;
            }
            if (t < t32 || (t == t32 && id < best_id)) {
                t32 = t;
                best_id = id;
                u32 = m.U / m.det;
                v32 = m.W / m.det;
                tlimit = t;
            }
        }
    }

    // Every leaf of subtree c, exactly: the second pass's answer when a
    // subtree finds no room on the stack (a tree deeper than the stack), so a
    // push is never dropped.  The span [smallest, largest sorted leaf] holds
    // the subtree's leaves (after treelet restructuring it may hold others of
    // the same mesh too; testing a triangle twice or one outside the subtree
    // never changes a result: each is decided exactly, and equal t count once).
    __device__ void test_span(const TravParams &p, int c) {
        int first = ~c, last = ~c;
        if (c >= 0) {
            const int4 r = p.nodes[c].refs;
            first = r.z;
            last = r.w;
        }
        for (int leaf = first; leaf <= last && leaf >= 0 && leaf < p.nt && !done; ++leaf)
            test_leaf(p, leaf);
    }

    __device__ void append(double t) {
        const int k = atomicAdd(list_len, 1);
        if (k < kCountList)
            list[k] = t;
    }

    __device__ void write(const TravParams &p, int64_t i, int toff) const {
        const int local = best_id >= 0 ? best_id - toff : -1;
        if (CERT)
            write_out(p.out, i, MODE, local, (float)bu, (float)bv, (float)bt);
        else
            write_out(p.out, i, MODE, local, u32, v32, t32);
    }

    // Wave-wide result: the smallest (t, triangle id) of all lanes' hits.
    __device__ void reduce_wave() {
        for (int off = 32; off > 0; off >>= 1) {
            const int oid = __shfl_xor(best_id, off);
            if (CERT) {
                const double ot = __shfl_xor(bt, off), ou = __shfl_xor(bu, off), ov = __shfl_xor(bv, off);
                if (oid >= 0 && (best_id < 0 || ot < bt || (ot == bt && oid < best_id))) {
                    best_id = oid;
                    bt = ot;
                    bu = ou;
                    bv = ov;
                }
            } else {
                const float ot = __shfl_xor(t32, off), ou = __shfl_xor(u32, off), ov = __shfl_xor(v32, off);
                if (oid >= 0 && (best_id < 0 || ot < t32 || (ot == t32 && oid < best_id))) {
                    best_id = oid;
                    t32 = ot;
                    u32 = ou;
                    v32 = ov;
                }
            }
        }
    }
};

__device__ __forceinline__ void segment_root(const TravParams &p, int64_t i, int &root, int &toff) {
    root = p.root;
    toff = 0;
    if (p.items) {
        const int m = mesh_of_segment(p.ray_off, p.n_meshes, i);
        root = p.mesh_root[m];
        toff = p.mesh_toff[m];
    }
}

// The wave's search for one segment from `root`: every lane's share of the
// candidates goes through f.test_leaf; the caller reduces across the wave.
template <int MODE, bool CERT>
__device__ void wave_search(const TravParams &p, Finish<MODE, CERT> &f, bool ok, int root, int *stk) {
    const int lane = threadIdx.x;
    const uint64_t lt_mask = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int n_internal = (int)p.nt - 1;
    if (root == kDone) {
        // empty mesh: nothing to test
    } else if (!ok) {
        if (CERT) {
            const int64_t first = root < 0 ? ~root : p.nodes[root].refs.z;
            const int64_t last = root < 0 ? ~root : p.nodes[root].refs.w;
            for (int64_t base = first; base <= last; base += 64) {
                if (base + lane <= last)
                    f.test_leaf(p, (int)(base + lane));
                if (MODE == MODE_BOOL && __ballot(f.done))
                    break;
            }
        }
    } else {
        int size = 1;
        if (lane == 0)
            stk[0] = root;
        __syncthreads();
        const int64_t max_steps = 2 * p.nt + 8;  // every step pops at least one of < 2 nt subtrees
        // soft limit: a step that pops k entries pushes at most 2k, and past
        // the soft limit single pops add at most one entry per tree level
        const int cap = p.wave_cap;
        const int soft = cap - (kDeepStack < cap / 2 ? kDeepStack : cap / 2);
        for (int64_t step = 0; step < max_steps && size > 0; ++step) {
            const int room = soft - size;
            int k = room < 1 ? 1 : (room < 64 ? room : 64);
            k = k < size ? k : size;
            const int ref = lane < k ? stk[size - 1 - lane] : kDone;
            __syncthreads();
            size -= k;
            int c0 = kDone, c1 = kDone;  // subtrees to push, nearer one on top
            if (ref >= 0 && ref < n_internal) {
                const Node *nd = p.nodes + ref;
                const float4 L = nd->xy_left, R = nd->xy_right, Z = nd->z_both;
                const int4 refs = nd->refs;
                float tl, tr;
                const bool hl = slab(L.x, L.y, L.z, L.w, Z.x, Z.y, f.r, f.tlimit, tl);
                const bool hr = slab(R.x, R.y, R.z, R.w, Z.z, Z.w, f.r, f.tlimit, tr);
                if (hl && hr) {
                    const bool left_first = tl <= tr;
                    c0 = left_first ? refs.y : refs.x;
                    c1 = left_first ? refs.x : refs.y;
                } else if (hl || hr) {
                    c0 = hl ? refs.x : refs.y;
                }
            } else if (ref != kDone && ref < 0 && ~ref < p.nt) {
                f.test_leaf(p, ~ref);
            }
            const uint64_t m0 = __ballot(c0 != kDone), m1 = __ballot(c1 != kDone);
            const int o = size + __popcll(m0 & lt_mask) + __popcll(m1 & lt_mask);
            // a subtree past the stack's capacity is searched leaf by leaf here
            if (c0 != kDone) {
                if (o < cap)
                    stk[o] = c0;
                else
                    f.test_span(p, c0);
            }
            if (c1 != kDone) {
                if (o + 1 < cap)
                    stk[o + 1] = c1;
                else
                    f.test_span(p, c1);
            }
            size += __popcll(m0) + __popcll(m1);
            size = size < cap ? size : cap;
            __syncthreads();
            if (MODE == MODE_BOOL) {
                if (__ballot(f.done))
                    break;
            } else {
                float tl = f.tlimit;  // any lane's hit bounds the nearest one
                for (int off = 32; off > 0; off >>= 1)
                    tl = fminf(tl, __shfl_xor(tl, off));
                f.tlimit = tl;
            }
        }
    }
    __syncthreads();  // the stack is reused by the next search
}

// One wave (the whole 64-thread block) finishes segment i.  Count mode
// collects the t of every hit in LDS and counts the distinct values; a
// segment with more hits than the list holds asks instead, round by round,
// for the nearest hit beyond the last counted t until there is none.
template <int MODE, bool CERT>
__device__ void finish_wave(const TravParams &p, int64_t i, int *stk) {
    int root, toff;
    segment_root(p, i, root, toff);
    Finish<MODE, CERT> f;
    const bool ok = f.init(p, i);
    if constexpr (MODE == MODE_COUNT) {
        // one search collecting every hit's t; the distinct values are then
        // counted in LDS.  Only a list that overflows falls back to rounds.
        __shared__ double list[kCountList];
        __shared__ int list_len;
        if (threadIdx.x == 0)
            list_len = 0;
        __syncthreads();
        f.list = list;
        f.list_len = &list_len;
        wave_search<MODE, CERT>(p, f, ok, root, stk);
        const int m = list_len;
        f.list = nullptr;
        if (m <= kCountList) {
            int distinct = 0;
            for (int j = threadIdx.x; j < m; j += blockDim.x) {
                const double v = list[j];
                bool first = true;
                for (int k = 0; k < j && first; ++k)
                    first = list[k] != v;
                distinct += first ? 1 : 0;
            }
            for (int off = 32; off > 0; off >>= 1)
                distinct += __shfl_xor(distinct, off);
            if (threadIdx.x == 0)
                write_count(p.out, i, distinct);
            __syncthreads();  // the list is reused by the block's next segment
            return;
        }
        int32_t cnt = 0;
        for (int64_t q = 0; q <= p.nt; ++q) {  // at most one round per triangle
            f.reset_best();
            wave_search<MODE, CERT>(p, f, ok, root, stk);
            f.reduce_wave();
            if (f.best_id < 0)
                break;
            ++cnt;
            if (CERT)
                f.floor64 = f.bt;
            else
                f.floor32 = f.t32;
        }
        if (threadIdx.x == 0)
            write_count(p.out, i, cnt);
        __syncthreads();
        return;
    } else {
        wave_search<MODE, CERT>(p, f, ok, root, stk);
        if (MODE == MODE_BOOL) {
            f.best_id = __ballot(f.best_id >= 0) ? 0 : -1;
            toff = 0;
        } else {
            f.reduce_wave();
        }
        if (threadIdx.x == 0)
            f.write(p, i, toff);
    }
}

// One lane finishes segment i with its private stack (stride kFinishThreads).
template <int MODE, bool CERT>
__device__ void finish_lane(const TravParams &p, int64_t i, int *stk) {
    int root, toff;
    segment_root(p, i, root, toff);
    Finish<MODE, CERT> f;
    const bool ok = f.init(p, i);
    if (root == kDone) {
        // empty mesh: nothing to test
    } else if (!ok) {
        if (CERT) {
            // brute force over every leaf under the root: the box test is not reliable here
            const int first = root < 0 ? ~root : p.nodes[root].refs.z;
            const int last = root < 0 ? ~root : p.nodes[root].refs.w;
            for (int leaf = first; leaf <= last && !f.done; ++leaf)
                f.test_leaf(p, leaf);
        }
    } else {
        int sp = 0;
        int ref = root;
        const int64_t max_steps = 2 * p.nt + 8;
        const int n_internal = (int)p.nt - 1;
        for (int64_t steps = 0; steps <= max_steps && ref < n_internal && ~ref < p.nt; ++steps) {
            if (ref >= 0) {
                const Node *nd = p.nodes + ref;
                const float4 L = nd->xy_left, R = nd->xy_right, Z = nd->z_both;
                const int4 refs = nd->refs;
                float tl, tr;
                const bool hl = slab(L.x, L.y, L.z, L.w, Z.x, Z.y, f.r, f.tlimit, tl);
                const bool hr = slab(R.x, R.y, R.z, R.w, Z.z, Z.w, f.r, f.tlimit, tr);
                if (hl && hr) {
                    const bool left_first = tl <= tr;
                    const int far = left_first ? refs.y : refs.x;
                    if (sp < p.deep_cap)
                        stk[(sp++) * kFinishThreads] = far;
                    else
                        f.test_span(p, far);  // deeper than the stack: that subtree leaf by leaf
                    if (f.done)
                        break;
                    ref = left_first ? refs.x : refs.y;
                    continue;
                }
                if (hl || hr) {
                    ref = hl ? refs.x : refs.y;
                    continue;
                }
            } else {
                f.test_leaf(p, ~ref);
                if (f.done)
                    break;
            }
            if (sp == 0)
                break;
            ref = stk[(--sp) * kFinishThreads];
        }
    }
    f.write(p, i, toff);
}

template <int MODE, bool CERT>
__global__ __launch_bounds__(kFinishThreads) void k_finish(TravParams p) {
    __shared__ int deep[kWaveCap<MODE>];
    const uint32_t count = *p.queue_len;
    if (MODE == MODE_COUNT || count <= (uint32_t)kWaveFinishMax) {
        for (uint32_t qi = blockIdx.x; qi < count; qi += gridDim.x)
            finish_wave<MODE, CERT>(p, p.queue[qi], deep);
    } else {
        if constexpr (MODE != MODE_COUNT)
            for (uint32_t qi = blockIdx.x * blockDim.x + threadIdx.x; qi < count; qi += gridDim.x * blockDim.x)
                finish_lane<MODE, CERT>(p, p.queue[qi], deep + threadIdx.x);
    }
}

// ------------------------------------------------------------ segment order
// Spatially coherent processing order: neighbouring lanes then take segments
// that start (or lie) close together and head the same way, so they share
// tree paths and cached nodes.  30-bit keys; in the batched form the top six
// bits are the mesh, so each mesh's segments stay in its own position range
// and the work items stay valid.
__device__ __forceinline__ uint32_t spread_bits(uint32_t v) {  // bit k -> bit 3k, 10 bits
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t cell(float x, float lo, float hi, int bits) {
    const float f = hi > lo ? (x - lo) / (hi - lo) : 0.0f;
    const float c = fminf(fmaxf(f, 0.0f), 1.0f) * (float)(1u << bits);  // NaN -> 0
    const uint32_t q = (uint32_t)c;
    return q < (1u << bits) ? q : (1u << bits) - 1u;
}

__global__ void k_ray_keys(const float *__restrict__ from, const float *__restrict__ to, int64_t n, int kind,
                           const float *__restrict__ bounds, const int32_t *__restrict__ ray_off, int n_meshes,
                           uint32_t *__restrict__ keys, int32_t *__restrict__ ids) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const int m = ray_off ? mesh_of_segment(ray_off, n_meshes, i) : 0;
    const float *b = bounds + 8 * m;
    const float ox = from[3 * i], oy = from[3 * i + 1], oz = from[3 * i + 2];
    const float ex = to[3 * i], ey = to[3 * i + 1], ez = to[3 * i + 2];
    const int mesh_bits = ray_off ? 6 : 0;
    const int oct_bits = kind == 2 ? 3 : 0;
    const int bits = (30 - mesh_bits - oct_bits) / 3;
    float px = ox, py = oy, pz = oz;
    if (kind == 1) {
        px = 0.5f * (ox + ex);
        py = 0.5f * (oy + ey);
        pz = 0.5f * (oz + ez);
    }
    const uint32_t code = (spread_bits(cell(pz, b[2], b[5], bits)) << 2) |
                          (spread_bits(cell(py, b[1], b[4], bits)) << 1) | spread_bits(cell(px, b[0], b[3], bits));
    uint32_t key = code;
    if (kind == 2) {
        const uint32_t oct = (ex < ox ? 1u : 0u) | (ey < oy ? 2u : 0u) | (ez < oz ? 4u : 0u);
        key |= oct << (3 * bits);
    }
    key |= (uint32_t)m << (30 - mesh_bits);
    keys[i] = key;
    ids[i] = (int32_t)i;
}

__global__ void k_reset(uint32_t *queue_len, unsigned long long *counters, int n_groups) {
    if (threadIdx.x < 2)
        queue_len[threadIdx.x] = 0;  // queue length, next segment of pass 1
    if (threadIdx.x < n_groups)
        queue_len[kGroupNext + threadIdx.x] = 0;  // next item of each group
    if (threadIdx.x < 4)
        counters[threadIdx.x] = 0;
}

// Certified barycentric output: the binary64 (u, v, t) of each segment's
// nearest triangle, from the original corners in the oracle's operation order.
// Run after both passes with a lane per segment, so the binary64 work is not
// spread over the traversal's divergent lanes.  Batched form: ray_off and toff
// give the mesh's first triangle, from which tri_id counts.
__global__ void k_bary64(const float *__restrict__ from, const float *__restrict__ to, const float *__restrict__ V,
                         const int32_t *__restrict__ F, const int32_t *__restrict__ tri_id, float *__restrict__ uvt,
                         int64_t n, const int32_t *__restrict__ ray_off, const int32_t *__restrict__ toff,
                         int n_meshes) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    int id = tri_id[i];
    if (id < 0)
        return;  // a miss: written by the passes
    if (ray_off)
        id += toff[mesh_of_segment(ray_off, n_meshes, i)];
    const MT64 h = mt64(from[3 * i], from[3 * i + 1], from[3 * i + 2], to[3 * i], to[3 * i + 1], to[3 * i + 2], V, F,
                        id);
    uvt[3 * i] = (float)h.u;
    uvt[3 * i + 1] = (float)h.v;
    uvt[3 * i + 2] = (float)h.t;
}

__global__ void k_fill_miss(Outs out, int64_t n, int mode) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        write_out(out, i, mode, -1, 0.0f, 0.0f, 0.0f);
}

// Default workgroup size: 256 for binary nodes; 1024 for 4-wide ones, whose
// workgroups keep the top of the tree in LDS (a larger workgroup holds more
// of it for the same resident waves: all 512 top nodes at 1024 threads and
// depth-20 stacks; 0.2-1% faster than 512 threads in every mode at the
// paper's scale).
constexpr int kDefaultBlock = 256, kDefaultBlockWide = 1024;

template <int MODE, bool CERT, bool STATS, bool PROP, bool WIDE>
void launch_pass1(const TravParams &p, int block, hipStream_t s) {
    if (block == 0)
        block = WIDE ? kDefaultBlockWide : kDefaultBlock;
    if (block > kMaxBlock<WIDE>)
        block = kMaxBlock<WIDE>;
    // spare slots per lane past stack_depth: one for the binary push, three
    // for the 4-wide one; the 4-wide traversal also keeps the top of the tree
    // in what is left of the CU's LDS for the resident workgroups asked for
    int dev = 0, cus = 256, per_cu = 0, lds_cu = 160 * 1024, lds_block = 64 * 1024;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev);
    if (hipDeviceGetAttribute(&lds_block, hipDeviceAttributeSharedMemPerBlockOptin, dev) != hipSuccess ||
        lds_block <= 0)
        (void)hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    // a workgroup whose stacks do not fit in LDS runs with fewer threads
    const size_t lane_bytes = (size_t)(p.stack_depth + (WIDE ? 3 : 1)) * sizeof(int);
    // the boolean staging windows (per wave), after the top nodes and the stacks
    const bool staged = MODE == MODE_BOOL && !STATS && p.stage_ok && p.items == nullptr && p.order == nullptr;
    const size_t wave_stage = staged ? kStageWaveWords * sizeof(uint32_t) : 0;
    const size_t spare = 64 * sizeof(int);  // the row below the first stack
    while (block > 64 && spare + lane_bytes * block + wave_stage * (block / 64) > (size_t)lds_block)
        block /= 2;
    const size_t stack_bytes = spare + lane_bytes * block;
    const size_t stage_bytes = wave_stage * (size_t)(block / 64);
    TravParams q = p;
    q.top_lds = 0;
    q.stage_ok = stage_bytes > 0 ? 1 : 0;
    if (WIDE) {
        int blocks_cu = p.waves_per_cu / (block / 64);
        blocks_cu = blocks_cu < 1 ? 1 : blocks_cu;
        int64_t room = lds_cu / blocks_cu;
        room = room < lds_block ? room : lds_block;
        room -= (int64_t)(stack_bytes + stage_bytes);
        const int64_t slots = room > 0 ? room / (int64_t)sizeof(Node4) : 0;
        q.top_lds = (int)(slots < kTopSlots ? slots : kTopSlots);
    }
    // a group's top replaces the combined one only when all of it is in LDS
    // (a slot fetched from memory is read at the combined top's address)
    q.top_group = (WIDE && p.items && p.top4g && q.top_lds == kTopSlots) ? 1 : 0;
    const size_t lds = stack_bytes + (size_t)q.top_lds * sizeof(Node4) + stage_bytes;
    void (*kern)(TravParams) = nullptr;
    if constexpr (MODE == MODE_COUNT)
        kern = &k_traverse_count<CERT, STATS, WIDE>;
    else
        kern = &k_traverse<MODE, CERT, STATS, PROP, WIDE>;
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern), block, lds);
    const int cap = p.waves_per_cu / (block / 64);  // resident blocks per CU asked for
    per_cu = per_cu < cap ? per_cu : cap;
    if (per_cu < 1)
        per_cu = 1;
    const int64_t want = (p.n + block - 1) / block;
    const int64_t resident = (int64_t)cus * per_cu;
    const int grid = (int)(want < resident ? want : resident);
    kern<<<grid, block, lds, s>>>(q);
}

// make_params leaves nodes4 NULL where the binary tree is walked; with the
// proposal order it names the proposal's own 4-wide tree.
template <int MODE, bool STATS, bool CERT>
void dispatch_order(const TravParams &p, bool prop, int block, hipStream_t s) {
    const bool wide = p.nodes4 != nullptr;
    if (prop)
        wide ? launch_pass1<MODE, CERT, STATS, true, true>(p, block, s)
             : launch_pass1<MODE, CERT, STATS, true, false>(p, block, s);
    else
        wide ? launch_pass1<MODE, CERT, STATS, false, true>(p, block, s)
             : launch_pass1<MODE, CERT, STATS, false, false>(p, block, s);
}

template <int MODE, bool STATS>
void dispatch_mode(const TravParams &p, bool cert, bool prop, int block, hipStream_t s) {
    cert ? dispatch_order<MODE, STATS, true>(p, prop, block, s) : dispatch_order<MODE, STATS, false>(p, prop, block, s);
}

template <bool STATS>
void dispatch_pass1(const TravParams &p, int mode, bool cert, int block, hipStream_t s) {
    const bool prop = p.bucket != nullptr;
    if (mode == MODE_BOOL)
        dispatch_mode<MODE_BOOL, STATS>(p, cert, prop, block, s);
    else if (mode == MODE_FIRST)
        dispatch_mode<MODE_FIRST, STATS>(p, cert, prop, block, s);
    else if (mode == MODE_BARY)
        dispatch_mode<MODE_BARY, STATS>(p, cert, prop, block, s);
    else if (cert)  // count mode has no proposal order
        p.nodes4 ? launch_pass1<MODE_COUNT, true, STATS, false, true>(p, block, s)
                 : launch_pass1<MODE_COUNT, true, STATS, false, false>(p, block, s);
    else
        p.nodes4 ? launch_pass1<MODE_COUNT, false, STATS, false, true>(p, block, s)
                 : launch_pass1<MODE_COUNT, false, STATS, false, false>(p, block, s);
}

TravParams make_params(const MeshDev &m, const TraverseArgs &a) {
    TravParams p;
    p.nodes = m.nodes;
    // the 4-wide tree for one mesh unless binary nodes are asked for: the
    // mesh's own in the plain order, the proposal's (frontier nodes start
    // 4-wide nodes) in the proposal order
    const bool wide = m.node_width == 4 && a.node_width != 2 && (a.items == nullptr || a.mesh_root4 != nullptr);
    if (wide && a.bucket == nullptr) {
        p.nodes4 = m.nodes4;
        p.top4 = m.top4;
    } else if (wide && m.prop.top4 != nullptr) {
        p.nodes4 = m.prop.top4 + kTopSlots;
        p.top4 = m.prop.top4;
    } else {
        p.nodes4 = nullptr;
        p.top4 = nullptr;
    }
    p.top_lds = 0;
    p.bary_after = 0;
    p.tris = m.tris;
    p.V = m.V;
    p.F = m.F;
    p.bounds = m.bounds;
    p.nv = m.nv;
    p.nt = m.nt;
    p.root = m.root;
    p.from = a.from;
    p.to = a.to;
    p.n = a.n;
    p.out = Outs{a.hit, a.tri_id, a.uvt, a.count};
    p.stack_depth = a.stack;
    p.waves_per_cu = a.waves_per_cu > 0 ? a.waves_per_cu : kDefaultWavesPerCU;
    p.queue = a.queue;
    p.queue_len = a.queue_len;
    p.next_ray = a.queue_len + 1;
    p.counters = reinterpret_cast<unsigned long long *>(a.counters);
    p.visits = a.visits;
    p.tests = a.tests;
    p.bucket = a.bucket;
    p.bucket_ref = p.nodes4 && a.bucket ? m.prop.bucket_ref4 : a.bucket_ref;
    p.items = a.items;
    p.n_items = a.n_items;
    p.group_start = a.items ? a.group_start : nullptr;
    p.n_groups = p.group_start ? a.n_groups : 0;
    p.n_meshes = a.n_meshes;
    p.mesh_root = a.mesh_root;
    p.mesh_root4 = p.nodes4 ? a.mesh_root4 : nullptr;
    p.top4g = p.nodes4 && a.items ? a.top4g : nullptr;
    p.roots4g = p.top4g ? a.roots4g : nullptr;
    p.top_group = 0;
    p.mesh_toff = a.mesh_toff;
    p.ray_off = a.ray_off;
    p.order = nullptr;
    p.stage_ok = (reinterpret_cast<uintptr_t>(a.hit) & 3u) == 0 ? 1 : 0;
    p.deep_cap = kDeepStack;
    p.wave_cap = a.mode == MODE_COUNT ? kWaveCap<MODE_COUNT> : kWaveCap<MODE_BOOL>;
    // RSI_DEBUG_PASS2_STACK=k (2..kDeepStack) shrinks both second-pass stacks
    // to k entries, so tests reach the leaf-span path that a tree deeper than
    // the stacks takes; results do not change
    if (const char *env = getenv("RSI_DEBUG_PASS2_STACK")) {
        const int k = atoi(env);
        if (k >= 2 && k <= kDeepStack) {
            p.deep_cap = k;
            p.wave_cap = k;
        }
    }
    // RSI_DEBUG_POOL_NODES=k (1..) shrinks the node stack of the pool form and
    // of a wave's last segments, so tests reach their overflow into the second pass
    p.pool_cap = INT32_MAX;
    if (const char *env = getenv("RSI_DEBUG_POOL_NODES"))
        if (atoi(env) >= 1)
            p.pool_cap = atoi(env);
    return p;
}

// Does the first pass run in pool form (pool.hip)?  In count mode always: it
// visits every candidate in any order, and the pool keeps the lanes busy
// (4e6 segments at the paper's scale 2.50 -> 1.74 ms).  In
// the other modes up to the lanes that are resident at once (262,144): below
// that a launch of the lane form is its slowest segments (1e4 segments 156 -> 35
// us, 1e5 against 522,242 triangles 150 -> 88, 2e5 at the paper's scale 134 ->
// 78); up to twice as many on meshes of at most kPoolSmallMesh triangles, whose
// nodes stay in an XCD's L2.  Above that a lane's nearest-first walk does less
// work (boolean, pool / lane form: 32,258 triangles 5e5 154 / 166 us, 6e5 187 /
// 178; 130,050 3e5 167 / 174, 3.9e5 200 / 186; 522,242 2.6e5 163 / 180, 3e5
// 190 / 178).  A launch shape the caller chose is the lane form's.
constexpr int64_t kPoolSmallMesh = 65536;
bool use_pool(const TravParams &p, const TraverseArgs &a) {
    if (!a.default_shape || p.nodes4 == nullptr || a.bucket != nullptr || p.nt > kMaxPoolTris)
        return false;
    if (a.mode == MODE_COUNT)
        return true;
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    return a.n <= (int64_t)cus * kDefaultWavesPerCU * 64 * (p.nt <= kPoolSmallMesh ? 2 : 1);
}

// Keys and a stable sort of the segment indices; p.order then lists them.
hipError_t order_segments(const TraverseArgs &a, TravParams &p, hipStream_t s) {
    if (a.ray_sort == 0 || a.n < 2)
        return hipSuccess;
    uint32_t *keys = static_cast<uint32_t *>(a.sort_ws);
    int32_t *ids = reinterpret_cast<int32_t *>(keys + ((a.n + 63) & ~int64_t(63)));
    void *tmp = ids + ((a.n + 63) & ~int64_t(63));
    k_ray_keys<<<(int)((a.n + 255) / 256), 256, 0, s>>>(a.from, a.to, a.n, a.ray_sort, a.key_bounds, a.ray_off,
                                                       a.n_meshes, keys, ids);
    const hipError_t e = sort_u32_pairs(keys, ids, tmp, a.n, s);
    p.order = ids;
    return e;
}

}  // namespace

size_t ray_sort_ws_bytes(int64_t n) {
    const int64_t padded = (n + 63) & ~int64_t(63);
    return 8 * (size_t)padded + sort_u32_tmp_bytes(n) + 256;
}

hipError_t launch_intersect(const MeshDev &m, const TraverseArgs &a, hipStream_t s) {
    TravParams p = make_params(m, a);
    k_reset<<<1, 64, 0, s>>>(a.queue_len, p.counters, p.group_start ? p.n_groups : 0);
    if (a.n == 0)
        return hipGetLastError();
    if (m.nt == 0) {
        k_fill_miss<<<(int)((a.n + 255) / 256), 256, 0, s>>>(p.out, a.n, a.mode);
        return hipGetLastError();
    }
    const hipError_t e = order_segments(a, p, s);
    if (e != hipSuccess)
        return e;
    // Certified barycentric: (u, v, t) by a launch of its own, except for a
    // batch in pool form, which writes them as it finishes a segment (5,000
    // segments in 7 meshes: 35.5 us, 37.2 with that launch)
    const bool pool = use_pool(p, a), bary_after = a.mode == MODE_BARY && a.certified && !(pool && a.items);
    p.bary_after = bary_after ? 1 : 0;
    if (pool)
        launch_pool(p, a.mode, a.certified != 0, s);
    else
        dispatch_pass1<false>(p, a.mode, a.certified != 0, a.block, s);
    // enough blocks for one per segment of a short queue; a long queue is
    // taken 64 segments per block (count mode: a wave per segment, with
    // small blocks that fit many per CU)
    const int64_t cap2 = a.mode == MODE_COUNT ? 8192 : 2048;
    const int grid2 = (int)(a.n < cap2 ? a.n : cap2);
    if (a.mode == MODE_BOOL)
        a.certified ? k_finish<MODE_BOOL, true><<<grid2, kFinishThreads, 0, s>>>(p) : k_finish<MODE_BOOL, false><<<grid2, kFinishThreads, 0, s>>>(p);
    else if (a.mode == MODE_FIRST)
        a.certified ? k_finish<MODE_FIRST, true><<<grid2, kFinishThreads, 0, s>>>(p) : k_finish<MODE_FIRST, false><<<grid2, kFinishThreads, 0, s>>>(p);
    else if (a.mode == MODE_BARY)
        a.certified ? k_finish<MODE_BARY, true><<<grid2, kFinishThreads, 0, s>>>(p) : k_finish<MODE_BARY, false><<<grid2, kFinishThreads, 0, s>>>(p);
    else
        a.certified ? k_finish<MODE_COUNT, true><<<grid2, kFinishThreads, 0, s>>>(p) : k_finish<MODE_COUNT, false><<<grid2, kFinishThreads, 0, s>>>(p);
    if (bary_after)
        k_bary64<<<(int)((a.n + 255) / 256), 256, 0, s>>>(a.from, a.to, m.V, m.F, a.tri_id, a.uvt, a.n,
                                                         a.items ? a.ray_off : nullptr, a.mesh_toff, a.n_meshes);
    return hipGetLastError();
}

namespace {
// Diagnostics of the certified test on given pairs: the same ray and triangle
// set-up as the traversal, then the binary32 quantities, their bounds and the
// classification.  vals[i] = det, U, W, T, B(det), B(U), B(W), B(T), tlo, thi.
__global__ void k_debug_certify(const float *__restrict__ from, const float *__restrict__ to,
                                const float *__restrict__ corners, int64_t n, float *__restrict__ vals,
                                int32_t *__restrict__ cls) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    Ray r;
    r.o = make_float3(from[3 * i], from[3 * i + 1], from[3 * i + 2]);
    r.d = make_float3(to[3 * i] - r.o.x, to[3 * i + 1] - r.o.y, to[3 * i + 2] - r.o.z);
    const float *c = corners + 9 * i;
    Tri tri;
    tri.a = make_float4(c[0], c[1], c[2], 0.0f);
    tri.e1 = make_float4(c[3] - c[0], c[4] - c[1], c[5] - c[2], 0.0f);
    tri.e2 = make_float4(c[6] - c[0], c[7] - c[1], c[8] - c[2], 0.0f);
    const MT32 m = mt32(tri, r);
    const Bounds b = mt_bounds(m, tri, r);
    float tlo = NAN, thi = NAN;
    cls[i] = classify(m, tri, r, tlo, thi);
    float *v = vals + 10 * i;
    v[0] = m.det; v[1] = m.U; v[2] = m.W; v[3] = m.T;
    v[4] = b.d; v[5] = b.U; v[6] = b.W; v[7] = b.T;
    v[8] = tlo; v[9] = thi;
}
}  // namespace

hipError_t launch_debug_certify(const float *from, const float *to, const float *corners, int64_t n, float *vals,
                                int32_t *cls, hipStream_t s) {
    if (n > 0)
        k_debug_certify<<<(int)((n + 255) / 256), 256, 0, s>>>(from, to, corners, n, vals, cls);
    return hipGetLastError();
}

hipError_t launch_stats(const MeshDev &m, const TraverseArgs &a, hipStream_t s) {
    TravParams p = make_params(m, a);
    k_reset<<<1, 64, 0, s>>>(a.queue_len, p.counters, p.group_start ? p.n_groups : 0);
    if (m.nt == 0 || a.n == 0)
        return hipGetLastError();
    const hipError_t e = order_segments(a, p, s);
    if (e != hipSuccess)
        return e;
    dispatch_pass1<true>(p, a.mode, a.certified != 0, a.block, s);
    return hipGetLastError();
}

}  // namespace rsi
