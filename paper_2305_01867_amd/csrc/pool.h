// pool.h -- one wave's segments traversed through a shared pool of pending
// nodes and leaves (4-wide tree).
//
// Each of the first `slots` lanes owns up to one segment ("slot" = the lane's
// number); the wave keeps one stack of (slot, node) entries and one list of
// (slot, leaf) entries in LDS.  A step pops up to 64 entries, one per lane,
// whichever segments they belong to: the lane fetches that segment's constants
// from its owner's registers (ds_bpermute), tests the node's four children and
// pushes those it meets; leaves are tested up to 64 at a time.  So a segment's
// work is not one lane's chain of dependent fetches (up to 200 nodes and 100
// triangles at the paper's scale, mean 18 and 3): with few segments it takes
// about the tree's depth in steps, and the last segments of a wave use all its
// lanes.  Results are those of the lane-per-segment form: every candidate whose
// box the segment meets below its limit is tested, with the same arithmetic,
// and the nearest of them (or their number) does not depend on the order.
#pragma once

#include "segment.h"

namespace rsi {
namespace {

constexpr int kPoolRefBits = 26;  // an entry: slot (6 bits) above a node or leaf number
constexpr uint32_t kPoolRefMask = (1u << kPoolRefBits) - 1u;
constexpr int64_t kMaxPoolTris = (int64_t(1) << kPoolRefBits) - kTopSlots;
// the leaves are below 64 before a node step adds up to four per lane
constexpr int kPoolLeafCap = 64 + 4 * 64;

__device__ __forceinline__ int lane_rank(uint64_t mask) {  // set bits of mask below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
__device__ __forceinline__ int from_lane(int byte_lane, int x) { return __builtin_amdgcn_ds_bpermute(byte_lane, x); }
__device__ __forceinline__ float from_lane(int byte_lane, float x) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(byte_lane, __float_as_int(x)));
}
__device__ __forceinline__ double from_lane(int byte_lane, double x) {
    return __hiloint2double(from_lane(byte_lane, __double2hiint(x)), from_lane(byte_lane, __double2loint(x)));
}
__device__ __forceinline__ float3 from_lane(int byte_lane, const float3 &v) {
    return make_float3(from_lane(byte_lane, v.x), from_lane(byte_lane, v.y), from_lane(byte_lane, v.z));
}
// LDS written by other lanes of the wave is read next (the LDS serves a wave's
// accesses in order: this only keeps the compiler from moving them)
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// A lane's own segment: set-up and answer so far.
template <int MODE, bool CERT>
struct PoolSegment {
    int ray;        // -1: none
    int toff;       // first triangle of its mesh
    float3 o, d, inv;
    float3 nn, nf;  // slab offsets of the near and far faces
    float tlimit;   // below 0: decided (boolean), the second pass's (count)
    int best_id;    // boolean: 0 once a hit is known
    float best_t, best_u, best_v;  // plain
    float best_lo, best_hi;        // certified: interval around the binary64 t
    bool best_exact;
    double best_t64;
    int redecided;  // pairs decided in binary64
    // proposal order: the proposed subtree is done (late), the answer was
    // found after it, the child to leave out
    bool late, best_late;
    int skip;

    __device__ __forceinline__ void reset() {
        tlimit = 1.0f;
        best_id = -1;
        best_t = best_lo = best_hi = INFINITY;
        best_u = best_v = 0.0f;
        best_exact = false;
        best_t64 = 0.0;
        redecided = 0;
        late = best_late = false;
        skip = kEmptyChild;
    }
    __device__ __forceinline__ void set(const Ray &r) {
        o = r.o;
        d = r.d;
        inv = r.inv;
        const bool sx = r.inv.x < 0.0f, sy = r.inv.y < 0.0f, sz = r.inv.z < 0.0f;
        nn = make_float3(sx ? r.nrb.x : r.nra.x, sy ? r.nrb.y : r.nra.y, sz ? r.nrb.z : r.nra.z);
        nf = make_float3(sx ? r.nra.x : r.nrb.x, sy ? r.nra.y : r.nrb.y, sz ? r.nra.z : r.nrb.z);
    }

    // plain nearest hit: smallest t, ties to the smaller triangle
    __device__ __forceinline__ void take(int id, float t, float u, float v) {
        if (t < best_t || (t == best_t && id < best_id)) {
            best_t = t;
            best_id = id;
            best_u = u;
            best_v = v;
            best_late = late;
            tlimit = t;
        }
    }
    // certified nearest hit: an interval [lo, hi] holding the hit's binary64 t
    // (itself when exact); where two intervals overlap the binary64 t decide,
    // ties to the smaller triangle
    __device__ __forceinline__ void take(const TravParams &p, int id, float lo, float hi, bool exact, double t64) {
        if (id == best_id)
            return;
        bool hit = true;
        if (!(best_id < 0 || hi < best_lo) && !(lo > best_hi)) {
            const float *a = p.from + 3 * (int64_t)ray, *e = p.to + 3 * (int64_t)ray;
            if (!exact) {
                t64 = mt64(a[0], a[1], a[2], e[0], e[1], e[2], p.V, p.F, id).t;
                exact = true;
            }
            if (!best_exact) {
                best_t64 = mt64(a[0], a[1], a[2], e[0], e[1], e[2], p.V, p.F, best_id).t;
                best_exact = true;
            }
            ++redecided;
            hit = t64 < best_t64 || (t64 == best_t64 && id < best_id);
            lo = __double2float_rd(t64);
            hi = __double2float_ru(t64);
        } else if (best_id >= 0 && !(hi < best_lo)) {
            hit = false;  // beyond the best hit
        }
        if (hit) {
            best_lo = lo;
            best_hi = hi;
            best_id = id;
            best_exact = exact;
            best_t64 = t64;
            best_late = late;
            tlimit = fminf(tlimit, hi * (1.0f + 0x1p-20f));
        }
    }
};

// Count mode: per slot the number of hits listed so far, above it whether the
// list had no room for one (kPoolFull) that met a listed one (kPoolMeet), and
// the list -- binary32 t (plain) or intervals (certified).
constexpr int kPoolFull = 1 << 29, kPoolMeet = 1 << 30;
// LDS words per slot: a mail word (nearest hits), or the hits and their list.
template <int MODE, bool CERT>
constexpr int kPoolSlotWords = MODE == MODE_COUNT ? 1 + kCountSlots<CERT> * (CERT ? 2 : 1) : 1;
// LDS words of one wave
template <int MODE, bool CERT>
constexpr int pool_words(int slots, int cap) {
    return (cap + kPoolLeafCap + slots * kPoolSlotWords<MODE, CERT> + 3) & ~3;
}

template <int MODE, bool CERT, bool PROP>
struct Pool {
    uint32_t *node, *leaf;  // this wave's entries (LDS)
    int *mail;              // [slots] a lane with news for the slot's owner; count mode: hits, then the lists
    int slots, cap;         // cap: entries of `node`
    int ns, ls;             // entries in use (wave-uniform)
    uint64_t lost;          // slots with an entry that found no room (wave-uniform)
    int top_lds;            // the tree's first top_lds nodes are in LDS, from address 0
    int ref_last;
    bool far;

    __device__ __forceinline__ void init(const TravParams &p, uint32_t *words, int n_slots, int node_cap) {
        node = words;
        leaf = words + node_cap;
        mail = reinterpret_cast<int *>(leaf + kPoolLeafCap);
        slots = n_slots;
        cap = node_cap;
        ns = ls = 0;
        lost = 0;
        top_lds = 0;
        far = far_nodes(p.nt);
        ref_last = (int)p.nt - 2 + kTopSlots;
    }
    __device__ __forceinline__ float *list(int slot) {
        return reinterpret_cast<float *>(mail + slots) + slot * kCountSlots<CERT> * (CERT ? 2 : 1);
    }

    // Entries (slot, ref) of the lanes with v: nodes onto the stack, leaves
    // (ref < 0) onto their list.
    __device__ __forceinline__ void push(bool v, int ref, uint32_t tag) {
        const bool inner = v && ref >= 0, outer = v && ref < 0;
        const uint64_t nm = __ballot(inner), lm = __ballot(outer);
        const int at = ns + lane_rank(nm);
        if (inner && at < cap)
            node[at] = tag | (uint32_t)ref;
        if (outer)
            leaf[ls + lane_rank(lm)] = tag | (uint32_t)~ref;
        ns += __popcll(nm);
        ls += __popcll(lm);
        if (ns > cap) {  // the segment goes to the second pass
            ns = cap;
            for (uint64_t m = __ballot(inner && at >= cap); m; m &= m - 1)
                lost |= 1ull << ((uint32_t)__builtin_amdgcn_readlane((int)tag, __builtin_ctzll(m)) >> kPoolRefBits);
        }
    }

    __device__ __forceinline__ void node_step(const TravParams &p, const PoolSegment<MODE, CERT> &s) {
        const int lane = threadIdx.x & 63;
        // every popped entry may add four: no more than the stack has room for
        // (one at a time when it is full, as a depth-first walk)
        const int fit = (cap - ns) / 3;
        int k = ns < 64 ? ns : 64;
        k = k < fit ? k : (fit > 1 ? fit : 1);
        const bool on = lane < k;
        const uint32_t it = on ? node[ns - 1 - lane] : 0u;
        ns -= k;
        const int from = (int)(it >> kPoolRefBits) << 2;
        const uint32_t tag = it & ~kPoolRefMask;
        int ref = (int)(it & kPoolRefMask);
        ref = ref < ref_last ? ref : ref_last;  // (a well-formed tree has no other)
        const float3 inv = from_lane(from, s.inv), nn = from_lane(from, s.nn), nf = from_lane(from, s.nf);
        const float tlimit = from_lane(from, s.tlimit);
        bool h0 = false, h1 = false, h2 = false, h3 = false;
        float k0 = INFINITY, k1 = INFINITY, k2 = INFINITY, k3 = INFINITY;
        int c0 = 0, c1 = 0, c2 = 0, c3 = 0;
        if (on && (MODE == MODE_FIRST || MODE == MODE_BARY || tlimit >= 0.0f)) {
            const int offx = inv.x < 0.0f ? 16 : 0, offy = inv.y < 0.0f ? 48 : 32, offz = inv.z < 0.0f ? 80 : 64;
            const NodeRows c = fetch_node(p.top4, ref, top_lds, far, offx, offy, offz);
            h0 = slab_nf<MODE == MODE_BOOL>(c.nx.x, c.fx.x, c.ny.x, c.fy.x, c.nz.x, c.fz.x, inv, nn, nf, tlimit, k0);
            h1 = slab_nf<MODE == MODE_BOOL>(c.nx.y, c.fx.y, c.ny.y, c.fy.y, c.nz.y, c.fz.y, inv, nn, nf, tlimit, k1);
            h2 = slab_nf<MODE == MODE_BOOL>(c.nx.z, c.fx.z, c.ny.z, c.fy.z, c.nz.z, c.fz.z, inv, nn, nf, tlimit, k2);
            h3 = slab_nf<MODE == MODE_BOOL>(c.nx.w, c.fx.w, c.ny.w, c.fy.w, c.nz.w, c.fz.w, inv, nn, nf, tlimit, k3);
            c0 = c.ch.x;
            c1 = c.ch.y;
            c2 = c.ch.z;
            c3 = c.ch.w;
        }
        if (PROP) {
            const int skip = from_lane(from, s.skip);
            h0 = h0 && c0 != skip;
            h1 = h1 && c1 != skip;
            h2 = h2 && c2 != skip;
            h3 = h3 && c3 != skip;
        }
        if (MODE != MODE_COUNT) {
            // each lane's first child (slab_nf) on top
            const int nh = (int)h0 + (int)h1 + (int)h2 + (int)h3;
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
            h0 = nh > 0;
            h1 = nh > 1;
            h2 = nh > 2;
            h3 = nh > 3;
        }
        push(h3, c3, tag);
        push(h2, c2, tag);
        push(h1, c1, tag);
        push(h0, c0, tag);
        wave_lds_fence();
    }

    // Boolean: the entries of decided segments leave the stack.
    __device__ __forceinline__ void drop_decided(const PoolSegment<MODE, CERT> &s) {
        const int lane = threadIdx.x & 63;
        const uint64_t decided = __ballot(s.tlimit < 0.0f);
        int kept = 0;
        for (int b = 0; b < ns; b += 64) {
            const bool in = b + lane < ns;
            const uint32_t it = in ? node[b + lane] : 0u;
            const bool keep = in && !(decided >> (it >> kPoolRefBits) & 1ull);
            const uint64_t m = __ballot(keep);
            if (keep)
                node[kept + lane_rank(m)] = it;
            kept += __popcll(m);
            wave_lds_fence();
        }
        ns = kept;
    }

    // Count mode, hits that found their segment's list full, lane by lane of
    // `past`.  Plain: the list drops repeated t (coincident triangles give one
    // t) and takes the hit's own unless it holds it.  Certified: intervals that
    // meet are the second pass's to count, so there is nothing to drop.  A list
    // without room sends the segment to the second pass, and nothing more is
    // looked for: its limit is below every entry t.  (16 sheets, doubled, 1e6
    // segments, plain: 5,895 us with the first 12 hits listed, repeated or not,
    // 2,817 so; certified 7,446 and 6,729.  3,000 triangles across the unit cube,
    // 4e5 segments with more hits than the list takes: 36.2 ms each walked to its
    // end, 30.3 so.)
    __device__ __forceinline__ void list_full(PoolSegment<MODE, CERT> &s, uint64_t past, int slot, float lo, float hi) {
        const int lane = threadIdx.x & 63;
        constexpr int kSlots = kCountSlots<CERT>;
        for (; past; past &= past - 1) {
            const int from = __builtin_ctzll(past), own = __builtin_amdgcn_readlane(slot, from);
            const float t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lo), from));
            float *l = list(own);
            const int had = __builtin_amdgcn_readfirstlane(mail[own]);
            if (had >= kPoolFull)
                continue;
            const int listed = had < kSlots ? had : kSlots;
            bool room = false;
            int now = kPoolFull;
            if (!CERT) {
                const float mine = lane < listed ? l[lane] : 0.0f;
                bool first = lane < listed;
#pragma unroll
                for (int j = 0; j + 1 < kSlots; ++j) {
                    const float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), j));
                    first = first && !(j < lane && x == mine);
                }
                const uint64_t keep = __ballot(first);
                const bool known = __ballot(first && mine == t) != 0;
                int kept = __popcll(keep);
                room = known || kept < kSlots;
                wave_lds_fence();  // every lane has read its entry
                if (first)
                    l[lane_rank(keep)] = mine;
                if (!known && room) {
                    if (lane == 0)
                        l[kept] = t;
                    ++kept;
                }
                now = room ? kept : kPoolFull;
            } else {
                const float h = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hi), from));
                if (__ballot(lane < kSlots && !(h < l[lane] || t > l[kSlots + lane])))
                    now |= kPoolMeet;
            }
            if (lane == 0)
                mail[own] = now;
            wave_lds_fence();
        }
        if (lane < slots && mail[lane] >= kPoolFull)
            s.tlimit = -1.0f;
    }

    // Up to 64 leaves, a lane each.
    __device__ __forceinline__ void leaf_step(const TravParams &p, PoolSegment<MODE, CERT> &s) {
        const int lane = threadIdx.x & 63;
        const int k = ls < 64 ? ls : 64;
        const bool on = lane < k;
        const uint32_t it = on ? leaf[ls - 1 - lane] : 0u;
        ls -= k;
        const int slot = (int)(it >> kPoolRefBits), from = slot << 2;
        const int at = (int)(it & kPoolRefMask);
        Ray q;
        q.o = from_lane(from, s.o);
        q.d = from_lane(from, s.d);
        const int ray = from_lane(from, s.ray);
        const float lim = MODE == MODE_COUNT ? 0.0f : from_lane(from, s.tlimit);
        bool hit = false, decided = false;
        float lo = 0.0f, hi = 0.0f, u = 0.0f, v = 0.0f;
        double t64 = 0.0;
        int id = -1;
        if (on && at < p.nt && (MODE != MODE_BOOL || lim >= 0.0f)) {
            const Tri tri = p.tris[at];
            const MT32 m = mt32(tri, q);
            id = __float_as_int(tri.a.w);
            if (!CERT) {
                hit = decide32(m);
                if (MODE != MODE_BOOL) {
                    lo = m.T / m.det;
                    if (MODE == MODE_BARY) {
                        u = m.U / m.det;
                        v = m.W / m.det;
                    }
                }
            } else {
                const int c = classify(m, tri, q, lo, hi);
                hit = c == kHit;
                if (c == kUnsure) {  // decided here, in the oracle's operation order
                    decided = true;
                    if (valid_tri(p.F, p.nv, id)) {
                        const float *o = p.from + 3 * (int64_t)ray, *e = p.to + 3 * (int64_t)ray;
                        const MT64 h = mt64(o[0], o[1], o[2], e[0], e[1], e[2], p.V, p.F, id);
                        hit = h.hit;
                        t64 = h.t;
                        lo = __double2float_rd(h.t);
                        hi = __double2float_ru(h.t);
                    }
                }
            }
            if (MODE == MODE_FIRST || MODE == MODE_BARY)
                hit = hit && !(lo > lim);
        }
        if (MODE == MODE_COUNT) {
            // every hit into its segment's list
            bool past = false;
            if (hit) {
                const int had = atomicAdd(mail + slot, 1);
                float *l = list(slot);
                past = had >= kCountSlots<CERT> && had < kPoolFull;
                if (had < kCountSlots<CERT>) {
                    l[had] = lo;
                    if (CERT)
                        l[kCountSlots<CERT> + had] = hi;
                }
            }
            wave_lds_fence();
            const uint64_t past_m = __ballot(past);
            if (past_m)
                list_full(s, past_m, slot, lo, hi);
            return;
        }
        if (CERT)
            for (uint64_t m = __ballot(decided); m; m &= m - 1)
                s.redecided += __builtin_amdgcn_readlane(slot, __builtin_ctzll(m)) == lane ? 1 : 0;
        // each owner takes its segment's hits one after the other, all owners
        // at once (a hit's lane leaves its number in the owner's mail)
        const bool any = __ballot(hit) != 0;
        while (__ballot(hit)) {
            if (lane < slots)
                mail[lane] = -1;
            wave_lds_fence();
            if (hit)
                mail[slot] = lane;
            wave_lds_fence();
            hit = hit && MODE != MODE_BOOL && mail[slot] != lane;
            const int w = lane < slots ? mail[lane] : -1;
            wave_lds_fence();
            if (MODE == MODE_BOOL) {
                if (w >= 0) {
                    s.best_id = 0;
                    s.best_late = s.late;
                    s.tlimit = -1.0f;
                }
            } else {
                const int wl = (w < 0 ? 0 : w) << 2;
                const int w_id = from_lane(wl, id);
                const float w_lo = from_lane(wl, lo);
                if (CERT) {
                    const float w_hi = from_lane(wl, hi);
                    const int w_exact = from_lane(wl, (int)decided);
                    const double w_t = from_lane(wl, t64);
                    if (w >= 0)
                        s.take(p, w_id, w_lo, w_hi, w_exact != 0, w_t);
                } else {
                    const float w_u = from_lane(wl, u), w_v = from_lane(wl, v);
                    if (w >= 0)
                        s.take(w_id, w_lo, w_u, w_v);
                }
            }
        }
        if (MODE == MODE_BOOL && any)
            drop_decided(s);
    }

    // Steps until at most `low` node entries are left (none, and no leaves, for
    // 0).  Leaves are tested once there are `leaves` of them (at most 64).
    __device__ __forceinline__ void run(const TravParams &p, PoolSegment<MODE, CERT> &s, int low, int leaves) {
        for (;;) {
            if (ls >= leaves || (ns == 0 && ls > 0)) {
                leaf_step(p, s);
                continue;
            }
            if (ns <= low)
                break;
            node_step(p, s);
        }
    }

    // Does this lane's segment have entries left?  (At most 64 nodes and fewer
    // leaves than that.)  Every lane takes part.
    __device__ __forceinline__ bool pending() {
        const int lane = threadIdx.x & 63;
        int *flag = reinterpret_cast<int *>(leaf + 64);  // (not in use: fewer than 64 leaves)
        flag[lane] = 0;
        wave_lds_fence();
        if (lane < ns)
            flag[node[lane] >> kPoolRefBits] = 1;
        if (lane < ls)
            flag[leaf[lane] >> kPoolRefBits] = 1;
        wave_lds_fence();
        const bool any = flag[lane] != 0;
        wave_lds_fence();
        return any;
    }
};

}  // namespace
}  // namespace rsi
