// segment.h -- device code shared by the traversal kernels: a segment's set-up,
// the slab tests, the binary32 and binary64 Moller-Trumbore tests with their
// bounds, the result writes and the kernels' parameters.
#pragma once

#include "rsi_internal.h"

namespace rsi {

struct Outs {
    uint8_t *hit;
    int32_t *id;
    float *uvt;
    int32_t *count;
};

struct TravParams {
    const Node *__restrict__ nodes;
    const Node4 *__restrict__ nodes4;  // the 4-wide tree the first pass walks, or NULL
    const Node4 *__restrict__ top4;    // its first kTopSlots nodes, breadth-first
    int top_lds;                       // how many of them each workgroup keeps in LDS
    int bary_after;                    // pool form, certified barycentric: (u, v, t) by k_bary64
    const Tri *__restrict__ tris;
    const float *__restrict__ V;
    const int32_t *__restrict__ F;
    const float *__restrict__ bounds;
    int64_t nv;
    int64_t nt;
    int root;
    const float *__restrict__ from;
    const float *__restrict__ to;
    int64_t n;
    Outs out;
    int stack_depth;
    int waves_per_cu;
    int32_t *queue;
    uint32_t *queue_len;
    uint32_t *next_ray;
    unsigned long long *counters;
    uint32_t *visits;
    uint32_t *tests;
    const uint8_t *bucket;
    const int32_t *bucket_ref;
    const int4 *items;
    int n_items;
    const int32_t *group_start;  // [n_groups + 1] first item of each group, or NULL: one queue
    int n_groups;
    int n_meshes;
    const int32_t *mesh_root;
    const int32_t *mesh_root4;  // the mesh roots as 4-wide references (first pass over 4-wide nodes)
    // batched form, 4-wide, every top slot in LDS: each workgroup keeps the
    // top of its item group's meshes (group blockIdx.x mod n_groups) instead
    // of the combined tree's, with the mesh roots as references in it
    const Node4 *top4g;
    const int32_t *roots4g;
    int top_group;
    const int32_t *mesh_toff;
    const int32_t *ray_off;
    const int32_t *order;  // segment at each processing position (NULL: input order)
    int pool_cap;          // pool form: node entries per wave at most
    int stage_ok;          // boolean results may be staged per wave (4-byte aligned output)
    int deep_cap;          // second pass: entries of a lane's private stack (<= kDeepStack)
    int wave_cap;          // second pass: entries of a wave's shared stack (<= its LDS array)
};

// The first pass in pool form (pool.hip).
void launch_pool(const TravParams &p, int mode, bool cert, hipStream_t s);

namespace {

constexpr float kEtaRel = 0x1p-20f;
constexpr float kBoundK = 12.0f * 0x1p-24f;  // >= 8 u32 (binary32) + 8 u64 (binary64) with slack
constexpr float kBoundTiny = 0x1p-140f;      // absorbs underflow in the products
constexpr int kMiss = 0, kHit = 1, kUnsure = 2;
enum { MODE_BOOL = 0, MODE_FIRST = 1, MODE_BARY = 2, MODE_COUNT = 3 };
// Distinct t that the first pass lists per segment in count mode: binary32 values
// (plain), or intervals of two floats each (certified).  The pool form's lists are
// in LDS; the lane form's in registers, where 11 intervals keep the kernel within
// its 128 VGPRs with few spills (1e7 segments at the paper's scale in that form:
// 6.28 ms with 11, 6.38 with 12).  Segments with more go to the second pass, 27k
// of those 1e7.
template <bool CERT>
constexpr int kCountSlots = CERT ? 11 : 12;

struct Ray {
    float3 o, d;   // start point, direction E - O (rounded)
    float3 inv;    // 1 / direction (components below eta/4 raised to eta/4)
    float3 nra;    // -(O + eta) * inv   (lower box faces)
    float3 nrb;    // -(O - eta) * inv   (upper box faces)
};

__device__ __forceinline__ bool finite3(float3 v) {
    return __builtin_isfinite(v.x) && __builtin_isfinite(v.y) && __builtin_isfinite(v.z);
}

__device__ __forceinline__ float widen_dir(float d, float dmin) {
    return fabsf(d) < dmin ? copysignf(dmin, d) : d;
}

// Returns false for segments whose setup is not finite.
__device__ __forceinline__ bool setup_ray(const float *__restrict__ from, const float *__restrict__ to,
                                          int64_t i, float scale, Ray &r) {
    // streamed once: non-temporal, so the segments do not push the tree out of L2
    r.o = make_float3(__builtin_nontemporal_load(from + 3 * i), __builtin_nontemporal_load(from + 3 * i + 1),
                      __builtin_nontemporal_load(from + 3 * i + 2));
    const float3 e = make_float3(__builtin_nontemporal_load(to + 3 * i), __builtin_nontemporal_load(to + 3 * i + 1),
                                 __builtin_nontemporal_load(to + 3 * i + 2));
    r.d = make_float3(e.x - r.o.x, e.y - r.o.y, e.z - r.o.z);
    float m = fmaxf(scale, fmaxf(fmaxf(fabsf(r.o.x), fabsf(r.o.y)), fabsf(r.o.z)));
    m = fmaxf(m, fmaxf(fmaxf(fabsf(e.x), fabsf(e.y)), fabsf(e.z)));
    const float eta = m * kEtaRel;
    const float dmin = 0.25f * eta;
    r.inv = make_float3(1.0f / widen_dir(r.d.x, dmin), 1.0f / widen_dir(r.d.y, dmin), 1.0f / widen_dir(r.d.z, dmin));
    r.nra = make_float3(-((r.o.x + eta) * r.inv.x), -((r.o.y + eta) * r.inv.y), -((r.o.z + eta) * r.inv.z));
    r.nrb = make_float3(-((r.o.x - eta) * r.inv.x), -((r.o.y - eta) * r.inv.y), -((r.o.z - eta) * r.inv.z));
    return finite3(r.o) && finite3(e) && finite3(r.d) && finite3(r.inv) && finite3(r.nra) && finite3(r.nrb) &&
           __builtin_isfinite(eta);
}

// Widened slab test of one box against t in [0, tlimit]; returns the entry t.
__device__ __forceinline__ bool slab(float xlo, float xhi, float ylo, float yhi, float zlo, float zhi,
                                     const Ray &r, float tlimit, float &tenter) {
    const float tx0 = fmaf(xlo, r.inv.x, r.nra.x), tx1 = fmaf(xhi, r.inv.x, r.nrb.x);
    const float ty0 = fmaf(ylo, r.inv.y, r.nra.y), ty1 = fmaf(yhi, r.inv.y, r.nrb.y);
    const float tz0 = fmaf(zlo, r.inv.z, r.nra.z), tz1 = fmaf(zhi, r.inv.z, r.nrb.z);
    const float tmin = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
    const float tmax = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fminf(fmaxf(tz0, tz1), tlimit));
    tenter = tmin;
    return tmin <= tmax;
}

// The same test with the near and far face of each axis given (the lower
// face is the near one for a direction component >= 0, the upper one
// otherwise, with the matching offsets nn / nf of nra / nrb).  For a box with
// lo <= hi the sign picks exactly the operands min / max pick in slab(), so
// the decisions are the same bit for bit; a box that is +inf on every face
// still misses.
// `order` is what the children a segment meets are visited by, the smallest
// first.  Nearest hits: the entry t, since a hit found early shrinks the limit.
// Boolean: minus the length of the segment's way through the box, since the
// longer it is the likelier a hit, and the first hit ends the search (by the entry
// t: 1e7 segments at the paper's scale 1,701 us, by this 1,629; 64 meshes 3,167 and
// 2,990; ways relative to the box, or weighted towards the near: no better).
template <bool ANY>
__device__ __forceinline__ bool slab_nf(float nx, float fx, float ny, float fy, float nz, float fz,
                                        const float3 &inv, const float3 &nn, const float3 &nf, float tlimit,
                                        float &order) {
    const float tnx = fmaf(nx, inv.x, nn.x), tfx = fmaf(fx, inv.x, nf.x);
    const float tny = fmaf(ny, inv.y, nn.y), tfy = fmaf(fy, inv.y, nf.y);
    const float tnz = fmaf(nz, inv.z, nn.z), tfz = fmaf(fz, inv.z, nf.z);
    const float tmin = fmaxf(fmaxf(tnx, tny), fmaxf(tnz, 0.0f));
    const float tmax = fminf(fminf(tfx, tfy), fminf(tfz, tlimit));
    order = ANY ? tmin - tmax : tmin;
    return tmin <= tmax;
}

struct MT32 {
    float det, U, W, T;
    float3 s;
};

// Binary32 Moller-Trumbore quantities.  The grouping into fused operations is
// written out, so that every kernel that has this in it gets the same values (the
// bound below holds for any grouping).
__device__ __forceinline__ float cross1(float a, float b, float c, float d) {  // a b - c d
#pragma clang fp contract(off)
    return __builtin_fmaf(a, b, -(c * d));
}
__device__ __forceinline__ float dot1(float ax, float bx, float ay, float by, float az, float bz) {
#pragma clang fp contract(off)
    return __builtin_fmaf(az, bz, __builtin_fmaf(ax, bx, ay * by));
}
__device__ __forceinline__ MT32 mt32(const Tri &tri, const Ray &r) {
    MT32 m;
    const float3 e1 = make_float3(tri.e1.x, tri.e1.y, tri.e1.z);
    const float3 e2 = make_float3(tri.e2.x, tri.e2.y, tri.e2.z);
    m.s = make_float3(r.o.x - tri.a.x, r.o.y - tri.a.y, r.o.z - tri.a.z);
    const float px = cross1(r.d.y, e2.z, r.d.z, e2.y);
    const float py = cross1(r.d.z, e2.x, r.d.x, e2.z);
    const float pz = cross1(r.d.x, e2.y, r.d.y, e2.x);
    const float qx = cross1(m.s.y, e1.z, m.s.z, e1.y);
    const float qy = cross1(m.s.z, e1.x, m.s.x, e1.z);
    const float qz = cross1(m.s.x, e1.y, m.s.y, e1.x);
    m.det = dot1(e1.x, px, e1.y, py, e1.z, pz);
    m.U = dot1(m.s.x, px, m.s.y, py, m.s.z, pz);
    m.W = dot1(r.d.x, qx, r.d.y, qy, r.d.z, qz);
    m.T = dot1(e2.x, qx, e2.y, qy, e2.z, qz);
    return m;
}

// The binary32 decision, same predicates as the definition.
__device__ __forceinline__ bool decide32(const MT32 &m) {
    if (!(m.det != 0.0f))
        return false;
    const float g = m.det > 0.0f ? 1.0f : -1.0f;
    const float a = g * m.U, b = g * m.W, tt = g * m.T, D = g * m.det;
    return a >= 0.0f && b >= 0.0f && a + b <= D && tt >= 0.0f && tt <= D;
}

// Certified classification.  Every binary32 quantity X (det, U, W, T) is a sum
// of six signed products of three rounded differences, formed with at most 8
// roundings per product; so |X32 - X| <= gamma_8 M(X) with M(X) the same sum
// over absolute values, and the binary64 evaluation obeys the same form with
// unit roundoff 2^-53.  B(X) = 12 * 2^-24 * M(X) covers both with room for the
// roundings of M itself.  For a hit the interval [tlo, thi] holds the exact t
// and the binary64 t.
struct Bounds {
    float d, U, W, T;
};

__device__ __forceinline__ Bounds mt_bounds(const MT32 &m, const Tri &tri, const Ray &r) {
    const float adx = fabsf(r.d.x), ady = fabsf(r.d.y), adz = fabsf(r.d.z);
    const float asx = fabsf(m.s.x), asy = fabsf(m.s.y), asz = fabsf(m.s.z);
    const float a1x = fabsf(tri.e1.x), a1y = fabsf(tri.e1.y), a1z = fabsf(tri.e1.z);
    const float a2x = fabsf(tri.e2.x), a2y = fabsf(tri.e2.y), a2z = fabsf(tri.e2.z);
    const float Pmx = ady * a2z + adz * a2y, Pmy = adz * a2x + adx * a2z, Pmz = adx * a2y + ady * a2x;
    const float Qmx = asy * a1z + asz * a1y, Qmy = asz * a1x + asx * a1z, Qmz = asx * a1y + asy * a1x;
    Bounds b;
    b.d = fmaf(kBoundK, a1x * Pmx + a1y * Pmy + a1z * Pmz, kBoundTiny);
    b.U = fmaf(kBoundK, asx * Pmx + asy * Pmy + asz * Pmz, kBoundTiny);
    b.W = fmaf(kBoundK, adx * Qmx + ady * Qmy + adz * Qmz, kBoundTiny);
    b.T = fmaf(kBoundK, a2x * Qmx + a2y * Qmy + a2z * Qmz, kBoundTiny);
    return b;
}

__device__ __forceinline__ int classify(const MT32 &m, const Tri &tri, const Ray &r, float &tlo, float &thi) {
    const Bounds bb = mt_bounds(m, tri, r);
    const float Bd = bb.d, BU = bb.U, BW = bb.W, BT = bb.T;
    const float aD = fabsf(m.det);
    // a hit needs |U|, |W|, |T| <= |det| in binary64; a sure excess is a sure miss
    const float cap = aD + Bd;
    if (fabsf(m.U) - BU > cap || fabsf(m.W) - BW > cap || fabsf(m.T) - BT > cap)
        return kMiss;
    if (!(aD > Bd))
        return kUnsure;  // sign of det (or det == 0) not certain; also NaN
    const float g = m.det > 0.0f ? 1.0f : -1.0f;
    const float a = g * m.U, b = g * m.W, tt = g * m.T;
    const float w = g * ((m.det - m.U) - m.W);  // D - a - b
    const float z = g * (m.det - m.T);          // D - tt
    const float Bw = Bd + BU + BW + 0x1p-22f * (aD + fabsf(m.U) + fabsf(m.W));
    const float Bz = Bd + BT + 0x1p-22f * (aD + fabsf(m.T));
    if (a < -BU || b < -BW || w < -Bw || tt < -BT || z < -Bz)
        return kMiss;
    if (a > BU && b > BW && w > Bw && tt > BT && z > Bz) {
        tlo = (tt - BT) / (aD + Bd) * (1.0f - 0x1p-21f);
        thi = (tt + BT) / (aD - Bd) * (1.0f + 0x1p-21f);
        return kHit;
    }
    return kUnsure;
}

// Binary64 test in the definition's operation order: differences, cross
// products, dot products summed left to right, no fused operations, correctly
// rounded division.
struct MT64 {
    bool hit;
    double u, v, t;
};

__device__ __forceinline__ MT64 mt64(double ox, double oy, double oz, double ex, double ey, double ez,
                                     const float *__restrict__ V, const int32_t *__restrict__ F, int t) {
#pragma clang fp contract(off)
    const int32_t i0 = F[3 * (int64_t)t], i1 = F[3 * (int64_t)t + 1], i2 = F[3 * (int64_t)t + 2];
    const double Ax = V[3 * (int64_t)i0], Ay = V[3 * (int64_t)i0 + 1], Az = V[3 * (int64_t)i0 + 2];
    const double Bx = V[3 * (int64_t)i1], By = V[3 * (int64_t)i1 + 1], Bz = V[3 * (int64_t)i1 + 2];
    const double Cx = V[3 * (int64_t)i2], Cy = V[3 * (int64_t)i2 + 1], Cz = V[3 * (int64_t)i2 + 2];
    const double dx = ex - ox, dy = ey - oy, dz = ez - oz;
    const double e1x = Bx - Ax, e1y = By - Ay, e1z = Bz - Az;
    const double e2x = Cx - Ax, e2y = Cy - Ay, e2z = Cz - Az;
    const double sx = ox - Ax, sy = oy - Ay, sz = oz - Az;
    const double px = dy * e2z - dz * e2y, py = dz * e2x - dx * e2z, pz = dx * e2y - dy * e2x;
    const double qx = sy * e1z - sz * e1y, qy = sz * e1x - sx * e1z, qz = sx * e1y - sy * e1x;
    const double det = (e1x * px + e1y * py) + e1z * pz;
    const double U = (sx * px + sy * py) + sz * pz;
    const double W = (dx * qx + dy * qy) + dz * qz;
    const double T = (e2x * qx + e2y * qy) + e2z * qz;
    MT64 r{false, 0.0, 0.0, 0.0};
    if (det == 0.0)
        return r;
    const double g = det > 0.0 ? 1.0 : -1.0;
    const double a = g * U, b = g * W, tt = g * T, D = g * det;
    if (a >= 0.0 && b >= 0.0 && a + b <= D && tt >= 0.0 && tt <= D) {
        r.hit = true;
        r.u = U / det;
        r.v = W / det;
        r.t = T / det;
    }
    return r;
}

__device__ __forceinline__ bool valid_tri(const int32_t *__restrict__ F, int64_t nv, int t) {
    const int32_t i0 = F[3 * (int64_t)t], i1 = F[3 * (int64_t)t + 1], i2 = F[3 * (int64_t)t + 2];
    return i0 >= 0 && i1 >= 0 && i2 >= 0 && i0 < nv && i1 < nv && i2 < nv;
}

// Batched form: the mesh of segment i.
__device__ __forceinline__ int mesh_of_segment(const int32_t *__restrict__ ray_off, int n_meshes, int64_t i) {
    int lo = 0, hi = n_meshes - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ray_off[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ void write_count(const Outs &o, int64_t i, int32_t c) {
    if (o.hit)
        o.hit[i] = c > 0 ? 1 : 0;
    o.count[i] = c;
}

__device__ __forceinline__ void write_out(const Outs &o, int64_t i, int mode, int id, float u, float v, float t) {
    if (mode == MODE_COUNT) {
        write_count(o, i, id >= 0 ? 1 : 0);
        return;
    }
    if (o.hit)
        o.hit[i] = id >= 0 ? 1 : 0;
    if (mode != MODE_BOOL)
        o.id[i] = id;
    if (mode == MODE_BARY) {
        o.uvt[3 * i] = id >= 0 ? u : NAN;
        o.uvt[3 * i + 1] = id >= 0 ? v : NAN;
        o.uvt[3 * i + 2] = id >= 0 ? t : NAN;
    }
}

__device__ __forceinline__ void enqueue(const TravParams &p, int64_t i, int why) {
    const uint32_t slot = atomicAdd(p.queue_len, 1u);
    p.queue[slot] = (int32_t)i;
    atomicAdd(p.counters + why, 1ull);
}


// Pointers into LDS by address space, so reads of the LDS copy of the tree's
// top compile to ds_read and are not merged with the global path.
typedef const __attribute__((address_space(3))) char *LdsBytes;
typedef float F4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 lds_f4(LdsBytes p) {
    const F4v v = *reinterpret_cast<const __attribute__((address_space(3))) F4v *>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

typedef __attribute__((address_space(3))) int *LdsInt;

// A 4-wide node as a segment sees it: each row a face of all four children,
// near and far faces chosen by the segment's signs (offx, offy, offz: byte
// offsets of the near rows, the far row being the other of each pair).  The
// first top_n nodes come from LDS, where the tree's top lies from address 0, so
// that a node's byte offset is its address there too; the others are at 32-bit
// offsets from the tree's first node (nodes4 follows top4: one address for both
// kinds of reference), or, from 4 GB of nodes on (far), at 64-bit addresses.
struct NodeRows {
    float4 nx, fx, ny, fy, nz, fz;
    int4 ch;
};
__device__ __forceinline__ float4 node_row(const char *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ bool far_nodes(int64_t nt) {
    return (nt + kTopSlots) * (int64_t)sizeof(Node4) > INT64_C(0xffffffff);
}
__device__ __forceinline__ NodeRows fetch_node(const Node4 *__restrict__ top4, int ref, int top_n, bool far, int offx,
                                               int offy, int offz) {
    NodeRows r;
    const uint32_t at = (uint32_t)ref << 7;
    auto fetch = [&](auto row) {
        r.nx = row(at + offx);
        r.fx = row(at + (offx ^ 16));
        r.ny = row(at + offy);
        r.fy = row(at + (offy ^ 16));
        r.nz = row(at + offz);
        r.fz = row(at + (offz ^ 16));
        const float4 cf = row(at + 96u);
        r.ch = make_int4(__float_as_int(cf.x), __float_as_int(cf.y), __float_as_int(cf.z), __float_as_int(cf.w));
    };
    if (ref < top_n)
        fetch([](uint32_t o) { return lds_f4((LdsBytes)o); });
    else if (!far)
        fetch([&](uint32_t o) { return node_row(reinterpret_cast<const char *>(top4) + o); });
    else  // (o - at: the row's offset in the node)
        fetch([&](uint32_t o) { return node_row(reinterpret_cast<const char *>(top4 + ref) + (o - at)); });
    // (the references are moved into their keys here, not in the branches,
    // which would wait for the loads there)
    asm("" : "+v"(r.ch.x), "+v"(r.ch.y), "+v"(r.ch.z), "+v"(r.ch.w));
    return r;
}

// A child's sort key: its order (slab_nf; +inf if the segment misses it) as the
// high word of a double, its reference as the low word.  Doubles order as their
// high words do as floats, and an infinite float makes a finite double, so two
// instructions exchange keys and references together where comparing the floats
// took a compare, a minimum, a maximum and two selects; equal t order by the
// references.  (Instructions, not fmin / fmax: those would first quiet
// signalling NaNs, which no key is.)
__device__ __forceinline__ double sort_key(bool h, float t, int c) {
    return __hiloint2double(h ? __float_as_int(t) : 0x7f800000, c);
}
__device__ __forceinline__ int key_child(double k) { return __double2loint(k); }
__device__ __forceinline__ void order2(double &a, double &b) {
    double lo, hi;
    asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(a), "v"(b));
    asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(a), "v"(b));
    a = lo;
    b = hi;
}

}  // namespace
}  // namespace rsi
