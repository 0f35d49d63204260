// Device-side building blocks of the gfx950 path tracer: vector math, Philox
// streams, decision hash, BVH traversal with LDS-staged stacks, the
// Torrance-Sparrow BRDF (evaluation, sampling, pdf and reverse-mode
// derivative), environment-map sampling, and the path estimator used by the
// adjoint replay and by the edge side paths.
//
// Method: Shape from Tracing, Sec. 3.2 (a differentiable physically based path
// tracer R(x, c_i) with gradients of pixels w.r.t. geometry) and Sec. 3.3
// (per-facet Torrance-Sparrow materials; global illumination).  The estimator is
// fixed by the library's stream and shading specification: point lights are
// all sampled at every vertex, one environment sample per vertex is combined
// with BRDF sampling by the balance heuristic, the BRDF is a Lambertian term
// plus a Beckmann / Smith microfacet lobe scaled by the specular colour.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace st {

constexpr float PI_F = 3.14159265358979323846f;
constexpr float INV_PI_F = 0.318309886183790671538f;
constexpr float INV_SQRT_PI_F = 0.564189583547756286948f;
constexpr float TMIN = 1e-4f;
constexpr float SHADOW_SHRINK = 1e-4f;
constexpr float ALPHA_MIN = 1e-3f;
constexpr float LOBE_SPEC_P = 0.5f;
constexpr double EPS_PRIMARY = 1e-3;    // pixels
constexpr float EPS_SECONDARY = 1e-4f;  // radians
constexpr double ZNEAR = 1e-3;
constexpr float SEC_COS_MIN = 1e-5f;    // secondary edge points this close to the tangent plane are skipped
constexpr float BOX_GROW = 1.0000004f;  // 1 + 2*gamma(3): conservative slab exit distance
#ifndef ST_LDS_STACK
#define ST_LDS_STACK 16
#endif
constexpr int LDS_STACK = ST_LDS_STACK; // per-lane traversal stack entries held in LDS
constexpr int SPILL_STACK = 64 - LDS_STACK;  // further entries spilled to HBM (64 in all)
constexpr int TRAV_BLOCK = 256;              // threads of every block that traverses (LDS stack stride)
constexpr uint32_t LEAF_BIT = 0x80000000u;
constexpr int MAX_LIGHTS = 16;
// slots of the traversal work counters (node visits, triangle tests, rays each):
// extension rays and shadow rays wherever traced, the adjoint, the single-kernel
// forward, and (counted a second time) the rays of the paired launch
constexpr int WORK_EXTEND = 0, WORK_SHADOW = 1, WORK_ADJOINT = 2, WORK_MEGA = 3, WORK_PAIR = 4, WORK_SLOTS = 5;

// error word bits (device -> host)
constexpr uint32_t ERR_STACK = 1u;
constexpr uint32_t ERR_NAN = 2u;
constexpr uint32_t ERR_QUEUE = 4u;
constexpr uint32_t ERR_LOOP = 8u;
constexpr int TRAVERSAL_CAP = 1 << 22;   // node visits per ray before the traversal gives up

// ---------------------------------------------------------------------------
struct V3 { float x, y, z; };
__device__ __forceinline__ V3 mk(float x, float y, float z) { return V3{x, y, z}; }
__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return V3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return V3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator-(V3 a) { return V3{-a.x, -a.y, -a.z}; }
__device__ __forceinline__ V3 operator*(V3 a, float s) { return V3{a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ V3 mul(V3 a, V3 b) { return V3{a.x * b.x, a.y * b.y, a.z * b.z}; }
__device__ __forceinline__ float dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
    return V3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ float len(V3 a) { return sqrtf(dot(a, a)); }
__device__ __forceinline__ V3 normalize(V3 a) { return a * (1.0f / len(a)); }
__device__ __forceinline__ float hsum(V3 a) { return a.x + a.y + a.z; }
template <class P> __device__ __forceinline__ V3 ld3(P p) { return V3{p[0], p[1], p[2]}; }
__device__ __forceinline__ V3 xyz(float4 a) { return V3{a.x, a.y, a.z}; }

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                        uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
        // one 64-bit product each: high and low word from a single quarter-rate multiply
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
    }
    return make_uint4(c0, c1, c2, c3);
}
__device__ __forceinline__ float unif(uint32_t r) { return (float)(r >> 8) * (1.0f / 16777216.0f); }

struct Ctr { uint32_t c0, c1, c2hi, c3; };
struct Key { uint32_t k0, k1; };

__device__ __forceinline__ float4 draw4(const Ctr& c, uint32_t bounce, uint32_t block, const Key& k) {
    uint4 r = philox(c.c0, c.c1, c.c2hi | (bounce << 8) | block, c.c3, k.k0, k.k1);
    return make_float4(unif(r.x), unif(r.y), unif(r.z), unif(r.w));
}

// FNV-1a over the little-endian bytes of 32-bit decision words
struct Hash {
    uint32_t h;
    bool on;
    __device__ void push(uint32_t w) {
        if (!on) return;
#pragma unroll
        for (int b = 0; b < 4; ++b) { h ^= (w >> (8 * b)) & 0xFFu; h *= 0x01000193u; }
    }
};
constexpr uint32_t FNV_INIT = 0x811C9DC5u;

// ---------------------------------------------------------------------------
// scene as the kernels see it
// ---------------------------------------------------------------------------
// one bin of the environment alias table: texel k of bin k is kept when the
// second uniform is below prob, otherwise the bin's alias texel is taken
struct __align__(16) EnvAlias {
    double prob;
    int alias;
    int pad;
};

// A pointer kept in a struct in memory, of which device code knows that it points to
// global memory: its loads are global, not flat (a flat load also occupies the LDS
// path, and its waits cannot be told from those of LDS accesses).
#if defined(__HIP_DEVICE_COMPILE__)
#define ST_GLOBAL __attribute__((address_space(1)))
#else
#define ST_GLOBAL
#endif
template <class T> struct GPtr {
    T* p;
    __host__ __device__ __forceinline__ GPtr& operator=(T* q) { p = q; return *this; }
    __host__ __device__ __forceinline__ operator T ST_GLOBAL*() const { return (T ST_GLOBAL*)p; }
};

struct DevScene {
    GPtr<const float> V;       // [nv,3]
    GPtr<const int> F;         // [nf,3]
    GPtr<const float> mat;     // [nf,7]
    GPtr<const float> lights;  // [nl,6]
    GPtr<const float4> fnorm;  // [nf] unit geometric normal
    GPtr<const float4> tri;    // [nf*3] node-ordered (v0, face bits) (e1) (e2)
    GPtr<const int> fleaf;     // [nf] record of each face in tri
    GPtr<const float4> nodes4; // 4-wide nodes, 8 float4 each: SoA child boxes + where the children start
    GPtr<const float> env;     // [he,we,3]
    GPtr<const double> marg;   // [he+1]
    GPtr<const double> cond;   // [he,we+1]
    GPtr<const float> texpdf;  // [he*we] solid-angle pdf of each texel
    GPtr<const float> rowcos;  // [2*(he+1)]: 1 - cos(pi r / he), then 1 + cos(pi r / he)
    GPtr<const int4> edges;    // [ne] (va, vb, f1, f2)
    GPtr<const double> ecdf;   // [ne+1] cumulative 3-D length / total
    GPtr<const float> etotal;  // total 3-D edge length
    GPtr<const int> eguide;    // guide table of ecdf, 2^eglog entries
    GPtr<const int> mguide;    // guide table of the env marginal CDF, 2^mglog entries
    GPtr<const int> cguide;    // guide tables of the env conditional CDFs, 2^cglog entries per row
    GPtr<const int> etchild;   // secondary-edge importance tree: children [ne-1, 2]
    GPtr<const float> etbox;   // node boxes [2ne-1, 6] (internal nodes, then leaves)
    GPtr<const float> etlen;   // node length sums [2ne-1]
    GPtr<const float> etnbox;  // node boxes of the adjacent faces' unit normals [2ne-1, 6]
    GPtr<const float4> etnode; // per internal node, both children's box, length, normal box and code
                          // in one 128-B record (8 float4, layout of k_epack) [ne-1]
    GPtr<const uint32_t> etedge; // sorted leaf -> edge
    GPtr<const EnvAlias> ealias; // [he*we] alias table of the texel probabilities, used when env_alias
    int env_alias;
    int vndf;             // specular lobe sampled from the visible normals
    int eglog, mglog, cglog;
    int nv, nf, nl, he, we, ne, has_env;
    int tex_res;          // mesh-colours resolution r: mat has nf (r+1)(r+2)/2 rows
    uint32_t scene_id;
};

// per-lane traversal stack: LDS_STACK entries in LDS (lane-interleaved), the
// rest in a per-thread HBM spill region
// address-space-qualified views: loads through them compile to global_load /
// ds_read instead of generic flat accesses
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const vf4 gfloat4;
typedef __attribute__((address_space(1))) uint32_t gu32;
typedef __attribute__((address_space(3))) uint32_t lu32;

struct TravStack {
    lu32* lds;         // this lane's LDS stack column: entry i at lds[i * TRAV_BLOCK]
    gu32* spill;       // spill base; entry i of thread g at spill[i*gstride + g]
    uint32_t gstride, gid;
    uint32_t* err;
    unsigned long long* work;   // optional: node visits, triangle tests, rays
    unsigned long long* work2;  // optional: a second set of the same counters
    __device__ __forceinline__ void put(int i, uint32_t v) {
        if (i < LDS_STACK) lds[i * TRAV_BLOCK] = v;
        else spill[(i - LDS_STACK) * gstride + gid] = v;
    }
    __device__ __forceinline__ uint32_t get(int i) const {
        if (i < LDS_STACK) return lds[i * TRAV_BLOCK];
        return spill[(i - LDS_STACK) * gstride + gid];
    }
    __device__ __forceinline__ bool push1(int& sp, uint32_t v) {
        if (sp >= LDS_STACK + SPILL_STACK) return false;
        put(sp++, v);
        return true;
    }
    // pushes m (0..3) entries: a, then b, then c; entries beyond the m-th are
    // written too when they stay in LDS (above the new top, so never read)
    __device__ __forceinline__ bool push3(int& sp, int m, uint32_t a, uint32_t b, uint32_t c) {
        if (sp + 3 <= LDS_STACK) {
            lds[sp * TRAV_BLOCK] = a;
            lds[(sp + 1) * TRAV_BLOCK] = b;
            lds[(sp + 2) * TRAV_BLOCK] = c;
            sp += m;
            return true;
        }
        if (sp + m > LDS_STACK + SPILL_STACK) return false;
        if (m > 0) put(sp++, a);
        if (m > 1) put(sp++, b);
        if (m > 2) put(sp++, c);
        return true;
    }
};

__device__ __forceinline__ TravStack make_trav_stack(uint32_t* lds, uint32_t* spill, uint32_t* err,
                                                     unsigned long long* work) {
    TravStack s;
    // the stack layout assumes TRAV_BLOCK threads per block
    if (blockDim.x != TRAV_BLOCK && threadIdx.x == 0) atomicOr(err, ERR_STACK);
    s.lds = (lu32*)lds + threadIdx.x;
    s.spill = (gu32*)spill;
    s.gstride = gridDim.x * blockDim.x;
    s.gid = blockIdx.x * blockDim.x + threadIdx.x;
    s.err = err;
    s.work = work;
    s.work2 = nullptr;
    return s;
}

// The geometry one traversal reads.  Where every ray of a launch is of one scene
// the pointers are wave-uniform (scalar registers): a node or triangle load is then
// a scalar base plus a 32-bit lane offset.  Rays of several scenes share waves (the
// compacted queues mix them), so there each lane keeps its own pointers.
typedef __attribute__((address_space(1))) const char gchar;
struct TraceGeo {
    const gchar* nodes;
    const gchar* tri;
    int nf;
};
__device__ __forceinline__ const gchar* uniform_ptr(const void* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (const gchar*)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ TraceGeo lane_geo(const DevScene& S) {
    return TraceGeo{(const gchar*)S.nodes4.p, (const gchar*)S.tri.p, S.nf};
}
// of a scene that is the same for every active lane
__device__ __forceinline__ TraceGeo wave_geo(const DevScene& S) {
    return TraceGeo{uniform_ptr(S.nodes4.p), uniform_ptr(S.tri.p), __builtin_amdgcn_readfirstlane(S.nf)};
}

// FAST traversals address nodes and triangles by 32-bit byte offsets, start at
// the constant TMIN and count no work; the others (scenes of more than
// TRAV_FAST_FACES faces, another tmin, or with work counters) use 64-bit offsets
// from the node or triangle index.  Both visit the same nodes in the same order.
constexpr int TRAV_FAST_FACES = 1 << 25;      // 128 B nodes, at most one per face: offsets below 2^32
constexpr uint32_t NODE_BYTES = 128, TRI_BYTES = 48;
constexpr float FAST_TFAR = 0x1.a36e2ap+114f;    // the largest distance a FAST key holds (bits of TMIN + 2^30 - 2)

// Moller-Trumbore, two-sided, on one triangle record.  Every rounding is written
// out: which of two triangles a ray near their common edge meets first hangs on
// them, and left to contraction the order of the two products that start the
// first barycentric sum differed from one call site to another.  YFIRST: that sum
// starts from the y product (the tests outside a traversal: a side ray's edge faces,
// the brute-force search), else from x.  Whether a ray within a rounding of a
// triangle's edge meets it can so differ between the two; t is the same in both.
template <bool YFIRST = false>
__device__ __forceinline__ bool tri_test(const gchar* rec, V3 o, V3 d, float tmin, float tmax, float& t, int& face) {
#pragma clang fp contract(off)
    const gfloat4* const r = (const gfloat4*)rec;
    const vf4 a = r[0], e1 = r[1], e2 = r[2];
    const V3 p{__builtin_fmaf(d.y, e2.z, -(d.z * e2.y)), __builtin_fmaf(d.z, e2.x, -(d.x * e2.z)),
               __builtin_fmaf(d.x, e2.y, -(d.y * e2.x))};
    const float det = __builtin_fmaf(e1.z, p.z, __builtin_fmaf(e1.x, p.x, e1.y * p.y));
    if (det == 0.0f) return false;
    const float inv = 1.0f / det;
    const V3 s{o.x - a.x, o.y - a.y, o.z - a.z};
    const float sp = YFIRST ? __builtin_fmaf(s.x, p.x, s.y * p.y) : __builtin_fmaf(s.y, p.y, s.x * p.x);
    const float b1 = __builtin_fmaf(s.z, p.z, sp) * inv;
    if (b1 < 0.0f || b1 > 1.0f) return false;
    const V3 q{__builtin_fmaf(s.y, e1.z, -(s.z * e1.y)), __builtin_fmaf(s.z, e1.x, -(s.x * e1.z)),
               __builtin_fmaf(s.x, e1.y, -(s.y * e1.x))};
    const float dq = __builtin_fmaf(d.z, q.z, __builtin_fmaf(d.x, q.x, d.y * q.y));
    if (dq * inv < 0.0f || __builtin_fmaf(dq, inv, b1) > 1.0f) return false;
    t = __builtin_fmaf(e2.z, q.z, __builtin_fmaf(e2.x, q.x, e2.y * q.y)) * inv;
    face = __float_as_int(a.w);
    return t > tmin && t < tmax;
}
__device__ __forceinline__ const gchar* tri_at(const gchar* tri, uint32_t i) { return tri + (size_t)i * TRI_BYTES; }

// distance along o + t d to the plane of face f, with the arithmetic of the
// triangle test (the hit distance of a recorded hit)
__device__ __forceinline__ float face_hit_t(const DevScene& S, int f, V3 o, V3 d) {
    const V3 a = ld3(S.V + 3 * (size_t)S.F[3 * f]);
    const V3 e1 = ld3(S.V + 3 * (size_t)S.F[3 * f + 1]) - a, e2 = ld3(S.V + 3 * (size_t)S.F[3 * f + 2]) - a;
    const V3 p = cross(d, e2);
    const float inv = 1.0f / dot(e1, p);
    const V3 q = cross(o - a, e1);
    return dot(e2, q) * inv;
}

__device__ __forceinline__ V3 safe_inv(V3 d) {
    auto f = [](float v) { return 1.0f / (fabsf(v) > 1e-30f ? v : copysignf(1e-30f, v)); };
    return V3{f(d.x), f(d.y), f(d.z)};
}

// A ray as the slab tests read it: origin, reciprocal direction, and for each
// axis the byte offset (0 or 16) of its near planes inside a node's pair of
// plane vectors: with them no plane pair has to be ordered by min and max.
struct RayBox {
    V3 o, inv;
    uint32_t sx, sy, sz;
};
__device__ __forceinline__ RayBox ray_box(V3 o, V3 d) {
    RayBox r;
    r.o = o;
    r.inv = safe_inv(d);
    r.sx = (__float_as_uint(r.inv.x) >> 27) & 16u;
    r.sy = (__float_as_uint(r.inv.y) >> 27) & 16u;
    r.sz = (__float_as_uint(r.inv.z) >> 27) & 16u;
    return r;
}

// Slab tests of the 4 child boxes of one 4-wide node (layout of k_pack4).  The
// traversal issues vector instructions most of its time (62-89 % of the SIMD
// cycles at 8 views of 256^2, 16 spp), so what counts is instructions per visit:
// planes picked by the ray's signs instead of ordered, leaves and children named
// by slot instead of by loaded codes, scalar base addresses.  Extension launch
// 4.43e8 -> 3.6e8 instructions, paired launch 7.12e8 -> 5.6e8; the latter
// 1295 -> 1204 us, a render of those views 3.46 -> 3.30 ms, the 40k-face step of
// 16 views of 512^2 99.5 -> 95.2 ms.  A
// node's internal children are consecutive nodes in consecutive slots, its leaf
// children consecutive triangles likewise, so a child is named by its slot: no
// child codes are loaded, selected or sorted.  t[s]: entry distance of slot s
// (hit or not); hit and inner: masks of the slots whose box is hit and of the
// internal ones.  node and first: byte offsets (FAST) or indices of the node and
// of what slot 0's node would be; tri0 likewise of slot 0's triangle.
template <bool FAST>
__device__ __forceinline__ void node4_test(const TraceGeo& G, uint32_t node, const RayBox& r, float tmin, float tmax,
                                           float t[4], bool hit[4], bool inner[4], uint32_t& first, uint32_t& tri0) {
    vf4 nx, fx, ny, fy, nz, fz, cc;
    if constexpr (FAST) {
        const uint32_t ox = node | r.sx, oy = node | r.sy, oz = node | r.sz;
        nx = *(const gfloat4*)(G.nodes + ox);      fx = *(const gfloat4*)(G.nodes + (ox ^ 16u));
        ny = *(const gfloat4*)(G.nodes + oy + 32); fy = *(const gfloat4*)(G.nodes + (oy ^ 16u) + 32);
        nz = *(const gfloat4*)(G.nodes + oz + 64); fz = *(const gfloat4*)(G.nodes + (oz ^ 16u) + 64);
        cc = *(const gfloat4*)(G.nodes + node + 96);
    } else {
        const gchar* const n = G.nodes + (size_t)node * NODE_BYTES;
        nx = *(const gfloat4*)(n + r.sx);      fx = *(const gfloat4*)(n + (r.sx ^ 16u));
        ny = *(const gfloat4*)(n + r.sy + 32); fy = *(const gfloat4*)(n + (r.sy ^ 16u) + 32);
        nz = *(const gfloat4*)(n + r.sz + 64); fz = *(const gfloat4*)(n + (r.sz ^ 16u) + 64);
        cc = *(const gfloat4*)(n + 112);
    }
    first = __float_as_uint(cc.x);
    tri0 = __float_as_uint(cc.y);
    // ni internal slots from 0, or (-1) slots 1..3
    const int ni = __float_as_int(cc.z);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const float ax = (nx[s] - r.o.x) * r.inv.x, bx = (fx[s] - r.o.x) * r.inv.x;
        const float ay = (ny[s] - r.o.y) * r.inv.y, by = (fy[s] - r.o.y) * r.inv.y;
        const float az = (nz[s] - r.o.z) * r.inv.z, bz = (fz[s] - r.o.z) * r.inv.z;
        const float tn = fmaxf(fmaxf(ax, ay), az);
        t[s] = FAST ? __builtin_amdgcn_fmed3f(tn, tmin, FAST_TFAR) : fmaxf(tn, tmin);
        const float t1 = fminf(fminf(bx, by), fminf(bz, tmax)) * BOX_GROW;
        hit[s] = t[s] <= t1;
        inner[s] = s == 0 ? ni > 0 : (uint32_t)ni > (uint32_t)s;
    }
}
// FAST sorts entry distances as integers that carry their slot: bits(t) -
// bits(TMIN), below 2^30 for t in [TMIN, FAST_TFAR], above the two slot bits,
// so the distance is exact.  (Entry distances are clamped to FAST_TFAR = 3.4e34,
// which only keeps boxes, and the far limit of the keys with them.)
constexpr uint32_t TMIN_BITS = 0x38d1b717u;                     // bits of 1e-4f
constexpr uint32_t KEY_MISS = 0xffffffffu;
__device__ __forceinline__ uint32_t dist_key(float t, uint32_t slot) {
    return (__float_as_uint(t) << 2) + (slot - (TMIN_BITS << 2));
}
__device__ __forceinline__ uint32_t leaf_mask(const bool hit[4], const bool inner[4]) {
    uint32_t m = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) m |= hit[s] && !inner[s] ? 1u << s : 0u;
    return m;
}
template <bool FAST> __device__ __forceinline__ uint32_t child_node(uint32_t first, uint32_t slot) {
    return first + slot * (FAST ? NODE_BYTES : 1u);
}
template <bool FAST> __device__ __forceinline__ const gchar* child_tri(const TraceGeo& G, uint32_t tri0, uint32_t slot) {
    if constexpr (FAST) return G.tri + (uint32_t)(tri0 + __umul24(slot, TRI_BYTES));
    else return G.tri + (size_t)(uint32_t)(tri0 + slot) * TRI_BYTES;
}
__device__ __forceinline__ void cswap(float& ta, uint32_t& ca, float& tb, uint32_t& cb) {
    if (tb < ta) {
        const float t = ta; ta = tb; tb = t;
        const uint32_t c = ca; ca = cb; cb = c;
    }
}
// The order in which a closest-hit traversal takes the internal children (key
// form: slot in the low two bits): by entry distance, ties as the exchange
// network (0 1)(2 3)(0 2)(1 3)(1 2) with strict comparisons leaves them.  Which
// of two triangles met within a rounding of the same distance is found first
// decides which box the running best hit culls, so ties are part of the result.
// The first four exchanges never meet an equal distance in descending slots, so
// minima and maxima of the keys make them; the last compares distances alone.
__device__ __forceinline__ void sort_keys(uint32_t k[4]) {
    const uint32_t a0 = min(k[0], k[1]), a1 = max(k[0], k[1]), a2 = min(k[2], k[3]), a3 = max(k[2], k[3]);
    const uint32_t b1 = min(a1, a3), b2 = max(a0, a2);
    const bool swap = b2 < (b1 & ~3u);
    k[0] = min(a0, a2);
    k[1] = swap ? b2 : b1;
    k[2] = swap ? b1 : b2;
    k[3] = max(a1, a3);
}
__device__ __forceinline__ void count_work(const TravStack& st, uint32_t visits, uint32_t tests) {
    for (unsigned long long* w : {st.work, st.work2})
        if (w) {
            atomicAdd(w, (unsigned long long)visits);
            atomicAdd(w + 1, (unsigned long long)tests);
            atomicAdd(w + 2, 1ull);
        }
}

// closest hit with t in (tmin, inf) excluding one face; ties go to the smaller face id.
// (t0, f0): a hit already known (f0 >= 0), which prunes the traversal and is its
// result unless a nearer one is met; tested YFIRST, it can be one that the
// traversal's own test lets pass by a rounding at the triangle's edge
template <bool FAST = false>
__device__ int trace_closest(const TraceGeo& G, V3 o, V3 d, float tmin, int exclude, float& thit, TravStack& st,
                             float t0 = __int_as_float(0x7f800000), int f0 = -1) {
    const float INF = __int_as_float(0x7f800000);
    float tbest = t0;
    int best = f0;
    if (G.nf <= 0) return -1;
    uint32_t tests = 0;
    auto leaf = [&](const gchar* rec) {
        if (!FAST) ++tests;
        float t; int f;
        if (tri_test(rec, o, d, tmin, INF, t, f) && f != exclude) {
            if (t < tbest || (t == tbest && f < best)) { tbest = t; best = f; }
        }
    };
    if (G.nf == 1) { leaf(G.tri); thit = tbest; return best; }
    const RayBox r = ray_box(o, d);
    uint32_t node = 0;
    int sp = 0;
    int iter = 0;
    for (;; ++iter) {
        if (iter >= TRAVERSAL_CAP) { atomicOr(st.err, ERR_LOOP); break; }
        float t[4];
        bool hit[4], inner[4];
        uint32_t first, tri0;
        node4_test<FAST>(G, node, r, FAST ? TMIN : tmin, tbest, t, hit, inner, first, tri0);
        uint32_t k[4];
        if (FAST) {
#pragma unroll
            for (int s = 0; s < 4; ++s) k[s] = hit[s] && inner[s] ? dist_key(t[s], (uint32_t)s) : KEY_MISS;
        }
        // hit leaf slots, tested in slot order at one site (a wave runs the
        // largest per-lane count of leaf tests, not one block per slot)
        for (uint32_t lv = leaf_mask(hit, inner); lv; lv &= lv - 1)
            leaf(child_tri<FAST>(G, tri0, (uint32_t)__builtin_ctz(lv)));
        // the hit internal slots not beyond the best hit, nearest first
        bool h0, h1, h2, h3;
        if (FAST) {
            sort_keys(k);
            const uint32_t kmax = dist_key(fminf(tbest, FAST_TFAR), 3u);
            h0 = k[0] <= kmax; h1 = k[1] <= kmax; h2 = k[2] <= kmax; h3 = k[3] <= kmax;
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                k[s] = (uint32_t)s;
                if (!(hit[s] && inner[s]) || t[s] > tbest) t[s] = INF;
            }
            cswap(t[0], k[0], t[1], k[1]); cswap(t[2], k[2], t[3], k[3]);
            cswap(t[0], k[0], t[2], k[2]); cswap(t[1], k[1], t[3], k[3]);
            cswap(t[1], k[1], t[2], k[2]);
            h0 = t[0] < INF; h1 = t[1] < INF; h2 = t[2] < INF; h3 = t[3] < INF;
        }
        if (h0) {
            // push the hit slots m-1 .. 1 of the order (farthest first)
            const int m = (int)h1 + (int)h2 + (int)h3;
            const uint32_t a = h3 ? k[3] : (h2 ? k[2] : k[1]);
            const uint32_t b = h3 ? k[2] : k[1];
            if (!st.push3(sp, m, child_node<FAST>(first, a & 3u), child_node<FAST>(first, b & 3u),
                          child_node<FAST>(first, k[1] & 3u))) {
                atomicOr(st.err, ERR_STACK);
                break;
            }
            node = child_node<FAST>(first, k[0] & 3u);
        } else {
            if (sp == 0) break;
            node = st.get(--sp);
        }
    }
    // node visits: one per iteration (the cap exit visits none)
    if (!FAST) count_work(st, (uint32_t)min(iter + 1, TRAVERSAL_CAP), tests);
    thit = tbest;
    return best;
}

template <bool FAST>
__device__ bool trace_any_impl(const TraceGeo& G, V3 o, V3 d, float tmin, float tmax, int exclude, TravStack& st,
                               uint32_t& visits, uint32_t& tests) {
    if (G.nf <= 0) return false;
    auto leaf = [&](const gchar* rec) -> bool {
        if (!FAST) ++tests;
        float t; int f;
        return tri_test(rec, o, d, tmin, tmax, t, f) && f != exclude;
    };
    if (G.nf == 1) return leaf(G.tri);
    const RayBox r = ray_box(o, d);
    uint32_t node = 0, group = 0;
    int sp = 0;
    for (int iter = 0;; ++iter) {
        if (iter >= TRAVERSAL_CAP) { atomicOr(st.err, ERR_LOOP); return false; }
        if (!FAST) ++visits;
        float t[4];
        bool hit[4], inner_s[4];
        uint32_t first, tri0;
        node4_test<FAST>(G, node, r, FAST ? TMIN : tmin, tmax, t, hit, inner_s, first, tri0);
        for (uint32_t lv = leaf_mask(hit, inner_s); lv; lv &= lv - 1)
            if (leaf(child_tri<FAST>(G, tri0, (uint32_t)__builtin_ctz(lv)))) return true;
        uint32_t inner = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) inner |= hit[s] && inner_s[s] ? 1u << s : 0u;
        if constexpr (FAST) {
            // the siblings still to visit form one group: the byte offset of slot 0's
            // node with their slot mask in its low bits; one entry holds a group
            if (inner) {
                if (group & 15u) {
                    if (!st.push1(sp, group)) { atomicOr(st.err, ERR_STACK); return false; }
                }
                group = first | inner;
            } else if (!(group & 15u)) {
                if (sp == 0) return false;
                group = st.get(--sp);
            }
            const uint32_t s = (uint32_t)__builtin_ctz(group);
            node = child_node<FAST>(group & ~15u, s);
            group &= group - 1;
        } else {
            // the first hit slot is visited next, the others are pushed in slot order
            if (inner) {
                node = first + (uint32_t)__builtin_ctz(inner);
                for (inner &= inner - 1; inner; inner &= inner - 1)
                    if (!st.push1(sp, first + (uint32_t)__builtin_ctz(inner))) { atomicOr(st.err, ERR_STACK); return false; }
            } else {
                if (sp == 0) return false;
                node = st.get(--sp);
            }
        }
    }
}

template <bool FAST = false>
__device__ __forceinline__ bool trace_any(const TraceGeo& G, V3 o, V3 d, float tmin, float tmax, int exclude,
                                          TravStack& st) {
    uint32_t visits = 0, tests = 0;
    const bool r = trace_any_impl<FAST>(G, o, d, tmin, tmax, exclude, st, visits, tests);
    if (!FAST) count_work(st, visits, tests);
    return r;
}

// ---------------------------------------------------------------------------
// Torrance-Sparrow BRDF: kd/pi + ks * D * G / (4 cos_i cos_o), Beckmann D,
// height-correlated Smith G of the Beckmann surface.
// ---------------------------------------------------------------------------
struct Mat { V3 kd, ks; float a; };
template <class P> __device__ __forceinline__ Mat load_mat(P m) {
    Mat r;
    r.kd = V3{m[0], m[1], m[2]};
    r.ks = V3{m[3], m[4], m[5]};
    r.a = m[6];
    return r;
}
__device__ __forceinline__ float alpha_eff(float a) { return a > ALPHA_MIN ? a : ALPHA_MIN; }

// Material row of the point x on face f.  Mesh colours (Sec. 3.3
// "Representation"): at resolution r the point with barycentric coordinates
// (alpha of the second vertex, beta of the third) uses texel
// f (r+1)(r+2)/2 + i (2r - i + 3)/2 + j, (i, j) = floor(r (alpha, beta)),
// clamped to 0 <= i <= r, 0 <= j <= r - i; r = 0 is one row per face.
__device__ __forceinline__ int texel_of(const DevScene& S, int f, V3 x) {
    const int r = S.tex_res;
    if (r == 0) return f;
    const V3 v0 = ld3(S.V + 3 * S.F[3 * f]), v1 = ld3(S.V + 3 * S.F[3 * f + 1]), v2 = ld3(S.V + 3 * S.F[3 * f + 2]);
    const V3 e1 = v1 - v0, e2 = v2 - v0, q = x - v0;
    const V3 N = cross(e1, e2);
    const float nn = dot(N, N);
    float a = dot(cross(q, e2), N) / nn, b = dot(cross(e1, q), N) / nn;
    a = fminf(fmaxf(a, -1.0f), 2.0f);   // also maps NaN to -1
    b = fminf(fmaxf(b, -1.0f), 2.0f);
    int i = (int)floorf((float)r * a), j = (int)floorf((float)r * b);
    i = min(max(i, 0), r);
    j = min(max(j, 0), r - i);
    return (f * (r + 1) * (r + 2) + i * (2 * r - i + 3)) / 2 + j;
}

// Beckmann D with tan^2 taken from |n x h|^2 / (n.h)^2: 1 - (n.h)^2 cancels in
// float32 near the highlight, the cross product does not
__device__ __forceinline__ float beckmann_D(V3 n, V3 h, float ch, float a) {
    const float c2 = ch * ch;
    const V3 nh = cross(n, h);
    const float t2 = dot(nh, nh) / c2;
    return expf(-t2 / (a * a)) / (PI_F * a * a * c2 * c2);
}

__device__ __forceinline__ float smith_lambda(float c, float a) {
    if (c >= 1.0f) return 0.0f;
    const float s = sqrtf(1.0f - c * c);
    const float x = c / (a * s);
    return (expf(-x * x) * INV_SQRT_PI_F / x - erfcf(x)) * 0.5f;
}

// Lambda(wo) of a shading point, for every evaluation there: an exponential and an
// erfc less in each (only read where n.wo > 0)
__device__ __forceinline__ float out_lambda(V3 wo, V3 n, const Mat& m) {
    const float co = dot(n, wo);
    return co > 0.0f ? smith_lambda(co, alpha_eff(m.a)) : 0.0f;
}

__device__ __forceinline__ V3 brdf_eval(V3 wi, V3 wo, V3 n, const Mat& m, float lambda_o) {
    const float ci = dot(n, wi), co = dot(n, wo);
    if (!(ci > 0.0f) || !(co > 0.0f)) return V3{0.f, 0.f, 0.f};
    const float a = alpha_eff(m.a);
    const V3 h = normalize(wi + wo);
    const float ch = dot(n, h);
    float spec = 0.0f;
    if (ch > 0.0f) {
        const float D = beckmann_D(n, h, ch, a);
        const float G = 1.0f / (1.0f + smith_lambda(ci, a) + lambda_o);
        spec = D * G / (4.0f * ci * co);
    }
    return m.kd * INV_PI_F + m.ks * spec;
}

// f(wi, wo) and the pdf of wi, of the one-sample mixture: 1/2 cosine-weighted + 1/2
// specular, whose half-vectors follow D(h) cos(theta_h), or with vndf the normals
// visible from wo, G1(wo) max(0, wo.h) D(h) / cos(theta_o) (Heitz and d'Eon 2014);
// either becomes a pdf of wi through 1 / (4 |wo.h|).  One half-vector, one D and the
// shading point's Lambda(wo) serve both.
__device__ __forceinline__ V3 brdf_eval_pdf(V3 wi, V3 wo, V3 n, const Mat& m, float lambda_o, bool vndf, float& pdf) {
    const float ci = dot(n, wi), co = dot(n, wo);
    pdf = 0.0f;
    if (!(ci > 0.0f)) return V3{0.f, 0.f, 0.f};
    const float a = alpha_eff(m.a);
    const V3 hv = wi + wo;
    const float hl = len(hv);
    float ps = 0.0f, spec = 0.0f;
    if (hl > 0.0f) {
        const V3 h = hv * (1.0f / hl);
        const float ch = dot(n, h);
        if (ch > 0.0f) {
            const float D = beckmann_D(n, h, ch, a);
            const float oh = dot(wo, h);
            if (!vndf) {
                if (fabsf(oh) > 0.0f) ps = LOBE_SPEC_P * D * ch / (4.0f * fabsf(oh));
            } else if (oh > 0.0f && co > 0.0f) {
                const float g1 = 1.0f / (1.0f + lambda_o);
                ps = LOBE_SPEC_P * g1 * D / (4.0f * co);
            }
            if (co > 0.0f) {
                const float G = 1.0f / (1.0f + smith_lambda(ci, a) + lambda_o);
                spec = D * G / (4.0f * ci * co);
            }
        }
    }
    pdf = (1.0f - LOBE_SPEC_P) * ci * INV_PI_F + ps;
    if (!(co > 0.0f)) return V3{0.f, 0.f, 0.f};
    return m.kd * INV_PI_F + m.ks * spec;
}

// Visible-normal sample of the Beckmann lobe in the local frame (z = normal):
// stretch wo by alpha; for the standard surface seen at cot(theta') = c the
// slope along the incident plane has density ~ (c - x) exp(-x^2) on x < c with
// integral F(x) = c sqrt(pi)/2 erfc(-x) + exp(-x^2)/2, inverted by bracketed
// Newton steps (from below on the lower half of u1, through F(c) - F(x) on the
// upper half); the other slope is erfinv(2 u2 - 1); rotate, unstretch.
constexpr float VNDF_COT_MAX = 1e4f;
constexpr float VNDF_Y_MAX = 1.0f - 1.0f / 8388608.0f;
constexpr float HALF_SQRT_PI_F = 0.886226925452758013649f;
__device__ __forceinline__ V3 vndf_normal(V3 wl, float a, float u1, float u2) {
    const V3 ws = normalize(V3{a * wl.x, a * wl.y, wl.z});
    const float st = sqrtf(ws.x * ws.x + ws.y * ws.y);
    const float cphi = st > 0.0f ? ws.x / st : 1.0f, sphi = st > 0.0f ? ws.y / st : 0.0f;
    const float c = st > 0.0f ? fminf(ws.z / st, VNDF_COT_MAX) : VNDF_COT_MAX;
    const bool upper = u1 > 0.5f;
    const float Fc = c * HALF_SQRT_PI_F * erfcf(-c) + 0.5f * expf(-c * c);
    const float target = (upper ? 1.0f - u1 : u1) * Fc;
    float lo = -8.0f, hi = fminf(c, 8.0f), x = fminf(0.0f, 0.5f * c);   // the root lies below 8
    const float erfc_c = erfcf(c), exp_c = expf(-c * c);
    // At most 24 steps; most lanes settle in 6 to 12.  Once the state of two steps before
    // comes back, at an even step, the steps left only repeat the two, and end on this one:
    // the same result bit for bit (k_shade of a 1024^2 view at 32 spp 1,610 -> 1,465 us;
    // one erfc per step instead of three).
    float lo1 = lo, hi1 = hi, x1 = x, lo2 = lo, hi2 = hi, x2 = __builtin_nanf("");
    for (int it = 0; it < 24; ++it) {
        if (((it & 1) == 0) && x == x2 && lo == lo2 && hi == hi2) break;
        const float ex = expf(-x * x);
        const float er = erfcf(upper ? x : -x);
        const float g = upper ? target - (c * HALF_SQRT_PI_F * (er - erfc_c) + 0.5f * (exp_c - ex))
                              : (c * HALF_SQRT_PI_F * er + 0.5f * ex) - target;
        lo2 = lo1; hi2 = hi1; x2 = x1;
        lo1 = lo; hi1 = hi; x1 = x;
        if (g > 0.0f) hi = x; else lo = x;
        const float dg = (c - x) * ex;
        float xn = dg > 0.0f ? x - g / dg : 0.5f * (lo + hi);
        if (!(xn >= lo && xn <= hi)) xn = 0.5f * (lo + hi);    // a converged step stays put
        x = xn;
    }
    const float y = erfinvf(fmaxf(-VNDF_Y_MAX, fminf(VNDF_Y_MAX, 2.0f * u2 - 1.0f)));
    const float sx = (cphi * x - sphi * y) * a, sy = (sphi * x + cphi * y) * a;
    return normalize(V3{-sx, -sy, 1.0f});
}

// orthonormal basis around n (Duff et al. 2017, branchless)
__device__ __forceinline__ void onb(V3 n, V3& t, V3& b) {
    const float sg = copysignf(1.0f, n.z);
    const float a = -1.0f / (sg + n.z);
    const float bb = n.x * n.y * a;
    t = V3{1.0f + sg * n.x * n.x * a, sg * bb, -sg * n.x};
    b = V3{bb, sg + n.y * n.y * a, -n.y};
}

__device__ __forceinline__ int bsdf_sample(float4 u, V3 wo, V3 n, float alpha, bool vndf, V3& wi) {
    V3 t, b;
    onb(n, t, b);
    const float a = alpha_eff(alpha);
    if (u.x < LOBE_SPEC_P && vndf) {
        const V3 hl = vndf_normal(V3{dot(wo, t), dot(wo, b), dot(wo, n)}, a, u.y, u.z);
        const V3 h = t * hl.x + b * hl.y + n * hl.z;
        wi = h * (2.0f * dot(wo, h)) - wo;
        return 0;
    }
    const float phi = 2.0f * PI_F * u.z;
    float sp, cp;
    sincosf(phi, &sp, &cp);
    if (u.x < LOBE_SPEC_P) {
        const float t2 = -a * a * logf(1.0f - u.y);
        const float ch = 1.0f / sqrtf(1.0f + t2);
        const float sh = sqrtf(t2 / (1.0f + t2));    // sin^2 = tan^2 / (1 + tan^2): no cancellation near the pole
        const V3 h = t * (sh * cp) + b * (sh * sp) + n * ch;
        wi = h * (2.0f * dot(wo, h)) - wo;
        return 0;
    }
    const float r = sqrtf(u.y);
    const float z = sqrtf(fmaxf(0.0f, 1.0f - u.y));
    wi = t * (r * cp) + b * (r * sp) + n * z;
    return 1;
}

// Secondary-edge importance hierarchy.  Node weight seen from the shading
// point p with normal nrm (contraction off, this operation order): zero when the
// node's box lies wholly behind the tangent plane of p (with a margin of 2^-16
// of the box's size plus distance, so that a box lying in the plane keeps its
// weight whatever the rounding of p), or (sil) when no edge in it can be a
// silhouette from p: the bound of N.(p - q) over q in the box and N in the
// node's box of face normals keeps one sign beyond the same margin; otherwise
// its length sum, times a cosine factor (reach + margin) / (L1 distance + half
// the box's edge sum + margin) in (0, 1], over (squared distance to the box
// centre + squared half diagonal).  The descent
// takes each child with probability proportional to its weight, by a fresh
// uniform per level (level l: component l % 4 of the draw of block 4 + l / 4 at
// vertex k); returns the edge and its probability pe, or -1 when all weights vanish.
template <class P>
__device__ __forceinline__ float edge_node_weight(P bx, float len, P nb, V3 p, V3 nrm, bool sil) {
#pragma clang fp contract(off)
    const float dx = (bx[0] + bx[3]) * 0.5f - p.x, dy = (bx[1] + bx[4]) * 0.5f - p.y, dz = (bx[2] + bx[5]) * 0.5f - p.z;
    const float ex = bx[3] - bx[0], ey = bx[4] - bx[1], ez = bx[5] - bx[2];
    const float reach = (dx * nrm.x + dy * nrm.y + dz * nrm.z) +
                        0.5f * ((fabsf(nrm.x) * ex + fabsf(nrm.y) * ey) + fabsf(nrm.z) * ez);
    const float tol = 0x1p-16f * (((fabsf(dx) + fabsf(dy)) + fabsf(dz)) + ((ex + ey) + ez));
    if (!(reach > -tol)) return 0.0f;
    if (sil) {
        const float a0 = -nb[0] * dx, b0 = -nb[3] * dx, a1 = -nb[1] * dy, b1 = -nb[4] * dy;
        const float a2 = -nb[2] * dz, b2 = -nb[5] * dz;
        const float lo = ((0.0f + fminf(a0, b0)) + fminf(a1, b1)) + fminf(a2, b2);
        const float hi = ((0.0f + fmaxf(a0, b0)) + fmaxf(a1, b1)) + fmaxf(a2, b2);
        const float rad = ((0.0f + fmaxf(fabsf(nb[0]), fabsf(nb[3])) * (0.5f * ex)) +
                           fmaxf(fabsf(nb[1]), fabsf(nb[4])) * (0.5f * ey)) +
                          fmaxf(fabsf(nb[2]), fabsf(nb[5])) * (0.5f * ez);
        if (lo - rad > tol || hi + rad < -tol) return 0.0f;
    }
    const float dl1 = ((fabsf(dx) + fabsf(dy)) + fabsf(dz)) + 0.5f * ((ex + ey) + ez);
    const float cb = (reach + tol) / (dl1 + tol);
    return len * cb / ((dx * dx + dy * dy + dz * dz) + 0.25f * ((ex * ex + ey * ey) + ez * ez));
}

// child j (0, 1) of a packed record: box (6), length, normal box (6), code
template <class P> __device__ __forceinline__ float edge_child_weight(P rec, int j, V3 p, V3 nrm, bool sil, int& code) {
    const vf4 a = *(const gfloat4*)(rec + 4 * j), b = *(const gfloat4*)(rec + 4 * j + 1), c = *(const gfloat4*)(rec + 4 * j + 2),
              d = *(const gfloat4*)(rec + 4 * j + 3);
    const float bx[6] = {a.x, a.y, a.z, a.w, b.x, b.y};
    const float nb[6] = {b.w, c.x, c.y, c.z, c.w, d.x};
    code = __float_as_int(d.y);
    return edge_node_weight<const float*>(bx, b.z, nb, p, nrm, sil);
}

__device__ __forceinline__ int edge_tree_sample(const DevScene& S, V3 p, V3 nrm, const Ctr& ctr, int k,
                                                const Key& key, bool sil, float& pe) {
#pragma clang fp contract(off)
    pe = 1.0f;
    if (S.ne <= 0) return -1;
    int code = S.ne == 1 ? (int)LEAF_BIT : 0;
    float4 u = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int level = 0; !(code & (int)LEAF_BIT); ++level) {
        if (level >= 128) return -1;
        if ((level & 3) == 0) u = draw4(ctr, k, 4 + (level >> 2), key);
        const auto rec = S.etnode + 8 * (size_t)code;
        int c0, c1;
        const float w0 = edge_child_weight(rec, 0, p, nrm, sil, c0), w1 = edge_child_weight(rec, 1, p, nrm, sil, c1);
        const float tot = w0 + w1;
        if (!(tot > 0.0f)) return -1;
        const float p0 = w0 / tot;
        const float ul = (level & 3) == 0 ? u.x : (level & 3) == 1 ? u.y : (level & 3) == 2 ? u.z : u.w;
        if (ul < p0) { code = c0; pe *= p0; }
        else { code = c1; pe *= w1 / tot; }
    }
    if (S.ne == 1 && !(edge_node_weight(S.etbox, S.etlen[0], S.etnbox, p, nrm, sil) > 0.0f)) return -1;
    return (int)S.etedge[code & 0x7FFFFFFF];
}

// Lambda of a direction with cosine c and its derivatives by c and by the roughness a
struct Lambda { float v, dc, da; };
__device__ __forceinline__ Lambda smith_lambda_grad(float c, float a) {
    // Lambda(x), x = c / (a sqrt(1-c^2)); dLambda/dx = -exp(-x^2) / (2 sqrt(pi) x^2)
    Lambda r{0.0f, 0.0f, 0.0f};
    if (c >= 1.0f) return r;
    const float s = sqrtf(1.0f - c * c);
    const float x = c / (a * s);
    const float e = expf(-x * x);
    r.v = (e * INV_SQRT_PI_F / x - erfcf(x)) * 0.5f;
    if (x > 12.0f) return r;
    const float dldx = -e * (0.5f * INV_SQRT_PI_F) / (x * x);
    r.da = dldx * (-x / a);
    r.dc = dldx / (a * s * s * s);
    return r;
}

// f(wi, wo, n, m) and the reverse-mode derivative of it contracted with gf (rgb), which
// accumulates into gn, gwi (only needed when wi depends on the geometry) and gm[7].  lo:
// Lambda of wo, the same for every wi of a shading point.  Value and derivative share
// the half-vector, D and both Lambdas.
__device__ __forceinline__ V3 brdf_eval_backward(V3 wi, V3 wo, V3 n, const Mat& m, const Lambda& lo, V3 gf, V3& gn,
                                                 V3& gwi, float* gm) {
    const float ci = dot(n, wi), co = dot(n, wo);
    if (!(ci > 0.0f) || !(co > 0.0f)) return V3{0.f, 0.f, 0.f};
    gm[0] += gf.x * INV_PI_F; gm[1] += gf.y * INV_PI_F; gm[2] += gf.z * INV_PI_F;
    const float a = alpha_eff(m.a);
    const V3 hv = wi + wo;
    const float hl = len(hv);
    const V3 h = hv * (1.0f / hl);
    const float ch = dot(n, h);
    if (!(ch > 0.0f)) return m.kd * INV_PI_F;
    const float D = beckmann_D(n, h, ch, a);
    const Lambda li = smith_lambda_grad(ci, a);
    const float G = 1.0f / (1.0f + li.v + lo.v);
    const float K = D * G / (4.0f * ci * co);
    gm[3] += gf.x * K; gm[4] += gf.y * K; gm[5] += gf.z * K;
    const float glnK = dot(gf, m.ks) * K;       // gradient w.r.t. ln K
    const float c2 = ch * ch;
    const float dlnD_dch = 2.0f / (c2 * ch * a * a) - 4.0f / ch;
    const V3 nh = cross(n, h);
    const float dlnD_da = 2.0f * dot(nh, nh) / (c2 * a * a * a) - 2.0f / a;
    if (m.a > ALPHA_MIN) gm[6] += glnK * (dlnD_da - G * (li.da + lo.da));
    const float gci = glnK * (-G * li.dc - 1.0f / ci);
    const float gco = glnK * (-G * lo.dc - 1.0f / co);
    const float gch = glnK * dlnD_dch;
    gn = gn + wi * gci + wo * gco + h * gch;
    // through h = normalize(wi + wo) (wo is fixed)
    const V3 gh = n * gch;
    const V3 ghv = (gh - h * dot(h, gh)) * (1.0f / hl);
    gwi = gwi + n * gci + ghv;
    return m.kd * INV_PI_F + m.ks * K;
}

// ---------------------------------------------------------------------------
// environment map: equirectangular, +y up, row 0 at theta = 0
// ---------------------------------------------------------------------------
// guide table of a CDF (cut-point method): guide[g] = largest i in [0, n-1] with
// C[i] <= g / G, G = 2^glog.  With g = floor(u G) the answer of cdf_find lies in
// [guide[g], guide[g + 1]], so a search of that (usually one- or two-entry)
// range returns exactly the index of the plain search.
template <class PC, class PG>
__device__ __forceinline__ int cdf_guided(PC C, int n, PG guide, int glog, double u) {
    const int G = 1 << glog;
    int g = (int)(u * (double)G);
    g = g < G - 1 ? g : G - 1;
    int lo = guide[g];
    int hi = g + 1 < G ? guide[g + 1] : n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (C[mid] <= u) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int cdf_find(const double* C, int n, double u) {
    // largest i in [0, n-1] with C[i] <= u (C[0] == 0 <= u)
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (C[mid] <= u) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int env_texel_of(const DevScene& S, V3 d) {
    const float y = fminf(1.0f, fmaxf(-1.0f, d.y));
    const float th = acosf(y);
    float ph = atan2f(d.x, d.z);
    if (ph < 0.0f) ph += 2.0f * PI_F;
    const int r = min((int)(th * (1.0f / PI_F) * S.he), S.he - 1);
    const int c = min((int)(ph * (0.5f / PI_F) * S.we), S.we - 1);
    return r * S.we + c;
}
__device__ __forceinline__ V3 env_rgb(const DevScene& S, int t) { return ld3(S.env + 3 * (size_t)t); }

__device__ __forceinline__ int env_sample(const DevScene& S, float4 u, V3& dir, float& pdf) {
    int r, c;
    if (S.env_alias) {
        // bin from the first uniform, the bin's texel or its alias from the second
        const int n = S.he * S.we;
        const int k = min((int)((double)u.x * (double)n), n - 1);
        const EnvAlias e = S.ealias[k];
        const int t = (double)u.y < e.prob ? k : e.alias;
        r = t / S.we;
        c = t - r * S.we;
    } else {
        r = cdf_guided(S.marg, S.he, S.mguide, S.mglog, (double)u.x);
        c = cdf_guided(S.cond + (size_t)r * (S.we + 1), S.we, S.cguide + ((size_t)r << S.cglog), S.cglog,
                       (double)u.y);
    }
    const float phi = 2.0f * PI_F * ((float)c + u.z) / (float)S.we;
    // cos(theta) uniform between the row's bounds; 1 -+ cos(theta) are taken
    // from the per-row tables of 1 - cos and 1 + cos so that sin(theta) keeps
    // full precision near both poles
    const float om0 = S.rowcos[r], om1 = S.rowcos[r + 1];                        // 1 - cos
    const float op0 = S.rowcos[S.he + 1 + r], op1 = S.rowcos[S.he + 2 + r];      // 1 + cos
    float a, b, cth;
    if (op0 + op1 >= om0 + om1) {       // upper half of the sphere: 1 - cos is the small one
        a = om0 + u.w * (om1 - om0);
        b = 2.0f - a;
        cth = 1.0f - a;
    } else {
        b = op0 - u.w * (op0 - op1);
        a = 2.0f - b;
        cth = b - 1.0f;
    }
    const float sth = sqrtf(fmaxf(0.0f, a * b));
    float sp, cp;
    sincosf(phi, &sp, &cp);
    dir = V3{sth * sp, cth, sth * cp};
    const int t = r * S.we + c;
    pdf = S.texpdf[t];
    return t;
}

// ---------------------------------------------------------------------------
// camera (precomputed basis; r and u already scaled by tan(fov/2) and aspect)
// ---------------------------------------------------------------------------
struct DevCam {
    float eye[3], f[3], rs[3], us[3];
    double deye[3], df[3], dr[3], du[3], dth, daspect;
    int W, H, scene;
    int rngview;         // view field of the random-stream counters: index among this scene's cameras
    long long qoff;      // processing-order path offset
    long long pixoff;    // canonical pixel offset
    long long eoff;      // primary edge sample offset
    long long ne;        // primary edge samples of this view
};

__device__ __forceinline__ V3 cam_dir(const DevCam& c, float sx, float sy) {
    const float nx = 2.0f * sx / (float)c.W - 1.0f, ny = 1.0f - 2.0f * sy / (float)c.H;
    const V3 d = ld3(c.f) + ld3(c.rs) * nx + ld3(c.us) * ny;
    return normalize(d);
}

// ---------------------------------------------------------------------------
// the path estimator (forward radiance only): used for the edge side paths and
// the single-kernel forward.  first_escape_full: a first-segment miss returns
// the environment radiance (secondary side rays) instead of black (camera).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void push_face(Hash& h, int f) { h.push(f < 0 ? 0xFFFFFFFFu : (uint32_t)f); }

template <bool FAST = false>
__device__ V3 trace_estimator(const DevScene& S, const TraceGeo& G, V3 o, V3 d, int exclude, int nvert, bool first_escape_full,
                              const Ctr& ctr, const Key& key, Hash& hash, TravStack& st) {
    V3 L{0.f, 0.f, 0.f}, beta{1.f, 1.f, 1.f};
    float p_prev = 0.0f;
    for (int k = 1; k <= nvert + 1; ++k) {
        float t;
        const int f = trace_closest<FAST>(G, o, d, TMIN, exclude, t, st);
        push_face(hash, f);
        if (f < 0) {
            if (S.has_env && (k > 1 || first_escape_full)) {
                const int tex = env_texel_of(S, d);
                hash.push((uint32_t)tex);
                const V3 Le = env_rgb(S, tex);
                float w = 1.0f;
                if (k > 1) { const float pe = S.texpdf[tex]; w = p_prev / (p_prev + pe); }
                L = L + mul(beta, Le) * w;
            }
            break;
        }
        if (k == nvert + 1) break;
        const V3 x = o + d * t;
        V3 n = xyz(S.fnorm[f]);
        const V3 wo = -d;
        if (dot(n, wo) < 0.0f) n = -n;
        const int tx = texel_of(S, f, x);
        if (S.tex_res) hash.push((uint32_t)tx);
        const Mat m = load_mat(S.mat + 7 * (size_t)tx);
        const float lo = out_lambda(wo, n, m);
        for (int l = 0; l < S.nl; ++l) {
            const auto lt = S.lights + 6 * l;
            const V3 dl = ld3(lt) - x;
            const float r2 = dot(dl, dl);
            uint32_t code = 0;
            if (r2 > 0.0f) {
                const float r = sqrtf(r2);
                const V3 wl = dl * (1.0f / r);
                const float c = dot(n, wl);
                if (c > 0.0f) {
                    const bool occ = trace_any<FAST>(G, x, wl, TMIN, r * (1.0f - SHADOW_SHRINK), f, st);
                    code = occ ? 1u : 2u;
                    if (!occ) L = L + mul(beta, mul(ld3(lt + 3), brdf_eval(wl, wo, n, m, lo))) * (c / r2);
                }
            }
            hash.push(code);
        }
        if (S.has_env) {
            const float4 u = draw4(ctr, k, 1, key);
            V3 we; float pe;
            const int tex = env_sample(S, u, we, pe);
            hash.push((uint32_t)tex);
            const float c = dot(n, we);
            uint32_t code = 0;
            if (c > 0.0f && pe > 0.0f) {
                const bool occ = trace_any<FAST>(G, x, we, TMIN, __int_as_float(0x7f800000), f, st);
                code = occ ? 1u : 2u;
                if (!occ) {
                    float pdf;
                    const V3 fv = brdf_eval_pdf(we, wo, n, m, lo, S.vndf, pdf);
                    const float den = pe + pdf;
                    L = L + mul(beta, mul(env_rgb(S, tex), fv)) * (c / den);
                }
            }
            hash.push(code);
        }
        if (!(k < nvert || S.has_env)) break;
        const float4 u = draw4(ctr, k, 2, key);
        V3 wi;
        const int lobe = bsdf_sample(u, wo, n, m.a, S.vndf, wi);
        const float ci = dot(n, wi);
        float pb;
        const V3 fi = brdf_eval_pdf(wi, wo, n, m, lo, S.vndf, pb);
        hash.push((uint32_t)lobe);
        if (!(ci > 0.0f) || !(pb > 0.0f)) { hash.push(0u); break; }
        hash.push(1u);
        beta = mul(beta, fi) * (ci / pb);
        p_prev = pb;
        o = x; d = wi; exclude = f;
    }
    return L;
}

__device__ __forceinline__ uint64_t lanemask_lt64() {
    const uint32_t lane = __lane_id();
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// processing order of path samples inside one view: sample-major, then 8x8
// pixel tiles (when the view is a multiple of 8 in both axes), then row-major
// (a call has fewer than 2^31 path samples: 32-bit divisions)
__device__ __forceinline__ void decode_path(const DevCam& c, long long local, int spp, int& x, int& y, int& j) {
    const uint32_t hw = (uint32_t)c.W * (uint32_t)c.H, l = (uint32_t)local;
    j = (int)(l / hw);
    const uint32_t p = l - (uint32_t)j * hw;
    if ((c.W & 7) == 0 && (c.H & 7) == 0) {
        const uint32_t tile = p >> 6, within = p & 63u, tw = (uint32_t)c.W >> 3, ty = tile / tw;
        x = (int)((tile - ty * tw) * 8 + (within & 7u));
        y = (int)(ty * 8 + (within >> 3));
    } else {
        y = (int)(p / (uint32_t)c.W);
        x = (int)(p - (uint32_t)y * (uint32_t)c.W);
    }
    (void)spp;
}

__device__ __forceinline__ int find_view(const long long* off, int ncam, long long q) {
    // largest v with off[v] <= q
    int lo = 0, hi = ncam - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= q) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// the view of entry q when entry base (uniform, base <= q) is of view vb: the same
// but for entries past that view's end
__device__ __forceinline__ int find_view_from(const long long* off, int ncam, int vb, long long q) {
    return q < off[vb + 1] ? vb : find_view(off, ncam, q);
}

// ---------------------------------------------------------------------------
// Normalised prefix sums of n doubles (out[0] = 0, out[i+1] = (w[0] + .. + w[i]) /
// total) in tiles of CDF_TILE, one block of CDF_BLOCK threads each, CDF_PER
// consecutive values a thread: the kernel that computes the weights leaves each
// tile's sum (cdf_tile_sum), the next one adds the tiles before (cdf_tile_write).
// One block over all values took 133 us for 60,000 edges (uncoalesced chunks, a
// serial scan of 1,024 partial sums); the two kernels take 9.
//
// Sums of different groupings of the same values differ by a rounding, so the values
// must not step back, nor rise over a weight of zero, where the groupings meet: a
// search would pick an edge that no sample may have.  A tile starts and ends at sums
// over tiles, all by one tree (a sum over more of its inputs is never less, and the
// same when they are zeros); inside, a value is the largest so far at a positive
// weight, at the tile's last one the tile's end.
// ---------------------------------------------------------------------------
constexpr int CDF_BLOCK = 256, CDF_PER = 4, CDF_TILE = CDF_BLOCK * CDF_PER;
__host__ __device__ __forceinline__ int cdf_tiles(int n) { return (n + CDF_TILE - 1) / CDF_TILE; }
// exclusive scan of v >= 0 over the block's threads, in thread order, and the block's
// total; op: sum or maximum
template <class Op>
__device__ __forceinline__ double block_excl(double v, double& total, double* lds /* CDF_BLOCK / 64 */, Op op) {
    double inc = v;
    const int lane = (int)__lane_id(), w = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double x = __shfl_up(inc, o, 64);
        if (lane >= o) inc = op(inc, x);
    }
    const double up = __shfl_up(inc, 1, 64);
    __syncthreads();
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    double before = 0.0, all = 0.0;
#pragma unroll
    for (int k = 0; k < CDF_BLOCK / 64; ++k) {
        if (k < w) before = op(before, lds[k]);
        all = op(all, lds[k]);
    }
    total = all;
    return op(before, lane > 0 ? up : 0.0);
}
__device__ __forceinline__ double block_excl_sum(double v, double& total, double* lds) {
    return block_excl(v, total, lds, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ void cdf_tile_sum(double thread_sum, double* tile_sums) {
    __shared__ double lds[CDF_BLOCK / 64];
    double total;
    block_excl_sum(thread_sum, total, lds);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}
// returns the total over all tiles
__device__ __forceinline__ double cdf_tile_write(const double* __restrict__ w, int n, const double* __restrict__ tile_sums,
                                                 double* __restrict__ out, double* total_out) {
    __shared__ double lds[CDF_BLOCK / 64];
    __shared__ int some[CDF_BLOCK / 64];
    const int t = threadIdx.x, b = blockIdx.x, nt = cdf_tiles(n);
    double bs = 0.0, es = 0.0, as = 0.0, start, end, total, dummy;
    for (int i = t; i < nt; i += CDF_BLOCK) {
        const double v = tile_sums[i];
        as += v;
        if (i < b) bs += v;
        if (i <= b) es += v;
    }
    block_excl_sum(bs, start, lds);
    block_excl_sum(es, end, lds);
    block_excl_sum(as, total, lds);
    const int i0 = b * CDF_TILE + t * CDF_PER;
    double v[CDF_PER], s = 0.0;
#pragma unroll
    for (int q = 0; q < CDF_PER; ++q) {
        v[q] = i0 + q < n ? w[i0 + q] : 0.0;
        s += v[q];
    }
    const uint64_t have = __ballot(s > 0.0);
    if (__lane_id() == 0) some[t >> 6] = have != 0;
    const double acc0 = start + block_excl_sum(s, dummy, lds);      // (synchronises the block)
    bool last = (have >> (t & 63)) == 1;      // no later thread of the wave, or of the waves after
    for (int k = (t >> 6) + 1; k < CDF_BLOCK / 64; ++k) last = last && !some[k];
    double most = 0.0, acc = acc0;
#pragma unroll
    for (int q = 0; q < CDF_PER; ++q) {
        acc += v[q];
        if (v[q] > 0.0) most = fmax(most, fmin(acc, end));
    }
    if (last) most = end;
    double at = fmax(start, block_excl(most, dummy, lds, [](double a, double c) { return fmax(a, c); }));
    acc = acc0;
#pragma unroll
    for (int q = 0; q < CDF_PER; ++q) {
        acc += v[q];
        bool ends = last;
#pragma unroll
        for (int r = q + 1; r < CDF_PER; ++r) ends = ends && !(v[r] > 0.0);
        if (v[q] > 0.0) at = ends ? end : fmax(at, fmin(acc, end));
        if (i0 + q < n) out[i0 + q + 1] = total > 0.0 ? at / total : 0.0;
    }
    if (b == 0 && t == 0) {
        out[0] = 0.0;
        *total_out = total;
    }
    return total;
}

// ---------------------------------------------------------------------------
// queue reservation with one atomic per block.  Atomics on one address are
// serialised by the memory system (about 11 ns apiece on this part), so one
// reservation per wave caps a compaction kernel at roughly 90 M waves/s;
// reserving per block of BS threads divides that cost by BS / 64.  Every thread
// of the block calls it (it synchronises the block); lanes with emit get M
// consecutive slots, the others -1.  lds holds BS / 64 + 1 ints.
// ---------------------------------------------------------------------------
template <int BS, int M>
__device__ __forceinline__ int block_reserve(bool emit, int* counter, int* lds) {
    const uint64_t mask = __ballot(emit);
    const int w = (int)(threadIdx.x >> 6);
    if (__lane_id() == 0) lds[w] = M * __popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int j = 0; j < BS / 64; ++j) {
            const int c = lds[j];
            lds[j] = acc;
            acc += c;
        }
        lds[BS / 64] = acc > 0 ? atomicAdd(counter, acc) : 0;
    }
    __syncthreads();
    const int o = lds[BS / 64] + lds[w] + M * __popcll(mask & lanemask_lt64());
    __syncthreads();
    return emit ? o : -1;
}

// m (0 <= m < 2^BITS) consecutive slots per thread from *counter, in thread
// order within the block, with one atomic per block; every thread of the block
// calls it (it synchronises the block).  lds holds BS / 64 + 1 ints.
template <int BS, int BITS>
__device__ __forceinline__ int block_reserve_n(int m, int* counter, int* lds) {
    constexpr int NW = BS / 64;
    const uint64_t lt = lanemask_lt64();
    int pre = 0, tot = 0;
    for (int b = 0; b < BITS; ++b) {
        const uint64_t bm = __ballot((m >> b) & 1);
        pre += __popcll(bm & lt) << b;
        tot += __popcll(bm) << b;
    }
    const int w = (int)(threadIdx.x >> 6);
    if (__lane_id() == 0) lds[w] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int j = 0; j < NW; ++j) {
            const int x = lds[j];
            lds[j] = acc;
            acc += x;
        }
        lds[NW] = acc > 0 ? atomicAdd(counter, acc) : 0;
    }
    __syncthreads();
    const int o = lds[NW] + lds[w] + pre;
    __syncthreads();
    return o;
}

// Two reservations in one pass: one slot per thread with emit from *ca, and m
// (0 <= m < 32) consecutive slots per thread from *cb.  Returns (slot or -1,
// first of the m slots).  lds holds 2 (BS / 64 + 1) ints.
template <int BS>
__device__ __forceinline__ int2 block_reserve2(bool emit, int m, int* ca, int* cb, int* lds) {
    constexpr int NW = BS / 64;
    const uint64_t lt = lanemask_lt64();
    const uint64_t mask = __ballot(emit);
    int pre = 0, tot = 0;
    for (int b = 0; b < 5; ++b) {
        const uint64_t bm = __ballot((m >> b) & 1);
        pre += __popcll(bm & lt) << b;
        tot += __popcll(bm) << b;
    }
    const int w = (int)(threadIdx.x >> 6);
    if (__lane_id() == 0) {
        lds[w] = __popcll(mask);
        lds[NW + 1 + w] = tot;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        // lane 0 scans and reserves for ca, lane 1 for cb: one atomic
        // instruction, so the two round trips overlap
        const int base = threadIdx.x == 0 ? 0 : NW + 1;
        int acc = 0;
        for (int j = 0; j < NW; ++j) {
            const int x = lds[base + j];
            lds[base + j] = acc;
            acc += x;
        }
        int* const ctr = threadIdx.x == 0 ? ca : cb;
        lds[base + NW] = acc > 0 ? atomicAdd(ctr, acc) : 0;
    }
    __syncthreads();
    const int oa = lds[NW] + lds[w] + __popcll(mask & lt);
    const int ob = lds[2 * NW + 1] + lds[NW + 1 + w] + pre;
    __syncthreads();
    return make_int2(emit ? oa : -1, ob);
}

// Block index remapped so that each XCD works on one contiguous range of the
// grid: the hardware hands block b to XCD b % 8, so XCD x receives blocks
// x, x + 8, ...; they become x's consecutive share [x G/8, (x+1) G/8) (the
// first G % 8 XCDs one block more), and neighbouring work shares one L2.
constexpr unsigned NUM_XCD = 8;
__device__ __forceinline__ unsigned xcd_block() {
    const unsigned G = gridDim.x, b = blockIdx.x;
    const unsigned per = G / NUM_XCD, rem = G % NUM_XCD, x = b % NUM_XCD, j = b / NUM_XCD;
    return x < rem ? x * (per + 1) + j : rem * (per + 1) + (x - rem) * per + j;
}
#ifndef ST_XCD_MAP
#define ST_XCD_MAP 1
#endif
// the block index the adjoint's grid-stride loop starts from (the traversal
// kernels keep the hardware order: contiguous shares per XCD made them slower,
// 69.8 -> 84.3 ms for k_extend, presumably because cheap and costly stretches
// of the queue then land on different XCDs)
__device__ __forceinline__ unsigned grid_block() { return ST_XCD_MAP ? xcd_block() : blockIdx.x; }

} // namespace st
