// Scene build on the GPU: per-face normals and bounds, the LBVH (30-bit Morton
// codes, stable LSD radix sort, Karras 2012 radix-tree hierarchy, bottom-up
// min/max refit), the leaf-ordered triangle records, the 3-D edge-length CDF of
// the secondary edge term, and the environment-map CDFs.
//
// The paper (Sec. 3.2, "Representation") relies on fast ray-surface
// intersection as the bulk of the cost without naming a structure; the LBVH is
// this library's choice.  Its integer part is bit-exact by specification:
// float32 centroids (min+max)*0.5, scale = float(1024 / (hi - lo)) evaluated in
// double, q = clamp(floor((c - lo) * s), 0, 1023), 10 bits per axis with x
// highest, key = morton << 32 | face, ascending.
#include "st_internal.h"

namespace st {

// ---------------------------------------------------------------------------
// Centroid bounds in two steps: each block of BND_TILE centroids leaves its own, and
// the blocks of k_morton reduce those of all blocks again (one block over all the
// centroids took 16 us at 40,000).
constexpr int BND_TILE = 1024, BND_BLOCK = 256;
struct Bounds {
    float lo[3], hi[3];
};
__device__ __forceinline__ Bounds bounds_none() {
    const float INF = __int_as_float(0x7f800000);
    return Bounds{{INF, INF, INF}, {-INF, -INF, -INF}};
}
// of the block's threads, in every thread
__device__ __forceinline__ Bounds block_bounds(Bounds b) {
    __shared__ Bounds lds[BND_BLOCK / 64];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
        for (int k = 0; k < 3; ++k) {
            b.lo[k] = fminf(b.lo[k], __shfl_xor(b.lo[k], o, 64));
            b.hi[k] = fmaxf(b.hi[k], __shfl_xor(b.hi[k], o, 64));
        }
    if (__lane_id() == 0) lds[threadIdx.x >> 6] = b;
    __syncthreads();
    for (int w = 0; w < BND_BLOCK / 64; ++w)
        for (int k = 0; k < 3; ++k) {
            b.lo[k] = fminf(b.lo[k], lds[w].lo[k]);
            b.hi[k] = fmaxf(b.hi[k], lds[w].hi[k]);
        }
    return b;
}
__device__ __forceinline__ void bounds_add(Bounds& b, float x, float y, float z) {
    b.lo[0] = fminf(b.lo[0], x); b.lo[1] = fminf(b.lo[1], y); b.lo[2] = fminf(b.lo[2], z);
    b.hi[0] = fmaxf(b.hi[0], x); b.hi[1] = fmaxf(b.hi[1], y); b.hi[2] = fmaxf(b.hi[2], z);
}

__global__ void __launch_bounds__(BND_BLOCK) k_face_prep(const float* __restrict__ V, const int* __restrict__ F, int nf,
                                                         float4* fnorm, float4* bmin, float4* bmax, float4* cen,
                                                         Bounds* bounds) {
#pragma clang fp contract(off)
    Bounds bb = bounds_none();
    for (int q = 0; q < BND_TILE / BND_BLOCK; ++q) {
        const int f = blockIdx.x * BND_TILE + q * BND_BLOCK + threadIdx.x;
        if (f >= nf) break;
        const V3 a = ld3(V + 3 * F[3 * f]), b = ld3(V + 3 * F[3 * f + 1]), c = ld3(V + 3 * F[3 * f + 2]);
        const V3 N = cross(b - a, c - a);
        const float l = len(N);
        const V3 n = l > 0.0f ? N * (1.0f / l) : V3{0.f, 0.f, 0.f};
        fnorm[f] = make_float4(n.x, n.y, n.z, 0.5f * l);
        const V3 mn{fminf(a.x, fminf(b.x, c.x)), fminf(a.y, fminf(b.y, c.y)), fminf(a.z, fminf(b.z, c.z))};
        const V3 mx{fmaxf(a.x, fmaxf(b.x, c.x)), fmaxf(a.y, fmaxf(b.y, c.y)), fmaxf(a.z, fmaxf(b.z, c.z))};
        bmin[f] = make_float4(mn.x, mn.y, mn.z, 0.f);
        bmax[f] = make_float4(mx.x, mx.y, mx.z, 0.f);
        const float cx = mn.x + mx.x, cy = mn.y + mx.y, cz = mn.z + mx.z;
        cen[f] = make_float4(cx * 0.5f, cy * 0.5f, cz * 0.5f, 0.f);
        bounds_add(bb, cx * 0.5f, cy * 0.5f, cz * 0.5f);
    }
    bb = block_bounds(bb);
    if (threadIdx.x == 0) bounds[blockIdx.x] = bb;
}

__device__ __forceinline__ uint32_t spread10(uint32_t v) {
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// ---------------------------------------------------------------------------
// stable LSD radix sort of (u32 key, u32 value), 8-bit digits, tiles of 1024
// ---------------------------------------------------------------------------
constexpr int RS_THREADS = 256;
constexpr int RS_ITEMS = 4;
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;

// digit counts of a block's tile: hist[256 block + digit]
__global__ void k_rs_hist(const uint32_t* __restrict__ keys, int n, int shift, uint32_t* hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * RS_TILE;
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = base + r * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & 0xFFu], 1u);
    }
    __syncthreads();
    hist[256 * (size_t)blockIdx.x + threadIdx.x] = h[threadIdx.x];
}

// Morton keys and the digit counts of the first sorting pass (of the same tiles)
__global__ void __launch_bounds__(BND_BLOCK) k_morton(const float4* __restrict__ cen, int nf, const Bounds* __restrict__ bounds,
                                                      int nbounds, uint32_t* keys, uint32_t* vals, uint32_t* hist) {
#pragma clang fp contract(off)
    static_assert(RS_TILE == BND_TILE && RS_THREADS == BND_BLOCK, "one tile for bounds, keys and counts");
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    Bounds bb = bounds_none();
    for (int i = threadIdx.x; i < nbounds; i += BND_BLOCK) {
        const Bounds o = bounds[i];
        bounds_add(bb, o.lo[0], o.lo[1], o.lo[2]);
        bounds_add(bb, o.hi[0], o.hi[1], o.hi[2]);
    }
    bb = block_bounds(bb);     // (synchronises the block)
    // one scale for all axes (cubic cells): 1024 cells along the longest extent
    double ext = 0.0;
    for (int k = 0; k < 3; ++k) ext = fmax(ext, (double)bb.hi[k] - (double)bb.lo[k]);
    const float scale = ext > 0.0 ? (float)(1024.0 / ext) : 0.0f;
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int f = blockIdx.x * RS_TILE + r * RS_THREADS + threadIdx.x;
        if (f >= nf) break;
        const float4 c = cen[f];
        const float cc[3] = {c.x, c.y, c.z};
        uint32_t q[3];
        for (int k = 0; k < 3; ++k) {
            const float d = cc[k] - bb.lo[k];
            const float p = d * scale;
            const int qi = (int)floorf(p);
            q[k] = (uint32_t)min(1023, max(0, qi));
        }
        const uint32_t key = (spread10(q[0]) << 2) | (spread10(q[1]) << 1) | spread10(q[2]);
        keys[f] = key;
        vals[f] = (uint32_t)f;
        atomicAdd(&h[key & 0xFFu], 1u);
    }
    __syncthreads();
    hist[256 * (size_t)blockIdx.x + threadIdx.x] = h[threadIdx.x];
}

// Where a tile's entries of each digit go: the entries of lower digits, then those
// of the same digit in the tiles before.  Up to RS_SUM_TILES tiles every tile adds
// the counts of all tiles itself (a coalesced row of 256 a tile: 40 rows take 2 us at
// 40,000 keys, where one block scanning them took 16); beyond, k_rs_scan prepares them.
constexpr int RS_SUM_TILES = 512;
// exclusive sum of v over the first 256 threads of the block (those with in)
__device__ __forceinline__ uint32_t block_excl_256(uint32_t v, uint32_t* lds /* 4 */, bool in = true) {
    uint32_t inc = v;
    const int lane = (int)__lane_id(), w = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(inc, o, 64);
        if (lane >= o) inc += x;
    }
    if (lane == 63 && in) lds[w] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int k = 0; in && k < w; ++k) before += lds[k];
    return before + inc - v;
}
// hist to these starts, in place; one block, a thread per digit and quarter of the tiles
constexpr int RS_SCAN_THREADS = 1024;
__global__ void __launch_bounds__(RS_SCAN_THREADS) k_rs_scan(uint32_t* hist, int nblocks) {
    __shared__ uint32_t lds[4];
    __shared__ uint32_t part[4][256], start[256];
    const int d = threadIdx.x & 255, q = threadIdx.x >> 8;
    const int b0 = (int)((long long)nblocks * q / 4), b1 = (int)((long long)nblocks * (q + 1) / 4);
    uint32_t tot = 0;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) tot += hist[256 * (size_t)b + d];
    part[q][d] = tot;
    __syncthreads();
    // the first 256 threads (four waves) scan; all synchronise
    uint32_t all = 0;
    for (int k = 0; k < 4; ++k) all += part[k][d];
    const uint32_t at0 = block_excl_256(q == 0 ? all : 0u, lds, q == 0);
    if (q == 0) start[d] = at0;
    __syncthreads();
    uint32_t at = start[d];
    for (int k = 0; k < q; ++k) at += part[k][d];
#pragma unroll 8
    for (int b = b0; b < b1; ++b) {
        const uint32_t c = hist[256 * (size_t)b + d];
        hist[256 * (size_t)b + d] = at;
        at += c;
    }
}

__global__ void k_rs_scatter(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* kout,
                             uint32_t* vout, int n, int shift, const uint32_t* __restrict__ hist, int nblocks) {
    constexpr int NW = RS_THREADS / 64;
    __shared__ uint32_t wcount[NW][256];
    __shared__ uint32_t running[256];
    __shared__ uint32_t gbase[256];
    __shared__ uint32_t scan[4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    running[t] = 0;
    if (nblocks > RS_SUM_TILES) {
        gbase[t] = hist[256 * (size_t)blockIdx.x + t];
    } else {
        uint32_t tot = 0, before = 0;
#pragma unroll 8
        for (int b = 0; b < nblocks; ++b) {
            const uint32_t c = hist[256 * b + t];
            tot += c;
            before += b < (int)blockIdx.x ? c : 0u;
        }
        gbase[t] = before + block_excl_256(tot, scan);
    }
    for (int k = 0; k < NW; ++k) wcount[k][t] = 0;
    __syncthreads();
    const int base = blockIdx.x * RS_TILE;
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int i = base + r * RS_THREADS + t;
        const bool valid = i < n;
        const uint32_t key = valid ? kin[i] : 0u;
        const uint32_t val = valid ? vin[i] : 0u;
        const uint32_t dg = (key >> shift) & 0xFFu;
        // lanes of this wave holding the same digit
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            const uint64_t bal = __ballot((dg >> b) & 1u);
            peers &= ((dg >> b) & 1u) ? bal : ~bal;
        }
        const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        if (valid && rank == 0) wcount[w][dg] = (uint32_t)__popcll(peers);
        __syncthreads();
        {   // per digit: offsets of each wave inside this round
            uint32_t acc = running[t];
            for (int k = 0; k < NW; ++k) { const uint32_t c = wcount[k][t]; wcount[k][t] = acc; acc += c; }
            running[t] = acc;
        }
        __syncthreads();
        if (valid) {
            const uint32_t pos = gbase[dg] + wcount[w][dg] + rank;
            kout[pos] = key;
            vout[pos] = val;
        }
        __syncthreads();
        for (int k = 0; k < NW; ++k) wcount[k][t] = 0;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Karras 2012 hierarchy over the sorted 64-bit keys (morton << 32 | face)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int kdelta(const uint32_t* m, const uint32_t* fa, int n, int i, int j) {
    if (j < 0 || j > n - 1) return -1;
    const uint64_t a = ((uint64_t)m[i] << 32) | fa[i];
    const uint64_t b = ((uint64_t)m[j] << 32) | fa[j];
    return __clzll(a ^ b);
}

// children codes of internal node i and the range [first, last] of leaves below it
__device__ __forceinline__ int2 karras_node(const uint32_t* __restrict__ m, const uint32_t* __restrict__ fa, int n, int i,
                                            int& left, int& right) {
    const int d = kdelta(m, fa, n, i, i + 1) > kdelta(m, fa, n, i, i - 1) ? 1 : -1;
    const int dmin = kdelta(m, fa, n, i, i - d);
    int lmax = 2;
    while (kdelta(m, fa, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (kdelta(m, fa, n, i, i + (l + t) * d) > dmin) l += t;
    const int j = i + l * d;
    const int dnode = kdelta(m, fa, n, i, j);
    int s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (kdelta(m, fa, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int split = i + s * d + min(d, 0);
    left = (min(i, j) == split) ? (int)(LEAF_BIT | (uint32_t)split) : split;
    right = (max(i, j) == split + 1) ? (int)(LEAF_BIT | (uint32_t)(split + 1)) : split + 1;
    return make_int2(min(i, j), max(i, j));
}

__global__ void k_karras(const uint32_t* __restrict__ m, const uint32_t* __restrict__ fa, int n, int* child,
                         int* parent) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    int left, right;
    karras_node(m, fa, n, i, left, right);
    child[2 * i] = left;
    child[2 * i + 1] = right;
    parent[(left & (int)LEAF_BIT) ? (n - 1) + (left & 0x7FFFFFFF) : left] = i;
    parent[(right & (int)LEAF_BIT) ? (n - 1) + (right & 0x7FFFFFFF) : right] = i;
    if (i == 0) parent[0] = -1;
}

// triangle record i of face f
__device__ __forceinline__ void put_tri(const float* __restrict__ V, const int* __restrict__ F, int f, uint32_t i,
                                        float4* tri, int* fleaf) {
    const V3 a = ld3(V + 3 * F[3 * f]), b = ld3(V + 3 * F[3 * f + 1]), c = ld3(V + 3 * F[3 * f + 2]);
    const V3 e1 = b - a, e2 = c - a;
    float4* const o = tri + 3 * (size_t)i;
    o[0] = make_float4(a.x, a.y, a.z, __int_as_float(f));
    o[1] = make_float4(e1.x, e1.y, e1.z, 0.f);
    o[2] = make_float4(e2.x, e2.y, e2.z, 0.f);
    fleaf[f] = (int)i;
}

// The radix tree over the sorted keys as k_treelets walks it: per node (internal
// nodes, then leaves) its parent and which child it is, (parent << 1) | side, -1 at
// the root; per internal node the leaves below it.  Also the 64-bit keys and the
// cleared arrival counters; with one face, its record and box.
__global__ void k_tree_init(const uint32_t* __restrict__ m, const uint32_t* __restrict__ fa, int n, int* up, int2* range,
                            uint64_t* keys, int* cnt, const float4* __restrict__ bmin, const float4* __restrict__ bmax,
                            const float* __restrict__ V, const int* __restrict__ F, float* aabb, float4* tri, int* fleaf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = ((uint64_t)m[i] << 32) | fa[i];
    if (n == 1) {
        put_tri(V, F, 0, 0, tri, fleaf);
        aabb[0] = bmin[0].x; aabb[1] = bmin[0].y; aabb[2] = bmin[0].z;
        aabb[3] = bmax[0].x; aabb[4] = bmax[0].y; aabb[5] = bmax[0].z;
    }
    if (i >= n - 1) return;
    cnt[i] = 0;
    int left, right;
    range[i] = karras_node(m, fa, n, i, left, right);
    up[(left & (int)LEAF_BIT) ? (n - 1) + (left & 0x7FFFFFFF) : left] = i << 1;
    up[(right & (int)LEAF_BIT) ? (n - 1) + (right & 0x7FFFFFFF) : right] = (i << 1) | 1;
    if (i == 0) up[0] = -1;
}

__device__ __forceinline__ float aload(const float* p) {
    return __uint_as_float(__hip_atomic_load((const uint32_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Before a wave counts its arrival at a node of a bottom-up pass: what it stored below is
// complete.  Not a release in the language's sense (a fence would write back and
// invalidate the L2 at every link of the chain); it holds because every store and load of
// the data handed over is a relaxed agent-scope access, which gfx950 takes past the L1s and
// the eight L2s to where all of them see it, because the counter of outstanding accesses
// reaches zero only when such a store is there, and because the loads come after the
// arrival's atomic has returned.  Plain accesses must not be handed over by it, but for
// those to a block's own LDS.
__device__ __forceinline__ void handoff_release() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);     // no compiler motion across this point
    __builtin_amdgcn_s_waitcnt(0);               // every store of this wave has completed
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}
__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Refit and treelet restructuring of the Karras tree (Karras and Aila, HPG 2013) in
// one bottom-up pass.  Every internal node r with at least TL_LEAVES triangles below
// it, once both of its subtrees are final, becomes the root of a treelet of
// TL_LEAVES entries: starting from r's two children, the internal entry with the
// largest box area (first in list order on ties) is replaced by its two children,
// appended at the end of the list.  The entries are re-arranged into the binary tree
// of least SAH cost (a triangle leaf costs its box area, an internal node C_INNER *
// area + the costs of its children), found by dynamic programming over the 2^7 - 1
// subsets of entries; the treelet's internal nodes are reused (r stays the root, the
// others in ascending id order along the preorder of the new tree).  All comparisons
// are in float32 with contraction off, in a fixed order, so the tree is a function of
// the mesh alone, not of the wave schedule.
//
// The time is that of the longest chain of hand-offs, root to leaf, so each link is
// made short.  A node is one 64-byte record, its two children's halves of 8 words:
// code, box (lower, upper), SAH cost; whoever finishes a subtree writes its half of
// the parent's record and counts its arrival, the second to arrive goes on with the
// parent.  A treelet reads one record per entry it opens, 8 lanes to a record.
// Subtrees that lie inside a block's leaves (a radix tree's nodes cover
// ranges of leaves, and node i's range has i at one end) are built in LDS; the nodes
// above go through global memory with agent-scope accesses (coherent across the XCDs'
// L2s without flushing them; a hand-off needs only the wave's own stores drained).
// One wave owns a treelet: its lanes share the list, the subset boxes and the subset
// programme, whose splits each lane holds in registers.
// ---------------------------------------------------------------------------
constexpr int TL_LEAVES = 7;
constexpr float TL_C_INNER = 1.2f;
// A wave starts from PER leaves and a block is two waves, whose 2 PER leaves make the
// part of the tree built in LDS.  The fewer leaves a wave has, the fewer treelets of one
// level it does in turn; but the waves should all be resident (four a SIMD: 4,096), so PER
// is the least of 16, 32 and 64 that keeps to that (tl_per_wave).  k_treelets at 320,
// 5,120, 40,000, 100k and 500k faces: with 16 leaves 70, 108, 145, 211, 739 us, with 32 92, 127, 160,
// 198, 558, with 64 117, 170, 197, 219, 466; blocks of 16 waves of 32, which left most
// CUs without one, took 88, 186, 234, 257, 805.
constexpr int TL_WAVES = 2;
constexpr int TL_BLOCK = 64 * TL_WAVES;
constexpr int TL_RESIDENT = 4096;
constexpr int TL_GUARD = 1 << 16;
static inline int tl_per_wave(int nf) {
    return nf <= 16 * TL_RESIDENT ? 16 : nf <= 32 * TL_RESIDENT ? 32 : 64;
}

__device__ __forceinline__ float tl_area(float dx, float dy, float dz) {
#pragma clang fp contract(off)
    return 2.0f * ((dx * dy + dy * dz) + dz * dx);
}

// a subtree as its parent's record holds it
struct TlHalf {
    uint32_t w[8];      // code, box lower xyz, box upper xyz, cost
};
struct TlLds {
    uint32_t ent[TL_LEAVES][8];
    float area[128], opt[128];
    uint32_t part[128];
    uint32_t ids[8];
};

// record words [2 j, 2 j + 1] of a node, j < 8
struct TlLocal {        // the block's records in LDS
    uint64_t* rec;
    int lo;
    __device__ __forceinline__ uint64_t load(int node, int j) const { return rec[8 * (node - lo) + j]; }
    __device__ __forceinline__ void store(int node, int j, uint64_t v) const { rec[8 * (node - lo) + j] = v; }
};
struct TlGlobal {
    uint64_t* rec;
    __device__ __forceinline__ uint64_t load(int node, int j) const {
        return __hip_atomic_load(rec + 8 * (size_t)node + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void store(int node, int j, uint64_t v) const {
        __hip_atomic_store(rec + 8 * (size_t)node + j, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// The splits (P, S ^ P) of the subsets a lane evaluates, as word offsets P | (S ^ P)
// << 8, and the subset itself; by subset size.  Subset S of size s is split at P =
// its lowest bit plus the bits of the rest that c selects, c = 2^(s-1) - 2 .. 0 (the
// order of preference among equal costs).  Sizes 2 to 4: one lane a subset; size 5:
// two lanes (c even, c odd), size 6: eight (c mod 8), size 7: one lane a split.
struct TlPlan {
    uint32_t set[6], s2[1], s3[3], s4[7], s5[8], s6[4], s7[1];     // set[s - 2]: the subset of size s, 0 for none
};
constexpr int TL_PLAN_WORDS = sizeof(TlPlan) / sizeof(uint32_t);
struct TlTable {
    uint32_t w[TL_PLAN_WORDS][64];      // the plan of every lane, word by word
};
constexpr int tl_count(uint32_t v) {
    int c = 0;
    for (; v; v &= v - 1) ++c;
    return c;
}
constexpr uint32_t tl_nth_subset(int size, int nth) {
    for (uint32_t S = 1; S < 128; ++S)
        if (tl_count(S) == size && nth-- == 0) return S;
    return 0;
}
constexpr uint32_t tl_split(uint32_t S, int c) {
    const uint32_t lb = S & (0u - S);
    uint32_t rest = S ^ lb, P = lb;
    for (int b = 0; rest; ++b) {
        const uint32_t low = rest & (0u - rest);
        if (c >> b & 1) P |= low;
        rest ^= low;
    }
    return P | ((S ^ P) << 8);
}
constexpr TlTable tl_table() {
    TlTable t{};
    for (int lane = 0; lane < 64; ++lane) {
        const uint32_t set[6] = {tl_nth_subset(2, lane), tl_nth_subset(3, lane), tl_nth_subset(4, lane),
                                 tl_nth_subset(5, lane >> 1), tl_nth_subset(6, lane >> 3), lane < 63 ? 127u : 0u};
        int w = 0;
        for (int q = 0; q < 6; ++q) t.w[w++][lane] = set[q];
        t.w[w++][lane] = tl_split(set[0], 0);
        for (int q = 0; q < 3; ++q) t.w[w++][lane] = tl_split(set[1], 2 - q);
        for (int q = 0; q < 7; ++q) t.w[w++][lane] = tl_split(set[2], 6 - q);
        for (int q = 0; q < 8; ++q) t.w[w++][lane] = tl_split(set[3], 14 - 2 * q - (lane & 1) < 0 ? 0 : 14 - 2 * q - (lane & 1));
        for (int q = 0; q < 4; ++q) t.w[w++][lane] = tl_split(set[4], 24 - 8 * q + (lane & 7) > 30 ? 30 : 24 - 8 * q + (lane & 7));
        t.w[w++][lane] = tl_split(set[5], lane);
    }
    return t;
}
__constant__ const TlTable TL_TABLE = tl_table();
__device__ __forceinline__ TlPlan tl_plan(int lane) {
    uint32_t w[TL_PLAN_WORDS];
#pragma unroll
    for (int i = 0; i < TL_PLAN_WORDS; ++i) w[i] = TL_TABLE.w[i][lane];
    return __builtin_bit_cast(TlPlan, w);
}

// value of lane + N / lane - N of the same 16 (DPP row shift)
template <int N> __device__ __forceinline__ uint32_t lane_up(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + N, 0xf, 0xf, true);
}
template <int N> __device__ __forceinline__ uint32_t lane_down(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + N, 0xf, 0xf, true);
}
// value of the lane at xor 1, xor 2, and mirrored within 8
__device__ __forceinline__ uint32_t lane_x1(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t lane_x2(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t lane_m8(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t pull(uint32_t v, int lane) { return (uint32_t)__shfl((int)v, lane, 64); }

// (cost, P) of the better split: less cost, on ties the larger P (larger c: P and c
// order alike within one subset)
__device__ __forceinline__ void tl_better(float& c, uint32_t& P, float c2, uint32_t P2) {
    if (c2 < c || (c2 == c && P2 > P)) { c = c2; P = P2; }
}
template <int N>
__device__ __forceinline__ void tl_try(const TlLds& T, const uint32_t (&sp)[N], float& c, uint32_t& P) {
#pragma clang fp contract(off)
    c = T.opt[sp[0] & 255u] + T.opt[sp[0] >> 8];
    P = sp[0] & 255u;
#pragma unroll
    for (int q = 1; q < N; ++q) {
        const float x = T.opt[sp[q] & 255u] + T.opt[sp[q] >> 8];
        if (x < c) { c = x; P = sp[q] & 255u; }     // in order of preference
    }
}

// Restructures the treelet of root r (its record complete, everything below final);
// returns the SAH cost of its new subtree.  Called by a whole wave.
template <class Mem>
__device__ __forceinline__ float treelet(const Mem& mem, int r, int lane, TlLds& T, const TlPlan& plan) {
#pragma clang fp contract(off)
    const int j = lane & 7, g = lane >> 3, base = lane & ~7;
    // the list: entry g in lanes 8 g .. 8 g + 7, one word of its half each (e), and
    // two words each of its own record (rx, ry) where it is internal
    uint32_t e = 0, rx = 0, ry = 0;
    if (g == 0) {
        const uint64_t v = mem.load(r, j);
        rx = (uint32_t)v;
        ry = (uint32_t)(v >> 32);
    }
    int b = 0, id[6];
    id[0] = r;
#pragma unroll
    for (int k = 0; k < TL_LEAVES - 1; ++k) {
        // entry b of the k (the root at k = 0) leaves the list, the later ones move
        // down, its children become entries k - 1 and k
        const int nk = k == 0 ? 2 : k + 2, c0 = nk - 2;
        const int from = g == c0 ? 8 * b + (j >> 1) : 8 * b + 4 + (j >> 1);
        const uint32_t cx = pull(rx, from), cy = pull(ry, from);
        const int mv = g >= b ? min(lane + 8, 63) : lane;
        const uint32_t me = pull(e, mv), mx = pull(rx, mv), my = pull(ry, mv);
        const bool fresh = g == c0 || g == c0 + 1;
        e = fresh ? (j & 1 ? cy : cx) : me;
        rx = mx;
        ry = my;
        if (k == TL_LEAVES - 2) break;
        const uint32_t code = pull(e, base);
        if (fresh && !(code & LEAF_BIT)) {
            const uint64_t v = mem.load((int)code, j);
            rx = (uint32_t)v;
            ry = (uint32_t)(v >> 32);
        }
        // the internal entry of largest area, first of the list on ties: box extents
        // in lanes j = 1..3 of an entry, its area in lane j = 1
        const float d = __uint_as_float(lane_up<3>(e)) - __uint_as_float(e);
        const float ar = tl_area(d, __uint_as_float(lane_up<1>(__float_as_uint(d))), __uint_as_float(lane_up<2>(__float_as_uint(d))));
        const uint32_t key = (lane_down<1>(e) & LEAF_BIT) ? 0u : ar >= 0.0f ? __float_as_uint(ar) + 1u : 1u;
        uint32_t best = 0;
#pragma unroll
        for (int i = 0; i < nk; ++i) {
            const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)key, 8 * i + 1);
            if (a > best) { best = a; b = i; }
        }
        id[k + 1] = __builtin_amdgcn_readlane((int)e, 8 * b);
    }
    wave_sync_lds();
    if (lane < 8 * TL_LEAVES) T.ent[g][j] = e;
    wave_sync_lds();
    // the internal nodes other than r in ascending id order
#pragma unroll
    for (int i = 2; i < 6; ++i)
#pragma unroll
        for (int q = i; q > 1; --q) {
            const int lo = min(id[q - 1], id[q]), hi = max(id[q - 1], id[q]);
            id[q - 1] = lo;
            id[q] = hi;
        }
    // boxes of the subsets lane (entries 0..5) and lane + 64 (with entry 6)
    float lo[3] = {__int_as_float(0x7f800000), __int_as_float(0x7f800000), __int_as_float(0x7f800000)};
    float hi[3] = {-__int_as_float(0x7f800000), -__int_as_float(0x7f800000), -__int_as_float(0x7f800000)};
#pragma unroll
    for (int i = 0; i < TL_LEAVES - 1; ++i)
        if (lane >> i & 1)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                lo[q] = fminf(lo[q], __uint_as_float(T.ent[i][1 + q]));
                hi[q] = fmaxf(hi[q], __uint_as_float(T.ent[i][4 + q]));
            }
    T.area[lane] = tl_area(hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        lo[q] = fminf(lo[q], __uint_as_float(T.ent[TL_LEAVES - 1][1 + q]));
        hi[q] = fmaxf(hi[q], __uint_as_float(T.ent[TL_LEAVES - 1][4 + q]));
    }
    T.area[lane + 64] = tl_area(hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2]);
    if (lane < TL_LEAVES) T.opt[1 << lane] = __uint_as_float(T.ent[lane][7]);
    if (lane < 6) T.ids[lane] = (uint32_t)(lane == 0 ? id[0] : lane == 1 ? id[1] : lane == 2 ? id[2] : lane == 3 ? id[3] : lane == 4 ? id[4] : id[5]);
    wave_sync_lds();
    float ar[8];
#pragma unroll
    for (int s = 2; s < 8; ++s) ar[s] = T.area[plan.set[s - 2]];
    float c;
    uint32_t P;
    auto settle = [&](int s, bool writes) {
        if (writes && plan.set[s - 2]) {
            T.opt[plan.set[s - 2]] = TL_C_INNER * ar[s] + c;
            T.part[plan.set[s - 2]] = P;
        }
        wave_sync_lds();
    };
    tl_try(T, plan.s2, c, P);
    settle(2, true);
    tl_try(T, plan.s3, c, P);
    settle(3, true);
    tl_try(T, plan.s4, c, P);
    settle(4, true);
    tl_try(T, plan.s5, c, P);
    tl_better(c, P, __uint_as_float(lane_x1(__float_as_uint(c))), lane_x1(P));
    settle(5, (lane & 1) == 0);
    tl_try(T, plan.s6, c, P);
    tl_better(c, P, __uint_as_float(lane_x1(__float_as_uint(c))), lane_x1(P));
    tl_better(c, P, __uint_as_float(lane_x2(__float_as_uint(c))), lane_x2(P));
    tl_better(c, P, __uint_as_float(lane_m8(__float_as_uint(c))), lane_m8(P));
    settle(6, j == 0);
    tl_try(T, plan.s7, c, P);
    if (!plan.set[5]) { c = __int_as_float(0x7f800000); P = 0; }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) tl_better(c, P, __uint_as_float(pull(__float_as_uint(c), lane ^ o)), pull(P, lane ^ o));
    settle(7, lane == 0);
    const float cost = T.opt[127];
    // the new tree's internal nodes along its preorder: node i's first child, where
    // internal, is node i + 1, its second node i + |first|
    uint64_t pre = 127u;
#pragma unroll
    for (int i = 0; i < TL_LEAVES - 1; ++i) {
        const uint32_t S = (uint32_t)(pre >> (8 * i)) & 255u;
        const uint32_t A = (uint32_t)__builtin_amdgcn_readfirstlane((int)T.part[S]), Q = S ^ A;
        if (A & (A - 1)) pre |= (uint64_t)A << (8 * (i + 1));
        if (Q & (Q - 1)) pre |= (uint64_t)Q << (8 * (i + __popc(A)));
    }
    // their records: node g, words 2 j and 2 j + 1
    if (g < TL_LEAVES - 1) {
        const uint32_t S = (uint32_t)(pre >> (8 * g)) & 255u, A = T.part[S];
        const uint32_t X = j < 4 ? A : S ^ A;
        const int w = 2 * (j & 3);
        uint32_t x, y;
        if (!(X & (X - 1))) {
            const int i = __ffs(X) - 1;
            x = T.ent[i][w];
            y = T.ent[i][w + 1];
        } else {
            float u = w < 4 ? __int_as_float(0x7f800000) : -__int_as_float(0x7f800000), v = w < 3 ? __int_as_float(0x7f800000) : -__int_as_float(0x7f800000);
#pragma unroll
            for (int i = 0; i < TL_LEAVES; ++i)
                if (X >> i & 1) {
                    const float p = __uint_as_float(T.ent[i][w]), q = __uint_as_float(T.ent[i][w + 1]);
                    u = w < 4 ? fminf(u, p) : fmaxf(u, p);
                    v = w < 3 ? fminf(v, q) : fmaxf(v, q);
                }
            x = w == 0 ? T.ids[j < 4 ? g + 1 : g + __popc(A)] : __float_as_uint(u);
            y = w == 6 ? __float_as_uint(T.opt[X]) : __float_as_uint(v);
        }
        mem.store((int)T.ids[g], j, (uint64_t)x | (uint64_t)y << 32);
    }
    wave_sync_lds();
    return cost;
}

// One wave's share of the bottom-up pass in one kind of memory.  h: the finished
// subtree a lane brings, up: its parent and side; lanes with on false have none.
// count(node) adds an arrival and returns those before; inside(node): whether this
// pass builds that node.  A lane whose subtree's parent is not inside keeps it and
// leaves the pass (on stays true).
template <class Mem, class Inside, class Count>
__device__ __forceinline__ void tl_climb(const Mem& mem, TlHalf& h, int& up, bool& on, int lane,
                                         const int* __restrict__ kup, const int2* __restrict__ range, TlLds& T,
                                         const TlPlan& plan, uint32_t* err, Inside inside, Count count) {
#pragma clang fp contract(off)
    bool active = on && up >= 0 && inside(up >> 1);
    for (int guard = 0; __ballot(active); ++guard) {
        if (guard == TL_GUARD) { atomicOr(err, ERR_LOOP); return; }
        const int node = up >> 1;
        bool own = false;
        if (active) {
#pragma unroll
            for (int q = 0; q < 4; ++q) mem.store(node, 4 * (up & 1) + q, (uint64_t)h.w[2 * q] | (uint64_t)h.w[2 * q + 1] << 32);
            handoff_release();
            own = count(node) != 0;                     // else the other subtree is not done yet
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            if (!own) active = on = false;
        }
        bool big = false;
        if (own) {
            uint32_t o[8];                              // the other child's half
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t v = mem.load(node, 4 * (~up & 1) + q);
                o[2 * q] = (uint32_t)v;
                o[2 * q + 1] = (uint32_t)(v >> 32);
            }
            const float k0 = __uint_as_float(up & 1 ? o[7] : h.w[7]), k1 = __uint_as_float(up & 1 ? h.w[7] : o[7]);
            float lo[3], hi[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                lo[q] = fminf(__uint_as_float(h.w[1 + q]), __uint_as_float(o[1 + q]));
                hi[q] = fmaxf(__uint_as_float(h.w[4 + q]), __uint_as_float(o[4 + q]));
                h.w[1 + q] = __float_as_uint(lo[q]);
                h.w[4 + q] = __float_as_uint(hi[q]);
            }
            const int2 rg = range[node];
            big = rg.y - rg.x + 1 >= TL_LEAVES;
            h.w[0] = (uint32_t)node;
            h.w[7] = __float_as_uint(TL_C_INNER * tl_area(hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2]) + (k0 + k1));
            up = kup[node];
            active = up >= 0 && inside(up >> 1);
        }
        for (uint64_t m = __ballot(big); m; m &= m - 1) {
            const int src = __ffsll((unsigned long long)m) - 1;
            const float c = treelet(mem, __builtin_amdgcn_readlane((int)h.w[0], src), lane, T, plan);
            if (lane == src) h.w[7] = __float_as_uint(c);
        }
    }
}

template <int PER>
__global__ __launch_bounds__(TL_BLOCK) void k_treelets(const int* __restrict__ kup, const int2* __restrict__ range,
                                                       const uint32_t* __restrict__ sface, const float4* __restrict__ bmin,
                                                       const float4* __restrict__ bmax, int n, uint32_t* rec, int* cnt,
                                                       uint32_t* err) {
    constexpr int SPAN = PER * TL_WAVES;
    __shared__ uint64_t recs[8 * SPAN];
    __shared__ int cnts[SPAN];
    __shared__ TlLds lds[TL_WAVES];
    const int lane = threadIdx.x & 63, w = (int)(threadIdx.x >> 6);
    TlLds& T = lds[w];
    const int lo = blockIdx.x * SPAN, hi = min(n, lo + SPAN) - 1;
    for (int i = threadIdx.x; i < SPAN; i += TL_BLOCK) cnts[i] = 0;
    const TlPlan plan = tl_plan(lane);
    const int leaf = lo + w * PER + lane;
    bool on = lane < PER && leaf <= hi;
    TlHalf h;
    int up = -1;
    if (on) {
        const int f = (int)sface[leaf];
        const float4 a = bmin[f], b = bmax[f];
        h.w[0] = LEAF_BIT | (uint32_t)leaf;
        h.w[1] = __float_as_uint(a.x); h.w[2] = __float_as_uint(a.y); h.w[3] = __float_as_uint(a.z);
        h.w[4] = __float_as_uint(b.x); h.w[5] = __float_as_uint(b.y); h.w[6] = __float_as_uint(b.z);
        h.w[7] = __float_as_uint(tl_area(b.x - a.x, b.y - a.y, b.z - a.z));
        up = kup[(n - 1) + leaf];
    }
    __syncthreads();
    auto local = [&](int node) {
        const int2 rg = range[node];
        return rg.x >= lo && rg.y <= hi;
    };
    const TlLocal lmem{recs, lo};
    tl_climb(lmem, h, up, on, lane, kup, range, T, plan, err, local, [&](int node) { return atomicAdd(&cnts[node - lo], 1); });
    __syncthreads();
    // the block's records, for the treelets above and the passes after
    const TlGlobal gmem{(uint64_t*)rec};
    for (int i = threadIdx.x; i < 8 * (hi - lo + 1); i += TL_BLOCK) {
        const int node = lo + (i >> 3);
        if (node < n - 1 && local(node)) gmem.store(node, i & 7, recs[i]);
    }
    handoff_release();
    __syncthreads();
    tl_climb(gmem, h, up, on, lane, kup, range, T, plan, err, [](int) { return true; }, [&](int node) { return atomicAdd(&cnt[node], 1); });
}

// the tree of the records as arrays: children, parents, boxes (internal nodes, then
// leaves); clears the arrival counters for the next pass
__global__ void k_tree_unpack(const uint32_t* __restrict__ rec, int n, int* child, int* parent, float* aabb, int* cnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    const uint32_t* const r = rec + 16 * (size_t)i;
    cnt[i] = 0;
    for (int s = 0; s < 2; ++s) {
        const int c = (int)r[8 * s];
        const size_t k = (c & (int)LEAF_BIT) ? (size_t)(n - 1) + (c & 0x7FFFFFFF) : (size_t)c;
        child[2 * i + s] = c;
        parent[k] = i;
        for (int q = 0; q < 6; ++q) aabb[6 * k + q] = __uint_as_float(r[8 * s + 1 + q]);
    }
    if (i == 0) {
        parent[0] = -1;
        for (int q = 0; q < 3; ++q) {
            aabb[q] = fminf(__uint_as_float(r[1 + q]), __uint_as_float(r[9 + q]));
            aabb[3 + q] = fmaxf(__uint_as_float(r[4 + q]), __uint_as_float(r[12 + q]));
        }
    }
}

// Collapse of the binary tree into 4-wide nodes with the least summed box area
// of the 4-wide nodes (under the surface-area measure, the expected number of
// node visits of a ray that meets the root box; every triangle stays one leaf
// slot, so triangle tests do not depend on the collapse).  Bottom-up, like the
// refit, every internal node x with children l, r gets
//   D[x][1] = A(x) + min over a, b >= 1, a + b <= 4 of D[l][a] + D[r][b]
//             (x heads a 4-wide node; as a slot of its parent it is one slot)
//   D[x][k] = min(D[x][k - 1], min over a + b = k of D[l][a] + D[r][b]),  k = 2..4
//             (x opened: its subtree fills up to k slots of the enclosing node)
// with D = 0 for a leaf.  Ties keep the first candidate in the order written,
// so the tree is a function of the binary tree alone.  cdec[x]: bits 0-1 and
// 2-3 hold a - 1 and b - 1 of the first line; bits 4 + 2 (k - 2), two per k,
// the a of the second line (0: k - 1 slots).
__device__ __forceinline__ float box_area(const float* b) {
    const float dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
    return 2.0f * (dx * dy + dy * dz + dz * dx);
}

__global__ void k_collapse_cost(const int* __restrict__ parent, const int* __restrict__ child,
                                const float* __restrict__ aabb, int n, int* cnt, float* cost, uint32_t* dec) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int node = parent[(n - 1) + i];
    for (int depth = 0; node >= 0 && depth < 128; ++depth) {
        handoff_release();
        if (atomicAdd(&cnt[node], 1) == 0) return;    // the other child is not done yet
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        float D[2][5];
        for (int j = 0; j < 2; ++j) {
            const int c = child[2 * node + j];
            D[j][0] = 0.0f;
            for (int k = 1; k <= 4; ++k) D[j][k] = (c & (int)LEAF_BIT) ? 0.0f : aload(cost + 4 * (size_t)c + (k - 1));
        }
        float head = __int_as_float(0x7f800000);
        uint32_t d = 0;
        for (int a = 1; a <= 3; ++a)
            for (int b = 1; a + b <= 4; ++b)
                if (D[0][a] + D[1][b] < head) {
                    head = D[0][a] + D[1][b];
                    d = (uint32_t)(a - 1) | ((uint32_t)(b - 1) << 2);
                }
        float Dx[5];
        Dx[1] = box_area(aabb + 6 * (size_t)node) + head;
        for (int k = 2; k <= 4; ++k) {
            float v = Dx[k - 1];
            uint32_t choice = 0;
            for (int a = 1; a < k; ++a)
                if (D[0][a] + D[1][k - a] < v) {
                    v = D[0][a] + D[1][k - a];
                    choice = (uint32_t)a;
                }
            Dx[k] = v;
            d |= choice << (4 + 2 * (k - 2));
        }
        for (int k = 1; k <= 4; ++k)
            __hip_atomic_store((uint32_t*)(cost + 4 * (size_t)node + (k - 1)), __float_as_uint(Dx[k]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        dec[node] = d;
        node = parent[node];
    }
}

// the number of slots (1..k) that node x's subtree takes in the enclosing 4-wide
// node when offered k: fewer while its choice for k is "k - 1 slots"
__device__ __forceinline__ int collapse_slots(uint32_t dx, int k) {
    while (k >= 2 && ((dx >> (4 + 2 * (k - 2))) & 3u) == 0u) --k;
    return k;
}

// flag[x] = 1 when internal node x heads a 4-wide node: the choices of its
// ancestors, replayed from the root down, leave it one slot (the root heads the
// tree).  The path is read upwards into a bit string first.
__global__ void k_collapse_flag(const int* __restrict__ parent, const int* __restrict__ child,
                                const uint32_t* __restrict__ dec, int n, int* flag, uint32_t* err) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    uint64_t bits[2] = {0ull, 0ull};   // bit j: the node at depth j + 1 on the path is a right child
    int depth = 0;
    for (int x = i; parent[x] >= 0; x = parent[x]) {
        if (depth >= 128) {
            // deeper than any radix tree over 64-bit keys: head a node (fewer slots
            // for the parent, never more)
            atomicOr(err, ERR_LOOP);
            flag[i] = 1;
            return;
        }
        const int px = parent[x];
        const uint64_t right = child[2 * px + 1] == x ? 1ull : 0ull;
        bits[depth >> 6] |= right << (depth & 63);
        ++depth;
    }
    // bits hold the path from i upwards: bit depth - 1 is the root's child
    int v = 0, k = 1;      // node on the path and its slot budget (1: heads a 4-wide node)
    for (int lvl = depth - 1; lvl >= 0; --lvl) {
        const uint32_t dv = dec[v];
        int a, b;
        if (k == 1) {
            a = (int)(dv & 3u) + 1;
            b = (int)((dv >> 2) & 3u) + 1;
        } else {
            a = (int)((dv >> (4 + 2 * (k - 2))) & 3u);
            b = k - a;
        }
        const int right = (int)((bits[lvl >> 6] >> (lvl & 63)) & 1ull);
        const int c = child[2 * v + right];
        k = collapse_slots(dec[c], right ? b : a);
        v = c;
    }
    flag[i] = k == 1 ? 1 : 0;
}

// The slots of the 4-wide node of a binary node x that heads one: its children,
// every internal one that does not head a node replaced by its own two children
// until only leaves and heads remain (at most 4 by the costs above), the internal
// ones first, each kind in tree order; but a leaf that tree order puts before the
// second of three internal ones comes first (lead), so that the traversal's order
// of equally near children stays that of the children in tree order.  Returns
// their number, ni of them internal.
__device__ __forceinline__ int node4_slots(const int* __restrict__ child, const int* __restrict__ flag, int x, int sl[4],
                                           int& ni, bool& lead, uint32_t* err) {
    int t[4] = {child[2 * x], child[2 * x + 1], 0, 0};
    int m = 2;
    for (int pass = 0; pass < 3; ++pass) {
        int at = -1;
        for (int s = 0; s < m; ++s)
            if (at < 0 && !(t[s] & (int)LEAF_BIT) && !flag[t[s]]) at = s;
        if (at < 0) break;
        if (m == 4) { atomicOr(err, ERR_LOOP); break; }   // cannot happen: the costs allow at most 4 slots
        const int y = t[at];
        for (int s = m; s > at + 1; --s) t[s] = t[s - 1];
        t[at] = child[2 * y];
        t[at + 1] = child[2 * y + 1];
        ++m;
    }
    ni = 0;
    for (int s = 0; s < m; ++s) ni += t[s] & (int)LEAF_BIT ? 0 : 1;
    lead = m == 4 && ni == 3 && ((t[0] | t[1]) & (int)LEAF_BIT);
    int in = lead ? 1 : 0, lf = lead ? 0 : ni;
    for (int s = 0; s < m; ++s) sl[t[s] & (int)LEAF_BIT ? lf++ : in++] = t[s];
    return m;
}

// Where the children of every 4-wide node start: the exclusive sums, over the
// binary nodes in index order, of the internal slots (nodes, after the root) and
// of the leaf slots (triangle records) of those that head one.  Tiles of
// PACK_TILE nodes: k_pack_count leaves each node's sum inside its tile and the
// tile's totals, k_pack_scan adds the tiles before.
__device__ __forceinline__ uint2 block_scan_pair(uint2 v, uint2& total, uint2* lds) {
    // exclusive over the block, in thread order; lds holds PACK_TILE / 64 + 1
    uint2 inc = v;
    const int lane = (int)__lane_id(), w = (int)(threadIdx.x >> 6);
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(inc.x, o, 64), y = __shfl_up(inc.y, o, 64);
        if (lane >= o) { inc.x += x; inc.y += y; }
    }
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    uint2 before = make_uint2(0u, 0u), all = make_uint2(0u, 0u);
    for (int j = 0; j < PACK_TILE / 64; ++j) {
        const uint2 x = lds[j];
        if (j < w) { before.x += x.x; before.y += x.y; }
        all.x += x.x; all.y += x.y;
    }
    __syncthreads();
    total = all;
    return make_uint2(before.x + inc.x - v.x, before.y + inc.y - v.y);
}

__global__ void __launch_bounds__(PACK_TILE) k_pack_count(const int* __restrict__ child, const int* __restrict__ flag, int n,
                                                          uint2* slots, uint2* tiles, uint32_t* err) {
    __shared__ uint2 lds[PACK_TILE / 64];
    const int i = blockIdx.x * PACK_TILE + threadIdx.x;
    uint2 v = make_uint2(0u, 0u);
    if (i < n - 1 && flag[i]) {
        int sl[4], ni;
        bool lead;
        const int m = node4_slots(child, flag, i, sl, ni, lead, err);
        v = make_uint2((uint32_t)ni, (uint32_t)(m - ni));
    }
    uint2 tot;
    const uint2 e = block_scan_pair(v, tot, lds);
    if (i < n - 1) slots[i] = e;
    if (threadIdx.x == 0) tiles[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(PACK_TILE) k_pack_scan(int n, uint2* slots, const uint2* __restrict__ tiles) {
    __shared__ uint2 lds[PACK_TILE / 64];
    uint2 v = make_uint2(0u, 0u), before;
    for (unsigned t = threadIdx.x; t < blockIdx.x; t += PACK_TILE) { v.x += tiles[t].x; v.y += tiles[t].y; }
    block_scan_pair(v, before, lds);
    const int i = blockIdx.x * PACK_TILE + threadIdx.x;
    if (i < n - 1) { slots[i].x += before.x + 1u; slots[i].y += before.y; }     // node 0 is the root
}

// 4-wide node of a binary node that heads one (8 float4: min x, max x, min y,
// max y, min z, max z of the 4 slots; byte offsets of slot 0's node and triangle
// record, internal slots (-1: slots 1..3, after a leaf); the same as indices) and
// the records of its triangles.  Slot 0's node or triangle is as if the kind's
// slots began there.  Its own place follows from its parent's.
__global__ void k_pack4(const int* __restrict__ child, const int* __restrict__ parent, const float* __restrict__ aabb,
                        const int* __restrict__ flag, const uint2* __restrict__ slots, const uint32_t* __restrict__ sface,
                        const float* __restrict__ V, const int* __restrict__ F, int n, float4* nodes4, float4* tri,
                        int* fleaf, uint32_t* err) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1 || !flag[i]) return;
    int sl[4], ni;
    bool lead;
    uint32_t id = 0;
    if (parent[i] >= 0) {
        int h = parent[i];
        while (!flag[h]) h = parent[h];
        node4_slots(child, flag, h, sl, ni, lead, err);
        id = slots[h].x;
        for (int s = lead ? 1 : 0; s < 3 && sl[s] != i; ++s) ++id;
    }
    const int m = node4_slots(child, flag, i, sl, ni, lead, err);
    const uint32_t first = slots[i].x - (lead ? 1u : 0u), tri0 = slots[i].y - (lead ? 0u : (uint32_t)ni);
    const int inner = lead ? -1 : ni;
    float v[6][4];
    for (int s = 0; s < 4; ++s) {
        if (s < m) {
            const int c = sl[s];
            const bool is_leaf = c & (int)LEAF_BIT;
            const float* bb = aabb + 6 * (is_leaf ? (size_t)(n - 1) + (c & 0x7FFFFFFF) : (size_t)c);
            v[0][s] = bb[0]; v[1][s] = bb[3]; v[2][s] = bb[1]; v[3][s] = bb[4]; v[4][s] = bb[2]; v[5][s] = bb[5];
            if (is_leaf) put_tri(V, F, (int)sface[c & 0x7FFFFFFF], tri0 + (uint32_t)s, tri, fleaf);
        } else {
            // an empty slot is an inverted box, min +inf and max -inf on every axis:
            // its near planes are at +inf and its far planes at -inf for any ray
            v[0][s] = v[2][s] = v[4][s] = __int_as_float(0x7f800000);
            v[1][s] = v[3][s] = v[5][s] = -__int_as_float(0x7f800000);
        }
    }
    float4* o = nodes4 + 8 * (size_t)id;
    for (int k = 0; k < 6; ++k) o[k] = make_float4(v[k][0], v[k][1], v[k][2], v[k][3]);
    o[6] = make_float4(__uint_as_float(first * NODE_BYTES), __uint_as_float(tri0 * TRI_BYTES), __int_as_float(inner), 0.f);
    o[7] = make_float4(__uint_as_float(first), __uint_as_float(tri0), __int_as_float(inner), 0.f);
}

__global__ void k_keys64(const uint32_t* __restrict__ m, const uint32_t* __restrict__ fa, int n, uint64_t* out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = ((uint64_t)m[i] << 32) | fa[i];
}

__global__ void __launch_bounds__(CDF_BLOCK) k_edge_len(const int4* __restrict__ edges, int ne, const float* __restrict__ V,
                                                        double* w, double* tiles) {
    double s = 0.0;
    for (int q = 0; q < CDF_PER; ++q) {
        const int e = blockIdx.x * CDF_TILE + threadIdx.x * CDF_PER + q;
        if (e >= ne) break;
        const int4 E = edges[e];
        const double dx = (double)V[3 * E.y] - (double)V[3 * E.x];
        const double dy = (double)V[3 * E.y + 1] - (double)V[3 * E.x + 1];
        const double dz = (double)V[3 * E.y + 2] - (double)V[3 * E.x + 2];
        w[e] = sqrt(dx * dx + dy * dy + dz * dz);
        s += w[e];
    }
    cdf_tile_sum(s, tiles);
}

__global__ void __launch_bounds__(CDF_BLOCK) k_edge_cdf(const double* w, const double* tiles, int ne, double* cdf,
                                                        double* total, float* ftotal) {
    const double t = cdf_tile_write(w, ne, tiles, cdf, total);
    if (blockIdx.x == 0 && threadIdx.x == 0) *ftotal = (float)t;
}

// environment map: per-row texel weights (mean rgb times row solid angle) and
// conditional CDFs, summed serially per row; marginal over rows serially.
__global__ void k_env_rows(const float* __restrict__ env, int he, int we, const double* __restrict__ dom,
                           double* cond, double* rows) {
#pragma clang fp contract(off)
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= he) return;
    double acc = 0.0;
    double* C = cond + (size_t)r * (we + 1);
    C[0] = 0.0;
    for (int c = 0; c < we; ++c) {
        const float* t = env + 3 * ((size_t)r * we + c);
        const double m = ((double)t[0] + (double)t[1] + (double)t[2]) / 3.0;
        acc += m * dom[r];
        C[c + 1] = acc;
    }
    rows[r] = acc;
    for (int c = 0; c <= we; ++c) C[c] = acc > 0.0 ? C[c] / acc : (double)c / we;
}

__global__ void k_env_marg(const double* rows, int he, double* marg, double* total) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double acc = 0.0;
    marg[0] = 0.0;
    for (int r = 0; r < he; ++r) { acc += rows[r]; marg[r + 1] = acc; }
    *total = acc;
    for (int r = 0; r <= he; ++r) marg[r] = acc > 0.0 ? marg[r] / acc : 0.0;
}

__global__ void k_env_pdf(const float* __restrict__ env, int he, int we, const double* __restrict__ dom,
                          const double* __restrict__ total, float* texpdf) {
#pragma clang fp contract(off)
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= he * we) return;
    const int r = i / we;
    const float* t = env + 3 * (size_t)i;
    const double m = ((double)t[0] + (double)t[1] + (double)t[2]) / 3.0;
    const double tot = *total;
    texpdf[i] = tot > 0.0 ? (float)((m * dom[r]) / tot / dom[r]) : 0.0f;
}

// guide tables: for CDF row y (blockIdx.y), guide[g] = largest i in [0, n-1]
// with C[i] <= g / 2^glog (C[0] == 0)
__global__ void k_guide(const double* __restrict__ C, int n, size_t cstride, int* guide, int glog) {
    const int G = 1 << glog;
    const double* Cr = C + cstride * blockIdx.y;
    int* gr = guide + ((size_t)blockIdx.y << glog);
    for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < G; g += gridDim.x * blockDim.x)
        gr[g] = cdf_find(Cr, n, (double)g / (double)G);
}

void launch_guide(const double* C, int n, size_t cstride, int rows, int* guide, int glog, hipStream_t st) {
    if (n <= 0 || rows <= 0) return;
    const int G = 1 << glog;
    ST_LAUNCH("k_guide", k_guide, dim3((G + 255) / 256 < 1024 ? (G + 255) / 256 : 1024, rows), dim3(256), 0, st, C, n,
              cstride, guide, glog);
}

int guide_log2(int n) {
    int l = 0;
    while ((1 << l) < n && l < 24) ++l;
    return l;
}

// 1 -> 4 subdivision (Sec. 3.2 "Subdivision": every edge split at its
// midpoint): vertices [V; midpoint of edge e at nv + e], face f ->
// (v0, m01, m20), (v1, m12, m01), (v2, m20, m12), (m01, m12, m20) at 4f.. 4f+3,
// which keeps every face's orientation
__global__ void k_subdivide(const float* __restrict__ V, const int* __restrict__ F, const int* __restrict__ fe,
                            const int4* __restrict__ edges, int nv, int nf, int ne, float* outV, int* outF) {
    const int stride = gridDim.x * blockDim.x;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 3 * nv; i += stride) outV[i] = V[i];
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += stride) {
        const int4 E = edges[e];
        for (int c = 0; c < 3; ++c) outV[3 * (size_t)(nv + e) + c] = (V[3 * E.x + c] + V[3 * E.y + c]) * 0.5f;
    }
    for (int f = blockIdx.x * blockDim.x + threadIdx.x; f < nf; f += stride) {
        const int v0 = F[3 * f], v1 = F[3 * f + 1], v2 = F[3 * f + 2];
        // a degenerate edge (both ends one vertex) has that vertex as its midpoint
        const int m01 = fe[3 * f] >= 0 ? nv + fe[3 * f] : v0;
        const int m12 = fe[3 * f + 1] >= 0 ? nv + fe[3 * f + 1] : v1;
        const int m20 = fe[3 * f + 2] >= 0 ? nv + fe[3 * f + 2] : v2;
        int* o = outF + 12 * (size_t)f;
        o[0] = v0;  o[1] = m01; o[2] = m20;
        o[3] = v1;  o[4] = m12; o[5] = m01;
        o[6] = v2;  o[7] = m20; o[8] = m12;
        o[9] = m01; o[10] = m12; o[11] = m20;
    }
}


// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static inline unsigned nb(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

void launch_subdivide(const SceneDev& s, float* out_V, int32_t* out_F, hipStream_t st) {
    const long long n = std::max<long long>(std::max<long long>(3ll * s.nv, s.ne), s.nf);
    ST_LAUNCH("k_subdivide", k_subdivide, dim3(nb(n, 256) < 4096 ? nb(n, 256) : 4096), dim3(256), 0, st, s.V, s.F,
              s.fe, s.edges, s.nv, s.nf, s.ne, out_V, out_F);
}


// ---------------------------------------------------------------------------
// secondary-edge importance tree: the same radix tree over the edges' boxes,
// each node also carrying the float sum of the edge lengths below it
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(BND_BLOCK) k_edge_prep(const float* __restrict__ V, const int4* __restrict__ edges, int ne,
                                                         float4* bmin, float4* bmax, float4* cen, Bounds* bounds) {
#pragma clang fp contract(off)
    Bounds bb = bounds_none();
    for (int q = 0; q < BND_TILE / BND_BLOCK; ++q) {
        const int e = blockIdx.x * BND_TILE + q * BND_BLOCK + threadIdx.x;
        if (e >= ne) break;
        const int4 E = edges[e];
        const V3 a = ld3(V + 3 * E.x), c = ld3(V + 3 * E.y);
        const V3 mn{fminf(a.x, c.x), fminf(a.y, c.y), fminf(a.z, c.z)};
        const V3 mx{fmaxf(a.x, c.x), fmaxf(a.y, c.y), fmaxf(a.z, c.z)};
        bmin[e] = make_float4(mn.x, mn.y, mn.z, 0.f);
        bmax[e] = make_float4(mx.x, mx.y, mx.z, 0.f);
        const float cx = mn.x + mx.x, cy = mn.y + mx.y, cz = mn.z + mx.z;
        cen[e] = make_float4(cx * 0.5f, cy * 0.5f, cz * 0.5f, 0.f);
        bounds_add(bb, cx * 0.5f, cy * 0.5f, cz * 0.5f);
    }
    bb = block_bounds(bb);
    if (threadIdx.x == 0) bounds[blockIdx.x] = bb;
}

// unit normal of face f: the double cross product of the float edge vectors over
// its double length, rounded to float; false for a degenerate face
__device__ __forceinline__ bool unit_normal_d(const float* __restrict__ V, const int* __restrict__ F, int f,
                                              float* un) {
#pragma clang fp contract(off)
    double q[3][3];
    for (int a = 0; a < 3; ++a) {
        const int v = F[3 * f + a];
        for (int k = 0; k < 3; ++k) q[a][k] = (double)V[3 * v + k];
    }
    const double e1x = q[1][0] - q[0][0], e1y = q[1][1] - q[0][1], e1z = q[1][2] - q[0][2];
    const double e2x = q[2][0] - q[0][0], e2y = q[2][1] - q[0][1], e2z = q[2][2] - q[0][2];
    const double cx = e1y * e2z - e1z * e2y, cy = e1z * e2x - e1x * e2z, cz = e1x * e2y - e1y * e2x;
    const double l = sqrt((cx * cx + cy * cy) + cz * cz);
    if (!(l > 0.0) || !isfinite(l)) return false;
    un[0] = (float)(cx / l); un[1] = (float)(cy / l); un[2] = (float)(cz / l);
    return true;
}

// leaves of the edge tree in sorted order: box, length (the double-precision
// length of the float endpoints, rounded to float) and the box of the adjacent
// faces' unit normals (the whole cube [-1, 1]^3, which never culls, for a
// boundary edge or a degenerate face); clears the refit counters
__global__ void k_eleaf_init(const uint32_t* __restrict__ sedge, const float4* __restrict__ bmin,
                             const float4* __restrict__ bmax, const int4* __restrict__ edges,
                             const float* __restrict__ V, const int* __restrict__ F, int n, float* aabb, float* len,
                             float* nbox, int* cnt) {
#pragma clang fp contract(off)
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n - 1) cnt[i] = 0;
    if (i >= n) return;
    const int e = (int)sedge[i];
    float* bx = aabb + 6 * ((size_t)(n - 1) + i);
    const float4 mn = bmin[e], mx = bmax[e];
    bx[0] = mn.x; bx[1] = mn.y; bx[2] = mn.z; bx[3] = mx.x; bx[4] = mx.y; bx[5] = mx.z;
    const int4 E = edges[e];
    const double dx = (double)V[3 * E.y] - (double)V[3 * E.x];
    const double dy = (double)V[3 * E.y + 1] - (double)V[3 * E.x + 1];
    const double dz = (double)V[3 * E.y + 2] - (double)V[3 * E.x + 2];
    len[(size_t)(n - 1) + i] = (float)sqrt((dx * dx + dy * dy) + dz * dz);
    float nb[6] = {-1.0f, -1.0f, -1.0f, 1.0f, 1.0f, 1.0f};
    float n1[3], n2[3];
    if (E.w >= 0 && unit_normal_d(V, F, E.z, n1) && unit_normal_d(V, F, E.w, n2))
        for (int k = 0; k < 3; ++k) {
            nb[k] = fminf(n1[k], n2[k]);
            nb[3 + k] = fmaxf(n1[k], n2[k]);
        }
    float* o = nbox + 6 * ((size_t)(n - 1) + i);
    for (int k = 0; k < 6; ++k) o[k] = nb[k];
}

// bottom-up boxes and length sums of the edge tree (second arrival at a node
// combines its two children, as in the refit)
__global__ void k_erefit(const int* __restrict__ parent, const int* __restrict__ child, int n, float* aabb,
                         float* len, float* nbox, int* cnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int node = parent[(n - 1) + i];
    for (int depth = 0; node >= 0 && depth < 4096; ++depth) {
        handoff_release();
        if (atomicAdd(&cnt[node], 1) == 0) return;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        const int c0 = child[2 * node], c1 = child[2 * node + 1];
        const size_t i0 = (c0 & (int)LEAF_BIT) ? (size_t)(n - 1) + (c0 & 0x7FFFFFFF) : (size_t)c0;
        const size_t i1 = (c1 & (int)LEAF_BIT) ? (size_t)(n - 1) + (c1 & 0x7FFFFFFF) : (size_t)c1;
        float box[6];
        for (int k = 0; k < 3; ++k) {
            box[k] = fminf(aload(aabb + 6 * i0 + k), aload(aabb + 6 * i1 + k));
            box[3 + k] = fmaxf(aload(aabb + 6 * i0 + 3 + k), aload(aabb + 6 * i1 + 3 + k));
        }
        for (int k = 0; k < 6; ++k)
            __hip_atomic_store((uint32_t*)(aabb + 6 * (size_t)node + k), __float_as_uint(box[k]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        for (int k = 0; k < 3; ++k) {
            box[k] = fminf(aload(nbox + 6 * i0 + k), aload(nbox + 6 * i1 + k));
            box[3 + k] = fmaxf(aload(nbox + 6 * i0 + 3 + k), aload(nbox + 6 * i1 + 3 + k));
        }
        for (int k = 0; k < 6; ++k)
            __hip_atomic_store((uint32_t*)(nbox + 6 * (size_t)node + k), __float_as_uint(box[k]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        const float l = aload(len + i0) + aload(len + i1);
        __hip_atomic_store((uint32_t*)(len + node), __float_as_uint(l), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        node = parent[node];
    }
}

// packed record of internal node i of the edge tree: for child j, float4s
// 4j..4j+3 hold its box (lower, upper), length, normal box (lower, upper) and code
__global__ void k_epack(const int* __restrict__ child, const float* __restrict__ aabb, const float* __restrict__ len,
                        const float* __restrict__ nbox, int n, float4* node) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    for (int j = 0; j < 2; ++j) {
        const int c = child[2 * i + j];
        const size_t k = (c & (int)LEAF_BIT) ? (size_t)(n - 1) + (c & 0x7FFFFFFF) : (size_t)c;
        const float* b = aabb + 6 * k;
        const float* nb = nbox + 6 * k;
        float4* o = node + 8 * (size_t)i + 4 * j;
        o[0] = make_float4(b[0], b[1], b[2], b[3]);
        o[1] = make_float4(b[4], b[5], len[k], nb[0]);
        o[2] = make_float4(nb[1], nb[2], nb[3], nb[4]);
        o[3] = make_float4(nb[5], __int_as_float(c), 0.0f, 0.0f);
    }
}

// Morton keys of n centres with these block bounds, stably sorted (4 LSD passes);
// returns the buffer index that holds the sorted (key, value) pairs
static int radix_sort_keys(const float4* cen, int n, const Bounds* bounds, uint32_t* const mk[2], uint32_t* const mv[2],
                           uint32_t* hist, hipStream_t st) {
    const int nblocks = (n + RS_TILE - 1) / RS_TILE;
    ST_LAUNCH("k_morton", k_morton, dim3(nblocks), dim3(RS_THREADS), 0, st, cen, n, bounds, nblocks, mk[0], mv[0], hist);
    int cur = 0;
    for (int shift = 0; shift < 32; shift += 8) {
        if (shift > 0) ST_LAUNCH("k_rs_hist", k_rs_hist, dim3(nblocks), dim3(RS_THREADS), 0, st, mk[cur], n, shift, hist);
        if (nblocks > RS_SUM_TILES) ST_LAUNCH("k_rs_scan", k_rs_scan, dim3(1), dim3(RS_SCAN_THREADS), 0, st, hist, nblocks);
        ST_LAUNCH("k_rs_scatter", k_rs_scatter, dim3(nblocks), dim3(RS_THREADS), 0, st, mk[cur], mv[cur], mk[cur ^ 1],
                  mv[cur ^ 1], n, shift, hist, nblocks);
        cur ^= 1;
    }
    return cur;
}

void launch_edge_tree(SceneDev& s, hipStream_t st) {
    const int n = s.ne;
    if (n <= 0) return;
    ST_LAUNCH("k_edge_prep", k_edge_prep, dim3(nb(n, BND_TILE)), dim3(BND_BLOCK), 0, st, s.V, s.edges, n, s.ebmin, s.ebmax,
              s.ecen, (Bounds*)s.ebounds);
    const int cur = radix_sort_keys(s.ecen, n, (const Bounds*)s.ebounds, s.emkeys, s.emvals, s.ers_hist, st);
    const uint32_t* sm = s.emkeys[cur];
    const uint32_t* se = s.emvals[cur];
    s.eleaf_edge = se;
    ST_LAUNCH("k_keys64", k_keys64, dim3(nb(n, 256)), dim3(256), 0, st, sm, se, n, s.ekeys64);
    if (n > 1) ST_LAUNCH("k_karras", k_karras, dim3(nb(n - 1, 256)), dim3(256), 0, st, sm, se, n, s.echild, s.eparent);
    ST_LAUNCH("k_eleaf_init", k_eleaf_init, dim3(nb(n, 256)), dim3(256), 0, st, se, s.ebmin, s.ebmax, s.edges, s.V,
              s.F, n, s.eaabb, s.elen, s.enbox, s.ecnt);
    if (n > 1) {
        ST_LAUNCH("k_erefit", k_erefit, dim3(nb(n, 256)), dim3(256), 0, st, s.eparent, s.echild, n, s.eaabb, s.elen,
                  s.enbox, s.ecnt);
        ST_LAUNCH("k_epack", k_epack, dim3(nb(n - 1, 256)), dim3(256), 0, st, s.echild, s.eaabb, s.elen, s.enbox, n,
                  s.enode);
    }
}

void launch_scene_geometry(SceneDev& s, hipStream_t st) {
    const int nf = s.nf;
    if (nf <= 0) return;
    ST_LAUNCH("k_face_prep", k_face_prep, dim3(nb(nf, BND_TILE)), dim3(BND_BLOCK), 0, st, s.V, s.F, nf, s.fnorm, s.bmin,
              s.bmax, s.cen, (Bounds*)s.bounds);
    const int cur = radix_sort_keys(s.cen, nf, (const Bounds*)s.bounds, s.mkeys, s.mvals, s.rs_hist, st);
    // after 4 passes the sorted data is back in buffer 0
    const uint32_t* sm = s.mkeys[cur];
    const uint32_t* sf = s.mvals[cur];
    ST_LAUNCH("k_tree_init", k_tree_init, dim3(nb(nf, 256)), dim3(256), 0, st, sm, sf, nf, s.kup, s.krange, s.keys64,
              s.refit_cnt, s.bmin, s.bmax, s.V, s.F, s.aabb, s.tri, s.fleaf);
    if (nf > 1) {
        const int per = tl_per_wave(nf);
        const auto treelets = per == 16 ? k_treelets<16> : per == 32 ? k_treelets<32> : k_treelets<64>;
        ST_LAUNCH("k_treelets", treelets, dim3(nb(nf, per * TL_WAVES)), dim3(TL_BLOCK), 0, st, s.kup, s.krange, sf, s.bmin,
                  s.bmax, nf, s.trec, s.refit_cnt, s.err);
        ST_LAUNCH("k_tree_unpack", k_tree_unpack, dim3(nb(nf - 1, 256)), dim3(256), 0, st, s.trec, nf, s.child, s.parent,
                  s.aabb, s.refit_cnt);
        ST_LAUNCH("k_collapse_cost", k_collapse_cost, dim3(nb(nf, 256)), dim3(256), 0, st, s.parent, s.child, s.aabb,
                  nf, s.refit_cnt, (float*)s.ccost, s.cdec);
        ST_LAUNCH("k_collapse_flag", k_collapse_flag, dim3(nb(nf - 1, 256)), dim3(256), 0, st, s.parent, s.child,
                  s.cdec, nf, s.flag4, s.err);
        const unsigned tiles = nb(nf - 1, PACK_TILE);
        ST_LAUNCH("k_pack_count", k_pack_count, dim3(tiles), dim3(PACK_TILE), 0, st, s.child, s.flag4, nf, s.slots4,
                  s.tiles4, s.err);
        ST_LAUNCH("k_pack_scan", k_pack_scan, dim3(tiles), dim3(PACK_TILE), 0, st, nf, s.slots4, s.tiles4);
        ST_LAUNCH("k_pack4", k_pack4, dim3(nb(nf - 1, 256)), dim3(256), 0, st, s.child, s.parent, s.aabb, s.flag4,
                  s.slots4, sf, s.V, s.F, nf, s.nodes4, s.tri, s.fleaf, s.err);
    }
    if (s.ne > 0) {
        const dim3 tiles((unsigned)cdf_tiles(s.ne));
        ST_LAUNCH("k_edge_len", k_edge_len, tiles, dim3(CDF_BLOCK), 0, st, s.edges, s.ne, s.V, s.edge_w, s.edge_tiles);
        ST_LAUNCH("k_edge_cdf", k_edge_cdf, tiles, dim3(CDF_BLOCK), 0, st, s.edge_w, s.edge_tiles, s.ne, s.ecdf,
                  s.etotal_d, s.etotal_f);
        launch_guide(s.ecdf, s.ne, 0, 1, s.eguide, guide_log2(s.ne), st);
    }
}

void launch_env_build(SceneDev& s, hipStream_t st) {
    if (s.he <= 0) return;
    ST_LAUNCH("k_env_rows", k_env_rows, dim3(nb(s.he, 64)), dim3(64), 0, st, s.env, s.he, s.we, s.row_dom, s.cond,
                       s.env_rows);
    ST_LAUNCH("k_env_marg", k_env_marg, dim3(1), dim3(64), 0, st, s.env_rows, s.he, s.marg, s.env_total);
    launch_guide(s.marg, s.he, 0, 1, s.mguide, guide_log2(s.he), st);
    launch_guide(s.cond, s.we, (size_t)(s.we + 1), s.he, s.cguide, guide_log2(s.we), st);
    ST_LAUNCH("k_env_pdf", k_env_pdf, dim3(nb((long long)s.he * s.we, 256)), dim3(256), 0, st, s.env, s.he, s.we,
                       s.row_dom, s.env_total, s.texpdf);
}

} // namespace st
