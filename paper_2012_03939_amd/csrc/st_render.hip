// Forward rendering R(x, m, c_i) (Shape from Tracing, Sec. 3.2) as a wavefront
// path tracer: per bounce a closest-hit kernel over a compacted ray queue, a
// shading kernel (next-event estimation set-up, BRDF sampling, block-wise
// compaction of the surviving paths and of the shadow entries) and the shadow rays
// of the listed entries, whose contributions are added in a fixed order.  Queues lie
// in HBM in blocks of 64 entries; per-sample radiance is kept for a final film pass
// that averages the samples of each pixel.
#include "st_internal.h"

namespace st {

// occupancy targets (waves per SIMD) the compiler fits the register budget to
#ifndef ST_SHADE_WAVES
#define ST_SHADE_WAVES 6
#endif
#ifndef ST_EXTEND_WAVES
#define ST_EXTEND_WAVES 8
#endif
#ifndef ST_SHADOW_WAVES
#define ST_SHADOW_WAVES 8
#endif
#define SHADE_OCC __attribute__((amdgpu_waves_per_eu(ST_SHADE_WAVES)))
#ifndef ST_SHADE_BLOCK
#define ST_SHADE_BLOCK 512
#endif
constexpr int SHADE_BLOCK = ST_SHADE_BLOCK;   // threads of a k_shade block (one queue reservation each)
#define EXTEND_OCC __attribute__((amdgpu_waves_per_eu(ST_EXTEND_WAVES)))
#define SHADOW_OCC __attribute__((amdgpu_waves_per_eu(ST_SHADOW_WAVES)))



// canonical path index of a (view, pixel, sample)
__device__ __forceinline__ long long canon(const DevCam& c, int x, int y, int j, int spp) {
    return (c.pixoff + (long long)y * c.W + x) * spp + j;
}

// final decision hash of a path: canonical debug slot, or the path's radiance slot
__device__ __forceinline__ void final_hash(const FwdParams& p, const RayRow& r, uint32_t h) {
    if (p.hash_by_q) {
        p.hash_by_q[r.u(QQ)] = h;
    } else if (p.dbg_hash) {
        const DevCam& c = p.cams[r.u(QVD) & 0xFFFFu];
        p.dbg_hash[(c.pixoff + (long long)r.u(QC0)) * p.spp + (r.u(QC1) & 0xFFFFu)] = h;
    }
}

// Clears what the kernels of a pass count in; n: rays of the first bounce.
__device__ __forceinline__ void clear_counters(const Queues& q, int n, int skip_set) {
    const int stride = gridDim.x * blockDim.x, g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < 64) q.cnt[g] = g == 1 ? n : 0;
    for (int j = g; j < TAKE_INTS; j += stride)
        if (j / (TAKE_NC * 32) != skip_set) q.take[j] = 0;
}
__global__ void k_pass_begin(Queues q, int n) { clear_counters(q, n, -1); }

// random counters, and with them camera direction, of path sample qq (processing
// order) of view c
__device__ __forceinline__ Ctr path_ctr(const FwdParams& p, const DevCam& c, long long qq) {
    int x, y, j;
    decode_path(c, qq - c.qoff, p.spp, x, y, j);
    return Ctr{(uint32_t)(y * c.W + x), ((uint32_t)c.rngview << 16) | (uint32_t)j, 0u, 0u};
}
__device__ __forceinline__ V3 path_dir(const FwdParams& p, const DevCam& c, const Ctr& ctr, uint32_t scene_id) {
    const float4 u = draw4(ctr, 0, 0, Key{p.seed, scene_id});
    const uint32_t y = ctr.c0 / (uint32_t)c.W, x = ctr.c0 - y * (uint32_t)c.W;
    return cam_dir(c, (float)(int)x + u.x, (float)(int)y + u.y);
}

// closest hit of queue entry i of bounce k >= 2.  ONE: the launch has one scene,
// whose geometry is GW; else each ray looks its own up
template <bool FAST, bool ONE>
__device__ __forceinline__ void extend_one(const FwdParams& p, const Queues& q, uint32_t* queue, uint32_t i, const TraceGeo& GW,
                                           TravStack& st) {
    const RayRow r(queue, i);
    const TraceGeo G = ONE ? GW : lane_geo(p.scenes[p.cams[r.u(QVD) & 0xFFFFu].scene]);
    const V3 o = r.v(QOX), d = r.v(QDX);
    float t;
    const int f = trace_closest<FAST>(G, o, d, TMIN, (int)r.u(QEXCL), t, st);
    const RecRow c(q.rec, i);
    c.f(RT, t);
    c.u(RF, (uint32_t)f);
}

// Closest hits of the first bounce, 64 consecutive rays per wave, traced in lockstep.
// Camera rays (SIDE false; path samples q0 .. q0 + n - 1) are made here from their
// index: a ray that misses, as most do around a small object, is never written; one
// that hits leaves its direction for k_shade.  Before, a kernel of its own wrote 40
// bytes a ray (0.22 of 5.1 ms for a 1024^2 view at 32 spp) that two kernels read back.
// Side rays come from the queue; each names its edge, whose faces are tested first,
// so that the traversal starts with their hit.
template <bool FAST, bool ONE, bool SIDE>
__global__ void __launch_bounds__(TRACE_BLOCK) EXTEND_OCC k_extend(FwdParams p, Queues q, long long q0, int n_cam) {
    __shared__ uint32_t lds[LDS_STACK * TRACE_BLOCK];
    TravStack st = make_trav_stack(lds, q.spill, p.err, p.work ? p.work + 3 * WORK_EXTEND : nullptr);
    const TraceGeo GW = wave_geo(p.scene);
    const int n = SIDE ? q.cnt[1] : n_cam;
    if (!SIDE) {
        // counters of the launches after this one (its own were cleared before it
        // when it needs them)
        clear_counters(q, n, 0);
        // the hit records are rewritten from here on: their key is cleared until k_film
        if (q0 == 0 && blockIdx.x == 0 && threadIdx.x == 0 && p.rec_key_dev) *p.rec_key_dev = 0ull;
    }
    wave_tiles(q.take, (uint32_t)n, [&](uint32_t tile) {
        const int i = (int)(tile + __lane_id());
        if (i >= n) return;
        float t0 = __int_as_float(0x7f800000);
        int f0 = -1;
        V3 o, d;
        TraceGeo G = GW;
        const RayRow r(q.ray[1], (uint32_t)i);
        if (SIDE) {
            const DevScene& S = p.scene;                // a backward has one scene
            o = ld3(p.cams[r.u(QVD) & 0xFFFFu].eye);
            d = r.v(QDX);
            const int4 E = S.edges[r.u(QEXCL) & 0x7FFFFFFFu];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int fe = j == 0 ? E.z : E.w;
                float th; int fh;
                if (fe >= 0 && tri_test<true>(tri_at(G.tri, (uint32_t)S.fleaf[fe]), o, d, TMIN, __int_as_float(0x7f800000),
                                              th, fh) &&
                    (th < t0 || (th == t0 && fh < f0))) {
                    t0 = th;
                    f0 = fh;
                }
            }
        } else {
            const int v = find_view_from(p.qoff, p.ncam, find_view(p.qoff, p.ncam, q0 + tile), q0 + i);
            const DevCam& c = p.cams[v];
            const DevScene& S = ONE ? p.scene : p.scenes[c.scene];
            if (!ONE) G = lane_geo(S);
            o = ld3(c.eye);
            d = path_dir(p, c, path_ctr(p, c, q0 + i), S.scene_id);
        }
        float t;
        const int f = trace_closest<FAST>(G, o, d, TMIN, -1, t, st, t0, f0);
        const RecRow c(q.rec, (uint32_t)i);
        c.f(RT, t);
        c.u(RF, (uint32_t)f);
        if (!SIDE && f >= 0) r.v(QDX, d);
    });
}

// With one shadow entry per shading point and no decision hashes, k_shadow adds
// each unoccluded contribution itself and records occlusion in the hit records,
// and k_shadow_sum is not launched (the sum over one entry is that entry).
__host__ __device__ __forceinline__ bool shadow_fused(const FwdParams& p, const Queues& q) {
    return q.nent == 1 && !(p.dbg_hash || p.hash_by_q);
}

// shading of bounce k: escapes, next-event set-up and BRDF continuation.
// MODE: one shadow entry per shading point (shadow_fused), several, or several with
// decision hashes asked for (p.dbg_hash or p.hash_by_q); compiled apart, because what
// one of them holds (an entry until its place is known; the hash) is spilled in all.
// ONE: the launch has one scene.  FROM: where the entries come from: later bounces
// (k >= 2), camera rays or side rays (k == 1).
// First bounces are bound by vector issue (80-89 % of the SIMD cycles, 55-66 % of the
// lanes: the misses idle), later ones by memory latency.  Six waves per SIMD: with the
// 80 registers the compiler spills at most 4 dwords; 5, 6 and 8 waves took 21.7, 19.8 and
// 21.1 ms of a 40k-face step of 16 views of 512^2.
enum { FROM_LATER, FROM_CAMERA, FROM_SIDE };
enum { MODE_FUSED, MODE_LISTED, MODE_HASH };
template <int MODE, bool ONE, int FROM>
__global__ void __launch_bounds__(SHADE_BLOCK) SHADE_OCC k_shade(FwdParams p, Queues q, int k, long long q0) {
    __shared__ int resv[2 * (SHADE_BLOCK / 64 + 1)];
    const int n = q.cnt[k];
    const int stride = gridDim.x * blockDim.x;
    constexpr bool hashing = MODE == MODE_HASH, fused = MODE == MODE_FUSED;
    // every thread of a block runs the same number of iterations: the
    // compaction below reserves queue slots per block
    for (int b0 = blockIdx.x * blockDim.x; b0 < n; b0 += stride) {
        const int i = b0 + (int)threadIdx.x;
        const bool active = i < n;
        const RayRow r(q.ray[k & 1], (uint32_t)i);
        const RecRow rec(q.rec, (uint32_t)i);
        bool emit = false;
        uint32_t rays = 0;          // shadow entries of this shading point that carry a ray
        V3 x{0.f, 0.f, 0.f}, wi{0.f, 0.f, 0.f}, beta{0.f, 0.f, 0.f};
        float pb = 0.0f;
        V3 ws{0.f, 0.f, 0.f}, cs{0.f, 0.f, 0.f};    // fused: the entry, until it has its place
        float ts = 0.0f;
        int f = -1;
        uint32_t hv = 0;
        // path identity (slot, counters, camera | domain), carried to the continuation
        uint32_t pq = 0, c0 = 0, c1 = 0, vd = 0;
        if (active) {
            // an entry's words are asked for together, one trip to memory before the
            // gathers; of a first-bounce entry, the hit alone: most of them are misses
            f = (int)rec.u(RF);
            float ht = 0.0f;
            V3 o{0.f, 0.f, 0.f}, d{0.f, 0.f, 0.f};
            beta = V3{1.f, 1.f, 1.f};
            if (FROM == FROM_LATER) {
                pq = r.u(QQ);
                c0 = r.u(QC0);
                c1 = r.u(QC1);
                vd = r.u(QVD);
                ht = rec.f(RT);
                d = r.v(QDX);
                beta = r.v(QBR);
            }
            if (FROM == FROM_CAMERA) {
                pq = (uint32_t)(q0 + i);
                float* L = q.L + 3 * (size_t)pq;
                L[0] = 0.0f; L[1] = 0.0f; L[2] = 0.0f;
            }
            if (FROM == FROM_LATER ? true : f >= 0 || hashing) {
                if (FROM == FROM_CAMERA) {
                    const int v = find_view_from(p.qoff, p.ncam, find_view(p.qoff, p.ncam, q0 + b0), q0 + i);
                    const Ctr cc = path_ctr(p, p.cams[v], q0 + i);
                    c0 = cc.c0;
                    c1 = cc.c1;
                    vd = (uint32_t)v;
                    // for the shadow kernels and the hashes of this bounce
                    if (!fused) {
                        r.u(QQ, pq);
                        r.u(QVD, vd);
                    }
                    if (hashing) { r.u(QC0, c0); r.u(QC1, c1); }
                }
                if (FROM == FROM_SIDE) {
                    pq = r.u(QQ);
                    c0 = r.u(QC0);
                    c1 = r.u(QC1);
                    vd = r.u(QVD);
                }
                if (FROM != FROM_LATER && f >= 0) {
                    ht = rec.f(RT);
                    d = r.v(QDX);
                }
            }
            const DevScene& S = ONE ? p.scene : p.scenes[p.cams[vd & 0xFFFFu].scene];
            const Key key{p.seed, S.scene_id};
            const Ctr ctr{c0, c1, 0u, vd >> 16};
            Hash h{hashing ? (FROM != FROM_LATER ? FNV_INIT : r.u(QHASH)) : 0u, hashing};
            push_face(h, f);
            // (the records belong to main paths: side paths come without them)
            if (FROM != FROM_SIDE && p.rec_face) qst(p.rec_face + (size_t)(k - 1) * p.rec_n + pq, f);
            if (!fused) rec.u(RFACE, 0xFFFFFFFFu);
            if (f < 0) {
                if (S.has_env && FROM == FROM_LATER) {
                    const int tex = env_texel_of(S, d);
                    h.push((uint32_t)tex);
                    const float pp = r.f(QPPREV);
                    const float w = pp / (pp + S.texpdf[tex]);
                    const V3 c = mul(beta, env_rgb(S, tex)) * w;
                    float* L = q.L + 3 * (size_t)pq;
                    L[0] += c.x; L[1] += c.y; L[2] += c.z;
                }
                if (hashing) final_hash(p, r, h.h);
            } else if (k > p.B) {
                if (hashing) final_hash(p, r, h.h);
            } else if (FROM == FROM_SIDE && (int)RecRow(q.rec, (uint32_t)(i ^ 1)).u(RF) == f) {
                // the two side rays of a primary edge sample (queue slots 2j and
                // 2j + 1 at bounce 1) met the same face first: the edge point is
                // hidden behind it, there is no jump to measure, and both side
                // paths end here with zero radiance
                if (hashing) final_hash(p, r, h.h);
            } else {
                o = FROM != FROM_LATER ? ld3(p.cams[vd & 0xFFFFu].eye) : r.v(QOX);
                x = o + d * ht;
                V3 n = xyz(S.fnorm[f]);
                const V3 wo = -d;
                if (dot(n, wo) < 0.0f) n = -n;
                const int tx = texel_of(S, f, x);
                if (S.tex_res) h.push((uint32_t)tx);
                const Mat m = load_mat(S.mat + 7 * (size_t)tx);
                const float lo = out_lambda(wo, n, m);
                for (int l = 0; l < S.nl; ++l) {
                    const auto lt = S.lights + 6 * l;
                    const V3 dl = ld3(lt) - x;
                    const float r2 = dot(dl, dl);
                    float tmax = -1.0f;
                    V3 wl{0.f, 0.f, 0.f}, ct{0.f, 0.f, 0.f};
                    if (r2 > 0.0f) {
                        const float rr = sqrtf(r2);
                        wl = dl * (1.0f / rr);
                        const float c = dot(n, wl);
                        if (c > 0.0f) {
                            tmax = rr * (1.0f - SHADOW_SHRINK);
                            ct = mul(beta, mul(ld3(lt + 3), brdf_eval(wl, wo, n, m, lo))) * (c / r2);
                        }
                    }
                    // an entry is read only when it carries a ray (listed for k_shadow;
                    // k_shadow_sum reads the contribution of an unoccluded one)
                    const size_t e = (size_t)l * q.cap + i;
                    if (tmax >= 0.0f) {
                        if (fused) {
                            ws = wl;
                            ts = tmax;
                            cs = ct;
                        } else {
                            const ShRow sh(q.sh, e);
                            sh.v(SWX, wl);
                            sh.f(STMAX, tmax);
                            sh.v(SCR, ct);
                        }
                        rays |= 1u << l;
                    } else if (!fused) {
                        q.socc[e] = 0;
                    }
                }
                int tex = 0;
                if (S.has_env) {
                    const float4 u = draw4(ctr, k, 1, key);
                    V3 we; float pe;
                    tex = env_sample(S, u, we, pe);
                    const float c = dot(n, we);
                    float tmax = -1.0f;
                    V3 ct{0.f, 0.f, 0.f};
                    if (c > 0.0f && pe > 0.0f) {
                        tmax = __int_as_float(0x7f800000);
                        float pdf;
                        const V3 fe = brdf_eval_pdf(we, wo, n, m, lo, S.vndf, pdf);
                        ct = mul(beta, mul(env_rgb(S, tex), fe)) * (c / (pe + pdf));
                    }
                    const size_t e = (size_t)S.nl * q.cap + i;
                    if (tmax >= 0.0f) {
                        if (fused) {
                            ws = we;
                            ts = tmax;
                            cs = ct;
                        } else {
                            const ShRow sh(q.sh, e);
                            sh.v(SWX, we);
                            sh.f(STMAX, tmax);
                            sh.v(SCR, ct);
                        }
                        rays |= 1u << S.nl;
                    } else if (!fused) {
                        q.socc[e] = 0;
                    }
                }
                uint32_t info = 0;
                if (k < p.B || S.has_env) {
                    const float4 u = draw4(ctr, k, 2, key);
                    const int lobe = bsdf_sample(u, wo, n, m.a, S.vndf, wi);
                    const float ci = dot(n, wi);
                    const V3 fi = brdf_eval_pdf(wi, wo, n, m, lo, S.vndf, pb);
                    info = 1u | ((uint32_t)lobe << 1);
                    if (ci > 0.0f && pb > 0.0f) {
                        info |= 4u;
                        emit = true;
                        beta = mul(beta, fi) * (ci / pb);
                    }
                }
                // the shading record: the shadow rays' origin and excluded face
                if (!fused) {
                    rec.u(RFACE, (uint32_t)f);
                    rec.v(RX0, x);
                }
                if (!fused) rec.u(RINFO, info);
                if (fused && FROM != FROM_SIDE && p.rec_occ)
                    p.rec_occ[(size_t)(k - 1) * p.rec_n + pq] = 0u;
                if (!fused) rec.u(RTEX, (uint32_t)tex);
                if (!fused) rec.u(RNEXT, 0xFFFFFFFFu);
            }
            hv = h.h;
        }
        // compaction of the continuing paths into the next queue, and of the
        // shadow entries that carry a ray (those of one shading point
        // consecutive) into the shadow list of this bounce
        const int2 oo = block_reserve2<SHADE_BLOCK>(emit, __popc(rays), &q.cnt[k + 1], &q.cnt[32 + k], resv);
        const int o = oo.x;
        // the next queue holds one continuation per path of the chunk and the
        // shadow list nent entries per shading point, so this never trips; a
        // reservation past either is reported (ST_ERR_QUEUE_OVERFLOW), not written
        if ((emit && o >= q.cap) || (rays && (long long)oo.y + __popc(rays) > (long long)q.cap * max(q.nent, 1))) {
            atomicOr(p.err, ERR_QUEUE);
            emit = false;
            rays = 0;
        }
        if (fused) {
            if (rays) {
                const ShRow sh(q.sh, (uint32_t)oo.y);
                sh.v(SWX, ws);
                sh.f(STMAX, ts);
                sh.v(SCR, cs);
                const RecRow so(q.rec, (uint32_t)oo.y);
                so.v(RX0, x);
                so.u(RFACE, (uint32_t)f);
                so.u(RSLOT, pq);
                // (the counting traversals look their scene up by ray in any launch)
                if (!ONE || !p.fast) so.u(RVD, vd);
            }
            rays = 0;
        }
        for (int so = oo.y; rays; rays &= rays - 1, ++so)
            qst(q.slist + so, (uint32_t)(__ffs(rays) - 1) * (uint32_t)q.cap + (uint32_t)i);
        if (emit) {
            const RayRow rn(q.ray[(k + 1) & 1], (uint32_t)o);
            rn.v(QOX, x);
            rn.v(QDX, wi);
            rn.u(QEXCL, (uint32_t)f);
            rn.f(QPPREV, pb);
            rn.u(QQ, pq);
            rn.u(QC0, c0);
            rn.u(QC1, c1);
            rn.u(QVD, vd);
            rn.v(QBR, beta);
            if (hashing) rn.u(QHASH, hv);
            if (!fused) rec.u(RNEXT, (uint32_t)o);
        }
        if (active && hashing) r.u(QHASH, hv);
    }
}

// shadow ray w of the list of bounce k: occlusion code, or (fused) the
// unoccluded contribution added and the occlusion recorded
template <bool FAST, bool ONE>
__device__ __forceinline__ void shadow_one(const FwdParams& p, const Queues& q, int k, int w, bool fused,
                                           const TraceGeo& GW, TravStack& st) {
    // fused: the records lie in list order (see SCol)
    const uint32_t e = fused ? (uint32_t)w : qld(q.slist + w);
    const uint32_t i = fused ? e : e % (uint32_t)q.cap;
    const RecRow rec(q.rec, i);
    const ShRow sh(q.sh, e);
    const int f = (int)rec.u(RFACE);
    const TraceGeo G = ONE ? GW : lane_geo(p.scenes[p.cams[(fused ? rec.u(RVD) : RayRow(q.ray[k & 1], i).u(QVD)) & 0xFFFFu].scene]);
    const float tmax = sh.f(STMAX);
    const V3 o = rec.v(RX0), dd = sh.v(SWX);
    const bool occluded = trace_any<FAST>(G, o, dd, TMIN, tmax, f, st);
    if (fused) {
        if (occluded) {
            if (p.rec_occ) p.rec_occ[(size_t)(k - 1) * p.rec_n + rec.u(RSLOT)] = 1u;
        } else {
            float* L = q.L + 3 * (size_t)rec.u(RSLOT);
            const V3 c = sh.v(SCR);
            L[0] += c.x; L[1] += c.y; L[2] += c.z;
        }
    } else {
        q.socc[e] = occluded ? 1 : 2;
    }
}

// shadow rays of bounce k: the entries listed by k_shade (entry l of shading
// point i is l * cap + i), one outcome code each (1 occluded, 2 unoccluded);
// k_shade wrote 0 (no ray) for the others
template <bool FAST, bool ONE>
__global__ void __launch_bounds__(TRACE_BLOCK) SHADOW_OCC k_shadow(FwdParams p, Queues q, int k) {
    __shared__ uint32_t lds[LDS_STACK * TRACE_BLOCK];
    TravStack st = make_trav_stack(lds, q.spill, p.err, p.work ? p.work + 3 * WORK_SHADOW : nullptr);
    const TraceGeo G = wave_geo(p.scene);
    const int items = q.cnt[32 + k];
    const bool fused = shadow_fused(p, q);
    // 64 consecutive listed rays per wave, traced in lockstep
    wave_tiles(q.take + TAKE_NC * 32 * k, (uint32_t)items, [&](uint32_t t) {
        const int w = (int)(t + __lane_id());
        if (w < items) shadow_one<FAST, ONE>(p, q, k, w, fused, G, st);
    });
}

// One launch for the extension rays of bounce k + 1 and the shadow rays of
// bounce k: both start at the shading points of bounce k and neither reads
// what the other writes (hits of the next queue; radiance, occlusion records
// or outcome codes of this bounce), so the two traversals share one grid and
// one drain at the end instead of two.  Waves take the listed shadow rays first
// (their count rounded up to whole waves), then the extension rays (this order
// measured 0.7 ms faster per step than the other).
template <bool FAST, bool ONE>
__global__ void __launch_bounds__(TRACE_BLOCK) EXTEND_OCC k_trace_pair(FwdParams p, Queues q, int k) {
    __shared__ uint32_t lds[LDS_STACK * TRACE_BLOCK];
    TravStack st = make_trav_stack(lds, q.spill, p.err, nullptr);
    st.work2 = p.work ? p.work + 3 * WORK_PAIR : nullptr;
    unsigned long long* const wext = p.work ? p.work + 3 * WORK_EXTEND : nullptr;
    unsigned long long* const wsh = p.work ? p.work + 3 * WORK_SHADOW : nullptr;
    const TraceGeo G = wave_geo(p.scene);
    const int n = q.cnt[k + 1];
    const int items = q.cnt[32 + k];
    const bool fused = shadow_fused(p, q);
    // unsigned: with many lights the two counts together can pass 2^31 (each is
    // below 2^31, the grid below 2^21, so the sum and the next index fit 32 bits)
    const uint32_t s64 = ((uint32_t)items + 63u) & ~63u;
    const uint32_t all = s64 + (uint32_t)n;
    wave_tiles(q.take + TAKE_NC * 32 * k, all, [&](uint32_t t) {
        const uint32_t i = t + __lane_id();
        if (t < s64) {
            if (i < (uint32_t)items) {
                st.work = wsh;
                shadow_one<FAST, ONE>(p, q, k, (int)i, fused, G, st);
            }
        } else if (i < all) {
            st.work = wext;
            extend_one<FAST, ONE>(p, q, q.ray[(k + 1) & 1], i - s64, G, st);
        }
    });
}

// Shadow contributions of bounce k added per shading point in entry order.  Bound by the
// chain of reads of a point: its face, its entries' outcomes, the contributions of those
// that see their light.  Four entries' outcomes and then their contributions are asked
// for together, and a launch of one scene takes the entry count from its arguments
// (three lights, 8 views of 256^2 at 16 spp: two launches 154 -> 105 us; 24-view batch of
// mixed scenes 781 -> 688 us).
template <bool ONE> __global__ void k_shadow_sum(FwdParams p, Queues q, int k) {
    constexpr int GROUP = 4;
    const int n = q.cnt[k];
    const int stride = gridDim.x * blockDim.x;
    const bool hashing = p.dbg_hash || p.hash_by_q;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const RayRow r(q.ray[k & 1], (uint32_t)i);
        const RecRow rec(q.rec, (uint32_t)i);
        const int f = (int)rec.u(RFACE);
        if (f < 0) continue;
        const uint32_t pq = r.u(QQ), info = hashing ? rec.u(RINFO) : 0u;
        const DevScene& S = ONE ? p.scene : p.scenes[p.cams[r.u(QVD) & 0xFFFFu].scene];
        Hash h{hashing ? r.u(QHASH) : 0u, hashing};
        V3 acc{0.f, 0.f, 0.f};
        const int nent = S.nl + (S.has_env ? 1 : 0);
        uint32_t occ = 0;
        for (int l0 = 0; l0 < nent; l0 += GROUP) {
            uint32_t code[GROUP];
            V3 c[GROUP];
#pragma unroll
            for (int g = 0; g < GROUP; ++g) code[g] = l0 + g < nent ? q.socc[(size_t)(l0 + g) * q.cap + i] : 0u;
#pragma unroll
            for (int g = 0; g < GROUP; ++g) {
                c[g] = V3{0.f, 0.f, 0.f};
                if (code[g] == 2u) c[g] = ShRow(q.sh, (size_t)(l0 + g) * q.cap + i).v(SCR);
            }
#pragma unroll
            for (int g = 0; g < GROUP; ++g) {
                const int l = l0 + g;
                if (l >= nent) break;
                if (l == S.nl) h.push(hashing ? rec.u(RTEX) : 0u);
                if (code[g] == 2u) acc = acc + c[g];
                if (code[g] == 1u) occ |= 1u << l;
                h.push(code[g]);
            }
        }
        if (p.rec_occ) p.rec_occ[(size_t)(k - 1) * p.rec_n + pq] = occ;
        if (info & 1u) {
            h.push((info >> 1) & 1u);
            h.push((info >> 2) & 1u);
        }
        float* L = q.L + 3 * (size_t)pq;
        L[0] += acc.x; L[1] += acc.y; L[2] += acc.z;
        if (hashing) {
            const int o = (int)rec.u(RNEXT);
            if (o >= 0) RayRow(q.ray[(k + 1) & 1], (uint32_t)o).u(QHASH, h.h);
            else final_hash(p, r, h.h);
        }
    }
}

// single-kernel forward (one thread per path sample); same estimator
__global__ void __launch_bounds__(TRACE_BLOCK) k_forward_mega(FwdParams p, float* L, long long total,
                                                              uint32_t* spill) {
    __shared__ uint32_t lds[LDS_STACK * TRACE_BLOCK];
    TravStack st = make_trav_stack(lds, spill, p.err, p.work ? p.work + 3 * WORK_MEGA : nullptr);
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long qq = blockIdx.x * (long long)blockDim.x + threadIdx.x; qq < total; qq += stride) {
        const int v = find_view(p.qoff, p.ncam, qq);
        const DevCam& c = p.cams[v];
        const DevScene& S = p.scenes[c.scene];
        int x, y, j;
        decode_path(c, qq - c.qoff, p.spp, x, y, j);
        const Ctr ctr{(uint32_t)(y * c.W + x), ((uint32_t)c.rngview << 16) | (uint32_t)j, 0u, 0u};
        const Key key{p.seed, S.scene_id};
        const float4 u = draw4(ctr, 0, 0, key);
        const V3 d = cam_dir(c, (float)x + u.x, (float)y + u.y);
        Hash h{FNV_INIT, true};
        const V3 r = trace_estimator(S, lane_geo(S), ld3(c.eye), d, -1, p.B, false, ctr, key, h, st);
        L[3 * qq] = r.x; L[3 * qq + 1] = r.y; L[3 * qq + 2] = r.z;
        if (p.dbg_hash) p.dbg_hash[canon(c, x, y, j, p.spp)] = h.h;
    }
}

// Film: the average of each pixel's spp samples, added in sample order.  Bound by the
// read of 12 bytes per sample.  Threads take the pixels in the order of the samples
// (8x8 tiles), so a wave reads 768 consecutive bytes of each sample plane, one 12-byte
// load a lane, four planes in flight; in scan order each line of a plane went to eight
// waves and was fetched twice (67M samples: 1.66 GB for 0.81, 297 us; now 135 us; a 1024^2
// view at 32 spp 135 -> 64 us).
typedef float film3 __attribute__((ext_vector_type(3), aligned(4)));
__global__ void k_film(const DevCam* __restrict__ cams, const long long* __restrict__ pixoff, int ncam, int spp,
                       const float* __restrict__ L, long long npix, float* out, uint32_t* err,
                       unsigned long long* key_dev, unsigned long long key) {
    if (key_dev && blockIdx.x == 0 && threadIdx.x == 0) *key_dev = key;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long g = blockIdx.x * (long long)blockDim.x + threadIdx.x; g < npix; g += stride) {
        const int v = find_view(pixoff, ncam, g);
        const DevCam& c = cams[v];
        int x, y, j0;
        decode_path(c, g - c.pixoff, spp, x, y, j0);
        const long long hw = (long long)c.W * c.H;
        const float* plane = L + 3 * (c.qoff + (g - c.pixoff));
        float a = 0.f, b = 0.f, cc = 0.f;
#pragma unroll 4
        for (int j = 0; j < spp; ++j, plane += 3 * hw) {
            const film3 s = __builtin_nontemporal_load((const film3*)plane);
            a += s.x; b += s.y; cc += s.z;
        }
        const float inv = 1.0f / (float)spp;
        float* const o = out + 3 * (c.pixoff + (long long)y * c.W + x);
        o[0] = a * inv; o[1] = b * inv; o[2] = cc * inv;
        if (!isfinite(a + b + cc)) atomicOr(err, ERR_NAN);
    }
}

// per-sample radiance in canonical order (debug output)
__global__ void k_sample_radiance(FwdParams p, const float* __restrict__ L, long long total, float* out) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long qq = blockIdx.x * (long long)blockDim.x + threadIdx.x; qq < total; qq += stride) {
        const int v = find_view(p.qoff, p.ncam, qq);
        const DevCam& c = p.cams[v];
        int x, y, j;
        decode_path(c, qq - c.qoff, p.spp, x, y, j);
        const long long g = canon(c, x, y, j, p.spp);
        out[3 * g] = L[3 * qq]; out[3 * g + 1] = L[3 * qq + 1]; out[3 * g + 2] = L[3 * qq + 2];
    }
}

__global__ void k_fill_f32(float* p, long long n, float v) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}
__global__ void k_fill_u32(uint32_t* p, long long n, uint32_t v) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// closest hit of caller-given rays (BVH, or brute force over all faces)
template <bool FAST>
__global__ void __launch_bounds__(TRACE_BLOCK) k_trace_debug(const DevScene* sc, const float* o, const float* d,
                                                             int n, float tmin, int brute, int* of, float* ot,
                                                             uint32_t* spill, uint32_t* err) {
    __shared__ uint32_t lds[LDS_STACK * TRACE_BLOCK];
    const DevScene& S = *sc;
    TravStack st = make_trav_stack(lds, spill, err, nullptr);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const TraceGeo G = wave_geo(S);
    const V3 oo = ld3(o + 3 * i), dd = ld3(d + 3 * i);
    float tb = __int_as_float(0x7f800000);
    int fb = -1;
    if (brute) {
        for (int l = 0; l < S.nf; ++l) {
            float t; int f;
            if (tri_test<true>(tri_at(G.tri, (uint32_t)l), oo, dd, tmin, __int_as_float(0x7f800000), t, f))
                if (t < tb || (t == tb && f < fb)) { tb = t; fb = f; }
        }
    } else {
        fb = trace_closest<FAST>(G, oo, dd, tmin, -1, tb, st);
    }
    of[i] = fb;
    ot[i] = tb;
}

// ---------------------------------------------------------------------------
static inline unsigned grid_for(long long n, int bs, unsigned cap) {
    long long g = (n + bs - 1) / bs;
    if (g < 1) g = 1;
    return (unsigned)(g < (long long)cap ? g : cap);
}


void launch_forward_wavefront(const FwdParams& p, Queues& q, long long total, int has_env_any, int nent,
                              hipStream_t st) {
    q.nent = nent;
    for (long long q0 = 0; q0 < total; q0 += q.cap) {
        const int n = (int)((total - q0) < q.cap ? (total - q0) : q.cap);
        launch_wavefront_bounces(p, q, n, q0, has_env_any, st);
    }
}

// Extension / shading / shadow kernels of every bounce for a chunk of n camera rays,
// path samples q0 .. q0 + n - 1, or (q0 < 0) of the side rays that fill queue 1 and
// whose count in cnt[1] n bounds (the counters cleared before).
void launch_wavefront_bounces(const FwdParams& p, Queues& q, int n, long long q0, int has_env_any, hipStream_t st,
                              LaunchHook* hook) {
    const unsigned gmax = (q.grid > 0 && (unsigned)q.grid < TRACE_GRID) ? (unsigned)q.grid : TRACE_GRID;
    const unsigned g = grid_for(n, TRACE_BLOCK, gmax);
    const int last = p.B + (has_env_any ? 1 : 0);
    const bool fused = shadow_fused(p, q), side = q0 < 0;
    const bool one = p.fast && p.nscenes == 1, hashing = p.dbg_hash || p.hash_by_q;
    using Shade = void (*)(FwdParams, Queues, int, long long);
    // (side rays come with one scene)
    constexpr Shade shades[3][2][3] = {      // [mode][one scene][from]
        {{k_shade<MODE_FUSED, false, FROM_LATER>, k_shade<MODE_FUSED, false, FROM_CAMERA>, nullptr},
         {k_shade<MODE_FUSED, true, FROM_LATER>, k_shade<MODE_FUSED, true, FROM_CAMERA>, k_shade<MODE_FUSED, true, FROM_SIDE>}},
        {{k_shade<MODE_LISTED, false, FROM_LATER>, k_shade<MODE_LISTED, false, FROM_CAMERA>, nullptr},
         {k_shade<MODE_LISTED, true, FROM_LATER>, k_shade<MODE_LISTED, true, FROM_CAMERA>, k_shade<MODE_LISTED, true, FROM_SIDE>}},
        {{k_shade<MODE_HASH, false, FROM_LATER>, k_shade<MODE_HASH, false, FROM_CAMERA>, nullptr},
         {k_shade<MODE_HASH, true, FROM_LATER>, k_shade<MODE_HASH, true, FROM_CAMERA>, k_shade<MODE_HASH, true, FROM_SIDE>}}};
    const int mode = hashing ? MODE_HASH : fused ? MODE_FUSED : MODE_LISTED;
    const auto extend = side ? (p.fast ? k_extend<true, true, true> : k_extend<false, true, true>)
                        : one ? k_extend<true, true, false>
                        : p.fast ? k_extend<true, false, false> : k_extend<false, false, false>;
    const auto shadow_rays = one ? k_shadow<true, true> : p.fast ? k_shadow<true, false> : k_shadow<false, false>;
    const auto pair = one ? k_trace_pair<true, true> : p.fast ? k_trace_pair<true, false> : k_trace_pair<false, false>;
    // (only a launch with more tiles than waves takes from its counters)
    if (!side && (unsigned)((n + 63) / 64) > g * (TRACE_BLOCK / 64))
        ST_LAUNCH("k_pass_begin", k_pass_begin, dim3(TAKE_INTS / 256), dim3(256), 0, st, q, n);
    ST_LAUNCH("k_extend", extend, dim3(g), dim3(TRACE_BLOCK), 0, st, p, q, q0, n);
    if (hook) hook->tick();
    for (int k = 1; k <= last; ++k) {
        // bounce k is traced: shade it, then trace its shadow rays together with
        // the extension rays of bounce k + 1
        ST_LAUNCH("k_shade", shades[mode][p.nscenes == 1][k > 1 ? FROM_LATER : side ? FROM_SIDE : FROM_CAMERA],
                  dim3(grid_for(n, SHADE_BLOCK, gmax)), dim3(SHADE_BLOCK), 0, st, p, q, k, q0);
        if (hook) hook->tick();
        if (k <= p.B && k < last) {
            ST_LAUNCH("k_trace_pair", pair, dim3(g), dim3(TRACE_BLOCK), 0, st, p, q, k);
            if (hook) hook->tick();
        } else if (k <= p.B) {
            ST_LAUNCH("k_shadow", shadow_rays, dim3(g), dim3(TRACE_BLOCK), 0, st, p, q, k);
            if (hook) hook->tick();
        }
        if (k <= p.B && !fused)
            ST_LAUNCH("k_shadow_sum", p.nscenes == 1 ? k_shadow_sum<true> : k_shadow_sum<false>, dim3(grid_for(n, 256, gmax)), dim3(256), 0, st, p, q, k);
    }
}

void launch_forward_mega(const FwdParams& p, float* L, long long total, uint32_t* spill, int grid,
                         hipStream_t st) {
    ST_LAUNCH("k_forward_mega", k_forward_mega, dim3(grid_for(total, TRACE_BLOCK, grid)), dim3(TRACE_BLOCK), 0, st, p, L,
                       total, spill);
}

void launch_film(const DevCam* cams, const long long* pixoff, int ncam, int spp, const float* L, long long npix,
                 float* out, uint32_t* err, hipStream_t st, unsigned long long* key_dev, unsigned long long key) {
    ST_LAUNCH("k_film", k_film, dim3(grid_for(npix, 256, 1u << 16)), dim3(256), 0, st, cams, pixoff, ncam, spp, L,
                       npix, out, err, key_dev, key);
}

void launch_sample_radiance(const FwdParams& p, const float* L, long long total, float* out, hipStream_t st) {
    ST_LAUNCH("k_sample_radiance", k_sample_radiance, dim3(grid_for(total, 256, 1u << 16)), dim3(256), 0, st, p, L, total,
                       out);
}

void launch_fill_f32(float* ptr, long long n, float v, hipStream_t st) {
    if (n > 0) ST_LAUNCH("k_fill_f32", k_fill_f32, dim3(grid_for(n, 256, 1u << 16)), dim3(256), 0, st, ptr, n, v);
}
// non-finite values among a[0..na) and b[0..nb) set ERR_NAN
__global__ void k_check_finite(const float* __restrict__ a, long long na, const float* __restrict__ b, long long nb,
                               uint32_t* err) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    bool bad = false;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < na + nb; i += stride)
        bad |= !isfinite(i < na ? a[i] : b[i - na]);
    if (__ballot(bad) && __lane_id() == 0) atomicOr(err, ERR_NAN);
}

void launch_check_finite(const float* a, long long na, const float* b, long long nb, uint32_t* err, hipStream_t st) {
    if (na + nb > 0)
        ST_LAUNCH("k_check_finite", k_check_finite, dim3(grid_for(na + nb, 256, 1u << 12)), dim3(256), 0, st, a, na, b,
                  nb, err);
}

// streaming copy of n 16-byte words (the achievable-bandwidth reference of the
// measurements): each thread moves 4 words per step with non-temporal loads and
// stores, consecutive lanes on consecutive words
__global__ void __launch_bounds__(256) k_stream_copy(vf4* __restrict__ dst, const vf4* __restrict__ src, long long n) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        const vf4 a = __builtin_nontemporal_load(src + i), b = __builtin_nontemporal_load(src + i + stride);
        const vf4 c = __builtin_nontemporal_load(src + i + 2 * stride), d = __builtin_nontemporal_load(src + i + 3 * stride);
        __builtin_nontemporal_store(a, dst + i);
        __builtin_nontemporal_store(b, dst + i + stride);
        __builtin_nontemporal_store(c, dst + i + 2 * stride);
        __builtin_nontemporal_store(d, dst + i + 3 * stride);
    }
    for (; i < n; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

void launch_stream_copy(float4* dst, const float4* src, long long n, hipStream_t st) {
    if (n > 0)
        ST_LAUNCH("k_stream_copy", k_stream_copy, dim3(grid_for(n, 256, 8192)), dim3(256), 0, st, (vf4*)dst,
                  (const vf4*)src, n);
}

// up to WORD_CHUNK words passed by value (so a captured launch carries its own
// copy) written to dst
constexpr int WORD_CHUNK = 480;
struct WordChunk {
    uint32_t n;
    uint32_t w[WORD_CHUNK];
};
__global__ void k_put_words(uint32_t* dst, WordChunk c) {
    for (uint32_t i = threadIdx.x; i < c.n; i += blockDim.x) dst[i] = c.w[i];
}

void launch_put_words(uint32_t* dst, const uint32_t* src, size_t nwords, hipStream_t st) {
    for (size_t i = 0; i < nwords; i += WORD_CHUNK) {
        WordChunk c;
        c.n = (uint32_t)(nwords - i < (size_t)WORD_CHUNK ? nwords - i : (size_t)WORD_CHUNK);
        for (uint32_t j = 0; j < c.n; ++j) c.w[j] = src[i + j];
        ST_LAUNCH("k_put_words", k_put_words, dim3(1), dim3(256), 0, st, dst + i, c);
    }
}

__global__ void k_put_u64(unsigned long long* p, unsigned long long v) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *p = v;
}

void launch_put_u64(unsigned long long* ptr, unsigned long long v, hipStream_t st) {
    ST_LAUNCH("k_put_u64", k_put_u64, dim3(1), dim3(64), 0, st, ptr, v);
}

void launch_fill_u32(uint32_t* ptr, long long n, uint32_t v, hipStream_t st) {
    if (n > 0) ST_LAUNCH("k_fill_u32", k_fill_u32, dim3(grid_for(n, 256, 1u << 16)), dim3(256), 0, st, ptr, n, v);
}

void launch_trace_debug(const DevScene* s, int nf, const float* o, const float* d, int n, float tmin, int brute,
                        int* out_face, float* out_t, uint32_t* spill, uint32_t* err, hipStream_t st) {
    const auto kern = tmin == TMIN && nf <= TRAV_FAST_FACES ? k_trace_debug<true> : k_trace_debug<false>;
    if (n > 0)
        ST_LAUNCH("k_trace_debug", kern, dim3((n + TRACE_BLOCK - 1) / TRACE_BLOCK), dim3(TRACE_BLOCK), 0, st, s, o,
                           d, n, tmin, brute, out_face, out_t, spill, err);
}

} // namespace st
