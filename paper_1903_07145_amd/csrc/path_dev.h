// Device code that every path kernel shares: the block's LDS tables, the BVH
// traversal with its short stack, and the shading of a path vertex.
#pragma once
#include <hip/hip_runtime.h>

#include "disney.h"
#include "ipt_internal.h"

namespace ipt {

struct Lds {
    __bf16* gact;       // this wave's guide activation rows (guided kernels)
    float* params;
    float* sparams;
    int* seg_emitter;
    float* cdf;
    int4* lights;
    double* grad;       // replay: block gradient, float64 (the terms of some entries cancel)
    int* stack;
    bool lights_in_lds;
};

// per-wave guide activation rows (64 x kGRowStride bf16), 4 waves per block
constexpr size_t kGuideLds = 4 * 64 * kGRowStride * sizeof(__bf16);

// PG (a compile-time copy of PathArgs::params_global) keeps each pointer's
// address space known, so LDS reads stay ds_read and the LDS gradient
// ds_add_f64 rather than flat accesses.
template <int PG>
__device__ void carve_lds(const PathArgs& a, int mode, unsigned char* smem, Lds& lds) {
    const int tid = threadIdx.x;
    unsigned char* p = smem;
    auto al = [](size_t x) { return (x + 15) & ~size_t(15); };
    constexpr int pg = PG;
    if constexpr (PG) {
        // parameters, segment table and the replay's gradient accumulator in global memory
        lds.params = (float*)a.params;
        lds.sparams = (float*)a.sparams;
        lds.seg_emitter = (int*)a.sc.seg_emitter;
    } else {
        lds.params = (float*)p; p += al(sizeof(float) * a.P);
        lds.sparams = lds.params;
        if (a.frozen) { lds.sparams = (float*)p; p += al(sizeof(float) * a.P); }
        lds.seg_emitter = (int*)p; p += al(sizeof(int) * a.sc.S);
    }
    lds.lights_in_lds = a.sc.nlt <= kMaxLdsLights;
    lds.cdf = nullptr;
    lds.lights = nullptr;
    if (lds.lights_in_lds) {
        lds.cdf = (float*)p; p += al(2 * sizeof(float) * a.sc.nlt);
        lds.lights = (int4*)p; p += al(sizeof(int4) * a.sc.nlt);
    }
    lds.grad = nullptr;
    if (mode == kReplay) {
        if constexpr (PG) lds.grad = a.grad_part + (size_t)(blockIdx.x % a.grad_copies) * a.P;
        else { lds.grad = (double*)p; p += al(sizeof(double) * a.P); }
    }
    lds.stack = (int*)p;
    p += sizeof(int) * kShortStack * kBlock;
    lds.gact = (__bf16*)p + (threadIdx.x >> 6) * 64 * kGRowStride;
    if constexpr (!pg) {
        for (int i = tid; i < a.P; i += kBlock) {
            lds.params[i] = a.params[i];
            if (a.frozen) lds.sparams[i] = a.sparams[i];
            if (mode == kReplay) lds.grad[i] = 0.0;
        }
        for (int i = tid; i < a.sc.S; i += kBlock) lds.seg_emitter[i] = a.sc.seg_emitter[i];
    }
    if (lds.lights_in_lds)
        for (int i = tid; i < a.sc.nlt; i += kBlock) {
            lds.cdf[i] = a.cdf[i];
            lds.cdf[a.sc.nlt + i] = a.cdf[a.sc.nlt + i];
            lds.lights[i] = a.sc.lights[i];
        }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Traversal with a per-lane short stack in LDS ([slot][lane] layout, so the
// 64 lanes of a wave hit 64 distinct banks) that spills its oldest entries to
// a per-lane global stack ([depth][thread], coalesced).
// ---------------------------------------------------------------------------
struct Stack {
    int* lds;     // kShortStack * kBlock
    int* ovf;
    int tid, gtid, gthreads;
    int sp;
    bool overflow;
    __device__ __forceinline__ void push(int x) {
        int slot = sp & (kShortStack - 1);
        if (sp >= kShortStack) {
            int d = sp - kShortStack;
            if (d >= kOvfDepth) { overflow = true; return; }
            ovf[(size_t)d * gthreads + gtid] = lds[slot * kBlock + tid];
        }
        lds[slot * kBlock + tid] = x;
        ++sp;
    }
    // Pushes the n (0..3) entries x0..x(n-1), x0 deepest.  With room for
    // three in the LDS window (and so no entry to move to the overflow
    // stack) all three slots are written, whatever n: the slots above the
    // new top hold no live entry.
    __device__ __forceinline__ void push_upto3(int n, int x0, int x1, int x2) {
        if (sp + 3 <= kShortStack) {
            int* s = lds + sp * kBlock + tid;
            s[0] = x0;
            s[kBlock] = x1;
            s[2 * kBlock] = x2;
            sp += n;
        } else {
            if (n > 0) push(x0);
            if (n > 1) push(x1);
            if (n > 2) push(x2);
        }
    }
    __device__ __forceinline__ int pop() {
        --sp;
        int slot = sp & (kShortStack - 1);
        int x = lds[slot * kBlock + tid];
        if (sp >= kShortStack) lds[slot * kBlock + tid] = ovf[(size_t)(sp - kShortStack) * gthreads + gtid];
        return x;
    }
};

__device__ __forceinline__ void init_stack(Stack& st, const PathArgs& a, int* lds_stack) {
    st.lds = lds_stack;
    st.ovf = a.ovf;
    st.tid = threadIdx.x;
    st.gtid = blockIdx.x * kBlock + threadIdx.x;
    st.gthreads = gridDim.x * kBlock;
    st.overflow = false;
    st.sp = 0;
}

struct Hit {
    int tri;     // leaf-ordered index, -1 on miss
    float t, u, v;
};

struct Work {
    uint32_t rays, nodes, tris, vertices, units;
};

__device__ __forceinline__ void load_tri(const SceneDev& sc, int i, V3& p0, V3& p1, V3& p2, int& orig,
                                         int& seg, int& light) {
    float4 a = sc.tris[3 * i], b = sc.tris[3 * i + 1], c = sc.tris[3 * i + 2];
    p0 = xyz(a); p1 = xyz(b); p2 = xyz(c);
    orig = __float_as_int(a.w);
    seg = __float_as_int(b.w);
    light = __float_as_int(c.w);
}

constexpr int kTravDone = (int)0x80000000;   // no node left (leaf codes are > INT_MIN)

// Bytes 0 and 2 (or 1 and 3) of a quantized plane row, zero-extended into the
// two 16-bit halves of a register: each half, read as fp16, is the subnormal
// q 2^-24 (kernels keep fp16 denormals, the default fp16/fp64 denormal mode;
// the BVH tests compare the hits with brute force bit for bit).
typedef _Float16 h2x __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h2x bytes02(uint32_t w) { return __builtin_bit_cast(h2x, w & 0x00ff00ffu); }
__device__ __forceinline__ h2x bytes13(uint32_t w) {
    return __builtin_bit_cast(h2x, __builtin_amdgcn_perm(w, w, 0x0c030c01u));
}

// Traversal state of one lane, kept across calls when a call returns early.
struct Trav {
    int cur;        // next node: inner (>= 0), leaf code (< 0) or kTravDone
    int pend;       // leaf held for the leaf phase
    int best_orig;  // original id of the best hit (tie rule)
    Hit best;
};

__device__ __forceinline__ void trav_init(Trav& tv, float tmax, Stack& st, Work& wk) {
    tv.cur = 0;
    tv.pend = kTravDone;
    tv.best_orig = 0x7FFFFFFF;
    tv.best = Hit{-1, tmax, 0.0f, 0.0f};
    st.sp = 0;
    wk.rays++;
}

// The node phase ends early once no more than this many lanes of the wave
// are still looking for their first leaf (0: it runs until none is).
// Apartment step with binary nodes: 166.7 ms at 0; 159.0 / 157.8 / 157.3 /
// 157.1 / 158.0 / 169.9 / 204.3 ms at 2 / 3 / 4 / 6 / 8 / 16 / 32.  With
// quantized four-child nodes and two-triangle leaves, whose leaf phase is
// cheaper (testing the held leaves sooner also shortens the rays' best
// distance): 125.9 / 123.2 / 122.4 ms at 2 / 4 / 8 in one run, and
// 123.8 / 123.0 / 124.8 / 129.7 / 141.1 ms at 4 / 8 / 12 / 16 / 24 in another.
#ifndef IPT_NODE_BREAK
#define IPT_NODE_BREAK 8
#endif


// Advances the lanes' traversals; returns true for a lane whose traversal
// has finished (its hit is then in tv.best).  With exit_lanes > 0 the call
// also returns, after at least one node phase and one leaf phase (so every
// call advances every unfinished lane), as soon as no more than exit_lanes
// lanes of the wave are still traversing: those keep their state and resume
// on the next call, while the others shade and start new rays, instead of
// idling through the slowest rays' tail.
__device__ bool traverse_resume(const SceneDev& sc, const Ray& r, float tmin, float tmax, int skip0, int skip1,
                                bool any, Stack& st, Work& wk, Trav& tv, int exit_lanes) {
    int cur = tv.cur, pend = tv.pend, best_orig = tv.best_orig;
    Hit best = tv.best;
    // direction signs: which byte row of a quantized node is an axis's near plane
    const bool negx = r.inv.x < 0.0f, negy = r.inv.y < 0.0f, negz = r.inv.z < 0.0f;
    auto next_from_stack = [&]() -> int { return (st.sp > 0 && !st.overflow) ? st.pop() : kTravDone; };
    while (true) {
        // ---- node phase ----
        while (true) {
            if (cur < 0 && cur != kTravDone && pend == kTravDone) {
                pend = cur;
                cur = next_from_stack();
            }
            const bool inner = cur >= 0;
            const uint64_t searching = __ballot(inner && pend == kTravDone);
            if (!searching) break;
            // few lanes still looking for their first leaf: test the leaves
            // the others hold now, and let those lanes descend again with
            // the rest after the leaf phase (at least one leaf is pending,
            // so every pass of the outer loop makes progress)
            if (IPT_NODE_BREAK > 0 && __popcll(searching) <= IPT_NODE_BREAK && __any(pend != kTravDone)) break;
            if (inner) {
                // four children: the nearest hit next, the others pushed far to near
                wk.nodes++;
                const float inf = __builtin_inff();
                float t[4];
                int c[4];
                // quantized child boxes: a plane is origin + q 2^e, so its
                // slab distance is fma(q, 2^e / d, (origin - o) / d); the
                // direction's sign picks each axis's near and far byte rows.
                // The exit distance gets a relative slack, so a triangle lying
                // on a box face is never culled.  The best hit so far gets an
                // absolute one (sc.tmin): the triangle test's t carries an error
                // of the order of the rounding of the scene coordinates, not of
                // t, so without it a flat box could be culled against a hit
                // whose t came out a few ulps of the coordinates short, and a
                // tie between coplanar triangles would be decided by the tree
                // instead of by the tie rule.
                // The byte enters the fma as an fp16 operand of the
                // mixed-precision fma (one instruction per plane instead of
                // a conversion and an fma; the same value bit for bit)
                const float4* n = sc.nodes + 4 * (size_t)cur;
                const float4 h = n[0], qa = n[1], qb = n[2], cr = n[3];
                c[0] = __float_as_int(cr.x); c[1] = __float_as_int(cr.y);
                c[2] = __float_as_int(cr.z); c[3] = __float_as_int(cr.w);
                // the references are needed only after the sort; tie them
                // to this point so their load issues with the box rows
                __asm__ volatile("" :: "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]));
                const uint32_t ew = __float_as_uint(h.w);
                // A carries an extra 2^24: a byte q, widened to 16 bits, is
                // read as the fp16 subnormal q 2^-24, so the mixed-precision
                // fma forms q 2^e / d + B exactly, with no conversion
                const V3 A = v3(ldexpf(r.inv.x, (int)(ew & 0xffu) - 103),
                                ldexpf(r.inv.y, (int)((ew >> 8) & 0xffu) - 103),
                                ldexpf(r.inv.z, (int)((ew >> 16) & 0xffu) - 103));
                const V3 B = v3((h.x - r.o.x) * r.inv.x, (h.y - r.o.y) * r.inv.y, (h.z - r.o.z) * r.inv.z);
                const uint32_t xl = __float_as_uint(qa.x), xh = __float_as_uint(qa.y);
                const uint32_t yl = __float_as_uint(qa.z), yh = __float_as_uint(qa.w);
                const uint32_t zl = __float_as_uint(qb.x), zh = __float_as_uint(qb.y);
                const uint32_t xn = negx ? xh : xl, xf = negx ? xl : xh;
                const uint32_t yn = negy ? yh : yl, yf = negy ? yl : yh;
                const uint32_t zn = negz ? zh : zl, zf = negz ? zl : zh;
                const float tmx = best.t + sc.tmin;
                // 16-bit lanes of children 0 and 2, and of children 1 and 3
                const h2x e02[6] = {bytes02(xn), bytes02(xf), bytes02(yn), bytes02(yf), bytes02(zn), bytes02(zf)};
                const h2x e13[6] = {bytes13(xn), bytes13(xf), bytes13(yn), bytes13(yf), bytes13(zn), bytes13(zf)};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const h2x* e = (i & 1) ? e13 : e02;
                    const int hi = i >> 1;
                    const float nx = fmaf((float)(hi ? e[0].y : e[0].x), A.x, B.x);
                    const float fx = fmaf((float)(hi ? e[1].y : e[1].x), A.x, B.x);
                    const float ny = fmaf((float)(hi ? e[2].y : e[2].x), A.y, B.y);
                    const float fy = fmaf((float)(hi ? e[3].y : e[3].x), A.y, B.y);
                    const float nz = fmaf((float)(hi ? e[4].y : e[4].x), A.z, B.z);
                    const float fz = fmaf((float)(hi ? e[5].y : e[5].x), A.z, B.z);
                    const float tn = fmaxf(fmaxf(nx, ny), fmaxf(nz, tmin));
                    const float tf = fminf(fminf(fx, fy), fminf(fz, tmx));
                    t[i] = tn <= tf * 1.0000005f ? tn : inf;
                }
                // sorting network on (t, child) with selects, no branches;
                // equal distances keep their slot order
                auto cas = [&](int i, int j) {
                    const bool sw = t[j] < t[i];
                    const float ti = t[i], tj = t[j];
                    const int ci = c[i], cj = c[j];
                    t[i] = sw ? tj : ti;
                    t[j] = sw ? ti : tj;
                    c[i] = sw ? cj : ci;
                    c[j] = sw ? ci : cj;
                };
                cas(0, 1); cas(2, 3); cas(0, 2); cas(1, 3); cas(1, 2);
                if (t[0] < inf) {
                    // the entered children are a prefix of the sorted slots:
                    // push the nf after the nearest, farthest first
                    const int nf = (t[1] < inf ? 1 : 0) + (t[2] < inf ? 1 : 0) + (t[3] < inf ? 1 : 0);
                    st.push_upto3(nf, nf == 3 ? c[3] : (nf == 2 ? c[2] : c[1]), nf == 3 ? c[2] : c[1], c[1]);
                    cur = c[0];
                } else {
                    cur = next_from_stack();
                }
            }
        }
        // ---- leaf phase ----
        if (pend != kTravDone) {
            int code = ~pend;
            int first = code >> 3, cnt = (code & 7) + 1;
            pend = kTravDone;
            wk.tris += cnt;
            for (int i = first; i < first + cnt; ++i) {
                if (i == skip0 || i == skip1) continue;
                V3 p0, p1, p2;
                int orig, seg, light;
                load_tri(sc, i, p0, p1, p2, orig, seg, light);
                float t, u, v;
                if (!tri_isect(r, p0, p1, p2, tmin, t, u, v)) continue;
                if (any) {
                    if (t < tmax) {
                        best.tri = i; best.t = t;
                        cur = kTravDone;
                        break;
                    }
                } else if (t < best.t || (t == best.t && orig < best_orig)) {
                    best.tri = i; best.t = t; best.u = u; best.v = v;
                    best_orig = orig;
                }
            }
        }
        const uint64_t live = __ballot(cur != kTravDone);
        if (!live) break;
        if (exit_lanes > 0 && __popcll(live) <= exit_lanes) break;
    }
    tv.cur = cur;
    tv.pend = pend;
    tv.best_orig = best_orig;
    const bool done = cur == kTravDone;
    if (done && !any && best.tri >= 0 && !(best.t < tmax)) best.tri = -1;
    tv.best = best;
    return done;
}

// Closest hit (any = false) or occlusion test (any = true: stops at the
// first hit in (tmin, tmax)), run to completion.  skip0/skip1 are leaf
// indices that are ignored.  Ties in t are resolved toward the smaller
// original id.
//
// Loop structure for 64-wide waves ("while-while" with speculative
// traversal, Aila and Laine 2009): the node phase visits inner nodes until
// every lane holds a leaf (a lane that already holds one keeps descending, and
// stops only at a second leaf), then the leaf phase tests the held leaves of
// all lanes together.  Node code and triangle code thus run with most lanes
// doing the same thing, instead of every iteration paying for both.
__device__ Hit traverse(const SceneDev& sc, const Ray& r, float tmin, float tmax, int skip0, int skip1, bool any,
                        Stack& st, Work& wk) {
    Trav tv;
    trav_init(tv, tmax, st, wk);
    traverse_resume(sc, r, tmin, tmax, skip0, skip1, any, st, wk, tv, 0);
    return tv.best;
}

// Brute-force closest hit (reference for the BVH).
__device__ Hit brute_closest(const SceneDev& sc, int64_t nt, const Ray& r, float tmin, int skip) {
    Hit best{-1, __builtin_inff(), 0.0f, 0.0f};
    int best_orig = 0x7FFFFFFF;
    for (int64_t i = 0; i < nt; ++i) {
        if ((int)i == skip) continue;
        V3 p0, p1, p2;
        int orig, seg, light;
        load_tri(sc, (int)i, p0, p1, p2, orig, seg, light);
        float t, u, v;
        if (!tri_isect(r, p0, p1, p2, tmin, t, u, v)) continue;
        if (t < best.t || (t == best.t && orig < best_orig)) {
            best.tri = (int)i; best.t = t; best.u = u; best.v = v;
            best_orig = orig;
        }
    }
    return best;
}

// ---------------------------------------------------------------------------
// Light selection from the cumulative table (first j with cdf[j] > u*total);
// cdf[n + j] holds light j's selection probability.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int pick_light(const float* cdf, int n, float u) {
    float x = u * cdf[n - 1];
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (cdf[mid] > x) hi = mid; else lo = mid + 1;
    }
    return lo;
}
__device__ __forceinline__ float light_prob(const float* cdf, int n, int j) {
    return cdf[n + j];
}

__device__ __forceinline__ void camera_ray(const PathArgs& a, int view, float px, float py, V3& o, V3& d) {
    const float* M = a.c2w + 16 * view;
    float th = tanf(0.5f * a.fov[view]);
    float asp = (float)a.W / (float)a.H;
    float cx = (2.0f * px / (float)a.W - 1.0f) * th * asp;
    float cy = (1.0f - 2.0f * py / (float)a.H) * th;
    V3 dw = v3(M[0] * cx + M[1] * cy - M[2], M[4] * cx + M[5] * cy - M[6], M[8] * cx + M[9] * cy - M[10]);
    o = v3(M[3], M[7], M[11]);
    d = normalize(dw);
}

__device__ __forceinline__ void lds_add(double* g, int i, float x) {
    if (x != 0.0f) atomicAdd(g + i, (double)x);
}
// n interleaved copies of the sums, [parameter][copy]; g points at the lane's copy.
struct GradCopies {
    double* g;
    int n;
};
__device__ __forceinline__ void lds_add(const GradCopies& c, int i, float x) {
    if (x != 0.0f) atomicAdd(c.g + i * c.n, (double)x);
}

// ---------------------------------------------------------------------------
// Shading shared by all passes.
// ---------------------------------------------------------------------------
struct Shade {
    V3 p0, e1, e2, x, ng, ngf, ns, wo;
    V3 tx, ty;   // tangent frame of the Disney model (set by mat_frame)
    int tri, orig, seg, light, em;
    float u, v, t, cos_emit;
};

// Geometry of a hit: position from barycentrics, geometric and shading
// normals, both flipped toward the incoming ray (two-sided reflection).
__device__ __forceinline__ void make_shade(const SceneDev& sc, const Lds& lds, const Hit& hit, V3 d, Shade& g) {
    V3 p1, p2;
    load_tri(sc, hit.tri, g.p0, p1, p2, g.orig, g.seg, g.light);
    g.tri = hit.tri;
    g.u = hit.u;
    g.v = hit.v;
    g.t = hit.t;
    g.e1 = p1 - g.p0;
    g.e2 = p2 - g.p0;
    g.x = g.p0 + g.e1 * hit.u + g.e2 * hit.v;
    g.ng = normalize(cross(g.e1, g.e2));
    g.em = lds.seg_emitter[g.seg];
    g.cos_emit = -dot(d, g.ng);
    g.wo = v3(-d.x, -d.y, -d.z);
    g.ns = g.ng;
    if (sc.nrm) {
        float b0 = 1.0f - hit.u - hit.v;
        V3 n0 = xyz(sc.nrm[3 * hit.tri]), n1 = xyz(sc.nrm[3 * hit.tri + 1]), n2 = xyz(sc.nrm[3 * hit.tri + 2]);
        g.ns = normalize(n0 * b0 + n1 * hit.u + n2 * hit.v);
    }
    g.ngf = g.ng;
    if (dot(g.ng, g.wo) < 0.0f) { g.ngf = g.ng * -1.0f; g.ns = g.ns * -1.0f; }
}

// ---------------------------------------------------------------------------
// Material models (compile-time): 0 Lambert + GGX, 7 parameters per segment;
// 1 Disney (Sec. 4.1), 13.  The kernels see a material through these
// overloads only.
// ---------------------------------------------------------------------------
template <int MAT> struct MatSel { using M = Mat; static constexpr int NP = 7; };
template <> struct MatSel<1> { using M = DMat; static constexpr int NP = kDisneyParams; };

template <int MAT>
__device__ __forceinline__ typename MatSel<MAT>::M mat_load(const float* p, int seg) {
    if constexpr (MAT == 1) return load_dmat(p, seg);
    else return load_mat(p, seg);
}
// The Disney model's anisotropy needs a tangent frame at the vertex.
template <int MAT>
__device__ __forceinline__ void mat_frame(Shade& g) {
    if constexpr (MAT == 1) disney_frame(g.ns, g.e1, g.tx, g.ty);
}
// f(wo, wi); for Lambert + GGX also the GGX factor and its alpha derivative,
// which the adjoint uses directly (the Disney adjoint differentiates f).
__device__ __forceinline__ V3 mat_f(const Mat& m, const Shade& g, V3 wi, float& spec, float& dspec) {
    spec_term(g.ns, g.wo, wi, m.alpha, spec, dspec);
    return m.kd * kInvPi + m.ks * spec;
}
__device__ __forceinline__ V3 mat_f(const DMat& m, const Shade& g, V3 wi, float& spec, float& dspec) {
    spec = dspec = 0.0f;
    return disney_value(m, disney_geom(g.ns, g.tx, g.ty, g.wo, wi));
}
__device__ __forceinline__ V3 mat_f_only(const Mat& m, const Shade& g, V3 wi) {
    return m.kd * kInvPi + m.ks * spec_only(g.ns, g.wo, wi, m.alpha);
}
__device__ __forceinline__ V3 mat_f_only(const DMat& m, const Shade& g, V3 wi) {
    return disney_value(m, disney_geom(g.ns, g.tx, g.ty, g.wo, wi));
}
__device__ __forceinline__ float mat_pdf(const Mat& m, const Shade& g, V3 wi) { return brdf_pdf(m, g.ns, g.wo, wi); }
__device__ __forceinline__ float mat_pdf(const DMat& m, const Shade& g, V3 wi) {
    return disney_pdf(m, g.ns, g.tx, g.ty, g.wo, wi);
}
__device__ __forceinline__ bool mat_sample(const Mat& m, const Shade& g, float u3, float u4, float u5, V3& wi,
                                           int& lobe) {
    return brdf_sample(m, g.ns, g.wo, u3, u4, u5, wi, lobe);
}
__device__ __forceinline__ bool mat_sample(const DMat& m, const Shade& g, float u3, float u4, float u5, V3& wi,
                                           int& lobe) {
    return disney_sample(m, g.ns, g.tx, g.ty, g.wo, u3, u4, u5, wi, lobe);
}
template <class M> struct MatNP { static constexpr int value = 7; };
template <> struct MatNP<DMat> { static constexpr int value = kDisneyParams; };

// Adjoint of f at one vertex: w . d f / d theta_seg added to the block's
// gradient, for a channel weight w (the Lambert + GGX terms use the factors
// spec, dspec kept from the evaluation; the Disney model its hand-written
// reverse sweep).
template <class G>
__device__ __forceinline__ void mat_grad(G grad, int mb, const Mat& m, const Shade&, V3, V3 w, float spec,
                                         float dspec) {
    lds_add(grad, mb + 0, w.x * kInvPi);
    lds_add(grad, mb + 1, w.y * kInvPi);
    lds_add(grad, mb + 2, w.z * kInvPi);
    lds_add(grad, mb + 3, w.x * spec);
    lds_add(grad, mb + 4, w.y * spec);
    lds_add(grad, mb + 5, w.z * spec);
    lds_add(grad, mb + 6, dot(w, m.ks) * dspec);
}
template <class G>
__device__ __forceinline__ void mat_grad(G grad, int mb, const DMat& m, const Shade& g, V3 wi, V3 w, float,
                                         float) {
    float d[kDisneyParams];
    disney_grad(m, disney_geom(g.ns, g.tx, g.ty, g.wo, wi), w, d);
#pragma unroll
    for (int j = 0; j < kDisneyParams; ++j) lds_add(grad, mb + j, d[j]);
}

// MIS weight of an emitter hit at vertex k reached by a direction sampled
// with pdf prev_pdf (balance or power heuristic against light sampling).
__device__ __forceinline__ float emit_weight(const PathArgs& a, const float* cdf, const int4* lights, const Shade& g,
                                             int k, float prev_pdf) {
    if (k == 1) return 1.0f;
    if (a.mis == 1) return 0.0f;
    if (a.mis == 0) return 1.0f;
    float pa = light_prob(cdf, a.sc.nlt, g.light) / __int_as_float(lights[g.light].z);
    float pl = pa * g.t * g.t / g.cos_emit;
    return mis_weight(prev_pdf, pl, a.mis);
}

struct NeeS {
    V3 wl;
    float d2, dist, cy, larea;
    int lj, ltri, lk;
    bool shoot;   // geometric tests passed: a shadow ray is needed
};

// How the forward passes round e1 u + e2 v in nee_setup (its UV), by proposal,
// parameter storage and material: what the state machine's variants were first
// compiled to, fixed here so that streams and state machine give the same bits
// whatever a compiler contracts.
__host__ __device__ constexpr int uv_rounding(int guide, int pg, int mat) {
    return guide == 1 || guide == 2 ? 0 : (mat == 0 && (pg == 0 || guide == 3) ? 2 : 1);
}

// Pick an emitter triangle from the table and a uniform point on it.  UV: how
// e1 u + e2 v is rounded: 0 as the compiler contracts it in this place, 1 with
// the first, 2 with the second product fused into the sum.
template <int UV = 0>
__device__ __forceinline__ NeeS nee_setup(const SceneDev& sc, const float* cdf, const int4* lights, const Shade& g,
                                          const float u[8]) {
    NeeS n;
    n.lj = pick_light(cdf, sc.nlt, u[0]);
    int4 lrec = lights[n.lj];
    n.ltri = lrec.x;
    n.lk = lrec.y;
    n.larea = __int_as_float(lrec.z);
    V3 q0, q1, q2;
    int lorig, lseg, llight;
    load_tri(sc, lrec.x, q0, q1, q2, lorig, lseg, llight);
    float su = sqrtf(u[1]);
    float b1 = (1.0f - u[2]) * su, b2 = u[2] * su;
    // y - x from vertex differences and edge terms: the light point and the
    // shading point are never rounded to world coordinates first
    V3 dl;
    if constexpr (UV == 0) {
        dl = (q0 - g.p0) + ((q1 - q0) * b1 + (q2 - q0) * b2 - (g.e1 * g.u + g.e2 * g.v));
    } else {
        const V3 at = UV == 1 ? fma3(g.e1, g.u, g.e2 * g.v) : fma3(g.e2, g.v, g.e1 * g.u);
        dl = (q0 - g.p0) + ((q1 - q0) * b1 + (q2 - q0) * b2 - at);
    }
    V3 lng = normalize(cross(q1 - q0, q2 - q0));
    n.d2 = dot(dl, dl);
    n.dist = sqrtf(n.d2);
    n.wl = dl * (1.0f / n.dist);
    n.cy = -dot(n.wl, lng);
    float cxg = dot(n.wl, g.ngf);
    // grazing configurations (cosines below 1e-6: the light triangle itself,
    // a coplanar emitter) are skipped
    n.shoot = n.cy > 1e-6f && cxg > 1e-6f;
    return n;
}

struct NeeC {
    V3 c;            // local contribution (without the prefix throughput)
    V3 e, f;         // emission and BRDF value
    float g;         // cos_x cos_y / d^2 * MIS weight / p_area * profile
    float spec, dspec;
    bool valid;
};

// The light-sample contribution assuming the shadow ray is unoccluded.
// pb >= 0 overrides the BRDF-sampling density of the light direction (the
// combined density when a guide is used).
template <class M>
__device__ __forceinline__ NeeC nee_contrib(const PathArgs& a, const Lds& lds, const float* cdf, const Shade& g,
                                            const M& m, const M& ms, const NeeS& n, float pb_in = -1.0f) {
    NeeC r;
    r.spec = r.dspec = 0.0f;
    float cx = dot(g.ns, n.wl);
    r.valid = cx > 0.0f;
    r.c = v3(0.0f, 0.0f, 0.0f);
    r.e = r.c;
    r.f = r.c;
    r.g = 0.0f;
    if (!r.valid) return r;
    float parea = light_prob(cdf, a.sc.nlt, n.lj) / n.larea;
    float w = 1.0f;
    if (a.mis >= 2) {
        float pl = parea * n.d2 / n.cy;
        float pb = pb_in >= 0.0f ? pb_in : mat_pdf(ms, g, n.wl);
        w = mis_weight(pl, pb, a.mis);
    }
    float prof = a.profile ? n.cy : 1.0f;
    r.g = cx * n.cy / n.d2 * w / parea * prof;
    const float* ep = lds.params + MatNP<M>::value * a.sc.S + 3 * n.lk;
    r.e = v3(ep[0], ep[1], ep[2]);
    r.f = mat_f(m, g, n.wl, r.spec, r.dspec);
    r.c = r.f * r.e * r.g;
    return r;
}

struct ContS {
    V3 wi, av, ts;     // av, ts: continuation weight at params / sampling params (before RR)
    float pdf, g, spec, dspec, qrr;
    int lobe;
    bool ok;           // a direction above the surface with pdf > 0
    bool alive;        // survived Russian roulette
};

// Continuation weight of a sampled direction wi with sampling density pdf:
// validity (above both the geometric and the shading surface, pdf > 0),
// a = f cos / pdf at params, the same at sampling params (for Russian
// roulette), and the roulette decision.
template <class M>
__device__ __forceinline__ ContS cont_eval(const PathArgs& a, const Shade& g, const M& m, const M& ms, V3 wi,
                                           float pdf, int lobe, const float u[8], int k, V3 Ts) {
    ContS c;
    c.wi = wi;
    c.lobe = lobe;
    c.pdf = pdf;
    c.qrr = 1.0f;
    c.alive = false;
    c.av = v3(0.0f, 0.0f, 0.0f);
    c.ts = c.av;
    c.g = c.spec = c.dspec = 0.0f;
    c.ok = pdf > 0.0f && dot(wi, g.ngf) > 0.0f && dot(wi, g.ns) > 0.0f;
    if (!c.ok) return c;
    const V3 f = mat_f(m, g, wi, c.spec, c.dspec);
    float ci = dot(g.ns, wi);
    c.g = ci / pdf;
    c.av = f * c.g;
    c.ts = c.av;
    if (a.frozen) c.ts = mat_f_only(ms, g, wi) * c.g;
    c.alive = true;
    if (a.rr_depth >= 0 && k >= a.rr_depth) {
        c.qrr = fminf(fmaxf(maxc(Ts * c.ts), 0.1f), 0.95f);
        c.alive = u[6] < c.qrr;
    }
    return c;
}

// Sample the continuation direction.  Without a guide (mix == NULL): the
// lobe mixture at sampling parameters.  With a guide: the technique is the
// guide with probability gmix (u[7]), the BRDF otherwise, and the density is
// the combined gmix q + (1 - gmix) p_brdf (one-sample MIS).
// Density and sample of the proposal: the mixture of the network's outputs
// (per-vertex kinds) or a cached row (kind 3).
template <int GUIDE>
__device__ __forceinline__ float guide_pdf(const float* mix, V3 w) {
    if (GUIDE == 3) return cached_pdf(mix, w);
    return mixture_pdf(mix, w);
}
template <int GUIDE>
__device__ __forceinline__ V3 guide_sample(const float* mix, float u3, float u4, float u5) {
    if (GUIDE == 3) return cached_sample(mix, u3, u4, u5);
    return mixture_sample(mix, u3, u4, u5);
}

template <int GUIDE, class M>
__device__ __forceinline__ ContS cont_sample(const PathArgs& a, const Shade& g, const M& m, const M& ms,
                                             const float u[8], int k, V3 Ts, const float* mix, bool& used_guide) {
    V3 wi = v3(0.0f, 0.0f, 1.0f);
    int lobe = 0;
    used_guide = false;
    float pdf = 0.0f;
    if (GUIDE && mix && u[7] < a.gmix) {
        used_guide = true;
        wi = guide_sample<GUIDE>(mix, u[3], u[4], u[5]);
        pdf = a.gmix * guide_pdf<GUIDE>(mix, wi) + (1.0f - a.gmix) * mat_pdf(ms, g, wi);
    } else {
        bool okd = mat_sample(ms, g, u[3], u[4], u[5], wi, lobe);
        if (okd && dot(wi, g.ngf) > 0.0f && dot(wi, g.ns) > 0.0f) {
            pdf = mat_pdf(ms, g, wi);
            if (GUIDE && mix) pdf = a.gmix * guide_pdf<GUIDE>(mix, wi) + (1.0f - a.gmix) * pdf;
        }
    }
    return cont_eval(a, g, m, ms, wi, pdf, lobe, u, k, Ts);
}

// The cached proposal's one-sample MIS in two steps, so that both densities a
// vertex needs (continuation direction, light sample) come from one pass over
// its row: first the technique (u[7]) and the direction (u[3..5]) ...
struct ContDir {
    V3 wi;
    int lobe;
    bool ok;      // BRDF technique: a direction above the surface
    bool guide;   // the proposal's technique was chosen
};
template <class M>
__device__ __forceinline__ ContDir cont_direction_cached(const PathArgs& a, const Shade& g, const M& ms,
                                                         const float u[8], const float* row) {
    ContDir c;
    c.lobe = 0;
    c.guide = u[7] < a.gmix;
    if (c.guide) {
        c.wi = cached_sample(row, u[3], u[4], u[5]);
        c.ok = true;
    } else {
        c.wi = v3(0.0f, 0.0f, 1.0f);
        c.ok = mat_sample(ms, g, u[3], u[4], u[5], c.wi, c.lobe) && dot(c.wi, g.ngf) > 0.0f &&
               dot(c.wi, g.ns) > 0.0f;
    }
    return c;
}
// ... then, with the proposal's density q of that direction, the combined
// density and the continuation weight (as cont_sample).
template <class M>
__device__ __forceinline__ ContS cont_finish_cached(const PathArgs& a, const Shade& g, const M& m, const M& ms,
                                                    const float u[8], int k, V3 Ts, const ContDir& c, float q) {
    float pdf = 0.0f;
    if (c.guide || c.ok) pdf = a.gmix * q + (1.0f - a.gmix) * mat_pdf(ms, g, c.wi);
    return cont_eval(a, g, m, ms, c.wi, pdf, c.lobe, u, k, Ts);
}

// Streaming store or load of one 16 B record of a checkpoint or list: it is read
// again only by a later kernel, so they should not displace the scene's nodes and
// triangles in the caches.
__device__ __forceinline__ void st_stream(float4* p, float4 v) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<f4*>(p));
}
__device__ __forceinline__ void st_stream(int4* p, int4 v) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    const i4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<i4*>(p));
}

__device__ __forceinline__ float4 ld_stream(const float4* p) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 x = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
    return make_float4(x.x, x.y, x.z, x.w);
}
__device__ __forceinline__ int4 ld_stream(const int4* p) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    const i4 x = __builtin_nontemporal_load(reinterpret_cast<const i4*>(p));
    return make_int4(x.x, x.y, x.z, x.w);
}

// Index of the records of vertex k (1..) of sample s of the chunk's pixel q.
__device__ __forceinline__ size_t ck_at(const PathArgs& a, int k, int s, int64_t q) {
    return (((size_t)(k - 1) * a.spp + s) * (size_t)a.pix_count + q) * a.ck_n;
}

// Backward sweep of the gradient forward pass: R_{k+1} into the c slot of
// vertex k; returns the path radiance.
__device__ __forceinline__ V3 suffix_sweep(const PathArgs& a, int klast, int s, int64_t q) {
    V3 R = v3(0.0f, 0.0f, 0.0f);
    for (int k = klast; k >= 1; --k) {
        const size_t ck = ck_at(a, k, s, q);
        float4 c = a.ck_c[ck], av = a.ck_a[ck];
        a.ck_c[ck] = make_float4(R.x, R.y, R.z, c.w);
        R = v3(c.x, c.y, c.z) + v3(av.x, av.y, av.z) * R;
    }
    return R;
}

// One atomic per wave (the first active lane's).
__device__ __forceinline__ void count_add(unsigned long long* c, uint32_t x) {
    unsigned long long s = x;
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0 && s) atomicAdd(c, s);
}

__device__ __forceinline__ void flush_stats(const PathArgs& a, int mode, const Work& wk, uint32_t npaths) {
    if (!a.count_stats) return;
    KStats* ks = &a.err->k[mode];
    count_add(&ks->rays, wk.rays);
    count_add(&ks->nodes, wk.nodes);
    count_add(&ks->tris, wk.tris);
    count_add(&ks->paths, npaths);
    count_add(&ks->vertices, wk.vertices);
    count_add(&ks->units, wk.units);
}

}  // namespace ipt
