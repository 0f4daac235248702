// Path streams (gfx950): the colour pass and the gradient forward pass of many
// paths as alternating kernels over dense lists instead of one state machine
// per lane.
//
//   ray generation -> [ray kernel -> shading kernel] per vertex -> finish
//
// All paths of a batch advance by one vertex at a time.  The ray kernel traces
// the closest-hit rays of vertex k and the shadow rays of vertex k - 1; the
// shading kernel turns every hit into a light sample and a continuation and
// appends both, compacted, to the lists of the next vertex.  A wave of the
// state machine (trace.hip) runs each phase for whichever lanes are in it:
// measured on the room workload 30% of the lanes of an issued VALU instruction
// were active (apartment 42%).  Here the lanes of the shading kernel are all
// in the same phase, and a lane of the ray kernel that has finished its ray
// takes the next one of the list.  The price is the path state in memory,
// about 250 B per path vertex, read and written in list order (coalesced) by
// streaming accesses, which leave the caches to the scene (apartment step 91.3 ->
// 90.2 ms, office floor render 19.8 -> 19.6).
//
// Measured, state machine -> streams: room step 17.4 -> 9.6 ms, apartment 132.6 ->
// 95.8 ms, and the passes of 4096 to 524288 paths 1.3-4 times faster.  The state
// machine serves single paths, the debug outputs, the proposal network evaluated
// per vertex and calls with little workspace (stream_batch in api.hip).
//
// Lists are split over 8 groups, one per XCD (blocks b mod 8): with one list
// for all, the appends' and chunk counters' atomics on one address took longer
// than the shading (they reach about 250 per us): apartment step 113 -> 102 ms.
//
// Every path draws the same numbers and does the same arithmetic in the same
// order as in the state machine: images and checkpoints agree bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "path_dev.h"
#include "ray_stream.h"

namespace ipt {

namespace {

// list positions of the lanes of a block that append to one of two lists: one
// atomic per block and list
struct Append {
    unsigned wave[2][kBlock / 64];
    unsigned base[2];
};
__device__ __forceinline__ void append2(Append& sh, unsigned* count, bool a, bool b, unsigned& ia, unsigned& ib) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t ma = __ballot(a), mb = __ballot(b);
    if (lane == 0) {
        sh.wave[0][w] = (unsigned)__popcll(ma);
        sh.wave[1][w] = (unsigned)__popcll(mb);
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned* c = sh.wave[threadIdx.x];
        unsigned s = 0;
        for (int i = 0; i < kBlock / 64; ++i) {
            const unsigned x = c[i];
            c[i] = s;
            s += x;
        }
        sh.base[threadIdx.x] = s ? atomicAdd(count + threadIdx.x, s) : 0u;
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    ia = sh.base[0] + sh.wave[0][w] + (unsigned)__popcll(ma & below);
    ib = sh.base[1] + sh.wave[1][w] + (unsigned)__popcll(mb & below);
    __syncthreads();   // the next tile writes sh again
}

// Path p of a batch: sample s of the batch's pixel q (consecutive lanes:
// consecutive pixels, same sample).
struct PathId {
    int s;
    int64_t q;       // pixel within the checkpoint chunk
    int64_t wi, pix;
    bool ok;
};
__device__ __forceinline__ PathId path_id(const PathArgs& a, const StreamArgs& t, unsigned p) {
    PathId r;
    r.s = (int)(p / t.nq);
    r.q = t.q0 + (int64_t)(p - (unsigned)r.s * t.nq);
    r.wi = a.pix_begin + r.q;
    r.pix = a.pixel_list ? a.pixel_list[r.wi] : r.wi;
    r.ok = r.pix >= 0 && r.pix < (int64_t)a.V * a.W * a.H;
    return r;
}

// The state machine's shading block sees the hit's geometry as loop-carried
// values.  Here the same code would follow the expressions that made them, and
// the compiler would fold, say, the negation in wo = -d into the products that
// use wo: other operand orders, other fused multiply-adds, other last bits.
// Hiding the values' origin keeps the two forms' arithmetic the same.
__device__ __forceinline__ void hide(float& x) { __asm__("" : "+v"(x)); }
__device__ __forceinline__ void hide(V3& a) { hide(a.x); hide(a.y); hide(a.z); }
__device__ __forceinline__ void hide(Shade& g) {
    hide(g.p0); hide(g.e1); hide(g.e2); hide(g.x); hide(g.ng); hide(g.ngf); hide(g.ns); hide(g.wo);
}

constexpr unsigned kCounts = (kMaxDepth + 2) * kStreamGroups * kStreamCount;
__device__ __forceinline__ unsigned* counters(const StreamArgs& t, int k, unsigned group) {
    return t.count + ((size_t)(k - 1) * kStreamGroups + group) * kStreamCount;
}
// Paths of a group among n.
__device__ __forceinline__ unsigned group_paths(unsigned n, unsigned group) {
    const unsigned tiles = (n + kBlock - 1) / kBlock;
    if (group >= tiles) return 0u;
    const unsigned own = (tiles - group + kStreamGroups - 1) / kStreamGroups * kBlock;
    return (tiles - 1) % kStreamGroups == group ? own - (tiles * kBlock - n) : own;
}

// Camera rays of all paths of the batch; a path of an invalid pixel traces a
// placeholder ray whose hit is ignored.
__global__ __launch_bounds__(kBlock) void stream_camera_kernel(PathArgs a, StreamArgs t) {
    const unsigned n = t.nq * (unsigned)a.spp;
    for (unsigned i = blockIdx.x * kBlock + threadIdx.x; i < kCounts; i += gridDim.x * kBlock)
        t.count[i] = i < kStreamGroups * kStreamCount && i % kStreamCount == 0 ? group_paths(n, i / kStreamCount) : 0u;
    for (unsigned p = blockIdx.x * kBlock + threadIdx.x; p < n; p += gridDim.x * kBlock) {
        const unsigned tile = p / kBlock;
        const unsigned i = (tile % kStreamGroups) * t.cap + (tile / kStreamGroups) * kBlock + p % kBlock;
        const PathId id = path_id(a, t, p);
        V3 o = v3(0.0f, 0.0f, 0.0f), d = v3(0.0f, 0.0f, 1.0f);
        unsigned tag = kNoPath;
        if (id.ok) {
            const uint64_t pid = (uint64_t)id.pix * (uint64_t)a.spp + (uint64_t)id.s;
            float j0 = 0.5f, j1 = 0.5f;
            if (a.jitter) jitter_uniforms(a.rng, pid, j0, j1);
            const int view = (int)(id.pix / ((int64_t)a.W * a.H));
            const int64_t rem = id.pix - (int64_t)view * a.W * a.H;
            const int py = (int)(rem / a.W), px = (int)(rem - (int64_t)py * a.W);
            camera_ray(a, view, (float)px + j0, (float)py + j1, o, d);
            tag = p;
        } else {
            t.L[p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        t.ray_o[0][i] = make_float4(o.x, o.y, o.z, __int_as_float(-1));
        t.ray_d[0][i] = make_float4(d.x, d.y, d.z, 0.0f);
        t.path[0][i] = make_float4(1.0f, 1.0f, 1.0f, __uint_as_float(tag));
    }
}

// Rays of one vertex: closest-hit rays [0, nc), then shadow rays.
template <int MODE>
struct PathRays {
    const PathArgs* a;
    const StreamArgs* t;
    unsigned nc, first;   // closest-hit rays of the group; its first list entry
    int cur;
    __device__ __forceinline__ void load(unsigned i, V3& o, V3& d, float& tmax, int& skip0, int& skip1, bool& any) const {
        any = i >= nc;
        const unsigned j = first + (any ? i - nc : i);
        const float4 A = ld_stream(any ? &t->sh_o[j] : &t->ray_o[cur][j]);
        const float4 B = any ? t->sh_d[j] : t->ray_d[cur][j];
        o = xyz(A);
        d = xyz(B);
        skip0 = __float_as_int(A.w);
        skip1 = any ? __float_as_int(t->sh_c[j].w) : -1;
        tmax = any ? B.w : __builtin_inff();
    }
    __device__ __forceinline__ void store(unsigned i, bool any, const Hit& h) const {
        if (!any) {
            st_stream(&t->hit[first + i], make_int4(h.tri, __float_as_int(h.u), __float_as_int(h.v), __float_as_int(h.t)));
        } else if (h.tri < 0) {
            // unoccluded: the light sample's contribution (one shadow ray per
            // path and vertex, so no two lanes touch the same record)
            const unsigned j = first + i - nc;
            const float4 c = t->sh_lt[j];
            const unsigned p = __float_as_uint(c.w);
            const float4 L = t->L[p];
            t->L[p] = make_float4(__fadd_rn(L.x, c.x), __fadd_rn(L.y, c.y), __fadd_rn(L.z, c.z), 0.0f);
            if (MODE == kGradFwd) {
                const int s = (int)(p / t->nq);
                const int64_t q = t->q0 + (int64_t)(p - (unsigned)s * t->nq);
                const size_t ck = ck_at(*a, t->k - 1, s, q);
                const float4 n = t->sh_c[j];
                const float4 v = a->ck_c[ck];
                a->ck_hit[ck].x |= (int)kCkVis;
                a->ck_c[ck] = make_float4(__fadd_rn(v.x, n.x), __fadd_rn(v.y, n.y), __fadd_rn(v.z, n.z), v.w);
            }
        }
    }
};

// Rays of vertex k (ray_stream.h says what bounds them): 31 + 34 ms of the
// apartment step's colour and gradient passes.
template <int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kRayBlocksPerCu, 8))) void stream_ray_kernel(PathArgs a,
                                                                                                        StreamArgs t) {
    __shared__ int stk[kRayStack * kBlock];
    const unsigned group = blockIdx.x % kStreamGroups;
    unsigned* count = counters(t, t.k, group);
    const unsigned nc = count[0], n = nc + count[1];
    const PathRays<MODE> src{&a, &t, nc, group * t.cap, (t.k - 1) & 1};
    const unsigned wave = __builtin_amdgcn_readfirstlane(blockIdx.x / kStreamGroups * (kBlock / 64) + (threadIdx.x >> 6));
    trace_stream(a.sc, a.sc.tmin, src, n, stk, t.ovf, wave, gridDim.x / kStreamGroups * (kBlock / 64), count + 2, a.err,
                 a.count_stats ? &a.err->k[MODE] : nullptr);
}

// Closest hits of a caller's rays.  Every gridDim-th 64 rays belong to a block
// (runs of consecutive rays cost unequally: 0.75 ms for 4.9 M camera rays of the
// apartment), its waves take chunks of them: 0.98 -> 0.68 ms.
struct BatchRays {
    const SceneDev* sc;
    const float* o;
    const float* d;
    const int* skip;
    int64_t nt;
    int* out_tri;
    float* out_tuv;
    static __device__ __forceinline__ int64_t ray(unsigned i) {
        return ((int64_t)(i >> 6) * gridDim.x + blockIdx.x) * 64 + (i & 63u);
    }
    __device__ __forceinline__ void load(unsigned i, V3& ro, V3& rd, float& tmax, int& skip0, int& skip1, bool& any) const {
        const int64_t j = ray(i);
        ro = v3(o[3 * j], o[3 * j + 1], o[3 * j + 2]);
        rd = v3(d[3 * j], d[3 * j + 1], d[3 * j + 2]);
        skip0 = (skip && skip[j] >= 0 && skip[j] < nt) ? sc->pos_of[skip[j]] : -1;
        skip1 = -1;
        tmax = __builtin_inff();
        any = false;
    }
    __device__ __forceinline__ void store(unsigned i, bool, const Hit& h) const {
        const int64_t j = ray(i);
        out_tri[j] = h.tri >= 0 ? __float_as_int(sc->tris[3 * (int64_t)h.tri].w) : -1;
        out_tuv[3 * j] = h.tri >= 0 ? h.t : 0.0f;
        out_tuv[3 * j + 1] = h.u;
        out_tuv[3 * j + 2] = h.v;
    }
};
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kRayBlocksPerCu, 8))) void batch_ray_kernel(
    SceneDev sc, const float* o, const float* d, const int* skip, int64_t n, float tmin, int64_t nt,
    int* out_tri, float* out_tuv, int* ovf, Counters* err) {
    __shared__ int stk[kRayStack * kBlock];
    __shared__ unsigned work;
    if (threadIdx.x == 0) work = 0u;
    __syncthreads();
    const int64_t sets = (n + 63) / 64, mine = (sets - blockIdx.x + gridDim.x - 1) / gridDim.x;   // sets of 64 rays
    const bool last = (sets - 1) % gridDim.x == blockIdx.x;
    const unsigned own = (unsigned)(64 * mine - (last ? 64 * sets - n : 0));
    const BatchRays src{&sc, o, d, skip, nt, out_tri, out_tuv};
    trace_stream(sc, tmin, src, own, stk, ovf, (unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                 (unsigned)(kBlock / 64), &work, err, (KStats*)nullptr);
}

// Shading of vertex k for every closest-hit ray of the list.  Bound by memory
// latency (78-80% of the lanes active; L1 waits 64-71% of the cycles): 7.3 and 12 ms of
// the apartment step's two passes.  No spills (98-157 VGPRs), unlike the state
// machine's 41-51; a forced fourth or fifth wave per SIMD changed nothing (97.0 ms)
// or spilled (102.2 ms).
template <int MODE, int GUIDE, int PG, int MAT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 8))) void stream_shade_kernel(PathArgs a,
                                                                                                          StreamArgs t) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ Append app;
    Lds lds;
    carve_lds<PG>(a, MODE, smem, lds);
    const SceneDev& sc = a.sc;
    const float* cdf = lds.lights_in_lds ? lds.cdf : a.cdf;
    const int4* lights = lds.lights_in_lds ? lds.lights : sc.lights;
    constexpr int UV = uv_rounding(GUIDE, PG, MAT);
    const int k = t.k, D = a.D;
    const int in = (k - 1) & 1, out = k & 1;
    const unsigned group = blockIdx.x % kStreamGroups, first = group * t.cap;
    const unsigned n = counters(t, k, group)[0];
    uint32_t npaths = 0, nvert = 0;
    for (unsigned tile = blockIdx.x / kStreamGroups * kBlock; tile < n; tile += gridDim.x / kStreamGroups * kBlock) {
        const unsigned i = first + tile + threadIdx.x;
        bool shoot = false, cont = false;
        NeeS nee;
        V3 nee_c = v3(0.0f, 0.0f, 0.0f), nee_LT = nee_c, T = nee_c, Ts = nee_c;
        ContS cs;
        Shade g;
        unsigned p = kNoPath;
        if (tile + threadIdx.x < n) {
            const float4 st = ld_stream(&t.path[in][i]);
            p = __float_as_uint(st.w);
            T = xyz(st);
        }
        if (p != kNoPath) {
            const PathId id = path_id(a, t, p);
            const uint64_t pid = (uint64_t)id.pix * (uint64_t)a.spp + (uint64_t)id.s;
            const size_t c1 = ck_at(a, 1, id.s, id.q);
            const size_t ck = ck_at(a, k, id.s, id.q);
            const int4 hb = ld_stream(&t.hit[i]);
            Hit hr;
            hr.tri = hb.x;
            hr.u = __int_as_float(hb.y);
            hr.v = __int_as_float(hb.z);
            hr.t = __int_as_float(hb.w);
            ++nvert;
            int klast = k;
            bool end_path = true;
            if (hr.tri < 0) {
                if (MODE == kGradFwd) a.ck_hit[ck] = make_int4(0, 0, 0, 0);
                klast = k - 1;   // a miss contributes nothing: the sweep starts below it
                if (k == 1) t.L[p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            } else {
                const float4 rd = ld_stream(&t.ray_d[in][i]);
                const V3 d = xyz(rd);
                const float prev_pdf = rd.w;
                make_shade(sc, lds, hr, d, g);
                V3 cpart = v3(0.0f, 0.0f, 0.0f);
                V3 L = cpart;
                bool emit = false;
                if (g.em >= 0 && g.cos_emit > 0.0f) {
                    float w = emit_weight(a, cdf, lights, g, k, prev_pdf);
                    if (w > 0.0f) {
                        float prof = a.profile ? g.cos_emit : 1.0f;
                        const float* e = lds.params + MatSel<MAT>::NP * sc.S + 3 * g.em;
                        V3 c = v3(e[0], e[1], e[2]) * (prof * w);
                        cpart = c;
                        if (k > 1) {
                            const float4 l = t.L[p];
                            L = xyz(l);
                        }
                        L = L + T * c;
                        emit = true;
                    }
                }
                if (emit || k == 1) t.L[p] = make_float4(L.x, L.y, L.z, 0.0f);
                if (k == D + 1 || dot(g.ns, g.wo) <= 0.0f) {
                    // x_{D+1} only counts its emission; a shading normal facing
                    // away ends the path
                    if (MODE == kGradFwd) {
                        a.ck_hit[ck] = make_int4(g.tri + 1, hb.y, hb.z, hb.w);
                        a.ck_a[ck] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        a.ck_c[ck] = make_float4(cpart.x, cpart.y, cpart.z, 0.0f);
                    }
                } else {
                    // ---- light sample and continuation of vertex k ----
                    hide(g);
                    const float* mix = nullptr;
                    if constexpr (GUIDE == 3) mix = cache_row_at(a.gd, g.tri, g.u, g.v, dot(g.ng, g.wo) < 0.0f);
                    if (a.rr_depth >= 0) Ts = k == 1 ? v3(1.0f, 1.0f, 1.0f) : xyz(ld_stream(&t.path_s[in][i]));
                    mat_frame<MAT>(g);
                    const typename MatSel<MAT>::M m = mat_load<MAT>(lds.params, g.seg);
                    const typename MatSel<MAT>::M ms = a.frozen ? mat_load<MAT>(lds.sparams, g.seg) : m;
                    float u[8];
                    vertex_uniforms(a.rng, pid, k, u);
                    float pb_nee = -1.0f;
                    nee.shoot = false;
                    const bool do_nee = a.mis != 0 && sc.nlt > 0;
                    auto take_nee = [&]() {
                        NeeC nc = nee_contrib(a, lds, cdf, g, m, ms, nee, pb_nee);
                        shoot = true;
                        if (nc.valid) {
                            nee_c = nc.c;
                            nee_LT = T * nc.c;
                        }
                    };
                    bool used_guide = false;
                    if constexpr (GUIDE == 3) {
                        if (do_nee) nee = nee_setup<UV>(sc, cdf, lights, g, u);
                        const ContDir cd = cont_direction_cached(a, g, ms, u, mix);
                        float q_wi, q_wl;
                        cached_pdf2(mix, cd.wi, nee.shoot ? nee.wl : cd.wi, q_wi, q_wl);
                        if (nee.shoot) {
                            pb_nee = a.gmix * q_wl + (1.0f - a.gmix) * mat_pdf(ms, g, nee.wl);
                            take_nee();
                        }
                        cs = cont_finish_cached(a, g, m, ms, u, k, Ts, cd, q_wi);
                    } else {
                        if (do_nee) {
                            nee = nee_setup<UV>(sc, cdf, lights, g, u);
                            if (nee.shoot) take_nee();
                        }
                        cs = cont_sample<GUIDE>(a, g, m, ms, u, k, Ts, mix, used_guide);
                    }
                    V3 av = v3(0.0f, 0.0f, 0.0f);
                    uint32_t flags = 0;
                    float rq = 1.0f;
                    cont = cs.ok && cs.alive;
                    if (cont) {
                        rq = 1.0f / cs.qrr;
                        av = cs.av * rq;
                        Ts = Ts * cs.ts * rq;
                        flags |= kCkCont;
                        T = T * av;
                    }
                    end_path = !cont;
                    if (MODE == kGradFwd) {
                        a.ck_hit[ck] = make_int4((int)((uint32_t)(g.tri + 1) | flags), hb.y, hb.z, hb.w);
                        a.ck_a[ck] = make_float4(av.x, av.y, av.z, cs.pdf);
                        if (a.guided) a.ck_d[ck] = make_float4(cs.wi.x, cs.wi.y, cs.wi.z, pb_nee);
                        a.ck_c[ck] = make_float4(cpart.x, cpart.y, cpart.z, rq);
                    }
                }
            }
            if (end_path) {
                ++npaths;
                // index of the path's last vertex, for the backward sweep
                if (MODE == kGradFwd) a.ck_c[c1].w = __int_as_float(klast);
            }
        }
        unsigned ic, is;
        append2(app, counters(t, k + 1, group), cont, shoot, ic, is);
        ic += first;
        is += first;
        if (cont) {
            st_stream(&t.ray_o[out][ic], make_float4(g.x.x, g.x.y, g.x.z, __int_as_float(g.tri)));
            st_stream(&t.ray_d[out][ic], make_float4(cs.wi.x, cs.wi.y, cs.wi.z, cs.pdf));
            st_stream(&t.path[out][ic], make_float4(T.x, T.y, T.z, __uint_as_float(p)));
            if (a.rr_depth >= 0) st_stream(&t.path_s[out][ic], make_float4(Ts.x, Ts.y, Ts.z, 0.0f));
        }
        if (shoot) {
            st_stream(&t.sh_o[is], make_float4(g.x.x, g.x.y, g.x.z, __int_as_float(g.tri)));
            st_stream(&t.sh_d[is], make_float4(nee.wl.x, nee.wl.y, nee.wl.z, nee.dist * (1.0f - 1e-5f)));
            st_stream(&t.sh_lt[is], make_float4(nee_LT.x, nee_LT.y, nee_LT.z, __uint_as_float(p)));
            st_stream(&t.sh_c[is], make_float4(nee_c.x, nee_c.y, nee_c.z, __int_as_float(nee.ltri)));
        }
    }
    if (a.count_stats) {
        KStats* ks = &a.err->k[MODE];
        count_add(&ks->paths, npaths);
        count_add(&ks->vertices, nvert);
    }
}

// Colour: pixel means (or, where a pixel's samples form several units, the
// units' sums) in sample order.
__global__ __launch_bounds__(kBlock) void stream_colour_kernel(PathArgs a, StreamArgs t) {
    const int64_t nunits = (int64_t)t.nq * a.nchunk;
    uint32_t units = 0;
    for (int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x; u < nunits; u += (int64_t)gridDim.x * kBlock) {
        const int c = (int)(u / t.nq);
        const int64_t q = t.q0 + (u - (int64_t)c * t.nq);
        const int64_t wi = a.pix_begin + q;
        const int64_t pix = a.pixel_list ? a.pixel_list[wi] : wi;
        const bool ok = pix >= 0 && pix < (int64_t)a.V * a.W * a.H;
        V3 acc = v3(0.0f, 0.0f, 0.0f);
        const int s_end = min(a.spp, (c + 1) * a.spc);
        for (int s = c * a.spc; ok && s < s_end; ++s) {
            const V3 L = xyz(t.L[(size_t)s * t.nq + (size_t)(q - t.q0)]);
            const size_t pidx = (size_t)wi * a.spp + s;
            const bool use = a.mask ? a.mask[pidx] != 0 : true;
            if (!finite3(L)) atomicAdd(&a.err->nonfinite, 1ull);
            else if (use) acc = acc + L;
            if (a.path_L) {
                a.path_L[3 * pidx] = L.x;
                a.path_L[3 * pidx + 1] = L.y;
                a.path_L[3 * pidx + 2] = L.z;
            }
        }
        if (a.nchunk > 1) {
            float* o = a.part + 3 * ((size_t)c * a.pix_count + q);
            o[0] = acc.x;
            o[1] = acc.y;
            o[2] = acc.z;
        } else {
            const float inv = 1.0f / (float)a.spp;
            a.image[3 * wi] = acc.x * inv;
            a.image[3 * wi + 1] = acc.y * inv;
            a.image[3 * wi + 2] = acc.z * inv;
        }
        ++units;
    }
    if (a.count_stats) count_add(&a.err->k[kColor].units, units);
}

// Gradient forward pass: drops paths whose radiance is not finite; with a
// guide attached also the backward sweep (its records read R_{k+1} before the
// replay runs).
__global__ __launch_bounds__(kBlock) void stream_grad_end_kernel(PathArgs a, StreamArgs t) {
    const unsigned n = t.nq * (unsigned)a.spp;
    for (unsigned p = blockIdx.x * kBlock + threadIdx.x; p < n; p += gridDim.x * kBlock) {
        const PathId id = path_id(a, t, p);
        if (!id.ok) continue;
        const size_t c1 = ck_at(a, 1, id.s, id.q);
        bool good = finite3(xyz(t.L[p]));
        if (a.guided) {
            const int klast = min(max(__float_as_int(a.ck_c[c1].w), 0), a.D + 1);
            good = finite3(suffix_sweep(a, klast, id.s, id.q)) && good;
        }
        if (!good) {
            a.ck_hit[c1].x = (int)((uint32_t)a.ck_hit[c1].x | kCkDrop);
            atomicAdd(&a.err->nonfinite, 1ull);
        }
    }
    if (a.count_stats && blockIdx.x == 0 && threadIdx.x == 0)
        atomicAdd(&a.err->k[kGradFwd].units, (unsigned long long)t.nq * a.nchunk);
}

// blocks for every group
int group_grid(int blocks) { return (blocks + kStreamGroups - 1) / kStreamGroups * kStreamGroups; }

// Launches the shading kernel on as many blocks as the chip holds at once:
// the blocks are persistent, a further one would run after the others.
template <class K>
hipError_t launch_resident(K kern, const PathArgs& a, const StreamArgs& t, int blocks, int num_cu, size_t lds,
                           hipStream_t st) {
    int per_cu = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kBlock, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(group_grid(std::min(blocks, num_cu * std::max(1, per_cu)))), dim3(kBlock), lds, st, a, t);
    return hipGetLastError();
}
template <int MODE, int PG, int MAT>
hipError_t launch_shade(const PathArgs& a, const StreamArgs& t, int blocks, int num_cu, size_t lds, hipStream_t st) {
    if (a.guide_kind == 3) return launch_resident(stream_shade_kernel<MODE, 3, PG, MAT>, a, t, blocks, num_cu, lds, st);
    return launch_resident(stream_shade_kernel<MODE, 0, PG, MAT>, a, t, blocks, num_cu, lds, st);
}
template <int MODE>
hipError_t launch_shade_kind(const PathArgs& a, const StreamArgs& t, int blocks, int num_cu, size_t lds,
                             hipStream_t st) {
    const int pg = a.params_global;
    if (a.mat == 1)
        return pg ? launch_shade<MODE, 1, 1>(a, t, blocks, num_cu, lds, st)
                  : launch_shade<MODE, 0, 1>(a, t, blocks, num_cu, lds, st);
    return pg ? launch_shade<MODE, 1, 0>(a, t, blocks, num_cu, lds, st)
              : launch_shade<MODE, 0, 0>(a, t, blocks, num_cu, lds, st);
}

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

size_t ray_stream_ovf_bytes(int blocks) { return sizeof(int) * (size_t)kRayOvf * blocks * kBlock; }

int batch_ray_blocks(int num_cu) { return num_cu * kRayBlocksPerCu; }

hipError_t launch_batch_rays(const SceneDev& sc, const float* o, const float* d, const int* skip, int64_t n, float tmin,
                             int64_t nt, int* out_tri, float* out_tuv, int* ovf, int num_cu, Counters* err,
                             hipStream_t st) {
    const int64_t blocks = std::min<int64_t>(batch_ray_blocks(num_cu), (n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(batch_ray_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st, sc, o, d, skip, n, tmin, nt,
                       out_tri, out_tuv, ovf, err);
    return hipGetLastError();
}

size_t stream_fixed_bytes(int num_cu) {
    // counters, overflow stacks, and what the lists need beyond one entry per path
    return al256(sizeof(unsigned) * kCounts) + ray_stream_ovf_bytes(num_cu * kRayBlocksPerCu) + 16 * 256 +
           kStreamPathBytes * (kStreamGroups + 1) * kBlock;
}

StreamArgs stream_layout(unsigned char* p, int num_cu, int64_t npaths) {
    StreamArgs t{};
    auto take = [&](size_t bytes) {
        unsigned char* r = p;
        p += al256(bytes);
        return r;
    };
    const int64_t tiles = (npaths + kBlock - 1) / kBlock;
    t.cap = (unsigned)((tiles + kStreamGroups - 1) / kStreamGroups * kBlock);
    const size_t n = (size_t)t.cap * kStreamGroups;
    t.count = (unsigned*)take(sizeof(unsigned) * kCounts);
    t.ovf = (int*)take(ray_stream_ovf_bytes(num_cu * kRayBlocksPerCu));
    for (int i = 0; i < 2; ++i) {
        t.ray_o[i] = (float4*)take(16 * n);
        t.ray_d[i] = (float4*)take(16 * n);
        t.path[i] = (float4*)take(16 * n);
        t.path_s[i] = (float4*)take(16 * n);
    }
    t.hit = (int4*)take(16 * n);
    t.L = (float4*)take(16 * n);
    t.sh_o = (float4*)take(16 * n);
    t.sh_d = (float4*)take(16 * n);
    t.sh_lt = (float4*)take(16 * n);
    t.sh_c = (float4*)take(16 * n);
    return t;
}

hipError_t launch_stream_pass(int mode, const PathArgs& a, StreamArgs t, int64_t batch_pixels, int num_cu,
                              hipStream_t st) {
    const size_t lds = path_lds_bytes(kColor, a.P, a.frozen, a.sc.S, a.sc.nlt, 0, a.params_global) -
                       sizeof(int) * kShortStack * kBlock;
    for (int64_t q = 0; q < a.pix_count; q += batch_pixels) {
        t.q0 = q;
        t.nq = (unsigned)std::min<int64_t>(batch_pixels, a.pix_count - q);
        const int64_t n = (int64_t)t.nq * a.spp;
        const int blocks = (int)((n + kBlock - 1) / kBlock);
        const int wide = std::min(blocks, num_cu * 8);
        // the waves of few rays get at least kRayFew of them; the fifth block of a
        // CU pays only where its waves have whole sets of 64 (room step of 65536
        // paths: 1.03 ms with four, 1.06 with five)
        const int per_cu = 2 * blocks <= 4 * num_cu ? 4 : kRayBlocksPerCu;
        const int ray = std::min(group_grid(2 * 64 / (int)kRayFew * blocks), num_cu * per_cu / kStreamGroups * kStreamGroups);
        hipLaunchKernelGGL(stream_camera_kernel, dim3(wide), dim3(kBlock), 0, st, a, t);
        for (t.k = 1; t.k <= a.D + 1; ++t.k) {
            hipError_t e;
            if (mode == kColor) {
                hipLaunchKernelGGL(stream_ray_kernel<kColor>, dim3(ray), dim3(kBlock), 0, st, a, t);
                e = launch_shade_kind<kColor>(a, t, blocks, num_cu, lds, st);
            } else {
                hipLaunchKernelGGL(stream_ray_kernel<kGradFwd>, dim3(ray), dim3(kBlock), 0, st, a, t);
                e = launch_shade_kind<kGradFwd>(a, t, blocks, num_cu, lds, st);
            }
            if (e != hipSuccess) return e;
        }
        if (mode == kColor) hipLaunchKernelGGL(stream_colour_kernel, dim3(wide), dim3(kBlock), 0, st, a, t);
        else hipLaunchKernelGGL(stream_grad_end_kernel, dim3(wide), dim3(kBlock), 0, st, a, t);
    }
    return hipGetLastError();
}

}  // namespace ipt
