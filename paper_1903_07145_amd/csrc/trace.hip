// Path kernels of the inverse path tracer (gfx950).
//
// Three passes share one set of shading functions, so they compute the same
// values:
//   kColor   - the Monte Carlo pixel estimate (Sec. 3.1, Eq. 1-2) with MIS of
//              BRDF sampling and light sampling (Appendix A.2, Appendix E);
//   kGradFwd - the gradient-stream forward pass: traces the independent
//              paths (Sec. 3.3: independent samples for the estimate and for
//              its gradient), stores per-vertex hit checkpoints, the local
//              contribution c_k and continuation weight a_k, then sweeps the
//              path backwards to turn them into the suffix radiance
//              R_{k+1} = c_{k+1} + a_{k+1} R_{k+2} (no division, so exact at
//              zero albedo or zero emission);
//   kReplay  - the adjoint: replays every path from its Philox counter (hits
//              from the checkpoints, or re-traced), carries the prefix
//              throughput T_{k-1} and adds, per vertex,
//              w . T_{k-1} (dc_k/dtheta + da_k/dtheta R_{k+1}) -- the product
//              rule of Eq. 5 (emission) and Eq. 6 (materials) -- into a block
//              private gradient in LDS.
//
// kColor and kGradFwd run as a per-lane state machine around ONE traversal
// call site that serves both closest-hit and shadow rays: every iteration
// each lane traces whatever ray it has pending, then advances its path.  A
// lane owns one pixel and walks its spp samples in order, so the pixel mean
// is formed in registers (deterministic, no atomics); a lane that finishes
// its pixel takes the next one at once (the wave takes as many pixels as it
// has idle lanes with one atomic).  The lanes of a wave thus stay in the same
// phase instead of serialising the divergent loops of a nested megakernel.
#include <hip/hip_runtime.h>

#include "path_dev.h"

namespace ipt {

size_t path_lds_bytes(int mode, int P, int frozen, int S, int nlt, int gk, int pglobal) {
    size_t b = 0;
    auto al = [](size_t x) { return (x + 15) & ~size_t(15); };
    if (pglobal) P = S = 0;                           // read from global memory
    b += al(sizeof(float) * P);                       // params
    if (frozen) b += al(sizeof(float) * P);           // sampling params
    b += al(sizeof(int) * S);                         // segment -> emitter
    if (nlt <= kMaxLdsLights) b += al(2 * sizeof(float) * nlt) + al(sizeof(int4) * nlt);
    if (mode == kReplay) b += al(sizeof(double) * P); // block gradient
    b += sizeof(int) * kShortStack * kBlock;          // short stacks
    if ((gk == 1 || gk == 2) && mode != kReplay) b += kGuideLds;   // network activations / outputs
    return b;
}

// ---------------------------------------------------------------------------
// Colour / gradient-forward kernel: per-lane state machine.
// ---------------------------------------------------------------------------
enum Phase { kNeedPixel = 0, kClosest = 1, kShadow = 2, kExit = 3 };

// At least 4 waves per SIMD: the path state needs ~158 VGPRs unconstrained
// (3 waves), and the fourth wave hides more node-fetch latency than the
// ~100 bytes of spilled state cost (apartment step 241 -> 214 ms).
#ifndef IPT_WAVES_PER_EU
#define IPT_WAVES_PER_EU 4
#endif
#define IPT_OCC __attribute__((amdgpu_waves_per_eu(IPT_WAVES_PER_EU, 8)))
// The guided kernels also hold the network's operands around the MLP call:
// at 2 waves per SIMD nothing spills (apartment guided step 537 ms at 4
// waves, 487 at 3, 449 at 2).
#ifndef IPT_WAVES_PER_EU_GUIDED
#define IPT_WAVES_PER_EU_GUIDED 2
#endif
// The Disney kernels hold two 13-float materials (rendering and sampling
// parameters) at each vertex: 3 waves per SIMD spill less (apartment with
// the Disney material: step 183.0 ms at 3 waves, 187.0 at 4, 215.2 at 2).
#ifndef IPT_WAVES_PER_EU_DISNEY
#define IPT_WAVES_PER_EU_DISNEY 3
#endif

// A traversal call returns once no more than this many lanes of the wave
// are still traversing (0: every traversal runs to completion in one call).
// Apartment step: 203 ms at 0, 188 / 187 / 190 / 195 ms at 8 / 16 / 24 / 32.
#ifndef IPT_TRAV_EXIT_LANES
#define IPT_TRAV_EXIT_LANES 16
#endif
// GUIDE: 0 none, 1 bfloat16 MFMA evaluation, 2 float32 VALU evaluation, 3 cached
// proposal; MAT: the material model (MatSel)
template <int MODE, int GUIDE, int PG, int MAT>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu((GUIDE == 1 || GUIDE == 2) ? IPT_WAVES_PER_EU_GUIDED
                                   : (MAT == 1 ? IPT_WAVES_PER_EU_DISNEY : IPT_WAVES_PER_EU),
                                   8))) void path_sm_kernel(
    PathArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    Lds lds;
    carve_lds<PG>(a, MODE, smem, lds);
    Stack st;
    init_stack(st, a, lds.stack);
    const SceneDev& sc = a.sc;
    const float* cdf = lds.lights_in_lds ? lds.cdf : a.cdf;
    const int4* lights = lds.lights_in_lds ? lds.lights : sc.lights;
    const int lane = threadIdx.x & 63;
    const int64_t npix_img = (int64_t)a.V * a.W * a.H;
    constexpr int UV = uv_rounding(GUIDE, PG, MAT);
    const int D = a.D;
    Work wk{0u, 0u, 0u, 0u, 0u};
    uint32_t npaths = 0;

    int ph = kNeedPixel;
    Trav tv;                 // traversal in progress (tracing) across iterations
    bool tracing = false;
    // work-unit state
    int64_t q = 0, wi = 0, pix = 0, unit = 0;
    int view = 0, px = 0, py = 0, s = 0, s_end = 0;
    const int64_t nunits = a.pix_count * a.nchunk;
    V3 acc = v3(0.0f, 0.0f, 0.0f);
    // path state: k = index of the vertex last processed
    uint64_t pid = 0, h = 0;
    int k = 0, klast = 0, prev_tri = -1;
    V3 T = acc, Ts = acc, L = acc, o = acc, d = acc;
    float prev_pdf = 0.0f;
    // vertex pending on a shadow ray
    V3 wl = acc, nee_LT = acc, nee_c = acc, cpart = acc;
    float rqk = 1.0f;   // roulette factor of vertex k
    float sdist = 0.0f;
    int sltri = -1;
    uint32_t ev = 0, evtail = 0, ckx = 0;
    bool nee_valid = false;
    float* dvk = nullptr;

    auto start_path = [&]() {
        pid = (uint64_t)pix * (uint64_t)a.spp + (uint64_t)s;
        float j0 = 0.5f, j1 = 0.5f;
        if (a.jitter) jitter_uniforms(a.rng, pid, j0, j1);
        camera_ray(a, view, (float)px + j0, (float)py + j1, o, d);
        k = 0;
        klast = 0;
        prev_tri = -1;
        prev_pdf = 0.0f;
        T = v3(1.0f, 1.0f, 1.0f);
        Ts = T;
        L = v3(0.0f, 0.0f, 0.0f);
        h = 0xCBF29CE484222325ull;
        if (MODE == kColor && a.dbg_vtx) {
            float* dv = a.dbg_vtx + ((size_t)wi * a.spp + s) * 8 * (size_t)(D + 1);
            for (int i = 0; i < 8 * (D + 1); ++i) dv[i] = -1.0f;
        }
        ph = kClosest;
    };

    while (true) {
        // ---- lanes without a pixel take the next pixels (one atomic per wave) ----
        uint64_t need = __ballot(ph == kNeedPixel);
        if (need) {
            int first = __ffsll((unsigned long long)need) - 1;
            unsigned base = 0;
            if (lane == first) base = atomicAdd(a.work, (unsigned)__popcll(need));
            base = __shfl(base, first);
            if (ph == kNeedPixel) {
                unsigned rank = (unsigned)__popcll(need & ((1ull << lane) - 1ull));
                unit = (int64_t)base + rank;
                if (unit >= nunits) {
                    ph = kExit;
                } else {
                    wk.units++;
                    const int c = (int)(unit / a.pix_count);
                    q = unit - (int64_t)c * a.pix_count;
                    s = c * a.spc;
                    s_end = min(a.spp, s + a.spc);
                    wi = a.pix_begin + q;
                    pix = a.pixel_list ? a.pixel_list[wi] : wi;
                    if (pix < 0 || pix >= npix_img) {
                        if (MODE == kColor) {
                            float* out = a.nchunk > 1 ? a.part + 3 * (size_t)unit : a.image + 3 * wi;
                            out[0] = 0.0f;
                            out[1] = 0.0f;
                            out[2] = 0.0f;
                        }
                    } else {
                        view = (int)(pix / ((int64_t)a.W * a.H));
                        int64_t rem = pix - (int64_t)view * a.W * a.H;
                        py = (int)(rem / a.W);
                        px = (int)(rem - (int64_t)py * a.W);
                        acc = v3(0.0f, 0.0f, 0.0f);
                        start_path();
                    }
                }
            }
        }
        if (__ballot(ph != kExit) == 0) break;

        bool end_path = false;
        bool shade = false;      // vertex k still needs light sampling and a continuation
        Shade g;
        Hit hr;
        hr.tri = -1;
        hr.t = hr.u = hr.v = 0.0f;
        size_t ck = 0;
        if (ph == kClosest || ph == kShadow) {
            // ---- one traversal call site for closest-hit and shadow rays ----
            // a lane whose traversal returned unfinished resumes it here and
            // skips the rest of the iteration until it is done
            const bool any = ph == kShadow;
            const float tmax = any ? sdist * (1.0f - 1e-5f) : __builtin_inff();
            Ray ray = make_ray(o, any ? wl : d);
            if (!tracing) {
                trav_init(tv, tmax, st, wk);
                tracing = true;
            }
            const bool done = traverse_resume(sc, ray, sc.tmin, tmax, prev_tri, any ? sltri : -1, any, st, wk, tv,
                                              IPT_TRAV_EXIT_LANES);
            if (done) tracing = false;
            hr = tv.best;
            if (!done) {
                // still traversing
            } else if (any) {
                // ---- finish the vertex that waited for its shadow ray ----
                bool vis = hr.tri < 0;
                ev |= (uint32_t)vis << 2;
                if (vis && nee_valid) {
                    cpart = cpart + nee_c;
                    L = L + nee_LT;
                    if (dvk) { dvk[4] = L.x; dvk[5] = L.y; dvk[6] = L.z; dvk[7] = 1.0f; }
                }
                h = fnv1a(h, ev | evtail);
                if (MODE == kGradFwd) {
                    ck = ck_at(a, k, s, q);
                    if (vis) a.ck_hit[ck].x = (int)(ckx | kCkVis);
                    st_stream(&a.ck_c[ck], make_float4(cpart.x, cpart.y, cpart.z, rqk));
                }
                end_path = evtail != 0;
                ph = kClosest;
            } else {
                // ---- closest hit: vertex k ----
                ++k;
                klast = k;
                wk.vertices++;
                ck = ck_at(a, k, s, q);
                if (hr.tri < 0) {
                    h = fnv1a(h, 0xFFFFFFFFu);
                    if (MODE == kGradFwd) st_stream(&a.ck_hit[ck], make_int4(0, 0, 0, 0));
                    klast = k - 1;   // a miss contributes nothing: the sweep starts below it
                    end_path = true;
                } else {
                    make_shade(sc, lds, hr, d, g);
                    h = fnv1a(h, (uint32_t)g.orig);
                    dvk = nullptr;
                    if (MODE == kColor && a.dbg_vtx) {
                        dvk = a.dbg_vtx + (((size_t)wi * a.spp + s) * (size_t)(D + 1) + (k - 1)) * 8;
                        dvk[0] = (float)g.orig; dvk[1] = hr.u; dvk[2] = hr.v; dvk[3] = hr.t;
                        dvk[4] = L.x; dvk[5] = L.y; dvk[6] = L.z; dvk[7] = 0.0f;
                    }
                    ev = 0;
                    evtail = 0;
                    cpart = v3(0.0f, 0.0f, 0.0f);
                    if (g.em >= 0 && g.cos_emit > 0.0f) {
                        float w = emit_weight(a, cdf, lights, g, k, prev_pdf);
                        if (w > 0.0f) {
                            float prof = a.profile ? g.cos_emit : 1.0f;
                            const float* e = lds.params + MatSel<MAT>::NP * sc.S + 3 * g.em;
                            V3 c = v3(e[0], e[1], e[2]) * (prof * w);
                            cpart = c;
                            L = L + T * c;
                            if (dvk) { dvk[4] = L.x; dvk[5] = L.y; dvk[6] = L.z; }
                        }
                        ev |= 1u;
                    }
                    if (k == D + 1 || dot(g.ns, g.wo) <= 0.0f) {
                        // x_{D+1} only counts its emission; a shading normal facing
                        // away ends the path
                        if (k != D + 1) ev |= 2u;
                        end_path = true;
                        h = fnv1a(h, ev);
                        prev_tri = g.tri;
                        if (MODE == kGradFwd) {
                            st_stream(&a.ck_hit[ck], make_int4(g.tri + 1, __float_as_int(hr.u),
                                                               __float_as_int(hr.v), __float_as_int(hr.t)));
                            st_stream(&a.ck_a[ck], make_float4(0.0f, 0.0f, 0.0f, 0.0f));
                            st_stream(&a.ck_c[ck], make_float4(cpart.x, cpart.y, cpart.z, 0.0f));
                        }
                    } else {
                        shade = true;
                    }
                }
            }
        }

        // ---- guide evaluation for the lanes about to sample (all lanes active here) ----
        const float* mix = nullptr;
        if (GUIDE == 3) {
            // cached row of the hit's cell, on the side the path arrives from
            if (shade) mix = cache_row_at(a.gd, g.tri, g.u, g.v, dot(g.ng, g.wo) < 0.0f);
        } else if (GUIDE) {
            float* row = (float*)(lds.gact + lane * kGRowStride);
            if (GUIDE == 1) {
                if (shade) {
                    float f[9];
                    guide_features(a.gd, g.x, g.ns, g.wo, f);
                    guide_put_inputs(a.gd, lds.gact, f, g.seg);
                }
                if (__ballot(shade)) guide_mlp_wave(a.gd, lds.gact);
            } else if (shade) {
                float f[9];
                guide_features(a.gd, g.x, g.ns, g.wo, f);
                guide_mlp_fp32(a.gd, f, g.seg, row);
            }
            if (shade) {
                mixture_from_raw(row);
                mix = row;
            }
        }

        if (shade) {
            // ---- light sample and continuation of vertex k ----
            uint32_t flags = 0;
            bool shoot = false;
            V3 av = v3(0.0f, 0.0f, 0.0f);
            rqk = 1.0f;
            mat_frame<MAT>(g);
            const typename MatSel<MAT>::M m = mat_load<MAT>(lds.params, g.seg);
            const typename MatSel<MAT>::M ms = a.frozen ? mat_load<MAT>(lds.sparams, g.seg) : m;
            float u[8];
            vertex_uniforms(a.rng, pid, k, u);
            float pb_nee = -1.0f;
            // light sample accepted: its contribution waits for the shadow ray
            auto take_nee = [&](const NeeS& n) {
                NeeC nc = nee_contrib(a, lds, cdf, g, m, ms, n, pb_nee);
                shoot = true;
                nee_valid = nc.valid;
                nee_c = nc.c;
                nee_LT = T * nc.c;
                wl = n.wl;
                sdist = n.dist;
                sltri = n.ltri;
            };
            bool used_guide = false;
            ContS cs;
            if constexpr (GUIDE == 3) {
                // cached proposal: direction first, then both densities in one pass over the row
                NeeS n;
                n.shoot = false;
                n.lj = 0;
                const bool do_nee = a.mis != 0 && sc.nlt > 0;
                if (do_nee) {
                    n = nee_setup<UV>(sc, cdf, lights, g, u);
                    ev |= (uint32_t)n.lj << 8;
                }
                const ContDir cd = cont_direction_cached(a, g, ms, u, mix);
                float q_wi, q_wl;
                cached_pdf2(mix, cd.wi, n.shoot ? n.wl : cd.wi, q_wi, q_wl);
                if (n.shoot) {
                    pb_nee = a.gmix * q_wl + (1.0f - a.gmix) * mat_pdf(ms, g, n.wl);
                    take_nee(n);
                }
                cs = cont_finish_cached(a, g, m, ms, u, k, Ts, cd, q_wi);
                used_guide = cd.guide;
            } else {
                if (a.mis != 0 && sc.nlt > 0) {
                    NeeS n = nee_setup<UV>(sc, cdf, lights, g, u);
                    ev |= (uint32_t)n.lj << 8;
                    if (n.shoot) {
                        if (GUIDE && mix)
                            pb_nee = a.gmix * guide_pdf<GUIDE>(mix, n.wl) + (1.0f - a.gmix) * mat_pdf(ms, g, n.wl);
                        take_nee(n);
                    }
                }
                cs = cont_sample<GUIDE>(a, g, m, ms, u, k, Ts, mix, used_guide);
            }
            // lobe 1 at bit 3, lobe 2 (the Disney clearcoat) at bit 7
            ev |= (uint32_t)(cs.lobe & 1) << 3 | (uint32_t)(cs.lobe >> 1) << 7;
            if (used_guide) ev |= 64u;
            if (!cs.ok) {
                evtail = 16u;
            } else if (!cs.alive) {
                evtail = 32u;
            } else {
                float rq = 1.0f / cs.qrr;
                rqk = rq;
                av = cs.av * rq;
                Ts = Ts * cs.ts * rq;
                flags |= kCkCont;
                prev_pdf = cs.pdf;
                T = T * av;
                d = cs.wi;
            }
            prev_tri = g.tri;
            o = g.x;
            if (MODE == kGradFwd) {
                ckx = (uint32_t)(g.tri + 1) | flags;
                st_stream(&a.ck_hit[ck], make_int4((int)ckx, __float_as_int(hr.u), __float_as_int(hr.v),
                                                   __float_as_int(hr.t)));
                st_stream(&a.ck_a[ck], make_float4(av.x, av.y, av.z, cs.pdf));
                if (a.guided) st_stream(&a.ck_d[ck], make_float4(cs.wi.x, cs.wi.y, cs.wi.z, pb_nee));
            }
            if (shoot) {
                ph = kShadow;   // the vertex finishes after its shadow ray
            } else {
                h = fnv1a(h, ev | evtail);
                if (MODE == kGradFwd) st_stream(&a.ck_c[ck], make_float4(cpart.x, cpart.y, cpart.z, rqk));
                end_path = evtail != 0;
            }
        }

        if (end_path) {
            ++npaths;
            size_t pidx = (size_t)wi * a.spp + s;
            bool use = a.mask ? a.mask[pidx] != 0 : true;
            if (MODE == kGradFwd) {
                const size_t c1 = ck_at(a, 1, s, q);
                if (a.guided) {
                    // the training records read R_{k+1} before the replay runs
                    V3 R = suffix_sweep(a, klast, s, q);
                    if (!finite3(R) || !finite3(L)) {
                        a.ck_hit[c1].x = (int)((uint32_t)a.ck_hit[c1].x | kCkDrop);
                        atomicAdd(&a.err->nonfinite, 1ull);
                    }
                } else if (!finite3(L)) {
                    a.ck_hit[c1].x = (int)((uint32_t)a.ck_hit[c1].x | kCkDrop);
                    atomicAdd(&a.err->nonfinite, 1ull);
                }
                // for the adjoint: the index of the path's last vertex, in the
                // fourth slot of vertex 1's c
                a.ck_c[c1].w = __int_as_float(klast);
            } else {
                if (!finite3(L)) atomicAdd(&a.err->nonfinite, 1ull);
                else if (use) acc = acc + L;
                if (a.path_L) {
                    a.path_L[3 * pidx] = L.x;
                    a.path_L[3 * pidx + 1] = L.y;
                    a.path_L[3 * pidx + 2] = L.z;
                }
            }
            if (a.hash) a.hash[pidx] = h;
            ++s;
            if (s < s_end) {
                start_path();
            } else {
                if (MODE == kColor) {
                    if (a.nchunk > 1) {   // sample sum of this unit; the reduce pass forms the mean
                        float* out = a.part + 3 * (size_t)unit;
                        out[0] = acc.x;
                        out[1] = acc.y;
                        out[2] = acc.z;
                    } else {
                        float inv = 1.0f / (float)a.spp;
                        a.image[3 * wi] = acc.x * inv;
                        a.image[3 * wi + 1] = acc.y * inv;
                        a.image[3 * wi + 2] = acc.z * inv;
                    }
                }
                ph = kNeedPixel;
            }
        }
    }
    if (st.overflow) atomicAdd(&a.err->overflow, 1ull);
    flush_stats(a, MODE, wk, npaths);
}

// ---------------------------------------------------------------------------
// Adjoint replay.  replay_kernel (one lane per pixel, tiles pulled by blocks)
// serves Lambert + GGX and the check mode that re-traces paths; replay_sm_kernel
// below the Disney model; adjoint.hip Lambert + GGX with a guide.
// ---------------------------------------------------------------------------
template <int MAT>
__device__ void replay_path(const PathArgs& a, const Lds& lds, Stack& st, Work& wk, uint64_t pid, int64_t q, int s,
                            V3 org, V3 dir, V3 wpix) {
    const SceneDev& sc = a.sc;
    const float* cdf = lds.lights_in_lds ? lds.cdf : a.cdf;
    const int4* lights = lds.lights_in_lds ? lds.lights : sc.lights;
    if ((uint32_t)a.ck_hit[ck_at(a, 1, s, q)].x & kCkDrop) return;
    // the backward sweep, here rather than at the end of each path in the
    // forward pass: every lane of the wave starts a path at once, so the
    // sweeps' round trips to memory overlap instead of holding up a wave
    // in which a few lanes end their paths
    const int klast = min(max(__float_as_int(a.ck_c[ck_at(a, 1, s, q)].w), 0), a.D + 1);
    const V3 R = suffix_sweep(a, klast, s, q);
    if (!finite3(R)) {
        atomicAdd(&a.err->nonfinite, 1ull);
        return;
    }
    V3 T = v3(1.0f, 1.0f, 1.0f), Ts = T;
    float prev_pdf = 0.0f;
    int prev_tri = -1;
    V3 o = org, d = dir;
    for (int k = 1; k <= a.D + 1; ++k) {
        size_t ck = ck_at(a, k, s, q);
        int4 rec = a.ck_hit[ck];
        uint32_t flags = (uint32_t)rec.x;
        Hit hit;
        if (!a.replay_traverse) {
            hit.tri = (int)(flags & kCkTriMask) - 1;
            hit.u = __int_as_float(rec.y);
            hit.v = __int_as_float(rec.z);
            hit.t = __int_as_float(rec.w);
        } else {
            Ray ray = make_ray(o, d);
            hit = traverse(sc, ray, sc.tmin, __builtin_inff(), prev_tri, -1, false, st, wk);
        }
        if (hit.tri < 0) return;
        wk.vertices++;
        float4 rr = a.ck_c[ck];
        V3 Rn = v3(rr.x, rr.y, rr.z);   // R_{k+1}
        Shade g;
        make_shade(sc, lds, hit, d, g);
        V3 wT = wpix * T;
        // emission at this vertex: d/de = w_hit * profile
        if (g.em >= 0 && g.cos_emit > 0.0f) {
            float w = emit_weight(a, cdf, lights, g, k, prev_pdf);
            if (w > 0.0f) {
                float prof = a.profile ? g.cos_emit : 1.0f;
                int eb = MatSel<MAT>::NP * sc.S + 3 * g.em;
                lds_add(lds.grad, eb + 0, wT.x * prof * w);
                lds_add(lds.grad, eb + 1, wT.y * prof * w);
                lds_add(lds.grad, eb + 2, wT.z * prof * w);
            }
        }
        if (k == a.D + 1 || dot(g.ns, g.wo) <= 0.0f) return;
        mat_frame<MAT>(g);
        const typename MatSel<MAT>::M m = mat_load<MAT>(lds.params, g.seg);
        const typename MatSel<MAT>::M ms = a.frozen ? mat_load<MAT>(lds.sparams, g.seg) : m;
        float u[8];
        vertex_uniforms(a.rng, pid, k, u);
        if (a.mis != 0 && sc.nlt > 0) {
            NeeS n = nee_setup(sc, cdf, lights, g, u);
            bool vis = false;
            if (n.shoot) {
                if (!a.replay_traverse) {
                    vis = (flags & kCkVis) != 0;
                } else {
                    Ray sr = make_ray(g.x, n.wl);
                    vis = traverse(sc, sr, sc.tmin, n.dist * (1.0f - 1e-5f), g.tri, n.ltri, true, st, wk).tri < 0;
                }
            }
            if (vis) {
                NeeC nc = nee_contrib(a, lds, cdf, g, m, ms, n);
                if (nc.valid) {
                    constexpr int NP = MatSel<MAT>::NP;
                    int mb = NP * g.seg, eb = NP * sc.S + 3 * n.lk;
                    V3 we = wT * nc.e * nc.g;
                    mat_grad(lds.grad, mb, m, g, n.wl, we, nc.spec, nc.dspec);
                    V3 wf = wT * nc.f * nc.g;
                    lds_add(lds.grad, eb + 0, wf.x);
                    lds_add(lds.grad, eb + 1, wf.y);
                    lds_add(lds.grad, eb + 2, wf.z);
                }
            }
        }
        if (!(flags & kCkCont)) return;
        bool ug;
        const ContS cs = cont_sample<0>(a, g, m, ms, u, k, Ts, nullptr, ug);
        float rq = 1.0f / cs.qrr;
        V3 wr = wT * Rn * (cs.g * rq);
        mat_grad(lds.grad, MatSel<MAT>::NP * g.seg, m, g, cs.wi, wr, cs.spec, cs.dspec);
        T = T * (cs.av * rq);
        Ts = Ts * cs.ts * rq;
        prev_pdf = cs.pdf;
        prev_tri = g.tri;
        o = g.x;
        d = cs.wi;
    }
}

template <int PG, int MAT>
__global__ __launch_bounds__(kBlock) void replay_kernel(PathArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned tile_sh;
    const int tid = threadIdx.x;
    Lds lds;
    carve_lds<PG>(a, kReplay, smem, lds);
    Stack st;
    init_stack(st, a, lds.stack);
    const int64_t npix_img = (int64_t)a.V * a.W * a.H;
    Work wk{0u, 0u, 0u, 0u, 0u};
    uint32_t npaths = 0;
    const int64_t nunits = a.pix_count * a.nchunk;
    while (true) {
        if (tid == 0) tile_sh = atomicAdd(a.work, 1u);
        __syncthreads();
        // every thread reads the tile before the second barrier: after it,
        // thread 0 may already be writing the next tile into tile_sh
        const int64_t tile0 = (int64_t)tile_sh * kBlock;
        __syncthreads();
        if (tile0 >= nunits) break;
        const int64_t unit = tile0 + tid;
        if (unit >= nunits) continue;
        wk.units++;
        const int c = (int)(unit / a.pix_count);
        const int64_t q = unit - (int64_t)c * a.pix_count;
        const int s_begin = c * a.spc, s_end = min(a.spp, s_begin + a.spc);
        int64_t wi = a.pix_begin + q;
        int64_t pix = a.pixel_list ? a.pixel_list[wi] : wi;
        if (pix < 0 || pix >= npix_img) continue;
        int view = (int)(pix / ((int64_t)a.W * a.H));
        int64_t rem = pix - (int64_t)view * a.W * a.H;
        int py = (int)(rem / a.W), px = (int)(rem - (int64_t)py * a.W);
        float inv = 1.0f / (float)a.spp;
        V3 wpix = v3(a.w[3 * wi] * inv, a.w[3 * wi + 1] * inv, a.w[3 * wi + 2] * inv);
        for (int s = s_begin; s < s_end; ++s) {
            uint64_t pid = (uint64_t)pix * (uint64_t)a.spp + (uint64_t)s;
            size_t pidx = (size_t)wi * a.spp + s;
            if (a.mask && a.mask[pidx] == 0) continue;
            float j0 = 0.5f, j1 = 0.5f;
            if (a.jitter) jitter_uniforms(a.rng, pid, j0, j1);
            V3 o, d;
            camera_ray(a, view, (float)px + j0, (float)py + j1, o, d);
            replay_path<MAT>(a, lds, st, wk, pid, q, s, o, d, wpix);
            ++npaths;
        }
    }
    if (st.overflow) atomicAdd(&a.err->overflow, 1ull);
    flush_stats(a, kReplay, wk, npaths);
    if constexpr (PG) return;   // the atomics went straight to the accumulator copies
    __syncthreads();
    double* out = a.grad_part + (size_t)blockIdx.x * a.P;
    for (int i = tid; i < a.P; i += kBlock) out[i] = lds.grad[i];
}

// Adjoint replay from vertex checkpoints as a per-lane state machine (the
// Disney material's replay): each pass of the loop replays one vertex of
// every lane's current path, and a lane whose path has ended takes the next
// one (the next sample of its unit, else a new unit, one atomic per wave)
// instead of idling until the longest path of the wave is done.  Same
// arithmetic, in the same order per path, as replay_path.
template <int PG, int MAT>
__global__ __launch_bounds__(kBlock) void replay_sm_kernel(PathArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    Lds lds;
    carve_lds<PG>(a, kReplay, smem, lds);
    const SceneDev& sc = a.sc;
    const float* cdf = lds.lights_in_lds ? lds.cdf : a.cdf;
    const int4* lights = lds.lights_in_lds ? lds.lights : sc.lights;
    const int64_t npix_img = (int64_t)a.V * a.W * a.H;
    const int64_t nunits = a.pix_count * a.nchunk;
    const float inv_spp = 1.0f / (float)a.spp;
    Work wk{0u, 0u, 0u, 0u, 0u};
    uint32_t npaths = 0;
    // unit of work: samples [s, s_end) of work pixel q
    bool have_unit = false, exhausted = false;
    int64_t q = 0, wi = 0, pix = 0;
    int view = 0, px = 0, py = 0, s = 0, s_end = 0;
    V3 wpix = v3(0.0f, 0.0f, 0.0f);
    // path being replayed
    bool in_path = false;
    uint64_t pid = 0;
    int k = 0;
    V3 T = wpix, Ts = wpix, d = wpix;
    float prev_pdf = 0.0f;

    while (true) {
        // ---- lanes without a path: next sample of the unit, else a new unit ----
        while (true) {
            if (!in_path && have_unit) {
                while (s < s_end && !in_path) {
                    pid = (uint64_t)pix * (uint64_t)a.spp + (uint64_t)s;
                    const size_t pidx = (size_t)wi * a.spp + s;
                    if (a.mask && a.mask[pidx] == 0) { ++s; continue; }
                    ++npaths;
                    if ((uint32_t)a.ck_hit[ck_at(a, 1, s, q)].x & kCkDrop) { ++s; continue; }
                    if (!a.guided) {
                        const int klast = min(max(__float_as_int(a.ck_c[ck_at(a, 1, s, q)].w), 0), a.D + 1);
                        const V3 R = suffix_sweep(a, klast, s, q);
                        if (!finite3(R)) {
                            atomicAdd(&a.err->nonfinite, 1ull);
                            ++s;
                            continue;
                        }
                    }
                    float j0 = 0.5f, j1 = 0.5f;
                    if (a.jitter) jitter_uniforms(a.rng, pid, j0, j1);
                    V3 o;
                    camera_ray(a, view, (float)px + j0, (float)py + j1, o, d);
                    T = v3(1.0f, 1.0f, 1.0f);
                    Ts = T;
                    prev_pdf = 0.0f;
                    k = 1;
                    in_path = true;
                }
                if (!in_path) have_unit = false;
            }
            const uint64_t need = __ballot(!in_path && !have_unit && !exhausted);
            if (!need) break;
            const int first = __ffsll((unsigned long long)need) - 1;
            unsigned base = 0;
            if (lane == first) base = atomicAdd(a.work, (unsigned)__popcll(need));
            base = __shfl(base, first);
            if (!in_path && !have_unit && !exhausted) {
                const int64_t unit = (int64_t)base + (int64_t)__popcll(need & ((1ull << lane) - 1ull));
                if (unit >= nunits) {
                    exhausted = true;
                } else {
                    wk.units++;
                    const int c = (int)(unit / a.pix_count);
                    q = unit - (int64_t)c * a.pix_count;
                    s = c * a.spc;
                    s_end = min(a.spp, s + a.spc);
                    wi = a.pix_begin + q;
                    pix = a.pixel_list ? a.pixel_list[wi] : wi;
                    if (pix >= 0 && pix < npix_img) {
                        view = (int)(pix / ((int64_t)a.W * a.H));
                        const int64_t rem = pix - (int64_t)view * a.W * a.H;
                        py = (int)(rem / a.W);
                        px = (int)(rem - (int64_t)py * a.W);
                        wpix = v3(a.w[3 * wi] * inv_spp, a.w[3 * wi + 1] * inv_spp, a.w[3 * wi + 2] * inv_spp);
                        have_unit = true;
                    }
                }
            }
        }
        if (__ballot(in_path) == 0) break;   // every lane is exhausted
        if (!in_path) continue;

        // ---- vertex k of the lane's path ----
        bool done = true;
        const size_t ck = ck_at(a, k, s, q);
        const int4 rec = a.ck_hit[ck];
        const uint32_t flags = (uint32_t)rec.x;
        Hit hit;
        hit.tri = (int)(flags & kCkTriMask) - 1;
        hit.u = __int_as_float(rec.y);
        hit.v = __int_as_float(rec.z);
        hit.t = __int_as_float(rec.w);
        if (hit.tri >= 0) {
            wk.vertices++;
            const float4 rr = a.ck_c[ck];
            const V3 Rn = v3(rr.x, rr.y, rr.z);   // R_{k+1}
            Shade g;
            make_shade(sc, lds, hit, d, g);
            const V3 wT = wpix * T;
            // emission at this vertex: d/de = w_hit * profile
            if (g.em >= 0 && g.cos_emit > 0.0f) {
                const float w = emit_weight(a, cdf, lights, g, k, prev_pdf);
                if (w > 0.0f) {
                    const float prof = a.profile ? g.cos_emit : 1.0f;
                    const int eb = MatSel<MAT>::NP * sc.S + 3 * g.em;
                    lds_add(lds.grad, eb + 0, wT.x * prof * w);
                    lds_add(lds.grad, eb + 1, wT.y * prof * w);
                    lds_add(lds.grad, eb + 2, wT.z * prof * w);
                }
            }
            if (k != a.D + 1 && dot(g.ns, g.wo) > 0.0f) {
                mat_frame<MAT>(g);
                const typename MatSel<MAT>::M m = mat_load<MAT>(lds.params, g.seg);
                const typename MatSel<MAT>::M ms = a.frozen ? mat_load<MAT>(lds.sparams, g.seg) : m;
                float u[8];
                vertex_uniforms(a.rng, pid, k, u);
                const float4 dk = a.guided ? a.ck_d[ck] : make_float4(0.0f, 0.0f, 0.0f, -1.0f);
                if (a.mis != 0 && sc.nlt > 0) {
                    const NeeS n = nee_setup(sc, cdf, lights, g, u);
                    if (n.shoot && (flags & kCkVis) != 0) {
                        // with a guide the forward pass stored the combined density of wl
                        const NeeC nc = nee_contrib(a, lds, cdf, g, m, ms, n, dk.w);
                        if (nc.valid) {
                            constexpr int NP = MatSel<MAT>::NP;
                            const int mb = NP * g.seg, eb = NP * sc.S + 3 * n.lk;
                            mat_grad(lds.grad, mb, m, g, n.wl, wT * nc.e * nc.g, nc.spec, nc.dspec);
                            const V3 wf = wT * nc.f * nc.g;
                            lds_add(lds.grad, eb + 0, wf.x);
                            lds_add(lds.grad, eb + 1, wf.y);
                            lds_add(lds.grad, eb + 2, wf.z);
                        }
                    }
                }
                if (flags & kCkCont) {
                    ContS cs;
                    if (a.guided) {
                        // the sampled direction and its density come from the checkpoint
                        cs = cont_eval(a, g, m, ms, v3(dk.x, dk.y, dk.z), a.ck_a[ck].w, 0, u, k, Ts);
                    } else {
                        bool ug;
                        cs = cont_sample<0>(a, g, m, ms, u, k, Ts, nullptr, ug);
                    }
                    const float rq = 1.0f / cs.qrr;
                    mat_grad(lds.grad, MatSel<MAT>::NP * g.seg, m, g, cs.wi, wT * Rn * (cs.g * rq), cs.spec, cs.dspec);
                    T = T * (cs.av * rq);
                    Ts = Ts * cs.ts * rq;
                    prev_pdf = cs.pdf;
                    d = cs.wi;
                    ++k;
                    done = false;
                }
            }
        }
        if (done) {
            in_path = false;
            ++s;
        }
    }
    flush_stats(a, kReplay, wk, npaths);
    if constexpr (PG) return;   // the atomics went straight to the accumulator copies
    __syncthreads();
    double* out = a.grad_part + (size_t)blockIdx.x * a.P;
    for (int i = tid; i < a.P; i += kBlock) out[i] = lds.grad[i];
}

// ---------------------------------------------------------------------------
// Guide training records from the gradient pass: after the forward pass and
// its backward sweep, vertex k of a path holds its hit, the sampled
// continuation direction w_i and density p_i, and R_{k+1}, the radiance
// arriving along w_i.  Every record_stride-th path contributes one record per
// continued vertex: (normalised position, shading normal, outgoing
// direction, segment, w_i, weight = luminance(R_{k+1}) / p_i).
//
// Bound by the reads of the vertices' records and triangles: consecutive lanes
// take consecutive pixels at one sample, as the records lie, and a block takes
// ring slots with one atomic per vertex index (consecutive samples of a pixel
// per lane and an atomic per wave: 1.58 ms of the guided room step, now 0.46).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void guide_records_kernel(PathArgs a) {
    __shared__ unsigned wave_n[4], wave_slot[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t plane = a.pix_count;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = (int)(p / plane);
    const int64_t q = p - (int64_t)s * plane;
    const int64_t wi = a.pix_begin + q;
    const int64_t gpath = wi * a.spp + s;
    bool on = p < plane * a.spp && gpath % a.grec_stride == 0 && !(a.mask && a.mask[gpath] == 0) &&
              !((uint32_t)a.ck_hit[p * a.ck_n].x & kCkDrop);
    V3 d = v3(0.0f, 0.0f, 0.0f);
    if (on) {
        const int64_t pix = a.pixel_list ? a.pixel_list[wi] : wi;
        const int64_t npix_img = (int64_t)a.V * a.W * a.H;
        on = pix >= 0 && pix < npix_img;
        if (on) {
            const int view = (int)(pix / ((int64_t)a.W * a.H));
            const int64_t rem = pix - (int64_t)view * a.W * a.H;
            const int py = (int)(rem / a.W), px = (int)(rem - (int64_t)py * a.W);
            const uint64_t pid = (uint64_t)pix * (uint64_t)a.spp + (uint64_t)s;
            float j0 = 0.5f, j1 = 0.5f;
            if (a.jitter) jitter_uniforms(a.rng, pid, j0, j1);
            V3 o;
            camera_ray(a, view, (float)px + j0, (float)py + j1, o, d);
        }
    }
    for (int k = 1; k <= a.D; ++k) {
        bool rec_on = false;
        float4 r0, r1, r2, r3;
        if (on) {
            const int64_t ck = ((int64_t)(k - 1) * a.spp * plane + p) * a.ck_n;
            const int4 rec = a.ck_hit[ck];
            const float4 dk = a.ck_d[ck];
            const float4 av = a.ck_a[ck];  // continuation factor f cos / p (and 1 / q_rr)
            const float4 R = a.ck_c[ck];   // R_{k+1} after the sweep
            const uint32_t fl = (uint32_t)rec.x;
            const int tri = (int)(fl & kCkTriMask) - 1;
            on = tri >= 0 && (fl & kCkCont);
            if (on) {
                // product target f cos L_i: its ratio to the sampling density is a_k R_{k+1}
                const float w = lum(v3(av.x * R.x, av.y * R.y, av.z * R.z));
                rec_on = w > 0.0f && isfinite(w);
                if (rec_on) {
                    V3 p0, p1, p2;
                    int orig, seg, light;
                    load_tri(a.sc, tri, p0, p1, p2, orig, seg, light);
                    float u = __int_as_float(rec.y), v = __int_as_float(rec.z);
                    V3 e1 = p1 - p0, e2 = p2 - p0;
                    V3 x = p0 + e1 * u + e2 * v;
                    V3 ng = normalize(cross(e1, e2));
                    V3 wo = v3(-d.x, -d.y, -d.z);
                    V3 ns = ng;
                    if (a.sc.nrm) {
                        float b0 = 1.0f - u - v;
                        ns = normalize(xyz(a.sc.nrm[3 * tri]) * b0 + xyz(a.sc.nrm[3 * tri + 1]) * u + xyz(a.sc.nrm[3 * tri + 2]) * v);
                    }
                    if (dot(ng, wo) < 0.0f) ns = ns * -1.0f;
                    float f[9];
                    guide_features(a.gd, x, ns, wo, f);
                    r0 = make_float4(f[0], f[1], f[2], __int_as_float(seg));
                    r1 = make_float4(f[3], f[4], f[5], w);
                    r2 = make_float4(f[6], f[7], f[8], __int_as_float((int)gpath));
                    r3 = make_float4(dk.x, dk.y, dk.z, __int_as_float(k));
                }
                d = v3(dk.x, dk.y, dk.z);
            }
        }
        const uint64_t m = __ballot(rec_on);
        if (lane == 0) wave_n[wv] = (unsigned)__popcll(m);
        if (!__syncthreads_or(on)) break;
        if (threadIdx.x == 0) {
            unsigned n = 0;
            for (int i = 0; i < 4; ++i) {
                wave_slot[i] = n;
                n += wave_n[i];
            }
            const unsigned base = n ? atomicAdd(a.grec_count, n) : 0u;
            for (int i = 0; i < 4; ++i) wave_slot[i] += base;
        }
        __syncthreads();
        if (rec_on) {
            const unsigned slot = (wave_slot[wv] + (unsigned)__popcll(m & ((1ull << lane) - 1ull))) % (unsigned)a.grec_cap;
            float4* r = (float4*)(a.grec + 16 * (size_t)slot);
            r[0] = r0;
            r[1] = r1;
            r[2] = r2;
            r[3] = r3;
        }
    }
}

hipError_t launch_guide_records(const PathArgs& a, hipStream_t st) {
    int64_t n = a.pix_count * a.spp;
    hipLaunchKernelGGL(guide_records_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <typename K>
static int occ(K kern, size_t lds) {
    int nb = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, kBlock, lds);
    return (e != hipSuccess || nb < 1) ? 1 : nb;
}

template <int MODE, int PG, int MAT>
static int path_occ(int gk, size_t lds) {
    switch (gk) {
        case 1: return occ(path_sm_kernel<MODE, 1, PG, MAT>, lds);
        case 2: return occ(path_sm_kernel<MODE, 2, PG, MAT>, lds);
        case 3: return occ(path_sm_kernel<MODE, 3, PG, MAT>, lds);
        default: return occ(path_sm_kernel<MODE, 0, PG, MAT>, lds);
    }
}

template <int MODE, int PG, int MAT>
static void launch_path_kind(int gk, const PathArgs& a, int grid, size_t lds, hipStream_t st) {
    switch (gk) {
        case 1: hipLaunchKernelGGL((path_sm_kernel<MODE, 1, PG, MAT>), dim3(grid), dim3(kBlock), lds, st, a); break;
        case 2: hipLaunchKernelGGL((path_sm_kernel<MODE, 2, PG, MAT>), dim3(grid), dim3(kBlock), lds, st, a); break;
        case 3: hipLaunchKernelGGL((path_sm_kernel<MODE, 3, PG, MAT>), dim3(grid), dim3(kBlock), lds, st, a); break;
        default: hipLaunchKernelGGL((path_sm_kernel<MODE, 0, PG, MAT>), dim3(grid), dim3(kBlock), lds, st, a); break;
    }
}

template <int MAT>
static int blocks_per_cu_mat(int mode, size_t lds, int gk, int pg) {
    if (mode == kColor) return pg ? path_occ<kColor, 1, MAT>(gk, lds) : path_occ<kColor, 0, MAT>(gk, lds);
    if (mode == kGradFwd) return pg ? path_occ<kGradFwd, 1, MAT>(gk, lds) : path_occ<kGradFwd, 0, MAT>(gk, lds);
    if constexpr (MAT == 1) return pg ? occ(replay_sm_kernel<1, MAT>, lds) : occ(replay_sm_kernel<0, MAT>, lds);
    return pg ? occ(replay_kernel<1, MAT>, lds) : occ(replay_kernel<0, MAT>, lds);
}

int path_blocks_per_cu(int mode, size_t lds, int gk, int pg, int mat) {
    return mat == 1 ? blocks_per_cu_mat<1>(mode, lds, gk, pg) : blocks_per_cu_mat<0>(mode, lds, gk, pg);
}

template <int MAT>
static void launch_paths_mat(int mode, const PathArgs& a, int grid, size_t lds, hipStream_t st) {
    const int pg = a.params_global;
    if (mode == kColor) {
        if (pg) launch_path_kind<kColor, 1, MAT>(a.guide_kind, a, grid, lds, st);
        else launch_path_kind<kColor, 0, MAT>(a.guide_kind, a, grid, lds, st);
    } else if (mode == kGradFwd) {
        if (pg) launch_path_kind<kGradFwd, 1, MAT>(a.guide_kind, a, grid, lds, st);
        else launch_path_kind<kGradFwd, 0, MAT>(a.guide_kind, a, grid, lds, st);
    } else if (a.replay_traverse || MAT == 0) {
        // the lanes of a wave replay the same sample and vertex index of
        // consecutive pixels, so their checkpoint reads coalesce: for the
        // Lambert + GGX adjoint, whose work per vertex is light, that beats
        // refilling idle lanes (apartment replay 12.9 ms here, 26.7 ms with
        // replay_sm_kernel); the Disney adjoint, ten times the arithmetic per
        // vertex, gains from the refill (27.1 -> 23.3 ms).  Also the check
        // mode that re-traces each path instead of reading its checkpoints.
        if (pg) hipLaunchKernelGGL((replay_kernel<1, MAT>), dim3(grid), dim3(kBlock), lds, st, a);
        else hipLaunchKernelGGL((replay_kernel<0, MAT>), dim3(grid), dim3(kBlock), lds, st, a);
    } else if constexpr (MAT == 1) {
        if (pg) hipLaunchKernelGGL((replay_sm_kernel<1, MAT>), dim3(grid), dim3(kBlock), lds, st, a);
        else hipLaunchKernelGGL((replay_sm_kernel<0, MAT>), dim3(grid), dim3(kBlock), lds, st, a);
    }
}

// The proposal is compiled in only when it is sampled (guide_mix > 0); kind
// as in PathArgs::guide_kind, material model as in PathArgs::mat.
hipError_t launch_paths(int mode, const PathArgs& a, int grid, size_t lds, hipStream_t st) {
    if (a.mat == 1) launch_paths_mat<1>(mode, a, grid, lds, st);
    else launch_paths_mat<0>(mode, a, grid, lds, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batch ray casting against every triangle (checks the BVH).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void brute_rays_kernel(SceneDev sc, const float* o, const float* d,
                                                            const int* skip, int64_t n, float tmin, int64_t nt,
                                                            int* out_tri, float* out_tuv) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        Ray r = make_ray(v3(o[3 * i], o[3 * i + 1], o[3 * i + 2]), v3(d[3 * i], d[3 * i + 1], d[3 * i + 2]));
        int sk = (skip && skip[i] >= 0 && skip[i] < nt) ? sc.pos_of[skip[i]] : -1;
        Hit h = brute_closest(sc, nt, r, tmin, sk);
        int orig = -1;
        if (h.tri >= 0) orig = __float_as_int(sc.tris[3 * h.tri].w);
        out_tri[i] = orig;
        out_tuv[3 * i] = h.tri >= 0 ? h.t : 0.0f;
        out_tuv[3 * i + 1] = h.u;
        out_tuv[3 * i + 2] = h.v;
    }
}

hipError_t launch_brute_rays(const SceneDev& sc, const float* o, const float* d, const int* skip, int64_t n, float tmin,
                             int64_t nt, int* out_tri, float* out_tuv, int num_cu, hipStream_t st) {
    hipLaunchKernelGGL(brute_rays_kernel, dim3(num_cu * 4), dim3(kBlock), 0, st, sc, o, d, skip, n, tmin, nt, out_tri,
                       out_tuv);
    return hipGetLastError();
}

}  // namespace ipt
