// Adjoint of a pass with a guide, Lambert + GGX (gfx950): the gradient of every path
// vertex from its records, a vertex per lane.
//
// A lane that walks a path (the replay kernels in trace.hip) idles until the
// longest path of its wave is done, and in the part of a vertex's work whose light
// sample does not count: 36-39% of the lanes of an issued VALU instruction are
// active there.  But the vertices of a path depend on each other only through the
// prefix throughput T_k, the suffix radiance R_{k+1}, the incoming direction and its
// density, and with a guide the forward pass keeps what these need: a_k (whose
// products are T), R, the directions and densities.  So a wave takes a tile of
// paths, sweeps them once (a path per lane, results in LDS), and then takes their
// vertices 64 at a time, in the order of their index, so that a pass mostly holds
// one index and its reads lie together; a tile has as many paths as fill whole
// passes.  Vertices with a light sample that counts wait in a list until there are
// 64.  No block barrier: the waves of a block share the parameters and the gradient
// sums.
//
// Measured on the guided room step, replay -> this kernel: 0.64 -> 0.41 ms.
// Elsewhere the replay stays, although this kernel took 7.3 ms where it takes 13
// (apartment; Disney model 2.0 and 5.4): without a guide it samples each direction
// again, in other last bits than the forward pass has, which narrow lobes turn into
// up to 4e-5 of the gradient, and so do the Disney model's weights here with a guide.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "path_dev.h"

namespace ipt {

namespace {

// Vertices of a tile: with more, fewer blocks fit into a CU's LDS (256: 0.43 ms;
// with many parameters 3.1 instead of 2.0); with 128, sweeps cost more (0.42).
constexpr int kEntries = 192;
constexpr int kLit = 127;                   // lit vertices: fewer than 64 wait, a pass adds at most 64
constexpr int kWaves = kBlock / 64;
constexpr int64_t kRec = 4;                 // ck_n with a guide
constexpr int kMaxChunk = 1024;             // paths that a wave takes at a time (below 2^24)
// LDS of a wave: T x, y, z, R x, y, z by vertex of the tile; the lit vertices'
// w T and (vertex index << 24 | path of the chunk); the paths by length
constexpr size_t kWaveLds = (24 * kEntries + 16 * kLit + 64 + 15) / 16 * 16;

// Order of a wave's LDS accesses (they complete in order; this holds the
// compiler to it).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Interleaved copies of a block's gradient sums, within 8 KiB of LDS: an LDS
// atomic takes 3 cycles per lane on one address, 3 / n on n copies in turn (0.42 ->
// 0.40 ms with four; with 16 KiB a block fewer fits and it is 0.43).
int sum_copies(int P) {
    int c = 1;
    while (c < 8 && sizeof(double) * P * 2 * c <= 8 << 10) c *= 2;
    return c;
}

// Direction of a path's camera ray.
__device__ __forceinline__ V3 camera_dir(const PathArgs& a, int64_t pix, uint64_t pid) {
    float jx = 0.5f, jy = 0.5f;
    if (a.jitter) jitter_uniforms(a.rng, pid, jx, jy);
    const int view = (int)(pix / ((int64_t)a.W * a.H));
    const int64_t rem = pix - (int64_t)view * a.W * a.H;
    const int py = (int)(rem / a.W), px = (int)(rem - (int64_t)py * a.W);
    V3 o, d;
    camera_ray(a, view, (float)px + jx, (float)py + jy, o, d);
    return d;
}
__device__ __forceinline__ Hit hit_of(int4 rec) {
    Hit h;
    h.tri = (int)((uint32_t)rec.x & kCkTriMask) - 1;
    h.u = __int_as_float(rec.y);
    h.v = __int_as_float(rec.z);
    h.t = __int_as_float(rec.w);
    return h;
}

template <int PG>
__global__ __launch_bounds__(kBlock) void adjoint_kernel(PathArgs a, int chunk, int copies) {   // chunk: paths per chunk
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int MAT = 0, NP = MatSel<MAT>::NP;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Lds lds;
    carve_lds<PG>(a, kColor, smem, lds);
    double* sums = (double*)((unsigned char*)lds.stack + kWaves * kWaveLds);
    GradCopies grad{sums + lane % copies, copies};
    if constexpr (PG) {
        grad = {a.grad_part + (size_t)(blockIdx.x % a.grad_copies) * a.P, 1};
    } else {
        for (int i = threadIdx.x; i < a.P * copies; i += kBlock) sums[i] = 0.0;
        __syncthreads();
    }
    unsigned char* mine = (unsigned char*)lds.stack + w * kWaveLds;
    float* ent = (float*)mine;
    float* lit = ent + 6 * kEntries;
    unsigned char* order = (unsigned char*)(lit + 4 * kLit);
    const SceneDev& sc = a.sc;
    const float* cdf = lds.lights_in_lds ? lds.cdf : a.cdf;
    const int4* lights = lds.lights_in_lds ? lds.lights : sc.lights;
    const int64_t plane = a.pix_count, npix_img = (int64_t)a.V * a.W * a.H;
    const int64_t stride = plane * a.spp;   // paths; records from a vertex to the next of its path
    const int levels = a.D + 1;
    const float inv_spp = 1.0f / (float)a.spp;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t npaths = 0, nvert = 0;

    const int64_t nchunks = (stride + chunk - 1) / chunk;
    for (int64_t ci = (int64_t)blockIdx.x * kWaves + w; ci < nchunks; ci += (int64_t)gridDim.x * kWaves) {
        const int64_t p0 = ci * chunk;
        const int len = (int)min((int64_t)chunk, stride - p0);
        const int s0 = (int)(p0 / plane);
        const int64_t q0 = p0 - (int64_t)s0 * plane;
        // path i of the chunk: sample, pixel
        struct Id {
            int s;
            int64_t wi, pix;
            uint64_t pid;
        };
        auto path_of = [&](int i) {
            Id d;
            d.s = s0;
            int64_t q = q0 + i;
            if (q >= plane) {
                if (plane >= 1 << 24) {   // i < 2^24: the next sample
                    ++d.s;
                    q -= plane;
                } else {
                    const uint32_t r = (uint32_t)q / (uint32_t)plane;
                    d.s += (int)r;
                    q -= (int64_t)r * plane;
                }
            }
            d.wi = a.pix_begin + q;
            d.pix = a.pixel_list ? a.pixel_list[d.wi] : d.wi;
            d.pid = (uint64_t)d.pix * (uint64_t)a.spp + (uint64_t)d.s;
            return d;
        };
        int nlit = 0;
        for (int at = 0; at < len;) {
            // ---- paths of the tile, one per lane, and their lengths ----
            int n = 0;
            bool counted = false;
            if (at + lane < len) {
                const Id id = path_of(at + lane);
                if (id.pix >= 0 && id.pix < npix_img && !(a.mask && a.mask[(size_t)id.wi * a.spp + id.s] == 0)) {
                    counted = true;
                    const int64_t p = p0 + at + lane;
                    const uint32_t f1 = (uint32_t)a.ck_hit[kRec * p].x;
                    n = min(max(__float_as_int(a.ck_c[kRec * p].w), 0), levels);
                    if (f1 & kCkDrop) n = 0;
                }
            }
            int upto = n;
            for (int o = 1; o < 64; o <<= 1) {
                const int x = __shfl_up(upto, o, 64);
                if (lane >= o) upto += x;
            }
            // as many paths as fill passes of 64 vertices, or the rest of the chunk
            const int all = __builtin_amdgcn_readlane(upto, 63);
            const int fit = min(all, kEntries);
            const int most = fit < 64 || (all <= kEntries && at + 64 >= len) ? fit : fit & ~63;
            const bool taken = upto <= most;
            const int ntaken = __popcll(__ballot(taken));
            if (!taken) n = 0;
            npaths += counted && taken ? 1u : 0u;
            // ---- longest paths first; off: vertices before vertex index lane + 1 ----
            int sum = 0, cnt = 0, rank = 0;
            for (int k = levels; k >= 1; --k) {
                const uint64_t m = __ballot(n == k);
                if (n == k) rank = sum + __popcll(m & below);
                sum += __popcll(m);
                if (lane == k - 1) cnt = sum;
            }
            if (n > 0) order[rank] = (unsigned char)lane;
            int off = cnt;
            for (int o = 1; o < 32; o <<= 1) {
                const int x = __shfl_up(off, o, 64);
                if (lane >= o) off += x;
            }
            const int nv = __builtin_amdgcn_readlane(off, levels - 1);
            off -= cnt;
            nvert += lane == 0 ? (uint32_t)nv : 0u;
            // ---- T and R of the vertices ----
            {
                const int64_t p = p0 + at + lane;
                // four vertices' loads at a time: one after the other their
                // latencies were most of a tile's time
                for (int k4 = levels; k4 >= 1; k4 -= 4) {
                    float4 av[4], R[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int k = k4 - i;
                        if (k >= 1 && n >= k) {
                            av[i] = a.ck_a[kRec * (p + (int64_t)(k - 1) * stride)];
                            R[i] = a.ck_c[kRec * (p + (int64_t)(k - 1) * stride)];   // R_{k+1}
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int k = k4 - i;
                        const int ok = __builtin_amdgcn_readlane(off, max(k, 1) - 1);
                        if (k >= 1 && n >= k) {
                            float* e = ent + ok + rank;
                            e[0] = av[i].x;
                            e[kEntries] = av[i].y;
                            e[2 * kEntries] = av[i].z;
                            e[3 * kEntries] = R[i].x;
                            e[4 * kEntries] = R[i].y;
                            e[5 * kEntries] = R[i].z;
                        }
                    }
                }
            }
            {
                V3 T = v3(1.0f, 1.0f, 1.0f);
                for (int k = 1; k <= levels; ++k) {
                    const int ok = __builtin_amdgcn_readlane(off, k - 1);
                    if (n >= k) {
                        float* e = ent + ok + rank;
                        const V3 av1 = v3(e[0], e[kEntries], e[2 * kEntries]);
                        e[0] = T.x;
                        e[kEntries] = T.y;
                        e[2 * kEntries] = T.z;
                        T = T * av1;
                    }
                }
            }
            wave_sync();

            const int base = at;
            at += ntaken;
            for (int j0 = 0; j0 < nv || (at >= len && nlit > 0);) {
                if (j0 < nv) {
                    // ---- a vertex per lane: emission and continuation ----
                    const int j = j0 + lane;
                    int k = 1, o = 0;
                    for (int l = 1; l < levels; ++l) {
                        const int ol = __builtin_amdgcn_readlane(off, l);
                        if (j >= ol) { k = l + 1; o = ol; }
                    }
                    j0 += 64;
                    bool is_lit = false;
                    V3 wT = v3(0.0f, 0.0f, 0.0f);
                    int i = 0;
                    const int src = j < nv ? order[j - o] : 0;
                    if (j < nv) {
                        i = base + src;
                        const Id id = path_of(i);
                        // everything that the vertex may need, at once: the branches
                        // below would each wait for a load of their own
                        const int64_t ck = kRec * (p0 + i + (int64_t)(k - 1) * stride), before = k > 1 ? ck - kRec * stride : ck;
                        const int4 rec = a.ck_hit[ck];
                        const float4 din = a.ck_d[before], dk = a.ck_d[ck];
                        const float pdf_in = a.ck_a[before].w;
                        const float* wp = a.w + 3 * id.wi;
                        const V3 wpix = v3(wp[0] * inv_spp, wp[1] * inv_spp, wp[2] * inv_spp);
                        const uint32_t flags = (uint32_t)rec.x;
                        const Hit hit = hit_of(rec);
                        if (hit.tri >= 0) {
                            const V3 d = k > 1 ? xyz(din) : camera_dir(a, id.pix, id.pid);
                            const float* e = ent + j;
                            const V3 T = v3(e[0], e[kEntries], e[2 * kEntries]);
                            wT = wpix * T;
                            is_lit = (flags & kCkVis) != 0;
                            Shade g;
                            make_shade(sc, lds, hit, d, g);
                            // emission at this vertex: d/de = w_hit * profile
                            if (g.em >= 0 && g.cos_emit > 0.0f) {
                                const float we = emit_weight(a, cdf, lights, g, k, pdf_in);
                                if (we > 0.0f) {
                                    const float prof = a.profile ? g.cos_emit : 1.0f;
                                    const int eb = NP * sc.S + 3 * g.em;
                                    lds_add(grad, eb + 0, wT.x * prof * we);
                                    lds_add(grad, eb + 1, wT.y * prof * we);
                                    lds_add(grad, eb + 2, wT.z * prof * we);
                                }
                            }
                            if (flags & kCkCont) {
                                // the sampled direction, its density and the roulette's
                                // factor come from the records
                                mat_frame<MAT>(g);
                                const typename MatSel<MAT>::M m = mat_load<MAT>(lds.params, g.seg);
                                const V3 out = xyz(dk);
                                const V3 Rn = v3(e[3 * kEntries], e[4 * kEntries], e[5 * kEntries]);   // R_{k+1}
                                float rq = k > 1 ? a.ck_c[ck].w : 1.0f, spec = 0.0f, dspec = 0.0f;
                                const V3 f = mat_f(m, g, out, spec, dspec);
                                const float cg = dot(g.ns, out) / a.ck_a[ck].w;
                                if (k == 1 && a.rr_depth >= 0 && a.rr_depth <= 1) {
                                    // the slot of vertex 1 holds the path's length; its roulette sees one weight
                                    V3 fs = f;
                                    if (a.frozen) fs = mat_f_only(mat_load<MAT>(lds.sparams, g.seg), g, out);
                                    rq = 1.0f / fminf(fmaxf(maxc(fs * cg), 0.1f), 0.95f);
                                }
                                mat_grad(grad, NP * g.seg, m, g, out, wT * Rn * (cg * rq), spec, dspec);
                            }
                        }
                    }
                    const uint64_t ml = __ballot(is_lit);
                    if (is_lit) {
                        float* r = lit + nlit + __popcll(ml & below);
                        r[0] = wT.x;
                        r[kLit] = wT.y;
                        r[2 * kLit] = wT.z;
                        r[3 * kLit] = __int_as_float(k << 24 | i);
                    }
                    nlit += __popcll(ml);
                    wave_sync();
                }
                // ---- a lit vertex per lane: the light sample ----
                if (nlit >= 64 || (at >= len && j0 >= nv && nlit > 0)) {
                    const int m0 = max(nlit - 64, 0);
                    if (m0 + lane < nlit) {
                        const float* r = lit + m0 + lane;
                        const V3 wT = v3(r[0], r[kLit], r[2 * kLit]);
                        const int ki = __float_as_int(r[3 * kLit]), k = ki >> 24, i = ki & 0xFFFFFF;
                        const Id id = path_of(i);
                        const int64_t ck = kRec * (p0 + i + (int64_t)(k - 1) * stride);
                        const float4 din = a.ck_d[k > 1 ? ck - kRec * stride : ck];
                        const Hit hit = hit_of(a.ck_hit[ck]);
                        const float pb = a.ck_d[ck].w;   // the combined density of wl
                        Shade g;
                        make_shade(sc, lds, hit, k > 1 ? xyz(din) : camera_dir(a, id.pix, id.pid), g);
                        mat_frame<MAT>(g);
                        const typename MatSel<MAT>::M m = mat_load<MAT>(lds.params, g.seg);
                        const typename MatSel<MAT>::M ms = a.frozen ? mat_load<MAT>(lds.sparams, g.seg) : m;
                        float u[8];
                        vertex_uniforms(a.rng, id.pid, k, u);
                        const NeeS ns = nee_setup(sc, cdf, lights, g, u);
                        if (ns.shoot) {
                            const NeeC nc = nee_contrib(a, lds, cdf, g, m, ms, ns, pb);
                            if (nc.valid) {
                                const int eb = NP * sc.S + 3 * ns.lk;
                                mat_grad(grad, NP * g.seg, m, g, ns.wl, wT * nc.e * nc.g, nc.spec, nc.dspec);
                                const V3 wf = wT * nc.f * nc.g;
                                lds_add(grad, eb + 0, wf.x);
                                lds_add(grad, eb + 1, wf.y);
                                lds_add(grad, eb + 2, wf.z);
                            }
                        }
                    }
                    nlit = m0;
                    wave_sync();
                }
            }
        }
    }
    if (a.count_stats) {
        KStats* ks = &a.err->k[kReplay];
        count_add(&ks->paths, npaths);
        count_add(&ks->vertices, nvert);
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&ks->units, (unsigned long long)(plane * a.nchunk));
    }
    if constexpr (PG) return;   // the atomics went straight to the accumulator copies
    __syncthreads();
    double* out = a.grad_part + (size_t)blockIdx.x * a.P;
    for (int i = threadIdx.x; i < a.P; i += kBlock) {
        double x = 0.0;
        for (int c = 0; c < copies; ++c) x += sums[i * copies + c];
        out[i] = x;
    }
}

template <class K>
hipError_t launch(K kern, const PathArgs& a, int max_blocks, int num_cu, size_t lds, int* grid, hipStream_t st) {
    int per_cu = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kBlock, lds);
    if (e != hipSuccess) return e;
    const int most = std::min(max_blocks, num_cu * std::max(1, per_cu));
    // chunks for several rounds of the resident waves; few paths take small
    // chunks, so that every wave has one
    const int64_t paths = a.pix_count * a.spp, share = (paths + most * kWaves - 1) / (most * kWaves);
    const int chunk = (int)std::max<int64_t>(8, std::min<int64_t>(kMaxChunk, share > 256 ? share / 4 : share));
    const int64_t chunks = (paths + chunk - 1) / chunk;
    *grid = (int)std::min<int64_t>(most, (chunks + kWaves - 1) / kWaves);
    hipLaunchKernelGGL(kern, dim3(*grid), dim3(kBlock), lds, st, a, chunk, a.params_global ? 1 : sum_copies(a.P));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint(const PathArgs& a, int max_blocks, int num_cu, int* grid, hipStream_t st) {
    const size_t lds = path_lds_bytes(kColor, a.P, a.frozen, a.sc.S, a.sc.nlt, 0, a.params_global) -
                       sizeof(int) * kShortStack * kBlock + kWaves * kWaveLds +
                       (a.params_global ? 0 : sizeof(double) * a.P * sum_copies(a.P));
    return a.params_global ? launch(adjoint_kernel<1>, a, max_blocks, num_cu, lds, grid, st)
                           : launch(adjoint_kernel<0>, a, max_blocks, num_cu, lds, grid, st);
}

}  // namespace ipt
