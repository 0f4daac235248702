// Ray streams: persistent waves trace a list of rays (closest hits and
// occlusion tests); a lane whose ray has finished takes the next one.  The
// same boxes, triangles and tie rule as the traversal of path_dev.h, so the
// same hits; only the order of visits can differ (children at equal distance).
//
// Bound by VALU issue with 4-cycle min/max, select and byte-permute instructions
// (fma, add, mul and bit operations take 2), then by the address unit and the
// latency of the node loads.  Rays of the apartment's path passes: VALU busy in
// 87-89% of the cycles, 59-60% of the lanes active, 0.81 accesses per clock and CU.
// A batch of 4.9 M camera rays: 75-82% and 52% (41% before), 63 instead of 89 wave
// instructions per ray, 5.0 -> 7.7 G rays/s.
#pragma once
#include "path_dev.h"

namespace ipt {

// The node phase ends once no more than this many lanes, or a quarter of those
// with a ray, are still looking for their first leaf (and some lane holds one).
// The quarter matters for waves that are running empty: passes of 4096 to 65536
// paths take 3-16% less with it (room, 4096: 366 -> 325 us).  Apartment step 98.1 / 96.8 / 96.0
// / 95.9 ms at 8 / 12 / 16 / 20, room 9.67 / 9.58 / 9.59 / 9.63 ms.
constexpr int kRayBreak = 16;
// Finished lanes take new rays once this many have finished: the refill costs
// about two node visits whoever takes part.  Apartment step 98.7 / 96.8 / 95.8
// ms at 16 / 24 / 32.
constexpr int kRayRefill = 32;
// Chunks of rays a wave takes one after the other, about: fewer leave waves idle
// at the end of a launch (apartment step 104.0 ms at 4, 102.5 at 8), more cost
// atomics on the groups' counters (103.2 at 16, 103.6 at 32).
constexpr int kRayChunks = 8;
// Few rays are spread over all waves, at least this many to a wave: a wave lasts as
// long as the phases of its lanes together.  Steps of 4096 / 16384 / 65536 paths of the
// apartment, depth 7: 1.02 / 1.21 / 1.32 ms with 64 rays to a wave, 1.00 / 1.15 / 1.28
// with 32, 0.94 / 1.08 / 1.27 with 8.
constexpr unsigned kRayFew = 8;
// Traversal stack: entries in LDS (24 KB per block, 5 blocks per CU), the rest
// in global memory; as many in all as the state machine's stack, which the
// scene build checks the tree against, and one for the bottom.
constexpr int kRayStack = 24;
constexpr int kRayOvf = kShortStack + kOvfDepth + 1 - kRayStack;
// Blocks per CU.  5 waves per SIMD hold the kernel's 95 VGPRs; a sixth spills 13
// of them (apartment step 105.1 against 103.2 ms).
constexpr int kRayBlocksPerCu = 5;

// A comparator of the sorting network on (entry distance, child reference) as
// one 64-bit word: read as a double it orders by the distance (which is
// positive or at least no NaN; its sign and exponent are the double's), so two
// full-rate instructions move both halves, where a compare and four selects
// moved them before.  The visit: 131 -> 108 VALU instructions.
__device__ __forceinline__ void cas64(double& a, double& b) {
    double lo, hi;
    __asm__("v_min_f64 %0, %2, %3\n\tv_max_f64 %1, %2, %3" : "=&v"(lo), "=&v"(hi) : "v"(a), "v"(b));
    a = lo;
    b = hi;
}
__device__ __forceinline__ double key64(float t, int c) {
    return __builtin_bit_cast(double, (uint64_t)__float_as_uint(t) << 32 | (uint32_t)c);
}
__device__ __forceinline__ float key_t(double k) { return __uint_as_float((uint32_t)(__builtin_bit_cast(uint64_t, k) >> 32)); }
// min and max without the canonicalisation of each operand that fminf and
// fmaxf bring (no operand here is a signalling NaN).
__device__ __forceinline__ float min_f(float a, float b) {
    float r;
    __asm__("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max_f(float a, float b) {
    float r;
    __asm__("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float min3_f(float a, float b, float c) {
    float r;
    __asm__("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float max3_f(float a, float b, float c) {
    float r;
    __asm__("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ int key_c(double k) { return (int)(uint32_t)__builtin_bit_cast(uint64_t, k); }

// tri_isect on a triangle stored by axis: X, Y, Z hold the three vertices'
// coordinates along the ray's kx, ky, kz, so no component has to be picked by
// selects (18 of about 95 VALU instructions).  Same operations in the same
// order, the fused ones spelled out.
__device__ __forceinline__ bool tri_isect_axes(float ox, float oy, float oz, float Sx, float Sy, float Sz, float4 X,
                                               float4 Y, float4 Z, float tmin, float& t, float& u, float& v) {
    const float Akz = Z.x - oz, Bkz = Z.y - oz, Ckz = Z.z - oz;
    const float Ax = fmaf(-Sx, Akz, X.x - ox), Ay = fmaf(-Sy, Akz, Y.x - oy);
    const float Bx = fmaf(-Sx, Bkz, X.y - ox), By = fmaf(-Sy, Bkz, Y.y - oy);
    const float Cx = fmaf(-Sx, Ckz, X.z - ox), Cy = fmaf(-Sy, Ckz, Y.z - oy);
    float U = fmaf(Cx, By, -(Cy * Bx));
    float V = fmaf(Ax, Cy, -(Ay * Cx));
    float W = fmaf(Bx, Ay, -(By * Ax));
    if (U == 0.0f || V == 0.0f || W == 0.0f) {
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    const float det = U + V + W;
    if (det == 0.0f) return false;
    const float T = fmaf(W, Sz * Ckz, fmaf(V, Sz * Bkz, U * (Sz * Akz)));
    const float rdet = 1.0f / det;
    t = T * rdet;
    if (!(t > tmin)) return false;
    u = V * rdet;
    v = W * rdet;
    return true;
}

// Traces rays [0, n) of a source: src.load(i, o, d, tmax, skip0, skip1, any)
// fetches a ray (any: stop at the first hit below tmax; skip0 and skip1 are
// leaf triangles to ignore), src.store(i, any, hit) takes its result.
// nwaves waves run it, this one as number `wave`; each takes chunks of
// consecutive rays: the next one of the counter `work` (zero at the start).
template <class SRC>
__device__ __forceinline__ void trace_stream(const SceneDev& sc, float tmin, const SRC& src, unsigned n, int* lds_stack,
                                             int* ovf, unsigned wave, unsigned nwaves, unsigned* work, Counters* err,
                                             KStats* stats) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int gtid = blockIdx.x * kBlock + tid, gthreads = gridDim.x * kBlock;
    // about kRayChunks per wave, of 64 to 512 rays; few rays over all waves
    const unsigned chunk = n < 64u * nwaves ? max(kRayFew, (n + nwaves - 1) / nwaves)
                                            : min(512u, max(64u, (n / (kRayChunks * nwaves)) & ~63u));
    const unsigned nchunks = (n + chunk - 1) / chunk;
    unsigned at = wave;                    // the wave's chunk
    auto next_chunk = [&]() {
        if (nchunks <= nwaves) {
            at = nchunks;
            return;
        }
        unsigned c = 0;
        if (lane == 0) c = atomicAdd(work, 1u);
        at = __builtin_amdgcn_readfirstlane(c) + nwaves;
    };
    unsigned base = at < nchunks ? at * chunk : n;         // next ray
    unsigned end = n - base > chunk ? base + chunk : n;
    bool more = base < n;
    bool overflow = false;
    uint32_t nrays = 0, nnodes = 0, ntris = 0;
    bool active = false;
    Ray r{};
    float ox = 0.0f, oy = 0.0f, oz = 0.0f;   // origin in the triangle test's axes
    float tmax = 0.0f;
    int skip0 = -1, skip1 = -1;
    bool any = false;
    int cur = kTravDone, pend = kTravDone, best_orig = 0x7FFFFFFF, sp = 0;
    Hit best{-1, 0.0f, 0.0f, 0.0f};
    unsigned tag = 0;
    // stack entry e of the lane is at byte (e kBlock + tid) 4 of the LDS window;
    // sp is the byte of the next free one
    constexpr int kEntry = kBlock * (int)sizeof(int), kWindow = kRayStack * kEntry;
    auto slot = [&](int at) -> int& { return *(int*)((char*)lds_stack + at); };
    auto spill = [&](int at) -> int& { return ovf[(size_t)((at - kWindow) / kEntry) * gthreads + gtid]; };
    auto push = [&](int x) {
        if (sp < kWindow) slot(sp) = x;
        else if (sp < kWindow + kRayOvf * kEntry) spill(sp) = x;
        else { overflow = true; return; }
        sp += kEntry;
    };
    auto pop = [&]() -> int {
        sp -= kEntry;
        return sp < kWindow ? slot(sp) : spill(sp);
    };
    while (true) {
        const uint64_t live = __builtin_amdgcn_ballot_w64(cur != kTravDone);
        if (__popcll(live) <= 64 - kRayRefill && (more || !live)) {
            // finished lanes store their hits and take the next rays
            if (cur == kTravDone) {
                if (active) {
                    if (!any && best.tri >= 0 && !(best.t < tmax)) best.tri = -1;
                    src.store(tag, any, best);
                    active = false;
                }
                const uint64_t idle = ~live;
                const int rank = __popcll(idle & ((1ull << lane) - 1ull));
                const unsigned i = base + rank;
                if (more && i < end) {
                    V3 o, d;
                    src.load(i, o, d, tmax, skip0, skip1, any);
                    r = make_ray(o, d);
                    ox = comp(o, r.kx);
                    oy = comp(o, r.ky);
                    oz = comp(o, r.kz);
                    tag = i;
                    active = true;
                    cur = 0;
                    pend = kTravDone;
                    best = Hit{-1, tmax, 0.0f, 0.0f};
                    best_orig = 0x7FFFFFFF;
                    slot(tid * 4) = kTravDone;   // bottom of the stack
                    sp = tid * 4 + kEntry;
                    ++nrays;
                }
            }
            base += (64 - __popcll(live));
            if (more && base >= end) {
                next_chunk();
                base = at < nchunks ? at * chunk : n;
                end = n - base > chunk ? base + chunk : n;
                more = base < n;
            }
            if (__builtin_amdgcn_ballot_w64(cur != kTravDone) == 0) {
                if (!more) break;
                continue;
            }
        }
        // ---- node phase ----
        const int few = min(kRayBreak, __popcll(__builtin_amdgcn_ballot_w64(cur != kTravDone)) >> 2);
        while (true) {
            if (cur < 0 && cur != kTravDone && pend == kTravDone) {
                pend = cur;
                cur = pop();
            }
            const bool inner = cur >= 0;
            const uint64_t searching = __builtin_amdgcn_ballot_w64(inner && pend == kTravDone);
            if (!searching) break;
            if (__popcll(searching) <= few && __builtin_amdgcn_ballot_w64(pend != kTravDone) != 0) break;
            if (inner) {
                ++nnodes;
                const float inf = __builtin_inff();
                const float4* nd = sc.nodes + 4 * (size_t)(uint32_t)cur;
                const float4 h = nd[0], qa = nd[1], qb = nd[2], cr = nd[3];
                int c[4] = {__float_as_int(cr.x), __float_as_int(cr.y), __float_as_int(cr.z), __float_as_int(cr.w)};
                __asm__ volatile("" ::"v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]));
                // the cells' sizes, 2^(e + 24), as the upper halves of floats
                const uint32_t exy = __float_as_uint(qb.z);
                const V3 A = v3(r.inv.x * __uint_as_float(exy & 0xffff0000u), r.inv.y * __uint_as_float(exy << 16),
                                r.inv.z * qb.w);
                const V3 B = v3((h.x - r.o.x) * r.inv.x, (h.y - r.o.y) * r.inv.y, (h.z - r.o.z) * r.inv.z);
                const uint32_t xl = __float_as_uint(qa.x), xh = __float_as_uint(qa.y);
                const uint32_t yl = __float_as_uint(qa.z), yh = __float_as_uint(qa.w);
                const uint32_t zl = __float_as_uint(qb.x), zh = __float_as_uint(qb.y);
                // near plane of a positive direction: bytes of the low row (0..3 of the pair); far: the high row (4..7)
                const uint32_t sx = r.inv.x < 0.0f ? 0x0c060c04u : 0x0c020c00u, sy = r.inv.y < 0.0f ? 0x0c060c04u : 0x0c020c00u,
                               sz = r.inv.z < 0.0f ? 0x0c060c04u : 0x0c020c00u;
                const float tmx = best.t + sc.tmin;
                auto pk = [](uint32_t hi, uint32_t lo, uint32_t s) { return __builtin_bit_cast(h2x, __builtin_amdgcn_perm(hi, lo, s)); };
                const uint32_t f = 0x00040004u, o1 = 0x00010001u;
                const h2x e02[6] = {pk(xh, xl, sx), pk(xh, xl, sx ^ f), pk(yh, yl, sy), pk(yh, yl, sy ^ f), pk(zh, zl, sz), pk(zh, zl, sz ^ f)};
                const h2x e13[6] = {pk(xh, xl, sx | o1), pk(xh, xl, (sx ^ f) | o1), pk(yh, yl, sy | o1), pk(yh, yl, (sy ^ f) | o1), pk(zh, zl, sz | o1), pk(zh, zl, (sz ^ f) | o1)};
                double k[4];
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
                    const float tn = max_f(max3_f(nx, ny, nz), tmin);
                    const float tf = min_f(min3_f(fx, fy, fz), tmx);
                    k[i] = key64(tn <= tf * 1.0000005f ? tn : inf, c[i]);
                }
                cas64(k[0], k[1]); cas64(k[2], k[3]); cas64(k[0], k[2]); cas64(k[1], k[3]); cas64(k[1], k[2]);
                if (sp < kWindow - 2 * kEntry) {
                    // farthest first
                    if (key_t(k[3]) < inf) { slot(sp) = key_c(k[3]); sp += kEntry; }
                    if (key_t(k[2]) < inf) { slot(sp) = key_c(k[2]); sp += kEntry; }
                    if (key_t(k[1]) < inf) { slot(sp) = key_c(k[1]); sp += kEntry; }
                } else {
                    if (key_t(k[3]) < inf) push(key_c(k[3]));
                    if (key_t(k[2]) < inf) push(key_c(k[2]));
                    if (key_t(k[1]) < inf) push(key_c(k[1]));
                }
                cur = key_t(k[0]) < inf ? key_c(k[0]) : pop();
            }
        }
        // ---- leaf phase ----
        // one triangle per pass for every lane that holds one; the wave leaves
        // when none does
        while (__builtin_amdgcn_ballot_w64(pend != kTravDone)) {
            if (pend != kTravDone) {
                const int code = ~pend;
                const int i = code >> 3;
                pend = (code & 7) ? ~(code + 7) : kTravDone;   // first + 1, count - 1
                ++ntris;
                if (i != skip0 && i != skip1) {
                    const float4* row = sc.tri_axis + 3 * (size_t)(uint32_t)i;
                    const float4 X = row[r.kx], Y = row[r.ky], Z = row[r.kz];
                    float t, u, v;
                    if (tri_isect_axes(ox, oy, oz, r.Sx, r.Sy, r.Sz, X, Y, Z, tmin, t, u, v)) {
                        const int orig = __float_as_int(X.w);
                        if (any) {
                            if (t < tmax) {
                                best.tri = i; best.t = t;
                                cur = kTravDone;
                                pend = kTravDone;
                            }
                        } else if (t < best.t || (t == best.t && orig < best_orig)) {
                            best.tri = i; best.t = t; best.u = u; best.v = v;
                            best_orig = orig;
                        }
                    }
                }
            }
        }
    }
    if (overflow) atomicAdd(&err->overflow, 1ull);
    if (stats) {
        count_add(&stats->rays, nrays);
        count_add(&stats->nodes, nnodes);
        count_add(&stats->tris, ntris);
    }
}

}  // namespace ipt
