// Quantization of a four-child node, shared by the host (bvh_wide.cpp) and the
// device (bvh_gpu.hip).
//
// Quantized nodes (after Ylitie, Karras and Laine 2017, "Efficient incoherent
// ray traversal on GPUs through compressed wide BVHs"): the four child boxes
// as 8-bit grid coordinates relative to a per-node origin, with a
// power-of-two cell size per axis.  Layout per node, 16 floats = 64 B:
//   row 0: origin x, y, z (float); biased exponents e_x, e_y, e_z (bytes 0-2)
//   row 1: x lo, x hi, y lo, y hi of the four children (one byte per child)
//   row 2: z lo, z hi; the cell sizes 2^(e + 24) of x and y (the upper 16 bits
//          of a float each, y's in the low half) and of z (float).  They are normal
//          floats: e >= -126, and e <= 34 since the scene build refuses coordinates
//          beyond 1e12
//   row 3: the four child references (as the float layout)
// A plane decodes to origin + q 2^e.  Every decoded box contains its child's
// float box widened by delta = 2^-20 of the node's largest extent on every
// side: that margin covers the rounding of the traversal's
// fma(q, 2^e / d, (origin - o) / d) for ray origins within or near the node,
// and the slab test's relative slack covers origins far from it.  An empty
// slot has q lo = 255, q hi = 0 (a box inside out, which the slab test
// rejects unless the ray starts some 10^6 node extents away) and, as its
// reference, the leaf code of the one-triangle leaf holding triangle 0
// (~0): should the slack ever admit the slot, the traversal tests a real
// triangle once more, which changes no hit, instead of following an
// invalid reference.  The traversal then needs no reference check.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

#ifdef __HIPCC__
#define IPT_HD __host__ __device__
#else
#define IPT_HD
#endif

namespace ipt {

constexpr int kQuantNone = 0x7FFFFFFF;   // empty child slot of the float layout

IPT_HD inline int quant_bits_i(float f) { int i; std::memcpy(&i, &f, sizeof i); return i; }
IPT_HD inline float quant_bits_f(int i) { float f; std::memcpy(&f, &i, sizeof f); return f; }

// o: the float node (32 floats), d: the quantized one (16 floats).
IPT_HD inline void quantize_node(const float* o, float* d) {
    float lo[3][4], hi[3][4];
    for (int a = 0; a < 3; ++a)
        for (int j = 0; j < 4; ++j) {
            lo[a][j] = o[4 * (2 * a) + j];
            hi[a][j] = o[4 * (2 * a + 1) + j];
        }
    const int ref[4] = {quant_bits_i(o[24]), quant_bits_i(o[25]), quant_bits_i(o[26]), quant_bits_i(o[27])};
    bool valid[4];
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int j = 0; j < 4; ++j) {
        valid[j] = ref[j] != kQuantNone;
        if (!valid[j]) continue;
        for (int a = 0; a < 3; ++a) {
            mn[a] = fmin(mn[a], (double)lo[a][j]);
            mx[a] = fmax(mx[a], (double)hi[a][j]);
        }
    }
    float org[3] = {0, 0, 0};
    int ex[3] = {0, 0, 0};
    uint8_t ql[3][4], qh[3][4];
    double ext = 0.0;
    for (int a = 0; a < 3; ++a)
        if (mx[a] >= mn[a]) ext = fmax(ext, mx[a] - mn[a]);
    // a node of points (extent 0) still gets a positive margin
    const double delta = ldexp(fmax(ext, 1e-30), -20);
    for (int a = 0; a < 3; ++a) {
        for (int j = 0; j < 4; ++j) { ql[a][j] = 255; qh[a][j] = 0; }
        if (!(mx[a] >= mn[a])) continue;   // no valid child
        // origin: a float at or below the lowest plane minus the margin
        float og = (float)(mn[a] - delta);
        while ((double)og > mn[a] - delta) og = nextafterf(og, -INFINITY);
        org[a] = og;
        const double span = mx[a] + delta - (double)og;
        int e;   // least power of two of at least span / 255
        if (frexp(span / 255.0, &e) == 0.5) --e;
        e = (e > -126 ? e : -126);
        for (;; ++e) {
            const double cell = ldexp(1.0, e);
            bool ok = true;
            for (int j = 0; j < 4 && ok; ++j) {
                if (!valid[j]) continue;
                double l = floor((lo[a][j] - delta - (double)og) / cell);
                double h = ceil((hi[a][j] + delta - (double)og) / cell);
                // the decoded planes (exact: og + q 2^e in double) enclose the widened box
                while (l > 0 && (double)og + l * cell > lo[a][j] - delta) l -= 1.0;
                while ((double)og + h * cell < hi[a][j] + delta) h += 1.0;
                if (l < 0 || h > 255) { ok = false; break; }
                ql[a][j] = (uint8_t)l;
                qh[a][j] = (uint8_t)h;
            }
            if (ok) break;
        }
        ex[a] = e;
    }
    auto pack = [](const uint8_t b[4]) {
        return quant_bits_f((int)((uint32_t)b[0] | (uint32_t)b[1] << 8 | (uint32_t)b[2] << 16 | (uint32_t)b[3] << 24));
    };
    const uint32_t ew = (uint32_t)(ex[0] + 127) | (uint32_t)(ex[1] + 127) << 8 | (uint32_t)(ex[2] + 127) << 16;
    d[0] = org[0]; d[1] = org[1]; d[2] = org[2]; d[3] = quant_bits_f((int)ew);
    d[4] = pack(ql[0]); d[5] = pack(qh[0]); d[6] = pack(ql[1]); d[7] = pack(qh[1]);
    d[8] = pack(ql[2]); d[9] = pack(qh[2]);
    // the traversal's cell sizes, with the 2^24 that turns a byte read as an
    // fp16 subnormal back into an integer
    auto size = [&](int a) { return (uint32_t)quant_bits_i((float)ldexp(1.0, ex[a] + 24)); };
    d[10] = quant_bits_f((int)(size(0) | size(1) >> 16));
    d[11] = quant_bits_f((int)size(2));
    for (int j = 0; j < 4; ++j) d[12 + j] = quant_bits_f(valid[j] ? ref[j] : ~0);
}

}  // namespace ipt
