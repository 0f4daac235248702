// Four-child BVH nodes from the binary tree's child-pair records (host side).
//
// Greedy collapse: a node starts from a binary node's two children and, while
// it has fewer than four, replaces its inner child of largest surface area by
// that child's two children (the greedy collapse of wide BVHs); leaves stay
// leaves, and the boxes are the binary tree's (padded) child boxes.  Against
// folding exactly every other binary level, the apartment's rays visit 15.0
// instead of 16.2 nodes.
#include "bvh_wide.h"

#include "bvh_quant.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>

namespace ipt {

namespace {

int bits_i(float f) { int i; std::memcpy(&i, &f, sizeof i); return i; }
float bits_f(int i) { float f; std::memcpy(&f, &i, sizeof f); return f; }

struct Child {
    float lo[3], hi[3];
    int ref;
};

}  // namespace

int64_t collapse_wide(const std::vector<float>& pairs, std::vector<float>& wide, int* depth) {
    auto children = [&](int r, Child out[2]) {
        const float* n = &pairs[16 * (size_t)r];
        out[0] = Child{{n[0], n[1], n[2]}, {n[3], n[4], n[5]}, bits_i(n[12])};
        out[1] = Child{{n[6], n[7], n[8]}, {n[9], n[10], n[11]}, bits_i(n[13])};
    };
    struct Node {
        int rec, level;                // binary record, node level
    };
    std::vector<Node> node{{0, 0}};    // by four-child node id
    node.reserve(pairs.size() / 32);
    wide.assign(32, 0.0f);
    wide.reserve(2 * pairs.size());
    std::vector<int> stack{0};         // four-child node ids to write
    int levels = 1;
    while (!stack.empty()) {
        const int id = stack.back();
        stack.pop_back();
        // the binary node's children, then, while a slot is free, the inner
        // child of largest surface area is replaced by its own children
        Child c2[2], g[4];
        children(node[id].rec, c2);
        int m = 0;
        for (int k = 0; k < 2; ++k)
            if (c2[k].ref != kWideNone) g[m++] = c2[k];
        while (m < 4) {
            int open = -1;
            double best_area = -1.0;
            for (int j = 0; j < m; ++j) {
                if (g[j].ref < 0) continue;
                const double dx = (double)g[j].hi[0] - g[j].lo[0], dy = (double)g[j].hi[1] - g[j].lo[1],
                             dz = (double)g[j].hi[2] - g[j].lo[2];
                const double area = dx * dy + dy * dz + dz * dx;
                if (area > best_area) { best_area = area; open = j; }
            }
            if (open < 0) break;
            Child gc[2];
            children(g[open].ref, gc);
            int k = 0;
            for (int j = 0; j < 2; ++j) {
                if (gc[j].ref == kWideNone) continue;
                if (k++ == 0) g[open] = gc[j];
                else g[m++] = gc[j];
            }
            if (k == 0) g[open] = g[--m];   // a record without children
        }
        int ref[4] = {kWideNone, kWideNone, kWideNone, kWideNone};
        int inner[4], ninner = 0;
        for (int j = 0; j < m; ++j) {
            if (g[j].ref >= 0) {
                ref[j] = (int)node.size();
                const int level = node[id].level + 1;
                node.push_back({g[j].ref, level});
                levels = std::max(levels, level + 1);
                inner[ninner++] = ref[j];
            } else {
                ref[j] = g[j].ref;
            }
        }
        for (int k = ninner; k-- > 0;) stack.push_back(inner[k]);
        wide.resize(32 * node.size());
        // an empty slot gets lo = hi = +inf on every axis: the slab test
        // gives it an entry distance of +inf (never entered)
        const float inf = std::numeric_limits<float>::infinity();
        float* o = &wide[32 * (size_t)id];
        for (int j = 0; j < 4; ++j)
            for (int a = 0; a < 3; ++a) {
                o[4 * (2 * a) + j] = j < m ? g[j].lo[a] : inf;
                o[4 * (2 * a + 1) + j] = j < m ? g[j].hi[a] : inf;
            }
        for (int j = 0; j < 4; ++j) {
            o[24 + j] = bits_f(ref[j]);
            o[28 + j] = 0.0f;
        }
    }
    if (depth) *depth = levels;
    return (int64_t)node.size();
}

void quantize_wide(std::vector<float>& wide) {
    const size_t n = wide.size() / 32;
    std::vector<float> q(16 * n);
    for (size_t id = 0; id < n; ++id) quantize_node(&wide[32 * id], &q[16 * id]);
    wide.swap(q);
}

}  // namespace ipt
