// Root cube, keys, level-10 cells and the leaf rule of the octree: what the
// kernels of one large input and the one-workgroup kernel of a small one share.
#pragma once

#include "common.hpp"

namespace gdn {

// Root cube: side S = largest bbox extent at the bbox minimum; depth limit from
// the minimum leaf side. Same FP64 expressions for every consumer.
__device__ __forceinline__ void frame_consts(const FrameStat* c, double min_leaf_side, FrameConst* f) {
    double S = 0.0;
    for (int a = 0; a < 3; ++a) {
        float lo = f32_from_ordered(~c->bbox_nmin[a]);
        float hi = f32_from_ordered(c->bbox_max[a]);
        f->lo[a] = lo;
        double H = (double)hi - (double)lo;
        if (H > S) S = H;
    }
    if (!(S > 0.0) || !(S < INFINITY)) S = 1.0;
    f->S = S;
    f->scale = 2097152.0 / S;
    int d = MORTON_BITS;
    if (min_leaf_side > 0.0) {
        d = 0;
        while (d < MORTON_BITS && ldexp(S, -(d + 1)) >= min_leaf_side) ++d;
    }
    f->dmax = d;
}

__device__ __forceinline__ uint32_t quantise(float x, float lo, double scale) {
    double q = floor(((double)x - (double)lo) * scale);
    if (!(q >= 0.0)) q = 0.0;
    if (q > (double)QMAX) q = (double)QMAX;
    return (uint32_t)q;
}

// A level-10 cell is the keys with one value of key >> CELL_SHIFT.
constexpr int CELL_SHIFT = 3 * (MORTON_BITS - SORT_SHORT_LEVEL);  // level-10 prefix = key >> 33

// First position in [lo, hi) whose level-10 cell prefix is >= c (the keys
// are in cell order everywhere).
__device__ __forceinline__ uint32_t cell_lower_bound(const uint64_t* keys, uint32_t lo, uint32_t hi, uint64_t c) {
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((keys[mid] >> CELL_SHIFT) < c) lo = mid + 1u;
        else hi = mid;
    }
    return lo;
}

// Number of leading octal digits two 63-bit Morton keys share (21 if equal).
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
    if (a == b) return MORTON_BITS;
    return (__clzll((long long)(a ^ b)) - 1) / 3;
}

// Leaves are the non-empty nodes reached by splitting every node that holds
// more than `cap` points above the depth limit. In the sorted key order a
// leaf boundary falls between positions j-1 and j exactly when the deepest
// cell holding both (level l = their common digits) is split, i.e. l < dmax
// and that cell holds more than `cap` points. The cell count is tested with
// one windowed binary search (window cap + 1).
//
// Boundary test of sorted position j inside its frame [fs, fe): the frame's
// first point starts a leaf; otherwise the rule above with the frame's depth
// limit and the search window clipped to the frame.
// Positions that share a level-10 cell lie in one leaf unless the cell is
// deep (more than leaf_cap points: it was re-sorted on the whole key, and the
// test below applies inside it).
__device__ __forceinline__ uint32_t leaf_boundary(const uint64_t* keys, uint32_t j, uint32_t fs, uint32_t fe, int dmax,
                                                  bool deep, uint32_t cap) {
    if (j == fs) return 1u;
    const uint64_t a = keys[j - 1], b = keys[j];
    const int l = common_digits(a, b);
    if (l >= dmax || (l >= SORT_SHORT_LEVEL && !deep)) return 0u;
    const int sh = 3 * (MORTON_BITS - l);
    const uint64_t P = b >> sh;
    uint32_t lo = (j - 1 - fs > cap) ? j - 1 - cap : fs;
    uint32_t hi = j - 1;
    while (lo < hi) {
        uint32_t mid = (lo + hi) >> 1;
        if ((keys[mid] >> sh) < P) lo = mid + 1;
        else hi = mid;
    }
    const uint64_t probe = (uint64_t)lo + cap;
    return (probe < fe && (keys[probe] >> sh) == P) ? 1u : 0u;
}

}  // namespace gdn
