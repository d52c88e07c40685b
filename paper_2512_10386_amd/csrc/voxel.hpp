// Voxel size, index and hash of the per-leaf voxel filter (Eq. 10-12).
#pragma once

#include "common.hpp"

namespace gdn {

__device__ __forceinline__ uint32_t vox_hash(uint64_t k) {
    return (uint32_t)((k * 0x9E3779B97F4A7C15ull) >> 32);
}

__device__ __forceinline__ uint64_t vox_key(float4 p, float mx_, float my_, float mz_, double h) {
    double v[3] = {floor(((double)p.x - (double)mx_) / h), floor(((double)p.y - (double)my_) / h),
                   floor(((double)p.z - (double)mz_) / h)};
    uint64_t k = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double f = v[a];
        if (!(f >= 0.0)) f = 0.0;
        if (f > (double)QMAX) f = (double)QMAX;
        k |= (uint64_t)f << (21 * a);
    }
    return k;
}

// Leaf voxel size (Eq. 10, 11) from its fp32 bbox: h = beta * cbrt(V / nt)
// rounded to fp32, 0 for a flat or degenerate leaf.
__device__ __forceinline__ float leaf_voxel_size(const float* lo, const float* hi, uint32_t nt, double beta) {
    double H[3];
    for (int a = 0; a < 3; ++a) H[a] = (double)hi[a] - (double)lo[a];
    const double V = (H[0] * H[1]) * H[2];
    float h32 = (float)(beta * cbrt(V / (double)nt));
    if (!(h32 > 0.0f) || !isfinite(h32)) h32 = 0.0f;
    return h32;
}

}  // namespace gdn
