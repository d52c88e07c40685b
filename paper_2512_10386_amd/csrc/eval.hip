// Evaluation kernels (include/gdn.h, gdn_nearest / gdn_eval_metrics): exact
// nearest neighbours between two clouds and the quality metrics of a
// denoised cloud, PSNR (Eq. 29) and the Chamfer distance (Eq. 30).
//
// Nearest, by groups (the second half of this file): both clouds in Hilbert
// order, the reference in groups of 64 points with boxes; a wave takes 16
// neighbouring queries and evaluates only the groups whose box lies within some
// query's best distance so far.
// Nearest, brute force (where sorting does not pay, or a workspace too small for
// the groups): one thread per query point, the reference cloud
// streamed through LDS in tiles; the reference is split into chunks, each with
// workgroups of its own, so that small query sets still fill the chip, and the
// chunks' answers are combined with a 64-bit atomic minimum on the key
// (fp32 d2 bits << 32 | index): d2 >= 0, so the bit order is the value
// order, and equal distances resolve to the smaller index.
#include <algorithm>

#include "kernels.hpp"
#include "radix.hpp"
#include "wave.hpp"

namespace gdn {

namespace {

constexpr int NN_BLOCK = 256;
constexpr int NN_TILE = 256;                // reference points per LDS tile (short, so that small clouds make many blocks)
constexpr unsigned NN_MIN_BLOCKS = 2048;    // split the reference until the grid has this many blocks
constexpr int EV_BLOCK = 256;
constexpr unsigned EV_BLOCKS_MAX = 1024;
constexpr int EV_STRIDE = 8;                // doubles per block partial

// One direction of a brute-force search: na queries, the best key of each; its
// workgroups are `blocks` blocks of queries times the chunks of the reference.
struct NnDir {
    const float* a;
    const float* b;
    uint32_t na, nb, chunk, blocks, chunks;
    unsigned long long* key;
};

// (the metrics run both directions in each launch: blockIdx.z here, one after
// the other in the search, whose grids differ: as one z-grid of both directions'
// largest sizes 300 against 10M points took 18 ms, nearly all of it workgroups
// without work)
__global__ __launch_bounds__(256) void nn_init_kernel(NnDir d0, NnDir d1) {
    const NnDir& d = blockIdx.z ? d1 : d0;
    const unsigned long long none = (unsigned long long)__float_as_uint(INFINITY) << 32;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < d.na; i += gridDim.x * blockDim.x) d.key[i] = none;
}

__global__ __launch_bounds__(NN_BLOCK) void nn_kernel(NnDir d0, NnDir d1) {
    __shared__ float s_x[NN_TILE], s_y[NN_TILE], s_z[NN_TILE];
    const uint32_t blocks0 = d0.blocks * d0.chunks;
    const bool second = blockIdx.x >= blocks0;
    const NnDir& d = second ? d1 : d0;
    const uint32_t blk = second ? blockIdx.x - blocks0 : blockIdx.x;
    const uint32_t i = blk % d.blocks * NN_BLOCK + threadIdx.x;
    const uint32_t c0 = blk / d.blocks * d.chunk;  // (below nb: the last chunk is not empty)
    const bool live = i < d.na;
    float ax = 0.f, ay = 0.f, az = 0.f;
    if (live) {
        ax = d.a[3 * (size_t)i];
        ay = d.a[3 * (size_t)i + 1];
        az = d.a[3 * (size_t)i + 2];
    }
    const uint32_t c1 = min(d.nb, c0 + d.chunk);
    // a thread's point of the next tile, read while the tile before is evaluated
    // (past the end: the last point again, which changes nothing)
    static_assert(NN_TILE == NN_BLOCK, "a point of the tile per thread");
    float nx, ny, nz;
    auto read = [&](uint32_t t0) {
        const size_t j = min(t0 + threadIdx.x, c1 - 1u);
        nx = d.b[3 * j];
        ny = d.b[3 * j + 1];
        nz = d.b[3 * j + 2];
    };
    read(c0);
    float best = INFINITY;
    uint32_t bi = 0;
    for (uint32_t t0 = c0; t0 < c1; t0 += NN_TILE) {
        __syncthreads();
        s_x[threadIdx.x] = nx;
        s_y[threadIdx.x] = ny;
        s_z[threadIdx.x] = nz;
        __syncthreads();
        if (t0 + NN_TILE < c1) read(t0 + NN_TILE);
        const uint32_t end = min((uint32_t)NN_TILE, (c1 - t0 + 7u) & ~7u);
#pragma unroll 8
        for (uint32_t e = 0; e < end; ++e) {
            const float dx = s_x[e] - ax, dy = s_y[e] - ay, dz = s_z[e] - az;
            const float v = (dx * dx + dy * dy) + dz * dz;  // compiled without contraction (no FMA)
            if (v < best) {
                best = v;
                bi = t0 + e;
            }
        }
    }
    if (live && best < INFINITY)
        atomicMin(&d.key[i], ((unsigned long long)__float_as_uint(best) << 32) | bi);
}

__global__ __launch_bounds__(256) void nn_out_kernel(const unsigned long long* __restrict__ key, uint32_t na,
                                                     uint32_t* __restrict__ idx, float* __restrict__ d2) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < na; i += gridDim.x * blockDim.x) {
        const unsigned long long k = key[i];
        idx[i] = (uint32_t)k;
        d2[i] = __uint_as_float((uint32_t)(k >> 32));
    }
}

__device__ __forceinline__ double wave_sum_d(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_min_f(float v) {
    return wave_fmin(v);
}
__device__ __forceinline__ float wave_max_f(float v) {
    return wave_fmax(v);
}

// Per block: sum of the FP64 squared distances from points of a to their
// matched points of b (slot 0), and, for the first direction, the fp32
// min/max per axis of a (slots 1..6).
__global__ __launch_bounds__(EV_BLOCK) void ev_sum_kernel(NnDir d0, NnDir d1, unsigned blocks0, double* __restrict__ part0,
                                                          double* __restrict__ part1) {
    const bool box = blockIdx.x < blocks0;
    const NnDir& d = box ? d0 : d1;
    const float* __restrict__ a = d.a;
    const float* __restrict__ b = d.b;
    const uint32_t na = d.na, blk = box ? blockIdx.x : blockIdx.x - blocks0;
    const uint32_t blks = box ? blocks0 : gridDim.x - blocks0;
    double* __restrict__ part = (box ? part0 : part1) + (size_t)blk * EV_STRIDE;
    __shared__ double s_sum[EV_BLOCK / 64];
    __shared__ float s_lo[EV_BLOCK / 64][3], s_hi[EV_BLOCK / 64][3];
    double s = 0.0;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (uint32_t i = blk * EV_BLOCK + threadIdx.x; i < na; i += blks * EV_BLOCK) {
        const uint32_t j = (uint32_t)d.key[i];
        double t = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float ac = a[3 * (size_t)i + c];
            const double e = (double)b[3 * (size_t)j + c] - (double)ac;
            t += e * e;
            lo[c] = fminf(lo[c], ac);
            hi[c] = fmaxf(hi[c], ac);
        }
        s += t;
    }
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    s = wave_sum_d(s);
    for (int c = 0; c < 3; ++c) {
        lo[c] = wave_min_f(lo[c]);
        hi[c] = wave_max_f(hi[c]);
    }
    if (lane == 0) {
        s_sum[w] = s;
        for (int c = 0; c < 3; ++c) {
            s_lo[w][c] = lo[c];
            s_hi[w][c] = hi[c];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < EV_BLOCK / 64; ++q) t += s_sum[q];
        part[0] = t;
        if (box) {
            for (int c = 0; c < 3; ++c) {
                float l = s_lo[0][c], h = s_hi[0][c];
                for (int q = 1; q < EV_BLOCK / 64; ++q) {
                    l = fminf(l, s_lo[q][c]);
                    h = fmaxf(h, s_hi[q][c]);
                }
                part[1 + c] = (double)l;
                part[4 + c] = (double)h;
            }
        }
    }
}

// One wave: MSE (clean -> denoised), mean denoised -> clean, CD, PSNR.
__global__ __launch_bounds__(64) void ev_final_kernel(const double* __restrict__ pc, uint32_t nbc,
                                                      const double* __restrict__ pd, uint32_t nbd, uint32_t nc,
                                                      uint32_t nd, double* __restrict__ out) {
    const uint32_t lane = threadIdx.x;
    double sc = 0.0, sd = 0.0;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (uint32_t q = lane; q < nbc; q += 64u) {
        sc += pc[(size_t)q * EV_STRIDE];
        for (int c = 0; c < 3; ++c) {
            lo[c] = fmin(lo[c], pc[(size_t)q * EV_STRIDE + 1 + c]);
            hi[c] = fmax(hi[c], pc[(size_t)q * EV_STRIDE + 4 + c]);
        }
    }
    for (uint32_t q = lane; q < nbd; q += 64u) sd += pd[(size_t)q * EV_STRIDE];
    sc = wave_sum_d(sc);
    sd = wave_sum_d(sd);
    for (int c = 0; c < 3; ++c) {
        for (int o = 32; o > 0; o >>= 1) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], o, 64));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], o, 64));
        }
    }
    if (lane == 0) {
        double m2 = 0.0;
        for (int c = 0; c < 3; ++c) m2 += (hi[c] - lo[c]) * (hi[c] - lo[c]);
        const double mse = sc / (double)nc;
        out[0] = mse;
        out[1] = sd / (double)nd;
        out[2] = out[0] + out[1];
        out[3] = 10.0 * log10(m2 / mse);
    }
}

unsigned ev_blocks(uint32_t n) {
    unsigned b = (n + EV_BLOCK - 1) / EV_BLOCK;
    if (b > EV_BLOCKS_MAX) b = EV_BLOCKS_MAX;
    return b == 0 ? 1u : b;
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---------------------------------------------------------------- nearest by groups
//
// Both clouds are put in Hilbert order (radix passes over 24- or 30-bit keys
// of a common cube, both clouds in each launch). The reference's sorted points
// form groups of 64 with boxes, and supers of 64 groups with boxes. A wave
// takes a tile of 16 consecutive queries. Each lane that holds a query first
// takes the points next to its key's place in the reference order; then the
// wave walks the supers and groups whose box lies within the tile's largest
// best distance of the tile's box, tests each such group's box against the
// queries, and evaluates the needed (query, group) pairs a point per lane. Box
// distances use the rounded operations of the point distance, which are
// monotone, and a box is skipped only if its distance exceeds the best so
// far, so the answer (ties included: equal distances compare indices) is the
// brute-force one.
//
// Key bits: 8 per axis cost a LiDAR sweep of 20k points 76 us, 10 bits 80, 5
// bits (two passes) 166 (70 for a scanned object of that size, where 8 bits
// take 73).
//
// A tile with far queries (noise between surfaces) reaches hundreds of
// groups; walked like the others, such tiles were the kernel's tail. A tile
// whose box reaches more than NN_HARD groups is put on a list instead, and
// nn_far_kernel takes its queries one per wave, the nearest boxes first.
//
// Bound by the latency of the chain (search the key, seeds, supers, groups,
// points) and, on large clouds, by the pair evaluations: the metrics of a 120k
// LiDAR sweep (114k against 111k points) take 143 us, 65 of them here, 18 the
// far queries, 56 the boxes, the keys and the sort; all pairs take 5162 us at
// 2.6 ms per direction. 16k against 16k points: 71 us, 119 by all pairs.

constexpr int NN_GRP = 64;                      // points per group (one per lane)
constexpr int NN_SUP = 64 * NN_GRP;             // points per super
constexpr uint32_t NN_TQ = 16;                  // queries per tile
constexpr uint32_t NN_HARD = 32;                // groups within reach of a tile, above: one wave per query
constexpr int NN_PASSES_MAX = 4;
constexpr uint32_t NN_SHORT_N = 1u << 15;       // clouds up to this size: 8 key bits per axis (3 passes), else 10 (4)
constexpr uint32_t NN_BOX_BLOCKS = 256;         // box records per cloud, at most
constexpr int NN_REC = 12;                      // floats per box record: finite min, max, then min, max of all points
constexpr float NN_TAIL = 16.0f;                // clouds reaching farther than this many times their middle half: see nn_key_kernel
constexpr uint32_t NN_FAR_BLOCKS = 512;         // far kernel: 16 waves each
constexpr uint32_t NN_FAR_MOST = 48;            // far kernel: groups one query evaluates by itself, at most,
constexpr uint32_t NN_FAR_SHARE = 16;           // or this share of all, if that is more
constexpr uint32_t NN_SUM_TILES = 1u << 14;     // tile sums one block adds up

struct NnBox {
    float4 lo, hi;  // groups: lo.w holds the bits of the smallest index
};

struct NnCloud {
    const float* p;       // [n][3]
    uint32_t n, tiles;
    uint32_t* key[2];     // Hilbert keys (ping-pong; sorted in key[0])
    uint32_t* idx[2];
    float4* pos;          // [whole supers] sorted x, y, z, index bits; NaN past n
    NnBox* gbox;          // per group
    uint32_t* sbox;       // per super [8]: ordered-uint max of ~min and of max (zeroed block)
    uint32_t* hist;       // [passes][256]
    uint32_t* status;     // [passes][tiles][256]
    float* rec;           // [box blocks][NN_REC]
    uint32_t box_blocks, key_blocks, supers;
    uint32_t qtiles;      // query tiles of this cloud
    uint2* seed;          // [n] best so far (bits, index) of the queries of hard tiles
    uint32_t* hard;       // [qtiles] list of hard tiles
    uint32_t* n_hard;     // (zeroed block)
    double* part;         // [qtiles] sums of the tiles' squared distances
    double* part2;        // [ceil(qtiles / NN_SUM_TILES)]
};

struct NnPlan {
    NnCloud c[2];
    int passes;
    uint32_t tile;        // keys per workgroup of the radix passes
    int first;            // buffer the first pass reads (the order ends in key[0], idx[0])
    char* zero;           // histograms, look-back words, flag
    size_t zero_bytes;
    uint32_t* flag;       // a look-back wait expired: the order is not usable
    float* core;          // [4] medians of both clouds' coordinates, and the extent of their middle half
    size_t bytes;
};

NnPlan nn_plan(const float* a, uint32_t na, const float* b, uint32_t nb, char* base) {
    NnPlan P{};
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        char* q = base ? base + off : nullptr;
        off += al256(bytes);
        return q;
    };
    const uint32_t big = na > nb ? na : nb;
    P.passes = big <= NN_SHORT_N ? 3 : NN_PASSES_MAX;
    P.first = P.passes & 1;
    P.tile = sort_tile_for(big);
    if (P.tile < 1024u) P.tile = 1024u;  // (the order and its look-backs are a small part there)
    P.c[0].p = a;
    P.c[0].n = na;
    P.c[1].p = b;
    P.c[1].n = nb;
    const size_t z0 = off;
    P.flag = (uint32_t*)take(4);
    for (NnCloud& c : P.c) {
        c.tiles = (c.n + P.tile - 1) / P.tile;
        c.supers = (c.n + NN_SUP - 1) / NN_SUP;
        c.n_hard = (uint32_t*)take(4);
        c.sbox = (uint32_t*)take(32 * (size_t)c.supers);
        c.hist = (uint32_t*)take((size_t)P.passes * 256 * 4);
        c.status = (uint32_t*)take((size_t)P.passes * c.tiles * 256 * 4);
    }
    P.zero = base ? base + z0 : nullptr;
    P.zero_bytes = off - z0;
    P.core = (float*)take(16);
    for (NnCloud& c : P.c) {
        const size_t padded = (size_t)c.supers * NN_SUP;
        for (int i = 0; i < 2; ++i) {
            c.key[i] = (uint32_t*)take(4 * (size_t)c.n);
            c.idx[i] = (uint32_t*)take(4 * (size_t)c.n);
        }
        c.pos = (float4*)take(16 * padded);
        c.gbox = (NnBox*)take(sizeof(NnBox) * (padded / NN_GRP));
        c.box_blocks = (c.n + 511) / 512;
        if (c.box_blocks > NN_BOX_BLOCKS) c.box_blocks = NN_BOX_BLOCKS;
        c.key_blocks = (c.n + 1023) / 1024;
        if (c.key_blocks > 512) c.key_blocks = 512;
        c.rec = (float*)take((size_t)4 * NN_REC * c.box_blocks);
        c.qtiles = (c.n + NN_TQ - 1) / NN_TQ;
        c.seed = (uint2*)take(8 * (size_t)c.n);
        c.hard = (uint32_t*)take(4 * (size_t)c.qtiles);
        c.part = (double*)take(8 * (size_t)c.qtiles);
        c.part2 = (double*)take(8 * (size_t)((c.qtiles + NN_SUM_TILES - 1) / NN_SUM_TILES));
    }
    P.bytes = off;
    return P;
}

// Medians and the extent of the middle half, per axis over 64 points taken at
// equal steps from both clouds; a wave per axis. One workgroup calls it.
__device__ void nn_core(const NnPlan& P, float* s_iqr) {
    const uint32_t lane = threadIdx.x & 63u, axis = threadIdx.x >> 6;
    if (axis < 3u) {
        const NnCloud& c = P.c[lane & 1u];
        const size_t i = (size_t)((uint64_t)(lane | 1u) * c.n / 64u);
        const float x = c.p[3 * i + axis];
        const uint32_t v = sort64_u32<true>(isfinite(x) ? f32_ordered(x) : 0xFFFFFFFFu, lane);
        const float lo = f32_from_ordered((uint32_t)__builtin_amdgcn_readlane((int)v, 16));
        const float mid = f32_from_ordered((uint32_t)__builtin_amdgcn_readlane((int)v, 32));
        const float hi = f32_from_ordered((uint32_t)__builtin_amdgcn_readlane((int)v, 47));
        if (lane == 0u) {
            P.core[axis] = mid;
            s_iqr[axis] = hi - lo;
        }
    }
    __syncthreads();
    // (not a number on an axis where a quarter of the points is not finite: it does not count)
    if (threadIdx.x == 0) P.core[3] = fmaxf(fmaxf(s_iqr[0], s_iqr[1]), s_iqr[2]);
}

// Boxes of both clouds, one record per block, and the control words cleared
// (nothing here uses them). The last block takes nn_core.
__global__ __launch_bounds__(256) void nn_box_kernel(NnPlan P) {
    __shared__ float s_v[4][NN_REC];
    uint4* z = (uint4*)P.zero;
    const size_t n16 = P.zero_bytes / 16;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        z[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == gridDim.x - 1u) {
        nn_core(P, s_v[0]);
        return;
    }
    const bool second = blockIdx.x >= P.c[0].box_blocks;
    const NnCloud& c = P.c[second ? 1 : 0];
    const uint32_t blk = second ? blockIdx.x - P.c[0].box_blocks : blockIdx.x;
    float v[NN_REC];
#pragma unroll
    for (int i = 0; i < NN_REC; ++i) v[i] = (i / 3) % 2 == 0 ? INFINITY : -INFINITY;
    for (uint32_t i = blk * 256u + threadIdx.x; i < c.n; i += c.box_blocks * 256u) {
        float x[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) x[a] = c.p[3 * (size_t)i + a];
        const bool fin = isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[a] = fminf(v[a], fin ? x[a] : INFINITY);
            v[3 + a] = fmaxf(v[3 + a], fin ? x[a] : -INFINITY);
            v[6 + a] = fminf(v[6 + a], x[a]);
            v[9 + a] = fmaxf(v[9 + a], x[a]);
        }
    }
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NN_REC; ++i) {
        v[i] = (i / 3) % 2 == 0 ? wave_min(v[i], lane) : wave_max(v[i], lane);
        if (lane == 0u) s_v[w][i] = v[i];
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)NN_REC) {
        const int i = (int)threadIdx.x;
        float r = s_v[0][i];
        for (int q = 1; q < 4; ++q) r = (i / 3) % 2 == 0 ? fminf(r, s_v[q][i]) : fmaxf(r, s_v[q][i]);
        c.rec[(size_t)blk * NN_REC + i] = r;
    }
}

__device__ __forceinline__ uint32_t spread3_10(uint32_t v) {
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    return (v | (v << 2)) & 0x09249249u;
}

// Place of cell (x, y, z) of a 2^BITS grid on the Hilbert curve (Skilling's
// transform of the coordinates, then the bits interleaved). Its runs are
// connected, so a group of consecutive points has a smaller box than in Morton
// order: a query needs 2.5 groups of a LiDAR sweep instead of 3.5, 2.3 of a
// scanned object instead of 4.7.
template <int BITS>
__device__ __forceinline__ uint32_t hilbert3(uint32_t x, uint32_t y, uint32_t z) {
#pragma unroll
    for (int b = BITS - 1; b >= 1; --b) {
        const uint32_t low = (1u << b) - 1u;
        auto step = [&](uint32_t& v) {
            const bool set = (v >> b) & 1u;
            const uint32_t t = set ? low : (x ^ v) & low;
            x ^= t;
            v ^= set ? 0u : t;
        };
        // (for the first axis itself the exchange is a no-op)
        x ^= (x >> b) & 1u ? low : 0u;
        step(y);
        step(z);
    }
    y ^= x;
    z ^= y;
    uint32_t t = 0u;
#pragma unroll
    for (int b = BITS - 1; b >= 1; --b) t ^= (z >> b) & 1u ? (1u << b) - 1u : 0u;
    return (spread3_10(x ^ t) << 2) | (spread3_10(y ^ t) << 1) | spread3_10(z ^ t);
}

// Hilbert keys of both clouds in the cube at their common minimum (non-finite
// coordinates quantise to a border cell: their points only need some place)
// and the digit histograms. A single stray point far out would leave all others
// in one cell, without an order. Clouds that reach farther from their median than
// NN_TAIL times the extent of their middle half take cells that grow with the
// distance from it instead, the logarithm's (18000 against 18000 points, one of
// them at a million times their size: 231 us all in one cell, 70 so, all pairs
// 77; 200k against 200k 12.6 ms and 187 us).
template <int PASSES>
__global__ __launch_bounds__(256) void nn_key_kernel(NnPlan P) {
    __shared__ float s_lo[4][3], s_hi[4][3];
    __shared__ float s_c[5];
    __shared__ uint32_t s_hist[PASSES][256];
    constexpr int BITS = PASSES == 3 ? 8 : 10;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
    const float4 core = *(const float4*)P.core;
    for (int p = 0; p < PASSES; ++p) s_hist[p][tid] = 0u;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int q = 0; q < 2; ++q)
        for (uint32_t r = tid; r < P.c[q].box_blocks; r += 256u)
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], P.c[q].rec[(size_t)r * NN_REC + a]);
                hi[a] = fmaxf(hi[a], P.c[q].rec[(size_t)r * NN_REC + 3 + a]);
            }
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(lo[a], lane);
        hi[a] = wave_max(hi[a], lane);
        if (lane == 0u) {
            s_lo[w][a] = lo[a];
            s_hi[w][a] = hi[a];
        }
    }
    __syncthreads();
    if (tid == 0u) {
        const float mid[3] = {core.x, core.y, core.z};
        float side = 0.0f, reach = 0.0f;
        for (int a = 0; a < 3; ++a) {
            float l = s_lo[0][a], h = s_hi[0][a];
            for (int q = 1; q < 4; ++q) {
                l = fminf(l, s_lo[q][a]);
                h = fmaxf(h, s_hi[q][a]);
            }
            s_c[a] = l;
            side = fmaxf(side, h - l);
            reach = fmaxf(reach, fmaxf(h - mid[a], mid[a] - l));
        }
        s_c[3] = side > 0.0f && side < INFINITY ? (float)(1 << BITS) / side : 0.0f;
        s_c[4] = 0.0f;
        if (core.w > 0.0f && reach > NN_TAIL * core.w && reach < INFINITY) {
            for (int a = 0; a < 3; ++a) s_c[a] = mid[a];
            s_c[3] = (float)(1 << (BITS - 1)) / log2f(1.0f + reach / core.w);
            s_c[4] = 1.0f / core.w;
        }
    }
    __syncthreads();
    const float c0 = s_c[0], c1 = s_c[1], c2 = s_c[2], sc = s_c[3], per = s_c[4];
    const bool second = blockIdx.x >= P.c[0].key_blocks;
    const NnCloud& c = P.c[second ? 1 : 0];
    const uint32_t blk = second ? blockIdx.x - P.c[0].key_blocks : blockIdx.x;
    auto q10 = [&](float x, float l) {
        float t = (x - l) * sc;
        if (per != 0.0f) {
            const float u = log2f(1.0f + fabsf(x - l) * per) * sc;
            t = (float)(1 << (BITS - 1)) + (x < l ? -u : u);
        }
        return (uint32_t)fminf(fmaxf(t, 0.0f), (float)((1 << BITS) - 1));
    };
    const uint32_t stride = c.key_blocks * 256u;
    constexpr int U = 4;
    for (uint32_t i0 = blk * 256u + tid; i0 < c.n; i0 += (uint32_t)U * stride) {
        float x[U], y[U], z[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = (uint64_t)i0 + (uint64_t)u * stride;
            const size_t j = i < c.n ? (size_t)i : (size_t)c.n - 1;
            x[u] = c.p[3 * j];
            y[u] = c.p[3 * j + 1];
            z[u] = c.p[3 * j + 2];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = (uint64_t)i0 + (uint64_t)u * stride;
            if (i >= c.n) break;
            const uint32_t k = hilbert3<BITS>(q10(x[u], c0), q10(y[u], c1), q10(z[u], c2));
            c.key[P.first][i] = k;
#pragma unroll
            for (int p = 0; p < PASSES; ++p) atomicAdd(&s_hist[p][(k >> (8 * p)) & 255u], 1u);
        }
    }
    __syncthreads();
    for (int p = 0; p < PASSES; ++p) {
        const uint32_t v = s_hist[p][tid];
        if (v) atomicAdd(&c.hist[p * 256 + tid], v);
    }
}

struct NnDigit {
    int shift;
    __device__ bool of_key() const { return true; }
    __device__ uint32_t key_digit(uint32_t k) const { return (k >> shift) & 255u; }
    __device__ uint32_t operator()(uint32_t k, uint32_t, bool) const { return key_digit(k); }
};

// One radix pass over both clouds (the first cloud's tiles, then the
// second's; each looks back over its own). The first pass's payload is the
// position itself.
template <int ITEMS, int BLOCK, bool FIRST>
__global__ __launch_bounds__(BLOCK) void nn_radix_kernel(NnPlan P, int pass) {
    const bool second = blockIdx.x >= P.c[0].tiles;
    const NnCloud& c = P.c[second ? 1 : 0];
    const uint32_t tile = second ? blockIdx.x - P.c[0].tiles : blockIdx.x;
    const int from = (pass + P.first) & 1, to = 1 - from;
    radix_tile<ITEMS, FIRST, BLOCK>((const uint32_t*)c.key[from], (const uint32_t*)c.idx[from], c.key[to], c.idx[to],
                                    c.n, tile, (const uint32_t*)c.hist + pass * 256,
                                    c.status + (size_t)pass * c.tiles * 256, P.flag, 1u, NnDigit{8 * pass});
}

// Sorted points and the boxes of groups and supers, NN_GATHER points per block.
constexpr int NN_GATHER = 1024;
__global__ __launch_bounds__(NN_GATHER) void nn_gather_kernel(NnPlan P) {
    __shared__ float s_b[6][NN_GATHER / NN_GRP];
    const uint32_t nb0 = P.c[0].supers * (uint32_t)(NN_SUP / NN_GATHER);
    const bool second = blockIdx.x >= nb0;
    const NnCloud& c = P.c[second ? 1 : 0];
    const uint32_t blk = second ? blockIdx.x - nb0 : blockIdx.x;
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    const float nan = __uint_as_float(0x7FC00000u);
    const size_t s = (size_t)blk * NN_GATHER + threadIdx.x;
    float4 q = make_float4(nan, nan, nan, __uint_as_float(0xFFFFFFFFu));
    if (s < c.n) {
        const uint32_t i = min(c.idx[0][s], c.n - 1u);  // (in range unless a look-back wait expired)
        q = make_float4(c.p[3 * (size_t)i], c.p[3 * (size_t)i + 1], c.p[3 * (size_t)i + 2], __uint_as_float(i));
    }
    c.pos[s] = q;  // (whole supers)
    // (NaN coordinates drop out of the box; an empty group's box is inverted)
    const float lx = wave_min(fminf(q.x, INFINITY), lane), hx = wave_max(fmaxf(q.x, -INFINITY), lane);
    const float ly = wave_min(fminf(q.y, INFINITY), lane), hy = wave_max(fmaxf(q.y, -INFINITY), lane);
    const float lz = wave_min(fminf(q.z, INFINITY), lane), hz = wave_max(fmaxf(q.z, -INFINITY), lane);
    uint32_t first = __float_as_uint(q.w);
    first = min(first, xor_lane<1>(first, lane));
    first = min(first, xor_lane<2>(first, lane));
    first = min(first, xor_lane<4>(first, lane));
    first = min(first, xor_lane<8>(first, lane));
    first = min(first, xor_lane<16>(first, lane));
    first = min(first, xor_lane<32>(first, lane));
    if (lane == 0u) {
        c.gbox[s / NN_GRP] = NnBox{make_float4(lx, ly, lz, __uint_as_float(first)), make_float4(hx, hy, hz, 0.f)};
        s_b[0][w] = lx;
        s_b[1][w] = ly;
        s_b[2][w] = lz;
        s_b[3][w] = hx;
        s_b[4][w] = hy;
        s_b[5][w] = hz;
    }
    __syncthreads();
    if (threadIdx.x < 6u) {
        const uint32_t a = threadIdx.x;
        float v = s_b[a][0];
        for (int q2 = 1; q2 < NN_GATHER / NN_GRP; ++q2) v = a < 3u ? fminf(v, s_b[a][q2]) : fmaxf(v, s_b[a][q2]);
        atomicMax(&c.sbox[8 * (size_t)(blk / (NN_SUP / NN_GATHER)) + a], a < 3u ? ~f32_ordered(v) : f32_ordered(v));
    }
}

__device__ __forceinline__ float box_gap2(const NnBox& B, float ax, float ay, float az, float bx, float by, float bz) {
    // squared distance between the box [a, b] (of queries) and B
    const float gx = fmaxf(fmaxf(B.lo.x - bx, ax - B.hi.x), 0.0f);
    const float gy = fmaxf(fmaxf(B.lo.y - by, ay - B.hi.y), 0.0f);
    const float gz = fmaxf(fmaxf(B.lo.z - bz, az - B.hi.z), 0.0f);
    return (gx * gx + gy * gy) + gz * gz;
}

// A group at the best distance itself can only hold a better match (an equal
// distance) with a smaller index: many copies of one place cost a query a few
// groups, not all of them.
__device__ __forceinline__ bool nn_needs(float gap, float first, float best, uint32_t bi) {
    return gap < best || (gap == best && __float_as_uint(first) < bi);
}

__device__ __forceinline__ NnBox super_box(const NnCloud& b, uint32_t s) {
    const uint4 u = *(const uint4*)(b.sbox + 8 * (size_t)s);
    const uint2 v = *(const uint2*)(b.sbox + 8 * (size_t)s + 4);
    return NnBox{make_float4(f32_from_ordered(~u.x), f32_from_ordered(~u.y), f32_from_ordered(~u.z), 0.f),
                 make_float4(f32_from_ordered(u.w), f32_from_ordered(v.x), f32_from_ordered(v.y), 0.f)};
}

__device__ __forceinline__ float lane_f32(float v, uint32_t l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), (int)l));
}
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}

__device__ __forceinline__ float nn_dist(float cx, float cy, float cz, float x, float y, float z) {
    const float dx = cx - x, dy = cy - y, dz = cz - z;
    return (dx * dx + dy * dy) + dz * dz;  // compiled without contraction (no FMA)
}

// Query j's best among the wave's points (one per lane: distance d, index
// id), given its best so far; false if none of them is as near. At the best
// distance itself only a smaller index counts.
__device__ __forceinline__ bool nn_best_of(float d, float id, uint32_t lane, float& bj, uint32_t& ij) {
    if (__builtin_amdgcn_ballot_w64(d <= bj) == 0ull) return false;
    const float m = wave_fmin(d);
    if (!(m < INFINITY)) return false;
    unsigned long long at = __builtin_amdgcn_ballot_w64(d == m);
    uint32_t i = m < bj ? 0xFFFFFFFFu : ij;
    while (at != 0ull) {
        i = min(i, lane_u32(__float_as_uint(id), (uint32_t)__ffsll((long long)at) - 1u));
        at &= at - 1ull;
    }
    bj = m;
    ij = i;
    return true;
}

// Tile of up to NN_TQ sorted queries of cloud a (lane l < NN_TQ holds query
// q, its key and whether its coordinates are finite: others match nothing).
// best = +inf and bi = 0 if there is no match (as brute force: no distance
// below +inf). Returns false, with the best among the seeds, for a hard tile.
__device__ __forceinline__ bool nn_tile(const NnCloud& b, bool lost, float4 q, uint32_t key, bool fin,
                                        uint32_t lane, float& best, uint32_t& bi) {
    best = fin ? INFINITY : -1.0f;
    bi = 0u;
    auto take = [&](float x, float y, float z, uint32_t id) {
        const float d = nn_dist(x, y, z, q.x, q.y, q.z);
        if (d < best || (d == best && id < bi)) {
            best = d;
            bi = id;
        }
    };
    if (lost) {  // every pair
        for (uint32_t j = 0; j < b.n; ++j)
            take(b.p[3 * (size_t)j], b.p[3 * (size_t)j + 1], b.p[3 * (size_t)j + 2], j);
        return true;
    }
    // the place of the first query's key in the reference order, 64 probes at a time
    const uint32_t* __restrict__ keys = b.key[0];
    const uint32_t k0 = lane_u32(key, 0u);
    uint32_t lo = 0, len = b.n;  // the place is in [lo, lo + len]
    while (len > 0u) {
        const uint32_t step = (len + 63u) / 64u;
        const uint32_t at = lane * step;
        const bool less = at < len && keys[lo + at] < k0;
        const uint32_t c = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(less));  // probes 0 .. c - 1 are below
        if (c == 0u) break;
        const uint32_t end = min(c * step, len);
        lo += (c - 1u) * step + 1u;
        len = end - ((c - 1u) * step + 1u);
    }
    // each query's place among the 64 keys from there on, and the points around it
    const uint32_t wk = lo + lane < b.n ? keys[lo + lane] : 0xFFFFFFFFu;
    uint32_t home = lo;
    for (uint32_t j = 0; j < NN_TQ; ++j) {
        const uint32_t c = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(wk < lane_u32(key, j)));
        if (lane == j) home = lo + c;
    }
    {
        constexpr int SEEDS = 8, BEFORE = 3;
        float4 c[SEEDS];
#pragma unroll
        for (int i = 0; i < SEEDS; ++i) {
            const uint32_t j = home + (uint32_t)i;
            c[i] = b.pos[j < (uint32_t)BEFORE ? 0u : min(j - (uint32_t)BEFORE, b.n - 1u)];
        }
#pragma unroll
        for (int i = 0; i < SEEDS; ++i) take(c[i].x, c[i].y, c[i].z, __float_as_uint(c[i].w));
    }
    const float far = wave_max(best, lane);
    if (!(far >= 0.0f)) return true;  // no query here
    const float ax = wave_min(fin ? q.x : INFINITY, lane), bx = wave_max(fin ? q.x : -INFINITY, lane);
    const float ay = wave_min(fin ? q.y : INFINITY, lane), by = wave_max(fin ? q.y : -INFINITY, lane);
    const float az = wave_min(fin ? q.z : INFINITY, lane), bz = wave_max(fin ? q.z : -INFINITY, lane);
    // the groups within reach, the i-th in lane i, and the lanes of the queries that need it
    uint32_t reach = 0, n = 0, my_g = 0, my_need = 0;
    for (uint32_t s0 = 0; s0 < b.supers; s0 += 64u) {
        const uint32_t s = s0 + lane;
        const float bd = box_gap2(super_box(b, min(s, b.supers - 1u)), ax, ay, az, bx, by, bz);
        unsigned long long ms = __builtin_amdgcn_ballot_w64(s < b.supers && !(bd > far));
        while (ms != 0ull) {
            const uint32_t su = s0 + (uint32_t)__ffsll((long long)ms) - 1u;
            ms &= ms - 1ull;
            const NnBox G = b.gbox[(size_t)su * 64u + lane];
            unsigned long long mg = __builtin_amdgcn_ballot_w64(!(box_gap2(G, ax, ay, az, bx, by, bz) > far));
            reach += (uint32_t)__popcll(mg);
            if (reach > NN_HARD) return false;
            while (mg != 0ull) {
                const uint32_t l = (uint32_t)__ffsll((long long)mg) - 1u;
                mg &= mg - 1ull;
                const NnBox B{make_float4(lane_f32(G.lo.x, l), lane_f32(G.lo.y, l), lane_f32(G.lo.z, l), 0.f),
                              make_float4(lane_f32(G.hi.x, l), lane_f32(G.hi.y, l), lane_f32(G.hi.z, l), 0.f)};
                const uint32_t need = (uint32_t)__builtin_amdgcn_ballot_w64(nn_needs(
                    box_gap2(B, q.x, q.y, q.z, q.x, q.y, q.z), lane_f32(G.lo.w, l), best, bi));
                if (need == 0u) continue;
                if (lane == n) {
                    my_g = su * 64u + l;
                    my_need = need;
                }
                ++n;
            }
        }
    }
    static_assert(NN_HARD <= 64 && NN_TQ <= 32, "a lane per group, a bit per query");
    if (n == 0u) return true;
    // NB groups' points in registers at a time, the next NB on their way
    constexpr uint32_t NB = 4;
    auto load = [&](uint32_t i, float4 (&c)[NB]) {
#pragma unroll
        for (uint32_t u = 0; u < NB; ++u) c[u] = b.pos[(size_t)lane_u32(my_g, min(i + u, n - 1u)) * NN_GRP + lane];
    };
    float4 next[NB];
    load(0u, next);
    for (uint32_t i0 = 0; i0 < n; i0 += NB) {
        float4 c[NB];
#pragma unroll
        for (uint32_t u = 0; u < NB; ++u) c[u] = next[u];
        if (i0 + NB < n) load(i0 + NB, next);
#pragma unroll
        for (uint32_t u = 0; u < NB; ++u) {
            if (i0 + u >= n) break;
            uint32_t need = lane_u32(my_need, i0 + u);
            while (need != 0u) {
                const uint32_t j = (uint32_t)__ffs((int)need) - 1u;
                need &= need - 1u;
                const float d = nn_dist(c[u].x, c[u].y, c[u].z, lane_f32(q.x, j), lane_f32(q.y, j), lane_f32(q.z, j));
                float bj = lane_f32(best, j);
                uint32_t ij = lane_u32(bi, j);
                if (nn_best_of(d, c[u].w, lane, bj, ij) && lane == j) {
                    best = bj;
                    bi = ij;
                }
            }
        }
    }
    return true;
}

// FP64 squared distance of a query and its match.
__device__ __forceinline__ double nn_dist64(const NnCloud& b, uint32_t bi, const float4& q) {
    const double dx = (double)b.p[3 * (size_t)bi] - (double)q.x;
    const double dy = (double)b.p[3 * (size_t)bi + 1] - (double)q.y;
    const double dz = (double)b.p[3 * (size_t)bi + 2] - (double)q.z;
    return dx * dx + dy * dy + dz * dz;
}

// Query tiles of cloud 0 against cloud 1 and, EVAL, after them those of cloud
// 1 against cloud 0; a wave per tile. EVAL: each tile's sum of the FP64
// squared distances of its matched pairs; else idx and d2 of cloud 0.
template <bool EVAL>
__global__ __launch_bounds__(256) void nn_tile_kernel(NnPlan P, uint32_t* __restrict__ idx, float* __restrict__ d2) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = (blockIdx.y * gridDim.x + blockIdx.x) * 4u +
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool back = EVAL && w >= P.c[0].qtiles;
    const NnCloud& a = P.c[back ? 1 : 0];
    const NnCloud& b = P.c[back ? 0 : 1];
    const uint32_t t = back ? w - P.c[0].qtiles : w;
    if (t >= a.qtiles) return;
    const uint32_t s = t * NN_TQ + lane;
    const bool in = lane < NN_TQ && s < a.n;
    const uint32_t sc = min(t * NN_TQ + min(lane, NN_TQ - 1u), a.n - 1u);
    // without an order the tile is of the cloud as it came, each query once
    const bool lost = *P.flag != 0u;
    float4 q = a.pos[sc];
    if (lost)
        q = make_float4(a.p[3 * (size_t)sc], a.p[3 * (size_t)sc + 1], a.p[3 * (size_t)sc + 2], __uint_as_float(sc));
    const bool fin = in && isfinite(q.x) && isfinite(q.y) && isfinite(q.z);
    float best;
    uint32_t bi;
    const bool done = nn_tile(b, lost, q, a.key[0][sc], fin, lane, best, bi);
    if (!done) {
        if (in) a.seed[s] = make_uint2(__float_as_uint(best), bi);
        if (lane == 0u) a.hard[atomicAdd(a.n_hard, 1u)] = t;
        return;
    }
    if constexpr (EVAL) {
        const double sum = wave_sum_d(in ? nn_dist64(b, bi, q) : 0.0);
        if (lane == 0u) a.part[t] = sum;
    } else if (in) {
        const uint32_t i = __float_as_uint(q.w);
        idx[i] = bi;
        d2[i] = fin ? best : INFINITY;
    }
}

// The best of up to four queries of a hard tile (bits of `left`, which they are
// taken from) over all points of b, by the whole workgroup: each lane takes
// points of its wave's share and compares each with the four queries, then the
// lanes' bests are combined in `key` (d2 bits, index). Ten instructions a pair
// where one group after another takes fifty.
__device__ __forceinline__ void nn_all_points(const NnCloud& b, uint32_t& left, const float4* s_pos,
                                              unsigned long long* s_key, uint32_t lane, uint32_t wave) {
    constexpr int N = 4;
    uint32_t q[N], bi[N];
    float x[N], y[N], z[N], bd[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        q[j] = left != 0u ? (uint32_t)__ffs((int)left) - 1u : q[0];  // (the first once more)
        left &= left - 1u;
        const float4 p = s_pos[q[j]];
        const unsigned long long k = s_key[q[j]];
        x[j] = lane_f32(p.x, 0u);  // (scalar registers)
        y[j] = lane_f32(p.y, 0u);
        z[j] = lane_f32(p.z, 0u);
        bd[j] = __uint_as_float((uint32_t)(k >> 32));
        bi[j] = (uint32_t)k;
    }
    // (whole groups of 64 points, NaN past the last)
    const uint32_t groups = (b.n + (uint32_t)NN_GRP - 1u) / (uint32_t)NN_GRP;
    for (uint32_t g = wave; g < groups; g += NN_TQ) {
        const float4 c = b.pos[(size_t)g * NN_GRP + lane];
        const uint32_t id = __float_as_uint(c.w);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float d = nn_dist(c.x, c.y, c.z, x[j], y[j], z[j]);
            if (d < bd[j] || (d == bd[j] && id < bi[j])) {
                bd[j] = d;
                bi[j] = id;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const unsigned long long k = wave_umin(((unsigned long long)__float_as_uint(bd[j]) << 32) | bi[j]);
        if (lane == 0u) atomicMin(&s_key[q[j]], k);
    }
}

// Queries of the hard tiles, a wave each: the nearest supers first, and in
// each the nearest groups first, four at a time, until the next box is
// farther than the best. A query that has evaluated NN_FAR_MOST groups (or more,
// by NN_FAR_SHARE) stops there: the points lie about as far from it in all
// directions, or in no useful order. The workgroup then takes such queries of its
// tile over all points together. It bounds what such clouds cost: 60000 queries
// in the middle of a shell of 60000 points take 1290 us so, without it 4870, all
// pairs 640. Clouds that lie apart stay below the line: 18000 points and 18000
// take 115 us, with a line at 24 groups 204 (all pairs 77).
// The minima over the wave go by DPP: with exchanges through the LDS unit two
// calls took 73.1 and 148.7 us, so 71.3 and 144.8 (metrics of an object of 20k
// points and a 120k sweep).
template <bool EVAL>
__global__ __launch_bounds__(64 * NN_TQ, 8) void nn_far_kernel(NnPlan P, uint32_t* __restrict__ idx,
                                                            float* __restrict__ d2) {
    __shared__ double s_e[NN_TQ];
    __shared__ float4 s_pos[NN_TQ];
    __shared__ unsigned long long s_key[NN_TQ];
    __shared__ uint32_t s_stop[NN_TQ];
    const uint32_t lane = threadIdx.x & 63u, wq = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t h0 = *P.c[0].n_hard, h1 = EVAL ? *P.c[1].n_hard : 0u;
    for (uint32_t h = blockIdx.x; h < h0 + h1; h += gridDim.x) {
        const bool back = h >= h0;
        const NnCloud& a = P.c[back ? 1 : 0];
        const NnCloud& b = P.c[back ? 0 : 1];
        const uint32_t t = a.hard[back ? h - h0 : h];
        const uint32_t s = t * NN_TQ + wq;
        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
        float best = -1.0f;
        uint32_t bi = 0;
        bool fin = false, stop = false;
        auto put = [&]() {  // the query's answer (lane 0)
            if constexpr (EVAL) {
                s_e[wq] = nn_dist64(b, bi, q);
            } else {
                const uint32_t i = __float_as_uint(q.w);
                idx[i] = bi;
                d2[i] = fin ? best : INFINITY;
            }
        };
        if (s < a.n) {
            q = a.pos[s];
            best = __uint_as_float(a.seed[s].x);
            bi = a.seed[s].y;
            fin = best >= 0.0f;
            const uint32_t most = max(NN_FAR_MOST, b.n / ((uint32_t)NN_GRP * NN_FAR_SHARE));
            uint32_t seen = 0;  // groups evaluated
            for (uint32_t s0 = 0; fin && !stop && s0 < b.supers; s0 += 64u) {
                const bool sok = s0 + lane < b.supers;
                const float sd = box_gap2(super_box(b, sok ? s0 + lane : s0), q.x, q.y, q.z, q.x, q.y, q.z);
                unsigned long long left = __builtin_amdgcn_ballot_w64(sok);
                while (left != 0ull && !stop) {
                    // the nearest super left (an unordered distance, from NaN boxes there are none, counts as far)
                    const float ds = ((left >> lane) & 1ull) ? sd : INFINITY;
                    const float ms = wave_fmin(ds);
                    if (ms > best) break;
                    const uint32_t l = (uint32_t)__ffsll((long long)(left & __builtin_amdgcn_ballot_w64(ds == ms))) - 1u;
                    left &= ~(1ull << l);
                    const uint32_t su = s0 + l;
                    const NnBox G = b.gbox[(size_t)su * 64u + lane];
                    const float gd = box_gap2(G, q.x, q.y, q.z, q.x, q.y, q.z);
                    unsigned long long lg = ~0ull;
                    bool more = true;
                    while (more && lg != 0ull) {
                        if (seen >= most) {
                            stop = true;
                            break;
                        }
                        constexpr int NB = 4;
                        float4 c[NB];
                        float dg[NB];
                        int nb = 0;
                        lg &= __builtin_amdgcn_ballot_w64(nn_needs(gd, G.lo.w, best, bi));
#pragma unroll
                        for (int u = 0; u < NB; ++u) {
                            const float dl = ((lg >> lane) & 1ull) ? gd : INFINITY;
                            dg[u] = wave_fmin(dl);
                            const unsigned long long m = lg & __builtin_amdgcn_ballot_w64(dl == dg[u]);
                            if (!more || m == 0ull || dg[u] > best) {
                                more = false;
                            } else {
                                const uint32_t g = (uint32_t)__ffsll((long long)m) - 1u;
                                lg &= ~(1ull << g);
                                c[u] = b.pos[((size_t)su * 64u + g) * NN_GRP + lane];
                                ++nb;
                            }
                        }
                        seen += (uint32_t)nb;
#pragma unroll
                        for (int u = 0; u < NB; ++u) {
                            if (u >= nb || dg[u] > best) break;
                            (void)nn_best_of(nn_dist(c[u].x, c[u].y, c[u].z, q.x, q.y, q.z), c[u].w, lane, best, bi);
                        }
                    }
                }
            }
            if (lane == 0u) {
                if (stop) {
                    s_pos[wq] = q;
                    s_key[wq] = ((unsigned long long)__float_as_uint(best) << 32) | bi;
                } else {
                    put();
                }
            }
        } else if (EVAL && lane == 0u) {
            s_e[wq] = 0.0;
        }
        if (lane == 0u) s_stop[wq] = stop ? 1u : 0u;
        __syncthreads();
        uint32_t open = (uint32_t)__builtin_amdgcn_ballot_w64(lane < NN_TQ && s_stop[lane % NN_TQ] != 0u);
        if (open != 0u) {
            while (open != 0u) nn_all_points(b, open, s_pos, s_key, lane, wq);
            __syncthreads();
            if (stop && lane == 0u) {
                best = __uint_as_float((uint32_t)(s_key[wq] >> 32));
                bi = (uint32_t)s_key[wq];
                put();
            }
            __syncthreads();
        }
        if constexpr (EVAL) {
            if (threadIdx.x == 0) {
                double sum = 0.0;
                for (uint32_t i = 0; i < NN_TQ; ++i) sum += s_e[i];
                a.part[t] = sum;
            }
        }
        __syncthreads();  // the LDS words are rewritten for the next tile
    }
}

// Sums of NN_SUM_TILES tile sums each (clouds of more tiles than one block adds up).
__global__ __launch_bounds__(1024) void nn_sum_kernel(NnPlan P) {
    __shared__ double s_s[16];
    const uint32_t n0 = (P.c[0].qtiles + NN_SUM_TILES - 1) / NN_SUM_TILES;
    const bool second = blockIdx.x >= n0;
    const NnCloud& c = P.c[second ? 1 : 0];
    const uint32_t blk = second ? blockIdx.x - n0 : blockIdx.x;
    const uint32_t end = min(c.qtiles, (blk + 1u) * NN_SUM_TILES);
    double s = 0.0;
    for (uint32_t i = blk * NN_SUM_TILES + threadIdx.x; i < end; i += 1024u) s += c.part[i];
    s = wave_sum_d(s);
    if ((threadIdx.x & 63u) == 0u) s_s[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < 16; ++i) t += s_s[i];
        c.part2[blk] = t;
    }
}

// One block: the metrics from the tile sums (`two`: from the sums of them)
// and the clean cloud's box records.
__global__ __launch_bounds__(1024) void nn_metrics_kernel(NnPlan P, bool two, double* __restrict__ out) {
    __shared__ double s_s[16][2];
    __shared__ float s_v[4][6];
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    float x[6];
    if (w < 4u) {
        const uint32_t r = min(threadIdx.x, P.c[0].box_blocks - 1u);
#pragma unroll
        for (int i = 0; i < 6; ++i) x[i] = P.c[0].rec[(size_t)r * NN_REC + 6 + i];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const NnCloud& c = P.c[q];
        const double* __restrict__ part = two ? c.part2 : c.part;
        const uint32_t n = two ? (c.qtiles + NN_SUM_TILES - 1) / NN_SUM_TILES : c.qtiles;
        constexpr uint32_t U = 4;
        double s = 0.0;
        for (uint32_t i0 = threadIdx.x; i0 < n; i0 += U * 1024u) {
            double v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = part[min(i0 + u * 1024u, n - 1u)];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (i0 + u * 1024u < n) s += v[u];
        }
        s = wave_sum_d(s);
        if (lane == 0u) s_s[w][q] = s;
    }
    if (w < 4u) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const float v = i < 3 ? wave_min(x[i], lane) : wave_max(x[i], lane);
            if (lane == 0u) s_v[w][i] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double m2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            float l = s_v[0][a], h = s_v[0][3 + a];
            for (int q = 1; q < 4; ++q) {
                l = fminf(l, s_v[q][a]);
                h = fmaxf(h, s_v[q][3 + a]);
            }
            m2 += ((double)h - (double)l) * ((double)h - (double)l);
        }
        double sc = 0.0, sd = 0.0;
        for (int i = 0; i < 16; ++i) {
            sc += s_s[i][0];
            sd += s_s[i][1];
        }
        const double mse = sc / (double)P.c[0].n;
        out[0] = mse;
        out[1] = sd / (double)P.c[1].n;
        out[2] = out[0] + out[1];
        out[3] = 10.0 * log10(m2 / mse);
    }
}
static_assert(NN_BOX_BLOCKS <= 256, "the metrics kernel reads one box record per thread of four waves");

__global__ void nn_lose_kernel(uint32_t* flag) { *flag = 1u; }

// Hilbert order, groups and boxes of both clouds. `lose`: no order is made, as
// if a wait of the radix passes had expired.
void nn_sort(const NnPlan& P, bool lose, hipStream_t st) {
    hipLaunchKernelGGL(nn_box_kernel, dim3(P.c[0].box_blocks + P.c[1].box_blocks + 1u), dim3(256), 0, st, P);
    hipLaunchKernelGGL(P.passes == 3 ? nn_key_kernel<3> : nn_key_kernel<NN_PASSES_MAX>,
                       dim3(P.c[0].key_blocks + P.c[1].key_blocks), dim3(256), 0, st, P);
    if (lose) hipLaunchKernelGGL(nn_lose_kernel, dim3(1), dim3(1), 0, st, P.flag);
    for (int pass = 0; pass < P.passes && !lose; ++pass) {
        auto kern = P.tile == 1024u ? (pass == 0 ? nn_radix_kernel<4, 256, true> : nn_radix_kernel<4, 256, false>)
                    : P.tile == 2048u ? (pass == 0 ? nn_radix_kernel<4, 512, true> : nn_radix_kernel<4, 512, false>)
                                      : (pass == 0 ? nn_radix_kernel<8, 512, true> : nn_radix_kernel<8, 512, false>);
        hipLaunchKernelGGL(kern, dim3(P.c[0].tiles + P.c[1].tiles), dim3(P.tile == 1024u ? 256 : 512), 0, st, P, pass);
    }
    hipLaunchKernelGGL(nn_gather_kernel, dim3((P.c[0].supers + P.c[1].supers) * (unsigned)(NN_SUP / NN_GATHER)),
                       dim3(NN_GATHER), 0, st, P);
}

template <bool EVAL>
void nn_search(const NnPlan& P, uint32_t* idx, float* d2, hipStream_t st) {
    const uint32_t tiles = P.c[0].qtiles + (EVAL ? P.c[1].qtiles : 0u);
    // (a grid dimension holds fewer than 2^32 threads, and a query takes four)
    constexpr uint32_t ROW = 1u << 22;
    const uint32_t blocks = (tiles + 3u) / 4u;
    hipLaunchKernelGGL(nn_tile_kernel<EVAL>, dim3(std::min(blocks, ROW), (blocks + ROW - 1u) / ROW), dim3(256), 0, st, P,
                       idx, d2);
    hipLaunchKernelGGL(nn_far_kernel<EVAL>, dim3(tiles < NN_FAR_BLOCKS ? tiles : NN_FAR_BLOCKS), dim3(64 * NN_TQ), 0, st,
                       P, idx, d2);
}

// Whether sorting pays for na queries in nb points (1 direction) or both clouds
// in each other (2). Brute force takes 0.21 us a million pairs; the sort and the
// search of groups are eight to ten launches, 55 to 70 us, and then some 0.24 us
// a thousand queries and 0.07 a thousand reference points; few queries or few
// reference points spread them over less of the chip. Brute force against
// groups, on a shell and a LiDAR sweep: nearest 15000 in 15000 points 58 us and
// 55 / 67, 18000 in 18000 82 and 57 / 69; 3000 in 100k 78 and 88 / 109, 5000 in
// 100k 118 and 108; 100 in 10M 540 and 713, 700 in 3M 474 and 275; 100k in 3000
// 73 and 86 / 117, 300k in 3000 196 and 135 / 167; 10M in 300 608 and 2047, 10M
// in 1500 2730 and 2104; metrics of 11500 and 11500 points 66 and 59 / 70, 12500
// and 12500 80 and 59 / 74, 3000 and 50k 78 and 90 / 102, 1M and 1000 405 and
// 316 / 343, 1M and 500 212 and 310.
constexpr uint32_t NN_EVEN = 8;  // clouds up to this many times the size of the other
bool nn_groups_pay(uint32_t na, uint32_t nb, uint32_t directions) {
    const uint64_t pairs = (uint64_t)na * nb * directions;
    if (directions == 2u) return pairs >= 260'000'000ull + 1300ull * ((uint64_t)na + nb);
    const bool even = std::max(na, nb) / NN_EVEN <= std::min(na, nb);
    return pairs >= (even ? 240'000'000ull : 310'000'000ull) + 1100ull * na + 300ull * nb;
}

// Whether it pays for any two clouds up to these sizes, for the workspaces: where
// it pays at all it pays for all larger clouds, but for even ones that grow
// uneven.
bool nn_groups_pay_within(uint32_t na, uint32_t nb, uint32_t directions) {
    constexpr uint32_t most = NN_EVEN, rest = NN_EVEN - 1u;  // the largest even clouds within
    return nn_groups_pay(na, nb, directions) ||
           nn_groups_pay((uint32_t)std::min<uint64_t>(na, (uint64_t)most * nb + rest),
                         (uint32_t)std::min<uint64_t>(nb, (uint64_t)most * na + rest), directions);
}

// Whether the search goes by groups: it pays, and the workspace holds the
// sorted clouds.
bool nn_by_groups(uint32_t na, uint32_t nb, uint32_t directions, size_t ws_bytes) {
    return nn_groups_pay(na, nb, directions) && nn_plan(nullptr, na, nullptr, nb, nullptr).bytes <= ws_bytes;
}

// Workspace bytes of the groups: the largest layout of any two clouds up to
// these sizes. (Just below an edge of the radix tiles there are more tiles, and
// look-back words, than just above it, and a workspace kept for larger clouds
// must not send those to brute force.)
size_t nn_groups_bytes(uint32_t na, uint32_t nb) {
    size_t bytes = nn_plan(nullptr, na, nullptr, nb, nullptr).bytes;
    for (const uint32_t edge : SORT_TILE_EDGES)
        if (edge < std::max(na, nb))
            bytes = std::max(bytes, nn_plan(nullptr, std::min(na, edge), nullptr, std::min(nb, edge), nullptr).bytes);
    return bytes;
}

}  // namespace

size_t nearest_workspace_bytes(uint32_t na) { return al256((size_t)8 * na); }

size_t nearest_best_workspace_bytes(uint32_t na, uint32_t nb) {
    const size_t brute = nearest_workspace_bytes(na);
    return nn_groups_pay_within(na, nb, 1u) ? std::max(brute, nn_groups_bytes(na, nb)) : brute;
}

// Brute-force keys of one direction, or of both in one launch each.
static void launch_nearest_keys(NnDir d0, NnDir d1, hipStream_t st) {
    const unsigned dirs = d1.key ? 2u : 1u;
    unsigned qb = 1, total = 0;
    for (unsigned i = 0; i < dirs; ++i) {
        NnDir& d = i ? d1 : d0;
        d.blocks = (d.na + NN_BLOCK - 1) / NN_BLOCK;
        const unsigned tiles = (d.nb + NN_TILE - 1) / NN_TILE;
        unsigned s = (NN_MIN_BLOCKS + d.blocks - 1) / d.blocks;
        if (s > tiles) s = tiles;
        if (s < 1) s = 1;
        d.chunk = ((d.nb + s - 1) / s + NN_TILE - 1) / NN_TILE * NN_TILE;
        d.chunks = (d.nb + d.chunk - 1) / d.chunk;
        qb = std::max(qb, d.blocks);
        total += d.blocks * d.chunks;
    }
    unsigned ib = qb;
    if (ib > 4096) ib = 4096;
    hipLaunchKernelGGL(nn_init_kernel, dim3(ib, 1, dirs), dim3(256), 0, st, d0, d1);
    hipLaunchKernelGGL(nn_kernel, dim3(total), dim3(NN_BLOCK), 0, st, d0, d1);
}

void launch_nearest(const float* a, uint32_t na, const float* b, uint32_t nb, void* ws, size_t ws_bytes, uint32_t* idx,
                    float* d2, bool lose_order, hipStream_t st) {
    if (nn_by_groups(na, nb, 1u, ws_bytes)) {
        const NnPlan P = nn_plan(a, na, b, nb, (char*)ws);
        nn_sort(P, lose_order, st);
        nn_search<false>(P, idx, d2, st);
        return;
    }
    unsigned long long* key = (unsigned long long*)ws;
    launch_nearest_keys(NnDir{a, b, na, nb, 0u, 0u, 0u, key}, NnDir{}, st);
    unsigned ob = (na + 255) / 256;
    if (ob > 4096) ob = 4096;
    hipLaunchKernelGGL(nn_out_kernel, dim3(ob), dim3(256), 0, st, key, na, idx, d2);
}

size_t eval_min_workspace_bytes(uint32_t nc, uint32_t nd) {
    return al256((size_t)8 * nc) + al256((size_t)8 * nd) + 2 * al256((size_t)8 * EV_STRIDE * EV_BLOCKS_MAX);
}

// (enough for gdn_nearest too)
size_t eval_workspace_bytes(uint32_t nc, uint32_t nd) {
    const size_t brute = eval_min_workspace_bytes(nc, nd);
    return nn_groups_pay_within(nc, nd, 1u) || nn_groups_pay(nc, nd, 2u) ? std::max(brute, nn_groups_bytes(nc, nd)) : brute;
}

void launch_eval(const float* clean, uint32_t nc, const float* den, uint32_t nd, void* ws, size_t ws_bytes, double* out,
                 bool lose_order, hipStream_t st) {
    if (nn_by_groups(nc, nd, 2u, ws_bytes)) {
        const NnPlan P = nn_plan(clean, nc, den, nd, (char*)ws);
        nn_sort(P, lose_order, st);
        nn_search<true>(P, nullptr, nullptr, st);
        auto sums = [](uint32_t t) { return (t + NN_SUM_TILES - 1) / NN_SUM_TILES; };
        const bool two = P.c[0].qtiles > NN_SUM_TILES || P.c[1].qtiles > NN_SUM_TILES;
        if (two)
            hipLaunchKernelGGL(nn_sum_kernel, dim3(sums(P.c[0].qtiles) + sums(P.c[1].qtiles)), dim3(1024), 0, st, P);
        hipLaunchKernelGGL(nn_metrics_kernel, dim3(1), dim3(1024), 0, st, P, two, out);
        return;
    }
    char* w = (char*)ws;
    unsigned long long* kc = (unsigned long long*)w;
    w += al256((size_t)8 * nc);
    unsigned long long* kd = (unsigned long long*)w;
    w += al256((size_t)8 * nd);
    double* pc = (double*)w;
    w += al256((size_t)8 * EV_STRIDE * EV_BLOCKS_MAX);
    double* pd = (double*)w;
    const NnDir d0{clean, den, nc, nd, 0u, 0u, 0u, kc}, d1{den, clean, nd, nc, 0u, 0u, 0u, kd};
    launch_nearest_keys(d0, d1, st);
    const unsigned bc = ev_blocks(nc), bd = ev_blocks(nd);
    hipLaunchKernelGGL(ev_sum_kernel, dim3(bc + bd), dim3(EV_BLOCK), 0, st, d0, d1, bc, pc, pd);
    hipLaunchKernelGGL(ev_final_kernel, dim3(1), dim3(64), 0, st, pc, bc, pd, bd, nc, nd, out);
}

}  // namespace gdn
