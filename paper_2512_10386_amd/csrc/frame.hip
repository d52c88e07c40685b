// Frame-level passes: zero-fill of the workspace control block, the frame
// bounding box (the octree root cube, Sec. 3 with Eq. 2), 63-bit Morton keys,
// the stable LSD radix sort of (key, original index) on the digits the octree
// needs, and the whole-key re-sort of deep level-10 cells.
#include <type_traits>

#include "kernels.hpp"
#include "radix.hpp"
#include "tree.hpp"
#include "wave.hpp"

namespace gdn {

// ---------------------------------------------------------------- zero fill, frame table

// Checked copy of the caller's frame offsets (int64[nf+1]): clamped to [0, n]
// and made non-decreasing (a running maximum), with foff[0] = 0 and
// foff[nf] = n. Any repair sets DEV_BAD_FRAMES; the batch is then processed
// with the repaired table (memory-safe, results unspecified). One workgroup;
// it also writes the first 16 bytes of the counters, the status word among
// them, which are otherwise zero.
__device__ __forceinline__ void frame_table(const int64_t* __restrict__ in, uint32_t nf, uint32_t n, uint32_t* foff,
                                            Counters* c) {
    __shared__ uint32_t s_max[4];
    constexpr uint32_t PER = (MAX_FRAMES + 1 + 255) / 256;
    const uint32_t t = threadIdx.x, b0 = t * PER;
    uint32_t v[PER];
    uint32_t m = 0, bad = 0;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        const uint32_t f = b0 + i;
        uint32_t x = 0;
        if (f <= nf) {
            const int64_t r = in[f];
            x = r < 0 ? 0u : (r > (int64_t)n ? n : (uint32_t)r);
            if (r < 0 || r > (int64_t)n) bad = 1;
            if (f == 0 && r != 0) bad = 1;
            if (f == nf && r != (int64_t)n) bad = 1;
            if (f > 0 && r < in[f - 1]) bad = 1;
        }
        m = x > m ? x : m;
        v[i] = m;  // running max within this thread's entries
    }
    // max over earlier threads: of this wave by a scan, of the waves before it
    const uint32_t inc = wave_incl_max(m);
    if ((t & 63u) == 63u) s_max[t >> 6] = inc;
    __syncthreads();
    uint32_t pre = (uint32_t)__shfl_up((int)inc, 1, 64);
    if ((t & 63u) == 0u) pre = 0u;
    for (uint32_t w = 0; w < (t >> 6); ++w) pre = s_max[w] > pre ? s_max[w] : pre;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        const uint32_t f = b0 + i;
        if (f <= nf) {
            uint32_t x = v[i] > pre ? v[i] : pre;
            if (f == 0) x = 0u;
            if (f == nf) x = n;
            foff[f] = x;
        }
    }
    const int any = __syncthreads_or((int)bad);
    static_assert(offsetof(Counters, status) == 0, "the status word opens the counters");
    if (t == 0) *(uint4*)c = make_uint4(any ? DEV_BAD_FRAMES : 0u, 0u, 0u, 0u);
}

// Clears the zeroed block (the counters first). A batch's frame table is made
// beside it by workgroup 0 (as a launch of its own it took 5 us of a batch of
// 12 objects' 232).
template <bool BATCH>
__global__ __launch_bounds__(256) void zero_kernel(Plan P, uint4* p, size_t n16, const int64_t* __restrict__ frame_off) {
    if (BATCH && blockIdx.x == 0) {
        frame_table(frame_off, P.nf, P.n, P.foff, P.ctr);
        return;
    }
    constexpr size_t B = BATCH ? 1 : 0;  // blocks and words that are the table's
    for (size_t i = B + (blockIdx.x - B) * (size_t)blockDim.x + threadIdx.x; i < n16; i += (gridDim.x - B) * (size_t)blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
    if (!BATCH && blockIdx.x == 0 && threadIdx.x == 0) {
        P.foff[0] = 0u;
        P.foff[1] = P.n;
    }
}

void launch_zero(const Plan& P, const int64_t* frame_off, hipStream_t st) {
    size_t n16 = P.zero_bytes / 16;
    unsigned blocks = (unsigned)((n16 + 255) / 256);
    if (blocks > 2048) blocks = 2048;
    if (blocks == 0) blocks = 1;
    if (frame_off)
        hipLaunchKernelGGL(zero_kernel<true>, dim3(blocks + 1), dim3(256), 0, st, P, (uint4*)P.zero_begin, n16, frame_off);
    else
        hipLaunchKernelGGL(zero_kernel<false>, dim3(blocks), dim3(256), 0, st, P, (uint4*)P.zero_begin, n16, frame_off);
}

// ---------------------------------------------------------------- bbox

// Waves take chunks of BBOX_CHUNK consecutive points (coalesced). A chunk
// inside one frame writes its reduced box to bbox_part[chunk] and a second
// kernel folds each frame's chunks (no contended atomics); a chunk across a
// frame border (at most nf - 1 of them) reduces each of its frames over the
// wave and adds them with atomics. With few chunks (`direct`) every chunk
// uses the atomics and there is no fold. Batches also record each point's
// frame.
constexpr uint32_t BBOX_CHUNK = 1024;

__device__ __forceinline__ void bbox_reduce_wave(float* mn, float* mx, uint32_t& bad) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        mn[a] = wave_fmin(mn[a]);
        mx[a] = wave_fmax(mx[a]);
    }
    bad = wave_sum(bad);
}

// Adds the points [lo, hi) to a lane's box (non-finite points are counted
// in `bad` instead), lane l taking points lo + l, lo + l + 64, ... in that
// order; BBOX_U loads per lane are issued before any is used (a lane past hi
// reads the last point and drops it). With fid, also records frame f of each
// point.
constexpr int BBOX_U = 8;
__device__ __forceinline__ void bbox_add_range(const float* __restrict__ xyz, uint32_t lo, uint32_t hi,
                                               uint32_t lane, float* mn, float* mx, uint32_t& bad, uint32_t* fid,
                                               uint32_t f) {
    for (uint32_t i0 = lo + lane; i0 < hi; i0 += 64u * BBOX_U) {
        float x[BBOX_U], y[BBOX_U], z[BBOX_U];
#pragma unroll
        for (int u = 0; u < BBOX_U; ++u) {
            const size_t j = min(i0 + 64u * (uint32_t)u, hi - 1u);
            x[u] = xyz[3 * j];
            y[u] = xyz[3 * j + 1];
            z[u] = xyz[3 * j + 2];
        }
#pragma unroll
        for (int u = 0; u < BBOX_U; ++u) {
            const uint32_t i = i0 + 64u * (uint32_t)u;
            const bool in = i < hi;
            const bool fin = isfinite(x[u]) && isfinite(y[u]) && isfinite(z[u]);
            const bool ok = in && fin;
            mn[0] = fminf(mn[0], ok ? x[u] : INFINITY); mx[0] = fmaxf(mx[0], ok ? x[u] : -INFINITY);
            mn[1] = fminf(mn[1], ok ? y[u] : INFINITY); mx[1] = fmaxf(mx[1], ok ? y[u] : -INFINITY);
            mn[2] = fminf(mn[2], ok ? z[u] : INFINITY); mx[2] = fmaxf(mx[2], ok ? z[u] : -INFINITY);
            bad += (in && !fin) ? 1u : 0u;
            if (fid && in) fid[i] = f;
        }
    }
}

__global__ __launch_bounds__(256) void bbox_kernel(const float* __restrict__ xyz, Plan P, bool direct,
                                                   uint32_t chunk) {
    __shared__ uint32_t s_foff[MAX_FRAMES + 1];
    const uint32_t n = P.n, nf = P.nf;
    if (nf > 1) {
        for (uint32_t f = threadIdx.x; f <= nf; f += blockDim.x) s_foff[f] = P.foff[f];
        __syncthreads();
    }
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wid = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t nchunks = (n + chunk - 1) / chunk;
    for (uint32_t c = wid; c < nchunks; c += nw) {
        const uint32_t base = c * chunk, end = min(n, base + chunk);
        const uint32_t f0 = nf > 1 ? frame_of(s_foff, nf, base) : 0u;
        const uint32_t f1 = nf > 1 ? frame_of(s_foff, nf, end - 1u) : 0u;
        for (uint32_t f = f0; f <= f1; ++f) {
            const uint32_t lo = f == f0 ? base : max(base, s_foff[f]);
            const uint32_t hi = f == f1 ? end : min(end, s_foff[f + 1]);
            float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
            uint32_t bad = 0;
            bbox_add_range(xyz, lo, hi, lane, mn, mx, bad, nf > 1 ? P.fid : nullptr, f);
            bbox_reduce_wave(mn, mx, bad);
            if (f0 == f1 && !direct) {
                // whole chunk in one frame: ordered-uint max of -min / max, bad count
                uint32_t* part = P.bbox_part + 8 * (size_t)c;
                if (lane < 3u) {
                    part[lane] = mn[lane] <= mx[lane] ? ~f32_ordered(mn[lane]) : 0u;
                    part[3 + lane] = mn[lane] <= mx[lane] ? f32_ordered(mx[lane]) : 0u;
                }
                if (lane == 3u) part[6] = bad;
            } else {
                FrameStat* fs = P.fstat + f;
                if (lane < 3u && mn[lane] <= mx[lane]) {
                    atomicMax(&fs->bbox_nmin[lane], ~f32_ordered(mn[lane]));
                    atomicMax(&fs->bbox_max[lane], f32_ordered(mx[lane]));
                }
                if (lane == 3u && bad) {
                    atomicAdd(&fs->nonfinite, bad);
                    atomicOr(&P.ctr->status, DEV_NONFINITE);
                }
            }
        }
    }
}

// A single frame with few points: each wave reduces its 512-point chunks and
// the block combines its four waves; each block writes its box (ordered-uint
// max of -min and max) and non-finite count to bbox_part[block], which the
// Morton kernel folds (no atomics, so the accumulators need no clearing). On a
// plain call the blocks also clear the workspace's zeroed block (counters,
// histograms, look-back status words: nothing here uses them) and write the
// one-frame offset table, in place of a separate fill launch.
__global__ __launch_bounds__(256) void bbox_one_kernel(const float* __restrict__ xyz, Plan P, uint32_t chunk,
                                                       bool clear) {
    __shared__ float s_mn[4][3], s_mx[4][3];
    __shared__ uint32_t s_bad[4];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t wid = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t n = P.n, nchunks = (n + chunk - 1) / chunk;
    if (clear) {
        uint4* z = (uint4*)P.zero_begin;
        const size_t n16 = P.zero_bytes / 16;
        for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
            z[i] = make_uint4(0u, 0u, 0u, 0u);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            P.foff[0] = 0u;
            P.foff[1] = n;
        }
    }
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    uint32_t bad = 0;
    for (uint32_t c = wid; c < nchunks; c += nw)
        bbox_add_range(xyz, c * chunk, min(n, (c + 1u) * chunk), lane, mn, mx, bad, nullptr, 0u);
    bbox_reduce_wave(mn, mx, bad);
    if (lane == 0u) {
        for (int a = 0; a < 3; ++a) {
            s_mn[wave][a] = mn[a];
            s_mx[wave][a] = mx[a];
        }
        s_bad[wave] = bad;
    }
    __syncthreads();
    uint32_t* part = P.bbox_part + 8 * (size_t)blockIdx.x;
    if (threadIdx.x < 3u) {
        const uint32_t a = threadIdx.x;
        float lo = s_mn[0][a], hi = s_mx[0][a];
        for (int w = 1; w < 4; ++w) {
            lo = fminf(lo, s_mn[w][a]);
            hi = fmaxf(hi, s_mx[w][a]);
        }
        part[a] = lo <= hi ? ~f32_ordered(lo) : 0u;
        part[3 + a] = lo <= hi ? f32_ordered(hi) : 0u;
    }
    if (threadIdx.x == 3u) part[6] = s_bad[0] + s_bad[1] + s_bad[2] + s_bad[3];
}

// One wave per frame: fold the frame's whole chunks into its accumulators.
__global__ __launch_bounds__(256) void bbox_fold_kernel(Plan P) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wid = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t f = wid; f < P.nf; f += nw) {
        const uint32_t fs = P.foff[f], fe = P.foff[f + 1];
        const uint32_t c0 = (fs + BBOX_CHUNK - 1) / BBOX_CHUNK;
        const uint32_t c1 = fe == P.n ? (fe + BBOX_CHUNK - 1) / BBOX_CHUNK : fe / BBOX_CHUNK;
        uint32_t v[7] = {0u, 0u, 0u, 0u, 0u, 0u, 0u};
        for (uint32_t c = c0 + lane; c < c1; c += 64u) {
            const uint32_t* part = P.bbox_part + 8 * (size_t)c;
#pragma unroll
            for (int a = 0; a < 6; ++a) v[a] = max(v[a], part[a]);
            v[6] += part[6];
        }
#pragma unroll
        for (int a = 0; a < 6; ++a) v[a] = wave_umax(v[a]);
        v[6] = wave_sum(v[6]);
        FrameStat* st = P.fstat + f;
        if (lane < 3u) {
            if (v[lane]) atomicMax(&st->bbox_nmin[lane], v[lane]);
            if (v[3 + lane]) atomicMax(&st->bbox_max[lane], v[3 + lane]);
        }
        if (lane == 3u && v[6]) atomicAdd(&st->nonfinite, v[6]);
        if (lane == 4u && (v[6] || st->nonfinite)) atomicOr(&P.ctr->status, DEV_NONFINITE);
    }
}

// Few points: 512-point chunks (one wave each, enough waves to cover the
// load latency); otherwise BBOX_CHUNK chunks and the fold.
static bool bbox_direct(const Plan& P) { return P.n <= (1u << 20); }
static unsigned bbox_blocks(const Plan& P) {
    const uint32_t chunk = bbox_direct(P) ? 512u : BBOX_CHUNK;
    const uint32_t nchunks = (P.n + chunk - 1) / chunk;
    unsigned blocks = (nchunks + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    return blocks ? blocks : 1u;
}
bool bbox_one_frame(const Plan& P) { return bbox_direct(P) && P.nf == 1; }

void launch_bbox(const Plan& P, const float* xyz, hipStream_t st, bool clear) {
    const bool direct = bbox_direct(P);
    const uint32_t chunk = direct ? 512u : BBOX_CHUNK;
    const unsigned blocks = bbox_blocks(P);
    if (bbox_one_frame(P)) {
        hipLaunchKernelGGL(bbox_one_kernel, dim3(blocks), dim3(256), 0, st, xyz, P, chunk, clear);
        return;
    }
    hipLaunchKernelGGL(bbox_kernel, dim3(blocks), dim3(256), 0, st, xyz, P, direct, chunk);
    if (direct) return;
    unsigned fb = (P.nf + 3) / 4;
    if (fb > 1024) fb = 1024;
    hipLaunchKernelGGL(bbox_fold_kernel, dim3(fb), dim3(256), 0, st, P);
}

// ---------------------------------------------------------------- Morton keys

// Frame constants of every frame of a large batch (one thread per frame); with
// up to FC_LDS frames each block of the key kernel computes them itself.
constexpr uint32_t FC_LDS = 64;
__global__ __launch_bounds__(256) void frame_const_kernel(Plan P, double min_leaf_side) {
    for (uint32_t f = threadIdx.x; f < P.nf; f += blockDim.x) frame_consts(P.fstat + f, min_leaf_side, P.fc + f);
}

// Keys (quantised with the point's own frame constants) and the digit
// histograms of the sort: key digits 4..7, then the frame id digits of a batch
// (from the frame table). A single frame computes its constants per block.
constexpr uint32_t MORTON_U = 8;
// nparts > 0: a single frame whose box is in nparts per-block records of
// bbox_one_kernel, folded here by every block (block 0 also stores the
// frame's statistics and constants and flags non-finite input).
// FRAMES: 1 for a single frame, otherwise FC_LDS or MAX_FRAMES, the most there
// can be.
template <uint32_t FRAMES>
__global__ __launch_bounds__(256) void morton_kernel(const float* __restrict__ xyz, Plan P, double min_leaf_side,
                                                     uint32_t nparts) {
    constexpr bool one = FRAMES == 1, fc_lds = FRAMES == FC_LDS;
    __shared__ FrameConst s_fc;
    __shared__ FrameConst s_fcs[fc_lds ? FC_LDS : 1];
    __shared__ FrameStat s_stat;
    if (fc_lds && threadIdx.x < P.nf) {
        frame_consts(P.fstat + threadIdx.x, min_leaf_side, s_fcs + threadIdx.x);
        if (blockIdx.x == 0) P.fc[threadIdx.x] = s_fcs[threadIdx.x];
    }
    __shared__ uint32_t s_hist[SORT_PASSES_MAX][256];
    const uint32_t n = P.n, nh = P.sort_passes;
    // MORTON_U points per thread at a time, their loads issued before any is
    // used (a point past n reads the last one and is dropped), the first ones
    // beside the fold of the boxes
    const uint32_t stride = gridDim.x * blockDim.x;
    uint32_t i0 = blockIdx.x * blockDim.x + threadIdx.x;
    float x[MORTON_U], y[MORTON_U], z[MORTON_U];
    uint32_t f[MORTON_U];
    auto load = [&]() {
#pragma unroll
        for (int u = 0; u < MORTON_U; ++u) {
            const uint32_t j = min(i0 + (uint32_t)u * stride, n - 1u);
            x[u] = xyz[3 * (size_t)j];
            y[u] = xyz[3 * (size_t)j + 1];
            z[u] = xyz[3 * (size_t)j + 2];
            f[u] = one ? 0u : P.fid[j];
        }
    };
    load();
    for (uint32_t i = threadIdx.x; i < nh * 256u; i += blockDim.x) (&s_hist[0][0])[i] = 0u;
    if (one && nparts > 0 && threadIdx.x < 64u) {
        const uint32_t lane = threadIdx.x;
        uint32_t v[7] = {0u, 0u, 0u, 0u, 0u, 0u, 0u};
        for (uint32_t c = lane; c < nparts; c += 64u) {
            const uint32_t* part = P.bbox_part + 8 * (size_t)c;
#pragma unroll
            for (int a = 0; a < 6; ++a) v[a] = max(v[a], part[a]);
            v[6] += part[6];
        }
#pragma unroll
        for (int a = 0; a < 6; ++a) v[a] = wave_umax(v[a]);
        v[6] = wave_sum(v[6]);
        if (lane == 0) {
            for (int a = 0; a < 3; ++a) {
                s_stat.bbox_nmin[a] = v[a];
                s_stat.bbox_max[a] = v[3 + a];
            }
            s_stat.nonfinite = v[6];
            s_stat.pad = 0u;
            frame_consts(&s_stat, min_leaf_side, &s_fc);
            if (blockIdx.x == 0) {
                *P.fstat = s_stat;
                *P.fc = s_fc;
                if (v[6]) atomicOr(&P.ctr->status, DEV_NONFINITE);
            }
        }
    } else if (one && threadIdx.x == 0) {
        frame_consts(P.fstat, min_leaf_side, &s_fc);
        if (blockIdx.x == 0) *P.fc = s_fc;
    }
    __syncthreads();
    if (!one && blockIdx.x == 0)  // a frame's points all count to its own digits
        for (uint32_t g = threadIdx.x; g < P.nf; g += blockDim.x) {
            const uint32_t m = P.foff[g + 1] - P.foff[g];
            for (uint32_t p = SORT_PASSES; m != 0u && p < nh; ++p)
                atomicAdd(&P.sort_hist[256u * p + ((g >> (8 * (p - SORT_PASSES))) & 255u)], m);
        }
    const float c0 = s_fc.lo[0], c1 = s_fc.lo[1], c2 = s_fc.lo[2];
    const double csc = s_fc.scale;
    while (i0 < n) {
        float l0[MORTON_U], l1[MORTON_U], l2[MORTON_U];
        double sc[MORTON_U];
#pragma unroll
        for (int u = 0; u < MORTON_U; ++u) {
            if (fc_lds) {
                const FrameConst& fc = s_fcs[f[u]];
                l0[u] = fc.lo[0];
                l1[u] = fc.lo[1];
                l2[u] = fc.lo[2];
                sc[u] = fc.scale;
            } else if (!one) {
                const FrameConst& fc = P.fc[f[u]];
                l0[u] = fc.lo[0];
                l1[u] = fc.lo[1];
                l2[u] = fc.lo[2];
                sc[u] = fc.scale;
            } else {
                l0[u] = c0;
                l1[u] = c1;
                l2[u] = c2;
                sc[u] = csc;
            }
        }
        // (an empty statement taking the loaded values keeps the compiler from
        // moving each load into the branch of its point)
#pragma unroll
        for (int u = 0; u < MORTON_U; ++u) asm volatile("" ::"v"(x[u]), "v"(y[u]), "v"(z[u]), "v"(f[u]));
#pragma unroll
        for (int u = 0; u < MORTON_U; ++u) {
            const uint32_t i = i0 + (uint32_t)u * stride;
            if (i >= n) break;
            const uint32_t qx = quantise(x[u], l0[u], sc[u]);
            const uint32_t qy = quantise(y[u], l1[u], sc[u]);
            const uint32_t qz = quantise(z[u], l2[u], sc[u]);
            const uint64_t key = morton3(qx, qy, qz);
            P.keys_src[i] = key;
#pragma unroll
            for (int p = SORT_SHORT_FIRST; p < SORT_PASSES; ++p)
                atomicAdd(&s_hist[p][(key >> (8 * p)) & 255u], 1u);
        }
        i0 += MORTON_U * stride;
        if (i0 < n) load();
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nh * 256u; i += blockDim.x) {
        uint32_t v = (&s_hist[0][0])[i];
        if (v) atomicAdd(&P.sort_hist[i], v);
    }
}

void launch_morton(const Plan& P, const Params& prm, const float* xyz, hipStream_t st) {
    if (P.nf > FC_LDS) hipLaunchKernelGGL(frame_const_kernel, dim3(1), dim3(256), 0, st, P, prm.min_leaf_side);
    unsigned blocks = (P.n + 2047) / 2048;
    if (blocks > 512) blocks = 512;
    const uint32_t nparts = bbox_one_frame(P) ? bbox_blocks(P) : 0u;
    auto kern = P.nf == 1 ? morton_kernel<1> : P.nf <= FC_LDS ? morton_kernel<FC_LDS> : morton_kernel<MAX_FRAMES>;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, st, xyz, P, prm.min_leaf_side, nparts);
}

// ---------------------------------------------------------------- radix sort

// Digit `pass` of the frame sort. Passes past the key's 8 take the digit from
// the frame of the payload (the original index, found in the frame offsets),
// so a batch ends sorted by (frame, key bits 32..62, index); only passes from
// SORT_SHORT_FIRST on are launched.
struct FrameDigit {
    int pass;
    const uint32_t* foff;    // frame offsets in memory
    const uint32_t* s_foff;  // the same staged in LDS, if `lds`
    bool lds;
    uint32_t nf;
    __device__ bool of_key() const { return pass < SORT_PASSES; }
    __device__ uint32_t key_digit(uint64_t k) const { return (uint32_t)((k >> (8 * pass)) & 255u); }
    __device__ uint32_t operator()(uint64_t k, uint32_t v, bool ok) const {
        if (of_key()) return key_digit(k);
        v = ok ? v : 0u;
        const uint32_t f = lds ? frame_of(s_foff, nf, v) : frame_of(foff, nf, v);
        return (f >> (8 * (pass - SORT_PASSES))) & 255u;
    }
};

// FIRST: the payload is the position itself.
template <int ITEMS, int BLOCK, bool FIRST>
__global__ __launch_bounds__(BLOCK) void radix_pass_kernel(const uint64_t* __restrict__ kin,
                                                                const uint32_t* __restrict__ vin,
                                                                uint64_t* __restrict__ kout,
                                                                uint32_t* __restrict__ vout, uint32_t n,
                                                                int pass, const uint32_t* __restrict__ hist,
                                                                uint32_t* status, uint32_t* dev_status,
                                                                const uint32_t* __restrict__ foff,
                                                                uint32_t nf) {
    __shared__ uint32_t s_foff[SORT_FOFF_LDS];
    // frame passes of batches with few frames search the offsets in LDS
    const bool foff_lds = pass >= SORT_PASSES && nf < SORT_FOFF_LDS;
    if (foff_lds)
        for (uint32_t i = threadIdx.x; i <= nf; i += BLOCK) s_foff[i] = foff[i];
    radix_tile<ITEMS, FIRST, BLOCK>(kin, vin, kout, vout, n, blockIdx.x, hist, status, dev_status, DEV_WAIT_LIMIT,
                             FrameDigit{pass, foff, s_foff, foff_lds, nf});
}

// ---------------------------------------------------------------- deep cells

constexpr int SEG_BLOCK = 256;
constexpr int SEG_PASSES = 6;  // key bits 0..47; bits 33..62 are the cell's own, and 6 passes end in keys_a

// Stable LSD radix sort of the keys and payloads of one level-10 cell [a, b)
// over key bits 0..47 (the cell's points share bits 33..62), by the whole
// block, tile by tile in order through keys_b / idx_b (scratch after the main
// sort): the cell's (original index) order becomes (key, index) order. A deep
// cell's positions are then flagged for the boundary test; a cell re-sorted
// only because it borders a deep one has its mark cleared.
__device__ void sort_cell(const Plan& P, uint32_t a, uint32_t b, bool deep, uint32_t* s_base,
                          uint32_t (*s_w)[256], uint32_t* s_scan) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int pass = 0; pass < SEG_PASSES; ++pass) {
        const int shift = 8 * pass;
        const uint64_t* ks = (pass & 1) ? P.keys_b : P.keys_a;
        const uint32_t* vs = (pass & 1) ? P.idx_b : P.idx_a;
        uint64_t* kd = (pass & 1) ? P.keys_a : P.keys_b;
        uint32_t* vd = (pass & 1) ? P.idx_a : P.idx_b;
        s_base[tid] = 0u;
        __syncthreads();
        for (uint32_t i = a + tid; i < b; i += SEG_BLOCK) atomicAdd(&s_base[(uint32_t)(ks[i] >> shift) & 255u], 1u);
        __syncthreads();
        uint32_t tot;
        const uint32_t ex = block_excl_scan(s_base[tid], s_scan, &tot);
        s_base[tid] = a + ex;
        for (uint32_t t0 = a; t0 < b; t0 += SEG_BLOCK) {
            for (int w = 0; w < SEG_BLOCK / 64; ++w) s_w[w][tid] = 0u;
            __syncthreads();
            const uint32_t i = t0 + tid;
            const bool ok = i < b;
            const uint64_t k = ok ? ks[i] : 0ull;
            const uint32_t v = ok ? vs[i] : 0u;
            const uint32_t d = ok ? (uint32_t)(k >> shift) & 255u : 256u;
            // lanes of this wave with the same digit
            const uint64_t m = match_digit(d, __ballot(ok));
            const uint32_t before = (uint32_t)__popcll(m & lt_mask);
            if (ok && (m >> lane) == 1ull) s_w[wave][d] = (uint32_t)__popcll(m);
            __syncthreads();
            uint32_t run = 0;
            for (int w = 0; w < SEG_BLOCK / 64; ++w) {
                const uint32_t c = s_w[w][tid];
                s_w[w][tid] = run;
                run += c;
            }
            __syncthreads();
            if (ok) {
                const uint32_t o = s_base[d] + s_w[wave][d] + before;
                if (o < b) {  // always true
                    kd[o] = k;
                    vd[o] = v;
                }
            }
            __syncthreads();
            s_base[tid] += run;
        }
        __syncthreads();  // the pass's writes are complete before the next reads them
    }
    if (deep) {
        for (uint32_t i = a + tid; i < b; i += SEG_BLOCK) P.deepf[i] = 1u;
    } else if (tid == 0) {
        P.deepf[a] = 0u;
    }
    __syncthreads();
}

// The same for a cell of up to SEG_BLOCK * SEG_ITEMS points, in LDS: five
// passes over key bits 0..39, the points in registers between them, read and
// written once.
constexpr int SEG_ITEMS = 4;
constexpr uint32_t SEG_LDS = (uint32_t)SEG_BLOCK * SEG_ITEMS;
__device__ void sort_cell_lds(const Plan& P, uint32_t a, uint32_t b, bool deep, uint64_t* s_k, uint32_t* s_v,
                              uint32_t* s_base, uint32_t (*s_w)[256], uint32_t* s_scan) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const uint32_t n = b - a;
    uint64_t key[SEG_ITEMS];
    uint32_t val[SEG_ITEMS];
    auto at = [&](int i) { return (uint32_t)(wave * 64 * SEG_ITEMS + i * 64 + lane); };
#pragma unroll
    for (int i = 0; i < SEG_ITEMS; ++i) {
        const bool ok = at(i) < n;
        key[i] = ok ? P.keys_a[a + at(i)] : 0ull;
        val[i] = ok ? P.idx_a[a + at(i)] : 0u;
    }
    for (int shift = 0; shift < 40; shift += 8) {
#pragma unroll
        for (int w = 0; w < SEG_BLOCK / 64; ++w) s_w[w][tid] = 0u;
        __syncthreads();
        uint32_t dig[SEG_ITEMS], rank[SEG_ITEMS];
#pragma unroll
        for (int i = 0; i < SEG_ITEMS; ++i) {
            const bool ok = at(i) < n;
            const uint32_t dg = (uint32_t)(key[i] >> shift) & 255u;
            const uint64_t m = match_digit(dg, __ballot(ok));
            const uint32_t before = (uint32_t)__popcll(m & lt_mask);
            const uint32_t wb = ok ? s_w[wave][dg] : 0u;
            dig[i] = dg;
            rank[i] = wb + before;
            if (ok && (m >> lane) == 1ull) s_w[wave][dg] = wb + (uint32_t)__popcll(m);
        }
        __syncthreads();
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < SEG_BLOCK / 64; ++w) {
            const uint32_t c = s_w[w][tid];
            s_w[w][tid] = run;
            run += c;
        }
        uint32_t tot;
        s_base[tid] = block_excl_scan(run, s_scan, &tot);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SEG_ITEMS; ++i)
            if (at(i) < n) {
                const uint32_t o = s_base[dig[i]] + s_w[wave][dig[i]] + rank[i];
                s_k[o] = key[i];
                s_v[o] = val[i];
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SEG_ITEMS; ++i)
            if (at(i) < n) {
                key[i] = s_k[at(i)];
                val[i] = s_v[at(i)];
            }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SEG_ITEMS; ++i)
        if (at(i) < n) {
            P.keys_a[a + at(i)] = key[i];
            P.idx_a[a + at(i)] = val[i];
            if (deep) P.deepf[a + at(i)] = 1u;
        }
    if (!deep && tid == 0) P.deepf[a] = 0u;
}

// The same for a cell of up to 64 points, by one wave: a bitonic sort of the
// cell's own key bits (0..32) and the position (points of equal keys keep
// their order).
__device__ void sort_cell_wave(const Plan& P, uint32_t a, uint32_t b, bool deep, uint32_t lane) {
    const bool ok = lane < b - a;
    const uint64_t key = ok ? P.keys_a[a + lane] : 0ull;
    const uint32_t val = ok ? P.idx_a[a + lane] : 0u;
    const unsigned long long own = key & ((1ull << CELL_SHIFT) - 1ull);
    const unsigned long long v = ok ? (own << 6) | lane : ~0ull >> 1;
    const unsigned long long srt = ~sort64_desc(~v, lane);
    const int src = (int)((uint32_t)srt & 63u);
    const uint32_t klo = (uint32_t)__shfl((int)(uint32_t)key, src, 64);
    const uint32_t khi = (uint32_t)__shfl((int)(uint32_t)(key >> 32), src, 64);
    const uint32_t vs = (uint32_t)__shfl((int)val, src, 64);
    if (ok) {
        P.keys_a[a + lane] = ((uint64_t)khi << 32) | klo;
        P.idx_a[a + lane] = vs;
        if (deep) P.deepf[a + lane] = 1u;
    }
    if (!deep && lane == 0u) P.deepf[a] = 0u;
}

// Frame of sorted position s and its range [fs, fe).
__device__ __forceinline__ uint32_t frame_range(const Plan& P, const uint32_t* s_foff, bool lds, uint32_t s,
                                                uint32_t* fs, uint32_t* fe) {
    uint32_t f = 0u;
    if (lds) {
        f = frame_of(s_foff, P.nf, s);
        *fs = s_foff[f];
        *fe = s_foff[f + 1];
    } else {
        if (P.nf > 1u) f = frame_of(P.foff, P.nf, s);
        *fs = P.foff[f];
        *fe = P.foff[f + 1];
    }
    return f;
}

// A level-10 cell splits when it holds more than `cap` points and lies above
// its frame's depth limit ("deep"). Its leaves lie below level 10, and so do
// the halo cells around them, which reach into the 26 level-10 cells next to
// it: every one of those needs its points in whole-key order too, so that a
// deeper cell is one contiguous key range. One thread per sorted position
// finds the positions that start a deep cell; the block then marks (deepf = 2)
// the start of each such cell and of each non-empty neighbouring cell in its
// frame, a thread per (cell, neighbour): each is a chain of ~20 dependent
// loads, and one thread walking all 26 made this 74 us on a 1.2M sweep (11
// now). The marks are plain stores of one value, so cells marked twice need no
// atomics.
// LDS: the frame offsets are staged in LDS (batches of fewer than
// SORT_FOFF_LDS frames), fixed at compile time so that they are read with LDS
// or global instructions, not generic ones.
template <bool LDS>
__global__ __launch_bounds__(SEG_BLOCK) void deep_mark_kernel(Plan P, uint32_t cap) {
    __shared__ uint32_t s_foff[SORT_FOFF_LDS];  // batches of fewer frames search the offsets here
    constexpr bool lds = LDS;
    if (lds)
        for (uint32_t i = threadIdx.x; i <= P.nf; i += blockDim.x) s_foff[i] = P.foff[i];
    __syncthreads();
    __shared__ uint32_t s_start[SEG_BLOCK];
    __shared__ uint32_t s_n;
    for (uint32_t base = blockIdx.x * SEG_BLOCK; base < P.n; base += gridDim.x * SEG_BLOCK) {
        if (threadIdx.x == 0) s_n = 0u;
        __syncthreads();
        const uint32_t s = base + threadIdx.x;
        if (s < P.n) {
            uint32_t fs, fe;
            const uint32_t f = frame_range(P, s_foff, lds, s, &fs, &fe);
            const uint64_t c = P.keys_a[s] >> CELL_SHIFT;
            const bool start = P.fc[f].dmax > SORT_SHORT_LEVEL &&
                               (s == fs || (P.keys_a[s - 1] >> CELL_SHIFT) != c) && (uint64_t)s + cap < fe &&
                               (P.keys_a[s + cap] >> CELL_SHIFT) == c;
            if (start) s_start[atomicAdd(&s_n, 1u)] = s;
        }
        __syncthreads();
        const uint32_t ns = s_n;
        if (ns != 0u && threadIdx.x == 0) P.ctr->n_deep = 1u;  // (any workgroup's store of the same value)
        for (uint32_t e = threadIdx.x; e < ns * 32u; e += SEG_BLOCK) {
            const uint32_t q0 = s_start[e / 32u];
            const int g = (int)(e % 32u);
            if (g >= 27) continue;
            if (g == 13) {
                P.deepf[q0] = 2u;
                continue;
            }
            uint32_t fs, fe;
            (void)frame_range(P, s_foff, lds, q0, &fs, &fe);
            const uint64_t c = P.keys_a[q0] >> CELL_SHIFT;
            const int32_t nx = (int32_t)compact3(c) + g % 3 - 1, ny = (int32_t)compact3(c >> 1) + (g / 3) % 3 - 1,
                          nz = (int32_t)compact3(c >> 2) + g / 9 - 1;
            const int32_t side = 1 << SORT_SHORT_LEVEL;
            if (nx < 0 || ny < 0 || nz < 0 || nx >= side || ny >= side || nz >= side) continue;
            const uint64_t nc = morton3((uint32_t)nx, (uint32_t)ny, (uint32_t)nz);
            const uint32_t q = cell_lower_bound(P.keys_a, fs, fe, nc);
            if (q < fe && (P.keys_a[q] >> CELL_SHIFT) == nc) P.deepf[q] = 2u;
        }
        __syncthreads();  // the list is refilled by the next round
    }
}

// One thread per sorted position: a marked position starts a cell to re-sort;
// it finds the cell's end, and the block then sorts the cells that start
// among its positions (deep ones flagged, the others unmarked): cells of up to
// 64 points a wave each, up to SEG_LDS points in LDS, larger ones through
// memory. (All of them through memory, one after another: 155 us on a 1.2M
// sweep, 32 now.) Blocks that
// read keys of a cell another block is sorting compare cell prefixes only,
// which the sort does not change; a mark is only read by the thread of its
// own position, and only that cell's block rewrites it.
template <bool LDS>
__global__ __launch_bounds__(SEG_BLOCK) void deep_cells_kernel(Plan P, uint32_t cap) {
    __shared__ uint32_t s_base[256];
    __shared__ uint32_t s_w[SEG_BLOCK / 64][256];
    __shared__ uint32_t s_scan[SEG_BLOCK / 64 + 1];
    __shared__ uint2 s_seg[SEG_BLOCK];
    __shared__ uint8_t s_deep[SEG_BLOCK];
    __shared__ uint64_t s_k[SEG_LDS];
    __shared__ uint32_t s_v[SEG_LDS];
    __shared__ uint32_t s_nseg;
    __shared__ uint32_t s_foff[SORT_FOFF_LDS];  // batches of fewer frames search the offsets here
    if (P.ctr->n_deep == 0u) return;  // (20k points 130.5 -> 129.6 us a call, 900k 757.5 -> 754)
    constexpr bool lds = LDS;
    if (lds)
        for (uint32_t i = threadIdx.x; i <= P.nf; i += blockDim.x) s_foff[i] = P.foff[i];
    // rounds of SEG_BLOCK positions, whose marks are read four rounds ahead:
    // those without one, nearly all of them, end there
    constexpr uint32_t U = 4;
    const uint32_t stride = gridDim.x * SEG_BLOCK;  // (at most 2^20)
    for (uint32_t base0 = blockIdx.x * SEG_BLOCK; base0 < P.n; base0 += U * stride) {
        // (four flags per load, a load per thread; they are padded with zeros past n)
        const uint32_t s4 = base0 + threadIdx.x / (SEG_BLOCK / U) * stride + threadIdx.x % (SEG_BLOCK / U) * 4u;
        const uint32_t f4 = s4 < P.n ? *(const uint32_t*)(P.deepf + s4) : 0u;
        if (!__syncthreads_or((int)(f4 & 0x02020202u))) continue;
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t base = base0 + u * stride;
            if (base >= P.n) break;
            if (threadIdx.x == 0) s_nseg = 0u;
            __syncthreads();
            const uint32_t s = base + threadIdx.x;
            if (s < P.n && P.deepf[s] == 2u) {
                uint32_t fs, fe;
                const uint32_t f = frame_range(P, s_foff, lds, s, &fs, &fe);
                const uint64_t c = P.keys_a[s] >> CELL_SHIFT;
                // the cell's end: doubling steps, then a search of the last one
                uint32_t lo = s, step = 64u;
                while (fe - lo > step && (P.keys_a[lo + step] >> CELL_SHIFT) == c) {
                    lo += step;
                    step *= 2u;
                }
                const uint32_t e = cell_lower_bound(P.keys_a, lo + 1u, fe - lo > step ? lo + step : fe, c + 1u);
                const uint32_t slot = atomicAdd(&s_nseg, 1u);
                s_seg[slot] = make_uint2(s, e);
                s_deep[slot] = (uint8_t)(P.fc[f].dmax > SORT_SHORT_LEVEL && e - s > cap);
            }
            __syncthreads();
            const uint32_t ns = s_nseg;
            for (uint32_t g = threadIdx.x >> 6; g < ns; g += SEG_BLOCK / 64)
                if (s_seg[g].y - s_seg[g].x <= 64u)
                    sort_cell_wave(P, s_seg[g].x, s_seg[g].y, s_deep[g] != 0u, threadIdx.x & 63u);
            for (uint32_t g = 0; g < ns; ++g) {
                const uint2 r = s_seg[g];
                if (r.y - r.x <= 64u) continue;
                if (r.y - r.x <= SEG_LDS)
                    sort_cell_lds(P, r.x, r.y, s_deep[g] != 0u, s_k, s_v, s_base, s_w, s_scan);
                else
                    sort_cell(P, r.x, r.y, s_deep[g] != 0u, s_base, s_w, s_scan);
                __syncthreads();
            }
            __syncthreads();
        }
    }
}

void launch_sort(const Plan& P, const Params& prm, hipStream_t st) {
    // the keys start where the launched passes leave them in keys_a
    const uint64_t* kin = P.keys_src;
    const uint32_t* vin = P.idx_src;
    uint64_t* kout = P.keys_src == P.keys_a ? P.keys_b : P.keys_a;
    uint32_t* vout = P.idx_src == P.idx_a ? P.idx_b : P.idx_a;
    for (uint32_t pass = SORT_SHORT_FIRST; pass < P.sort_passes; ++pass) {
        // small inputs: many small tiles (latency); large: fewer, fuller tiles
        auto pick = [&](auto first) {
            constexpr bool F = decltype(first)::value;
            return P.sort_tile == 512u    ? radix_pass_kernel<2, 256, F>
                   : P.sort_tile == 1024u ? radix_pass_kernel<4, 256, F>
                   : P.sort_tile == 2048u ? radix_pass_kernel<4, 512, F>
                                          : radix_pass_kernel<8, 512, F>;
        };
        auto kern = pass == SORT_SHORT_FIRST ? pick(std::true_type{}) : pick(std::false_type{});
        hipLaunchKernelGGL(kern, dim3(P.sort_tiles), dim3(P.sort_tile <= 1024u ? 256 : 512), 0, st, kin, vin, kout, vout,
                           P.n, (int)pass, P.sort_hist + 256 * pass,
                           P.sort_status + (size_t)(pass - SORT_SHORT_FIRST) * P.sort_tiles * 256, &P.ctr->status,
                           (const uint32_t*)P.foff, P.nf);
        const uint64_t* tk = kout;
        const uint32_t* tv = vout;
        kout = (uint64_t*)kin;
        vout = (uint32_t*)vin;
        kin = tk;
        vin = tv;
    }
    if (P.n <= (uint32_t)prm.leaf_cap) return;  // no deep cells
    unsigned blocks = (P.n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks == 0) blocks = 1;
    const bool lds = P.nf > 1u && P.nf < SORT_FOFF_LDS;
    hipLaunchKernelGGL(lds ? deep_mark_kernel<true> : deep_mark_kernel<false>, dim3(blocks), dim3(SEG_BLOCK), 0, st, P,
                       (uint32_t)prm.leaf_cap);
    hipLaunchKernelGGL(lds ? deep_cells_kernel<true> : deep_cells_kernel<false>, dim3(blocks), dim3(SEG_BLOCK), 0, st,
                       P, (uint32_t)prm.leaf_cap);
}

}  // namespace gdn
