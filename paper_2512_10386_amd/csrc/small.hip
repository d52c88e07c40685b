// The octree of a small frame in one workgroup: bounding box, Morton keys,
// their sort and the leaves, held in registers and LDS from the first load to
// the last store.
#include "kernels.hpp"
#include "tree.hpp"

namespace gdn {

constexpr int SMALL_BLOCK = 1024;
constexpr int SMALL_WAVES = SMALL_BLOCK / 64;
constexpr uint32_t SMALL_WHOLE = 1u << 31;  // payload: sorted on the whole key
constexpr uint32_t SMALL_DEEP = 1u << 30;   // payload: in a deep level-10 cell
constexpr uint32_t SMALL_IDX = SMALL_DEEP - 1u;

// One stable counting pass over digit(key, payload) < 256: ranks inside each
// wave by ballots, the 16 waves' digit counts scanned by all threads (four
// waves' counts of one digit each), then through LDS to the sorted place. The
// points come from registers (wave w's item i of lane l is position
// (w * ITEMS + i) * 64 + l) and return to them in their new order.
template <int ITEMS, class Digit>
__device__ __forceinline__ void small_pass(uint64_t (&key)[ITEMS], uint32_t (&val)[ITEMS], uint32_t n, uint64_t* s_key,
                                           uint32_t* s_val, uint32_t (*s_w)[256], uint32_t (*s_part)[256],
                                           uint32_t* s_scan, Digit&& digit) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint64_t below = lane == 0u ? 0ull : (~0ull >> (64u - lane));
    auto at = [&](int i) { return (wave * ITEMS + (uint32_t)i) * 64u + lane; };
#pragma unroll
    for (int i = 0; i < SMALL_WAVES * 256 / SMALL_BLOCK; ++i) (&s_w[0][0])[i * SMALL_BLOCK + tid] = 0u;
    __syncthreads();
    uint32_t dig[ITEMS], rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool ok = at(i) < n;
        const uint32_t d = digit(key[i], val[i]);
        const uint64_t m = match_digit(d, __ballot(ok));
        const uint32_t before = ok ? s_w[wave][d] : 0u;
        dig[i] = d;
        rank[i] = before + (uint32_t)__popcll(m & below);
        if (ok && (m >> lane) == 1ull) s_w[wave][d] = before + (uint32_t)__popcll(m);
    }
    __syncthreads();
    // thread (q, d): digit d of waves 4q .. 4q + 3
    const uint32_t d = tid & 255u, q = tid >> 8;
    uint32_t c[4], sum = 0;
#pragma unroll
    for (uint32_t w = 0; w < 4u; ++w) {
        c[w] = s_w[4u * q + w][d];
        sum += c[w];
    }
    s_part[q][d] = sum;
    __syncthreads();
    uint32_t all = 0, base = 0;
#pragma unroll
    for (uint32_t r = 0; r < 4u; ++r) {
        const uint32_t v = s_part[r][d];
        base += r < q ? v : 0u;
        all += v;
    }
    const uint32_t inc = wave_incl_scan(all);  // (each q scans the same 256 totals)
    if (lane == 63u) s_scan[wave] = inc;
    __syncthreads();
    base += inc - all;
    for (uint32_t w = wave & ~3u; w < wave; ++w) base += s_scan[w];
#pragma unroll
    for (uint32_t w = 0; w < 4u; ++w) {
        s_w[4u * q + w][d] = base;
        base += c[w];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (at(i) < n) {
            const uint32_t o = s_w[wave][dig[i]] + rank[i];
            s_key[o] = key[i];
            s_val[o] = val[i];
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (at(i) < n) {
            key[i] = s_key[at(i)];
            val[i] = s_val[at(i)];
        }
}

// n <= SMALL_BLOCK * ITEMS points of one frame. Latency bounds it: at these
// sizes each kernel of the general path (box, keys, four sort passes, two for
// deep cells, leaf borders, their scan) takes the few microseconds that any
// launch and its first loads take, so one workgroup that keeps the points on
// chip is faster than ten launches over the whole chip. Whole calls, general
// path and this one: 65 points 90 and 69 us, 500 101 and 78, 1501 112 and 89.
template <int ITEMS>
__global__ __launch_bounds__(SMALL_BLOCK) void small_tree_kernel(const float* __restrict__ xyz, Plan P,
                                                                 double min_leaf_side, uint32_t cap) {
    __shared__ uint64_t s_key[SMALL_BLOCK * ITEMS];
    __shared__ uint32_t s_val[SMALL_BLOCK * ITEMS];
    __shared__ uint32_t s_w[SMALL_WAVES][256];
    __shared__ uint32_t s_part[4][256];
    __shared__ uint32_t s_scan[SMALL_WAVES + 1];
    __shared__ uint8_t s_mark[SMALL_BLOCK * ITEMS];
    __shared__ float s_box[6][SMALL_WAVES];
    __shared__ uint32_t s_bad[SMALL_WAVES];
    __shared__ FrameConst s_fc;
    __shared__ uint32_t s_n;
    const uint32_t n = P.n, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint64_t below = lane == 0u ? 0ull : (~0ull >> (64u - lane));
    auto at = [&](int i) { return (wave * ITEMS + (uint32_t)i) * 64u + lane; };

    // the workspace's zeroed block, as bbox_one_kernel clears it
    for (size_t i = tid; i < P.zero_bytes / 16; i += SMALL_BLOCK) ((uint4*)P.zero_begin)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) {
        P.foff[0] = 0u;
        P.foff[1] = n;
    }

    // bounding box of the finite points
    float x[ITEMS], y[ITEMS], z[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const size_t j = min(at(i), n - 1u);
        x[i] = xyz[3 * j];
        y[i] = xyz[3 * j + 1];
        z[i] = xyz[3 * j + 2];
    }
    float b[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};  // min, min of -x
    uint32_t bad = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool in = at(i) < n;
        const bool fin = isfinite(x[i]) && isfinite(y[i]) && isfinite(z[i]);
        if (in && fin) {
            b[0] = fminf(b[0], x[i]); b[3] = fminf(b[3], -x[i]);
            b[1] = fminf(b[1], y[i]); b[4] = fminf(b[4], -y[i]);
            b[2] = fminf(b[2], z[i]); b[5] = fminf(b[5], -z[i]);
        }
        bad += in && !fin ? 1u : 0u;
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) b[a] = wave_fmin(b[a]);
    bad = wave_sum(bad);
    if (lane == 0u) {
#pragma unroll
        for (int a = 0; a < 6; ++a) s_box[a][wave] = b[a];
        s_bad[wave] = bad;
    }
    __syncthreads();
    if (tid < 64u) {
        const uint32_t w = lane & (SMALL_WAVES - 1u);
#pragma unroll
        for (int a = 0; a < 6; ++a) b[a] = s_box[a][w];
        bad = lane < (uint32_t)SMALL_WAVES ? s_bad[w] : 0u;
#pragma unroll
        for (int a = 0; a < 6; ++a) b[a] = wave_fmin(b[a]);
        bad = wave_sum(bad);
        if (lane == 0u) {
            FrameStat fs;
            for (int a = 0; a < 3; ++a) {
                const bool any = b[a] <= -b[3 + a];
                fs.bbox_nmin[a] = any ? ~f32_ordered(b[a]) : 0u;
                fs.bbox_max[a] = any ? f32_ordered(-b[3 + a]) : 0u;
            }
            fs.nonfinite = bad;
            fs.pad = 0u;
            frame_consts(&fs, min_leaf_side, &s_fc);
            *P.fstat = fs;
            *P.fc = s_fc;
            if (bad) P.ctr->status = DEV_NONFINITE;  // (the first to write it)
        }
    }
    __syncthreads();

    uint64_t key[ITEMS];
    uint32_t val[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        key[i] = morton3(quantise(x[i], s_fc.lo[0], s_fc.scale), quantise(y[i], s_fc.lo[1], s_fc.scale),
                         quantise(z[i], s_fc.lo[2], s_fc.scale));
        val[i] = at(i);
    }
    const int dmax = s_fc.dmax;

    // Sort by key bits 32..62 (index order at ties). If some level-10 cell is
    // deep (more than cap points above the depth limit), the points of deep
    // cells and of the cells next to them are marked, and a second round sorts
    // on the low bits too, read as zero where a point has no mark.
    for (int round = 0;; ++round) {
        for (int pass = round == 0 ? SORT_SHORT_FIRST : 0; pass < SORT_PASSES; ++pass)
            small_pass<ITEMS>(key, val, n, s_key, s_val, s_w, s_part, s_scan, [&](uint64_t k, uint32_t v) {
                const uint32_t d = (uint32_t)(k >> (8 * pass)) & 255u;
                return pass >= SORT_SHORT_FIRST || (v & SMALL_WHOLE) ? d : 0u;
            });
        if (round == 1 || dmax <= SORT_SHORT_LEVEL || cap >= n) break;
        uint32_t* s_start = s_val;  // first positions of the deep cells (the payloads are in registers)
        if (tid == 0) s_n = 0u;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (at(i) < n) s_mark[at(i)] = 0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t s = at(i);
            if (s < n) {
                const uint64_t c = key[i] >> CELL_SHIFT;
                if ((s == 0u || (s_key[s - 1u] >> CELL_SHIFT) != c) && cap < n - s &&
                    (s_key[s + cap] >> CELL_SHIFT) == c)
                    s_start[atomicAdd(&s_n, 1u)] = s;
            }
        }
        __syncthreads();
        const uint32_t ns = s_n;
        if (ns == 0u) break;
        for (uint32_t e = tid; e < ns * 32u; e += SMALL_BLOCK) {
            const uint32_t s = s_start[e / 32u];
            const int g = (int)(e % 32u);
            if (g >= HALO) continue;
            const uint64_t c = s_key[s] >> CELL_SHIFT;
            const int32_t nx = (int32_t)compact3(c) + g % 3 - 1, ny = (int32_t)compact3(c >> 1) + (g / 3) % 3 - 1,
                          nz = (int32_t)compact3(c >> 2) + g / 9 - 1;
            const int32_t side = 1 << SORT_SHORT_LEVEL;
            if (nx < 0 || ny < 0 || nz < 0 || nx >= side || ny >= side || nz >= side) continue;
            const uint64_t nc = morton3((uint32_t)nx, (uint32_t)ny, (uint32_t)nz);
            const uint32_t o = cell_lower_bound(s_key, 0u, n, nc);
            if (o < n && (s_key[o] >> CELL_SHIFT) == nc) s_mark[o] = 1u;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (at(i) < n) {
                const uint64_t c = key[i] >> CELL_SHIFT;
                const uint32_t o = cell_lower_bound(s_key, 0u, at(i), c);
                if (s_mark[o])
                    val[i] |= SMALL_WHOLE |
                              (cap < n - o && (s_key[o + cap] >> CELL_SHIFT) == c ? SMALL_DEEP : 0u);
            }
        __syncthreads();  // (the passes overwrite what these reads use)
    }

    // leaf borders, leaf ids and the points in sorted order
    uint32_t ex[ITEMS];
    bool flag[ITEMS];
    uint32_t cnt = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t s = at(i);
        flag[i] = s < n && leaf_boundary(s_key, s, 0u, n, dmax, (val[i] & SMALL_DEEP) != 0u, cap) != 0u;
        const uint64_t m = __ballot(flag[i]);
        ex[i] = cnt + (uint32_t)__popcll(m & below);
        cnt += (uint32_t)__popcll(m);
    }
    if (lane == 0u) s_scan[wave] = cnt;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)SMALL_WAVES; ++w) {
        const uint32_t c = s_scan[w];
        base += w < wave ? c : 0u;
        total += c;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t s = at(i);
        if (s < n) {
            const uint32_t o = val[i] & SMALL_IDX, e = base + ex[i];
            P.keys_a[s] = key[i];
            P.idx_a[s] = o;
            P.pos4[s] = make_float4(xyz[3 * (size_t)o], xyz[3 * (size_t)o + 1], xyz[3 * (size_t)o + 2], __uint_as_float(o));
            P.leaf_of[s] = e + (flag[i] ? 1u : 0u) - 1u;
            if (flag[i]) P.leaf_begin[e] = s;
            if (P.big_leaves)  // the leaf boxes of launch_big_voxel start empty
                for (uint32_t a = 0; a < 6u; ++a) P.leaf_box[6 * (size_t)s + a] = 0u;
        }
    }
    if (tid == 0) {
        P.ctr->n_leaves = total;
        P.leaf_begin[total] = n;
    }
}

// One frame of so few points that the workgroup is done sooner than the chip
// (3000 points 125 us the general way and 109 this way, 4096 132 and 120, but
// 6000 130 and 136, with eight points per thread).
bool small_tree(const Plan& P) { return P.nf == 1 && P.n <= 4u * SMALL_BLOCK; }

void launch_small_tree(const Plan& P, const Params& prm, const float* xyz, hipStream_t st) {
    auto kern = P.n <= (uint32_t)SMALL_BLOCK       ? small_tree_kernel<1>
                : P.n <= 2u * (uint32_t)SMALL_BLOCK ? small_tree_kernel<2>
                                                    : small_tree_kernel<4>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(SMALL_BLOCK), 0, st, xyz, P, prm.min_leaf_side, (uint32_t)prm.leaf_cap);
}

}  // namespace gdn
