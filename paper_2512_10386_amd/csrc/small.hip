// The octree of a small frame in one workgroup: bounding box, Morton keys,
// their sort and the leaves, then the voxel filter and P1, held in registers
// and LDS from the first load to the last store.
#include "kernels.hpp"
#include "tree.hpp"
#include "voxel.hpp"

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

// One step of the running minima m[0..2] and maxima m[3..5] over the lanes of
// one leaf (leaves are runs of lanes), in the manner of wave_incl_scan.
template <int CTRL, int ROWS>
__device__ __forceinline__ void run_step(uint32_t leaf, float (&m)[6]) {
    const bool same = dpp_from<CTRL, ROWS>(leaf, ~leaf) == leaf;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        const float v = dpp_from<CTRL, ROWS>(m[a], m[a]);
        m[a] = same ? (a < 3 ? fminf(m[a], v) : fmaxf(m[a], v)) : m[a];
    }
}

// n <= SMALL_BLOCK * ITEMS points of one frame. Latency bounds it: at these
// sizes each kernel of the general path (box, keys, four sort passes, two for
// deep cells, leaf borders, their scan) takes the few microseconds that any
// launch and its first loads take, so one workgroup that keeps the points on
// chip is faster than ten launches over the whole chip. Whole calls of a scanned
// object, general path and this one: 65 points 66.5 and 49.6 us, 500 74.6 and
// 52.9, 1501 88.3 and 66.3, 3000 98.2 and 85.0, 4096 102.5 and 91.5. Most of it is
// the sort: a pass is six barriers over 16 waves, 3 us.
// P1: the voxel filter and the P1 compaction too, by all threads over the
// points (leaf boxes, then hash tables, in the LDS that the sort is done with):
// 500 points 59.1 us a call without and 52.9 with it, 1501 68.2 and 66.3, 2048
// 73.7 and 70.4, but 3000 84.9 and 85.7, 4096, where a workgroup per leaf does
// more at once, 91.4 and 94.1.
template <int ITEMS, bool P1>
__global__ __launch_bounds__(SMALL_BLOCK) void small_tree_kernel(const float* __restrict__ xyz, Plan P,
                                                                 double min_leaf_side, uint32_t cap, double beta,
                                                                 uint32_t nv) {
    constexpr uint32_t N = SMALL_BLOCK * ITEMS;
    constexpr uint32_t SORT_BYTES = 13u * N + 4u * SMALL_WAVES * 256u, P1_BYTES = P1 ? 32u * N + 16u : 0u;
    __shared__ __align__(16) char s_raw[SORT_BYTES > P1_BYTES ? SORT_BYTES : P1_BYTES];
    uint64_t* const s_key = (uint64_t*)s_raw;
    uint32_t* const s_val = (uint32_t*)(s_raw + 8u * N);
    uint32_t(*const s_w)[256] = (uint32_t(*)[256])(s_raw + 12u * N);
    uint8_t* const s_mark = (uint8_t*)(s_raw + 12u * N + 4u * SMALL_WAVES * 256u);
    __shared__ uint32_t s_part[4][256];
    __shared__ uint32_t s_scan[SMALL_WAVES + 1];
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
    float4 p[ITEMS];
    uint32_t leaf[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const size_t o = at(i) < n ? val[i] & SMALL_IDX : 0u;
        p[i] = make_float4(xyz[3 * o], xyz[3 * o + 1], xyz[3 * o + 2], __uint_as_float((uint32_t)o));
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t s = at(i);
        const uint32_t e = base + ex[i];
        leaf[i] = s < n ? e + (flag[i] ? 1u : 0u) - 1u : ~0u;
        if (s < n) {
            P.keys_a[s] = key[i];
            P.idx_a[s] = __float_as_uint(p[i].w);
            P.pos4[s] = p[i];
            P.leaf_of[s] = leaf[i];
            if (flag[i]) P.leaf_begin[e] = s;
            if (!P1 && P.big_leaves)  // the leaf boxes of launch_big_voxel start empty
                for (uint32_t a = 0; a < 6u; ++a) P.leaf_box[6 * (size_t)s + a] = 0u;
        }
    }
    if (tid == 0) {
        P.ctr->n_leaves = total;
        P.leaf_begin[total] = n;
    }
    if constexpr (P1) {
        // first points and boxes of the leaves (ordered-uint minima, maxima)
        uint32_t* const s_lbox = (uint32_t*)s_raw;           // [6][N]
        uint32_t* const s_begin = (uint32_t*)s_raw + 6u * N;  // [N + 1]
        float* const s_h = (float*)s_raw + 7u * N + 1u;       // [N]
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (flag[i]) s_begin[leaf[i]] = at(i);
        if (tid == 0) s_begin[total] = n;
        for (uint32_t t = tid; t < total; t += SMALL_BLOCK)
#pragma unroll
            for (uint32_t a = 0; a < 6u; ++a) s_lbox[a * N + t] = f32_ordered(a < 3u ? INFINITY : -INFINITY);
        __syncthreads();
        // a leaf's run of lanes is reduced into its last lane, which adds it to
        // the leaf's box
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const float c[3] = {p[i].x, p[i].y, p[i].z};
            float m[6];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                m[a] = fminf(c[a], INFINITY);
                m[3 + a] = fmaxf(c[a], -INFINITY);
            }
            run_step<0x111, 0xF>(leaf[i], m);
            run_step<0x112, 0xF>(leaf[i], m);
            run_step<0x114, 0xF>(leaf[i], m);
            run_step<0x118, 0xF>(leaf[i], m);
            run_step<0x142, 0xA>(leaf[i], m);
            run_step<0x143, 0xC>(leaf[i], m);
            const uint32_t next = (uint32_t)__shfl_down((int)leaf[i], 1, 64);
            if (leaf[i] != ~0u && (lane == 63u || next != leaf[i])) {
#pragma unroll
                for (uint32_t a = 0; a < 6u; ++a) {
                    if (a < 3u) atomicMin(&s_lbox[a * N + leaf[i]], f32_ordered(m[a]));
                    else atomicMax(&s_lbox[a * N + leaf[i]], f32_ordered(m[a]));
                }
            }
        }
        __syncthreads();
        for (uint32_t t = tid; t < total; t += SMALL_BLOCK) {
            float lo[3], hi[3];
#pragma unroll
            for (uint32_t a = 0; a < 3u; ++a) {
                lo[a] = f32_from_ordered(s_lbox[a * N + t]);
                hi[a] = f32_from_ordered(s_lbox[(3u + a) * N + t]);
            }
            const float h = leaf_voxel_size(lo, hi, s_begin[t + 1u] - s_begin[t], beta);
            s_h[t] = h;
            P.leaf_h[t] = h;
        }
        __syncthreads();
        uint64_t vk[ITEMS];
        float h[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t t = min(leaf[i], total - 1u);
            h[i] = s_h[t];
            vk[i] = h[i] == 0.0f ? 0ull
                                 : vox_key(p[i], f32_from_ordered(s_lbox[t]), f32_from_ordered(s_lbox[N + t]),
                                           f32_from_ordered(s_lbox[2u * N + t]), (double)h[i]);
        }
        __syncthreads();  // the boxes have been read
        // occupancy: an open-addressing table of 2 nt slots per leaf
        constexpr unsigned long long EMPTY = ~0ull;
        unsigned long long* const s_tk = (unsigned long long*)s_raw;  // [2 N], 16 N bytes
        uint32_t* const s_tc = (uint32_t*)(s_raw + 16u * N);          // [2 N], up to byte 24 N
        for (uint32_t j = tid; j < 2u * n; j += SMALL_BLOCK) {
            s_tk[j] = EMPTY;
            s_tc[j] = 0u;
        }
        __syncthreads();
        uint32_t slot[ITEMS], nt[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (leaf[i] == ~0u) continue;
            const uint32_t lb = s_begin[leaf[i]];
            nt[i] = s_begin[leaf[i] + 1u] - lb;
            if (h[i] == 0.0f) continue;
            const uint32_t slots = 2u * nt[i];
            uint32_t r = __umulhi(vox_hash(vk[i]), slots);
            for (uint32_t probe = 0; probe < slots; ++probe) {
                const unsigned long long prev = atomicCAS(&s_tk[2u * lb + r], EMPTY, (unsigned long long)vk[i]);
                if (prev == EMPTY || prev == vk[i]) break;
                r = r + 1u == slots ? 0u : r + 1u;
            }
            slot[i] = 2u * lb + r;
            atomicAdd(&s_tc[slot[i]], 1u);
        }
        __syncthreads();
        // P1 and its places
        bool in1[ITEMS];
        cnt = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t s = at(i);
            in1[i] = false;
            if (s < n) {
                const uint32_t occ = h[i] == 0.0f ? nt[i] : s_tc[slot[i]];
                in1[i] = occ >= nv;
                P.occ[s] = occ;
                P.p1[s] = in1[i];
            }
            const uint64_t m = __ballot(in1[i]);
            ex[i] = cnt + (uint32_t)__popcll(m & below);
            cnt += (uint32_t)__popcll(m);
        }
        if (lane == 0u) s_scan[wave] = cnt;
        __syncthreads();
        base = 0;
        total = 0;
#pragma unroll
        for (uint32_t w = 0; w < (uint32_t)SMALL_WAVES; ++w) {
            const uint32_t c = s_scan[w];
            base += w < wave ? c : 0u;
            total += c;
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t s = at(i), q = base + ex[i];
            if (s < n) P.p1pos[s] = q;
            if (in1[i]) {
                P.cand4[q] = p[i];
                P.cand_leaf[q] = leaf[i];
                P.inv_p1[__float_as_uint(p[i].w)] = q;
            }
        }
        if (tid == 0) {
            P.ctr->n_p1 = total;
            P.ctr->knn_tq = knn_tile_queries(total);
            P.p1pos[n] = total;
        }
    }
}

// One frame of so few points that the workgroup is done sooner than the chip
// (4096 points 102.5 us the general way and 91.5 this way, but 6000 106.7 and
// 109.4, with eight points per thread).
bool small_tree(const Plan& P) { return P.nf == 1 && P.n <= 4u * SMALL_BLOCK; }

void launch_small_tree(const Plan& P, const Params& prm, const float* xyz, hipStream_t st) {
    auto kern = P.n <= (uint32_t)SMALL_BLOCK        ? small_tree_kernel<1, true>
                : P.n <= 2u * (uint32_t)SMALL_BLOCK ? small_tree_kernel<2, true>
                                                    : small_tree_kernel<4, false>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(SMALL_BLOCK), 0, st, xyz, P, prm.min_leaf_side, (uint32_t)prm.leaf_cap,
                       prm.beta, (uint32_t)prm.min_vox_count);
    if (P.n > 2u * (uint32_t)SMALL_BLOCK) {
        launch_voxel(P, prm, st);
        launch_p1_compact(P, st);
    }
}

}  // namespace gdn
