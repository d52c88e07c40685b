// Voxel filter (Eq. 10-12), density with percentile cut and median (Eq. 13, 14,
// 16) and top-lambda for octrees whose leaves are big (big_leaf_path): the
// per-point work runs over all positions, one thread each, and only the selects
// run one workgroup per leaf, on values held in registers. Same expressions as
// the per-leaf kernels, so the results are the same bits.
#include "density.hpp"
#include "kernels.hpp"
#include "voxel.hpp"
#include "wave.hpp"

namespace gdn {

namespace {

unsigned point_blocks(uint32_t n) {
    unsigned b = (n + 255) / 256;
    if (b > 8192) b = 8192;
    return b ? b : 1u;
}

// ---------------------------------------------------------------- voxel filter

// Leaf boxes, and the hash slots cleared: position s clears slots 2s and 2s + 1,
// so leaf [b, e) finds its region [2b, 2e) empty. A workgroup takes BOX_CHUNK
// positions at a time and reduces them first if they lie in one leaf, else
// each wave its part of every leaf: the atomics of a leaf all meet on six words
// (one leaf of 20k points: 24 us with a reduction per wave alone, this 5; 20
// leaves: 200 us with one atomic per point at the borders, this 11).
constexpr uint32_t BOX_CHUNK = 1024;
__global__ __launch_bounds__(256) void big_box_kernel(Plan P) {
    __shared__ float s_v[4][6];
    constexpr unsigned long long EMPTY = ~0ull;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    for (uint32_t c0 = blockIdx.x * BOX_CHUNK; c0 < P.n; c0 += gridDim.x * BOX_CHUNK) {
        const uint32_t c1 = min(P.n, c0 + BOX_CHUNK);
        const bool whole = P.leaf_of[c0] == P.leaf_of[c1 - 1u];  // leaf ids do not decrease
        float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
        for (uint32_t s0 = c0 + (tid & ~63u); s0 < c1; s0 += 256u) {
            const uint32_t s = s0 + lane;
            const bool in = s < c1;
            float x[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (in) {
                const float4 p = P.pos4[s];
                P.vox_keys[2 * (size_t)s] = EMPTY;
                P.vox_keys[2 * (size_t)s + 1] = EMPTY;
                P.vox_cnt[2 * (size_t)s] = 0u;
                P.vox_cnt[2 * (size_t)s + 1] = 0u;
                // (NaN coordinates drop out, as in a running fminf / fmaxf)
                x[0] = fminf(p.x, INFINITY), x[1] = fminf(p.y, INFINITY), x[2] = fminf(p.z, INFINITY);
                x[3] = fmaxf(p.x, -INFINITY), x[4] = fmaxf(p.y, -INFINITY), x[5] = fmaxf(p.z, -INFINITY);
            }
            if (whole) {
#pragma unroll
                for (int a = 0; a < 6; ++a) v[a] = a < 3 ? fminf(v[a], x[a]) : fmaxf(v[a], x[a]);
                continue;
            }
            // the leaves of these 64 positions in turn
            const uint32_t t = P.leaf_of[in ? s : c1 - 1u];
            unsigned long long left = __builtin_amdgcn_ballot_w64(in);
            while (left != 0ull) {
                const uint32_t lt = (uint32_t)__builtin_amdgcn_readlane((int)t, __ffsll((long long)left) - 1);
                const bool mine = in && t == lt;
                left &= ~__builtin_amdgcn_ballot_w64(mine);
#pragma unroll
                for (int a = 0; a < 6; ++a) {
                    const float none = a < 3 ? INFINITY : -INFINITY;
                    const float y = mine ? x[a] : none;
                    const float r = a < 3 ? wave_min(y, lane) : wave_max(y, lane);
                    if (lane == 0u)
                        atomicMax(P.leaf_box + 6 * (size_t)lt + a, a < 3 ? ~f32_ordered(r) : f32_ordered(r));
                }
            }
        }
        if (whole) {
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                v[a] = a < 3 ? wave_min(v[a], lane) : wave_max(v[a], lane);
                if (lane == 0u) s_v[wave][a] = v[a];
            }
            __syncthreads();
            if (tid < 6u) {
                float r = s_v[0][tid];
                for (int w = 1; w < 4; ++w) r = tid < 3u ? fminf(r, s_v[w][tid]) : fmaxf(r, s_v[w][tid]);
                atomicMax(P.leaf_box + 6 * (size_t)P.leaf_of[c0] + tid, tid < 3u ? ~f32_ordered(r) : f32_ordered(r));
            }
            __syncthreads();
        }
    }
}

struct BigLeaf {
    uint32_t b, nt;
    float lo[3], h;
};
__device__ __forceinline__ BigLeaf big_leaf(const Plan& P, uint32_t t, double beta) {
    BigLeaf L;
    L.b = P.leaf_begin[t];
    L.nt = P.leaf_begin[t + 1] - L.b;
    float hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        L.lo[a] = f32_from_ordered(~P.leaf_box[6 * (size_t)t + a]);
        hi[a] = f32_from_ordered(P.leaf_box[6 * (size_t)t + 3 + a]);
    }
    L.h = leaf_voxel_size(L.lo, hi, L.nt, beta);
    return L;
}

// Counts the points of each voxel in the leaf's hash region.
__global__ __launch_bounds__(256) void big_count_kernel(Plan P, double beta) {
    constexpr unsigned long long EMPTY = ~0ull;
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < P.n; s += gridDim.x * blockDim.x) {
        const uint32_t t = P.leaf_of[s];
        const BigLeaf L = big_leaf(P, t, beta);
        if (s == L.b) P.leaf_h[t] = L.h;
        if (L.h == 0.0f) continue;
        const unsigned long long k = vox_key(P.pos4[s], L.lo[0], L.lo[1], L.lo[2], (double)L.h);
        unsigned long long* tk = (unsigned long long*)P.vox_keys + 2 * (size_t)L.b;
        const uint32_t slots = 2u * L.nt;
        uint32_t slot = vox_hash(k) % slots;
        for (uint32_t probe = 0; probe < slots; ++probe) {
            const unsigned long long prev = atomicCAS(&tk[slot], EMPTY, k);
            if (prev == EMPTY || prev == k) {
                atomicAdd(&P.vox_cnt[2 * (size_t)L.b + slot], 1u);
                break;
            }
            slot = (slot + 1 == slots) ? 0u : slot + 1;
        }
    }
}

__global__ __launch_bounds__(256) void big_occ_kernel(Plan P, double beta, uint32_t nv) {
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < P.n; s += gridDim.x * blockDim.x) {
        const BigLeaf L = big_leaf(P, P.leaf_of[s], beta);
        uint32_t c = L.nt;
        if (L.h != 0.0f) {
            const unsigned long long k = vox_key(P.pos4[s], L.lo[0], L.lo[1], L.lo[2], (double)L.h);
            const unsigned long long* tk = (const unsigned long long*)P.vox_keys + 2 * (size_t)L.b;
            const uint32_t slots = 2u * L.nt;
            uint32_t slot = vox_hash(k) % slots;
            c = 0;
            for (uint32_t probe = 0; probe < slots; ++probe) {
                if (tk[slot] == k) {
                    c = P.vox_cnt[2 * (size_t)L.b + slot];
                    break;
                }
                slot = (slot + 1 == slots) ? 0u : slot + 1;
            }
        }
        P.occ[s] = c;
        P.p1[s] = c >= nv;
    }
}

// ---------------------------------------------------------------- selects

constexpr int BIG_BLOCK = 1024;
constexpr int BIG_WAVES = BIG_BLOCK / 64;

// The values a workgroup selects from: in registers (up to V * BIG_BLOCK of
// them), or read again in every pass.
template <class T, int V>
struct RegVals {
    T v[V];
    uint32_t n;
    template <class G>
    __device__ RegVals(uint32_t count, G get) : n(count) {
#pragma unroll
        for (int u = 0; u < V; ++u) v[u] = get(min(threadIdx.x + (uint32_t)u * BIG_BLOCK, n - 1u));
    }
    template <class F>
    __device__ void each(F f) const {
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const uint32_t i = threadIdx.x + (uint32_t)u * BIG_BLOCK;
            if (i < n) f(v[u], i);
        }
    }
};
template <class T, class G>
struct MemVals {
    G get;
    uint32_t n;
    template <class F>
    __device__ void each(F f) const {
        for (uint32_t i = threadIdx.x; i < n; i += BIG_BLOCK) f((T)get(i), i);
    }
};

// The non-zero values of another set. Points that a select has to rank below
// all others hold zeros; left in, a single zero makes the values differ from
// the top bit on, and the first passes then count nearly all of them in one bin.
template <class Vals>
struct NonZero {
    const Vals& vals;
    template <class F>
    __device__ void each(F f) const {
        vals.each([&](auto v, uint32_t i) {
            if (v != 0) f(v, i);
        });
    }
};

struct BigShared {
    uint32_t hist[256];
    uint32_t sel[4];
    unsigned long long red[BIG_WAVES][2];
    unsigned long long val;
};

// Value of ascending rank r (0-based, r < n). Radix select: the bits all
// values share are fixed first (otherwise every value would land in one bin of
// the first histograms), then digits of up to 8 bits from the highest
// differing bit down; a bin holding one value ends it. Whole workgroup.
template <class T, class Vals>
__device__ T big_select(const Vals& vals, uint32_t r, BigShared& sh) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    T a = ~(T)0, o = 0;
    vals.each([&](T v, uint32_t) {
        a &= v;
        o |= v;
    });
    a = wave_and(a);
    o = wave_or(o);
    __syncthreads();
    if (lane == 0u) {
        sh.red[wave][0] = a;
        sh.red[wave][1] = o;
    }
    __syncthreads();
    for (int w = 0; w < BIG_WAVES; ++w) {
        a &= (T)sh.red[w][0];
        o |= (T)sh.red[w][1];
    }
    if (a == o) return a;
    int top = 63 - __builtin_clzll((unsigned long long)(T)(a ^ o));
    T mask = top + 1 >= 8 * (int)sizeof(T) ? (T)0 : (T)(~(T)0 << (top + 1));
    T prefix = a & mask;
    while (true) {
        const int lo = top >= 7 ? top - 7 : 0;
        const uint32_t dm = (2u << (top - lo)) - 1u;
        __syncthreads();
        if (threadIdx.x < 256u) sh.hist[threadIdx.x] = 0u;
        __syncthreads();
        vals.each([&](T v, uint32_t) {
            if ((v & mask) == prefix) atomicAdd(&sh.hist[(uint32_t)(v >> lo) & dm], 1u);
        });
        __syncthreads();
        if (wave == 0u) {
            uint32_t h[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) h[q] = sh.hist[4u * lane + (uint32_t)q];
            const uint32_t s = h[0] + h[1] + h[2] + h[3];
            const uint32_t inc = wave_incl_scan(s), ex = inc - s;
            if (ex <= r && r < inc) {
                uint32_t acc = ex, b = 0;
                while (r >= acc + h[b]) acc += h[b++];
                sh.sel[0] = 4u * lane + b;
                sh.sel[1] = acc;
                sh.sel[2] = h[b];
            }
        }
        __syncthreads();
        r -= sh.sel[1];
        prefix |= (T)sh.sel[0] << lo;
        mask |= (T)dm << lo;
        if (lo == 0) return prefix;
        if (sh.sel[2] == 1u) {
            vals.each([&](T v, uint32_t) {
                if ((v & mask) == prefix) sh.val = v;
            });
            __syncthreads();
            return (T)sh.val;
        }
        top = lo - 1;
    }
}

// Given a = the value of ascending rank r, the value of rank r + 1: a again
// if more than r + 1 values are <= a, else the smallest value above a.
template <class T, class Vals>
__device__ T big_next_rank(const Vals& vals, uint32_t r, T a, BigShared& sh) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t le = 0;
    T mn = ~(T)0;
    vals.each([&](T v, uint32_t) {
        if (v <= a) ++le;
        else if (v < mn) mn = v;
    });
    le = wave_sum(le);
    mn = wave_umin(mn);
    __syncthreads();
    if (lane == 0u) {
        sh.red[wave][0] = le;
        sh.red[wave][1] = mn;
    }
    __syncthreads();
    uint32_t L = 0;
    T M = ~(T)0;
    for (int w = 0; w < BIG_WAVES; ++w) {
        L += (uint32_t)sh.red[w][0];
        const T x = (T)sh.red[w][1];
        M = x < M ? x : M;
    }
    return L > r + 1u ? a : M;
}

// Sums of two counts over the workgroup.
__device__ __forceinline__ uint2 big_sums(uint32_t a, uint32_t b, BigShared& sh) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    a = wave_sum(a);
    b = wave_sum(b);
    __syncthreads();
    if (lane == 0u) {
        sh.red[wave][0] = a;
        sh.red[wave][1] = b;
    }
    __syncthreads();
    uint2 t = make_uint2(0u, 0u);
    for (int w = 0; w < BIG_WAVES; ++w) {
        t.x += (uint32_t)sh.red[w][0];
        t.y += (uint32_t)sh.red[w][1];
    }
    return t;
}

// Density of every P1 point.
__global__ __launch_bounds__(256) void big_density_kernel(Plan P, uint32_t k) {
    const uint32_t np1 = P.ctr->n_p1;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < np1; q += gridDim.x * blockDim.x)
        (void)density_finish(P, k, q, density_load(P, q));
}

// Percentile cut (role 0, even blocks) and median density (role 1) of each leaf.
template <class R2, class Rho>
__device__ void big_cut_median(const Plan& P, const Params& prm, uint32_t role, uint32_t t, uint32_t n1, const R2& r2,
                               const Rho& rho, BigShared& sh) {
    if (role == 0u) {
        const float cut = __uint_as_float(big_select<uint32_t>(r2, n1 - percentile_rank(n1, prm.rho_percentile), sh));
        if (threadIdx.x == 0) P.leaf_r2cut[t] = cut;
    } else {
        // points without k candidates have density 0 and rank first
        uint32_t z = 0;
        rho.each([&](unsigned long long v, uint32_t) { z += v == 0ull ? 1u : 0u; });
        z = big_sums(z, 0u, sh).x;
        const uint32_t r = (n1 - 1u) / 2u;
        const NonZero<Rho> pos{rho};
        const unsigned long long ab = r < z ? 0ull : big_select<unsigned long long>(pos, r - z, sh);
        double med = __longlong_as_double((long long)ab);
        if ((n1 & 1u) == 0u) {
            const unsigned long long bb = big_next_rank<unsigned long long>(rho, r, ab, sh);
            med = (med + __longlong_as_double((long long)bb)) / 2.0;
        }
        if (threadIdx.x == 0) P.leaf_rho_med[t] = med;
    }
}

constexpr int BIG_V = 20;  // values per thread in registers: leaves of up to 20480 P1 points

__global__ __launch_bounds__(BIG_BLOCK) void big_select_kernel(Plan P, Params prm) {
    __shared__ BigShared sh;
    const uint32_t nl = P.ctr->n_leaves, role = blockIdx.x & 1u;
    for (uint32_t t = blockIdx.x >> 1; t < nl; t += gridDim.x >> 1) {
        const uint32_t qb = P.p1pos[P.leaf_begin[t]], n1 = P.p1pos[P.leaf_begin[t + 1]] - qb;
        if (n1 == 0u) {
            if (threadIdx.x == 0 && role == 1u) P.leaf_rho_med[t] = 0.0;
            continue;
        }
        auto r2 = [&](uint32_t i) { return __float_as_uint(P.r2k[qb + i]); };
        auto rho = [&](uint32_t i) { return (unsigned long long)__double_as_longlong(P.rho_c[qb + i]); };
        if (n1 > (uint32_t)(BIG_V * BIG_BLOCK)) {
            const MemVals<uint32_t, decltype(r2)> a{r2, n1};
            const MemVals<unsigned long long, decltype(rho)> b{rho, n1};
            big_cut_median(P, prm, role, t, n1, a, b, sh);
        } else if (role == 0u) {
            const RegVals<uint32_t, BIG_V> a(n1, r2);
            big_cut_median(P, prm, 0u, t, n1, a, MemVals<unsigned long long, decltype(rho)>{rho, n1}, sh);
        } else {
            const RegVals<unsigned long long, BIG_V> b(n1, rho);
            big_cut_median(P, prm, 1u, t, n1, MemVals<uint32_t, decltype(r2)>{r2, n1}, b, sh);
        }
        __syncthreads();
    }
}

// P2, the weight factors and the density powers from the leaf's cut and median.
template <bool SQRT>
__global__ __launch_bounds__(256) void big_weights_kernel(Plan P, Params prm) {
    const uint32_t np1 = P.ctr->n_p1;
    const double ha = prm.alpha / 2.0;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < np1; q += gridDim.x * blockDim.x) {
        const uint32_t t = P.cand_leaf[q];
        const double med = P.leaf_rho_med[t], rho = P.rho_c[q];
        const double den = med * med + prm.eps, sr = prm.sigma * P.r64_c[q];
        P.p2[q] = (P.krec[q].x != NO_NBR && P.r2k[q] <= P.leaf_r2cut[t]) ? 1 : 0;
        P.afac_c[q] = make_double2(pow_ha<SQRT>(rho / den, ha), 1.0 / (2.0 * sr * sr));
        P.gpow_p[q] = pow_ha<SQRT>(rho, ha);
    }
}

// Top-lambda cut of a leaf: the m-th largest key and, among the keys equal to
// it, the largest original index kept.
template <class Keys, class Idx>
__device__ void big_topl_cut(const Plan& P, double lambda, uint32_t t, uint32_t n1, const Keys& keys, Idx idx,
                             BigShared& sh) {
    uint32_t c = 0;
    keys.each([&](unsigned long long k, uint32_t) { c += k != 0ull ? 1u : 0u; });  // keys of P2 points are > 0
    const uint32_t n2 = big_sums(c, 0u, sh).x;
    const uint32_t m = topl_count(lambda, n2);
    unsigned long long theta = ~0ull;
    uint32_t icut = 0;
    if (m > 0u) {
        theta = big_select<unsigned long long>(NonZero<Keys>{keys}, n2 - m, sh);
        uint32_t g = 0, e = 0;
        keys.each([&](unsigned long long k, uint32_t) {
            g += k > theta ? 1u : 0u;
            e += k == theta ? 1u : 0u;
        });
        const uint2 ge = big_sums(g, e, sh);
        icut = 0xFFFFFFFFu;
        if (ge.y != m - ge.x) {
            // some of the keys equal to theta are dropped: the largest indices among them
            auto tie = [&](uint32_t i) -> uint32_t { return keys.at(i) == theta ? idx(i) : 0xFFFFFFFFu; };
            const MemVals<uint32_t, decltype(tie)> ties{tie, n1};
            icut = big_select<uint32_t>(ties, m - ge.x - 1u, sh);
        }
    }
    if (threadIdx.x == 0) {
        P.leaf_theta[t] = theta;
        P.leaf_icut[t] = icut;
    }
}

template <class Vals, class G>
struct WithAt {
    const Vals& vals;
    G get;
    template <class F>
    __device__ void each(F f) const { vals.each(f); }
    __device__ unsigned long long at(uint32_t i) const { return get(i); }
};

__global__ __launch_bounds__(BIG_BLOCK) void big_topl_kernel(Plan P, double lambda) {
    __shared__ BigShared sh;
    const uint32_t nl = P.ctr->n_leaves;
    for (uint32_t t = blockIdx.x; t < nl; t += gridDim.x) {
        const uint32_t qb = P.p1pos[P.leaf_begin[t]], n1 = P.p1pos[P.leaf_begin[t + 1]] - qb;
        if (n1 == 0u) continue;
        auto key = [&](uint32_t i) { return score_key(P.p2[qb + i] != 0, P.score_c[qb + i]); };
        auto idx = [&](uint32_t i) { return __float_as_uint(P.cand4[qb + i].w); };
        if (n1 > (uint32_t)(BIG_V * BIG_BLOCK)) {
            const MemVals<unsigned long long, decltype(key)> a{key, n1};
            big_topl_cut(P, lambda, t, n1, WithAt<decltype(a), decltype(key)>{a, key}, idx, sh);
        } else {
            const RegVals<unsigned long long, BIG_V> a(n1, key);
            big_topl_cut(P, lambda, t, n1, WithAt<decltype(a), decltype(key)>{a, key}, idx, sh);
        }
        __syncthreads();
    }
}

// Stage codes from the leaf's cut, and the outputs in input order.
__global__ __launch_bounds__(256) void big_stage_kernel(Plan P, ToplOut out) {
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < P.n; s += gridDim.x * blockDim.x) {
        const uint32_t i = P.idx_a[s];
        uint8_t st = 0;
        double sc = 0.0;
        if (P.p1[s]) {
            const uint32_t q = P.p1pos[s], t = P.leaf_of[s];
            const bool p2 = P.p2[q] != 0;
            sc = P.score_c[q];
            const unsigned long long k = score_key(p2, sc), theta = P.leaf_theta[t];
            st = !p2 ? 1 : (k > theta || (k == theta && i <= P.leaf_icut[t])) ? 3 : 2;
            P.stage_c[q] = st;
        }
        out.put(i, st, sc);
    }
}

// Workgroups for the selects: the leaves are few, but their number is only
// known on the device.
unsigned big_leaf_blocks(uint32_t n) {
    unsigned b = n / 256u + 1u;
    return b > 512u ? 512u : b;
}

}  // namespace

void launch_big_voxel(const Plan& P, const Params& prm, hipStream_t st) {
    const unsigned blocks = point_blocks(P.n);
    hipLaunchKernelGGL(big_box_kernel, dim3(blocks), dim3(256), 0, st, P);
    hipLaunchKernelGGL(big_count_kernel, dim3(blocks), dim3(256), 0, st, P, prm.beta);
    hipLaunchKernelGGL(big_occ_kernel, dim3(blocks), dim3(256), 0, st, P, prm.beta, (uint32_t)prm.min_vox_count);
}

void launch_big_select(const Plan& P, const Params& prm, hipStream_t st) {
    const unsigned blocks = point_blocks(P.n);
    hipLaunchKernelGGL(big_density_kernel, dim3(blocks), dim3(256), 0, st, P, (uint32_t)prm.k);
    hipLaunchKernelGGL(big_select_kernel, dim3(2 * big_leaf_blocks(P.n)), dim3(BIG_BLOCK), 0, st, P, prm);
    hipLaunchKernelGGL(prm.alpha == 1.0 ? big_weights_kernel<true> : big_weights_kernel<false>, dim3(blocks), dim3(256),
                       0, st, P, prm);
}

void launch_big_topl(const Plan& P, double lambda, const ToplOut& out, hipStream_t st) {
    hipLaunchKernelGGL(big_topl_kernel, dim3(big_leaf_blocks(P.n)), dim3(BIG_BLOCK), 0, st, P, lambda);
    hipLaunchKernelGGL(big_stage_kernel, dim3(point_blocks(P.n)), dim3(256), 0, st, P, out);
}

}  // namespace gdn
