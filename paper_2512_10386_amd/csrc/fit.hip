// Score fit (include/gdn.h, gdn_fit_loss_grad): the loss of a relaxed
// threshold on ln F_i and its gradient over alpha, sigma, gamma and tau, on
// the neighbour sets, densities, medians and P2 of the last pipeline pass.
//
// F_i follows Eq. 21 with the kernel of Eq. 20 raised to gamma/2:
//   t_ij = exp(alpha/2 * ln(rho_i rho_j / (rho_med^2 + eps)))     (Eq. 17)
//        * exp(-d_ij^2 / (2 sigma^2 r_K,i^2))                      (Eq. 18, 19)
//        * exp(-gamma/2 * ln(d_ij^2 + eps))                        (Eq. 20)
// and its log-derivatives are, term by term,
//   d/dalpha ln t = ln(ratio) / 2, d/dsigma ln t = d^2 / (sigma^3 r^2),
//   d/dgamma ln t = -ln(d^2 + eps) / 2.
// With y_i = 1 for a clean point, z_i = (ln F_i - tau) / T and
// p_i = sigmoid(z_i), the loss is the mean binary cross-entropy over the P2
// points with 0 < F_i < inf, and dL/dz_i = (p_i - y_i) / count.
//
// One lane per neighbour (as the score kernel); per-block partial sums in a
// fixed order, then one block sums the partials: the result does not depend
// on scheduling.
#include <algorithm>
#include <limits>

#include "kernels.hpp"
#include "wave.hpp"

namespace gdn {

namespace {

constexpr int FIT_PARTS = 6;        // loss, d/dalpha, d/dsigma, d/dgamma, d/dtau, count
constexpr int FIT_STRIDE = 8;       // doubles per block partial
constexpr unsigned FIT_BLOCKS_MAX = 1024;

__device__ __forceinline__ double seg_sum_f(double v, uint32_t kp) {
    for (uint32_t o = kp >> 1; o > 0; o >>= 1) v += __shfl_xor(v, (int)o, 64);
    return v;
}

__device__ __forceinline__ double wave_sum_f(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ln rho of every P1 point, at its P1 position (where the neighbour lists
// point). rho = 0 (fewer than k candidates) gives -inf.
__global__ __launch_bounds__(256) void fit_prep_kernel(Plan P, double* __restrict__ lrho_p) {
    const uint32_t np1 = P.ctr->n_p1;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < np1; q += gridDim.x * blockDim.x)
        lrho_p[q] = log(P.rho_c[q]);
}

template <int M>
__device__ __forceinline__ double xor_f64(double v, uint32_t lane) {
    return __longlong_as_double((long long)xor_lane_key<M>((unsigned long long)__double_as_longlong(v), lane));
}

// Sums of v[0..3] over each segment of kp >= 4 lanes: lanes 0, 1, 2, 3 of the
// segment get the sums of v[0], v[2], v[1], v[3]. The first two exchanges each
// halve the number of values a lane carries: 5 exchanges for 16 lanes instead
// of 16.
__device__ __forceinline__ double seg_sum4(const double (&v)[4], uint32_t kp, uint32_t lane) {
    const bool b0 = (lane & 1u) != 0u, b1 = (lane & 2u) != 0u;
    const double u0 = (b0 ? v[2] : v[0]) + xor_f64<1>(b0 ? v[0] : v[2], lane);
    const double u1 = (b0 ? v[3] : v[1]) + xor_f64<1>(b0 ? v[1] : v[3], lane);
    double w = (b1 ? u1 : u0) + xor_f64<2>(b1 ? u0 : u1, lane);
    if (kp > 4u) w += xor_f64<4>(w, lane);
    if (kp > 8u) w += xor_f64<8>(w, lane);
    if (kp > 16u) w += xor_f64<16>(w, lane);
    if (kp > 32u) w += xor_f64<32>(w, lane);
    return w;
}

// FP64 exponentials and logarithms bound this kernel. Each wave takes
// FIT_TILE queries at a time: what depends on the query alone (ln rho -
// ln(rho_med^2 + eps) and 1 / r_K^2) one lane per query, into LDS; the neighbour
// terms one lane per neighbour, with one logarithm and one exponential per term
// (the three exponents are added first, their rounding errors carried along),
// the sums into LDS; then the loss of the tile's queries one lane per query. (With three
// logarithms and three exponentials per term and the loss evaluated by one
// lane per segment: 62 us for 107k P1 points at k = 16, this 27.)
constexpr uint32_t FIT_TILE = 32;

// -1 / (2 sigma^2) in two parts, and 1 / sigma^3.
struct FitSigma {
    double hi, lo, cube;
};

__global__ __launch_bounds__(256) void fit_kernel(Plan P, const uint8_t* __restrict__ label,
                                                  const double* __restrict__ lrho_p, int kk, FitArgs a, FitSigma S,
                                                  double* __restrict__ part) {
    __shared__ double s_red[4][FIT_PARTS];
    __shared__ double2 s_own[4][FIT_TILE];    // per wave and query: its part of ln(ratio), 1 / r_K^2
    __shared__ double s_sum[4][4][FIT_TILE];  // per wave and query: F and its three weighted sums
    const uint32_t np1 = P.ctr->n_p1;
    const uint32_t k = (uint32_t)kk;
    uint32_t kp = 1;
    while (kp < k) kp <<= 1;
    const uint32_t qpw = min(64u / kp, FIT_TILE);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, seg = lane / kp, r = lane % kp;
    const uint32_t wid = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const double ha = 0.5 * a.alpha, hg = -0.5 * a.gamma;
    double acc[FIT_PARTS] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // what a tile's queries read (lane l: query l of the tile) is fetched while
    // the tile before it is worked on, the leaf's median one step behind the leaf
    bool mine = false;
    uint32_t leaf = 0;
    double lrho = 0.0, r64 = 1.0, med = 0.0;
    auto fetch = [&](uint32_t q0) {
        const uint32_t ql = q0 + lane;
        mine = lane < FIT_TILE && ql < np1;
        if (mine) {
            mine = P.p2[ql] != 0;
            leaf = P.cand_leaf[ql];
            lrho = lrho_p[ql];
            r64 = P.r64_c[ql];
        }
    };
    auto fetch_median = [&]() {
        if (mine) med = P.leaf_rho_med[leaf];
    };
    const uint32_t first = wid * FIT_TILE;
    fetch(first);
    fetch_median();
    for (uint32_t q0 = first; q0 < np1; q0 += nw * FIT_TILE) {
        const bool live = mine;  // the loss of query q0 + lane is this lane's
        if (lane < FIT_TILE)  // (queries outside P2: a radius that none has)
            s_own[wave][lane] = live ? make_double2(lrho - log(med * med + a.eps), 1.0 / (r64 * r64)) : make_double2(0.0, -1.0);
        wave_lds_fence();
        fetch(q0 + nw * FIT_TILE);
        for (uint32_t i0 = 0; i0 < FIT_TILE; i0 += qpw) {
            const uint32_t qi = q0 + i0 + seg;
            double v[4] = {0.0, 0.0, 0.0, 0.0};
            const double2 own = seg < qpw ? s_own[wave][i0 + seg] : make_double2(0.0, -1.0);
            if (r < k && !(own.y < 0.0)) {
                const uint32_t j = P.nbr[(size_t)qi * k + r];
                if (j < P.n) {
                    const double lr = own.x + lrho_p[j];
                    // the neighbour (P1 position j) and the query from their sorted
                    // copies of the input coordinates
                    const float4 cj = P.cand4[j], ci = P.cand4[qi];
                    const double dx = (double)cj.x - (double)ci.x;
                    const double dy = (double)cj.y - (double)ci.y;
                    const double dz = (double)cj.z - (double)ci.z;
                    const double d2 = dx * dx + dy * dy + dz * dz;
                    const double lk = log(d2 + a.eps);
                    // d^2 / r^2 (0 for a neighbour at d = 0, also when r = 0)
                    const double dr = d2 != 0.0 ? d2 * own.y : 0.0;
                    const double ea = ha * lr, es = S.hi * dr, eg = hg * lk;
                    // x = ea + es + eg, and what the products and sums rounded off
                    const double p = ea + eg, pb = p - ea;
                    const double x = p + es, xb = x - p;
                    const double xe = (((ea - (p - pb)) + (eg - pb)) + ((p - (x - xb)) + (es - xb))) +
                                      ((fma(ha, lr, -ea) + fma(hg, lk, -eg)) + (fma(S.hi, dr, -es) + S.lo * dr));
                    double tt = exp(x);
                    if (tt != 0.0) {
                        tt += isfinite(x) ? tt * xe : 0.0;
                        v[0] = tt;
                        v[1] = tt * 0.5 * lr;
                        v[2] = tt * dr;  // over sigma^3 at the end
                        v[3] = tt * (-0.5 * lk);
                    }
                }
            }
            if (kp >= 4u) {
                const double w = seg_sum4(v, kp, lane);
                if (r < 4u) s_sum[wave][r == 1u ? 2u : r == 2u ? 1u : r][i0 + seg] = w;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double w = seg_sum_f(v[c], kp);
                    if (r == 0u && seg < qpw) s_sum[wave][c][i0 + seg] = w;
                }
            }
        }
        wave_lds_fence();
        fetch_median();
        if (live) {
            const double F = s_sum[wave][0][lane];
            if (F > 0.0 && F < INFINITY) {
                const double y = label[__float_as_uint(P.cand4[q0 + lane].w)] ? 0.0 : 1.0;
                const double z = (log(F) - a.tau) / a.T;
                const double p = 1.0 / (1.0 + exp(-z));
                acc[0] += (z > 0.0 ? z + log1p(exp(-z)) : log1p(exp(z))) - y * z;
                const double g = (p - y) / a.T;
                acc[1] += g * s_sum[wave][1][lane] / F;
                acc[2] += g * s_sum[wave][2][lane] / F;
                acc[3] += g * s_sum[wave][3][lane] / F;
                acc[4] -= g;
                acc[5] += 1.0;
            }
        }
        wave_lds_fence();  // the sums are read before the next tile's are written
    }
#pragma unroll
    for (int c = 0; c < FIT_PARTS; ++c) {
        const double v = wave_sum_f(c == 2 ? acc[c] * S.cube : acc[c]);
        if (lane == 0) s_red[wave][c] = v;
    }
    __syncthreads();
    if (threadIdx.x < FIT_PARTS) {
        const uint32_t c = threadIdx.x;
        part[(size_t)blockIdx.x * FIT_STRIDE + c] = ((s_red[0][c] + s_red[1][c]) + s_red[2][c]) + s_red[3][c];
    }
}

// One block: sums the block partials in a fixed order and normalises by the
// count. Each thread reads one partial's six values at once (one wave alone
// took 18 us for 1024 partials: 16 round trips in turn).
constexpr int FIT_FINAL = 1024;
static_assert(FIT_BLOCKS_MAX <= (unsigned)FIT_FINAL, "a thread per partial");
__global__ __launch_bounds__(FIT_FINAL) void fit_final_kernel(const double* __restrict__ part, uint32_t nb,
                                                              double* __restrict__ out) {
    __shared__ double s_red[FIT_FINAL / 64][FIT_PARTS];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    double v[FIT_PARTS];
#pragma unroll
    for (int c = 0; c < FIT_PARTS; ++c)
        v[c] = threadIdx.x < nb ? part[(size_t)threadIdx.x * FIT_STRIDE + c] : 0.0;
#pragma unroll
    for (int c = 0; c < FIT_PARTS; ++c) {
        const double w = wave_sum_f(v[c]);
        if (lane == 0u) s_red[wave][c] = w;
    }
    __syncthreads();
    if (threadIdx.x < FIT_PARTS) {
        double cnt = 0.0, t = 0.0;
        for (int w = 0; w < FIT_FINAL / 64; ++w) {
            cnt += s_red[w][5];
            t += s_red[w][threadIdx.x];
        }
        out[threadIdx.x] = threadIdx.x == 5 ? cnt : t / (cnt > 0.0 ? cnt : 1.0);
    }
}

unsigned fit_blocks(uint32_t n) {
    uint64_t b = ((uint64_t)n + 4 * FIT_TILE - 1) / (4 * FIT_TILE);
    if (b > FIT_BLOCKS_MAX) b = FIT_BLOCKS_MAX;
    return b == 0 ? 1u : (unsigned)b;
}

}  // namespace

size_t fit_workspace_bytes(uint32_t n) {
    return (((size_t)8 * n + 255) & ~(size_t)255) + (size_t)FIT_STRIDE * 8 * FIT_BLOCKS_MAX;
}

void launch_fit(const Plan& P, const float*, const uint8_t* label, const FitArgs& a, void* workspace,
                double* out, hipStream_t st) {
    double* lrho_p = (double*)workspace;
    double* part = (double*)((char*)workspace + (((size_t)8 * P.n + 255) & ~(size_t)255));
    unsigned pb = (P.n + 255) / 256;
    if (pb > 4096) pb = 4096;
    if (pb == 0) pb = 1;
    hipLaunchKernelGGL(fit_prep_kernel, dim3(pb), dim3(256), 0, st, P, lrho_p);
    const unsigned nb = fit_blocks(P.n);
    // (a bandwidth so small that its powers overflow leaves the neighbours at
    // d = 0 alone, whose d^2 / r^2 = 0 must not meet an infinity)
    const long double top = std::numeric_limits<double>::max();
    const long double s2 = (long double)a.sigma * a.sigma, h = std::max(-0.5L / s2, -top);
    const FitSigma S{(double)h, (double)(h - (double)h), (double)std::min(1.0L / (s2 * a.sigma), top)};
    hipLaunchKernelGGL(fit_kernel, dim3(nb), dim3(256), 0, st, P, label, lrho_p, P.k, a, S, part);
    hipLaunchKernelGGL(fit_final_kernel, dim3(1), dim3(FIT_FINAL), 0, st, part, nb, out);
}

}  // namespace gdn
