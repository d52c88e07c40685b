// Per-point pieces the select and output kernels share: the density (Eq. 13),
// the density weight's power, the top-lambda key and the output record.
#pragma once

#include "common.hpp"

namespace gdn {

constexpr uint32_t NO_NBR = 0xFFFFFFFFu;
constexpr double PI_D = 3.14159265358979323846;

// x^(alpha/2) of the density weight (Eq. 17): the square root for the
// default alpha = 1 (a few instructions instead of a general FP64 power; the
// two agree to an ulp), pow otherwise. The select kernels are instantiated
// for either, so each holds only the code it runs.
template <bool SQRT>
__device__ __forceinline__ double pow_ha(double x, double ha) {
    if constexpr (SQRT) return sqrt(x);
    else return pow(x, ha);
}

// Density of P1 query qi. The list is sorted by fp32 d2, and fp32 d2 is
// within ~6e-7 relative of the exact value, so only the neighbours whose fp32
// d2 is within 2^-16 of the k-th can hold the FP64 maximum. Usually that is
// the k-th alone (the (k-1)-th lies below), read from the dense record the
// kNN writes; otherwise walk the list down from the k-th and stop at the
// first one below. Stores r^2_K, rho and r densely (the selects run it for
// their leaf's points, so the density needs no launch of its own).
struct Dens {
    float r2;
    double rho, r64;
    bool short_list;  // fewer than k candidates
};

// What the density of a query starts from: its k-th neighbour record and the
// coordinates of the query and of that neighbour (the query's again when it
// has none), all loaded at once.
struct DensIn {
    uint4 kr;
    float4 cq, cj;
};
__device__ __forceinline__ DensIn density_load(const Plan& P, uint32_t qi) {
    DensIn d;
    d.kr = P.krec[qi];
    d.cq = P.cand4[qi];
    d.cj = P.cand4[d.kr.x < P.n ? d.kr.x : qi];
    return d;
}

__device__ __forceinline__ Dens density_finish(const Plan& P, uint32_t k, uint32_t qi, const DensIn& in) {
    const uint4 kr = in.kr;
    const uint32_t jk = kr.x;
    Dens out;
    out.r2 = __uint_as_float(kr.z);
    out.short_list = jk == NO_NBR;
    if (out.short_list) {
        out.rho = 0.0;
        out.r64 = INFINITY;
    } else {
        // the query's coordinates: cand4 holds bit copies of the input
        const double xi = in.cq.x, yi = in.cq.y, zi = in.cq.z;
        // a neighbour's sorted copy of the input coordinates
        auto d2_of = [&](const float4 cj) -> double {
            const double dx = (double)cj.x - xi;
            const double dy = (double)cj.y - yi;
            const double dz = (double)cj.z - zi;
            return dx * dx + dy * dy + dz * dz;
        };
        auto d2_to = [&](uint32_t j) -> double { return d2_of(P.cand4[j]); };
        const float thr = out.r2 * (1.0f - 1.0f / 65536.0f);
        double m2 = 0.0;
        if (k == 1u || __uint_as_float(kr.y) < thr) {
            if (jk < P.n) m2 = fmax(m2, d2_of(in.cj));
        } else {
            const uint32_t* nb = P.nbr + (size_t)qi * k;
            const float* d2 = P.nbr_d2 + (size_t)qi * k;
            for (int r = (int)k - 1; r >= 0; --r) {
                if (d2[r] < thr) break;
                const uint32_t j = nb[r];
                if (j >= P.n) continue;
                const double v = d2_to(j);
                if (v > m2) m2 = v;
            }
        }
        out.r64 = sqrt(m2);
        out.rho = (double)k / ((4.0 / 3.0) * PI_D * (out.r64 * out.r64 * out.r64));
    }
    P.r2k[qi] = out.r2;
    P.rho_c[qi] = out.rho;
    P.r64_c[qi] = out.r64;
    return out;
}

__device__ __forceinline__ unsigned long long score_key(bool p2, double f) {
    if (!p2) return 0ull;
    if (isnan(f)) return 1ull;
    return (unsigned long long)__double_as_longlong(f) + 2ull;
}
// Outputs in input order for every point of each leaf: keep, score and stage
// as outputs_kernel writes them, or (rec) packed records as outputs_pack_kernel
// does, so that those passes are not needed.
struct ToplOut {
    uint2* rec;
    uint8_t* keep;
    float* score;
    uint8_t* stage;
    __device__ void put(uint32_t i, uint8_t st, double sc) const {
        if (rec) {
            rec[i] = make_uint2(__float_as_uint(st >= 2 ? (float)sc : -1.0f), st);
            return;
        }
        keep[i] = st == 3;
        score[i] = st >= 2 ? (float)sc : -1.0f;
        if (stage) stage[i] = st;
    }
};

// Number of the leaf's n1 densities that stay below the percentile cut's rank:
// MATLAB prctile keeps the densities >= the c-th smallest, c = ceil(n1*q/100 +
// 0.5) clamped to [1, n1].
__device__ __forceinline__ uint32_t percentile_rank(uint32_t n1, double q) {
    double cd = ceil((double)n1 * q / 100.0 + 0.5);
    if (cd < 1.0) cd = 1.0;
    if (cd > (double)n1) cd = (double)n1;
    return (uint32_t)cd;
}

// Points kept by top-lambda: min(n2, ceil(lambda * n2)).
__device__ __forceinline__ uint32_t topl_count(double lambda, uint32_t n2) {
    if (n2 == 0u) return 0u;
    const double mf = ceil(lambda * (double)n2);
    return mf >= (double)n2 ? n2 : (uint32_t)mf;
}

}  // namespace gdn
