// One tile of a stable LSD radix pass (8-bit digits) in the onesweep style:
// local ranks by wave-level digit matching, digit offsets of earlier tiles by
// decoupled look-back (bounded waits), global digit bases from the histogram.
#pragma once

#include "common.hpp"

namespace gdn {

// Sorts tile `tile` of n (key, payload) pairs by digit(key, payload, in
// range); a BLOCK-thread workgroup calls it with nothing pending on its
// LDS. IDENT: the payload is the position itself and vin is not read.
//   hist    this pass's digit totals [256]
//   status  look-back words [tiles][256], zero before the launch
//   flag    word that gets `flag_bit` when a look-back wait expires
//   Digit   operator()(K, uint32_t, bool ok); of_key(): the digit is
//           key_digit(key) alone (otherwise it is staged beside the key)
template <int ITEMS, bool IDENT, int BLOCK, class K, class Digit>
__device__ __forceinline__ void radix_tile(const K* __restrict__ kin, const uint32_t* __restrict__ vin,
                                           K* __restrict__ kout, uint32_t* __restrict__ vout, uint32_t n,
                                           uint32_t tile, const uint32_t* __restrict__ hist, uint32_t* status,
                                           uint32_t* flag, uint32_t flag_bit, const Digit digit) {
    constexpr int Q = BLOCK / 256;  // threads per digit, each for four waves
    __shared__ uint32_t s_w[BLOCK / 64][256];
    __shared__ uint32_t s_part[Q > 1 ? Q : 1][Q > 1 ? 256 : 1];
    __shared__ uint32_t s_base[256];
    __shared__ uint32_t s_scan[BLOCK / 64 + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // this digit's total over the pass, needed only after the ranking: read first
    const uint32_t hv = tid < 256 ? hist[tid] : 0u;
    for (int i = tid; i < (BLOCK / 64) * 256; i += BLOCK) (&s_w[0][0])[i] = 0u;

    K key[ITEMS];
    uint32_t val[ITEMS], dig[ITEMS], rank[ITEMS];
    // Tile = workgroup index. Each XCD starts its workgroups in index order,
    // so every tile a look-back waits on has been started and only waits on
    // lower tiles in turn; the waits are bounded anyway (SPIN_LIMIT, then a
    // status bit). A tile counter taken with an atomic cost a round trip
    // before the loads, and on large inputs, where the workgroups that start
    // together race for it, a second load of the tile.
    const uint32_t tbase = tile * (BLOCK * ITEMS) + wave * (64 * ITEMS);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t pos = tbase + i * 64 + lane;
        const bool ok = pos < n;
        key[i] = ok ? kin[pos] : (K)0;
        if constexpr (IDENT) val[i] = pos;
        else val[i] = ok ? vin[pos] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t pos = tbase + i * 64 + lane;
        const bool ok = pos < n;
        const uint32_t d = digit(key[i], val[i], ok);
        dig[i] = ok ? d : 256u;
    }
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t d = dig[i];
        const bool ok = d < 256u;
        const uint64_t m = match_digit(d, __ballot(ok));
        uint32_t before = __popcll(m & lt_mask);
        uint32_t cnt = __popcll(m);
        uint32_t wb = ok ? s_w[wave][d & 255u] : 0u;
        rank[i] = wb + before;
        bool leader = ok && ((m >> lane) == 1ull);
        if (leader) s_w[wave][d] = wb + cnt;
    }
    __syncthreads();

    // per digit: offsets of the waves of this tile, tile total
    uint32_t tcnt = 0;
    {
        const int d = tid & 255, q = tid >> 8;
        uint32_t c[4], run = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            c[w] = s_w[4 * q + w][d];
            tcnt += c[w];
        }
        if constexpr (Q > 1) {
            s_part[q][d] = tcnt;
            __syncthreads();
            tcnt = 0;
#pragma unroll
            for (int r = 0; r < Q; ++r) {
                const uint32_t v = s_part[r][d];
                run += r < q ? v : 0u;
                tcnt += v;
            }
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            s_w[4 * q + w][d] = run;
            run += c[w];
        }
    }
    // look-back over earlier tiles, digit by digit
    uint32_t* st = status + (size_t)tile * 256 + tid;
    uint32_t excl = 0;
    if (Q == 1 || tid < 256) st_relaxed_agent(st, (tile == 0 ? LB_FLAG_PRE : LB_FLAG_AGG) | tcnt);
    // global base of each digit (while the earlier tiles publish theirs)
    uint32_t total;
    const uint32_t gex = block_excl_scan(hv, s_scan, &total);
    if (tile != 0 && (Q == 1 || tid < 256)) {
        // LB_WINDOW predecessors per round trip; consume ready words nearest
        // first until an inclusive prefix, stop at the first one not ready
        int j = (int)tile - 1;
        uint32_t spins = 0;
        while (j >= 0) {
            uint32_t w[LB_WINDOW];
#pragma unroll
            for (int b = 0; b < LB_WINDOW; ++b)
                w[b] = j - b >= 0 ? ld_relaxed_agent(status + (size_t)(j - b) * 256 + tid) : 0u;
            int used = 0;
            bool stop = false, pre = false;
#pragma unroll
            for (int b = 0; b < LB_WINDOW; ++b) {
                if (!stop) {
                    if (j - b < 0 || (w[b] & ~LB_VALUE) == 0u) {
                        stop = true;
                    } else {
                        excl += w[b] & LB_VALUE;
                        ++used;
                        if (w[b] & LB_FLAG_PRE) pre = stop = true;
                    }
                }
            }
            if (pre) break;
            j -= used;
            if (used == 0) {
                if (++spins > SPIN_LIMIT) {
                    atomicOr(flag, flag_bit);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        st_relaxed_agent(st, LB_FLAG_PRE | ((excl + tcnt) & LB_VALUE));
    }
    if (Q == 1 || tid < 256) s_base[tid] = gex + excl;
    if constexpr (ITEMS * BLOCK >= 4096) {
        // Large tiles (inputs above 2^20): stage the tile in LDS in digit order, then write each
        // digit's run with consecutive threads (coalesced) instead of
        // scattering from registers.
        __shared__ K s_k[BLOCK * ITEMS];
        __shared__ uint32_t s_v[BLOCK * ITEMS];
        __shared__ uint8_t s_dg[BLOCK * ITEMS];  // digits that are not of the key, found once per element
        __shared__ uint32_t s_toff[256];
        uint32_t ttot;
        const uint32_t tex = block_excl_scan(Q == 1 || tid < 256 ? tcnt : 0u, s_scan, &ttot);
        if (Q == 1 || tid < 256) s_toff[tid] = tex;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t d = dig[i];
            if (d < 256u) {
                const uint32_t lp = s_toff[d] + s_w[wave][d] + rank[i];
                s_k[lp] = key[i];
                s_v[lp] = val[i];
                if (!digit.of_key()) s_dg[lp] = (uint8_t)d;
            }
        }
        __syncthreads();
        for (uint32_t p = tid; p < ttot; p += BLOCK) {
            const K kk = s_k[p];
            const uint32_t vv = s_v[p];
            const uint32_t d = digit.of_key() ? digit.key_digit(kk) : (uint32_t)s_dg[p];
            const uint32_t o = s_base[d] + (p - s_toff[d]);
            if (o < n) {  // always true unless a look-back wait expired
                kout[o] = kk;
                vout[o] = vv;
            }
        }
    } else {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t d = dig[i];
            if (d < 256u) {
                const uint32_t o = s_base[d] + s_w[wave][d] + rank[i];
                if (o < n) {  // always true unless a look-back wait expired
                    kout[o] = key[i];
                    vout[o] = val[i];
                }
            }
        }
    }
}

}  // namespace gdn
