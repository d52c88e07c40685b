// Shared device helpers and the workspace plan of the gfx950 denoiser.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gdn {

constexpr int MORTON_BITS = 21;
constexpr uint32_t QMAX = (1u << MORTON_BITS) - 1u;

// Tile sizes.
constexpr int SORT_PASSES = 8;                // 8-bit digits over the 63-bit key
constexpr int SORT_FRAME_PASSES_MAX = 2;      // 8-bit digits of the frame id (batches)
constexpr int SORT_PASSES_MAX = SORT_PASSES + SORT_FRAME_PASSES_MAX;
constexpr uint32_t SORT_FOFF_LDS = 2048;      // frame offsets staged in LDS by frame passes (nf < this)
// Short sort: the radix passes cover only digits 4..7 (key bits 32..62),
// which hold every level-10 cell prefix (bits 33..62); the points end in
// (frame, bits 32..62, original index) order. A level-10 cell that holds
// more than leaf_cap points (and lies above the depth limit) splits further:
// such "deep" cells are found after the sort and each is sorted on its whole
// key by one workgroup, so the octree sees full key order wherever it goes
// below level 10.
constexpr int SORT_SHORT_LEVEL = 10;
constexpr int SORT_SHORT_FIRST = 4;
static_assert(3 * (MORTON_BITS - SORT_SHORT_LEVEL) >= 8 * SORT_SHORT_FIRST, "short sort must hold the cell prefix");
static_assert(SORT_SHORT_FIRST % 2 == 0, "skipped passes keep the ping-pong parity");
constexpr uint32_t MAX_FRAMES = 4096;         // frames per batched call (frame table staged in LDS)
constexpr int SCAN_BLOCK = 512;                // look-back scan workgroup (fewer tiles to look back over than 256)
constexpr int SCAN_ITEMS = 16;
constexpr uint32_t SCAN_SMALL_N = 1u << 20;   // scans up to this size: 4 items per thread
constexpr int SCAN_SLOTS = 3;                 // scans per call: leaves, P1, keep
constexpr int PLAN_CLASSES = 4;               // queue classes of unchunked leaves
constexpr int PLAN_COUNTERS = 2 + PLAN_CLASSES;
constexpr int PLAN_CLASS_SHIFT = 29;          // leaf_item of such plans: counter, place among its items
// Inputs whose kNN queue is ordered by class. A sweep of 1M points ends on
// its few heaviest items unless they start first: 1404 us a call in leaf order
// and 1245 by class (caps 512 and 1024, three seeds each: 3 to 14 % less); nine
// sweeps of 100k gain up to 3 % at cap 256 and 0 to 1 % above. At 64 sweeps, 6.2M
// points, the end is short against the rest, and leaf order, where items that
// run together share their candidates, is ahead: 3992 and 4028 us.
constexpr uint32_t PLAN_CLASS_MAX_N = 1u << 21;
static_assert(2ull * PLAN_CLASS_MAX_N + 64 < 1ull << PLAN_CLASS_SHIFT, "a place fits below the class");
constexpr uint32_t PLAN_ONE_MAX_N = 1u << 19;  // kNN plan: one workgroup up to this size, parallel above
constexpr int PLAN_LEVELS = 8;                // candidate chunk lengths chunk0 << 0..7 (parallel plan)
// Default initial candidate chunk: in effect none (lengths double up to 2^30
// from here). A query tests few of a leaf's culling groups, so a split walks
// the group boxes sooner at the price of a partial list per chunk, their merge
// and a weaker bound in each. Whole calls with chunks of 8192 / 32768 / none:
// 120k sweep at cap 1024 309 / 288 / 276 us, 250k 446 / 423 / 416, 100k at cap
// 4096 442 / 392 / 338, 300k in one leaf - / 3647 / 3252, 20k objects 138 / 135
// / 135. Up to this size the merge and the plan's check are not launched.
constexpr int KNN_CC0 = 1 << 23;
static_assert((long long)KNN_CC0 << (PLAN_LEVELS - 1) <= 1ll << 30, "the candidate chunk lengths are 32-bit");
constexpr int KNN_TQ = 8;                     // queries per kNN work item (one wave), at most
constexpr int KNN_NCH_MAX = 32;               // max candidate chunks per leaf
constexpr int KNN_GRP = 64;                   // P1 positions per culling group of the kNN (one per lane)
constexpr uint32_t KNN_STREAMS = 64;          // kNN work-queue streams (cursors)
constexpr int HALO = 27;
constexpr int VOX_BLOCK = 256;
constexpr int VOX_LDS_SLOTS = 4096;           // LDS hash slots (leaves <= 2048 pts)
constexpr int SEL_BLOCK = 256;

// Status word packing for decoupled look-back: 2 flag bits + 30 value bits.
constexpr uint32_t LB_FLAG_AGG = 1u << 30;
constexpr uint32_t LB_FLAG_PRE = 2u << 30;
constexpr uint32_t LB_VALUE = (1u << 30) - 1u;
constexpr uint32_t SPIN_LIMIT = 1u << 22;

constexpr uint32_t DEV_NONFINITE = 1u;
constexpr uint32_t DEV_WAIT_LIMIT = 2u;
constexpr uint32_t DEV_BAD_FRAMES = 4u;

// Per-frame bounding-box accumulators (inside the zeroed block).
struct FrameStat {
    uint32_t bbox_max[3];   // ordered-uint max of x, y, z
    uint32_t bbox_nmin[3];  // ordered-uint max of ~x (i.e. the min)
    uint32_t nonfinite;
    uint32_t pad;
};

// Scalars the kernels share through device memory (inside the zeroed block).
struct Counters {
    uint32_t status;
    uint32_t n_leaves;
    uint32_t n_p1;
    uint32_t n_items;
    uint32_t n_kept;
    unsigned long long pairs;
    uint32_t n_chunked_items; // kNN items of chunked leaves (they come first)
    uint32_t pad;
    uint32_t knn_tq;          // queries per kNN work item (a power of two)
    // plans that give each class its own count (halo kernel, parallel plan):
    // partial lists, items of chunked leaves, items of each class
    uint32_t plan_q[PLAN_COUNTERS];
    uint32_t n_deep;          // 1: some level-10 cell is marked for the re-sort
    uint32_t n_vox_big;       // 1: some leaf is left to voxel_kernel by voxel_wave_kernel
    uint32_t n_big;           // 1: some leaf has more than SMALL_LEAF P1 points
    unsigned long long plan_acc[PLAN_LEVELS][3];  // per candidate chunk length: lists, items, chunked items
    unsigned long long plan_pairs;
    // kNN work queue: item i belongs to stream i % KNN_STREAMS; one cursor
    // per stream, each on its own 128-byte line
    uint32_t knn_q[KNN_STREAMS][32];
};

// Frame constants derived on the device from the bounding box.
struct FrameConst {
    float lo[3];
    int32_t dmax;
    double S;
    double scale;
};

// Bounding box of the P1 points at positions [KNN_GRP g, KNN_GRP (g + 1)).
struct GroupBox {
    float4 lo, hi;  // w unused
};

// One kNN work item: queries [q0, q1) of leaf `leaf` against candidate chunk
// `chunk`.
struct __align__(16) KnnItem {
    uint32_t leaf, q0, q1, chunk;
};

// Leaves of at most SMALL_LEAF P1 points take one wave in the density and
// top-lambda selects (four values per lane, no block barriers) where the input
// has so many of them that a workgroup per leaf runs in many rounds: above
// 2^20 points, above 2^19 with a leaf cap of at most 512, or above 3 * 2^16
// with one of at most 256. Whole calls, workgroups against waves: 120k points
// at cap 256 206 and 209 us, 250k 299.5 and 289, 500k 495 and 458, 200k on a
// torus 205.5 and 196.7; at cap 512 900k in nine frames 936 and 926.
constexpr uint32_t SMALL_LEAF = 256;
constexpr uint32_t SEL_LDS_MAX = 2048;  // leaves up to this size are selected from LDS
inline bool small_leaf_path(uint32_t n, int32_t leaf_cap) {
    return n > (1u << 20) || (n > (1u << 19) && leaf_cap <= 512) || (n > (3u << 16) && leaf_cap <= 256);
}

// Leaf caps above SEL_LDS_MAX (the octree switched off, or nearly) leave a
// frame with few leaves of many points. One workgroup per leaf then holds the
// whole frame up: one leaf of 20k points took 250 us in the voxel filter, 142
// in the density select and 201 in top-lambda (now 15, 33 and 27). Such calls
// run the per-point work of these steps over all positions instead, and only
// the selects themselves in one (larger) workgroup per leaf. Inputs with many
// leaves fill the chip with the per-leaf kernels: 500k points at cap 4096 take
// 1339 us with those, 1387 this way; 120k 490 and 426, 100k in one leaf 3598
// and 733. Where frames are small, or split at once into leaves that are, there
// are no big leaves after all: 1000 frames of 200 points 264 us with the per-leaf
// kernels and 455 this way, 250 of 1000 306 and 385 (60 of 4000, each in one leaf,
// 505 and 424); at cap 4096 50 frames of 5000 points 354 and 444, 20 of 10000 348
// and 390 (10 of 20000 436 and 401); at cap 2100 a 120k object 254 and 324, 20k
// 138 and 174 (at cap 4096 365 and 319, 262 and 197). A leaf holds an eighth of
// its parent and more, up to the cap where the density varies, so only low caps
// are judged by it. (Over-full leaves at the depth limit of smaller caps stay with
// the per-leaf kernels.)
constexpr uint32_t BIG_FRAME_MIN = 1024;   // smaller frames (on average): no big leaves
constexpr uint32_t BIG_CAP_LOW = 4096;     // up to this cap,
constexpr uint32_t BIG_SPLIT_MIN = 2400;   // an eighth of a frame or the cap, if not above this: none either
inline bool big_leaf_path(uint32_t n, uint32_t nf, int32_t leaf_cap) {
    const uint32_t cap = (uint32_t)leaf_cap, frame = n / nf;
    if (n <= SEL_LDS_MAX || cap <= SEL_LDS_MAX || frame <= BIG_FRAME_MIN) return false;
    if (frame > cap && cap <= BIG_CAP_LOW && (cap <= BIG_SPLIT_MIN || frame / 8u <= BIG_SPLIT_MIN)) return false;
    return n <= (1u << 18) || (n <= (1u << 20) && cap >= n / 16u);
}

// Queries per kNN work item of inputs with n1 P1 points. A wave takes an
// item's queries in turn, so few points make short items to fill the chip's
// waves, and many points long ones, which share the walk over the leaf's
// groups. Whole calls with 8 / 4 / 2 / 1 queries (and four waves per SIMD): 914
// points 131 / 120 / 115 / 112 us; 12.2k 180 / 161 / 157 / 164; 35.6k 309 / 272
// / 264 / 291; 52k 248 / 245 / 258 / 297; 96k 307 / 313 / 353 / 442. With five
// waves 52k take 222 / 217, 96k 268.4 / 268.7. Tiles of 16 need more LDS than
// six waves per SIMD have: 1.2M points 1009 us with 16 (five waves) and 941 with
// 8, 64 sweeps 3860 and 3697, with 4 1002 and 4028.
__host__ __device__ inline uint32_t knn_tile_queries(uint32_t n1) {
    return n1 <= 4096u ? 1u : n1 <= 20480u ? 2u : n1 <= 65536u ? 4u : (uint32_t)KNN_TQ;
}

// Queries per kNN item of a leaf in counter q of the plan (1: chunked, 2 .. the
// classes). A leaf of the first class has 128 candidates and more per query:
// few isolated points, whose far neighbours make a query test many groups. As
// items of several such queries they set the run of a small input; alone they
// spread over the chip: 200k points at caps 512 / 1024 232 / 301 us a call with
// whole items, 219 / 243 so. Above 2^18 points there is enough other work to
// fill in (1.2M 1016 and 1022 us, 400k at cap 4096 860 and 872).
__host__ __device__ inline uint32_t knn_leaf_tile(uint32_t q, uint32_t tq, uint32_t n) {
    return q == 2u && n <= (1u << 18) ? 1u : tq;
}

// Inputs whose halo kernel plans the kNN items as it goes, each workgroup (8
// leaves) by additions to six counters that all share, at some 10 ns each.
// The plan kernel, one workgroup of 1024 leaves a round, takes 8 us for few
// leaves and 16 for 1500. Thousands of workgroups would wait for the counters
// longer than that: the line is at some 8000 leaves of a surface, four to the
// leaf cap.
inline bool plan_in_halo(uint32_t n, int32_t leaf_cap) {
    return n <= PLAN_ONE_MAX_N && n / 2048u <= (uint32_t)leaf_cap;
}

// Keys per workgroup of a radix pass. Below some 100k keys a pass is the
// latency of one workgroup plus a few round trips of look-back, and few keys
// per workgroup are read, ranked and written sooner; above, the look-back's
// traffic (1 KB of status words per tile and round trip) weighs more. Whole
// calls with tiles of 512 / 1024 / 2048 keys: 10k points 135.9 / 136.9 / 140.5
// us, 20k 147.5 / 147.7 / 151.1, 80k 226 / 222.8 / 224.6; with 1024 / 2048, on a
// sweep and a torus: 30k 137.7 / 139.1 and 131.4 / 134.4, 60k 164.1 / 164.4 and
// 146.9 / 148.7, 90k 193.5 / 192.3 and 167.0 / 167.7, 114k 215.8 / 213.9 and 178.1
// / 178.6, 130k 223.9 / 220.7 and 185.3 / 185.9 (from 60k on the two differ by
// about what calls do); 900k 875 / 863. 4096 keys, staged in LDS, by 512 threads
// of 8 keys against 256 of 16 (the same LDS with twice the waves): 1.2M points
// 1051 and 1042 us, 6.2M 3990 and 3948.
constexpr uint32_t SORT_TILE_EDGES[] = {1u << 14, 7u << 14, 1u << 20};  // the largest n of each tile but the last
inline uint32_t sort_tile_for(uint32_t n) {
    uint32_t tile = 512u;
    for (const uint32_t edge : SORT_TILE_EDGES) tile <<= n > edge ? 1 : 0;
    return tile;
}

// Method parameters as the kernels use them.
struct Params {
    int32_t k;
    int32_t leaf_cap;
    double min_leaf_side;
    double beta;
    int32_t min_vox_count;
    double rho_percentile;
    double alpha;
    double sigma;
    double eps;
    double keep_ratio;
    int32_t knn_chunk;        // initial kNN candidate chunk length (performance only)
    double gamma;             // kernel exponent: (d^2 + eps)^(-gamma/2); 2 = Eq. 20
    double log_thr;           // NaN: top-lambda; else keep P2 points with ln F >= log_thr
    int32_t stages;           // enabled modules: 1 voxel filter, 2 density filter, 4 score
};

// First candidate chunk length of the kNN plan.
inline uint32_t plan_chunk0(const Params& prm) { return prm.knn_chunk > 0 ? (uint32_t)prm.knn_chunk : (uint32_t)KNN_CC0; }

// Parameters of the score fit (loss and gradient of a relaxed ln F threshold).
struct FitArgs {
    double alpha, sigma, gamma, tau, T, eps;
};

// Pointers into the caller's workspace for a batch of nf frames, n points in
// all (a plain call is the batch of one frame). Frames are contiguous runs of
// the input; after the sort (frame id most significant) frame f occupies the
// same positions [foff[f], foff[f+1]) in sorted order.
struct Plan {
    uint32_t n;
    int k;
    uint32_t nf;
    uint32_t sort_passes;     // SORT_PASSES + frame-id passes
    size_t bytes;
    // zero-initialised block
    char* zero_begin;
    size_t zero_bytes;
    Counters* ctr;
    FrameStat* fstat;         // [nf]
    uint32_t* sort_hist;      // [SORT_PASSES_MAX][256]
    uint32_t* sort_status;    // [sort_passes - SORT_SHORT_FIRST][sort_tiles][256]
    uint32_t* scan_status;    // [SCAN_SLOTS][scan_tiles]
    uint32_t* plan_status;    // [PLAN_COUNTERS][plan_tiles] (parallel kNN plan)
    uint32_t sort_tiles, scan_tiles, plan_tiles;
    uint32_t sort_tile;       // keys per workgroup of the radix passes (sort_tile_for)
    bool plan_halo;           // the halo kernel plans the kNN items (plan_in_halo)
    bool big_leaves;          // leaves of more than SEL_LDS_MAX points are ordinary here (big_leaf_path)
    uint8_t* deepf;           // [n] 1 at sorted positions inside deep level-10 cells; between the two
                              // deep-cell kernels, 2 marks the start of a cell to re-sort (zeroed block)
    // frames
    uint32_t* foff;           // [nf+1] frame offsets (checked copy of the caller's)
    uint32_t* fid;            // [n] frame of each point (original order; nf > 1 only)
    uint32_t* bbox_part;      // [ceil(n / 1024)][8] per-chunk box (chunks inside one frame)
    FrameConst* fc;           // [nf]
    uint32_t* keep_ex;        // [n+1] exclusive count of kept points (original order; nf > 1)
    // sort (sorted order = s)
    uint64_t* keys_a;         // sorted keys end here
    uint64_t* keys_b;
    uint32_t* idx_a;          // sorted original indices end here
    uint32_t* idx_b;
    uint64_t* keys_src;       // where the keys are written before the sort (a or b by pass parity)
    uint32_t* idx_src;
    float4* pos4;             // [n] sorted x, y, z, original index bits
    uint32_t* leaf_of;        // [n] sorted
    uint32_t* occ;            // [n] sorted
    uint8_t* p1;              // [n] sorted
    uint8_t* bflag;           // [n] sorted: a leaf starts here
    uint32_t* p1pos;          // [n+1] exclusive scan of p1
    // leaves (at most n)
    uint32_t* leaf_begin;     // [n+1]
    uint32_t* leaf_level;     // [n]
    float* leaf_h;            // [n]
    uint32_t* leaf_nr;        // [n] number of candidate ranges
    uint2* leaf_ranges;       // [n][HALO] compacted candidate ranges
    uint2* leaf_own;          // [n] the candidate range holding the leaf's own P1 points
    uint32_t* leaf_ncand;     // [n]
    uint32_t* leaf_nch;       // [n] candidate chunks
    uint32_t* leaf_cc;        // [n] chunk length
    uint32_t* leaf_plist;     // [n] first partial list of the leaf
    uint32_t* leaf_item;      // [n] queue index of the leaf's first kNN item
    double* leaf_rho_med;     // [n]
    uint64_t* vox_keys;       // [2n] global hash fallback
    uint32_t* vox_cnt;        // [2n]
    // compacted P1 (query/candidate index q)
    float4* cand4;            // [n]
    uint32_t* cand_leaf;      // [n]
    uint32_t* nbr;            // [n][k] P1 positions of the neighbours (sorted by d2, then original index)
    uint32_t* inv_p1;         // [n] by original index: the P1 position of a P1 point
    float* nbr_d2;            // [n][k]
    float* r2k;               // [n] (written by the density kernel from krec)
    uint4* krec;              // [n] k-th neighbour's P1 position (none: 0xFFFFFFFF), fp32 bits of the (k-1)-th and k-th d2
    uint2* outrec;            // [n] by original index: fp32 score bits, stage (large inputs' outputs)
    float* tau_c;             // [n] per-query upper bound of r^2_K (-1: none)
    GroupBox* gbox;           // [ceil(n / KNN_GRP)] boxes of aligned groups of the P1 order
    double* rho_c;            // [n]
    double* r64_c;            // [n]
    double2* afac_c;          // [n] (rho_i / (rho_med^2 + eps))^(alpha/2), 1 / (2 (sigma r_K,i)^2)
    uint8_t* p2;              // [n]
    uint8_t* stage_c;         // [n] 1 density-removed, 2 score-removed, 3 kept
    double* score_c;          // [n]
    double* gpow_p;           // [n] P1 order: rho^(alpha/2)
    // kNN work
    KnnItem* items;           // [items_max]
    uint32_t items_max;
    uint64_t* plist;          // [plist_max][k] partial top-k keys
    uint32_t plist_max;
    // big leaves: short-lived arrays inside plist (before the kNN, then after its merge)
    uint32_t* leaf_box;       // [6n] ordered-uint max of ~min and of max, per leaf
    unsigned long long* leaf_theta;  // [n] top-lambda cut: key, and the largest index kept at that key
    uint32_t* leaf_icut;      // [n]
    float* leaf_r2cut;        // [n] percentile cut
};

// ------------------------------------------------------------------ helpers

// Whether the halo kernel's plan holds: it was made and fits the workspace.
__device__ __forceinline__ bool halo_plan_stands(const Plan& P) {
    if (!P.plan_halo) return false;
    unsigned long long items = 0;
#pragma unroll
    for (int i = 1; i < PLAN_COUNTERS; ++i) items += P.ctr->plan_q[i];
    return P.ctr->plan_q[0] <= P.plist_max && items <= P.items_max;
}

__device__ __forceinline__ uint32_t f32_ordered(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float f32_from_ordered(uint32_t o) {
    uint32_t u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    return __uint_as_float(u);
}

// Look-back status words carry their whole payload (flag + count), so relaxed
// device-scope atomics suffice: no other data is published through them.
constexpr int LB_WINDOW = 4;                  // predecessors fetched per look-back round trip

__device__ __forceinline__ uint32_t ld_relaxed_agent(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed_agent(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-level inclusive scan and sum (wave64, every lane active), by DPP: row
// shifts inside the rows of 16 lanes, then the rows' last lanes broadcast to
// the rows after them. A step takes the VALU's latency where a shuffle through
// the LDS unit takes some hundred cycles, and the scans of a workgroup wait for
// six of them in a row.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15 to rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31 to rows 2, 3
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v), 63);
}

// Inclusive running maximum (every lane active).
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v) {
    auto step = [&](uint32_t o) { v = o > v ? o : v; };
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));
    return v;
}

// Any associative, commutative f over the wave (every lane active) the same
// way, 32- or 64-bit values, result in every lane; f(ident, v) = v.
template <int CTRL, int ROWS, class T>
__device__ __forceinline__ T dpp_from(T v, T ident) {
    uint32_t a[sizeof(T) / 4], b[sizeof(T) / 4];
    __builtin_memcpy(a, &v, sizeof(T));
    __builtin_memcpy(b, &ident, sizeof(T));
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i)
        a[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)b[i], (int)a[i], CTRL, ROWS, 0xF, false);
    __builtin_memcpy(&v, a, sizeof(T));
    return v;
}
template <class T, class F>
__device__ __forceinline__ T wave_reduce(T v, T ident, F f) {
    v = f(v, dpp_from<0x111, 0xF>(v, ident));
    v = f(v, dpp_from<0x112, 0xF>(v, ident));
    v = f(v, dpp_from<0x114, 0xF>(v, ident));
    v = f(v, dpp_from<0x118, 0xF>(v, ident));
    v = f(v, dpp_from<0x142, 0xA>(v, ident));
    v = f(v, dpp_from<0x143, 0xC>(v, ident));
    uint32_t a[sizeof(T) / 4];
    __builtin_memcpy(a, &v, sizeof(T));
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) a[i] = (uint32_t)__builtin_amdgcn_readlane((int)a[i], 63);
    __builtin_memcpy(&v, a, sizeof(T));
    return v;
}
__device__ __forceinline__ float wave_fmin(float v) {
    return wave_reduce(v, INFINITY, [](float a, float b) { return fminf(a, b); });
}
__device__ __forceinline__ float wave_fmax(float v) {
    return wave_reduce(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
    return wave_reduce(v, 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
template <class T>
__device__ __forceinline__ T wave_umin(T v) {
    return wave_reduce(v, (T)~(T)0, [](T a, T b) { return a < b ? a : b; });
}
template <class T>
__device__ __forceinline__ T wave_and(T v) {
    return wave_reduce(v, (T)~(T)0, [](T a, T b) { return (T)(a & b); });
}
template <class T>
__device__ __forceinline__ T wave_or(T v) {
    return wave_reduce(v, (T)0, [](T a, T b) { return (T)(a | b); });
}

// The lanes of `m` whose digit (8 bits) is this lane's. Per bit one ballot and
// one three-input logic operation on each half of the mask.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t m) {
    uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint32_t s = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);  // all ones where the bit is set
        const uint64_t bb = __builtin_amdgcn_ballot_w64(s != 0u);
        lo &= ~((uint32_t)bb ^ s);
        hi &= ~((uint32_t)(bb >> 32) ^ s);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Workgroups are dealt to the chip's eight XCDs in turn (workgroup b runs on
// XCD b % 8). xcd_part gives the workgroups of one XCD one contiguous eighth
// of [0, n) to stride through: a kernel over sorted positions that gathers
// from, or scatters to, input order then touches only the lines of its own
// part's few frames, which stay in its XCD's L2 instead of being fetched by
// all eight. The grid must hold a whole number of workgroups per XCD
// (xcd_grid).
constexpr unsigned N_XCD = 8;
struct XcdPart {
    uint32_t first, end, step;
};
__device__ __forceinline__ XcdPart xcd_part(uint32_t n) {
    const uint32_t per = (n + N_XCD - 1u) / N_XCD;
    const uint32_t lo = min(n, (blockIdx.x % N_XCD) * per);
    return XcdPart{lo + (blockIdx.x / N_XCD) * blockDim.x + threadIdx.x, min(n, lo + per),
                   (gridDim.x / N_XCD) * blockDim.x};
}
inline unsigned xcd_grid(unsigned blocks) { return (blocks + N_XCD - 1u) / N_XCD * N_XCD; }

// Block exclusive scan of one value per thread (blockDim multiple of 64, <= 1024).
// `smem` needs blockDim/64 + 1 words. Returns the exclusive prefix; *total gets
// the block sum. Contains __syncthreads.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* smem, uint32_t* total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == 63u) smem[wave] = inc;
    __syncthreads();
    // every wave scans the wave totals
    const uint32_t t = wave_incl_scan(lane < nw ? smem[lane] : 0u);
    const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)t, (int)wave - 1) : 0u;
    *total = (uint32_t)__builtin_amdgcn_readlane((int)t, 63);
    __syncthreads();
    return before + inc - v;
}

// 3D bit interleave (x in the lowest bit), magic-number spreading.
__device__ __forceinline__ uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x1F00000000FFFFull;
    x = (x | (x << 16)) & 0x1F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}
__device__ __forceinline__ uint32_t compact3(uint64_t x) {
    x &= 0x1249249249249249ull;
    x = (x ^ (x >> 2)) & 0x10C30C30C30C30C3ull;
    x = (x ^ (x >> 4)) & 0x100F00F00F00F00Full;
    x = (x ^ (x >> 8)) & 0x1F0000FF0000FFull;
    x = (x ^ (x >> 16)) & 0x1F00000000FFFFull;
    x = (x ^ (x >> 32)) & 0x1FFFFFull;
    return (uint32_t)x;
}
__device__ __forceinline__ uint64_t morton3(uint32_t x, uint32_t y, uint32_t z) {
    return spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
}

// Frame holding position j of a batch: frames are contiguous runs both of
// the input and of the sorted order (the frame id is the most significant
// sort digit), so the frame is the last f with foff[f] <= j (empty frames
// share their end with the next start). foff is tiny and stays in cache.
__device__ __forceinline__ uint32_t frame_of(const uint32_t* foff, uint32_t nf, uint32_t j) {
    uint32_t lo = 0, hi = nf;
    while (hi - lo > 1u) {
        const uint32_t mid = (lo + hi) >> 1;
        if (foff[mid] <= j) lo = mid;
        else hi = mid;
    }
    return lo;
}

}  // namespace gdn
