// Internal definitions shared by the gfx950 kernels and the host ABI layer.
// Nothing here is part of the public C ABI (include/xg.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xg.h"

namespace xg {

constexpr int kWave = 64;

// Workspace header words (first 256 bytes of the workspace).
struct WsHeader {
    int32_t status;        // XG_OK / XG_ECAPACITY
    int32_t n_pairs;       // pairs requested by the scan (may exceed capacity)
    int32_t item_sel;      // which item key/value buffer holds the depth-sorted items
    uint32_t depth_min;    // min float32 depth bits over kept (view, Gaussian)
    uint32_t depth_max;    // max float32 depth bits
    int32_t queue_fwd;     // persistent forward tile queue head
    int32_t queue_bwd;     // persistent backward tile queue head
    int32_t done_fwd;      // persistent forward workgroups finished
    int32_t done_bwd;      // persistent backward workgroups finished
    int32_t item_passes;   // item-sort passes that moved data
    int32_t pad[54];
};
static_assert(sizeof(WsHeader) == 256, "header is one 256-byte block");

// Render record of one (view, Gaussian), written by the preprocess and read
// by every tile that lists the Gaussian: 64 bytes, one cache line, so a
// staged list entry is a single aligned gather.
//   a: (u_x - floor(u_x), u_y - floor(u_y), qa, qb)
//   b: (qc, -log2(opacity), intensity, float bits of depth)
//   c: (floor(u_x), floor(u_y), x_lo | x_hi << 16, y_lo | y_hi << 16), with
//      kRecPlain in the x word (bounds are below 2^15)
//   d: unused
// (qa, qb, qc) factor the inverse 2-D covariance scaled by k = log2(e)/2:
//   k * d^T Sigma''^-1 d = (qa dx + qb dy)^2 + (qc dy)^2
// so that exp(-d^T Sigma''^-1 d / 2) = exp2(-(that)), and the opacity times
// it, the a of Eq. 10, is exp2(-(that - log2 opacity)): the blend kernels
// evaluate one exponential and no product.
struct alignas(64) Record {
    float4 a;
    float4 b;
    int4 c;
    float4 d;
};
static_assert(sizeof(Record) == 64, "one cache line per record");

// The blend needs neither the rectangle test nor the alpha clamp for this
// (view, Gaussian): no pixel outside the rectangle reaches alpha_min, and no
// pixel alpha_max, with a margin far above float rounding.
constexpr int kRecPlain = 1 << 15;
__host__ __device__ __forceinline__ int rec_x_lo(int xword) { return xword & 0x7fff; }

// Number of XCDs workgroups are dealt to round-robin (MI355X: 8).  Used to
// give each XCD a contiguous range of tiles, so the records its L2 caches
// are shared by the tiles it renders.
constexpr int kXcds = 8;

// Tile of workgroup b in a grid of n tiles such that XCD b % kXcds takes a
// contiguous block of tiles.  A bijection on [0, n) for any n.
__device__ __forceinline__ int xcd_tile(int b, int n) {
    const int x = b % kXcds, i = b / kXcds;
    const int q = n / kXcds, r = n % kXcds;
    return x * q + min(x, r) + i;
}

// Tile of workgroup b of a one-workgroup-per-tile launch over n tiles: XCD
// b % kXcds walks its share of the tiles in the order the list builder left
// in `order` (longest list first, so the longest tiles start early and none
// is left to run alone at the end of the launch).  An entry outside [0, n)
// (a workspace whose lists were never built) falls back to the natural
// order of contiguous blocks instead of reading out of bounds.
__device__ __forceinline__ int ordered_tile(const int32_t *order, int b, int n) {
    const int i = xcd_tile(b, n);
    const int t = order[i];
    return (unsigned)t < (unsigned)n ? t : i;
}

// How the items of a frame are sorted: by the radix passes over all views,
// or each view by one workgroup, with or without the counting of the tile
// lists in the same launch.
enum class ViewSort : int32_t { kNone, kItems, kLists };
constexpr int kViewSortThreads = 1024;
constexpr int kViewSortItems = 8;                                   // most items per thread
constexpr int kViewSortMax = kViewSortThreads * kViewSortItems;
constexpr int kViewListsItems = 4;                                  // the same where it counts the lists
constexpr int kViewSortParts = 64;                                  // most list partitions of a view
constexpr int64_t kViewListsMax = 65536;                            // most items of a frame counted in the launch
// LDS words of the one-workgroup sort: keys, 16-bit item numbers, per
// wavefront a digit histogram and a table of 64-bit lane masks
constexpr int view_sort_words(int items) {
    return kViewSortThreads * items * 3 / 2 + kViewSortThreads / kWave * 256 * 3;
}

// Device view of a workspace, resolved on the host from the layout.
struct Ws {
    WsHeader *hdr;
    Record *rec;
    uint32_t *counts;      // tiles per (view, Gaussian), in (view, Gaussian) order
    uint32_t *icounts;     // the same counts in depth-sorted item order
    uint32_t *offsets;     // exclusive scan of icounts
    uint32_t *scan_tmp;
    uint32_t *depth_part;  // (min, max) depth bits of each preprocess workgroup's kept items: kept until the
                           // next preprocess, every list build reads them
    uint32_t *ikeys[2];    // item sort keys (float32 depth bits; 0xffffffff when culled)
    uint64_t *ivals[2];    // item sort values: (view, Gaussian) index | tile rectangle << 32
    uint32_t *ptile[2];    // pair sort keys (global tile id)
    uint32_t *pval[2];     // pair sort values (Gaussian index)
    uint32_t *ghist;       // radix sort: digit histograms [kMaxPasses][kRadix], one 128-byte line each
    uint32_t *vhist;       // item sort (within each view): digit totals [view][kMaxPasses][kRadix]
    uint32_t *vctr;        // item sort: partition counters [view][kMaxPasses], one 128-byte line each
    bool sort_fold;        // item sort: its histogram launch folds the depth partials (no clearing launch)
    uint32_t *bin_cnt;     // tile lists by counting: [view][partition][local tile] pair counts,
                           // then their exclusive scan down each column
    uint32_t *bin_csum;    // tile lists by counting: pairs of every 64 tiles of a view
    uint32_t *bin_ptot;    // tile lists by counting: pairs of each [view][partition]
    uint32_t *bin_pstart;  // tile lists by counting: first pair slot of each [view][partition]
    uint32_t *pctr;        // radix sort: partition counters [kMaxPasses]
    uint64_t *lookback[2]; // radix sort: per (partition, digit) aggregate / prefix words
    uint32_t *ranges;
    void *entry_mask;      // per list entry: the 8 x 8 sub-blocks the blending kernels visit
                           // (written by the forward, read by the backward; 1 byte, 2 for 32 x 32 tiles)
    float *grad2d;
    float *ssim;           // loss: three per-pixel SSIM partial-derivative maps, then one
                           // loss share per 48 x 8 loss strip
    int32_t *tile_order;   // persistent queue: tiles in work order
    int32_t *xcd_order;    // each XCD's contiguous block of tiles, longest list first
    int32_t *blend_order;  // one-workgroup-per-tile launches: each XCD's tiles, longest list first
    int64_t cap;
    int64_t n_items;       // n_views * n
    int64_t total_tiles;
    int64_t total_pixels;
    int32_t n;
    int32_t n_views;
    int32_t tile_bits;     // bits of the largest global tile id
    int32_t item_blocks;   // radix-sort blocks over the items
    int32_t item_per;      // their items per thread (2, 4 or 8)
    int32_t pair_blocks;   // radix-sort blocks over the pair capacity
    int32_t pair_passes;   // 8-bit passes over the tile id
    int32_t pair_sel;      // buffer holding the tile-sorted pairs (pair_passes & 1)
    // Packed pairs: when the tile id and the Gaussian index fit one word,
    // ptile holds tile << pair_gbits | index and pval is not used
    // (pair_gbits = 0: two arrays).  The blending kernels read the index as
    // pair_vals[p] & pair_gmask.
    int32_t pair_gbits;
    uint32_t pair_gmask;
    const uint32_t *pair_vals;
    // Tile lists by counting (bin_tiles > 0): the row length of bin_cnt (the
    // most tiles of any view), and per view the partitions of bin_items items.
    // bin_tiles = 0: emission and the radix sort of the pairs by tile.
    int32_t bin_tiles;
    int32_t bin_bands;     // bands of at most 1024 tiles (whole rows) of the view with the most
    int32_t bin_ppv;
    int32_t bin_items;
    ViewSort view_sort;
};

// Scalar constants of one rendering.
struct Params {
    float lowpass, alpha_min, alpha_max, t_min, near_z;
    float kappa;           // float32(-2 ln alpha_min): rectangle radius^2
    int32_t tile;
    int32_t lds_batch;
};

constexpr float kLog2eHalf = 0.72134752044448170368f;   // log2(e) / 2
constexpr float kInvLog2eHalf = 1.38629436111989061883f; // 2 ln 2

// Preprocess workgroups: 256 threads, one per (view, Gaussian).
constexpr int kPreThreads = 256;

// The tile rectangle of a (view, Gaussian) item packed in 32 bits and
// carried through the item sort, so the pair emission reads no record:
// first tile column and row (10 bits each), extra columns and rows (5 bits
// each), bit 30 set when the rectangle fits (else the record is read).
__host__ __device__ __forceinline__ uint32_t pack_tile_rect(int tx0, int tx1, int ty0, int ty1) {
    const int dx = tx1 - tx0, dy = ty1 - ty0;
    if (tx0 < 0 || ty0 < 0 || tx0 >= 1024 || ty0 >= 1024 || dx < 0 || dy < 0 || dx >= 32 || dy >= 32)
        return 0u;
    return (1u << 30) | (uint32_t)tx0 | ((uint32_t)ty0 << 10) | ((uint32_t)dx << 20) | ((uint32_t)dy << 25);
}
struct TileRect {
    int tx0, tx1, ty0, ty1;
};
__device__ __forceinline__ bool unpack_tile_rect(uint32_t r, TileRect &t) {
    if (!(r & (1u << 30))) return false;
    t.tx0 = (int)(r & 1023u);
    t.ty0 = (int)((r >> 10) & 1023u);
    t.tx1 = t.tx0 + (int)((r >> 20) & 31u);
    t.ty1 = t.ty0 + (int)((r >> 25) & 31u);
    return true;
}

// Tile rectangle (first/last tile column and row, view-local) of a sorted
// item from its sort value: the packed rectangle, else the record.
__device__ __forceinline__ TileRect item_tile_rect(const Ws &ws, uint64_t val, int tile) {
    TileRect tr;
    if (!unpack_tile_rect((uint32_t)(val >> 32), tr)) {
        const int4 rc = ws.rec[(uint32_t)val].c;
        tr.tx0 = rec_x_lo(rc.z) / tile;
        tr.tx1 = (rc.z >> 16) / tile;
        tr.ty0 = (rc.w & 0xffff) / tile;
        tr.ty1 = (rc.w >> 16) / tile;
    }
    return tr;
}

// Lanes of the wavefront whose BITS-bit key equals this lane's (one ballot
// per key bit), restricted to `valid` lanes.
// Per bit: the bit spread over a word, one compare (a wavefront-uniform mask)
// and, per half of the mask, one three-operand instruction.
template <int BITS>
__device__ __forceinline__ uint64_t match_peers(uint32_t d, bool valid) {
    const uint64_t v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const int bit = (int)(d << (31 - b)) >> 31;   // all ones when the bit is set
        const uint64_t bal = __ballot(bit < 0);
        lo &= ~((uint32_t)bal ^ (uint32_t)bit);
        hi &= ~((uint32_t)(bal >> 32) ^ (uint32_t)bit);
    }
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Tile lists by counting: most items per partition (all of one view), pairs
// per LDS window of the ranking kernel, and which frames take this path (the
// others use emission and the radix sort of the pairs; the rule and its
// figures are where the frame's plan is made): no view with more than
// kBinMaxTilesX tiles in a row, and either none with more than kBinMaxTiles
// tiles, or none with more than kBinMostTiles and at most kBinMostGroups
// ranking workgroups.
constexpr int kBinItems = 2048;
constexpr int kBinItemsMin = 256;
constexpr int kBinResident = 512;   // ranking workgroups the device holds at once (two per CU)
constexpr int kBinWindow = 4096;
constexpr int kBinMaxTiles = 4096;
constexpr int kBinMaxTilesX = 1024;             // a band of the ranking kernel holds a row
constexpr int kBinMostTiles = 65536;
constexpr int kBinMostGroups = 4096;
constexpr int kColTiles = 64;                   // tiles of a workgroup of the column scans

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanBlock = kScanThreads * kScanItems;   // 2048 elements

// Radix-sort partitions (keys per workgroup = threads x keys per thread);
// larger partitions shorten the look-back chains, smaller ones the chain of
// phases inside a workgroup.  The items' hold 8192, 4096 or 2048: the smallest
// that make no more partitions than the device has CUs (a workgroup of 8192 fills a
// CU's LDS) and no longer chains in a view than 128 of 4096 or 64 of 2048.
// Forward passes with 8192 / 4096 / 2048: one view of 43k items 108 / 95 / 89 us;
// one of 400k 147.6 / 143.9 / 149.7, of 1M (245 partitions of 4096) 185 / 188 /
// 208; 8 views of 50k 155 / 147 / 145; 4 of 200k 212 / 207 / 217; 8 of 200k (392
// of 4096), a training step, 452 / 472 / 482.  1024: 43k 88.5, 10k 82.7
// against 83.7, but 8 views of 50k 155.
constexpr int kItemSortThreads = 1024;
constexpr int kItemSortItems = 8;        // most items per thread
constexpr int kItemSortMost = 256;       // most partitions of the smaller sizes
constexpr int kItemSortChain = 32;       // and of a view, times the items per thread
constexpr int kPairSortThreads = 1024, kPairSortItems = 16;   // 16384 pairs
constexpr int kPairSortBlock = kPairSortThreads * kPairSortItems;
// packed pairs move 4-byte keys only, so a partition holds more of them
constexpr int kPackedSortThreads = 1024, kPackedSortItems = 16;
constexpr int kPackedSortBlock = kPackedSortThreads * kPackedSortItems;
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;
constexpr int kMaxPasses = 4;                            // 32 depth bits, 8 at a time
constexpr int kGhStride = 32;   // words between histogram bins (spreads their atomics over channels)
constexpr int kSortCtlWords = (kMaxPasses * kRadix + kMaxPasses) * kGhStride;

// Preprocess workgroups (depth partials) up to which the item sort's
// histogram launch folds them in every workgroup, instead of a clearing
// launch that folds a share in each: 8192 pairs are 8 loads a thread; at
// 62 500 (16 M items) the launch is the cheaper one.
constexpr int64_t kFoldParts = 8192;

// The item sort's words that are zero before its histogram launch where that
// launch folds the depth partials (ws.sort_fold): the digit totals of every
// view and the partition counters.  The preprocess zeroes them, and the launch
// after the sort again, so that a second list build of the same preprocess
// finds them zero too.
__device__ __forceinline__ int64_t item_sort_zeros(const Ws &ws) {
    return (int64_t)ws.n_views * kMaxPasses * (kRadix + 1);
}
__device__ __forceinline__ void zero_item_sort(const Ws &ws, int64_t i) {
    const int64_t bins = (int64_t)ws.n_views * kMaxPasses * kRadix;
    if (i < bins)
        ws.vhist[i] = 0;
    else
        ws.vctr[(i - bins) * kGhStride] = 0;
}

// ---- launchers (one translation unit per stage) --------------------------
hipError_t launch_preprocess(const Ws &ws, const xg_gaussians &g, const xg_camera *cams,
                             const Params &p, bool colours, hipStream_t s);
hipError_t launch_scan(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp,
                       int32_t *total, int32_t *status, int64_t cap, hipStream_t s);
hipError_t launch_sort_items(const Ws &ws, const xg_camera *cams, const Params &p, hipStream_t s);
hipError_t launch_emit(const Ws &ws, const xg_camera *cams, const Params &p, hipStream_t s);
hipError_t launch_sort_pairs(const Ws &ws, hipStream_t s);
hipError_t launch_ranges(const Ws &ws, bool cleared, hipStream_t s);  // cleared: by the pair sort
hipError_t launch_tile_order(const Ws &ws, hipStream_t s);
hipError_t launch_xcd_order(const Ws &ws, hipStream_t s);
hipError_t launch_bin_lists(const Ws &ws, const xg_camera *cams, const Params &p, hipStream_t s);
hipError_t launch_pair_keys(const Ws &ws, const xg_camera *cams, uint64_t *keys, uint32_t *vals,
                            int64_t cap, hipStream_t s);
// Per-pixel stored transmittances of the stored-list variant: count[tile][px]
// contributors, then t[tile][slot][px] = T before contributor `slot` (the
// first `slots` contributors of each pixel; px = thread index in the tile).
struct TStore {
    float *t;
    int32_t *count;
    int slots;
};

// Optional L1 epilogue of the forward blend: dl[o] = scale * sign(image[o] -
// target[o]) (sign(0) = 0), written with the image (dl null: none).
struct L1Fuse {
    const float *target;
    float *dl;
    float scale;
};
hipError_t launch_render_fwd(const Ws &ws, const xg_camera *cams, const Params &p,
                             float *image, float *final_t, int32_t *n_contrib,
                             int persistent, const TStore &ts, const L1Fuse &l1, hipStream_t s);
hipError_t launch_render_bwd(const Ws &ws, const xg_camera *cams, const Params &p,
                             const float *dl_dimage, const float *final_t,
                             const int32_t *n_contrib, int persistent, const TStore &ts,
                             hipStream_t s);
hipError_t launch_render_counts(const Ws &ws, const xg_camera *cams, const Params &p,
                                int32_t *counts, hipStream_t s);
hipError_t launch_preprocess_bwd(const Ws &ws, const xg_gaussians &g, const xg_camera *cams, bool accumulate,
                                 const Params &p, const xg_grads &gr, hipStream_t s);
hipError_t launch_sh_color(const Ws &ws, const xg_camera *cams_dev, const float *means, const float *sh,
                           int degree, hipStream_t s);
hipError_t launch_render_fwd_rgb(const Ws &ws, const xg_camera *cams, const Params &p, float *image,
                                 float *final_t, int32_t *n_contrib, hipStream_t s);
hipError_t launch_acui_grid(const double size[3], const int32_t grid[3], double d, const int32_t k[3],
                            int64_t count, float *means, hipStream_t s);
int64_t loss_tiles(const xg_camera *cams_host, int n_views);
// this device's address of the static scratch array of xg_loss_grad_static
// (resolved on the first call on each device)
hipError_t static_scratch(float **out);
hipError_t launch_loss_grad(const Ws &ws, const xg_camera *cams_dev, int64_t tiles,
                            const float *image, const float *target, float gamma, float *dl,
                            float *loss, hipStream_t s);
hipError_t launch_l1_grad(const float *image, const float *target, float *out, int64_t n,
                          float scale, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s);
hipError_t launch_rirf_fwd(const float *features, const float *weights, int64_t n, int nf,
                           float *intensity, hipStream_t s);
hipError_t launch_rirf_bwd(const float *features, const float *weights, int64_t n, int nf,
                           const float *dl_di, float *grad_f, hipStream_t s);
hipError_t launch_adam(const xg_params &p, const xg_grads &g, float *m, float *v, int32_t *step,
                       const xg_adam &c, float *scales, float *opacity, float *intensity,
                       const int32_t *gate, hipStream_t s);

// ---- device helpers ------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Wave-wide inclusive prefix sum of a uint32 (64 lanes, all active): within
// each row of 16 by DPP shifts, then the rows' last lanes broadcast onward
// (six VALU instructions; as LDS permutes each step costs an LDS round trip).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
#define XG_SCAN_STEP(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false)
    XG_SCAN_STEP(0x111, 0xf);   // row_shr:1
    XG_SCAN_STEP(0x112, 0xf);   // row_shr:2
    XG_SCAN_STEP(0x114, 0xf);   // row_shr:4
    XG_SCAN_STEP(0x118, 0xf);   // row_shr:8
    XG_SCAN_STEP(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
    XG_SCAN_STEP(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef XG_SCAN_STEP
    return v;
}

// Block-wide exclusive prefix sums of Q values at once, over blockDim.x
// threads (multiple of 64, at most 1024).  `lds` must hold Q rows of
// kScanLds words, 16-byte aligned.  v[q] becomes the exclusive prefix,
// total[q] the block sum.  Two barriers: every thread adds up the wavefront
// totals itself.
constexpr int kScanLds = 1024 / kWave;
template <int Q>
__device__ __forceinline__ void block_excl_scans(uint32_t (&v)[Q], uint32_t *lds, uint32_t (&total)[Q]) {
    const int w = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    uint32_t inc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        inc[q] = wave_incl_scan(v[q]);
        if (lane_id() == kWave - 1) lds[q * kScanLds + w] = inc[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        uint32_t before = 0, sum = 0;
        const uint4 *rows = reinterpret_cast<const uint4 *>(lds + q * kScanLds);
#pragma unroll
        for (int k4 = 0; k4 < kScanLds / 4; ++k4) {
            const uint4 r = rows[k4];   // words past the block's wavefronts: never written, not added
            const uint32_t x[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                before += 4 * k4 + k < w ? x[k] : 0u;
                sum += 4 * k4 + k < nw ? x[k] : 0u;
            }
        }
        v[q] = before + inc[q] - v[q];
        total[q] = sum;
    }
    __syncthreads();
}

// The same for one value; `lds` holds kScanLds words.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *lds, uint32_t *total) {
    uint32_t a[1] = {v}, t[1];
    block_excl_scans<1>(a, lds, t);
    *total = t[0];
    return a[0];
}

// Work-order buckets of list lengths: eight per octave, longest first.
constexpr int kOrderBuckets = 256;
__device__ __forceinline__ int order_bucket(const Ws &ws, int64_t t) {
    const uint32_t len = ws.ranges[2 * t + 1] - ws.ranges[2 * t];
    const int l = (int)(8.0f * __log2f((float)len + 1.0f));
    return kOrderBuckets - 1 - min(l, kOrderBuckets - 1);
}

// How the blend launches deal the tiles to the XCDs.  Every XCD takes the
// same number of tiles (workgroup b runs on XCD b % kXcds), as `rounds`
// chunks of `chunk` consecutive tiles, chunk k of the frame going to XCD
// k % kXcds, and what is left over in kXcds contiguous pieces.  rounds = 0
// is one contiguous block per XCD.  A bijection for any chunk > 0.
struct TileDeal {
    int chunk, rounds, base, q, rem;
    __host__ __device__ __forceinline__ TileDeal(int n, int c, bool contiguous)
        : chunk(c), rounds(contiguous ? 0 : n / (kXcds * c)) {
        base = rounds * kXcds * chunk;
        q = (n - base) / kXcds;
        rem = (n - base) % kXcds;
    }
    // tiles of XCD x
    __host__ __device__ __forceinline__ int tiles(int x) const { return rounds * chunk + q + (x < rem ? 1 : 0); }
    // tile j (from 0) of XCD x
    __host__ __device__ __forceinline__ int tile(int x, int j) const {
        const int dealt = rounds * chunk;
        if (j < dealt) return (j / chunk * kXcds + x) * chunk + j % chunk;
        return base + x * q + (x < rem ? x : rem) + (j - dealt);
    }
};

// The chunkings that xcd_order_block chooses from: step 0 is one contiguous
// block per XCD, step m chunks of about n / (8 * 2^m) tiles, whole groups of g.
constexpr int kDealSteps = 7;
constexpr int kDealParts = 8;                        // threads per (step, XCD) sum
constexpr float kDealSlack = 1.1f;
__host__ __device__ __forceinline__ int deal_chunk(int n, int g, int step) {
    const int c = n / (kXcds << step) / g * g;
    return c > g ? c : g;
}

// List entries of XCD x under deal d: the share of thread `part` of
// kDealParts.  Whole groups of the dealt chunks (`group`: entries of every g
// consecutive tiles); the left-over pieces start and end inside groups, whose
// entries are taken as even over their tiles, in sixteenths.  Every workgroup
// makes the choice for itself and all have to make the same one, or tiles are
// rendered twice and others never: integers, whose sum no order of adding
// changes (a frame has fewer than 2^31 entries).
__host__ __device__ __forceinline__ uint32_t deal_share(const uint32_t *group, int g, const TileDeal &d, int x,
                                                        int part) {
    const int tiles = d.tiles(x);
    uint32_t sum = 0;
    for (int j = part * g; j < tiles; j += kDealParts * g) {
        const uint32_t len = group[d.tile(x, j) / g];
        sum += tiles - j >= g ? len : (uint32_t)((uint64_t)len * (uint32_t)((tiles - j) / (g / 16)) >> 4);
    }
    return sum;
}

// The largest XCD's load over the mean (1: even).
__host__ __device__ __forceinline__ float deal_excess(uint32_t largest, uint32_t total) {
    return (float)largest * (kXcds / (float)(total > 0 ? total : 1));
}

// The coarsest step within kDealSlack of an even split, else the most even one.
__host__ __device__ __forceinline__ int deal_choice(const float (&excess)[kDealSteps]) {
    int best = 0;
    float least = excess[0];
#pragma unroll
    for (int step = 1; step < kDealSteps; ++step) {
        if (least > kDealSlack && excess[step] < least) {
            best = step;
            least = excess[step];
        }
    }
    return best;
}

// Writes the cnt tiles tile_of(j) longest list first to out, and to also
// unless null (buckets of an eighth of an octave; the order inside a bucket
// is arbitrary).  The
// workgroup has at least kOrderBuckets threads; hist: kOrderBuckets words
// of LDS; scan_lds: kScanLds words.  Contains barriers.
template <class TileOf>
__device__ __forceinline__ void order_tiles(const Ws &ws, int cnt, TileOf tile_of, int32_t *out, int32_t *also,
                                            uint32_t *hist, uint32_t *scan_lds) {
    for (int b = threadIdx.x; b < kOrderBuckets; b += blockDim.x) hist[b] = 0;
    __syncthreads();
    for (int j = (int)threadIdx.x; j < cnt; j += blockDim.x) atomicAdd(&hist[order_bucket(ws, tile_of(j))], 1u);
    __syncthreads();
    const uint32_t v = threadIdx.x < kOrderBuckets ? hist[threadIdx.x] : 0u;
    uint32_t tot;
    const uint32_t ex = block_excl_scan(v, scan_lds, &tot);
    if (threadIdx.x < kOrderBuckets) hist[threadIdx.x] = ex;
    __syncthreads();
    for (int j = (int)threadIdx.x; j < cnt; j += blockDim.x) {
        const int t = tile_of(j);
        const uint32_t pos = atomicAdd(&hist[order_bucket(ws, t)], 1u);
        out[pos] = (int32_t)t;
        if (also) also[pos] = (int32_t)t;
    }
    __syncthreads();
}

// The blend launches' tile orders, one XCD's part.  xcd_order: the
// contiguous block of tiles of XCD x (xcd_tile), longest list first.
// blend_order, which the launches read: the same when the contiguous
// blocks hold about the same number of list entries, else the tiles dealt
// in smaller chunks (TileDeal), longest first within the XCD.  A block of
// rows of one view ends with a light XCD (the edge of the detector) and a
// heavy one (its centre), and so do mixed view sizes, whose smallest views
// have the longest lists; large chunks keep neighbouring tiles, which
// share records, on one L2.  Of the chunkings n / (8 m) tiles, m = 1, 2,
// 4 ... 64, the coarsest within kDealSlack of an even split is taken, else
// the most even one.  The entries are counted in groups of consecutive
// tiles (`group` words of LDS, kOrderGroups of them), every workgroup over
// the whole frame, by 16 tiles of a group (order_sample): all of them up to
// 32 768 tiles, and never more than those reads.  The workgroup has 512 or
// 1024 threads.  (64 Gaussians in 1000 views of 512 x 512, 1M tiles, the list
// scatter with these workgroups in it: 509 us with every tile read, now 171;
// 1000 Gaussians in 500 such views 266 -> 117.)
// Measured (whole step, contiguous blocks -> dealt): 300k Gaussians, 32
// views of 128^2, 256^2 and 512^2 in that order 2.87 -> 2.04 ms; 200k, one
// view of 2048 x 1536 0.585 -> 0.518 ms, of 512^2 0.400 -> 0.389 ms; 200k,
// 8 views of 512^2 (one view per XCD, kept contiguous) unchanged.
constexpr int kOrderGroups = 2048;

// The tile that lane l of 16 reads of group k of g tiles (g a power of two
// from 16 on): one of its g / 16, at a place that differs from group to group
// and lane to lane, or it would be the same column of the detector every time.
__host__ __device__ __forceinline__ int64_t order_sample(int k, int l, int g) {
    const uint32_t h = ((uint32_t)k * 16u + (uint32_t)l) * 0x9e3779b1u;   // (multiplicative hashing)
    return (int64_t)k * g + (int64_t)l * (g / 16) + (int64_t)((h >> 8) & (uint32_t)(g / 16 - 1));
}

__device__ __forceinline__ void xcd_order_block(const Ws &ws, int x, uint32_t *hist, uint32_t *scan_lds,
                                                uint32_t *group) {
    static_assert(kXcds * kDealParts == kWave && kDealSteps * kWave <= 512, "a wavefront per step");
    const int n = (int)ws.total_tiles;
    const TileDeal own(n, n, true);
    const int cnt = own.tiles(x);
    const int t0 = x * own.q + min(x, own.rem);
    // list entries of every group of g consecutive tiles (16 lanes a group),
    // four groups' loads together
    int g = 16;
    while ((n + g - 1) / g > kOrderGroups) g *= 2;
    const int ng = (n + g - 1) / g, lanes = (int)blockDim.x / 16;
    const uint2 *rg = reinterpret_cast<const uint2 *>(ws.ranges);
    for (int k0 = (int)threadIdx.x / 16; k0 - (int)threadIdx.x / 16 < ng; k0 += 4 * lanes) {
        uint2 r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t t = order_sample(k0 + u * lanes, (int)threadIdx.x % 16, g);
            r[u] = t < n ? rg[t] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t len = r[u].y - r[u].x;
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) len += (uint32_t)__shfl_xor((int)len, o, kWave);
            if (k0 + u * lanes < ng && threadIdx.x % 16 == 0) group[k0 + u * lanes] = len;
        }
    }
    __shared__ float s_excess[kDealSteps];
    __syncthreads();
    if (threadIdx.x < kDealSteps * kWave) {   // a wavefront per step
        const int part = threadIdx.x % kDealParts, xx = threadIdx.x / kDealParts % kXcds;
        const int step = threadIdx.x / kWave;
        const TileDeal d(n, deal_chunk(n, g, step), step == 0);
        uint32_t load = deal_share(group, g, d, xx, part);
#pragma unroll
        for (int o = 1; o < kDealParts; o <<= 1) load += (uint32_t)__shfl_xor((int)load, o, kWave);
        uint32_t total = load;
#pragma unroll
        for (int o = kDealParts; o < kWave; o <<= 1) {
            load = max(load, (uint32_t)__shfl_xor((int)load, o, kWave));
            total += (uint32_t)__shfl_xor((int)total, o, kWave);
        }
        if (threadIdx.x % kWave == 0) s_excess[step] = deal_excess(load, total);
    }
    __syncthreads();
    const int best = deal_choice(s_excess);
    order_tiles(ws, cnt, [&](int j) { return own.tile(x, j); }, ws.xcd_order + t0,
                best == 0 ? ws.blend_order + t0 : nullptr, hist, scan_lds);
    if (best != 0) {
        const TileDeal d(n, deal_chunk(n, g, best), false);
        order_tiles(ws, cnt, [&](int j) { return d.tile(x, j); }, ws.blend_order + t0, nullptr, hist, scan_lds);
    }
}

// Resets the header words of a new frame other than the depth range.
__device__ __forceinline__ void frame_header_reset(WsHeader *h) {
    h->status = XG_OK;
    h->n_pairs = 0;
    h->item_sel = 0;
    h->item_passes = 0;
    h->queue_fwd = 0;
    h->queue_bwd = 0;
    h->done_fwd = 0;
    h->done_bwd = 0;
}

// Folds this workgroup's share of the preprocess's per-block depth partials
// ((min, max) pairs) into the header's depth range, which the preprocess
// set to (0xffffffff, 0).  Called by every thread of the workgroup
// (contains a barrier; at most 1024 threads).
__device__ __forceinline__ void depth_range_fold(WsHeader *h, const uint32_t *part, int64_t nparts) {
    uint32_t dmin = 0xffffffffu, dmax = 0u;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nparts;
         k += (int64_t)gridDim.x * blockDim.x) {
        dmin = min(dmin, part[2 * k]);
        dmax = max(dmax, part[2 * k + 1]);
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        dmin = min(dmin, (uint32_t)__shfl_xor((int)dmin, off, kWave));
        dmax = max(dmax, (uint32_t)__shfl_xor((int)dmax, off, kWave));
    }
    __shared__ uint32_t smin[16], smax[16];
    const int w = threadIdx.x / kWave;
    if (lane_id() == 0) { smin[w] = dmin; smax[w] = dmax; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < (int)(blockDim.x / kWave); ++k) {
            dmin = min(dmin, smin[k]);
            dmax = max(dmax, smax[k]);
        }
        if (dmin != 0xffffffffu) atomicMin(&h->depth_min, dmin);
        if (dmax != 0u) atomicMax(&h->depth_max, dmax);
    }
}

// View index of a global tile id: the last view whose tile_offset <= tile.
__device__ __forceinline__ int view_of_tile(const xg_camera *cams, int n_views, int tile) {
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (cams[mid].tile_offset <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

}  // namespace xg
