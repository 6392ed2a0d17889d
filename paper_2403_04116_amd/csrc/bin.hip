// Stage 2 (Sec. 3.2), the per-tile depth-ordered Gaussian lists, built by
// counting instead of sorting the pairs.
//
// The items (view, Gaussian) are sorted by depth within each view, so the
// items of view v sit in [v n, (v + 1) n) in (depth, Gaussian index)
// order, and their scanned tile counts give every item its pair slots.  A
// tile only lists Gaussians of its own view, in item order.  The lists are
// therefore a stable counting sort of each view's pairs by view-local tile
// id, whose digit range (the view's tiles, bounded by the plan) is small
// enough to count in LDS, in bands of whole tile rows where a view has more
// tiles than one workgroup's counters (each band a workgroup of its own, its
// items' rectangles clipped to it):
//   1. k_bin_count: per partition (ws.bin_items consecutive items of one
//      view), the number of pairs of each tile (LDS atomics over the items'
//      tile rectangles) -> one row of bin_cnt;
//   2. k_bin_columns: down each (view, tile) column of bin_cnt, the
//      exclusive scan over the view's partitions (segments in parallel),
//      and the tile's total;
//   3. k_bin_starts: the exclusive scan of a view's tile totals from the
//      view's first pair slot -> the tile ranges [start, end);
//   4. k_bin_scatter: per partition, the pairs in windows of kBinWindow
//      slots: a lane finds its slot's pair, the pairs are ranked stably within the
//      window (each row of 64 slots matched by tile through an LDS table of
//      lane masks, per-wavefront counters, then a prefix over the
//      wavefronts), reordered in LDS so that each tile's pairs are
//      adjacent, and written at tile start + column prefix + rank (runs of
//      consecutive entries per tile, not one scattered word per pair).
// The result is the same (tile, depth, index) order as the radix sort of
// the pairs, element for element; no pair is read back from memory.
#include "common.h"

namespace xg {

namespace {

struct BinPart {
    int view, q;
    int64_t j0, j1;   // items [j0, j1) of the partition
    int tiles_x, tiles_y, tiles, toff;
};

// Rows [y0, y1] of tiles of band `band`, and its first tile and tile count;
// bands hold at most `most` tiles, and tiles_x is at most that.  A band past
// the view's last row is empty.
struct Band {
    int y0, y1, first, tiles;
    __device__ __forceinline__ Band(const BinPart &b, int band, int most) {
        const int rows = most / b.tiles_x;
        y0 = min(band * rows, b.tiles_y);
        y1 = min(y0 + rows, b.tiles_y) - 1;
        first = y0 * b.tiles_x;
        tiles = (y1 - y0 + 1) * b.tiles_x;
    }
};

__device__ __forceinline__ BinPart bin_part(const Ws &ws, const xg_camera *cams, int tile, int part) {
    BinPart b;
    b.view = part / ws.bin_ppv;
    b.q = part - b.view * ws.bin_ppv;
    const int64_t vbase = (int64_t)b.view * ws.n;
    b.j0 = vbase + (int64_t)b.q * ws.bin_items;
    b.j1 = min(b.j0 + ws.bin_items, vbase + ws.n);
    const xg_camera &c = cams[b.view];
    b.tiles_x = (c.width + tile - 1) / tile;
    b.tiles_y = (c.height + tile - 1) / tile;
    b.tiles = b.tiles_x * b.tiles_y;
    b.toff = c.tile_offset;
    return b;
}

constexpr int kCountThreads = 1024;
constexpr int kCountTiles = 4096;     // tiles of a band of the counting kernel
constexpr int kScatterTiles = 1024;   // and of the ranking kernel
static_assert(kBinMaxTilesX <= kScatterTiles && kBinMaxTilesX <= kCountTiles, "a band holds a row of tiles");
static_assert(kBinItems % kCountThreads == 0, "whole items per thread");

// An item adds 1 where a row of its rectangle of tiles begins and takes 1 away
// where it ends (two LDS atomics a row whatever its length); the counts are
// the prefix sums of that along the rows.  What bounds the kernel is the item
// with the most work in each wavefront: with an atomic per tile, ACUI scan of
// 100 views (17 tiles an item) 1.293 ms, now 1.276; one 2048 x 1536 view of
// 200k Gaussians 379 -> 373 us; 1M x 16 views (3 tiles an item) 2.207 -> 2.201 ms.
// Taking differences along the columns too (four atomics an item, two more
// barriers) loses what it gains: 1.275, 374, 2.217.
__global__ __launch_bounds__(kCountThreads) void k_bin_count(Ws ws, const xg_camera *cams, int tile, int bands) {
    __shared__ uint32_t cnt[kCountTiles];
    const int part = (int)blockIdx.x / bands;
    const BinPart b = bin_part(ws, cams, tile, part);
    const Band bd(b, (int)blockIdx.x - part * bands, kCountTiles);
    // the item sort is over: leave its digit totals and counters zero
    if (ws.sort_fold)
        for (int64_t i = (int64_t)blockIdx.x * kCountThreads + threadIdx.x; i < item_sort_zeros(ws);
             i += (int64_t)gridDim.x * kCountThreads)
            zero_item_sort(ws, i);
    for (int t = threadIdx.x; t < bd.tiles; t += kCountThreads) cnt[t] = 0;
    __syncthreads();
    const int W = b.tiles_x;
    const int sel = ws.hdr->item_sel & 1;
    // every item's count and sort value loaded before any is used
    constexpr int kPer = kBinItems / kCountThreads;
    uint32_t n_t[kPer];
    uint64_t val[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t j = b.j0 + (int64_t)k * kCountThreads + threadIdx.x;
        n_t[k] = j < b.j1 ? ws.icounts[j] : 0u;
        val[k] = j < b.j1 ? ws.ivals[sel][j] : 0ull;
    }
    uint32_t mine = 0;   // this thread's pairs
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (n_t[k] == 0) continue;
        mine += n_t[k];
        const TileRect r = item_tile_rect(ws, val[k], tile);
        const int y0 = max(r.ty0, bd.y0), y1 = min(r.ty1, bd.y1);
        for (int ty = y0; ty <= y1; ++ty) {
            uint32_t *c = cnt + (ty * W - bd.first);
            atomicAdd(c + r.tx0, 1u);
            if (r.tx1 + 1 < W) atomicAdd(c + r.tx1 + 1, ~0u);
        }
    }
    // the partition's pair total, by its first band's workgroup (at most
    // kBinItems * kBinMostTiles)
    __shared__ uint32_t s_tot[kCountThreads / kWave];
    for (int off = kWave / 2; off > 0; off >>= 1) mine += (uint32_t)__shfl_xor((int)mine, off, kWave);
    if (lane_id() == 0) s_tot[threadIdx.x / kWave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0;
#pragma unroll
        for (int w = 0; w < kCountThreads / kWave; ++w) tot += s_tot[w];
        if (bd.y0 == 0) ws.bin_ptot[part] = tot;
    }
    // the prefix sums along the rows, a wavefront per row of tiles
    uint32_t *row = ws.bin_cnt + (int64_t)part * ws.bin_tiles + bd.first;
    const int H = bd.y1 - bd.y0 + 1, lane = lane_id();
    for (int y = threadIdx.x / kWave; y < H; y += kCountThreads / kWave) {
        uint32_t carry = 0;
        for (int x = lane; x - lane < W; x += kWave) {
            const uint32_t v = wave_incl_scan(x < W ? cnt[y * W + x] : 0u) + carry;
            if (x < W) row[y * W + x] = v;
            carry = (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
        }
    }
}

// Exclusive scan down each (view, local tile) column of bin_cnt over the
// view's partitions, rewritten in place; the column total goes to the
// tile's range start word until k_bin_starts replaces it, and the sum of the
// workgroup's columns to bin_csum.  A workgroup takes 64 columns; its wavefronts split each column's partitions into
// kColSegs consecutive segments: each sums its segment, the segment totals are
// scanned through LDS, and each rewrites its segment from its offset.
static_assert(kColTiles == kWave, "a wavefront adds up a workgroup's columns");
constexpr int kColSegs = 8;
constexpr int kColThreads = kColTiles * kColSegs;

__global__ __launch_bounds__(kColThreads) void k_bin_columns(Ws ws, const xg_camera *cams, int tile,
                                                             int chunks) {
    __shared__ uint32_t part[kColSegs][kColTiles];
    const int v = blockIdx.x / chunks;
    const int seg = threadIdx.x / kColTiles;
    const int t = (blockIdx.x - v * chunks) * kColTiles + (threadIdx.x % kColTiles);
    const xg_camera &c = cams[v];
    const int tiles = ((c.width + tile - 1) / tile) * ((c.height + tile - 1) / tile);
    const int64_t stride = ws.bin_tiles;
    const int per = (ws.bin_ppv + kColSegs - 1) / kColSegs;
    const int q0 = min(seg * per, ws.bin_ppv), q1 = min(q0 + per, ws.bin_ppv);
    uint32_t *col = ws.bin_cnt + (int64_t)v * ws.bin_ppv * stride + t;
    const bool live = t < tiles;
    uint32_t sum = 0;
    if (live) {
        int q = q0;
        for (; q + 8 <= q1; q += 8) {   // eight loads in flight per step
            uint32_t x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = col[(int64_t)(q + k) * stride];
#pragma unroll
            for (int k = 0; k < 8; ++k) sum += x[k];
        }
        for (; q < q1; ++q) sum += col[(int64_t)q * stride];
    }
    part[seg][threadIdx.x % kColTiles] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (int k = 0; k < kColSegs; ++k) {
        const uint32_t x = part[k][threadIdx.x % kColTiles];
        run += k < seg ? x : 0u;
        total += x;
    }
    if (seg == 0) {   // one wavefront: the pairs of the workgroup's tiles
        uint32_t sum = total;
        for (int off = kWave / 2; off > 0; off >>= 1) sum += (uint32_t)__shfl_xor((int)sum, off, kWave);
        if (lane_id() == 0) ws.bin_csum[blockIdx.x] = sum;
    }
    if (!live) return;
    int q = q0;
    for (; q + 8 <= q1; q += 8) {
        uint32_t x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = col[(int64_t)(q + k) * stride];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            col[(int64_t)(q + k) * stride] = run;
            run += x[k];
        }
    }
    for (; q < q1; ++q) {
        const uint32_t x = col[(int64_t)q * stride];
        col[(int64_t)q * stride] = run;
        run += x;
    }
    if (seg == kColSegs - 1) ws.ranges[2 * ((int64_t)c.tile_offset + t)] = total;
}

// One workgroup per kStartThreads tiles of a view.  The view's first pair
// slot is the sum of the pair totals of the partitions of the views before
// it; the pair count of the whole frame (every workgroup sums all
// partitions) is checked against the capacity (XG_ECAPACITY, and the pair
// count, written by the first workgroup).  The view's first workgroup scans
// its partition totals into each partition's first slot.  The tile ranges
// are the scan of the tile totals, from the sums of the column workgroups
// before.  Empty tiles, and all tiles once the capacity is exceeded, read
// (0, 0).  (One workgroup for a whole view reads a large view's totals at
// the rate of one CU's outstanding loads: 15 us for 12 288 tiles.)
constexpr int kStartThreads = 1024;

__global__ __launch_bounds__(kStartThreads) void k_bin_starts(Ws ws, const xg_camera *cams, int tile, int blocks,
                                                              int chunks) {
    __shared__ alignas(16) uint32_t lds[kScanLds];
    __shared__ uint64_t s_sum[3][kStartThreads / kWave];
    const int v = (int)blockIdx.x / blocks, blk = (int)blockIdx.x - v * blocks;
    const xg_camera &c = cams[v];
    const int tiles = ((c.width + tile - 1) / tile) * ((c.height + tile - 1) / tile);
    uint2 *rg = reinterpret_cast<uint2 *>(ws.ranges) + c.tile_offset;
    const int t = blk * kStartThreads + (int)threadIdx.x;
    const uint32_t n = t < tiles ? rg[t].x : 0u;
    const int ppv = ws.bin_ppv;
    const int64_t nparts = (int64_t)ws.n_views * ppv;
    uint64_t before = 0, all = 0, columns = 0;
    for (int64_t k = threadIdx.x; k < nparts; k += kStartThreads) {
        const uint32_t x = ws.bin_ptot[k];
        all += x;
        if (k < (int64_t)v * ppv) before += x;
    }
    for (int k = threadIdx.x; k < min(blk * (kStartThreads / kColTiles), chunks); k += kStartThreads)
        columns += ws.bin_csum[(int64_t)v * chunks + k];
    for (int off = kWave / 2; off > 0; off >>= 1) {
        before += __shfl_xor(before, off, kWave);
        all += __shfl_xor(all, off, kWave);
        columns += __shfl_xor(columns, off, kWave);
    }
    if (lane_id() == 0) {
        s_sum[0][threadIdx.x / kWave] = before;
        s_sum[1][threadIdx.x / kWave] = all;
        s_sum[2][threadIdx.x / kWave] = columns;
    }
    __syncthreads();
    before = 0;
    all = 0;
    columns = 0;
#pragma unroll
    for (int w = 0; w < kStartThreads / kWave; ++w) {
        before += s_sum[0][w];
        all += s_sum[1][w];
        columns += s_sum[2][w];
    }
    const bool st_ok = ws.hdr->status == XG_OK;   // an item sort that gave up keeps its XG_EHIP
    const bool ok = st_ok && all <= (uint64_t)ws.cap;
    uint32_t tot;
    const uint32_t start = (uint32_t)(before + columns) + block_excl_scan(n, lds, &tot);
    if (t < tiles) rg[t] = ok && n > 0 ? make_uint2(start, start + n) : make_uint2(0u, 0u);
    if (blk > 0) return;
    if (v == 0 && threadIdx.x == 0) {
        ws.hdr->n_pairs = (int32_t)(all > 0x7fffffffull ? 0x7fffffffull : all);
        if (st_ok && all > (uint64_t)ws.cap) ws.hdr->status = XG_ECAPACITY;
    }
    // partition starts (below the capacity whenever they are used)
    uint32_t carry = (uint32_t)before;
    for (int q0 = 0; q0 < ppv; q0 += kStartThreads) {
        const int q = q0 + threadIdx.x;
        const uint32_t x = q < ppv ? ws.bin_ptot[(int64_t)v * ppv + q] : 0u;
        const uint32_t ex = block_excl_scan(x, lds, &tot);
        if (q < ppv) ws.bin_pstart[(int64_t)v * ppv + q] = carry + ex;
        carry += tot;
    }
}

// Stable ranking and placement of one partition's pairs in one band of its
// view's tile rows (LT tiles at most; most views have a single band).  The
// pairs of the band are numbered in item order (slots).  Per window: the
// slots [w0, w0 + kBinWindow) at which items begin are marked, and each lane
// counts its way to its slot's item, whose rectangle gives the pair's tile;
// wavefront w ranks its kBinWindow / NW consecutive slots, row by row (the
// lanes of a row holding a tile found through the lane-mask table), with a
// 16-bit counter per tile (two per word, LDS atomics from one leader lane
// per tile in a row); a prefix over the wavefronts then turns the counters
// into each wavefront's offset inside the window.  Every pair belongs at
// base[tile] + that offset + its rank, where base[tile] = the tile's start
// + the column prefix of the partition + the window's predecessors; the
// pairs are first permuted in LDS into blocks of one tile each (a
// wavefront scan of the tile totals), so that the stores of a row write
// runs of consecutive list entries.
// (16 wavefronts, at most 64 registers, so that two workgroups share a CU.
// Bands of 4096 tiles, whose counters leave 8 wavefronts on a CU: 200k
// Gaussians, 8 views of 4096 tiles, 0.64 ms a forward pass where bands of 1024
// take 0.52.)
// What bounds it: barriers and LDS round trips with two workgroups on a CU
// (HBM and VALU are both below half).  A lane per slot, loads issued together at the
// start and one base word per tile for the placement, against a thread per item
// that wrote its pairs one by one: ACUI scan of 100 views
// (17 pairs an item) 1.355 -> 1.320 ms, one 2048 x 1536 view of 200k Gaussians 0.396 -> 0.375,
// 200k x 8 views 0.468 -> 0.464, 1M x 16 views 2.31 -> 2.28; 1k Gaussians at
// 64 x 64, which is all latency, 42.8 -> 43.1 us.
// MI = items per thread: the partitions hold at most MI NT items.
template <int MI>
__global__ __launch_bounds__(1024, 8) void k_bin_scatter(Ws ws, const xg_camera *cams, int tile, int bands) {
    constexpr int LT = kScatterTiles, NW = 16;
    constexpr int NT = NW * kWave;
    constexpr int LB = 10;
    constexpr int kRows = kBinWindow / NT;         // rows of 64 slots per wavefront
    constexpr int kMyItems = MI;
    static_assert(LT <= (1 << LB) && kBinWindow % NT == 0, "shape");
    static_assert(kBinWindow <= 65535, "window offsets and counts fit 16 bits");
    __shared__ alignas(16) uint32_t h16[NW][LT / 2];
    __shared__ uint32_t base[LT];
    // the items with pairs in the band, in order: first tile | columns << 16 |
    // first slot << 32
    static_assert(LT <= 1 << 10, "fields of an item");
    __shared__ uint64_t s_item[MI * NT];
    // the slots of a window at which an item begins, a word for each row of 64
    __shared__ uint64_t s_begin[2][kBinWindow / kWave];
    static_assert(kBinWindow / kWave == kWave, "one word per lane");
    // the window's pairs in tile order, and each tile's first window position
    // (two 16-bit starts per word)
    __shared__ alignas(16) uint32_t s_gi[kBinWindow];
    __shared__ alignas(16) uint16_t s_lt[kBinWindow];
    __shared__ alignas(16) uint32_t s_lst[LT / 2];
    __shared__ uint32_t s_alloc;
    // ranking: per wavefront, a 64-bit lane mask for each value of a tile's
    // low kHashBits bits (zero between rows), in the words that hold the
    // window's pairs afterwards
    constexpr int kHashBits = 6, kHash = 1 << kHashBits;
    static_assert(kHash == kWave && sizeof(s_gi) >= NW * kHash * sizeof(uint64_t), "one word per lane");
    uint64_t *s_tab = reinterpret_cast<uint64_t *>(s_gi) + threadIdx.x / kWave * kHash;
    // the items' indices, until the window's tiles take their words
    static_assert(sizeof(s_lt) >= MI * NT * sizeof(uint32_t), "a word per item");
    uint32_t *s_igi = reinterpret_cast<uint32_t *>(s_lt);

    // the first kXcds workgroups write the blend launches' tile order (the
    // ranges are final; every status, since the blends read it even when
    // the lists are empty), in slots the partitions leave idle
    if ((int)blockIdx.x < kXcds) {
        static_assert(NW * (LT / 2) >= kOrderGroups && LT >= kOrderBuckets && LT / 2 >= kScanLds, "scratch of the order");
        xcd_order_block(ws, blockIdx.x, base, s_lst, &h16[0][0]);
        return;
    }
    const int part = ((int)blockIdx.x - kXcds) / bands;
    const BinPart b = bin_part(ws, cams, tile, part);
    const Band bd(b, (int)blockIdx.x - kXcds - part * bands, LT);
    if (b.j0 >= b.j1 || bd.tiles <= 0) return;

    // everything that depends on no other load is loaded before anything is
    // used: two round trips to memory before the first window, where testing
    // each in turn took five
    const uint32_t status = ws.hdr->status;
    const int sel = __builtin_amdgcn_readfirstlane((int)ws.hdr->item_sel) & 1;
    const uint32_t pstart = ws.bin_pstart[part];
    const int64_t j0 = b.j0 + (int64_t)threadIdx.x * kMyItems;   // this thread's items
    uint32_t icnt[kMyItems];
#pragma unroll
    for (int k = 0; k < kMyItems; ++k) icnt[k] = j0 + k < b.j1 ? ws.icounts[j0 + k] : 0u;
    const uint32_t *colp = ws.bin_cnt + (int64_t)part * ws.bin_tiles + bd.first;
    static_assert(LT == NT, "a tile per thread");
    const bool mine = (int)threadIdx.x < bd.tiles;
    const uint32_t tstart = mine ? ws.ranges[2 * ((int64_t)b.toff + bd.first + threadIdx.x)] : 0u;
    const uint32_t tcol = mine ? colp[threadIdx.x] : 0u;
    uint64_t ival[kMyItems];
#pragma unroll
    for (int k = 0; k < kMyItems; ++k) ival[k] = j0 + k < b.j1 ? ws.ivals[sel][j0 + k] : 0ull;
    if (status != XG_OK) return;
    if (threadIdx.x < 2 * kWave) (&s_begin[0][0])[threadIdx.x] = 0ull;
    base[threadIdx.x] = tstart + tcol;

    // this thread's items: slot range (the exclusive scan of the items'
    // pairs in the band, in item order), tile rectangle clipped to the band,
    // index
    // (counts and tile coordinates in the band fit 16 bits)
    uint32_t i_off[kMyItems], i_gi[kMyItems];
    uint32_t i_cy[kMyItems];  // pair count | first tile row of the band << 16
    uint32_t i_x[kMyItems];   // first | last tile column << 16
#pragma unroll
    for (int k = 0; k < kMyItems; ++k) {
        i_cy[k] = 0;
        i_x[k] = 0;
        i_gi[k] = (uint32_t)ival[k] - (uint32_t)b.view * (uint32_t)ws.n;
        if (icnt[k] > 0) {
            const TileRect r = item_tile_rect(ws, ival[k], tile);
            const int y0 = max(r.ty0, bd.y0), y1 = min(r.ty1, bd.y1);
            i_x[k] = (uint32_t)r.tx0 | ((uint32_t)r.tx1 << 16);
            if (y0 <= y1)
                i_cy[k] = (uint32_t)((r.tx1 - r.tx0 + 1) * (y1 - y0 + 1)) | ((uint32_t)(y0 - bd.y0) << 16);
        }
    }
    // a thread's items are consecutive (j0 + thread kMyItems + k): one block
    // scan of the thread sums, of the band's pairs, of the items that have any
    // and, for the first band's workgroup, of the items' whole counts (the
    // offsets, from the partition's first pair)
    uint32_t E, ord;
    {
        __shared__ alignas(16) uint32_t s_scan[3 * kScanLds];
        uint32_t sums[3] = {0, 0, 0}, tot[3];
#pragma unroll
        for (int k = 0; k < kMyItems; ++k) {
            const uint32_t cnt = i_cy[k] & 0xffffu;
            sums[0] += cnt;
            sums[1] += cnt != 0;
            sums[2] += icnt[k];
        }
        block_excl_scans<3>(sums, s_scan, tot);
        E = tot[0];
        uint32_t run = sums[0], off = pstart + sums[2], o = sums[1];
        ord = o;
#pragma unroll
        for (int k = 0; k < kMyItems; ++k) {
            const uint32_t cnt = i_cy[k] & 0xffffu;
            i_off[k] = cnt ? run : ~0u;   // (none: past every window)
            if (cnt) {
                const uint32_t tx0 = i_x[k] & 0xffffu, cols = (i_x[k] >> 16) - tx0 + 1u;
                s_item[o++] = (uint64_t)(((i_cy[k] >> 16) * (uint32_t)b.tiles_x + tx0) | (cols << 16)) | ((uint64_t)run << 32);
            }
            run += cnt;
            if (bd.y0 == 0 && j0 + k < b.j1) ws.offsets[j0 + k] = off;
            off += icnt[k];
        }
    }

    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int lane = lane_id();
    const int gb = ws.pair_gbits;
    uint32_t *out_t = ws.ptile[ws.pair_sel];
    uint32_t *out_v = ws.pval[ws.pair_sel];

    uint32_t first = 0;   // items begun before the window
    int buf = 0;
    for (uint32_t w0 = 0; w0 < E; w0 += kBinWindow, buf ^= 1) {
        const uint32_t w1 = min(E, w0 + (uint32_t)kBinWindow);
        const int wn = (int)(w1 - w0);
        for (int k = threadIdx.x; k < NW * (LT / 2) / 4; k += NT)
            reinterpret_cast<uint4 *>(&h16[0][0])[k] = make_uint4(0u, 0u, 0u, 0u);
        if (threadIdx.x == 0) s_alloc = 0u;
        uint32_t o = ord;
#pragma unroll
        for (int k = 0; k < kMyItems; ++k) {
            if (i_off[k] != ~0u) s_igi[o++] = i_gi[k];
            const uint32_t a = i_off[k] - w0;   // (wraps if begun before the window)
            if (a < (uint32_t)wn)
                atomicOr(reinterpret_cast<unsigned long long *>(&s_begin[buf][a / kWave]), 1ull << (a % kWave));
        }
        __syncthreads();
        // emission, a lane for each slot: the items begun up to the slot are
        // counted, which numbers the slot's item, and the slot's place in the
        // item's rectangle (row-major) gives the tile.  Every lane has the same
        // work whatever the items' sizes; where a thread wrote its items' pairs
        // one by one, a wavefront took as long as its largest
        const uint64_t begin = s_begin[buf][lane];
        if (threadIdx.x < kWave) s_begin[buf ^ 1][threadIdx.x] = 0ull;
        s_tab[lane] = 0ull;
        const uint32_t begun = wave_incl_scan((uint32_t)__popcll(begin));
        uint32_t tt[kRows], gi[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int row = w * kRows + r;
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)begin, row);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(begin >> 32), row);
            const uint64_t m = (uint64_t)lo | ((uint64_t)hi << 32);
            // the last item begun before the row's second slot, then one for
            // every beginning from there up to the lane's slot
            const uint32_t id0 = first + (uint32_t)__builtin_amdgcn_readlane((int)begun, row) - (uint32_t)__popcll(m >> 1) - 1u;
            const uint32_t id = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 33), __builtin_amdgcn_mbcnt_lo((uint32_t)(m >> 1), id0));
            const uint64_t it = s_item[id];
            const uint32_t tc = (uint32_t)it;
            gi[r] = s_igi[id];
            const uint32_t cols = tc >> 16;
            const uint32_t k = w0 + (uint32_t)(row * kWave + lane) - (uint32_t)(it >> 32);
            // k / cols, both at most 1024 (LT): with half a unit added to k the
            // quotient is at least 0.5 / 1024 of itself from a whole number
            const uint32_t y = (uint32_t)(((float)k + 0.5f) * __builtin_amdgcn_rcpf((float)cols));
            tt[r] = (tc & 0xffffu) + k + __umul24(y, (uint32_t)b.tiles_x - cols);
        }
        first += (uint32_t)__builtin_amdgcn_readlane((int)begun, kWave - 1);
        // ranking: wavefront w owns slots [w kRows 64, (w + 1) kRows 64)
        uint32_t rt[kRows];   // rank in the wavefront | tile << 16 (both below 2^16)
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int slot = (w * kRows + r) * kWave + lane;
            const bool valid = slot < wn;
            const uint32_t t = valid ? tt[r] : 0u;
            // lanes of the row with this tile: the lanes whose low kHashBits
            // agree (one bit each, OR-ed into this wavefront's table slot,
            // read back, then cleared; a wavefront's LDS operations complete
            // in order) that also agree in the high bits (one ballot each)
            uint64_t *slotp = &s_tab[t & (kHash - 1)];
            if (valid) atomicOr(reinterpret_cast<unsigned long long *>(slotp), 1ull << lane);
            const uint64_t same_low = *slotp;
            *slotp = 0ull;
            const uint64_t peers = valid ? same_low & match_peers<LB - kHashBits>(t >> kHashBits, valid) : 0ull;
            // every lane reads its tile's count, then the first lane of each
            // tile adds the row's (two tiles share a word: an atomic, whose
            // result nothing waits for)
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            const uint32_t sh = 16u * (t & 1u);
            const uint32_t old = (h16[w][t >> 1] >> sh) & 0xffffu;
            if (valid && below == 0) atomicAdd(&h16[w][t >> 1], (uint32_t)__popcll(peers) << sh);
            rt[r] = (old + below) | (t << 16);
        }
        __syncthreads();
        // prefix over the wavefronts, two tiles (one word) per step; then each
        // tile's block of window positions: a wavefront scan of the word
        // totals and one allocation per wavefront (blocks in any order, each
        // tile's block contiguous)
        constexpr int kPairsPerThread = (LT / 2 + NT - 1) / NT;
        uint32_t adv[kPairsPerThread], pos[kPairsPerThread];
#pragma unroll
        for (int k = 0; k < kPairsPerThread; ++k) {
            const int tw = k * NT + threadIdx.x;
            uint32_t run = 0;   // two 16-bit sums
            if (tw < LT / 2) {
#pragma unroll
                for (int x = 0; x < NW; ++x) {
                    const uint32_t hcur = h16[x][tw];
                    h16[x][tw] = run;
                    run += hcur;   // neither half exceeds kBinWindow: no carry
                }
            }
            adv[k] = run;
            const uint32_t lo = run & 0xffffu;
            const uint32_t tot = lo + (run >> 16);
            const uint32_t incl = wave_incl_scan(tot);
            const uint32_t wsum = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
            uint32_t wbase = 0;
            if (lane == 0 && wsum) wbase = atomicAdd(&s_alloc, wsum);
            wbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)wbase);
            const uint32_t st = wbase + incl - tot;
            pos[k] = st;
            if (tw < LT / 2 && tot) {
                s_lst[tw] = st | ((st + lo) << 16);
                // for the placement: the list entry of window position 0
                base[2 * tw] -= st;
                base[2 * tw + 1] -= st + lo;
            }
        }
        __syncthreads();
        // each slot's window position: its tile's block, the wavefronts
        // before it, its rank in the wavefront
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int slot = (w * kRows + r) * kWave + lane;
            if (slot < wn) {
                const uint32_t t = rt[r] >> 16;
                const uint32_t sh = 16u * (t & 1u);
                const uint32_t off = (h16[w][t >> 1] >> sh) & 0xffffu;
                const uint32_t st = (s_lst[t >> 1] >> sh) & 0xffffu;
                const uint32_t k = st + off + (rt[r] & 0xffffu);
                s_lt[k] = (uint16_t)t;
                s_gi[k] = gi[r];
            }
        }
        __syncthreads();
        // placement in tile order: consecutive positions of a tile go to
        // consecutive list entries (coalesced stores)
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int k = (w * kRows + r) * kWave + lane;
            if (k < wn) {
                const uint32_t t = s_lt[k];
                const uint32_t gi = s_gi[k];
                const uint32_t dst = base[t] + (uint32_t)k;
                const uint32_t gt = (uint32_t)(b.toff + bd.first) + t;
                if (dst >= (uint64_t)ws.cap) continue;   // never: the counts add up to the slots
                if (gb) {
                    out_t[dst] = (gt << gb) | gi;
                } else {
                    out_t[dst] = gt;
                    out_v[dst] = gi;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPairsPerThread; ++k) {
            const int tw = k * NT + threadIdx.x;
            if (tw < LT / 2 && adv[k]) {   // past the window's pairs
                const uint32_t lo = adv[k] & 0xffffu;
                base[2 * tw] += pos[k] + lo;
                base[2 * tw + 1] += pos[k] + lo + (adv[k] >> 16);
            }
        }
        // the next window's counters are cleared before its ranking, after
        // the barrier that follows its emission; base is next read after that
    }
}

}  // namespace

hipError_t launch_bin_lists(const Ws &ws, const xg_camera *cams, const Params &p, hipStream_t s) {
    if (ws.bin_tiles <= 0 || ws.bin_tiles > kBinMostTiles || ws.bin_bands <= 0 || ws.bin_ppv <= 0 ||
        ws.bin_items <= 0 || ws.bin_items > kBinItems)
        return hipErrorInvalidValue;
    const int64_t parts = (int64_t)ws.n_views * ws.bin_ppv;
    // (a counting band of 4 ranking bands' tiles holds at least 4 of them)
    const int cbands = (ws.bin_bands + kCountTiles / kScatterTiles - 1) / (kCountTiles / kScatterTiles);
    if (parts * ws.bin_bands + kXcds > 0x7fffffff) return hipErrorInvalidValue;
    if (ws.view_sort != ViewSort::kLists) {   // else counted by the item sort's launch
        hipLaunchKernelGGL(k_bin_count, dim3((unsigned)(parts * cbands)), dim3(kCountThreads), 0, s, ws, cams, p.tile,
                           cbands);
        const int chunks = (ws.bin_tiles + kColTiles - 1) / kColTiles;
        hipLaunchKernelGGL(k_bin_columns, dim3((unsigned)(ws.n_views * chunks)), dim3(kColThreads), 0, s, ws,
                           cams, p.tile, chunks);
        const int blocks = (ws.bin_tiles + kStartThreads - 1) / kStartThreads;
        hipLaunchKernelGGL(k_bin_starts, dim3((unsigned)(ws.n_views * blocks)), dim3(kStartThreads), 0, s, ws, cams,
                           p.tile, blocks, chunks);
    }
    // kXcds extra workgroups write the blend launches' tile order
    const dim3 grid((unsigned)(parts * ws.bin_bands) + kXcds);
    if (ws.bin_items > 1024)
        hipLaunchKernelGGL(k_bin_scatter<2>, grid, dim3(1024), 0, s, ws, cams, p.tile, ws.bin_bands);
    else
        hipLaunchKernelGGL(k_bin_scatter<1>, grid, dim3(1024), 0, s, ws, cams, p.tile, ws.bin_bands);
    return hipGetLastError();
}

}  // namespace xg
