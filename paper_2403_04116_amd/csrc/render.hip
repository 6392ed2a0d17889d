// Stage 3 and its adjoint: front-to-back blending (Eq. 10) of every pixel
// over its tile's depth-sorted list, and the reverse-order backward.
//
// Work decomposition (gfx950, 64-lane wavefronts): one workgroup per tile
// of T x T pixels (T = 8, 16, 32), one lane per pixel, and each wavefront
// owns an 8 x 8 sub-block of the tile.  Gaussians of the tile's list are
// staged through LDS in batches of B; every wavefront then walks the batch
// with the Gaussian's data broadcast from LDS.  A wavefront skips a
// Gaussian whose bounding rectangle misses its 8 x 8 sub-block (a scalar
// test), leaves the batch as soon as all its lanes have terminated, and the
// workgroup stops staging once every lane is done.
//
// Numerics: positions are relative to the centre of the enclosing 32 x 32
// pixel block (the preprocess stores the centre as integer + fraction), the
// same reference for every tile size, so a pixel's arithmetic does not
// depend on the tiling; and the Mahalanobis form is factored
// (k d^T Sigma''^-1 d = (qa dx + qb dy)^2 + (qc dy)^2) so the exponent has
// no catastrophic cancellation; alpha is computed by one inline function
// shared by both kernels, so the backward recomputes the forward's alpha
// bit for bit and can divide the transmittance back.
#include "common.h"

#include <type_traits>

namespace xg {

namespace {

struct Eval {
    float dx, dy, y1, y2, a, alpha;
};

// Records marked kRecPlain (almost all: the bounding rectangle is taken for
// opacity 1, so with its own opacity a Gaussian falls below alpha_min
// inside it) need neither the rectangle test nor the alpha clamp.  A
// wavefront whose list of a batch holds only such records walks it without
// them: 3 of about 20 VALU instructions a visit in the forward, 4 of 43 in
// the backward.  The results are the same bit for bit.  200k Gaussians x 8
// views of 512 x 512: step 0.511 -> 0.495 ms; ACUI scan, 100 views: 1.45 ->
// 1.40 ms.
//
// alpha of one staged Gaussian at a pixel centre (px, py), both relative
// to the block reference point.  sa = (ux, uy, qa, qb), sb = (qc, -log2 o,
// intensity, rectangle word): a = o G = exp2(-(E - log2 o)), with E the
// scaled Mahalanobis term, so the opacity enters the exponent's sum.
// PLAIN: the alpha cannot reach the clamp.
template <bool PLAIN>
__device__ __forceinline__ Eval splat_eval(const float4 &sa, const float4 &sb, float px, float py,
                                           float amax) {
#pragma clang fp contract(off)
    Eval e;
    e.dx = px - sa.x;
    e.dy = py - sa.y;
    e.y1 = fmaf(sa.w, e.dy, sa.z * e.dx);
    e.y2 = sb.x * e.dy;
    const float E = fmaf(e.y2, e.y2, fmaf(e.y1, e.y1, sb.y));
    e.a = __builtin_amdgcn_exp2f(-E);
    e.alpha = PLAIN ? e.a : fminf(e.a, amax);
    return e;
}

struct TileGeom {
    int view, x0, y0, W, H, pix_off;
    int rx, ry;   // reference point: centre of the enclosing 32 x 32 block
};

__device__ __forceinline__ TileGeom tile_geom(const xg_camera *cams, int n_views, int tile, int T) {
    TileGeom t;
    t.view = view_of_tile(cams, n_views, tile);
    const xg_camera &c = cams[t.view];
    t.W = c.width;
    t.H = c.height;
    t.pix_off = c.pixel_offset;
    const int txn = (t.W + T - 1) / T;
    const int lt = tile - c.tile_offset;
    const int ty = lt / txn;
    t.x0 = (lt - ty * txn) * T;
    t.y0 = ty * T;
    t.rx = (t.x0 & ~31) + 16;
    t.ry = (t.y0 & ~31) + 16;
    return t;
}

// The tile-local rectangle [xl, xh] x [yl, yh] of a staged entry, in the
// form the blend loops test it.  T <= 16: bit x of the low half and bit y of
// the high half are set for the columns and rows the rectangle covers, and a
// lane at (lx, ly) is inside iff both of its two bits are set: one AND and
// one compare per entry against a per-lane constant.  T = 32 (32 columns do
// not fit a half word): the four bounds as bytes, compared one by one.
template <int T>
__device__ __forceinline__ uint32_t rect_word(int xl, int xh, int yl, int yh) {
    if constexpr (T <= 16) {
        const uint32_t xm = ((2u << xh) - 1u) & ~((1u << xl) - 1u);
        const uint32_t ym = ((2u << yh) - 1u) & ~((1u << yl) - 1u);
        return xm | (ym << 16);
    } else {
        return (uint32_t)xl | ((uint32_t)xh << 8) | ((uint32_t)yl << 16) | ((uint32_t)yh << 24);
    }
}

template <int T>
__device__ __forceinline__ uint32_t rect_lane_key(int lx, int ly) {
    return T <= 16 ? (1u << lx) | (1u << (16 + ly)) : 0u;
}

template <int T>
__device__ __forceinline__ bool in_rect(uint32_t rect, uint32_t key, int lx, int ly) {
    if constexpr (T <= 16) {
        return (rect & key) == key;
    } else {
        const int rxl = rect & 255, rxh = (rect >> 8) & 255;
        const int ryl = (rect >> 16) & 255, ryh = rect >> 24;
        return lx >= rxl && lx <= rxh && ly >= ryl && ly <= ryh;
    }
}

// Bit s of the result: the tile-local rectangle [xl, xh] x [yl, yh] touches
// the 8 x 8 sub-block s (row-major, SB sub-blocks per row).
template <int SB>
__device__ __forceinline__ uint32_t subblock_mask(int xl, int xh, int yl, int yh) {
    const int cx0 = xl >> 3, cx1 = xh >> 3, cy0 = yl >> 3, cy1 = yh >> 3;
    const uint32_t row = ((1u << (cx1 - cx0 + 1)) - 1u) << cx0;
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < SB; ++r)
        if (r >= cy0 && r <= cy1) m |= row << (r * SB);
    return m;
}

// Sub-block culling (in stage below): the smallest value over a box
// [X0, X1] x [Y0, Y1] of the exponent
// E(dx, dy) = (qa dx + qb dy)^2 + (qc dy)^2 (qa > 0, qb^2 + qc^2 > 0), whose
// minimum 0 is at the origin.  For a box point p, the segment from p to the
// origin leaves the box through an edge facing the origin, at a point q
// with E(q) <= E(p) (E is convex); so the minimum lies on the vertical edge
// x = Xn and the horizontal edge y = Yn nearest the origin, Xn and Yn the
// origin's coordinates clamped to the box (a clamped coordinate that the
// box already spans gives a line through the box, whose minimum is no
// smaller, and for a box holding the origin both lines give 0).  Along each
// line E is a one-dimensional quadratic minimised at -rx Yn resp. -ry Xn
// (rx = qb / qa, ry = qa qb / (qb^2 + qc^2)), clamped to the edge.
// (X0 <= X1 and Y0 <= Y1, all finite: each clamp is one median of three)
__device__ __forceinline__ float box_min_exponent(float qa, float qb, float qc, float rx, float ry,
                                                  float X0, float X1, float Y0, float Y1) {
    const float xn = __builtin_amdgcn_fmed3f(0.0f, X0, X1);
    const float yn = __builtin_amdgcn_fmed3f(0.0f, Y0, Y1);
    const float x = __builtin_amdgcn_fmed3f(-rx * yn, X0, X1);
    const float e1 = qa * x + qb * yn, e2 = qc * yn;
    const float y = __builtin_amdgcn_fmed3f(-ry * xn, Y0, Y1);
    const float f1 = qa * xn + qb * y, f2 = qc * y;
    return fminf(e1 * e1 + e2 * e2, f1 * f1 + f2 * f2);
}

// Stages list entries [b0, b0 + cnt) of the tile into LDS, with the mask of
// the 8 x 8 sub-blocks each entry must be visited for.  A sub-block is in
// the mask when the entry's rectangle touches it and (CULL) the entry's
// alpha can reach alpha_min somewhere in that part of the rectangle: the
// smallest exponent over the part, a lower bound of every pixel's, is
// compared with log2(o / alpha_min) plus a margin far above float
// rounding.  Dropping the others skips only evaluations that the
// per-pixel alpha test would skip, so results do not change.
// DUAL (the counting forward): s_mask keeps the rectangle-only mask and
// s_cmask receives the culled one.
// MASKIO: 1 (the blending forward) also writes the culled mask of list
// entry p to the workspace's per-entry mask array; 2 (the backward) reads it
// from there instead of testing the sub-blocks again.  Every entry the
// backward stages was staged by the forward of the same lists (a pixel's
// last contributor lies in a batch the forward staged), and both would
// compute the same mask.
//
// Tiles of at most 16 x 16 (four sub-blocks) also carry kMaskExact: set
// unless the record is marked kRecPlain.
constexpr uint32_t kMaskExact = 0x8000u;
template <int T>
using SubMask = std::conditional_t<(T > 16), uint16_t, uint8_t>;

template <int T, int NT, bool CULL, bool DUAL = false, int MASKIO = 0>
__device__ __forceinline__ void stage(const Ws &ws, const uint32_t *vals, uint32_t b0, int cnt,
                                      const TileGeom &tg, float amin, float4 *s_a, float4 *s_b,
                                      uint16_t *s_mask, uint32_t *s_rid, float4 *s_c = nullptr,
                                      uint16_t *s_cmask = nullptr) {
    constexpr int SB = T / 8;
    static_assert(!(MASKIO && DUAL), "the counting forward neither stores nor loads masks");
    SubMask<T> *gmask = reinterpret_cast<SubMask<T> *>(ws.entry_mask);
    const float lg_amin = -__builtin_amdgcn_logf(amin);   // log2(1 / alpha_min)
    for (int k = threadIdx.x; k < cnt; k += NT) {
        const uint32_t gi = vals[b0 + k] & ws.pair_gmask;   // Gaussian index (packed or not)
        const int64_t rid = (int64_t)tg.view * ws.n + gi;
        const Record &rec = ws.rec[rid];
        const float4 ra = rec.a;
        const float4 rb = rec.b;
        const int4 rc = rec.c;
        const float ux = (float)(rc.x - tg.rx) + ra.x;
        const float uy = (float)(rc.y - tg.ry) + ra.y;
        const int xl = max(rec_x_lo(rc.z) - tg.x0, 0), xh = min((rc.z >> 16) - tg.x0, T - 1);
        const int yl = max((rc.w & 0xffff) - tg.y0, 0), yh = min((rc.w >> 16) - tg.y0, T - 1);
        const uint32_t rect = rect_word<T>(xl, xh, yl, yh);
        s_a[k] = make_float4(ux, uy, ra.z, ra.w);
        s_b[k] = make_float4(rb.x, rb.y, rb.z, __uint_as_float(rect));
        uint32_t m = subblock_mask<SB>(xl, xh, yl, yh);
        uint32_t mc = m;
        if (MASKIO == 2) {
            m = gmask[b0 + k];
        } else if (CULL || DUAL) {
            const float thr = (lg_amin - rb.y) * 1.00001f + 1e-3f;   // log2(o / alpha_min) + margin
            // the edge minimisers' slopes, with approximate reciprocals: an
            // argmin off by a rounding error raises the minimum by a
            // second-order amount, far inside the margin of thr
            const float qa = ra.z, qb = ra.w, qc = rb.x;
            const float rx = qb * __builtin_amdgcn_rcpf(qa);
            const float ry = qa * qb * __builtin_amdgcn_rcpf(qb * qb + qc * qc);
            // pixel centres relative to the Gaussian centre; the box edges
            // clamp the rectangle's (offset once) to each sub-block's, which
            // rounds the same as offsetting the clamped integer (a rounded
            // sum is monotone in its operands)
            const float ox = (float)(tg.x0 - tg.rx) + 0.5f - ux;
            const float oy = (float)(tg.y0 - tg.ry) + 0.5f - uy;
            const float rxl = ox + (float)xl, rxh = ox + (float)xh;
            const float ryl = oy + (float)yl, ryh = oy + (float)yh;
            // A sub-block the rectangle touches has its edges on the right
            // sides of the rectangle's: each clamp is a median of three (for
            // the others the result is masked off).
            if constexpr (SB > 2) {   // 32 x 32 tiles: one box at a time (registers)
#pragma unroll
                for (int sb = 0; sb < SB * SB; ++sb) {
                    if (!((m >> sb) & 1u)) continue;
                    const int bx = (sb % SB) * 8, by = (sb / SB) * 8;
                    const float X0 = __builtin_amdgcn_fmed3f(rxl, ox + (float)bx, rxh);
                    const float X1 = __builtin_amdgcn_fmed3f(rxl, ox + (float)(bx + 7), rxh);
                    const float Y0 = __builtin_amdgcn_fmed3f(ryl, oy + (float)by, ryh);
                    const float Y1 = __builtin_amdgcn_fmed3f(ryl, oy + (float)(by + 7), ryh);
                    if (box_min_exponent(qa, qb, qc, rx, ry, X0, X1, Y0, Y1) > thr) mc &= ~(1u << sb);
                }
            } else {
            // the same minimum with everything that depends on one coordinate
            // only computed once per sub-block column (x) or row (y)
            float X0[SB], X1[SB], xn[SB], ryxn[SB], qaxn[SB];
            float Y0[SB], Y1[SB], yn[SB], rxyn[SB], qbyn[SB], e2s[SB];
#pragma unroll
            for (int c = 0; c < SB; ++c) {
                X0[c] = __builtin_amdgcn_fmed3f(rxl, ox + (float)(8 * c), rxh);
                X1[c] = __builtin_amdgcn_fmed3f(rxl, ox + (float)(8 * c + 7), rxh);
                xn[c] = __builtin_amdgcn_fmed3f(0.0f, X0[c], X1[c]);
                ryxn[c] = -ry * xn[c];
                qaxn[c] = qa * xn[c];
                Y0[c] = __builtin_amdgcn_fmed3f(ryl, oy + (float)(8 * c), ryh);
                Y1[c] = __builtin_amdgcn_fmed3f(ryl, oy + (float)(8 * c + 7), ryh);
                yn[c] = __builtin_amdgcn_fmed3f(0.0f, Y0[c], Y1[c]);
                rxyn[c] = -rx * yn[c];
                qbyn[c] = qb * yn[c];
                const float e2 = qc * yn[c];
                e2s[c] = e2 * e2;
            }
#pragma unroll
            for (int sb = 0; sb < SB * SB; ++sb) {
                const int c = sb % SB, r = sb / SB;
                // nearest point of the box to the centre along the edge x = x(y)
                // facing it, and along y = y(x)
                const float x = __builtin_amdgcn_fmed3f(rxyn[r], X0[c], X1[c]);
                const float e1 = fmaf(qa, x, qbyn[r]);
                const float E = fmaf(e1, e1, e2s[r]);
                const float y = __builtin_amdgcn_fmed3f(ryxn[c], Y0[r], Y1[r]);
                const float f1 = fmaf(qb, y, qaxn[c]), f2 = qc * y;
                const float F = fmaf(f1, f1, f2 * f2);
                if (fminf(E, F) > thr) mc &= ~(1u << sb);
            }
            }
            if (CULL) m = mc;
            if (DUAL) s_cmask[k] = (uint16_t)mc;
            if (MASKIO == 1) gmask[b0 + k] = (SubMask<T>)m;
        }
        s_mask[k] = (uint16_t)(T <= 16 && !(rc.z & kRecPlain) ? m | kMaskExact : m);
        if (s_rid) s_rid[4 * k] = (uint32_t)rid;   // 16-byte slots, like the records
        if (s_c) s_c[k] = rec.d;   // RGB colour of the view (comparison model)
    }
}

// Compacts, in list order, the staged entries [0, cnt) whose rectangle
// touches this wavefront's sub-block w into list[]; returns their number
// (wavefront-uniform).  An entry k is stored as 16 k, the byte offset of its
// slot in the float4 record arrays, and the blend loops read records without
// scaling the index.  The kListPad words after the last entry name the empty
// slot.  exact: one of the entries needs the rectangle test and the alpha
// clamp.
constexpr int kListPad = 8;
template <int B>
__device__ __forceinline__ int wave_list(const uint16_t *s_mask, int cnt, int w, uint32_t *list, bool &exact) {
    const int lane = lane_id();
    const uint64_t lt = (1ull << lane) - 1ull;
    int n = 0;
    uint64_t ex = 0;
    for (int c = 0; c < cnt; c += kWave) {
        const int k = c + lane;
        const uint32_t m = k < cnt ? s_mask[k] : 0u;
        const bool sel = (m >> w) & 1u;
        const uint64_t bal = __ballot(sel);
        ex |= __ballot(sel && (m & kMaskExact));
        if (sel) list[n + __popcll(bal & lt)] = 16u * (uint32_t)k;
        n += __popcll(bal);
    }
    if (lane < kListPad) list[n + lane] = 16u * B;
    exact = ex != 0;
    return n;
}

// Record slot at byte offset `off` (16 x its index) of a float4 array.
__device__ __forceinline__ float4 slot16(const float4 *base, uint32_t off) {
    return *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(base) + off);
}

// LDS of one blending workgroup (rid and wmax: the backward's;
// c holds the staged RGB colours of the CH = 3 forward, cmask the culled
// sub-block masks of the counting forward).
template <int T, int B, bool BWD = false, int CH = 1, bool CNT = false>
struct BlendLds {
    static constexpr int NW = T * T / kWave;
    // slot B is the empty one (empty_slot)
    float4 a[B + 1];
    float4 b[B + 1];
    float4 c[CH == 3 ? B + 1 : 1];
    uint32_t rid[BWD ? 4 * (B + 1) : 1];   // record index of entry k at rid[4 k] (read at the entry's byte offset)
    uint16_t mask[B];
    uint16_t cmask[CNT ? B + 1 : 1];
    alignas(16) uint32_t list[NW][B + kListPad];
    int wmax[NW];
    int next;
};

// The record that fills the blend loops' last group of entries: no pixel
// takes it.  Its exponent is NaN, so its alpha passes no comparison with
// alpha_min (0 included), and where the clamp would turn that into alpha_max,
// the rectangle covers no pixel.
template <int T, typename Lds>
__device__ __forceinline__ void empty_slot(Lds &sh, int B) {
    sh.a[B] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    sh.b[B] = make_float4(0.0f, __builtin_nanf(""), 0.0f, __uint_as_float(T <= 16 ? 0u : 255u));
}

// CH = 1: the radiative intensity of the record (Eq. 10).  CH = 3: the
// three colour channels of the record's fourth slot (the comparison model),
// image planar [3][total pixels]; the blending decisions are the same.
// COUNT: the work counts of xg_render_counts (rows documented there)
// instead of the image.  The walk then covers every list entry whose
// rectangle touches the wavefront's 8 x 8 block (the definition's
// evaluations); the culled mask tells which of them the blending kernels
// visit.
template <int T, int B, bool COUNT, bool STORE, int CH = 1>
__device__ __forceinline__ void fwd_tile(int tile, const Ws &ws, const xg_camera *cams,
                                         const Params &p, float *image, float *final_t,
                                         int32_t *n_contrib, int32_t *counts, const TStore &ts,
                                         const L1Fuse &l1, BlendLds<T, B, false, CH, COUNT> &sh) {
    static_assert(CH == 1 || (CH == 3 && !COUNT && !STORE), "RGB forward: plain variant only");
    constexpr int NT = T * T;
    constexpr int SB = T / 8;
    float4 *s_a = sh.a;
    float4 *s_b = sh.b;
    uint16_t *s_mask = sh.mask;

    const TileGeom tg = tile_geom(cams, ws.n_views, tile, T);
    const int w = threadIdx.x / kWave;
    const int lane = lane_id();
    const int sx = (w % SB) * 8, sy = (w / SB) * 8;
    const int lx = sx + (lane & 7), ly = sy + (lane >> 3);
    const int px = tg.x0 + lx, py = tg.y0 + ly;
    const bool inside = px < tg.W && py < tg.H;
    const float pxr = (float)(px - tg.rx) + 0.5f;
    const float pyr = (float)(py - tg.ry) + 0.5f;
    const uint32_t rkey = rect_lane_key<T>(lx, ly);

    const uint32_t s = ws.ranges[2 * (int64_t)tile];
    const uint32_t e = ws.ranges[2 * (int64_t)tile + 1];
    const uint32_t *vals = ws.pair_vals;
    const float amin = p.alpha_min, amax = p.alpha_max, tmin = p.t_min;
    const uint32_t *list = sh.list[w];

    float Tr = 1.0f, C = 0.0f, Cg = 0.0f, Cb = 0.0f;
    int last = 0;
    // counting variant: per lane (rows 0-2, 6, 7) and per wavefront (3-5)
    int n_eval = 0, n_con = 0, n_upto = 0, n_fev = 0, n_bev = 0, bev_run = 0;
    int w_red = 0, w_bvis = 0, w_fvis = 0, w_cvis = 0;
    if (threadIdx.x == 0) {
        empty_slot<T>(sh, B);
        if (COUNT) sh.cmask[B] = 0;
    }
    uint64_t live = __ballot(inside);   // lanes that have not terminated
    int nc = 0;   // contributors so far (stored variant)
    float *tbase = STORE ? ts.t + (int64_t)tile * ts.slots * NT + threadIdx.x : nullptr;
    for (uint32_t b0 = s; b0 < e; b0 += B) {
        const int cnt = (int)min((uint32_t)B, e - b0);
        if (!__syncthreads_or(live != 0)) break;
        // the counting variant keeps every rectangle evaluation (the work
        // count of the definition), the others skip sub-blocks out of reach
        stage<T, NT, !COUNT, COUNT, (COUNT || CH == 3) ? 0 : 1>(ws, vals, b0, cnt, tg, amin, s_a, s_b, s_mask, nullptr,
                                    CH == 3 ? sh.c : nullptr, COUNT ? sh.cmask : nullptr);
        __syncthreads();
        if (live == 0) continue;
        bool exact;
        const int nl = wave_list<B>(s_mask, cnt, w, sh.list[w], exact);
        exact = exact || T > 16 || COUNT;
        int lk = -1;   // 16 x batch index of this lane's last contributor in the batch
        // the entry at byte offset `off` (16 x its batch index) of the record
        // arrays, with its evaluation and its colour; inr: the lanes whose
        // pixel the rectangle holds
        auto composite = [&](uint32_t off, uint64_t inr, const Eval &ev, float c0, float c1, float c2) {
            const uint64_t act_m = live & inr;
            const bool any_live = live != 0;   // before this entry
            const uint64_t con = act_m & __ballot(ev.alpha >= amin);
            const float Tn = fmaf(-Tr, ev.alpha, Tr);   // T (1 - alpha), one rounding
            const uint64_t keep_m = con & __ballot(!(Tn < tmin));
            const bool keep = __builtin_amdgcn_inverse_ballot_w64(keep_m);
            live &= ~(con ^ keep_m);   // con without keep: the lane terminates
            if (STORE) {
                if (keep && nc < ts.slots) tbase[(int64_t)nc * NT] = Tr;
                nc += keep ? 1 : 0;
            }
            if constexpr (CH == 3) {
                C = keep ? fmaf(c0 * ev.alpha, Tr, C) : C;
                Cg = keep ? fmaf(c1 * ev.alpha, Tr, Cg) : Cg;
                Cb = keep ? fmaf(c2 * ev.alpha, Tr, Cb) : Cb;
            } else {
                C = keep ? fmaf(c0 * ev.alpha, Tr, C) : C;
            }
            Tr = keep ? Tn : Tr;
            lk = keep ? (int)off : lk;
            if (COUNT) {
                const bool act = __builtin_amdgcn_inverse_ballot_w64(act_m);
                n_eval += act ? 1 : 0;
                n_con += keep ? 1 : 0;
                n_upto = keep ? n_eval : n_upto;
                const bool any_keep = __any(keep);
                w_red += any_keep ? 1 : 0;
                if ((sh.cmask[off >> 4] >> w) & 1u) {   // an entry the blend kernels visit
                    ++w_cvis;
                    if (any_live) {
                        ++w_fvis;
                        n_fev += act ? 1 : 0;
                    }
                    bev_run += __builtin_amdgcn_inverse_ballot_w64(inr) ? 1 : 0;
                    if (any_keep) w_bvis = w_cvis;
                    n_bev = keep ? bev_run : n_bev;
                }
            }
        };
        // plain: every record of the wavefront's list is marked kRecPlain, so
        // the rectangle test and the clamp change nothing
        auto walk = [&](auto plain) {
            constexpr bool PLAIN = decltype(plain)::value;
            auto covers = [&](const float4 &sb) {
                return PLAIN ? ~0ull : __ballot(in_rect<T>(__float_as_uint(sb.w), rkey, lx, ly));
            };
            // Groups of 4 entries, their offsets in one 16-byte read, the last
            // group filled up with the empty slot (no test between entries);
            // the wavefront leaves the batch after a group once all its lanes
            // have terminated.  Each entry's record is loaded one entry ahead
            // of its use, also from one group to the next (the read after the
            // last group stays in the row's padding; the barrier keeps the
            // scheduler from moving the loads back down).  A visit is 16 VALU
            // instructions and, the lane masks being kept as scalar words
            // rather than lane booleans, 4 scalar ones; with 16-bit offsets to
            // unpack, a tested partial group and booleans it was 17 and 5.  A
            // wavefront alone on its SIMD issues an instruction every 6 cycles
            // or so and gains most.  Measured (with the same groups in the
            // backward): one view of 50k Gaussians at 256 x 256, a step 168 ->
            // 159 us; 1M x 16 views 2.29 -> 2.25 ms; ACUI scan of 100 views 1.35 ->
            // 1.32 ms; three channels, 200k x 4 views 220 -> 215 us.  Computing
            // the next entry's alpha beside the current entry's update, to
            // hide the exponential's latency, gained nothing.
            if (nl == 0) return;
            uint4 q = *reinterpret_cast<const uint4 *>(list);
            float4 sa_n = slot16(s_a, q.x), sb_n = slot16(s_b, q.x);
            auto group = [&](const uint4 &g, uint32_t next) {
                const uint32_t off[5] = {g.x, g.y, g.z, g.w, next};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 sa = sa_n, sb = sb_n;
                    sa_n = slot16(s_a, off[u + 1]);
                    sb_n = slot16(s_b, off[u + 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    const float4 sc = CH == 3 ? slot16(sh.c, off[u]) : make_float4(sb.z, 0.0f, 0.0f, 0.0f);
                    composite(off[u], covers(sb), splat_eval<PLAIN>(sa, sb, pxr, pyr, amax), sc.x, sc.y, sc.z);
                }
            };
            for (int j0 = 4;; j0 += 8) {
                const uint4 q1 = *reinterpret_cast<const uint4 *>(list + j0);
                group(q, q1.x);
                if (j0 >= nl || live == 0) break;
                q = *reinterpret_cast<const uint4 *>(list + j0 + 4);
                group(q1, q.x);
                if (j0 + 4 >= nl || live == 0) break;
            }
        };
        if (exact)
            walk(std::false_type{});
        else if constexpr (T <= 16 && !COUNT)
            walk(std::true_type{});
        if (lk >= 0) last = (int)(b0 - s) + (lk >> 4) + 1;
    }
    if (STORE) ts.count[(int64_t)tile * NT + threadIdx.x] = nc;
    if (inside) {
        const int64_t o = (int64_t)tg.pix_off + (int64_t)py * tg.W + px;
        if (COUNT) {
            const int64_t tp = ws.total_pixels;
            const bool first = lane == 0;   // the block's first pixel
            counts[o] = n_eval;
            counts[tp + o] = n_con;
            counts[2 * tp + o] = n_upto;
            counts[3 * tp + o] = first ? w_red : 0;
            counts[4 * tp + o] = first ? w_bvis : 0;
            counts[5 * tp + o] = first ? w_fvis : 0;
            counts[6 * tp + o] = n_fev;
            counts[7 * tp + o] = n_bev;
        } else {
            image[o] = C;
            if constexpr (CH == 3) {
                image[ws.total_pixels + o] = Cg;
                image[2 * ws.total_pixels + o] = Cb;
            }
            final_t[o] = Tr;
            n_contrib[o] = last;
            if (l1.dl) {
                const float d = C - l1.target[o];
                l1.dl[o] = d > 0.0f ? l1.scale : (d < 0.0f ? -l1.scale : 0.0f);
            }
        }
    }
}

// Pops the next tile of the heavy-first work order (-1 when exhausted).
template <typename Lds>
__device__ __forceinline__ int pop_tile(const Ws &ws, int32_t *queue, Lds &sh) {
    if (threadIdx.x == 0) {
        const int q = atomicAdd(queue, 1);
        sh.next = q < ws.total_tiles ? ws.tile_order[q] : -1;
    }
    __syncthreads();
    const int t = sh.next;
    __syncthreads();
    return t;
}

// The last workgroup of a persistent launch to finish rewinds the queue, so
// the next launch on this workspace starts from the first tile again.
__device__ __forceinline__ void finish_queue(int32_t *queue, int32_t *done) {
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(done, 1) == (int)gridDim.x - 1) {
            atomicExch(queue, 0);
            atomicExch(done, 0);
        }
    }
}

// COUNT = true: instead of the image, write the per-pixel work counts
// (evaluations, contributors, evaluations up to the last contributor) into
// counts[3][total pixels]; the blending decisions are the same.
// PERSIST = true: a grid sized to the device's resident capacity takes
// tiles from the work queue; otherwise one workgroup per tile.
// STORE = true: also keep the transmittance before each of the first
// ts.slots contributors of every pixel (one workgroup per tile only).
// (64 registers for all variants of several wavefronts but the persistent
// ones: as for the backward below)
template <int T, int B, bool COUNT, bool PERSIST, bool STORE>
__global__ __launch_bounds__(T * T, T > 8 && !PERSIST ? 8 : 2) void k_render_fwd(Ws ws, const xg_camera *cams, Params p,
                                                      float *image, float *final_t,
                                                      int32_t *n_contrib, int32_t *counts,
                                                      TStore ts, L1Fuse l1) {
    __shared__ BlendLds<T, B, false, 1, COUNT> sh;
    if (!PERSIST) {
        fwd_tile<T, B, COUNT, STORE>(ordered_tile(ws.blend_order, blockIdx.x, (int)ws.total_tiles), ws, cams, p, image,
                                     final_t, n_contrib, counts, ts, l1, sh);
        return;
    }
    for (;;) {
        const int tile = pop_tile(ws, &ws.hdr->queue_fwd, sh);
        if (tile < 0) break;
        fwd_tile<T, B, COUNT, false>(tile, ws, cams, p, image, final_t, n_contrib, counts, ts, l1, sh);
    }
    finish_queue(&ws.hdr->queue_fwd, &ws.hdr->done_fwd);
}

// Forward of the comparison model: three colour channels per pixel, one
// workgroup per tile.
template <int T, int B>
__global__ __launch_bounds__(T * T, T > 8 ? 8 : 2) void k_render_fwd_rgb(Ws ws, const xg_camera *cams, Params p,
                                                          float *image, float *final_t,
                                                          int32_t *n_contrib) {
    __shared__ BlendLds<T, B, false, 3> sh;
    fwd_tile<T, B, false, false, 3>(ordered_tile(ws.blend_order, blockIdx.x, (int)ws.total_tiles), ws, cams, p, image,
                                    final_t, n_contrib, nullptr, TStore{nullptr, nullptr, 0},
                                    L1Fuse{nullptr, nullptr, 0.0f}, sh);
}

// DPP lane permutations (row = 16 lanes): quad xor 1, quad xor 2, lane
// i^8 within a row (rotate by 8), and mirror within each half row.  Every
// permutation reads a lane of the same row and all lanes are active, so the
// bound control (a lane with no source reads 0) never applies; it spares
// the compiler materialising the old value.
#define XG_DPP(x, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, true))
constexpr int kDppQuadXor1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int kDppRowRor8 = 0x128;   // row_ror:8
constexpr int kDppHalfMirror = 0x141; // row_half_mirror

// Sums over a wavefront's 8 x 8 pixels of the 7 gradient terms of 4 list
// entries.  The terms are gp dx^a dy^b (a + b <= 2) and w, and dy depends
// on the pixel row only, so the rows are summed first: 4 values per entry
// (gp, gp dy, gp dy^2, w) over lane bits 5-3, then the row sums times 1, dx,
// dx^2 over lane bits 2-0.  Both are reduce-scatters, which halve the live
// values at every step; bits 5 and 4 swap wavefront halves and rows (gfx950
// permlane swaps: one swap and one add per pair of values), the others read
// a partner lane through DPP (two selects and one add per pair).  All VALU,
// no LDS traffic.  The kernel issues VALU most of its cycles, so what counts
// is instructions: 13 an entry here with the moment products, where forming
// all 7 terms per pixel and summing two entries together took 21.  200k
// Gaussians x 8 views of 512 x 512: backward 257 -> 207 us; one such view
// 81 -> 56 us (with the tiles dealt to the XCDs by work).
//
// row_sums: acc[e][q] of entry e -> c[0], c[1] at lane 16 e + 8 h + x:
// (sum gp, sum gp dy^2) for h = 0, (sum gp dy, sum w) for h = 1, of column x.
// 30 instructions; an entry's sums depend on its own values alone.
__device__ __forceinline__ void row_sums(const float (&acc)[4][4], int lane, float (&c)[2]) {
    float b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float a[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[e][q]), __float_as_uint(acc[e + 2][q]),
                                                            false, false);
            a[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[0]), __float_as_uint(a[1]), false, false);
        b[q] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const bool h = lane & 8;
    c[0] = (h ? b[1] : b[0]) + XG_DPP(h ? b[0] : b[1], kDppRowRor8);
    c[1] = (h ? b[3] : b[2]) + XG_DPP(h ? b[2] : b[3], kDppRowRor8);
}

// column_sums: value v of (c0, c0 dx, c0 dx^2, c1) summed over the columns
// at the lanes of bits 2-1 = v.
__device__ __forceinline__ float column_sums(const float (&c)[2], float dx, int lane) {
    const float m1 = c[0] * dx, m2 = m1 * dx;
    const bool h2 = lane & 4, h1 = lane & 2;
    const float d0 = (h2 ? m2 : c[0]) + XG_DPP(h2 ? c[0] : m2, kDppHalfMirror);
    const float d1 = (h2 ? c[1] : m1) + XG_DPP(h2 ? m1 : c[1], kDppHalfMirror);
    float x = (h1 ? d1 : d0) + XG_DPP(h1 ? d0 : d1, kDppQuadXor2);
    x += XG_DPP(x, kDppQuadXor1);
    return x;
}

// List entries whose gradient terms are summed over the wavefront together,
// entry e's sums ending in its row of 16 lanes.
constexpr int kBwdGroup = 4;

// Gradient word (of the 8 per (view, Gaussian)) that a lane's sum adds to;
// -1: none (the upper lane of a pair, and the column sum of gp dx^2 dy).
__device__ __forceinline__ int sum_word(int lane) {
    if (lane & 1) return -1;
    const int v = (lane >> 1) & 3;
    if (lane & 8) return v == 0 ? 1 : v == 1 ? 3 : v == 3 ? 6 : -1;
    return v == 0 ? 5 : v == 1 ? 0 : v == 2 ? 2 : 4;
}

template <int T, int B, bool STORE>
__device__ __forceinline__ void bwd_tile(int tile, const Ws &ws, const xg_camera *cams,
                                         const Params &p, const float *dl_dimage,
                                         const float *final_t, const int32_t *n_contrib,
                                         const TStore &ts, BlendLds<T, B, true> &sh) {
    constexpr int NT = T * T;
    constexpr int NW = NT / kWave;
    constexpr int SB = T / 8;
    float4 *s_a = sh.a;
    float4 *s_b = sh.b;
    uint32_t *s_rid = sh.rid;
    uint16_t *s_mask = sh.mask;
    int *s_max = sh.wmax;

    const TileGeom tg = tile_geom(cams, ws.n_views, tile, T);
    const int w = threadIdx.x / kWave;
    const int lane = lane_id();
    const int sx = (w % SB) * 8, sy = (w / SB) * 8;
    const int lx = sx + (lane & 7), ly = sy + (lane >> 3);
    const int px = tg.x0 + lx, py = tg.y0 + ly;
    const bool inside = px < tg.W && py < tg.H;
    const float pxr = (float)(px - tg.rx) + 0.5f;
    const float pyr = (float)(py - tg.ry) + 0.5f;
    const uint32_t rkey = rect_lane_key<T>(lx, ly);

    const uint32_t s = ws.ranges[2 * (int64_t)tile];
    const uint32_t *vals = ws.pair_vals;
    const float amin = p.alpha_min, amax = p.alpha_max;
    const uint32_t *list = sh.list[w];

    float g = 0.0f, Tr = 1.0f;
    int last = 0;
    if (inside) {
        const int64_t o = (int64_t)tg.pix_off + (int64_t)py * tg.W + px;
        g = dl_dimage[o];
        Tr = final_t[o];
        last = n_contrib[o];
        if (g == 0.0f) last = 0;
    }
    // stored variant: index of the next contributor (counting down) and its
    // stored transmittance, loaded one contributor ahead of its use;
    // contributors past the stored slots divide the transmittance back
    int c = -1;
    float tnext = 0.0f;
    const float *tbase = STORE ? ts.t + (int64_t)tile * ts.slots * NT + threadIdx.x : nullptr;
    if (STORE) {
        c = ts.count[(int64_t)tile * NT + threadIdx.x] - 1;
        if (c >= 0 && c < ts.slots) tnext = tbase[(int64_t)c * NT];
    }
    int wmax = last;
    for (int off = kWave / 2; off > 0; off >>= 1) wmax = max(wmax, __shfl_xor(wmax, off, kWave));
    if (lane == 0) s_max[w] = wmax;
    if (threadIdx.x == 0) empty_slot<T>(sh, B);
    __syncthreads();
    int bmax = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) bmax = max(bmax, s_max[k]);
    wmax = __builtin_amdgcn_readfirstlane(wmax);

    float R = 0.0f;   // intensity behind, seen from just after the current Gaussian
    // the lane's share of a group's sums: its entry (its row of 16 lanes) and
    // the gradient word it adds to
    constexpr int G = kBwdGroup;
    static_assert(G == kWave / 16, "one row of lanes per entry");
    const int lane_e = lane >> 4;
    const int lane_q = sum_word(lane);
    const uint32_t lane_q4 = 4u * (uint32_t)lane_q;
    const uint32_t lane_bit = lane_q < 0 ? 0u : 1u << lane_e;   // tested against the live entries
    const bool small_rid = ws.n_items < (int64_t)1 << 27;   // 32 B x records below 4 GiB
    for (int end = bmax; end > 0; end -= B) {
        const int b0 = max(end - B, 0);
        const int cnt = end - b0;
        __syncthreads();
        stage<T, NT, true, false, 2>(ws, vals, s + (uint32_t)b0, cnt, tg, amin, s_a, s_b, s_mask, s_rid);
        __syncthreads();
        if (b0 >= wmax) continue;
        bool exact;
        const int nl = wave_list<B>(s_mask, min(cnt, wmax - b0), w, sh.list[w], exact);
        // 16 x batch index of this lane's last contributor (-16: none in the batch)
        const int lastk16 = 16 * max(last - b0 - 1, -1);
        // (plain: as in the forward)
        auto walk = [&](auto plain) {
            constexpr bool PLAIN = decltype(plain)::value;
            // groups of G entries from the back, each group's offsets in one
            // 16-byte read; the last is filled up with the empty slot.  Each
            // entry's record is loaded one entry ahead of its use.
            if (nl == 0) return;
            int j0 = (nl - 1) & ~(G - 1);
            uint4 q = *reinterpret_cast<const uint4 *>(list + j0);
            float4 sa_n = slot16(s_a, q.w), sb_n = slot16(s_b, q.w);
            for (;;) {
              const uint32_t eoff = list[j0 + lane_e];   // the group's entry of this lane, for the sums
              const int jn = j0 - G;
              const uint4 qn = *reinterpret_cast<const uint4 *>(list + max(jn, 0));
              const uint32_t offs[G] = {q.x, q.y, q.z, q.w};
              uint32_t live = 0;   // entries of the group that some lane contributes to (bit e)
              float acc[G][4];     // gp, gp dy, gp dy^2 and w of the group's entries
#pragma unroll
              for (int e = G - 1; e >= 0; --e) {
                const uint32_t off = offs[e];   // 16 x batch index
                const float4 sa = sa_n;
                const float4 sb = sb_n;
                const uint32_t off_n = e > 0 ? offs[e - 1] : qn.w;
                sa_n = slot16(s_a, off_n);
                sb_n = slot16(s_b, off_n);
                const bool inr = (int)off <= lastk16 && (PLAIN || in_rect<T>(__float_as_uint(sb.w), rkey, lx, ly));
                const Eval ev = splat_eval<PLAIN>(sa, sb, pxr, pyr, amax);
                const bool act = inr && ev.alpha >= amin;
                if (__any(act)) {
                    // Every lane runs the same arithmetic; a lane that is not a
                    // contributor adds exact zeros to the sums (its alpha
                    // taken as 0, its alpha gradient masked) and keeps its
                    // transmittance and R.
                    const float aact = act ? ev.alpha : 0.0f;
                    float gT;   // dL/dI times T before this Gaussian
                    if (STORE) {
                        const float om = 1.0f - ev.alpha;
                        const float Tj = act ? (c < ts.slots ? tnext : Tr * __builtin_amdgcn_rcpf(om)) : Tr;
                        const int cn = act ? c - 1 : c;
                        if (act && cn >= 0 && cn < ts.slots) tnext = tbase[(int64_t)cn * NT];
                        c = cn;
                        Tr = Tj;
                        gT = g * Tj;
                    } else {
                        // T before this Gaussian = T after it / (1 - alpha); a
                        // lane that is not a contributor divides by 1 - 0 (the
                        // reciprocal of 1 is exact) and keeps its T.  T itself is
                        // carried, not dL/dI x T: T stays a normal float down to
                        // t_min, a product with a small dL/dI might not.
                        const float Tj = Tr * __builtin_amdgcn_rcpf(1.0f - aact);
                        Tr = Tj;
                        gT = g * Tj;
                    }
                    const float it = sb.z;
                    const float wi = gT * aact;                    // dL/d intensity
                    const float dR = it - R;
                    const float galpha = gT * dR;                  // dL/d alpha
                    // R after this Gaussian: i alpha + (1 - alpha) R
                    R = fmaf(aact, dR, R);
                    // no alpha gradient through the clamp, nor for a lane that is
                    // not a contributor
                    const float ga = act && (PLAIN || ev.a <= amax) ? galpha : 0.0f;
                    // dL/d power, power = -d^T Q d / 2.  Its sum is the opacity
                    // times dL/d opacity (a = o G); its moments over the pixel
                    // offsets d = pixel - u give the gradients of u and Sigma''
                    // (the inverse covariance is applied once per (view, Gaussian))
                    const float gp = ga * ev.a;
                    acc[e][0] = gp;
                    acc[e][1] = gp * ev.dy;
                    acc[e][2] = acc[e][1] * ev.dy;
                    acc[e][3] = wi;
                    live |= 1u << e;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[e][q] = 0.0f;
                }
              }
              if (live != 0) {
                const float eux = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(s_a) + eoff);
                const uint32_t rid = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(s_rid) + eoff);
                float c2[2];
                row_sums(acc, lane, c2);
                const float x = column_sums(c2, pxr - eux, lane);
                if (live & lane_bit) {
                    if (small_rid) {   // 32-bit byte offset from the array base
                        atomicAdd(reinterpret_cast<float *>(reinterpret_cast<char *>(ws.grad2d) + (rid << 5 | lane_q4)), x);
                    } else {
                        atomicAdd(ws.grad2d + 8 * (int64_t)rid + lane_q, x);
                        __asm__ volatile("" ::: "memory");   // keeps the two atomics apart
                    }
                }
              }
              if (jn < 0) break;
              j0 = jn;
              q = qn;
            }
        };
        if (exact || T > 16)
            walk(std::false_type{});
        else if constexpr (T <= 16)
            walk(std::true_type{});
    }
}

// (64 registers for the plain variants of several wavefronts: 8 wavefronts
// per SIMD, and two workgroups per CU of 32 x 32 tiles.  The stored variant
// of 32 x 32 tiles too, for the same reason: with 72 registers one workgroup
// to a CU, 200k Gaussians x 8 views of 512 x 512 forward 421 us and backward
// 887 where two take 301 and 632, four spilled registers included.  At 16 x 16
// a workgroup is 4 wavefronts and 70 registers cost nothing: 442 and 441.)
template <int T, int B, bool PERSIST, bool STORE>
__global__ __launch_bounds__(T * T, T > 8 && !PERSIST && (T > 16 || !STORE) ? 8 : 2) void k_render_bwd(Ws ws, const xg_camera *cams, Params p,
                                                      const float *dl_dimage, const float *final_t,
                                                      const int32_t *n_contrib, TStore ts) {
    __shared__ BlendLds<T, B, true> sh;
    if (!PERSIST) {
        bwd_tile<T, B, STORE>(ordered_tile(ws.blend_order, blockIdx.x, (int)ws.total_tiles), ws, cams, p, dl_dimage,
                              final_t, n_contrib, ts, sh);
        return;
    }
    for (;;) {
        const int tile = pop_tile(ws, &ws.hdr->queue_bwd, sh);
        if (tile < 0) break;
        bwd_tile<T, B, false>(tile, ws, cams, p, dl_dimage, final_t, n_contrib, ts, sh);
        __syncthreads();
    }
    finish_queue(&ws.hdr->queue_bwd, &ws.hdr->done_bwd);
}

// Workgroups of `kernel` that fit on the device at once (persistent grid).
template <typename K>
unsigned resident_grid(K kernel, int threads, int64_t work) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) return 0;
    int64_t g = (int64_t)cus * (per_cu > 0 ? per_cu : 1);
    if (g > work) g = work;
    return (unsigned)(g > 0 ? g : 1);
}

template <int T, int B>
hipError_t fwd_t(const Ws &ws, const xg_camera *cams, const Params &p, float *image, float *final_t,
                 int32_t *n_contrib, int persistent, const TStore &ts, const L1Fuse &l1, hipStream_t st) {
    const unsigned nb = (unsigned)(ws.total_tiles > 0 ? ws.total_tiles : 1);
    if (ts.t) {
        if (persistent) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_render_fwd<T, B, false, false, true>), dim3(nb), dim3(T * T), 0, st, ws,
                           cams, p, image, final_t, n_contrib, nullptr, ts, l1);
    } else if (persistent) {
        const unsigned g = resident_grid(k_render_fwd<T, B, false, true, false>, T * T, ws.total_tiles);
        if (g == 0) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_render_fwd<T, B, false, true, false>), dim3(g), dim3(T * T), 0, st, ws,
                           cams, p, image, final_t, n_contrib, nullptr, ts, l1);
    } else {
        hipLaunchKernelGGL((k_render_fwd<T, B, false, false, false>), dim3(nb), dim3(T * T), 0, st, ws,
                           cams, p, image, final_t, n_contrib, nullptr, ts, l1);
    }
    return hipGetLastError();
}

template <int T, int B>
hipError_t fwd_rgb_t(const Ws &ws, const xg_camera *cams, const Params &p, float *image,
                     float *final_t, int32_t *n_contrib, hipStream_t st) {
    const unsigned nb = (unsigned)(ws.total_tiles > 0 ? ws.total_tiles : 1);
    hipLaunchKernelGGL((k_render_fwd_rgb<T, B>), dim3(nb), dim3(T * T), 0, st, ws, cams, p, image,
                       final_t, n_contrib);
    return hipGetLastError();
}

template <int T, int B>
hipError_t counts_t(const Ws &ws, const xg_camera *cams, const Params &p, int32_t *counts,
                    hipStream_t st) {
    const unsigned nb = (unsigned)(ws.total_tiles > 0 ? ws.total_tiles : 1);
    hipLaunchKernelGGL((k_render_fwd<T, B, true, false, false>), dim3(nb), dim3(T * T), 0, st, ws,
                       cams, p, nullptr, nullptr, nullptr, counts, TStore{nullptr, nullptr, 0},
                       L1Fuse{nullptr, nullptr, 0.0f});
    return hipGetLastError();
}

template <int T, int B>
hipError_t bwd_t(const Ws &ws, const xg_camera *cams, const Params &p, const float *dl,
                 const float *final_t, const int32_t *n_contrib, int persistent, const TStore &ts,
                 hipStream_t st) {
    const unsigned nb = (unsigned)(ws.total_tiles > 0 ? ws.total_tiles : 1);
    if (ts.t) {
        if (persistent) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_render_bwd<T, B, false, true>), dim3(nb), dim3(T * T), 0, st, ws, cams,
                           p, dl, final_t, n_contrib, ts);
    } else if (persistent) {
        const unsigned g = resident_grid(k_render_bwd<T, B, true, false>, T * T, ws.total_tiles);
        if (g == 0) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_render_bwd<T, B, true, false>), dim3(g), dim3(T * T), 0, st, ws, cams, p,
                           dl, final_t, n_contrib, ts);
    } else {
        hipLaunchKernelGGL((k_render_bwd<T, B, false, false>), dim3(nb), dim3(T * T), 0, st, ws, cams,
                           p, dl, final_t, n_contrib, ts);
    }
    return hipGetLastError();
}

}  // namespace

#define XG_DISPATCH(FN, ...)                                                   \
    switch (p.tile * 1000 + p.lds_batch) {                                     \
        case 8064: return FN<8, 64>(__VA_ARGS__);                              \
        case 8128: return FN<8, 128>(__VA_ARGS__);                             \
        case 8256: return FN<8, 256>(__VA_ARGS__);                             \
        case 16064: return FN<16, 64>(__VA_ARGS__);                            \
        case 16128: return FN<16, 128>(__VA_ARGS__);                           \
        case 16256: return FN<16, 256>(__VA_ARGS__);                           \
        case 32064: return FN<32, 64>(__VA_ARGS__);                            \
        case 32128: return FN<32, 128>(__VA_ARGS__);                           \
        case 32256: return FN<32, 256>(__VA_ARGS__);                           \
        default: return hipErrorInvalidValue;                                  \
    }

hipError_t launch_render_fwd(const Ws &ws, const xg_camera *cams, const Params &p, float *image,
                             float *final_t, int32_t *n_contrib, int persistent, const TStore &ts,
                             const L1Fuse &l1, hipStream_t s) {
    XG_DISPATCH(fwd_t, ws, cams, p, image, final_t, n_contrib, persistent, ts, l1, s)
}

hipError_t launch_render_fwd_rgb(const Ws &ws, const xg_camera *cams, const Params &p, float *image,
                                 float *final_t, int32_t *n_contrib, hipStream_t s) {
    XG_DISPATCH(fwd_rgb_t, ws, cams, p, image, final_t, n_contrib, s)
}

hipError_t launch_render_bwd(const Ws &ws, const xg_camera *cams, const Params &p,
                             const float *dl_dimage, const float *final_t,
                             const int32_t *n_contrib, int persistent, const TStore &ts,
                             hipStream_t s) {
    XG_DISPATCH(bwd_t, ws, cams, p, dl_dimage, final_t, n_contrib, persistent, ts, s)
}

hipError_t launch_render_counts(const Ws &ws, const xg_camera *cams, const Params &p,
                                int32_t *counts, hipStream_t s) {
    XG_DISPATCH(counts_t, ws, cams, p, counts, s)
}

}  // namespace xg
