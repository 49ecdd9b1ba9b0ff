// Hybrid binning and compositing for scenes with screen-covering splats.
//
// A record whose tile footprint exceeds a per-view threshold ("wide") is not
// duplicated into every tile it covers but into every region (REGION x
// REGION tiles) its footprint overlaps; the remaining ("narrow") records are
// duplicated per tile.  Both kinds of entry share one key space (tile ids,
// then region ids) and one stable sort, so each tile and each region holds
// its entries in (depth, record) order.  A tile's list in the sense of
// Sec. 3.1 -- every record whose footprint covers the tile, in depth order --
// is then the merge of the tile's narrow entries with the entries of its
// region whose rectangle contains the tile.  The compositing kernels form
// that merged list batch by batch in LDS (merge path over two ordered
// windows), so the entries, their order and the per-pixel results are
// exactly those of fully duplicated lists, while the instance sort shrinks
// from every (tile, wide splat) pair to one entry per region.
//
// With culling, an entry is kept only where the splat can pass the per-pixel
// filters at some pixel centre of the cell (exact test, conservative
// margin): narrow entries per tile at duplication, wide entries per region
// at duplication and per tile before the merge.  Dropped entries contribute
// nothing to any pixel; the merged lists are shorter, the results the same.
//
// Records are copied once into (view, depth, record) order ("sorted
// records"); list entries hold positions in that order, which are unique and
// order exactly as (depth, record) within a view, so the merge compares plain
// 32-bit positions and the record gathers of a tile walk memory upwards.
//
// The forward records, per tile and batch, the stream cursors where the batch
// began; the backward replays the same batches in reverse from those
// checkpoints, so the merge is deterministic and nothing per pixel beyond the
// final transmittance and the last blended entry is stored.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "composite_common.hpp"
#include "kernels.hpp"
#include "staged.hpp"

namespace mgs {
namespace {

// The tile's pixel centres span [X0, X1] x [Y0, Y1].
struct TileBox {
    float X0, X1, Y0, Y1;
};

// Whether an entry can pass the per-pixel filters (Q <= q_max and
// alpha >= alpha_min) at any pixel centre of the tile: the minimum of its
// quadratic form over the box (zero if the centre is inside, else the
// smallest of the clamped minima along the four edges) against the cut
// min(q_max, 2 ln(opacity / alpha_min)).  The test is conservative (a small
// margin over the cut), so an entry it drops contributes nothing to any
// pixel of the tile in the forward or the backward pass; dropping it leaves
// every result unchanged.
struct TouchPrep {
    float u, v, a, beta, gamma;
    float nbc;       // -b / c: minimiser along a vertical edge (-beta along a horizontal one)
    float cut;       // +huge: no cut (always touches); < 0: reaches no pixel
};

// Every operation below is written out (fmaf where a fused product is meant)
// and contraction is off, so the rounding of each step is fixed by the
// source: the binning kernels inline the test and still take identical
// decisions for the same record and cell.
__device__ __forceinline__ TouchPrep touch_prep(const float4& A, const float4& B, float q_max, float alpha_min) {
#pragma clang fp contract(off)
    TouchPrep p;
    p.u = A.x;
    p.v = A.y;
    p.a = A.z;
    p.beta = A.w;
    p.gamma = B.x;
    // -b / c = -a beta / (a beta^2 + gamma); a reciprocal approximation only
    // moves the edge minimiser slightly, which raises the computed minimum by
    // a second-order amount far inside the margin below
    const float ab = p.a * p.beta;
    p.nbc = -ab * __builtin_amdgcn_rcpf(fmaf(ab, p.beta, p.gamma));
    float cut = q_max;
    if (alpha_min > 0.f) cut = fminf(cut, 2.f * __logf(B.y / alpha_min));
    if (cut >= 3.0e38f) p.cut = 3.4e38f;          // no finite cut
    else if (!(cut > -3.0e38f)) p.cut = -1.f;     // zero opacity
    else p.cut = fmaf(1e-3f, 1.f + fabsf(cut), cut);
    return p;
}

__device__ __forceinline__ TouchPrep touch_prep(const float4& A, const float4& B, const DevSettings& st) {
    return touch_prep(A, B, st.q_max, st.alpha_min);
}

// a (dx + beta dy)^2 + gamma dy^2
__device__ __forceinline__ float touch_q(const TouchPrep& p, float dx, float dy) {
#pragma clang fp contract(off)
    const float t = fmaf(p.beta, dy, dx);
    const float at = p.a * t;
    const float gdy = p.gamma * dy;
    return fmaf(at, t, gdy * dy);
}

__device__ __forceinline__ bool touch_test(const TouchPrep& p, const TileBox& tb) {
#pragma clang fp contract(off)
    if (p.cut >= 3.0e38f) return true;  // no cut (exact mode)
    if (p.cut < 0.f) return false;
    if (p.u >= tb.X0 && p.u <= tb.X1 && p.v >= tb.Y0 && p.v <= tb.Y1) return true;
    const float dyl = p.v - tb.Y1, dyh = p.v - tb.Y0, dxl = p.u - tb.X1, dxh = p.u - tb.X0;
    // along the vertical edges dy minimises at -b/c dx, along the horizontal
    // ones dx at -beta dy, each clamped to the edge
    float q = touch_q(p, dxh, fminf(fmaxf(p.nbc * dxh, dyl), dyh));
    q = fminf(q, touch_q(p, dxl, fminf(fmaxf(p.nbc * dxl, dyl), dyh)));
    q = fminf(q, touch_q(p, fminf(fmaxf(-p.beta * dyh, dxl), dxh), dyh));
    q = fminf(q, touch_q(p, fminf(fmaxf(-p.beta * dyl, dxl), dxh), dyl));
    return q <= p.cut;
}

__device__ __forceinline__ bool may_touch(const float4& A, const float4& B, const TileBox& tb,
                                          const DevSettings& st) {
    return touch_test(touch_prep(A, B, st), tb);
}

// ---------------------------------------------------------------------------
// binning: (view, depth) order of records, sorted records, per-tile and
// per-region lists, batch checkpoints
// ---------------------------------------------------------------------------

// Depth keys of the records, sorted per view (the records of view v are the
// segment [v n, (v + 1) n)): the float bits of the view-space depth (positive,
// so the bits order like the values), all ones for a record without tiles,
// which sorts it after every listed record of its view.
// The cells a record is listed in: the tiles of its rectangle for a narrow
// record, the regions (REGION x REGION tiles) its rectangle overlaps for a
// wide one.  Cell j of the rectangle is (x0 + j % w, y0 + j / w).
struct Cells {
    int x0, y0, w;
    uint32_t area;   // 0: the record is listed nowhere
    int cw, ch;      // cell size in pixels
    int h;
};

__device__ __forceinline__ Cells cells_of(const float4& A, const float4& B, bool wide, const DevView& cam,
                                          const DevSettings& st) {
    Cells c{0, 0, 1, 0u, st.tile_w, st.tile_h, 0};
    const Rect q = rect_of(A.x, A.y, B.w, cam, st);
    if (q.x1 < q.x0 || q.y1 < q.y0) return c;
    if (wide) {
        c.x0 = q.x0 / REGION;
        c.y0 = q.y0 / REGION;
        c.w = q.x1 / REGION - c.x0 + 1;
        c.h = q.y1 / REGION - c.y0 + 1;
        c.cw = REGION * st.tile_w;
        c.ch = REGION * st.tile_h;
    } else {
        c.x0 = q.x0;
        c.y0 = q.y0;
        c.w = q.x1 - q.x0 + 1;
        c.h = q.y1 - q.y0 + 1;
    }
    c.area = (uint32_t)c.w * (uint32_t)c.h;
    return c;
}

// Sort key of cell (cx, cy): tile ids first, then region ids.
__device__ __forceinline__ uint32_t cell_key(bool wide, int cx, int cy, const DevView& cam, const ViewSet& views) {
    return wide ? views.total_tiles + cam.reg_off + (uint32_t)cy * (uint32_t)cam.reg_w + (uint32_t)cx
                : cam.tile_off + (uint32_t)cy * (uint32_t)cam.grid_w + (uint32_t)cx;
}

// Row-wise culling of the binning.  Within a band of pixel-centre rows
// [Y0, Y1] the points where an entry can pass the per-pixel filters form the
// band's slice of the ellipse a (ex + beta ey)^2 + gamma ey^2 <= cut (ex, ey
// offsets from the centre; cut = min(q_max, 2 ln(opacity / alpha_min)) plus a
// margin), and the slice's x-extent is an interval: the chord's right end
// -beta ey + sqrt((cut - gamma ey^2) / a) is concave in ey, so its maximum
// over the band is at the ellipse's rightmost point (ey = eyR) clamped to the
// band, and the left end's minimum at -eyR.  A cell of the row is kept iff
// the interval meets the cell's pixel-centre columns -- the decision of a
// test of the quadratic form's minimum over each cell's box, taken once per
// row.  Every operation is written out and contraction is off, so the
// classification (which counts) and the duplication (which emits) take
// identical decisions; culled cells contribute nothing to any pixel.
// Reciprocals and square roots are the hardware's single instructions (about
// one ulp): their error is orders of magnitude inside the margins (1e-3 of
// the cut, 1e-3 pixel), so the test stays conservative.
struct RowCull {
    float u, v, beta, gamma, inva, cut, H, eyR;
    int mode;  // 0: cull, 1: every cell (no finite cut), 2: no cell
};

__device__ __forceinline__ RowCull row_prep(const float4& A, const float4& B, const DevSettings& st) {
#pragma clang fp contract(off)
    RowCull p;
    p.u = A.x;
    p.v = A.y;
    p.beta = A.w;
    p.gamma = B.x;
    const float a = A.z;
    float cut = st.q_max;
    if (st.alpha_min > 0.f) cut = fminf(cut, 2.f * __logf(B.y / st.alpha_min));
    p.mode = 0;
    p.cut = 0.f;
    if (cut >= 3.0e38f) {
        p.mode = 1;
    } else if (!(cut > -3.0e38f)) {
        p.mode = 2;
    } else {
        p.cut = fmaf(1e-3f, 1.f + fabsf(cut), cut);
        if (!(p.cut >= 0.f)) p.mode = 2;
    }
    p.inva = __builtin_amdgcn_rcpf(a);
    p.H = __builtin_amdgcn_sqrtf(p.cut * __builtin_amdgcn_rcpf(p.gamma));
    const float D = fmaf(a * p.beta, p.beta, p.gamma);  // c = gamma + a beta^2
    p.eyR = -p.beta * __builtin_amdgcn_sqrtf(p.cut * a * __builtin_amdgcn_rcpf(p.gamma * D));
    return p;
}

// Columns [lo, hi] (within [x0, x1]) of cell row cy, cells of cw x ch pixels
// (powers of two), that the entry can reach; false if none.
__device__ __forceinline__ bool row_cells(const RowCull& p, int cy, int cw, int ch, int x0, int x1, int width,
                                          int height, int& lo, int& hi) {
#pragma clang fp contract(off)
    lo = x0;
    hi = x1;
    if (p.mode == 1) return true;
    if (p.mode == 2) return false;
    const float Y0 = (float)(cy * ch) + 0.5f, Y1 = (float)min((cy + 1) * ch, height) - 0.5f;
    const float e0 = fmaxf(Y0 - p.v, -p.H), e1 = fminf(Y1 - p.v, p.H);
    if (!(e0 <= e1)) return false;
    const float eR = fminf(fmaxf(p.eyR, e0), e1), eL = fminf(fmaxf(-p.eyR, e0), e1);
    const float gR = p.gamma * eR, gL = p.gamma * eL;
    const float sR = __builtin_amdgcn_sqrtf(fmaxf(0.f, (p.cut - gR * eR) * p.inva));
    const float sL = __builtin_amdgcn_sqrtf(fmaxf(0.f, (p.cut - gL * eL) * p.inva));
    const float xhi = p.u + (sR - p.beta * eR) + 1e-3f;
    const float xlo = p.u - (sL + p.beta * eL) - 1e-3f;
    if (!(xlo <= (float)width - 0.5f && xhi >= 0.5f)) return false;
    // cell cx spans pixel centres [cx cw + 0.5, (cx + 1) cw - 0.5]
    const float icw = ldexpf(1.f, -__builtin_ctz((unsigned)cw));  // exact: cw is a power of two
    const float flo = fmaxf(ceilf((xlo + 0.5f) * icw - 1.f), (float)x0);
    const float fhi = fminf(floorf((xhi - 0.5f) * icw), (float)x1);
    if (!(flo <= fhi)) return false;
    lo = (int)flo;
    hi = (int)fhi;
    return true;
}

// The four 4x4 pixel blocks (bit 2 (y / 4) + x / 4) of the 8x8 pixels at
// (x0, y0) that an entry can reach: row_cells' band test with the bands and
// columns of the blocks.  The margin grows with the centre's distance, whose
// rounding the per-pixel evaluation shares, and a comparison with a NaN
// counts as reached, so a block left out holds no pixel that passes the
// filters.
__device__ __forceinline__ uint32_t block_mask(const float4& A, const float4& B, int x0, int y0, int height,
                                               const DevSettings& st) {
    const RowCull p = row_prep(A, B, st);
    if (p.mode == 1) return 15u;
    if (p.mode == 2) return 0u;
    uint32_t mask = 0;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const float Y0 = (float)(y0 + 4 * r) + 0.5f, Y1 = (float)min(y0 + 4 * r + 4, height) - 0.5f;
        const float e0 = fmaxf(Y0 - p.v, -p.H), e1 = fminf(Y1 - p.v, p.H);
        if (e0 > e1) continue;
        const float eR = fminf(fmaxf(p.eyR, e0), e1), eL = fminf(fmaxf(-p.eyR, e0), e1);
        const float sR = __builtin_amdgcn_sqrtf(fmaxf(0.f, (p.cut - p.gamma * eR * eR) * p.inva));
        const float sL = __builtin_amdgcn_sqrtf(fmaxf(0.f, (p.cut - p.gamma * eL * eL) * p.inva));
        const float mg = 1e-3f + 1e-6f * (fabsf(p.u) + fabsf(p.beta) * fmaxf(fabsf(eR), fabsf(eL)));
        const float xhi = p.u + (sR - p.beta * eR) + mg, xlo = p.u - (sL + p.beta * eL) - mg;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float X0 = (float)(x0 + 4 * c) + 0.5f;
            if (!(xhi < X0 || xlo > X0 + 3.f)) mask |= 1u << (2 * r + c);
        }
    }
    return mask;
}

// A value equal in all lanes, in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)uniform((int)v); }
__device__ __forceinline__ uint2 uniform(uint2 v) { return make_uint2(uniform(v.x), uniform(v.y)); }

// Inclusive maximum scan over the 64 lanes of a wave, for values >= -1:
// shifts within each 16-lane row, then the broadcasts of lane 15 into rows
// 1 and 3 and of lane 31 into rows 2 and 3 (a lane with no source keeps -1).
__device__ __forceinline__ int wave_max_scan(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x111, 0xf, 0xf, false));  // row_shr 1
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x112, 0xf, 0xf, false));  // row_shr 2
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x114, 0xf, 0xf, false));  // row_shr 4
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x118, 0xf, 0xf, false));  // row_shr 8
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x142, 0xa, 0xf, false));  // row_bcast 15
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x143, 0xc, 0xf, false));  // row_bcast 31
    return x;
}

// Owner of each of the slots [w0, w0 + 64) of a wave, one per lane: items (one
// per lane, at most; has: this lane's holds slots) own consecutive runs of
// slots, item `lane` from slot `first` on; the owner is the last item whose
// first slot is at or before the slot.  Every item marks its first slot in the
// wave's 64 words, a running maximum fills the rest; carry: the last owner of
// the slots before (-1 at first).  LDS operations of one wave complete in
// program order.
__device__ __forceinline__ int slot_owner(int* words, int lane, bool has, uint32_t first, uint32_t w0, int& carry) {
    words[lane] = -1;
    __builtin_amdgcn_wave_barrier();
    if (has && first - w0 < 64u) words[first - w0] = lane;  // (first below w0 wraps)
    __builtin_amdgcn_wave_barrier();
    const int own = max(wave_max_scan(words[lane]), carry);
    carry = __builtin_amdgcn_readlane(own, 63);
    __builtin_amdgcn_wave_barrier();
    return own;
}

// What the classification hands to the duplication per listed position (x:
// key of the first cell; y: row stride of the keys << 14).  A rectangle of at
// most CULL_MAX cells: y also width and height << 7, (z, w) the kept cells as
// a bit mask (bit j: cell j, row-major).  A larger one: y also CELLS_LARGE, z
// first column and row << 16, w width and height << 16; its rows are found
// again.  (Grids have at most 2048 x 2048 cells.)
constexpr uint32_t CULL_MAX = 64;
constexpr uint32_t CELLS_LARGE = 0x80000000u;
// Key of an emitted slot the duplication could not fill: past every cell,
// so it sorts last and no range includes it.
constexpr uint32_t KEY_NONE = 0xffffffffu;
// Bit of a position's entry count that marks a wide record (listed per
// region); the count itself is below 2^24.
constexpr uint32_t CNT_WIDE = 0x80000000u;
// Splats of a larger radius (pixels) cover most of the tiles they reach.
constexpr float LARGE_RADIUS = 24.f;

// Sorted position i holds record order[i] with depth key skeys[i]; positions
// [v n, (v + 1) n) belong to view v.  Writes the sorted record copy (radius in
// B.w, record id bits in C.w), the wide flag and the number of list entries
// (tiles or regions, after culling) of every position, and per workgroup the
// number of wide records and of their region entries (part[b], part[nb +
// b]), and per wave the number of all list entries (part[2 nb + wave]; a
// position has fewer than 2^24 entries, so a wave's 64 stay below 2^32).
// With sizes, also per workgroup the tiles of all footprints and those of
// splats larger than LARGE_RADIUS (part[6 nb + b], part[7 nb + b]; at most
// 2^22 tiles each): the compositing's choice of kernel.
// A record without tiles (key all ones, last in its view: from lives[view] on,
// if given) is listed
// nowhere: it gets no copy, which nothing uses.
// Bound by the gather of the records (8 views of 1 M, 70 % listed: 0.82 GB, 159
// us at the copy rate).  The wave loads its records three lanes to each, and
// walks their rows 64 at a time: with a record per lane throughout, the lanes
// wait for the one with most rows.  227 -> 209 us (8.5e7 -> 6.3e7 vector
// instructions of a wave), 1.5 M records of one view 41.5 -> 40.6 us, though
// the duplication now gets the rectangle too (16 bytes for 8).
__global__ void __launch_bounds__(256) permute_classify_kernel(
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ skeys, const uint32_t* __restrict__ lives,
    const float4* __restrict__ rec, int64_t R, int64_t n, ViewSet views, DevSettings st, uint32_t* __restrict__ cnt_out,
    uint4* __restrict__ cells, float4* __restrict__ srec,
    uint32_t* __restrict__ part, int sizes) {
    __shared__ uint32_t s_part[4][4];
    // per wave 3 x 64: its records as they are laid out, then for the walk over
    // rows, per record: RowCull (two), columns, rows and the view's size
    __shared__ float4 s_rec[3 * 256];
    __shared__ uint32_t s_cnt[256];
    __shared__ unsigned long long s_mask[256];
    __shared__ int s_own[256];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = lane_id();
    const bool live = i < R;
    float4 A = make_float4(0.f, 0.f, 0.f, 0.f), B = A;
    uint32_t c = 0;
    bool wide = false;
    int vi = 0;
    // both loads of the position in one round trip, then the record
    if (live && lives) vi = (int)((uint32_t)i / (uint32_t)n);  // positions are below 2^32
    const bool has =
        live && (lives ? (uint32_t)i - (uint32_t)vi * (uint32_t)n < lives[vi] : skeys[i] != 0xffffffffu);
    const uint32_t r = live ? order[i] : 0u;
    float4* wrec = s_rec + 3 * (threadIdx.x & ~63u);
    if (ballot(has)) {
        // the wave's records (radius in B.w, tile count in C.w), three
        // neighbouring lanes to a record: a load touches 22 records' lines
        // instead of 64, and the copy's stores are contiguous
        const uint32_t rid = has ? r : 0xffffffffu;
        float4* out4 = srec + 3 * (i - lane);
        float4 v[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int q = j * 64 + lane, part = q % 3;
            const uint32_t rq = (uint32_t)__shfl((int)rid, q / 3);
            v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (rq != 0xffffffffu) v[j] = rec[3 * (size_t)rq + part];
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int q = j * 64 + lane;
            const uint32_t rq = (uint32_t)__shfl((int)rid, q / 3);
            wrec[q] = v[j];
            if (q % 3 == 2) v[j].w = __uint_as_float(rq);
            if (rq != 0xffffffffu) out4[q] = v[j];
        }
        __builtin_amdgcn_wave_barrier();
        A = wrec[3 * lane];
        B = wrec[3 * lane + 1];
        c = __float_as_uint(wrec[3 * lane + 2].w);
        if (has) {
            vi = (int)((uint32_t)i / (uint32_t)n);
            wide = c > views.v[vi].wide_min;
        }
        __builtin_amdgcn_wave_barrier();
    }
    Cells cl{0, 0, 1, 0u, st.tile_w, st.tile_h, 0};
    if (live && c > 0) cl = cells_of(A, B, wide, views.v[vi], st);
    uint32_t cnt = cl.area;
    uint64_t mask = cl.area >= 64u ? ~0ull : (1ull << cl.area) - 1ull;
    if (st.tile_cull) {
        // the rows of the wave's records, one per lane and round
        const int t = threadIdx.x, wb = t & ~63;
        const uint32_t rows = cl.area > 0 ? (uint32_t)cl.h : 0u;
        const uint32_t x = wave_add_scan(rows);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)x, 63), first = x - rows;
        if (rows) {
            const RowCull rc = row_prep(A, B, st);
            wrec[lane] = make_float4(rc.u, rc.v, rc.beta, rc.gamma);
            wrec[64 + lane] = make_float4(rc.inva, rc.cut, rc.H, rc.eyR);
            reinterpret_cast<uint4*>(wrec)[128 + lane] =
                make_uint4(first, (uint32_t)cl.x0 | (uint32_t)cl.y0 << 16,
                           (uint32_t)cl.w | (uint32_t)rc.mode << 16 | (wide ? 1u << 18 : 0u),
                           (uint32_t)views.v[vi].width | (uint32_t)views.v[vi].height << 16);
        }
        s_cnt[t] = 0u;
        s_mask[t] = 0ull;
        int carry = -1;
        for (uint32_t w0 = 0; w0 < total; w0 += 64) {
            const int own = slot_owner(s_own + wb, lane, rows > 0, first, w0, carry), k = wb + own;
            const uint32_t e = w0 + (uint32_t)lane;
            if (e >= total) continue;
            const float4 p0 = wrec[own], p1 = wrec[64 + own];
            const uint4 g = reinterpret_cast<const uint4*>(wrec)[128 + own];
            const int ry = (int)(e - g.x), w = (int)(g.z & 0xffffu), x0 = (int)(g.y & 0xffffu);
            const RowCull rc{p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w, (int)(g.z >> 16) & 3};
            const int scale = (g.z >> 18) & 1u ? REGION : 1;
            int lo, hi;
            if (!row_cells(rc, (int)(g.y >> 16) + ry, scale * st.tile_w, scale * st.tile_h, x0, x0 + w - 1,
                           (int)(g.w & 0xffffu), (int)(g.w >> 16), lo, hi))
                continue;
            const uint32_t nb = (uint32_t)(hi - lo + 1);
            atomicAdd(&s_cnt[k], nb);
            // bits ry w + (lo - x0) .. ry w + (hi - x0); of no use past 64 cells
            const uint32_t b0 = (uint32_t)(ry * w + (lo - x0));
            if (b0 < 64u) atomicOr(&s_mask[k], (nb >= 64 ? ~0ull : ((1ull << nb) - 1ull)) << b0);
        }
        __builtin_amdgcn_wave_barrier();
        cnt = s_cnt[t];
        mask = s_mask[t];
    }
    if (live) {
        // the wide flag rides in bit 31 (counts stay below 2^24); the cells
        // are kept only for positions with entries
        cnt_out[i] = cnt | (wide ? CNT_WIDE : 0u);
        if (cnt != 0) {
            const DevView& cam = views.v[vi];
            uint4 o;
            o.x = cell_key(wide, cl.x0, cl.y0, cam, views);
            o.y = (uint32_t)(wide ? cam.reg_w : cam.grid_w) << 14;
            if (cl.area <= CULL_MAX) {
                o.y |= (uint32_t)cl.w | (uint32_t)cl.h << 7;
                o.z = (uint32_t)mask;
                o.w = (uint32_t)(mask >> 32);
            } else {
                o.y |= CELLS_LARGE;
                o.z = (uint32_t)cl.x0 | (uint32_t)cl.y0 << 16;
                o.w = (uint32_t)cl.w | (uint32_t)cl.h << 16;
            }
            cells[i] = o;
        }
    }
    // wide records and their list entries of the workgroup (no atomics: one
    // address updated by every wave serialises)
    const uint64_t wb = __ballot(live && wide);
    // the wave's totals land in lane 63
    const uint32_t e = wave_add_scan(live && wide ? cnt : 0u);
    const uint32_t ea = wave_add_scan(live ? cnt : 0u);
    const int wid = threadIdx.x >> 6;
    if (sizes) {
        const uint32_t all = wave_add_scan(c), large = wave_add_scan(B.w > LARGE_RADIUS ? c : 0u);
        if (lane == 63) {
            s_part[2][wid] = all;
            s_part[3][wid] = large;
        }
    }
    if (lane == 63) {
        s_part[0][wid] = (uint32_t)__popcll(wb);
        s_part[1][wid] = e;
        part[2 * gridDim.x + (blockIdx.x * blockDim.x + threadIdx.x) / 64] = ea;
    }
    __syncthreads();
    if (threadIdx.x < 4u) {
        const uint32_t k = threadIdx.x;
        const uint32_t a = s_part[k][0] + s_part[k][1] + s_part[k][2] + s_part[k][3];
        if (k < 2 || sizes) part[(k < 2 ? k : k + 4) * gridDim.x + blockIdx.x] = a;
    }
}

// List offsets from the classification's counts, in two steps.  A group is
// LO_GROUP waves (LO_GROUP / 4 classification workgroups).  Step 1, one
// workgroup per group: each wave's first entry relative to its group (an
// exclusive scan of the per-wave entry counts), the group's entry total and
// its totals of wide records, their region entries and the footprint tiles.
// Step 2, one workgroup: the groups' first entries, the entry total (*total),
// the wide totals (wide[0], wide[2]) and the footprint tiles, all and of large
// splats (wide[3], wide[4]).  A wave's first entry is then
// wave_rel[wave] + group_off[wave / LO_GROUP].  Integer sums: no result
// depends on an order.
constexpr int LO_GROUP = 1024;
struct ListOffsets {
    uint64_t* wave_rel;   // [waves]
    uint64_t* group_tot;  // [groups, 5]: entries, wide records, region entries, footprint tiles (all, large)
    uint64_t* group_off;  // [groups]
};

// Inclusive sums within each 16 lanes, and a lane's value in every lane.
__device__ __forceinline__ uint64_t waves_scan(uint64_t x) {
    static_assert(LO_GROUP / 64 == 16, "one lane per wave");
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const uint64_t y = __shfl_up(x, d, 16);
        if ((lane_id() & 15) >= d) x += y;
    }
    return x;
}
// (only where the whole wave is active: in a branch, what the compiler moved
// into it is missing in the lanes that are not)
__device__ __forceinline__ uint64_t read_lane(uint64_t x, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l) << 32 | lo;
}

__global__ void __launch_bounds__(LO_GROUP) list_offsets_group_kernel(const uint32_t* __restrict__ part, int64_t nb,
                                                                     int64_t nw, ListOffsets lo, int sizes) {
    __shared__ uint64_t s_w[LO_GROUP / 64][5];
    const int t = threadIdx.x, lane = lane_id(), wid = uniform(t >> 6);
    const int64_t w = (int64_t)blockIdx.x * LO_GROUP + t;  // this thread's wave
    const uint64_t c = w < nw ? part[2 * nb + w] : 0u;
    // the group's classification workgroups: LO_GROUP / 4 of them
    const int64_t b = (int64_t)blockIdx.x * (LO_GROUP / 4) + t;
    uint64_t sum[4] = {0, 0, 0, 0};
    if (t < LO_GROUP / 4 && b < nb) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < 2 || sizes) sum[k] = part[(k < 2 ? k : k + 4) * nb + b];
    }
    uint64_t x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_w[wid][0] = x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        for (int off = 32; off > 0; off >>= 1) sum[k] += __shfl_xor(sum[k], off);
        if (lane == 0) s_w[wid][1 + k] = sum[k];
    }
    __syncthreads();
    const uint64_t ws = waves_scan(s_w[lane & 15][0]);
    const uint64_t before = wid > 0 ? read_lane(ws, wid - 1) : 0u;
    if (w < nw) lo.wave_rel[w] = before + x - c;
    if (t < 5) {
        uint64_t tot = 0;
#pragma unroll
        for (int v = 0; v < LO_GROUP / 64; ++v) tot += s_w[v][t];
        lo.group_tot[5 * blockIdx.x + t] = tot;
    }
}

// What step 2 leaves: on the device, and (host, optional) in pinned host
// memory with the flag words and the staged-entry counter, so that the plain
// path's one read needs no copy.
struct ListTotals {
    uint64_t* total;
    uint64_t* wide;
    const uint32_t* flags;   // two words
    const uint32_t* staged;
    uint64_t* host;
};
// thread k of the workgroup holds total k (0: entries, 1 .. 4: as group_tot)
__device__ __forceinline__ void put_totals(const ListTotals& o, int k, uint64_t v) {
    if (k > 4) return;
    const int w = k <= 1 ? 0 : k;  // place in wide
    if (k == 0) *o.total = v;
    else o.wide[w] = v;
    if (o.host) {
        if (k == 0) {
            o.host[1] = v;
            o.host[0] = (uint64_t)o.flags[0] | (uint64_t)o.flags[1] << 32;
            o.host[24] = (uint64_t)*o.staged * STG_CHUNK;
        } else {
            o.host[2 + w] = v;
        }
        __threadfence_system();
    }
}

__global__ void __launch_bounds__(LO_GROUP) list_offsets_total_kernel(int64_t ng, ListOffsets lo, ListTotals out) {
    __shared__ uint64_t s_w[LO_GROUP / 64][5];
    const int t = threadIdx.x, lane = lane_id(), wid = uniform(t >> 6);
    uint64_t carry = 0, sum[4] = {0, 0, 0, 0};
    for (int64_t base = 0; base < ng; base += LO_GROUP) {
        const int64_t g = base + t;
        const uint64_t c = g < ng ? lo.group_tot[5 * g] : 0u;
        if (g < ng) {
#pragma unroll
            for (int k = 0; k < 4; ++k) sum[k] += lo.group_tot[5 * g + 1 + k];
        }
        uint64_t x = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t y = __shfl_up(x, d);
            if (lane >= d) x += y;
        }
        if (lane == 63) s_w[wid][0] = x;
        __syncthreads();
        const uint64_t ws = waves_scan(s_w[lane & 15][0]);
        const uint64_t before = wid > 0 ? read_lane(ws, wid - 1) : 0u;
        if (g < ng) lo.group_off[g] = carry + before + x - c;
        carry += read_lane(ws, 15);
        __syncthreads();  // s_w is written again by the next round
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        for (int off = 32; off > 0; off >>= 1) sum[k] += __shfl_xor(sum[k], off);
        if (lane == 0) s_w[wid][1 + k] = sum[k];
    }
    __syncthreads();
    if (t < 5) {
        uint64_t tot = carry;
        if (t > 0) {
            tot = 0;
#pragma unroll
            for (int v = 0; v < LO_GROUP / 64; ++v) tot += s_w[v][t];
        }
        put_totals(out, t, tot);
    }
}

// Both steps in one workgroup, for at most LO_ONE groups, whose loads and scans
// go side by side (10.4 -> 8.9 us for four; the two launches: 10.3 us; a second
// round of groups: 12.6 us).
constexpr int64_t LO_ONE = 4;
constexpr int LO_ROUND = 4;
__global__ void __launch_bounds__(LO_GROUP) list_offsets_one_kernel(const uint32_t* __restrict__ part, int64_t nb,
                                                                   int64_t nw, int64_t ng, ListOffsets lo, int sizes,
                                                                   ListTotals out) {
    __shared__ uint64_t s_w[LO_GROUP / 64][5];
    const int t = threadIdx.x, lane = lane_id(), wid = uniform(t >> 6);
    uint64_t carry = 0, sum[4] = {0, 0, 0, 0};
    for (int64_t b = t; b < nb; b += LO_GROUP) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < 2 || sizes) sum[k] += part[(k < 2 ? k : k + 4) * nb + b];
    }
    __shared__ uint64_t s_g[LO_GROUP / 64][LO_ROUND];
    for (int64_t g0 = 0; g0 < ng; g0 += LO_ROUND) {
        // the groups' loads and scans side by side
        uint64_t c[LO_ROUND], x[LO_ROUND];
#pragma unroll
        for (int j = 0; j < LO_ROUND; ++j) {
            const int64_t w = (g0 + j) * LO_GROUP + t;
            x[j] = c[j] = w < nw ? part[2 * nb + w] : 0u;
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
            for (int j = 0; j < LO_ROUND; ++j) {
                const uint64_t y = __shfl_up(x[j], d);
                if (lane >= d) x[j] += y;
            }
        }
#pragma unroll
        for (int j = 0; j < LO_ROUND; ++j)
            if (lane == 63) s_g[wid][j] = x[j];
        __syncthreads();
        // lanes 16 j + v: the inclusive sums of group j's waves up to v
        const uint64_t ws = waves_scan(s_g[lane & 15][lane >> 4]);
#pragma unroll
        for (int j = 0; j < LO_ROUND; ++j) {
            const int64_t w = (g0 + j) * LO_GROUP + t;
            const uint64_t wo = wid > 0 ? read_lane(ws, 16 * j + wid - 1) : 0u;
            if (w < nw) lo.wave_rel[w] = wo + x[j] - c[j];
            if (t == 0 && g0 + j < ng) lo.group_off[g0 + j] = carry;
            carry += read_lane(ws, 16 * j + 15);
        }
        __syncthreads();  // s_g is written again
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        for (int off = 32; off > 0; off >>= 1) sum[k] += __shfl_xor(sum[k], off);
        if (lane == 0) s_w[wid][1 + k] = sum[k];
    }
    __syncthreads();
    if (t < 5) {
        uint64_t tot = carry;
        if (t > 0) {
            tot = 0;
#pragma unroll
            for (int v = 0; v < LO_GROUP / 64; ++v) tot += s_w[v][t];
        }
        put_totals(out, t, tot);
    }
}

// List entries in sorted-position order: cell keys (tile or region ids) as
// keys, positions as values, for the cells the classification counted.  Each
// wave walks its records' rows 64 at a time, one per lane: a row's kept cells
// are one run, read off the record's cell mask, or found again where the
// rectangle has more than CULL_MAX cells.  It then walks the runs' entries 64
// at a time, so that every lane is busy and consecutive lanes write
// consecutive entries.  Bound by VALU issue where lists are short: selecting
// each entry's cell as the r-th bit of its mask, deriving every rectangle again
// from the record, and one large record at a time, this took 187 us for 8
// views of 1 M records (20.2 M entries), 63 us for 1.5 M (4.1 M) and 32 us for
// 300 k (1.6 M); walking runs 104, 23 and 14 us (20.2 M entries: 41 us of
// traffic for them, 27 us for the cells).  Writes never leave the wave's counted slots; a slot
// the emission does not fill gets KEY_NONE.  No step waits on another wave.
// Words that a thread clears at most: few records over many tiles take further
// workgroups, which only clear (left to the records', 256 of one view in 32,400
// tiles: stage 56 -> 14 us, of 16 views in 518,400 tiles 58 -> 20 us).
constexpr int DUP_CLEAR = 4;
__global__ void __launch_bounds__(256) duplicate_kernel(
    const float4* __restrict__ srec, const uint32_t* __restrict__ cnt_sorted,
    const uint4* __restrict__ cells, ListOffsets lo, int64_t R, int64_t n, ViewSet views, DevSettings st,
    void* __restrict__ keys, bool keys16, uint32_t* __restrict__ vals, int64_t capacity,
    uint32_t* __restrict__ flags, FillSet fs) {
    // the clears of the later stages ride along (a launch of their own: 4 us)
    for (int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x; f < fs.total; f += (int64_t)gridDim.x * 256)
        fill_element(fs, f);
    __shared__ uint4 s_c[256];   // per record: first row | flags, key, width | stride << 16, column | row << 16
    __shared__ unsigned long long s_mask[256];
    __shared__ float4 s_p0[256], s_p1[256];  // large records: RowCull, in part
    __shared__ int2 s_wh[256];               // ... and the view's size
    __shared__ uint2 s_run[256];             // per row: key of its first entry less the entry's slot, position
    __shared__ int s_own[256];
    constexpr uint32_t LARGE = 1u << 24, MODE = 25, WIDE = 1u << 27;  // flags beside the first row (below 2^24)
    const int t = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x;
    const int64_t i = i0 + t;
    const int lane = lane_id();
    const int wb = t & ~63;  // the wave's first thread
    uint32_t cnt = 0;
    bool wide = false;
    if (i < R) {
        const uint32_t cw = cnt_sorted[i];
        cnt = cw & ~CNT_WIDE;
        wide = (cw & CNT_WIDE) != 0;
    }
    if (!ballot(cnt != 0)) return;  // (no barrier below is the workgroup's)
    uint32_t rows = 0;
    uint4 c = make_uint4(0u, 0u, 0u, 0u);
    if (cnt != 0) {
        c = cells[i];
        rows = c.y & CELLS_LARGE ? c.w >> 16 : (c.y >> 7) & 0x7fu;
    }
    const uint32_t rx = wave_add_scan(rows), ax = wave_add_scan(cnt);
    const uint32_t total_rows = (uint32_t)__builtin_amdgcn_readlane((int)rx, 63), first = rx - rows;
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)ax, 63);
    if (cnt != 0) {
        const uint32_t stride = (c.y & ~CELLS_LARGE) >> 14;
        if (c.y & CELLS_LARGE) {
            uint32_t fl = LARGE | (wide ? WIDE : 0u);
            if (st.tile_cull) {
                const DevView& cam = views.v[(uint32_t)i / (uint32_t)n];  // positions are below 2^32
                const RowCull rc = row_prep(srec[3 * i], srec[3 * i + 1], st);
                s_p0[t] = make_float4(rc.u, rc.v, rc.beta, rc.gamma);
                s_p1[t] = make_float4(rc.inva, rc.cut, rc.H, rc.eyR);
                s_wh[t] = make_int2(cam.width, cam.height);
                fl |= (uint32_t)rc.mode << MODE;
            }
            s_c[t] = make_uint4(first | fl, c.x, (c.w & 0xffffu) | stride << 16, c.z);
        } else {
            s_c[t] = make_uint4(first, c.x, (c.y & 0x7fu) | stride << 16, 0u);
            s_mask[t] = (unsigned long long)c.w << 32 | c.z;
        }
    }
    // the wave's slots: its offset within its group of waves plus the group's
    const int64_t wave = uniform((int)(i0 / 64) + (t >> 6));
    const int64_t base = (int64_t)(lo.wave_rel[wave] + lo.group_off[wave / LO_GROUP]);
    const uint32_t lim = (uint32_t)max((int64_t)0, min((int64_t)total, capacity - base));
    uint32_t* kw = reinterpret_cast<uint32_t*>(keys) + base;
    uint16_t* kh = reinterpret_cast<uint16_t*>(keys) + base;
    uint32_t* vw = vals + base;
    uint32_t out = 0;
    int rcarry = -1;
    for (uint32_t r0 = 0; r0 < total_rows; r0 += 64) {
        const int k = wb + slot_owner(s_own + wb, lane, rows > 0, first, r0, rcarry);
        uint32_t nrun = 0, key = 0;
        if (r0 + (uint32_t)lane < total_rows) {
            const uint4 g = s_c[k];
            const uint32_t ry = r0 + (uint32_t)lane - (g.x & 0xffffffu), w = g.z & 0xffffu;
            key = g.y + ry * (g.z >> 16);
            if (!(g.x & LARGE)) {
                const uint64_t m = (s_mask[k] >> (ry * w)) & (w >= 64u ? ~0ull : (1ull << w) - 1ull);
                nrun = (uint32_t)__popcll(m);
                key += (uint32_t)__builtin_ctzll(m | 1ull << 63);
            } else if (!st.tile_cull) {
                nrun = w;
            } else {
                const float4 p0 = s_p0[k], p1 = s_p1[k];
                const int2 wh = s_wh[k];
                const RowCull rc{p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w, (int)(g.x >> MODE) & 3};
                const int scale = g.x & WIDE ? REGION : 1, x0 = (int)(g.w & 0xffffu);
                int cl, ch;
                if (row_cells(rc, (int)((g.w >> 16) + ry), scale * st.tile_w, scale * st.tile_h, x0, x0 + (int)w - 1,
                              wh.x, wh.y, cl, ch)) {
                    nrun = (uint32_t)(ch - cl + 1);
                    key += (uint32_t)(cl - x0);
                }
            }
        }
        const uint32_t nx = wave_add_scan(nrun), nfirst = nx - nrun;
        const uint32_t ntot = (uint32_t)__builtin_amdgcn_readlane((int)nx, 63);
        s_run[t] = make_uint2(key - nfirst, (uint32_t)(i0 + k));
        int ecarry = -1;
        for (uint32_t e0 = 0; e0 < ntot; e0 += 64) {
            const uint2 run = s_run[wb + slot_owner(s_own + wb, lane, nrun > 0, nfirst, e0, ecarry)];
            const uint32_t e = e0 + (uint32_t)lane, o = out + e;
            if (e < ntot && o < lim) {
                if (keys16) kh[o] = (uint16_t)(run.x + e);
                else kw[o] = run.x + e;
                vw[o] = run.y;
            }
        }
        __builtin_amdgcn_wave_barrier();  // s_run is written again
        out += ntot;
    }
    for (uint32_t o = out + (uint32_t)lane; o < lim; o += 64) {
        if (keys16) kh[o] = (uint16_t)KEY_NONE;
        else kw[o] = KEY_NONE;
        vw[o] = 0u;
    }
    if (lim < total && lane == 0) atomicOr(flags, FLAG_CAPACITY);
}

// Cell of the region that holds tile (tx, ty).
__device__ __forceinline__ uint32_t region_of_tile(int tx, int ty, const DevView& cam, const ViewSet& views) {
    return views.total_tiles + cam.reg_off + (uint32_t)(ty / REGION) * (uint32_t)cam.reg_w + (uint32_t)(tx / REGION);
}

// Per tile: the batch checkpoints it may take (a batch either emits `batch`
// merged entries or exhausts a whole window of one of the two streams), as
// an exclusive prefix within the workgroup (cur_off) and the workgroup's
// total (blk); the forward's cost key (cost: the entries of the two lists in
// units of 8, at most 255); and the workgroup's histogram of the tile-order
// key (key[t], or the cost key when key is null), added into hist[256].
__global__ void __launch_bounds__(256) batch_caps_kernel(const uint2* __restrict__ ranges, ViewSet views, int batch,
                                                          const uint32_t* __restrict__ key, uint32_t* __restrict__ cost,
                                                          uint32_t* __restrict__ cur_off, uint32_t* __restrict__ blk,
                                                          uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[256];
    __shared__ uint32_t s_w[4];
    const int tid = threadIdx.x, lane = lane_id();
    h[tid] = 0u;
    __syncthreads();
    const uint32_t t = blockIdx.x * 256u + (uint32_t)tid;
    uint32_t c = 0;
    if (t < views.total_tiles) {
        int vi = 0;
        while (vi + 1 < views.n_views && t >= views.v[vi + 1].tile_off) ++vi;
        const DevView& cam = views.v[vi];
        const uint32_t lt = t - cam.tile_off;
        const int tx = (int)(lt % (uint32_t)cam.grid_w), ty = (int)(lt / (uint32_t)cam.grid_w);
        const uint2 r2 = ranges[region_of_tile(tx, ty, cam, views)];
        const uint32_t len1 = ranges[t].y - ranges[t].x;
        const uint32_t len2 = r2.y - r2.x;
        c = 2u * ((len1 + batch - 1) / batch + (len2 + batch - 1) / batch) + 2u;
        const uint32_t ck = min((len1 + len2) >> 3, 255u);
        if (cost) cost[t] = ck;
        atomicAdd(&h[255u - min(key ? key[t] : ck, 255u)], 1u);
    }
    uint32_t x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_w[tid >> 6] = x;
    __syncthreads();
    uint32_t wo = 0;
    for (int v = 0; v < (tid >> 6); ++v) wo += s_w[v];
    if (t < views.total_tiles) cur_off[t] = wo + x - c;
    if (tid == 255) blk[blockIdx.x] = wo + x;
    if (h[tid]) atomicAdd(&hist[tid], h[tid]);
}

// Launch order of the tiles, most expensive first, so that the last
// workgroups to start are cheap (a launch's tail is the cost of the tiles
// still running when none is left to start).  A counting sort on a per-tile
// cost key (0..255, descending): order_hist_kernel adds every workgroup's
// histogram of the keys into hist[256]; order_place_kernel scans hist for the
// bins' starts, takes for each of its bins a run of slots with one atomic
// on cursor[256] and places its tiles in the run (ties in any order: the
// tiles are independent).  hist and cursor are zero before the first kernel.
__global__ void __launch_bounds__(256) order_hist_kernel(const uint32_t* __restrict__ key, uint32_t n,
                                                          uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[256];
    const int t = threadIdx.x;
    h[t] = 0u;
    __syncthreads();
    const uint32_t i = blockIdx.x * 256u + (uint32_t)t;
    if (i < n) atomicAdd(&h[255u - min(key[i], 255u)], 1u);
    __syncthreads();
    if (h[t]) atomicAdd(&hist[t], h[t]);
}

__global__ void __launch_bounds__(256) order_place_kernel(const uint32_t* __restrict__ key, uint32_t n,
                                                           const uint32_t* __restrict__ hist,
                                                           uint32_t* __restrict__ cursor, uint32_t* __restrict__ order) {
    __shared__ uint32_t s_base[256];
    __shared__ uint32_t s_cnt[256];
    __shared__ uint32_t s_wsum[4];
    const int t = threadIdx.x, lane = lane_id();
    // bin starts: exclusive scan of hist
    const uint32_t c = hist[t];
    uint32_t x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wsum[t >> 6] = x;
    s_cnt[t] = 0u;
    __syncthreads();
    uint32_t start = x - c;
    for (int v = 0; v < (t >> 6); ++v) start += s_wsum[v];
    // this workgroup's tiles per bin, and each tile's rank within its bin
    const uint32_t i = blockIdx.x * 256u + (uint32_t)t;
    const uint32_t b = i < n ? 255u - min(key[i], 255u) : 0u;
    const uint32_t rank = i < n ? atomicAdd(&s_cnt[b], 1u) : 0u;
    __syncthreads();
    // a run of slots per non-empty bin
    if (s_cnt[t]) s_base[t] = start + atomicAdd(&cursor[t], s_cnt[t]);
    __syncthreads();
    if (i < n) order[s_base[b] + rank] = i;
}

// order_place_kernel for the forward's set-up (the keys: key[t], or cost[t]
// when key is null), which also completes the checkpoint offsets: cur_off[t]
// (a prefix within its workgroup of 256 tiles) plus the totals of the
// earlier workgroups (blk), and *cur_need = the grand total.  The batch
// counts of the tiles (nbatch, which key may be) are cleared for the forward.
__global__ void __launch_bounds__(256) order_offsets_kernel(const uint32_t* key,
                                                             const uint32_t* __restrict__ cost, uint32_t n,
                                                             const uint32_t* __restrict__ hist,
                                                             uint32_t* __restrict__ cursor,
                                                             uint32_t* __restrict__ order,
                                                             uint32_t* __restrict__ cur_off,
                                                             const uint32_t* __restrict__ blk,
                                                             uint64_t* __restrict__ cur_need,
                                                             uint32_t* nbatch) {
    __shared__ uint32_t s_base[256];
    __shared__ uint32_t s_cnt[256];
    __shared__ uint32_t s_wsum[4];
    __shared__ uint64_t s_pre[4];
    const int t = threadIdx.x, lane = lane_id();
    const uint32_t c = hist[t];
    uint32_t x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    // checkpoints of the earlier workgroups
    uint64_t pre = 0;
    for (uint32_t b0 = 0; b0 < blockIdx.x; b0 += 256u) {
        const uint32_t b = b0 + (uint32_t)t;
        if (b < blockIdx.x) pre += blk[b];
    }
    for (int off = 32; off > 0; off >>= 1) pre += __shfl_xor(pre, off);
    if (lane == 63) s_wsum[t >> 6] = x;
    if (lane == 0) s_pre[t >> 6] = pre;
    s_cnt[t] = 0u;
    __syncthreads();
    uint32_t start = x - c;
    for (int v = 0; v < (t >> 6); ++v) start += s_wsum[v];
    const uint64_t before = s_pre[0] + s_pre[1] + s_pre[2] + s_pre[3];
    const uint32_t i = blockIdx.x * 256u + (uint32_t)t;
    if (i < n) cur_off[i] += (uint32_t)before;
    if (blockIdx.x == gridDim.x - 1 && t == 0) *cur_need = before + blk[blockIdx.x];
    const uint32_t b = i < n ? 255u - min(key ? key[i] : cost[i], 255u) : 0u;
    const uint32_t rank = i < n ? atomicAdd(&s_cnt[b], 1u) : 0u;
    __syncthreads();
    if (s_cnt[t]) s_base[t] = start + atomicAdd(&cursor[t], s_cnt[t]);
    __syncthreads();
    if (i < n) {
        order[s_base[b] + rank] = i;
        nbatch[i] = 0u;  // (key may be the same array: read above by this thread only)
    }
}

// batch_caps_kernel and order_offsets_kernel in one workgroup, for at most
// SETUP_ONE tiles (64 tiles 4 us, 478 tiles 5.2 us; 2,500 tiles 8.5 us, 4,080
// tiles 11.5 us, where the two launches take 8 to 9 us).
constexpr int SETUP_DT = 1024, SETUP_PER = 2;
constexpr uint32_t SETUP_ONE = SETUP_DT * SETUP_PER;
__global__ void __launch_bounds__(SETUP_DT) tile_setup_kernel(const uint2* __restrict__ ranges, ViewSet views, int batch,
                                                               const uint32_t* key, uint32_t* __restrict__ cost,
                                                               uint32_t* __restrict__ cur_off,
                                                               uint64_t* __restrict__ cur_need,
                                                               uint32_t* __restrict__ order, uint32_t* nbatch) {
    __shared__ uint32_t h[256];
    __shared__ uint32_t s_w[SETUP_DT / 64];
    __shared__ uint32_t s_bin[4];
    const int t = threadIdx.x, lane = lane_id(), wid = t >> 6;
    if (t < 256) h[t] = 0u;
    __syncthreads();
    uint32_t c[SETUP_PER], bin[SETUP_PER];
    uint2 r1[SETUP_PER], r2[SETUP_PER];
#pragma unroll
    for (int k = 0; k < SETUP_PER; ++k) {  // the loads first
        const uint32_t i = min((uint32_t)(k * SETUP_DT + t), views.total_tiles - 1u);
        int vi = 0;
        while (vi + 1 < views.n_views && i >= views.v[vi + 1].tile_off) ++vi;
        const DevView& cam = views.v[vi];
        const uint32_t lt = i - cam.tile_off;
        const int ty = (int)(lt / (uint32_t)cam.grid_w), tx = (int)(lt - (uint32_t)ty * (uint32_t)cam.grid_w);
        r1[k] = ranges[i];
        r2[k] = ranges[region_of_tile(tx, ty, cam, views)];
        bin[k] = key ? key[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < SETUP_PER; ++k) {
        const uint32_t i = (uint32_t)(k * SETUP_DT + t);
        c[k] = 0u;
        if (i >= views.total_tiles) continue;
        const uint32_t len1 = r1[k].y - r1[k].x, len2 = r2[k].y - r2[k].x;
        c[k] = 2u * ((len1 + batch - 1) / batch + (len2 + batch - 1) / batch) + 2u;
        const uint32_t ck = min((len1 + len2) >> 3, 255u);
        cost[i] = ck;
        bin[k] = 255u - min(key ? bin[k] : ck, 255u);
        atomicAdd(&h[bin[k]], 1u);
    }
    // checkpoint offsets: exclusive prefix over the tiles in index order
    uint64_t carry = 0;
#pragma unroll
    for (int k = 0; k < SETUP_PER; ++k) {
        const uint32_t i = (uint32_t)(k * SETUP_DT + t);
        const uint32_t x = wave_add_scan(c[k]);
        if (lane == 63) s_w[wid] = x;
        __syncthreads();
        uint32_t wo = 0, tot = 0;
        for (int v = 0; v < SETUP_DT / 64; ++v) {
            if (v < wid) wo += s_w[v];
            tot += s_w[v];
        }
        if (i < views.total_tiles) cur_off[i] = (uint32_t)carry + wo + x - c[k];
        carry += tot;
        __syncthreads();  // s_w is written again
    }
    if (t == 0) *cur_need = carry;
    // bin starts, then the tiles in descending cost (ties in any order)
    uint32_t n = 0, x = 0;
    if (t < 256) {
        n = h[t];
        x = wave_add_scan(n);
        if (lane == 63) s_bin[wid] = x;
    }
    __syncthreads();
    if (t < 256) {
        for (int v = 0; v < wid; ++v) x += s_bin[v];
        h[t] = x - n;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SETUP_PER; ++k) {
        const uint32_t i = (uint32_t)(k * SETUP_DT + t);
        if (i >= views.total_tiles) continue;
        order[atomicAdd(&h[bin[k]], 1u)] = i;
        nbatch[i] = 0u;  // (key may be the same array: read above by this thread only)
    }
}

// ---------------------------------------------------------------------------
// merging two ordered streams in LDS
// ---------------------------------------------------------------------------

// Dynamic LDS of one workgroup for batch depth B: the staged records of the
// batch (3 float4 per entry) share their space with the merge windows, which
// are dead once the merged positions are known.
struct Lds {
    uint32_t* xk;     // narrow window (sorted positions)
    uint32_t* yraw;   // region window (sorted positions), before the tile test
    uint32_t* yk;     // entries of the region window that belong to this tile
    uint8_t* ypass;   // tile test of the region window
    // staged records of the batch, three float4 per entry (A, B, C): one
    // LDS address per entry, the three reads at fixed offsets
    float4* E;
    uint32_t* m;      // merged positions of the batch
    uint8_t* bm;      // the 4x4 blocks each staged entry can reach (kernels for small splats)
    uint32_t* wsum;   // per-wave partial counts
};

__host__ __device__ constexpr size_t lds_bytes(int batch) { return (size_t)batch * (48 + 4 + 1) + 64; }

__device__ __forceinline__ Lds carve(char* smem, int batch) {
    Lds L;
    L.E = reinterpret_cast<float4*>(smem);
    L.xk = reinterpret_cast<uint32_t*>(smem);
    L.yraw = L.xk + batch;
    L.yk = L.yraw + batch;
    L.ypass = reinterpret_cast<uint8_t*>(L.yk + batch);
    L.m = reinterpret_cast<uint32_t*>(smem + 48 * (size_t)batch);
    L.bm = reinterpret_cast<uint8_t*>(L.m + batch);
    L.wsum = reinterpret_cast<uint32_t*>(L.bm + batch);
    return L;
}

__device__ __forceinline__ int count_le(const uint32_t* a, int n, uint32_t key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] <= key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int count_lt(const uint32_t* a, int n, uint32_t key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Exclusive scan over a block of any multiple of 64 threads.
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* wsum, uint32_t* total) {
    const int lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        if (i < w) before += wsum[i];
        tot += wsum[i];
    }
    *total = tot;
    return before + x - v;
}

struct Batch {
    int M;      // staged entries (those that can reach a pixel of the tile)
    int Mfull;  // merged entries of the batch, staged or not
    int nX;     // narrow entries consumed
    int nYraw;  // region entries consumed (including those not belonging to the tile)
};

// Stages a record as entry j of the batch: a and gamma scaled for eval_entry,
// the entry's index k in the tile's full list in B.w (which held the radius,
// unused here), and, for the kernels for small splats, the blocks of the part
// at (qx0, qy0) it can reach.
template <bool FINE>
__device__ __forceinline__ void put_entry(const Lds& L, int j, const float4& A, const float4& B, const float4& C,
                                          int k, int qx0, int qy0, int height, const DevSettings& st) {
    float4 Bs = stage_b(B);
    Bs.w = __int_as_float(k);
    L.E[3 * j] = stage_a(A);
    L.E[3 * j + 1] = Bs;
    L.E[3 * j + 2] = C;
    if constexpr (FINE) L.bm[j] = (uint8_t)block_mask(A, B, qx0, qy0, height, st);
}

// ... the record at sorted position p
template <bool FINE>
__device__ __forceinline__ void stage_entry(const Lds& L, int j, const float4* __restrict__ srec, size_t p, int k,
                                            int qx0, int qy0, int height, const DevSettings& st) {
    put_entry<FINE>(L, j, srec[3 * p], srec[3 * p + 1], srec[3 * p + 2], k, qx0, qy0, height, st);
}

// Hides where a value comes from: what is computed from it is computed again
// behind this point, not kept in (spilled) registers from before it.
__device__ __forceinline__ void opaque(int& v) { asm volatile("" : "+v"(v)); }

// Stages the next (at most `batch`) entries of the tile's merged list in LDS.
// Every thread of the block calls it; the result is uniform.  The first
// stream is the tile's narrow list, the second its region list, of which
// only the entries that reach the tile belong to the tile's list: with
// culling, those that pass the exact touch test (narrow lists are already
// culled the same way, so every merged entry is staged); without, those
// whose tile rectangle contains the tile (the list of Sec. 3.1), and the
// touch test then only decides which merged entries are staged.
template <bool FINE>
__device__ Batch merge_batch(const Lds& L, const uint32_t* __restrict__ vals, const float4* __restrict__ srec,
                             int i1, int e1, int i2, int e2, int batch, int tcx, int tcy, const TileBox& tb,
                             const DevView& cam, const DevSettings& st, int kbase, int qx0 = 0, int qy0 = 0) {
    int t = threadIdx.x;
    opaque(t);
    const int NT = blockDim.x;
    if (st.tile_cull && i2 >= e2) {
        // no region entries left: the next narrow entries are the batch
        const int M = min(batch, e1 - i1);
        for (int j = t; j < M; j += NT) {
            const uint32_t p = vals[i1 + j];
            L.m[j] = p;
            stage_entry<FINE>(L, j, srec, p, kbase + j, qx0, qy0, cam.height, st);
        }
        __syncthreads();
        return Batch{uniform(M), uniform(M), uniform(M), 0};
    }
    const int cX = min(batch, e1 - i1), cY = min(batch, e2 - i2);
    for (int l = t; l < cX; l += NT) L.xk[l] = vals[i1 + l];
    for (int l = t; l < cY; l += NT) {
        const uint32_t p = vals[i2 + l];
        L.yraw[l] = p;
        const float4 A = srec[3 * (size_t)p], B = srec[3 * (size_t)p + 1];
        bool pass;
        if (st.tile_cull) {
            pass = may_touch(A, B, tb, st);
        } else {
            const Rect q = rect_of(A.x, A.y, B.w, cam, st);
            pass = tcx >= q.x0 && tcx <= q.x1 && tcy >= q.y0 && tcy <= q.y1;
        }
        L.ypass[l] = pass ? 1 : 0;
    }
    __syncthreads();
    // entries up to the smaller of the two window ends are final (positions
    // are below 2^31, so the all-ones value means "no bound")
    uint32_t F = 0xffffffffu;
    if (i1 + cX < e1) F = L.xk[cX - 1];
    if (i2 + cY < e2) F = min(F, L.yraw[cY - 1]);
    int nX = count_le(L.xk, cX, F);
    int nYr = count_le(L.yraw, cY, F);
    // compact the passing entries among the consumed raw ones
    const int per = (cY + NT - 1) / NT;
    uint32_t cnt = 0;
    for (int q = 0; q < per; ++q) {
        const int l = t * per + q;
        if (l < nYr) cnt += L.ypass[l];
    }
    uint32_t nYu;
    uint32_t pos = block_scan_excl(cnt, L.wsum, &nYu);
    for (int q = 0; q < per; ++q) {
        const int l = t * per + q;
        if (l < nYr && L.ypass[l]) L.yk[pos++] = L.yraw[l];
    }
    __syncthreads();
    int nY = (int)nYu;
    if (nX + nY > batch) {
        // keep the `batch` smallest: co-rank of the diagonal d = batch
        const int d = batch;
        int lo = max(0, d - nY), hi = min(d, nX);
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (L.xk[mid] < L.yk[d - mid - 1]) lo = mid + 1;
            else hi = mid;
        }
        const int a = lo;
        uint32_t last = 0;
        if (a > 0) last = L.xk[a - 1];
        if (d - a > 0) last = max(last, L.yk[d - a - 1]);
        nX = a;
        nY = d - a;
        nYr = count_le(L.yraw, nYr, last);
    }
    for (int a = t; a < nX; a += NT) L.m[a + count_lt(L.yk, nY, L.xk[a])] = L.xk[a];
    for (int b = t; b < nY; b += NT) L.m[b + count_lt(L.xk, nX, L.yk[b])] = L.yk[b];
    __syncthreads();
    // the windows are dead: stage over them, in merged order, the records
    // that can reach a pixel of the tile; an entry's index in the tile's full
    // list is kbase (the merged entries of the earlier batches) plus its
    // index within the merged batch
    const int M = nX + nY;
    if (st.tile_cull) {
        for (int j = t; j < M; j += NT) stage_entry<FINE>(L, j, srec, L.m[j], kbase + j, qx0, qy0, cam.height, st);
        __syncthreads();
        return Batch{uniform(M), uniform(M), uniform(nX), uniform(nYr)};
    }
    const int run = (M + NT - 1) / NT;  // contiguous entries per thread (<= MAXB / 64)
    uint32_t keep = 0, nkeep = 0;
    for (int q = 0; q < run; ++q) {
        const int j = t * run + q;
        if (j < M) {
            const size_t i = L.m[j];
            if (may_touch(srec[3 * i], srec[3 * i + 1], tb, st)) {
                keep |= 1u << q;
                ++nkeep;
            }
        }
    }
    uint32_t Mc;
    uint32_t p = block_scan_excl(nkeep, L.wsum, &Mc);
    for (int q = 0; q < run; ++q) {
        if (!((keep >> q) & 1u)) continue;
        const int j = t * run + q;
        stage_entry<FINE>(L, (int)p, srec, L.m[j], kbase + j, qx0, qy0, cam.height, st);
        ++p;
    }
    __syncthreads();
    return Batch{uniform((int)Mc), uniform(M), uniform(nX), uniform(nYr)};
}

// Wave totals of ten per-lane quantities, each left in the lanes that
// issue its atomic.  The gfx950 lane swaps halve the data without selects:
// permlane32_swap trades the upper half of its first operand for the lower
// half of its second, so the sum of its two results holds the first
// quantity's total over lanes l, l + 32 in the lower half and the second's in
// the upper half; permlane16_swap trades rows 1 and 3 of its first operand
// for rows 0 and 2 of its second, which halves again across the row pairs.
// Four DPP steps within each 16-lane row then complete the totals.
__device__ __forceinline__ float dpp_xor1(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xb1, 0xf, 0xf, false));
}
__device__ __forceinline__ float dpp_xor2(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4e, 0xf, 0xf, false));
}
__device__ __forceinline__ float dpp_ror4(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false));
}
__device__ __forceinline__ float dpp_ror8(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false));
}
__device__ __forceinline__ float halves_pair(float a, float b) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float rows_pair(float a, float b) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// total over the 16 lanes of each row, in every lane of the row
__device__ __forceinline__ float row_total(float x) {
    x += dpp_ror8(x);
    x += dpp_ror4(x);
    x += dpp_xor2(x);
    return x + dpp_xor1(x);
}

// the same for maxima
__device__ __forceinline__ float halves_pair_max(float a, float b) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float rows_pair_max(float a, float b) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float row_max(float x) {
    x = fmaxf(x, dpp_ror8(x));
    x = fmaxf(x, dpp_ror4(x));
    x = fmaxf(x, dpp_xor2(x));
    return fmaxf(x, dpp_xor1(x));
}

// Quantity whose wave total lane holds after wave_sum_swap10 (-1: none).
// Column 0 of the rows holds quantities 0, 2, 1, 3 (rows 0 to 3), column 1
// quantities 4, 6, 5, 7, column 2 of rows 0 and 2 quantities 8 and 9.
__device__ __forceinline__ int swap10_quantity(int lane) {
    const int row = lane >> 4, c = lane & 15;
    if (c == 0) return (row & 1) * 2 + (row >> 1);
    if (c == 1) return 4 + (row & 1) * 2 + (row >> 1);
    if (c == 2 && (row & 1) == 0) return 8 + (row >> 1);
    return -1;
}

__device__ __forceinline__ float wave_sum_swap10(const float (&v)[10], int lane) {
    const float s0 = halves_pair(v[0], v[1]), s1 = halves_pair(v[2], v[3]), s2 = halves_pair(v[4], v[5]);
    const float s3 = halves_pair(v[6], v[7]), s4 = halves_pair(v[8], v[9]);
    const float t0 = row_total(rows_pair(s0, s1));  // rows: quantities 0, 2, 1, 3
    const float t1 = row_total(rows_pair(s2, s3));  // rows: 4, 6, 5, 7
    const float t2 = row_total(rows_pair(s4, s4));  // rows: 8, 8, 9, 9
    const int c = lane & 15;
    return c == 0 ? t0 : (c == 1 ? t1 : t2);
}

// Pixel of slot i of thread t: every wave's slot covers one 8x8 block of
// the tile (block w PPT + i of the tile's TW / 8 x TH / 8 blocks), so that an
// entry whose footprint covers part of the tile leaves fewer lanes idle than
// with rows of the tile per slot.
template <int TW, int PPT>
__device__ __forceinline__ void pixel_of(int t, int i, const TileGeom& tg, int& x, int& y) {
    const int b = (t >> 6) * PPT + i, l = t & 63;
    x = tg.tx0 + (b % (TW / 8)) * 8 + (l & 7);
    y = tg.ty0 + (b / (TW / 8)) * 8 + (l >> 3);
}

// Words of Lds::wsum behind the scan's, of the workgroup's staged-list chunk:
// next free entry, entries left, where the batch's entries go (both
// STG_NOWHERE: nowhere).
constexpr int STG_BASE = 8, STG_LEFT = 9, STG_OFF = 10;

struct HybridLists {
    const uint32_t* vals;      // list entries (sorted positions) in (cell, position) order
    const uint2* ranges;       // [start, end) per tile, then per region
    uint4* cur;                // batch checkpoints (narrow cursor, region cursor, merged index)
    const uint32_t* cur_off;   // first checkpoint of each tile
    uint32_t* nbatch;          // batches the forward took per tile
    const uint64_t* cur_need;  // checkpoints the tiles may take (device)
    uint64_t cur_cap;          // checkpoints the buffer holds
    uint32_t* flags;
    // entries the forward staged per batch, kept for the backward:
    // per checkpoint (offset into stg or all ones, count), and per staged
    // entry (sorted position, index within the merged batch)
    uint2* cur_stg;
    uint2* stg;                // null: the backward merges again
    uint32_t* stg_count;       // the next chunk, in units of STG_CHUNK entries (behind the first chunks)
    uint32_t stg_cap;
    double* drec_clear;        // the backward's FP64 accumulators, cleared by the forward
    uint64_t drec_clear_n2;    // their size in pairs of doubles
    const uint32_t* order;     // optional: tile of each workgroup
};

// Tile-wide compositing, one workgroup per tile in launch order.  Both kernels
// are bound by instruction issue, and take no loop over a device queue: with
// the loop, the launch's arguments stay live in registers across it, and
// resident workgroups that pop one counter wait for each other.  What the tile
// and the batch determine is read into scalar registers (`uniform`), so that a
// thread holds its pixels and the entry only: 56 registers for the forward at
// two pixels per thread (72 and spills before), 90 for the backward at four.
// Measured on splats of an unbounded scene, batches of 128, two pixels per
// thread forward and four backward, queue loop -> now: 4,346 tiles forward 143
// -> 64 us, backward 186 -> 152 us; 8,664 tiles 222 -> 134 and 317 -> 252 us;
// 24,937 tiles 432 -> 341 and 663 -> 585 us (of the forward, the tests every
// 16 entries as a loop of their own: 69 -> 64, 147 -> 134 and 362 -> 341 us).
// With the counters, batches of 256, one workgroup per tile before and after:
// 4,346 tiles 107 -> 86 us, 24,937 tiles 512 -> 480 us.
// Waves per SIMD the register use is held to: forward eight (seven with the
// counters, which at eight spill: 485 -> 505 us at 24,937 tiles), backward
// five (six spill at four pixels per thread: 254 -> 268 us at 8,664 tiles).
// STATS: write the per-pixel work counters (stats_out, eval_out).
// IMP: accumulate every Gaussian's blending weights M alpha T over the
// pixels it enters: the tile's sum (of FP32 sums over the waves, in FP64) into
// imp_sum and its maximum (as float bits, the weights being non-negative) into
// imp_max.
template <int TW, int TH, int PPT, bool STATS, bool IMP>
__global__ void __launch_bounds__(TW * TH / PPT, PPT >= 4 ? 5 : STATS ? 7 : 8) hybrid_fwd_kernel(
    const float4* __restrict__ srec, HybridLists hl, ViewSet views, DevSettings st, float* __restrict__ images,
    float* __restrict__ t_final, int32_t* __restrict__ last_out, int4* __restrict__ stats_out,
    int4* __restrict__ eval_out, int64_t n, double* __restrict__ imp_sum,
    uint32_t* __restrict__ imp_max) {
    constexpr int NT = TW * TH / PPT;
    // entries per round: with IMP four, whose reductions over the wave share
    // their steps (2 views of 400 k Gaussians: 154 -> 138 us against one)
    constexpr int ROUND = IMP ? 4 : 1;
    // IMP: the batch's sums and maxima over the tile, added to the Gaussians'
    // once per tile, a lane to an entry (138 -> 102 us against atomics of
    // every wave and round); zero between batches
    __shared__ double s_isum[IMP ? MAXB : 1];
    __shared__ uint32_t s_imax[IMP ? MAXB : 1];
    extern __shared__ __align__(16) char smem[];
    int t = threadIdx.x;
    const int batch = st.batch;
    const Lds L = carve(smem, batch);
    const EvalConsts ek = eval_consts(st);
    if (*hl.cur_need > hl.cur_cap) {  // a fixed workspace too small: report, write nothing
        if (blockIdx.x == 0 && t == 0) atomicOr(hl.flags, FLAG_CAPACITY);
        return;
    }
    // staged-list chunk of this workgroup (used by thread 0 only)
    if (hl.stg && t == 0) {
        const uint32_t first = staged_first(gridDim.x);
        L.wsum[STG_BASE] = staged_first_base(blockIdx.x, first);
        L.wsum[STG_LEFT] = first;
    }
    const uint32_t tile = uniform(hl.order ? hl.order[blockIdx.x] : blockIdx.x);
    const TileGeom tg = tile_geom(views, tile, TW, TH);
    if constexpr (IMP) {
        for (int p = t; p < MAXB; p += NT) {
            s_isum[p] = 0.0;
            s_imax[p] = 0u;
        }
    }
    const DevView& cam = views.v[tg.vi];
    float px[PPT], py[PPT], T[PPT], C0[PPT], C1[PPT], C2[PPT];
    // stopk: the entry at which the pixel stopped, -1 while it runs
    // (and 0 for a pixel outside the view, which never runs): the
    // pixel's done flag, tested with one compare per slot and entry; its
    // value changes only when the pixel stops
    // (STATS: nev, nev_last: staged entries up to the one at which the
    // pixel stopped and up to the one it blended last, from the entry's
    // place in the staged order, so that an entry a pixel skips costs no
    // counter; staged: entries staged in the batches before)
    int last[PPT], stopk[PPT], nblend[PPT], nmasked[PPT], nev[PPT], nev_last[PPT];
    int staged = 0;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        int x, y;
        pixel_of<TW, PPT>(t, i, tg, x, y);
        const bool inside = x < cam.width && y < cam.height;
        px[i] = (float)x + 0.5f;
        py[i] = (float)y + 0.5f;
        T[i] = 1.f;
        C0[i] = C1[i] = C2[i] = 0.f;
        last[i] = -1;
        stopk[i] = inside ? -1 : 0;
        nblend[i] = nmasked[i] = nev[i] = nev_last[i] = 0;
    }
    const int tcx = tg.tx0 / TW, tcy = tg.ty0 / TH;
    const uint2 r1 = uniform(hl.ranges[tile]);
    const uint2 r2 = uniform(hl.ranges[region_of_tile(tcx, tcy, cam, views)]);
    const int e1 = (int)r1.y, e2 = (int)r2.y;
    int i1 = (int)r1.x, i2 = (int)r2.x, m = 0, b = 0;
    const TileBox tb{(float)tg.tx0 + 0.5f, (float)min(tg.tx0 + TW, cam.width) - 0.5f, (float)tg.ty0 + 0.5f,
                     (float)min(tg.ty0 + TH, cam.height) - 0.5f};
    uint4* cur = hl.cur + uniform(hl.cur_off[tile]);
    while (i1 < e1 || i2 < e2) {
        bool active = false;
#pragma unroll
        for (int i = 0; i < PPT; ++i) active |= stopk[i] < 0;
        if (!__syncthreads_or(active)) break;
        if (t == 0) cur[b] = make_uint4((uint32_t)i1, (uint32_t)i2, (uint32_t)m, 0u);
        const Batch bt =
            merge_batch<false>(L, hl.vals, srec, i1, e1, i2, e2, batch, tcx, tcy, tb, cam, st, m);
        // room for the staged entries in the list kept for the backward:
        // thread 0 sub-allocates from a chunk the workgroup took from the
        // global counter (one atomic per chunk, not per batch)
        if (hl.stg && t == 0) {
            uint32_t cbase = L.wsum[STG_BASE], cleft = L.wsum[STG_LEFT];
            if ((uint32_t)bt.M > cleft) {
                cbase = staged_base(atomicAdd(hl.stg_count, 1u));
                cleft = STG_CHUNK;
            }
            const uint32_t off = staged_offset(cbase, (uint32_t)bt.M, hl.stg_cap);
            L.wsum[STG_OFF] = off;
            L.wsum[STG_BASE] = staged_next(off, (uint32_t)bt.M);
            L.wsum[STG_LEFT] = cleft - (uint32_t)bt.M;
            hl.cur_stg[hl.cur_off[tile] + b] = make_uint2(off, (uint32_t)bt.M);
        }
        for (int j0 = 0; j0 < bt.M; j0 += 16) {
            // the wave leaves the batch once all its pixels are done,
            // tested every 16 entries (a done pixel's slot costs only
            // its skip; a test per entry costs more than it saves)
            active = false;
#pragma unroll
            for (int i = 0; i < PPT; ++i) active |= stopk[i] < 0;
            if (!__any(active)) break;
            const int j1 = min(j0 + 16, bt.M);
            int j = j0;
            do {
                float isum[ROUND], imax[ROUND];
#pragma unroll
                for (int u = 0; u < ROUND; ++u) {
                    const int je = j + u;
                    isum[u] = imax[u] = 0.f;
                    if (u > 0 && je >= j1) continue;  // uniform
                    const float4 A = L.E[3 * je], B = L.E[3 * je + 1], Cc = L.E[3 * je + 2];
                    const int k = __float_as_int(B.w);  // index in the tile's full list
#pragma unroll
                    for (int i = 0; i < PPT; ++i) {
                        if (stopk[i] >= 0) continue;
                        Eval e;
                        if (!eval_entry(A, B, px[i], py[i], ek, e)) continue;
                        const float ma = B.z * e.alpha;
                        const float test = T[i] * (1.f - ma);
                        // one select, not a branch with copies on both sides
                        const bool stop = test < st.t_min;
                        stopk[i] = stop ? k : stopk[i];
                        asm volatile("" : "+v"(stopk[i]));  // keeps the select here
                        if (STATS) nev[i] = staged + je + 1;  // the last entry that passed the cuts
                        if (stop) continue;
                        const float wgt = ma * T[i];
                        C0[i] += wgt * Cc.x;
                        C1[i] += wgt * Cc.y;
                        C2[i] += wgt * Cc.z;
                        T[i] = test;
                        last[i] = k;
                        if (STATS) {
                            ++nblend[i];
                            nmasked[i] += B.z == 0.f;
                            nev_last[i] = nev[i];
                        }
                        if (IMP) {
                            isum[u] += wgt;
                            imax[u] = fmaxf(imax[u], wgt);
                        }
                    }
                }
                if constexpr (IMP) {
                    // the four entries' sums and maxima over the wave, each
                    // entry's in one row, whose first lane adds them
                    if (ballot((isum[0] > 0.f) | (isum[1] > 0.f) | (isum[2] > 0.f) | (isum[3] > 0.f))) {
                        const float ws = row_total(rows_pair(halves_pair(isum[0], isum[1]),
                                                             halves_pair(isum[2], isum[3])));
                        const float wm = row_max(rows_pair_max(halves_pair_max(imax[0], imax[1]),
                                                               halves_pair_max(imax[2], imax[3])));
                        const int row = lane_id() >> 4;  // rows: entries 0, 2, 1, 3
                        const int je = j + (row >> 1) + 2 * (row & 1);
                        if ((lane_id() & 15) == 0 && je < j1 && !(ws <= 0.f)) {
                            atomicAdd(&s_isum[je], (double)ws);
                            atomicMax(&s_imax[je], __float_as_uint(wm));
                        }
                    }
                }
                j += ROUND;
            } while (j < j1);
        }
        active = false;
#pragma unroll
        for (int i = 0; i < PPT; ++i) active |= stopk[i] < 0;
        if (hl.stg) {
            __syncthreads();
            const uint32_t off = L.wsum[STG_OFF];
            if (off != STG_NOWHERE) {
                for (int p = t; p < bt.M; p += NT) {
                    const uint32_t jj = __float_as_uint(L.E[3 * p + 1].w) - (uint32_t)m;
                    hl.stg[off + p] = make_uint2(L.m[jj], jj);
                }
            }
        }
        if constexpr (IMP) {
            __syncthreads();
            for (int p = t; p < bt.M; p += NT) {
                const double ws = s_isum[p];
                if (ws == 0.0) continue;
                const int64_t g = (int64_t)__float_as_uint(L.E[3 * p + 2].w) - (int64_t)tg.vi * n;
                atomicAdd(imp_sum + g, ws);
                atomicMax(imp_max + g, s_imax[p]);
                s_isum[p] = 0.0;
                s_imax[p] = 0u;
            }
        }
        i1 += bt.nX;
        i2 += bt.nYraw;
        m += bt.Mfull;
        if (STATS) staged += bt.M;
        ++b;
        __syncthreads();  // the next batch overwrites the LDS
    }
    opaque(t);
    if (t == 0) hl.nbatch[tile] = (uint32_t)b;
    if (hl.drec_clear) {
        // the backward's FP64 accumulator of per-record gradients is
        // cleared here, one slice per tile: this kernel is bound by VALU
        // issue and leaves HBM bandwidth idle, the projection backward
        // (HBM-bound) then only reads the rows
        const uint64_t per = (hl.drec_clear_n2 + views.total_tiles - 1) / views.total_tiles;
        const uint64_t q0 = (uint64_t)tile * per;
        const uint64_t q1 = min(q0 + per, hl.drec_clear_n2);
        double2* z = reinterpret_cast<double2*>(hl.drec_clear);
        for (uint64_t q = q0 + (uint64_t)t; q < q1; q += NT) z[q] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        int x, y;
        pixel_of<TW, PPT>(t, i, tg, x, y);
        if (x >= cam.width || y >= cam.height) continue;
        const int64_t pv = (int64_t)cam.width * cam.height;
        const int64_t loc = (int64_t)y * cam.width + x;
        float* im = images + 3 * (int64_t)cam.px_off;
        im[loc] = C0[i] + T[i] * st.bg[0];
        im[pv + loc] = C1[i] + T[i] * st.bg[1];
        im[2 * pv + loc] = C2[i] + T[i] * st.bg[2];
        const int64_t p = (int64_t)cam.px_off + loc;
        t_final[p] = T[i];
        last_out[p] = last[i];
        // a pixel that never stopped saw the whole merged list (m entries);
        // entries it evaluated are those of the list that can reach the tile
        if (STATS) {
            stats_out[p] = make_int4(stopk[i] >= 0 ? stopk[i] + 1 : m, nblend[i], nmasked[i], last[i] + 1);
            eval_out[p] = make_int4(stopk[i] >= 0 ? nev[i] : staged, nev_last[i], 0, 0);
        }
    }
}

// SUM (several waves to a tile): the waves' totals of BWD_ROUND entries meet in
// LDS and are added to the accumulators once per tile and entry, a lane to a
// quantity: fewer atomics, which wait for each other where tiles reach the same
// splats at the same time, for two barriers a round.  Splats of an unbounded
// scene, 1,392 to 24,937 tiles of 256 pixels, summed against every wave for
// itself:
//   one pixel per thread (two or four waves): 0.45 to 0.94 of the time at any
//   number of tiles and batch depth (4,346 tiles 349 -> 188 us, 24,937 tiles
//   1,450 -> 1,060 us)
//   two pixels per thread (two waves), batches of 32 to 128: 0.74 to 1.02 (4,346
//   tiles 220 -> 167, 8,664 tiles 305 -> 294, 24,937 tiles 785 -> 747 us)
//   two pixels per thread, batches of 256 (whose LDS leaves room for fewer
//   workgroups with the sums): 1,392 tiles 104 / 107 us, 4,346 tiles 237 /
//   174, 6,000 tiles 256 / 253, 7,110 tiles 320 / 279, 7,740 tiles 302 / 309,
//   8,664 tiles 320 / 334, 24,937 tiles 778 / 838
// So the waves sum, but with two pixels per thread and batches of 256 only up
// to SUM_TILES tiles.
constexpr int BWD_ROUND = 32;
constexpr uint32_t SUM_TILES = 7424;
template <int TW, int TH, int PPT, bool SUM>
__global__ void __launch_bounds__(TW * TH / PPT, 5) hybrid_bwd_kernel(
    const float4* __restrict__ srec, HybridLists hl, ViewSet views, DevSettings st, const float* __restrict__ t_final,
    const int32_t* __restrict__ last_in, const float* __restrict__ dl_dimages, int64_t n, double* __restrict__ d_rec,
    double* __restrict__ d_masks) {
    constexpr int NT = TW * TH / PPT, NW = SUM ? NT / 64 : 1;
    // SUM: the waves' totals of BWD_ROUND entries; zero between rounds
    __shared__ float s_acc[SUM ? NW * BWD_ROUND * 10 : 1];
    extern __shared__ __align__(16) char smem[];
    __shared__ int s_top;
    const int t = threadIdx.x;
    const int lane = lane_id();
    const int batch = st.batch;
    const Lds L = carve(smem, batch);
    const float bg0 = st.bg[0], bg1 = st.bg[1], bg2 = st.bg[2];
    const EvalConsts ek = eval_consts(st);
    // the quantity whose wave total this lane adds into the accumulator
    // (-1: none); the totals of the sums over t^2 and dy^2 (quantities 2
    // and 4) are rescaled by QSCALE / 2 to give dL/da and dL/dgamma (see the
    // pixel loop)
    const int qi = swap10_quantity(lane);
    const float qscale = (qi == 2 || qi == 4) ? 0.5f * QSCALE : 1.f;
    if (*hl.cur_need > hl.cur_cap) return;  // the forward reported it
    const uint32_t tile = uniform(hl.order ? hl.order[blockIdx.x] : blockIdx.x);
    const TileGeom tg = tile_geom(views, tile, TW, TH);
    const DevView& cam = views.v[tg.vi];
    const int64_t rec_base = (int64_t)tg.vi * n;
    // s = w . b: the loss weights of the pixel dotted with the colour
    // composited behind the current entry (scaled by its transmittance)
    float px[PPT], py[PPT], T[PPT], Tf[PPT], w0[PPT], w1[PPT], w2[PPT], wbg[PPT], sb[PPT];
    int lastk[PPT];
    int mylast = -1;
    const int64_t pv = (int64_t)cam.width * cam.height;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
        int x, y;
        pixel_of<TW, PPT>(t, i, tg, x, y);
        px[i] = (float)x + 0.5f;
        py[i] = (float)y + 0.5f;
        sb[i] = 0.f;
        if (x < cam.width && y < cam.height) {
            const int64_t loc = (int64_t)y * cam.width + x;
            const int64_t p = (int64_t)cam.px_off + loc;
            const float* dl = dl_dimages + 3 * (int64_t)cam.px_off;
            lastk[i] = last_in[p];
            Tf[i] = t_final[p];
            w0[i] = dl[loc];
            w1[i] = dl[pv + loc];
            w2[i] = dl[2 * pv + loc];
        } else {
            lastk[i] = -1;
            Tf[i] = 1.f;
            w0[i] = w1[i] = w2[i] = 0.f;
        }
        T[i] = Tf[i];
        wbg[i] = w0[i] * bg0 + w1[i] * bg1 + w2[i] * bg2;
        mylast = max(mylast, lastk[i]);
    }
    for (int off = 32; off > 0; off >>= 1) mylast = max(mylast, __shfl_xor(mylast, off));
    if (t == 0) s_top = -1;
    __syncthreads();
    if (lane == 0) atomicMax(&s_top, mylast);
    __syncthreads();
    const int top = uniform(s_top);
    const uint4* cur = hl.cur + uniform(hl.cur_off[tile]);
    const int tcx = tg.tx0 / TW, tcy = tg.ty0 / TH;
    const uint2 r1 = uniform(hl.ranges[tile]);
    const uint2 r2 = uniform(hl.ranges[region_of_tile(tcx, tcy, cam, views)]);
    const TileBox tb{(float)tg.tx0 + 0.5f, (float)min(tg.tx0 + TW, cam.width) - 0.5f, (float)tg.ty0 + 0.5f,
                     (float)min(tg.ty0 + TH, cam.height) - 0.5f};
    // the batch holding the largest last-blended entry, then backwards
    int bstar = -1;
    if (top >= 0) {
        const int nb = (int)hl.nbatch[tile];
        for (int b = 0; b < nb; ++b)
            if ((int)cur[b].z <= top) bstar = b;
    }
    float* acc = s_acc + (SUM ? (t >> 6) * BWD_ROUND * 10 : 0);
    if constexpr (SUM)
        for (int i = t; i < NW * BWD_ROUND * 10; i += NT) s_acc[i] = 0.f;
    const uint2* cstg = hl.stg ? hl.cur_stg + uniform(hl.cur_off[tile]) : nullptr;
    // per-entry partial sums of this lane's pixels; zero between entries
    // (reset after each reduction), so no per-entry initialisation
    float gu = 0.f, gv = 0.f, ga = 0.f, gb = 0.f, gc = 0.f, go = 0.f, gr = 0.f, gg = 0.f, gbl = 0.f, gm = 0.f;
    for (int b = bstar; b >= 0; --b) {
        const uint4 c = cur[b];
        const int m = (int)c.z;
        const uint2 cs = cstg ? cstg[b] : make_uint2(STG_NOWHERE, 0u);
        int Mb;
        if (cs.x != STG_NOWHERE) {
            // the entries the forward staged for this batch
            Mb = (int)cs.y;
            for (int p = t; p < Mb; p += NT) {
                const uint2 e = hl.stg[cs.x + p];
                const size_t i = e.x;
                float4 B = stage_b(srec[3 * i + 1]);
                B.w = __int_as_float(m + (int)e.y);
                L.E[3 * p] = stage_a(srec[3 * i]);
                L.E[3 * p + 1] = B;
                L.E[3 * p + 2] = srec[3 * i + 2];
            }
            __syncthreads();
        } else {
            Mb = merge_batch<false>(L, hl.vals, srec, (int)c.x, (int)r1.y, (int)c.y, (int)r2.y, batch, tcx,
                                        tcy, tb, cam, st, m).M;
        }
        for (int j1 = Mb; j1 > 0; j1 -= BWD_ROUND) {
            const int j0 = SUM ? max(j1 - BWD_ROUND, 0) : 0;
            for (int j = j1 - 1; j >= j0; --j) {
                const float4 A = L.E[3 * j], B = L.E[3 * j + 1], Cc = L.E[3 * j + 2];
                const int k = __float_as_int(B.w);  // index in the tile's full list
                if (k > top) continue;                  // uniform: past every pixel's last entry
                const float M = B.z;
                const float okq = B.y * QSCALE_NINV;
                bool any = false;
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    if (k > lastk[i]) continue;
                    Eval e;
                    if (!eval_entry(A, B, px[i], py[i], ek, e)) continue;
                    any = true;
                    const float ma = M * e.alpha;
                    const float one_m = 1.f - ma;
                    const float inv = __builtin_amdgcn_rcpf(one_m);
                    const float Ti = T[i] * inv;
                    const float d = fmaf(w0[i], Cc.x, fmaf(w1[i], Cc.y, w2[i] * Cc.z)) - sb[i];
                    const float X = Ti * d - Tf[i] * inv * wbg[i];
                    gm += e.alpha * X;
                    const float wt = ma * Ti;
                    gr += wt * w0[i];
                    gg += wt * w1[i];
                    gbl += wt * w2[i];
                    if (e.oG <= ek.amax) {
                        // dL/dalpha = M X, dL/dQ = -o G M X / 2; with a' = QSCALE a,
                        // gamma' = QSCALE gamma: dL/du = kq a' t, dL/dv =
                        // kq (beta a' t + gamma' dy), dL/dbeta = kq a' t dy, and
                        // dL/da, dL/dgamma are QSCALE / 2 times the sums of kq t^2,
                        // kq dy^2, where kq = 2 dL/dQ / QSCALE
                        const float GdA = e.G * (M * X);
                        go += GdA;
                        const float kq = GdA * okq;
                        const float kapt = kq * e.apt;
                        gu += kapt;
                        gv += kq * fmaf(A.w, e.apt, e.gdy);
                        gb += kapt * e.dy;
                        ga += (kq * e.t) * e.t;
                        gc += (kq * e.dy) * e.dy;
                    }
                    sb[i] = fmaf(ma, d, sb[i]);
                    T[i] = Ti;
                }
                if (__any(any)) {
                    const uint32_t r = __float_as_uint(Cc.w);
                    const int64_t g = (int64_t)r - rec_base;
                    if (M != 0.f) {
                        // ten lanes receive the wave totals, quantity qi each
                        const float v[10] = {gu, gv, ga, gb, gc, go, gr, gg, gbl, gm};
                        const float x = wave_sum_swap10(v, lane) * qscale;
                        if constexpr (SUM) {
                            if (qi >= 0) acc[(j - j0) * 10 + qi] = x;
                        } else {
                            if ((unsigned)qi < (unsigned)DREC) atomicAdd(d_rec + (size_t)r * DREC + qi, (double)x);
                            else if (qi == DREC) atomicAdd(d_masks + g, (double)x);
                        }
                    } else {
                        const float sm = wave_sum(gm);
                        if (lane == 0) {
                            if constexpr (SUM) acc[(j - j0) * 10 + DREC] = sm;
                            else atomicAdd(d_masks + g, (double)sm);
                        }
                    }
                    gu = gv = ga = gb = gc = go = gr = gg = gbl = gm = 0.f;
                }
        
            }
            if constexpr (!SUM) break;  // the whole batch
            __syncthreads();
            for (int i = t; i < (j1 - j0) * 10; i += NT) {
                double x = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    x += (double)s_acc[w * BWD_ROUND * 10 + i];
                    s_acc[w * BWD_ROUND * 10 + i] = 0.f;
                }
                if (x == 0.0) continue;
                const int j = i / 10, q = i - j * 10;
                const uint32_t r = __float_as_uint(L.E[3 * (j0 + j) + 2].w);
                if (q < DREC) atomicAdd(d_rec + (size_t)r * DREC + q, x);
                else atomicAdd(d_masks + ((int64_t)r - rec_base), x);
            }
            __syncthreads();
        }
        __syncthreads();  // the next batch overwrites the LDS
    }
}

// ---------------------------------------------------------------------------
// compositing of small splats: four list entries of a 4x4 pixel block at a time
// ---------------------------------------------------------------------------

// A wave of the kernels above takes a tile's entries one after the other; a
// wave that has its SIMD to itself needs about 650 (forward) and 1100
// (backward) cycles per entry, and where splats are small, most pixels of the
// tile evaluate an entry in vain and a few long lists decide the launch's
// time.  Here a workgroup of four waves owns an 8x8 pixel part of a tile and
// each wave a 4x4 block of it.  The block's list is the staged batch without
// the entries that cannot reach the block, and the wave's four 16-lane rows
// take four consecutive entries of it at a time; the transmittance passes
// along the rows through the gfx950 lane swaps.  Per pixel and entry this
// issues about three times the instructions of the kernels above, so it pays
// where splats reach a fraction of the tile or the tiles leave the device idle
// (rule: use_fine).  Measured against the kernels above, which then popped a
// device queue: 200 k small splats at 800x800, 16x16 tiles with the work
// counters, forward 304 -> 77 us, backward 449 -> 109 us; 8x8 tiles without
// them 291 -> 66 and 321 -> 105 us; 4096 splats at 128x128, 216 -> 33 and 336
// -> 42 us.  The forward issues VALU instructions at 0.41 to 0.65 of the chip's
// rate and the backward at 0.5 to 0.58 (200 k splats), and their waves wait half
// of the time: a few parts hold long lists, whose entries depend on each other.
// Launches are plain (one workgroup per part, the tiles in launch order): a loop
// over a device queue keeps the kernel arguments live and spills more (forward
// 97 -> 80 us without it).  At six waves per SIMD the forward spills 36 bytes a
// lane, with the counters or the scores 56.
constexpr int FINE_NT = 256;
constexpr int FINE_BATCH = 256;  // entries per batch: one per thread

// Row exchanges of a value x with rows (x0, x1, x2, x3): the even and the odd
// row of each row pair (x0, x0, x2, x2), (x1, x1, x3, x3); the lower and the
// upper half (xa, xa), (xb, xb).
struct Rows2 {
    float lo, hi;
};
__device__ __forceinline__ Rows2 row_pairs(float x) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return Rows2{__uint_as_float(s[0]), __uint_as_float(s[1])};
}
__device__ __forceinline__ Rows2 row_halves(float x) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return Rows2{__uint_as_float(s[0]), __uint_as_float(s[1])};
}
// maximum and sum over the four rows, per column
__device__ __forceinline__ int rows_max(int x) {
    const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    const int y = max((int)a[0], (int)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)y, (uint32_t)y, false, false);
    return max((int)b[0], (int)b[1]);
}
__device__ __forceinline__ int rows_add(int x) {
    const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    const int y = (int)(a[0] + a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)y, (uint32_t)y, false, false);
    return (int)(b[0] + b[1]);
}
// The bit of row r and this lane's column in a mask over the wave's lanes.
__device__ __forceinline__ bool row_in_all_rows(uint64_t mask, int r) {
    uint32_t m = (uint32_t)(mask >> (16 * r)) & 0xffffu;
    m |= m << 16;
    return __builtin_amdgcn_inverse_ballot_w64((uint64_t)m << 32 | m);
}

// LDS of one workgroup after the staging area of lds_bytes: per wave the
// block's list (byte offsets of its entries in L.E, two rounds of padding)
// and, in the backward, twice ten partial sums per staged entry.
constexpr int FINE_LIST = FINE_BATCH + 8;
constexpr size_t fine_lds_bytes(bool bwd) {
    return lds_bytes(FINE_BATCH) + (FINE_NT / 64) * FINE_LIST * 2 + (bwd ? 2 * FINE_BATCH * 40 : 0);
}

// Part q of a launch over the 8x8 parts of every tile, tiles in launch order.
struct FinePart {
    uint32_t tile;
    TileGeom tg;
    int qx0, qy0;  // first pixel of the part
};
__device__ __forceinline__ FinePart fine_part(const ViewSet& views, const HybridLists& hl, const DevSettings& st,
                                              uint32_t q, uint32_t parts) {
    FinePart f;
    const uint32_t s = q / parts, part = q - s * parts;
    f.tile = hl.order ? hl.order[s] : s;
    f.tg = tile_geom(views, f.tile, st.tile_w, st.tile_h);
    const uint32_t pw = (uint32_t)st.tile_w / 8u;
    f.qx0 = f.tg.tx0 + (int)(part % pw) * 8;
    f.qy0 = f.tg.ty0 + (int)(part / pw) * 8;
    return f;
}

// The staged entries that can reach this wave's block (and have index at most
// kmax in the tile's list) as a list of their offsets in order, followed by
// zeros; returns their number (uniform).  LDS operations of one wave complete
// in program order.
__device__ __forceinline__ int block_list(const Lds& L, int M, int wave, int lane, int kmax, uint16_t* list) {
    uint32_t bm[FINE_BATCH / 64];
    int k[FINE_BATCH / 64];
#pragma unroll
    for (int i = 0; i < FINE_BATCH / 64; ++i) {
        const int j = 64 * i + lane;
        bm[i] = L.bm[j];
        k[i] = __float_as_int(L.E[3 * j + 1].w);
    }
    int n = 0;
#pragma unroll
    for (int i = 0; i < FINE_BATCH / 64; ++i) {
        const int j = 64 * i + lane;
        const bool in = (j < M) & (((bm[i] >> wave) & 1u) != 0) & (k[i] <= kmax);
        const uint64_t m = ballot(in);
        if (in) list[n + (int)__popcll(m & lanemask_lt())] = (uint16_t)(48 * j);
        n += (int)__popcll(m);
    }
    if (lane < 8) list[n + lane] = 0;
    __builtin_amdgcn_wave_barrier();
    return n;
}

// A part's batches.  While a batch whose tile has no region entries left is
// composited, the thread's record of the next batch and its position of the
// one after are on their way.
struct FineStream {
    float4 A, B, C;
    uint32_t p, pn;
    bool have;  // A, B, C, p hold the next batch's record (uniform)
};

__device__ __forceinline__ Batch fine_batch(const Lds& L, FineStream& fs, const HybridLists& hl,
                                            const float4* __restrict__ srec, int i1, int e1, int i2, int e2, int tcx,
                                            int tcy, const TileBox& tb, const DevView& cam, const DevSettings& st,
                                            int kbase, int qx0, int qy0) {
    if (!(st.tile_cull && i2 >= e2)) {
        fs.have = false;
        return merge_batch<true>(L, hl.vals, srec, i1, e1, i2, e2, FINE_BATCH, tcx, tcy, tb, cam, st, kbase, qx0, qy0);
    }
    const int t = threadIdx.x;
    const int M = min(FINE_BATCH, e1 - i1);
    if (!fs.have) {
        fs.p = t < M ? hl.vals[i1 + t] : 0u;
        if (t < M) {
            fs.A = srec[3 * (size_t)fs.p];
            fs.B = srec[3 * (size_t)fs.p + 1];
            fs.C = srec[3 * (size_t)fs.p + 2];
        }
        fs.pn = i1 + FINE_BATCH + t < e1 ? hl.vals[i1 + FINE_BATCH + t] : 0u;
    }
    if (t < M) put_entry<true>(L, t, fs.A, fs.B, fs.C, kbase + t, qx0, qy0, cam.height, st);
    __syncthreads();
    fs.have = i1 + FINE_BATCH < e1;
    if (fs.have) {
        fs.p = fs.pn;
        if (i1 + FINE_BATCH + t < e1) {
            fs.A = srec[3 * (size_t)fs.p];
            fs.B = srec[3 * (size_t)fs.p + 1];
            fs.C = srec[3 * (size_t)fs.p + 2];
        }
        fs.pn = i1 + 2 * FINE_BATCH + t < e1 ? hl.vals[i1 + 2 * FINE_BATCH + t] : 0u;
    }
    return Batch{M, M, M, 0};
}

template <bool STATS, bool IMP>
__global__ void __launch_bounds__(FINE_NT, 6) hybrid_fwd_fine_kernel(
    const float4* __restrict__ srec, HybridLists hl, ViewSet views, DevSettings st, float* __restrict__ images,
    float* __restrict__ t_final, int32_t* __restrict__ last_out, int4* __restrict__ stats_out,
    int4* __restrict__ eval_out, int64_t n, double* __restrict__ imp_sum, uint32_t* __restrict__ imp_max,
    uint32_t parts) {
    extern __shared__ __align__(16) char smem[];
    // IMP: as in hybrid_fwd_kernel, over the part (against atomics of every row
    // and round: 300 k splats of an unbounded scene at 420x300 129 -> 62 us,
    // 200 k small ones in two views of 800x700 207 -> 133 us; 45 and 110 us
    // without the scores)
    __shared__ double s_isum[IMP ? FINE_BATCH : 1];
    __shared__ uint32_t s_imax[IMP ? FINE_BATCH : 1];
    static_assert(FINE_BATCH == FINE_NT, "one entry per thread");
    const int t = threadIdx.x;
    if constexpr (IMP) {
        s_isum[t] = 0.0;
        s_imax[t] = 0u;
    }
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int row = lane >> 4, col = lane & 15;
    const bool odd = (row & 1) != 0, upper = row >= 2;
    const Lds L = carve(smem, FINE_BATCH);
    uint16_t* list = reinterpret_cast<uint16_t*>(smem + lds_bytes(FINE_BATCH)) + wave * FINE_LIST;
    const uint2* list4 = reinterpret_cast<const uint2*>(list);
    const int chan = 32 + 4 * min(row, 2);  // offset of this row's channel in a staged entry
    const float bgr = row == 0 ? st.bg[0] : (row == 1 ? st.bg[1] : st.bg[2]);
    const EvalConsts ek = eval_consts(st);
    if (*hl.cur_need > hl.cur_cap) {  // a fixed workspace too small: report, write nothing
        if (blockIdx.x == 0 && t == 0) atomicOr(hl.flags, FLAG_CAPACITY);
        return;
    }
    const uint32_t q = blockIdx.x;
    const FinePart fp = fine_part(views, hl, st, q, parts);
    const uint32_t tile = fp.tile;
    const TileGeom tg = fp.tg;
    const DevView& cam = views.v[tg.vi];
    const int x = fp.qx0 + (wave & 1) * 4 + (col & 3), y = fp.qy0 + (wave >> 1) * 4 + (col >> 2);
    const bool inside = x < cam.width && y < cam.height;
    const float px = (float)x + 0.5f, py = (float)y + 0.5f;
    // T: the pixel's transmittance (the same in its four lanes); C: the
    // channel of this row; the last blended index and the counters are
    // those of the entries this row took
    float T = 1.f, C = 0.f;
    int last = -1, stopk = 0x7fffffff, nblend = 0, nmasked = 0, nev = 0x7fffffff, nev_last = 0, staged = 0;
    bool run = inside;
    const int tcx = tg.tx0 / st.tile_w, tcy = tg.ty0 / st.tile_h;
    const uint2 r1 = uniform(hl.ranges[tile]);
    const uint2 r2 = uniform(hl.ranges[region_of_tile(tcx, tcy, cam, views)]);
    const int e1 = (int)r1.y, e2 = (int)r2.y;
    int i1 = (int)r1.x, i2 = (int)r2.x, m = 0, b = 0;
    const TileBox tb{(float)tg.tx0 + 0.5f, (float)min(tg.tx0 + st.tile_w, cam.width) - 0.5f,
                     (float)tg.ty0 + 0.5f, (float)min(tg.ty0 + st.tile_h, cam.height) - 0.5f};
    uint4* cur = hl.cur + uniform(hl.cur_off[tile]);
    FineStream fs;
    fs.have = false;
    while (i1 < e1 || i2 < e2) {
        if (!__syncthreads_or(run)) break;
        // (every part of the tile that gets here writes the same values)
        if (t == 0) cur[b] = make_uint4((uint32_t)i1, (uint32_t)i2, (uint32_t)m, 0u);
        const Batch bt = fine_batch(L, fs, hl, srec, i1, e1, i2, e2, tcx, tcy, tb, cam, st, m, fp.qx0, fp.qy0);
        const int ne = ballot(run) ? block_list(L, bt.M, wave, lane, 0x7fffffff, list) : 0;
        // one entry per row and round; the offsets of the four are read
        // two rounds ahead, the geometry one round ahead
        uint2 o0 = make_uint2(0u, 0u), o1 = o0;
        if (ne > 0) {  // (without a list its words hold anything)
            o0 = list4[0];
            o1 = list4[1];
        }
        uint32_t own = ((upper ? o0.y : o0.x) >> (odd ? 16 : 0)) & 0xffffu;
        float4 A = *reinterpret_cast<const float4*>(smem + own);
        float4 B = *reinterpret_cast<const float4*>(smem + own + 16);
        for (int e0 = 0; e0 < ne; e0 += 4) {
            const uint2 o2 = list4[e0 / 4 + 2 < FINE_LIST / 4 ? e0 / 4 + 2 : 0];
            const uint32_t ownn = ((upper ? o1.y : o1.x) >> (odd ? 16 : 0)) & 0xffffu;
            const float4 An = *reinterpret_cast<const float4*>(smem + ownn);
            const float4 Bn = *reinterpret_cast<const float4*>(smem + ownn + 16);
            const float c0 = *reinterpret_cast<const float*>(smem + (o0.x & 0xffffu) + chan);
            const float c1 = *reinterpret_cast<const float*>(smem + (o0.x >> 16) + chan);
            const float c2 = *reinterpret_cast<const float*>(smem + (o0.y & 0xffffu) + chan);
            const float c3 = *reinterpret_cast<const float*>(smem + (o0.y >> 16) + chan);
            const int k = __float_as_int(B.w);  // index in the tile's full list
            Eval e;
            bool hit = eval_entry(A, B, px, py, ek, e) & (e0 + row < ne) & run;
            const float f = hit ? fmaf(-B.z, e.alpha, 1.f) : 1.f;
            // the transmittance after each entry, by one product after
            // the other as in hybrid_fwd_kernel: images do not depend on
            // the kernel
            const Rows2 fr = row_pairs(f);
            const Rows2 fa = row_halves(fr.lo), fb = row_halves(fr.hi);
            const float t1 = T * fa.lo, t2 = t1 * fb.lo, t3 = t2 * fa.hi, t4 = t3 * fb.hi;
            const float Tb = upper ? (odd ? t3 : t2) : (odd ? t1 : T);
            float Tn = t4;
            const bool over = run & (t4 < st.t_min);
            const uint64_t om = ballot(over);
            if (om) {
                // the first entry that would leave less than t_min stops
                // the pixel and is excluded, as are those behind it
                const int s = !over ? 4 : (t1 < st.t_min ? 0 : (t2 < st.t_min ? 1 : (t3 < st.t_min ? 2 : 3)));
                if (over) Tn = s == 0 ? T : (s == 1 ? t1 : (s == 2 ? t2 : t3));
                if (STATS && row == s) {
                    stopk = k;
                    nev = staged + (int)(own / 48u) + 1;
                }
                hit = hit & (row < s);
                run = run & !over;
            }
            T = Tn;
            const float wgt = hit ? B.z * e.alpha * Tb : 0.f;
            const Rows2 wr = row_pairs(wgt);
            const Rows2 wa = row_halves(wr.lo), wb = row_halves(wr.hi);
            // an entry that does not reach the pixel must not touch its
            // colour, which may be infinite; one that does always adds to it,
            // also with weight 0, as in hybrid_fwd_kernel
            const uint64_t hm = ballot(hit);
            if (row_in_all_rows(hm, 0)) C = fmaf(wa.lo, c0, C);
            if (row_in_all_rows(hm, 1)) C = fmaf(wb.lo, c1, C);
            if (row_in_all_rows(hm, 2)) C = fmaf(wa.hi, c2, C);
            if (row_in_all_rows(hm, 3)) C = fmaf(wb.hi, c3, C);
            if (hit) {
                last = k;
                if (STATS) {
                    ++nblend;
                    nmasked += B.z == 0.f;
                    nev_last = staged + (int)(own / 48u) + 1;
                }
            }
            if (IMP && ballot(wgt > 0.f)) {
                const float ws = row_total(wgt), wm = row_max(wgt);
                if (col == 0 && !(ws <= 0.f)) {
                    const uint32_t j = own / 48u;
                    atomicAdd(&s_isum[j], (double)ws);
                    atomicMax(&s_imax[j], __float_as_uint(wm));
                }
            }
            if (om && !ballot(run)) break;
            own = ownn;
            A = An;
            B = Bn;
            o0 = o1;
            o1 = o2;
        }
        if constexpr (IMP) {
            __syncthreads();
            if (t < bt.M && s_isum[t] != 0.0) {
                const int64_t g = (int64_t)__float_as_uint(L.E[3 * t + 2].w) - (int64_t)tg.vi * n;
                atomicAdd(imp_sum + g, s_isum[t]);
                atomicMax(imp_max + g, s_imax[t]);
                s_isum[t] = 0.0;
                s_imax[t] = 0u;
            }
        }
        i1 += bt.nX;
        i2 += bt.nYraw;
        m += bt.Mfull;
        staged += bt.M;
        ++b;
        __syncthreads();  // the next batch overwrites the LDS
    }
    if (t == 0) atomicMax(hl.nbatch + tile, (uint32_t)b);
    if (hl.drec_clear) {
        // the backward's accumulator, one slice per part (as in
        // hybrid_fwd_kernel)
        const uint64_t np = (uint64_t)views.total_tiles * parts;
        const uint64_t per = (hl.drec_clear_n2 + np - 1) / np;
        const uint64_t q0 = (uint64_t)q * per;
        const uint64_t q1 = min(q0 + per, hl.drec_clear_n2);
        double2* z = reinterpret_cast<double2*>(hl.drec_clear);
        for (uint64_t zq = q0 + (uint64_t)t; zq < q1; zq += FINE_NT) z[zq] = make_double2(0.0, 0.0);
    }
    last = rows_max(last);
    const int64_t pv = (int64_t)cam.width * cam.height;
    const int64_t loc = (int64_t)y * cam.width + x;
    const int64_t p = (int64_t)cam.px_off + loc;
    if (inside) {
        // row r writes channel r, the last row the per-pixel state
        if (row < 3) {
            images[3 * (int64_t)cam.px_off + row * pv + loc] = fmaf(T, bgr, C);
        } else {
            t_final[p] = T;
            last_out[p] = last;
        }
    }
    if (STATS) {
        stopk = -rows_max(-stopk);
        nev = -rows_max(-nev);
        nev_last = rows_max(nev_last);
        nblend = rows_add(nblend);
        nmasked = rows_add(nmasked);
        if (inside && row == 0) {
            stats_out[p] = make_int4(stopk != 0x7fffffff ? stopk + 1 : m, nblend, nmasked, last + 1);
            eval_out[p] = make_int4(nev != 0x7fffffff ? nev : staged, nev_last, 0, 0);
        }
    }
}

// Row sums of ten per-lane quantities, folded pairwise while the lanes are
// halved: after the step over 8 lanes a lane holds one of two quantities, and
// so on; the quantity whose row total lane col ends with is
// fold10_quantity(col) (-1: none).  The step that chooses on bit 2 pairs lanes
// l and l ^ 7 (the mirror within 8 lanes): the four lanes of a quad then still
// cover the eight.
__device__ __forceinline__ float dpp_xor7(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, false));
}
__device__ __forceinline__ int fold10_quantity(int col) {
    const int q = ((col >> 3) & 1) + ((col >> 2) & 1) * 2 + ((col >> 1) & 1) * 4;
    if ((col & 1) == 0) return q;
    return (col & 6) == 0 ? 8 + ((col >> 3) & 1) : -1;
}
__device__ __forceinline__ float row_fold10(const float (&v)[10], int col) {
    const bool b3 = (col & 8) != 0, b2 = (col & 4) != 0, b1 = (col & 2) != 0, b0 = (col & 1) != 0;
    float a[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) a[i] = (b3 ? v[2 * i + 1] : v[2 * i]) + dpp_ror8(b3 ? v[2 * i] : v[2 * i + 1]);
    // a[i]: quantity 2 i + b3
    const float c0 = (b2 ? a[1] : a[0]) + dpp_xor7(b2 ? a[0] : a[1]);
    const float c1 = (b2 ? a[3] : a[2]) + dpp_xor7(b2 ? a[2] : a[3]);
    const float c2 = a[4] + dpp_xor7(a[4]);
    const float d0 = (b1 ? c1 : c0) + dpp_xor2(b1 ? c0 : c1);
    const float d1 = c2 + dpp_xor2(c2);
    return (b0 ? d1 : d0) + dpp_xor1(b0 ? d0 : d1);
}

__global__ void __launch_bounds__(FINE_NT, 5) hybrid_bwd_fine_kernel(
    const float4* __restrict__ srec, HybridLists hl, ViewSet views, DevSettings st, const float* __restrict__ t_final,
    const int32_t* __restrict__ last_in, const float* __restrict__ dl_dimages, int64_t n, double* __restrict__ d_rec,
    double* __restrict__ d_masks, uint32_t parts) {
    extern __shared__ __align__(16) char smem[];
    __shared__ int s_top;
    const int t = threadIdx.x;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int row = lane >> 4, col = lane & 15;
    const bool odd = (row & 1) != 0, upper = row >= 2;
    const Lds L = carve(smem, FINE_BATCH);
    uint16_t* list = reinterpret_cast<uint16_t*>(smem + lds_bytes(FINE_BATCH)) + wave * FINE_LIST;
    // ten partial sums per staged entry over the part's blocks, in two sets: one
    // of waves 0 and 1, one of waves 2 and 3.  A sum of two does not depend on
    // which wave comes first, so that the FP32 sums repeat to the bit.  (The LDS
    // then holds four workgroups instead of five: 200 k small splats at 800x800
    // 139 -> 140 us, 4096 splats at 128x128 44.5 -> 45.5 us.)
    constexpr int SET = FINE_BATCH * 10;
    float* acc = reinterpret_cast<float*>(smem + lds_bytes(FINE_BATCH) + (FINE_NT / 64) * FINE_LIST * 2);
    float* wacc = acc + (wave >> 1) * SET;
    const int qi = fold10_quantity(col);
    const EvalConsts ek = eval_consts(st);
    if (*hl.cur_need > hl.cur_cap) return;  // the forward reported it
    for (int i = t; i < SET / 2; i += FINE_NT) reinterpret_cast<float4*>(acc)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    const uint32_t q = blockIdx.x;
    const FinePart fp = fine_part(views, hl, st, q, parts);
    const uint32_t tile = fp.tile;
    const TileGeom tg = fp.tg;
    const DevView& cam = views.v[tg.vi];
    const int64_t rec_base = (int64_t)tg.vi * n;
    const int64_t pv = (int64_t)cam.width * cam.height;
    const int x = fp.qx0 + (wave & 1) * 4 + (col & 3), y = fp.qy0 + (wave >> 1) * 4 + (col >> 2);
    const float px = (float)x + 0.5f, py = (float)y + 0.5f;
    float Tf = 1.f, w0 = 0.f, w1 = 0.f, w2 = 0.f;
    int lastk = -1;
    if (x < cam.width && y < cam.height) {
        const int64_t loc = (int64_t)y * cam.width + x;
        const int64_t p = (int64_t)cam.px_off + loc;
        const float* dl = dl_dimages + 3 * (int64_t)cam.px_off;
        lastk = last_in[p];
        Tf = t_final[p];
        w0 = dl[loc];
        w1 = dl[pv + loc];
        w2 = dl[2 * pv + loc];
    }
    // T and sb (the loss weights dotted with the colour behind) of the
    // pixel are the same in its four lanes
    float T = Tf, sb = 0.f;
    const float wbg = w0 * st.bg[0] + w1 * st.bg[1] + w2 * st.bg[2];
    const int wlast = __builtin_amdgcn_readlane(wave_max_scan(lastk), 63);  // the block's last blended index
    if (t == 0) s_top = -1;
    __syncthreads();
    if (lane == 0) atomicMax(&s_top, wlast);
    __syncthreads();
    const int top = uniform(s_top);
    const uint4* cur = hl.cur + uniform(hl.cur_off[tile]);
    const int tcx = tg.tx0 / st.tile_w, tcy = tg.ty0 / st.tile_h;
    const uint2 r1 = uniform(hl.ranges[tile]);
    const uint2 r2 = uniform(hl.ranges[region_of_tile(tcx, tcy, cam, views)]);
    const TileBox tb{(float)tg.tx0 + 0.5f, (float)min(tg.tx0 + st.tile_w, cam.width) - 0.5f,
                     (float)tg.ty0 + 0.5f, (float)min(tg.ty0 + st.tile_h, cam.height) - 0.5f};
    // the batch holding the largest last-blended entry (the batches'
    // first indices ascend), then backwards.  A tile without region entries
    // has its narrow list as its batches, one after the other: there the
    // thread's record of the next batch and its position of the one after
    // are on their way while a batch is worked on.
    const bool plain = st.tile_cull != 0 && r2.x >= r2.y;
    int bstar = -1;
    if (top >= 0 && plain) {
        bstar = top / FINE_BATCH;
    } else if (top >= 0) {
        const int nb = (int)hl.nbatch[tile];
        for (int b0 = 0; b0 < nb; b0 += 64)
            bstar += (int)__popcll(ballot(b0 + lane < nb && (int)cur[min(b0 + lane, nb - 1)].z <= top));
    }
    float4 nA, nB, nC;
    uint32_t np = 0;
    if (plain && bstar >= 0) {
        if (bstar * FINE_BATCH + t <= top) {
            const size_t p = hl.vals[r1.x + (uint32_t)(bstar * FINE_BATCH + t)];
            nA = srec[3 * p];
            nB = srec[3 * p + 1];
            nC = srec[3 * p + 2];
        }
        if (bstar > 0) np = hl.vals[r1.x + (uint32_t)((bstar - 1) * FINE_BATCH + t)];
    }
    for (int b = bstar; b >= 0; --b) {
        int m, Mb;
        if (plain) {
            m = b * FINE_BATCH;
            Mb = min(FINE_BATCH, top + 1 - m);
            if (t < Mb) put_entry<true>(L, t, nA, nB, nC, m + t, fp.qx0, fp.qy0, cam.height, st);
            __syncthreads();
            if (b > 0) {
                nA = srec[3 * (size_t)np];
                nB = srec[3 * (size_t)np + 1];
                nC = srec[3 * (size_t)np + 2];
                if (b > 1) np = hl.vals[r1.x + (uint32_t)((b - 2) * FINE_BATCH + t)];
            }
        } else {
            const uint4 c = cur[b];
            m = (int)c.z;
            Mb = merge_batch<true>(L, hl.vals, srec, (int)c.x, (int)r1.y, (int)c.y, (int)r2.y, FINE_BATCH, tcx, tcy,
                                   tb, cam, st, m, fp.qx0, fp.qy0).M;
        }
        const int ne = wlast >= m ? block_list(L, Mb, wave, lane, wlast, list) : 0;
        for (int e0 = (ne - 1) & ~3; e0 >= 0; e0 -= 4) {
            const uint32_t own = list[e0 + row];
            const float4 A = *reinterpret_cast<const float4*>(smem + own);
            const float4 B = *reinterpret_cast<const float4*>(smem + own + 16);
            const float4 Cc = *reinterpret_cast<const float4*>(smem + own + 32);
            Eval e;
            const bool reach = eval_entry(A, B, px, py, ek, e);
            const bool hit = reach & (e0 + row < ne) & (__float_as_int(B.w) <= lastk);
            if (!ballot(hit)) continue;
            const float M = B.z;
            const float ma = hit ? M * e.alpha : 0.f;
            const float f = 1.f - ma;
            // the entries behind this one among the four: their factors,
            // and their colours against the loss weights
            const float wc = fmaf(w0, Cc.x, fmaf(w1, Cc.y, w2 * Cc.z));
            const float S = hit ? ma * wc : 0.f;
            const Rows2 f1 = row_pairs(f), s1 = row_pairs(S);
            const Rows2 f2 = row_halves(f1.lo * f1.hi), s2 = row_halves(fmaf(f1.lo, s1.hi, s1.lo));
            const float mid = fmaf(f2.hi, sb, s2.hi);  // behind the first two
            const float base = upper ? sb : mid;       // behind this one's pair
            const float behind = odd ? base : fmaf(f1.hi, base, s1.hi);
            const float Ti = T * __builtin_amdgcn_rcpf((odd ? f : f1.lo * f1.hi) * (upper ? 1.f : f2.hi));
            sb = fmaf(f2.lo, mid, s2.lo);
            T *= __builtin_amdgcn_rcpf(f2.lo * f2.hi);
            float v[10] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (hit) {
                const float X = Ti * (wc - behind) - Tf * __builtin_amdgcn_rcpf(f) * wbg;
                const float wt = ma * Ti;
                v[6] = wt * w0;
                v[7] = wt * w1;
                v[8] = wt * w2;
                v[9] = e.alpha * X;
                if (e.oG <= ek.amax) {
                    // as in hybrid_bwd_kernel
                    const float GdA = e.G * (M * X);
                    const float kq = GdA * (B.y * QSCALE_NINV);
                    const float kapt = kq * e.apt;
                    v[0] = kapt;
                    v[1] = kq * fmaf(A.w, e.apt, e.gdy);
                    v[2] = (kq * e.t) * e.t;
                    v[3] = kapt * e.dy;
                    v[4] = (kq * e.dy) * e.dy;
                    v[5] = GdA;
                }
            }
            const float x10 = row_fold10(v, col);
            // (own / 48) 10 + qi
            if (qi >= 0 && x10 != 0.f) atomicAdd(wacc + (own / 48u) * 10u + (uint32_t)qi, x10);
        }
        __syncthreads();
        for (int i = t; i < Mb * 10; i += FINE_NT) {
            const float x0 = acc[i], x1 = acc[i + SET];
            if (x0 == 0.f && x1 == 0.f) continue;
            acc[i] = acc[i + SET] = 0.f;
            const float xs = x0 + x1;
            const int j = i / 10, k = i - j * 10;
            const uint32_t r = __float_as_uint(L.E[3 * j + 2].w);
            // (the totals of t^2 and dy^2 rescaled, as in hybrid_bwd_kernel)
            if (k < DREC)
                atomicAdd(d_rec + (size_t)r * DREC + k, (double)(xs * (k == 2 || k == 4 ? 0.5f * QSCALE : 1.f)));
            else
                atomicAdd(d_masks + ((int64_t)r - rec_base), (double)xs);
        }
        __syncthreads();  // the next batch overwrites the LDS
    }
}

template <int TW, int TH, int PPT, bool STATS, bool IMP>
void hybrid_fwd_s(hipStream_t s, const float* srec, const HybridLists& hl, const ViewSet& views,
                  const DevSettings& st, float* images, float* t_final, int32_t* last, int32_t* stats,
                  int32_t* evals, int64_t n, double* imp_sum, uint32_t* imp_max) {
    hipLaunchKernelGGL((hybrid_fwd_kernel<TW, TH, PPT, STATS, IMP>), dim3(views.total_tiles), dim3(TW * TH / PPT),
                       lds_bytes(st.batch), s, reinterpret_cast<const float4*>(srec), hl, views, st, images, t_final,
                       last, reinterpret_cast<int4*>(stats), reinterpret_cast<int4*>(evals), n, imp_sum, imp_max);
}

template <int TW, int TH, int PPT>
void hybrid_fwd_t(hipStream_t s, const float* srec, const HybridLists& hl, const ViewSet& views,
                  const DevSettings& st, float* images, float* t_final, int32_t* last, int32_t* stats,
                  int32_t* evals, int64_t n, double* imp_sum, uint32_t* imp_max) {
    if (imp_sum && imp_max)
        hybrid_fwd_s<TW, TH, PPT, false, true>(s, srec, hl, views, st, images, t_final, last, nullptr,
                                               nullptr, n, imp_sum, imp_max);
    else if (stats && evals)
        hybrid_fwd_s<TW, TH, PPT, true, false>(s, srec, hl, views, st, images, t_final, last, stats, evals,
                                               n, nullptr, nullptr);
    else
        hybrid_fwd_s<TW, TH, PPT, false, false>(s, srec, hl, views, st, images, t_final, last, nullptr,
                                                nullptr, n, nullptr, nullptr);
}

template <bool STATS, bool IMP>
void hybrid_fwd_fine(hipStream_t s, const float* srec, const HybridLists& hl, const ViewSet& views,
                     const DevSettings& st, float* images, float* t_final, int32_t* last, int32_t* stats,
                     int32_t* evals, int64_t n, double* imp_sum, uint32_t* imp_max) {
    const uint32_t parts = (uint32_t)(st.tile_w * st.tile_h / 64);
    hipLaunchKernelGGL((hybrid_fwd_fine_kernel<STATS, IMP>), dim3(views.total_tiles * parts), dim3(FINE_NT),
                       fine_lds_bytes(false), s, reinterpret_cast<const float4*>(srec), hl, views, st, images, t_final,
                       last, reinterpret_cast<int4*>(stats), reinterpret_cast<int4*>(evals), n, imp_sum, imp_max,
                       parts);
}

void hybrid_bwd_fine(hipStream_t s, const float* srec, const HybridLists& hl, const ViewSet& views,
                     const DevSettings& st, const float* t_final, const int32_t* last, const float* dl, int64_t n,
                     double* d_rec, double* d_masks) {
    const uint32_t parts = (uint32_t)(st.tile_w * st.tile_h / 64);
    hipLaunchKernelGGL(hybrid_bwd_fine_kernel, dim3(views.total_tiles * parts), dim3(FINE_NT), fine_lds_bytes(true), s,
                       reinterpret_cast<const float4*>(srec), hl, views, st, t_final, last, dl, n, d_rec, d_masks,
                       parts);
}

template <int TW, int TH, int PPT>
void hybrid_bwd_t(hipStream_t s, const float* srec, const HybridLists& hl, const ViewSet& views,
                  const DevSettings& st, const float* t_final, const int32_t* last, const float* dl, int64_t n,
                  double* d_rec, double* d_masks) {
    auto launch = [&](auto sum) {
        hipLaunchKernelGGL((hybrid_bwd_kernel<TW, TH, PPT, decltype(sum)::value>), dim3(views.total_tiles),
                           dim3(TW * TH / PPT), lds_bytes(st.batch), s, reinterpret_cast<const float4*>(srec), hl, views,
                           st, t_final, last, dl, n, d_rec, d_masks);
    };
    if constexpr (TW * TH / PPT == 64) {
        launch(std::false_type{});
    } else if constexpr (PPT == 1) {
        launch(std::true_type{});
    } else {
        if (st.batch < MAXB || views.total_tiles <= SUM_TILES) launch(std::true_type{});
        else launch(std::false_type{});
    }
}

#define MGS_HYBRID_SHAPES(X) \
    X(8, 8, 1)               \
    X(16, 8, 1)              \
    X(16, 8, 2)              \
    X(16, 16, 1)             \
    X(16, 16, 2)             \
    X(16, 16, 4)             \
    X(32, 8, 1)              \
    X(32, 8, 2)              \
    X(32, 8, 4)

HybridLists make_lists(const HybridBuffers& b) {
    HybridLists hl;
    hl.vals = b.vals;
    hl.ranges = reinterpret_cast<const uint2*>(b.ranges);
    hl.cur = reinterpret_cast<uint4*>(b.cur);
    hl.cur_off = b.cur_off;
    hl.nbatch = b.nbatch;
    hl.cur_need = b.cur_need;
    hl.cur_cap = b.cur_cap;
    hl.flags = b.flags;
    hl.cur_stg = reinterpret_cast<uint2*>(b.cur_stg);
    hl.stg = reinterpret_cast<uint2*>(b.stg);
    hl.stg_count = b.stg_count;
    hl.order = b.order;
    hl.stg_cap = (uint32_t)std::min<uint64_t>(b.stg_cap, STG_NOWHERE);
    hl.drec_clear = b.drec_clear;
    hl.drec_clear_n2 = b.drec_clear_n2;
    return hl;
}

unsigned blocks_of(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// Which compositing kernels a forward (and its backward) takes: those for
// small splats or the tile-wide ones.  Measured, tile-wide / small-splat time
// of forward and backward together (16x16 tiles; the library's default
// settings, and batches of 128 with 2 and 4 pixels per thread):
//   192 and 600 tiles, splats of every size: 0.97 (600 tiles of a scene of
//   screen-filling splats) to 7.4;  960 tiles, screen-filling: 0.65 to 1.07
//   1,750 tiles, share of large splats' tiles 0.07 / 0.72 / 0.94: 3.5, 3.6 /
//   3.1, 3.0 / 0.6, 0.7;  3,300 tiles, 0.18 / 0.89 / 0.97: 2.0, 2.1 / 2.0, 2.4
//   / 0.55, 0.42;  5,400 tiles, 0.13 / 0.84 / 0.96: 1.4, 1.4 / 1.4, 1.7 / 0.5,
//   0.4;  8,800 tiles, 0.10 / 0.79: 0.96, 0.91 / 0.94, 1.15;  16,000 tiles,
//   0.29: 0.6, 0.5
// So the line lies at 640 tiles, or at 7,168 tiles where splats larger than
// LARGE_RADIUS hold at most three quarters of the footprint tiles.  Tiles of
// other sizes count by their pixels.
constexpr int64_t FINE_PIXELS_ANY = 640 * 256, FINE_PIXELS_SMALL = 7168 * 256;

bool fine_needs_sizes(int64_t pixels) { return pixels > FINE_PIXELS_ANY && pixels <= FINE_PIXELS_SMALL; }

bool use_fine(int64_t pixels, uint64_t tiles_all, uint64_t tiles_large) {
    return pixels <= FINE_PIXELS_ANY || (pixels <= FINE_PIXELS_SMALL && 4 * tiles_large <= 3 * tiles_all);
}

bool composite_config_supported(const CompositeConfig& c) {
#define MGS_MATCH(A, B, P) \
    if (c.tile_w == A && c.tile_h == B && c.ppt == P) return true;
    MGS_HYBRID_SHAPES(MGS_MATCH)
#undef MGS_MATCH
    return false;
}

void launch_permute_classify(hipStream_t stream, const uint32_t* order, const uint32_t* skeys, const uint32_t* live,
                             const float* rec, int64_t R, int64_t n, const ViewSet& views, const DevSettings& st, uint32_t* cnt,
                             uint32_t* cells, float* srec, uint32_t* part, bool sizes) {
    if (R == 0) return;
    const unsigned nb = blocks_of(R);
    hipLaunchKernelGGL(permute_classify_kernel, dim3(nb), dim3(256), 0, stream, order, skeys, live,
                       reinterpret_cast<const float4*>(rec), R, n, views, st, cnt, reinterpret_cast<uint4*>(cells),
                       reinterpret_cast<float4*>(srec), part, sizes ? 1 : 0);
}

// part: 2 nb + 4 nb + 2 nb u32 counts (per workgroup, per wave, per
// workgroup), then (8-byte aligned) the list offsets: per wave, per group (5
// totals and the offset)
namespace {
int64_t waves_of(int64_t R) { return (int64_t)blocks_of(R) * 4; }
int64_t groups_of(int64_t R) { return (waves_of(R) + LO_GROUP - 1) / LO_GROUP; }
size_t counts_bytes(int64_t R) { return ((size_t)blocks_of(R) * 32 + 15) / 8 * 8; }
ListOffsets list_offsets(uint32_t* part, int64_t R) {
    char* p = reinterpret_cast<char*>(part) + counts_bytes(R);
    ListOffsets lo;
    lo.wave_rel = reinterpret_cast<uint64_t*>(p);
    lo.group_tot = lo.wave_rel + waves_of(R);
    lo.group_off = lo.group_tot + 5 * groups_of(R);
    return lo;
}
}  // namespace

size_t classify_parts_bytes(int64_t R) { return counts_bytes(R) + (size_t)(waves_of(R) + 6 * groups_of(R)) * 8 + 8; }

void launch_list_offsets(hipStream_t stream, uint32_t* part, int64_t R, uint64_t* total, uint64_t* wide_counts,
                         bool sizes, const uint32_t* flags, const uint32_t* staged, uint64_t* host) {
    const ListOffsets lo = list_offsets(part, R);
    const ListTotals out{total, wide_counts, flags, staged, host};
    const int64_t ng = R > 0 ? groups_of(R) : 0, nb = (int64_t)blocks_of(R);
    if (ng > 0 && ng <= LO_ONE) {
        hipLaunchKernelGGL(list_offsets_one_kernel, dim3(1), dim3(LO_GROUP), 0, stream, part, nb, waves_of(R), ng, lo,
                           sizes ? 1 : 0, out);
        return;
    }
    if (ng > 0)
        hipLaunchKernelGGL(list_offsets_group_kernel, dim3((unsigned)ng), dim3(LO_GROUP), 0, stream, part, nb,
                           waves_of(R), lo, sizes ? 1 : 0);
    hipLaunchKernelGGL(list_offsets_total_kernel, dim3(1), dim3(LO_GROUP), 0, stream, ng, lo, out);
}

void launch_duplicate_lists(hipStream_t stream, const float* srec, const uint32_t* cnt_sorted,
                            const uint32_t* cells, uint32_t* part, int64_t R,
                            int64_t n, const ViewSet& views, const DevSettings& st, void* keys, bool keys16,
                            uint32_t* vals, int64_t capacity, uint32_t* flags, const FillSpan* fill,
                            int fill_count) {
    if (R == 0) {
        launch_fill_spans(stream, fill, fill_count);
        return;
    }
    const FillSet fs = make_fill_set(fill, fill_count);
    const unsigned grid = std::max(blocks_of(R), blocks_of((fs.total + DUP_CLEAR - 1) / DUP_CLEAR));
    hipLaunchKernelGGL(duplicate_kernel, dim3(grid), dim3(256), 0, stream, reinterpret_cast<const float4*>(srec),
                       cnt_sorted, reinterpret_cast<const uint4*>(cells), list_offsets(part, R), R, n, views, st, keys,
                       keys16, vals, capacity, flags, fs);
}

void launch_tile_order(hipStream_t stream, const uint32_t* key, uint32_t tiles, uint32_t* hist_cursor,
                       uint32_t* order, bool cleared) {
    if (tiles == 0) return;
    if (!cleared) launch_fill_u32(stream, hist_cursor, 512, 0u);
    hipLaunchKernelGGL(order_hist_kernel, dim3(blocks_of(tiles)), dim3(256), 0, stream, key, tiles, hist_cursor);
    hipLaunchKernelGGL(order_place_kernel, dim3(blocks_of(tiles)), dim3(256), 0, stream, key, tiles,
                       (const uint32_t*)hist_cursor, hist_cursor + 256, order);
}

void launch_tile_setup(hipStream_t stream, const uint32_t* ranges, const ViewSet& views, int batch,
                       const uint32_t* key, uint32_t* cost, uint32_t* cur_off, uint64_t* cur_need, uint32_t* blk,
                       uint32_t* hist_cursor, uint32_t* order, uint32_t* nbatch) {
    const uint32_t T = views.total_tiles;
    if (T == 0) return;
    if (T <= SETUP_ONE) {
        hipLaunchKernelGGL(tile_setup_kernel, dim3(1), dim3(SETUP_DT), 0, stream,
                           reinterpret_cast<const uint2*>(ranges), views, batch, key, cost, cur_off, cur_need, order,
                           nbatch);
        return;
    }
    hipLaunchKernelGGL(batch_caps_kernel, dim3(blocks_of(T)), dim3(256), 0, stream,
                       reinterpret_cast<const uint2*>(ranges), views, batch, key, cost, cur_off, blk, hist_cursor);
    hipLaunchKernelGGL(order_offsets_kernel, dim3(blocks_of(T)), dim3(256), 0, stream, key, (const uint32_t*)cost, T,
                       (const uint32_t*)hist_cursor, hist_cursor + 256, order, cur_off, (const uint32_t*)blk,
                       cur_need, nbatch);
}

void launch_hybrid_fwd(hipStream_t stream, const CompositeConfig& cfg, const float* srec, const HybridBuffers& bufs,
                       const ViewSet& views, const DevSettings& st, float* images, float* t_final, int32_t* last,
                       int32_t* stats, int32_t* evals, int64_t n, double* imp_sum,
                       uint32_t* imp_max) {
    if (views.total_tiles == 0) return;
    const HybridLists hl = make_lists(bufs);
    if (bufs.fine) {
        if (imp_sum && imp_max)
            hybrid_fwd_fine<false, true>(stream, srec, hl, views, st, images, t_final, last, nullptr, nullptr, n,
                                         imp_sum, imp_max);
        else if (stats && evals)
            hybrid_fwd_fine<true, false>(stream, srec, hl, views, st, images, t_final, last, stats, evals, n, nullptr,
                                         nullptr);
        else
            hybrid_fwd_fine<false, false>(stream, srec, hl, views, st, images, t_final, last, nullptr, nullptr, n,
                                          nullptr, nullptr);
        return;
    }
#define MGS_HFWD(A, B, P)                                                                               \
    if (cfg.tile_w == A && cfg.tile_h == B && cfg.ppt == P) {                                           \
        hybrid_fwd_t<A, B, P>(stream, srec, hl, views, st, images, t_final, last, stats, evals, n,      \
                              imp_sum, imp_max);                                                        \
        return;                                                                                         \
    }
    MGS_HYBRID_SHAPES(MGS_HFWD)
#undef MGS_HFWD
}

void launch_hybrid_bwd(hipStream_t stream, const CompositeConfig& cfg, const float* srec, const HybridBuffers& bufs,
                       const ViewSet& views, const DevSettings& st, const float* t_final, const int32_t* last,
                       const float* dl_dimages, int64_t n, double* d_rec, double* d_masks) {
    if (views.total_tiles == 0) return;
    const HybridLists hl = make_lists(bufs);
    if (bufs.fine) {
        hybrid_bwd_fine(stream, srec, hl, views, st, t_final, last, dl_dimages, n, d_rec, d_masks);
        return;
    }
#define MGS_HBWD(A, B, P)                                                                               \
    if (cfg.tile_w == A && cfg.tile_h == B && cfg.ppt == P) {                                           \
        hybrid_bwd_t<A, B, P>(stream, srec, hl, views, st, t_final, last, dl_dimages, n, d_rec, d_masks); \
        return;                                                                                         \
    }
    MGS_HYBRID_SHAPES(MGS_HBWD)
#undef MGS_HBWD
}

}  // namespace mgs
