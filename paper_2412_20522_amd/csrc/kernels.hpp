// Host-side launchers of the gfx950 kernels (one translation unit each).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "common.hpp"

namespace mgs {

// projection (radius optional: the record's B.w holds it too)
// rkeys (optional): the keys of the per-view depth order of the records (depth
// bits, all ones for records without tiles)
void launch_project_fwd(hipStream_t stream, const mgs_gaussians& g, const ViewSet& views, const DevSettings& st,
                        float* rec, float* depth, float* radius, uint32_t* tiles, uint32_t* flags,
                        uint32_t* rkeys = nullptr);
// out[r] = field `field` (0..11) of record r (the radius is field 7, B.w)
void launch_record_field(hipStream_t stream, const float* rec, int64_t R, int field, float* out);
void launch_project_bwd(hipStream_t stream, const mgs_gaussians& g, const ViewSet& views, const DevSettings& st,
                        const float* d_rec, const mgs_gradients& out);
// Whole path: FP64 per-record gradients (zeroed by the forward compositing
// before the backward accumulates them); dm_acc (FP64 mask gradients) is
// rounded into out.d_masks.  order_hist: the [512] words of the backward's
// tile order (launch_tile_order), left zero for the next backward.
void launch_project_bwd64(hipStream_t stream, const mgs_gaussians& g, const ViewSet& views, const DevSettings& st,
                          double* d_rec, const double* dm_acc, const mgs_gradients& out,
                          const uint32_t* tiles, uint32_t* order_hist);

// scan / binning / sort / ranges
size_t scan_scratch_bytes(int64_t n);
// Exclusive scan of n u32; total (u64) to total_dev.  count_dev (optional)
// holds the live element count on the device (<= n); elements at or past it
// are treated as zero.
void launch_scan_u32(hipStream_t stream, const uint32_t* in, int64_t n, uint32_t* out, uint64_t* total_dev,
                     void* scratch);
// The allocation-free scan: a library-owned device array of
// SCAN_NOALLOC_BYTES per GPU holds its scratch.  scan_noalloc_init, called
// with `device` current, returns that GPU's address of the array (looked up
// once per device); scan_noalloc_max_n is the largest n it serves.
constexpr size_t SCAN_NOALLOC_BYTES = MGS_SCAN_NOALLOC_BYTES;
hipError_t scan_noalloc_init(int device, void** out);
int64_t scan_noalloc_max_n();
void launch_duplicate(hipStream_t stream, const float* rec, const float* radius, const float* depth,
                      const uint32_t* tiles, const uint32_t* offsets, int64_t n_records, int64_t n_per_view,
                      const ViewSet& views, const DevSettings& st, uint64_t* keys, uint32_t* vals, int64_t capacity,
                      uint32_t* flags);
size_t sort_scratch_bytes(int64_t K);
// Sorts (keys, vals) by the low key_bits bits; K_dev (optional) is the live
// count on the device (<= K).  Returns through *out_in_alt whether the
// result ended in the alternate buffers.
void launch_radix_sort(hipStream_t stream, uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt,
                       int64_t K, const uint64_t* K_dev, int key_bits, void* scratch, bool* out_in_alt);
void launch_tile_ranges(hipStream_t stream, const uint64_t* keys, int64_t K, const uint64_t* K_dev,
                        int64_t total_tiles, uint32_t* ranges);
// Whether the keys of a list of K entries (or room for K) over `cells` cells
// take 16 bits: fewer than 65535 cells (all ones is no cell's key), and more
// entries than are sorted in one workgroup.  20.2 M entries of 26 k cells:
// duplication, sort and ranges 376 -> 349 us; up to 4 M entries no difference.
bool cell_keys16(int64_t K, int64_t cells);
// Cell keys sorted on their low `bits` bits (stable), and the cells' ranges
// (cleared).  A sort in one workgroup also writes the ranges; returns whether
// it did.
bool launch_cell_sort(hipStream_t stream, void* keys, uint32_t* vals, void* keys_alt, uint32_t* vals_alt, bool keys16,
                      int64_t K, const uint64_t* K_dev, int bits, void* scratch, bool* out_in_alt, uint32_t* ranges,
                      int64_t nbins);
// Stable sort of the indices 0 .. K - 1 (written to vals) by their 32-bit keys
// within consecutive segments of seg_len keys each (at most 16 segments; the
// last may be shorter).  Keys of all ones come last in their segment.  Returns
// whether live[segment] was written: the number of other keys, behind which
// the sorted keys hold anything; if not, all keys are there, sorted.
bool launch_depth_sort(hipStream_t stream, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                       int64_t K, int64_t seg_len, void* scratch, bool* out_in_alt, uint32_t* live);
void launch_cell_ranges(hipStream_t stream, const void* keys, bool keys16, int64_t K, const uint64_t* K_dev,
                        int64_t cells, uint32_t* ranges);
void launch_fill_u32(hipStream_t stream, uint32_t* p, int64_t n, uint32_t value);
// Several u32 fills in one launch (at most FILL_SPANS; null or empty spans
// are skipped).
constexpr int FILL_SPANS = 8;
struct FillSpan {
    uint32_t* p;
    int64_t n;
    uint32_t value;
};
// Spans as a kernel argument: element i of their concatenation belongs to the
// first span whose end exceeds it.
struct FillSet {
    uint32_t* p[FILL_SPANS];
    int64_t end[FILL_SPANS];  // cumulative element counts
    uint32_t v[FILL_SPANS];
    int64_t total;
    int count;
};
FillSet make_fill_set(const FillSpan* spans, int count);
__device__ __forceinline__ void fill_element(const FillSet& fs, int64_t i) {
    int64_t start = 0;
    for (int k = 0; k < fs.count; ++k) {
        if (i < fs.end[k]) {
            fs.p[k][i - start] = fs.v[k];
            return;
        }
        start = fs.end[k];
    }
}
void launch_fill_spans(hipStream_t stream, const FillSpan* spans, int count);
void launch_fill_f32(hipStream_t stream, float* p, int64_t n, float value);
// Column sums of an [n, 4] int32 array into out_dev[4] (u64); scratch holds
// 4 * scan_scratch_bytes(n) bytes.
void launch_sum_i32x4(hipStream_t stream, const int32_t* in, int64_t n, uint64_t* out_dev, void* scratch);

// compositing
struct CompositeConfig {
    int tile_w, tile_h, ppt;  // pixels per thread; threads per block = tile_w * tile_h / ppt
};
bool composite_config_supported(const CompositeConfig& c);

// hybrid binning: records in (view, depth, record) order are copied once
// ("sorted records": radius in B.w, record id bits in C.w); narrow records
// are listed per tile, wide records per region (one key space: tile ids, then
// region ids), with sorted positions as values, and merged per tile while
// compositing
// part: classify_parts_bytes(R) bytes of per-workgroup counts (written by
// the classification) and list offsets (by launch_list_offsets, read by the
// duplication)
size_t classify_parts_bytes(int64_t R);
// skeys, live: as launch_depth_sort left them; live null if not written
void launch_permute_classify(hipStream_t stream, const uint32_t* order, const uint32_t* skeys, const uint32_t* live,
                             const float* rec, int64_t R, int64_t n, const ViewSet& views, const DevSettings& st, uint32_t* cnt,
                             uint32_t* cells, float* srec, uint32_t* part, bool sizes);
// From the classification's per-workgroup counts: each workgroup's first list
// entry, the entry total (device u64 *total) and wide_counts (device u64):
// [0] = wide records, [2] = their region entries, and with sizes (as given to
// the classification; else 0) [3] = tiles of all footprints, [4] = of those
// of large splats; host (optional, pinned memory the device can write)
// receives for the host [0] = the two flag words, [1] = the entry total, [2] ..
// [6] = wide_counts, [24] = *staged in entries
void launch_list_offsets(hipStream_t stream, uint32_t* part, int64_t R, uint64_t* total, uint64_t* wide_counts,
                         bool sizes, const uint32_t* flags, const uint32_t* staged, uint64_t* host);
// The rule that picks the compositing kernels (pixels over all views; the two
// counts above, needed where fine_needs_sizes).
bool fine_needs_sizes(int64_t pixels);
bool use_fine(int64_t pixels, uint64_t tiles_all, uint64_t tiles_large);
// (fill: the spans the later stages need cleared, set in the same launch)
void launch_duplicate_lists(hipStream_t stream, const float* srec, const uint32_t* cnt_sorted,
                            const uint32_t* cells, uint32_t* part, int64_t R,
                            int64_t n, const ViewSet& views, const DevSettings& st, void* keys, bool keys16,
                            uint32_t* vals, int64_t capacity, uint32_t* flags, const FillSpan* fill, int fill_count);
// Launch order of the tiles: the tiles by descending cost key
// (key[t] in 0..255, ties in any order), so that the most expensive start
// first.  hist_cursor: [512] u32 of scratch (cleared here unless cleared).
void launch_tile_order(hipStream_t stream, const uint32_t* key, uint32_t tiles, uint32_t* hist_cursor,
                       uint32_t* order, bool cleared = false);
// The forward's per-tile set-up after the ranges: each tile's first batch
// checkpoint (cur_off, and the total into the device u64 *cur_need: per tile
// 2 (ceil(narrow / batch) + ceil(region / batch)) + 2), its cost key (cost:
// the entries of its two lists in units of 8, at most 255), and the tile
// order by descending key (key[t], or the cost key when key is null).
// hist_cursor: [512] u32, zero before; blk: blocks of 256 tiles, u32 scratch.
// nbatch (which key may be) is cleared once the order is taken.
void launch_tile_setup(hipStream_t stream, const uint32_t* ranges, const ViewSet& views, int batch,
                       const uint32_t* key, uint32_t* cost, uint32_t* cur_off, uint64_t* cur_need, uint32_t* blk,
                       uint32_t* hist_cursor, uint32_t* order, uint32_t* nbatch);
struct HybridBuffers {
    const uint32_t* vals;        // list entries (sorted positions), (cell, position) order
    const uint32_t* ranges;      // [tiles + regions, 2]
    uint32_t* cur;               // [checkpoints, 4]
    const uint32_t* cur_off;     // [tiles]
    uint32_t* nbatch;            // [tiles]
    const uint64_t* cur_need;    // device: checkpoints the tiles may take
    uint64_t cur_cap;            // checkpoints the buffer holds
    uint32_t* flags;             // device flags (capacity)
    uint32_t* cur_stg;           // [checkpoints, 2] staged-list offset (or ~0) and count
    uint32_t* stg;               // [stg_cap, 2] staged entries; null: the backward merges again
    uint32_t* stg_count;         // the staged list in use, in units of STG_CHUNK entries; before the
                                 // forward staged_first_units
    uint64_t stg_cap;
    double* drec_clear;          // optional: FP64 gradient accumulators (per record, then the masks') the forward clears
    uint64_t drec_clear_n2;      // their size in pairs of doubles
    const uint32_t* order;       // optional [tiles]: tile of each workgroup
    bool fine;                   // the kernels for small splats (the same for a forward and its backward)
};
// stats [P, 4] (examined, blended, blended with mask 0, last + 1) and evals
// [P, 4] (evaluated, evaluated up to the last blended entry, 0, 0) are
// written only when both are non-null.
// imp_sum (FP64, zeroed) and imp_max (float bits, zeroed), both [n] or both
// null: per-Gaussian sum and maximum of the blending weights M alpha T.
void launch_hybrid_fwd(hipStream_t stream, const CompositeConfig& cfg, const float* srec, const HybridBuffers& bufs,
                       const ViewSet& views, const DevSettings& st, float* images, float* t_final, int32_t* last,
                       int32_t* stats, int32_t* evals, int64_t n = 0,
                       double* imp_sum = nullptr, uint32_t* imp_max = nullptr);
void launch_round_f64(hipStream_t stream, const double* in, float* out, int64_t n);
void launch_hybrid_bwd(hipStream_t stream, const CompositeConfig& cfg, const float* srec, const HybridBuffers& bufs,
                       const ViewSet& views, const DevSettings& st, const float* t_final, const int32_t* last,
                       const float* dl_dimages, int64_t n, double* d_rec, double* d_masks);

// masks, loss, optimiser
size_t reduce_scratch_bytes(int64_t n);
// step_off (optional, device): added to step
void launch_sample_masks(hipStream_t stream, const float* scores, int64_t n, float tau, uint64_t seed, uint64_t step,
                         const uint64_t* step_off, float* m_hard, float* y_soft);
void launch_threshold_masks(hipStream_t stream, const float* scores, int64_t n, double threshold, float* m_hard,
                            float* y_soft);
void launch_prune_sample(hipStream_t stream, const float* scores, int64_t n, uint64_t seed, uint64_t step0,
                         int n_draws, uint32_t* keep);
// pos: exclusive scan of keep
void launch_compact_rows(hipStream_t stream, const uint32_t* keep, const uint32_t* pos, int64_t n, int n_arrays,
                         const float* const* in, float* const* out, const int* widths);
void launch_mask_loss(hipStream_t stream, const float* m_hard, int64_t n, float* loss_m, void* scratch);
// lambda_scale (optional, device): multiplies lambda_m
void launch_mask_grad(hipStream_t stream, const float* d_masks, const float* m_hard, const float* y_soft, int64_t n,
                      float tau, float lambda_m, const float* lambda_scale, float* d_scores, float* loss_m,
                      void* scratch);
// d_images and loss optional; grad_scale (optional, device) multiplies d_images
void launch_l1_loss_grad(hipStream_t stream, const float* images, const float* targets, int64_t m, float* d_images,
                         const float* grad_scale, float* loss, void* scratch);
struct AdamArray {
    float* params;
    const float* grads;
    float* m;
    float* v;
    int64_t n;
    float lr;
};
int adam_multi_max();
// step_off (optional, device): added to step for the bias corrections
void launch_adam_multi(hipStream_t stream, const AdamArray* arrays, int n_arrays, float b1, float b2, float eps,
                       int64_t step, const int64_t* step_off);
void launch_step_advance(hipStream_t stream, int64_t* counter, int64_t delta);
void launch_adam(hipStream_t stream, float* params, const float* grads, float* m, float* v, int64_t n, float lr,
                 float b1, float b2, float eps, int64_t step);

}  // namespace mgs
