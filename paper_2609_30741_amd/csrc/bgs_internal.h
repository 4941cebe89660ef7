// Internal declarations of the HIP library behind include/bgs.h.
// gfx950 (CDNA4): wave64, 160 KiB LDS per CU, 256 CUs in 8 XCDs.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "bgs.h"

namespace bgs {

constexpr int kTile = 16;            // rasteriser tile edge (pixels)
constexpr int kBinChunk = 256;       // entries a wave expands at a time
constexpr int kBinMaxChunks = 4096;  // chunks of the compositing order
constexpr int kBinFine = 64;         // surfels per chunk at the front of the order

// Per-surfel record written by the preprocess and staged through LDS by the
// blend kernel.  64 bytes.
//   a = (mu_x, mu_y, C1, C2)    projected centre; u numerator coefficients
//   b = (D1, D2, N1, N2)        v numerator; common denominator
//   c = (lam_num, z_c, opacity, band direction)
//   d = (r, g, b, band interval)
// With dx = i - mu_x, dy = j - mu_y and den = 1 + N1 dx + N2 dy the
// surfel-plane coordinates of pixel (i, j), times sqrt(1/2), are
// u = (C1 dx + C2 dy)/den, v = (D1 dx + D2 dy)/den and the ray meets the
// plane at depth
// lam_num/den (lam_num < 0 marks a surfel seen exactly edge-on, or one
// without extent: only its low-pass term counts).  The
// strip band bounds every pixel x the surfel can reach by
// |n.(x - mu) - c| <= w, with n a pair of snorm16 (x low, y high) and c, w
// a pair of fp16 (c low, w high).
struct alignas(16) SurfelRec {
    float4 a, b, c, d;
};

// Camera constants for the preprocess (fp64 geometry).
struct PreCam {
    double Rt[9];  // world-to-camera rotation R^T, row-major
    double t[3];   // camera centre
    double fx, fy, cx, cy;
    double z_near;
    float zc[4];   // fp32 centre-depth key coefficients (r20, r21, r22, tz)
    int W, H, tiles_x, tiles_y;
};

struct SceneArgs {
    const float* pos;
    const float* quat;
    const float* scale;
    const float* opacity;
    const float* sh;
    int n;
    int sh_degree;
};

// Optional ROI restriction of the binning: bit 8 (ty & 7) + (tx & 7) of
// cells[cell] says whether the tile is masked (cell = (ty / 8) * cells_x +
// tx / 8); null: every tile.
struct CellMask {
    const uint64_t* cells;
    int cells_x;
};

// Binning of one pass (raster.hip): scene, image and scratch.
struct BinArgs {
    const uint32_t* order;  // surfels in compositing order
    const uint2* rects;     // tile rects (x | y << 16, inclusive), empty when .x > .y
    const SurfelRec* recs;
    int n;
    uint32_t chunks;   // chunks of the order, at most kBinMaxChunks:
    uint32_t fine;     //   the first `fine` hold kBinFine surfels each,
    int per;           //   the others this many (a multiple of 256)
    int tiles_x, tiles_y, cells_x;
    uint32_t n_cells;
    uint32_t cap;      // key capacity: list words
    uint32_t ecap;     // entry capacity (bin_max_entries)
    CellMask mask;
    uint4* band;       // per position of the order: rect, band direction and interval (empty rect: no entries)
    float2* mu;        // and the projected centre
    uint32_t* matrix;  // [n_cells][chunks] entries, then their exclusive scan over the chunks
    uint2* kpart;      // per chunk: keys (then their running sum, at most 2^32 - 1), whether it has any
    uint32_t* ctot;    // per cell: entries
    uint32_t* cstart;  // n_cells + 1: first entry
    uint32_t* cpre;    // n_cells + 1: first expansion chunk (kBinChunk entries each)
    uint64_t* emask;   // per entry: its tiles within the cell
    uint32_t* eid;     // per entry: its surfel
    uint32_t* tcount;  // [expansion chunk][64]: keys per tile, then their scan over the cell's chunks
    uint32_t* ttot;    // per tile: keys
    uint32_t* vals;    // the tile lists
};

// The split of n surfels over n_cells cells.  The nearest surfels span the
// image and carry most of the entries, so the front of the order goes in
// small chunks (which also gives small scenes enough workgroups).  The
// count table is bounded: 4 MiB, or 256 chunks where the cells alone exceed
// that.
inline void bin_split(int64_t n, int64_t n_cells, uint32_t* chunks, uint32_t* fine, int* per) {
    const int64_t most = n_cells * kBinMaxChunks <= (1 << 20) ? kBinMaxChunks : (1 << 20) / n_cells;
    const int64_t limit = most < 256 ? 256 : most;
    const int64_t all_fine = (n + kBinFine - 1) / kBinFine;
    const int64_t f = all_fine < limit / 8 ? all_fine : limit / 8;
    const int64_t subs = n > f * kBinFine ? (n - f * kBinFine + 255) / 256 : 0;
    const int64_t p = subs ? 256 * ((subs + (limit - f) - 1) / (limit - f)) : 256;
    const int64_t c = f + (subs * 256 + p - 1) / p;
    *chunks = (uint32_t)(c < 1 ? 1 : c);
    *fine = (uint32_t)f;
    *per = (int)p;
}
// Words of the count table for images of up to n_cells cells.
inline size_t bin_table_words(int64_t n, int64_t n_cells) {
    const int64_t all_fine = (n + kBinFine - 1) / kBinFine;  // no more chunks than this
    const int64_t c = all_fine < 1 ? 1 : all_fine < kBinMaxChunks ? all_fine : kBinMaxChunks;
    const int64_t w = n_cells * c, b = n_cells * 256 > (1 << 20) ? n_cells * 256 : (1 << 20);
    return (size_t)(w < b ? w : b);
}
// Every entry holds a key, except those of the one surfel that the capacity
// cuts, which has at most one per cell.
inline uint64_t bin_max_entries(uint64_t key_cap, uint64_t n_cells) {
    return key_cap + n_cells < 0xFFFFFFFFull ? key_cap + n_cells : 0xFFFFFFFFull;
}
inline uint64_t bin_max_expand_chunks(uint64_t entry_cap, uint64_t n_cells) { return entry_cap / kBinChunk + n_cells; }

struct BlendArgs {
    int W, H, tiles_x;
    float alpha_min, alpha_max, t_min;
    int lowpass;
    float bg0, bg1, bg2;
    float a_min;     // patch mode: depth proxy written only when A >= a_min
    float z_near;
    int patch;       // 0: write rgb/depth_raw/alpha; 1: write rgb/z/alpha/cls
    // ROI patch with 8-pixel ROI tiles: the 8x8 ROI tile mask (qmask_w tiles
    // per row); an 8x8 quadrant of a 16x16 tile that it leaves out is neither
    // composited nor written.  Null otherwise.
    const uint8_t* qmask;
    int qmask_w;
    // View-colour transfer (dominant eye of a stereo frame only; an option
    // outside the paper's method): xrecs are the records of the affiliated
    // eye, whose last float4 holds each surfel's colour seen from that eye;
    // the blend composites them with the dominant eye's weights into
    // xrgb[3][H][W] (plus T bg).  Null otherwise.
    const SurfelRec* xrecs;
    float* xrgb;
};

// Continuation of long tile lists in the blend (k_blend, k_blend_seg,
// k_blend_chain, k_blend_fix in raster.hip).  All arrays live in the
// workspace.  A continued tile takes a slot and a run of consecutive items,
// one per segment of its remaining records.
struct ContArgs {
    uint32_t cap;          // records a tile composites before its rest is continued; 0: never
    uint32_t seg_len;      // records per continuation segment (at most kContMaxSeg segments)
    uint32_t max_slots;    // tiles that may be continued per pass
    uint32_t min_far;      // continue a tile only if some pixel is expected to composite this many more records
    uint32_t* n_slots;     // counters (DevStatus), cleared before each pass
    uint32_t* n_items;
    uint4* slot_desc;      // per slot: tile id, first continued record, end record, item base | nseg << kContSegShift
    uint32_t* item_slot;   // per item: its slot
    float4* st1;           // per slot: 256 pixels x 2 float4 after the capped walk
    float4* part;          // per item: 256 pixels x 2 float4, the segment's walk from the slot's transmittance
};
constexpr uint32_t kContMaxSeg = 32;
constexpr uint32_t kContSegShift = 26;  // item base in the low 26 bits, segment count above


// Device status block kept in the workspace.
struct DevStatus {
    uint32_t n_keys;       // keys of the last binning (may exceed capacity)
    uint32_t n_sort;       // min(n_keys, capacity): keys in the tile lists
    uint32_t n_masked;     // masked tiles of the last ROI patch
    uint32_t n_keys_dom;
    uint32_t n_keys_roi;
    uint32_t overflow;     // bit 0 key capacity, bit 1 box capacity
    uint32_t n_holes, n_gap, n_center, n_rowfill, n_boxes, n_roi_tiles, n_edge;
    // Overflow bits of every earlier frame since the last bgs_poll_status:
    // the per-frame reset folds the previous frame's overflow into it, and
    // only the poll clears it.
    uint32_t sticky;
    // Depth-range reduction over positive fp32 bits: the complement of the
    // minimum (so that a zeroed block means "none yet") and the maximum.
    uint32_t dmin_inv, dmax_bits;
    uint32_t pad2[2];
    uint32_t n_slots, n_items;  // blend continuation of the current pass
    // Counting mode only, dominant then ROI pass, 6 each: evaluated pairs,
    // contributing pairs, records walked (summed over waves), records past
    // the strip test (summed over waves), longest walk of one wave, longest
    // tile list.
    unsigned long long pairs[12];
    int32_t edge_boxes[4 * 6];
    int32_t widths[4];
};

// ---- status and fills (sort.hip) --------------------------------------------
// Start-of-frame reset of the status block by a kernel (no memset node, so a
// frame can be captured in a graph): full = 1 zeroes every word; full = 0
// keeps the sticky overflow word and ORs the previous frame's overflow bits
// into it.
hipError_t launch_status_reset(DevStatus* st, int full, hipStream_t s);
// dst[i] = value for i < n, by a kernel.
hipError_t launch_fill_u32(uint32_t* dst, int64_t n, uint32_t value, hipStream_t s);

// ---- sort (sort.hip) --------------------------------------------------------
size_t radix_tmp_bytes(int64_t n_cap);
// Stable LSD radix sort of n (key, value) pairs by the low key_bits bits of
// the keys, with digits of up to 8 bits.  (ka, va) is the input, (kb, vb)
// the ping-pong buffer; iota = true ignores the input values and uses the
// input positions instead.  Returns in *in_b whether the result is in
// (kb, vb).
hipError_t radix_sort(uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb, int64_t n, int key_bits, bool iota,
                      void* tmp, hipStream_t s, bool* in_b);

// ---- rasteriser (raster.hip) --------------------------------------------------
// cam2 (optional): also the keys, rects and records of a second camera.
// counts (optional, without cam2): the tiles of each surfel's band.  With a
// mask, surfels whose rect holds no masked tile get an empty rect.
hipError_t launch_preprocess(const SceneArgs& sc, const PreCam& cam, float alpha_min, int lowpass,
                             const CellMask& mask, SurfelRec* recs, uint32_t* zkeys, uint2* rects,
                             uint32_t* counts, const PreCam* cam2, SurfelRec* recs2, uint32_t* zkeys2,
                             uint2* rects2, hipStream_t s);
// The cells' masks of an ROI tile mask with T x T tiles (T = 8, 16 or 32)
// for a W x H image: a 16-tile is set iff it overlaps a set T-tile.
hipError_t launch_cell_masks(const uint8_t* tmask, int T, int W, int H, uint64_t* cells, hipStream_t s);
// Entries of the pass's surfels by cell, in compositing order; the key count
// goes to the status block (which: 0 dominant, 1 ROI).
hipError_t launch_bin_entries(const BinArgs& a, DevStatus* st, int which, hipStream_t s);
// Tile ranges, and the dispatch order of the (masked) tiles, heaviest first;
// with a mask also their number, in the status block.
hipError_t launch_tile_plan(const BinArgs& a, uint2* ranges, uint32_t* order, DevStatus* st, hipStream_t s);
// The tile lists (a.vals).
hipError_t launch_tile_write(const BinArgs& a, const uint2* ranges, hipStream_t s);
// One block per tile, in `order`; n_live (device, optional) limits
// the blocks that do work when the tile count is only known on the device.
// pair_counts (optional): the six blend counters of DevStatus::pairs.
hipError_t launch_blend(const SurfelRec* recs, const uint32_t* vals, const uint2* ranges, const uint32_t* order,
                        const uint32_t* n_live, int n_blocks,
                        const BlendArgs& a, const ContArgs& ca, float* rgb, float* d_or_z, float* alpha, uint8_t* cls,
                        unsigned long long* pair_counts, long long* trace, hipStream_t s);
// One frame's blend of a batch (one eye of one stereo pair), in device
// memory: a persistent launch renders the tiles of every frame of the batch
// from a shared work queue.
struct BatchBlendDesc {
    const SurfelRec* recs;
    const uint32_t* vals;
    const uint2* ranges;
    const uint32_t* order;      // dispatch order of the (masked) tiles, heaviest first
    const uint32_t* n_live;     // masked tiles (masked passes); null: n_tiles
    uint32_t n_tiles;
    uint32_t reserved;
    BlendArgs a;
    float* rgb;
    float* dz;
    float* alpha;
    uint8_t* cls;
};
// Copy a descriptor (a kernel argument) into device memory.
hipError_t launch_put_desc(const BatchBlendDesc& d, BatchBlendDesc* dst, hipStream_t s);
// Blend every tile of n frames: item prefix over the frames, then one
// persistent launch of `grid` workgroups that take (frame, tile) items from
// a queue counter in turn until all are done (no waits between workgroups).
// scratch: n + 2 words (prefix and counter).  patch: the frames are ROI
// passes (the patch writes).
hipError_t launch_blend_batch(const BatchBlendDesc* descs, int n, uint32_t* scratch, int grid, bool patch,
                              hipStream_t s);

// ---- reprojection and classification (warp.hip, no fp contraction) -------
struct WarpCam {
    int W, H;
    double fx, fy, cx, cy, z_near, z_far;
};
struct RelPose {
    double M[9], c[3];
};
RelPose rel_pose(const bgs_camera& src, const bgs_camera& dst);

// Per-block partials the reprojection leaves in wpart (row-preserving form:
// one per row; the scatter form reduces with atomics and leaves none).
int warp_parts(const WarpCam& src, const WarpCam& dst, const RelPose& P);
// reset: clear the status fields the reprojection and classification
// accumulate (not needed when the whole status block was zeroed);
// depth_range (optional): fold the partials into the status block and
// write the covered depth-proxy range there; without it the classification
// that follows folds them.
hipError_t launch_reproject(const WarpCam& src, const WarpCam& dst, const RelPose& P, float a_min,
                            const float* rgb, const float* draw, const float* alpha, unsigned long long* zbuf,
                            float* rgb_dst, float* z_dst, float* alpha_dst, uint8_t* hole, float* depth_range,
                            bool reset, uint4* wpart, DevStatus* st, hipStream_t s);
struct ClassifyBufs {
    uint8_t* hole;     // interpolation tags
    uint8_t* hole2;    // center-hole mask
    uint32_t* bcount;  // component roots per 1024-pixel block, then their exclusive scan
    unsigned long long* rmask;  // per 64 pixels: bit mask of the component roots
    uint8_t* pflag;    // tile-local piece roots
    int4* pbox;        // piece boxes, indexed by root pixel; then the component's at its root
    uint4* wpart;      // reprojection partials (warp_parts entries)
    uint2* gpart;      // gap-fill partials, one per gap-fill block
};
// depth_range null: take the range from the reprojection just run (its
// partials in b.wpart and its status fields).
hipError_t launch_classify(const WarpCam& src, const WarpCam& dst, const RelPose& P, const bgs_roi_params& roi,
                           const float bg[3], const float* depth_range, float* rgb, float* z, float* alpha,
                           uint8_t* cls, int32_t* labels, bgs_box* boxes, int32_t box_cap, int32_t* n_boxes,
                           uint8_t* tile_mask, const ClassifyBufs& b, DevStatus* st, hipStream_t s);
hipError_t launch_label_components(const uint8_t* mask, int W, int H, int conn, int32_t* labels,
                                   hipStream_t s);

}  // namespace bgs
