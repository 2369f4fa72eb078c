// Internal declarations shared by the rkhsba HIP translation units.
// Device data layout (all frames concatenated, HBM-resident between calls):
//   pts   float4[N_total]  frame-local xyz of each frame's points in cell-key order;
//                          .w holds the class id bits (class features) or 0
//   feat  float[N_total*Dp] dense feature rows in the same order (zero padded to Dp)
//   perm  int32[N_total]   sorted position -> original index within the frame
//   keys  uint32[N_total]  sorted cell keys, ((kz' * NY) + ky) * NX + kx with kz' = kz, or for class ids in a
//                          label-stacked frame kz' = label * NZ + kz (each class id has a layer of NZ cells)
//   rows  int4[sum NY*NZ*L] per (ky,kz') row of cells: (x_lo, x_hi, xtab offset, 0); L label layers (1 unstacked)
//   xtab  uint32[...]      per row, for x in [x_lo, x_hi+1]: first point of cell x
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <string>
#include <vector>

namespace rkhsba {

// Binning keys: a 30-bit Morton code of the source point's target-frame cell (clamped to the grid and its
// margin), with this bit set when the point lies outside both (it has no pair).  The last 8-bit digit of codes of
// more than 24 bits includes it, so that those points come last; shorter codes leave them at their clamped place.
constexpr uint32_t kOutsideBit = 0x80000000u;
constexpr int kMaxDense = 64;

enum Mode { MODE_LOSS = 0, MODE_NORMAL = 1 };
// Feature paths (values equal the public feature kinds): class ids, dense
// FP32 rows, dense rows stored in bfloat16 or fp8 e4m3 (inner products on the
// matrix cores with FP32 accumulation).
enum FeatPath { FEAT_CLASS = 0, FEAT_DENSE = 1, FEAT_BF16 = 2, FEAT_FP8 = 3 };
__host__ __device__ constexpr bool feat_low_precision(int f) { return f == FEAT_BF16 || f == FEAT_FP8; }
__host__ __device__ constexpr int feat_elem_bytes(int f) { return f == FEAT_DENSE ? 4 : f == FEAT_BF16 ? 2 : 1; }

// Per-frame grid description (device and host copies).
struct FrameInfo {
  int64_t pt_off;    // first point of the frame in pts/feat/perm/keys
  int32_t n;         // points
  int32_t org[3];    // cell coordinates of the grid origin
  int32_t dim[3];    // cells per axis
  int32_t mort_shift;  // source-binning Morton code: (k + reach) >> mort_shift
  int64_t row_off;   // first row descriptor of the frame
  int64_t xt_off;    // first xtab entry of the frame
  int32_t n_lab;     // label layers of a label-stacked frame (class id + 1 of its largest id), 0: not stacked
  int32_t key_sub;   // source-binning key resolution: 2^key_sub sub-cells per cell and axis
};

// First row descriptor (relative to row_off) of the layer of class id lbl: 0 in a frame that is not
// label-stacked, -1 where the frame has no layer for that id (no point of the frame carries it).
__host__ __device__ inline int64_t label_rows(const FrameInfo& T, uint32_t lbl) {
  if (T.n_lab <= 0) return 0;
  if (lbl >= (uint32_t)T.n_lab) return -1;
  return (int64_t)lbl * T.dim[1] * T.dim[2];
}

// Static per-edge layout of one edge list (host-computed once per list).
struct EdgeInfo {
  int32_t m, n;      // source frame, target frame
  int64_t ent_off;   // first binning entry (one per source point)
  int32_t n_src;     // source points (= frame m's count)
  int32_t pass_size; // source points per sweep pass of the edge (its problem's choice)
  int32_t n_pass;
  int32_t fin_off;   // first finalize block of the edge
  int32_t n_fin;
  int32_t fin_pt;    // entries per finalize thread (a block covers kFinThreads * fin_pt entries)
  int32_t prob;      // problem of the edge within the evaluated set (constants, system)
  int32_t pass0;     // first pass of the edge in the set's pass table
  int32_t seg0;      // first binning segment of the edge (one per class id of a label-stacked source frame,
  int32_t n_seg;     // else one): passes never straddle a segment
};

// One sweep pass: up to pass-size consecutive binning entries of one segment of an edge.
struct PassInfo {
  int64_t entry0;    // first binning entry
  int64_t src_off;   // pool offset of the source frame's points
  int32_t e;         // edge (set-wide)
  int32_t count;     // entries in the pass
  int32_t tgt;       // target frame slot
  int32_t prob;      // problem (constants)
};

// Relative transform of an edge, T_nm = T_n^-1 T_m (FP64), written on device.
struct EdgeXf {
  double R[9];
  double t[3];
};

// Kernel constants derived from the options (host-computed in FP64).
struct KConst {
  double inv_cell;   // 1 / cell edge
  double cell;       // cell edge = r_c / cell_subdiv
  double reach;      // r_c * (1 + 2^-12): covers every pair the FP32 rule accepts
  double reach2;
  float rc2;         // float(r_c * r_c), the FP32 membership threshold
  float alpha;       // log2(e) / (2 ell^2), so that exp(-r^2/2l^2) = exp2(-alpha r^2)
  int reach_cells;   // cell_subdiv + 1
  int clamp;         // clamp negative c to 0 (only set when some feature value is negative)
  int Dp;            // padded dense feature width (0 for class ids)
  int topk;          // > 0: only the topk pairs with the largest kernel values per source point (per edge)
  double inv2l2;     // 1 / (2 ell^2), for the FP64 ranking key of the topk selection
  int c_positive;    // FP32 dense features, none negative, and one dimension >= 1e-18 in every row: every
                     // inner product is > 0 (its term in that dimension is >= 1e-36, above FLT_MIN)
  float r_c;           // truncation radius
  float spread_limit;  // class-id sweeps: passes whose box is wider than this walk per source point
};
constexpr int kMaxTopK = 8;

// A piece of a segment to be sorted: a tile of the LSD radix sort, or a run that one workgroup sorts in LDS.
struct SortTile {
  int64_t start;     // first element
  int32_t count;     // elements (<= kSortTile)
  int32_t seg;       // segment id
  int32_t edge;      // edge of the binning entries (edge sorts), or the frame (point sorts)
  int32_t runs;      // runs of the segment (tiles: 0)
};
struct SortSeg {
  int64_t start;
  int32_t count;     // elements (a frame's or a class id's points, < 2^31)
  int32_t owner;     // edge of the binning entries (edge sorts), or the frame (point sorts)
  int32_t tile0;     // first tile
  int32_t n_tiles;   // 0: sorted in runs (at most kMergeMax elements)
};
constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;
// Segments of at most this many elements are sorted in runs of kSortTile, all digits in one launch, and the runs of a
// segment of several are merged by a second.  Larger ones take two launches per digit.  The merge reads a segment's
// keys once per run (four times up to 128 runs, whose workgroups it splits) and searches every other run: 12 segments
// of 16,000 elements 12.8 + 12 us, and 28 of 30,000 18 + 55, where the tiles take 63.
constexpr int kMergeMax = 16384;

// How the segments of one launch are sorted.
struct SortPlan {
  int n_segs = 0;
  int n_tiles = 0;        // tiles of the segments above kMergeMax
  int max_seg_tiles = 0;  // most tiles of one segment
  int n_multi = 0;        // runs of the segments of several runs
  int n_runs = 0;         // those and the segments of one run
  int max_multi = 0;      // largest segment of several runs
};
// The tables of a plan: segments, and pieces in the order tiles, runs of several, single runs.
struct SortTables {
  SortPlan plan;
  std::vector<SortSeg> segs;
  void add(int64_t start, int64_t count, int32_t owner) {
    SortSeg S{};
    S.start = start;
    S.count = (int32_t)count;
    S.owner = owner;
    S.tile0 = plan.n_tiles;
    const int pieces = (int)((count + kSortTile - 1) / kSortTile);
    const bool tiled = count > kMergeMax;
    std::vector<SortTile>& list = tiled ? tiles_ : pieces > 1 ? multi_ : single_;
    for (int64_t s = 0; s < count; s += kSortTile)
      list.push_back(SortTile{start + s, (int32_t)(count - s < kSortTile ? count - s : kSortTile), plan.n_segs, owner,
                              tiled ? 0 : pieces});
    if (tiled) {
      S.n_tiles = pieces;
      plan.n_tiles += pieces;
      if (pieces > plan.max_seg_tiles) plan.max_seg_tiles = pieces;
    } else {
      plan.n_runs += pieces;
      if (pieces > 1) plan.n_multi += pieces;
      if (pieces > 1 && S.count > plan.max_multi) plan.max_multi = S.count;
    }
    segs.push_back(S);
    ++plan.n_segs;
  }
  std::vector<SortTile> pieces() const {
    std::vector<SortTile> all(tiles_);
    all.insert(all.end(), multi_.begin(), multi_.end());
    all.insert(all.end(), single_.begin(), single_.end());
    return all;
  }

 private:
  std::vector<SortTile> tiles_, multi_, single_;
};

// ---------------------------------------------------------------- launchers
// Each returns hipSuccess or the first HIP error.  All run on `st`.

// Digit passes of the tiled segments, over key bits [0, bits); the tiles' counts of digit 0 are in `hist` already.
// keep_keys: the sorted keys are wanted too, not only the values.  The result ends in (keys, vals) or, for an odd
// number of digits, in (keys_tmp, vals_tmp): sort_ends_in_tmp(bits).
hipError_t launch_radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_tmp, uint32_t* vals_tmp,
                             uint32_t* hist, const SortTile* d_tiles, const SortSeg* d_segs, const SortPlan& plan,
                             int bits, bool keep_keys, hipStream_t st);
// Merges the sorted runs of the segments of several, from (keys, vals) to (out_keys, out_vals); out_keys may be null.
hipError_t launch_merge(const uint32_t* keys, const uint32_t* vals, const SortTile* d_pieces, const SortSeg* d_segs,
                        const SortPlan& plan, uint32_t* out_keys, uint32_t* out_vals, hipStream_t st);
inline bool sort_ends_in_tmp(int bits) { return (((bits + 7) / 8) & 1) != 0; }

hipError_t launch_exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* tmp, uint64_t* d_total,
                                 hipStream_t st);
constexpr int kScanTileElems = 2048;

// Padded feature row length: 8, 16, 24, 32 or 64 (FP32), 32 or 64 (bfloat16, fp8: whole 32-wide MFMA slices).
int dense_pad(int D, int feat_path);

// Smallest and largest coordinate of every frame, [6 f + 0..2] and [6 f + 3..5] of d_bounds (which the caller sets to
// all ones and zero), as the floats' bits in unsigned order; *d_bad is set where a coordinate is not finite.  n_max:
// points of the largest frame.  d_label_max (class ids, else null): per frame, the largest class id (max-combined;
// the caller sets -1).
hipError_t launch_frame_bounds(const float* const* d_xyz_ptrs, const int64_t* d_in_off, int K, int64_t n_max,
                               const void* const* d_class_ptrs, uint32_t* d_bounds, int32_t* d_bad,
                               int32_t* d_label_max, hipStream_t st);
inline float float_of_ordered(uint32_t o) {
  const uint32_t u = (o & 0x80000000u) ? o & 0x7fffffffu : ~o;
  float v;
  std::memcpy(&v, &u, sizeof(v));
  return v;
}
// Cell keys (frames with n_lab > 0 take the class ids, d_class_ptrs, into kz') and their sort by frame, stable.
// Frames of at most kMergeMax points end in (d_sorted_keys, d_sorted_vals), by way of (d_run_keys, d_run_vals); the
// keys and values of the others are left in (d_keys, d_vals), with their tiles' counts of digit 0, for
// launch_radix_sort.
hipError_t launch_cell_sort(const float* const* d_xyz_ptrs, double inv_cell, const FrameInfo* d_frames,
                            const void* const* d_class_ptrs, const SortTile* d_tiles, const SortSeg* d_segs,
                            const SortPlan& plan, int bits, uint32_t* d_keys, uint32_t* d_vals, uint32_t* d_hist,
                            uint32_t* d_run_keys, uint32_t* d_run_vals, uint32_t* d_sorted_keys,
                            uint32_t* d_sorted_vals, hipStream_t st);
// For every label-stacked frame f (frame-local key order) and class id l in [0, n_lab]: the first point
// of layer l (l = n_lab: the frame's count), at d_out[d_lab_off[f] + l].
hipError_t launch_label_starts(const uint32_t* d_keys, const FrameInfo* d_frames, const int64_t* d_lab_off, int K,
                               int32_t* d_out, hipStream_t st);
hipError_t launch_gather(const float* const* d_xyz_ptrs, const void* const* d_feat_ptrs, int feat_kind, int D, int Dp,
                         const int64_t* d_in_off, int K, int64_t n_total, const uint32_t* d_sorted_keys,
                         const uint32_t* d_sorted_vals, float4* d_pts, void* d_feat, int32_t* d_perm,
                         uint32_t* d_keys, int32_t* d_neg_flag, hipStream_t st);
// Per feature dimension d < Dp (<= 64), the smallest stored FP32 value over n rows, as its bit pattern (values
// >= 0; negative values count as 0), min-combined into d_min[d], which the caller sets to +inf first.
hipError_t launch_feature_min(const float* d_feat, int64_t n, int Dp, uint32_t* d_min, hipStream_t st);
// Row tables (x extents and x-table offsets) of sorted frames; d_totals[0] = x-table entries, [1] = occupied cells.
hipError_t launch_rows(const uint32_t* d_keys, const FrameInfo* d_frames, const int64_t* d_in_off, int K,
                       int64_t n_total, int4* d_rows, int64_t n_rows, uint32_t* d_sizes, uint32_t* d_scan_tmp,
                       uint64_t* d_totals, hipStream_t st);
hipError_t launch_xtab(const uint32_t* d_keys, const FrameInfo* d_frames, const int64_t* d_in_off, int K,
                       int64_t n_total, const int4* d_rows, uint32_t* d_xtab, hipStream_t st);

// Small transfers (transfer.hip): up to kMaxPieces pieces of whole 32-bit words in one launch.
constexpr int kMaxPieces = 6;
constexpr size_t kPutBytes = 3584;   // an upload's payload (a kernel's arguments are at most 4 KB)
constexpr size_t kGetBytes = 16384;  // a download's pieces together
struct Upload {
  void* dst;        // device
  const void* src;  // host, free again on return
  size_t bytes;
};
struct Download {
  void* dst;        // host
  const void* src;  // device
  size_t item;      // bytes of an item
  size_t count = 1;
  size_t stride = 0;  // bytes from one item to the next
};
bool put_fits(const Upload* up, int n);
hipError_t launch_put(const Upload* up, int n, hipStream_t st);
hipError_t launch_get(const Download* dn, int n, void* pinned, hipStream_t st);

// Mean of n points' xyz in FP64 (one workgroup, fixed summation order) -> out[3].
hipError_t launch_frame_centroid(const float4* d_pts, int n, double* d_out, hipStream_t st);

// The pass table of a set from its edge table: passes pass0 .. pass0 + n_pass - 1
// of each edge cover each of its segments in runs of pass_size (64 for per-point walks).
hipError_t launch_fill_passes(const EdgeInfo* d_edges, int E, const FrameInfo* d_frames, const SortSeg* d_segs,
                              PassInfo* d_passes, hipStream_t st);
// d_n_items (nullable): the sweep's item counter, cleared here.
hipError_t launch_edge_setup(const double* d_poses, const EdgeInfo* d_edges, int E, EdgeXf* d_xf, uint32_t* d_n_items,
                             hipStream_t st);
// Source binning.  Segments of at most kMergeMax entries: their sorted source indices written to d_sorted, by way of
// (d_keys, d_run_vals), d_run_vals another array than d_sorted.  The others: keys and source indices of every entry, one block per tile,
// with the tile's counts of digit 0, for launch_radix_sort.
hipError_t launch_bin(const float4* d_pts, const FrameInfo* d_frames, const EdgeInfo* d_edges,
                      const SortTile* d_tiles, const SortSeg* d_segs, const SortPlan& plan, const EdgeXf* d_xf,
                      const KConst* d_kcs, int bits, uint32_t* d_keys, uint32_t* d_vals, uint32_t* d_hist,
                      uint32_t* d_run_vals, uint32_t* d_sorted, hipStream_t st);

// Passes whose box spans more rows than this skip the batches of rows that no source of theirs is near.  The
// sources of such a pass lie in a few places far apart (a jump of the Morton order), and most rows of the box
// around them all lie between: a box across a frame of 8 m in cells of 3 cm has 70,000 rows.  One wavefront
// enumerates them 64 at a time, and such passes set the time of a launch.  Tested 64 batches at once, one per
// lane.  The batches kept are enumerated as without the test, so the order of a source's candidates is the same.
// Sweep of 8 depth frames x 30,000 points, 23 dimensions, 28 edges: 1342 -> 1000 us; 5 x 12,345 points, fp8:
// 282 -> 163 us; 4 x 8,000 points, 20 dimensions: 180 -> 102 us.  Boxes of fewer rows would pay more for the test
// (a compact pass has about (2 + box / r_c)^2 cell_subdiv^2 rows: 450 at 8 cells per r_c) than the few batches it
// could skip.
constexpr int kManyRows = 512;

// Dense-feature passes whose box is wider than split_factor(passes of the launch) truncation radii and spans more
// than kSplitRows rows are split over their sources (sweep_dense.hip).  A split pass costs more work in all, and
// ends sooner: few passes are bound by the longest one, many by the work.  Sweep times in us, split at 2 / 4 r_c
// (not at all): 8 x 30,000 points, 52,500 passes 907 / 844 (1004); 3 x 60,000, 11,250 passes 1987 / 2268 (2350); 3 x
// 9,000 bfloat16, 1,700 passes 48 / 73 (86); 4 x 8,000, 3,000 passes 70 / 82 (113).  Boxes of a few rows (two to four
// batches) are walked faster than they are split: 5 x 12,345 fp8 102 from 256 rows on, 111 from 128.
constexpr int kSplitRows = 256;
inline float split_factor(int64_t n_pass) { return n_pass <= 16384 ? 2.f : 4.f; }
// Room for the items of a launch of n_pass passes.  The sweep's grid holds a workgroup for every pass and every item
// that could be listed, so the list of a large set, which is bound by its work and not by its longest passes, ends at
// 65,536; and it leaves the grid below 2^26 workgroups of 64, the most that a launch takes.
inline uint32_t max_items(int64_t n_pass) {
  const int64_t room = (1ll << 26) - 1 - n_pass, most = n_pass + 64 < 65536 ? n_pass + 64 : 65536;
  return n_pass <= 0 || room <= 0 ? 0u : (uint32_t)(most < room ? most : room);
}

struct PairArgs {
  const float4* pts;
  const void* feat;       // feature rows (element type by feature path), Dp elements per point
  const int4* rows;
  const uint32_t* xtab;
  const FrameInfo* frames;
  const EdgeInfo* edges;
  const EdgeXf* xf;
  const uint32_t* vals;   // source points in binning order (frame-local sorted index)
  float* mom;             // moments, component-major: mom[c * n_entries + entry]
  uint32_t* cnt;          // in-radius pair count per entry
  const KConst* kcs;      // per problem of the set, indexed by EdgeInfo::prob
  const int32_t* perm;    // sorted position -> original index (ties of the topk selection)
  const PassInfo* passes; // per sweep pass
  int64_t n_entries;
  int32_t E;
  int32_t pass0;          // first pass of this launch in the pass table
  int32_t n_pass;         // passes of this launch
  KConst kc;              // set-wide: Dp and clamp (clamping is exact for non-negative features)
  uint2* items;           // the spread passes of dense features, split: (pass, source mask); null: not split
  uint32_t* n_items;      // items listed (zero when the sweep's first kernel begins)
  uint8_t* split;         // per pass of the launch: listed as items
  uint32_t item_cap;
  float split_factor;     // passes whose box is wider than this many truncation radii count as spread
  int32_t stacked;        // every frame of the set is label-stacked (class ids): a candidate of the pass's
                          // layer always carries the pass's class id, and the sweeps skip that test
};
// Passes of pass_points sources: 1 = each lane walks its own point's cells,
// 8 (class ids) and 16 (launch_sweep), 32, 64 = shared walk over the pass's box.
hipError_t launch_pairs(const PairArgs& a, int mode, int feat_path, int pass_points, bool topk, hipStream_t st);

// Tiled sweep for passes of 16 sources, or 8 with class ids.  source_counts (Gauss-Newton moments on the
// VALU only): each entry of a.cnt receives its own source point's pair count instead of the pass total on
// the pass's first entry (the per-edge sums are the same).
hipError_t launch_sweep(const PairArgs& a, int mode, int feat_path, int pass_points, bool matrix_moments,
                        bool source_counts, hipStream_t st);

// Tiled sweep of dense features, passes of 16 sources, moments on the VALU; source_counts as above.
hipError_t launch_sweep_dense(const PairArgs& a, int mode, int feat_path, bool source_counts, hipStream_t st);

// Where element k of a dense feature row is stored: FP32 rows are stored column by column of the 16x16x4 matrix
// instruction's operand (elements 4i + g for i = 0, 1, ... at g * Dp / 4), the others in order.
__host__ __device__ constexpr int feat_slot(int feat_path, int Dp, int k) {
  return feat_path == FEAT_DENSE ? (k & 3) * (Dp / 4) + (k >> 2) : k;
}

struct FinArgs {
  const float4* pts;
  const EdgeInfo* edges;
  const EdgeXf* xf;
  const FrameInfo* frames;
  const uint32_t* vals;
  const float* mom;
  const uint32_t* cnt;
  const KConst* kcs;      // per problem of the set, indexed by EdgeInfo::prob
  double* partial;        // [n_fin_total][kFinStats]
  int64_t n_entries;
  int32_t E;
  int32_t n_fin_total;
};
constexpr int kEdgeVals = 93;  // F, b_m(6), b_n(6), H_mm(21), H_nn(21), H_mn(36), pair count, sum w r^2
constexpr int kFinThreads = 256;
constexpr int kFinStats = 40;  // per-edge sums the normal-equation blocks are expanded from, sum w r^2, F, pair count
// fp32_sums: per-point terms and their sums in FP32 with Kahan compensation,
// else FP64.  Pair counts are summed in FP64.
hipError_t launch_finalize(const FinArgs& a, const int32_t* d_fin_off, int mode, bool fp32_sums, hipStream_t st);
hipError_t launch_edge_reduce(const double* d_partial, const EdgeInfo* d_edges, const EdgeXf* d_xf, int E, int mode,
                              bool fp32_sums, double* d_edge_out, hipStream_t st);

// One problem's Gauss-Newton system within an evaluated set.
struct ProbSys {
  int32_t K;          // frames
  int32_t fixed;      // frame removed from the system (-1: none)
  int32_t n;          // system size: 6K, or 6(K-1) with a fixed frame
  int32_t e0, E;      // edges of the problem in the set's edge table
  int32_t blk0;       // first entry of the problem's K*K+1 block-contributor starts
  int32_t vec0;       // first entry of the problem's K+1 vector-contributor starts
  int32_t n_iter;     // Gauss-Newton iterations; solves stop once iter reaches it
  int64_t slot0;      // first frame slot (frame table, poses)
  int64_t h_off;      // offset of the problem's n x n matrix in the set's H buffer
  int64_t v_off;      // offset of its n-vectors in b and delta
  int64_t hist_off;   // offset of its loss and pair-count histories (n_iter + 1 each)
  int64_t state_off;  // offset of its (iter, status) pair
  double sigma2;
  double damping_rel;
  int32_t plan0;      // first word of its block-sparse elimination plan in the set's plans (-1: none)
  int32_t pad_;
};

struct SolveArgs {
  const double* edge_out;  // [E][kEdgeVals]
  const ProbSys* sys;      // [n_prob]
  int32_t n_prob;
  int32_t n_max;           // largest system size of the set
  double* H;
  double* b;
  double* delta;
  double* poses;           // [slot][12], updated in place by the solve
  double* loss_hist;       // F per evaluation, at hist_off + iter
  double* pairs_hist;      // in-radius pair count per evaluation
  int32_t* state;          // per problem: iter (evaluations whose solve ran), status (0 ok, -4 not PD; sticky)
  // contributors of each 6x6 block (frame a, frame c) of a problem's H, CSR over blk0 + a*K + c:
  // entries e*4 + role (set-wide edge index), role 0 H_mm, 1 H_nn, 2 H_mn, 3 H_mn^T
  const int32_t* blk_start;
  const int32_t* blk_list;
  // contributors of each frame's 6-vector of b, CSR over vec0 + a: entries e*2 + role, role 0 b_m, 1 b_n
  const int32_t* vec_start;
  const int32_t* vec_list;
  const uint16_t* plans;   // block-sparse elimination plans (solve_plan.h)
};
// What follows an evaluation's finalisation: nothing but the per-edge values, the loss and pair-count history
// entry, also H and b, or the whole Gauss-Newton step.
enum Step { STEP_NONE = 0, STEP_LOSS = 1, STEP_SYSTEM = 2, STEP_SOLVE = 3 };
struct StepArgs {
  const double* partial;   // finalisation partial sums (null: edge_out holds the edges' values already)
  const EdgeInfo* edges;
  EdgeXf* xf;              // STEP_SOLVE leaves those of the moved poses
  double* edge_out;
  uint32_t* n_items;       // cleared (nullable)
};
// Whether one workgroup takes a problem's whole step: the system fits in LDS, and assembling it reads few edges.  It
// takes their sums too where each wavefront has one edge and few finalisation blocks (sum_in_step; 2 edges each: 7 us
// of one CU, as much as a launch that spreads them; 28 edges of 118 blocks: 1 MB through one CU, 30 us).
constexpr int kStepEdges = 64;
bool small_step(const ProbSys& S);
inline bool sum_in_step(int edges, int64_t fin_blocks) { return edges <= 16 && fin_blocks <= 512; }
// The step of every problem of a set of small ones.
hipError_t launch_step(const SolveArgs& a, const StepArgs& u, int mode, int step, bool fp32_sums, hipStream_t st);
// Writes H, b of every problem (and the loss / pair-count history entry of the
// current iteration).
hipError_t launch_assemble(const SolveArgs& a, hipStream_t st);
// Loss / pair-count history entry only (loss evaluations).
hipError_t launch_loss_only(const SolveArgs& a, hipStream_t st);
// Damped Cholesky solve and pose update of every problem whose iteration count
// is below its n_iter; advances the iteration count of every problem.
hipError_t launch_solve_update(const SolveArgs& a, hipStream_t st);

// out[0] = sum of F, out[1] = sum of pair counts over the E per-edge rows of edge_out (edge order).
hipError_t launch_edge_totals(const double* d_edge_out, int E, double* d_out, hipStream_t st);

hipError_t launch_export_pairs(const float4* d_pts, const int4* d_rows, const uint32_t* d_xtab,
                               const FrameInfo* d_frames, int n_src, const int32_t* d_perm, const void* d_feat,
                               const EdgeXf* d_xf, int m, int n, int feat_path, KConst kc, int64_t cap, int32_t* d_out,
                               unsigned long long* d_count, hipStream_t st);

}  // namespace rkhsba
