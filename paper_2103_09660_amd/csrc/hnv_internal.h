// Internal declarations shared by the host code (hnv_host.cpp) and the HIP
// kernels (hnv_kernels.hip).  Not part of the public ABI.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "hnv.h"

typedef struct ihipStream_t *hipStream_t;

#ifdef __HIP__
#define HNV_HD __attribute__((host)) __attribute__((device))
#else
#define HNV_HD
#endif

namespace hnv {

constexpr int kBlock = 256;   // threads per workgroup (4 wavefronts of 64)
constexpr int kWave = 64;
constexpr int kWavesPerBlock = kBlock / kWave;

// A work item: `len` neighbours of side-local row `row` starting at `start`
// in the side's neighbour array.
//   lane-group tier: len = the row's degree, aux = the row of the next
//     coarser level its value is projected from (0 at the coarsest level);
//   wavefront tier: aux = -1 if the item is the whole row (len = its
//     degree), else the partial slot it writes; a finalize pass combines a
//     split row's slots in order.
struct alignas(16) Item {
    int32_t row, start, len, aux;
};
// The first kInlineIds neighbour ids of a lane-group row (unused entries 0),
// kept beside its work item so that a row of that many neighbours or fewer
// needs no load of its own index list.
constexpr int kInlineIds = 4;
struct alignas(16) InlineIds {
    int32_t id[kInlineIds];
};
// A row split over n_slots consecutive partial slots starting at first_slot.
struct alignas(16) Split {
    int32_t row, first_slot, n_slots, deg;
};

// One side of the star expansion of a level, as device arrays.
//   side 0: hyperedge rows, neighbours = member nodes (hyperedge->members)
//   side 1: node rows, neighbours = incident hyperedges (node->hyperedges)
struct DevSide {
    int32_t n_rows = 0;
    int32_t row_base = 0;            // Z row of local row 0 (n_nodes for side 0, 0 for side 1)
    const int32_t *ptr = nullptr;    // [n_rows + 1]
    const int32_t *idx = nullptr;    // [nnz] neighbour Z row at this level
    const int32_t *cidx = nullptr;   // [nnz] neighbour Z row at the next coarser level, or null
    float *wn = nullptr;             // [nnz] weight of each star edge (side 1 only)
    float *sn = nullptr;             // [nnz] reverse-mode scale: reciprocal of the neighbour's row sum
    const Item *small = nullptr;
    const InlineIds *small_ids = nullptr;    // [n_small] first ids of each small row, from idx
    const InlineIds *small_cids = nullptr;   // [n_small] the same from cidx, or null
    int32_t n_small = 0;
    const Item *chunks = nullptr;
    int32_t n_chunks = 0;
    const Split *splits = nullptr;
    int32_t n_splits = 0;
};

// Device-side state of a refinement that stops a level early (Section 3.3's
// epsilon rule) without reading residuals back on the host.  The sweeps and
// projections of such a refinement take their input and output matrices
// from here; the last kernel of each operation advances them, and the
// residual of each sweep is compared with tol on the device, setting the
// level's stop flag, after which that level's remaining sweeps do nothing.
struct SweepCtl {
    const void *cur;      // matrix holding the latest iterate
    void *next;           // buffer the next operation writes
    void *buf[2];         // the two buffers the refinement alternates between
    double *res;          // residual of each sweep run, packed in run order, or null
    double *res_tmp;      // [1] residual of the last sweep when res is null
    int32_t *stop;        // [n_levels] 1 once a sweep of the level changed Z by <= tol
    int32_t *done;        // [n_levels] sweeps run per level
    double tol;
    int64_t n_res;        // sweeps run so far (next index into res)
};

struct LevelPlan {
    int64_t n_nodes = 0, n_edges = 0, nnz = 0, rows = 0;
    int64_t rows_coarse = 0;         // rows of level + 1 (0 at the coarsest level)
    bool has_coarse = false;
    bool unit_w = true;
    int small_max = 0;               // lane-group tier bound of the level
    int long_len = 0;                // items of more neighbours than this take a workgroup,
    int few_items = 0;               // or all of them if there are at most this many
    int chunk = 0;                   // rows of more neighbours than this are cut,
    int split_over = 0;              // than this if the level has a row of more than a chunk,
    int cut = 0;                     // into items of this many
    int slot_pieces = 1;             // pieces per such item in the order that serves gradients
    bool deep = false;               // the level doesn't fill the chip: more loads in flight there
    bool scales_ready = false;       // the reverse-mode scales (side[*].sn) hold the current weights
    DevSide side[2];
    float *r = nullptr;              // [rows] 1 / (row weight sum), 0 for rows without neighbours
    float *w = nullptr;              // [n_edges] current hyperedge weights
    int32_t *rowmap = nullptr;       // [rows] -> row of level + 1
    int32_t *inv_ptr = nullptr;      // [rows_coarse + 1]
    int32_t *inv_idx = nullptr;      // [rows] fine rows grouped by coarse row, ascending
    int32_t n_slots = 0;             // partial slots used by split rows (both sides)
    // host copies of the work-list sizes (for launch geometry)
    int32_t n_small[2] = {0, 0}, n_chunks[2] = {0, 0}, n_splits[2] = {0, 0};
    int32_t n_long[2] = {0, 0};      // leading chunks that a whole workgroup takes
    // in the order that serves gradients: leading chunks of more than a piece,
    // and of more than lane_most neighbours (the others take a lane group)
    int32_t n_pieced[2] = {0, 0}, n_wide[2] = {0, 0};
};

}  // namespace hnv

namespace hnv {
// Sweeps of one level whose residuals a fixed-count refinement reduces
// together (their per-block partials wait in as many slots).
constexpr int kResidBatch = 8;
// Per-block residual partials one workgroup of a residual stage sums, and the
// most that one workgroup takes where that ends the reduction: each stage is a
// launch of about 4 us, as much as a sweep of a small level.
constexpr int kResidPer = kBlock * 8;
constexpr int kResidLast = 4 * kResidPer;
// Sweeps of a small level that one launch runs from LDS when residuals are
// wanted, and the LDS bytes that it takes.
constexpr int kResidentBatch = 2 * kResidBatch;
constexpr int64_t kResidentLds = 160 * 1024;
}  // namespace hnv

struct hnv_plan {
    int n_levels = 0;
    int d = 0;
    hnv_dtype dtype = HNV_F32;
    hnv_options opts{};
    std::vector<hnv::LevelPlan> lv;
    void *zbuf = nullptr;            // scratch embedding [rows of level 0 x d]
    float *partials = nullptr;       // [max_slots x pstride]
    int32_t pstride = 0;             // floats per partial slot (d + 8)
    int64_t max_slots = 0;
    // the order that serves gradients: rows of up to lane_most neighbours one
    // after another, longer ones in pieces
    int lane_most = 0, piece = 0;
    double *resid_part = nullptr;    // [kResidBatch x max_resid_blocks] per-block partials, one slot per sweep
    int64_t max_resid_blocks = 0;
    double *resid_stage = nullptr;   // [2 x kResidBatch x resid_stage_len] partial sums of the residual stages
    int64_t resid_stage_len = 0;
    uint32_t *resident_trace = nullptr;  // [resident_words] rows before and after sweeps run from LDS
    int64_t resident_words = 0;
    double *resident_part = nullptr;     // [kResidentBatch x resident_blocks] their per-block partials
    int64_t resident_blocks = 0;
    float *cscratch = nullptr;       // [max n_nodes] per-node scalar of the reverse sweep
    double *resid_tmp = nullptr;     // [1]
    hnv::SweepCtl *ctl = nullptr;    // [1] early-stop control (device)
    int32_t *ctl_flags = nullptr;    // [2 x n_levels] its stop flags and sweep counts
    int panels = 1;                  // column passes of a forward sweep
    int dp = 0;                      // columns per pass
    int g_fwd = 1;                   // lanes per row in a forward pass
    int epl_fwd = 8;                 // elements per lane in a forward pass
    int g_full = 1;                  // lanes per full-width row
    int epl_full = 8;                // elements per lane of a full-width row
    size_t ws_bytes = 0;
    // kernel timing (hnv_plan_set_profiling)
    struct ProfRecord {
        int kind, level;
        void *ev_begin, *ev_end;   // hipEvent_t
    };
    bool profiling = false;
    std::vector<ProfRecord> prof;
    std::vector<void *> ev_pool;
    ~hnv_plan();
};

namespace hnv {

// thread-local error text
hnv_status fail(hnv_status st, const std::string &msg);
void clear_error();

int next_pow2(int x);
// Sort key of a wavefront-tier item of `len` of at most `chunk` neighbours:
// ascending keys put the longest first, to within 1/512 of a chunk, so that
// both sides' keys (2 chunk_keys) fit one counting pass of the GPU builder.
inline int chunk_shift(int chunk)
{
    int s = 0;
    while ((chunk - 1) >> s >= 512)
        ++s;
    return s;
}
inline int chunk_keys(int chunk) { return ((chunk - 1) >> chunk_shift(chunk)) + 1; }
// (an item of a split row counts as one of at least 65 neighbours, so that the
// last ones of an ascending list are whole rows)
constexpr int kSplitKeyLen = 65;
HNV_HD inline int item_key(int chunk, int shift, int len, bool split)
{
    const int least = chunk < kSplitKeyLen ? chunk : kSplitKeyLen;
    return (chunk - (split && len < least ? least : len)) >> shift;
}
inline int item_key(int chunk, int len, bool split) { return item_key(chunk, chunk_shift(chunk), len, split); }
// Items of more than `len` neighbours have keys below this (to within 1/512 of a chunk).
inline int key_above(int chunk, int len) { return (chunk > len ? chunk - len : 0) >> chunk_shift(chunk); }
// Lane layout of a row slice of `cols` elements of `elem` bytes: lanes move
// 16 B each, or 32 B for FP32 slices of 128 columns or more.
void lane_layout(int cols, int elem, int *lanes, int *elems_per_lane);
constexpr int kIdxRegs = 4;          // neighbour indices a lane preloads in the lane-group tier
int64_t blocks_for(int64_t items, int64_t per_block);

// Sizes and work-list counts of one level of a plan.
struct LevelShape {
    int64_t nV = 0, nE = 0, nnz = 0, rows = 0, rows_c = 0;
    bool has_coarse = false, unit_w = true;
    int32_t n_small[2] = {0, 0}, n_chunks[2] = {0, 0}, n_splits[2] = {0, 0}, n_long[2] = {0, 0};
    int32_t n_pieced[2] = {0, 0}, n_wide[2] = {0, 0};
    int32_t n_slots = 0;
};

// Where a level's lists of items are divided: an item's list is ascending by
// key, and its leading items below each of these keys are counted.
constexpr int kItemMarks = 3;   // LevelPlan's n_long (unless all items are), n_pieced, n_wide
struct ItemMarks {
    int32_t key[kItemMarks];
};
ItemMarks item_marks(const hnv_plan *p, const LevelPlan &L);
void set_item_counts(const hnv_plan *p, const LevelPlan &L, const int32_t (&n_chunks)[2],
                     const int32_t (&marks)[kItemMarks][2], int32_t (&n_long)[2], int32_t (&n_pieced)[2],
                     int32_t (&n_wide)[2]);

// Plan set-up shared by the host-built and the device-built plan
// (hnv_host.cpp): option defaults and limits, the plan's shape, and the
// workspace layout (base == nullptr: sizing only; sets p->ws_bytes).
void resolve_options(const hnv_options *in, int d, hnv_dtype dtype, hnv_options *out);
hnv_status check_plan_options(int d, hnv_dtype dtype, const hnv_options &o);
void init_plan_shape(hnv_plan *p, const std::vector<LevelShape> &shape, int d, hnv_dtype dtype,
                     const hnv_options &o);
void carve(hnv_plan *p, const std::vector<LevelShape> &shape, char *base);

// Forward-sweep launch geometry of a level (blocks per panel and finalize blocks).
void forward_geometry(const hnv_plan *p, const LevelPlan &L, int64_t *main_blocks, int64_t *fin_blocks);

// Where a level's arrays lie in the LDS of a launch that runs many of its
// sweeps (bytes past the node rows), and whether the level allows such a launch:
// by its sizes, one column panel of 4 to 16 lanes per row (so that a long
// item's lanes are one wavefront and a row's serial chain is no longer than a
// lane group's), its LDS bytes and its 16-bit offsets; and, once its work lists
// are known, no split rows, a workgroup for every wavefront-tier item (as
// levels of this size have it unless settle_long_items undid it), and residual
// partials that one workgroup adds.
struct ResidentLayout {
    int64_t off_e[2], off_idx[2], off_wn, off_items, off_mix, off_wide, total;
};
ResidentLayout resident_layout(const hnv_plan *p, const LevelPlan &L);
bool resident_sizes(const hnv_plan *p, const LevelPlan &L);
bool resident_fits(const hnv_plan *p, const LevelPlan &L);

// A level's sweep scratch in the static array of hnv_sweep_noalloc: residual
// partials and stages (only with a residual), then the split-row slots.
struct NoallocLayout {
    int64_t stage_len, off_stage, off_slots, total;
};
NoallocLayout noalloc_layout(const hnv_plan *p, const LevelPlan &L, bool resid);
// Called once a level's work lists are known: a level whose scratch passes the
// static array with a workgroup per long item has a wavefront per item, a
// quarter of those residual partials, in every sweep, so that both sweep
// entry points give the same bits.
void settle_long_items(const hnv_plan *p, LevelPlan &L);

// Device arrays of a candidate-scoring plan (carved from the caller's workspace)
struct ScorePlan {
    const int32_t *idx = nullptr;
    const Item *small = nullptr;
    int32_t n_small = 0;
    const Item *chunks = nullptr;
    int32_t n_chunks = 0;
    const Split *splits = nullptr;
    int32_t n_splits = 0;
    float *partials = nullptr;
};

constexpr int kScoreChunk = 512;     // members per wavefront work item of the scoring kernel

// Device-side pieces implemented in hnv_kernels.hip
hnv_status dev_recompute_reciprocals(hnv_plan *p, int level, void *stream);
// Fills both sides' small_ids / small_cids of a level of a host-built plan
// from its work items and neighbour arrays (the device-built plan fills them
// as it writes its work items).
hnv_status dev_fill_inline_ids(hnv_plan *p, int level, hipStream_t s);
hnv_status dev_check(const char *what);
hnv_status dev_score(const ScorePlan &sp, const void *z, hnv_dtype dtype, int d, int op, float *out,
                     hipStream_t s);

}  // namespace hnv

// A candidate-scoring plan: the device arrays above plus the sizes.
struct hnv_score_plan {
    hnv::ScorePlan sp;
    int64_t n_cand = 0, z_rows = 0;
    int d = 0;
    hnv_dtype dtype = HNV_F32;
};
