// psl_launch.h -- host-side launchers of the libpsl kernels (internal).
#pragma once

#include "psl_device.h"

namespace psl {

hipError_t launch_power_table(double *T, uint32_t n, uint32_t alpha, hipStream_t s);
// Slabs zeroed, records written and pivots set (bits: the staged words of given
// pivots) of nb walks of at most max_bytes of slab and max_nw words.
hipError_t launch_init(WalkDev *walks, const InitRec *recs, const uint64_t *bits, uint32_t nb, uint64_t max_bytes,
                       uint32_t max_nw, hipStream_t s);
// Lengths of the walks a correlation covers: the shortest, the longest, and the
// work, in 32-position chunks per 4096 shifts (add each walk once).
struct CorrDims {
    uint32_t min_L = UINT32_MAX, max_L = 0;
    uint64_t chunks = 0;
    void add(uint32_t L, uint64_t count = 1)
    {
        if (L < min_L) min_L = L;
        if (L > max_L) max_L = L;
        chunks += count * ((uint64_t)L * L / (2ull * 4096 * 32) + 1);
    }
};
// C (Eq. (2)) from the pivot's bits (psl_corr.hip). mode 0: every walk (init; C
// of local_best = C as well); 1: walks left pending by a switch whose Rand_flip
// is too large for the one-flip rebuild; 2: every walk, C only (restore).
hipError_t launch_corr(WalkDev *walks, const BatchEntry *batch, uint32_t nb, const CorrDims &dims, int mode,
                       hipStream_t s);
constexpr uint32_t kPendUnit = 1024;   // shifts per work unit of the pending-walk rebuild

// F and PSL of the walks on the pending list (pend: count, then batch positions)
// whose switch flipped more than kFlipIncremental elements, after launch_corr
// rebuilt C (units: work units of kPendUnit shifts the batch's nb walks hold in
// all).
hipError_t launch_pending(WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint64_t units,
                          const Tables &tabs, const uint32_t *pend, hipStream_t s);
// F and PSL of the pivots from C. The segments' sums go through the entries'
// chunk arrays (2 and 1 entries per segment).
hipError_t launch_fit(WalkDev *walks, const BatchEntry *batch, uint32_t nb, const Tables &tabs, const SegMap &map,
                      int mode, hipStream_t s);
// tab (batches with a matrix path): the number of the batch's walks left to
// this evaluation in this step; with none, its blocks return at once.
hipError_t launch_eval(const WalkDev *walks, const BatchEntry *batch, const EvalItem *items,
                       uint32_t n_items, const Tables &tabs, const EvalShape &shape,
                       EvalQueues *queues, const uint32_t *tab, uint32_t n_cu, hipStream_t s);
// The step's chunk arrays and near-peak list (and, with pend, the step's pending
// list emptied), turned into suffix values when scan != 0 (the evaluation in
// 16-wavefront blocks reads those; smaller blocks add the chunk values
// themselves).
hipError_t launch_suffix(const WalkDev *walks, BatchEntry *batch, uint32_t nb, const Tables &tabs, const SegMap *map,
                         uint32_t *pend, int scan, const EvalCall &call, hipStream_t s);
hipError_t launch_seg_scan(const WalkDev *walks, const BatchEntry *batch, const SegMap &map, hipStream_t s);
// Zero the near-peak counts of a batch, its pending count, its counters (done: nb;
// with left, kCombMaxBlocks more for each walk) and its matrix walks' zero
// records after its scratch is allocated.
hipError_t launch_batch_reset(const WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint32_t *pend, uint32_t *done,
                              bool left, hipStream_t s);
// F and PSL per candidate from the partials, then the selection, its
// ambiguity flags (margin: their relative margin) and, pure == 0, the step's
// bookkeeping (pend: the pending list the walks that switch phase join), by
// each walk's last combine block in launches of at most 256 combine blocks
// (done: one zeroed counter per batch position, left zero; without it the
// selection takes a launch of its own): pure != 0 writes the choice record
// `out` (one walk), else the walks' step records. pure == 1: the table
// evaluation has not run, and the record of a walk it is left to says so
// (choice_dev_table) instead.
hipError_t launch_select(WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint32_t comb_blocks,
                         uint32_t comb_group, const Tables &tabs, int pure, void *out, uint32_t *pend,
                         uint32_t *done, double margin, hipStream_t s);
// launch_select of a step whose walks are all matrix walks, where
// select_left_blocks (updates: N_lmt x (L-1) of the walk with the most) gives the
// blocks per walk (grid) and not 0: a walk left to the table evaluation is
// evaluated here, so that no launch_eval comes before. done: nb counters, then
// kCombMaxBlocks for each walk; entries' red: kCombMaxBlocks.
uint32_t select_left_blocks(uint32_t nb, uint32_t comb_blocks, uint64_t updates);
hipError_t launch_select_left(WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint32_t comb_blocks,
                              uint32_t comb_group, uint32_t grid, const Tables &tabs, uint32_t *pend, uint32_t *done,
                              double margin, hipStream_t s);
size_t choice_dev_size();
bool choice_dev_table(const void *p);
void choice_dev_unpack(const void *p, uint32_t *i_best, uint32_t *j_best, double *F_best,
                       double *F_min, uint32_t *j_psl, int32_t *psl_min, int32_t *psl_k, uint32_t *flags);
// The C update of each walk's recorded move (j_fixed < 0, after the
// bookkeeping; for a walk that switched phase, C, F and PSL of its new pivot) or
// of a forced flip of element j_fixed, with F, PSL and the element's bit. done:
// one zeroed counter per batch position, left zero.
hipError_t launch_apply(WalkDev *walks, const BatchEntry *batch, const SegMap &map, const Tables &tabs,
                        int64_t j_fixed, uint32_t *done, hipStream_t s);
// Units of launch_pending for walks of length L.
inline uint64_t pending_units(uint32_t L) { return (L - 1 + kPendUnit - 1) / kPendUnit; }

// Matrix path (psl_split.hip), in a step of a batch with matrix walks: the
// first pass over C in place of launch_suffix (the matrix walks' near-peak
// lists, digits and prefix sums, the other walks' chunk arrays, with scan
// their suffix values; *pend and *tab zeroed), then the matrix products
// (items: walk, kMxTile-element tile, k-split), whose first items choose each
// walk's path; *tab counts the walks left to the table evaluation, launched
// after them.
hipError_t launch_prep(const WalkDev *walks, BatchEntry *batch, uint32_t nb, const Tables &tabs,
                       const SegMap &map, int scan, uint32_t *pend, uint32_t *tab, const EvalCall &call,
                       hipStream_t s);
hipError_t launch_mx(const WalkDev *walks, const BatchEntry *batch, const EvalItem *items, uint32_t n_items,
                     const Tables &tabs, uint32_t *tab, hipStream_t s);

}  // namespace psl
