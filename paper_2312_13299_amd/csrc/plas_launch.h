// plas_launch.h -- host-side launchers of the PLAS kernels (plas_kernels.hip).
// Each enqueues work on `stream` and returns the launch status; none
// synchronises. `dp` is the padded channel stride of the working layout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plas_device.h"

namespace plas {

struct plas_level_out {  // same layout as plas_level_stat in plas.h
  double phi;
  int32_t r;
  int32_t beta;
  int64_t reorders;
  uint64_t energy_fixed;
  uint64_t moved;
};

// Storage of the working grids.
constexpr int kStorageF32 = 0;
constexpr int kStorageBF16 = 1;

// What an ingest and an energy query leave on the device.
struct QueryOut {
  float lo[64], hi[64];       // range of the stored values per channel, d of them
  int32_t bad_value;          // nonzero: some value is NaN or infinite
  int32_t bad_perm;           // nonzero: the permutation is not a bijection
  int32_t s;                  // energy scale (scale_shift of the ranges)
  int32_t pad;
  unsigned long long energy;  // fixed-point energy
  double vad[2];              // of a VAD: the mean (in place only) and the variance
};

// Clears out's flags and energy; writes float32 1/c (correctly rounded) for c
// = 1..w and 0 for c = 0 to counts (NULL: not); writes the inverse of perm
// (device int32[n], NULL: none) to inv, for launch_ingest to check and follow.
hipError_t launch_begin(QueryOut* out, const int32_t* perm, int64_t n, int32_t* inv, float* counts, int w,
                        hipStream_t stream);
// P[p] = bijection(n, keys)(p), inv its inverse (NULL: not written).
hipError_t launch_start_perm(int32_t* P, int32_t* inv, int64_t n, const uint64_t keys[4], hipStream_t stream);
// Sets out->bad_perm if perm (int32[n]) is not a bijection of [0, n), and
// clears the rest as launch_begin does. inv: scratch int32[n].
hipError_t launch_check_perm(const int32_t* perm, int64_t n, int32_t* inv, QueryOut* out, hipStream_t stream);
// features (layout CN [d][n] or NC [n][d]; float32, or bfloat16 bits if
// input_bf16) -> G [n][dp] in `storage`, feature i at G[inv[i]] (inv NULL:
// G[i]), channels >= d zero; out's ranges, bad_value and s. With perm (the
// permutation launch_begin inverted; NULL: inv is known good) sets
// out->bad_perm if it is no bijection; places it does not name are then left
// unwritten. part: scratch of ingest_partial_floats(dp) floats. Few blocks
// keep the fold of their ranges short (1024^2 x 59, ingest and fold: 512
// blocks 112 + 6 us, 1024 blocks 105 + 9).
constexpr int kIngestBlocks = 512;
constexpr size_t ingest_partial_floats(int dp) { return static_cast<size_t>(kIngestBlocks) * 2 * dp; }
hipError_t launch_ingest(const void* features, int input_bf16, int64_t n, int d, int layout, int dp, int storage,
                         const int32_t* inv, const int32_t* perm, void* G, float* part, QueryOut* out,
                         hipStream_t stream);
// The grouping table a reorder's first row pass fills after its lines, from
// the state's beta and keys.
struct TableArgs {
  int32_t* table;
  int64_t max_cells;  // largest beta^2 of the sort: the pass launches enough blocks to fill it quickly
};

// One blur pass (vertical = 0: rows, 1: columns) with radius st->r, or
// `radius` if st is NULL (a pass queued after the end of the sort returns at
// once). With st, `radius` is the one the caller last saw there: it helps to
// choose the kernel, and every kernel is right at every radius. inv: float32 1/c for c = 0..w (the register kernel's multipliers).
hipError_t launch_blur_pass(const void* in, void* out, int w, int dp, int storage, const DevState* st,
                            int radius, int vertical, const float* inv, hipStream_t stream,
                            const TableArgs* table = nullptr);
// Grouping table of the current reorder: table[t] = packed pi(t), t < beta^2.
hipError_t launch_group_table(int32_t* table, const DevState* st, int64_t max_cells,
                              hipStream_t stream);
// What the control step at the end of a sort's assignment needs: the level
// table and the per-level trace (may be NULL).
struct ControlArgs {
  const LevelInfo* levels;
  plas_level_out* trace;
};

// One blockwise assignment with the parameters in st. max_items bounds the
// items (groups, and packs of four singles) of every level this launch may
// see. With `control`,
// the last block to finish runs the control step of the reorder on st in
// place (the energy and moved sums, the stall test, the schedule, the next
// shift and grouping keys); without it, st keeps the sums for the caller.
hipError_t launch_assign(void* G, const void* T, int32_t* P, const int32_t* table, DevState* st, int dp,
                         int storage, int64_t max_items, hipStream_t stream, const ControlArgs* control = nullptr);
// VAD (App. C) of a grid [w * w][dp] of d channels, the rest zero: the variance
// of |a - b| over neighbour pairs and channels, to *out (device). part: device
// scratch of vad_partial_doubles() doubles.
size_t vad_partial_doubles();
hipError_t launch_vad_grid(const void* G, int d, int w, int dp, int storage, double* part, double* out,
                           hipStream_t stream);
// The same of features[perm] without a grid: out[0] the mean, out[1] the
// variance.
hipError_t launch_vad_in_place(const void* features, int input_bf16, const int32_t* perm, int64_t n, int d, int w,
                               int layout, double* part, double* out, hipStream_t stream);

// ---- batches of sorts (BatchGrid in plas_device.h). A launch's block map
// (device uint32[blocks]) holds (grid index << 16) | block index within the
// grid's blocks; a grid's entries run from 0 to its block count - 1.
// Blocks each grid takes per launch kind.
// Whether blur passes of this shape go through LDS (cells of at least 16
// bytes): the relay or the ring kernel; groups_per_block applies to those only.
bool staged_blur(int dp, int storage);
// Whether the grids in flight (the one grid of a sort, every running grid
// of a batch) are a large working set, more than 128 MiB: then column passes
// stream their loads, and float32 passes may take the ring kernel (ring_rows,
// batch_ring).
bool blur_large_working_set(int64_t working_bytes);
// Groups of 64 / dp lines of a pass.
int64_t blur_groups(int w, int dp);
// What the ring kernel gains (or, negative, costs) a float32 grid of a batch at
// radius r, in percent of a reorder times cells; and whether the grids of one
// width (16 channels or more) of a large working set take it, from the sums of
// their groups, cells, bytes and gains.
int64_t batch_ring_gain(int w, int dp, int r);
bool batch_ring(int64_t groups, int64_t cells, int64_t bytes, int64_t gain);
// groups_per_block of blur launches: 1, 2 or 4 line groups per block of the
// relay kernel, or kBatchRing for the ring kernel.
constexpr int kBatchRing = -1;
// Blur blocks: enough for every line, and for filling a grouping table of
// max_cells entries at about one entry per thread.
int batch_blur_blocks(int w, int dp, int storage, int groups_per_block, int64_t max_cells);
int batch_assign_blocks(int64_t max_items, int dp, int storage, int cap);  // cap <= 0: the single-sort default
int assign_blocks_cap(int storage);  // blocks of an assignment launch without a tuned value
// A batch blur pass's route: its axis (vertical 0: rows, 1: columns), its
// source and destination grids (0 G, 1 H, 2 T; the destination H or T, not
// the source) and whether it fills each grid's grouping table after its
// lines (the first row pass of a reorder).
int blur_route(int vertical, int src, int dst, int with_table);
// One blur pass along `route` of every mapped grid, all of dp channels and
// `storage`; large: blur_large_working_set holds for the running grids.
hipError_t launch_blur_batch(const BatchGrid* grids, const uint32_t* map, int blocks, int dp, int storage,
                             int groups_per_block, int route, int large, hipStream_t stream);
// One assignment of every mapped grid; each grid's last block runs its
// control step.
hipError_t launch_assign_batch(const BatchGrid* grids, const uint32_t* map, int blocks, int dp, int storage,
                               hipStream_t stream);
// out[i] = (done, k) of grids[list[i]]'s state, i < count.
hipError_t launch_batch_status(const BatchGrid* grids, const int32_t* list, int count, HostStatus* out,
                               hipStream_t stream);

// energy_out (device u64) += sum over cells of floor(d(G[p], T[p]) * 2^s);
// s is *s_device if that is not NULL.
hipError_t launch_energy(const void* G, const void* T, int64_t n, int dp, int storage, int s,
                         const int32_t* s_device, unsigned long long* energy_out, hipStream_t stream);

// ---- the device scratch of the no-allocation energy query. One array per
// GPU, allocated with the code object and held until the process ends;
// every call on a GPU shares it.
constexpr int64_t kNoAllocMaxCells = 65536;  // side <= 256
constexpr int kNoAllocMaxSide = 256;
struct NoAllocLayout {
  static constexpr size_t kGrid = static_cast<size_t>(kNoAllocMaxCells) * 64 * 4;  // widest cell, float32
  static constexpr size_t kG = 0, kH = kGrid, kT = 2 * kGrid;
  static constexpr size_t kRangePart = 3 * kGrid;
  static constexpr size_t kOut = kRangePart + ingest_partial_floats(64) * 4;  // QueryOut
  static constexpr size_t kInv = kOut + 1024;
  static constexpr size_t kBytes = kInv + 4096;  // (kNoAllocMaxSide + 1) floats, rounded up
};
// The array's device address on `device`, which must be current (looked up
// once per device, then remembered).
hipError_t noalloc_scratch(int device, void** out);

}  // namespace plas
