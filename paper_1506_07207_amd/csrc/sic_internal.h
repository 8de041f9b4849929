// sic_internal.h - device-side layout shared by the kernels and the host
// side of libsic (not part of the public ABI).
//
// Tracer storage.  Tracers live in 64-slot chunks, one wavefront per chunk;
// every sheet starts on a chunk boundary (its last chunk may be partly
// empty), so a wavefront never straddles two sheets.  State is two arrays of
// 8-byte words per tracer slot:
//   word 0: x (float64)                      - SIC_FP64
//           index (low 32 bits) | offset (high) - split forms: U32 the cell
//           and a uint32 fraction of it; F32 an index of 2^-20-cell
//           sub-cells (cell = index >> 20) and a float32 offset in [0, 1)
//           of the sub-cell
//   word 1: v (float64)
// Every chunk also keeps a copy of its first tracer's state in a "halo"
// array.  A step that moves tracers and deposits their new positions in the
// same kernel needs, for the last tracer of each chunk, the new position of
// the first tracer of the next chunk, which another workgroup may already
// have overwritten; it recomputes that move from the halo copy written by the
// previous step.  The halo is double-buffered (read one, write the other).
//
// Charges.  By default every segment of a sheet carries the sheet's charge,
// kept in the chunk descriptor.  Pools created for per-segment charges (and
// refinement, which halves segments) keep a third 8-byte word per tracer
// slot: the charge of the segment that starts at that tracer (float64, or
// int64 fixed point in the split forms), plus per chunk the charge of the
// segment that ends at its first tracer and of the segment that starts at
// its partner tracer ("charge edges").
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sic {

constexpr int kChunk = 64;          // tracer slots per chunk = wavefront width
constexpr int kMaxCells = 4096;     // mirrors SIC_MAX_CELLS
// Copies of a single simulation's charge accumulators (P, D, R): its work
// items merge into copy (item mod copies), so each address takes that
// fraction of the atomics, and the solve sums the copies in order.  Four for
// meshes of up to kSolveThreads cells; two for larger ones, whose every
// solve-first workgroup reads all copies of the whole mesh (the reads then
// cost more than the contention saves).  Batches, with few items per
// simulation, keep one copy.
constexpr int kSmallMeshRep = 4;
constexpr int single_rep(int max_cells) { return max_cells <= 256 ? kSmallMeshRep : 2; }
constexpr int kSolveThreads = 256;  // field-solve workgroup
// The mesh sizes that the solve is built for (1, 4 and 16 cells per thread),
// and the smallest of them that holds a mesh.
constexpr int kSolveCells[3] = {kSolveThreads, 4 * kSolveThreads, 16 * kSolveThreads};
constexpr int solve_class(int n_cells) { return n_cells <= kSolveCells[0] ? 0 : (n_cells <= kSolveCells[1] ? 1 : 2); }
constexpr int kComputeUnits = 256;  // of an MI355X

enum Prec : int { kFP64 = 0, kSplitF32 = 1, kSplitU32 = 2 };

// Tracer-kernel modes (bit set).
enum Mode : int {
  kDeposit = 1,      // deposit the (possibly new) positions into the mesh
  kPush = 2,         // kick with E and drift
  kKickHalf = 4,     // start-up: v <- v - dt/2 E(x), positions unchanged
};

// Solve-kernel flags.
enum SolveFlags : int {
  kHavePush = 1,     // a push ran since the last solve: step += 1, KE/momentum rows
  kHaveDeposit = 2,  // partials hold the max segment of the deposited positions
  kBatchStep = 4,    // count the step against steps_left; finish at zero
};

struct alignas(16) InstDesc {
  double L, half_L, dx, inv_dx;
  double dt, q_unit;      // q_unit: charge of one fixed-point unit (split forms)
  int64_t mesh_off;       // first cell of this slot in the mesh arrays
  int64_t hist_off;       // first row of this slot in the history array
  int64_t hist_cap;       // rows in the ring
  int64_t step;           // positions are x^step
  int64_t steps_left;     // batch: steps still to run (< 0: unlimited)
  int32_t n_cells;
  int32_t active;         // 1: advanced by batch steps
  int32_t flags;          // sticky sic_diag flags
  int32_t live;           // slot holds a simulation
};

struct alignas(16) ChunkDesc {
  double q;               // segment charge
  int64_t q_fix;          // segment charge in fixed-point units
  int32_t partner;        // chunk whose first tracer follows this chunk's last
                          // valid tracer in the sheet; -1: open sheet end
  int32_t n_valid;        // valid tracer slots (1..64)
  int32_t inst;           // slot
  int32_t flags;          // kChunkOpenStart
};

enum ChunkFlags : int {
  kChunkOpenStart = 1,    // lane 0 is the first tracer of an open sheet (no segment before it)
};

struct alignas(16) Item {
  int32_t inst;
  int32_t chunk_begin;
  int32_t chunk_end;
  int32_t pad;
};

struct alignas(32) Partial {
  double ke, mom, maxseg, pad;
};

// Row layout of the history ring (matches sic_diag).
struct alignas(64) DiagRow {
  int64_t step;
  double t, W_E, KE, momentum, total_charge, max_segment;
  int64_t flags;
};

// Links from a chunk to single tracers of other chunks (piecewise-linear
// segments need two tracers past a chunk's end and one before its start):
// (chunk << 2) | which, which = 0 first, 1 second, 2 last tracer of that
// chunk; -1 when there is no such tracer (ends of an open sheet, or a closed
// sheet too short to have a gradient).
enum HaloWhich : int { kHaloFirst = 0, kHaloSecond = 1, kHaloLast = 2 };

struct SolveArgs {
  InstDesc *inst;
  const int2 *slot_items;    // per slot: (first item, item count) in the item list
  const int32_t *slot_list;  // NULL: slot = blockIdx.x
  const Partial *partials;
  void *meshP;
  void *meshD;
  void *meshR;               // order 1 only
  double *meshE;
  double *meshRho;           // n_j - nbar of the newest solve
  DiagRow *hist;
  int32_t *done;             // per slot: set to 1 when a batch run finishes
  int32_t flags;
  int32_t respect_active;
  int32_t order;             // deposit order of the pool (0, 1 or 2); R exists only for 1
  const int32_t *gate = nullptr;  // non-NULL: the launch does nothing unless *gate > 0
  // P, D and R are held in rep copies rep_stride words apart; the solve
  // sums them in copy order and clears each
  int32_t rep = 1;
  int64_t rep_stride = 0;
  // further accumulators to clear (those that the last of a run of
  // solve-first steps read)
  void *zero = nullptr;
  int64_t zero_words = 0;
  // the end of a run of refining solve-first steps: the partials' count (>= 0)
  // and, where the last step refined, the partials of the refined deposit
  int32_t n_partials = -1;
  int32_t n_refined = 0;
  const Partial *refined = nullptr;
};

// Refinement done entirely on the device (one simulation, steps in a row):
// int32 words of its state.
//   kRefChunks      chunks of the slot now
//   kRefInserted    whether the last pass inserted tracers (> 0) or re-laid out
//                   nothing (0)
//   kRefHalt        set when a pass would exceed the capacity (sticky; the
//                   following steps do nothing)
//   kRefMarks       set when a segment was marked since the last plan
//   kRefCur         which of the two sets of state arrays holds the state
//   kRefSteps       steps taken
//   kRefStepChunks  chunks at the newest step, before its refinement
enum RefineState : int {
  kRefChunks = 0,
  kRefInserted = 1,
  kRefHalt = 2,
  kRefMarks = 3,
  kRefCur = 4,
  kRefSteps = 5,
  kRefStepChunks = 6,
  kRefWords = 8
};

// The second set of a refining simulation's state arrays and its state
// words; state NULL: the launch does not refine.
struct RefineSel {
  const int32_t *state = nullptr;
  uint64_t *xs = nullptr;
  double *vs = nullptr;
  uint64_t *segq = nullptr;
  ChunkDesc *chunks = nullptr;
};

// Where a step marks the segments longer than l_max: per chunk from
// chunk_begin on their count and lane mask, and whether there are any; cnt
// NULL: none.
struct MarkArgs {
  int32_t *cnt = nullptr;
  uint64_t *mask = nullptr;
  int32_t *any = nullptr;
  double l_max = 0.0;
  int32_t chunk_begin = 0;
};

// Work items of a simulation that refines on the device: enough for one per
// compute unit but one (which writes the rows), of 8 to kRefineMaxTile chunks.
constexpr int kRefineGroups = kComputeUnits - 1;
constexpr int kRefineMaxTile = 256;
__host__ __device__ inline int refine_tile(int n_chunks, int fixed) {
  if (fixed > 0) return fixed;
  const int t = ((n_chunks + kRefineGroups - 1) / kRefineGroups + 7) / 8 * 8;
  return t < 8 ? 8 : (t > kRefineMaxTile ? kRefineMaxTile : t);
}
__host__ __device__ inline int refine_items(int n_chunks, int fixed) {
  const int t = refine_tile(n_chunks, fixed);
  return (n_chunks + t - 1) / t;
}

struct TracerArgs {
  const Item *items;
  const int32_t *n_items;  // device-side item count
  const InstDesc *inst;
  const ChunkDesc *chunks;
  const int2 *links;       // per chunk (prev link, next-but-one link); order 1
  const double2 *halo3_in; // per chunk: first, second, last tracer; order 1
  double2 *halo3_out;
  void *meshR;             // second-difference array for linear ramps; order 1
  uint64_t *xs;            // word 0 per slot
  double *vs;              // word 1 per slot
  const double2 *halo_in;  // (x word as bits, v) per chunk
  double2 *halo_out;
  void *meshP;             // direct cell charge (double or int64)
  void *meshD;             // difference array for covered cell runs
  const double *meshE;
  Partial *partials;       // per item
  const uint64_t *segq;    // per slot: charge of the segment starting there (per-segment pools)
  const uint64_t *cedge;   // per chunk: charge ending at lane 0, charge starting at the partner
  int32_t mesh_cells;      // LDS capacity in cells (max n_cells of the pool)
  int32_t tile_cap;        // LDS capacity in chunks per work item
  int32_t respect_active;  // skip slots with active == 0
  const int32_t *gate = nullptr;  // non-NULL: the launch does nothing unless *gate > 0
  // copies of P, D and R, rep_stride words apart: work item i merges into
  // copy i mod rep (fewer atomics on one address when many items share a
  // mesh)
  int32_t rep = 1;
  int64_t rep_stride = 0;
  // deposit alone, one simulation: consecutive items that a workgroup may take
  // with one clearing and one merge of its mesh (the grid covers the items)
  int32_t run = 1;
  RefineSel sel;           // per-segment pools
  MarkArgs mark;
};

// A solve-first step of a single simulation (slot 0).  The accumulators of a
// step are one block of (P, D and for linear segments R) x single_rep copies
// x nc words.
struct StepArgs {
  double L, half_L, dx, inv_dx, dt, q_unit;
  int32_t nc;
  int32_t n_items, tile;          // item i: chunks [chunk_begin + i tile, + tile), n_chunks in all
  int32_t chunk_begin, n_chunks;
  int64_t hist_cap;
  const ChunkDesc *chunks;
  const int2 *links;              // order 1
  const uint64_t *segq, *cedge;   // per-segment charges
  uint64_t *xs;
  double *vs;
  const double2 *halo_in;         // orders 0, 2: one copy per chunk; order 1: three
  double2 *halo_out;
  const double *meshE;            // the field of a run's first step
  const void *acc_in;             // the previous step's charge; NULL: a run's first step
  void *acc_out;                  // this step's charge
  void *acc_zero;                 // accumulators to clear, or NULL
  const Partial *part_in;         // the previous step's work-item partials
  Partial *part_out;
  SolveArgs sf;                   // what the diagnostics go to
  // refining on the device (per-segment pools; sel.state set): the chunk count
  // is the device's, the items are those of refine_tile(count, tile_fixed)
  RefineSel sel;
  MarkArgs mark;
  int32_t tile_fixed = 0;
  const Partial *part_ref = nullptr;  // partials of the refined state's deposit
  int32_t row_group = 0;          // set by launch_step: workgroup 0 has no item
  int32_t zero_slice = 0;         // words of acc_zero per workgroup
};

struct IngestArgs {
  const double *x_in;
  const uint64_t *w_in;       // raw state words instead of x_in (re-layout), or NULL
  const double *v_in;
  const double *c_in;         // per-segment charges (float64), or NULL
  const uint64_t *cw_in;      // raw per-segment charge words (re-layout), or NULL
  uint64_t *segq;             // NULL: the pool keeps no per-segment charges
  double q_scale;             // fixed-point units per unit charge (split forms)
  const int64_t *chunk_in_off;  // per chunk of the range: first input index
  int32_t chunk_begin;
  int32_t n_chunks;
  const ChunkDesc *chunks;
  const InstDesc *inst;
  uint64_t *xs;
  double *vs;
  double2 *halo;
  double2 *halo3;  // order 1 (NULL otherwise)
};

struct ExtractArgs {
  const int64_t *chunk_in_off;
  int32_t chunk_begin;
  int32_t n_chunks;
  const ChunkDesc *chunks;
  const InstDesc *inst;
  const uint64_t *xs;
  const double *vs;
  const uint64_t *segq;  // with c_out: per-segment charges
  double *x_out;
  double *v_out;
  double *c_out;         // NULL: positions and velocities only
  int64_t *step_out = nullptr;  // host memory that takes the slot's step, or NULL
};

// What a diagnostics call reads of a slot, written in one launch to a block
// of host memory: its descriptor (at 0), the newest row (kExportRow), the
// density and the field (kExportMesh, nc words each; where wanted) and the
// newest rows of the history that the call takes, oldest first, unless they
// are more than max_rows.
constexpr size_t kExportRow = 128, kExportMesh = 192;
struct ExportArgs {
  const InstDesc *inst;    // the slot's
  const DiagRow *hist;     // the slot's ring
  const double *rho, *E;   // both or neither
  int32_t nc;
  int64_t hist_from;       // the step the history starts at
  int64_t rows;            // that the call takes at most
  int64_t max_rows;        // that the block has room for
  unsigned char *out;
};

// Refinement (section 2.6) of one slot's chunk range: a marking pass counts
// per chunk the segments longer than l_max (and keeps their lane mask); the
// scatter pass writes every tracer, plus a centre tracer after each marked
// one, to flat sheet-major output arrays (chunk cl starts at out_off[cl]).
struct RefineArgs {
  const ChunkDesc *chunks;
  const InstDesc *inst;
  const uint64_t *xs;
  const double *vs;
  const uint64_t *segq;
  int32_t chunk_begin;
  int32_t n_chunks;
  double l_max;
  int32_t *cnt;            // per chunk of the range
  uint64_t *mask;          // per chunk of the range
  const int64_t *out_off;  // per chunk of the range (scatter)
  uint64_t *w_out;
  double *v_out;
  uint64_t *c_out;
};

// A refinement pass of one simulation on the device, after a step that
// marked its segments: the plan and the rebuild.  State arrays come in two
// sets; the rebuild reads one and writes the other.
struct RefinePassArgs {
  ChunkDesc *chunks[2];
  uint64_t *xs[2];
  double *vs[2];
  uint64_t *segq[2];
  double2 *halo;           // the halo copies the next step reads (orders 0, 2: one per chunk, 1: three)
  uint64_t *cedge;
  int2 *links;             // order 1 (NULL otherwise)
  Item *items;             // the slot's item range (room for the capacity)
  int2 *slot_items;        // per slot: (first item, item count)
  int32_t *n_items;        // item count the tracer kernel walks
  InstDesc *inst;
  const int32_t *cnt;      // per chunk of the range: segments to split
  const uint64_t *mask;    // per chunk of the range: their lanes
  int64_t *out_off;        // per chunk of the range: its first tracer's index in the new order
  int32_t *nt;             // per sheet: tracers now
  const int32_t *closed;   // per sheet
  const double *q;         // per sheet: charge kept in the descriptors
  int64_t *work;           // 4 n_sheets + 2 entries (per sheet: new count, new first chunk, index of its
                           // first tracer, old first chunk)
  int32_t *state;          // RefineState words
  void *acc_zero;          // accumulators to clear when the pass inserts, or NULL
  int64_t acc_words;
  int64_t max_tracers;
  double q_scale;
  int32_t n_sheets;
  int32_t chunk_begin;
  int32_t chunk_cap;       // chunks reserved for the slot
  int32_t tile_fixed;      // refine_tile
  int32_t slot;
  int32_t item_begin;
  int32_t order;
  int32_t fixed;           // split forms: descriptors carry fixed-point charges
};

// Launchers (sic_kernels.hip).  All return hipError_t as int.
int launch_tracers(int prec, int mode, int order, bool seg, const TracerArgs &a, int grid, int block,
                   size_t lds_bytes, void *stream);
// A solve-first step of a single simulation: grid workgroups over the items,
// of block threads, at least kSolveThreads and at least a.tile.
int launch_step(int prec, int order, bool seg, const StepArgs &a, int grid, int block, void *stream);
bool step_supported(int order, int max_cells);
// The tracer launch of a step whose charge a solve launch solves (a.acc_in,
// acc_zero NULL), in at most *grid workgroups and at most as many as run at a
// time; *grid: the workgroups launched, each of which writes one partial.
int launch_run(int prec, int order, bool seg, const StepArgs &a, int block, void *stream, int *grid);
// The tracer kernels' dynamic LDS limit, for every mesh and item size.
int set_tracer_lds_limit(int prec, int order, bool seg);
size_t tracer_lds_size(int prec, int order, bool seg, int mesh_cells, int tile_cap);
// max_cells: the largest mesh of the slots the launch may solve.
int launch_solve(int prec, const SolveArgs &a, int n_blocks, int max_cells, void *stream);
int launch_ingest(int prec, const IngestArgs &a, void *stream);
int launch_extract(int prec, const ExtractArgs &a, void *stream);
// Clears the meshes of the listed slots in all rep copies (rep_stride words
// apart); step >= 0 sets their step.
int launch_zero_mesh(int prec, void *meshP, void *meshD, void *meshR, InstDesc *inst,
                     const int32_t *slot_list, int n_blocks, int rep, int64_t rep_stride, void *stream,
                     int64_t step = -1);
int launch_export(const ExportArgs &a, void *stream);
// grid: workgroups of 256 threads
int launch_copy_bench(const double *src, double *dst, int64_t n, int grid, void *stream);
// Charge edges of chunks [chunk_begin, chunk_begin + n_chunks): prev_slot[c]
// is the slot of the tracer before chunk c's first one (-1: none).
int launch_charge_edges(const ChunkDesc *chunks, const int64_t *prev_slot, const uint64_t *segq, uint64_t *cedge,
                        int32_t chunk_begin, int32_t n_chunks, void *stream);
// A small simulation's n_steps fused steps (push, deposit, solve) in one
// launch of one workgroup; chunks [chunk_begin, chunk_begin + n_chunks) of
// slot 0.  a.halo_out (order 1: a.halo3_out) receives the halos of the final
// state.
bool resident_supported(int order, int n_chunks, int n_cells);
int launch_resident(int prec, int order, bool seg, const TracerArgs &a, const SolveArgs &sa, int chunk_begin,
                    int n_chunks, int n_cells, int64_t n_steps, void *stream);
int launch_refine_mark(int prec, const RefineArgs &a, void *stream);
int launch_refine_scatter(int prec, const RefineArgs &a, void *stream);
// A pass on the device: the plan (one workgroup) and the rebuild.
int launch_refine_plan(const RefinePassArgs &a, void *stream);
int launch_refine_rebuild(int prec, const RefinePassArgs &a, void *stream);

}  // namespace sic
