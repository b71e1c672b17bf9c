// Internal declarations shared by the host planner and the HIP launch code.
// Not part of the public ABI (include/superkernel.h is).
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "superkernel.h"

namespace sk {

enum : int32_t {
  FLAG_VEC_A = 1,  // activation rows can be read in aligned 16-byte pieces
  FLAG_VEC_B = 2,  // weight rows can be read in aligned 16-byte pieces
  FLAG_VEC_C = 4,  // four consecutive outputs of a row can be stored as one vector
  FLAG_ROWS = 16,         // the host plans the operator as one of run_tile_rows (mark_rows)
  FLAG_ROWS_FORM = 32,    // run_tile_rows serves the operator's form (rows_form)
  FLAG_PLANES_FORM = 64,  // run_tile_planes does (planes_form)
  FLAG_PAST_CACHES = 8,  // outputs of whole tiles go past the caches (of every operator of the plan, or of none)
};

enum : uint16_t {
  CLS_SKINNY_FIRST = 0,  // 0..8: 3*log2(rm) + log2(wk), rm = 1, 2, 4 blocks of 16 activation rows
  CLS_TILE_128x128 = 9,
  CLS_TILE_128x64 = 10,  // operators with at most 64 output columns
  CLS_WINDOW = 11,       // device's list only: a run of output pixels of a 3x3 convolution of 64 channels (run_window)
};

// Device-side description of one operator in its canonical GEMM view
//   C[Mg,Ng] = A'[Mg,Kg] . Bs[Ng,Kg]^T
// where A' is either a plain row-major matrix (gather == 0) or the implicit
// patch matrix of an image (gather == 1; Section 5.3: a convolution is
// executed through the GEMM that backs it), NHWC or, with nchw set, NCHW.
struct DevProblem {
  const void *A;
  const void *B;
  void *C;
  int64_t lda, ldb, ldc;  // row strides in elements (lda unused when gather)
  int32_t Mg, Ng, Kg;
  int32_t dtype;
  int32_t gather;
  int32_t H, W, Cin, Ho, Wo, R, S, pad_h, pad_w;
  int32_t flags;
  int32_t tile_first, tile_count;
  int32_t stride;  // of a convolution, both directions (>= 1)
  int32_t nchw;    // convolution on channel-major arrays: X[Nb,Cin,H,W], W[Cout,Cin,R,S], Y[Nb,Cout,Ho,Wo]
  // convolution: bytes from the corner of the padded image (row -pad_h, column -pad_w; channel-major: of channel 0) to the end of the
  // last element that any output pixel meets under any tap, in the image or not; 2^31 stands for more
  uint32_t reach;
  // Division by a convolution's Ho*Wo, Wo, Cin and S as multiply and shift (see FastDiv): the tile set-up
  // divides row and reduction indices by them for every row a thread stages.
  uint32_t div_hw[2], div_wo[2], div_cin[2], div_s[2];
};
static_assert(sizeof(DevProblem) % 8 == 0, "DevProblem must stay 8-byte sized");

#ifdef __HIPCC__
#define SK_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SK_HOST_DEVICE inline
#endif
// Whether every offset that an element of a convolution's images b .. b + later can get, counted from the corner of image b's
// padding (a pixel's offset plus its tap's, and the element itself), lies below `limit` bytes, 2^31 at most.
SK_HOST_DEVICE bool offsets_below(const DevProblem &d, int64_t later, int64_t es, int64_t limit) {
  // (limit <= 2^31; a shift, not a 64-bit comparison: see lean_operands)
  return (uint64_t)(later * ((int64_t)d.H * d.W * d.Cin * es) + (int64_t)d.reach + (((int64_t)1 << 31) - limit)) >> 31 == 0;
}

// Whether a channel-major convolution's outputs lie in the order of the pixels under each of its taps (run_tile_planes): stride 1, one or
// three filter columns that keep the images' width, at most four filter rows, images and weight rows of at least a piece.
SK_HOST_DEVICE bool planes_form(const DevProblem &d, int64_t es) {
  const int64_t piece = 16 / es;
  return d.nchw && d.stride == 1 && (d.S == 1 || d.S == 3) && 2 * d.pad_w == d.S - 1 && d.R <= 4 && d.Kg >= piece &&
         (int64_t)d.H * d.W * d.Cin >= piece && (uint64_t)(128 * d.ldb * es) >> 31 == 0;
}

// How run_tile_rows holds an NHWC convolution of few channels in LDS: `pieces` of 16 bytes per filter row's run of S * Cin elements, a weight row of
// `weight_row` bytes, a row of the image (its padding included) of `image_row`, of which a tile needs `rows` at most.  ok: it serves the
// operator (filters and images small enough, at most 64 output channels, runs of one to four or six pieces, image rows of at least one).
// What it leaves out, which runs as patches: windows of more than ROWS_LOADS pieces a thread, which wait in registers for a block (7x7 on 224x224 RGB in fp32,
// 30.6 KB against 24, and on 448 columns in 16 bits); more channels than the two fragments a wave multiplies a pixel by; runs of five pieces (11x11 on
// RGB in 16 bits), an instantiation of the products more per type.
struct RowsForm {
  bool ok;
  int32_t pieces, weight_row, image_row, rows;
};
constexpr int32_t ROWS_LOADS = 6;               // pieces of an image window per thread, at most
constexpr int32_t ROWS_LDS = 512 * 144;         // LDS_TILE_BYTES of the kernels
SK_HOST_DEVICE RowsForm rows_form(const DevProblem &d, int32_t es) {
  const int32_t ce = 16 / es;
  RowsForm f{false, 0, 0, 0, 0};
  if (!d.gather || d.nchw || d.Ng > 64 || d.R > 16 || d.S > 16 || d.Cin > 16 || d.Wo > 4096 || d.stride > 16) return f;
  const int32_t run = d.S * d.Cin;
  if (run < ce || (int64_t)d.W * d.Cin < ce || ((uint64_t)d.H * (uint64_t)d.W * (uint64_t)(d.Cin * es)) >> 31 != 0 || ((uint64_t)64 * (uint64_t)d.ldb * (uint64_t)es) >> 31 != 0) return f;
  f.pieces = (run + ce - 1) / ce;
  if (f.pieces == 5 || f.pieces > 6) return f;
  f.weight_row = ((d.R * f.pieces + 1) / 2 * 2 + 1) * 16;  // (an odd number of pieces: the rows' banks)
  f.image_row = (((d.Wo - 1) * d.stride * d.Cin + f.pieces * ce) * es + 31) / 16 * 16;
  f.rows = (126 + d.Wo) / d.Wo * d.stride + d.R;
  const int32_t window = f.rows * f.image_row, outputs = 128 * (64 * es + 16);
  f.ok = window <= ROWS_LOADS * 256 * 16 && 64 * f.weight_row + (window > outputs ? window : outputs) <= ROWS_LDS;
  return f;
}

// n / d for 0 <= n < 2^31 as (n * mul) >> shift with mul = floor(2^(31+l) / d) + 1, l = ceil(log2 d), shift = 31 + l:
// mul * d = 2^(31+l) + e with 0 < e <= d <= 2^l, so the quotient is off by less than n / (d * 2^31) < 1 / d.
struct FastDiv {
  uint32_t mul, shift;
};
inline FastDiv fast_div_of(uint32_t d) {
  if (d == 0) return FastDiv{0u, 0u};
  uint32_t l = 0;
  while (((uint64_t)1 << l) < d) ++l;
  const uint64_t mul = (((uint64_t)1 << (31 + l)) / d) + 1;  // < 2^32 + 1; equals 2^32 only for d = 1 ... see below
  // d = 1: l = 0, mul = 2^31 + 1, shift 31: (n * (2^31 + 1)) >> 31 = n for n < 2^31
  return FastDiv{(uint32_t)mul, 31u + l};
}

// What the device reads per tile: the record of the tile table with a copy of its operator's
// descriptor beside it, so that one fetch (and one prefetch) brings everything a workgroup
// needs to start the tile.
struct TileWork {
  sk_tile tile;
  DevProblem prob;
};
static_assert(sizeof(TileWork) == 192, "TileWork layout");

// How the device's list slices a rectangle of the table anew: into S slices of that many reduction elements (S == 0: as the table has it).
struct Slicing {
  int64_t S = 0, slice = 0;
};

// The records the device runs, with output rectangles and a split-K workspace numbered for them, and the per-die lists over them.
struct WorkList {
  std::vector<sk_tile> work;
  std::vector<int64_t> count;    // per operator
  std::vector<uint32_t> ws_off;  // per output rectangle
  int64_t ws_f32x4 = 0;
  std::vector<uint32_t> xorder;
  uint32_t xoff[9] = {};
  std::vector<Slicing> slicing;  // of the table's rectangles, up to the last that is sliced anew
  bool window = false;  // has runs of pixels: only the general kernels of one element type take it
};

struct HostPlan {
  std::vector<sk_problem> problems;
  std::vector<DevProblem> dev;
  std::vector<sk_tile> tiles;
  std::vector<int32_t> order;
  std::vector<int64_t> first, count;
  std::vector<uint32_t> ws_off;  // per output rectangle: offset of its split-K partials, in 16-byte units
  int64_t ws_f32x4 = 0;          // size of the split-K workspace, in 16-byte units
  // The LDS tiles of the table once more, as eight lists (one per accelerator die): xorder[xoff[x] .. xoff[x+1])
  // are the table indices of the tiles die x takes, in the order it takes them.  Empty when xcd_part is 0.
  std::vector<uint32_t> xorder;
  uint32_t xoff[9] = {};
  sk_plan_params params;
  int64_t target_tile_bytes = 0;
  bool rows = false;  // some operators are planned as ones of run_tile_rows (FLAG_ROWS)
  // what the device runs in place of the table (see device_list); without records: the table itself
  WorkList run;
  const std::vector<sk_tile> &records() const { return run.work.empty() ? tiles : run.work; }
  int64_t record_count(size_t i) const { return run.work.empty() ? count[i] : run.count[i]; }
  const std::vector<uint32_t> &rect_off() const { return run.work.empty() ? ws_off : run.ws_off; }
  int64_t ws_units() const { return run.work.empty() ? ws_f32x4 : run.ws_f32x4; }
  const std::vector<uint32_t> &die_order() const { return run.work.empty() ? xorder : run.xorder; }
  const uint32_t *die_offsets() const { return run.work.empty() ? xoff : run.xoff; }
};

// Pure host planning (no HIP call).  Returns SK_OK or an error with `err` set.
sk_status plan_host(const sk_problem *problems, int32_t n, const sk_plan_params *params,
                    HostPlan &out, std::string &err);

// The device's work list for a launch of that many workgroups: the table's records, of which those of operators without 16-byte
// pieces that the launch would wait for are cut into parts of 64 x 64 outputs (`work`; `count` of them per operator; false
// and untouched if nothing is to be cut).
bool refine_tiles(const HostPlan &hp, int64_t workgroups, std::vector<sk_tile> &work, std::vector<int64_t> &count);

// Operators that run_window serves as runs of output pixels, where that pays (false: none).
bool window_operator(const HostPlan &hp, size_t i);
bool window_records(const HostPlan &hp, int64_t workgroups, std::vector<sk_tile> &records, std::vector<int64_t> &count);
// What the device runs in place of the plan's table (false: the table itself): these and refine_tiles, long records cut, operators of one
// deadline the longest first.  tiles_only: runs of pixels or nothing; without `slices`: none that the table does not have.
bool device_list(const HostPlan &hp, int64_t workgroups, bool tiles_only, WorkList &out, bool slices = true);
// The same for every operator of the baseline's tables (plan_host_each_alone), each a launch of its own, as tiles; false: nothing changed.
bool balance_each_alone(HostPlan &alone, int64_t workgroups);

// Whether every tile of the plan, and of each of its operators planned alone, is a 128 x 64 LDS tile whose operands can
// be read through 32-bit descriptors (the device's lean_operands, for the whole operator instead of tile by tile).
bool narrow_plan(const HostPlan &hp);
// Whether a launch of that many such tiles, the longest of so many stages of the reduction, is faster in the kernel of which three
// workgroups share a compute unit than in the general one.
bool narrow_pays(bool fp32, int64_t stages, int64_t tiles, int64_t compute_units);
// The tile tables of the one-launch-per-operator baseline: every operator of `whole` planned
// by plan_host as if it were submitted alone, with its long records cut as for a launch of its own on that many workgroups,
// concatenated in submission order.
sk_status plan_host_each_alone(const HostPlan &whole, int64_t workgroups, HostPlan &out, std::string &err);

inline int elem_size(int32_t dtype) { return dtype == SK_F32 ? 4 : 2; }

// SK_STATIC_SCRATCH_BYTES is what a plan's table may need for sk_launch_static.  The device's list slices further than the table, and both
// launch calls have to slice alike, so such plans have a larger array (of 3300 random plans whose tables fit, 52 lists need more than
// SK_STATIC_SCRATCH_BYTES, the largest 46 MiB).  Its address on the current device goes to *ptr (a hipError_t; scratch.hip).
constexpr size_t LARGE_SCRATCH_BYTES = 3 * (size_t)SK_STATIC_SCRATCH_BYTES;
int large_scratch_address(void **ptr);

// Sets the calling thread's sk_last_error() text and passes the status through (superkernel.hip).
sk_status set_last_error(sk_status st, const std::string &msg);

// sk_launch of a plan with stamps, which leave for `host_stamps` (the n completion stamps and the start; memory that the device can
// write) behind it; `done` (a hipEvent_t) completes when they are there.  Not under stream capture (superkernel.hip).
sk_status launch_with_stamps(sk_plan *plan, void *hip_stream, uint64_t *host_stamps, void *done);

// ---- the arrival queue's decisions, free of HIP calls so that they can be exercised on the host ----

// One submitted operator as the batch selection sees it.
struct QueuedOp {
  double deadline_ms;  // absolute: submit time + budget (+inf if none)
  int64_t bytes;       // operand bytes, for the duration estimate
  const void *C;       // its output buffer
};

// Operand bytes of an operator (activations + weights + output, each once), 0 for a malformed one.
int64_t operand_bytes(const sk_problem &p);

// Estimated duration of a launch over `bytes` of operands.
double estimate_launch_ms(int64_t bytes, double bytes_per_ms, double floor_ms);

// Which of `ops` (any order) go into the next launch, as indices in the order they are to be planned:
// earliest deadline first, ties by index; an operator whose output buffer is in `busy` (sorted) or was
// taken by an earlier pick waits; SK_QUEUE_OOO closes the batch before the operator that would take
// the estimate (times `corr`) past cap_ms, unless the batch is still empty; SK_QUEUE_SEQUENTIAL takes
// the first submitted operator only (index 0), whatever its deadline.
std::vector<size_t> select_batch(const std::vector<QueuedOp> &ops, const std::vector<const void *> &busy, int policy,
                                 double cap_ms, double corr, double bytes_per_ms, double floor_ms);

// Bookkeeping of one plan's launches, free of HIP calls so that it can be exercised on the host.
// A plan has one tile queue, one set of split-reduction counters and one workspace: a launch may only
// start when the one before it has finished or precedes it on the same stream.  The ledger says when
// the caller has to ask the event behind the latest launch, and what sk_plan_destroy must wait for.
struct LaunchLedger {
  enum Ask { GO, QUERY_EVENT };            // QUERY_EVENT: launch only if the event has completed, else SK_ERR_BUSY
  enum Wait { NOTHING, EVENT, DEVICE };
  bool has_event = false;                  // an event sits behind the latest launch made outside a stream capture
  uintptr_t last_stream = 0;
  bool device_wide = false;                // launches the event does not cover (captured into a graph, or the
                                           // event could not be recorded): only a device-wide wait covers them
  Ask before_launch(uintptr_t stream, bool capturing) const;
  // event_recorded: the caller recorded the plan's event behind the launch (never under capture)
  void after_launch(uintptr_t stream, bool capturing, bool event_recorded);
  Wait before_destroy() const;
};

}  // namespace sk
