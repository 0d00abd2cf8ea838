// Internal declarations shared by the host planner (ttc_plan.cpp) and the device side
// (ttc_device.hip).  Nothing here is part of the C ABI.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "ttc.h"
#include "ttc_aux.h"

namespace ttc {

constexpr int kMaxDim = TTC_MAX_DIM;
constexpr int kWave = 64;                 // CDNA wavefront
constexpr int kMaxThreads = 512;          // launch bound of every kernel
constexpr int kMaxLdsBytes = 160 * 1024;  // per workgroup: all of a CU's LDS (gfx950); smaller tiles let several workgroups share it

// Exact unsigned division by a run-time constant d >= 1 for any 32-bit x whose
// quotient sum does not overflow (x < 2^31 is enough):
//   q = (mulhi(x, mul) + x) >> shift,   mul = floor(2^32 (2^shift - d) / d) + 1,  shift = ceil(log2 d).
struct FastDiv {
    uint32_t mul;
    uint32_t shift;
    uint32_t div;
};
FastDiv make_fastdiv(uint32_t d);

constexpr int kBoxDims = 4;               // a box spans at most this many indices
constexpr int kMaxIters = 2048;           // sub-box positions per tile and walk (size of the position table)
constexpr int kMaxDigitExtent = 32000;    // flat extent of one digit of a walk: coordinates are compared 16 bits at a time

// A box spans at most kBoxDims indices of the tensor; "slot" j is the j-th of them in A order.
// Each walk ("side") sees the box as up to kBoxDims digits.  A digit is one index, or -- when
// the leading indices of the walk's tensor lie whole inside the box -- the chain of those
// indices merged into one flat index (the tile-level form of the paper's index fusion): the
// flat digit is contiguous in memory over the whole chain.  Digits are stored at the slot of
// the chain's outermost index, the only one the tensor's edge can cut; a slot whose index is
// an inner member of a chain holds an empty digit (tile = 1).
struct Digit {
    int32_t  tile;                   // flat extent of the digit inside the box
    int32_t  lane;                   // flat extent of the sub-box the 64 lanes cover
    int32_t  iters;                  // ceil(tile / lane): sub-box positions along the digit
    int32_t  lane_mul;               // flat elements per lane step: vec on the vector digit, else 1
    int32_t  slot_mul;               // flat elements per step of the slot's index (product of merged inner extents)
    int32_t  lstride;                // LDS element stride of one flat step
    int32_t  ragged;                 // 1: lane does not divide tile (the last sub-box position overhangs)
    int32_t  pad;
    FastDiv  lane_below, lane_cnt;   // lane id -> lane coordinate: (lane / below) % cnt
    FastDiv  iter_below, iter_cnt;   // position id -> position digit
    int64_t  gstride;                // element stride of one flat step in the tensor the walk follows
    int64_t  g2stride;               // direct kernel: element stride in B
};

struct Side {
    int32_t  vec;                    // elements per lane per access, along the walk's first digit
    int32_t  lanes;                  // active lanes of a wavefront
    int32_t  n_iter;                 // sub-box positions per tile = prod(iters)
    int32_t  vec_lds_stride;         // LDS element stride between the vec elements of one lane
    int32_t  exact;                  // 1: lane divides tile on every digit (no ragged sub-boxes)
    int32_t  chunk;                  // positions per wavefront, rounded up: ceil(n_iter / waves)
    int32_t  chunk_rem;              // wavefronts that really have `chunk` positions (the others have one less)
    int32_t  partial;                // 1: the first digit's extent is not a multiple of vec: the last vector of a run is cut
    int32_t  vec_slot;               // slot (0..3) that holds the walk's first digit, the one vectors run along
    FastDiv  chunk_div;
    Digit    d[kBoxDims];
};

struct Slot {
    int32_t  tile;                   // box extent along the slot's index
    int32_t  pad;
    int64_t  size;                   // extent of the index in the tensor
    FastDiv  tile_below, tile_cnt;   // tile id -> tile coordinate along this index
};

// The micro-tile kernel: a tile spans ta columns and tb rows and nothing else.  The column index is A's stride-1
// index (index 0), or A's indices 0 and 1 taken as one index where rows are short (together they are one contiguous
// run of A, and a column's place in B follows from its two parts); the row index is B's stride-1 index (A's index
// p0), or B's first two indices taken as one.  Lanes load 16-byte vectors along the columns and park them in LDS with
// one 128-bit write; after the barrier a lane reads the vec x vec block it owns with vec 128-bit reads, transposes
// it in registers and stores vec 16-byte vectors along the rows.  Rows of the LDS tile are `pitch`
// 16-byte chunks long (a multiple of eight); chunk c of row r sits at chunk position c ^ ((r / vec) & 7), which
// makes both the writes (lanes along c) and the reads (lanes along r in steps of vec) free of bank conflicts.
struct MicroParams {
    int32_t  ta, tb;                 // tile extents along the column index and along the row index (multiples of vec)
    int32_t  p0;                     // the index of A that is B's stride-1 index
    int32_t  merged_a, merged_b;     // 1: the column index is A's indices 0 and 1 taken as one (contiguous in A), the row
                                     // index B's first two indices taken as one (contiguous in B); 0: one index each
    int32_t  vec, vec_log;           // elements in 16 bytes, and its log2
    int32_t  la, lb;                 // ta / vec and tb / vec: vectors per row of the tile, blocks per column
    int32_t  pitch;                  // 16-byte chunks per row of the LDS tile: la rounded up to a multiple of 8
    uint32_t swizzle;                // 7: chunk c of row r sits at c ^ ((r / vec) & 7); 0: rows laid out plainly (measurement aid)
    // One pair of fields for both kernels, which never read each other's: as fields of their own (448 bytes of arguments
    // instead of 440) they cost the line kernel 1-6 % of a 4 us launch (25 x 1257 x 6 fp64 -> fp32 4.19 us, 4.36 with them
    // here, 4.21 with them at the end).
    union {
        int32_t loads;               // vectors a lane loads per tile: ceil(la * tb / threads)
        int32_t lines;               // line kernel: LineShape::lines (a skewed tile writes one line less per column)
    };
    union {
        int32_t blocks;              // vec x vec blocks a lane owns: ceil(la * lb / threads)
        int32_t skewed;              // line kernel: 1: the columns of B start at different places inside a line, so every
                                     // column of a tile is cut where its own lines end; 0: tiles are cut at the same row everywhere
    };
    FastDiv  la_div, lb_div;
    int64_t  size_a0, size_p0;       // extents of the column index and of the row index (the product where two are merged)
    // A column x sits at element x of A's run and at (x % in) * stride_in + (x / in) * stride_out in B, where `in`
    // is the extent of A's index 0; a row likewise with the tensors exchanged.  Not merged: x / in is always 0.
    FastDiv  col_in_div, row_in_div;
    int64_t  col_b_in, col_b_out;    // element strides in B of the column index's inner and outer part
    int64_t  row_a_in, row_a_out;    // element strides in A of the row index's inner and outer part
};

// The line kernel's tile: `cols` columns (the contiguous direction of A) by the rows of `lines` 128-byte lines of B.
// Everything follows from those two and the element sizes; the kernels take it at compile time, the planner and the
// replay at run time.
struct LineShape {
    int32_t  cols, lines;
    int32_t  va, vb;                 // elements in 16 bytes of A and of B
    int32_t  line;                   // elements of B in a line
    int32_t  rows;                   // rows of A held in LDS: lines * line
    int32_t  lanes;                  // lanes that load one row (16 bytes each)
    int32_t  pass;                   // rows the workgroup loads at once
    int32_t  passes;                 // 16-byte loads per lane
    int32_t  side;                   // columns the workgroup stores at once, eight lanes each ...
    int32_t  groups;                 // ... and how many lines of each: 32 / side
    int32_t  pitch;                  // elements from one row to the next in LDS
    int32_t  lds_bytes;
};
constexpr int kLineThreads = 256;
constexpr int kLineBytes = 128;
constexpr int64_t kLineMaxExtent = (int64_t(1) << 31) - 4096;    // rows and columns: tile limits are worked out in 32 bits
// LDS pitch: a lane of the store phase reads the elements of one column, eight lanes with rows 16 bytes of B apart
// times eight neighbouring columns per instruction.  cols + 2 (4- and 8-byte elements) or cols + 1 (16-byte) keeps the
// row starts aligned for the 8- and 16-byte LDS writes and spreads the reads of one precision of 4 or 8 bytes evenly
// over the banks; by the bank model two precisions and 16-byte elements meet some bank twice, and so do the writes of rows of
// 128 bytes (a plan's lds_conflict_a and lds_conflict_b).  Measured, LDS cycles per instruction and conflicts among them: 384^3
// fp32 -> fp64 5.3 and 0.0, 1024^2 fp32 8.0 and 2.7, complex128 9.8 and 3.6; the micro-tile kernel's swizzled tile 8.0 and 2.0.
constexpr LineShape line_shape(int cols, int lines, int eb_a, int eb_b)
{
    LineShape s = {};
    s.cols = cols;
    s.lines = lines;
    s.va = 16 / eb_a;
    s.vb = 16 / eb_b;
    s.line = kLineBytes / eb_b;
    s.rows = lines * s.line;
    s.lanes = cols / s.va;
    s.pass = kLineThreads / s.lanes;
    s.passes = s.rows / s.pass;
    s.side = cols < kLineThreads / 8 ? cols : kLineThreads / 8;
    s.groups = kLineThreads / 8 / s.side;
    s.pitch = cols + (eb_a == 16 ? 1 : 2);
    s.lds_bytes = s.rows * s.pitch * eb_a;
    return s;
}
// which tiles exist as kernels: rows of 128 to 512 bytes, whole passes, at most 44 KB of LDS (three workgroups per compute unit)
constexpr bool line_shape_ok(int cols, int lines, int eb_a, int eb_b)
{
    const LineShape s = line_shape(cols, lines, eb_a, eb_b);
    return (cols == 16 || cols == 32 || cols == 64) && (lines == 2 || lines == 4 || lines == 8) &&
           cols * eb_a >= 128 && cols * eb_a <= 512 && s.rows % s.pass == 0 && lines % s.groups == 0 && s.lds_bytes <= 44 * 1024;
}

// HIP launches fewer than 2^32 work items; kernels that give every tile or chunk a workgroup of its own reach that.
constexpr bool launchable(int64_t grid, int threads)
{
    return grid >= 1 && grid <= INT32_MAX && grid * threads < (int64_t(1) << 32);
}

// Everything a kernel launch needs; passed by value as the kernel argument.
struct KernelParams {
    int32_t  n;                      // fused number of indices
    int32_t  xcd_remap;              // how tile ids map to the 8 XCDs: 0 round robin, 1 one contiguous range each,
                                     // k >= 2: chunks of 2^k consecutive tiles dealt round robin
    uint32_t num_tiles;
    uint32_t tiles_per_xcd;          // num_tiles / 8
    uint32_t tiles_rem_xcd;          // num_tiles % 8
    uint32_t grid;                   // workgroups launched (filled at launch; <= num_tiles)
    uint32_t grid_per_xcd;           // grid / 8
    uint32_t grid_rem_xcd;           // grid % 8
    uint32_t xcd_tiles[8];           // chunked mapping: tiles of each XCD
    int32_t  lds_data_off;           // byte offset of the first data buffer in dynamic LDS
    int32_t  lds_tile_elems;         // elements per LDS data buffer (padded tile)
    int32_t  lds_buffers;            // 2: tile buffers alternate, one barrier per tile; 1: one buffer, two barriers
    int32_t  nt_a;                   // 1: loads of A carry the non-temporal hint (streamed, not kept in cache)
    int32_t  nslots;                 // indices the box spans
    int32_t  nt_b;                   // 1: stores to B, and loads of B when beta != 0, carry the non-temporal hint
    Slot     slot[kBoxDims];
    int32_t  tile[kMaxDim];          // box extent per fused index of A (1 = index not blocked)
    FastDiv  tile_below[kMaxDim];    // prod of tile counts of the indices that vary faster in the tile order
    FastDiv  tile_cnt[kMaxDim];      // ceil(size[k] / tile[k])
    int64_t  stride_a[kMaxDim];      // element stride of fused index k in A
    int64_t  stride_b[kMaxDim];      // element stride of fused index k in B
    Side     a;                      // load walk (A order)
    Side     b;                      // store walk (B order); unused by the direct kernel
    double   alpha[2];               // re, im (im = 0 for real types)
    double   beta[2];
    int32_t  debug_stop;             // measurement aid: 1 = every workgroup returns after its set-up (micro-tile kernel: 2 = after its loads)
    int32_t  pad_end;
    MicroParams micro;               // micro-tile kernel only
};

// The micro-tile kernel's whole argument: what it needs of KernelParams and nothing else, seven 64-byte lines
// instead of twenty-six.  Every workgroup reads its arguments through the scalar cache before it can issue a
// load, and that shows: a copy kernel that first reads 1.6 KB of arguments takes 0.9 us longer per launch than the
// same kernel with 24 bytes (8 MB: 3.8 against 2.9 us; 32 MB: 8.3 against 7.2 us).  Built from the candidate at
// launch (micro_args()), so that the tile mapping and the streaming hints are the plan's current ones.
struct MicroArgs {
    int32_t  xcd_remap;              // the fields of KernelParams that tile_sequence() reads, under the same names
    uint32_t num_tiles, tiles_per_xcd, tiles_rem_xcd;
    uint32_t grid, grid_per_xcd, grid_rem_xcd;
    uint32_t xcd_tiles[8];
    int32_t  nt_a, nt_b;
    int32_t  debug_stop;
    int32_t  col_pos, row_pos;       // where the column index and the row index stand in the tile order
    int32_t  pad;
    FastDiv  cnt[kMaxDim];           // tile id -> tile coordinates, mixed radix in tile order: tiles along the i-th index of the order
    int64_t  step_a[kMaxDim];        // element offset in A, and in B, of one tile step along it (the column index: its place
    int64_t  step_b[kMaxDim];        // in A's run only; the row index: its place in B's run only; see MicroTile)
    double   alpha[2], beta[2];
    MicroParams micro;
};
static_assert(sizeof(MicroArgs) == 440, "seven lines of arguments, with room for the first of the two pointers");

// Parameters of the row kernel (stride-1 index fixed: rows are contiguous in both tensors), and of the gather kernel.  B is walked in
// the order of its multi-index, so the writes of consecutive workgroups are consecutive in memory.
struct RowsParams {
    int32_t  n;                      // fused number of indices; index 0 is the row
    int32_t  vec;                    // elements per lane and access
    int32_t  unroll;                 // accesses a lane keeps in flight
    int32_t  overlap;                // 1: rows are not a multiple of vec: the last vector of a row is moved back to end with it
    uint32_t row;                    // extent of index 0
    uint32_t slots;                  // vectors per row: ceil(row / vec); flat: elements per row
    uint32_t chunk;                  // vectors a workgroup moves: threads * unroll
    int32_t  nt_a, nt_b;             // non-temporal accesses per side
    int32_t  flat;                   // 1: B is dense: vectors are counted through B from its first element, across the ends of rows
    int32_t  xcd_remap;              // how the workgroups' chunks are dealt to the XCDs (as KernelParams::xcd_remap)
    uint32_t blocks;                 // chunks, one per workgroup
    uint32_t per_xcd;                // gather kernel, round robin over the XCDs (xcd_remap 0): 0, or chunks are numbered so that every
                                     // eighth is the next one in B (eight ranges of this many chunks side by side)
    uint32_t rows;                   // rows of the tensor
    FastDiv  slot_div;               // x / slots
    FastDiv  size_div[kMaxDim];      // extent of B's index d, d = 1 .. n-1 (entry 0: gather kernel only)
    int64_t  stride_a[kMaxDim];      // element stride in A of B's index d
    int64_t  stride_b[kMaxDim];      // element stride in B of B's index d
    int64_t  vectors;                // rows * slots; flat: ceil(elements / vec)
    int64_t  elements;
    double   alpha[2];
    double   beta[2];
};

// The block kernel: a tile is a box whose leading indices are one contiguous run of A (run_a elements, `rows` of them) and one
// contiguous run of B (run_b elements, `outs` of them); an index may be part of both runs.  At most two indices are cut into
// tiles: the last one of A's run and the last one of B's (they may be one and the same); all others of the box lie whole in it.
// LDS holds the tile in A's order, a row every `pitch` elements.
struct BlockParams {
    int32_t  run_a, run_b;           // elements of a whole tile's runs
    int32_t  inner_a, inner_b;       // elements of a run per step of the index it ends with
    int32_t  tile_a, tile_b;         // tile extents of the two indices the runs end with
    int32_t  pos_a, pos_b;           // where these stand in the tile order
    int32_t  cut_row, cut_out;       // which digit of a row's place (0, 1; -1: none) is the index B's run ends with, and which
                                     // digit of an out's place the one A's run ends with
    int32_t  rows, outs, pitch, even;// even: B's first index is a multiple of the vector
    int32_t  unroll, pad;            // vectors a lane loads
    int64_t  size_a, size_b;         // extents of the two indices in the tensor
    FastDiv  va_div, vb_div;         // vectors of a run
    FastDiv  row_div, out_div;       // extent of digit 0 of a row's place, of an out's place
    FastDiv  x_div[2];               // place in B's run -> indices: extents of the first two
    int32_t  x_lds[3], out_lds[2];   // LDS strides of B's run's indices and of an out's digits
    int32_t  pad_end;
    int64_t  row_step[2], out_step[2];   // element strides in A of a row's digits, in B of an out's
};

// The block kernel's whole argument.
struct BlockArgs {
    int32_t  xcd_remap;              // how the tiles are dealt to the XCDs (as KernelParams::xcd_remap)
    uint32_t blocks;                 // tiles, one per workgroup
    int32_t  nt_a, nt_b;
    FastDiv  cnt[kMaxDim];
    int64_t  step_a[kMaxDim], step_b[kMaxDim];
    double   alpha[2], beta[2];
    BlockParams block;
};
constexpr int kBlockThreads = 256;
constexpr int kBlockMaxLds = 64 * 1024;
// vectors a lane stores where it loads `unroll`
constexpr int block_stores(int unroll, int eb_a, int eb_b) { return unroll * eb_b / eb_a < 1 ? 1 : unroll * eb_b / eb_a; }

// RowsParams of a small problem, packed.  Launches with up to 96 bytes of arguments, the two pointers included, leave the host
// at 2.6-2.8 us each, larger ones at 3.4-3.6 (112 to 456 bytes; empty kernels in a row), which is most of what a small problem
// takes; and its workgroups begin sooner.  70 x 33 x 45 fp32 (2,0,1) 3.46 -> 2.78 us a launch, 600 x 600 fp32 4.05 -> 3.44,
// 96 x 80 x 70 fp32 (0,2,1) 3.3 -> 2.87.  Where chunks are dealt to the XCDs in groups parameters go whole, and where they
// do not fit (six indices, strides beyond 32 bits).  Four words (elements, chunks, per_xcd, rows), then per division two (the multiplier; divisor and shift), the
// strides in A, and at an 8-byte boundary the scalars that the epilogue reads.
// The line kernel's MicroArgs are packed the same way: a word of places and flags, the first two divisions of the tile id, the
// third index's steps, the extents, where columns lie in B and rows in A, and (MERGED) how a merged index is taken apart.
struct SmallArgs { uint32_t w[20]; };
constexpr int kSmallMaxDim = 5;
constexpr int64_t kSmallMaxElements = int64_t(1) << 26;       // divisors leave five bits of their word to the shift

// The line kernel's internal class.  Plans report it as TTC_KERNEL_LDS (its tile is staged through LDS) with a
// non-zero `unroll`.
constexpr int kKernelLines = 4;
// The gather kernel's; reported as TTC_KERNEL_ROWS (B is walked front to back).
constexpr int kKernelGather = 5;
// The block kernel's; reported as TTC_KERNEL_MICRO with bit 2 of `merged` set.
constexpr int kKernelBlock = 6;

// One candidate launch configuration ("candidate" in the paper's Section 3).
struct Candidate {
    int      kernel_class;           // TTC_KERNEL_*, kKernelLines or kKernelGather
    int      threads;
    int      wg_per_cu;              // workgroups launched per compute unit (each walks several tiles)
    int      lds_bytes;              // dynamic LDS per workgroup: shared tile records, spare slots, position tables, one or two tile buffers
    int      tile_order[kMaxDim];
    int      tile[kMaxDim], lds_stride[kMaxDim];   // by fused index of A
    int      digits_a, digits_b;                   // digits of each walk, in the walk's own order:
    int      dtile_a[kBoxDims], dlane_a[kBoxDims]; //   flat extent and lane sub-box extent
    int      dtile_b[kBoxDims], dlane_b[kBoxDims];
    int      lds_conflict_a, lds_conflict_b;
    double   score;                  // heuristic cost, smaller is better
    double   model_us;               // gather kernel: modelled time
    float    tuned_ms;
    KernelParams kp;                 // box kernels (staged and direct); the streaming flags and the tile mapping of every class
    RowsParams rows;                 // row kernel
    BlockParams block;               // block kernel
};

// Element kinds of one tensor (the two tensors of a mixed-precision problem differ).
enum { kKindF32 = 0, kKindF64 = 1, kKindC64 = 2, kKindC128 = 3 };

struct Problem {
    int      dtype;                  // TTC_* code the plan was created with
    int      kind_a, kind_b;         // element kind of A and of B
    int      eb_a, eb_b;             // element bytes of A (also the LDS tile's) and of B
    int      epilogue;               // TTC_EPI_*
    int      ndim;                   // fused
    int64_t  size[kMaxDim];
    int      perm[kMaxDim];
    int64_t  stride_a[kMaxDim];      // by fused index of A; from the leading dimensions, dense if none were given
    int64_t  stride_b[kMaxDim];      // by fused index of A (stride it has in B)
    int64_t  elements;
    int64_t  span_a, span_b;         // elements from the first to the last element of each (sub-)tensor, inclusive
    double   alpha[2], beta[2];
};

}  // namespace ttc

struct ttc_plan_s {
    ttc::Problem prob;
    std::vector<ttc::Candidate> cands;     // complete: candidate 0 is ttc_plan_create's choice, the others follow ranked
                                           // by the heuristic cost; not complete: only that choice
    int selected;
    bool complete;
};

namespace ttc {

// Host planner.  Returns TTC_OK and fills *out, or a status.
int build_plan(int dtype, int ndim, const int64_t* sizes, const int* perm, const int64_t* lda, const int64_t* ldb,
               const void* alpha, const void* beta, ttc_plan_s* out);
int complete_plan(ttc_plan_s* plan);
void set_last_status(int status);
bool verbose();
// Plan store (ttc_cache.cpp).
int cache_store(const ttc_plan_s* plan, const char* path);
int cache_lookup(ttc_plan_s* plan, const char* path);
// Workgroups to launch for a candidate on a device with `cus` compute units.
uint32_t launch_grid(const Candidate& c, int cus);
void set_grid(KernelParams* kp, uint32_t grid);
// tile ids -> XCDs: 0 round robin, 1 one contiguous range per XCD, 2..10: chunks of 2^mode tiles dealt in turn
// mode -1: the default, chunks of 32 tiles; round robin below 2048 tiles (line and row kernel: default_tile_mapping() has the say)
constexpr int kDefaultTileMapping = -1;
constexpr int kMaxTileMapping = 10;                  // chunks of 2^10
bool set_tile_mapping(KernelParams* kp, int mode);
void default_streaming(const Problem& P, Candidate* c);
MicroArgs micro_args(const Candidate& c);
BlockArgs block_args(const Candidate& c);

}  // namespace ttc
