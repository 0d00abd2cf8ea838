// Index arithmetic of a tile walk, shared by the device kernels and by the host-side bounds
// checker (ttc_debug_emulate_map), so that what the checker proves in bounds is the code the
// GPU runs.
//
// A walk covers the tile with copies of one fixed sub-box.  Two small tables make a step of
// the walk cost a handful of instructions whatever the number of indices:
//   * per lane (vector registers, built once per workgroup): where the lane sits inside the
//     sub-box -- its offset in the tensor, its offset in the LDS tile, its coordinates;
//   * per sub-box position (LDS, built once per workgroup, the same for every tile): where
//     the sub-box sits inside the tile -- the same three things.
// A memory access of the walk is then  tile base + position entry + lane entry.
#pragma once

#include "ttc_internal.h"

#if defined(__HIPCC__)
#define TTC_HD __host__ __device__ __forceinline__
#else
#define TTC_HD inline
#endif

namespace ttc {

TTC_HD uint32_t fdiv(uint32_t x, const FastDiv& d)
{
    return ((uint32_t)(((uint64_t)x * d.mul) >> 32) + x) >> d.shift;
}
TTC_HD uint32_t fdigit(uint32_t x, const FastDiv& below, const FastDiv& cnt)
{
    const uint32_t q = fdiv(x, below);
    return q - fdiv(q, cnt) * cnt.div;
}

// ---- row kernel: where a logical element of B (position in the order of B's multi-index) lies ----------
// `row_index` counts rows in B's order (all indices but the first), `col` is the position inside the row.
struct RowPlace { int64_t a, b; };

TTC_HD RowPlace rows_place(const RowsParams& p, uint32_t row_index, uint32_t col)
{
    RowPlace r;
    r.a = col; r.b = col;
    uint32_t rest = row_index;
#pragma unroll
    for (int d = 1; d < kMaxDim; ++d) {             // unused indices: extent 1, stride 0
        const uint32_t q = fdiv(rest, p.size_div[d]);
        const uint32_t j = rest - q * p.size_div[d].div;
        r.a += (int64_t)j * p.stride_a[d];
        r.b += (int64_t)j * p.stride_b[d];
        rest = q;
    }
    return r;
}

// One access of the row kernel: `k` is the number of its vector inside the workgroup's chunk, which starts at
// vector `base` = row `row0`, slot `slot0` (a row holds `slots` vectors; where the row is not a multiple of the
// vector, the last one is moved back so that it ends with the row and repeats elements of its neighbour).
// (slot0 + k stays far below 2^31: rows are shorter than 2^30 elements and a chunk holds at most 2^20 vectors.)
struct RowAccess { RowPlace at; bool valid; };

TTC_HD RowAccess rows_access(const RowsParams& p, int64_t base, uint32_t row0, uint32_t slot0, uint32_t k)
{
    const uint32_t x = slot0 + k;
    const uint32_t rl = fdiv(x, p.slot_div);
    const uint32_t sl = x - rl * p.slots;
    uint32_t c = sl * (uint32_t)p.vec;
    if (c + (uint32_t)p.vec > p.row) c = p.row - (uint32_t)p.vec;      // only with overlap: the last slot of a row
    RowAccess r;
    r.valid = (base + (int64_t)k < p.vectors);
    r.at = rows_place(p, r.valid ? row0 + rl : 0u, r.valid ? c : 0u);  // past the end: the first vector, never stored
    return r;
}

// Flat: vector `k` of the workgroup's chunk, which starts at element `base` of a dense B = row `row0`, column `col0`.  Its first
// `head` elements end row r (all of them unless the row ends inside the vector), the others begin the next row: `a` is where
// a whole vector of row r lies that holds the head (as its last elements if the row ends), `a_next` where row r + 1 begins.
// left: elements of B from the vector's first on (fewer than vec only at the end of B).  Rows hold at least one vector.
struct FlatAccess { int64_t a, a_next, b, left; uint32_t head; bool valid, split; };

TTC_HD FlatAccess flat_access(const RowsParams& p, int64_t base, uint32_t row0, uint32_t col0, uint32_t k)
{
    const uint32_t vec = (uint32_t)p.vec, x = col0 + k * vec;
    const uint32_t rl = fdiv(x, p.slot_div);
    const uint32_t c = x - rl * p.row;
    FlatAccess f;
    f.b = base + (int64_t)k * vec;
    f.left = p.elements - f.b;
    f.valid = f.left > 0;
    const uint32_t r = f.valid ? row0 + rl : 0u, col = f.valid ? c : 0u;      // past the end: the first vector, never stored
    f.head = p.row - col < vec ? p.row - col : vec;
    f.split = f.head < vec;
    f.a = rows_place(p, r, f.split ? p.row - vec : col).a;
    f.a_next = f.split ? rows_place(p, r + 1u < p.rows ? r + 1u : r, 0u).a : 0;
    return f;
}

// ---- gather kernel: where element `e` of B, in the order of B's multi-index, lies in both tensors ----
struct GatherPlace { int64_t a, b; uint32_t first; };        // first: its coordinate along B's index 0

TTC_HD GatherPlace gather_place(const RowsParams& p, uint32_t e)
{
    GatherPlace r = {0, 0, 0};
    uint32_t rest = e;
#pragma unroll
    for (int d = 0; d < kMaxDim; ++d) {             // unused indices: extent 1, stride 0
        const uint32_t q = fdiv(rest, p.size_div[d]);
        const uint32_t j = rest - q * p.size_div[d].div;
        if (d == 0) r.first = j;
        r.a += (int64_t)j * p.stride_a[d];
        r.b += (int64_t)j * p.stride_b[d];
        rest = q;
    }
    return r;
}

// Workgroup `wg`'s place where each XCD has one range of `per_xcd` places.
TTC_HD uint32_t range_place(uint32_t per_xcd, uint32_t wg) { return (wg & 7u) * per_xcd + (wg >> 3); }

// First element of lane `tid` of chunk `block` (past the end of B: nothing to do).
TTC_HD uint32_t gather_first(const RowsParams& p, uint32_t block, uint32_t tid)
{
    if (p.per_xcd && p.xcd_remap == 0) block = range_place(p.per_xcd, block);
    return (block * p.chunk + tid) * (uint32_t)p.vec;
}

// Whether a lane's `count` elements of B, the first at `g`, are one contiguous vector of it (the kernel then stores them as
// one): a whole vector, inside one run of B unless B is dense.
TTC_HD bool gather_whole(const RowsParams& p, const GatherPlace& g, int32_t count)
{
    return count == p.vec && (p.flat || g.first + (uint32_t)p.vec <= p.row);
}

// Element e + j of B, given element e's place: a step along B's index 0 unless that ends before (past the end of B: the last element).
TTC_HD GatherPlace gather_next(const RowsParams& p, const GatherPlace& g, uint32_t e, uint32_t j)
{
    if (g.first + j < p.row) {
        GatherPlace r = {g.a + (int64_t)j * p.stride_a[0], g.b + (int64_t)j * p.stride_b[0], g.first + j};
        return r;
    }
    const uint32_t last = (uint32_t)(p.elements - 1);
    return gather_place(p, e + j < last ? e + j : last);
}

// Which chunk workgroup `wg` of a row-kernel launch moves (p.blocks: none): consecutive chunks, which share a line of
// B and lines of A, go to one XCD a few at a time, as with tiles.  The block kernel's tiles likewise.
template <typename Params>       // RowsParams, BlockArgs or SmallDeal
TTC_HD uint32_t rows_block(const Params& p, uint32_t wg)
{
    if (p.xcd_remap == 0) return wg;
    const uint32_t x = wg & 7u, q = wg >> 3;
    if (p.xcd_remap == 1) {
        const uint32_t per = (p.blocks + 7u) / 8u, block = x * per + q;
        return q < per && block < p.blocks ? block : p.blocks;
    }
    const uint32_t log = (uint32_t)p.xcd_remap, block = ((x + 8u * (q >> log)) << log) + (q & ((1u << log) - 1u));
    return block < p.blocks ? block : p.blocks;
}

// Workgroups to launch so that every chunk has one: whole rounds of chunks over the XCDs.
template <typename Params>
TTC_HD int64_t rows_grid(const Params& p)
{
    if (p.xcd_remap == 0) return p.blocks;
    const int64_t round = p.xcd_remap == 1 ? 8 : int64_t(8) << p.xcd_remap;
    return (p.blocks + round - 1) / round * round;
}

// ---- the arguments of small problems ---------------------------------------------------------
// Words before the scalars.  Gather kernel: divisions for B's indices 0 ... n-2, strides of all; row kernel (flat): divisions for
// the row and B's indices 1 ... n-2, strides of indices 1 ... n-1.
constexpr int small_words(bool gather, int n) { return (4 + 2 * (n - 1) + (gather ? n : n - 1) + 1) / 2 * 2; }
constexpr int small_scalars(int epilogue, bool is_complex) { return (epilogue == TTC_EPI_COPY ? 0 : epilogue == TTC_EPI_SCALE ? 1 : 2) * (is_complex ? 2 : 1); }
constexpr bool small_fits(bool gather, int n, int epilogue, bool is_complex) { return small_words(gather, n) + 2 * small_scalars(epilogue, is_complex) <= 20; }

// Which number of indices the kernels are compiled for serves this launch; 0: none, its arguments go unpacked.  nt_a, nt_b: the
// hints the packed kernels are compiled with.
inline int small_dims(const RowsParams& p, bool gather, int epilogue, bool is_complex, int nt_a, int nt_b)
{
    const int n = p.n < 2 ? 2 : p.n;
    if (!p.flat || p.xcd_remap > (gather ? 0 : 1) || p.nt_a != nt_a || p.nt_b != nt_b || n > kSmallMaxDim || p.elements >= kSmallMaxElements ||
        !small_fits(gather, n, epilogue, is_complex)) return 0;
    for (int d = 0; d < n; ++d)
        if (p.stride_a[d] > INT32_MAX || (p.size_div[d].div > 1 && (p.size_div[d].div - 1) * p.stride_a[d] > INT32_MAX)) return 0;
    return n;
}

inline SmallArgs small_pack(const RowsParams& p, bool gather, int n, int epilogue, bool is_complex)
{
    SmallArgs s = {};
    int at = 0;
    s.w[at++] = (uint32_t)p.elements;
    s.w[at++] = p.blocks;
    s.w[at++] = p.per_xcd;
    s.w[at++] = p.rows;
    for (int d = 0; d < n - 1; ++d) {
        const FastDiv& f = !gather && d == 0 ? p.slot_div : p.size_div[d];
        s.w[at++] = f.mul;
        s.w[at++] = f.div | f.shift << 27;
    }
    for (int d = gather ? 0 : 1; d < n; ++d) s.w[at++] = (uint32_t)p.stride_a[d];
    at = small_words(gather, n);
    const int count = small_scalars(epilogue, is_complex), each = is_complex ? 2 : 1;
    for (int k = 0; k < count; ++k) {
        const double v = k < each ? p.alpha[k] : p.beta[k - each];
        uint64_t bits;
        __builtin_memcpy(&bits, &v, 8);
        s.w[at++] = (uint32_t)bits;
        s.w[at++] = (uint32_t)(bits >> 32);
    }
    return s;
}

// The parameters as the index code reads them; what is not packed follows from the rest or is never read.  The last index's
// division only has to give quotient 0.
template <bool GATHER, int N, int MODE, bool COMPLEX>
TTC_HD RowsParams small_unpack(const SmallArgs& s, int vec, uint32_t chunk)
{
    RowsParams p;
    p.n = N; p.vec = vec; p.unroll = 1; p.overlap = 0; p.flat = 1; p.xcd_remap = 0; p.chunk = chunk;
    p.elements = (int64_t)s.w[0];
    p.blocks = s.w[1];
    p.per_xcd = s.w[2];
    p.rows = s.w[3];
    p.nt_a = 0; p.nt_b = GATHER ? 0 : 1;
    p.vectors = 0;
    int64_t b = 1;
#pragma unroll
    for (int d = 0; d < kMaxDim; ++d) {
        FastDiv f = {0u, d == N - 1 ? 31u : 0u, d == N - 1 ? 0u : 1u};
        if (d < N - 1) { f.mul = s.w[4 + 2 * d]; f.div = s.w[5 + 2 * d] & 0x7ffffffu; f.shift = s.w[5 + 2 * d] >> 27; }
        if (d == 0) { p.row = f.div; p.slots = f.div; p.slot_div = f; }
        p.size_div[d] = f;
        p.stride_a[d] = d < N && (GATHER || d > 0) ? (int64_t)(int32_t)s.w[4 + 2 * (N - 1) + (GATHER ? d : d - 1)] : 0;
        p.stride_b[d] = GATHER && d < N ? b : 0;
        b *= (int64_t)f.div;
    }
    p.alpha[0] = p.alpha[1] = p.beta[0] = p.beta[1] = 0.0;
    constexpr int kCount = small_scalars(MODE, COMPLEX), kEach = COMPLEX ? 2 : 1, kAt = small_words(GATHER, N);
#pragma unroll
    for (int k = 0; k < kCount; ++k) {
        const uint64_t bits = (uint64_t)s.w[kAt + 2 * k] | (uint64_t)s.w[kAt + 2 * k + 1] << 32;
        double v;
        __builtin_memcpy(&v, &bits, 8);
        if (k < kEach) p.alpha[k] = v; else p.beta[k - kEach] = v;
    }
    return p;
}

// Where workgroup `wg` of the row kernel with packed arguments starts: its first element of B, the row that one lies in and its place
// there.  RANGES: each XCD has one range of chunks; the workgroups behind the last chunk start past the end of B and find nothing valid.
struct SmallRowsStart { uint32_t first, row0, col0; };

template <bool RANGES>
TTC_HD SmallRowsStart small_rows_start(const RowsParams& p, uint32_t wg)
{
    SmallRowsStart s;
    s.first = (RANGES ? range_place(p.per_xcd, wg) : wg) * (p.chunk * (uint32_t)p.vec);
    s.row0 = fdiv(s.first, p.slot_div);
    s.col0 = s.first - s.row0 * p.row;
    return s;
}

// ---- which tiles a workgroup walks ---------------------------------------------------------
// Consecutive workgroup ids land on consecutive XCDs (8 of them, each with its own L2).  Every
// XCD owns one contiguous range of tile ids; its workgroups take the tiles of that range round
// robin, so tiles that are neighbours in memory are in flight on the same XCD at the same time.
// A workgroup walks positions first, first + step, ... < end of its XCD's sequence of tiles; tile_of() turns a
// position into a tile id.  Three mappings: plain round robin over all workgroups (one window that advances
// through the tensor: the lowest memory latency when tiles share no cache lines); one contiguous range of
// tile ids per XCD (neighbouring tiles always meet in one L2); and chunks of 2^k consecutive tiles dealt to the
// XCDs in turn (neighbours inside a chunk share an L2 and the window still advances as one).
struct TileSeq { uint32_t first, end, step, base, xcd, chunk_log; };

template <typename Params>       // KernelParams, or the micro-tile kernel's MicroArgs
TTC_HD TileSeq tile_sequence(const Params& p, uint32_t wg)
{
    TileSeq s;
    s.base = 0; s.xcd = 0; s.chunk_log = 0;
    if (!p.xcd_remap || p.grid < 8u) {
        s.first = wg; s.end = p.num_tiles; s.step = p.grid;
        return s;
    }
    const uint32_t x = wg & 7u, slot = wg >> 3;
    s.first = slot;
    s.step = p.grid_per_xcd + (x < p.grid_rem_xcd ? 1u : 0u);
    if (p.xcd_remap == 1) {
        s.base = x * p.tiles_per_xcd + (x < p.tiles_rem_xcd ? x : p.tiles_rem_xcd);
        s.end = p.tiles_per_xcd + (x < p.tiles_rem_xcd ? 1u : 0u);
    } else {
        s.xcd = x;
        s.chunk_log = (uint32_t)p.xcd_remap;
        s.end = p.xcd_tiles[x];
    }
    return s;
}

TTC_HD uint32_t tile_of(const TileSeq& s, uint32_t q)
{
    if (s.chunk_log == 0) return s.base + q;
    return ((s.xcd + 8u * (q >> s.chunk_log)) << s.chunk_log) + (q & ((1u << s.chunk_log) - 1u));
}

// tile id -> element offsets of the box origin in A and in B
struct TileBase { int64_t a, b; };
// what one wavefront works out for the others about a tile (two of these sit at the start of LDS)
// (per walk: the tile's limits in the walk's digits, packed for the bounds test, and whether the walk has to
// test its positions in this tile, so that the other wavefronts read all of it instead of deriving it again)
struct alignas(16) SideShare { int32_t lim[kBoxDims]; uint32_t t01, t23, dynamic, pad; };
struct alignas(16) TileShare { int64_t a, b; SideShare sa, sb; };
constexpr int kTileShareBytes = 2 * (int)sizeof(TileShare);
// after them: one spare slot of 16 bytes per lane of a wavefront, where lanes outside a tile park what they loaded
constexpr int kSpareBytes = 64 * 16;
constexpr int kTablesOff = kTileShareBytes + kSpareBytes;

TTC_HD TileBase tile_base(const KernelParams& p, uint32_t tile)
{
    TileBase t;
    t.a = 0; t.b = 0;
    // straight-line over all kMaxDim entries: unused ones hold neutral values (one tile, stride 0), and code
    // without branches lets the compiler fetch every parameter in one batch instead of index by index
#pragma unroll
    for (int k = 0; k < kMaxDim; ++k) {
        const int64_t origin = (int64_t)fdigit(tile, p.tile_below[k], p.tile_cnt[k]) * p.tile[k];
        t.a += origin * p.stride_a[k];
        t.b += origin * p.stride_b[k];
    }
    return t;
}

// How much of the box lies inside the tensor along each slot.  whole: nothing is cut off.
struct TileLim { int32_t lim[kBoxDims]; bool whole; };

TTC_HD TileLim tile_lim(const KernelParams& p, uint32_t tile)
{
    TileLim t;
    t.whole = true;
#pragma unroll
    for (int j = 0; j < kBoxDims; ++j) {            // unused slots: extent 1, size 1, one tile
        const Slot& sl = p.slot[j];
        const int64_t origin = (int64_t)fdigit(tile, sl.tile_below, sl.tile_cnt) * sl.tile;
        const int64_t left = sl.size - origin;
        t.lim[j] = (int32_t)(left < (int64_t)sl.tile ? left : (int64_t)sl.tile);
        t.whole = t.whole && (t.lim[j] == sl.tile);
    }
    return t;
}

// The same limits in the flat units of one walk's digits, and packed for the bounds test.
//
// The test "coordinate of the lane + coordinate of the sub-box < limit" runs on all four digits
// at once, 16 bits per digit: with g = 0x8000 a guard bit per field,
//     x = (g + limit - 1)  -  position  -  lane        (field by field; no field can borrow from its
//                                                      neighbour because extents stay below 32000)
// keeps its guard bit exactly where the element lies inside the limit.
constexpr uint32_t kGuard = 0x80008000u;
struct SideLim { int32_t lim[kBoxDims]; uint32_t t01, t23; };

TTC_HD SideLim side_lim(const Side& s, const TileLim& t)
{
    SideLim r;
#pragma unroll
    for (int j = 0; j < kBoxDims; ++j) r.lim[j] = t.lim[j] * s.d[j].slot_mul;
    r.t01 = (kGuard + (uint32_t)(r.lim[0] - 1)) + ((uint32_t)(r.lim[1] - 1) << 16);
    r.t23 = (kGuard + (uint32_t)(r.lim[2] - 1)) + ((uint32_t)(r.lim[3] - 1) << 16);
    return r;
}

// ---- micro-tile kernel -----------------------------------------------------------------------
// Where a tile lies and how much of it is inside the tensor along its two indices.  A remainder tile that holds
// less than one vector along an index is moved back along it until it holds one (the elements it shares with its
// neighbour are then written twice, with the same value), so lim_a and lim_b are at least vec.
// a, b: element offsets in A and B of everything but the tile's two indices, plus (a) the first column's place in A's
// run and (b) the first row's place in B's run; col0, row0: the tile's first column and row (where a column lies in
// B and a row in A follows from those, see micro_col_b / micro_row_a).
// own_a, own_b: the first column and row that are this tile's own (not 0 where the tile was moved back over its neighbour).
struct MicroTile { int64_t a, b; uint32_t col0, row0, lim_a, lim_b, own_a, own_b; };

// Tile id -> what the tile contributes to the offsets in A and B, and its coordinates along the column and row index.
struct TilePlace { int64_t a, b; uint32_t col, row; };

TTC_HD TilePlace tile_place(const MicroArgs& p, uint32_t tile)
{
    // mixed radix in tile order; straight-line over all kMaxDim places (unused ones hold one tile and no step).
    // The steps leave out what depends on the column in B and on the row in A.
    TilePlace t = {0, 0, 0, 0};
    uint32_t rest = tile;
#pragma unroll
    for (int i = 0; i < kMaxDim; ++i) {
        const uint32_t next = fdiv(rest, p.cnt[i]);
        const uint32_t d = rest - next * p.cnt[i].div;
        rest = next;
        t.a += (int64_t)d * p.step_a[i];
        t.b += (int64_t)d * p.step_b[i];
        if (i == p.col_pos) t.col = d;
        if (i == p.row_pos) t.row = d;
    }
    return t;
}

TTC_HD MicroTile micro_tile(const MicroArgs& p, uint32_t tile)
{
    const MicroParams& m = p.micro;
    const TilePlace t = tile_place(p, tile);
    const uint32_t da = t.col, db = t.row;
    const int64_t oa = (int64_t)da * m.ta, ob = (int64_t)db * m.tb;
    int64_t lim_a = m.size_a0 - oa < (int64_t)m.ta ? m.size_a0 - oa : (int64_t)m.ta;
    int64_t lim_b = m.size_p0 - ob < (int64_t)m.tb ? m.size_p0 - ob : (int64_t)m.tb;
    const int64_t back_a = lim_a < m.vec ? m.vec - lim_a : 0, back_b = lim_b < m.vec ? m.vec - lim_b : 0;
    MicroTile r;
    r.a = t.a - back_a;
    r.b = t.b - back_b;
    r.col0 = (uint32_t)(oa - back_a);
    r.row0 = (uint32_t)(ob - back_b);
    r.own_a = (uint32_t)back_a;
    r.own_b = (uint32_t)back_b;
    r.lim_a = (uint32_t)(lim_a + back_a);
    r.lim_b = (uint32_t)(lim_b + back_b);
    return r;
}

// Element offset in B of column x (of the whole tensor), and in A of row y.
TTC_HD int64_t micro_col_b(const MicroParams& m, uint32_t x)
{
    const uint32_t out = fdiv(x, m.col_in_div);
    return (int64_t)(x - out * m.col_in_div.div) * m.col_b_in + (int64_t)out * m.col_b_out;
}

TTC_HD int64_t micro_row_a(const MicroParams& m, uint32_t y)
{
    const uint32_t out = fdiv(y, m.row_in_div);
    return (int64_t)(y - out * m.row_in_div.div) * m.row_a_in + (int64_t)out * m.row_a_out;
}

// Where the vector (or block side) that nominally starts at x really starts in a tile holding lim (at least vec)
// elements along that index: the last one is moved back so that it ends with the tile.  Both phases apply the same
// rule, so the LDS slot of lane (row, lane_a) holds the same columns for its writer and its readers.
TTC_HD uint32_t micro_back(uint32_t x, uint32_t lim, uint32_t vec) { return x + vec > lim ? lim - vec : x; }

// The 16-byte LDS slot of row `row` of the tile, column group `lane_c`.
TTC_HD uint32_t micro_slot(const MicroParams& m, uint32_t row, uint32_t lane_c)
{
    return row * (uint32_t)m.pitch + (lane_c ^ ((row >> m.vec_log) & m.swizzle));
}

// Load walk: vector k of lane `tid` (vectors are numbered row by row, so consecutive lanes load consecutive
// vectors of a row).  row runs along A's index p0 (B's stride-1 index), col along A's index 0; chunk is the
// 16-byte slot of the LDS tile the vector is parked in.  valid: the vector is one of the tile's.
struct MicroLoad { uint32_t row, col, chunk; bool valid; };

TTC_HD MicroLoad micro_load(const MicroParams& m, uint32_t threads, uint32_t tid, uint32_t k)
{
    const uint32_t g = tid + k * threads;
    MicroLoad r;
    r.row = fdiv(g, m.la_div);
    const uint32_t lane_a = g - r.row * (uint32_t)m.la;
    r.col = lane_a << m.vec_log;
    r.chunk = micro_slot(m, r.row, lane_a);
    r.valid = r.row < (uint32_t)m.tb;
    return r;
}

// Store walk: block b of lane `tid` (blocks are numbered along B's stride-1 index first): vec rows x vec columns
// nominally starting at (row, col).  Row r of the tile, column group lane_c, sits in LDS slot micro_slot(m, r, lane_c).
struct MicroBlock { uint32_t row, col, lane_c; bool valid; };

TTC_HD MicroBlock micro_block(const MicroParams& m, uint32_t threads, uint32_t tid, uint32_t b)
{
    const uint32_t h = tid + b * threads;
    MicroBlock r;
    r.lane_c = fdiv(h, m.lb_div);
    const uint32_t lane_r = h - r.lane_c * (uint32_t)m.lb;
    r.row = lane_r << m.vec_log;
    r.col = r.lane_c << m.vec_log;
    r.valid = r.lane_c < (uint32_t)m.la;
    return r;
}

// ---- line kernel -----------------------------------------------------------------------------
// A tile holds m.ta columns.  Along the rows it is cut where lines of B end: with `phase` = the place inside its line
// of row 0 of a column (in elements, 0 unless m.skewed), tile number g writes rows g * tb - phase ... (g + 1) * tb -
// phase of that column, as far as they exist.  Skewed, it needs rows from line - 1 before g * tb on and writes one
// line less than LDS holds rows for (tb = (lines - 1) * line); else tb = lines * line.  row0 is the row of LDS row 0.
struct LineTile { int64_t a, b; uint32_t col0; int32_t row0, cols, first; };

TTC_HD LineTile line_tile(const MicroArgs& p, const LineShape& s, uint32_t tile)
{
    const MicroParams& m = p.micro;
    const TilePlace t = tile_place(p, tile);
    LineTile r;
    r.col0 = t.col * (uint32_t)m.ta;
    r.row0 = (int32_t)(t.row * (uint32_t)m.tb) - (m.skewed ? s.line : 0);
    r.a = t.a;                                                       // the first column included
    r.b = t.b - (int64_t)t.row * m.tb;                               // row 0 of the tensor
    const int64_t left = m.size_a0 - (int64_t)r.col0;
    r.cols = (int32_t)(left < (int64_t)m.ta ? left : (int64_t)m.ta);
    r.first = r.row0 < 0 ? s.line : 0;                               // LDS rows before this one are not needed
    return r;
}

// Load `k` of lane `tid`: LDS row, the column the vector nominally starts at, the one it really starts at (moved back to
// end with the tensor; negative if the tile holds fewer columns than a vector: it then starts in the tile before),
// and the row of the tensor (clamped into it: rows outside are loaded from its edge and never stored).
struct LineLoad { int32_t lds_row, col, start; uint32_t row; bool needed; };

TTC_HD LineLoad line_load(const MicroParams& m, const LineShape& s, const LineTile& t, uint32_t tid, int k)
{
    LineLoad r;
    r.lds_row = (int32_t)tid / s.lanes + k * s.pass;
    r.col = (int32_t)tid % s.lanes * s.va;
    r.start = r.col < t.cols - s.va ? r.col : t.cols - s.va;
    const int32_t y = t.row0 + r.lds_row, last = (int32_t)m.size_p0 - 1;
    r.row = (uint32_t)(y < 0 ? 0 : (y > last ? last : y));
    // uniform over the workgroup: whole passes may lie before the first or behind the last row that is needed
    r.needed = (k + 1) * s.pass > t.first && t.row0 + k * s.pass <= last;
    return r;
}

// Stores: lane `tid` keeps column line_column(tid, g) of the tile, g = 0 ... cols / side - 1, and writes 16 bytes of every
// groups-th of its lines: rows y ... y + vb - 1 with y = line_row() + i * groups * line, i = 0 ... lines / groups - 1,
// taken from LDS rows y - row0 on.  The last line of a skewed tile is not the tile's (line_last()).
TTC_HD int32_t line_column(const LineShape& s, uint32_t tid, int g) { return (int32_t)(tid >> 3) % s.side + g * s.side; }
TTC_HD int32_t line_group(const LineShape& s, uint32_t tid) { return (int32_t)(tid >> 3) / s.side; }

TTC_HD int32_t line_row(const MicroParams& m, const LineShape& s, const LineTile& t, int32_t phase, uint32_t tid)
{
    return t.row0 + (m.skewed ? s.line - phase : 0) + line_group(s, tid) * s.line + (int32_t)(tid & 7u) * s.vb;
}

TTC_HD bool line_last(const MicroParams& m, const LineShape& s, uint32_t tid, int i)
{
    return m.skewed && line_group(s, tid) + i * s.groups == s.lines - 1;
}

// ---- block kernel ------------------------------------------------------------------------------
// a, b: element offsets of the tile in A and in B; run_a, run_b: elements of its runs that exist; lim_row, lim_out: how far
// the cut digit of a row's, of an out's place goes.
struct BlockTile { int64_t a, b; int32_t run_a, run_b, lim_row, lim_out; };

TTC_HD BlockTile block_tile(const BlockArgs& p, uint32_t tile)
{
    const BlockParams& m = p.block;
    BlockTile t;
    t.a = 0; t.b = 0;
    uint32_t rest = tile, ca = 0, cb = 0;
#pragma unroll
    for (int i = 0; i < kMaxDim; ++i) {
        const uint32_t next = fdiv(rest, p.cnt[i]);
        const uint32_t d = rest - next * p.cnt[i].div;
        rest = next;
        t.a += (int64_t)d * p.step_a[i];
        t.b += (int64_t)d * p.step_b[i];
        if (i == m.pos_a) ca = d;
        if (i == m.pos_b) cb = d;
    }
    const int64_t left_a = m.size_a - (int64_t)ca * m.tile_a, left_b = m.size_b - (int64_t)cb * m.tile_b;
    const int32_t lim_a = left_a < m.tile_a ? (int32_t)left_a : m.tile_a, lim_b = left_b < m.tile_b ? (int32_t)left_b : m.tile_b;
    t.run_a = m.inner_a * lim_a;
    t.run_b = m.inner_b * lim_b;
    t.lim_row = lim_b;
    t.lim_out = lim_a;
    return t;
}

// Vector `g` of the tile in A's order: where it starts in A (relative to the tile) and in LDS.  start: its place in the run,
// moved back to end with the run (negative, that is inside the tile before, if the run holds less than a vector).
// ok: it is one of the tile's; if not, the tile's first vector is loaded in its place.
struct BlockLoad { int64_t a; int32_t lds, col, start; bool ok; };

TTC_HD BlockLoad block_load(const BlockParams& m, const BlockTile& t, uint32_t g, int32_t vec)
{
    BlockLoad r;
    const uint32_t row = fdiv(g, m.va_div);
    const uint32_t r1 = fdiv(row, m.row_div), r0 = row - r1 * m.row_div.div;
    r.col = (int32_t)(g - row * m.va_div.div) * vec;
    r.ok = row < (uint32_t)m.rows && r.col < t.run_a && (int32_t)(m.cut_row == 0 ? r0 : m.cut_row == 1 ? r1 : 0u) < t.lim_row;
    r.start = r.ok ? r.col : 0;
    if (r.start + vec > t.run_a) r.start = t.run_a - vec;
    r.a = (r.ok ? (int64_t)r0 * m.row_step[0] + (int64_t)r1 * m.row_step[1] : 0) + r.start;
    r.lds = (int32_t)row * m.pitch + r.start;
    return r;
}

// Vector `h` of the tile in B's order: where it starts in B (relative to the tile), its first element's place in LDS, that
// element's places along the first two indices of B's run, and how many of its elements are the tile's (0: none; fewer than
// a vector at the end of a run).  from: where the whole vector starts in B that B is read with before an update.
struct BlockStore { int64_t b, from; int32_t lds, x0, x1, count; };

TTC_HD BlockStore block_store(const BlockParams& m, const BlockTile& t, uint32_t h, int32_t vec)
{
    BlockStore r;
    const uint32_t out = fdiv(h, m.vb_div);
    const uint32_t o1 = fdiv(out, m.out_div), o0 = out - o1 * m.out_div.div;
    const int32_t x = (int32_t)(h - out * m.vb_div.div) * vec;
    const bool ok = out < (uint32_t)m.outs && x < t.run_b && (int32_t)(m.cut_out == 0 ? o0 : m.cut_out == 1 ? o1 : 0u) < t.lim_out;
    r.count = !ok ? 0 : t.run_b - x < vec ? t.run_b - x : vec;
    const uint32_t q0 = fdiv((uint32_t)x, m.x_div[0]), q1 = fdiv(q0, m.x_div[1]);
    r.x0 = x - (int32_t)(q0 * m.x_div[0].div);
    r.x1 = (int32_t)(q0 - q1 * m.x_div[1].div);
    r.lds = r.x0 * m.x_lds[0] + r.x1 * m.x_lds[1] + (int32_t)q1 * m.x_lds[2] + (int32_t)o0 * m.out_lds[0] + (int32_t)o1 * m.out_lds[1];
    const int64_t place = ok ? (int64_t)o0 * m.out_step[0] + (int64_t)o1 * m.out_step[1] : 0;
    r.b = place + x;
    r.from = place + (!ok || x + vec > t.run_b ? (ok ? t.run_b - vec : t.run_b < vec ? t.run_b - vec : 0) : x);
    if (!ok) r.lds = 0;
    return r;
}

// The next element of a vector that runs across B's indices: its place in LDS and along the first two.
TTC_HD void block_next(const BlockParams& m, int32_t* lds, int32_t* x0, int32_t* x1)
{
    *lds += m.x_lds[0];
    if (++*x0 < (int32_t)m.x_div[0].div) return;
    *x0 = 0;
    *lds += m.x_lds[1] - (int32_t)m.x_div[0].div * m.x_lds[0];
    if (++*x1 < (int32_t)m.x_div[1].div) return;
    *x1 = 0;
    *lds += m.x_lds[2] - (int32_t)m.x_div[1].div * m.x_lds[1];
}

// The line kernel's arguments, packed.
constexpr int small_line_words(bool merged) { return merged ? 18 : 12; }
constexpr bool small_line_fits(bool merged, int epilogue, bool is_complex) { return small_line_words(merged) + 2 * small_scalars(epilogue, is_complex) <= 20; }

// Which packed kernel a launch needs: tiles as they come, one range per XCD, or any dealing and A streamed.
constexpr int kDealNone = 0, kDealRanges = 1, kDealAll = 2;
inline int small_line_dealing(const MicroArgs& a) { return a.nt_a != 0 || a.xcd_remap > 1 ? kDealAll : a.xcd_remap == 1 ? kDealRanges : kDealNone; }

// Whether there is a packed kernel for tiles dealt in any way (kDealAll); `passes`: vectors of A a lane loads.
// Updates of many tiles whose lanes load eight vectors of A keep the whole arguments there: that kernel waits for arguments between
// its loads, the packed one issues eight of A and up to eight of B in a row, and is slower by 3 % (fp32, 18 problems; 40 x 1064 x 344
// (1,0,2) in chunks of 32 36.8 -> 40.3 us), 2 % (fp64, 10), 1 % (complex64, 8; complex128, 6) and 10 and 7 % (complex128 -> complex64, fp64 -> fp32, 3 and
// 2).  With four vectors it is 1-3 % faster, and 5 % and more where there are fewer tiles.
// With one range per XCD (kDealRanges) it is the packed kernel that is faster with eight vectors as well: 0.94-0.96 of the time from 700 tiles
// on (130 problems of every type, in rotation; one pair 0.95, new tensors 0.96), 0.99 below (23, from 0.77 to 1.18); 40 x 1064 x 344 29.8 us,
// whole arguments 30.7 (and 31.0 in chunks of 32).
constexpr bool small_line_deals(int epilogue, int passes) { return epilogue != TTC_EPI_AXPBY || passes < 8; }

// 0: the arguments go unpacked; 1: packed; 2: packed with merged indices.
inline int small_line(const MicroArgs& a, int epilogue, bool is_complex, int passes)
{
    const bool merged = a.micro.merged_a || a.micro.merged_b;
    if (small_line_dealing(a) == kDealAll && !small_line_deals(epilogue, passes)) return 0;
    if (!small_line_fits(merged, epilogue, is_complex) || a.micro.size_a0 > INT32_MAX || a.micro.size_p0 > INT32_MAX) return 0;
    int used = 0;                                              // places in the tile order that hold more than one tile, or a column or row
    for (int i = 0; i < kMaxDim; ++i) {
        if (a.cnt[i].div >= (1u << 27)) return 0;
        if (a.cnt[i].div > 1 || i == a.col_pos || i == a.row_pos) ++used;
        if (i != a.col_pos && i != a.row_pos && (a.step_a[i] > INT32_MAX || a.step_b[i] > INT32_MAX)) return 0;
    }
    const MicroParams& m = a.micro;
    if (used > 3 || m.col_in_div.div >= (1u << 27) || m.row_in_div.div >= (1u << 27) || m.col_b_in > INT32_MAX || m.col_b_out > INT32_MAX ||
        m.row_a_in > INT32_MAX || m.row_a_out > INT32_MAX) return 0;
    return merged ? 2 : 1;
}

inline SmallArgs small_line_pack(const MicroArgs& a, int epilogue, bool is_complex)
{
    SmallArgs s = {};
    const MicroParams& m = a.micro;
    const bool merged = m.merged_a || m.merged_b;
    uint32_t col = 0, row = 0, other = 3;
    int place[3] = {-1, -1, -1}, n = 0;
    for (int i = 0; i < kMaxDim; ++i) {
        if (!(a.cnt[i].div > 1 || i == a.col_pos || i == a.row_pos)) continue;
        if (i == a.col_pos) col = (uint32_t)n; else if (i == a.row_pos) row = (uint32_t)n; else other = (uint32_t)n;
        place[n++] = i;
    }
    s.w[0] = col | row << 2 | other << 4 | (uint32_t)m.skewed << 6 | (uint32_t)a.nt_b << 7 | (uint32_t)a.nt_a << 8 | (uint32_t)a.xcd_remap << 9;
    for (int k = 0; k < 2; ++k) {
        s.w[1 + 2 * k] = a.cnt[place[k]].mul;
        s.w[2 + 2 * k] = a.cnt[place[k]].div | a.cnt[place[k]].shift << 27;
    }
    if (other < 3) { s.w[5] = (uint32_t)a.step_a[place[other]]; s.w[6] = (uint32_t)a.step_b[place[other]]; }
    s.w[7] = (uint32_t)m.size_a0; s.w[8] = (uint32_t)m.size_p0;
    s.w[9] = (uint32_t)m.col_b_in; s.w[10] = (uint32_t)m.row_a_in;
    if (merged) {
        s.w[11] = m.merged_a ? m.col_in_div.mul : 0u;          // not merged: quotient 0
        s.w[12] = m.merged_a ? m.col_in_div.div | m.col_in_div.shift << 27 : 31u << 27;
        s.w[13] = (uint32_t)m.col_b_out;
        s.w[14] = m.merged_b ? m.row_in_div.mul : 0u;
        s.w[15] = m.merged_b ? m.row_in_div.div | m.row_in_div.shift << 27 : 31u << 27;
        s.w[16] = (uint32_t)m.row_a_out;
    }
    s.w[merged ? 17 : 11] = a.num_tiles;
    int at = small_line_words(merged);
    const int count = small_scalars(epilogue, is_complex), each = is_complex ? 2 : 1;
    for (int k = 0; k < count; ++k) {
        const double v = k < each ? a.alpha[k] : a.beta[k - each];
        uint64_t bits;
        __builtin_memcpy(&bits, &v, 8);
        s.w[at++] = (uint32_t)bits;
        s.w[at++] = (uint32_t)(bits >> 32);
    }
    return s;
}

// How its tiles are dealt: one workgroup each, as the row kernel's chunks.
struct SmallDeal { int32_t xcd_remap; uint32_t blocks; };
TTC_HD SmallDeal small_line_deal(const SmallArgs& s, bool merged) { return SmallDeal{(int32_t)(s.w[0] >> 9 & 15u), s.w[merged ? 17 : 11]}; }

// The tile of workgroup `wg` with one range per XCD (num_tiles or more: none).
TTC_HD uint32_t small_line_range(const SmallDeal& d, uint32_t wg) { return range_place((d.blocks + 7u) / 8u, wg); }

// The arguments as the line kernel's index code reads them (the fields of the dealing are not set).
// DEALT: what a small problem does without: tiles dealt to the XCDs in chunks, A streamed.
template <int MODE, bool COMPLEX, bool MERGED, bool DEALT>
TTC_HD MicroArgs small_line_unpack(const SmallArgs& s, int cols, const LineShape& shape)
{
    MicroArgs a;
    a.xcd_remap = 0; a.debug_stop = 0;
    a.nt_a = DEALT ? (int32_t)(s.w[0] >> 8 & 1u) : 0;
    a.nt_b = (int32_t)(s.w[0] >> 7 & 1u);
    a.col_pos = (int32_t)(s.w[0] & 3u);
    a.row_pos = (int32_t)(s.w[0] >> 2 & 3u);
    const int32_t other = (int32_t)(s.w[0] >> 4 & 3u);
    MicroParams& m = a.micro;
    m.skewed = (int32_t)(s.w[0] >> 6 & 1u);
    m.lines = shape.lines;
    m.ta = cols;
    m.tb = (shape.lines - m.skewed) * shape.line;
    m.size_a0 = (int64_t)s.w[7]; m.size_p0 = (int64_t)s.w[8];
#pragma unroll
    for (int i = 0; i < kMaxDim; ++i) {
        FastDiv f = {0u, i == 2 ? 31u : 0u, i == 2 ? 0u : 1u};
        if (i < 2) { f.mul = s.w[1 + 2 * i]; f.div = s.w[2 + 2 * i] & 0x7ffffffu; f.shift = s.w[2 + 2 * i] >> 27; }
        a.cnt[i] = f;
        a.step_a[i] = i > 2 ? 0 : i == a.col_pos ? (int64_t)cols : i == other ? (int64_t)s.w[5] : 0;
        a.step_b[i] = i > 2 ? 0 : i == a.row_pos ? (int64_t)m.tb : i == other ? (int64_t)s.w[6] : 0;
    }
    m.col_b_in = (int64_t)s.w[9]; m.row_a_in = (int64_t)s.w[10];
    if (MERGED) {
        m.col_in_div = FastDiv{s.w[11], s.w[12] >> 27, s.w[12] & 0x7ffffffu};
        m.col_b_out = (int64_t)s.w[13];
        m.row_in_div = FastDiv{s.w[14], s.w[15] >> 27, s.w[15] & 0x7ffffffu};
        m.row_a_out = (int64_t)s.w[16];
    } else {
        m.col_in_div = m.row_in_div = FastDiv{0u, 31u, 0u};
        m.col_b_out = m.row_a_out = 0;
    }
    a.alpha[0] = a.alpha[1] = a.beta[0] = a.beta[1] = 0.0;
    constexpr int kCount = small_scalars(MODE, COMPLEX), kEach = COMPLEX ? 2 : 1, kAt = small_line_words(MERGED);
#pragma unroll
    for (int k = 0; k < kCount; ++k) {
        const uint64_t bits = (uint64_t)s.w[kAt + 2 * k] | (uint64_t)s.w[kAt + 2 * k + 1] << 32;
        double v;
        __builtin_memcpy(&v, &bits, 8);
        if (k < kEach) a.alpha[k] = v; else a.beta[k - kEach] = v;
    }
    return a;
}

// ---- lane entry ------------------------------------------------------------------------------
// Offsets are in BYTES.  A walk has three element sizes: of the tensor it follows (g), of B in
// the direct kernel (g2), and of the LDS tile, which holds elements of A (l).
struct Scales { int32_t g, g2, l; };

struct LaneState {
    int64_t g;                 // byte offset into the tensor the walk follows
    int64_t g2;                // direct kernel: byte offset into B
    int32_t l;                 // byte offset into the LDS tile
    uint32_t c01, c23;         // flat coordinate along each digit, in elements, 16 bits per digit
    bool    active;
};

template <bool DIRECT>
TTC_HD LaneState lane_setup(const Side& s, uint32_t lane, const Scales& scale)
{
    LaneState L;
    L.g = 0; L.g2 = 0; L.l = 0;
    L.active = lane < (uint32_t)s.lanes;
    uint32_t cs[kBoxDims];
#pragma unroll
    for (int j = 0; j < kBoxDims; ++j) {            // empty digits: one lane step, stride 0
        const Digit& d = s.d[j];
        const int32_t c = (int32_t)fdigit(lane, d.lane_below, d.lane_cnt) * d.lane_mul;
        cs[j] = (uint32_t)c;
        L.g += (int64_t)c * d.gstride;
        if (DIRECT) L.g2 += (int64_t)c * d.g2stride;
        else L.l += c * d.lstride;
    }
    L.g *= scale.g; L.g2 *= scale.g2; L.l *= scale.l;
    L.c01 = cs[0] | (cs[1] << 16);
    L.c23 = cs[2] | (cs[3] << 16);
    return L;
}

// ---- position entry --------------------------------------------------------------------------
// 16 + 8 bytes per sub-box position: offsets of the sub-box origin, and its coordinates inside
// the tile packed 16 bits per digit (flat extents of a digit stay below 32000).
struct alignas(16) PosEntry {
    int64_t g;                 // byte offset in the tensor the walk follows
    int64_t l_or_g2;           // staged kernel: LDS byte offset; direct kernel: byte offset in B
};
struct alignas(8) PosCoord { uint32_t c01, c23; };

template <bool DIRECT>
TTC_HD void make_position(const Side& s, uint32_t it, const Scales& scale, PosEntry* e, PosCoord* c)
{
    int64_t g = 0, x = 0;
    uint32_t pc[kBoxDims];
#pragma unroll
    for (int i = 0; i < kBoxDims; ++i) {            // digits with one position contribute 0
        const Digit& d = s.d[i];
        const uint32_t q = fdigit(it, d.iter_below, d.iter_cnt) * (uint32_t)d.lane;
        pc[i] = q;
        g += (int64_t)q * d.gstride;
        x += (int64_t)q * (DIRECT ? d.g2stride : (int64_t)d.lstride);
    }
    e->g = g * scale.g;
    e->l_or_g2 = x * (DIRECT ? scale.g2 : scale.l);
    c->c01 = pc[0] | (pc[1] << 16);
    c->c23 = pc[2] | (pc[3] << 16);
}

// Limits of one tile as one lane sees them: the lane's own coordinates already taken off.
struct LaneLim { uint32_t x01, x23; };

TTC_HD LaneLim lane_lim(const LaneState& L, const SideLim& lim)
{
    LaneLim r;
    r.x01 = lim.t01 - L.c01;
    r.x23 = lim.t23 - L.c23;
    return r;
}

// does this lane's element (the first one of its vector) at this sub-box position lie inside the
// box and the tensor?
TTC_HD bool lane_valid(const LaneLim& x, const PosCoord& pc)
{
    return (((x.x01 - pc.c01) & (x.x23 - pc.c23)) & kGuard) == kGuard;
}

// Vectors of V elements along the walk's first digit whose extent is not a multiple of V: by how many
// elements must the lane's vector move back so that it ends inside the limit?  0 .. V-1, or -1 if not
// even its first element lies inside (the limit is at least V, so a moved vector never starts before 0).
template <int V>
TTC_HD int lane_back(const LaneLim& x, const PosCoord& pc, int vec_slot)
{
    const uint32_t a = x.x01 - pc.c01, b = x.x23 - pc.c23;
    if (((a & b) & kGuard) != kGuard) return -1;
    const uint32_t w = (vec_slot & 2) ? b : a;
    const uint32_t f = (vec_slot & 1) ? (w >> 16) : w;
    const int left = (int)(f & 0x7fffu) + 1;          // the field holds limit - 1 - coordinate
    return left < V ? V - left : 0;
}

// Which sub-box positions a wavefront takes, and where their table entries sit.  Wavefront w of
// nwave takes positions w, w + nwave, w + 2 nwave, ...; the tables are stored wave-major, the
// k-th position of wavefront w at index w * chunk + k, so that a wavefront reads consecutive
// entries.
TTC_HD uint32_t wave_positions(const Side& s, uint32_t wave)
{
    return (uint32_t)s.chunk - (wave >= (uint32_t)s.chunk_rem ? 1u : 0u);
}

// How a group of positions treats the bounds: no test at all, whole vectors tested, or vectors
// that are moved back where the run ends inside them.
enum { kWalkFull = 0, kWalkMasked = 1, kWalkPartial = 2 };

// U positions at a time: stage1 for all U (issue the loads), then stage2 for all U (consume
// them), so that U memory instructions are in flight per wavefront.  stage(u, entry, back, ok):
// u = slot 0..U-1, back = elements the lane's vector is moved back by (0 unless the walk is partial),
// ok = the lane's element lies inside the tile.  Stages run for every lane: a lane that is not ok must
// do something harmless (load the tile's first vector, write to a spare LDS slot, skip a global store),
// so that no load sits inside divergent control flow, where it would be waited for on the spot.
template <int U, int V, int MODE, class Stage1, class Stage2>
TTC_HD void walk_group(const LaneLim& x, int vec_slot, const PosEntry* e_ptr, const PosCoord* c_ptr,
                       Stage1&& stage1, Stage2&& stage2)
{
    PosEntry e[U];
    int back[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        e[u] = e_ptr[u];
        if (MODE == kWalkFull) back[u] = 0;
        else if (MODE == kWalkMasked) back[u] = lane_valid(x, c_ptr[u]) ? 0 : -1;
        else back[u] = lane_back<V>(x, c_ptr[u], vec_slot);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        stage1(u, e[u], (MODE == kWalkPartial && back[u] > 0) ? back[u] : 0, MODE == kWalkFull ? true : back[u] >= 0);
#pragma unroll
    for (int u = 0; u < U; ++u)
        stage2(u, e[u], (MODE == kWalkPartial && back[u] > 0) ? back[u] : 0, MODE == kWalkFull ? true : back[u] >= 0);
}

// What a walk has to test per lane in one tile.  Digits with a single sub-box position are
// tested once per tile (lane_ok); only digits that step AND are cut by the tensor's edge or
// overhang the tile need the test at every position (dynamic, wave-uniform).
struct WalkMask { bool lane_ok; bool dynamic; };

// bit j: digit j has a single sub-box position (the same for every tile)
TTC_HD uint32_t single_digits(const Side& s)
{
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < kBoxDims; ++j) m |= (s.d[j].iters == 1 ? 1u : 0u) << j;
    return m;
}

// the wave-uniform half: does the walk have to test its positions in this tile?
TTC_HD bool walk_dynamic(const Side& s, const SideLim& lim)
{
    bool dynamic = (s.partial != 0);
#pragma unroll
    for (int j = 0; j < kBoxDims; ++j) {
        const Digit& d = s.d[j];
        if (d.iters != 1) dynamic = dynamic | (lim.lim[j] != d.tile) | (d.ragged != 0);
    }
    return dynamic;
}

// the per-lane half: is the lane inside the tile along the digits that do not step?
TTC_HD bool lane_inside(uint32_t single, const LaneState& L, const SideLim& lim)
{
    bool ok = L.active;
#pragma unroll
    for (int j = 0; j < kBoxDims; ++j) {
        const int32_t c = (int32_t)(((j & 2) ? L.c23 : L.c01) >> ((j & 1) ? 16 : 0)) & 0xffff;
        if ((single >> j) & 1u) ok = ok & (c < lim.lim[j]);
    }
    return ok;
}

// one walk's part of the shared tile record
TTC_HD SideShare make_side_share(const Side& s, const TileLim& tl)
{
    const SideLim sl = side_lim(s, tl);
    SideShare v;
    v.lim[0] = sl.lim[0]; v.lim[1] = sl.lim[1]; v.lim[2] = sl.lim[2]; v.lim[3] = sl.lim[3];
    v.t01 = sl.t01; v.t23 = sl.t23;
    v.dynamic = walk_dynamic(s, sl) ? 1u : 0u;
    v.pad = 0;
    return v;
}

TTC_HD WalkMask walk_mask(const Side& s, const LaneState& L, const SideLim& lim)
{
    WalkMask m;
    m.lane_ok = lane_inside(single_digits(s), L, lim);
    m.dynamic = walk_dynamic(s, lim);
    return m;
}

template <int U, int V, int MODE, class Stage1, class Stage2>
TTC_HD void walk_mode(const LaneLim& x, int vec_slot, const PosEntry* my, const PosCoord* myc, uint32_t cnt,
                      Stage1&& stage1, Stage2&& stage2)
{
    uint32_t k = 0;
    for (; k + U <= cnt; k += U) walk_group<U, V, MODE>(x, vec_slot, my + k, myc + k, stage1, stage2);
    for (; k < cnt; ++k) walk_group<1, V, MODE>(x, vec_slot, my + k, myc + k, stage1, stage2);
}

// Drive one wavefront through its share of a walk with V elements per lane and access.
template <int U, int V, class Stage1, class Stage2>
TTC_HD void walk(const Side& s, const LaneState& L, const SideLim& lim, const WalkMask& m, const PosEntry* tab,
                 const PosCoord* tabc, uint32_t wave, Stage1&& stage1, Stage2&& stage2)
{
    if (!m.lane_ok) return;
    const uint32_t cnt = wave_positions(s, wave);
    const PosEntry* my = tab + wave * (uint32_t)s.chunk;
    const PosCoord* myc = tabc + wave * (uint32_t)s.chunk;
    const LaneLim x = lane_lim(L, lim);
    if (!m.dynamic) walk_mode<U, V, kWalkFull>(x, 0, my, myc, cnt, stage1, stage2);
    else if (V == 1 || !s.partial) walk_mode<U, V, kWalkMasked>(x, 0, my, myc, cnt, stage1, stage2);
    else walk_mode<U, V, kWalkPartial>(x, s.vec_slot, my, myc, cnt, stage1, stage2);
}

// Fill the two tables of one walk (all threads of the workgroup take part).
template <bool DIRECT>
TTC_HD void build_tables(const Side& s, uint32_t nwave, uint32_t thread, uint32_t nthreads, const Scales& scale,
                         PosEntry* tab, PosCoord* tabc)
{
    const uint32_t total = nwave * (uint32_t)s.chunk;
    for (uint32_t j = thread; j < total; j += nthreads) {
        const uint32_t w = fdiv(j, s.chunk_div);
        const uint32_t it = w + (j - w * (uint32_t)s.chunk) * nwave;
        if (it < (uint32_t)s.n_iter) make_position<DIRECT>(s, it, scale, &tab[j], &tabc[j]);
    }
}

}  // namespace ttc
