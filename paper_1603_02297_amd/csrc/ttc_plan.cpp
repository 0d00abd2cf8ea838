// Host planner: validation, size-1 removal, index fusion (paper Section 3, stage (1)),
// case split (Section 3.1), candidate enumeration with a heuristic ranking (Sections 3.2,
// 3.3 and the candidate queue of Section 3).  Pure host C++: no device is touched here.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <type_traits>
#include <unordered_map>

#include "ttc_internal.h"
#include "ttc_walk.h"

namespace ttc {

static thread_local int g_last_status = TTC_OK;
void set_last_status(int status) { g_last_status = status; }

// TTC_VERBOSE=1 in the environment: one line on stderr per plan, per completed candidate list and per search
bool verbose()
{
    static const bool on = [] { const char* e = std::getenv("TTC_VERBOSE"); return e && *e && *e != '0'; }();
    return on;
}

FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f;
    if (d <= 1) { f.div = 1; f.shift = 0; f.mul = 1; return f; }      // (x * 1 >> 32) + x >> 0 = x for x < 2^32
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    f.div = d;
    f.shift = s;
    f.mul = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << s) - d)) / d + 1);
    return f;
}

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline int64_t round_up(int64_t a, int64_t m) { return ceil_div(a, m) * m; }

// ---------------------------------------------------------------------------------
// Normalisation: element kinds, strides from the leading dimensions, drop extents of 1, merge
// indices that stay adjacent and in order and are contiguous in both tensors.
// ---------------------------------------------------------------------------------
static int kind_bytes(int kind) { return kind == kKindF32 ? 4 : (kind == kKindC128 ? 16 : 8); }

static bool dtype_kinds(int dtype, int* ka, int* kb)
{
    switch (dtype) {
    case TTC_F32:      *ka = kKindF32;  *kb = kKindF32;  return true;
    case TTC_F64:      *ka = kKindF64;  *kb = kKindF64;  return true;
    case TTC_C64:      *ka = kKindC64;  *kb = kKindC64;  return true;
    case TTC_C128:     *ka = kKindC128; *kb = kKindC128; return true;
    case TTC_F32_F64:  *ka = kKindF32;  *kb = kKindF64;  return true;
    case TTC_F64_F32:  *ka = kKindF64;  *kb = kKindF32;  return true;
    case TTC_C64_C128: *ka = kKindC64;  *kb = kKindC128; return true;
    case TTC_C128_C64: *ka = kKindC128; *kb = kKindC64;  return true;
    default: return false;
    }
}

static int normalise(int dtype, int ndim, const int64_t* sizes, const int* perm, const int64_t* lda,
                     const int64_t* ldb, const void* alpha, const void* beta, Problem* P)
{
    if (!sizes || !perm) return TTC_ERR_NULL_POINTER;
    int ka, kb;
    if (!dtype_kinds(dtype, &ka, &kb)) return TTC_ERR_UNSUPPORTED_DTYPE;
    if (ndim < 1 || ndim > kMaxDim) return TTC_ERR_INVALID_VALUE;
    bool seen[kMaxDim] = {false};
    for (int j = 0; j < ndim; ++j) {
        if (perm[j] < 0 || perm[j] >= ndim || seen[perm[j]]) return TTC_ERR_INVALID_PERM;
        seen[perm[j]] = true;
    }
    int64_t total = 1, alloc_a = 1, alloc_b = 1;
    for (int k = 0; k < ndim; ++k)
        if (sizes[k] < 1) return TTC_ERR_INVALID_VALUE;
    for (int k = 0; k < ndim; ++k) {
        const int64_t la = lda ? lda[k] : sizes[k], lb = ldb ? ldb[k] : sizes[perm[k]];
        if (la < sizes[k] || lb < sizes[perm[k]]) return TTC_ERR_INVALID_VALUE;
        if (total > (INT64_MAX / 16) / sizes[k]) return TTC_ERR_OVERFLOW;
        if (alloc_a > (INT64_MAX / 16) / la || alloc_b > (INT64_MAX / 16) / lb) return TTC_ERR_OVERFLOW;
        total *= sizes[k];
        alloc_a *= la;
        alloc_b *= lb;
    }
    // strides in the caller's index space (paper Table 1, --lda / --ldb: the tensor may be a part of
    // a larger one whose extents are the leading dimensions)
    int64_t sa[kMaxDim], sb[kMaxDim];          // sa by index of A; sb by index (position) of B
    sa[0] = 1; sb[0] = 1;
    for (int k = 1; k < ndim; ++k) {
        sa[k] = sa[k - 1] * (lda ? lda[k - 1] : sizes[k - 1]);
        sb[k] = sb[k - 1] * (ldb ? ldb[k - 1] : sizes[perm[k - 1]]);
    }
    int64_t span_a = 1, span_b = 1;
    for (int k = 0; k < ndim; ++k) {
        span_a += (sizes[k] - 1) * sa[k];
        span_b += (sizes[perm[k]] - 1) * sb[k];
    }

    // 1. drop size-1 extents (they contribute offset 0 on both sides)
    int newidx[kMaxDim], m = 0;
    int64_t s1[kMaxDim], sa1[kMaxDim];
    for (int k = 0; k < ndim; ++k) {
        newidx[k] = -1;
        if (sizes[k] > 1) { newidx[k] = m; s1[m] = sizes[k]; sa1[m] = sa[k]; ++m; }
    }
    int p1[kMaxDim], mp = 0;
    int64_t sb1[kMaxDim];                      // by kept position of B
    for (int j = 0; j < ndim; ++j)
        if (sizes[perm[j]] > 1) { p1[mp] = newidx[perm[j]]; sb1[mp] = sb[j]; ++mp; }
    if (m == 0) { m = 1; s1[0] = 1; p1[0] = 0; sa1[0] = 1; sb1[0] = 1; }

    // 2. merge: B positions j, j+1 holding A indices a, a+1 form one index if the pair is contiguous in
    //    both tensors: ld(i_{m+1}) = size(i_m) * ld(i_m), the condition of the footnote in Section 3.
    int group_start[kMaxDim], group_len[kMaxDim], group_pos[kMaxDim], ng = 0;     // groups in B order
    for (int j = 0; j < m;) {
        int len = 1;
        while (j + len < m && p1[j + len] == p1[j + len - 1] + 1 &&
               sa1[p1[j + len]] == sa1[p1[j + len - 1]] * s1[p1[j + len - 1]] &&
               sb1[j + len] == sb1[j + len - 1] * s1[p1[j + len - 1]]) ++len;
        group_start[ng] = p1[j];
        group_len[ng] = len;
        group_pos[ng] = j;
        ++ng;
        j += len;
    }
    // fused index of A = rank of the group's first A index
    int rank_of_group[kMaxDim];
    for (int g = 0; g < ng; ++g) {
        int r = 0;
        for (int h = 0; h < ng; ++h) if (group_start[h] < group_start[g]) ++r;
        rank_of_group[g] = r;
    }
    P->dtype = dtype;
    P->kind_a = ka; P->kind_b = kb;
    P->eb_a = kind_bytes(ka); P->eb_b = kind_bytes(kb);
    P->ndim = ng;
    P->elements = total;
    P->span_a = span_a; P->span_b = span_b;
    for (int k = 0; k < kMaxDim; ++k) { P->size[k] = 0; P->perm[k] = 0; P->stride_a[k] = 0; P->stride_b[k] = 0; }
    for (int g = 0; g < ng; ++g) {
        int64_t sz = 1;
        for (int i = 0; i < group_len[g]; ++i) sz *= s1[group_start[g] + i];
        const int r = rank_of_group[g];
        P->size[r] = sz;
        P->perm[g] = r;
        P->stride_a[r] = sa1[group_start[g]];
        P->stride_b[r] = sb1[group_pos[g]];
    }

    // scalars (defaults of the paper's Table 1: alpha = 1, beta = 0), in the precision the arithmetic
    // runs in: the data type's, or double for mixed precision
    const bool wide = (ka == kKindF64 || ka == kKindC128 || kb == kKindF64 || kb == kKindC128);
    const bool cplx = (ka == kKindC64 || ka == kKindC128);
    auto read = [&](const void* src, double* dst) {
        if (wide) { dst[0] = ((const double*)src)[0]; dst[1] = cplx ? ((const double*)src)[1] : 0.0; }
        else      { dst[0] = ((const float*)src)[0];  dst[1] = cplx ? ((const float*)src)[1] : 0.0; }
    };
    P->alpha[0] = 1.0; P->alpha[1] = 0.0; P->beta[0] = 0.0; P->beta[1] = 0.0;
    if (alpha) read(alpha, P->alpha);
    if (beta) read(beta, P->beta);
    const bool beta0 = (P->beta[0] == 0.0 && P->beta[1] == 0.0);
    const bool alpha1 = (P->alpha[0] == 1.0 && P->alpha[1] == 0.0);
    P->epilogue = beta0 ? (alpha1 ? TTC_EPI_COPY : TTC_EPI_SCALE) : TTC_EPI_AXPBY;
    return TTC_OK;
}

// ---------------------------------------------------------------------------------
// Tile (box) construction
// ---------------------------------------------------------------------------------

// Extent near `want` along an index of size s, a multiple of mult (s % mult == 0).
// Divisors of s are preferred (no remainder tiles: the second rule of the paper's blocking
// heuristic, Section 3.2); otherwise the index is cut into equal pieces.
static int pick_extent(int64_t s, int64_t want, int mult, int style = 0, int nice = 1)
{
    if (want < mult) want = mult;
    if (want >= s) return (int)s;
    if (style == 1) {
        // cache-line friendly: a multiple of `nice` elements (64 bytes) even if that leaves a remainder tile
        const int64_t unit = std::max<int64_t>(nice, mult);
        for (int64_t t = round_up(want, unit); t <= std::min<int64_t>(s, 2 * want); t += unit)
            if (s % t == 0) return (int)t;
        const int64_t t = round_up(want, unit);
        if (t < s) return (int)t;
    }
    for (int64_t t = round_up(want, mult); t <= std::min<int64_t>(s, 2 * want); t += mult)
        if (s % t == 0) return (int)t;
    for (int64_t t = (want / mult) * mult; t >= mult && 4 * t >= 3 * want; t -= mult)
        if (s % t == 0) return (int)t;
    const int64_t parts = ceil_div(s, want);
    int64_t t = round_up(ceil_div(s, parts), mult);
    return (int)std::min<int64_t>(t, s);
}

// Leading indices of one tensor, in that tensor's order, until the contiguous run they
// span reaches `target` elements.  All but the last are taken whole.
static void build_group(const Problem& P, const int* order, int eb, int64_t target, int vec, int max_dims, int* t,
                        int style = 0)
{
    for (int k = 0; k < kMaxDim; ++k) t[k] = 1;
    int64_t run = 1;
    for (int i = 0; i < P.ndim && i < max_dims; ++i) {
        const int k = order[i];
        const int64_t need = ceil_div(target, run);
        if (need <= 1) break;
        const int mult = (i == 0) ? vec : 1;
        int ext;
        if (P.size[k] <= need + need / 2) ext = (int)P.size[k];
        else ext = pick_extent(P.size[k], need, mult, style, std::max(1, 64 / eb));
        t[k] = ext;
        run *= ext;
        if (ext < P.size[k]) break;
    }
}

// ---------------------------------------------------------------------------------
// Walks: how each side sees the box
// ---------------------------------------------------------------------------------
struct DigitSpec {
    int first_dim;      // innermost index of the chain (the stride-1 end)
    int outer_dim;      // outermost index of the chain: the only one the tensor's edge can cut
    int tile;           // flat extent inside the box
    int inner;          // product of the box extents of the chain's inner indices
    int lane;           // flat extent of the lane sub-box (filled by choose_lanes)
};
struct WalkSpec { int nd; DigitSpec d[kBoxDims]; };

// Digits of one walk in the walk's own order.  With `merge`, the leading indices that lie whole
// inside the box fuse with their successor into one flat digit (tile-level index fusion); an
// index whose bit is set in `no_tail` may not be appended to a chain.
static bool build_walk(const Problem& P, const int* order, const int64_t* stride, const int* t, bool merge,
                       unsigned no_tail, WalkSpec* w)
{
    w->nd = 0;
    bool leading = true;
    for (int i = 0; i < P.ndim; ++i) {
        const int k = order[i];
        if (t[k] <= 1) { leading = false; continue; }
        if (merge && leading && w->nd == 1) {
            DigitSpec& d = w->d[0];
            const int prev = d.outer_dim;
            if (i > 0 && order[i - 1] == prev && t[prev] == P.size[prev] && !(no_tail & (1u << k)) &&
                stride[k] == stride[prev] * P.size[prev] && (int64_t)d.tile * t[k] <= kMaxDigitExtent) {
                d.inner = d.tile;
                d.tile *= t[k];
                d.outer_dim = k;
                continue;
            }
        }
        if (w->nd >= 1) leading = false;
        if (w->nd == kBoxDims) return false;
        DigitSpec& d = w->d[w->nd++];
        d.first_dim = d.outer_dim = k;
        d.tile = t[k];
        d.inner = 1;
        d.lane = 1;
        if (t[k] > kMaxDigitExtent) return false;
    }
    return w->nd >= 1;
}

// Largest vector width (elements) for a walk: vectors lie along the first digit and must not
// straddle its end, in whole tiles and in the tiles the tensor's edge cuts.
// A limit above 16 also admits vectors that do not divide the run (*partial = true): the last vector of every
// run is then moved back to end with the run and overlaps its neighbour.  That needs every run, also the
// shortened ones of the tiles the tensor's edge cuts, to hold at least one vector, and pays only for runs of
// several vectors.
static int walk_vec(const Problem& P, const WalkSpec& w, const int* t, int limit, int eb, bool unit_stride,
                    bool* partial)
{
    *partial = false;
    if (!unit_stride) return 1;      // a dropped size-1 index with a padded leading dimension: no stride-1 index
    const int widest = std::max(1, std::min(std::min(limit, 16), std::max(1, 16 / eb)));
    const DigitSpec& d = w.d[0];
    const int64_t rest = P.size[d.outer_dim] % t[d.outer_dim];
    int v = widest;
    while (v > 1 && (d.tile % v != 0 || (rest * d.inner) % v != 0)) v /= 2;
    v = std::max(v, 1);
    if (limit > 16 && v < widest && d.tile >= 4 * widest && (rest == 0 || rest * d.inner >= widest)) {
        *partial = true;
        return widest;
    }
    return v;
}

// Lane mapping: which sub-box of the tile one wavefront instruction covers.
static void choose_lanes(const Problem& P, WalkSpec* w, int vec, int eb, int* n_iter_out, int* lanes_out)
{
    int best_lane[kBoxDims] = {1, 1, 1, 1};
    int64_t best_cost = INT64_MAX;
    int best_iter = 1, best_lanes = 1;
    const int t0 = w->d[0].tile;
    std::vector<int> opts;
    const int cap = (int)std::min<int64_t>(round_up(t0, vec), kWave * vec);
    for (int l = vec; l <= cap; l += vec)
        if (t0 % l == 0 || l == cap) opts.push_back(l);
    if (opts.empty()) opts.push_back(vec);
    for (int l0 : opts) {
        int lane[kBoxDims] = {1, 1, 1, 1};
        lane[0] = l0;
        int lanes = l0 / vec;
        int rem = kWave / std::max(lanes, 1);
        int64_t iters = ceil_div(t0, l0);
        bool ragged = (t0 % l0) != 0;
        for (int i = 1; i < w->nd; ++i) {
            const int ti = w->d[i].tile;
            int l = 1;
            if (rem > 1) {
                l = std::min(rem, ti);
                // prefer a divisor of the extent if it costs at most one position in four
                int div = l;
                while (div > 1 && ti % div != 0) --div;
                if (4 * ceil_div(ti, div) <= 5 * ceil_div(ti, l)) l = div;
                else l = (int)ceil_div(ti, ceil_div(ti, l));      // same count, less ragged
                rem /= l;
                lanes *= l;
            }
            lane[i] = l;
            iters *= ceil_div(ti, l);
            if (ti % l != 0) ragged = true;
        }
        // short segments along the stride-1 index cost coalescing: ask for a 128-byte line unless the tile is
        // shorter; an overhanging sub-box makes every position test its bounds
        const bool short_seg = (l0 < t0) && (l0 * eb < 128);
        const int64_t cost = iters * (short_seg ? 8 : 4) * (ragged ? 5 : 4);
        if (cost < best_cost || (cost == best_cost && l0 > best_lane[0])) {
            best_cost = cost;
            for (int i = 0; i < kBoxDims; ++i) best_lane[i] = lane[i];
            best_iter = (int)std::min<int64_t>(iters, INT32_MAX);
            best_lanes = lanes;
        }
    }
    for (int i = 0; i < w->nd; ++i) w->d[i].lane = best_lane[i];
    *n_iter_out = best_iter;
    *lanes_out = best_lanes;
}

// Lay one walk out for the kernel: digits go to the slot of their outermost index.
static bool fill_side(const Problem& P, const WalkSpec& w, int vec, const int* slot_of_dim,
                      const int* lds_stride, bool follows_b, Side* s)
{
    std::memset(s, 0, sizeof(*s));
    s->vec = vec;
    s->exact = 1;
    for (int j = 0; j < kBoxDims; ++j) {
        Digit& d = s->d[j];
        d.tile = 1; d.lane = 1; d.iters = 1; d.lane_mul = 1; d.slot_mul = 1;
        d.lane_below = d.lane_cnt = d.iter_below = d.iter_cnt = make_fastdiv(1);
    }
    uint32_t lane_below = 1, iter_below = 1;
    int64_t n_iter = 1;
    for (int i = 0; i < w.nd; ++i) {
        const DigitSpec& ds = w.d[i];
        const int j = slot_of_dim[ds.outer_dim];
        if (j < 0 || j >= kBoxDims) return false;
        Digit& d = s->d[j];
        const int mul = (i == 0) ? vec : 1;
        if (ds.lane % mul != 0) return false;
        const int cnt = ds.lane / mul;
        const int its = (int)ceil_div(ds.tile, ds.lane);
        d.tile = ds.tile;
        d.lane = ds.lane;
        d.iters = its;
        d.lane_mul = mul;
        d.slot_mul = ds.inner;
        d.lane_below = make_fastdiv(lane_below);
        d.lane_cnt = make_fastdiv((uint32_t)cnt);
        d.iter_below = make_fastdiv(iter_below);
        d.iter_cnt = make_fastdiv((uint32_t)its);
        d.gstride = follows_b ? P.stride_b[ds.first_dim] : P.stride_a[ds.first_dim];
        d.g2stride = P.stride_b[ds.first_dim];
        d.lstride = lds_stride ? lds_stride[ds.first_dim] : 0;
        d.ragged = (ds.tile % ds.lane != 0) ? 1 : 0;
        if (d.ragged) s->exact = 0;
        lane_below *= (uint32_t)cnt;
        iter_below *= (uint32_t)its;
        n_iter *= its;
        if (n_iter > kMaxIters || lane_below > (uint32_t)kWave) return false;
    }
    s->lanes = (int)lane_below;
    s->n_iter = (int)n_iter;
    s->vec_lds_stride = lds_stride ? lds_stride[w.d[0].first_dim] : 0;
    s->vec_slot = slot_of_dim[w.d[0].outer_dim];
    return true;
}

// ---------------------------------------------------------------------------------
// LDS layout.  Indices that a walk merged into one flat digit must be affine in LDS as well:
// stride(next) = extent(cur) * stride(cur).  These links form chains; the chain holding A's
// stride-1 index comes first, the others follow, each chain head on a small pad chosen by
// simulating which banks the 64 lanes of one LDS instruction touch.
// ---------------------------------------------------------------------------------
// Lane coordinates of one walk, per digit slot, in flat elements: what the bank simulation needs besides the
// LDS strides (computed once per layout search; the strides change from one trial layout to the next).
struct LaneCoords { int lanes, vec; int c[kWave][kBoxDims]; };

static void lane_coords(const Side& s, LaneCoords* out)
{
    out->lanes = s.lanes;
    out->vec = s.vec;
    for (int lane = 0; lane < s.lanes; ++lane)
        for (int i = 0; i < kBoxDims; ++i) {
            const Digit& d = s.d[i];
            out->c[lane][i] = (int)((lane / d.lane_below.div) % d.lane_cnt.div) * d.lane_mul;
        }
}

// Worst number of distinct addresses that the lanes of one LDS instruction send to one bank, relative to the
// unavoidable number (ceil(addresses / banks)), for 32 and for 64 banks; the two are added (2 = conflict-free).
static int bank_multiplicity(const LaneCoords& lc, const int* lstride /* per slot */, int vec_stride, int words)
{
    int worst32 = 1, worst64 = 1;
    int64_t base[kWave], addr[kWave];
    for (int lane = 0; lane < lc.lanes; ++lane) {
        int64_t a = 0;
        for (int i = 0; i < kBoxDims; ++i) a += (int64_t)lc.c[lane][i] * lstride[i];
        base[lane] = a;
    }
    for (int j = 0; j < lc.vec; ++j) {
        int n = lc.lanes;
        for (int lane = 0; lane < n; ++lane) addr[lane] = (base[lane] + (int64_t)j * vec_stride) * words;
        // distinct word addresses per bank (same address = broadcast, no conflict)
        std::sort(addr, addr + n);
        n = (int)(std::unique(addr, addr + n) - addr);
        int cnt32[32] = {0}, cnt64[64] = {0};
        for (int i = 0; i < n; ++i)
            for (int w = 0; w < words; ++w) {
                const uint64_t x = (uint64_t)(addr[i] + w);
                cnt32[x & 31u]++;
                cnt64[x & 63u]++;
            }
        int mx32 = 0, mx64 = 0;
        for (int b = 0; b < 32; ++b) mx32 = std::max(mx32, cnt32[b]);
        for (int b = 0; b < 64; ++b) mx64 = std::max(mx64, cnt64[b]);
        const int ideal32 = std::max(1, (int)ceil_div((int64_t)n * words, 32));
        const int ideal64 = std::max(1, (int)ceil_div((int64_t)n * words, 64));
        worst32 = std::max(worst32, (int)ceil_div(mx32, ideal32));
        worst64 = std::max(worst64, (int)ceil_div(mx64, ideal64));
    }
    return worst32 + worst64;
}

// The same for the line kernel's tile, one instruction of a wavefront each: writes of 8 bytes (4-byte elements) or 16
// along the rows, reads of one element, eight lanes with rows 16 bytes of B apart times eight neighbouring columns.
static void line_conflicts(const LineShape& S, int eb_a, int* writes, int* reads)
{
    const int unit = eb_a == 16 ? 1 : 2;            // elements per write; rows are whole numbers of them
    LaneCoords w, r;
    w.lanes = r.lanes = kWave;
    w.vec = r.vec = 1;
    std::memset(w.c, 0, sizeof(w.c));
    std::memset(r.c, 0, sizeof(r.c));
    for (int lane = 0; lane < kWave; ++lane) {
        w.c[lane][0] = lane / S.lanes;              // row
        w.c[lane][1] = lane % S.lanes * S.va / unit;
        r.c[lane][0] = (lane & 7) * S.vb;
        r.c[lane][1] = (lane >> 3) % S.side;
    }
    const int write_stride[kBoxDims] = {S.pitch / unit, 1, 0, 0}, read_stride[kBoxDims] = {S.pitch, 1, 0, 0};
    *writes = bank_multiplicity(w, write_stride, 0, unit * eb_a / 4);
    *reads = bank_multiplicity(r, read_stride, 0, eb_a / 4);
}

struct LdsLayout { int stride[kMaxDim]; int elems; int conflict_a, conflict_b; };

static LdsLayout choose_lds_layout(const Problem& P, const int* t, const int* slot_of_dim,
                                   const WalkSpec& wa, const WalkSpec& wb, int va, int vb,
                                   const int* next_in_chain /* by dim, -1 = chain end */,
                                   const bool* is_head /* by dim */)
{
    LdsLayout best;
    best.elems = 0; best.conflict_a = best.conflict_b = 1 << 20;
    // chain heads in layout order: the chain of index 0 first, then by index
    int heads[kMaxDim], nh = 0;
    for (int k = 0; k < P.ndim; ++k) if (t[k] > 1 && is_head[k]) heads[nh++] = k;
    // TTC_LDS_PAD=0 in the environment lays every tile out without pads (the ablation of the studies)
    const char* pad_env = std::getenv("TTC_LDS_PAD");
    const bool pads = !(pad_env && pad_env[0] == '0');
    const int npad = pads ? std::max(0, std::min(nh - 1, 3)) : 0;
    // the walks' lane mappings do not depend on the LDS strides: lay the sides out once
    Side sa, sb;
    const int zero[kMaxDim] = {0, 0, 0, 0, 0, 0};
    if (!fill_side(P, wa, va, slot_of_dim, zero, false, &sa)) return best;
    if (!fill_side(P, wb, vb, slot_of_dim, zero, true, &sb)) return best;
    LaneCoords la, lb;
    lane_coords(sa, &la);
    lane_coords(sb, &lb);
    int dim_of_slot_a[kBoxDims] = {-1, -1, -1, -1}, dim_of_slot_b[kBoxDims] = {-1, -1, -1, -1};
    for (int i = 0; i < wa.nd; ++i) dim_of_slot_a[slot_of_dim[wa.d[i].outer_dim]] = wa.d[i].first_dim;
    for (int i = 0; i < wb.nd; ++i) dim_of_slot_b[slot_of_dim[wb.d[i].outer_dim]] = wb.d[i].first_dim;
    const int words = P.eb_a / 4;               // the LDS tile holds elements of A
    int64_t best_cost = INT64_MAX;
    const int combos = 1 << (2 * npad);
    for (int c = 0; c < combos; ++c) {
        LdsLayout L;
        for (int k = 0; k < kMaxDim; ++k) L.stride[k] = 0;
        int64_t run = 1;
        for (int h = 0; h < nh; ++h) {
            if (h >= 1 && h - 1 < npad) run += (c >> (2 * (h - 1))) & 3;
            for (int k = heads[h]; k >= 0; k = next_in_chain[k]) {
                L.stride[k] = (int)run;
                run *= t[k];
            }
        }
        L.elems = (int)run;
        if ((int64_t)L.elems * P.eb_a > kMaxLdsBytes) continue;
        int ls_a[kBoxDims], ls_b[kBoxDims];
        for (int j = 0; j < kBoxDims; ++j) {
            ls_a[j] = dim_of_slot_a[j] >= 0 ? L.stride[dim_of_slot_a[j]] : 0;
            ls_b[j] = dim_of_slot_b[j] >= 0 ? L.stride[dim_of_slot_b[j]] : 0;
        }
        L.conflict_a = bank_multiplicity(la, ls_a, L.stride[wa.d[0].first_dim], words);
        L.conflict_b = bank_multiplicity(lb, ls_b, L.stride[wb.d[0].first_dim], words);
        const int64_t cost = ((int64_t)(L.conflict_a + L.conflict_b) << 24) + L.elems;
        if (cost < best_cost) { best_cost = cost; best = L; }
        if (L.conflict_a + L.conflict_b == 4) break;             // conflict-free under both bank counts
    }
    return best;
}

// ---------------------------------------------------------------------------------
// Candidate assembly
// ---------------------------------------------------------------------------------
// The LDS layout depends on the box and the walks only, not on the launch shape or the tile
// order: candidates that differ only in those share one layout search.
struct LayoutKey {
    int t[kMaxDim]; int vec_limit; bool merge_a, merge_b;
    bool operator==(const LayoutKey& o) const
    {
        for (int k = 0; k < kMaxDim; ++k) if (t[k] != o.t[k]) return false;
        return vec_limit == o.vec_limit && merge_a == o.merge_a && merge_b == o.merge_b;
    }
};
struct LayoutCache { std::vector<std::pair<LayoutKey, LdsLayout>> items; };

static bool make_candidate(const Problem& P, const int* t_in, int vec_limit, bool direct, int threads,
                           int wg_per_cu, const int* tile_order, int xcd_remap, Candidate* out,
                           bool merge_a = true, bool merge_b = true, LayoutCache* cache = nullptr, int nbuf = 2)
{
    Candidate C;
    std::memset(&C, 0, sizeof(C));
    int t[kMaxDim];
    for (int k = 0; k < kMaxDim; ++k) t[k] = (k < P.ndim) ? t_in[k] : 1;
    int order_a[kMaxDim], order_b[kMaxDim];
    for (int k = 0; k < kMaxDim; ++k) { order_a[k] = k; order_b[k] = (k < P.ndim) ? P.perm[k] : k; }

    KernelParams& kp = C.kp;
    kp.n = P.ndim;
    int64_t ntiles = 1;
    for (int k = 0; k < kMaxDim; ++k) {
        kp.stride_a[k] = (k < P.ndim) ? P.stride_a[k] : 0;
        kp.stride_b[k] = (k < P.ndim) ? P.stride_b[k] : 0;
        kp.tile[k] = t[k];
        kp.tile_below[k] = make_fastdiv(1);
        kp.tile_cnt[k] = make_fastdiv(1);
    }
    for (int i = 0; i < P.ndim; ++i) {
        const int k = tile_order[i];
        const int64_t cnt = ceil_div(P.size[k], t[k]);
        if (ntiles > INT32_MAX / 2 || cnt > INT32_MAX / 2) return false;
        kp.tile_below[k] = make_fastdiv((uint32_t)ntiles);
        kp.tile_cnt[k] = make_fastdiv((uint32_t)cnt);
        ntiles *= cnt;
        if (ntiles > INT32_MAX / 2) return false;
        C.tile_order[i] = k;
    }
    kp.num_tiles = (uint32_t)ntiles;
    kp.tiles_per_xcd = kp.num_tiles / 8;
    kp.tiles_rem_xcd = kp.num_tiles % 8;
    if (!set_tile_mapping(&kp, xcd_remap)) return false;
    kp.alpha[0] = P.alpha[0]; kp.alpha[1] = P.alpha[1];
    kp.beta[0] = P.beta[0];   kp.beta[1] = P.beta[1];

    // slots: the indices the box spans, in A order
    int slot_of_dim[kMaxDim];
    int nslots = 0;
    for (int k = 0; k < kMaxDim; ++k) {
        slot_of_dim[k] = -1;
        if (k < P.ndim && t[k] > 1) {
            if (nslots == kBoxDims) return false;
            Slot& sl = kp.slot[nslots];
            sl.tile = t[k];
            sl.size = P.size[k];
            sl.tile_below = kp.tile_below[k];
            sl.tile_cnt = kp.tile_cnt[k];
            slot_of_dim[k] = nslots++;
        }
    }
    for (int j = nslots; j < kBoxDims; ++j) {
        kp.slot[j].tile = 1; kp.slot[j].size = 1;
        kp.slot[j].tile_below = kp.slot[j].tile_cnt = make_fastdiv(1);
    }
    kp.nslots = nslots;
    if (nslots == 0) {                      // a one-element tensor: give the walks one trivial digit
        kp.nslots = 1;
        slot_of_dim[0] = 0;
    }

    for (int k = 0; k < kMaxDim; ++k) { C.tile[k] = t[k]; C.lds_stride[k] = 0; }
    WalkSpec wa, wb;
    auto trivial_walk = [&](WalkSpec* w) {
        w->nd = 1;
        w->d[0].first_dim = w->d[0].outer_dim = 0;
        w->d[0].tile = 1; w->d[0].inner = 1; w->d[0].lane = 1;
    };
    if (direct) {
        if (nslots == 0) trivial_walk(&wa);
        else if (!build_walk(P, order_a, P.stride_a, t, false, 0u, &wa)) return false;
        const int eb_max = std::max(P.eb_a, P.eb_b);        // every lane stores what it loaded: one width for both
        // overlapping vectors would read elements of B that a neighbour may already have updated
        if (P.epilogue == TTC_EPI_AXPBY) vec_limit = std::min(vec_limit, 16);
        bool part = false;
        const int v = (nslots == 0) ? 1 : walk_vec(P, wa, t, vec_limit, eb_max,
                                                  P.stride_a[wa.d[0].first_dim] == 1 && P.stride_b[wa.d[0].first_dim] == 1,
                                                  &part);
        int n_iter, lanes;
        choose_lanes(P, &wa, v, eb_max, &n_iter, &lanes);
        if (!fill_side(P, wa, v, slot_of_dim, nullptr, false, &kp.a)) return false;
        kp.a.partial = part ? 1 : 0;
        kp.b = kp.a;
        wb = wa;
        C.kernel_class = TTC_KERNEL_DIRECT;
        C.lds_bytes = (int)round_up(24 * (int64_t)kp.a.n_iter, 16);
        kp.lds_data_off = C.lds_bytes;
        kp.lds_tile_elems = 0;
        kp.lds_buffers = 1;
        C.lds_conflict_a = C.lds_conflict_b = 0;
    } else {
        if (nslots == 0) return false;
        if (!build_walk(P, order_a, P.stride_a, t, merge_a, 0u, &wa)) return false;
        // LDS chains from A's merged digit; B may chain its own leading indices only where that
        // does not give an index a second predecessor or a second successor
        int next_in_chain[kMaxDim];
        bool is_head[kMaxDim];
        unsigned in_a_chain = 0, a_nonlast = 0;
        for (int k = 0; k < kMaxDim; ++k) { next_in_chain[k] = -1; is_head[k] = true; }
        if (wa.d[0].first_dim != wa.d[0].outer_dim)
            for (int k = wa.d[0].first_dim; k <= wa.d[0].outer_dim; ++k) {      // A's chain is consecutive indices
                in_a_chain |= 1u << k;
                if (k < wa.d[0].outer_dim) { next_in_chain[k] = k + 1; is_head[k + 1] = false; a_nonlast |= 1u << k; }
            }
        const bool b_may_merge = merge_b && !(a_nonlast & (1u << order_b[0]));
        if (!build_walk(P, order_b, P.stride_b, t, b_may_merge, in_a_chain, &wb)) return false;
        if (wb.d[0].first_dim != wb.d[0].outer_dim) {
            int prev = -1;
            for (int i = 0; i < P.ndim; ++i) {
                const int k = order_b[i];
                if (prev >= 0) { next_in_chain[prev] = k; is_head[k] = false; }
                prev = k;
                if (k == wb.d[0].outer_dim) break;
            }
        }
        bool part_a = false, part_b = false;
        const int va = walk_vec(P, wa, t, vec_limit, P.eb_a, P.stride_a[wa.d[0].first_dim] == 1, &part_a);
        const int vb = walk_vec(P, wb, t, P.epilogue == TTC_EPI_AXPBY ? std::min(vec_limit, 16) : vec_limit, P.eb_b,
                                P.stride_b[wb.d[0].first_dim] == 1, &part_b);     // see the direct case
        int ia, la_, ib, lb_;
        choose_lanes(P, &wa, va, P.eb_a, &ia, &la_);
        choose_lanes(P, &wb, vb, P.eb_b, &ib, &lb_);
        LdsLayout L;
        bool cached = false;
        LayoutKey key;
        for (int k = 0; k < kMaxDim; ++k) key.t[k] = t[k];
        key.vec_limit = vec_limit; key.merge_a = merge_a; key.merge_b = merge_b;
        if (cache)
            for (const auto& it : cache->items) if (it.first == key) { L = it.second; cached = true; break; }
        if (!cached) {
            L = choose_lds_layout(P, t, slot_of_dim, wa, wb, va, vb, next_in_chain, is_head);
            if (cache) cache->items.emplace_back(key, L);
        }
        if (L.elems == 0) return false;
        for (int k = 0; k < kMaxDim; ++k) C.lds_stride[k] = L.stride[k];
        if (!fill_side(P, wa, va, slot_of_dim, L.stride, false, &kp.a)) return false;
        if (!fill_side(P, wb, vb, slot_of_dim, L.stride, true, &kp.b)) return false;
        kp.a.partial = part_a ? 1 : 0;
        kp.b.partial = part_b ? 1 : 0;
        C.kernel_class = TTC_KERNEL_LDS;
        kp.lds_data_off = (int)round_up(24 * (int64_t)(kp.a.n_iter + kp.b.n_iter), 16);
        kp.lds_tile_elems = (int)round_up(L.elems, std::max(1, 16 / P.eb_a));
        kp.lds_buffers = nbuf;
        C.lds_bytes = kp.lds_data_off + nbuf * kp.lds_tile_elems * P.eb_a;
        if (C.lds_bytes > kMaxLdsBytes) return false;
        C.lds_conflict_a = L.conflict_a;
        C.lds_conflict_b = L.conflict_b;
    }
    C.digits_a = wa.nd;
    C.digits_b = wb.nd;
    for (int i = 0; i < kBoxDims; ++i) {
        C.dtile_a[i] = i < wa.nd ? wa.d[i].tile : 0;  C.dlane_a[i] = i < wa.nd ? wa.d[i].lane : 0;
        C.dtile_b[i] = i < wb.nd ? wb.d[i].tile : 0;  C.dlane_b[i] = i < wb.nd ? wb.d[i].lane : 0;
    }
    C.threads = threads;
    const int nwave = threads / kWave;
    auto set_chunks = [&](Side* sd) {
        sd->chunk = (int)ceil_div(sd->n_iter, nwave);
        sd->chunk_rem = sd->n_iter - (sd->chunk - 1) * nwave;
        sd->chunk_div = make_fastdiv((uint32_t)sd->chunk);
    };
    set_chunks(&kp.a);
    set_chunks(&kp.b);
    const int64_t tab_entries = (int64_t)nwave * (kp.a.chunk + (direct ? 0 : kp.b.chunk));
    const int tab_bytes = (int)round_up(kTablesOff + 24 * tab_entries, 16);
    C.lds_bytes += tab_bytes - kp.lds_data_off;
    kp.lds_data_off = tab_bytes;
    if (C.lds_bytes > kMaxLdsBytes) return false;
    // wg_per_cu <= 0: as many workgroups as a compute unit holds at once (LDS in granules of 1280 bytes, 32
    // wavefronts, 16 workgroups that need a barrier), so that every workgroup is resident from the start and its
    // set-up is paid once per slot instead of once per round
    if (wg_per_cu <= 0) {
        const int by_lds = (int)(kMaxLdsBytes / round_up(std::max(C.lds_bytes, 1), 1280));
        const int by_waves = 32 / nwave;
        wg_per_cu = std::max(1, std::min(std::min(by_lds, by_waves), nwave > 1 ? 16 : 32));
    }
    C.wg_per_cu = wg_per_cu;
    set_grid(&kp, launch_grid(C, 256));
    C.tuned_ms = 0.f;
    *out = C;
    return true;
}

// The micro-tile kernel's candidate: a tile of ta columns x tb rows.  The column index is A's index 0, or A's
// indices 0 and 1 taken as one (merge_a: together they are one contiguous run of A); the row index is B's
// stride-1 index p0, or B's first two indices taken as one (merge_b).  Needs one element type of 4 or 8 bytes on
// both sides, indices contiguous in their tensor, four different indices where both sides merge, both (merged)
// extents at least one 16-byte vector, ta and tb multiples of the vector, a tile of at most 64 KB.  Extents that
// are not multiples of the vector make some elements be moved twice; where B is updated (beta != 0) the kernel
// writes such an element once, from the block that owns it.
static bool make_micro_candidate(const Problem& P, int ta, int tb, int threads, const int* tile_order, bool merge_a, bool merge_b,
                                 Candidate* out)
{
    if (P.ndim < 2 || P.perm[0] == 0 || P.kind_a != P.kind_b || (P.eb_a != 4 && P.eb_a != 8)) return false;
    const int p0 = P.perm[0], vec = 16 / P.eb_a;
    const int a1 = 1, p1 = P.ndim >= 2 ? P.perm[1] : -1;         // the second index of A and of B
    if (P.stride_a[0] != 1 || P.stride_b[p0] != 1) return false;
    if (merge_a && (P.ndim < 3 || a1 == p0 || P.stride_a[a1] != P.size[0] || (merge_b && a1 == p1))) return false;
    if (merge_b && (P.ndim < 3 || p1 == 0 || P.stride_b[p1] != P.size[p0] || (merge_a && p1 == a1))) return false;
    const int64_t cols = merge_a ? P.size[0] * P.size[a1] : P.size[0], rows = merge_b ? P.size[p0] * P.size[p1] : P.size[p0];
    if (cols >= (int64_t(1) << 31) || rows >= (int64_t(1) << 31)) return false;
    if (cols < vec || rows < vec || ta % vec != 0 || tb % vec != 0 || ta < vec || tb < vec) return false;
    const int la = ta / vec, lb = tb / vec;
    const int pitch = (la + 7) / 8 * 8;
    if ((int64_t)tb * pitch * 16 > 64 * 1024) return false;
    const int loads = (int)ceil_div((int64_t)la * tb, threads), blocks = (int)ceil_div((int64_t)la * lb, threads);
    if (blocks > 8) return false;
    Candidate C;
    std::memset(&C, 0, sizeof(C));
    C.kernel_class = TTC_KERNEL_MICRO;
    C.threads = threads;
    C.wg_per_cu = 0;                   // one tile per workgroup
    C.lds_bytes = tb * pitch * 16;
    KernelParams& kp = C.kp;
    kp.n = P.ndim;
    int64_t ntiles = 1;
    // what the tile decode sees: the (merged) column index in the place of index 0, the row index in the place of
    // p0, an index merged into one of them as a single tile that contributes nothing, every other index one
    // element per tile.  The decode adds the column's place in A and the row's place in B (stride 1); where the
    // column lies in B and the row in A depends on more than a stride and is left to the kernel.
    int64_t extent[kMaxDim];
    for (int k = 0; k < kMaxDim; ++k) {
        extent[k] = (k < P.ndim) ? P.size[k] : 1;
        C.tile[k] = 1;
        kp.stride_a[k] = (k < P.ndim) ? P.stride_a[k] : 0;
        kp.stride_b[k] = (k < P.ndim) ? P.stride_b[k] : 0;
        kp.tile_below[k] = kp.tile_cnt[k] = make_fastdiv(1);
    }
    extent[0] = cols; C.tile[0] = ta; kp.stride_a[0] = 1; kp.stride_b[0] = 0;
    extent[p0] = rows; C.tile[p0] = tb; kp.stride_a[p0] = 0; kp.stride_b[p0] = 1;
    if (merge_a) { extent[a1] = 1; kp.stride_a[a1] = kp.stride_b[a1] = 0; }
    if (merge_b) { extent[p1] = 1; kp.stride_a[p1] = kp.stride_b[p1] = 0; }
    for (int k = 0; k < kMaxDim; ++k) kp.tile[k] = C.tile[k];
    uint32_t ordered = 0;                        // the order has to name every index of the problem once
    for (int i = 0; i < P.ndim; ++i) if (tile_order[i] >= 0 && tile_order[i] < P.ndim) ordered |= 1u << tile_order[i];
    if (ordered != (1u << P.ndim) - 1u) return false;
    for (int i = 0; i < P.ndim; ++i) {
        const int k = tile_order[i];
        const int64_t cnt = ceil_div(extent[k], C.tile[k]);
        if (cnt > INT32_MAX / 2 || ntiles > INT32_MAX / 2) return false;
        kp.tile_below[k] = make_fastdiv((uint32_t)ntiles);
        kp.tile_cnt[k] = make_fastdiv((uint32_t)cnt);
        ntiles *= cnt;
        if (ntiles > INT32_MAX / 2) return false;
        C.tile_order[i] = k;
    }
    if (!launchable(ntiles, C.threads)) return false;
    kp.num_tiles = (uint32_t)ntiles;
    kp.tiles_per_xcd = kp.num_tiles / 8;
    kp.tiles_rem_xcd = kp.num_tiles % 8;
    if (!set_tile_mapping(&kp, kDefaultTileMapping)) return false;
    set_grid(&kp, kp.num_tiles);
    kp.alpha[0] = P.alpha[0]; kp.alpha[1] = P.alpha[1];
    kp.beta[0] = P.beta[0];   kp.beta[1] = P.beta[1];
    kp.a.vec = kp.b.vec = vec;
    kp.lds_buffers = 1;
    kp.lds_tile_elems = ta * tb;
    for (int j = 0; j < kBoxDims; ++j) {            // the box kernels' slots, so that shared helpers see neutral values
        kp.slot[j].tile = 1; kp.slot[j].size = 1;
        kp.slot[j].tile_below = kp.slot[j].tile_cnt = make_fastdiv(1);
    }
    MicroParams& m = kp.micro;
    m.ta = ta; m.tb = tb; m.p0 = p0; m.vec = vec;
    m.merged_a = merge_a ? 1 : 0; m.merged_b = merge_b ? 1 : 0;
    m.la = la; m.lb = lb; m.pitch = pitch; m.loads = loads; m.blocks = blocks;
    {   // TTC_LDS_PAD=0 in the environment: no swizzle either (the ablation of the studies)
        const char* pad_env = std::getenv("TTC_LDS_PAD");
        m.swizzle = (pad_env && pad_env[0] == '0') ? 0u : 7u;
    }
    m.la_div = make_fastdiv((uint32_t)la); m.lb_div = make_fastdiv((uint32_t)lb);
    m.vec_log = (vec == 4) ? 2 : 1;
    m.size_a0 = cols; m.size_p0 = rows;
    m.col_in_div = make_fastdiv((uint32_t)P.size[0]);
    m.row_in_div = make_fastdiv((uint32_t)P.size[p0]);
    m.col_b_in = P.stride_b[0];  m.col_b_out = merge_a ? P.stride_b[a1] : 0;
    m.row_a_in = P.stride_a[p0]; m.row_a_out = merge_b ? P.stride_a[p1] : 0;
    // the tile per index of A, as the plan reports it: a merged index takes what the tile spans of it
    if (merge_a) { C.tile[0] = (int)std::min<int64_t>(ta, P.size[0]); C.tile[a1] = (int)std::min<int64_t>(ceil_div(ta, P.size[0]), P.size[a1]); }
    if (merge_b) { C.tile[p0] = (int)std::min<int64_t>(tb, P.size[p0]); C.tile[p1] = (int)std::min<int64_t>(ceil_div(tb, P.size[p0]), P.size[p1]); }
    C.digits_a = C.digits_b = 2;
    C.dtile_a[0] = ta; C.dtile_a[1] = tb; C.dlane_a[0] = std::min(ta, kWave * vec); C.dlane_a[1] = std::max(1, kWave / la);
    C.dtile_b[0] = tb; C.dtile_b[1] = ta; C.dlane_b[0] = std::min(tb, kWave * vec); C.dlane_b[1] = std::max(1, kWave / lb) * vec;
    C.dlane_a[2] = m.merged_a; C.dlane_b[2] = m.merged_b;       // part of what names the configuration
    C.lds_conflict_a = C.lds_conflict_b = 2;       // conflict-free by construction (the value the bank model gives such a layout)
    C.lds_stride[0] = 1;
    C.lds_stride[p0] = pitch * vec;
    *out = C;
    return true;
}

static int default_tile_mapping(const Problem& P, const Candidate& C);

// The line kernel's candidate: `cols` columns by `lines` lines of B per column.  Columns and rows are what the
// micro-tile kernel takes (A's index 0 and B's first index, each possibly merged with the next), for every type pair.
static bool make_line_candidate(const Problem& P, int cols_tile, int lines, const int* tile_order, bool merge_a, bool merge_b, Candidate* out)
{
    if (P.ndim < 2 || P.perm[0] == 0 || !line_shape_ok(cols_tile, lines, P.eb_a, P.eb_b)) return false;
    const LineShape S = line_shape(cols_tile, lines, P.eb_a, P.eb_b);
    const int p0 = P.perm[0], p1 = P.perm[1], a1 = 1;
    if (P.stride_a[0] != 1 || P.stride_b[p0] != 1) return false;
    if (merge_a && (P.ndim < 3 || a1 == p0 || P.stride_a[a1] != P.size[0])) return false;
    if (merge_b && (P.ndim < 3 || p1 == 0 || P.stride_b[p1] != P.size[p0])) return false;
    if (merge_a && merge_b && a1 == p1) return false;
    const int64_t cols = merge_a ? P.size[0] * P.size[a1] : P.size[0], rows = merge_b ? P.size[p0] * P.size[p1] : P.size[p0];
    if (cols >= kLineMaxExtent || rows >= kLineMaxExtent || cols < S.va || rows < S.vb) return false;
    // do all columns of B start at the same place inside a line?
    bool skewed = false;
    for (int k = 0; k < P.ndim; ++k)
        if (k != p0 && !(merge_b && k == p1) && P.stride_b[k] * P.eb_b % kLineBytes != 0) skewed = true;
    const int tb = (lines - (skewed ? 1 : 0)) * S.line;
    Candidate C;
    std::memset(&C, 0, sizeof(C));
    C.kernel_class = kKernelLines;
    C.threads = kLineThreads;
    C.wg_per_cu = 0;                   // one tile per workgroup
    C.lds_bytes = S.lds_bytes;
    KernelParams& kp = C.kp;
    kp.n = P.ndim;
    int64_t extent[kMaxDim];           // as the tile decode sees the indices: see make_micro_candidate
    for (int k = 0; k < kMaxDim; ++k) {
        extent[k] = (k < P.ndim) ? P.size[k] : 1;
        C.tile[k] = 1;
        kp.stride_a[k] = (k < P.ndim) ? P.stride_a[k] : 0;
        kp.stride_b[k] = (k < P.ndim) ? P.stride_b[k] : 0;
        kp.tile_below[k] = kp.tile_cnt[k] = make_fastdiv(1);
    }
    extent[0] = cols; C.tile[0] = cols_tile; kp.stride_a[0] = 1; kp.stride_b[0] = 0;
    extent[p0] = rows + (skewed ? S.line - 1 : 0); C.tile[p0] = tb; kp.stride_a[p0] = 0; kp.stride_b[p0] = 1;
    if (merge_a) { extent[a1] = 1; kp.stride_a[a1] = kp.stride_b[a1] = 0; }
    if (merge_b) { extent[p1] = 1; kp.stride_a[p1] = kp.stride_b[p1] = 0; }
    for (int k = 0; k < kMaxDim; ++k) kp.tile[k] = C.tile[k];
    uint32_t ordered = 0;
    for (int i = 0; i < P.ndim; ++i) if (tile_order[i] >= 0 && tile_order[i] < P.ndim) ordered |= 1u << tile_order[i];
    if (ordered != (1u << P.ndim) - 1u) return false;
    int64_t ntiles = 1;
    for (int i = 0; i < P.ndim; ++i) {
        const int k = tile_order[i];
        const int64_t cnt = ceil_div(extent[k], C.tile[k]);
        if (cnt > INT32_MAX / 2 || ntiles > INT32_MAX / 2) return false;
        kp.tile_below[k] = make_fastdiv((uint32_t)ntiles);
        kp.tile_cnt[k] = make_fastdiv((uint32_t)cnt);
        ntiles *= cnt;
        if (ntiles > INT32_MAX / 2) return false;
        C.tile_order[i] = k;
    }
    if (!launchable(ntiles, C.threads)) return false;
    kp.num_tiles = (uint32_t)ntiles;
    kp.tiles_per_xcd = kp.num_tiles / 8;
    kp.tiles_rem_xcd = kp.num_tiles % 8;
    set_grid(&kp, kp.num_tiles);
    kp.alpha[0] = P.alpha[0]; kp.alpha[1] = P.alpha[1];
    kp.beta[0] = P.beta[0];   kp.beta[1] = P.beta[1];
    kp.a.vec = S.va; kp.b.vec = S.vb;
    kp.lds_buffers = 1;
    kp.lds_tile_elems = S.rows * S.pitch;
    for (int j = 0; j < kBoxDims; ++j) {
        kp.slot[j].tile = 1; kp.slot[j].size = 1;
        kp.slot[j].tile_below = kp.slot[j].tile_cnt = make_fastdiv(1);
    }
    MicroParams& m = kp.micro;
    m.ta = cols_tile; m.tb = tb; m.p0 = p0; m.vec = S.va;
    m.merged_a = merge_a ? 1 : 0; m.merged_b = merge_b ? 1 : 0;
    m.lines = lines; m.skewed = skewed ? 1 : 0;
    m.la_div = m.lb_div = make_fastdiv(1);
    m.size_a0 = cols; m.size_p0 = rows;
    m.col_in_div = make_fastdiv((uint32_t)P.size[0]);
    m.row_in_div = make_fastdiv((uint32_t)P.size[p0]);
    m.col_b_in = P.stride_b[0];  m.col_b_out = merge_a ? P.stride_b[a1] : 0;
    m.row_a_in = P.stride_a[p0]; m.row_a_out = merge_b ? P.stride_a[p1] : 0;
    if (!set_tile_mapping(&kp, default_tile_mapping(P, C))) return false;
    // the tile per index of A, as the plan reports it
    C.tile[0] = (int)std::min<int64_t>(cols_tile, P.size[0]);
    if (merge_a) C.tile[a1] = (int)std::min<int64_t>(ceil_div(cols_tile, P.size[0]), P.size[a1]);
    C.tile[p0] = (int)std::min<int64_t>(tb, P.size[p0]);
    if (merge_b) C.tile[p1] = (int)std::min<int64_t>(ceil_div(tb, P.size[p0]), P.size[p1]);
    C.digits_a = C.digits_b = 2;
    C.dtile_a[0] = cols_tile; C.dtile_a[1] = S.rows; C.dlane_a[0] = cols_tile; C.dlane_a[1] = std::max(1, kWave / S.lanes);
    C.dtile_b[0] = tb; C.dtile_b[1] = cols_tile; C.dlane_b[0] = S.line; C.dlane_b[1] = std::min(S.side, kWave / 8);
    C.dlane_a[2] = m.merged_a; C.dlane_b[2] = m.merged_b;       // part of what names the configuration
    C.lds_stride[0] = 1;
    C.lds_stride[p0] = S.pitch;
    *out = C;
    return true;
}

// The argument block of the micro-tile and the line kernel from a candidate as it stands (tile mapping, streaming hints and grid are
// the plan's current ones).
MicroArgs micro_args(const Candidate& c)
{
    const KernelParams& kp = c.kp;
    MicroArgs a;
    std::memset(&a, 0, sizeof(a));
    a.xcd_remap = kp.xcd_remap;
    a.num_tiles = kp.num_tiles; a.tiles_per_xcd = kp.tiles_per_xcd; a.tiles_rem_xcd = kp.tiles_rem_xcd;
    a.grid = kp.grid; a.grid_per_xcd = kp.grid_per_xcd; a.grid_rem_xcd = kp.grid_rem_xcd;
    for (int x = 0; x < 8; ++x) a.xcd_tiles[x] = kp.xcd_tiles[x];
    a.nt_a = kp.nt_a; a.nt_b = kp.nt_b;
    a.debug_stop = 0;
    a.col_pos = a.row_pos = -1;
    for (int i = 0; i < kMaxDim; ++i) {
        a.cnt[i] = make_fastdiv(1);
        a.step_a[i] = a.step_b[i] = 0;
    }
    for (int i = 0; i < kp.n && i < kMaxDim; ++i) {
        const int k = c.tile_order[i];
        a.cnt[i] = kp.tile_cnt[k];
        a.step_a[i] = (int64_t)kp.tile[k] * kp.stride_a[k];
        a.step_b[i] = (int64_t)kp.tile[k] * kp.stride_b[k];
        if (k == 0) a.col_pos = i;
        if (k == kp.micro.p0) a.row_pos = i;
    }
    a.alpha[0] = kp.alpha[0]; a.alpha[1] = kp.alpha[1];
    a.beta[0] = kp.beta[0];   a.beta[1] = kp.beta[1];
    a.micro = kp.micro;
    return a;
}

// The block kernel's candidate: a box of extents t[] (whole indices, but for the last ones of A's and of B's run), tile ids in
// the order `tile_order`.  Needs both unit strides to be 1.
static bool make_block_candidate(const Problem& P, const int* t, const int* tile_order, Candidate* out)
{
    if (P.ndim < 2 || P.stride_a[0] != 1 || P.stride_b[P.perm[0]] != 1) return false;
    const int va = 16 / P.eb_a, vb = 16 / P.eb_b;
    // the runs: leading indices, contiguous in the tensor, all whole but the last
    struct Run { int n, last; int dim[kMaxDim]; int64_t elems; uint32_t in; } run[2];
    for (int side = 0; side < 2; ++side) {
        Run& r = run[side];
        r.n = 0; r.last = -1; r.elems = 1; r.in = 0;
        const int64_t* stride = side ? P.stride_b : P.stride_a;
        for (int i = 0; i < P.ndim; ++i) {
            const int k = side ? P.perm[i] : i;
            if (stride[k] != r.elems || (t[k] == 1 && r.n > 0)) break;
            r.dim[r.n++] = k; r.last = k; r.in |= 1u << k;
            r.elems *= t[k];
            if (t[k] < P.size[k]) break;
        }
        if (r.n < 1) return false;
    }
    int row[2] = {-1, -1}, outd[2] = {-1, -1}, nrow = 0, nout = 0;
    int64_t volume = 1;
    for (int i = 0; i < P.ndim; ++i) {
        const int k = P.perm[i];
        if (t[k] < 1 || t[k] > P.size[k]) return false;
        volume *= t[k];
        if (volume * P.eb_a > kBlockMaxLds) return false;
        if (t[k] == 1 || ((run[0].in >> k) & 1u)) continue;
        if (nrow == 2 || (t[k] < P.size[k] && k != run[1].last)) return false;
        row[nrow++] = k;
    }
    for (int k = 0; k < P.ndim; ++k) {
        if (t[k] == 1 || ((run[1].in >> k) & 1u)) continue;
        if (nout == 2 || (t[k] < P.size[k] && k != run[0].last)) return false;
        outd[nout++] = k;
    }
    if (run[1].n > 3) return false;
    Candidate C;
    std::memset(&C, 0, sizeof(C));
    BlockParams& m = C.block;
    const int sa = run[0].last, sb = run[1].last;
    m.run_a = (int32_t)run[0].elems; m.run_b = (int32_t)run[1].elems;
    m.tile_a = t[sa]; m.tile_b = t[sb];
    m.inner_a = m.run_a / m.tile_a; m.inner_b = m.run_b / m.tile_b;
    m.size_a = P.size[sa]; m.size_b = P.size[sb];
    if (m.run_a < va || m.run_b < vb) return false;              // a cut run may hold less: its vectors then begin in the tile before
    // runs of one index each that are not the same are the micro-tile kernel's; so are those that an index of 1 KB and more begins
    if (run[0].n == 1 && run[1].n == 1) return false;
    if ((run[0].n > 1 && P.size[0] * P.eb_a > 1024) || (run[1].n > 1 && P.size[P.perm[0]] * P.eb_b > 1024)) return false;
    m.rows = (int32_t)(volume / m.run_a); m.outs = (int32_t)(volume / m.run_b);
    const int64_t per_row = ceil_div(m.run_a, va), per_out = ceil_div(m.run_b, vb);
    int unroll = 0;
    for (int u : {2, 4, 8})
        if (!unroll && per_row * m.rows <= u * kBlockThreads && per_out * m.outs <= block_stores(u, P.eb_a, P.eb_b) * kBlockThreads) unroll = u;
    if (!unroll) return false;
    m.unroll = unroll;
    m.va_div = make_fastdiv((uint32_t)per_row); m.vb_div = make_fastdiv((uint32_t)per_out);
    m.cut_row = m.cut_out = -1;
    for (int d = 0; d < 2; ++d) {
        m.row_step[d] = row[d] >= 0 ? P.stride_a[row[d]] : 0;
        m.out_step[d] = outd[d] >= 0 ? P.stride_b[outd[d]] : 0;
        if (row[d] >= 0 && row[d] == sb) m.cut_row = d;
        if (outd[d] >= 0 && outd[d] == sa) m.cut_out = d;
    }
    m.row_div = make_fastdiv((uint32_t)(row[0] >= 0 ? t[row[0]] : 1));
    m.out_div = make_fastdiv((uint32_t)(outd[0] >= 0 ? t[outd[0]] : 1));
    m.even = t[P.perm[0]] % vb == 0 ? 1 : 0;
    m.x_div[0] = make_fastdiv((uint32_t)t[run[1].dim[0]]);
    m.x_div[1] = make_fastdiv((uint32_t)(run[1].n > 1 ? t[run[1].dim[1]] : 1));
    // The LDS tile: A's order, rows padded by up to three vectors, so that the first elements of 64 neighbouring vectors of B
    // meet as few banks twice as may be.
    int64_t best = INT64_MAX;
    int lstride[kMaxDim] = {0};
    for (int pad = 0; pad < 4; ++pad) {
        const int pitch = (int)((per_row + pad) * va);
        if ((int64_t)m.rows * pitch * P.eb_a > kBlockMaxLds || (pad > 0 && m.rows == 1)) break;
        int ls[kMaxDim] = {0}, step = 1;
        for (int i = 0; i < run[0].n; ++i) { ls[run[0].dim[i]] = step; step *= t[run[0].dim[i]]; }
        if (row[0] >= 0) ls[row[0]] = pitch;
        if (row[1] >= 0) ls[row[1]] = pitch * t[row[0]];
        int bank[32] = {0};
        const int words = P.eb_a / 4;
        int worst = 0;
        for (int lane = 0; lane < kWave; ++lane) {
            const int64_t o = lane / per_out, x = lane % per_out * vb;
            if (o >= m.outs) break;
            const int64_t x0 = x % t[run[1].dim[0]], q = x / t[run[1].dim[0]], e1 = run[1].n > 1 ? t[run[1].dim[1]] : 1;
            int64_t at = x0 * ls[run[1].dim[0]] + (run[1].n > 1 ? q % e1 * ls[run[1].dim[1]] : 0) + (run[1].n > 2 ? q / e1 * ls[run[1].dim[2]] : 0);
            const int64_t e0 = outd[0] >= 0 ? t[outd[0]] : 1;
            if (outd[0] >= 0) at += o % e0 * ls[outd[0]];
            if (outd[1] >= 0) at += o / e0 * ls[outd[1]];
            for (int w = 0; w < words; ++w) worst = std::max(worst, ++bank[(at * words + w) & 31]);
        }
        const int64_t cost = (int64_t)worst * 16 + pad;
        if (cost >= best) continue;
        best = cost;
        m.pitch = pitch;
        for (int k = 0; k < kMaxDim; ++k) lstride[k] = ls[k];
        C.lds_conflict_b = 2 * std::max(1, worst / (2 * words));
    }
    if (m.pitch == 0) return false;
    C.lds_conflict_a = 2;
    for (int i = 0; i < 3; ++i) m.x_lds[i] = i < run[1].n ? lstride[run[1].dim[i]] : 0;
    for (int d = 0; d < 2; ++d) m.out_lds[d] = outd[d] >= 0 ? lstride[outd[d]] : 0;
    C.kernel_class = kKernelBlock;
    C.threads = kBlockThreads;
    C.wg_per_cu = 0;
    C.lds_bytes = m.rows * m.pitch * P.eb_a;
    KernelParams& kp = C.kp;
    kp.n = P.ndim;
    int64_t ntiles = 1;
    for (int k = 0; k < kMaxDim; ++k) {
        C.tile[k] = kp.tile[k] = k < P.ndim ? t[k] : 1;
        C.lds_stride[k] = lstride[k];
        kp.stride_a[k] = k < P.ndim ? P.stride_a[k] : 0;
        kp.stride_b[k] = k < P.ndim ? P.stride_b[k] : 0;
        kp.tile_below[k] = kp.tile_cnt[k] = make_fastdiv(1);
    }
    m.pos_a = m.pos_b = -1;
    for (int i = 0; i < P.ndim; ++i) {
        const int k = tile_order[i];
        const int64_t cnt = ceil_div(P.size[k], t[k]);
        if (cnt > INT32_MAX / 2 || ntiles > INT32_MAX / 2) return false;
        kp.tile_below[k] = make_fastdiv((uint32_t)ntiles);
        kp.tile_cnt[k] = make_fastdiv((uint32_t)cnt);
        ntiles *= cnt;
        if (ntiles > INT32_MAX / 2) return false;
        C.tile_order[i] = k;
        if (k == sa) m.pos_a = i;
        if (k == sb) m.pos_b = i;
    }
    if (!launchable(ntiles + (8 << kMaxTileMapping), C.threads)) return false;       // a launch rounds up to whole rounds over the XCDs
    kp.num_tiles = (uint32_t)ntiles;
    kp.tiles_per_xcd = kp.num_tiles / 8;
    kp.tiles_rem_xcd = kp.num_tiles % 8;
    if (!set_tile_mapping(&kp, kDefaultTileMapping)) return false;
    set_grid(&kp, kp.num_tiles);
    kp.alpha[0] = P.alpha[0]; kp.alpha[1] = P.alpha[1];
    kp.beta[0] = P.beta[0];   kp.beta[1] = P.beta[1];
    kp.a.vec = va; kp.b.vec = vb;
    kp.lds_buffers = 1;
    kp.lds_tile_elems = m.rows * m.pitch;
    for (int j = 0; j < kBoxDims; ++j) {
        kp.slot[j].tile = 1; kp.slot[j].size = 1;
        kp.slot[j].tile_below = kp.slot[j].tile_cnt = make_fastdiv(1);
    }
    C.digits_a = C.digits_b = 2;
    C.dtile_a[0] = m.run_a; C.dtile_a[1] = m.rows; C.dlane_a[0] = std::min(m.run_a, kWave * va); C.dlane_a[1] = 1;
    C.dtile_b[0] = m.run_b; C.dtile_b[1] = m.outs; C.dlane_b[0] = std::min(m.run_b, kWave * vb); C.dlane_b[1] = 1;
    *out = C;
    return true;
}

// The argument block of the block kernel from a candidate as it stands.
BlockArgs block_args(const Candidate& c)
{
    const KernelParams& kp = c.kp;
    BlockArgs a;
    std::memset(&a, 0, sizeof(a));
    a.xcd_remap = kp.xcd_remap;
    a.blocks = kp.num_tiles;
    a.nt_a = kp.nt_a; a.nt_b = kp.nt_b;
    for (int i = 0; i < kMaxDim; ++i) a.cnt[i] = make_fastdiv(1);
    for (int i = 0; i < kp.n && i < kMaxDim; ++i) {
        const int k = c.tile_order[i];
        a.cnt[i] = kp.tile_cnt[k];
        a.step_a[i] = (int64_t)kp.tile[k] * kp.stride_a[k];
        a.step_b[i] = (int64_t)kp.tile[k] * kp.stride_b[k];
    }
    a.alpha[0] = kp.alpha[0]; a.alpha[1] = kp.alpha[1];
    a.beta[0] = kp.beta[0];   a.beta[1] = kp.beta[1];
    a.block = c.block;
    return a;
}

// The row kernel's candidate: B walked front to back, `vec` elements per lane and access; `flat`: vectors counted through
// a dense B.  Needs rows that are contiguous in both tensors and hold at least one vector, fewer than 2^31 rows, rows
// shorter than 2^30.
static bool make_rows_candidate(const Problem& P, int vec, int unroll, bool flat, Candidate* out)
{
    if (P.perm[0] != 0 || P.stride_a[0] != 1 || P.stride_b[0] != 1) return false;
    const int64_t row = P.size[0], rows = P.elements / P.size[0];
    if (row < vec || row >= (int64_t(1) << 30) || rows >= (int64_t(1) << 31)) return false;
    if (flat && P.span_b != P.elements) return false;
    // rows that are not a multiple of the vector: their last vector overlaps its neighbour, which is only
    // harmless where B is not read
    if (!flat && row % vec != 0 && P.epilogue == TTC_EPI_AXPBY) return false;
    Candidate C;
    std::memset(&C, 0, sizeof(C));
    C.kernel_class = TTC_KERNEL_ROWS;
    C.threads = 256;
    C.wg_per_cu = 0;                   // one-shot workgroups: nothing to choose
    C.lds_bytes = 0;
    RowsParams& r = C.rows;
    r.n = P.ndim;
    r.vec = vec;
    r.unroll = unroll;
    r.row = (uint32_t)row;
    r.rows = (uint32_t)rows;
    r.elements = P.elements;
    r.flat = flat ? 1 : 0;
    r.slots = (uint32_t)(flat ? row : ceil_div(row, vec));
    r.chunk = (uint32_t)(C.threads * r.unroll);
    r.overlap = (!flat && row % vec != 0) ? 1 : 0;
    r.slot_div = make_fastdiv(r.slots);
    r.vectors = flat ? ceil_div(P.elements, vec) : rows * (int64_t)r.slots;
    for (int d = 0; d < kMaxDim; ++d) {
        r.size_div[d] = make_fastdiv(1);
        r.stride_a[d] = 0;
        r.stride_b[d] = 0;
        if (d >= 1 && d < P.ndim) {
            const int k = P.perm[d];                       // B's index d is A's index k
            r.size_div[d] = make_fastdiv((uint32_t)P.size[k]);
            r.stride_a[d] = P.stride_a[k];
            r.stride_b[d] = P.stride_b[k];
        }
    }
    r.alpha[0] = P.alpha[0]; r.alpha[1] = P.alpha[1];
    r.beta[0] = P.beta[0];   r.beta[1] = P.beta[1];
    // what the other kernels' fields say about this one
    KernelParams& kp = C.kp;
    kp.n = P.ndim;
    kp.a.vec = vec; kp.b.vec = vec;
    kp.lds_buffers = 1;
    const int64_t grid = ceil_div(r.vectors, r.chunk);
    if (!launchable(grid + (8 << kMaxTileMapping), C.threads)) return false;       // a launch rounds up to whole rounds over the XCDs
    kp.a.partial = kp.b.partial = r.overlap;
    kp.num_tiles = (uint32_t)grid;
    kp.grid = (uint32_t)grid;
    r.blocks = (uint32_t)grid;
    if (!set_tile_mapping(&kp, default_tile_mapping(P, C))) return false;
    for (int k = 0; k < kMaxDim; ++k) {
        C.tile[k] = (k == 0) ? (int)row : 1;
        C.tile_order[k] = (k < P.ndim) ? P.perm[k] : k;
        kp.tile[k] = C.tile[k];
        kp.tile_below[k] = kp.tile_cnt[k] = make_fastdiv(1);
        kp.stride_a[k] = (k < P.ndim) ? P.stride_a[k] : 0;
        kp.stride_b[k] = (k < P.ndim) ? P.stride_b[k] : 0;
    }
    C.digits_a = C.digits_b = 1;
    C.dtile_a[0] = C.dtile_b[0] = (int)row;
    C.dlane_a[0] = C.dlane_b[0] = (int)std::min<int64_t>(row, (int64_t)kWave * vec);
    *out = C;
    return true;
}

static double traffic_bytes(const Problem& P)
{
    return (double)P.elements * (P.eb_a + (P.epilogue == TTC_EPI_AXPBY ? 2 : 1) * P.eb_b);
}

// What the loads of the gather kernel ask of the memory system, counted over two pairs of neighbouring workgroups: lines
// that the 64 lanes of one load instruction touch (per wavefront, all of its loads), lines that a workgroup touches, and
// which part of its lines a workgroup shares with the next one.
struct GatherLines { double requests, lines, shared; };

static GatherLines gather_lines(const Problem& P, const RowsParams& r)
{
    GatherLines g = {0, 0, 0};
    const uint32_t vec = (uint32_t)r.vec, last = (uint32_t)(P.elements - 1);
    constexpr uint32_t kSlots = 4096;                      // at most 2 x 1024 lines a pair
    struct Slot { int64_t line; uint32_t loads; };         // bit 16 w + 4 wave + j: load j of that wavefront touches it
    std::vector<Slot> slot(kSlots);                        // 64 KB: more than a thread's stack may have
    double both = 0, single = 0;
    for (int s = 0; s < 2; ++s) {
        const uint32_t wg = (uint32_t)((int64_t)r.blocks * (1 + 2 * s) / 4);
        for (Slot& x : slot) x.loads = 0;
        for (uint32_t t = 0; t < 512; ++t) {
            const uint32_t e = (wg * 256 + t) * vec;
            const GatherPlace first = gather_place(r, std::min(e, last));
            for (uint32_t j = 0; j < vec; ++j) {
                const GatherPlace at = j == 0 ? first : (e + j <= last ? gather_next(r, first, e, j) : gather_place(r, last));
                const int64_t line = at.a * P.eb_a / kLineBytes;
                uint32_t h = (uint32_t)((uint64_t)line * 0x9e3779b97f4a7c15ull >> 52);
                while (slot[h].loads != 0 && slot[h].line != line) h = (h + 1) % kSlots;
                slot[h].line = line;
                slot[h].loads |= 1u << (16 * (t / 256) + 4 * (t / kWave % 4) + j);
            }
        }
        for (const Slot& x : slot) {
            if (x.loads == 0) continue;
            g.requests += (double)__builtin_popcount(x.loads) / 16.0;         // per wavefront: 4 workgroups of 4
            single += (x.loads & 0xffffu ? 1 : 0) + (x.loads >> 16 ? 1 : 0);
            both += 1;
        }
    }
    g.lines = single / 4.0;
    g.shared = 2.0 * (1.0 - both / single);
    return g;
}

// The gather kernel's candidate: every lane writes 16 bytes of B and fetches their elements one by one from A.  Any
// problem of at most 64 MB of traffic (beyond that its repeated line requests never win) whose B has a unit stride along
// its first index: what a lane writes is one vector (of one element where that has 16 bytes: any stride will do).
static bool make_gather_candidate(const Problem& P, Candidate* out)
{
    if (traffic_bytes(P) > 64e6) return false;
    if (P.eb_b < 16 && P.stride_b[P.perm[0]] != 1) return false;      // an index of extent 1 in front of it, padded by ldb
    Candidate C;
    std::memset(&C, 0, sizeof(C));
    C.kernel_class = kKernelGather;
    C.threads = 256;
    C.wg_per_cu = 0;
    RowsParams& r = C.rows;
    r.n = P.ndim;
    r.vec = 16 / P.eb_b;
    r.unroll = 1;
    r.row = (uint32_t)P.size[P.perm[0]];
    r.elements = P.elements;
    r.flat = P.span_b == P.elements ? 1 : 0;
    r.chunk = 256;
    r.vectors = ceil_div(P.elements, r.vec);
    r.blocks = (uint32_t)ceil_div(r.vectors, r.chunk);
    for (int d = 0; d < kMaxDim; ++d) {
        r.size_div[d] = make_fastdiv(1);
        if (d >= P.ndim) continue;
        const int k = P.perm[d];                           // B's index d is A's index k
        r.size_div[d] = make_fastdiv((uint32_t)P.size[k]);
        r.stride_a[d] = P.stride_a[k];
        r.stride_b[d] = P.stride_b[k];
    }
    r.alpha[0] = P.alpha[0]; r.alpha[1] = P.alpha[1];
    r.beta[0] = P.beta[0];   r.beta[1] = P.beta[1];
    KernelParams& kp = C.kp;
    kp.n = P.ndim;
    kp.a.vec = kp.b.vec = r.vec;           // what a lane moves
    kp.lds_buffers = 1;
    for (int k = 0; k < kMaxDim; ++k) {
        // nothing is tiled: the fields say whole vectors along either unit-stride index, as for every kernel
        C.tile[k] = kp.tile[k] = (k == P.perm[0]) ? (int)std::min<int64_t>(P.size[k], 256 * r.vec) : (k == 0 ? r.vec : 1);
        C.tile_order[k] = (k < P.ndim) ? P.perm[k] : k;
        kp.tile_below[k] = kp.tile_cnt[k] = make_fastdiv(1);
        kp.stride_a[k] = (k < P.ndim) ? P.stride_a[k] : 0;
        kp.stride_b[k] = (k < P.ndim) ? P.stride_b[k] : 0;
    }
    // Workgroups that share lines of A with their neighbours belong on one XCD: one contiguous range each, dealt round robin
    // at any size (transposes, against chunks numbered as they lie in B: 600 x 600 fp32 4.1 us and 5.3, 1500 x 1500 12.7
    // and 17.6, 700 x 500 fp64 4.0 and 6.0; in chunks of 32 1500 x 1500 takes 13.2).  Where they share none the ranges may
    // only spread the reads further (40 x 50 x 60 x 20 complex64, reversed, 45 against 31); that workgroups further apart
    // share some is not seen (581 x 783 complex128 runs at 9.9, 5.3 in ranges; the line kernel is ranked first there).
    const GatherLines g = gather_lines(P, r);
    const uint32_t chunks = r.blocks;
    if (chunks >= 64 && g.shared > 0.25) {
        r.per_xcd = (chunks + 7) / 8;
        r.blocks = 8 * r.per_xcd;
    }
    kp.num_tiles = kp.grid = r.blocks;
    if (!set_tile_mapping(&kp, r.per_xcd ? 0 : kDefaultTileMapping)) return false;
    // Fitted to 170 problems of 0.1 to 60 MB: 20 % rms.
    C.model_us = 2.5 + 0.105e-6 * traffic_bytes(P) + 2.25e-6 * g.requests * 4.0 * chunks + 4.3e-6 * g.lines * chunks;
    C.digits_a = C.digits_b = 1;
    C.dtile_a[0] = 1; C.dlane_a[0] = 1;
    C.dtile_b[0] = C.dlane_b[0] = kWave * r.vec;
    *out = C;
    return true;
}

// The row kernel's chunks: rows that share lines of A (they start inside lines, and the next one begins in the line where this one ends)
// lie in chunks that are far apart in B and meet in one L2 where each XCD has one range of chunks; and a launch without groups of
// chunks (none or ranges) packs its arguments.  Time of ranges over the rule of set_tile_mapping(), pairs in rotation, 19 000 random
// problems with a dense A.  Packed copies: 8-16, 16-32, 32-64, 64-128 MB of traffic, rows
// below 64 bytes 0.72, 0.80, 0.82, 0.86, to 128 0.80, 0.83, 0.85, 0.84, to 512 0.92, 0.85, 0.89, 0.88, longer 0.95, 0.86, 0.91, 0.91,
// whole lines 0.96, 0.91, 0.93, 0.93; 128-200 MB below 512 bytes 0.90-0.92, longer and whole lines 0.96-1.05, beyond 200 MB 0.94-1.06.  (6 x 258 x 2475 fp32
// (0,2,1) reads 18 MB instead of 50, of 15: 11.9 -> 7.6 us.)  Packed updates of rows that split lines: below 128 bytes 0.80-0.94 from 8 MB on, to
// 512 0.92-0.97 from 16 MB on, longer 0.94-0.99; others from 16 MB on as they come: 0.95-0.99 (ranges 0.97-1.02).  Not packed: split rows below
// 256 bytes 0.76-0.99 (copies to 512 0.92-0.98) from 8 to 200 MB; the others 0.99-1.06.
// With a padded A it is the distance of the rows that counts, not their length.  Ranges over chunks as they come, 400 problems: shared
// lines 0.79 (copies) and 0.84 (updates) in rows below 128 bytes, 0.95 and 0.98 in longer ones; rows on lines of their own, or a line
// and more apart, 0.99-1.02; not packed, rows of whole lines that share others gain nothing (123 below 512 bytes: 0.99 over chunks of 32, 1.04 on
// new tensors).  400 problems where that is another mapping than the rows' length gives: 0.990 of the time in rotation, 0.992
// on one pair, 0.985 on new tensors (32 x 800 x 331 fp32 (0,2,1) at a distance of 33 with an update 20.0 -> 16.8 us, a copy of 64 x 560 x 558
// at 65 32.0 -> 25.0).
// An XCD has about 1 MB of B under way (32 compute units, eight chunks of 4 KB each): rows below 128 bytes whose neighbours in A lie `apart`
// further than that do not meet (1.00-1.10, as they come 0.92-0.99); up to 512 KB 0.63-0.93, up to 1 MB 0.79-0.99.
static int rows_tile_mapping(const Problem& P, const Candidate& C)
{
    const double traffic = traffic_bytes(P);
    const int64_t row = P.size[0] * P.eb_a;
    const int64_t apart = P.ndim > 1 ? P.stride_b[1] * P.eb_b : 0, step = P.ndim > 1 ? P.stride_a[1] * P.eb_a : 0;
    const bool update = P.epilogue == TTC_EPI_AXPBY;
    const bool shared = step % kLineBytes != 0 && step - row < kLineBytes;       // (strides of later indices are multiples of index 1's)
    if (traffic < 8e6 || traffic > 200e6) return kDefaultTileMapping;
    Candidate rule = C;
    default_streaming(P, &rule);
    RowsParams r = C.rows;
    r.nt_a = rule.kp.nt_a;
    r.nt_b = rule.kp.nt_b;
    r.xcd_remap = 1;
    const bool packed = r.unroll == 1 && small_dims(r, false, P.epilogue, P.kind_a >= kKindC64, 0, 1) != 0;
    if (row < 128 && apart > (row < 64 && traffic < 32e6 ? int64_t(1) << 19 : int64_t(1) << 20)) return packed ? 0 : kDefaultTileMapping;
    if (!packed) return shared && row % kLineBytes != 0 && row < (update ? 256 : 512) ? 1 : kDefaultTileMapping;
    if (!update) return traffic <= 128e6 || (shared && row < 512) ? 1 : kDefaultTileMapping;
    if (traffic < 16e6) return shared && row < 128 ? 1 : kDefaultTileMapping;
    return shared && row < 2048 ? 1 : 0;
}

// Tiles from one to the next along A's run, in the candidate's order.
static int64_t tiles_between(const Problem& P, const Candidate& C)
{
    int64_t between = 1;
    for (int i = 0; i < P.ndim && C.tile_order[i] != 0; ++i) between *= (int64_t)C.kp.tile_cnt[C.tile_order[i]].div;
    return between;
}

// The line kernel's tiles read lines that their neighbours read as well: rows of A at the edge along B's runs where columns are cut at
// their own lines (skewed), lines of A at the edge along A's runs where those split lines.  One contiguous range of tiles per XCD lets
// neighbours meet in one L2; from 200 MB on the eight distant windows cost more than that gives.  Time of one range over the rule of
// set_tile_mapping(), pairs in rotation, 21 000 random problems: skewed, copies of 8-16, 16-32, 32-64, 64-128 and 128-200 MB of
// traffic 0.89, 0.83, 0.87, 0.90, 0.95 (4-8 MB 0.98-1.03), updates from 2 MB on 0.94, 0.93, 0.92, 0.86, 0.88, 0.92, 0.93; 200-300 MB 1.01, beyond
// 1.03.  (2334 x 4390 fp32 reads 93 MB from beyond the L2s instead of 45, of 41 that it has to, and a request takes 1073 cycles instead of
// 688: 20.0 -> 13.8 us; 7145 x 536 9.7 -> 6.9, 2001^2 10.9 -> 7.0.)  Where A's lines are split the next tile along A's
// run has to be under way at the same time, `between` tiles later: up to 160 of them 0.90, 192-256 0.93-0.99, beyond 0.95-1.01 and
// up to 1.5 (25 x 143639 complex64); where a range is shorter than that 0.93, with a twentieth of them above 1.1.  Not skewed, lines split at multiples of 32 bytes or less, 8 to 200 MB and up to 64 tiles
// between 0.91; at 64 bytes or with more between 0.98-1.06; whole lines on both sides share nothing (0.99-1.02).
static int default_tile_mapping(const Problem& P, const Candidate& C)
{
    if (C.kernel_class == TTC_KERNEL_ROWS) return rows_tile_mapping(P, C);
    if (C.kernel_class != kKernelLines) return C.rows.per_xcd ? 0 : kDefaultTileMapping;
    const MicroParams& m = C.kp.micro;
    int64_t align = kLineBytes;
    for (int k = 1; k < P.ndim; ++k)
        while (!(m.merged_a && k == 1) && P.stride_a[k] * P.eb_a % align != 0) align /= 2;
    const int64_t between = tiles_between(P, C);
    const double traffic = traffic_bytes(P);
    const bool near = between <= 160 && between * 8 <= (int64_t)C.kp.num_tiles;
    const bool ranges = m.skewed ? traffic >= (P.epilogue == TTC_EPI_AXPBY ? 2e6 : 8e6) && (align == kLineBytes || near)
                                 : traffic >= 8e6 && align <= 32 && between <= 64;
    return ranges && traffic <= 200e6 ? 1 : kDefaultTileMapping;
}

bool set_tile_mapping(KernelParams* kp, int mode)
{
    if (mode == kDefaultTileMapping) {
        mode = kp->num_tiles >= 2048u ? 5 : 0;      // few tiles (a workgroup gets one or two): round robin spreads them best
    }
    if (mode < 0 || mode > kMaxTileMapping) return false;
    kp->xcd_remap = mode;
    for (int x = 0; x < 8; ++x) kp->xcd_tiles[x] = 0;
    if (mode >= 2) {
        const uint32_t C = 1u << mode;
        const uint32_t chunks = (kp->num_tiles + C - 1) / C;             // the last one may be partial
        for (uint32_t x = 0; x < 8; ++x) {
            const uint32_t mine = chunks > x ? (chunks - x + 7) / 8 : 0;
            kp->xcd_tiles[x] = mine * C;
            if (mine > 0 && (chunks - 1) % 8 == x) kp->xcd_tiles[x] -= chunks * C - kp->num_tiles;
        }
    }
    return true;
}

uint32_t launch_grid(const Candidate& c, int cus)
{
    if (c.kernel_class == TTC_KERNEL_MICRO || c.kernel_class == TTC_KERNEL_ROWS || c.kernel_class == kKernelLines ||
        c.kernel_class == kKernelGather || c.kernel_class == kKernelBlock) return c.kp.num_tiles;    // one-shot workgroups
    const uint64_t want = (uint64_t)std::max(cus, 1) * (uint64_t)std::max(c.wg_per_cu, 1);
    return (uint32_t)std::min<uint64_t>(want, c.kp.num_tiles);
}

void set_grid(KernelParams* kp, uint32_t grid)
{
    kp->grid = grid;
    kp->grid_per_xcd = grid / 8;
    kp->grid_rem_xcd = grid % 8;
}

// Heuristic cost of a candidate (smaller is better).  It plays the role of the paper's cost
// estimate that admits candidates to the bounded queue; the paper does not define one, this
// one prices coalescing (length and alignment of the contiguous runs on both sides),
// remainder tiles, tile size, lane use and vector width.
// How a candidate touches memory, in bytes per side: the contiguous run the tile spans, the
// contiguous piece one wavefront instruction covers, and the power of two (up to 128) that
// divides the byte offset of every run start.
struct AccessShape { int run[2], seg[2], align[2]; };

static int segment_elems(const Side& s, bool second)
{
    struct Item { int64_t stride; int lane, tile; } it[kBoxDims];
    int n = 0;
    for (int j = 0; j < kBoxDims; ++j)
        if (s.d[j].tile > 1) { it[n].stride = second ? s.d[j].g2stride : s.d[j].gstride; it[n].lane = s.d[j].lane; it[n].tile = s.d[j].tile; ++n; }
    std::sort(it, it + n, [](const Item& x, const Item& y) { return x.stride < y.stride; });
    int64_t seg = 1, expect = 1;
    for (int i = 0; i < n; ++i) {
        if (it[i].stride != expect) break;
        seg *= it[i].lane;
        if (it[i].lane < it[i].tile) break;
        expect = it[i].stride * it[i].tile;
    }
    return (int)std::min<int64_t>(seg, 1 << 20);
}

static AccessShape access_shape(const Problem& P, const Candidate& C)
{
    AccessShape r;
    const bool direct = (C.kernel_class == TTC_KERNEL_DIRECT);
    for (int side = 0; side < 2; ++side) {
        int order[kMaxDim];
        for (int k = 0; k < kMaxDim; ++k) order[k] = side ? ((k < P.ndim) ? P.perm[k] : k) : k;
        const int64_t* stride = side ? P.stride_b : P.stride_a;
        const int eb = side ? P.eb_b : P.eb_a;
        int64_t run = 1, g = 0;
        bool open = true;
        for (int i = 0; i < P.ndim; ++i) {
            const int k = order[i];
            if (open && stride[k] != run) open = false;
            if (open) {
                run *= C.kp.tile[k];
                if (C.kp.tile[k] < P.size[k]) open = false;
            } else if (P.size[k] > 1) {
                int64_t a = stride[k] * eb, b = g;
                while (b) { const int64_t t = a % b; a = b; b = t; }
                g = a;
            }
        }
        int64_t a = run * eb, b = g;
        while (b) { const int64_t t = a % b; a = b; b = t; }
        int al = 1;
        while (al < 128 && a % (2 * al) == 0) al *= 2;
        r.run[side] = (int)std::min<int64_t>(run * eb, INT32_MAX);
        r.align[side] = al;
        const Side& s = (side && !direct) ? C.kp.b : C.kp.a;
        r.seg[side] = segment_elems(s, side && direct) * eb;
    }
    return r;
}

// The row kernel against the tiled kernels, fitted to the times of both on 330 problems: rows of 16 bytes to 64 KB, 2 to
// 200 MB, fp32, fp64, complex128 and fp32 -> fp64, dense and padded.
// Dense B: whole lines are ahead from 128-byte rows on (200 MB: 66-68 us against 72-75), rows that start inside lines
// from 264-byte rows on (71-79 us against 88-91; 68-byte rows 102 against 93), updates of ragged rows by more (340-byte
// rows 104 against 153-166: no narrow vectors).  Padded B: tiles split lines as well there, and rows are ahead from
// 36 bytes on (64-byte rows 87-115 us against 130-156, 800-byte ones 72 against 100; 32-byte ones 164 against 139).
// Below 8 MB rows always are (2.6-4 us against 5.4-8: no tables, no barrier).
static double rows_cost(const Problem& P, const Candidate& C)
{
    const double row_bytes = (double)P.size[0] * P.eb_a;
    auto oct_below = [](double x, double ref) { return x < ref ? std::log2(ref / x) : 0.0; };
    const bool update = P.epilogue == TTC_EPI_AXPBY, whole = P.size[0] * P.eb_a % kLineBytes == 0;
    const double traffic = traffic_bytes(P);
    double e = traffic < 8e6 ? -0.425 : (traffic < 1e8 ? -0.128 : 0.0);
    if (P.span_b == P.elements) {
        e -= 0.373;
        if (!C.rows.flat) e += 0.05;                                        // pieces of B that start at any element
        if (!whole) e += 0.124;
        if (traffic >= 1e8) e += 0.049 * oct_below(row_bytes, 128.0) + (whole ? 0.0 : 0.094 * oct_below(row_bytes, 512.0));
        if (traffic >= 1e8 && !whole && !update && row_bytes < 160.0) e += 0.02;     // 140 bytes: 35^5 98 us, tiles 88; 35 x 63 x 115 x 208 100
                                                                            // and 97 (184 bytes 71 and 74, 208 bytes 106 and 113)
        else if (!whole) e += 0.103 * oct_below(row_bytes, 128.0);
        if (update && P.size[0] % (16 / std::max(P.eb_a, P.eb_b)) != 0 && C.rows.flat) e -= 0.131;
    } else {
        e -= 0.30;
        e += traffic >= 1e8 ? 0.10 * oct_below(row_bytes, 128.0) : 0.05 * oct_below(row_bytes, 64.0);
        if (row_bytes <= 32.0 && traffic >= 8e6) e += 2.0;
    }
    // access width, and the bytes of A a lane keeps in flight: 16; every doubling costs 1-5 %, eight bytes (the narrow
    // side of fp32 -> fp64) 10 % unless B is loaded too
    e += 0.05 * oct_below(C.rows.vec * std::max(P.eb_a, P.eb_b), 16.0);
    const double flight = (double)C.rows.vec * C.rows.unroll * P.eb_a;
    e += flight < 16.0 ? (update ? 0.0 : 0.10) * std::log2(16.0 / flight) : 0.03 * std::log2(flight / 16.0);
    return std::exp(e);
}

// The micro-tile kernel's ranking model: log-linear like the box kernels' below, with the family's own features
// (it has no tables, no barriers per walk, no bank conflicts).  Weights fitted to the timings of every micro-tile
// candidate of 68 problems (the 57-case benchmark and the search study's 30, the suite included; weighted least
// squares, penalties constrained to be penalties, checked by holding problems out: the first candidate reaches
// 93.8 % of the family's best on problems the fit has not seen, the first ten 98.5 %) and rounded; the offset
// against the box kernels' model is the one that makes the first candidate of the joint ranking best on the same
// problems.  Guard rails for small problems as below.
static double micro_cost(const Problem& P, const Candidate& C)
{
    auto below = [](double x, double ref) { return x < ref ? std::log2(ref / x) : 0.0; };
    auto above = [](double x, double ref) { return x > ref ? std::log2(x / ref) : 0.0; };
    const MicroParams& m = C.kp.micro;
    const double run_a = (double)m.ta * P.eb_a, run_b = (double)m.tb * P.eb_a;
    const int64_t line = 128 / P.eb_a;
    const bool un_a = m.size_a0 % line != 0 || m.ta % line != 0;          // runs of A start inside lines
    const bool un_b = m.size_p0 % line != 0 || m.tb % line != 0;
    double e = -0.22;
    e += 0.05 * below(run_a, 128.0) + 0.012 * below(run_b, 128.0);
    e += -0.01 * above(run_a, 1024.0) - 0.03 * above(run_b, 1024.0);
    const double padded = ((double)ceil_div(m.size_a0, m.ta) * m.ta / (double)m.size_a0) *
                          ((double)ceil_div(m.size_p0, m.tb) * m.tb / (double)m.size_p0);
    e += 0.11 * (padded - 1.0);                                          // idle lanes in the remainder tiles
    if (un_a) e += 0.028 * below(run_a, 512.0);                          // the shorter the run, the larger the share of split lines
    if (un_b) e += 0.072 * below(run_b, 512.0);
    if (C.threads == 128) e += 0.04; else if (C.threads == 64) e += 0.068;
    bool b_order = true;
    for (int i = 0; i < P.ndim; ++i) if (C.tile_order[i] != P.perm[i]) b_order = false;
    if (!b_order) e += 0.054;
    e += 0.009 * std::log2((double)std::max(1, m.blocks));
    e += 0.114 * (double)C.lds_bytes / 65536.0;                          // fewer workgroups per compute unit
    if (m.merged_a) e += 0.006;
    if (m.merged_b) e += 0.011;
    e += 0.27 * (1.0 - (double)m.la * m.lb / ((double)m.blocks * C.threads));   // lanes without a block
    const double tiles_wanted = std::min(2048.0, std::max(1.0, (double)P.elements * P.eb_a / 8192.0));
    if (C.kp.num_tiles < tiles_wanted) e += 1.28 * (tiles_wanted - C.kp.num_tiles) / 2048.0;
    const double cus_wanted = std::min(256.0, std::max(1.0, (double)P.elements * P.eb_a / 4096.0));
    if (C.kp.num_tiles < cus_wanted) e += 1.5 * (cus_wanted - C.kp.num_tiles) / 256.0;
    return std::exp(e);
}

// 0 up to `from`, 1 from `to` on, even in the logarithm between: terms of the ranking models set in without a jump.
static double octaves(double x, double from, double to)
{
    return x <= from ? 0.0 : x >= to ? 1.0 : std::log(x / from) / std::log(to / from);
}

// The line kernel's ranking model, log-linear like the others, fitted to the timings of every line candidate of 300
// problems (the 57-case benchmark in fp32, fp64, complex128 and fp32 -> fp64, and random problems of every type, 64 KB
// to 240 MB) against the candidate that the other models rank first.  Two sets of weights: from 16 MB of traffic on a
// tile costs what it loads and stores, below what counts is how long one tile takes.  Choosing by it takes 7 % (large)
// and 15 % (small) off the time of the other families' first candidate, geometric mean over all problems, those that
// stay with the other families included (held-out problems: 7 % and 15 %).
static double line_cost(const Problem& P, const Candidate& C)
{
    const MicroParams& m = C.kp.micro;
    const LineShape S = line_shape(m.ta, m.lines, P.eb_a, P.eb_b);
    const double rows = (double)m.size_p0, cols = (double)m.size_a0;
    const int64_t segs = (int64_t)C.kp.tile_cnt[m.p0].div;
    const bool update = P.epilogue == TTC_EPI_AXPBY;
    bool split_a = m.ta * P.eb_a % kLineBytes != 0;                       // runs of A that start or end inside lines
    for (int k = 1; k < P.ndim; ++k)
        if (!(m.merged_a && k == 1) && P.stride_a[k] * P.eb_a % kLineBytes != 0) split_a = true;
    const double run_a = std::min<double>(m.ta, cols) * P.eb_a;
    const double split = split_a ? (double)kLineBytes / run_a : 0.0;
    const double pad_cols = std::log((double)ceil_div(m.size_a0, m.ta) * m.ta / cols);
    // Columns of B start inside lines unless B's first two indices are taken as one: such a problem's other candidates split
    // lines as those of a skewed one do, and the kernel gains as much on them, whichever way its own tiles are cut.
    bool odd = m.skewed != 0;
    for (int k = 0; k < P.ndim; ++k) if (k != P.perm[0] && P.stride_b[k] * P.eb_b % kLineBytes != 0) odd = true;
    const bool one_precision = P.eb_a == P.eb_b && P.eb_a < 16;           // the others' first is then a micro-tile candidate, ranked by its own model
    const double line_rows = rows / S.line;                               // lines per column
    const double traffic = traffic_bytes(P);
    double e;
    if (traffic >= 16e6) {
        const int64_t last_row0 = (segs - 1) * (int64_t)m.tb - (m.skewed ? S.line : 0);
        int64_t loaded = segs * (int64_t)S.rows;                          // rows loaded per column: whole passes
        loaded -= S.rows - std::min<int64_t>(S.rows, ceil_div(m.size_p0 - last_row0, S.pass) * S.pass);
        if (m.skewed) loaded -= S.line / S.pass * S.pass;                 // the first tile needs no rows before it
        e = -0.245 - (odd ? 0.082 : 0.0) - (update ? 0.083 : 0.0);
        if (one_precision) e += odd ? -0.073 : (split_a || update ? -0.010 : 0.075);     // whole lines on both sides: the micro-tile kernel is as good
        // Updates with whole lines on both sides, where neither kernel splits one: line against micro-tile kernel on one pair
        // of tensors, on pairs in rotation and on new ones, geometric means.  Tensors beyond the 256 MB of the last-level
        // cache (14 problems): 1.15, 1.01 and 1.30 times the micro-tile kernel's time (288 x 608 x 221 complex64 (1,0,2):
        // 144 us against 130, 146 against 158, 189 against 138).  Smaller ones of 4-byte elements (12): 0.98, 1.09 and
        // 1.06; of 8-byte elements (15): 0.99, 0.97 and 1.04.  Held-out problems (24) agree.
        if (one_precision && update && !m.skewed && !split_a) {
            if (P.elements * P.eb_a >= (int64_t(256) << 20)) e += 0.30;
            else if (P.eb_a == 4) e += 0.17;
        }
        // Copies of 8-byte elements whose columns of B start inside lines, both tensors together a quarter to a half of the
        // last-level cache: the line kernel takes 1.09, 1.02 and 1.09 times the micro-tile kernel's time (one pair, pairs in
        // rotation, new ones; 28 problems of 32 to 64 MB per tensor, tiles dealt by number: 795 x 6248 fp64 19.7 us against 17.2, 22.7 against 21.3
        // and 22.2 against 20.3).  Below, 0.93, 0.94 and 0.95 (15 problems from 9 MB on); above, 1.01, 0.97 and 1.04 (17 up to 127 MB).
        // Not where its tiles have one range per XCD: there it takes 0.84, 0.80 and 0.94 times what the first candidate with this term does (60
        // problems of three to six indices), 0.84, 0.77 and 0.92 with two (80; 1379 x 5230 fp64 23.3 -> 19.2, 27.4 -> 19.2 and 29.2 -> 25.5 us).
        const bool ranges = C.kp.xcd_remap == 1, short_runs = P.span_b != P.elements && rows * P.eb_b < 512.0;
        if (one_precision && !update && m.skewed && P.eb_a == 8 && traffic >= 64e6 && traffic < 128e6 && !ranges) {
            e += 0.16;
        } else if (ranges && !short_runs) {
            // With ranges, what the fit (tiles dealt by number) does not know: how much they are worth depends on how far away the next tile along
            // A's run is, and without skewed columns they are worth half; it sets in and ends where ranges do, or with this branch.  In copies columns of
            // 128 bytes go before 256 in 4-byte elements, and in the wider ones eight lines before four in the narrowest tiles.  Runs of B below 512
            // bytes between leading dimensions gain less.  Each by itself: time of the first candidate with it over that without, in rotation, on one
            // pair and on new tensors, drawn problems of 8 to 200 MB that it decides.  The share of ranges 0.94, 0.93 and 0.99 (150; at 16-32, 32-64,
            // 64-128, 128-200 MB 0.96, 0.92, 0.93 and 0.93 in rotation; instead of the block kernel 0.91, 0.92 and 0.98, of another tile of this kernel 0.95, 0.94
            // and 0.99, of the micro-tile kernel 0.86, 0.91 and 0.99); 128 bytes before 256 0.93, 0.93 and 0.99 (90); eight lines 0.99, 0.92 and 0.99 (75);
            // short runs left out 0.90, 0.89 and 0.97 (27).
            const double between = (double)tiles_between(P, C);
            e -= m.skewed ? 0.12 * (1.0 - octaves(between, 64.0, 160.0)) : 0.06 * (1.0 - octaves(between, 16.0, 64.0));
            if (!update) e += P.eb_a == 4 ? (m.ta == 64 ? 0.04 : 0.0) : m.lines == 4 && m.ta == 16 ? 0.03 : 0.0;
        }
        if (update && m.merged_a && P.size[0] * P.eb_a >= 512) e += 0.08 + (P.perm[1] == 0 ? 0.12 : 0.0);    // a tile that crosses the end of a row
                                                                          // reads and writes B in two places, and leaves a contiguous block
        e += 0.343 * std::log((double)loaded / rows) + 0.340 * pad_cols + 0.293 * std::log((double)segs * m.tb / rows) + 0.087 * split;
        // Columns of 256 bytes before 128 in 4-byte elements, four lines before eight.  With `odd` above, over 120 problems of 16 to
        // 500 MB: 2.4 % off the geometric mean, 7 % where both ways of cutting exist, none slower by more than 2 % (408^3 fp32 reversed
        // 149 -> 115 us, 300^3 fp64 103 -> 95, 408 x 200 x 408 fp32 with an update 91 -> 76, 360^3 fp64 -> fp32 138 -> 125; with their
        // arguments packed as well 113, 84, 75 and 108).
        if (m.skewed) e += (P.eb_a == 4 && m.ta == 64 ? -0.03 : 0.0) + (m.lines == 8 ? 0.02 : 0.0);
        if (m.skewed) e += 0.178 * 2.0 / (line_rows + 1.0);               // lines that no tile writes whole: a column's first and last
        if (m.size_p0 < S.line) e += 0.258;
        if (m.lines == 2) e += 0.10;
        if (update && m.ta == 64 && m.lines >= 4) e += 0.20;              // eight old vectors a lane: half the wavefronts fit
        const double tiles_wanted = std::min(2048.0, std::max(1.0, (double)P.elements * P.eb_a / 8192.0));
        if (C.kp.num_tiles < tiles_wanted) e += 0.30 * (tiles_wanted - C.kp.num_tiles) / 2048.0;
    } else {
        e = -0.40 + (m.skewed ? 0.057 : 0.0) + (one_precision ? (update && m.skewed ? 0.16 : 0.08) : 0.0) - (update ? 0.126 : 0.0);
        e += 0.05 * pad_cols + 0.167 * split + 0.18 * C.lds_bytes / 65536.0;
        e -= 0.058 * std::log2(std::min<double>(m.lines - m.skewed, std::ceil(line_rows)));
        // vectors a lane stores: the fewer the quicker the tile
        e += std::min(0.14, std::max(0.05, 0.12 - 0.025 * std::log2(traffic / 2e6))) * std::log2((double)(m.ta / S.side) * (m.lines / S.groups));
        // two lines' rows: the quickest tile, the best one below 2 MB; one line of a skewed tile's two is its neighbour's
        if (m.lines == 2) e += 0.016 + 0.061 * std::min(3.0, std::max(-2.0, std::log2(traffic / 2e6)));
        if (m.size_p0 < S.line) e += 0.374;
        const double cus_wanted = std::min(256.0, std::max(1.0, (double)P.elements * P.eb_a / 4096.0));
        if (C.kp.num_tiles < cus_wanted) e += 0.38 * (cus_wanted - C.kp.num_tiles) / 256.0;
    }
    // The models were fitted before this kernel's arguments were packed.  Time of its first candidate over the micro-tile kernel's,
    // beyond what the two models have: packed 0.76 below 8 MB (196 problems), 0.81 from 8 to 20 (161), 0.75 to 40 (107), 0.89 to 60
    // (69) and 0.92 to 100 (90); not packed 0.99, 1.04 and 0.90 (210 up to 40 MB).  More than this would take places from the gather
    // kernel, whose arguments are packed as well.  Over 3760 problems of 2.5 MB to 1.9 GB this, gather_cost()'s bonus and block_cost()'s
    // choose 0.9 % better than 0.12 here between 8 and 40 MB alone, packed or not, did, and 86 problems instead of 130 take more than 1.05
    // times what they took before any arguments were packed (13061 x 72 fp64 -> fp32 (1,0) 6.0 -> 4.3 us).
    // Updates whose lanes load eight vectors of A are packed in ranges only: with half for these, 1.01, 0.99 and 1.01 (rotation, one pair, new
    // tensors; 170 problems whose first candidate that changes).
    const bool packed = small_line(micro_args(C), P.epilogue, P.kind_a >= kKindC64, S.passes) != 0;
    e -= (packed ? 0.12 : 0.06) * octaves(traffic, 4e6, 8e6) * (1.0 - octaves(traffic, 40e6, 80e6));
    bool b_order = true;
    for (int i = 0; i < P.ndim; ++i) if (C.tile_order[i] != P.perm[i]) b_order = false;
    if (!b_order) e += 0.08;
    if (rows * P.eb_b < 64.0) e += 0.25 * std::log2(64.0 / (rows * P.eb_b));          // outside the fitted range: most of a tile's rows are not there
    return std::exp(e);
}

// Whether the line kernel has candidates, tiles in B's order, that run in one range per XCD.
static bool lines_in_ranges(const Problem& P)
{
    for (int merged = 0; merged < 4; ++merged)
        for (int cols : {16, 32, 64})
            for (int lines : {4, 8, 2}) {
                Candidate c;
                if (make_line_candidate(P, cols, lines, P.perm, (merged & 1) != 0, (merged & 2) != 0, &c) && c.kp.xcd_remap == 1) return true;
            }
    return false;
}

// The gather kernel against the others.  For problems that the caches hold the families' first candidates take, to
// within 10-13 %, 3.4 us + 0.18 us per MB of traffic (line), 3.9 + 0.19 (micro-tile), 2.4 + 0.15 (row) and 5.6 + 0.20 (box), by
// timings from before arguments were packed; the gather kernel's modelled time against the line kernel's, whose candidates cost
// about 0.86 there.  (Large problems are further from the fit: a margin.)  Packed, it gained what the line kernel did, and has that
// one's bonus up to 12 MB, fading out to 20, where the stride-1 index moves (elsewhere the row kernel is the alternative).  From 16 MB on it
// keeps its distance to the line kernel's candidates with one range per XCD, which rank up to 12 % better there, if the problem has such
// candidates and B is dense, or A's first index is B's second (neighbouring columns of B then read the same lines of A).  Time of the gather kernel over that of the first candidate without this
// term, in rotation, on one pair and on new tensors, problems of 15 to 65 MB in which it decides: 0.88, 0.84 and 1.00 (169); in the others,
// without line tiles in ranges or between leading dimensions, it would be 1.23, 1.23 and 1.22 (77; 5 x 14 x 20 x 102 x 12 complex64 reversed
// 34 us, box kernel 11.7).
static double gather_cost(const Problem& P, const Candidate& C)
{
    const double traffic = traffic_bytes(P), mb = traffic * 1e-6;
    const double packed = P.perm[0] != 0 ? 0.12 * octaves(traffic, 4e6, 8e6) * (1.0 - octaves(traffic, 12e6, 20e6)) : 0.0;
    const double distance = traffic >= 16e6 && (C.rows.flat || P.perm[1] == 0) && lines_in_ranges(P) ? 0.05 : 0.0;       // (P.perm[0] == 0: there are none)
    return 0.86 * (1.0 + 0.004 * mb) * C.model_us / (3.4 + 0.18 * mb) * std::exp(-packed - distance);
}

// The block kernel's ranking model, log-linear, fitted to the timings of every block candidate of 112 problems of 9 MB to 1.9 GB of
// traffic (every type; the first index of A or of B short, or the two runs overlapping) against the candidate that the other
// models rank first, above and below 100 MB.  By it the first block candidate is 3-4 % behind the best one, and the joint
// choice takes 8 % (large) and 10 % (small) off the time of the others' first; the best of all would take 10 % and 13 %.  The
// constants are 0.04 above the fit's, widening 0.06 to 0.1, so that near ties stay where they were.
static double block_cost(const Problem& P, const Candidate& C)
{
    const BlockParams& m = C.block;
    const AccessShape sh = access_shape(P, C);
    const bool update = P.epilogue == TTC_EPI_AXPBY;
    const double traffic = traffic_bytes(P);
    const bool large = traffic >= 100e6;
    double e = large ? -0.344 + (update ? 0.056 : 0.0) + (P.eb_b > P.eb_a ? 0.22 : 0.0)
                     : -0.351 - (update ? 0.042 : 0.0) + (P.eb_b > P.eb_a ? 0.22 : 0.0);
    // The device starts a workgroup of 256 threads every 1.7 ns (tiles of 0.5 to 4 KB, every type): what a small tile costs.
    const double starts = 1.7e-3 * C.kp.num_tiles / (traffic / 6.2e6);
    e += std::log(1.0 + std::pow(starts, 6.0)) / 6.0;
    const double tile_bytes = (double)m.rows * m.run_a * P.eb_a;
    if (tile_bytes > 8192.0) e += (large ? 0.044 : 0.085) * std::log2(tile_bytes / 8192.0);
    // eight vectors of A and eight of B a lane: few wavefronts fit, which a short launch does not make up for (25 x 13 x 4 x 26 x 19 x 5
    // fp32 reversed with an update 17.0 us, the line kernel 14.6)
    if (!large && update && m.unroll == 8) e += 0.12;
    // lines that a run shares with another one, per line of the run
    e += (large ? 0.072 : 0.18) * (1.0 - sh.align[0] / 128.0) * 128.0 / sh.run[0];
    e += (large && update ? 0.106 : 0.34) * (1.0 - sh.align[1] / 128.0) * 128.0 / sh.run[1];
    for (int k = 0; k < P.ndim && large; ++k) e += 0.19 * std::log((double)ceil_div(P.size[k], C.tile[k]) * C.tile[k] / (double)P.size[k]);
    e += 0.025 * std::log2(std::max(1.0, C.lds_conflict_b / 2.0));
    for (int i = 0; i < P.ndim; ++i) if (C.tile_order[i] != P.perm[i]) { e += large ? 0.054 : 0.006; break; }
    if (C.kp.num_tiles < 512) e += 0.19 * std::log2(512.0 / C.kp.num_tiles);
    // Against the micro-tile kernel where neither splits lines: time of this kernel's first candidate over that one's, beyond what the
    // two models have.  Copies and scaled copies, pairs in rotation and one pair: 0.93 and 0.91 below 40 MB (62 problems), 1.13 and
    // 0.95 up to 100 (23), 1.02 and 1.09 above (55).  Updates of 90 to 700 MB per tensor, in rotation, on one pair and on new tensors (60
    // problems, medians of six first passes), where the models have 0.92 in the mean: if A's first index is not B's second, 0.98, 1.11 and
    // 1.07 below 256 MB, 1.00, 1.18 and 1.14 above; if it is, 0.93, 1.00 and 0.98 below, and above 0.98, 1.09 and 1.10 but for three
    // fp32 problems at 0.74 to 0.80.
    // whether no index but the first starts inside a piece of a line that long; `joined`: first and second taken as one
    auto whole = [&](int bytes, bool joined) {
        for (int i = 1; i < P.ndim; ++i) {
            const bool second = joined && i == 1 && P.ndim > 2;
            if (!(second && P.stride_a[1] == P.size[0]) && P.stride_a[i] * P.eb_a % bytes != 0) return false;
            if (!(second && P.stride_b[P.perm[1]] == P.size[P.perm[0]]) && P.stride_b[P.perm[i]] * P.eb_b % bytes != 0) return false;
        }
        return true;
    };
    if (P.eb_a == P.eb_b && P.eb_a < 16) {                               // the micro-tile kernel's types
        if (!update && whole(64, false)) e += 0.06 * octaves(traffic, 30e6, 40e6);
        if (update && whole(128, true))
            e += P.perm[1] == 0 ? 0.12 * octaves((double)P.elements * P.eb_b, 190e6, 380e6) : 0.10 * octaves(traffic, 30e6, 40e6);
    }
    // Small problems: the line and the gather kernel have a bonus for their packed arguments, of which half is this kernel's due.
    e -= 0.06 * octaves(traffic, 4e6, 8e6) * (1.0 - octaves(traffic, 12e6, 20e6));
    // towards the end of the fitted range and below it a launch is what a problem costs, and the gather kernel is ahead (12 x 28 x
    // 1898 complex64 (1,0,2) with an update, 15 MB: 4.5 us against 5.6)
    if (traffic < 48e6) e += 0.1 * std::log2(48e6 / traffic);
    return std::exp(e);
}

static double heuristic_cost(const Problem& P, const Candidate& C)
{
    if (C.kernel_class == kKernelBlock) return block_cost(P, C);
    if (C.kernel_class == kKernelGather) return gather_cost(P, C);
    if (C.kernel_class == TTC_KERNEL_ROWS) return rows_cost(P, C);
    if (C.kernel_class == kKernelLines) return line_cost(P, C);
    if (C.kernel_class == TTC_KERNEL_MICRO) return micro_cost(P, C);
    // Weights fitted to timings of every candidate of 105 problems on MI355X (the benchmark workloads, 3-D and
    // 5-D problems with odd extents, a 57-case benchmark drawn by the paper's rules, power-of-two shapes): log-linear least
    // squares weighted towards the fast candidates, penalties constrained to be penalties, a small ridge term,
    // checked by holding problems out; rounded, with guard rails outside the measured range (runs under 64
    // bytes, small problems).
    const KernelParams& kp = C.kp;
    const double eb_a = P.eb_a, eb_b = P.eb_b;
    const bool direct = (C.kernel_class == TTC_KERNEL_DIRECT);
    const bool reads_b = (P.epilogue == TTC_EPI_AXPBY);
    auto oct_below = [](double x, double ref) { return x < ref ? std::log2(ref / x) : 0.0; };
    double volume = 1, padded = 1;
    for (int k = 0; k < P.ndim; ++k) {
        volume *= kp.tile[k];
        padded *= (double)ceil_div(P.size[k], kp.tile[k]) * kp.tile[k] / (double)P.size[k];
    }
    const double tile_bytes = volume * eb_a;
    const AccessShape sh = access_shape(P, C);
    const double run_a = sh.run[0], run_b = sh.run[1], seg_a = sh.seg[0], seg_b = sh.seg[1];
    const int vec_b = direct ? kp.a.vec : kp.b.vec;
    bool b_order = true, a_order = true;
    for (int i = 0; i < P.ndim; ++i) {
        if (C.tile_order[i] != P.perm[i]) b_order = false;
        if (C.tile_order[i] != i) a_order = false;
    }
    const bool order_a = !b_order && a_order, order_mixed = !b_order && !a_order;
    double e = 0.0;
    // coalescing: the contiguous run per tile and the contiguous piece per wavefront instruction; where runs
    // are whole lines their length counts for more (nothing is shared with a neighbour that could hide it)
    e += 0.002 * oct_below(run_a, 1024.0) + 0.016 * oct_below(run_b, 1024.0);
    e += 0.15 * oct_below(run_a, 64.0) + 0.20 * oct_below(run_b, 64.0);
    e += 0.015 * oct_below(seg_a, 256.0) + 0.025 * oct_below(seg_b, 256.0);
    e += 0.066 * oct_below(seg_a, 64.0) + 0.10 * oct_below(seg_b, 64.0);
    if (sh.align[0] >= 128) e += 0.026 * oct_below(run_a, 1024.0) - 0.004 * oct_below(run_a, 256.0);
    if (sh.align[1] >= 128) e += 0.007 * oct_below(run_b, 2048.0);
    // runs that start or end inside a line: lines_shared = what a run shares with its neighbours per 128
    // bytes it moves; requests = line (A) or 64-byte write (B) requests per line or 64 bytes moved, minus one.
    // On the B side both cost more when the tiles that share the line run far apart in time (tile ids in
    // A's order).
    const double lines_shared_a = (1.0 - sh.align[0] / 128.0) * 128.0 / run_a;
    const double requests_a = ((run_a + 128.0 - std::min(sh.align[0], 128)) / 128.0) * 128.0 / run_a - 1.0;
    const double lines_shared = (1.0 - sh.align[1] / 128.0) * 128.0 / run_b;
    const double requests = ((run_b + 64.0 - std::min(sh.align[1], 64)) / 64.0) * 64.0 / run_b - 1.0;
    e += 0.014 * lines_shared_a + 0.014 * requests_a + 0.0705 * requests;
    if (order_a) e += 0.002 + 0.065 * lines_shared + 0.124 * requests;
    if (order_mixed) e += -0.010 + 0.021 * lines_shared;
    e -= 0.0568 * (kp.nt_a + kp.nt_b);                                  // sides that stream (whole lines only)
    e += (kp.a.vec * eb_a >= 16 ? 0.0 : (kp.a.vec * eb_a >= 8 ? 0.037 : 0.057));
    e += (vec_b * eb_b >= 8 ? 0.0 : 0.005);
    if (!direct && kp.b.partial) e -= 0.016;
    e += 0.214 * (padded - 1.0);                                        // lanes idle in remainder tiles
    // tile size and occupancy
    e += 0.2035 * oct_below(tile_bytes, 8192.0);
    if (tile_bytes > 16384.0) e -= 0.0626 * std::log2(tile_bytes / 16384.0);
    if (tile_bytes > 32768.0) e += 0.0629 * std::log2(tile_bytes / 32768.0);
    const double lane_a = (double)kp.a.n_iter * kWave * kp.a.vec / volume;
    e += 0.052 * (lane_a - 1.0);
    double groups = 16.0, resident_waves = 32.0;
    if (direct) {
        // no regrouping through LDS: every instruction's piece meets memory as it is
        e += 0.0436 + 0.0555 * ((1.0 - sh.align[0] / 128.0) * 128.0 / seg_a + (1.0 - sh.align[1] / 128.0) * 128.0 / seg_b);
    } else {
        groups = std::min(16.0, std::floor(160.0 * 1024 / C.lds_bytes));
        resident_waves = std::min(32.0, groups * (C.threads / kWave));
        if (kp.lds_buffers == 1) e += reads_b ? 0.005 : 0.002;
        const double lane_b = (double)kp.b.n_iter * kWave * kp.b.vec / volume;
        e += 0.006 * (lane_b - 1.0);
    }
    if (resident_waves < 16.0) e += 0.233 * (16.0 - resident_waves) / 16.0;
    if (resident_waves < 8.0) e += 0.277 * (8.0 - resident_waves) / 8.0;
    if (groups < 4.0) e += 0.061 * (4.0 - groups) / 4.0;
    // launch shape: measured preference
    if (C.threads == 128) e -= reads_b ? 0.0744 : 0.0259;
    else if (C.threads == 512) e += 0.0285;
    if (C.wg_per_cu == 4) e += 0.022;
    else if (C.wg_per_cu == 8) e += 0.0225;
    // too few tiles to fill the chip (a problem too small for 2048 tiles of 8 KB is not pushed below 8 KB)
    const double tiles_wanted = std::min(2048.0, std::max(1.0, (double)P.elements * eb_a / 8192.0));
    if (kp.num_tiles < tiles_wanted) e += 1.28 * (tiles_wanted - kp.num_tiles) / 2048.0;
    // small problems (outside the fitted range): a tile per compute unit comes before large tiles
    const double cus_wanted = std::min(256.0, std::max(1.0, (double)P.elements * eb_a / 4096.0));
    if (kp.num_tiles < cus_wanted) e += 1.5 * (cus_wanted - kp.num_tiles) / 256.0;
    // ... and what tables, set-up and barriers cost in a problem that the caches hold (the times beside gather_cost): 33 %
    // at 1 MB, 13 % at 16 MB
    const double mb = traffic_bytes(P) * 1e-6;
    e += std::max(0.0, std::log((5.56 + 0.199 * mb) / (3.4 + 0.18 * mb)) - 0.207);
    return std::exp(e);
}

static bool same_config(const Candidate& x, const Candidate& y)
{
    if (x.kernel_class != y.kernel_class || x.threads != y.threads || x.wg_per_cu != y.wg_per_cu) return false;
    if (x.rows.unroll != y.rows.unroll) return false;
    if (x.kp.a.vec != y.kp.a.vec || x.kp.b.vec != y.kp.b.vec || x.kp.lds_buffers != y.kp.lds_buffers) return false;
    for (int k = 0; k < kMaxDim; ++k) {
        if (x.tile[k] != y.tile[k]) return false;
        if (x.kp.tile_below[k].div != y.kp.tile_below[k].div) return false;
    }
    for (int i = 0; i < kBoxDims; ++i)
        if (x.dlane_a[i] != y.dlane_a[i] || x.dlane_b[i] != y.dlane_b[i] || x.dtile_a[i] != y.dtile_a[i] ||
            x.dtile_b[i] != y.dtile_b[i]) return false;
    return true;
}

// Non-temporal hints by rule: a side streams if all its runs are whole 128-byte lines.  Then no line is
// shared with a neighbouring tile, and keeping it in cache would only displace lines that are.  (The timed
// search tries the other settings on its finalists.)
void default_streaming(const Problem& P, Candidate* c)
{
    if (c->kernel_class == kKernelGather) { c->kp.nt_a = c->kp.nt_b = 0; return; }      // lines of A are fetched several times, B is small
    if (c->kernel_class == TTC_KERNEL_ROWS) {
        // B is written front to back: streamed.  A is read once, but rows that start inside lines share them, and a
        // tensor of a quarter of the last-level cache may still be there: streamed only if it is larger and its rows
        // are whole lines or long (25 MB problems run 13 % faster without, 200 MB ones with 128-byte to 64 KB rows
        // 3 % faster with the hint, 340- and 532-byte rows 5-8 % slower).
        const int64_t row_bytes = P.size[0] * P.eb_a;
        bool whole = row_bytes % kLineBytes == 0;
        for (int k = 1; k < P.ndim; ++k) if (P.stride_a[k] * P.eb_a % kLineBytes != 0) whole = false;
        c->kp.nt_a = P.elements * P.eb_a >= (int64_t(64) << 20) && (whole || row_bytes >= 1024) ? 1 : 0;
        c->kp.nt_b = 1;
        return;
    }
    if (c->kernel_class == kKernelLines) {
        // B's lines are written once and whole: streamed (A's rows then stay in the caches: tiles share them where
        // they are skewed or A's runs split lines; both sides streamed is 14 % slower on the average of such problems,
        // neither side 13 %).  A is streamed too where nothing of it is shared, B is not read and A exceeds half the
        // last-level cache (1.6 % faster; at smaller sizes 14 % slower if A was written not long ago; with an update 0-12 %).  Below 8 MB of traffic everything stays in the
        // caches and the hints make no difference: none, B's reader comes next.
        const MicroParams& m = c->kp.micro;
        bool whole_a = !m.skewed && P.epilogue != TTC_EPI_AXPBY && P.elements * P.eb_a >= (int64_t(128) << 20);
        for (int k = 1; k < P.ndim; ++k)
            if (!(m.merged_a && k == 1) && P.stride_a[k] * P.eb_a % kLineBytes != 0) whole_a = false;
        c->kp.nt_a = whole_a ? 1 : 0;
        c->kp.nt_b = traffic_bytes(P) >= 8e6 ? 1 : 0;
        return;
    }
    const AccessShape sh = access_shape(P, *c);
    if (c->kernel_class == kKernelBlock) {
        // Whole lines of B, and long runs, which share their two ends only, are streamed: 5-10 % faster from 1 KB runs on in
        // problems of 100 MB and more (256-byte runs 3-7 % slower, shorter ones up to 30 %), and from 256 bytes on in smaller ones.
        // So are A's in the large problems if they are whole lines (2 %) or at least 4 KB long (1 %); smaller problems keep
        // A in the caches (2 %).  By the medians of 112 problems.
        const bool large = traffic_bytes(P) >= 100e6;
        c->kp.nt_a = large && (sh.align[0] >= 128 || sh.run[0] >= 4096) ? 1 : 0;
        c->kp.nt_b = sh.align[1] >= 128 || sh.run[1] >= (large ? 1024 : 256) ? 1 : 0;
        return;
    }
    c->kp.nt_a = (sh.align[0] >= 128) ? 1 : 0;
    c->kp.nt_b = (sh.align[1] >= 128) ? 1 : 0;
    if (c->kernel_class == TTC_KERNEL_MICRO && P.epilogue == TTC_EPI_AXPBY && sh.align[0] >= 32 && sh.align[1] >= 32) {
        // B is read and written by the same lane within a few hundred cycles, and runs that start on 32-byte
        // boundaries split no memory transaction with a neighbour: with both sides streamed 72^4 fp64 (rows of 576
        // bytes) runs at 98-105 % of a copy against 77-88 % by the rule above.  (Runs that start anywhere,
        // 24x20x16x18x22x17 with its 68-byte steps in B, lose up to 20 % that way and keep the rule.)
        c->kp.nt_a = c->kp.nt_b = 1;
    }
    if (c->kernel_class == TTC_KERNEL_DIRECT) c->kp.nt_a = c->kp.nt_b = (c->kp.nt_a && c->kp.nt_b) ? 1 : 0;   // both or neither
}

// what same_config() compares, folded into one number: candidates are looked up by it instead of being
// compared with every earlier one
static uint64_t config_hash(const Candidate& c)
{
    uint64_t h = 1469598103934665603ull;
    auto mix = [&](int64_t x) { h = (h ^ (uint64_t)x) * 1099511628211ull; };
    mix(c.kernel_class); mix(c.threads); mix(c.wg_per_cu); mix(c.rows.unroll);
    mix(c.kp.a.vec); mix(c.kp.b.vec); mix(c.kp.lds_buffers);
    for (int k = 0; k < kMaxDim; ++k) { mix(c.tile[k]); mix(c.kp.tile_below[k].div); }
    for (int i = 0; i < kBoxDims; ++i) { mix(c.dlane_a[i]); mix(c.dlane_b[i]); mix(c.dtile_a[i]); mix(c.dtile_b[i]); }
    return h;
}

struct CandidateList {
    std::vector<Candidate>& v;
    std::unordered_multimap<uint64_t, size_t> seen;
    explicit CandidateList(std::vector<Candidate>& out) : v(out) {}
};

static void add_candidate(const Problem& P, CandidateList& L, const Candidate& c)
{
    const uint64_t h = config_hash(c);
    const auto range = L.seen.equal_range(h);
    for (auto it = range.first; it != range.second; ++it)
        if (same_config(L.v[it->second], c)) return;
    L.seen.emplace(h, L.v.size());
    L.v.push_back(c);
    default_streaming(P, &L.v.back());
    L.v.back().score = heuristic_cost(P, L.v.back());
}

static int max_vec(int eb, int64_t extent)
{
    int v = std::max(1, 16 / eb);
    while (v > 1 && extent % v != 0) v /= 2;
    return v;
}

// Launch shapes tried for every tile shape: workgroup size and workgroups per compute unit.
struct LaunchShape { int threads, wg_per_cu; };
static const LaunchShape kLaunchShapes[] = {{256, 16}, {128, 8}, {256, 8}, {128, 16}, {256, 4}, {512, 8}, {64, 32},
                                            {256, 0}, {128, 0}, {512, 0}};      // 0: what a compute unit holds at once

// Different run-length targets often ask for the same box: each (box, vector rule, kernel family) is expanded once.
struct ShapesSeen {
    struct Key { int t[kMaxDim]; int vec, family; };
    std::vector<Key> keys;
    bool first_time(const int* t, int vec, int family)
    {
        for (const Key& k : keys) {
            bool same = (k.vec == vec && k.family == family);
            for (int i = 0; same && i < kMaxDim; ++i) same = (k.t[i] == t[i]);
            if (same) return false;
        }
        Key k;
        for (int i = 0; i < kMaxDim; ++i) k.t[i] = t[i];
        k.vec = vec; k.family = family;
        keys.push_back(k);
        return true;
    }
};

// quick: only the variants the ranking prefers (both walks merged, the two favoured launch shapes) -- what
// ttc_plan_create pays for; the full list is built when something first asks for it.
static void enumerate(const Problem& P, std::vector<Candidate>& out_list, bool quick)
{
    out_list.reserve(quick ? 2048 : 16384);      // a candidate is a few KB: no regrowth copies
    CandidateList out(out_list);
    ShapesSeen shapes;
    LayoutCache cache;
    const int n = P.ndim;
    const int eb = std::max(P.eb_a, P.eb_b);
    int order_a[kMaxDim], order_b[kMaxDim];
    for (int k = 0; k < kMaxDim; ++k) { order_a[k] = k; order_b[k] = (k < n) ? P.perm[k] : k; }
    const bool stride1_fixed = (P.perm[0] == 0);
    // Tile orders (which index varies fastest from one tile id to the next): B's index order, A's, and the
    // two mixed ones that put the other tensor's stride-1 index first, so that tiles sharing a cache line
    // at the end of a run are in flight together on BOTH sides.
    int order_ab[kMaxDim], order_ba[kMaxDim];
    {
        int na = 0, nb = 0;
        order_ab[na++] = 0;
        for (int i = 0; i < kMaxDim; ++i) if (order_b[i] != 0) order_ab[na++] = order_b[i];
        order_ba[nb++] = order_b[0];
        for (int i = 0; i < kMaxDim; ++i) if (order_a[i] != order_b[0]) order_ba[nb++] = order_a[i];
    }
    const int* orders[4] = {order_b, order_a, order_ab, order_ba};
    const int norders = stride1_fixed ? 2 : 4;
    const int nshapes = quick ? 2 : (int)(sizeof(kLaunchShapes) / sizeof(kLaunchShapes[0]));

    // -- the row kernel: only when the stride-1 index keeps its place (or there is one index only)
    if (stride1_fixed) {
        const int vwide = std::max(1, 16 / eb);
        for (int v = vwide; v >= 1; v /= 2) {
            for (int unroll : {1, 2, 4, 8}) {
                Candidate c;
                // a dense B is taken flat; only in the narrow forms, which the widest vector makes pointless, row by row
                if (v == vwide ? make_rows_candidate(P, v, unroll, true, &c) || make_rows_candidate(P, v, unroll, false, &c)
                               : make_rows_candidate(P, v, unroll, false, &c)) add_candidate(P, out, c);
                if (quick && unroll == 2) break;
            }
        }
    }

    // -- direct candidates: only when the stride-1 index keeps its place.  The box takes leading
    //    indices of A and of B so that both sides move a few long contiguous chunks per tile.
    if (stride1_fixed) {
        const int vfull = max_vec(eb, P.size[0]);
        const int64_t chunk_bytes[7] = {16384, 4096, 32768, 8192, 2048, 65536, 1024};
        const int vwide = std::max(1, 16 / eb);
        for (int vsel = 0; vsel < 3; ++vsel) {
            if (vsel == 1 && vfull == 1) continue;
            if (vsel == 2 && (vfull == vwide || P.stride_a[0] != 1 || P.stride_b[0] != 1)) continue;
            // 0: the widest vector that divides the rows; 1: scalar; 2: the widest vector, cut at the end of a run
            const int v = vsel == 0 ? vfull : (vsel == 1 ? 1 : 32);
            const int vmult = vsel == 0 ? vfull : 1;
            for (int style = 0; style < 2; ++style)
            for (int64_t ra : chunk_bytes)
                for (int64_t rb : chunk_bytes) {
                    int ta[kMaxDim], tb[kMaxDim], t[kMaxDim];
                    build_group(P, order_a, P.eb_a, ra / P.eb_a, vmult, kBoxDims, ta, style);
                    build_group(P, order_b, P.eb_b, rb / P.eb_b, vmult, kBoxDims, tb, style);
                    int64_t vol = 1;
                    int spanned = 0;
                    for (int k = 0; k < kMaxDim; ++k) t[k] = std::max(ta[k], tb[k]);
                    for (int k = 0; k < n; ++k) { vol *= t[k]; spanned += (t[k] > 1); }
                    if (spanned > kBoxDims || vol * eb > 128 * 1024) continue;
                    if (vol * eb < 4096 && vol < P.elements) continue;
                    if (!shapes.first_time(t, v, 0)) continue;
                    for (int o = 0; o < norders; ++o)
                        for (int li = 0; li < nshapes; ++li) {
                            const LaunchShape& ls = kLaunchShapes[li];
                            Candidate c;
                            if (make_candidate(P, t, v, true, ls.threads, ls.wg_per_cu, orders[o], kDefaultTileMapping, &c))
                                add_candidate(P, out, c);
                        }
                }
        }
    }

    // -- the micro-tile kernel: a tile over the two stride-1 indices.  Tile extents in vectors: powers of two, and
    // the divisors of the extent (no remainder tiles)
    if (!stride1_fixed && n >= 2) {
        const int vec = std::max(1, 16 / P.eb_a);
        auto extents = [&](int64_t size, bool divisors, std::vector<int>* v) {
            const int64_t whole = size / vec;
            for (int l = 8; l <= 64; l *= 2) if (l <= 2 * whole) v->push_back(l);
            if (size % vec == 0 && divisors)
                for (int l = 6; l <= 96; ++l)
                    if (whole % l == 0 && (l & (l - 1)) != 0) v->push_back(l);
            if (whole >= 1 && whole < 8) v->push_back((int)ceil_div(size, vec));
            if (size % vec != 0 && whole >= 8) {               // the whole extent in one tile, or in two: no run shared between tiles
                const int64_t all = ceil_div(size, vec);
                if (all <= 96) v->push_back((int)all);
                if (all >= 16 && ceil_div(all, 2) <= 96) v->push_back((int)ceil_div(all, 2));
            }
        };
        // the column index: A's index 0, or (short rows) indices 0 and 1 as one; the row index likewise on B's side
        const int p0 = P.perm[0], p1 = P.perm[1];
        for (int merge_a = 0; merge_a < 2; ++merge_a)
            for (int merge_b = 0; merge_b < 2; ++merge_b) {
                if (merge_a && (n < 3 || P.size[0] * P.eb_a > 1024 || p0 == 1)) continue;
                if (merge_b && (n < 3 || P.size[p0] * P.eb_a > 1024 || p1 == 0)) continue;
                if (merge_a && merge_b && p1 == 1) continue;
                const int64_t cols = merge_a ? P.size[0] * P.size[1] : P.size[0], rows = merge_b ? P.size[p0] * P.size[p1] : P.size[p0];
                std::vector<int> las, lbs;
                extents(cols, !(quick && merge_a), &las);       // the short list: a merged index is cut at powers of two and whole rows only
                extents(rows, !(quick && merge_b), &lbs);
                // whole rows of the inner index: tiles that end where a run of the other tensor ends
                if (merge_a) for (int64_t k = 1; k * P.size[0] <= 96 * vec && k <= P.size[1]; ++k) if (k * P.size[0] % vec == 0) las.push_back((int)(k * P.size[0] / vec));
                if (merge_b) for (int64_t k = 1; k * P.size[p0] <= 96 * vec && k <= P.size[p1]; ++k) if (k * P.size[p0] % vec == 0) lbs.push_back((int)(k * P.size[p0] / vec));
                for (int threads : {256, 128, 64}) {
                    if (quick && threads == 64) continue;          // the model ranks one-wavefront workgroups behind the others
                    for (int la : las)
                        for (int lb : lbs) {
                            const int64_t blocks = ceil_div((int64_t)la * lb, threads);
                            if (blocks > 6 || (int64_t)la * lb * 5 < blocks * threads * 4) continue;      // lanes mostly busy
                            for (int o = 0; o < (quick ? 1 : 2); ++o) {       // the mixed orders, and the indices outside the tile first, time the same (384^3, 72^4, 6-D reversals)
                                Candidate c;
                                if (make_micro_candidate(P, la * vec, lb * vec, threads, orders[o], merge_a != 0, merge_b != 0, &c))
                                    add_candidate(P, out, c);
                            }
                        }
                }
            }
    }

    // -- the line kernel
    if (!stride1_fixed && n >= 2) {
        const int p0 = P.perm[0], p1 = P.perm[1];
        for (int merge_a = 0; merge_a < 2; ++merge_a)
            for (int merge_b = 0; merge_b < 2; ++merge_b) {
                if (merge_a && (n < 3 || p0 == 1)) continue;
                if (merge_b && (n < 3 || p1 == 0)) continue;
                for (int cols : {16, 32, 64})
                    for (int lines : {4, 8, 2})
                        for (int o = 0; o < (quick ? 1 : 2); ++o) {
                            Candidate c;
                            if (make_line_candidate(P, cols, lines, orders[o], merge_a != 0, merge_b != 0, &c)) add_candidate(P, out, c);
                        }
            }
    }

    // -- the block kernel
    if (!stride1_fixed && n >= 2) {
        std::vector<std::vector<int>> tried;
        for (int64_t ra : {128, 256, 512, 1024, 2048, 4096, 8192, 16384, 32768})
            for (int64_t rb : {128, 256, 512, 1024, 2048, 4096, 8192, 16384, 32768})
                for (int style = 0; style < 2; ++style) {
                    int ta[kMaxDim], tb[kMaxDim], t[kMaxDim];
                    build_group(P, order_a, P.eb_a, ra / P.eb_a, max_vec(P.eb_a, P.size[0]), 3, ta, style);
                    build_group(P, order_b, P.eb_b, rb / P.eb_b, max_vec(P.eb_b, P.size[P.perm[0]]), 3, tb, style);
                    for (int k = 0; k < kMaxDim; ++k) t[k] = std::max(ta[k], tb[k]);
                    // the other tensor's group may have cut an index that vectors run along anywhere
                    const int p0 = P.perm[0];
                    t[0] = (int)std::min<int64_t>(P.size[0], round_up(t[0], max_vec(P.eb_a, P.size[0])));
                    t[p0] = (int)std::min<int64_t>(P.size[p0], round_up(t[p0], max_vec(P.eb_b, P.size[p0])));
                    const std::vector<int> key(t, t + kMaxDim);
                    if (std::find(tried.begin(), tried.end(), key) != tried.end()) continue;
                    tried.push_back(key);
                    for (int o = 0; o < (quick ? 1 : 2); ++o) {
                        Candidate c;
                        if (make_block_candidate(P, t, orders[o], &c)) add_candidate(P, out, c);
                    }
                }
    }

    // -- staged candidates: a box spanning the leading indices of A and of B
    if (n >= 2) {
        const int p0 = P.perm[0];
        const int va_full = max_vec(P.eb_a, P.size[0]);
        const int vb_full = max_vec(P.eb_b, P.size[p0]);
        const int64_t run_bytes[8] = {256, 512, 128, 1024, 64, 2048, 4096, 8192};
        const bool odd_rows = va_full < std::max(1, 16 / P.eb_a) || vb_full < std::max(1, 16 / P.eb_b);
        for (int vsel = 0; vsel < 3; ++vsel) {
            if (vsel == 2 && !odd_rows) continue;
            // 0: the widest vectors that divide the runs; 1: scalar; 2: the widest vectors, cut at the end of a run
            const int va = vsel == 0 ? va_full : 1;       // multiples the group builder keeps on the stride-1 extents
            const int vb = vsel == 0 ? vb_full : 1;
            const int vec_limit = vsel == 0 ? 16 : (vsel == 1 ? 1 : 32);
            for (int md = 3; md >= 1; --md)
              for (int style = 0; style < 2; ++style)
                for (int64_t ra : run_bytes)
                    for (int64_t rb : run_bytes) {
                        int ta[kMaxDim], tb[kMaxDim], t[kMaxDim];
                        build_group(P, order_a, P.eb_a, std::max<int64_t>(1, ra / P.eb_a), va, md, ta, style);
                        build_group(P, order_b, P.eb_b, std::max<int64_t>(1, rb / P.eb_b), vb, md, tb, style);
                        int64_t vol = 1;
                        int spanned = 0;
                        for (int k = 0; k < kMaxDim; ++k) t[k] = std::max(ta[k], tb[k]);
                        for (int k = 0; k < n; ++k) { vol *= t[k]; spanned += (t[k] > 1); }
                        if (spanned > kBoxDims) continue;
                        if (vol * P.eb_a > kMaxLdsBytes - 2048) continue;
                        if (vol * eb < 2048 && md > 1 && vol < P.elements) continue;
                        if (!shapes.first_time(t, vec_limit, 1)) continue;
                        for (int nbuf = 2; nbuf >= 1; --nbuf) {
                            if (nbuf == 1 && vol * eb < 8192) continue;     // small tiles can afford two buffers
                            for (int mg = 0; mg < (quick ? 1 : 4); ++mg)
                                for (int o = 0; o < norders; ++o)
                                    for (int li = 0; li < nshapes; ++li) {
                                        const LaunchShape& ls = kLaunchShapes[li];
                                        Candidate c;
                                        if (make_candidate(P, t, vec_limit, false, ls.threads, ls.wg_per_cu, orders[o], kDefaultTileMapping,
                                                           &c, (mg & 1) == 0, (mg & 2) == 0, &cache, nbuf))
                                            add_candidate(P, out, c);
                                    }
                        }
                    }
        }
    }

    // -- the gather kernel
    {
        Candidate c;
        if (make_gather_candidate(P, &c)) add_candidate(P, out, c);
    }

    // -- last resort so that every problem has a candidate: scalar direct walk in A order
    if (out_list.empty() || n == 1) {
        int t[kMaxDim];
        build_group(P, order_a, P.eb_a, 16384 / eb, 1, kBoxDims, t);
        Candidate c;
        if (make_candidate(P, t, 1, true, 256, 8, order_a, kDefaultTileMapping, &c)) add_candidate(P, out, c);
    }
}

int build_plan(int dtype, int ndim, const int64_t* sizes, const int* perm, const int64_t* lda, const int64_t* ldb,
               const void* alpha, const void* beta, ttc_plan_s* plan)
{
    Problem& P = plan->prob;
    int st = normalise(dtype, ndim, sizes, perm, lda, ldb, alpha, beta, &P);
    if (st != TTC_OK) return st;
    std::vector<Candidate> quick;
    enumerate(P, quick, true);
    if (quick.empty()) enumerate(P, quick, false);
    if (quick.empty()) return TTC_ERR_OVERFLOW;
    size_t best = 0;
    for (size_t i = 1; i < quick.size(); ++i) if (quick[i].score < quick[best].score) best = i;
    plan->cands.assign(1, quick[best]);
    plan->selected = 0;
    plan->complete = false;
    if (verbose()) {
        const Candidate& c = plan->cands[0];
        static const char* const names[] = {"direct", "staged", "row", "micro-tile", "line", "gather", "block"};       // by kernel class
        constexpr int kClasses = (int)(sizeof(names) / sizeof(names[0]));
        static_assert(TTC_KERNEL_MICRO == 3 && kKernelLines == 4 && kKernelGather == 5 && kKernelBlock == kClasses - 1, "one name per class");
        std::fprintf(stderr, "ttc: plan dtype %d, %d fused indices, %s kernel, tile", P.dtype, P.ndim, names[c.kernel_class]);
        for (int k = 0; k < P.ndim; ++k) std::fprintf(stderr, " %d", c.tile[k]);
        size_t per_class[kClasses] = {0};
        for (const Candidate& q : quick) ++per_class[q.kernel_class];
        std::fprintf(stderr, ", vectors %d/%d, %d threads, %d B LDS, cost %.4f (best of %zu candidates of the short list:",
                     c.kp.a.vec, c.kp.b.vec, c.threads, c.lds_bytes, c.score, quick.size());
        for (int k = 0; k < kClasses; ++k) std::fprintf(stderr, "%s %zu %s", k ? "," : "", per_class[k], names[k]);
        std::fprintf(stderr, ")\n");
    }
    return TTC_OK;
}

// The ranked list of all candidates, built on first use.  Candidate 0 stays what ttc_plan_create chose (with
// whatever the caller has set on it since); the others follow in the order of the heuristic cost.
int complete_plan(ttc_plan_s* plan)
{
    if (plan->complete) return TTC_OK;
    const Candidate first = plan->cands[plan->selected];
    std::vector<Candidate> all;
    enumerate(plan->prob, all, false);
    std::stable_sort(all.begin(), all.end(), [](const Candidate& x, const Candidate& y) { return x.score < y.score; });
    std::vector<Candidate> ranked;
    ranked.reserve(all.size() + 1);
    ranked.push_back(first);
    for (const Candidate& c : all) if (!same_config(c, first)) ranked.push_back(c);
    plan->cands.swap(ranked);
    plan->selected = 0;
    plan->complete = true;
    if (verbose()) std::fprintf(stderr, "ttc: %zu candidates ranked\n", plan->cands.size());
    return TTC_OK;
}

}  // namespace ttc

// Nothing may throw across the C boundary: allocation failures and anything unexpected become status codes.
template <class F> static int guarded(F&& body)
{
    try { return body(); }
    catch (const std::bad_alloc&) { return TTC_ERR_ALLOC; }
    catch (...) { return TTC_ERR_INTERNAL; }
}

// The kernels instantiate a walk for a compile-time vector width; the replay picks the same one.
template <class S1, class S2>
static void emu_walk(const ttc::Side& s, const ttc::LaneState& L, const ttc::SideLim& lim, const ttc::WalkMask& m,
                     const ttc::PosEntry* tab, const ttc::PosCoord* tabc, uint32_t wave, S1&& s1, S2&& s2)
{
    switch (s.vec) {
    case 1: ttc::walk<4, 1>(s, L, lim, m, tab, tabc, wave, s1, s2); break;
    case 2: ttc::walk<4, 2>(s, L, lim, m, tab, tabc, wave, s1, s2); break;
    default: ttc::walk<4, 4>(s, L, lim, m, tab, tabc, wave, s1, s2); break;
    }
}

// ---------------------------------------------------------------------------------
// Host-only part of the C ABI
// ---------------------------------------------------------------------------------
extern "C" {

ttc_plan_t ttc_plan_create(int dtype, int ndim, const int64_t* sizes, const int* perm,
                           const void* alpha, const void* beta)
{
    return ttc_plan_create_ex(dtype, ndim, sizes, perm, nullptr, nullptr, alpha, beta);
}

ttc_plan_t ttc_plan_create_ex(int dtype, int ndim, const int64_t* sizes, const int* perm,
                              const int64_t* lda, const int64_t* ldb, const void* alpha, const void* beta)
{
    ttc_plan_s* plan = new (std::nothrow) ttc_plan_s();
    if (!plan) { ttc::set_last_status(TTC_ERR_ALLOC); return nullptr; }
    int st;
    try {
        st = ttc::build_plan(dtype, ndim, sizes, perm, lda, ldb, alpha, beta, plan);
    } catch (const std::bad_alloc&) {
        st = TTC_ERR_ALLOC;
    } catch (...) {
        st = TTC_ERR_INVALID_VALUE;
    }
    ttc::set_last_status(st);
    if (st != TTC_OK) { delete plan; return nullptr; }
    return plan;
}

int ttc_plan_destroy(ttc_plan_t plan)
{
    delete plan;
    return TTC_OK;
}

int ttc_last_status(void) { return ttc::g_last_status; }

const char* ttc_status_string(int status)
{
    switch (status) {
    case TTC_OK: return "ok";
    case TTC_ERR_INVALID_VALUE: return "invalid value";
    case TTC_ERR_INVALID_PERM: return "perm is not a permutation";
    case TTC_ERR_UNSUPPORTED_DTYPE: return "unsupported data type";
    case TTC_ERR_NULL_POINTER: return "null pointer";
    case TTC_ERR_ALIAS: return "A and B overlap";
    case TTC_ERR_OVERFLOW: return "size overflow";
    case TTC_ERR_HIP: return "HIP runtime error";
    case TTC_ERR_ALLOC: return "allocation failed";
    case TTC_ERR_MISALIGNED: return "pointer not aligned to the element size";
    case TTC_ERR_INTERNAL: return "internal error: a candidate's walk is not a bijection in bounds";
    case TTC_ERR_NOT_FOUND: return "no stored plan for this problem";
    case TTC_ERR_IO: return "the plan store could not be written";
    default: return "unknown status";
    }
}

int ttc_plan_get_info(ttc_plan_t plan, ttc_plan_info_t* out)
{
    if (!plan || !out) return TTC_ERR_NULL_POINTER;
    return guarded([&]() -> int {
    const ttc::Problem& P = plan->prob;
    const ttc::Candidate& C = plan->cands[plan->selected];
    std::memset(out, 0, sizeof(*out));
    out->dtype = P.dtype;
    out->ndim = P.ndim;
    for (int k = 0; k < P.ndim; ++k) {
        out->sizes[k] = P.size[k];
        out->perm[k] = P.perm[k];
        out->tile[k] = C.tile[k];
        out->tile_order[k] = C.tile_order[k];
        out->lds_stride[k] = C.lds_stride[k];
    }
    out->digits_a = C.digits_a;
    out->digits_b = C.digits_b;
    for (int i = 0; i < ttc::kBoxDims; ++i) {
        out->digit_tile_a[i] = C.dtile_a[i];  out->digit_lane_a[i] = C.dlane_a[i];
        out->digit_tile_b[i] = C.dtile_b[i];  out->digit_lane_b[i] = C.dlane_b[i];
    }
    out->stride1_fixed = (P.perm[0] == 0) ? 1 : 0;
    out->kernel_class = C.kernel_class == ttc::kKernelLines ? TTC_KERNEL_LDS : C.kernel_class == ttc::kKernelGather ? TTC_KERNEL_ROWS :
                        C.kernel_class == ttc::kKernelBlock ? TTC_KERNEL_MICRO : C.kernel_class;
    out->epilogue = P.epilogue;
    out->vec_a = C.kp.a.vec;
    out->vec_b = C.kp.b.vec;
    out->partial_a = C.kp.a.partial;
    out->partial_b = C.kp.b.partial;
    out->threads = C.threads;
    out->wg_per_cu = C.wg_per_cu;
    out->xcd_remap = C.kp.xcd_remap;
    out->lds_bytes = C.lds_bytes;
    out->lds_buffers = C.kp.lds_buffers;
    out->nt_a = C.kp.nt_a;
    out->nt_b = C.kp.nt_b;
    out->lds_conflict_a = C.lds_conflict_a;
    out->lds_conflict_b = C.lds_conflict_b;
    if (C.kernel_class == ttc::kKernelLines)
        ttc::line_conflicts(ttc::line_shape(C.kp.micro.ta, C.kp.micro.lines, P.eb_a, P.eb_b), P.eb_a, &out->lds_conflict_a, &out->lds_conflict_b);
    {
        const ttc::AccessShape sh = ttc::access_shape(P, C);
        out->run_bytes_a = sh.run[0]; out->run_bytes_b = sh.run[1];
        out->seg_bytes_a = sh.seg[0]; out->seg_bytes_b = sh.seg[1];
        out->align_a = sh.align[0];   out->align_b = sh.align[1];
    }
    out->num_tiles = C.kp.num_tiles;
    out->elements = P.elements;
    out->bytes_moved = P.elements * (P.eb_a + (P.epilogue == TTC_EPI_AXPBY ? 2 : 1) * P.eb_b);
    out->span_a = P.span_a;
    out->span_b = P.span_b;
    for (int k = 0; k < P.ndim; ++k) { out->stride_a[k] = P.stride_a[k]; out->stride_b[k] = P.stride_b[k]; }
    out->candidate_index = plan->selected;
    out->candidate_count = (int)plan->cands.size();
    out->tuned_ms = C.tuned_ms;
    out->heuristic_cost = C.score;
    out->merged = (C.kernel_class == TTC_KERNEL_MICRO || C.kernel_class == ttc::kKernelLines) ? (C.kp.micro.merged_a | (C.kp.micro.merged_b << 1)) :
                  C.kernel_class == ttc::kKernelBlock ? 4 : 0;
    out->unroll = C.kernel_class == TTC_KERNEL_ROWS ? C.rows.unroll :
                  C.kernel_class == TTC_KERNEL_MICRO ? C.kp.micro.blocks : C.kernel_class == ttc::kKernelLines ? C.kp.micro.lines :
                  C.kernel_class == ttc::kKernelBlock ? C.block.unroll : 0;
    return TTC_OK;
    });
}

int ttc_plan_set_streaming(ttc_plan_t plan, int stream_a, int stream_b)
{
    if (!plan) return TTC_ERR_NULL_POINTER;
    if (stream_a < -1 || stream_a > 1 || stream_b < -1 || stream_b > 1) return TTC_ERR_INVALID_VALUE;
    return guarded([&]() -> int {
        ttc::Candidate& C = plan->cands[plan->selected];
        ttc::Candidate rule = C;
        ttc::default_streaming(plan->prob, &rule);
        C.kp.nt_a = stream_a < 0 ? rule.kp.nt_a : stream_a;
        C.kp.nt_b = stream_b < 0 ? rule.kp.nt_b : stream_b;
        if (C.kernel_class == TTC_KERNEL_DIRECT) C.kp.nt_a = C.kp.nt_b = (C.kp.nt_a && C.kp.nt_b) ? 1 : 0;
        return TTC_OK;
    });
}

int ttc_plan_set_tile_mapping(ttc_plan_t plan, int mode)
{
    if (!plan) return TTC_ERR_NULL_POINTER;
    if (mode < -1 || mode > ttc::kMaxTileMapping) return TTC_ERR_INVALID_VALUE;
    ttc::Candidate& C = plan->cands[plan->selected];
    return ttc::set_tile_mapping(&C.kp, mode < 0 ? ttc::default_tile_mapping(plan->prob, C) : mode) ? TTC_OK : TTC_ERR_INVALID_VALUE;
}

int ttc_plan_candidate_count(ttc_plan_t plan)
{
    if (!plan) return -TTC_ERR_NULL_POINTER;
    const int st = guarded([&] { return ttc::complete_plan(plan); });
    return st == TTC_OK ? (int)plan->cands.size() : -st;
}

int ttc_plan_select_candidate(ttc_plan_t plan, int index)
{
    if (!plan) return TTC_ERR_NULL_POINTER;
    if (index < 0) return TTC_ERR_INVALID_VALUE;
    if (index == 0 && plan->selected == 0) return TTC_OK;          // the choice of ttc_plan_create: no list needed
    const int st = guarded([&] { return ttc::complete_plan(plan); });
    if (st != TTC_OK) return st;
    if (index >= (int)plan->cands.size()) return TTC_ERR_INVALID_VALUE;
    plan->selected = index;
    return TTC_OK;
}

// Host-side bounds checker: replays the selected candidate's walk (the same index code the
// kernels run) lane by lane and records, for every offset of B, the offset of A that lands
// there.  Fails on any access outside the (sub-)tensors or the LDS tile, any access that is
// not element-aligned, any element of B written twice or never, and any LDS slot read before
// it was written.
static int emulate_map(ttc_plan_t plan, int64_t* b_from_a);

int ttc_debug_emulate_map(ttc_plan_t plan, int64_t* b_from_a)
{
    if (!plan || !b_from_a) return TTC_ERR_NULL_POINTER;
    return guarded([&] { return emulate_map(plan, b_from_a); });
}

}  // extern "C"

// What the kernels of small problems see of the parameters: packed and unpacked again, if such a kernel runs.
template <bool GATHER, int MODE, bool COMPLEX, int N = 2>
static void small_round_trip(ttc::RowsParams* p)
{
    using namespace ttc;
    if constexpr (N <= kSmallMaxDim) {
        if constexpr (small_fits(GATHER, N, MODE, COMPLEX))
            if (small_dims(*p, GATHER, MODE, COMPLEX, 0, GATHER ? 0 : 1) == N) {
                const RowsParams q = small_unpack<GATHER, N, MODE, COMPLEX>(small_pack(*p, GATHER, N, MODE, COMPLEX), p->vec, p->chunk);
                *p = q;
                return;
            }
        small_round_trip<GATHER, MODE, COMPLEX, N + 1>(p);
    }
}

template <bool GATHER>
static void small_round_trip(const ttc::Problem& P, ttc::RowsParams* p)
{
    const bool cplx = P.kind_a >= ttc::kKindC64;
    switch (P.epilogue) {
    case TTC_EPI_COPY:  cplx ? small_round_trip<GATHER, TTC_EPI_COPY, true>(p) : small_round_trip<GATHER, TTC_EPI_COPY, false>(p); break;
    case TTC_EPI_SCALE: cplx ? small_round_trip<GATHER, TTC_EPI_SCALE, true>(p) : small_round_trip<GATHER, TTC_EPI_SCALE, false>(p); break;
    default:            cplx ? small_round_trip<GATHER, TTC_EPI_AXPBY, true>(p) : small_round_trip<GATHER, TTC_EPI_AXPBY, false>(p); break;
    }
}

// Replay of the row kernel: every workgroup, every lane, the index code the kernel runs.
static int emulate_rows(const ttc::Problem& P, const ttc::Candidate& C, int64_t* b_from_a)
{
    using namespace ttc;
    RowsParams p = C.rows;
    p.xcd_remap = C.kp.xcd_remap;               // as the launch does
    p.nt_a = C.kp.nt_a; p.nt_b = C.kp.nt_b;
    for (int64_t i = 0; i < P.span_b; ++i) b_from_a[i] = -1;
    const int64_t rows = P.elements / P.size[0];
    if ((p.vec != 1 && p.vec != 2 && p.vec != 4) || (p.unroll != 1 && p.unroll != 2 && p.unroll != 4 && p.unroll != 8) || C.threads != 256 ||
        p.chunk != (uint32_t)(C.threads * p.unroll) || p.row < (uint32_t)p.vec || p.row != (uint32_t)P.size[0] || p.rows != (uint32_t)rows ||
        p.elements != P.elements || (p.flat && P.span_b != P.elements) || p.slot_div.div != p.slots ||
        p.slots != (p.flat ? p.row : (p.row + (uint32_t)p.vec - 1) / (uint32_t)p.vec) ||
        p.vectors != (p.flat ? (P.elements + p.vec - 1) / p.vec : rows * (int64_t)p.slots) || (int64_t)p.blocks != (p.vectors + p.chunk - 1) / p.chunk ||
        p.overlap != (!p.flat && P.size[0] % p.vec != 0 ? 1 : 0) || (p.overlap && P.epilogue == TTC_EPI_AXPBY) ||
        P.size[0] >= (int64_t(1) << 30) || rows >= (int64_t(1) << 31))
        return TTC_ERR_INTERNAL;
    p.per_xcd = p.xcd_remap == 1 ? (p.blocks + 7u) / 8u : 0u;
    const bool packed = p.unroll == 1 && small_dims(p, false, P.epilogue, P.kind_a >= kKindC64, 0, 1) != 0;
    if (packed) small_round_trip<false>(P, &p);
    p.xcd_remap = C.kp.xcd_remap;               // packed: none, or ranges by per_xcd
    auto inside = [&](int64_t off, const int64_t* stride, bool b_side) {
        if (off < 0) return false;
        for (int i = P.ndim - 1; i >= 0; --i) {
            const int k = b_side ? P.perm[i] : i;
            const int64_t c = off / stride[k];
            if (c >= P.size[k]) return false;
            off -= c * stride[k];
        }
        return off == 0;
    };
    int64_t written = 0;
    bool bad = false;
    const int64_t grid = rows_grid(p);
    std::vector<char> seen((size_t)p.blocks, 0);
    for (int64_t wg = 0; wg < grid && !bad; ++wg) {
        // the packed kernel runs every workgroup of the grid, those behind the last chunk too; the other one returns there
        const uint32_t block = !packed ? rows_block(p, (uint32_t)wg) : p.xcd_remap == 1 ? range_place(p.per_xcd, (uint32_t)wg) : (uint32_t)wg;
        if (block >= p.blocks && !packed) continue;
        if (block < p.blocks) {
            if (seen[block]) return TTC_ERR_INTERNAL;
            seen[block] = 1;
        }
        const int64_t base = block * (int64_t)p.chunk * (p.flat ? p.vec : 1);
        const int64_t row0_wide = base / (int64_t)p.slots;
        const uint32_t row0 = (uint32_t)row0_wide, slot0 = (uint32_t)(base - row0_wide * (int64_t)p.slots);
        if (packed) {
            const SmallRowsStart at = p.xcd_remap == 1 ? small_rows_start<true>(p, (uint32_t)wg) : small_rows_start<false>(p, (uint32_t)wg);
            if ((int64_t)at.first != base || at.row0 != row0 || at.col0 != slot0) return TTC_ERR_INTERNAL;
        }
        for (uint32_t i = 0; p.flat && i < p.chunk && !bad; ++i) {
            const FlatAccess x = flat_access(p, base, row0, slot0, i);
            for (int j = 0; j < p.vec; ++j) {                // what is loaded: whole vectors inside the tensors
                if (!inside(x.a + j, P.stride_a, false) || (x.split && !inside(x.a_next + j, P.stride_a, false))) bad = true;
                if (!x.valid || j >= x.left) continue;
                const int64_t ea = j < (int)x.head ? x.a + j + (x.split ? p.vec - (int)x.head : 0) : x.a_next + j - (int)x.head, eo = x.b + j;
                if (bad || !inside(ea, P.stride_a, false) || !inside(eo, P.stride_b, true) || b_from_a[eo] != -1) { bad = true; break; }
                b_from_a[eo] = ea;
                ++written;
            }
        }
        if (p.flat) continue;
        for (int u = 0; u < p.unroll && !bad; ++u)
            for (uint32_t tid = 0; tid < (uint32_t)C.threads && !bad; ++tid) {
                const RowAccess x = rows_access(p, base, row0, slot0, (uint32_t)u * (uint32_t)C.threads + tid);
                for (int j = 0; j < p.vec; ++j) {            // loads happen for every lane: they must stay inside
                    const int64_t ea = x.at.a + j, eo = x.at.b + j;
                    if (!inside(ea, P.stride_a, false) || !inside(eo, P.stride_b, true)) { bad = true; break; }
                    if (!x.valid) continue;
                    // an overlapping vector repeats its neighbour's elements: same source
                    if (b_from_a[eo] != -1 && (b_from_a[eo] != ea || !p.overlap)) { bad = true; break; }
                    if (b_from_a[eo] == -1) ++written;
                    b_from_a[eo] = ea;
                }
            }
    }
    return (bad || written != P.elements) ? TTC_ERR_INTERNAL : TTC_OK;
}

// Replay of the gather kernel.
static int emulate_gather(const ttc::Problem& P, const ttc::Candidate& C, int64_t* b_from_a)
{
    using namespace ttc;
    RowsParams p = C.rows;
    p.xcd_remap = C.kp.xcd_remap;
    if (p.vec * P.eb_b != 16 || p.elements != P.elements || p.elements >= (int64_t(1) << 30) || p.chunk != 256 || C.threads != 256 ||
        p.row != (uint32_t)P.size[P.perm[0]] || p.size_div[0].div != p.row || (p.flat != 0) != (P.span_b == P.elements) ||
        (int64_t)p.per_xcd != (p.per_xcd ? (((p.elements + p.vec - 1) / p.vec + p.chunk - 1) / p.chunk + 7) / 8 : 0) ||
        (int64_t)p.blocks != (p.per_xcd ? 8 * (int64_t)p.per_xcd : ((p.elements + p.vec - 1) / p.vec + p.chunk - 1) / p.chunk))
        return TTC_ERR_INTERNAL;
    p.nt_a = C.kp.nt_a; p.nt_b = C.kp.nt_b;
    small_round_trip<true>(P, &p);
    for (int64_t i = 0; i < P.span_b; ++i) b_from_a[i] = -1;
    auto inside = [&](int64_t off, const int64_t* stride, bool b_side) {
        if (off < 0) return false;
        for (int i = P.ndim - 1; i >= 0; --i) {
            const int k = b_side ? P.perm[i] : i;
            const int64_t c = off / stride[k];
            if (c >= P.size[k]) return false;
            off -= c * stride[k];
        }
        return off == 0;
    };
    std::vector<char> seen((size_t)p.blocks, 0);
    int64_t written = 0;
    for (int64_t wg = 0; wg < rows_grid(p); ++wg) {
        const uint32_t block = rows_block(p, (uint32_t)wg);
        if (block >= p.blocks) continue;
        if (seen[block]) return TTC_ERR_INTERNAL;
        seen[block] = 1;
        for (uint32_t tid = 0; tid < p.chunk; ++tid) {
            const uint32_t e = gather_first(p, block, tid);
            if ((int64_t)e >= p.elements) continue;
            const GatherPlace g = gather_place(p, e);
            const bool whole = gather_whole(p, g, (int32_t)std::min<int64_t>(p.elements - (int64_t)e, p.vec));
            for (uint32_t j = 0; j < (uint32_t)p.vec; ++j) {
                const bool there = (int64_t)(e + j) < p.elements;
                const GatherPlace x = gather_next(p, g, e, j);
                if (!inside(x.a, P.stride_a, false) || !inside(x.b, P.stride_b, true)) return TTC_ERR_INTERNAL;      // loaded even if not stored
                if (!there) continue;
                if (p.flat && x.b != (int64_t)(e + j)) return TTC_ERR_INTERNAL;
                if (whole && x.b != g.b + (int64_t)j) return TTC_ERR_INTERNAL;       // the vector that the kernel stores
                if (b_from_a[x.b] != -1) return TTC_ERR_INTERNAL;
                b_from_a[x.b] = x.a;
                ++written;
            }
        }
    }
    return written == P.elements ? TTC_OK : TTC_ERR_INTERNAL;
}

// Replay of the micro-tile kernel: every workgroup, every lane, the index code the kernel runs; every LDS slot
// must be written before it is read, inside the tile buffer.
static int emulate_micro(const ttc::Problem& P, const ttc::Candidate& C, int64_t* b_from_a)
{
    using namespace ttc;
    const MicroArgs p = micro_args(C);          // what the launch hands to the kernel
    const MicroParams& m = p.micro;
    for (int64_t i = 0; i < P.span_b; ++i) b_from_a[i] = -1;
    const uint32_t threads = (uint32_t)C.threads;
    const int vec = m.vec;
    if (p.col_pos < 0 || p.row_pos < 0 || p.col_pos == p.row_pos) return TTC_ERR_INTERNAL;
    if ((vec != 2 && vec != 4) || vec * P.eb_a != 16 || P.eb_a != P.eb_b ||
        (threads != 64 && threads != 128 && threads != 256) || m.ta != vec * m.la || m.tb != vec * m.lb ||
        m.la < 1 || m.lb < 1 || m.pitch < m.la || (m.pitch & 7) || (m.swizzle != 7u && m.swizzle != 0u) || m.la_div.div != (uint32_t)m.la || m.lb_div.div != (uint32_t)m.lb ||
        (int64_t)m.loads * threads < (int64_t)m.la * m.tb || (int64_t)m.blocks * threads < (int64_t)m.la * m.lb ||
        (1 << m.vec_log) != vec || C.lds_bytes != m.tb * m.pitch * 16 || C.lds_bytes > 64 * 1024 || p.grid != p.num_tiles ||
        m.p0 != P.perm[0] || m.p0 == 0 || P.ndim < 2 || P.stride_a[0] != 1 || P.stride_b[m.p0] != 1 ||
        (m.merged_a != 0 && m.merged_a != 1) || (m.merged_b != 0 && m.merged_b != 1))
        return TTC_ERR_INTERNAL;
    const int a1 = 1, p1 = P.perm[1];
    if (m.merged_a && (P.ndim < 3 || a1 == m.p0 || P.stride_a[a1] != P.size[0] || (m.merged_b && a1 == p1))) return TTC_ERR_INTERNAL;
    if (m.merged_b && (P.ndim < 3 || p1 == 0 || P.stride_b[p1] != P.size[m.p0] || (m.merged_a && p1 == a1))) return TTC_ERR_INTERNAL;
    const int64_t cols = m.merged_a ? P.size[0] * P.size[a1] : P.size[0], rows = m.merged_b ? P.size[m.p0] * P.size[p1] : P.size[m.p0];
    if (m.size_a0 != cols || m.size_p0 != rows || cols < vec || rows < vec || cols >= (int64_t(1) << 31) || rows >= (int64_t(1) << 31) ||
        m.col_in_div.div != (uint32_t)P.size[0] || m.row_in_div.div != (uint32_t)P.size[m.p0] ||
        m.col_b_in != P.stride_b[0] || m.col_b_out != (m.merged_a ? P.stride_b[a1] : 0) ||
        m.row_a_in != P.stride_a[m.p0] || m.row_a_out != (m.merged_b ? P.stride_a[p1] : 0))
        return TTC_ERR_INTERNAL;
    const bool whole = cols % vec == 0 && rows % vec == 0;                   // else some elements are written twice ...
    const bool update = P.epilogue == TTC_EPI_AXPBY;                         // ... unless B is read as well: then blocks write only their own
    auto inside = [&](int64_t off, const int64_t* stride, bool b_side) {
        if (off < 0) return false;
        for (int i = P.ndim - 1; i >= 0; --i) {
            const int k = b_side ? P.perm[i] : i;
            const int64_t c = off / stride[k];
            if (c >= P.size[k]) return false;
            off -= c * stride[k];
        }
        return off == 0;
    };
    const int64_t slots = (int64_t)m.tb * m.pitch;              // 16-byte slots of the tile buffer
    std::vector<int64_t> lds((size_t)(slots * vec));
    std::vector<char> seen(p.num_tiles, 0);
    int64_t written = 0;
    for (uint32_t wg = 0; wg < p.grid; ++wg) {
        const TileSeq seq = tile_sequence(p, wg);
        for (uint32_t q = seq.first; q < seq.end; q += seq.step) {
            const uint32_t tile = tile_of(seq, q);
            if (tile >= p.num_tiles || seen[tile]) return TTC_ERR_INTERNAL;
            seen[tile] = 1;
            const MicroTile t = micro_tile(p, tile);
            if (t.lim_a < (uint32_t)vec || t.lim_b < (uint32_t)vec || t.lim_a > (uint32_t)m.ta || t.lim_b > (uint32_t)m.tb) return TTC_ERR_INTERNAL;
            if (whole && (t.lim_a % vec || t.lim_b % vec)) return TTC_ERR_INTERNAL;
            std::fill(lds.begin(), lds.end(), (int64_t)-1);
            for (int i = 0; i < vec; ++i)                         // lanes outside load the tile's first vector or block
                for (int j = 0; j < vec; ++j)
                    if (!inside(t.a + micro_row_a(m, t.row0 + (uint32_t)i) + j, P.stride_a, false) ||
                        !inside(t.b + micro_col_b(m, t.col0 + (uint32_t)j) + i, P.stride_b, true))
                        return TTC_ERR_INTERNAL;
            for (uint32_t tid = 0; tid < threads; ++tid)
                for (int k = 0; k < (m.loads + 3) / 4 * 4; ++k) { // the kernel walks its loads four at a time
                    const MicroLoad x = micro_load(m, threads, tid, (uint32_t)k);
                    if (!x.valid) continue;
                    if (x.chunk >= (uint64_t)slots) return TTC_ERR_INTERNAL;
                    const bool ok = x.row < t.lim_b && x.col < t.lim_a;
                    const uint32_t col = ok ? micro_back(x.col, t.lim_a, (uint32_t)vec) : 0u;
                    for (int j = 0; j < vec; ++j) {
                        int64_t src = -2;                         // parked by a lane outside the tensor: must never be read
                        if (ok) {
                            src = t.a + micro_row_a(m, t.row0 + x.row) + col + j;
                            if (!inside(src, P.stride_a, false)) return TTC_ERR_INTERNAL;
                        }
                        if (lds[(size_t)x.chunk * vec + j] != -1) return TTC_ERR_INTERNAL;       // every slot has one writer
                        lds[(size_t)x.chunk * vec + j] = src;
                    }
                }
            for (uint32_t tid = 0; tid < threads; ++tid)
                for (int b = 0; b < m.blocks; ++b) {
                    const MicroBlock x = micro_block(m, threads, tid, (uint32_t)b);
                    if (!(x.valid && x.row < t.lim_b && x.col < t.lim_a)) continue;
                    const uint32_t row = micro_back(x.row, t.lim_b, (uint32_t)vec), col = micro_back(x.col, t.lim_a, (uint32_t)vec);
                    const bool edge = update && (row != x.row || col != x.col || x.row < t.own_b || x.col < t.own_a);
                    const uint32_t first_row = std::max(x.row, t.own_b), first_col = std::max(x.col, t.own_a);
                    for (int i = 0; i < vec; ++i) {
                        const uint64_t chunk = micro_slot(m, row + (uint32_t)i, x.lane_c);
                        if (chunk >= (uint64_t)slots) return TTC_ERR_INTERNAL;
                        for (int j = 0; j < vec; ++j) {
                            const int64_t src = lds[(size_t)chunk * vec + j];
                            const int64_t dst = t.b + micro_col_b(m, t.col0 + col + (uint32_t)j) + row + i;
                            // what sits in the slot must be the element of the tile at (row + i, col + j)
                            if (src != t.a + micro_row_a(m, t.row0 + row + (uint32_t)i) + col + j) return TTC_ERR_INTERNAL;
                            if (!inside(dst, P.stride_b, true)) return TTC_ERR_INTERNAL;
                            if (edge && !(col + (uint32_t)j >= first_col && row + (uint32_t)i >= first_row)) continue;   // not this block's to update
                            if (b_from_a[dst] == -1) ++written;
                            else if (whole || update || b_from_a[dst] != src) return TTC_ERR_INTERNAL;   // a second write brings the same element
                            b_from_a[dst] = src;
                        }
                    }
                }
        }
    }
    return written == P.elements ? TTC_OK : TTC_ERR_INTERNAL;
}

// Replay of the line kernel, every workgroup and every lane, for a B that starts `phase0` elements behind the start of a line.
static int emulate_lines(const ttc::Problem& P, const ttc::Candidate& C, int phase0, int64_t* b_from_a)
{
    using namespace ttc;
    const MicroArgs whole = micro_args(C);
    MicroArgs p = whole;
    const MicroParams& m = p.micro;
    const int p0 = P.perm[0], p1 = P.ndim >= 2 ? P.perm[1] : -1, a1 = 1;
    if (p0 == 0 || P.ndim < 2 || !line_shape_ok(m.ta, m.lines, P.eb_a, P.eb_b)) return TTC_ERR_INTERNAL;
    const LineShape S = line_shape(m.ta, m.lines, P.eb_a, P.eb_b);
    const int64_t cols = m.merged_a ? P.size[0] * P.size[a1] : P.size[0], rows = m.merged_b ? P.size[p0] * P.size[p1] : P.size[p0];
    if (p.col_pos < 0 || p.row_pos < 0 || p.col_pos == p.row_pos || p.grid != p.num_tiles || C.threads != kLineThreads || C.lds_bytes != S.lds_bytes ||
        S.passes * S.pass != S.rows || S.lanes * S.pass != kLineThreads || S.lanes * S.va != m.ta || 8 * S.vb != S.line ||
        S.side * S.groups * 8 != kLineThreads || m.ta % S.side != 0 || m.lines % S.groups != 0 || m.tb != (m.lines - m.skewed) * S.line || m.p0 != p0 ||
        P.stride_a[0] != 1 || P.stride_b[p0] != 1 || (m.merged_a | 1) != 1 || (m.merged_b | 1) != 1 || (m.skewed | 1) != 1 ||
        (m.merged_a && (P.ndim < 3 || a1 == p0 || P.stride_a[a1] != P.size[0] || (m.merged_b && a1 == p1))) ||
        (m.merged_b && (P.ndim < 3 || p1 == 0 || P.stride_b[p1] != P.size[p0])) ||
        m.size_a0 != cols || m.size_p0 != rows || cols < S.va || rows < S.vb || cols >= kLineMaxExtent || rows >= kLineMaxExtent ||
        m.col_in_div.div != (uint32_t)P.size[0] || m.row_in_div.div != (uint32_t)P.size[p0] ||
        m.col_b_in != P.stride_b[0] || m.col_b_out != (m.merged_a ? P.stride_b[a1] : 0) ||
        m.row_a_in != P.stride_a[p0] || m.row_a_out != (m.merged_b ? P.stride_a[p1] : 0))
        return TTC_ERR_INTERNAL;
    const bool cplx = P.kind_a >= kKindC64;
    const int packed = small_line(whole, P.epilogue, cplx, S.passes);
    SmallDeal deal = {0, 0};
    const int dealing = small_line_dealing(whole);
    if (packed) {                                              // as the kernel of small problems sees them
        const SmallArgs small = small_line_pack(whole, P.epilogue, cplx);
        auto unpack = [&](auto cx, auto merged) {
            constexpr bool kComplex = decltype(cx)::value, kMerged = decltype(merged)::value;
            return dealing == kDealAll ? small_line_unpack<TTC_EPI_COPY, kComplex, kMerged, true>(small, m.ta, S) : small_line_unpack<TTC_EPI_COPY, kComplex, kMerged, false>(small, m.ta, S);
        };
        p = packed == 2 ? (cplx ? unpack(std::true_type(), std::true_type()) : unpack(std::false_type(), std::true_type()))
                        : (cplx ? unpack(std::true_type(), std::false_type()) : unpack(std::false_type(), std::false_type()));
        deal = small_line_deal(small, packed == 2);
        p.num_tiles = p.grid = whole.num_tiles;
        if (p.nt_a != whole.nt_a || deal.blocks != whole.num_tiles || deal.xcd_remap != whole.xcd_remap || p.nt_b != whole.nt_b || m.tb != whole.micro.tb || m.skewed != whole.micro.skewed) return TTC_ERR_INTERNAL;
    }
    for (int64_t i = 0; i < P.span_b; ++i) b_from_a[i] = -1;
    auto inside = [&](int64_t off, const int64_t* stride, bool b_side) {
        if (off < 0) return false;
        for (int i = P.ndim - 1; i >= 0; --i) {
            const int k = b_side ? P.perm[i] : i;
            const int64_t c = off / stride[k];
            if (c >= P.size[k]) return false;
            off -= c * stride[k];
        }
        return off == 0;
    };
    std::vector<int64_t> lds((size_t)(S.rows * S.pitch));
    std::vector<char> seen(p.num_tiles, 0);
    int64_t written = 0;
    const int64_t grid = packed ? rows_grid(deal) : (int64_t)p.grid;
    for (int64_t wg = 0; wg < grid; ++wg) {
        TileSeq seq = {(uint32_t)wg, (uint32_t)wg + 1u, 1u, 0u, 0u, 0u};
        const uint32_t mine = dealing == kDealAll ? rows_block(deal, (uint32_t)wg) : dealing == kDealRanges ? small_line_range(deal, (uint32_t)wg) : (uint32_t)wg;
        if (packed) {
            if (mine >= deal.blocks) continue;
        } else {
            seq = tile_sequence(p, (uint32_t)wg);
        }
        for (uint32_t q = seq.first; q < seq.end; q += seq.step) {
            const uint32_t tile = packed ? mine : tile_of(seq, q);
            if (tile >= p.num_tiles || seen[tile]) return TTC_ERR_INTERNAL;
            seen[tile] = 1;
            const LineTile t = line_tile(p, S, tile);
            if (t.cols < 1 || t.cols > m.ta) return TTC_ERR_INTERNAL;
            std::fill(lds.begin(), lds.end(), (int64_t)-1);
            for (int k = 0; k < S.passes; ++k)
                for (uint32_t tid = 0; tid < (uint32_t)kLineThreads; ++tid) {
                    const LineLoad x = line_load(m, S, t, tid, k);
                    if (!x.needed) continue;
                    const int64_t y = (int64_t)t.row0 + x.lds_row;
                    for (int j = 0; j < S.va; ++j) {             // every lane loads, whether it keeps what it got or not
                        const int64_t src = t.a + micro_row_a(m, x.row) + x.start + j;
                        if (!inside(src, P.stride_a, false)) return TTC_ERR_INTERNAL;
                        if (x.col >= t.cols || x.start + j < 0) continue;
                        const int64_t slot = (int64_t)x.lds_row * S.pitch + x.start + j;
                        if (x.start + j >= m.ta || slot < 0 || slot >= (int64_t)lds.size()) return TTC_ERR_INTERNAL;
                        if (x.start == x.col && (slot - j) * P.eb_a % (P.eb_a == 4 ? 8 : 16) != 0) return TTC_ERR_INTERNAL;     // the wide LDS write
                        const int64_t value = y >= 0 && y < rows ? src : -2;            // rows outside the tensor: parked, never stored
                        if (lds[(size_t)slot] != -1 && lds[(size_t)slot] != value) return TTC_ERR_INTERNAL;
                        lds[(size_t)slot] = value;
                    }
                }
            for (uint32_t tid = 0; tid < (uint32_t)kLineThreads; ++tid)
                for (int g = 0; g < m.ta / S.side; ++g) {
                    const int32_t c = line_column(S, tid, g);
                    if (c >= t.cols) continue;
                    const int64_t col = t.b + micro_col_b(m, t.col0 + (uint32_t)c);
                    const int32_t phase = (int32_t)((col + phase0) % S.line);
                    for (int i = 0; i < m.lines / S.groups; ++i)
                        for (int j = 0; j < S.vb; ++j) {
                            if (line_last(m, S, tid, i)) continue;
                            const int64_t y = (int64_t)line_row(m, S, t, phase, tid) + i * S.groups * S.line + j, slot = (y - t.row0) * S.pitch + c;
                            if (slot < 0 || slot >= (int64_t)lds.size()) return TTC_ERR_INTERNAL;
                            if (y < 0 || y >= rows) continue;
                            const int64_t dst = col + y;
                            if (lds[(size_t)slot] < 0 || !inside(dst, P.stride_b, true) || b_from_a[dst] != -1) return TTC_ERR_INTERNAL;
                            b_from_a[dst] = lds[(size_t)slot];
                            ++written;
                        }
                }
        }
    }
    return written == P.elements ? TTC_OK : TTC_ERR_INTERNAL;
}

// Replay of the block kernel: every workgroup, every lane, the index code the kernel runs.
static int emulate_block(const ttc::Problem& P, const ttc::Candidate& C, int64_t* b_from_a)
{
    using namespace ttc;
    const BlockArgs p = block_args(C);
    const BlockParams& m = p.block;
    const int va = 16 / P.eb_a, vb = 16 / P.eb_b, stores = block_stores(m.unroll, P.eb_a, P.eb_b);
    if (P.stride_a[0] != 1 || P.stride_b[P.perm[0]] != 1 || p.blocks != C.kp.num_tiles || C.threads != kBlockThreads || C.lds_bytes > kBlockMaxLds ||
        (int64_t)m.rows * m.pitch * P.eb_a != C.lds_bytes || m.pitch % va != 0 || m.run_a > m.pitch ||
        (int64_t)m.va_div.div * m.rows > m.unroll * kBlockThreads || (int64_t)m.vb_div.div * m.outs > stores * kBlockThreads ||
        (int64_t)m.rows * m.run_a != (int64_t)m.outs * m.run_b)
        return TTC_ERR_INTERNAL;
    for (int64_t i = 0; i < P.span_b; ++i) b_from_a[i] = -1;
    auto inside = [&](int64_t off, const int64_t* stride, bool b_side) {
        if (off < 0) return false;
        for (int i = P.ndim - 1; i >= 0; --i) {
            const int k = b_side ? P.perm[i] : i;
            const int64_t c = off / stride[k];
            if (c >= P.size[k]) return false;
            off -= c * stride[k];
        }
        return off == 0;
    };
    std::vector<int64_t> lds((size_t)(m.rows * (int64_t)m.pitch));
    std::vector<char> seen(p.blocks, 0);
    int64_t written = 0;
    for (int64_t wg = 0; wg < rows_grid(p); ++wg) {
        const uint32_t block = rows_block(p, (uint32_t)wg);
        if (block >= p.blocks) continue;
        if (seen[block]) return TTC_ERR_INTERNAL;
        seen[block] = 1;
        const BlockTile t = block_tile(p, block);
        if (t.run_a < 1 || t.run_b < 1 || t.run_a > m.run_a || t.run_b > m.run_b) return TTC_ERR_INTERNAL;
        std::fill(lds.begin(), lds.end(), (int64_t)-1);
        for (uint32_t g = 0; g < (uint32_t)(m.unroll * kBlockThreads); ++g) {
            const BlockLoad x = block_load(m, t, g, va);
            for (int j = 0; j < va; ++j) {                       // every lane loads, whether it keeps what it got or not
                const int64_t src = t.a + x.a + j;
                if (!inside(src, P.stride_a, false)) return TTC_ERR_INTERNAL;
                if (!x.ok || x.start + j < 0) continue;
                const int64_t slot = (int64_t)x.lds + j;
                if (slot < 0 || slot >= (int64_t)lds.size() || (x.start == x.col && x.lds % va != 0)) return TTC_ERR_INTERNAL;
                if (lds[(size_t)slot] != -1 && lds[(size_t)slot] != src) return TTC_ERR_INTERNAL;
                lds[(size_t)slot] = src;
            }
        }
        for (uint32_t h = 0; h < (uint32_t)(stores * kBlockThreads); ++h) {
            const BlockStore x = block_store(m, t, h, vb);
            if (P.epilogue == TTC_EPI_AXPBY)
                for (int j = 0; j < vb; ++j) if (!inside(t.b + x.from + j, P.stride_b, true)) return TTC_ERR_INTERNAL;
            int32_t at = x.lds, x0 = x.x0, x1 = x.x1;
            for (int j = 0; j < x.count; ++j) {
                if (m.even) at = x.lds + j * m.x_lds[0];
                else if (j > 0) block_next(m, &at, &x0, &x1);
                const int64_t dst = t.b + x.b + j;
                if (at < 0 || at >= (int64_t)lds.size() || lds[(size_t)at] < 0 || !inside(dst, P.stride_b, true) || b_from_a[dst] != -1) return TTC_ERR_INTERNAL;
                b_from_a[dst] = lds[(size_t)at];
                ++written;
            }
        }
    }
    return written == P.elements ? TTC_OK : TTC_ERR_INTERNAL;
}

static int emulate_map(ttc_plan_t plan, int64_t* b_from_a)
{
    using namespace ttc;
    const Problem& P = plan->prob;
    const Candidate& C = plan->cands[plan->selected];
    if (C.kernel_class == TTC_KERNEL_ROWS) return emulate_rows(P, C, b_from_a);
    if (C.kernel_class == kKernelGather) return emulate_gather(P, C, b_from_a);
    if (C.kernel_class == TTC_KERNEL_MICRO) return emulate_micro(P, C, b_from_a);
    if (C.kernel_class == kKernelBlock) return emulate_block(P, C, b_from_a);
    if (C.kernel_class == kKernelLines) {
        // where a tile is cut depends on the address B will have: every place inside a line that matters (the first,
        // the last, one between), the aligned one last
        const int line = kLineBytes / P.eb_b;
        for (int phase : {line - 1, line / 2 + 1, 0}) {
            const int st = emulate_lines(P, C, phase, b_from_a);
            if (st != TTC_OK) return st;
        }
        return TTC_OK;
    }
    KernelParams p = C.kp;
    set_grid(&p, launch_grid(C, 256));
    const int32_t eba = P.eb_a, ebb = P.eb_b;
    for (int64_t i = 0; i < P.span_b; ++i) b_from_a[i] = -1;
    const uint32_t nwave = (uint32_t)C.threads / kWave;
    if (nwave < 1 || C.threads % kWave) return TTC_ERR_INTERNAL;
    const bool direct = (C.kernel_class == TTC_KERNEL_DIRECT);
    if ((p.lds_buffers != 1 && p.lds_buffers != 2) ||
        p.lds_data_off + p.lds_buffers * (int64_t)p.lds_tile_elems * eba != C.lds_bytes || C.lds_bytes > kMaxLdsBytes)
        return TTC_ERR_INTERNAL;
    // is this element offset an element of the sub-tensor?  (decode by strides, slowest index first)
    auto inside = [&](int64_t off, const int64_t* stride, bool b_side) {
        if (off < 0) return false;
        for (int i = P.ndim - 1; i >= 0; --i) {
            const int k = b_side ? P.perm[i] : i;
            const int64_t c = off / stride[k];
            if (c >= P.size[k]) return false;
            off -= c * stride[k];
        }
        return off == 0;
    };
    // position tables, as a workgroup builds them
    const uint32_t ta = nwave * (uint32_t)p.a.chunk, tbn = direct ? 0u : nwave * (uint32_t)p.b.chunk;
    if (kTablesOff + (int64_t)24 * (ta + tbn) > p.lds_data_off) return TTC_ERR_INTERNAL;
    if (p.a.chunk_rem < 1 || p.a.chunk_rem > (int)nwave || (p.a.chunk - 1) * (int)nwave + p.a.chunk_rem != p.a.n_iter)
        return TTC_ERR_INTERNAL;
    if (!direct && (p.b.chunk_rem < 1 || p.b.chunk_rem > (int)nwave ||
                    (p.b.chunk - 1) * (int)nwave + p.b.chunk_rem != p.b.n_iter)) return TTC_ERR_INTERNAL;
    const Scales sc_a = {eba, ebb, eba};       // walk over A (direct: g2 addresses B)
    const Scales sc_b = {ebb, ebb, eba};       // walk over B of the staged kernel
    std::vector<PosEntry> tab_a(ta), tab_b(tbn);
    std::vector<PosCoord> tabc_a(ta), tabc_b(tbn);
    for (uint32_t th = 0; th < (uint32_t)C.threads; ++th) {
        if (direct) build_tables<true>(p.a, nwave, th, (uint32_t)C.threads, sc_a, tab_a.data(), tabc_a.data());
        else {
            build_tables<false>(p.a, nwave, th, (uint32_t)C.threads, sc_a, tab_a.data(), tabc_a.data());
            build_tables<false>(p.b, nwave, th, (uint32_t)C.threads, sc_b, tab_b.data(), tabc_b.data());
        }
    }

    const int64_t lds_bytes = (int64_t)p.lds_tile_elems * eba;
    std::vector<int64_t> lds((size_t)p.lds_tile_elems);          // which element offset of A each slot holds
    std::vector<char> seen(p.num_tiles, 0);
    bool bad = false;
    int fail_line = 0;
    auto fail_at = [&](int line) { if (!bad) fail_line = line; bad = true; };
#define fail() fail_at(__LINE__)
    auto nop = [](int, const PosEntry&, int, bool) {};
    const bool axpby = (P.epilogue == TTC_EPI_AXPBY);
    std::vector<int64_t> writer((size_t)P.span_b, -1);      // which instruction wrote an element of B
    int64_t written = 0;
    for (uint32_t wg = 0; wg < p.grid && !bad; ++wg) {
        const TileSeq seq = tile_sequence(p, wg);
        for (uint32_t q = seq.first; q < seq.end && !bad; q += seq.step) {
            const uint32_t tile = tile_of(seq, q);
            if (tile >= p.num_tiles || seen[tile]) return TTC_ERR_INTERNAL;
            seen[tile] = 1;
            const TileBase tb = tile_base(p, tile);
            const int64_t base_a = tb.a * eba, base_b = tb.b * ebb;
            const TileLim tl = tile_lim(p, tile);
            const SideLim la = side_lim(p.a, tl);
            // lanes outside the tile load the tile's first vector instead (and read the LDS tile's first slots)
            for (int j = 0; j < p.a.vec; ++j) if (!inside(tb.a + j, P.stride_a, false)) return TTC_ERR_INTERNAL;
            for (int j = 0; j < (direct ? p.a.vec : p.b.vec); ++j)
                if (!inside(tb.b + j, P.stride_b, true)) return TTC_ERR_INTERNAL;
            if (!direct && (int64_t)(p.b.vec - 1) * p.b.vec_lds_stride >= p.lds_tile_elems) return TTC_ERR_INTERNAL;
            if (direct) {
                for (uint32_t wave = 0; wave < nwave; ++wave)
                    for (uint32_t lane = 0; lane < (uint32_t)kWave; ++lane) {
                        const LaneState L = lane_setup<true>(p.a, lane, sc_a);
                        const WalkMask wm = walk_mask(p.a, L, la);
                        auto st = [&](int, const PosEntry& e, int back, bool ok) {
                            if (!ok) return;
                            const int64_t oa = base_a + e.g + L.g, ob = base_b + e.l_or_g2 + L.g2;
                            if (oa % eba || ob % ebb || back < 0 || back >= p.a.vec) return fail();
                            const int64_t who = ((int64_t)tile << 32) | (wave << 16) | (uint32_t)(&e - tab_a.data());
                            for (int j = -back; j < p.a.vec - back; ++j) {
                                const int64_t ea = oa / eba + j, eo = ob / ebb + j;
                                if (!inside(ea, P.stride_a, false) || !inside(eo, P.stride_b, true)) return fail();
                                // a moved-back vector repeats its neighbour's elements: same source, same instruction
                                // if B is read as well as written
                                if (b_from_a[eo] != -1 && (b_from_a[eo] != ea || (axpby && writer[eo] != who))) return fail();
                                if (b_from_a[eo] == -1) ++written;
                                b_from_a[eo] = ea;
                                writer[eo] = who;
                            }
                        };
                        emu_walk(p.a, L, la, wm, tab_a.data(), tabc_a.data(), wave, st, nop);
                    }
                continue;
            }
            std::fill(lds.begin(), lds.end(), (int64_t)-1);
            for (uint32_t wave = 0; wave < nwave; ++wave)
                for (uint32_t lane = 0; lane < (uint32_t)kWave; ++lane) {
                    const LaneState L = lane_setup<false>(p.a, lane, sc_a);
                    const WalkMask wm = walk_mask(p.a, L, la);
                    auto st = [&](int, const PosEntry& e, int back, bool ok) {
                        if (!ok) return;
                        const int64_t oa = base_a + e.g + L.g;
                        const int64_t lo = (int64_t)(int32_t)e.l_or_g2 + L.l;
                        if (oa % eba || lo % eba || back < 0 || back >= p.a.vec) return fail();
                        if (lo < 0 || lo >= lds_bytes) return fail();
                        for (int j = -back; j < p.a.vec - back; ++j) {
                            const int64_t ea = oa / eba + j;
                            if (!inside(ea, P.stride_a, false)) return fail();
                            const int64_t li = lo / eba + (int64_t)j * p.a.vec_lds_stride;
                            if (li < 0 || li >= p.lds_tile_elems) return fail();
                            if (lds[li] != -1 && lds[li] != ea) return fail();
                            lds[li] = ea;
                        }
                    };
                    emu_walk(p.a, L, la, wm, tab_a.data(), tabc_a.data(), wave, st, nop);
                }
            const SideLim lb = side_lim(p.b, tl);
            for (uint32_t wave = 0; wave < nwave; ++wave)
                for (uint32_t lane = 0; lane < (uint32_t)kWave; ++lane) {
                    const LaneState L = lane_setup<false>(p.b, lane, sc_b);
                    const WalkMask wm = walk_mask(p.b, L, lb);
                    auto st = [&](int, const PosEntry& e, int back, bool ok) {
                        if (!ok) return;
                        const int64_t ob = base_b + e.g + L.g;
                        const int64_t lo = (int64_t)(int32_t)e.l_or_g2 + L.l;
                        if (ob % ebb || lo % eba || back < 0 || back >= p.b.vec) return fail();
                        const int64_t who = ((int64_t)tile << 32) | (wave << 16) | (uint32_t)(&e - tab_b.data());
                        for (int j = -back; j < p.b.vec - back; ++j) {
                            const int64_t eo = ob / ebb + j;
                            if (!inside(eo, P.stride_b, true)) return fail();
                            const int64_t li = lo / eba + (int64_t)j * p.b.vec_lds_stride;
                            if (li < 0 || li >= p.lds_tile_elems) return fail();
                            if (lds[li] == -1) return fail();
                            if (b_from_a[eo] != -1 && (b_from_a[eo] != lds[li] || (axpby && writer[eo] != who))) return fail();
                            if (b_from_a[eo] == -1) ++written;
                            b_from_a[eo] = lds[li];
                            writer[eo] = who;
                        }
                    };
                    emu_walk(p.b, L, lb, wm, tab_b.data(), tabc_b.data(), wave, st, nop);
                }
        }
    }
#undef fail
    if (bad || written != P.elements) {
        if (std::getenv("TTC_EMU_DEBUG")) std::fprintf(stderr, "ttc_debug_emulate_map: check at line %d failed, %lld of %lld elements written\n", fail_line, (long long)written, (long long)P.elements);
        return TTC_ERR_INTERNAL;
    }
    return TTC_OK;
}
