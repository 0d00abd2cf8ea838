// The tile ("box") kernels for gfx950 (MI355X) and their launch templates.  Included by one
// translation unit per group of element types (ttc_launch_*.hip), so that the groups compile in parallel.
//
// One kernel template serves both cases of the paper's Section 3.1.
//   * staged (stride-1 index changes):  a workgroup owns one box of the tensor that spans the
//     leading indices of A *and* of B.  Wavefronts walk the box in A order with vector loads
//     (lanes along A's stride-1 index), park it in LDS, and after one barrier walk it again in B
//     order (lanes along B's stride-1 index), apply the alpha/beta epilogue and store vectors.
//   * direct (stride-1 index fixed, or 1-D):  the same walk, but every lane stores what it
//     loaded; no LDS, no barrier.
// A walk is factorised CDNA-style: the 64 lanes of a wavefront cover a fixed sub-box (lane
// offsets are computed once and live in VGPRs), and the position of that sub-box inside the
// tile is wave-uniform, so the per-instruction index arithmetic runs on the scalar unit.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <climits>
#include <cstdlib>
#include <type_traits>

#include "ttc_internal.h"
#include "ttc_walk.h"

namespace ttc {

// ---------------------------------------------------------------------------------
// Element types and the alpha/beta epilogue (fixed evaluation order; built with
// -ffp-contract=off so the only fused operations are the ones written here).
//   real:    copy: r = a | scale: r = alpha*a | axpby: t = beta*b, r = fma(alpha, a, t)
//   complex: product z = s*x as z.re = fma(s.re, x.re, -(s.im*x.im)), z.im = fma(s.re, x.im, s.im*x.re);
//            scale: r = alpha*a | axpby: r = alpha*a + beta*b componentwise
// Mixed precision (A and B of different precision): elements are widened to double, the same
// formulas run in double, the result is rounded once (to nearest even) to B's type.
// ---------------------------------------------------------------------------------
struct alignas(8) cfloat { float re, im; };
struct alignas(8) cdouble { double re, im; };

// Global vectors are only guaranteed element alignment (gfx950 global dwordx2/x4 accesses need
// no more); the hardware runs them at full rate at any 4-byte boundary.
template <typename T, int V> struct alignas(alignof(T)) Pack { T v[V]; };

template <typename To, typename From> struct Convert;
template <typename T> struct Convert<T, T> { __device__ static __forceinline__ T go(T x) { return x; } };
template <> struct Convert<double, float> { __device__ static __forceinline__ double go(float x) { return (double)x; } };
template <> struct Convert<float, double> { __device__ static __forceinline__ float go(double x) { return (float)x; } };
template <> struct Convert<cdouble, cfloat> {
    __device__ static __forceinline__ cdouble go(cfloat x) { cdouble r; r.re = (double)x.re; r.im = (double)x.im; return r; }
};
template <> struct Convert<cfloat, cdouble> {
    __device__ static __forceinline__ cfloat go(cdouble x) { cfloat r; r.re = (float)x.re; r.im = (float)x.im; return r; }
};

__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

// the arithmetic, in the type it runs in
template <typename C, int MODE> struct Core {                    // C = float or double
    C al, be;
    __device__ Core(const double* alpha, const double* beta) : al((C)alpha[0]), be((C)beta[0]) {}
    __device__ __forceinline__ C operator()(C a, C b) const
    {
        if (MODE == TTC_EPI_COPY) return a;
        if (MODE == TTC_EPI_SCALE) return al * a;
        const C t = be * b;
        return fused(al, a, t);
    }
};

template <typename Z, typename R, int MODE> struct ComplexCore {  // Z = cfloat / cdouble over R = float / double
    R ar, ai, br, bi;
    __device__ ComplexCore(const double* alpha, const double* beta)
        : ar((R)alpha[0]), ai((R)alpha[1]), br((R)beta[0]), bi((R)beta[1]) {}
    __device__ __forceinline__ Z operator()(Z a, Z b) const
    {
        if (MODE == TTC_EPI_COPY) return a;
        Z p;
        p.re = fused(ar, a.re, -(ai * a.im));
        p.im = fused(ar, a.im, ai * a.re);
        if (MODE == TTC_EPI_SCALE) return p;
        Z q;
        q.re = fused(br, b.re, -(bi * b.im));
        q.im = fused(br, b.im, bi * b.re);
        Z r;
        r.re = p.re + q.re;
        r.im = p.im + q.im;
        return r;
    }
};
template <int MODE> struct Core<cfloat, MODE> : ComplexCore<cfloat, float, MODE> { using ComplexCore<cfloat, float, MODE>::ComplexCore; };
template <int MODE> struct Core<cdouble, MODE> : ComplexCore<cdouble, double, MODE> { using ComplexCore<cdouble, double, MODE>::ComplexCore; };

template <typename T> struct IsComplex { static constexpr bool value = std::is_same<T, cfloat>::value || std::is_same<T, cdouble>::value; };

// type the arithmetic runs in: the common type, or the double-precision one when they differ
template <typename TA, typename TB> struct Wider;
template <typename T> struct Wider<T, T> { using type = T; };
template <> struct Wider<float, double> { using type = double; };
template <> struct Wider<double, float> { using type = double; };
template <> struct Wider<cfloat, cdouble> { using type = cdouble; };
template <> struct Wider<cdouble, cfloat> { using type = cdouble; };

template <typename TA, typename TB, int MODE> struct Epilogue {
    using C = typename Wider<TA, TB>::type;
    Core<C, MODE> core;
    __device__ Epilogue(const double* alpha, const double* beta) : core(alpha, beta) {}
    __device__ __forceinline__ TB operator()(TA a, TB b) const
    {
        return Convert<TB, C>::go(core(Convert<C, TA>::go(a), Convert<C, TB>::go(b)));
    }
};

// ---------------------------------------------------------------------------------
// The kernel.  Dynamic LDS: [two shared tile records][spare slots][position tables of both walks][tile buffer 0][tile buffer 1].
// Cut vectors: where a run is not a multiple of the vector width, the lane that would overhang moves its
// vector back so that it ends with the run (`back` elements, handed to the stages).  It then repeats what
// its neighbour does for those elements, with the same values, so nothing diverges and every access stays a
// full vector.
// A workgroup walks several tiles; with two tile buffers one barrier per tile is enough: a
// wavefront can only start filling buffer (t+1)%2 after it passed the barrier of tile t, and
// every wavefront reached that barrier after it had finished reading that buffer for tile t-1.
// ---------------------------------------------------------------------------------
// memory instructions a wavefront keeps in flight per walk step: four 16-byte accesses per lane, more of the
// narrow ones (the bytes in flight per wavefront are what hides the memory latency)
template <typename T, int V> struct Unroll { static constexpr int value = (V * sizeof(T) >= 16) ? 4 : 8; };

__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Non-temporal accesses (the paper's streaming stores, Table 1 / Section 3.4, and their load counterpart):
// data that is touched once need not displace what neighbouring tiles will share.  The hint is a compile-time
// property of an access; a walk exists in both forms and the (wave-uniform) flag picks one per tile.
template <int N> struct Words;
template <> struct Words<1> { typedef uint32_t type; };
template <> struct Words<2> { typedef uint32_t type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Words<4> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Words<8> { typedef uint32_t type __attribute__((ext_vector_type(8), aligned(4))); };

template <typename T, int V, bool NT>
__device__ __forceinline__ Pack<T, V> load_pack(const unsigned char* base, int64_t off)
{
    typedef typename Words<V * sizeof(T) / 4>::type W;
    if (NT) {
        union { W w; Pack<T, V> p; } u;
        u.w = __builtin_nontemporal_load(reinterpret_cast<const W*>(base + off));
        return u.p;
    }
    return *reinterpret_cast<const Pack<T, V>*>(base + off);
}

template <typename T, int V, bool NT>
__device__ __forceinline__ void store_pack(unsigned char* base, int64_t off, const Pack<T, V>& v)
{
    typedef typename Words<V * sizeof(T) / 4>::type W;
    if (NT) {
        union { W w; Pack<T, V> p; } u;
        u.p = v;
        __builtin_nontemporal_store(u.w, reinterpret_cast<W*>(base + off));
    } else {
        *reinterpret_cast<Pack<T, V>*>(base + off) = v;
    }
}

// what one wavefront left in LDS about a tile and a walk, as the (wave-uniform) limits and the lane's own verdict
__device__ __forceinline__ void take_side(const SideShare& v, uint32_t single, const LaneState& L, SideLim* sl, WalkMask* wm)
{
    sl->lim[0] = __builtin_amdgcn_readfirstlane(v.lim[0]); sl->lim[1] = __builtin_amdgcn_readfirstlane(v.lim[1]);
    sl->lim[2] = __builtin_amdgcn_readfirstlane(v.lim[2]); sl->lim[3] = __builtin_amdgcn_readfirstlane(v.lim[3]);
    sl->t01 = __builtin_amdgcn_readfirstlane(v.t01); sl->t23 = __builtin_amdgcn_readfirstlane(v.t23);
    wm->dynamic = __builtin_amdgcn_readfirstlane(v.dynamic) != 0;
    wm->lane_ok = lane_inside(single, L, *sl);
}

template <typename TA, typename TB, int MODE, int VA, int VB, bool DIRECT>
__global__ __launch_bounds__(kMaxThreads) void box_kernel(const KernelParams params_by_value, const TA* __restrict__ A,
                                                          TB* __restrict__ B)
{
    // The parameter block is read where the launch put it, at the start of the kernel-argument segment (constant
    // memory, scalar loads).  Reading the by-value argument instead leaves it to the optimiser to see through the
    // copy the language asks for, and past a certain number of uses it keeps the copy: 1.4 KB of scratch per lane.
    const KernelParams& p = *reinterpret_cast<const KernelParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    extern __shared__ __align__(16) unsigned char smem[];
    {   // Bring the whole parameter block into the scalar cache at once (read-only scalar loads of one word per
        // 64-byte line): the set-up code below reads it piece by piece, and each piece would otherwise be a miss.
        typedef const uint32_t __attribute__((address_space(4))) ConstWord;
        const ConstWord* args = (const ConstWord*)__builtin_amdgcn_kernarg_segment_ptr();
        uint32_t touched = 0;
#pragma unroll
        for (int i = 0; i < (int)(sizeof(KernelParams) / 64); ++i) touched ^= args[i * 16];
        asm volatile("" :: "s"(touched));
    }
    constexpr int32_t kScaleA = (int32_t)sizeof(TA), kScaleB = (int32_t)sizeof(TB);
    const Scales sc_a = {kScaleA, kScaleB, kScaleA};     // walk over A; the LDS tile holds elements of A
    const Scales sc_b = {kScaleB, kScaleB, kScaleA};     // walk over B
    const uint32_t nwave = blockDim.x >> 6;
    const uint32_t n_a = nwave * (uint32_t)p.a.chunk, n_b = DIRECT ? 0u : nwave * (uint32_t)p.b.chunk;
    TileShare* share = reinterpret_cast<TileShare*>(smem);            // two slots, kTileShareBytes in all
    PosEntry* tab_a = reinterpret_cast<PosEntry*>(smem + kTablesOff);
    PosEntry* tab_b = tab_a + n_a;
    PosCoord* tabc_a = reinterpret_cast<PosCoord*>(tab_b + n_b);
    PosCoord* tabc_b = tabc_a + n_a;

    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    build_tables<DIRECT>(p.a, nwave, threadIdx.x, blockDim.x, sc_a, tab_a, tabc_a);
    if (!DIRECT) build_tables<false>(p.b, nwave, threadIdx.x, blockDim.x, sc_b, tab_b, tabc_b);
    const LaneState LA = lane_setup<DIRECT>(p.a, lane, sc_a);
    const LaneState LB = DIRECT ? LA : lane_setup<false>(p.b, lane, sc_b);
    const Epilogue<TA, TB, MODE> epi(p.alpha, p.beta);
    const bool nt_a = p.nt_a != 0, nt_b = p.nt_b != 0;
    unsigned char* spare = smem + kTileShareBytes + lane * 16;      // where this lane parks what it must not keep
    const TileSeq seq = tile_sequence(p, blockIdx.x);

    // Staged kernel: the last wavefront works out where a tile lies (scalar divisions and
    // multiplications) one tile ahead and leaves the result in LDS; the barrier that already
    // separates the two walks of the current tile publishes it to the other wavefronts.
    auto publish = [&](uint32_t tile, uint32_t slot) __attribute__((always_inline)) {     // (not inlined, it would need the parameter block in memory)
        const TileBase tb = tile_base(p, tile);
        const TileLim tl = tile_lim(p, tile);
        TileShare v;
        v.a = tb.a; v.b = tb.b;
        v.sa = make_side_share(p.a, tl);
        v.sb = make_side_share(p.b, tl);
        share[slot] = v;
    };
    const uint32_t single_a = single_digits(p.a), single_b = DIRECT ? 0u : single_digits(p.b);
    if (!DIRECT && wave == nwave - 1 && seq.first < seq.end) publish(tile_of(seq, seq.first), 0);
    __syncthreads();
    if (p.debug_stop) return;

    uint32_t parity = 0;
    for (uint32_t q = seq.first; q < seq.end; q += seq.step) {
        const uint32_t tile = tile_of(seq, q);
        TileBase tb;
        SideLim sla, slb;
        WalkMask wma, wmb;
        if (DIRECT) {
            tb = tile_base(p, tile);
            const TileLim tl = tile_lim(p, tile);
            sla = side_lim(p.a, tl);
            wma = walk_mask(p.a, LA, sla);
            slb = sla; wmb = wma;
        } else {
            const TileShare v = share[parity];
            tb.a = uniform64(v.a); tb.b = uniform64(v.b);
            take_side(v.sa, single_a, LA, &sla, &wma);
            take_side(v.sb, single_b, LB, &slb, &wmb);
        }
        const unsigned char* At = reinterpret_cast<const unsigned char*>(A + tb.a);
        unsigned char* Bt = reinterpret_cast<unsigned char*>(B + tb.b);
        if (DIRECT) {
            auto run = [&](auto stream) {            // the direct kernel streams both tensors or neither
                constexpr bool NT = decltype(stream)::value;
                constexpr int kUnroll = Unroll<TA, VA>::value;
                Pack<TA, VA> ra[kUnroll];
                Pack<TB, VA> rb[kUnroll];
                auto load = [&](int u, const PosEntry& e, int back, bool ok) {
                    ra[u] = load_pack<TA, VA, NT>(At, ok ? e.g + LA.g - back * kScaleA : 0);
                    if (MODE == TTC_EPI_AXPBY) rb[u] = load_pack<TB, VA, NT>(Bt, ok ? e.l_or_g2 + LA.g2 - back * kScaleB : 0);
                };
                auto store = [&](int u, const PosEntry& e, int back, bool ok) {
                    if (!ok) return;
                    Pack<TB, VA> out;
#pragma unroll
                    for (int j = 0; j < VA; ++j) {
                        TB old = TB();
                        if (MODE == TTC_EPI_AXPBY) old = rb[u].v[j];
                        out.v[j] = epi(ra[u].v[j], old);
                    }
                    store_pack<TB, VA, NT>(Bt, e.l_or_g2 + LA.g2 - back * kScaleB, out);
                };
                walk<kUnroll, VA>(p.a, LA, sla, wma, tab_a, tabc_a, wave, load, store);
            };
            if (nt_a && nt_b) run(std::true_type()); else run(std::false_type());
            continue;
        }

        unsigned char* lds = smem + p.lds_data_off +
                             (parity & (uint32_t)(p.lds_buffers - 1)) * (uint32_t)(p.lds_tile_elems * kScaleA);
        parity ^= 1u;
        // ---- walk 1: A order, global -> LDS
        {
            auto run = [&](auto stream) {
                constexpr bool NT = decltype(stream)::value;
                const int32_t vs = p.a.vec_lds_stride;
                constexpr int kUnroll = Unroll<TA, VA>::value;
                Pack<TA, VA> ra[kUnroll];
                auto load = [&](int u, const PosEntry& e, int back, bool ok) {
                    ra[u] = load_pack<TA, VA, NT>(At, ok ? e.g + LA.g - back * kScaleA : 0);
                };
                auto park = [&](int u, const PosEntry& e, int back, bool ok) {
                    unsigned char* dst = lds + ((int32_t)e.l_or_g2 + LA.l - back * vs * kScaleA);
#pragma unroll
                    for (int j = 0; j < VA; ++j)
                        *reinterpret_cast<TA*>(ok ? dst + j * vs * kScaleA : spare) = ra[u].v[j];
                };
                walk<kUnroll, VA>(p.a, LA, sla, wma, tab_a, tabc_a, wave, load, park);
            };
            if (nt_a) run(std::true_type()); else run(std::false_type());
        }
        if (wave == nwave - 1 && q + seq.step < seq.end) publish(tile_of(seq, q + seq.step), parity);   // parity already flipped
        __syncthreads();
        // ---- walk 2: B order, LDS -> epilogue -> global
        {
            auto run = [&](auto stream) {
                constexpr bool NT = decltype(stream)::value;
                const int32_t vs = p.b.vec_lds_stride;
                constexpr int kUnroll = Unroll<TB, VB>::value;
                Pack<TB, VB> rb[kUnroll];
                Pack<TA, VB> rl[kUnroll];
                auto load = [&](int u, const PosEntry& e, int back, bool ok) {
                    if (MODE == TTC_EPI_AXPBY) rb[u] = load_pack<TB, VB, NT>(Bt, ok ? e.g + LB.g - back * kScaleB : 0);
                    const TA* src = reinterpret_cast<const TA*>(lds + (ok ? (int32_t)e.l_or_g2 + LB.l - back * vs * kScaleA : 0));
#pragma unroll
                    for (int j = 0; j < VB; ++j) rl[u].v[j] = src[j * vs];
                };
                auto store = [&](int u, const PosEntry& e, int back, bool ok) {
                    if (!ok) return;
                    Pack<TB, VB> out;
#pragma unroll
                    for (int j = 0; j < VB; ++j) {
                        TB old = TB();
                        if (MODE == TTC_EPI_AXPBY) old = rb[u].v[j];
                        out.v[j] = epi(rl[u].v[j], old);
                    }
                    store_pack<TB, VB, NT>(Bt, e.g + LB.g - back * kScaleB, out);
                };
                walk<kUnroll, VB>(p.b, LB, slb, wmb, tab_b, tabc_b, wave, load, store);
            };
            if (nt_b) run(std::true_type()); else run(std::false_type());
        }
        if (p.lds_buffers == 1) __syncthreads();      // the one buffer is refilled by the next tile
    }
}

// ---------------------------------------------------------------------------------
// The row kernel, for the case where the stride-1 index keeps its place and rows are contiguous in both tensors
// (paper Section 3.1, case 1: the first column is copied, inside loops over the other indices).  B is walked in the order of its
// multi-index: a workgroup moves a chunk of consecutive vectors, so consecutive chunks are consecutive memory (a dense B
// is written front to back like a copy), and every lane gathers its vectors from the rows of A.  No tiles, no LDS, no
// tables: a lane finds its row by one division and the row's place in both tensors by one division per index.
// Dense B (FLAT): vectors are counted from B's first element, 16-byte aligned as B itself is, whatever the rows' length;
// one that spans the end of a row takes its two parts from two rows of A (a second load for the few lanes that need
// it), and every element of B is written once, so it serves an update too.  917 x 374 x 153 fp32 (0,2,1): 70 us; with
// vectors counted row by row, 4-byte aligned, 76 us.
// Else: a row holds `slots` vectors; where it is not a multiple of the vector, its last one is moved back to end with the
// row and repeats up to V-1 elements of its neighbour with the same values (only where B is not read: with beta != 0
// the planner picks a vector that divides the row).
// Chunks are dealt to the XCDs 32 at a time: neighbours share lines of A, and of B where a chunk ends inside a line; dealt
// one by one to eight L2s the same 917 x 374 x 153 takes 69.9 us, in groups 69.1; 384^3 74.0 and 72.9 us.
// ---------------------------------------------------------------------------------
constexpr int kRowsThreads = 256;

template <typename TA, typename TB, int MODE, int V, int U, bool FLAT>
__device__ __forceinline__ void rows_chunk(const RowsParams& p, int64_t base, uint32_t row0, uint32_t slot0, const TA* __restrict__ A, TB* __restrict__ B)
{
    constexpr int32_t kScaleA = (int32_t)sizeof(TA), kScaleB = (int32_t)sizeof(TB);
    const Epilogue<TA, TB, MODE> epi(p.alpha, p.beta);
    const unsigned char* Ab = reinterpret_cast<const unsigned char*>(A);
    unsigned char* Bb = reinterpret_cast<unsigned char*>(B);
    auto run = [&](auto stream_a, auto stream_b) {
        constexpr bool NTA = decltype(stream_a)::value, NTB = decltype(stream_b)::value;
        Pack<TA, V> ra[U];
        Pack<TB, V> rb[U];
        int64_t to[U];
        int32_t count[U];                                               // elements to store: V, 0 past the end, fewer at the end of a flat B
        // a lane past the end of the tensor loads the first vector instead and stores nothing, so that no load
        // sits in divergent control flow (the second part of a split vector is the exception)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t k = (uint32_t)u * kRowsThreads + threadIdx.x;
            if (FLAT) {
                const FlatAccess x = flat_access(p, base, row0, slot0, k);
                count[u] = x.valid ? (int32_t)(x.left < V ? x.left : V) : 0;
                to[u] = (count[u] == V ? x.b : p.elements - V) * kScaleB;               // where B is loaded from
                ra[u] = load_pack<TA, V, NTA>(Ab, x.a * kScaleA);
                if (MODE == TTC_EPI_AXPBY) rb[u] = load_pack<TB, V, NTB>(Bb, to[u]);
                if (V > 1 && x.split) {
                    const Pack<TA, V> next = load_pack<TA, V, false>(Ab, x.a_next * kScaleA);
                    Pack<TA, V> both;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        TA v = next.v[0];
#pragma unroll
                        for (int e = 0; e < V; ++e) {
                            if (e == j + V - (int)x.head) v = ra[u].v[e];                // j < head: the last elements of row r
                            if (e == j - (int)x.head) v = next.v[e];
                        }
                        both.v[j] = v;
                    }
                    ra[u] = both;
                }
                if (V > 1 && MODE == TTC_EPI_AXPBY && count[u] > 0 && count[u] < V) {    // the last vector of B: what was loaded ends with B
                    Pack<TB, V> last;
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        TB v = rb[u].v[0];
#pragma unroll
                        for (int e = 0; e < V; ++e) if (e == j + V - count[u]) v = rb[u].v[e];
                        last.v[j] = v;
                    }
                    rb[u] = last;
                }
                if (count[u] > 0) to[u] = x.b * kScaleB;
            } else {
                const RowAccess x = rows_access(p, base, row0, slot0, k);
                count[u] = x.valid ? V : 0;
                to[u] = x.at.b * kScaleB;
                ra[u] = load_pack<TA, V, NTA>(Ab, x.at.a * kScaleA);
                if (MODE == TTC_EPI_AXPBY) rb[u] = load_pack<TB, V, NTB>(Bb, to[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (count[u] == 0) continue;
            Pack<TB, V> out;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                TB old = TB();
                if (MODE == TTC_EPI_AXPBY) old = rb[u].v[j];
                out.v[j] = epi(ra[u].v[j], old);
            }
            if (!FLAT || V == 1 || count[u] == V) {
                store_pack<TB, V, NTB>(Bb, to[u], out);
            } else {
#pragma unroll
                for (int j = 0; j < V; ++j) if (j < count[u]) reinterpret_cast<TB*>(Bb + to[u])[j] = out.v[j];
            }
        }
    };
    if (p.nt_a) { if (p.nt_b) run(std::true_type(), std::true_type()); else run(std::true_type(), std::false_type()); }
    else        { if (p.nt_b) run(std::false_type(), std::true_type()); else run(std::false_type(), std::false_type()); }
}

template <typename TA, typename TB, int MODE, int V, int U, bool FLAT>
__global__ __launch_bounds__(kRowsThreads) void rows_kernel(const RowsParams p, const TA* __restrict__ A, TB* __restrict__ B)
{
    const uint32_t block = rows_block(p, blockIdx.x);
    if (block >= p.blocks) return;
    const int64_t base = (int64_t)block * (int64_t)p.chunk * (FLAT ? V : 1);
    const int64_t row0_wide = base / (int64_t)p.slots;                  // wave-uniform: once per workgroup
    rows_chunk<TA, TB, MODE, V, U, FLAT>(p, base, (uint32_t)row0_wide, (uint32_t)(base - row0_wide * (int64_t)p.slots), A, B);
}

// The same for small problems over a dense B, with its arguments packed (SmallArgs) and the usual hints (A kept, B streamed).  RANGES: each
// XCD has one range of chunks.
template <typename TA, typename TB, int MODE, int V, int N, bool RANGES>
__global__ __launch_bounds__(kRowsThreads) void rows_small_kernel(const SmallArgs args_by_value, const TA* __restrict__ A, TB* __restrict__ B)
{
    const SmallArgs& s = *reinterpret_cast<const SmallArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    const RowsParams p = small_unpack<false, N, MODE, IsComplex<TA>::value>(s, V, kRowsThreads);
    const SmallRowsStart at = small_rows_start<RANGES>(p, blockIdx.x);
    rows_chunk<TA, TB, MODE, V, 1, true>(p, (int64_t)at.first, at.row0, at.col0, A, B);
}

// ---------------------------------------------------------------------------------
// The micro-tile kernel (the paper's w x w in-register transposition, Section 3.2, in its gfx950 form): a tile over
// the two stride-1 indices only (each possibly merged with the index next to it in its tensor, see MicroParams),
// every access 128 bits wide.  Lanes load 16-byte vectors along A's stride-1 index and park each with one 128-bit
// LDS write; after the barrier a lane reads the V x V block it owns with V 128-bit LDS reads (rows of the tile are
// XOR-swizzled at 16-byte granularity: neither phase has bank conflicts), transposes it in registers -- no
// cross-lane traffic: row i of the block is one register quad, column j is element j of each -- and stores V
// 16-byte vectors along B's stride-1 index.  Extents need not be multiples of V: the last vector of a row and the
// last block of a column are moved back to end with the tensor (micro_back), and where B is updated as well a
// moved block writes only what is its own.  Both tensors have one element type of 4 or 8 bytes.
// ---------------------------------------------------------------------------------
template <typename T, int MODE, int V>
__global__ __launch_bounds__(256) void micro_kernel(const MicroArgs args_by_value, const T* __restrict__ A, T* __restrict__ B)
{
    static_assert(V * sizeof(T) == 16, "one 16-byte vector");
    const MicroArgs& p = *reinterpret_cast<const MicroArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    extern __shared__ __align__(16) unsigned char smem[];
    typedef uint32_t Quad __attribute__((ext_vector_type(4)));
    Quad* lds = reinterpret_cast<Quad*>(smem);
    constexpr int U = 4;                                       // loads a lane keeps in flight (eight: 0-5 % slower on the suite)
    constexpr int32_t kScale = (int32_t)sizeof(T);
    const MicroParams& m = p.micro;
    const Epilogue<T, T, MODE> epi(p.alpha, p.beta);
    const uint32_t tid = threadIdx.x, threads = blockDim.x;
    const uint32_t loads = (uint32_t)m.loads, blocks = (uint32_t)m.blocks;
    const TileSeq seq = tile_sequence(p, blockIdx.x);
    for (uint32_t q = seq.first; q < seq.end; q += seq.step) {
        const MicroTile t = micro_tile(p, tile_of(seq, q));
        if (p.debug_stop == 1) return;                        // measurement aid: launch, parameters and tile decode only
        const unsigned char* At = reinterpret_cast<const unsigned char*>(A + t.a);
        unsigned char* Bt = reinterpret_cast<unsigned char*>(B + t.b);
        auto run = [&](auto stream_a, auto stream_b) {
            constexpr bool NTA = decltype(stream_a)::value, NTB = decltype(stream_b)::value;
            union Vec { Pack<T, V> p; Quad q; };
            // ---- A order: global -> LDS, U vectors at a time.  A lane whose vector lies outside the tensor loads the
            // tile's first vector instead (no load in divergent control flow); what it parks nobody reads.
            for (uint32_t k0 = 0; k0 < loads; k0 += U) {
                Vec in[U];
                MicroLoad x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    x[u] = micro_load(m, threads, tid, k0 + (uint32_t)u);
                    const bool ok = x[u].valid && x[u].row < t.lim_b && x[u].col < t.lim_a;
                    const uint32_t col = ok ? micro_back(x[u].col, t.lim_a, V) : 0u;
                    in[u].p = load_pack<T, V, NTA>(At, (micro_row_a(m, t.row0 + (ok ? x[u].row : 0u)) + (int64_t)col) * kScale);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (x[u].valid) lds[x[u].chunk] = in[u].q;
            }
            __syncthreads();
            if (p.debug_stop == 2) return;                     // measurement aid: ... and the loads of A into LDS
            // ---- B order: LDS -> registers (V x V block) -> epilogue -> global
            for (uint32_t b = 0; b < blocks; ++b) {
                const MicroBlock x = micro_block(m, threads, tid, b);
                const bool ok = x.valid && x.row < t.lim_b && x.col < t.lim_a;
                const uint32_t row = ok ? micro_back(x.row, t.lim_b, V) : 0u, col = ok ? micro_back(x.col, t.lim_a, V) : 0u;
                const uint32_t lane_c = ok ? x.lane_c : 0u;
                int64_t to[V];                                  // byte offsets of the block's V columns in B
#pragma unroll
                for (int j = 0; j < V; ++j) to[j] = (micro_col_b(m, t.col0 + col + (uint32_t)j) + (int64_t)row) * kScale;
                Pack<T, V> old[V];
                if (MODE == TTC_EPI_AXPBY) {
#pragma unroll
                    for (int j = 0; j < V; ++j) old[j] = load_pack<T, V, NTB>(Bt, to[j]);
                }
                Vec blk[V];
#pragma unroll
                for (int i = 0; i < V; ++i) blk[i].q = lds[micro_slot(m, row + (uint32_t)i, lane_c)];
                // Where B is read as well as written an element must be updated once: a block that was moved back, or
                // lies in a tile that was, updates only what is its own (from its nominal place on, and not the
                // neighbouring tile's elements), element by element.  Such blocks exist at the tensor's edge only.
                const bool edge = MODE == TTC_EPI_AXPBY && ok && (row != x.row || col != x.col || x.row < t.own_b || x.col < t.own_a);
                if (MODE == TTC_EPI_AXPBY && edge) {
                    const uint32_t first_row = x.row > t.own_b ? x.row : t.own_b, first_col = x.col > t.own_a ? x.col : t.own_a;
#pragma unroll
                    for (int j = 0; j < V; ++j)
#pragma unroll
                        for (int i = 0; i < V; ++i)
                            if (col + (uint32_t)j >= first_col && row + (uint32_t)i >= first_row) {
                                T* pb = reinterpret_cast<T*>(Bt + to[j]) + i;
                                *pb = epi(blk[i].p.v[j], *pb);
                            }
                } else if (ok) {
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        Pack<T, V> out;
#pragma unroll
                        for (int i = 0; i < V; ++i) {
                            T b_old = T();
                            if (MODE == TTC_EPI_AXPBY) b_old = old[j].v[i];
                            out.v[i] = epi(blk[i].p.v[j], b_old);
                        }
                        store_pack<T, V, NTB>(Bt, to[j], out);
                    }
                }
            }
        };
        if (p.nt_a) { if (p.nt_b) run(std::true_type(), std::true_type()); else run(std::true_type(), std::false_type()); }
        else        { if (p.nt_b) run(std::false_type(), std::true_type()); else run(std::false_type(), std::false_type()); }
        __syncthreads();                                       // the tile buffer is refilled by the next tile
    }
}

template <typename TA, typename TB, int MODE>
inline hipError_t launch_micro(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    if constexpr (std::is_same<TA, TB>::value && (sizeof(TA) == 4 || sizeof(TA) == 8)) {
        constexpr int V = 16 / (int)sizeof(TA);
        const KernelParams& kp = c.kp;
        const MicroParams& m = kp.micro;
        const uint32_t grid = kp.num_tiles;                    // one tile per workgroup: the hardware deals them
        const int64_t th = c.threads;
        if (m.vec != V || (1 << m.vec_log) != V || (th != 64 && th != 128 && th != 256) || m.la < 1 || m.lb < 1 ||
            m.ta != m.la * V || m.tb != m.lb * V || m.pitch < m.la || (m.pitch & 7) || (m.swizzle != 7u && m.swizzle != 0u) || m.la_div.div != (uint32_t)m.la ||
            m.lb_div.div != (uint32_t)m.lb || (int64_t)m.loads * th < (int64_t)m.la * m.tb || (int64_t)m.blocks * th < (int64_t)m.la * m.lb ||
            (int64_t)(m.loads + 4) * th >= (int64_t(1) << 31) ||
            c.lds_bytes != m.tb * m.pitch * 16 || c.lds_bytes > 64 * 1024 || !launchable(grid, c.threads) || grid != kp.grid ||
            m.size_a0 < V || m.size_p0 < V || m.size_a0 >= (int64_t(1) << 31) || m.size_p0 >= (int64_t(1) << 31) ||
            m.col_in_div.div < 1 || m.row_in_div.div < 1)
            return hipErrorInvalidValue;
        const void* fn = reinterpret_cast<const void*>(&micro_kernel<TA, MODE, V>);
        const TA* a = static_cast<const TA*>(A);
        TA* b = static_cast<TA*>(B);
        // TTC_DEBUG_STOP=1 or 2 in the environment: workgroups return early (how the parts of a launch were timed)
        static const int stop = std::getenv("TTC_DEBUG_STOP") ? std::atoi(std::getenv("TTC_DEBUG_STOP")) : 0;
        MicroArgs ready = micro_args(c);
        ready.debug_stop = stop;
        void* args[] = {&ready, &a, &b};
        return hipLaunchKernel(fn, dim3(grid), dim3(c.threads), args, (size_t)c.lds_bytes, stream);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------
// The line kernel: a tile of COLS columns by the rows of LINES 128-byte lines of B.
// What it is for: columns of B that do not start on lines (odd extents, leading dimensions).  A tile cut at one row
// for all its columns then begins and ends inside a line in almost every column, and a line written in two parts by
// two workgroups costs two masked writes: 7200 x 7200 fp32 took 72 us with both tensors' leading dimension 7232
// (whole lines) and 99 us (82 searched) with B's 7241, although the bytes are the same.  Here every column is cut
// where its own lines end, so each line is written once and whole; the price is that a tile reads up to a line's
// worth of rows of its neighbour again, and both tiles the line of A that their common edge splits.  77 us, whatever B's
// leading dimension; 79 against 92-105 us with both at 7241.
// How much of that comes from the caches depends on the order of the tiles.  The 6-D reversal 24 x 20 x 16 x 18 x 22 x 17
// (merged on both sides, 24-element runs of A) asks for 1.32 lines per line of A and reads 1.03 times A from memory (81 us);
// 85^4 reversed asks for 1.98 and reads A 1.51 times (90 us; in tiles of 32 columns 2.25, 2.03 times and 97 us): the next tile along A
// comes tens of tiles later there, on another XCD.
// It also takes what the micro-tile kernel does not: 16-byte elements and two precisions (B's lines aligned or not).
//
// Loads: 16 bytes a lane along A, all of a tile's rows in flight at once, parked row by row in LDS.
// Stores: eight lanes per line and eight neighbouring columns per instruction; a lane keeps its column for the whole
// tile, so a line costs it LDS reads at constant offsets and one 16-byte store.  With an update, B's lines are loaded
// before the barrier, beside the loads of A.  One tile per workgroup.
// ---------------------------------------------------------------------------------
template <typename TA, typename TB, int MODE, int COLS, int LINES>
__device__ __forceinline__ void line_tile_move(const MicroArgs& p, uint32_t tile, const TA* __restrict__ A, TB* __restrict__ B)
{
    constexpr LineShape S = line_shape(COLS, LINES, (int)sizeof(TA), (int)sizeof(TB));
    static_assert(line_shape_ok(COLS, LINES, (int)sizeof(TA), (int)sizeof(TB)), "no such tile");
    constexpr int VA = S.va, VB = S.vb, L = S.line, U = S.passes;
    constexpr int G = COLS / S.side, N = LINES / S.groups;     // columns a lane stores, and lines of each
    __shared__ __align__(16) unsigned char smem[S.lds_bytes];
    TA* const lds = reinterpret_cast<TA*>(smem);
    const MicroParams& m = p.micro;
    const Epilogue<TA, TB, MODE> epi(p.alpha, p.beta);
    const uint32_t tid = threadIdx.x;
    const int32_t rows = (int32_t)m.size_p0;
    const LineTile t = line_tile(p, S, tile);
    auto run = [&](auto stream_a, auto stream_b) {
        constexpr bool NTA = decltype(stream_a)::value, NTB = decltype(stream_b)::value;
        union Vec { Pack<TA, VA> p; uint32_t w[4]; };
        Vec in[U];
        const unsigned char* At = reinterpret_cast<const unsigned char*>(A + t.a);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const LineLoad x = line_load(m, S, t, tid, u);
            if (x.needed) in[u].p = load_pack<TA, VA, NTA>(At, (micro_row_a(m, x.row) + (int64_t)x.start) * (int64_t)sizeof(TA));
        }
        // the lane's columns: where row 0 of each lies in B, and at which place of a line
        unsigned char* to[G];
        int32_t y0[G];
        bool mine[G];
        Pack<TB, VB> old[G][N];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int32_t c = line_column(S, tid, g);
            mine[g] = c < t.cols;
            TB* col = B + (t.b + micro_col_b(m, t.col0 + (uint32_t)(mine[g] ? c : 0)));
            const int32_t phase = (int32_t)((reinterpret_cast<uintptr_t>(col) & (kLineBytes - 1)) / sizeof(TB));
            y0[g] = line_row(m, S, t, phase, tid);
            to[g] = reinterpret_cast<unsigned char*>(col);
            if (MODE == TTC_EPI_AXPBY) {
#pragma unroll
                for (int i = 0; i < N; ++i) {               // a vector that is not whole is loaded from the column's edge
                    const int32_t y = y0[g] + i * S.groups * L, top = rows - VB;
                    old[g][i] = load_pack<TB, VB, NTB>(to[g], (int64_t)(y < 0 ? 0 : (y > top ? top : y)) * (int64_t)sizeof(TB));
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const LineLoad x = line_load(m, S, t, tid, u);
            if (!x.needed || x.col >= t.cols) continue;
            TA* dst = lds + x.lds_row * S.pitch + x.start;
            if (x.start == x.col) {
                typedef uint32_t Half __attribute__((ext_vector_type(2)));
                typedef uint32_t Quad __attribute__((ext_vector_type(4)));
                if (sizeof(TA) == 4) {                     // rows start on 8-byte boundaries
                    Half* h = reinterpret_cast<Half*>(dst);
                    h[0] = Half{in[u].w[0], in[u].w[1]};
                    h[1] = Half{in[u].w[2], in[u].w[3]};
                } else {
                    *reinterpret_cast<Quad*>(dst) = Quad{in[u].w[0], in[u].w[1], in[u].w[2], in[u].w[3]};
                }
            } else {                                       // moved back: what lies before the tile belongs to another one
#pragma unroll
                for (int j = 0; j < VA; ++j)
                    if (x.start + j >= 0) dst[j] = in[u].p.v[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (!mine[g]) continue;
            const TA* src = lds + (y0[g] - t.row0) * S.pitch + line_column(S, tid, g);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (line_last(m, S, tid, i)) continue;
                const int32_t y = y0[g] + i * S.groups * L;
                TA a[VB];
#pragma unroll
                for (int j = 0; j < VB; ++j) a[j] = src[(i * S.groups * L + j) * S.pitch];
                const int64_t at = (int64_t)y * (int64_t)sizeof(TB);
                if (y >= 0 && y + VB <= rows) {
                    Pack<TB, VB> out;
#pragma unroll
                    for (int j = 0; j < VB; ++j) {
                        TB b_old = TB();
                        if (MODE == TTC_EPI_AXPBY) b_old = old[g][i].v[j];
                        out.v[j] = epi(a[j], b_old);
                    }
                    store_pack<TB, VB, NTB>(to[g], at, out);
                } else {
                    // The first and the last vector of a column: element by element.  What B held was loaded from
                    // the column's edge: row y + j is element j + (y - edge) of that vector.  (Loads here, one
                    // waiting for the other, made 85^4 fp32 (3,0,2,1) with an update 40 % slower.)
                    const int32_t shift = y < 0 ? y : y - (rows - VB);
#pragma unroll
                    for (int j = 0; j < VB; ++j) {
                        TB b_old = TB();
                        if (MODE == TTC_EPI_AXPBY) {
#pragma unroll
                            for (int e = 0; e < VB; ++e) if (e == j + shift) b_old = old[g][i].v[e];
                        }
                        if (y + j >= 0 && y + j < rows) reinterpret_cast<TB*>(to[g] + at)[j] = epi(a[j], b_old);
                    }
                }
            }
        }
    };
    if (p.nt_a) { if (p.nt_b) run(std::true_type(), std::true_type()); else run(std::true_type(), std::false_type()); }
    else        { if (p.nt_b) run(std::false_type(), std::true_type()); else run(std::false_type(), std::false_type()); }
}

template <typename TA, typename TB, int MODE, int COLS, int LINES>
__global__ __launch_bounds__(kLineThreads) void line_kernel(const MicroArgs args_by_value, const TA* __restrict__ A, TB* __restrict__ B)
{
    const MicroArgs& p = *reinterpret_cast<const MicroArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    const TileSeq seq = tile_sequence(p, blockIdx.x);
    for (uint32_t q = seq.first; q < seq.end; q += seq.step) {
        line_tile_move<TA, TB, MODE, COLS, LINES>(p, tile_of(seq, q), A, B);
        __syncthreads();                                       // the tile buffer is refilled by the next tile
    }
}

// The same with its arguments packed (SmallArgs), one tile per workgroup, where small_line() finds room for them: 96 of 154 plans of
// random problems of 64 KB to 1.9 GB (not four places in the tile order, not updates over merged indices).  Three ways of dealing tiles.
// kDealNone, for fewer than 2048 tiles that share nothing: a workgroup's number is its tile's (1024 x 1024 fp32 2.77 us, with kDealAll
// 3.04; 1680 x 289 complex64 with an update 4.26 and 5.18; a kernel that serves kDealRanges too, and so has to look at its arguments
// before it may go on, is 1-2 % slower in the mean over 5000 problems below 32 MB and 6-8 % on a tenth of them).  kDealRanges: one
// range per XCD.  kDealAll: any mapping, and A may be streamed.
template <typename TA, typename TB, int MODE, int COLS, int LINES, bool MERGED, int DEAL>
__global__ __launch_bounds__(kLineThreads) void line_small_kernel(const SmallArgs args_by_value, const TA* __restrict__ A, TB* __restrict__ B)
{
    const SmallArgs& s = *reinterpret_cast<const SmallArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    constexpr LineShape S = line_shape(COLS, LINES, (int)sizeof(TA), (int)sizeof(TB));
    uint32_t tile = blockIdx.x;
    if (DEAL != kDealNone) {
        const SmallDeal deal = small_line_deal(s, MERGED);
        tile = DEAL == kDealAll ? rows_block(deal, tile) : small_line_range(deal, tile);
        if (tile >= deal.blocks) return;
    }
    const MicroArgs p = small_line_unpack<MODE, IsComplex<TA>::value, MERGED, DEAL == kDealAll>(s, COLS, S);
    line_tile_move<TA, TB, MODE, COLS, LINES>(p, tile, A, B);
}

// The packed kernel for a way of dealing.  Where there is none for kDealAll (small_line_deals()), such a launch is not packed.
template <typename TA, typename TB, int MODE, int COLS, int LINES, bool MERGED>
inline const void* small_line_function(int deal)
{
    constexpr LineShape S = line_shape(COLS, LINES, (int)sizeof(TA), (int)sizeof(TB));
    if (deal == kDealNone) return reinterpret_cast<const void*>(&line_small_kernel<TA, TB, MODE, COLS, LINES, MERGED, kDealNone>);
    if (deal == kDealRanges) return reinterpret_cast<const void*>(&line_small_kernel<TA, TB, MODE, COLS, LINES, MERGED, kDealRanges>);
    if constexpr (small_line_deals(MODE, S.passes)) return reinterpret_cast<const void*>(&line_small_kernel<TA, TB, MODE, COLS, LINES, MERGED, kDealAll>);
    return nullptr;
}

template <typename TA, typename TB, int MODE, int COLS, int LINES>
inline hipError_t launch_line_shape(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    if constexpr (line_shape_ok(COLS, LINES, (int)sizeof(TA), (int)sizeof(TB))) {
        constexpr LineShape S = line_shape(COLS, LINES, (int)sizeof(TA), (int)sizeof(TB));
        const KernelParams& kp = c.kp;
        const MicroParams& m = kp.micro;
        if (m.ta != COLS || m.lines != LINES || (m.skewed | 1) != 1 || m.tb != (LINES - m.skewed) * S.line || c.threads != kLineThreads ||
            c.lds_bytes != S.lds_bytes || !launchable(kp.num_tiles, kLineThreads) || kp.grid != kp.num_tiles || m.size_a0 < S.va || m.size_p0 < S.vb ||
            m.size_a0 >= kLineMaxExtent || m.size_p0 >= kLineMaxExtent || m.col_in_div.div < 1 || m.row_in_div.div < 1)
            return hipErrorInvalidValue;
        const void* fn = reinterpret_cast<const void*>(&line_kernel<TA, TB, MODE, COLS, LINES>);
        const TA* a = static_cast<const TA*>(A);
        TB* b = static_cast<TB*>(B);
        MicroArgs ready = micro_args(c);
        const int packed = small_line(ready, MODE, IsComplex<TA>::value, S.passes);
        if (packed) {
            SmallArgs small = small_line_pack(ready, MODE, IsComplex<TA>::value);
            void* args[] = {&small, &a, &b};
            const void* small_fn = nullptr;
            const int deal = small_line_dealing(ready);
            if constexpr (small_line_fits(false, MODE, IsComplex<TA>::value))
                if (packed == 1) small_fn = small_line_function<TA, TB, MODE, COLS, LINES, false>(deal);
            if constexpr (small_line_fits(true, MODE, IsComplex<TA>::value))
                if (packed == 2) small_fn = small_line_function<TA, TB, MODE, COLS, LINES, true>(deal);
            const int64_t grid = rows_grid(small_line_deal(small, packed == 2));
            if (small_fn && launchable(grid, kLineThreads)) return hipLaunchKernel(small_fn, dim3((uint32_t)grid), dim3(kLineThreads), args, 0, stream);
        }
        void* args[] = {&ready, &a, &b};
        return hipLaunchKernel(fn, dim3(kp.num_tiles), dim3(kLineThreads), args, 0, stream);
    }
    return hipErrorInvalidValue;
}

template <typename TA, typename TB, int MODE, int COLS>
inline hipError_t launch_line_cols(const Candidate& c, const void* A, void* B, hipStream_t s)
{
    switch (c.kp.micro.lines) {
    case 2: return launch_line_shape<TA, TB, MODE, COLS, 2>(c, A, B, s);
    case 4: return launch_line_shape<TA, TB, MODE, COLS, 4>(c, A, B, s);
    case 8: return launch_line_shape<TA, TB, MODE, COLS, 8>(c, A, B, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename TA, typename TB, int MODE>
inline hipError_t launch_lines(const Candidate& c, const void* A, void* B, hipStream_t s)
{
    switch (c.kp.micro.ta) {
    case 16: return launch_line_cols<TA, TB, MODE, 16>(c, A, B, s);
    case 32: return launch_line_cols<TA, TB, MODE, 32>(c, A, B, s);
    case 64: return launch_line_cols<TA, TB, MODE, 64>(c, A, B, s);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------------
// The block kernel: a box of the tensor that is one or a few long contiguous runs of B and runs of whole lines of A, moved by
// a one-shot workgroup.
// What it is for: problems whose leading indices in A and in B overlap, or are short.  The box kernel moves the same boxes, but
// a workgroup first builds position tables and then walks several tiles between barriers; here a lane finds its U vectors
// by a few divisions, has all of them in flight at once (an update: B's as well), and one barrier separates loads from stores.
// What bounds it is memory, then how fast the device starts workgroups: one of 256 threads every 1.7 ns, so a tile of 6-12 KB is
// best (24 x 20 x 16 x 18 x 22 x 17 fp32 (1,0,2,3,5,4), tiles of 1.9, 3.8, 5.8, 11.5 and 31 KB: 181, 97, 75, 70 and 74 us).  Kernels that
// only read reach 6.0-6.9 TB/s in any order of whole lines, kernels that only write 6.4 TB/s front to back but 4.7-5.8 where a launch writes 32 and more
// places at once: as much of B's run as the tile can hold is better than more of A's.
// Box kernel -> here: the same problem as an update 109 -> 95 us (6.5 TB/s), 3 x 307200 x 64 fp32 (1,0,2) 82.4 -> 74.0
// (6.4 TB/s), 12 x 1000 x 12 x 300 fp32 (2,1,0,3) 62 -> 56, 8 x 9 x 7 x 96 x 104 complex128 (1,2,3,4,0) 35.5 -> 28.6.  The first two
// pass 1.0002 and 1.0006 times what they have to through memory; of 9.6 and 8.0 LDS cycles an instruction 6.4 and 4.8 are bank conflicts,
// which the memory hides.
// One tile per workgroup, and no loop over tiles around it: with one the same two problems took 111 and 89 us.
// ---------------------------------------------------------------------------------
template <typename TA, typename TB, int MODE, int U>
__global__ __launch_bounds__(kBlockThreads) void block_kernel(const BlockArgs args_by_value, const TA* __restrict__ A, TB* __restrict__ B)
{
    const BlockArgs& p = *reinterpret_cast<const BlockArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    constexpr int VA = 16 / (int)sizeof(TA), VB = 16 / (int)sizeof(TB), UB = block_stores(U, (int)sizeof(TA), (int)sizeof(TB));
    extern __shared__ __align__(16) unsigned char smem[];
    TA* const lds = reinterpret_cast<TA*>(smem);
    const BlockParams& m = p.block;
    const Epilogue<TA, TB, MODE> epi(p.alpha, p.beta);
    const uint32_t tid = threadIdx.x;
    const uint32_t block = rows_block(p, blockIdx.x);
    if (block >= p.blocks) return;
    const BlockTile t = block_tile(p, block);
    const unsigned char* At = reinterpret_cast<const unsigned char*>(A + t.a);
    unsigned char* Bt = reinterpret_cast<unsigned char*>(B + t.b);
    auto run = [&](auto stream_a, auto stream_b) {
        constexpr bool NTA = decltype(stream_a)::value, NTB = decltype(stream_b)::value;
        union Vec { Pack<TA, VA> p; uint32_t w[4]; };
        typedef uint32_t Quad __attribute__((ext_vector_type(4)));
        Vec in[U];
        Pack<TB, VB> old[UB];
#pragma unroll
        for (int u = 0; u < U; ++u)
            in[u].p = load_pack<TA, VA, NTA>(At, block_load(m, t, tid + (uint32_t)(u * kBlockThreads), VA).a * (int64_t)sizeof(TA));
        if (MODE == TTC_EPI_AXPBY) {
#pragma unroll
            for (int u = 0; u < UB; ++u)
                old[u] = load_pack<TB, VB, NTB>(Bt, block_store(m, t, tid + (uint32_t)(u * kBlockThreads), VB).from * (int64_t)sizeof(TB));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const BlockLoad x = block_load(m, t, tid + (uint32_t)(u * kBlockThreads), VA);
            if (!x.ok) continue;
            if (x.start == x.col) {
                *reinterpret_cast<Quad*>(lds + x.lds) = Quad{in[u].w[0], in[u].w[1], in[u].w[2], in[u].w[3]};
            } else {                                           // moved back: what lies before the tile belongs to another one
#pragma unroll
                for (int j = 0; j < VA; ++j)
                    if (x.start + j >= 0) lds[x.lds + j] = in[u].p.v[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const BlockStore x = block_store(m, t, tid + (uint32_t)(u * kBlockThreads), VB);
            if (x.count == 0) continue;
            TA a[VB];
            if (m.even) {
#pragma unroll
                for (int j = 0; j < VB; ++j) a[j] = lds[x.lds + j * m.x_lds[0]];
            } else {
                int32_t at = x.lds, x0 = x.x0, x1 = x.x1;
#pragma unroll
                for (int j = 0; j < VB; ++j) {
                    a[j] = lds[at];
                    if (j + 1 < x.count) block_next(m, &at, &x0, &x1);
                }
            }
            if (x.count == VB) {
                Pack<TB, VB> out;
#pragma unroll
                for (int j = 0; j < VB; ++j) {
                    TB b_old = TB();
                    if (MODE == TTC_EPI_AXPBY) b_old = old[u].v[j];
                    out.v[j] = epi(a[j], b_old);
                }
                store_pack<TB, VB, NTB>(Bt, x.b * (int64_t)sizeof(TB), out);
            } else {
                // the end of a run: element j of it is element j + (x.b - x.from) of the vector that B was read with
                const int32_t shift = (int32_t)(x.b - x.from);
#pragma unroll
                for (int j = 0; j < VB; ++j) {
                    TB b_old = TB();
                    if (MODE == TTC_EPI_AXPBY) {
#pragma unroll
                        for (int e = 0; e < VB; ++e) if (e == j + shift) b_old = old[u].v[e];
                    }
                    if (j < x.count) reinterpret_cast<TB*>(Bt + x.b * (int64_t)sizeof(TB))[j] = epi(a[j], b_old);
                }
            }
        }
    };
    if (p.nt_a) { if (p.nt_b) run(std::true_type(), std::true_type()); else run(std::true_type(), std::false_type()); }
    else        { if (p.nt_b) run(std::false_type(), std::true_type()); else run(std::false_type(), std::false_type()); }
}

template <typename TA, typename TB, int MODE, int U>
inline hipError_t launch_block_unrolled(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    constexpr int VA = 16 / (int)sizeof(TA), VB = 16 / (int)sizeof(TB), UB = block_stores(U, (int)sizeof(TA), (int)sizeof(TB));
    const KernelParams& kp = c.kp;
    const BlockParams& m = c.block;
    if (c.threads != kBlockThreads || m.unroll != U || m.rows < 1 || m.outs < 1 || m.run_a < 1 || m.run_b < 1 || m.pitch < m.run_a ||
        m.pitch % VA != 0 || c.lds_bytes > kBlockMaxLds || (int64_t)m.rows * m.pitch * (int64_t)sizeof(TA) > c.lds_bytes ||
        (int64_t)m.va_div.div * VA < m.run_a || (int64_t)m.vb_div.div * VB < m.run_b ||
        (int64_t)m.va_div.div * m.rows > U * kBlockThreads || (int64_t)m.vb_div.div * m.outs > UB * kBlockThreads ||
        (int64_t)m.rows * m.run_a != (int64_t)m.outs * m.run_b || m.run_a != m.inner_a * m.tile_a || m.run_b != m.inner_b * m.tile_b ||
        m.run_a < VA || m.run_b < VB || kp.grid != kp.num_tiles)
        return hipErrorInvalidValue;
    const TA* a = static_cast<const TA*>(A);
    TB* b = static_cast<TB*>(B);
    BlockArgs ready = block_args(c);
    const int64_t grid = rows_grid(ready);
    if (!launchable(grid, kBlockThreads)) return hipErrorInvalidValue;
    void* args[] = {&ready, &a, &b};
    return hipLaunchKernel(reinterpret_cast<const void*>(&block_kernel<TA, TB, MODE, U>), dim3((uint32_t)grid), dim3(kBlockThreads), args,
                           (size_t)c.lds_bytes, stream);
}

template <typename TA, typename TB, int MODE>
inline hipError_t launch_block(const Candidate& c, const void* A, void* B, hipStream_t s)
{
    switch (c.block.unroll) {
    case 2: return launch_block_unrolled<TA, TB, MODE, 2>(c, A, B, s);
    case 4: return launch_block_unrolled<TA, TB, MODE, 4>(c, A, B, s);
    case 8: return launch_block_unrolled<TA, TB, MODE, 8>(c, A, B, s);
    default: return hipErrorInvalidValue;
    }
}

// Compute units of the current device (256 on MI355X), asked once per process and device.
inline int device_cus()
{
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

// ---------------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------------
template <typename TA, typename TB, int MODE, int VA, int VB, bool DIRECT>
inline hipError_t launch_one(const KernelParams& kp, const void* A, void* B, uint32_t grid, int threads,
                             int lds_bytes, hipStream_t stream)
{
    if (grid != kp.grid || grid < 1 || grid > kp.num_tiles) return hipErrorInvalidValue;
    const void* fn = reinterpret_cast<const void*>(&box_kernel<TA, TB, MODE, VA, VB, DIRECT>);
    // more than 64 KB of dynamic LDS has to be asked for, once per kernel and device (a CU of gfx950 has 160 KB)
    if (lds_bytes > 64 * 1024) {
        static std::atomic<uint64_t> raised{0};                 // bit d: done on device d
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        if (!((raised.load(std::memory_order_acquire) >> dev) & 1u)) {
            const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
            if (e != hipSuccess) return e;
            raised.fetch_or(uint64_t(1) << dev, std::memory_order_release);
        }
    }
    const TA* a = static_cast<const TA*>(A);
    TB* b = static_cast<TB*>(B);
    void* args[] = {const_cast<KernelParams*>(&kp), &a, &b};
    // the launch's own status: an error left behind by an earlier, unrelated call on this thread is not ours
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), args, (size_t)lds_bytes, stream);
}

// ---------------------------------------------------------------------------------
// The gather kernel: B is walked front to back, a lane writes 16 bytes of it and fetches their elements from A one by one.
// No tiles, no LDS, no barrier: one memory latency between launch and store, which is what a small problem costs.
// 70 x 33 x 45 fp32 (2,0,1): 2.3-2.8 us a launch, from host to host (3.3-3.5 with its arguments whole, box kernel 4.2), 2.4 line requests
// per line of A, all but 0.4 of them from L2.
// ---------------------------------------------------------------------------------
template <typename TA, typename TB, int MODE, int V>
__device__ __forceinline__ void gather_chunk(const RowsParams& p, uint32_t block, const TA* __restrict__ A, TB* __restrict__ B)
{
    static_assert(V * sizeof(TB) == 16, "one 16-byte vector of B");
    const uint32_t e = gather_first(p, block, threadIdx.x);
    if ((int64_t)e >= p.elements) return;
    const Epilogue<TA, TB, MODE> epi(p.alpha, p.beta);
    const int32_t count = p.elements - (int64_t)e < V ? (int32_t)(p.elements - (int64_t)e) : V;
    auto run = [&](auto stream_a, auto stream_b) {
        constexpr bool NTA = decltype(stream_a)::value, NTB = decltype(stream_b)::value;
        const GatherPlace g = gather_place(p, e);
        GatherPlace x[V];
#pragma unroll
        for (int j = 0; j < V; ++j) x[j] = j == 0 ? g : gather_next(p, g, e, (uint32_t)j);
        const bool whole = gather_whole(p, g, count);
        Pack<TA, 1> a[V];
#pragma unroll
        for (int j = 0; j < V; ++j) a[j] = load_pack<TA, 1, NTA>(reinterpret_cast<const unsigned char*>(A), x[j].a * (int64_t)sizeof(TA));
        Pack<TB, V> out;
        unsigned char* Bb = reinterpret_cast<unsigned char*>(B);
        Pack<TB, V> old;
        if (MODE == TTC_EPI_AXPBY) {
            if (whole) {
                old = load_pack<TB, V, NTB>(Bb, g.b * (int64_t)sizeof(TB));
            } else {
#pragma unroll
                for (int j = 0; j < V; ++j) old.v[j] = B[x[j].b];
            }
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
            TB b_old = TB();
            if (MODE == TTC_EPI_AXPBY) b_old = old.v[j];
            out.v[j] = epi(a[j].v[0], b_old);
        }
        if (whole) {
            store_pack<TB, V, NTB>(Bb, g.b * (int64_t)sizeof(TB), out);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) if (j < count) B[x[j].b] = out.v[j];
        }
    };
    if (p.nt_a) { if (p.nt_b) run(std::true_type(), std::true_type()); else run(std::true_type(), std::false_type()); }
    else        { if (p.nt_b) run(std::false_type(), std::true_type()); else run(std::false_type(), std::false_type()); }
}

template <typename TA, typename TB, int MODE, int V>
__global__ __launch_bounds__(kRowsThreads) void gather_kernel(const RowsParams p, const TA* __restrict__ A, TB* __restrict__ B)
{
    const uint32_t block = rows_block(p, blockIdx.x);
    if (block >= p.blocks) return;
    gather_chunk<TA, TB, MODE, V>(p, block, A, B);
}

// The same over a dense B with its arguments packed (SmallArgs), nothing streamed.
template <typename TA, typename TB, int MODE, int V, int N>
__global__ __launch_bounds__(kRowsThreads) void gather_small_kernel(const SmallArgs args_by_value, const TA* __restrict__ A, TB* __restrict__ B)
{
    const SmallArgs& s = *reinterpret_cast<const SmallArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    const RowsParams p = small_unpack<true, N, MODE, IsComplex<TA>::value>(s, V, kRowsThreads);
    gather_chunk<TA, TB, MODE, V>(p, blockIdx.x, A, B);
}

// Launch of either small kernel: the one compiled for `dims` indices (small_dims()).
template <typename TA, typename TB, int MODE, int V, bool GATHER, int N = 2>
inline hipError_t launch_small(const RowsParams& rp, int dims, int64_t grid, const TA* a, TB* b, hipStream_t stream)
{
    if constexpr (N <= kSmallMaxDim) {
        if constexpr (small_fits(GATHER, N, MODE, IsComplex<TA>::value)) {
            if (dims == N) {
                SmallArgs ready = small_pack(rp, GATHER, N, MODE, IsComplex<TA>::value);
                void* args[] = {&ready, &a, &b};
                const void* fn = GATHER ? reinterpret_cast<const void*>(&gather_small_kernel<TA, TB, MODE, 16 / (int)sizeof(TB), N>)
                               : rp.xcd_remap == 1 ? reinterpret_cast<const void*>(&rows_small_kernel<TA, TB, MODE, V, N, true>)
                                                   : reinterpret_cast<const void*>(&rows_small_kernel<TA, TB, MODE, V, N, false>);
                return hipLaunchKernel(fn, dim3((uint32_t)grid), dim3(kRowsThreads), args, 0, stream);
            }
        }
        return launch_small<TA, TB, MODE, V, GATHER, N + 1>(rp, dims, grid, a, b, stream);
    }
    return hipErrorInvalidValue;
}

template <typename TA, typename TB, int MODE>
inline hipError_t launch_gather(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    constexpr int V = 16 / (int)sizeof(TB);
    RowsParams rp = c.rows;
    rp.nt_a = c.kp.nt_a;
    rp.nt_b = c.kp.nt_b;
    rp.xcd_remap = c.kp.xcd_remap;
    if (rp.vec != V || c.threads != kRowsThreads || rp.chunk != kRowsThreads || rp.elements < 1 || rp.elements >= (int64_t(1) << 30) ||
        rp.row < 1 || rp.size_div[0].div != rp.row || (V > 1 && rp.stride_b[0] != 1)) return hipErrorInvalidValue;
    const int64_t chunks = ((rp.elements + V - 1) / V + kRowsThreads - 1) / kRowsThreads;
    if ((int64_t)rp.per_xcd != (rp.per_xcd ? (chunks + 7) / 8 : 0) || (int64_t)rp.blocks != (rp.per_xcd ? 8 * (int64_t)rp.per_xcd : chunks)) return hipErrorInvalidValue;
    const int64_t grid = rows_grid(rp);
    if (!launchable(grid, kRowsThreads)) return hipErrorInvalidValue;
    const TA* a = static_cast<const TA*>(A);
    TB* b = static_cast<TB*>(B);
    const int dims = small_dims(rp, true, MODE, IsComplex<TA>::value, 0, 0);
    if (dims) return launch_small<TA, TB, MODE, V, true>(rp, dims, grid, a, b, stream);
    void* args[] = {&rp, &a, &b};
    return hipLaunchKernel(reinterpret_cast<const void*>(&gather_kernel<TA, TB, MODE, V>), dim3((uint32_t)grid), dim3(kRowsThreads), args, 0, stream);
}

template <typename TA, typename TB, int MODE, int V, int U, bool FLAT>
inline hipError_t launch_rows_unrolled(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    RowsParams rp = c.rows;
    rp.nt_a = c.kp.nt_a;
    rp.nt_b = c.kp.nt_b;
    rp.xcd_remap = c.kp.xcd_remap;
    if (rp.vec != V || rp.unroll != U || c.threads != kRowsThreads || rp.chunk != (uint32_t)(kRowsThreads * U) || rp.row < (uint32_t)V ||
        rp.slots != (FLAT ? rp.row : (rp.row + V - 1) / V) || rp.slot_div.div != rp.slots || rp.flat != (FLAT ? 1 : 0) || rp.vectors < 1 || rp.rows < 1 ||
        (MODE == TTC_EPI_AXPBY && rp.overlap) || (int64_t)rp.blocks != (rp.vectors + rp.chunk - 1) / rp.chunk ||
        (FLAT && (rp.vectors != (rp.elements + V - 1) / V || rp.elements != (int64_t)rp.rows * rp.row))) return hipErrorInvalidValue;
    const int64_t grid = rows_grid(rp);
    if (!launchable(grid, kRowsThreads)) return hipErrorInvalidValue;
    const TA* a = static_cast<const TA*>(A);
    TB* b = static_cast<TB*>(B);
    if constexpr (FLAT && U == 1) {
        rp.per_xcd = rp.xcd_remap == 1 ? (rp.blocks + 7u) / 8u : 0u;
        const int dims = small_dims(rp, false, MODE, IsComplex<TA>::value, 0, 1);
        if (dims) return launch_small<TA, TB, MODE, V, false>(rp, dims, grid, a, b, stream);
    }
    void* args[] = {&rp, &a, &b};
    return hipLaunchKernel(reinterpret_cast<const void*>(&rows_kernel<TA, TB, MODE, V, U, FLAT>), dim3((uint32_t)grid), dim3(kRowsThreads), args, 0, stream);
}

template <typename TA, typename TB, int MODE, int V>
inline hipError_t launch_rows_one(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    switch (c.rows.unroll) {
    case 1: return launch_rows_unrolled<TA, TB, MODE, V, 1, false>(c, A, B, stream);
    case 2: return launch_rows_unrolled<TA, TB, MODE, V, 2, false>(c, A, B, stream);
    case 4: return launch_rows_unrolled<TA, TB, MODE, V, 4, false>(c, A, B, stream);
    case 8: return launch_rows_unrolled<TA, TB, MODE, V, 8, false>(c, A, B, stream);
    default: return hipErrorInvalidValue;
    }
}

template <typename TA, typename TB, int MODE, int V>
inline hipError_t launch_rows_flat(const Candidate& c, const void* A, void* B, hipStream_t stream)
{
    switch (c.rows.unroll) {
    case 1: return launch_rows_unrolled<TA, TB, MODE, V, 1, true>(c, A, B, stream);
    case 2: return launch_rows_unrolled<TA, TB, MODE, V, 2, true>(c, A, B, stream);
    case 4: return launch_rows_unrolled<TA, TB, MODE, V, 4, true>(c, A, B, stream);
    case 8: return launch_rows_unrolled<TA, TB, MODE, V, 8, true>(c, A, B, stream);
    default: return hipErrorInvalidValue;
    }
}

// VMAXA / VMAXB: elements of each type in 16 bytes
template <typename TA, typename TB, int MODE, int VMAXA, int VMAXB>
inline hipError_t launch_vec(const Candidate& c, const void* A, void* B, hipStream_t s)
{
    constexpr int VD = VMAXA < VMAXB ? VMAXA : VMAXB;      // direct and row kernel: one width for both sides
    if (c.kernel_class == TTC_KERNEL_MICRO) return launch_micro<TA, TB, MODE>(c, A, B, s);
    if (c.kernel_class == kKernelLines) return launch_lines<TA, TB, MODE>(c, A, B, s);
    if (c.kernel_class == kKernelGather) return launch_gather<TA, TB, MODE>(c, A, B, s);
    if (c.kernel_class == kKernelBlock) return launch_block<TA, TB, MODE>(c, A, B, s);
    if (c.kernel_class == TTC_KERNEL_ROWS) {
        const int v = c.rows.vec;
        if (c.rows.flat) return v == VD ? launch_rows_flat<TA, TB, MODE, VD>(c, A, B, s) : hipErrorInvalidValue;
        if (v == 1) return launch_rows_one<TA, TB, MODE, 1>(c, A, B, s);
        if (v == 2 && VD >= 2) return launch_rows_one<TA, TB, MODE, (VD >= 2 ? 2 : 1)>(c, A, B, s);
        if (v == 4 && VD >= 4) return launch_rows_one<TA, TB, MODE, (VD >= 4 ? 4 : 1)>(c, A, B, s);
        return hipErrorInvalidValue;
    }
    // the candidate's parameter block is launch-ready for a device of 256 compute units (every MI355X); it is
    // copied and re-gridded only for another device, or for the set-up measurement (TTC_DEBUG_STOP in the
    // environment: every workgroup returns after its set-up)
    static const bool stop = std::getenv("TTC_DEBUG_STOP") != nullptr;
    const uint32_t grid = launch_grid(c, device_cus());
    KernelParams other;
    const KernelParams* ready = &c.kp;
    if (grid != c.kp.grid || stop) {
        other = c.kp;
        set_grid(&other, grid);
        other.debug_stop = stop ? 1 : 0;
        ready = &other;
    }
    const KernelParams& kp = *ready;
    const int va = kp.a.vec, vb = kp.b.vec;
    if (c.kernel_class == TTC_KERNEL_DIRECT) {
        if (va == 1) return launch_one<TA, TB, MODE, 1, 1, true>(kp, A, B, grid, c.threads, c.lds_bytes, s);
        if (va == 2 && VD >= 2) return launch_one<TA, TB, MODE, (VD >= 2 ? 2 : 1), (VD >= 2 ? 2 : 1), true>(kp, A, B, grid, c.threads, c.lds_bytes, s);
        if (va == 4 && VD >= 4) return launch_one<TA, TB, MODE, (VD >= 4 ? 4 : 1), (VD >= 4 ? 4 : 1), true>(kp, A, B, grid, c.threads, c.lds_bytes, s);
        return hipErrorInvalidValue;
    }
#define TTC_CASE(VA_, VB_)                                                                                   \
    if (va == VA_ && vb == VB_ && VA_ <= VMAXA && VB_ <= VMAXB)                                              \
        return launch_one<TA, TB, MODE, (VA_ <= VMAXA ? VA_ : 1), (VB_ <= VMAXB ? VB_ : 1), false>(          \
            kp, A, B, grid, c.threads, c.lds_bytes, s);
    TTC_CASE(1, 1) TTC_CASE(1, 2) TTC_CASE(2, 1) TTC_CASE(2, 2)
    TTC_CASE(1, 4) TTC_CASE(2, 4) TTC_CASE(4, 1) TTC_CASE(4, 2) TTC_CASE(4, 4)
#undef TTC_CASE
    return hipErrorInvalidValue;
}

template <typename TA, typename TB, int VMAXA, int VMAXB>
inline hipError_t launch_mode(const Problem& P, const Candidate& c, const void* A, void* B, hipStream_t s)
{
    switch (P.epilogue) {
    case TTC_EPI_COPY:  return launch_vec<TA, TB, TTC_EPI_COPY, VMAXA, VMAXB>(c, A, B, s);
    case TTC_EPI_SCALE: return launch_vec<TA, TB, TTC_EPI_SCALE, VMAXA, VMAXB>(c, A, B, s);
    default:            return launch_vec<TA, TB, TTC_EPI_AXPBY, VMAXA, VMAXB>(c, A, B, s);
    }
}

}  // namespace ttc
