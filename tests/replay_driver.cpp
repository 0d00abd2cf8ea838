// Which workgroups of the row kernel the host replay (ttc_debug_emulate_map) looks at (built and run by tests/test_rows_kernel.py; plain
// C++, no GPU): the library's index code with a record of where every replayed workgroup starts.  A launch over ranges has up
// to seven workgroups behind the last chunk; the packed kernel runs them like any other, so the replay has to check them too.
#include <cstdio>
#include <vector>

#define flat_access library_flat_access
#include "ttc_walk.h"
#undef flat_access

namespace ttc {
static std::vector<int64_t> g_starts;
inline FlatAccess flat_access(const RowsParams& p, int64_t base, uint32_t row0, uint32_t col0, uint32_t k)
{
    if (g_starts.empty() || g_starts.back() != base) g_starts.push_back(base);
    return library_flat_access(p, base, row0, col0, k);
}
}

#include "ttc_plan.cpp"

// dtype, extents, beta: row problems whose chunk counts are no multiple of eight
struct Case { int dtype; int64_t sizes[3]; double beta; };
static const Case kCases[] = {{TTC_F32, {27, 40, 33}, 0.0}, {TTC_F32, {27, 40, 33}, 1.0}, {TTC_F64, {64, 9, 17}, 0.0}, {TTC_C64, {33, 7, 29}, 0.0}, {TTC_F32_F64, {13, 51, 20}, 1.0}};

int main()
{
    int failures = 0;
    for (const Case& c : kCases) {
        const int perm[3] = {0, 2, 1};
        float alpha_f[2] = {1.0f, 0.0f}, beta_f[2] = {(float)c.beta, 0.0f};
        double alpha_d[2] = {1.0, 0.0}, beta_d[2] = {c.beta, 0.0};
        const bool single = c.dtype == TTC_F32 || c.dtype == TTC_C64;
        ttc_plan_t plan = ttc_plan_create(c.dtype, 3, c.sizes, perm, single ? (void*)alpha_f : (void*)alpha_d, single ? (void*)beta_f : (void*)beta_d);
        std::vector<int64_t> map((size_t)(c.sizes[0] * c.sizes[1] * c.sizes[2]));
        int ran = 0;
        for (int k = 0; plan && k < ttc_plan_candidate_count(plan); ++k) {
            ttc_plan_select_candidate(plan, k);
            const ttc::Candidate& C = plan->cands[(size_t)k];
            if (C.kernel_class != TTC_KERNEL_ROWS || !C.rows.flat || C.rows.unroll != 1) continue;
            for (int mapping = 0; mapping <= 1; ++mapping) {
                ttc_plan_set_tile_mapping(plan, mapping);
                ttc::g_starts.clear();
                const int status = ttc_debug_emulate_map(plan, map.data());
                const size_t launched = mapping ? (C.rows.blocks + 7u) / 8u * 8u : C.rows.blocks;
                if (status != TTC_OK || C.rows.blocks % 8 == 0 || ttc::g_starts.size() != launched) {
                    ++failures;
                    std::printf("FAIL type %d, %lld x %lld x %lld, mapping %d: status %d, %zu of %zu workgroups replayed (%u chunks)\n", c.dtype, (long long)c.sizes[0],
                                (long long)c.sizes[1], (long long)c.sizes[2], mapping, status, ttc::g_starts.size(), launched, C.rows.blocks);
                }
                ++ran;
            }
        }
        if (ran == 0) { ++failures; std::printf("FAIL no row candidate for type %d\n", c.dtype); }
        ttc_plan_destroy(plan);
    }
    if (failures == 0) std::printf("replay driver ok\n");
    return failures != 0;
}
