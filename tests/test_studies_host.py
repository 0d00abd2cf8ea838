"""Host-side checks of the study helpers (no GPU): the benchmark's permutations and shapes, the rule by which the
search fills its places (mirrored from the library), and the feature functions the ranking models are fitted with."""
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_1603_02297_amd as ttc
from paper_1603_02297_amd import studies as st
from paper_1603_02297_amd import workloads as wl


def test_benchmark_has_57_cases_without_mergeable_indices():
    perms = st.benchmark_permutations()
    assert len(perms) == 19 and len(perms) * 3 == 57
    for perm, cls in perms:
        assert sorted(perm) == list(range(len(perm)))
        assert not st.mergeable(perm)
        assert cls in ("stride-1", "inverse", "general")
        assert (perm[0] == 0) == (cls == "stride-1")
    for n in range(2, 7):
        for cfg in (0, 1, 2):
            sizes = st.shape_for(n, cfg)
            assert len(sizes) == n and 150e6 < 4 * np.prod(sizes) < 260e6


def test_benchmark_takes_problems_of_one_type_only():
    """bench.py sizes both tensors, its copies and its traffic by one element size: two precisions are refused before
    anything is allocated (B of a widening problem would be half as large as what is written to it)."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "bench.py", "--problem", "f32f64:8x8:10:1:0"], cwd=root, capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "one type" in r.stderr, r.stderr
    for dtype in (wl.F32_F64, wl.F64_F32, wl.C64_C128, wl.C128_C64, wl.C64, wl.F64):
        a, b = wl.case_inputs(wl.Case(9, dtype, (4, 3), (1, 0), 1.0, 0.0))
        assert a.nbytes == 12 * wl.ELEM_BYTES[dtype] and b.nbytes == 12 * wl.ELEM_BYTES_B[dtype]


def test_search_set_keeps_places_for_both_micro_tile_families():
    fam = [0] * 300
    for i in (5, 150, 210):
        fam[i] = 1
    for i in (220, 230, 280):
        fam[i] = 2
    assert st.search_set(fam, 1) == [0]
    assert st.search_set(fam, 10) == [0, 1, 2, 3, 4, 5, 6, 150, 220, 230]      # two places per family, candidate 5 was in anyway
    chosen = st.search_set(fam, 100)
    assert len(set(chosen)) == 100 and {150, 210, 220, 230, 280} <= set(chosen)
    assert st.search_set(fam, 400) == list(range(300))
    # where few others are left to give way, the line kernel's candidates keep their places
    fam = [3, 0, 3, 1] + [1] * 30 + [2] * 100
    assert st.search_set(fam, 20) == [0, 37] + list(range(2, 20))


def test_every_kernel_has_a_family_of_its_own():
    """The line, the gather and the block kernel report another kernel's class: the studies, the benchmark and the smoke run
    tell them apart by it, and nothing but box kernels enters the box model's fit and its ablation."""
    def families(dtype, sizes, perm):
        p = ttc.ttc_plan_create(dtype, len(sizes), sizes, perm, 1.0, 0.0)
        seen = {}
        for k in range(ttc.ttc_plan_candidate_count(p)):
            ttc.ttc_plan_select_candidate(p, k)
            info = ttc.ttc_plan_get_info(p)
            seen.setdefault(ttc.kernel_family(info), []).append(info)
        ttc.ttc_plan_destroy(p)
        return seen

    moved, fixed = families(ttc.TTC_F32, (70, 33, 45), (2, 0, 1)), families(ttc.TTC_F32, (96, 20, 31), (0, 2, 1))
    assert set(moved) == {"lds", "line", "gather", "micro", "block"} and set(fixed) == {"direct", "lds", "rows", "gather"}
    assert len(moved["gather"]) == len(fixed["gather"]) == 1             # one candidate, whatever the problem
    assert set(moved) | set(fixed) == set(ttc.KERNEL_FAMILIES)
    assert {i["unroll"] for i in moved["block"]} <= {2, 4, 8} and {i["merged"] for i in moved["micro"]} <= {0, 1, 2, 3}
    assert {st.micro_family(i) for i in moved["block"]} == {3}           # no micro-tile candidate of either kind, and none that gives way to one
    assert {i["unroll"] for i in moved["line"]} <= {2, 4, 8} and {i["unroll"] for i in fixed["rows"]} <= {1, 2, 4, 8}
    assert all(i["wg_per_cu"] == 0 for f in ("line", "gather", "micro", "block") for i in moved[f])
    assert all(i["wg_per_cu"] > 0 for f in st.BOX for i in moved.get(f, []) + fixed.get(f, []))
    rows = [(i, 1.0 if f in st.BOX else 0.5) for f in moved for i in moved[f]]
    rows.sort(key=lambda r: r[0]["candidate_index"])
    abl = st.ablations(rows)
    assert abl["kernel family"] == 2.0 and abl["LDS buffering"] == abl["launch shape"] == 1.0
    assert st.ablations([r for r in rows if ttc.kernel_family(r[0]) in ("lds", "line")])["launch shape"] == 1.0


def test_micro_tile_features_mirror_the_library_model():
    """micro_cost() of the library = exp(offset + sum of the fitted weights times these features)."""
    weights = {"A<128": 0.05, "B<128": 0.012, "A>1K": -0.01, "B>1K": -0.03, "pad": 0.11, "unA*A<512": 0.028,
               "unB*B<512": 0.072, "t128": 0.04, "t64": 0.068, "ordNotB": 0.054, "blocks": 0.009, "lds": 0.114,
               "mergeA": 0.006, "mergeB": 0.011, "idle": 0.27}
    p = ttc.ttc_plan_create(ttc.TTC_F32, 5, (512, 20, 9, 22, 768), (4, 3, 2, 1, 0), 1.0, 0.0)   # large enough that no small-problem term applies
    seen = 0
    for k in range(ttc.ttc_plan_candidate_count(p)):
        ttc.ttc_plan_select_candidate(p, k)
        info = ttc.ttc_plan_get_info(p)
        if ttc.kernel_family(info) != "micro":
            continue
        seen += 1
        assert st.micro_family(info) == (2 if info["merged"] else 1)
        f = st.fit_micro_features(info)
        model = np.exp(-0.22 + sum(weights[q] * v for q, v in f.items() if q in weights))
        assert model == pytest.approx(info["heuristic_cost"], rel=1e-12), (k, info["tile"], f)
    assert seen >= 20
    ttc.ttc_plan_destroy(p)
