"""The row kernel over a dense B, whose vectors run across the ends of rows, and over a padded one, and the gather kernel
(reported as the same class), which takes any permutation: every candidate and
every way of dealing its chunks to the XCDs against the oracle, replayed on the host and run on the GPU.  Sizes: rows
of one vector, one element more, odd ones; a tensor that is no multiple of the vector; chunks that do not fill a round."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_1603_02297_amd as ttc
from paper_1603_02297_amd import workloads as wl

# sizes, perm, lda, ldb
SHAPES = [
    ((4, 3, 5), (0, 2, 1), None, None),
    ((5, 3, 7), (0, 2, 1), None, None),
    ((7, 31, 29), (0, 2, 1), None, None),
    ((45, 9, 37), (0, 2, 1), (47, 9, 37), None),          # A padded, B dense
    ((45, 9, 37), (0, 2, 1), None, (48, 37, 9)),          # B padded: counted row by row
    ((13, 5, 6, 4), (0, 3, 1, 2), None, None),
    ((1001,), (0,), (1003,), None),                       # one row
    # the stride-1 index moves: the gather kernel alone
    ((3, 50), (1, 0), None, None),                        # B's runs longer than a vector, shorter, of two elements
    ((50, 3), (1, 0), None, None),
    ((2, 7, 2, 9), (2, 0, 3, 1), None, None),
    ((5, 4, 3, 6), (3, 1, 0, 2), (6, 4, 5, 6), (7, 4, 5, 3)),
    ((1, 8, 6, 10), (1, 2, 0, 3), (2, 9, 8, 10), (9, 7, 3, 14)),     # A has no stride-1 index
    # nor has B: an index of extent 1 is its first, inside a larger one, so its elements lie apart
    ((1, 64, 6, 10), (0, 2, 1, 3), None, (2, 6, 64, 10)),
    ((64, 1, 60), (1, 2, 0), None, (3, 60, 64)),
    ((1, 1000), (0, 1), None, (2, 1000)),
]
DTYPES = [wl.F32, wl.F64, wl.C128, wl.F32_F64, wl.F64_F32]


# B's elements lie apart: an index of extent 1 is its first, inside a larger one
NO_UNIT_STRIDE_IN_B = [
    ((1, 64, 60, 10), (0, 2, 1, 3), None, (2, 60, 64, 10)),
    ((64, 1, 60), (1, 2, 0), None, (3, 60, 64)),
    ((1, 1000), (0, 1), None, (2, 1000)),
    ((300, 1, 200), (1, 2, 0), None, (2, 200, 300)),
]


def rows_candidates(plan):
    for k in range(ttc.ttc_plan_candidate_count(plan)):
        ttc.ttc_plan_select_candidate(plan, k)
        info = ttc.ttc_plan_get_info(plan)
        if info["kernel_class"] == ttc.TTC_KERNEL_ROWS:
            for mapping in (0, 1, 2, 5):
                ttc.ttc_plan_set_tile_mapping(plan, mapping)
                yield k, mapping, info


@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_walks_of_every_row_candidate(dtype):
    seen = 0
    for sizes, perm, lda, ldb in SHAPES:
        for beta in (0.0, 1.0):
            p = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, 1.0, beta)
            want = [-1] * ttc.ttc_plan_get_info(p)["span_b"]
            for off_a, off_b in oracle.element_pairs(sizes, perm, lda, ldb):
                want[off_b] = off_a
            for k, mapping, info in rows_candidates(p):
                assert list(ttc.ttc_debug_emulate_map(p)) == want, (sizes, perm, k, mapping, info)
                seen += 1
            ttc.ttc_plan_destroy(p)
    assert seen >= 100


@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_plans_as_created_where_b_has_no_unit_stride(dtype):
    """Elements of B that lie apart are never written as one vector; only 16-byte elements may take the gather kernel."""
    for sizes, perm, lda, ldb in NO_UNIT_STRIDE_IN_B:
        for beta in (0.0, 1.0):
            p = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, 1.0, beta)
            want = [-1] * ttc.ttc_plan_get_info(p)["span_b"]
            for off_a, off_b in oracle.element_pairs(sizes, perm, lda, ldb):
                want[off_b] = off_a
            assert list(ttc.ttc_debug_emulate_map(p)) == want, (sizes, perm, ttc.ttc_plan_get_info(p))
            for k in range(ttc.ttc_plan_candidate_count(p)):
                ttc.ttc_plan_select_candidate(p, k)
                info = ttc.ttc_plan_get_info(p)
                assert info["kernel_class"] != ttc.TTC_KERNEL_ROWS or wl.ELEM_BYTES_B[dtype] == 16, (sizes, perm, k)
            ttc.ttc_plan_destroy(p)


# sizes, perm, type, whether neighbouring workgroups of the gather kernel share lines of A: several hundred to 2200 chunks of 256
# vectors, the numbers of chunks no multiples of eight
GATHER_CHUNKS = [
    ((301, 203), (1, 0), wl.C128, True),
    ((301, 509), (1, 0), wl.F32, True),
    ((1500, 1500), (1, 0), wl.F32, True),
    ((301, 37, 21), (2, 1, 0), wl.F64, True),
    ((581, 783), (1, 0), wl.C128, False),
    ((700, 900), (1, 0), wl.C128, False),
]


def gather_candidate(plan):
    for k in range(ttc.ttc_plan_candidate_count(plan)):
        ttc.ttc_plan_select_candidate(plan, k)
        if ttc.kernel_family(ttc.ttc_plan_get_info(plan)) == "gather":
            return ttc.ttc_plan_get_info(plan)
    raise AssertionError("no gather candidate")


@pytest.mark.parametrize("sizes,perm,dtype,shared", GATHER_CHUNKS)
def test_gather_chunks_are_dealt_one_way(sizes, perm, dtype, shared):
    """Where neighbours share lines the chunks are numbered range by range and dealt round robin, whatever their number: a
    second dealing on top would give every XCD pieces of all ranges.  Else by the number of chunks, as tiles are.
    Every mapping covers B."""
    p = ttc.ttc_plan_create(dtype, len(sizes), sizes, perm, 1.0, 0.0)
    info = gather_candidate(p)
    chunks = -(-int(np.prod(sizes)) * wl.ELEM_BYTES_B[dtype] // 4096)
    assert chunks >= 64 and chunks % 8 != 0
    assert info["num_tiles"] == (-(-chunks // 8) * 8 if shared else chunks)
    default = 0 if shared or chunks < 2048 else 5
    assert info["xcd_remap"] == default
    n = len(sizes)
    stride = np.cumprod([1] + list(sizes[:-1]))                       # B in its own order: where each element comes from
    want = (np.indices([sizes[k] for k in perm][::-1]) * np.array([stride[k] for k in perm][::-1]).reshape((n,) + (1,) * n)).sum(0).ravel()
    for mode in (-1, 0, 1, 5, -1):
        ttc.ttc_plan_set_tile_mapping(p, mode)
        assert ttc.ttc_plan_get_info(p)["xcd_remap"] == (default if mode < 0 else mode)
        assert np.array_equal(np.array(ttc.ttc_debug_emulate_map(p)), want), mode
    ttc.ttc_plan_destroy(p)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_row_kernel_against_the_oracle(dtype):
    """Every epilogue; what lies behind B stays as it was.  Fixed evaluation order on both sides: bit-equal but for the
    ulp the library allows."""
    import torch
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    prod = lambda v: int(np.prod(v))  # noqa: E731
    ran = 0
    cplx = wl.COMPONENTS[dtype] == 2
    for shape, (sizes, perm, lda, ldb) in enumerate(SHAPES):
        na, nb = prod(lda or sizes), prod(ldb or sizes)
        A = wl.uniform_tensor(dtype, na, 7200 + shape, "a")
        B0 = wl.uniform_tensor(dtype, nb, 7300 + shape, "b")
        comp, room = wl.COMPONENTS[dtype], 16
        dA = torch.from_numpy(A).to(dev)
        for alpha, beta in ((1.0, 0.0), (0.5 + 0.5j if cplx else 1.5, 0.0), (0.75, 1.0 + 0.5j if cplx else -1.25)):
            want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4, lda=lda, ldb=ldb)
            plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, alpha, beta)
            try:
                for k, mapping, info in rows_candidates(plan):
                    buf = torch.full((nb * comp + 2 * room,), 77.0, dtype=torch.from_numpy(B0).dtype, device=dev)
                    buf[room:room + nb * comp] = torch.from_numpy(B0).to(dev)
                    ttc.ttc_execute(plan, dA.data_ptr(), buf.data_ptr() + room * buf.element_size(), stream)
                    torch.cuda.synchronize()
                    got = buf.cpu().numpy()
                    assert (got[:room] == 77).all() and (got[room + nb * comp:] == 77).all(), (sizes, perm, k, info)
                    got = got[room:room + nb * comp]
                    if complex(alpha) == 1 and complex(beta) == 0:
                        assert np.array_equal(got, want), (sizes, perm, k, mapping, info)
                    else:
                        assert np.abs(got - want).max() <= np.spacing(np.abs(want).max()), (sizes, perm, alpha, beta, k, mapping, info)
                    ran += 1
            finally:
                ttc.ttc_plan_destroy(plan)
    assert ran >= 100


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_plans_as_created_where_b_has_no_unit_stride_on_the_gpu(dtype):
    """The plan as created writes the elements of the sub-tensor and nothing between them."""
    import torch
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    for shape, (sizes, perm, lda, ldb) in enumerate(NO_UNIT_STRIDE_IN_B):
        A = wl.uniform_tensor(dtype, int(np.prod(sizes)), 7400 + shape, "a")
        B0 = wl.uniform_tensor(dtype, int(np.prod(ldb)), 7500 + shape, "b")
        dA = torch.from_numpy(A).to(dev)
        for alpha, beta in ((1.0, 0.0), (0.75, -1.25)):
            want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4, lda=lda, ldb=ldb)
            plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, alpha, beta)
            dB = torch.from_numpy(B0).to(dev)
            ttc.ttc_execute(plan, dA.data_ptr(), dB.data_ptr(), stream)
            got = dB.cpu().numpy()
            ttc.ttc_plan_destroy(plan)
            allowed = 0.0 if beta == 0 else np.spacing(np.abs(want).max())      # the one ulp the library allows an update
            assert np.abs(got - want).max() <= allowed, (sizes, perm, ldb, beta)


def execute_and_compare(plan, dtype, dA, B0, want, moved_only, setup, tag):
    """One ttc_execute on a B that starts `first` elements behind an aligned address, `setup` = (streaming hint, first): what
    lies around B stays as it was, B is the oracle's: bit-equal where elements are only moved, else within the one ulp the
    library allows (same evaluation order)."""
    import torch
    comp, room = wl.COMPONENTS[dtype], 64
    nt, first = setup
    ttc.ttc_plan_set_streaming(plan, nt, nt)
    buf = torch.full((B0.size + 2 * room,), 77.0, dtype=torch.from_numpy(B0).dtype, device=dA.device)
    at = room + int(first * comp)
    buf[at:at + B0.size] = torch.from_numpy(B0).to(dA.device)
    ttc.ttc_execute(plan, dA.data_ptr(), buf.data_ptr() + at * buf.element_size(), torch.cuda.current_stream().cuda_stream)
    got = buf.cpu().numpy()
    assert (got[:at] == 77).all() and (got[at + B0.size:] == 77).all(), tag
    got = got[at:at + B0.size]
    if moved_only:
        assert np.array_equal(got, want), tag
    else:
        assert np.abs(got - want).max() <= np.spacing(np.abs(want).max()), tag


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_streaming_and_odd_addresses_against_the_oracle(dtype):
    """Every row and gather candidate with both settings of the streaming hints, and on a B aligned to its element only."""
    import torch
    dev = torch.device("cuda:0")
    cplx, ran = wl.COMPONENTS[dtype] == 2, 0
    setups = ((0, 1), (1, 3), (1, 0)) + (((0, 0.5),) if dtype == wl.C128 else ())          # 8 bytes are enough for complex128
    for shape, (sizes, perm, lda, ldb) in enumerate(SHAPES):
        A = wl.uniform_tensor(dtype, int(np.prod(lda or sizes)), 7600 + shape, "a")
        B0 = wl.uniform_tensor(dtype, int(np.prod(ldb or sizes)), 7700 + shape, "b")
        dA = torch.from_numpy(A).to(dev)
        for alpha, beta in ((1.0, 0.0), (0.75, 1.0 + 0.5j if cplx else -1.25)):
            want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4, lda=lda, ldb=ldb)
            plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, alpha, beta)
            try:
                for k in range(ttc.ttc_plan_candidate_count(plan)):
                    ttc.ttc_plan_select_candidate(plan, k)
                    if ttc.kernel_family(ttc.ttc_plan_get_info(plan)) not in ("rows", "gather"):
                        continue
                    for setup in setups:
                        execute_and_compare(plan, dtype, dA, B0, want, beta == 0, setup, (sizes, perm, beta, k, setup))
                        ran += 1
            finally:
                ttc.ttc_plan_destroy(plan)
    assert ran >= 100


@pytest.mark.gpu
@pytest.mark.parametrize("sizes,perm,dtype,shared", GATHER_CHUNKS)
def test_many_gather_chunks_against_the_oracle(sizes, perm, dtype, shared):
    """Hundreds of chunks, their numbers no multiples of eight: every dealing of them, with and without an update of B."""
    import torch
    dev = torch.device("cuda:0")
    A = wl.uniform_tensor(dtype, int(np.prod(sizes)), 7800, "a")
    B0 = wl.uniform_tensor(dtype, int(np.prod(sizes)), 7801, "b")
    dA = torch.from_numpy(A).to(dev)
    for alpha, beta in ((1.0, 0.0), (0.75, -1.25)):
        want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4)
        plan = ttc.ttc_plan_create(dtype, len(sizes), sizes, perm, alpha, beta)
        gather_candidate(plan)
        for mapping in (-1, 0, 1, 5):
            ttc.ttc_plan_set_tile_mapping(plan, mapping)
            for setup in ((0, 1), (1, 0)):
                execute_and_compare(plan, dtype, dA, B0, want, beta == 0, setup, (sizes, perm, beta, mapping, setup))
        ttc.ttc_plan_destroy(plan)


# sizes, perm: two to six indices (what is packed ends between four and six, by the scalars), rows of one vector, one row
SMALL_SHAPES = [((40, 30), (1, 0)), ((9, 7, 5), (2, 0, 1)), ((5, 4, 3, 6), (3, 1, 0, 2)), ((3, 4, 2, 5, 6), (4, 2, 0, 3, 1)), ((2, 3, 2, 5, 4, 3), (5, 3, 1, 0, 4, 2)),
                ((4, 5, 3), (0, 2, 1)), ((16, 4, 3, 5), (0, 3, 2, 1)), ((6, 3, 4, 2, 5), (0, 4, 2, 1, 3)), ((513,), (0,))]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", range(8), ids=[wl.DTYPE_NAME[d] for d in range(8)])
def test_small_problems_with_packed_parameters(dtype):
    """Every number of indices and every epilogue through the row and the gather kernel of small problems, next to those whose
    parameters are not packed: as created, with the hints and the dealing of tiles that only the unpacked form has."""
    import torch
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    cplx = wl.COMPONENTS[dtype] == 2
    ran = 0
    for shape, (sizes, perm) in enumerate(SMALL_SHAPES):
        n = int(np.prod(sizes))
        A = wl.uniform_tensor(dtype, n, 9000 + shape, "a")
        B0 = wl.uniform_tensor(dtype, n, 9100 + shape, "b")
        dA = torch.from_numpy(A).to(dev)
        for alpha, beta in ((1.0, 0.0), (0.5 + 0.25j if cplx else 1.5, 0.0), (0.5 - 0.25j if cplx else 0.75, 1.0 + 0.5j if cplx else -1.25)):
            want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4)
            plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, None, None, alpha, beta)
            try:
                for k in range(ttc.ttc_plan_candidate_count(plan)):
                    ttc.ttc_plan_select_candidate(plan, k)
                    if ttc.kernel_family(ttc.ttc_plan_get_info(plan)) not in ("rows", "gather"):
                        continue
                    for packed in (True, False):
                        if not packed:
                            ttc.ttc_plan_set_streaming(plan, 1, 1)
                            ttc.ttc_plan_set_tile_mapping(plan, 2)
                        dB = torch.from_numpy(B0).to(dev)
                        ttc.ttc_execute(plan, dA.data_ptr(), dB.data_ptr(), stream)
                        got = dB.cpu().numpy()
                        allowed = 0.0 if complex(alpha) == 1 and complex(beta) == 0 else np.spacing(np.abs(want).max())
                        assert np.abs(got - want).max() <= allowed, (sizes, perm, alpha, beta, k, packed)
                        ran += 1
            finally:
                ttc.ttc_plan_destroy(plan)
    assert ran >= 50


# (type, extents, permutation, beta, mapping that the rule gives a row plan, leading dimensions of A): either side of the lines of the rule
ROWS_DEALT_BY_DEFAULT = [
    (wl.F32, (27, 211, 199), (0, 2, 1), 0.0, 1, None), (wl.F32, (27, 199, 173), (0, 2, 1), 0.0, 0, None),          # 9.1 and 7.4 MB of traffic
    (wl.F32, (13, 91, 3001), (0, 2, 1), 0.0, 1, None), (wl.F32, (13, 21, 12001), (0, 2, 1), 0.0, 0, None),         # neighbours 156 and 624 KB apart, 28 and 26 MB
    (wl.F32, (64, 300, 299), (0, 2, 1), 0.0, 1, None),                                                       # whole lines: ranges, packed
    (wl.F32, (13, 331, 307), (0, 2, 1), 1.0, 1, None), (wl.F32, (31, 331, 307), (0, 2, 1), 1.0, 1, None),          # updates, 15.9 and 37.8 MB
    (wl.F32, (37, 231, 107), (0, 2, 1), 1.0, 0, None), (wl.F32, (64, 300, 299), (0, 2, 1), 1.0, 0, None),          # rows beyond 128 bytes below 16 MB; whole lines
    (wl.C128, (5, 7, 5, 9, 11, 61), (0, 2, 1, 5, 4, 3), 1.0, 1, None), (wl.C128, (35, 5, 9, 11, 7, 13), (0, 5, 2, 4, 3, 1), 0.0, 5, None),     # six indices: not packed
    # rows of a larger A: each on lines of its own, or starting inside lines that they share, whatever their own length is; the third and the sixth lie
    # more than a line apart
    (wl.F32, (27, 800, 331), (0, 2, 1), 1.0, 0, (32, 800, 331)), (wl.F32, (32, 800, 331), (0, 2, 1), 1.0, 1, (33, 800, 331)), (wl.F32, (27, 800, 331), (0, 2, 1), 1.0, 0, (60, 800, 331)),
    (wl.F32, (64, 560, 558), (0, 2, 1), 0.0, 1, (65, 560, 558)), (wl.F32, (63, 560, 558), (0, 2, 1), 0.0, 5, (64, 560, 558)), (wl.F32, (63, 560, 558), (0, 2, 1), 0.0, 5, (97, 560, 558)),
    # not packed: rows that share lines and are not whole lines themselves, rows of whole lines, rows on lines of their own
    (wl.C128, (7, 7, 9, 11, 13, 15), (0, 2, 1, 5, 4, 3), 1.0, 1, (9, 7, 9, 11, 13, 15)), (wl.C128, (8, 7, 9, 11, 13, 15), (0, 2, 1, 5, 4, 3), 1.0, 5, (9, 7, 9, 11, 13, 15)),
    (wl.C128, (7, 7, 9, 11, 13, 15), (0, 2, 1, 5, 4, 3), 1.0, 5, (8, 7, 9, 11, 13, 15)),
    (wl.F32, (33, 800, 331), (0, 2, 1), 1.0, 1, (33, 801, 331)),                                       # dense rows, padded behind the second index
]


@pytest.mark.parametrize("dtype,sizes,perm,beta,mapping,lda", ROWS_DEALT_BY_DEFAULT)
def test_rows_that_share_lines_are_dealt_in_ranges(dtype, sizes, perm, beta, mapping, lda):
    p = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, None, 1.5, beta)
    for k in range(ttc.ttc_plan_candidate_count(p)):
        ttc.ttc_plan_select_candidate(p, k)
        info = ttc.ttc_plan_get_info(p)
        if ttc.kernel_family(info) == "rows" and info["unroll"] == 1 and info["partial_a"] == 0 and info["vec_a"] == 16 // max(wl.ELEM_BYTES[dtype], wl.ELEM_BYTES_B[dtype]):
            break
    else:
        raise AssertionError("no row candidate of whole vectors")
    assert info["xcd_remap"] == mapping
    ttc.ttc_plan_set_tile_mapping(p, 2)
    ttc.ttc_plan_set_tile_mapping(p, -1)
    assert ttc.ttc_plan_get_info(p)["xcd_remap"] == mapping
    ttc.ttc_plan_destroy(p)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,sizes,perm,beta,mapping,lda", [c for c in ROWS_DEALT_BY_DEFAULT if c[4] == 1])
def test_row_ranges_against_the_oracle(dtype, sizes, perm, beta, mapping, lda):
    """Every row candidate with one range of chunks per XCD, the plan as created first; chunk counts that do not divide by eight, B with a last vector
    that is not whole."""
    import torch
    n, stream, cplx = int(np.prod(sizes)), torch.cuda.current_stream().cuda_stream, wl.COMPONENTS[dtype] == 2
    A, B0 = wl.uniform_tensor(dtype, int(np.prod(lda or sizes)), 7400, "a"), wl.uniform_tensor(dtype, n, 7401, "b")
    alpha = 0.5 + 0.5j if cplx else 1.5
    want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 8, lda=lda)
    dA, dB0 = torch.from_numpy(A).cuda(), torch.from_numpy(B0).cuda()
    plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, None, alpha, beta)
    ran = 0
    for k in range(ttc.ttc_plan_candidate_count(plan)):
        ttc.ttc_plan_select_candidate(plan, k)
        if k and ttc.kernel_family(ttc.ttc_plan_get_info(plan)) != "rows":
            continue
        if k:
            ttc.ttc_plan_set_tile_mapping(plan, 1)
        dB = dB0.clone()
        ttc.ttc_execute(plan, dA.data_ptr(), dB.data_ptr(), stream)
        assert np.abs(dB.cpu().numpy() - want).max() <= np.spacing(np.abs(want).max()), (k, ttc.ttc_plan_get_info(plan))     # one ulp
        ran += 1
    assert ran >= 2
    ttc.ttc_plan_destroy(plan)


def test_the_replay_runs_every_workgroup_of_a_packed_launch(tmp_path):
    """Over ranges a launch has up to seven workgroups behind the last chunk; the packed kernel loads there as everywhere, so the host replay
    has to follow them (replay_driver.cpp records where each replayed workgroup starts)."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    csrc, exe = os.path.join(root, "paper_1603_02297_amd", "csrc"), str(tmp_path / "replay_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-Wno-unknown-pragmas", "-I", os.path.join(root, "include"), "-I", csrc,
                    os.path.join(root, "tests", "replay_driver.cpp"), os.path.join(csrc, "ttc_cache.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "replay driver ok" in res.stdout, res.stdout + res.stderr
