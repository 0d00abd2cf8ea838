"""The line kernel (tiles cut where lines of B end): every candidate against the oracle, replayed on the host and run on
the GPU, at the sizes where its tiles can go wrong: fewer columns than a vector in the last tile, rows that end
inside the first line, one row or one column more than a tile, columns of B at every place inside a line."""
import numpy as np
import pytest

import oracle
import paper_1603_02297_amd as ttc
from paper_1603_02297_amd import workloads as wl

# sizes, perm, lda, ldb
SHAPES = [
    ((33, 129), (1, 0), None, None),                 # one column and one row more than a tile
    ((65, 31), (1, 0), None, None),                  # rows shorter than a line of fp32
    ((64, 256), (1, 0), None, None),                 # B's columns on whole lines: tiles not skewed
    ((34, 70), (1, 0), (37, 70), (71, 34)),          # leading dimensions on both sides
    ((4, 4), (1, 0), None, None),                    # the smallest tensor: one vector each way
    ((7, 11, 9), (2, 1, 0), None, None),
    ((5, 13, 40), (2, 0, 1), None, None),            # fuses to (65, 40)
    ((12, 5, 7, 9), (3, 2, 1, 0), None, None),       # two indices taken as one on both sides
    ((6, 7, 5, 9), (3, 1, 0, 2), (6, 8, 5, 9), None),
    ((9, 4, 3, 5, 8), (4, 1, 3, 0, 2), None, (9, 4, 5, 9, 3)),
]
DTYPES = [wl.F32, wl.F64, wl.C64, wl.C128, wl.F32_F64, wl.F64_F32, wl.C64_C128, wl.C128_C64]


def line_candidates(plan):
    """Indices of the plan's line-kernel candidates: staged through LDS, and `unroll` (lines per tile) is set."""
    for k in range(ttc.ttc_plan_candidate_count(plan)):
        ttc.ttc_plan_select_candidate(plan, k)
        info = ttc.ttc_plan_get_info(plan)
        if info["kernel_class"] == ttc.TTC_KERNEL_LDS and info["unroll"] > 0:
            yield k, info


def form(info, dtype):
    """How a line candidate's arguments go to the kernel, mirrored from the library: "whole", or packed, for tiles as they come ("small": a
    workgroup's number is its tile's), for one range of tiles per XCD ("ranges") or for any other dealing, or A streamed ("dealt"); and whether
    its indices are merged."""
    cols, lines, ea, eb = info["digit_tile_a"][0], info["unroll"], wl.ELEM_BYTES[dtype], wl.ELEM_BYTES_B[dtype]
    merged, update = bool(info["merged"]), info["epilogue"] == ttc.TTC_EPI_AXPBY
    dealing = "dealt" if info["xcd_remap"] > 1 or info["nt_a"] != 0 else "ranges" if info["xcd_remap"] == 1 else "small"
    passes = lines * (128 // eb) * (cols * ea // 16) // 256              # vectors of A a lane loads
    words = (18 if merged else 12) + 2 * info["epilogue"] * wl.COMPONENTS[dtype]
    used = {k for k in range(info["ndim"]) if info["tile"][k] < info["sizes"][k]} | {0, info["perm"][0]}
    whole = words > 20 or len(used) > 3 or (update and passes >= 8 and dealing == "dealt")
    return ("whole" if whole else dealing), merged


FORMS = {(f, m) for f in ("whole", "small", "ranges", "dealt") for m in (False, True)}


def scalars(dtype):
    cplx = wl.COMPONENTS[dtype] == 2
    return [(1.0, 0.0), (0.5 + 0.5j if cplx else 1.5, 0.0), (0.5 - 0.25j if cplx else 0.75, 1.0 + 0.5j if cplx else -1.25)]


@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_walks_of_every_line_candidate(dtype):
    seen, forms = 0, set()
    for sizes, perm, lda, ldb in SHAPES:
        for beta in (0.0, 1.0):
            p = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, 1.0, beta)
            want = [-1] * ttc.ttc_plan_get_info(p)["span_b"]
            for off_a, off_b in oracle.element_pairs(sizes, perm, lda, ldb):
                want[off_b] = off_a
            for k, info in line_candidates(p):
                for mode, nt in ((-1, 0), (1, 0), ((1, 2, 5)[seen % 3], seen // 3 % 2)):      # tiles dealt to the XCDs, surplus workgroups among them
                    ttc.ttc_plan_set_tile_mapping(p, mode)
                    ttc.ttc_plan_set_streaming(p, nt, nt)
                    forms.add(form(ttc.ttc_plan_get_info(p), dtype))
                    assert list(ttc.ttc_debug_emulate_map(p)) == want, (sizes, perm, k, mode, nt, info)
                seen += 1
            ttc.ttc_plan_destroy(p)
    assert seen >= 40 and forms == FORMS


def multiplicity(addresses, words):
    """Distinct addresses that the lanes of one LDS instruction (`words` 4-byte words each) send to one bank, over the
    unavoidable number: for 32 and for 64 banks, added (2: no conflict)."""
    total = 0
    for banks in (32, 64):
        load = np.bincount([(a + w) % banks for a in set(addresses) for w in range(words)], minlength=banks).max()
        total += -(-int(load) // max(1, -(-len(set(addresses)) * words // banks)))
    return total


@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_reported_bank_conflicts_are_those_of_the_tile(dtype):
    ea, eb = wl.ELEM_BYTES[dtype], wl.ELEM_BYTES_B[dtype]
    p = ttc.ttc_plan_create(dtype, 2, (301, 203), (1, 0), 1.0, 0.0)
    seen = set()
    for k, info in line_candidates(p):
        cols, pitch = info["digit_tile_a"][0], info["lds_stride"][1]            # elements
        per_row, wide = cols * ea // 16, 8 if ea == 4 else 16                   # lanes that write a row, bytes of a write
        writes = [(t // per_row * pitch + t % per_row * (16 // ea)) * ea // 4 for t in range(64)]
        reads = [((t % 8) * (16 // eb) * pitch + t // 8) * ea // 4 for t in range(64)]
        want = (multiplicity(writes, wide // 4), multiplicity(reads, ea // 4))
        assert (info["lds_conflict_a"], info["lds_conflict_b"]) == want, (cols, info["unroll"])
        seen.add(cols)
    assert len(seen) >= 2
    ttc.ttc_plan_destroy(p)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES, ids=[wl.DTYPE_NAME[d] for d in DTYPES])
def test_line_kernel_against_the_oracle(dtype):
    """Every candidate, every epilogue, both streaming settings, tiles as they come, in ranges and dealt otherwise (packed and whole arguments of each); B at
    four places inside a line; what lies around the sub-tensor stays as it was.  Fixed evaluation order on both sides: bit-equal
    but for the ulp the library allows."""
    import torch
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    prod = lambda v: int(np.prod(v))  # noqa: E731
    ran, forms = 0, set()
    for shape, (sizes, perm, lda, ldb) in enumerate(SHAPES):
        na, nb = prod(lda or sizes), prod(ldb or sizes)
        A = wl.uniform_tensor(dtype, na, 7000 + shape, "a")
        B0 = wl.uniform_tensor(dtype, nb, 7100 + shape, "b")
        comp, room = wl.COMPONENTS[dtype], 128
        dA = torch.from_numpy(A).to(dev)
        for alpha, beta in scalars(dtype):
            want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4, lda=lda, ldb=ldb)
            plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, alpha, beta)
            try:
                for k, info in line_candidates(plan):
                    for nt, phase, mode in ((0, 0, -1), (1, 1, (-1, 1, 2, 5)[k % 4]), (0, 3, 1), (0, 7, (2, 5)[k % 2])):
                        ttc.ttc_plan_set_streaming(plan, nt, nt)
                        ttc.ttc_plan_set_tile_mapping(plan, mode)
                        forms.add(form(ttc.ttc_plan_get_info(plan), dtype))
                        buf = torch.full((nb * comp + 2 * room,), 77.0, dtype=torch.from_numpy(B0).dtype, device=dev)
                        at = room + phase * comp
                        buf[at:at + nb * comp] = torch.from_numpy(B0).to(dev)
                        ttc.ttc_execute(plan, dA.data_ptr(), buf.data_ptr() + at * buf.element_size(), stream)
                        torch.cuda.synchronize()
                        got = buf.cpu().numpy()
                        assert (got[:at] == 77).all() and (got[at + nb * comp:] == 77).all(), (sizes, perm, k, info)
                        got = got[at:at + nb * comp]
                        if complex(alpha) == 1 and complex(beta) == 0:
                            assert np.array_equal(got, want), (sizes, perm, k, info)
                        else:
                            ulp = np.spacing(np.abs(want).max())
                            assert np.abs(got - want).max() <= ulp, (sizes, perm, alpha, beta, k, info)
                        ran += 1
            finally:
                ttc.ttc_plan_destroy(plan)
    assert ran >= 100 and forms == FORMS


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.C128, wl.C64_C128, wl.C128_C64], ids=["c128", "c64c128", "c128c64"])
def test_elements_that_start_halfway(dtype):
    """complex128 operands need 8-byte alignment only: elements, and lines of B, that start in the middle of 16 bytes."""
    import torch
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    shift_a, shift_b = (1 if wl.ELEM_BYTES[dtype] == 16 else 2), (1 if wl.ELEM_BYTES_B[dtype] == 16 else 2)        # in components
    ran = 0
    for shape, (sizes, perm, lda, ldb) in enumerate(SHAPES[:4] + SHAPES[-2:]):
        A = wl.uniform_tensor(dtype, int(np.prod(lda or sizes)), 7900 + shape, "a")
        B0 = wl.uniform_tensor(dtype, int(np.prod(ldb or sizes)), 7950 + shape, "b")
        bufa = torch.zeros(A.size + 4, dtype=torch.from_numpy(A).dtype, device=dev)
        bufa[shift_a:shift_a + A.size] = torch.from_numpy(A).to(dev)
        for alpha, beta in scalars(dtype)[::2]:
            want = oracle.transpose(dtype, sizes, perm, alpha, beta, A, B0.copy(), 4, lda=lda, ldb=ldb)
            plan = ttc.ttc_plan_create_ex(dtype, len(sizes), sizes, perm, lda, ldb, alpha, beta)
            try:
                for k, info in line_candidates(plan):
                    buf = torch.full((B0.size + 128,), 77.0, dtype=torch.from_numpy(B0).dtype, device=dev)
                    at = 64 + shift_b
                    buf[at:at + B0.size] = torch.from_numpy(B0).to(dev)
                    ttc.ttc_execute(plan, bufa.data_ptr() + shift_a * bufa.element_size(), buf.data_ptr() + at * buf.element_size(), stream)
                    got = buf.cpu().numpy()
                    assert (got[:at] == 77).all() and (got[at + B0.size:] == 77).all(), (sizes, perm, k, info)
                    allowed = 0.0 if complex(alpha) == 1 and complex(beta) == 0 else np.spacing(np.abs(want).max())
                    assert np.abs(got[at:at + B0.size] - want).max() <= allowed, (sizes, perm, alpha, beta, k, info)
                    ran += 1
            finally:
                ttc.ttc_plan_destroy(plan)
    assert ran >= 40


# (type, extents, permutation, beta, whether each XCD gets one range of tiles): either side of every line of the rule
DEALT_BY_DEFAULT = [
    (wl.F32, (1301, 1303), (1, 0), 0.0, True), (wl.F32, (901, 903), (1, 0), 0.0, False),           # 13.6 MB, 6.5 MB of traffic
    (wl.F32, (521, 503), (1, 0), 1.0, True), (wl.F32, (301, 303), (1, 0), 1.0, False),             # updates of 3.1 and 1.1 MB
    (wl.F64, (17, 40009), (1, 0), 0.0, False), (wl.F64, (16, 40009), (1, 0), 0.0, True),           # hundreds of tiles before the next one along A: lines split, or none
    (wl.F32, (1031, 1024), (1, 0), 0.0, True), (wl.F32, (1032, 1024), (1, 0), 0.0, True),          # whole lines of B, A's split at 4 and 32 bytes
    (wl.F32, (1040, 1024), (1, 0), 0.0, False), (wl.F32, (1024, 1024), (1, 0), 0.0, False),        # at 64 bytes, and none
    (wl.C64, (37, 41, 701), (2, 1, 0), 0.0, True), (wl.C64, (37, 41, 701), (2, 1, 0), 1.0, True),  # merged indices: packed, and whole arguments with an update
    (wl.C128_C64, (13, 47, 611), (2, 1, 0), 0.0, True), (wl.F32_F64, (299, 19, 203), (2, 0, 1), 0.0, True),        # two types
    (wl.F32, (23, 31, 41, 101), (3, 2, 1, 0), 0.0, True),                                          # more places in the tile order than are packed
]


def default_of(plan):
    """The mapping that the first line candidate in B's order has."""
    perm = ttc.ttc_plan_get_info(plan)["perm"]
    for k, info in line_candidates(plan):
        if info["tile_order"] == perm:
            return info
    raise AssertionError("no line candidate")


@pytest.mark.parametrize("dtype,sizes,perm,beta,ranges", DEALT_BY_DEFAULT)
def test_tiles_that_share_lines_are_dealt_in_ranges(dtype, sizes, perm, beta, ranges):
    p = ttc.ttc_plan_create(dtype, len(sizes), sizes, perm, 1.0, beta)
    info = default_of(p)
    plain = 5 if info["num_tiles"] >= 2048 else 0
    assert info["xcd_remap"] == (1 if ranges else plain)
    ttc.ttc_plan_set_tile_mapping(p, 3)
    ttc.ttc_plan_set_tile_mapping(p, -1)
    assert ttc.ttc_plan_get_info(p)["xcd_remap"] == (1 if ranges else plain)
    ttc.ttc_plan_destroy(p)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,sizes,perm,beta,ranges", [c for c in DEALT_BY_DEFAULT if c[-1]])
def test_ranges_against_the_oracle(dtype, sizes, perm, beta, ranges):
    """The plan as created and its line candidates over ranges: tile counts that do not divide by eight, packed arguments, with merged indices too,
    and whole ones."""
    import torch
    n, stream = int(np.prod(sizes)), torch.cuda.current_stream().cuda_stream
    A, B0 = wl.uniform_tensor(dtype, n, 7300, "a"), wl.uniform_tensor(dtype, n, 7301, "b")
    want = oracle.transpose(dtype, sizes, perm, 1.0, beta, A, B0.copy(), 8)
    dA, dB0 = torch.from_numpy(A).cuda(), torch.from_numpy(B0).cuda()
    plan = ttc.ttc_plan_create(dtype, len(sizes), sizes, perm, 1.0, beta)
    seen, forms = 0, set()
    for k, info in [(0, None)] + list(line_candidates(plan)):
        ttc.ttc_plan_select_candidate(plan, k)
        ttc.ttc_plan_set_tile_mapping(plan, -1 if info is None else 1)
        seen += ttc.ttc_plan_get_info(plan)["num_tiles"] % 8 != 0
        if info is not None:
            forms.add(form(ttc.ttc_plan_get_info(plan), dtype))
        dB = dB0.clone()
        ttc.ttc_execute(plan, dA.data_ptr(), dB.data_ptr(), stream)
        allowed = 0.0 if beta == 0 else np.spacing(np.abs(want).max())          # bits are copied; one ulp with an update
        assert np.abs(dB.cpu().numpy() - want).max() <= allowed, (k, ttc.ttc_plan_get_info(plan))
    few, merged = len(sizes) < 4, sizes == (37, 41, 701) or sizes == (13, 47, 611)
    assert seen and (("ranges", False) in forms) == few and (("ranges", True) in forms) == (merged and beta == 0)
    ttc.ttc_plan_destroy(plan)
