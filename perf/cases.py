"""Performance cases of the transposition library: problems as its callers have them, from a few hundred KB to 1.9 GB
of traffic, through the public entry points (a plan that the program keeps, ttc_execute on resident tensors).

A case names the element type (A's, and B's where the two differ), the extents of A (index 0 has stride 1), the
permutation (perm[j] is the index of A that becomes index j of B), alpha and beta, the extents of the enclosing
tensors where the operands are parts of larger ones (lda, ldb), whether the program had the plan searched on its
own buffers (ttc_plan_tune) or runs it as created, and how many tensors it moves with that plan one after the other
(small problems come in numbers).
"""
import math
import weakref

import torch

import paper_1603_02297_amd as ttc

# name: (library code, torch type of A, of B, of the 64-bit result)
TYPES = {
    "f32": (ttc.TTC_F32, torch.float32, torch.float32, torch.float64),
    "f64": (ttc.TTC_F64, torch.float64, torch.float64, torch.float64),
    "c64": (ttc.TTC_C64, torch.complex64, torch.complex64, torch.complex128),
    "c128": (ttc.TTC_C128, torch.complex128, torch.complex128, torch.complex128),
    "f32_f64": (ttc.TTC_F32_F64, torch.float32, torch.float64, torch.float64),
    "f64_f32": (ttc.TTC_F64_F32, torch.float64, torch.float32, torch.float64),
    "c64_c128": (ttc.TTC_C64_C128, torch.complex64, torch.complex128, torch.complex128),
    "c128_c64": (ttc.TTC_C128_C64, torch.complex128, torch.complex64, torch.complex128),
}


def _case(dtype, sizes, perm, alpha=1.0, beta=0.0, lda=None, ldb=None, search=False, tensors=1, name=None):
    """alpha and beta of complex types are (re, im) pairs; the extents travel as text."""
    are, aim = alpha if isinstance(alpha, tuple) else (alpha, 0.0)
    bre, bim = beta if isinstance(beta, tuple) else (beta, 0.0)
    text = lambda v: "x".join(str(int(x)) for x in v)  # noqa: E731
    c = {"dtype": dtype, "sizes": text(sizes), "perm": text(perm), "alpha_re": float(are), "alpha_im": float(aim),
         "beta_re": float(bre), "beta_im": float(bim), "lda": text(lda) if lda else "", "ldb": text(ldb) if ldb else "",
         "search": bool(search), "tensors": int(tensors)}
    return dict(c, name=name) if name else c


def listed():
    return [
        # small tensors re-ordered inside a longer computation: what counts is the cost of a call
        _case("f32", (70, 33, 45), (2, 0, 1), tensors=4, name="small-3d"),
        # matrices that fit the caches, both operands of a product
        _case("f32", (1024, 1024), (1, 0), tensors=2, name="matrix-1024"),
        # index reversal (column-major <-> row-major) with a scale, extents that are whole cache lines
        _case("f32", (384, 384, 384), (2, 1, 0), alpha=1.5, name="reversal-3d"),
        # the same change of storage order with odd extents: no run starts or ends on a line
        _case("f32", (85, 85, 85, 85), (3, 2, 1, 0), name="reversal-odd-4d"),
        # a long-running program that reverses one six-index tensor over and over: the plan is searched first
        _case("f32", (24, 20, 16, 18, 22, 17), (5, 4, 3, 2, 1, 0), search=True, name="reversal-6d-searched"),
        # contraction set-up: pairs of indices exchanged, the result subtracted from a scaled operand
        _case("f32", (24, 20, 16, 18, 22, 17), (1, 0, 2, 3, 5, 4), alpha=2.0, beta=-1.0, name="pairs-6d-update"),
        # two blocks of larger tensors (leading dimensions on both sides), accumulated in double precision
        _case("f64", (72, 72, 72, 72), (3, 2, 1, 0), alpha=0.75, beta=1.0, lda=(80, 72, 75, 72), ldb=(72, 76, 72, 72),
              name="block-4d-f64-update"),
        # complex amplitudes with a short leading index, accumulated: the largest case (1.9 GB of traffic)
        _case("c64", (8, 64, 48, 40, 80), (2, 0, 4, 3, 1), alpha=(0.5, 0.5), beta=(1.0, 0.0), name="complex-5d-update"),
        # the stride-1 index keeps its place: rows of 3.6 KB gathered in another order
        _case("f32", (917, 374, 153), (0, 2, 1), name="rows-3d"),
        # 16-byte elements, four indices, accumulated
        _case("c128", (72, 40, 72, 72), (3, 0, 2, 1), alpha=(0.5, 0.5), beta=(1.0, 0.0), name="complex128-4d-update"),
        # single-precision data handed to a double-precision solver, re-ordered on the way
        _case("f32_f64", (384, 384, 384), (2, 1, 0), alpha=1.5, name="widen-3d"),
        # records of three values turned into three planes, in a batch (array of structures -> structure of arrays)
        _case("f32", (3, 307200, 64), (1, 0, 2), name="records-to-planes"),
    ]


def draw(rng):
    """Any type, 2 to 6 indices, tensors of 64 KB to 240 MB, odd extents and short leading indices among them."""
    dtype = rng.choice(["f32"] * 4 + ["f64"] * 3 + ["c64"] * 3 + ["c128"] * 2 + ["f32_f64", "f64_f32", "c64_c128", "c128_c64"])
    widest = max(torch.empty(0, dtype=t).element_size() for t in TYPES[dtype][1:3])
    n = rng.choice([2, 2, 3, 3, 3, 4, 4, 5, 6])
    while True:
        elements = math.exp(rng.uniform(math.log(64 * 1024 / 4), math.log(230e6 / widest)))
        share = [0.35 + rng.random() for _ in range(n)]
        share = [s / sum(share) for s in share]
        sizes = [max(2, round(elements ** s)) for s in share]
        if n >= 3 and rng.random() < 0.25:                       # a short index at the front of A or of B: records, components
            sizes[0] = rng.randint(2, 9)
        if rng.random() < 0.35:                                  # extents as programs choose them: multiples of eight
            sizes = [max(8, 8 * round(s / 8)) if s > 12 else s for s in sizes]
        total = math.prod(sizes)
        if 64 * 1024 <= total * widest <= 240e6:
            break
    kind = rng.random()
    if kind < 0.25:
        perm = list(range(n))[::-1]
    elif kind < 0.45 and n >= 3:
        rest = list(range(1, n))
        while rest == list(range(1, n)):
            rng.shuffle(rest)
        perm = [0] + rest
    else:
        perm = list(range(n))
        while perm == list(range(n)) or perm[0] == 0:
            rng.shuffle(perm)
    if rng.random() < 0.15:                                      # the short index may also be B's first
        sizes = [sizes[k] for k in perm]
    complex_ = dtype.startswith("c")
    epilogue = rng.random()
    alpha, beta = 1.0, 0.0
    if epilogue >= 0.4:
        alpha = (0.5, 0.5) if complex_ else rng.choice([1.5, 0.75, 2.0])
    if epilogue >= 0.6:
        beta = (1.0, 0.0) if complex_ else rng.choice([1.0, -1.0])
    lda = ldb = None
    if rng.random() < 0.2:                                       # a block of a larger tensor, on either side
        lda = [s + (rng.randint(0, 1 + s // 8) if k < n - 1 else 0) for k, s in enumerate(sizes)]
        ldb = [sizes[p] + (rng.randint(0, 1 + sizes[p] // 8) if j < n - 1 else 0) for j, p in enumerate(perm)]
        room = 300e6 / widest
        if math.prod(lda) > room or math.prod(ldb) > room:
            lda = ldb = None
    size = math.prod(sizes) * widest
    return _case(dtype, sizes, perm, alpha, beta, lda, ldb, search=rng.random() < 0.15,
                 tensors=4 if size < 2e6 else 2 if size < 12e6 else 1)


def _numbers(text):
    return [int(x) for x in text.split("x")] if text else None


def _operands(case, seed):
    """(list of A, list of B, sizes, perm, lda, ldb, alpha, beta): flat device buffers, values uniform on [-1, 1)."""
    _, ta, tb, _ = TYPES[case["dtype"]]
    sizes, perm = _numbers(case["sizes"]), _numbers(case["perm"])
    lda, ldb = _numbers(case["lda"]), _numbers(case["ldb"])
    g = torch.Generator(device="cuda").manual_seed(seed)

    def uniform(n, dtype):
        real = torch.empty(0, dtype=dtype).real.dtype
        x = torch.rand(n * (2 if dtype.is_complex else 1), dtype=real, device="cuda", generator=g).mul_(2).sub_(1)
        return torch.view_as_complex(x.view(n, 2)) if dtype.is_complex else x

    count = case["tensors"]
    A = [uniform(math.prod(lda or sizes), ta) for _ in range(count)]
    nb = math.prod(ldb or sizes)
    alpha, beta = complex(case["alpha_re"], case["alpha_im"]), complex(case["beta_re"], case["beta_im"])
    B = [uniform(nb, tb) if beta != 0 else torch.zeros(nb, dtype=tb, device="cuda") for _ in range(count)]
    if not ta.is_complex:
        alpha, beta = alpha.real, beta.real
    return A, B, sizes, perm, lda, ldb, alpha, beta


class Plan:
    """A plan handle that is given back with its owner."""

    def __init__(self, *args):
        self.handle = ttc.ttc_plan_create_ex(*args)
        weakref.finalize(self, ttc.ttc_plan_destroy, self.handle)


def prepare(case, seed):
    A, B, sizes, perm, lda, ldb, alpha, beta = _operands(case, seed)
    plan = Plan(TYPES[case["dtype"]][0], len(sizes), sizes, perm, lda, ldb, alpha, beta)
    stream = torch.cuda.current_stream().cuda_stream
    if case["search"]:
        scratch = torch.empty_like(B[0])                         # the search overwrites its target
        ttc.ttc_plan_tune(plan.handle, A[0].data_ptr(), scratch.data_ptr(), stream)
        del scratch
    return {"plan": plan, "A": A, "B": B, "stream": stream}


def run(state):
    for a, b in zip(state["A"], state["B"]):
        ttc.ttc_execute(state["plan"].handle, a.data_ptr(), b.data_ptr(), state["stream"])
    return state["B"]


def work(case):
    _, ta, tb, _ = TYPES[case["dtype"]]
    n = math.prod(_numbers(case["sizes"])) * case["tensors"]
    ea, eb = (torch.empty(0, dtype=t).element_size() for t in (ta, tb))
    update = case["beta_re"] != 0 or case["beta_im"] != 0
    scaled = update or case["alpha_re"] != 1 or case["alpha_im"] != 0
    flops = (3 if update else 1 if scaled else 0) if not ta.is_complex else (14 if update else 6 if scaled else 0)
    return {"bytes": n * (ea + eb * (2 if update else 1)), "flops": n * flops}


def tolerance(case):
    """A pure copy moves bits.  Otherwise a result differs by how its one product and sum are rounded: about four times
    the error against 64 bits that this path shows (2.8e-8 in 32 bits), and in 64 bits four times what one more
    rounding, of the product before the sum, gives (1e-16)."""
    update = case["beta_re"] != 0 or case["beta_im"] != 0
    if not update and case["alpha_re"] == 1 and case["alpha_im"] == 0 and "_" not in case["dtype"]:
        return "exact"
    single = TYPES[case["dtype"]][2] in (torch.float32, torch.complex64)
    return {"rel": 1.2e-7, "max": 5e-7} if single else {"rel": 4e-16, "max": 2e-15}


def exact(case, seed):
    A, B, sizes, perm, lda, ldb, alpha, beta = _operands(case, seed)
    wide = TYPES[case["dtype"]][3]
    n = len(sizes)
    results = []
    for x, y in zip(A, B):
        # column-major extents are a torch shape read backwards
        a = x.view((lda or sizes)[::-1])[tuple(slice(s) for s in sizes[::-1])]
        result = y.to(wide, copy=True)
        b = result.view((ldb or [sizes[p] for p in perm])[::-1])[tuple(slice(sizes[p]) for p in perm[::-1])]
        moved = a.permute([n - 1 - p for p in perm[::-1]]).to(wide)
        b.copy_(alpha * moved + beta * b if beta != 0 else alpha * moved)
        results.append(result)
    return results
