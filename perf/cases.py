"""What a program of this library's users has it do, as cases that can be timed.

A case is one call of a public entry point on operands that are already on the GPU, as in a query
plan or a learning loop that keeps its matrices there: R += task(A, B, params), or the join count.
The sizes are the named workloads of amulet_workloads.py where there is one for the use, and
ordinary or odd table sizes else; the value distributions are the ones of that module's recipes,
drawn on the GPU.

  listed()           the cases
  draw(rng)          one more case of the same ranges
  prepare(case, s)   operands, parameters, result (and workspace) of a case, from seed s
  run(state)         one pass: the call; returns the result matrix
  work(case)         bytes and operations that no implementation can do without
  tolerance(case)    what two right implementations may differ by
"""
import math

import torch

import paper_2305_08872_amd as am

TASKS = {"identity": am.AMULET_IDENTITY, "discount": am.AMULET_DISCOUNT, "boost": am.AMULET_BOOST,
         "count_gt": am.AMULET_COUNT_GT}
FORMS = {"col": am.AMULET_THRES_COL, "row": am.AMULET_THRES_ROW, "const": am.AMULET_THRES_CONST,
         "elem": am.AMULET_THRES_ELEM}


def _case(name, op, task, M, N, K, form="col", trans_a=False, trans_b=False):
    c = {"op": op, "task": task, "M": M, "N": N, "K": K, "form": form, "trans_a": trans_a, "trans_b": trans_b}
    return dict(c, name=name) if name else c


def listed():
    return [
        # Query 1 on a small table: one of many short calls, where launch and latency count
        _case("discount_f32_256", "f32", "discount", 256, 256, 256),
        # Query 1 on tables whose row counts are whatever they are (odd pitches, ragged tiles)
        _case("discount_f32_odd", "f32", "discount", 1003, 1501, 777),
        # Query 1 at the headline size, the largest
        _case("discount_f32_8192", "f32", "discount", 8192, 8192, 8192),
        # Query 1 with a threshold per output and B stored by columns
        _case("discount_f32_elem_bt", "f32_general", "discount", 3000, 2000, 1200, form="elem", trans_b=True),
        # Query 2 (signal strengths), the mid-size named workload
        _case("boost_f32_2048", "f32", "boost", 2048, 2048, 2048),
        # Query 3 (count over a threshold) at the paper's square size
        _case("count_gt_f32_4096", "f32", "count_gt", 4096, 4096, 4096),
        # plain matrix multiplication through the same interface, few tiles and many
        _case("identity_f32_1024", "f32", "identity", 1024, 1024, 1024),
        _case("identity_f32_4096", "f32", "identity", 4096, 4096, 4096),
        # join count as a matrix product: the named workload, accumulated
        _case("join_i8_8192x8192x4096", "i8", "join", 8192, 8192, 4096),
        # join count of relations with arbitrary key counts, the count written
        _case("join_i8_odd_assign", "i8_assign", "join", 2999, 4001, 2503),
        # Query 1 in the paper's own element type
        _case("discount_f64_2048", "f64", "discount", 2048, 2048, 2048),
        # plain matrix multiplication in the paper's own element type
        _case("identity_f64_1024", "f64", "identity", 1024, 1024, 1024),
    ]


def _size(rng, low, high):
    """A row or column count, even over the logarithm; one in two padded to whole 64s as tables kept
    for a GPU often are, the others as they fall."""
    n = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
    return max(64, n // 64 * 64) if rng.random() < 0.5 else n


def draw(rng):
    """A call of any of the entry points above on 64 to 8192 rows, columns and inner length (no more
    products than 2^38; fp64, whose rate is half, 2^36), every task, threshold form and layout."""
    op = rng.choice(["f32", "f32", "f32_general", "f64", "i8", "i8_assign", "i8_general"])
    while True:
        M, N, K = (_size(rng, 64, 8192) for _ in range(3))
        if M * N * K <= (2 ** 36 if op == "f64" else 2 ** 38):
            break
    if op.startswith("i8"):
        general = op == "i8_general"
        return _case(None, op, "join", M, N, K, trans_a=general and rng.random() < 0.5, trans_b=general and rng.random() < 0.5)
    task = rng.choice(["identity", "discount", "discount", "boost", "count_gt"])
    form, ta, tb = "col", False, False
    if op != "f32":
        form = rng.choice(["col", "row", "const", "elem"])
        ta, tb = rng.random() < 0.3, rng.random() < 0.3
    return _case(None, op, task, M, N, K, form, ta, tb)


def prepare(case, seed):
    M, N, K, op, task = case["M"], case["N"], case["K"], case["op"], case["task"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = torch.float64 if op == "f64" else torch.float32
    sa = (K, M) if case["trans_a"] else (M, K)
    sb = (N, K) if case["trans_b"] else (K, N)

    def uniform(lo, hi, *shape):
        return torch.empty(shape, dtype=dt, device="cuda").uniform_(lo, hi, generator=g)

    def normal(*shape):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(generator=g)

    s = dict(case, workspace=None, params=None, thres=None, dis=None)
    if task == "join":
        # indicator matrices, one key in twenty present
        s["A"] = (torch.empty(sa, device="cuda").uniform_(generator=g) < 0.05).to(torch.int8)
        s["B"] = (torch.empty(sb, device="cuda").uniform_(generator=g) < 0.05).to(torch.int8)
        s["R"] = torch.zeros(M, N, dtype=torch.int32, device="cuda")
        if op == "i8_general":
            s["workspace"] = torch.empty(am.amulet_count_i8_repack_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
        return s
    n_thres = {"col": (N,), "row": (M,), "const": (1,), "elem": (M, N)}[case["form"]]
    if task == "identity":
        s["A"], s["B"] = uniform(-1, 1, *sa), uniform(-1, 1, *sb)
    elif task == "boost":
        s["A"], s["B"] = normal(*sa), normal(*sb)
        s["thres"] = normal(*n_thres).abs_() + 1
    else:
        # units bought, list prices, and a threshold per seller (and discount)
        s["A"] = torch.randint(0, 10, sa, generator=g, device="cuda").to(dt)
        s["B"] = uniform(1, 100, *sb)
        s["thres"] = uniform(100, 500, *n_thres) if task == "discount" else uniform(50, 150, *n_thres)
        if task == "discount":
            s["dis"] = uniform(0.05, 0.3, N)
    if op == "f32" and s["thres"] is not None:
        s["params"] = torch.stack([s["thres"], s["dis"]]) if task == "discount" else s["thres"][None, :].contiguous()
    s["R"] = torch.zeros(M, N, dtype=dt, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "f32":
        am.amulet_mmlike_f32(TASKS[s["task"]], s["A"], s["B"], s["params"], s["R"])
    elif op == "f32_general":
        am.amulet_mmlike_f32_general(TASKS[s["task"]], s["A"], s["B"], s["thres"], s["dis"], s["R"],
                                     thres_form=FORMS[s["form"]], trans_a=s["trans_a"], trans_b=s["trans_b"])
    elif op == "f64":
        am.amulet_mmlike_f64(TASKS[s["task"]], s["A"], s["B"], s["thres"], s["dis"], s["R"],
                             thres_form=FORMS[s["form"]], trans_a=s["trans_a"], trans_b=s["trans_b"])
    elif op == "i8":
        am.amulet_count_i8(s["A"], s["B"], s["R"])
    elif op == "i8_assign":
        am.amulet_count_i8_assign(s["A"], s["B"], s["R"])
    else:
        am.amulet_count_i8_general(s["A"], s["B"], s["R"], s["workspace"], trans_a=s["trans_a"], trans_b=s["trans_b"])
    return s["R"]


def work(case):
    M, N, K, op, task = case["M"], case["N"], case["K"], case["op"], case["task"]
    e = {"f64": 8, "f32": 4, "f32_general": 4}.get(op, 1)     # bytes of an operand's element
    r = 8 if op == "f64" else 4                               # and of a result's
    b = e * (M * K + K * N) + r * M * N * (1 if op == "i8_assign" else 2)
    if task in ("discount", "boost", "count_gt"):
        b += e * {"col": N, "row": M, "const": 1, "elem": M * N}[case["form"]]
    if task == "discount":
        b += e * N
    return {"bytes": b, "flops": 2 * M * N * K}


def tolerance(case):
    if case["task"] in ("join", "count_gt"):
        return "exact"                                        # whole numbers
    return {"rel": 1e-13} if case["op"] == "f64" else {"rel": 1e-5}
