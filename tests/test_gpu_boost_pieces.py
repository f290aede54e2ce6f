"""GPU parity of BOOST with its plain sum on the matrix cores: remainders of tiles and of K, K in parts, every threshold
form and layout, and the values that send a workgroup to its second way of forming a tile."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FORMS = ("col", "row", "const", "elem")


@pytest.fixture(scope="module")
def am():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_08872_amd as am
    am.load_library()
    am.amulet_clear_selections()
    return am


def run(am, A, B, th, R, form, tA, tB, must=True):
    am.amulet_mmlike_f32_general(am.AMULET_BOOST, A, B, th, None, R, thres_form=FORMS.index(form), trans_a=tA, trans_b=tB)
    kernel = am.amulet_recent_kernel()
    torch.cuda.synchronize()
    assert "bf16_pieces" in kernel or not must, kernel
    return "bf16_pieces" in kernel


def check(R, R0, A, B, th, form, tA, tB, bound):
    """Sampled rows (the first and last tile's, some between) against 64 bits: |error| within `bound` of the sum of magnitudes."""
    a, b = (A.T if tA else A), (B.T if tB else B).double()
    M = a.shape[0]
    rows = sorted(set(list(range(0, M, max(1, M // 23))) + [M - 1, M - 2, 31, 32]) & set(range(M)))
    for i in rows:
        t = {"col": lambda: th, "row": lambda: th[i], "const": lambda: th[0], "elem": lambda: th[i]}[form]().double()
        p = a[i].double()[:, None] * b
        term = p + (p - t).clamp_min(0)
        want, mag = term.sum(0) + R0, term.abs().sum(0)
        err = (R[i].double() - want).abs() - 2.0 ** -23 * want.abs() - 2.0 ** -149
        assert bool((err <= bound * mag).all()), (i, float((err / mag.clamp_min(1e-300)).max()))


def make(g, M, N, K, form, tA, tB, pad=0):
    def normal(r, c):
        return torch.empty(r, c + pad, device="cuda").normal_(generator=g)[:, :c]
    A, B = normal(*((K, M) if tA else (M, K))), normal(*((N, K) if tB else (K, N)))
    shape = {"col": (N,), "row": (M,), "const": (1,), "elem": (M, N)}[form]
    return A, B, torch.empty(*shape, device="cuda").normal_(generator=g)


# whole tiles; a part of K per workgroup and its remainders 1 .. 15; rows and columns one past and one short of a tile; an unaligned pitch
# (the sizes whose plan it is differ between forms and layouts: the rest are checked all the same)
SIZES = [(2048, 2048, 64, 0), (2048, 2048, 79, 0), (2049, 2047, 65, 1), (2017, 2015, 66, 3), (1024, 2048, 2033, 3), (1024, 1024, 1009, 0), (2079, 1793, 527, 2)]


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("form", FORMS)
def test_remainders_forms_and_layouts(am, form, tA, tB):
    ran = []
    for M, N, K, pad in SIZES:
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        A, B, th = make(g, M, N, K, form, tA, tB, pad)
        R = torch.full((M, N + pad), 0.25, device="cuda")[:, :N]
        print("boost pieces", form, tA, tB, M, N, K, pad, flush=True)
        ran.append(run(am, A, B, th, R, form, tA, tB, must=False))
        # partial sums over 64 k: 64 + 24 roundings of at most half an ulp each, then one per part
        check(R, 0.25, A, B, th, form, tA, tB, 100 * 2.0 ** -24)
    assert ran[0] and ran[1] and ran[3] and (ran[4] or (tA and form == "elem")), ran


@pytest.mark.parametrize("tA,tB", [(False, False), (True, True)])
@pytest.mark.parametrize("what", ["tiny a", "tiny b", "large sums", "thresholds", "subnormal"])
def test_values_of_the_second_way(am, what, tA, tB):
    M, N, K = 2040, 2047, 79
    for form in FORMS:
        g = torch.Generator(device="cuda").manual_seed(3)
        A, B, th = make(g, M, N, K, form, tA, tB)
        a, b = (A.T if tA else A), (B.T if tB else B)
        if what == "tiny a":
            a[5] *= 2.0 ** -60
            a[31, 3] = 2.0 ** -120
            a[31, 4:] = 0
        elif what == "tiny b":
            b[7, 40] = 2.0 ** -100
            b[:7, 40] = 0
            b[8:, 40] = 0
            a[9] *= 2.0 ** 90
        elif what == "large sums":
            a[33] *= 2.0 ** 40
            b[:, 300] *= 2.0 ** 30
            a[64] *= 2.0 ** 100
        elif what == "thresholds":
            special = torch.tensor([0.0, -0.0, 1e-30, -1e-30, float("inf"), -1e30, 2.0 ** 60, 1e-45], device="cuda")
            th.view(-1)[:8] = special[: min(8, th.numel())] if th.numel() >= 8 else special[2:3]
        else:
            A *= 2.0 ** -63
            B *= 2.0 ** -64
            th *= 2.0 ** -127
        R = torch.zeros(M, N, device="cuda")
        print("boost pieces special", what, form, tA, tB, flush=True)
        run(am, A, B, th, R, form, tA, tB)
        # (subnormal: a product of some 2^-128 is rounded to 2^-149, in each of the three places it is used)
        check(R, 0.0, A, B, th, form, tA, tB, 3 * 2.0 ** -20 if what == "subnormal" else 1e-5)


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("form", FORMS)
def test_where_the_second_way_begins(am, form, tA, tB):
    """One value that the pieces do not take, found after the first partial sum, the second, some later one or at the end
    only; in tiles of their own, beside tiles without one, and where K is in parts and their remainders."""
    for M, N, K, pad in [(2048, 2048, 300, 0), (2049, 2047, 143, 1), (1024, 2048, 2033, 3)]:
        g = torch.Generator(device="cuda").manual_seed(K)
        A, B, th = make(g, M, N, K, form, tA, tB, pad)
        a, b = (A.T if tA else A), (B.T if tB else B)
        for i, k in enumerate([0, 63, 64, 100, 128, K // 2, K - 1]):
            a[40 * i + 1, k] = 1e-12 if i % 2 else 1e-40
        b[K - 2, 700] = -1e-30
        R = torch.full((M, N + pad), 0.25, device="cuda")[:, :N]
        print("boost pieces second way", form, tA, tB, M, N, K, pad, flush=True)
        run(am, A, B, th, R, form, tA, tB, must=K == 300 and not (tA and form == "elem"))
        check(R, 0.25, A, B, th, form, tA, tB, 100 * 2.0 ** -24)
        rows = [40 * i + 1 for i in range(7)]      # (check samples rows: these, and one beside them in the tile)
        rows += [r + 1 for r in rows]
        t = {"col": lambda: th[None], "row": lambda: th[rows][:, None], "const": lambda: th[0], "elem": lambda: th[rows]}[form]().double()
        want, mag = torch.full((len(rows), N), 0.25, dtype=torch.float64, device="cuda"), torch.zeros(len(rows), N, dtype=torch.float64, device="cuda")
        for k in range(K):
            p = a[rows, k].double()[:, None] * b[k].double()[None]
            term = p + (p - t).clamp_min(0)
            want, mag = want + term, mag + term.abs()
        assert bool(((R[rows].double() - want).abs() - 2.0 ** -23 * want.abs() <= 100 * 2.0 ** -24 * mag).all())


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("size", [46, 52, 60])
def test_a_term_beyond_the_clamp_is_found_beside_large_sums(am, size, form):
    """Negative products of 2^size and, after two folds, one large positive one in a row of each tile: its term counts as
    2^52 where the clamp goes unnoticed, as it does where the partial sum began below zero with what a fold had rounded away."""
    M, N, K = 2048, 2048, 256
    g = torch.Generator(device="cuda").manual_seed(size)
    A = -(torch.rand(M, K, device="cuda", generator=g) + 0.5) * 2.0 ** size
    rows = torch.arange(0, M, 32, device="cuda") + torch.randint(0, 32, (M // 32,), device="cuda", generator=g)
    A[rows, torch.randint(128, K, (M // 32,), device="cuda", generator=g)] = 2.0 ** (max(size, 52) + 8)
    B, th = torch.ones(K, N, device="cuda"), torch.ones({"col": (N,), "row": (M,), "const": (1,), "elem": (M, N)}[form], device="cuda")
    R = torch.zeros(M, N, device="cuda")
    print("boost pieces clamp", size, form, flush=True)
    run(am, A, B, th, R, form, False, False)
    term = A.double() + (A.double() - 1).clamp_min(0)
    worst = ((R.double() - term.sum(1)[:, None]).abs() / term.abs().sum(1)[:, None]).max()
    assert float(worst) <= 1e-5, float(worst)


def test_infinities_and_nan_stay_with_their_rows(am):
    M, N, K = 1024, 1024, 1024
    g = torch.Generator(device="cuda").manual_seed(4)
    A, B, th = make(g, M, N, K, "col", False, False)
    B[0] = 1.0
    A[3, 0], A[70, 0], A[100, 0] = float("inf"), float("-inf"), float("nan")
    R = torch.zeros(M, N, device="cuda")
    run(am, A, B, th, R, "col", False, False)
    assert bool((R[3] == float("inf")).all()) and bool((R[70] == float("-inf")).all()) and bool(R[100].isnan().all())
    rest = torch.ones(M, dtype=torch.bool, device="cuda")
    rest[[3, 70, 100]] = False
    assert bool(R[rest].isfinite().all())
    th[7] = float("-inf")         # always triggers
    A[3, 0] = A[70, 0] = A[100, 0] = 1.0
    R.zero_()
    run(am, A, B, th, R, "col", False, False)
    assert bool((R[:, 7] == float("inf")).all()) and bool(R[:, :7].isfinite().all()) and bool(R[:, 8:].isfinite().all())
