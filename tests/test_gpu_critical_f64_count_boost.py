"""GPU parity of fp64 COUNT by critical values and BOOST by a clamp: products at the threshold, remainders of tiles and of K, forms
and layouts, rows left to the tile kernels, and the values that send a tile to the task's own operations; of COUNT and DISCOUNT
thresholds of 0 and below."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def am():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_08872_amd as am
    am.load_library()
    am.amulet_clear_selections()
    return am


def run(am, task, A, B, th, R, form, tA=False, tB=False):
    """The kernels it was, the last one first."""
    am.amulet_mmlike_f64(getattr(am, "AMULET_" + task.upper()), A, B, th, None, R, thres_form=getattr(am, "AMULET_THRES_" + form.upper()),
                         trans_a=tA, trans_b=tB)
    kernels = [am.amulet_recent_kernel(0), am.amulet_recent_kernel(1)]
    torch.cuda.synchronize()
    return kernels


def reference(task, A, B, th, form, R0, tA=False, tB=False):
    """Sum and sum of magnitudes, product by product in 64 bits."""
    a, b = (A.T if tA else A), (B.T if tB else B)
    if form == "row":
        th = th[:, None]
    want, mag = torch.full((a.shape[0], b.shape[1]), R0, dtype=torch.float64, device="cuda"), 0.0
    for k in range(a.shape[1]):
        p = a[:, k, None] * b[k]
        if task == "count_gt":
            want += (p > th).double()
        else:
            over = torch.where(p > th, p - th, 0.0)
            want += p
            want += over
            mag = mag + p.abs() + over
    return want, mag


def close(task, R, want, mag, K):
    if task == "count_gt":
        return R == want
    # 2 K sums here and in the reference, whose product is rounded before the threshold is taken off, and the last one
    ok = (R - want).abs() <= 2.0 ** -53 * ((4 * K + 3) * mag + 2 * want.abs())
    odd = ~torch.isfinite(want)
    return ok | odd & (torch.isnan(R) == torch.isnan(want)) & (torch.isnan(want) | (R == want))


def make(seed, M, N, K, form, tA=False, tB=False, pad=0):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(r, c):
        return torch.empty(r, c + pad, dtype=torch.float64, device="cuda").normal_(generator=g)[:, :c]
    A, B = normal(*((K, M) if tA else (M, K))), normal(*((N, K) if tB else (K, N)))
    n = {"col": N, "row": M, "const": 1}[form]
    return A, B, torch.empty(n, dtype=torch.float64, device="cuda").uniform_(0.05, 2, generator=g)


@pytest.mark.parametrize("form", ["col", "row"])
@pytest.mark.parametrize("sign", [1, -1])
def test_products_at_the_threshold(am, sign, form):
    """One product per sum, thresholds one ulp below, at and above some of them: every decision shows."""
    M, N, K = 3072 if form == "col" else 4096, 2048, 64       # (each a size whose plan it is)
    g = torch.Generator(device="cuda").manual_seed(64)
    for bits in (53, 27, 14):       # 27: products of 53 and 54 bits, ties among them; 14: exact products
        def value(n):
            v = torch.empty(n, dtype=torch.float64, device="cuda").uniform_(1, 2, generator=g)
            return torch.round(v * 2.0 ** (bits - 1)) * 2.0 ** (1 - bits) * 2.0 ** torch.randint(-3, 12, (n,), generator=g, device="cuda").double()
        a, b = sign * value(M), sign * value(N)
        A, B = torch.zeros(M, K, dtype=torch.float64, device="cuda"), torch.zeros(K, N, dtype=torch.float64, device="cuda")
        A[:, K - 3], B[K - 3] = a, b
        th = a[torch.arange(N, device="cuda") % M] * b if form == "col" else a * b[torch.arange(M, device="cuda") % N]
        step = torch.arange(len(th), device="cuda") % 3
        th = torch.where(step == 0, th, torch.nextafter(th, (step == 1).double() * 1e9))
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        assert "critical_rows 128" in run(am, "count_gt", A, B, th, R, form)[0]
        assert torch.equal(R, (a[:, None] * b > (th if form == "col" else th[:, None])).double()), (bits, sign)


@pytest.mark.parametrize("task", ["count_gt", "discount"])
@pytest.mark.parametrize("sign", [1, -1])
def test_negative_thresholds(am, task, sign):
    """As above with products below 0, K one past a stage; what is nothing times something is above such a threshold."""
    M, N, K = 3072, 2048, 65
    g = torch.Generator(device="cuda").manual_seed(65)
    for bits in (53, 27, 14):
        def value(n):
            v = torch.empty(n, dtype=torch.float64, device="cuda").uniform_(1, 2, generator=g)
            return torch.round(v * 2.0 ** (bits - 1)) * 2.0 ** (1 - bits) * 2.0 ** torch.randint(-3, 12, (n,), generator=g, device="cuda").double()
        a, b = sign * value(M), -sign * value(N)
        b[5] = 0.0
        A, B = torch.zeros(M, K, dtype=torch.float64, device="cuda"), torch.zeros(K, N, dtype=torch.float64, device="cuda")
        A[:, K - 1], B[K - 1] = a, b
        th = a[torch.arange(N, device="cuda") % M] * b
        th[5], th[6] = -1.0, -4.0          # (a power of two: the number below it in magnitude is nearer)
        step = torch.arange(N, device="cuda") % 3
        th = torch.where((step == 0) | (b == 0), th, torch.nextafter(th, (step == 1).double() * 2e9 - 1e9))
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        dis = torch.ones(N, dtype=torch.float64, device="cuda")
        am.amulet_mmlike_f64(getattr(am, "AMULET_" + task.upper()), A, B, th, dis if task == "discount" else None, R)
        assert "critical_rows" in am.amulet_recent_kernel(0)
        p = a[:, None] * b
        want = K - 1 + (p > th).double() if task == "count_gt" else torch.where(p > th, 0.0, p)
        assert torch.equal(R, want), (bits, sign)


@pytest.mark.parametrize("task", ["count_gt", "discount"])
@pytest.mark.parametrize("least", [1e-12, 1e-90, 1e-160])
def test_thresholds_of_zero(am, task, least):
    """Both signs of both operands, zeros among them; 1e-160: products of 0 from operands that are not, by the plain way."""
    M, N, K = 4093, 2047, 67
    g = torch.Generator(device="cuda").manual_seed(3)

    def value(*n):
        v = torch.empty(n, dtype=torch.float64, device="cuda").normal_(generator=g)
        s = torch.where(torch.randint(0, 2, n, generator=g, device="cuda") == 0, 1.0, least).double()
        return v * s * (torch.randint(0, 5, n, generator=g, device="cuda") != 0)
    A, B, th = value(M, K), value(K, N), torch.zeros(N, dtype=torch.float64, device="cuda")
    th[::2], th[::3] = -0.0, 0.5
    dis = torch.empty(N, dtype=torch.float64, device="cuda").uniform_(0, 1, generator=g)
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    am.amulet_mmlike_f64(getattr(am, "AMULET_" + task.upper()), A, B, th, dis if task == "discount" else None, R)
    assert "critical_rows" in " ".join(am.amulet_recent_kernel(i) for i in range(2))
    if task == "count_gt":
        assert torch.equal(R, reference(task, A, B, th, "col", 0.0)[0])
        return
    want, mag = torch.zeros_like(R), torch.zeros_like(R)
    for k in range(K):
        p = A[:, k, None] * B[k]
        term = torch.where(p > th, p * (1.0 - dis), p)
        want += term
        mag += p.abs()
    assert bool(((R - want).abs() <= 2.0 ** -53 * (2 * K + 5) * mag).all())


SIZES = [(4096, 2048, 64, 0), (4095, 2047, 67, 1), (4161, 2050, 271, 3), (8193, 1029, 79, 1)]


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("task,form", [("count_gt", "col"), ("count_gt", "row"), ("count_gt", "const"), ("boost", "col"), ("boost", "row"), ("boost", "const")])
def test_remainders_forms_and_layouts(am, task, form, tA, tB):
    ran = []
    for M, N, K, pad in SIZES:
        A, B, th = make(M + N + K, M, N, K, form, tA, tB, pad)
        whole = torch.full((M, N + pad), 0.25, dtype=torch.float64, device="cuda")
        R = whole[:, :N]
        print("critical f64", task, form, M, N, K, tA, tB, flush=True)
        ran.append(" ".join(run(am, task, A, B, th, R, form, tA, tB)))
        want, mag = reference(task, A, B, th, form, 0.25, tA, tB)
        assert bool(close(task, R, want, mag, K).all()), (M, N, K)
        assert bool((whole[:, N:] == 0.25).all())
    assert sum("critical_rows" in r for r in ran) >= 3, ran


@pytest.mark.parametrize("form,tA,tB", [("col", False, False), ("row", True, False), ("const", False, True), ("col", True, True)])
@pytest.mark.parametrize("K", [65, 71, 72, 263])
def test_boost_below_zero_stops_at_the_last_k(am, form, K, tA, tB):
    """Thresholds of both signs: a k past the last one, nothing times nothing, would be over those below 0."""
    M, N = 4093, 2047
    A, B, th = make(K, M, N, K, form, tA, tB)
    th[::2] *= -1.0
    if form != "const":
        th[1], th[3], th[5], th[150], th[151] = 2.0 ** 100, 2.0 ** 101, 1e200, 1.7976931348623157e308, float("inf")
    R = torch.full((M, N), 0.25, dtype=torch.float64, device="cuda")
    assert "critical_rows 64" in run(am, "boost", A, B, th, R, form, tA, tB)[0]
    want, mag = reference("boost", A, B, th, form, 0.25, tA, tB)
    assert bool(close("boost", R, want, mag, K).all())


@pytest.mark.parametrize("task,form", [("count_gt", "col"), ("count_gt", "row"), ("boost", "row")])
def test_rows_left_to_the_tile_kernels(am, task, form):
    left = 0
    for M, N, K in [(2560, 1751, 1792), (5120, 1751, 1300), (1751, 5120, 1300), (9000, 1100, 900)]:
        A, B, th = make(M, M, N, K, form)
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        kernels = run(am, task, A, B, th, R, form)
        left += "critical" not in kernels[0] and "critical_rows" in kernels[1]
        want, mag = reference(task, A, B, th, form, 0.0)
        assert bool(close(task, R, want, mag, K).all()), (M, N, K)
    assert left > 0


@pytest.mark.parametrize("tA,tB", [(False, False), (True, True)])
@pytest.mark.parametrize("what", ["thresholds", "tiny", "large", "late", "not numbers", "limits"])
@pytest.mark.parametrize("task,form", [("count_gt", "col"), ("count_gt", "row"), ("boost", "col"), ("boost", "row")])
def test_values_of_the_plain_way(am, task, form, what, tA, tB):
    if (task, what) == ("count_gt", "not numbers"):
        pytest.skip("a count of products that are no numbers is not specified")
    inf = float("inf")
    for M, N, K in [(4093, 2046, 75), (4097, 2048, 264)]:
        A, B, th = make(K, M, N, K, form, tA, tB)
        a, b = (A.T if tA else A), (B.T if tB else B)
        if what == "thresholds":
            th[:8] = torch.tensor([0.0, -0.0, -1.5, 1e-200, 1e200, inf, -inf, 5e-324], dtype=torch.float64, device="cuda")
            th[300], th[1000], th[1500] = float("nan"), inf, -0.5
        elif what == "tiny":
            b[K // 2, 5::7] = 2.0 ** -1000
            b[K // 2, 6::7] = -5e-324
            b[3, 1::9] = 0.0
            a[::5, 4] *= 1e-200
        elif what == "large":
            b[1, 40] = -1e200
            a[9, :K // 2] *= 1e100
            b[2, 700] = 1e308
        elif what == "late":
            b[K - 1, ::2] = 1e-300
            b[min(K - 1, 200), 1000] = 1e50
        elif what == "limits":
            lo, hi = (-400, 100) if task == "boost" else (-600, 100)
            for i, v in enumerate([2.0 ** hi, 2.0 ** hi * (1 - 2.0 ** -53), 2.0 ** hi * 1.5, 2.0 ** lo, 2.0 ** lo * (1 - 2.0 ** -53)]):
                b[i, 130 * i + 2], b[K - 1 - i, 130 * i + 40] = v, -v
            th[:6] = torch.tensor([2.0 ** 100, 2.0 ** 100 * (1 + 2.0 ** -52), 2.0 ** -100, 2.0 ** -101, -(2.0 ** 100), -(2.0 ** -100)], dtype=torch.float64, device="cuda")
        else:
            a[3, 4], a[5, 6], b[7, 8], b[9, 10] = inf, float("nan"), float("nan"), -inf
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        assert "critical" in " ".join(run(am, task, A, B, th, R, form, tA, tB))
        want, mag = reference(task, A, B, th, form, 0.0, tA, tB)
        ok = close(task, R, want, mag, K)
        assert bool(ok.all()), (what, M, N, K, (~ok).nonzero()[:4])


@pytest.mark.parametrize("task", ["discount", "boost"])
@pytest.mark.parametrize("M,N,K", [(4096, 2048, 256), (4096, 2048, 2048), (4096, 2048, 8192)])
def test_sums_are_added_up_in_parts(am, task, M, N, K):
    """No more error than four sums of a quarter of K each: the n roundings of a growing sum are, as independent ones of up to
    2^-54 of it (uniform: 1 / sqrt 3 of that), sqrt(n) / 3 of 2^-53 of it together, and four of a quarter half of that."""
    import numpy as np
    g = torch.Generator(device="cuda").manual_seed(K)

    def uniform(lo, hi, *shape):
        return torch.empty(*shape, dtype=torch.float64, device="cuda").uniform_(lo, hi, generator=g)
    A, B, th, dis = uniform(0, 10, M, K), uniform(1, 100, K, N), uniform(100, 500, N), uniform(0.05, 0.3, N)
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    am.amulet_mmlike_f64(getattr(am, "AMULET_" + task.upper()), A, B, th, dis if task == "discount" else None, R)
    assert "critical_rows" in am.amulet_recent_kernel(0)

    def long(x):
        return x.cpu().numpy().astype(np.longdouble)
    rows, b, t, d = [0, 77, 1999, M - 1], long(B[:, ::8]), long(th[::8]), long(1.0 - dis[::8])
    if np.finfo(np.longdouble).nmant <= 52:
        pytest.skip("no wider type to compare with")
    error = []
    for i, got in zip(rows, long(R[rows][:, ::8])):
        p = long(A[i])[:, None] * b
        term = p + np.maximum(p - t, 0) if task == "boost" else np.where(p.astype(np.float64) > t, p * d, p)
        error.append((got - term.sum(0)) / term.sum(0))
    assert np.sqrt(np.mean(np.square(error))) * 2.0 ** 53 <= np.sqrt(K / 4) / 6 + 1


def test_a_count_of_every_k(am):
    """Every product over its threshold, more of them than 16 bits hold."""
    M, N, K = 4096, 2048, 70000
    A = torch.full((M, K), 2.0, dtype=torch.float64, device="cuda")
    B = torch.where(torch.arange(N, device="cuda") % 2 == 0, 3.0, -3.0).double().repeat(K, 1)
    A[::3] = -2.0
    th = torch.tensor([5.999999999999999], dtype=torch.float64, device="cuda")
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    assert "critical" in " ".join(run(am, "count_gt", A, B, th, R, "const"))
    assert torch.equal(R, torch.where((A[:, :1] > 0) == (B[:1] > 0), float(K), 0.0).double())
