"""GPU parity of fp64 DISCOUNT by critical values: products at the threshold, remainders of tiles and of K, forms and layouts,
rows left to the tile kernels, and the values that send a tile to the task's own operations."""
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


def run(am, A, B, th, dis, R, tA=False, tB=False):
    """The kernels it was, the last one first."""
    form = am.AMULET_THRES_CONST if th.numel() == 1 and R.shape[1] > 1 else am.AMULET_THRES_COL
    am.amulet_mmlike_f64(am.AMULET_DISCOUNT, A, B, th, dis, R, thres_form=form, trans_a=tA, trans_b=tB)
    kernels = [am.amulet_recent_kernel(0), am.amulet_recent_kernel(1)]
    torch.cuda.synchronize()
    return kernels


def reference(A, B, th, dis, R0, tA=False, tB=False):
    """Sum and sum of magnitudes, product by product in 64 bits."""
    a, b = (A.T if tA else A), (B.T if tB else B)
    want, mag = torch.full((a.shape[0], b.shape[1]), R0, dtype=torch.float64, device="cuda"), 0.0
    for k in range(a.shape[1]):
        p = a[:, k, None] * b[k]
        term = torch.where(p > th, p * (1.0 - dis), p)
        want += term
        mag = mag + term.abs()
    return want, mag


def make(seed, M, N, K, tA=False, tB=False, pad=0, const=False):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(r, c):
        return torch.empty(r, c + pad, dtype=torch.float64, device="cuda").normal_(generator=g)[:, :c]
    A, B = normal(*((K, M) if tA else (M, K))), normal(*((N, K) if tB else (K, N)))
    th = torch.empty(1 if const else N, dtype=torch.float64, device="cuda").uniform_(0.05, 2, generator=g)
    return A, B, th, torch.empty(N, dtype=torch.float64, device="cuda").uniform_(0, 1, generator=g)


# (rows of the tile, M, N, K): each the plan at its size
@pytest.mark.parametrize("rows,M,N,K", [(64, 3072, 2048, 64), (128, 2048, 2048, 256)])
@pytest.mark.parametrize("sign", [1, -1])
def test_products_at_the_threshold(am, rows, M, N, K, sign):
    """One product per sum, thresholds one ulp below, at and above some of them, nothing left of what is over: every decision shows."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    for bits in (53, 27, 14):       # 27: products of 53 and 54 bits, ties among them; 14: exact products
        def value(n):
            v = torch.empty(n, dtype=torch.float64, device="cuda").uniform_(1, 2, generator=g)
            return torch.round(v * 2.0 ** (bits - 1)) * 2.0 ** (1 - bits) * 2.0 ** torch.randint(-3, 12, (n,), generator=g, device="cuda").double()
        a, b = sign * value(M), sign * value(N)
        A, B = torch.zeros(M, K, dtype=torch.float64, device="cuda"), torch.zeros(K, N, dtype=torch.float64, device="cuda")
        k = K - 3
        A[:, k], B[k] = a, b
        th = a[torch.arange(N, device="cuda") % M] * b
        step = torch.arange(N, device="cuda") % 3
        th = torch.where(step == 0, th, torch.nextafter(th, (step == 1).double() * 1e9))
        dis = torch.ones(N, dtype=torch.float64, device="cuda")
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        assert "critical_rows %d" % rows in run(am, A, B, th, dis, R)[0]
        p = a[:, None] * b
        assert torch.equal(R, torch.where(p > th, 0.0, p)), (bits, sign)


@pytest.mark.parametrize("rows,M,N,K", [(64, 3072, 2048, 64), (128, 2048, 2048, 256)])
@pytest.mark.parametrize("rest", [(1.0, 0.7, 0.5, 0.0), (0.3,), (0.3, 0.1, 1e-2, 1e-4), (1e-6, 1e-9, 1e-12, 2.0 ** -52), (1.5, 3.0, -0.25, -5.0)])
def test_error_of_a_term(am, rest, rows, M, N, K):
    """One product per sum, discounts that leave `rest` of what is over: two roundings if it is, one if it is not, whatever is left."""
    import numpy as np
    g = torch.Generator(device="cuda").manual_seed(K)

    def value(n):
        v = torch.empty(n, dtype=torch.float64, device="cuda").uniform_(1, 8, generator=g)
        return v * (torch.randint(0, 2, (n,), generator=g, device="cuda") * 2 - 1)
    a, b = value(M), value(N)
    A, B = torch.zeros(M, K, dtype=torch.float64, device="cuda"), torch.zeros(K, N, dtype=torch.float64, device="cuda")
    A[:, K - 3], B[K - 3] = a, b
    th = torch.empty(N, dtype=torch.float64, device="cuda").uniform_(0.5, 20, generator=g)
    dis = 1.0 - torch.tensor(rest, dtype=torch.float64, device="cuda").repeat(N)[:N]
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    assert "critical_rows %d" % rows in run(am, A, B, th, dis, R)[0]
    if np.finfo(np.longdouble).nmant <= 52:
        pytest.skip("no wider type to compare with")
    long = [x.cpu().numpy().astype(np.longdouble) for x in (a, b, 1.0 - dis)]
    over = (a[:, None] * b > th).cpu().numpy()
    want = long[0][:, None] * long[1] * np.where(over, long[2], 1.0)
    error = np.abs(R.cpu().numpy() - want)
    assert (error <= 2.0 ** -53 * np.where(over, 2, 1) * np.abs(want) * (1 + 2.0 ** -9)).all(), rest


@pytest.mark.parametrize("M,N,K", [(3072, 2048, 64), (2048, 2048, 2048)])
@pytest.mark.parametrize("left", [1e-3, 1e-6, 2.0 ** -52])
def test_error_where_everything_is_over(am, left, M, N, K):
    A, B, th, dis = make(K, M, N, K)
    A, B, th, dis = A.abs() + 0.5, B.abs() + 0.5, th * 0.1, torch.full_like(dis, 1.0 - left)
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    assert "critical_rows" in run(am, A, B, th, dis, R)[0]
    want, mag = reference(A, B, th, dis, 0.0)
    # K sums, and a product's two roundings, here and in the reference
    assert bool(((R - want).abs() <= 2.0 ** -53 * (2 * K + 4) * mag).all())


def test_products_past_the_largest_number(am):
    """Infinite before the discount is taken off."""
    for M, N, K in [(3072, 2048, 64), (2048, 2048, 256)]:
        A, B, th, dis = make(K, M, N, K)
        A[7, 9], A[2040, K - 1], A[5, 5] = 1.5e308, -1.7e308, 2.0 ** 900
        B[9], B[K - 1], B[5] = B[9] * 3 + torch.sign(B[9]), B[K - 1] * 5 + torch.sign(B[K - 1]), 2.0 ** 99
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        assert "critical_rows" in run(am, A, B, th, dis, R)[0]
        want, mag = reference(A, B, th, dis, 0.0)
        big = ~torch.isfinite(want)
        assert int(big.sum()) > N and bool((R == want)[big].all())
        assert bool(((R - want).abs() <= 2.0 ** -53 * (2 * K + 4) * mag)[~big].all())


SIZES = [(3072, 2048, 64, 0), (2048, 2048, 256, 0), (3071, 2047, 67, 1), (2049, 2045, 263, 3), (4481, 1025, 79, 0), (1985, 2050, 271, 1)]


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("const", [False, True])
def test_remainders_forms_and_layouts(am, const, tA, tB):
    ran = []
    for M, N, K, pad in SIZES:
        A, B, th, dis = make(M + N + K, M, N, K, tA, tB, pad, const)
        whole = torch.full((M, N + pad), 0.25, dtype=torch.float64, device="cuda")
        R = whole[:, :N]
        print("critical f64", M, N, K, tA, tB, flush=True)
        ran.append(" ".join(run(am, A, B, th, dis, R, tA, tB)))
        want, mag = reference(A, B, th, dis, 0.25, tA, tB)
        # K sums, a product's two roundings and those of 1 - dis and of the value that a product over the threshold is formed with
        assert bool(((R - want).abs() <= 2.0 ** -53 * ((K + 5) * mag + 2 * want.abs())).all()), (M, N, K)
        assert bool((whole[:, N:] == 0.25).all())
    assert any("critical_rows 64" in r for r in ran) and any("critical_rows 128" in r for r in ran), ran


@pytest.mark.parametrize("M,N,K", [(2560, 1751, 1792), (5120, 1751, 1300)])
def test_rows_left_to_the_tile_kernels(am, M, N, K):
    A, B, th, dis = make(M, M, N, K)
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    kernels = run(am, A, B, th, dis, R)
    assert "critical" not in kernels[0] and "critical_rows" in kernels[1], kernels
    want, mag = reference(A, B, th, dis, 0.0)
    assert bool(((R - want).abs() <= 2.0 ** -53 * (K + 7) * mag).all())
    again = torch.zeros_like(R)
    run(am, A, B, th, dis, again)
    assert torch.equal(R, again)       # (K in one part: the same bits every time)


@pytest.mark.parametrize("tA,tB", [(False, False), (True, True)])
@pytest.mark.parametrize("what", ["thresholds", "tiny b", "large", "discounts", "late", "not numbers", "limits", "always and never"])
def test_values_of_the_plain_way(am, what, tA, tB):
    for M, N, K in [(3071, 2046, 75), (2047, 2048, 259)]:
        A, B, th, dis = make(K, M, N, K, tA, tB)
        a, b = (A.T if tA else A), (B.T if tB else B)
        if what == "thresholds":
            th[:8] = torch.tensor([0.0, -0.0, -1.5, 1e-200, 1e200, float("inf"), float("-inf"), 5e-324], dtype=torch.float64, device="cuda")
            th[300], th[1000] = float("nan"), float("inf")
        elif what == "always and never":
            top = 1.7976931348623157e308
            th[:10] = torch.tensor([float("inf"), float("-inf"), top, -top, 2.0 ** 1000, -(2.0 ** 1000), 0.0, -1.0, 1.0, -0.0], dtype=torch.float64, device="cuda")
            th[200:205], th[1000:], b[4, ::3], b[7] = -top, float("-inf"), 0.0, 2.0 ** 99
            a[40, 7], a[41, 7] = 2.0 ** 899, -(2.0 ** 899)
        elif what == "tiny b":
            b[K // 2, 5::7] = 2.0 ** -1000
            b[K // 2, 6::7] = -5e-324
            b[3, 1::9] = 0.0
            a[::5] *= 2.0 ** 900
        elif what == "large":
            b[1, 40] = -1e200
            a[9] *= 1e100
            b[2, 700] = 1e308
        elif what == "discounts":
            dis[5], dis[6], dis[400], dis[900] = 1.5, -0.5, 1.0, 0.0
        elif what == "late":
            b[K - 1, ::2] = 1e-300
            b[min(K - 1, 200), 1000] = 1e50
        elif what == "limits":
            lo, hi = -600, 100
            for i, v in enumerate([2.0 ** hi, 2.0 ** hi * (1 - 2.0 ** -53), 2.0 ** hi * 1.5, 2.0 ** lo, 2.0 ** lo * (1 - 2.0 ** -53)]):
                b[i, 130 * i + 2], b[K - 1 - i, 130 * i + 40] = v, -v
            th[:6] = torch.tensor([2.0 ** 100, 2.0 ** 100 * (1 + 2.0 ** -52), 2.0 ** -100, 2.0 ** -101, -(2.0 ** 100), -(2.0 ** -100)], dtype=torch.float64, device="cuda")
        else:
            a[3, 4], a[5, 6], b[7, 8], b[9, 10] = float("inf"), float("nan"), float("nan"), float("-inf")
        R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        assert "critical" in run(am, A, B, th, dis, R, tA, tB)[0]
        want, mag = reference(A, B, th, dis, 0.0, tA, tB)
        ok = (R - want).abs() <= 2.0 ** -53 * (K + 7) * mag
        both = ~torch.isfinite(want)
        ok |= both & (torch.isnan(R) == torch.isnan(want)) & (torch.isnan(want) | (R == want))
        assert bool(ok.all()), (what, M, N, K, (~ok).nonzero()[:4])
