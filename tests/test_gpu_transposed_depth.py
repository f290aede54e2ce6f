"""GPU parity of the discount's wide kernel with A transposed, whose stage is 32 k deep: every remainder of K class, K shorter
than a stage and in parts, rows and columns beside the tile's, all threshold forms."""
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


@pytest.mark.parametrize("tB", [False, True])
@pytest.mark.parametrize("form", FORMS)
def test_remainders(am, form, tB):
    shape = next(i for i in range(am.amulet_shape_count(am.AMULET_DISCOUNT))
                 if am.amulet_shape_name(am.AMULET_DISCOUNT, i) == "valu_32x256_w8_k16")
    for M, N, K in [(64, 256, 64), (33, 257, 31), (31, 255, 65), (65, 300, 95), (96, 512, 1), (40, 260, 33), (300, 700, 1003)]:
        g = torch.Generator(device="cuda").manual_seed(M + K)
        A = torch.randint(0, 10, (M, K), device="cuda", generator=g).float()
        B = torch.empty(K, N, device="cuda").uniform_(1, 100, generator=g)
        th = torch.empty(*{"col": (N,), "row": (M,), "const": (1,), "elem": (M, N)}[form], device="cuda").uniform_(100, 500, generator=g)
        dis = torch.empty(N, device="cuda").uniform_(0.05, 0.3, generator=g)
        R = torch.full((M, N), 0.5, device="cuda")
        am.amulet_mmlike_f32_general(am.AMULET_DISCOUNT, A.t().contiguous(), B.t().contiguous() if tB else B, th, dis, R,
                                     thres_form=FORMS.index(form), trans_a=True, trans_b=tB, shape=shape)
        t = {"col": lambda: th[None, :], "row": lambda: th[:, None], "const": lambda: th[0], "elem": lambda: th}[form]()
        want = torch.full((M, N), 0.5, device="cuda", dtype=torch.float64)
        for k in range(K):
            p = A[:, k:k + 1] * B[k:k + 1]
            want += torch.where(p > t, p.double() * (1 - dis).double()[None, :], p.double())
        # partial sums over 64 k of terms of one sign: 64 + K / 64 roundings, one per part, and one of 1 - dis
        assert bool(((R - want).abs() <= (66 + K / 64 + 16) * 2.0 ** -24 * want).all()), (form, tB, M, N, K)
