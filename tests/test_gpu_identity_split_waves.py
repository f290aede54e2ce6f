"""GPU parity of the fp32 identity task from bf16 pieces where the waves of a workgroup share K: remainders of tiles, of K and of its
parts, layouts, pitches, and values that the pieces do not carry."""
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


def make(seed, M, N, K, tA, tB, pad=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.empty(r, c + pad, device="cuda").uniform_(-1, 1, generator=g)[:, :c] for r, c in ((K, M) if tA else (M, K), (N, K) if tB else (K, N))]


def run(am, A, B, R, tA, tB):
    am.amulet_mmlike_f32_general(am.AMULET_IDENTITY, A, B, None, None, R, trans_a=tA, trans_b=tB)
    kernel = am.amulet_recent_kernel()
    torch.cuda.synchronize()
    return "tile_rows 64" in kernel


# one round and more; a wave's part of K whole, short, of a few k, or nothing; one past and one to three short of a tile; odd pitches
SIZES = [(1024, 1024, 1024, 0), (1015, 1021, 1009, 15), (961, 1023, 1040, 1), (1021, 1019, 2033, 15), (3844, 197, 2100, 12), (65, 7681, 1153, 15)]


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
def test_remainders_and_layouts(am, tA, tB):
    ran = 0
    for M, N, K, pad in SIZES:
        A, B = make(M + K, M, N, K, tA, tB, pad)
        whole = torch.full((M, N + pad), 0.25, device="cuda")
        R = whole[:, :N]
        print("identity waves", M, N, K, pad, tA, tB, flush=True)
        ran += run(am, A, B, R, tA, tB)
        a, b = (A.T if tA else A).double().cpu(), (B.T if tB else B).double().cpu()
        want, mag = a @ b + 0.25, a.abs() @ b.abs()
        # an eighth of K in steps of 16 that round once each, seven sums of those, R's own rounding
        assert bool(((R.double().cpu() - want).abs() <= 2.0 ** -24 * ((K / 128 + 12) * mag + 2 * want.abs())).all()), (M, N, K)
        assert bool((whole[:, N:] == 0.25).all())
    assert ran >= 3


@pytest.mark.parametrize("tA,tB", [(False, False), (True, True)])
@pytest.mark.parametrize("what", ["tiny", "tiny in one part", "infinite", "rounds to infinite", "integers"])
def test_values_the_pieces_do_not_carry(am, what, tA, tB):
    M, N, K = 1023, 1021, 1019
    A, B = make(5, M, N, K, tA, tB)
    a, b = (A.T if tA else A), (B.T if tB else B)
    if what == "tiny":
        A *= 2.0 ** -70
        B *= 2.0 ** -50
        a[7] *= 2.0 ** -60
    elif what == "tiny in one part":
        a[100, 900] = 2.0 ** -140 * 1.2345
        b[900, 3] = 2.0 ** 100
    elif what == "infinite":
        a[3, 5], b[700, 9], b[1018, 1020] = float("inf"), float("nan"), float("-inf")
    elif what == "rounds to infinite":
        a[3, 5] = 3.4e38
        b[5] *= 2.0 ** -20
    else:
        A.copy_(torch.round(A * 2047))
        B.copy_(torch.round(B * 2047))
    R = torch.zeros(M, N, device="cuda")
    assert run(am, A, B, R, tA, tB)
    got, x, y = R.double().cpu(), a.double().cpu(), b.double().cpu()
    want, mag = x @ y, x.abs() @ y.abs()
    if what == "integers":       # |sums| below 2^33: exact in each piece product, rounded where they pass 2^24
        assert bool(((got - want).abs() <= 2.0 ** -24 * 12 * mag).all())
        return
    fine = torch.isfinite(want)
    # (the fp32 instruction rounds every product: K / 8 of a part more)
    assert bool(((got - want).abs() <= 2.0 ** -24 * (K / 8 + 16) * mag + 2.0 ** -140)[fine].all())
    assert bool((torch.isnan(got) == torch.isnan(want)).all()) and bool((got == want)[~fine & ~torch.isnan(want)].all())
