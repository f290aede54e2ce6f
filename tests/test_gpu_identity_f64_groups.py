"""GPU parity of the fp64 identity task where groups of waves share a tile's K: bit for bit on whole numbers, with stages that the
groups share unevenly, remainders of K and of tiles, all layouts."""
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


# one tile of 64 x 64 to a compute unit: two groups from 256 k on, four from 1024 on; two whole ones to a unit: two from 512 on
@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K", [(1024, 1024, 256), (1001, 1023, 263), (1024, 1000, 1024), (1015, 1024, 1055), (961, 961, 1037),
                                   (2048, 1024, 520), (1985, 1023, 535), (768, 768, 768), (769, 700, 1799)])
def test_whole_numbers(am, M, N, K, tA, tB):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)

    def whole(*shape):
        return torch.randint(-9, 10, shape, generator=g, device="cuda").double()
    A, B = whole(*((K, M) if tA else (M, K))), whole(*((N, K) if tB else (K, N)))
    R = torch.full((M, N + 3), 7.0, dtype=torch.float64, device="cuda")
    print("identity f64", M, N, K, tA, tB, flush=True)
    am.amulet_mmlike_f64(am.AMULET_IDENTITY, A, B, None, None, R[:, :N], trans_a=tA, trans_b=tB)
    want = (A.T if tA else A).cpu() @ (B.T if tB else B).cpu() + 7.0
    assert torch.equal(R[:, :N].cpu(), want)
    assert bool((R[:, N:] == 7.0).all())
