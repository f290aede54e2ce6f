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


# one tile of 64 x 64 to a compute unit: two groups from 256 k on, four from 1024 on; two whole ones to a unit: two from 512 on; ranges of K
# over several workgroups, the last one short; and one group where a rule stops
SIZES = [(2, 1024, 1024, 256), (2, 1001, 1023, 263), (4, 1024, 1000, 1024), (4, 1015, 1024, 1055), (4, 961, 961, 1037),
         (2, 2048, 1024, 520), (2, 1985, 1023, 535), (2, 512, 512, 2048), (2, 500, 512, 1040), (2, 320, 300, 2060), (2, 128, 128, 8199),
         (1, 768, 768, 768), (1, 769, 700, 1799), (1, 1024, 1024, 255), (1, 2048, 1024, 511)]


def run(am, groups, A, B, R, tA, tB):
    print("identity f64", groups, R.shape, tA, tB, flush=True)
    groups = 1 if groups == 2 and tB and not tA else groups       # (both operands stored along k)
    am.amulet_mmlike_f64(am.AMULET_IDENTITY, A, B, None, None, R, trans_a=tA, trans_b=tB)
    kernel = am.amulet_recent_kernel()
    torch.cuda.synchronize()
    assert kernel.startswith("mfma_f64_64x64_dma4 ") and (" k_groups %d" % groups in kernel if groups > 1 else "k_groups" not in kernel), kernel


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("groups,M,N,K", SIZES)
def test_whole_numbers(am, groups, M, N, K, tA, tB):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)

    def whole(*shape):
        return torch.randint(-9, 10, shape, generator=g, device="cuda").double()
    A, B = whole(*((K, M) if tA else (M, K))), whole(*((N, K) if tB else (K, N)))
    R = torch.full((M, N + 3), 7.0, dtype=torch.float64, device="cuda")
    run(am, groups, A, B, R[:, :N], tA, tB)
    want = (A.T if tA else A).cpu() @ (B.T if tB else B).cpu() + 7.0
    assert torch.equal(R[:, :N].cpu(), want)
    assert bool((R[:, N:] == 7.0).all())


@pytest.mark.parametrize("groups,M,N,K", SIZES)
def test_error(am, groups, M, N, K):
    import numpy as np
    if np.finfo(np.longdouble).nmant <= 52:
        pytest.skip("no wider type to compare with")
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, B = (torch.empty(*s, dtype=torch.float64, device="cuda").uniform_(-1, 1, generator=g) for s in ((M, K), (K, N)))
    R = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    run(am, groups, A, B, R, False, False)
    a, b = (x.cpu().numpy().astype(np.longdouble) for x in (A[::97], B[:, ::53]))
    # (each of K sums rounds to 2^-53 of the magnitudes at most, in whatever order)
    assert (np.abs(R[::97, ::53].cpu().numpy() - a @ b) <= K * 2.0 ** -53 * (np.abs(a) @ np.abs(b))).all()
