"""GPU parity of the join count's tile of 192 x 256 (rows at any byte address, through registers), where one wave in three
has a load more than the others and the image's pieces do not divide over the waves: one row, column or k past
and short of a tile and a stage, both layouts of B, R written and added to."""
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


@pytest.mark.parametrize("M,N,K", [(11 * 192 + 1, 20 * 256 + 1, 11 * 64 + 1), (11 * 192 - 1, 21 * 256 - 1, 12 * 64 - 1),
                                   (7 * 192, 27 * 256 + 129, 48 * 64 + 31), (16 * 192 - 73, 15 * 256 + 161, 39 * 64 + 7)])
def test_edges(am, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M)

    def draw(r, c):      # rows at odd addresses
        return torch.randint(-128, 128, (r, c | 1), device="cuda", generator=g, dtype=torch.int16).to(torch.int8)[:, :c]
    for tB in (False, True):
        A, B = draw(M, K), draw(N, K) if tB else draw(K, N)
        b = (B.t() if tB else B).double().contiguous()
        want = (A.double() @ b).to(torch.int32)
        R = torch.full((M, N), 7, device="cuda", dtype=torch.int32)
        ws = torch.empty(am.amulet_count_i8_repack_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
        am.amulet_count_i8_general(A, B, R, ws, trans_a=False, trans_b=tB)
        assert am.amulet_recent_kernel().startswith("i8_tile_192x256_registers "), am.amulet_recent_kernel()
        assert torch.equal(R, want + 7)
    A, B = draw(M, K), draw(K, N)
    R = torch.full((M, N), 7, device="cuda", dtype=torch.int32)
    am.amulet_count_i8_assign(A, B, R)
    assert am.amulet_recent_kernel().startswith("i8_tile_192x256_registers "), am.amulet_recent_kernel()
    assert torch.equal(R, (A.double() @ B.double().contiguous()).to(torch.int32))
