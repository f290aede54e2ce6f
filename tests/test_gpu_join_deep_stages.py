"""The join count's smaller tiles with stages of 128 k: less than a ring of them, ranges with a short last stage of
one to four k-steps, K over several workgroups, ragged rows and columns, every layout; exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,split,M,N,K", [
    ("i8_tile_64x64", False, 1020, 960, 768),         # three stages to a group of waves
    ("i8_tile_64x64", False, 1020, 1024, 3328),       # whole stages, ragged rows
    ("i8_tile_64x64", False, 640, 1156, 4228),        # the second group's last stage has 4 k
    ("i8_tile_64x64", True, 132, 1000, 8068),         # parts; the last one's groups end in 128 and 4 k
    ("i8_tile_64x64", False, 1024, 960, 3520),        # rows of an odd number of 64 bytes
    ("i8_tile_128x128", False, 2412, 896, 4184),      # a last stage of 88 k
    ("i8_tile_128x128", False, 448, 5012, 5040),      # ... of 48
    ("i8_tile_128x128", True, 260, 2052, 8068),
    ("i8_tile_128x128", False, 300, 7000, 3520),      # a last stage of 64: not with A transposed
    ("i8_tile_128x128", False, 1500, 1500, 5040),     # rows of neither operand whole parts of lines
])
def test_stages_of_128_k(kernel, split, M, N, K):
    import paper_2305_08872_amd as am
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randint(-3, 4, (M, K), generator=g, device="cuda", dtype=torch.int8)
    B = torch.randint(-3, 4, (K, N), generator=g, device="cuda", dtype=torch.int8)
    want = (A.float() @ B.float()).to(torch.int32)    # |sum| < 2^24: exact
    am.amulet_clear_selections()
    for tA, tB in [(False, False), (True, False), (False, True), (True, True)]:
        print(kernel, split, tA, tB, M, N, K, flush=True)
        sA, sB = A.t().contiguous() if tA else A, B.t().contiguous() if tB else B
        R = torch.full((M, N), 11, dtype=torch.int32, device="cuda")
        ws = torch.empty(am.amulet_count_i8_workspace_bytes(tA, tB, M, N, K) + 16, dtype=torch.int8, device="cuda")
        am.amulet_count_i8_general(sA, sB, R, ws, trans_a=tA, trans_b=tB)
        torch.cuda.synchronize()
        ran = am.amulet_recent_kernel().split()
        # (the 64 x 64 tile keeps stages of 64 k for operands across k, and of such rows where either lies so; the 128 x 128 tile of such rows with A
        # across k, and for operands across k whose rows are not multiples of 64 bytes apart, where the last stage is short)
        if kernel == "i8_tile_128x128":
            deep = not tA if K % 128 == 64 else not tA or tB or K % 128 == 0 or M % 64 == 0 or N % 64 == 0
        else:
            deep = (not tA and tB) if K % 128 == 64 else (not tA or tB)
        assert ran[0] == kernel and (ran[-2:] == ["stage_k", "128"]) == deep and (int(ran[4]) > 1) == split, ran
        assert torch.equal(R, want + 11), (tA, tB)
    am.amulet_count_i8_assign(A, B, R)
    torch.cuda.synchronize()
    assert torch.equal(R, want)


def test_stages_of_128_k_of_padded_rows():
    """Operands and R with pitches of their own, an odd number of 64 bytes where K is not and the other way round; every layout."""
    import paper_2305_08872_amd as am
    M, N = 640, 1156
    am.amulet_clear_selections()
    for K, pad in [(4096, 64), (3520, 64), (4228, 28)]:
        g = torch.Generator(device="cuda").manual_seed(K)
        A = torch.randint(-3, 4, (M, K), generator=g, device="cuda", dtype=torch.int8)
        B = torch.randint(-3, 4, (K, N), generator=g, device="cuda", dtype=torch.int8)
        want = (A.float() @ B.float()).to(torch.int32)    # |sum| < 2^24: exact
        for tA, tB in [(False, False), (True, False), (False, True), (True, True)]:
            print(tA, tB, M, N, K, pad, flush=True)
            sA, sB = A.t() if tA else A, B.t() if tB else B
            pA, pB = torch.full((sA.shape[0], sA.shape[1] + pad), 99, dtype=torch.int8, device="cuda"), torch.full((sB.shape[0], sB.shape[1] + pad), 99, dtype=torch.int8, device="cuda")
            pA[:, :sA.shape[1]] = sA
            pB[:, :sB.shape[1]] = sB
            R = torch.full((M, N + 4), 11, dtype=torch.int32, device="cuda")
            ws = torch.empty(am.amulet_count_i8_workspace_bytes(tA, tB, M, N, K) + 16, dtype=torch.int8, device="cuda")
            am.amulet_count_i8_general(pA[:, :sA.shape[1]], pB[:, :sB.shape[1]], R[:, :N], ws, trans_a=tA, trans_b=tB)
            torch.cuda.synchronize()
            assert am.amulet_recent_kernel().startswith("i8_tile_64x64 ")
            assert torch.equal(R[:, :N], want + 11) and (R[:, N:] == 11).all(), (tA, tB)
