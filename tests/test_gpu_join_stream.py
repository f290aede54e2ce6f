"""R += of the join count by the kernel that reads R during its K loop (count_i8_stream.hip): every count of R, from an R that
holds other values and has a pitch of its own, at the least K it takes and at K whose groups of stages are uneven, with tiles that
do and do not divide over the workgroups."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("named,M,N,K,pad,ran", [      # (named: by the shape's id; else as the library chooses)
    (False, 4096, 8192, 3392, 0, ("4", "1")),       # two tiles to a workgroup, three stages to each group of four of R's values
    (True, 4096, 8192, 3328, 0, ("8", "1")),        # a stage too few: groups of eight
    (True, 4096, 4096, 1856, 4, ("8", "0")),        # one tile to a workgroup, three stages to each group of eight
    (True, 4096, 8192, 1792, 0, (None, None)),      # a stage too few: the kernel with its own write-back of R
    (False, 8192, 4096, 1856, 8, ("8", "0")),       # R written through the caches, its stores under way behind the next tile's stages
    (False, 4352, 8192, 3456, 8, ("4", "0")),       # ... places without a tile, a last round of few tiles
    (False, 8192, 4864, 4160, 4, ("4", "1")),       # groups of 3 and 4 stages
])
def test_count_i8_r_read_during_the_k_loop(named, M, N, K, pad, ran):
    import paper_2305_08872_amd as am
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    A = torch.randint(-128, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    B = torch.randint(-128, 128, (K, N), generator=g, device="cuda", dtype=torch.int8)
    held = torch.randint(-2 ** 31, 2 ** 31 - 1, (M, N + pad), generator=g, device="cuda", dtype=torch.int32)
    # (whole numbers below 2^53 throughout: exact in 64 bits)
    product = A.double() @ B.double()
    for _ in range(2):           # (the second call finds the first one's counts)
        want = held.long()
        want[:, :N] += product.long()
        want = ((want + 2 ** 31) % 2 ** 32 - 2 ** 31).int()
        print("join stream", M, N, K, pad, flush=True)
        if named:
            am.amulet_count_i8_shape(8, A, B, held[:, :N])
        else:
            am.amulet_clear_selections()
            am.amulet_count_i8(A, B, held[:, :N])
        torch.cuda.synchronize()
        words = am.amulet_recent_kernel().split()
        fields = dict(zip(words[1::2], words[2::2]))
        assert words[0] == "mfma_i8_256x256_w16_dma4_persistent" and "workgroups" in fields, words
        assert (fields.get("r_in_k_loop"), fields.get("r_bypass")) == ran, words
        assert torch.equal(held, want)
