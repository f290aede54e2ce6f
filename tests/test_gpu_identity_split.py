"""GPU parity of the identity task's bf16-piece kernel (problems that fill the chip): tile and K remainders, the four
layouts, pitches that leave rows unaligned, and the values its pieces do not carry."""
import numpy as np
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


def operand(g, rows, cols, pad, scale=None):
    """A rows x cols view into rows cols + pad apart, uniform in -1 .. 1."""
    x = torch.empty(rows, cols + pad, device="cuda").uniform_(-1, 1, generator=g)
    return x[:, :cols]


def run(am, A, B, R, tA, tB):
    am.amulet_mmlike_f32_general(am.AMULET_IDENTITY, A, B, None, None, R, trans_a=tA, trans_b=tB)
    kernel = am.amulet_recent_kernel().split()
    torch.cuda.synchronize()
    assert "bf16_pieces" in kernel, kernel
    return int(kernel[kernel.index("tile_rows") + 1])


def exact(A, B, tA, tB):
    a, b = (A.T if tA else A).double().contiguous(), (B.T if tB else B).double().contiguous()
    return a @ b, a.abs() @ b.abs()


# the least K the kernel is chosen for, one stage's remainders, an odd K; both tile heights; edges by one line and by less than a block
SIZES = [(2048, 2048, 96, 0, 128), (2047, 1921, 111, 3, 128), (1985, 1985, 257, 1, 128), (1985, 2047, 112, 2, 128),
         (4096, 4096, 96, 0, 256), (3841, 4095, 97, 1, 256), (4095, 4001, 113, 5, 256)]


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K,pad,tile_rows", SIZES)
def test_remainders_and_layouts(am, M, N, K, pad, tile_rows, tA, tB):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = operand(g, *((K, M) if tA else (M, K)), pad)
    B = operand(g, *((N, K) if tB else (K, N)), pad)
    R = torch.full((M, N + pad), 0.5, device="cuda")[:, :N]
    print("identity pieces", M, N, K, pad, tA, tB, flush=True)
    assert run(am, A, B, R, tA, tB) == tile_rows
    ref, ab = exact(A, B, tA, tB)
    # fp32 accumulators over K: the library's own bound is 1e-5 of the sum of magnitudes; here K <= 257, at most 6 roundings per
    # 16 k of at most half an ulp of a partial sum
    err = (R.double() - (ref + 0.5)).abs() - 2.0 ** -23 * (ref + 0.5).abs()
    assert float((err / ab).max()) <= 6 * (K / 16 + 1) * 2.0 ** -24
    # nothing outside R, and R += twice
    if pad:
        full = R._base if R._base is not None else R
        assert torch.equal(full[:, N:], torch.full_like(full[:, N:], 0.5))
    assert run(am, A, B, R, tA, tB) == tile_rows
    assert float(((R.double() - (2 * ref + 0.5)).abs() / (ab + 1)).max()) <= 1e-5


@pytest.mark.parametrize("M,N,K", [(2048, 2048, 1000), (4096, 4096, 1000)])
def test_no_less_precise_than_the_fp32_matrix_instruction(am, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(5)
    for low in (-1.0, 0.0):
        A = torch.empty(M, K, device="cuda").uniform_(low, 1, generator=g)
        B = torch.empty(K, N, device="cuda").uniform_(low, 1, generator=g)
        ref, _ = exact(A, B, False, False)
        R, F = torch.zeros(M, N, device="cuda"), torch.zeros(M, N, device="cuda")
        run(am, A, B, R, False, False)
        am.amulet_mmlike_f32_shape(am.AMULET_IDENTITY, 8, A, B, None, F)   # register-staged fp32 kernel
        assert (R.double() - ref).norm() <= (F.double() - ref).norm()


@pytest.mark.parametrize("size,most", [(2048, 1.02 * 2.0 ** -23), (4096, 1.5 * 2.0 ** -23)])
def test_a_product_alone_in_its_sum(am, size, most):
    """A row of A with one value: every result is one product, of which the pieces leave out at most 2^-24; the sum of the
    rest is rounded once with two sets of accumulators (2048), and to an ulp by the matrix instruction with one (4096)."""
    K = 128
    g = torch.Generator(device="cuda").manual_seed(17)
    A = torch.zeros(size, K, device="cuda")
    A[torch.arange(size, device="cuda"), torch.randint(0, K, (size,), device="cuda", generator=g)] = torch.empty(size, device="cuda").uniform_(1, 2, generator=g)
    B = torch.empty(K, size, device="cuda").normal_(generator=g)
    R = torch.zeros(size, size, device="cuda")
    run(am, A, B, R, False, False)
    ref, ab = exact(A, B, False, False)
    err = (R.double() - ref).abs() / ab
    assert float(err.max()) <= most and float(err.mean()) <= 2.0 ** -25


@pytest.mark.parametrize("M,N", [(2048, 2048), (4096, 4096)])
def test_values_the_pieces_do_not_carry(am, M, N):
    """Small, subnormal and near-overflow values are as exact as any other; infinities and NaN reach the results that
    plain fp32 would give them in."""
    K = 112
    g = torch.Generator(device="cuda").manual_seed(7)
    A, B = operand(g, M, K, 0), operand(g, K, N, 0)
    A[3] *= 2.0 ** -120              # a row below what three pieces hold, times a column that makes it count
    A[200, 5] = 2.0 ** -140          # one value of a tile, and its partners' products the only ones that are not zero
    A[200, :5] = 0
    A[200, 6:] = 0
    B[5, :] = 2.0 ** 100
    B[:, 64] *= 2.0 ** 20
    A[700] = 0
    A[700, 9] = 3.4e38               # rounds to an infinite bf16
    B[9, :] = 0.5
    ref, ab = exact(A, B, False, False)
    R = torch.zeros(M, N, device="cuda")
    print("identity pieces special", M, N, flush=True)
    run(am, A, B, R, False, False)
    # (the least representable result, and fp32 accumulators)
    assert float((((R.double() - ref).abs() - 2.0 ** -149) / ab.clamp_min(1e-300)).max()) <= 1e-5
    A[40, 0], A[41, 1], A[42, 2] = float("inf"), float("-inf"), float("nan")
    B[0, :], B[1, :] = 1.0, 0.25
    R.zero_()
    run(am, A, B, R, False, False)
    assert bool((R[40] == float("inf")).all()) and bool((R[41] == float("-inf")).all()) and bool(R[42].isnan().all())
    rest = torch.ones(M, dtype=torch.bool, device="cuda")
    rest[40:43] = False
    assert bool(R[rest].isfinite().all())


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,pad,tile_rows", [(2047, 1921, 3, 128), (4095, 4001, 5, 256)])
def test_where_the_second_way_begins(am, M, N, pad, tile_rows, tA, tB):
    """One value that the pieces do not carry in some tiles, found in the first stage or at the end only, beside tiles
    without one; remainders of K and of the tiles; every value of a block of rows."""
    K = 300
    g = torch.Generator(device="cuda").manual_seed(13)
    A = operand(g, *((K, M) if tA else (M, K)), pad)
    B = operand(g, *((N, K) if tB else (K, N)), pad)
    a = A.T if tA else A
    for i, k in enumerate([0, 11, 100, 128, 143, 200, 256, K - 1]):
        a[256 * (i % 7) + 3 + i, k] = 1.2345e-40 * (i + 1)
    a[M - 5:] *= 1e-36
    a[M - 1, 7] = float("inf")
    R = torch.full((M, N + pad), 0.5, device="cuda")[:, :N]
    print("identity pieces second way", M, N, tA, tB, flush=True)
    assert run(am, A, B, R, tA, tB) == tile_rows
    ref, ab = exact(A, B, tA, tB)
    rest = slice(0, M - 1)
    # fp32 accumulators over K <= 300, one rounding per product where the tile is formed in fp32, and what R += rounds
    err = (R[rest].double() - (ref[rest] + 0.5)).abs() - 2.0 ** -23 * (ref[rest] + 0.5).abs() - 2.0 ** -149
    assert float((err / ab[rest]).max()) <= K * 2.0 ** -24
    assert torch.equal(R[M - 1].double(), ref[M - 1])          # infinities and the NaN of 0 inf, where the products have them
    assert bool(R[rest].isfinite().all())


@pytest.mark.parametrize("M,N", [(2048, 2048), (4096, 4096)])
@pytest.mark.parametrize("what", ["subnormal products", "subnormal pieces"])
def test_subnormals_on_the_bf16_matrix_cores(am, what, M, N):
    """Pieces and piece products below the smallest normal number count like any other."""
    K = 112
    g = torch.Generator(device="cuda").manual_seed(11)
    A, B = operand(g, M, K, 0), operand(g, K, N, 0)
    if what == "subnormal products":     # the products straddle 2^-126, no piece is subnormal
        A, B = A * 2.0 ** -63, B * 2.0 ** -63
    else:                                # 16 bits from 2^-133 up: the pieces carry all of them, most in subnormal bf16 numbers
        A = (A * 65535).round() * 2.0 ** -126 * 2.0 ** -7
        B = B * 2.0 ** 100
    ref, ab = exact(A, B, False, False)
    R = torch.zeros(M, N, device="cuda")
    print("identity pieces", what, M, N, flush=True)
    run(am, A, B, R, False, False)
    # fp32 accumulators, and of each product six pieces that round to a multiple of 2^-149
    worst = float((((R.double() - ref).abs() - 6 * K * 2.0 ** -150) / ab).max())
    print("worst", worst, flush=True)
    assert worst <= 1e-5
