"""The fp32 count by rounding (csrc/count_rounding.h): its arithmetic on the CPU against exact fractions, and the kernel
against the definition on the GPU, where products tie with their thresholds and where a tile needs its second way."""
import random
import struct
from fractions import Fraction

import pytest

torch = pytest.importorskip("torch")

FORMS = ("col", "row", "const", "elem")


def as_float(bits):
    return struct.unpack("f", struct.pack("I", bits & 0xFFFFFFFF))[0]


def as_bits(x):
    return struct.unpack("I", struct.pack("f", x))[0]


def round32(x):
    """The float nearest to a fraction, ties to even (normal results)."""
    if x == 0:
        return Fraction(0)
    m, e = abs(x), 0
    while m >= 1 << 24:
        m, e = m / 2, e + 1
    while m < 1 << 23:
        m, e = m * 2, e - 1
    n, rest = divmod(m, 1)
    n = int(n) + (1 if rest > Fraction(1, 2) or (rest == Fraction(1, 2) and int(n) % 2) else 0)
    return Fraction(n) * Fraction(2) ** e * (1 if x > 0 else -1)


def test_rounding_is_the_comparison():
    """g, s and both operations as the header gives them, in exact arithmetic rounded where the hardware rounds, against
    RN(a b) > th: products around a threshold, every tie, and thresholds next to powers of two of both signs."""
    rng = random.Random(5)
    ties = above = 0
    for _ in range(6000):
        kind = rng.randrange(3)
        a = Fraction(rng.getrandbits(24) | 1 << 23 if kind else rng.getrandbits(12) | 1 << 11 | 1) * rng.choice((1, -1))
        b = Fraction(rng.getrandbits(24) | 1 << 23 if kind else rng.getrandbits(13) | 1 << 12 | 1) * rng.choice((1, -1)) / 2 ** rng.randrange(24, 70)
        p = round32(a * b)
        bits = as_bits(float(p))
        if kind == 2:      # a threshold at a power of two, and a product next to it
            bits &= 0xFF800000
            b = round32(Fraction(as_float(bits)) * (1 + Fraction(rng.randrange(-4, 5), 2 ** 25)) / a)
            p = round32(a * b)
        bits += rng.choice((-2, -1, -1, 0, 0, 1, 2))
        th = Fraction(as_float(bits))
        exponent = ((bits >> 23) & 255) - 127
        if not -40 <= exponent < 24:
            continue
        e = exponent - (1 if bits & 0x807FFFFF == 0x80000000 else 0)
        g = Fraction(2) ** (23 - e)
        s = 1 + Fraction(1, 2 ** 23) if bits & 1 else 1 - Fraction(1, 2 ** 24)
        assert round32(th * g) == th * g and abs(th * g) <= 2 ** 24
        t = min(max(round32(a * (b * g) - th * g), Fraction(0)), Fraction(1))
        n = rng.randrange(2 ** 23)
        total = 2 ** 23 + n + t * s
        got = int(total // 1) + (1 if total % 1 > Fraction(1, 2) else 0)
        assert total % 1 != Fraction(1, 2)       # never a tie of its own: the sum's last bit does not matter
        assert got == 2 ** 23 + n + (1 if p > th else 0), (float(a), float(b), float(th))
        ties += a * b != p and t == Fraction(1, 2)
        above += p > th
    assert ties > 20 and 1000 < above < 5000


def test_zero_by_rounding_is_the_comparison():
    """The factors of a threshold of zero, in exact arithmetic rounded where the hardware rounds and infinite where fp32
    overflows, against RN(a b) > 0: products around 2^-150, subnormal operands, and factors that overflow."""
    rng = random.Random(6)
    top = Fraction(2) ** 128

    def up(x, e):       # x 2^e as fp32 has it: exact, or infinite
        y = x * Fraction(2) ** e
        return y if abs(y) < top else (None if y > 0 else -1)
    near = seen = 0
    for _ in range(6000):
        ea = rng.randrange(-126, 127)
        a = Fraction(rng.getrandbits(23) | 1 << 23) * Fraction(2) ** (ea - 23)
        eb = rng.choice((-150 - ea + rng.randrange(-2, 3), rng.randrange(-149, 127)))
        b = Fraction(rng.getrandbits(23) | 1 << 23) * Fraction(2) ** (eb - 23)
        if rng.random() < 0.5:      # the partner that makes 2^-150, or its neighbours
            b = round32(Fraction(2) ** -150 / a) * (1 + Fraction(rng.randrange(-1, 2), 2 ** 23))
        b = Fraction(int(b * 2 ** 149), 2 ** 149)           # (fp32 below its normal numbers)
        if not 0 < b < top:
            continue
        above = a * b > Fraction(2) ** -150
        for first, then in ((99, 98), (98, None)):          # on B alone; on A, with 99 on B
            if then is not None:
                if a < Fraction(2) ** -80:
                    continue
                x, y = a, up(b, first)
                y = None if y is None else up(y, then)
            else:
                x, y = up(a, 98), up(b, 99)
            t = 1 if x is None or y is None else min(max(round32(x * y - Fraction(2) ** 47), Fraction(0)), Fraction(1))
            assert t == (1 if above else 0), (float(a), float(b), first)
            seen += 1
        near += abs(a * b * Fraction(2) ** 150 - 1) < Fraction(1, 2 ** 20)
    assert near > 500 and seen > 6000


@pytest.fixture(scope="module")
def am():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_08872_amd as am
    am.load_library()
    am.amulet_clear_selections()
    return am


def check(am, A, B, th, form, tA, tB, shape, want=None, pad=0):
    M, K = A.shape
    N = B.shape[1]
    t = {"col": lambda: th[None, :], "row": lambda: th[:, None], "const": lambda: th[0], "elem": lambda: th}[form]()
    if want is None:
        want = torch.zeros(M, N, device="cuda")
        for k in range(K):
            want += (A[:, k:k + 1] * B[k:k + 1, :] > t).float()

    def stored(X, transposed):
        X = X.t() if transposed else X
        buf = torch.empty(X.shape[0], X.shape[1] + pad, device="cuda")
        buf[:, :X.shape[1]] = X
        return buf[:, :X.shape[1]]
    R = torch.full((M, N), 2.0, device="cuda")
    am.amulet_mmlike_f32_general(am.AMULET_COUNT_GT, stored(A, tA), stored(B, tB), th, None, R, thres_form=FORMS.index(form),
                                 trans_a=tA, trans_b=tB, shape=shape)
    assert ("valu_" if shape >= 0 else "f32_tile_") in am.amulet_recent_kernel(), am.amulet_recent_kernel()
    assert torch.equal(R, want + 2.0), (form, tA, tB, shape, int((R != want + 2.0).sum()))
    return want


def thresholds(form, M, N):
    return {"col": (N,), "row": (M,), "const": (1,), "elem": (M, N)}[form]


def some(g, pool, shape):
    return pool[torch.randint(0, pool.numel(), shape, device="cuda", generator=g)]


# remainders of K beside the 16 and 32 k of a stage, rows and columns beside the tile's, K in parts (512 x 512), an unaligned pitch
SIZES = [(33, 257, 31, 0), (64, 256, 64, 0), (31, 255, 97, 1), (512, 512, 200, 0), (5, 3, 18, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("form", FORMS)
def test_ties_and_neighbours(am, form, tA, tB):
    """Odd factors of 13 and 14 bits, whose products end half way between two floats, from few values, so that thresholds
    taken from the products and their neighbours are met often: every count must be the definition's."""
    shapes = [am_id for am_id in range(am.amulet_shape_count(am.AMULET_COUNT_GT))
              if am.amulet_shape_name(am.AMULET_COUNT_GT, am_id) in ("valu_16x256_k16", "valu_32x256_w8_k16", "valu_16x256_k8")]
    assert len(shapes) == 3
    for M, N, K, pad in SIZES:
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        a = torch.randint(-4096, 4096, (5,), device="cuda", generator=g).float() * 2 + 1
        b = (torch.randint(-8192, 8192, (5,), device="cuda", generator=g).float() * 2 + 1) * 2.0 ** -20
        th = (a[:, None] * b[None, :]).flatten()
        below, over = torch.full_like(th, -1e38), torch.full_like(th, 1e38)
        th = torch.cat([th, torch.nextafter(th, over), torch.nextafter(th, below), torch.tensor([0.015625, -0.015625], device="cuda")])
        b = torch.cat([b, torch.nextafter(torch.tensor([0.015625, -0.015625]), torch.zeros(2)).cuda()])
        a = torch.cat([a, torch.ones(1, device="cuda")])
        A, B, T = some(g, a, (M, K)), some(g, b, (K, N)), some(g, th, thresholds(form, M, N))
        want = None
        for shape in shapes:
            want = check(am, A, B, T, form, tA, tB, shape, want, pad)


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("form", ("col", "row", "const"))
def test_tile_kernels(am, form, tA, tB):
    """The same in the tile kernels, at sizes from which they round: both tiles, K shared by their waves and in parts, remainders of
    its stages, ragged edges; and what sends a tile to its second way."""
    for M, N, K, pad in [(801, 701, 799, 0), (129, 4003, 515, 1), (65, 2001, 2047, 3), (640, 512, 720, 0)]:
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        a = torch.randint(-4096, 4096, (6,), device="cuda", generator=g).float() * 2 + 1
        b = (torch.randint(-8192, 8192, (6,), device="cuda", generator=g).float() * 2 + 1) * 2.0 ** -20
        th = (a[:, None] * b[None, :]).flatten()
        th = torch.cat([th, torch.nextafter(th, torch.full_like(th, 1e38)), torch.nextafter(th, torch.full_like(th, -1e38))])
        A, B, T = some(g, a, (M, K)), some(g, b, (K, N)), some(g, th, thresholds(form, M, N))
        check(am, A, B, T, form, tA, tB, -1, pad=pad)
        B[K // 2, N // 3] = 3e38      # (in the rows' form A carries the factor)
        A[M // 2, K // 3] = -3e38
        A[:, K // 2] = 0.0
        check(am, A, B, T, form, tA, tB, -1, pad=pad)
        T.view(-1)[::3] = 0.0
        check(am, A, B, T, form, tA, tB, -1, pad=pad)


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("form", ("col", "row", "const"))
def test_threshold_zero(am, form, tA, tB):
    """Products at 2^-150 and next to it, subnormal operands, and factors whose scaled value overflows, against a threshold of
    zero (of either sign) alone; then with values that leave it to the comparison, and with other thresholds beside it."""
    f32 = lambda *v: torch.tensor(v, device="cuda")  # noqa: E731
    odd = torch.tensor([1 + 2.0 ** -12, 1 + 2.0 ** -23, 1.7], dtype=torch.float32)
    part = (1 / odd.double()).float()
    part = torch.cat([part, torch.nextafter(part, torch.full_like(part, 9.0)), torch.nextafter(part, torch.zeros_like(part))])
    a = torch.cat([odd.cuda() * 2.0 ** -75, f32(0.0, -0.0, -1.0, 2.0 ** -80, 2.0 ** -75, 1.5, -3e38, 1e30, 2.0 ** -79)])
    b = torch.cat([part.cuda() * 2.0 ** -75, f32(0.0, 2.0 ** -149, -1e-45, 2.0 ** -70, 2.0 ** -71, 2.0 ** -75, 3e38, -1e30, 2.0 ** -126, 1.0)])
    small = f32(1e-45, -2.0 ** -149, 2.0 ** -81, 1e-40)
    tiles = [(801, 701, 799, 0), (129, 4003, 515, 1), (65, 2001, 2047, 3), (640, 512, 720, 0)]      # (the tile kernels', from 15 us on)
    for M, N, K, pad in SIZES + [(40, 260, 3, 1), (70, 300, 2100, 3)] + tiles:
        g = torch.Generator(device="cuda").manual_seed(M + N + K)
        T = some(g, f32(0.0, -0.0), thresholds(form, M, N))
        for pool in (a, torch.cat([a, f32(float("inf"), -float("inf"), float("nan"))]), torch.cat([a, small])):
            A, B = some(g, pool, (M, K)), some(g, b, (K, N))
            want = None
            for shape in (-1,) if (M, N, K, pad) in tiles else (4, 5, 0):
                want = check(am, A, B, T, form, tA, tB, shape, want, pad)
        T.view(-1)[::3] = 0.5
        check(am, A, B, T, form, tA, tB, -1 if (M, N, K, pad) in tiles else 5, pad=pad)


@pytest.mark.gpu
@pytest.mark.parametrize("form", FORMS)
def test_values_that_need_the_comparison(am, form):
    """Thresholds the rounding does not take, mixed with others and alone, and operands whose scaled value overflows beside
    factors (zero, subnormal) for which the overflow would count."""
    M, N, K = 65, 300, 70
    g = torch.Generator(device="cuda").manual_seed(11)
    special = torch.tensor([0.0, -0.0, 1e-30, -1e-30, 2.0 ** 24, -2.0 ** 24, 1e30, 2.0 ** -41, 1e-45], device="cuda")
    inside = torch.tensor([float("inf"), -float("inf"), 2.0 ** -40, -2.0 ** -40, 0.5, -2.0, 2.0 ** 24 - 1, 3e-5], device="cuda")
    normal = lambda *s: torch.empty(*s, device="cuda").normal_(generator=g)  # noqa: E731
    for tA, tB in [(False, False), (True, True)]:
        for pool in (special, inside, torch.cat([special, inside])):
            A, B = normal(M, K), normal(K, N)
            A.view(-1)[::7] = 0.0
            B.view(-1)[::5] = 0.0
            A.view(-1)[1::17] = 1e-40
            check(am, A, B, some(g, pool, thresholds(form, M, N)), form, tA, tB, 5)
        A, B, T = normal(M, K), normal(K, N), -normal(*thresholds(form, M, N)).abs() * 1e-3
        A.view(-1)[::3] = 0.0
        A.view(-1)[1::3] = 1e-40
        B.view(-1)[::37] = 3e38
        check(am, A, B, T, form, tA, tB, 5)
        A.view(-1)[::3] = -3e38      # (in the rows' form A carries the factor)
        B.view(-1)[::37] = 0.0
        check(am, A, B, T, form, tA, tB, 5)
        A, B, T = normal(M, K), normal(K, N), normal(*thresholds(form, M, N))
        A.view(-1)[3::11] = float("inf")
        B.view(-1)[2::13] = -float("inf")
        check(am, A, B, T, form, tA, tB, 5)
