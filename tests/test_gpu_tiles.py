"""GPU parity of the tile kernels: of the predicate tasks (32 x 64 and 16 x 64 tiles whose K a
workgroup's waves share), which built-in calls take at small, narrow and odd sizes, on exact dyadic
data with ties, so that every form, layout and size must agree bit for bit with the oracle; and of
the join count (64 x 64 to 256 x 256), exact against a float32 product of small integers."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# edges of the tiles (16, 32 rows; 64 columns; 16-byte units of 4 and 2), of a stage (16 and 8 k) and
# of the k ranges: the smallest problem of each layout, one more and one less than whole tiles and
# stages, ranges of unequal length, K over several workgroups, more than one round of them
SIZES = [(4, 4, 16), (1, 5, 16), (15, 63, 17), (16, 64, 64), (17, 65, 31), (33, 130, 100), (32, 64, 777), (100, 70, 2047),
         (509, 515, 130)]


@pytest.fixture(scope="module")
def am():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_08872_amd as am
    am.load_library()
    return am


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("task", [1, 2, 3])
@pytest.mark.parametrize("form", [0, 1, 2, 3])
def test_tile_kernels_at_the_edges_of_tiles_stages_and_k_ranges(am, dtype, task, form):
    ref = oracle.mmlike_f32_general if dtype == np.float32 else oracle.mmlike_f64_general
    call = am.amulet_mmlike_f32_general if dtype == np.float32 else am.amulet_mmlike_f64
    for idx, (M, N, K) in enumerate(SIZES):
        g = np.random.Generator(np.random.PCG64(7100 + 10 * task + form + 100 * idx))
        A, B = g.integers(-8, 9, (M, K)).astype(dtype), g.integers(-8, 9, (K, N)).astype(dtype)
        th = (g.integers(-24, 25, {0: (N,), 1: (M,), 2: (1,), 3: (M, N)}[form]) / 2.0).astype(dtype)
        dis = (g.integers(0, 9, N) / 8.0).astype(dtype)
        R_in = g.integers(-5, 6, (M, N)).astype(dtype)
        R_ref, _, _ = ref(task, A, B, th, dis if task == 1 else None, R_in, thres_form=form)
        for tA, tB in [(False, False), (True, False), (False, True), (True, True)]:
            dR = torch.from_numpy(R_in.copy()).cuda()
            print("tile", dtype.__name__, task, form, tA, tB, M, N, K, flush=True)
            call(task, torch.from_numpy(np.ascontiguousarray(A.T if tA else A)).cuda(),
                 torch.from_numpy(np.ascontiguousarray(B.T if tB else B)).cuda(), torch.from_numpy(th).cuda(),
                 torch.from_numpy(dis).cuda() if task == 1 else None, dR, thres_form=form, trans_a=tA, trans_b=tB)
            torch.cuda.synchronize()
            assert np.array_equal(dR.cpu().numpy(), R_ref.astype(dtype)), (M, N, K, tA, tB)


# edges of the join count's tiles (64 ... 256), of its 16-byte units and of its stages (64 k, 128 in two
# groups): the smallest problem, one more and one less than whole tiles, units and stages, a short last
# stage in either group, K over several workgroups, an R that is read and written around the caches (which
# kernel a size gets follows from a model of its time; every kernel at a size of its own: I8_KERNELS below)
I8_SIZES = [(16, 16, 64), (17, 31, 65), (63, 65, 127), (64, 64, 128), (65, 80, 193), (130, 100, 1055), (100, 260, 4097),
            (1000, 1000, 250), (1100, 1500, 300), (2100, 1900, 130), (2048, 4096, 192), (1900, 3000, 1000), (2300, 4112, 208), (3000, 4400, 75), (8500, 8400, 70)]


@pytest.mark.parametrize("layout", [(False, False), (True, False), (False, True), (True, True)])
def test_count_tile_kernels_at_the_edges_of_tiles_units_and_stages(am, layout):
    tA, tB = layout
    for idx, (M, N, K) in enumerate(I8_SIZES):
        g = torch.Generator().manual_seed(9300 + idx)
        A = torch.randint(-3, 4, (M, K), dtype=torch.int8, generator=g).cuda()
        B = torch.randint(-3, 4, (K, N), dtype=torch.int8, generator=g).cuda()
        want = A.float() @ B.float()          # |sum| < 2^24: exact
        R_in = torch.randint(-9, 10, (M, N), dtype=torch.int32, generator=g).cuda()
        ws = torch.empty(am.amulet_count_i8_workspace_bytes(tA, tB, M, N, K) + 16, dtype=torch.int8, device="cuda")
        # rows as they are, at odd addresses (through registers) and at a pitch of whole 16 bytes (streamed)
        for pad in (0, 1, 16):
            def stored(X, trans):
                X = X.t() if trans else X
                pitch = X.shape[1] if pad == 0 else (X.shape[1] + 15) // 16 * 16 + pad
                buf = torch.zeros(X.shape[0] * pitch + pad, dtype=torch.int8, device="cuda")
                view = buf[pad % 16:][:X.shape[0] * pitch].view(X.shape[0], pitch)[:, :X.shape[1]]
                view.copy_(X)
                return view
            print("count tile", layout, pad, M, N, K, flush=True)
            sA, sB = stored(A, tA), stored(B, tB)
            R = R_in.clone()
            am.amulet_count_i8_general(sA, sB, R, ws, trans_a=tA, trans_b=tB)
            torch.cuda.synchronize()
            assert torch.equal(R - R_in, want.to(torch.int32)), (M, N, K, pad)
            if not tA and not tB:
                R = R_in.clone()
                am.amulet_count_i8_assign(sA, sB, R)
                torch.cuda.synchronize()
                assert torch.equal(R, want.to(torch.int32)), (M, N, K, pad)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("form", [0, 3])
def test_boost_terms_enter_the_sum_with_the_unrounded_product(am, dtype, form):
    """Row i holds -fl(x * x) * 1 at an even k and x * x at the next one, x = 1 + 2^-13 (fp64: 2^-28), below any
    threshold: in whichever k range the two stand, the sum is the product's own rounding error, 2^-26
    (2^-56), if the product goes into the fused add as it is, and 0 if it was rounded first."""
    e = 13 if dtype == np.float32 else 28
    x, want = dtype(1 + 2.0 ** -e), dtype(2.0 ** (-2 * e))
    call = am.amulet_mmlike_f32_general if dtype == np.float32 else am.amulet_mmlike_f64
    for M, N, K in [(40, 70, 16), (40, 70, 18), (300, 70, 577), (40, 260, 1024)]:
        A, B = np.zeros((M, K), dtype), np.ones((K, N), dtype)
        k = 2 * (np.arange(M) % (K // 2))
        A[np.arange(M), k], A[np.arange(M), k + 1] = -(1 + 2.0 ** (1 - e)), x
        B[1::2] = x
        th = np.full({0: (N,), 3: (M, N)}[form], 1e30, dtype)
        for tA, tB in [(False, False), (True, False), (False, True), (True, True)]:
            dR = torch.zeros((M, N), dtype=torch.from_numpy(A).dtype, device="cuda")
            call(2, torch.from_numpy(np.ascontiguousarray(A.T if tA else A)).cuda(),
                 torch.from_numpy(np.ascontiguousarray(B.T if tB else B)).cuda(), torch.from_numpy(th).cuda(), None, dR,
                 thres_form=form, trans_a=tA, trans_b=tB)
            torch.cuda.synchronize()
            assert "tile" in am.amulet_recent_kernel()
            assert np.all(dR.cpu().numpy() == want), (M, N, K, tA, tB)


def _kernel(am, back=0):
    """amulet_recent_kernel without the rows."""
    words = am.amulet_recent_kernel(back).split()
    return [words[0]] + words[3:]


@pytest.mark.parametrize("M,N,K", [(16384, 8192, 2048), (12001, 16003, 130)])
def test_adaptive_count_times_as_the_built_in_kernel_what_a_plain_call_runs(am, monkeypatch, M, N, K):
    """The first trial of an adaptive call is what a plain call would run, and if it wins the rest runs with
    it: decided for the slab alone, one of 4096 rows of 16384 x 8192 x 2048 went to the tile kernels, which the
    whole count does not take."""
    monkeypatch.setenv("AMULET_ADAPTIVE_MIN_TASK_MS", "0")   # (lift the no-trials limit)
    g = torch.Generator(device="cuda").manual_seed(77)
    A = torch.randint(-3, 4, (M, K), dtype=torch.int8, device="cuda", generator=g)
    B = torch.randint(-3, 4, (K, N), dtype=torch.int8, device="cuda", generator=g)
    am.amulet_clear_selections()
    R = torch.zeros(M, N, dtype=torch.int32, device="cuda")
    am.amulet_count_i8(A, B, R)
    plain, built_in = _kernel(am), am.amulet_selected_shape(am.AMULET_TASK_COUNT_I8, M, N, K)
    R.fill_(5)
    chosen, trials = am.amulet_count_i8_adaptive(A, B, R)
    torch.cuda.synchronize()
    am.amulet_clear_selections()
    assert trials >= 2
    assert _kernel(am, trials) == plain
    assert _kernel(am, 0) == (plain if chosen == built_in else [am.amulet_shape_name(am.AMULET_TASK_COUNT_I8, chosen)])
    assert torch.equal(R, (A.float() @ B.float()).to(torch.int32) + 5)      # |sum| < 2^24: exact


@pytest.mark.parametrize("task", [1, 2, 3])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_adaptive_calls_time_as_the_built_in_kernel_what_a_plain_call_runs(am, monkeypatch, task, dtype):
    monkeypatch.setenv("AMULET_ADAPTIVE_MIN_TASK_MS", "0")
    M, N, K = 24576, 2048, 72
    g = torch.Generator(device="cuda").manual_seed(78)
    A, B, th, dis = (torch.randint(-9, 10, s, device="cuda", generator=g).to(dtype) for s in ((M, K), (K, N), (N,), (N,)))
    R, call = torch.zeros(M, N, dtype=dtype, device="cuda"), am.amulet_mmlike_f32_general if dtype == torch.float32 else am.amulet_mmlike_f64
    adaptive = am.amulet_mmlike_f32_adaptive_general if dtype == torch.float32 else am.amulet_mmlike_f64_adaptive
    am.amulet_clear_selections()
    call(task, A, B, th, dis / 8, R)
    plain, whole = _kernel(am), R.clone()
    R.zero_()
    _, trials = adaptive(task, A, B, th, dis / 8, R)
    torch.cuda.synchronize()
    am.amulet_clear_selections()
    assert trials >= 2 and _kernel(am, trials) == plain
    assert torch.equal(R, whole)        # multiples of 1/8 well below 2^24 of them: exact in any order


# Every kernel of the join count's tile family at a size whose plan it is: (kernel, K over several workgroups,
# R = instead of R +=, M, N, K).  Streamed ones on tight rows, the ones through registers on rows at odd
# addresses; ragged in all three.  A model of the kernels' times makes the plans: where a constant of it changes,
# the size here has to follow, or that kernel goes untested.
I8_KERNELS = [
    ("i8_tile_64x64", False, False, 100, 68, 76), ("i8_tile_64x64", True, False, 72, 68, 460), ("i8_tile_64x64", True, True, 64, 68, 3780),
    ("i8_tile_64x64_registers", False, False, 65, 67, 103), ("i8_tile_64x64_registers", True, False, 77, 65, 385),
    ("i8_tile_64x64_registers", True, True, 71, 89, 2109),
    ("i8_tile_128x128", False, False, 6660, 268, 72), ("i8_tile_128x128", False, True, 8820, 208, 68),
    ("i8_tile_128x128", True, False, 72, 8684, 1148), ("i8_tile_128x128", True, True, 8336, 68, 3144),
    ("i8_tile_128x128_registers", False, False, 8321, 77, 277), ("i8_tile_128x128_registers", True, False, 8961, 67, 617),
    ("i8_tile_128x128_registers", True, True, 67, 8769, 1917),
    ("i8_tile_128x256", False, False, 4648, 2564, 68), ("i8_tile_128x256", False, True, 7620, 1576, 76),
    ("i8_tile_128x256_bypass", False, False, 8852, 8096, 96),
    ("i8_tile_128x256_ring6", False, False, 2400, 1724, 1352), ("i8_tile_128x256_ring6", False, True, 5980, 704, 1088),
    ("i8_tile_256x256", False, False, 2724, 2948, 2204), ("i8_tile_256x256", False, True, 1388, 5964, 1672),
    ("i8_tile_256x256_bypass", False, False, 7644, 8236, 2388),
    ("i8_tile_256x256_registers", False, False, 6949, 1785, 65), ("i8_tile_256x256_registers", False, True, 1625, 7825, 69),
    ("i8_tile_256x256_registers_bypass", False, False, 8741, 8897, 69),
    # whole aligned tiles: the streamed kernels that have shape ids (transposed operands copied first, from K = 4096 on)
    ("mfma_i8_256x256_w16_dma4_persistent", False, False, 8192, 8192, 4096),
    ("mfma_i8_256x256_w16_dma4_persistent", False, False, 8192, 8192, 2048), ("mfma_i8_256x256_w16_dma4_persistent", False, True, 8192, 8192, 320),
    ("mfma_i8_128x256_dma3", False, True, 4096, 4352, 256),
]


@pytest.mark.parametrize("kernel,split,assign,M,N,K", I8_KERNELS)
def test_every_count_kernel_at_a_size_of_its_own(am, kernel, split, assign, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = torch.randint(-3, 4, (M, K), dtype=torch.int8, device="cuda", generator=g)
    B = torch.randint(-3, 4, (K, N), dtype=torch.int8, device="cuda", generator=g)
    want = (A.float() @ B.float()).to(torch.int32)      # |sum| < 2^24: exact
    odd = 1 if "registers" in kernel else 0
    am.amulet_clear_selections()
    for tA, tB in [(False, False)] if assign or (kernel.startswith("mfma") and K < 4096) else [(False, False), (True, False), (False, True), (True, True)]:
        def stored(X, trans):
            X = X.t() if trans else X
            buf = torch.zeros(X.numel() + odd, dtype=torch.int8, device="cuda")
            view = buf[odd:].view(X.shape)
            view.copy_(X)
            return view
        print(kernel, split, assign, tA, tB, M, N, K, flush=True)
        sA, sB = stored(A, tA), stored(B, tB)
        R = torch.full((M, N), 11, dtype=torch.int32, device="cuda")
        if assign:
            am.amulet_count_i8_assign(sA, sB, R)
        else:
            am.amulet_count_i8_general(sA, sB, R, torch.empty(am.amulet_count_i8_workspace_bytes(tA, tB, M, N, K) + 16, dtype=torch.int8,
                                                              device="cuda"), trans_a=tA, trans_b=tB)
        torch.cuda.synchronize()
        ran = _kernel(am)
        assert ran[0] == kernel and ("parts" in ran and int(ran[2]) > 1) == split, ran
        assert ("r_in_k_loop" in ran) == (kernel.endswith("persistent") and not assign), ran
        assert torch.equal(R, want if assign else want + 11), (tA, tB)


@pytest.mark.parametrize("dtype,kernel,split,M,N,K", [
    (np.float32, "f32_tile_32x64", True, 815, 141, 265), (np.float32, "f32_tile_32x64", False, 600, 1301, 333),
    (np.float32, "f32_tile_16x64", False, 903, 145, 243), (np.float32, "f32_tile_16x64", True, 71, 67, 1003),
    (np.float64, "f64_tile_32x64", True, 815, 141, 265), (np.float64, "f64_tile_32x64", False, 600, 1301, 333),
    (np.float64, "f64_tile_16x64", False, 903, 145, 243), (np.float64, "f64_tile_16x64", True, 71, 67, 1003)])
@pytest.mark.parametrize("task", [1, 2, 3])
def test_every_predicate_tile_at_a_size_of_its_own(am, dtype, kernel, split, M, N, K, task):
    """Both tiles, K whole and over several workgroups, with K loops of many stages, a short last one and
    ragged edges: as above, on data whose sums are exact in any order."""
    ref = oracle.mmlike_f32_general if dtype == np.float32 else oracle.mmlike_f64_general
    call = am.amulet_mmlike_f32_general if dtype == np.float32 else am.amulet_mmlike_f64
    g = np.random.Generator(np.random.PCG64(7900 + task + M))
    A, B = g.integers(-8, 9, (M, K)).astype(dtype), g.integers(-8, 9, (K, N)).astype(dtype)
    th, dis = (g.integers(-24, 25, N) / 2.0).astype(dtype), (g.integers(0, 9, N) / 8.0).astype(dtype)
    R_in = g.integers(-5, 6, (M, N)).astype(dtype)
    R_ref, _, _ = ref(task, A, B, th, dis if task == 1 else None, R_in, thres_form=0)
    am.amulet_clear_selections()
    for tA, tB in [(False, False), (True, False), (False, True), (True, True)]:
        dR = torch.from_numpy(R_in.copy()).cuda()
        print(kernel, split, task, tA, tB, M, N, K, flush=True)
        call(task, torch.from_numpy(np.ascontiguousarray(A.T if tA else A)).cuda(), torch.from_numpy(np.ascontiguousarray(B.T if tB else B)).cuda(),
             torch.from_numpy(th).cuda(), torch.from_numpy(dis).cuda() if task == 1 else None, dR, trans_a=tA, trans_b=tB)
        torch.cuda.synchronize()
        ran = _kernel(am)
        assert ran[0] == kernel and (int(ran[2]) > 1) == split, ran
        assert np.array_equal(dR.cpu().numpy(), R_ref.astype(dtype)), (tA, tB)


def test_a_tuned_shape_runs_on_copies_of_operands_it_cannot_take(am):
    """With a shape selected that is not the built-in one, the general join count copies operands that are
    transposed, unaligned or ragged into the workspace.  100 and 250 rows share a selection and have different
    built-in shapes (at most 256 tiles of 128 x 256, and more), so whatever the tuner picks, one of the two
    does not run the built-in choice."""
    N, K, on_copies = 33000, 1000, 0
    am.amulet_clear_selections()
    try:
        assert am.amulet_selected_shape(100, 100, N, K) != am.amulet_selected_shape(100, 250, N, K)
        chosen = am.amulet_tune(am.AMULET_TASK_COUNT_I8, 250, N, K)
        for M in (100, 250):
            g = torch.Generator(device="cuda").manual_seed(M)
            A = torch.randint(-3, 4, (M, K), dtype=torch.int8, device="cuda", generator=g)
            B = torch.randint(-3, 4, (K, N), dtype=torch.int8, device="cuda", generator=g)
            want = (A.float() @ B.float()).to(torch.int32) + 5
            for tA, tB, off in [(False, False, 1), (True, False, 3), (False, True, 0), (True, True, 1)]:
                def stored(X, trans):
                    X = X.t() if trans else X
                    view = torch.zeros(X.numel() + off, dtype=torch.int8, device="cuda")[off:].view(X.shape)
                    view.copy_(X)
                    return view
                ws = torch.full((am.amulet_count_i8_repack_workspace_bytes(M, N, K),), 77, dtype=torch.int8, device="cuda")
                R = torch.full((M, N), 5, dtype=torch.int32, device="cuda")
                print("tuned join", chosen, M, tA, tB, off, flush=True)
                am.amulet_count_i8_general(stored(A, tA), stored(B, tB), R, ws, trans_a=tA, trans_b=tB)
                torch.cuda.synchronize()
                on_copies += _kernel(am) == [am.amulet_shape_name(am.AMULET_TASK_COUNT_I8, chosen)]
                assert torch.equal(R, want), (chosen, M, tA, tB)
        assert on_copies >= 4
    finally:
        am.amulet_clear_selections()
