"""Which kernel a call runs, as amulet_recent_kernel tells it.  Every launch here is refused on the host (the
library's own seam), so this runs without a GPU: pointers are never read, only their alignment is."""
import ctypes
import os

import pytest

import paper_2305_08872_amd as am


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(am.library_path()):
        from paper_2305_08872_amd import build
        build.build()
    lib = am.load_library()
    am.amulet_clear_selections()
    yield lib
    am.amulet_debug_fail_launches(0)


def kernel(lib, call):
    """amulet_recent_kernel after a call whose launch is refused, as (name, fields)."""
    am.amulet_debug_fail_launches(1)
    try:
        assert call() == -5
    finally:
        am.amulet_debug_fail_launches(0)
    words = am.amulet_recent_kernel().split()
    return words[0], dict(zip(words[1::2], map(int, words[2::2])))


def ptr(address=1 << 20):
    return ctypes.c_void_p(address)


def f32(lib, task, M, N, K, shape=-1):
    return kernel(lib, lambda: lib.amulet_mmlike_f32_general(task, 0, 0, 0, shape, M, N, K, ptr(), K, ptr(), N, ptr(), 0, ptr(), ptr(), N, None))


def f64(lib, task, M, N, K, shape=-1):
    return kernel(lib, lambda: lib.amulet_mmlike_f64_shape(task, shape, 0, 0, 0, M, N, K, ptr(), K, ptr(), N, ptr(), 0, ptr(), ptr(), N, None))


def i8(lib, M, N, K, shape=None, at=1 << 20):
    if shape is not None:
        return kernel(lib, lambda: lib.amulet_count_i8_shape(shape, M, N, K, ptr(at), K, ptr(at), N, ptr(), N, None))
    return kernel(lib, lambda: lib.amulet_count_i8(M, N, K, ptr(at), K, ptr(at), N, ptr(), N, None))


def test_a_call_that_names_no_shape_tells_which_kernel_it_ran(lib):
    """The selected shape is what runs only where no tile kernel does: amulet_selected_shape alone
    would name a kernel for these sizes that does not run."""
    for task in (1, 2, 3):
        name, got = f32(lib, task, 256, 256, 256)
        assert name in ("f32_tile_16x64", "f32_tile_32x64") and got["rows"] == 256 and got["kpart"] * got["parts"] >= 256
        name, got = f64(lib, task, 1024, 1024, 1024)
        assert name in ("f64_tile_16x64", "f64_tile_32x64") and got["rows"] == 1024 and got["parts"] == 1
        rows = 64 if task == 2 else 128
        assert f64(lib, task, 4096, 4096, 4096) == ("f64_critical_%dx128" % rows, {"rows": 4096, "critical_rows": rows})
    name, got = i8(lib, 1000, 1000, 1000)
    assert name.startswith("i8_tile_") and got["rows"] == 1000
    # where no tile kernel runs: the selected shape
    assert f32(lib, 1, 8192, 8192, 8192)[0] == am.amulet_shape_name(1, am.amulet_selected_shape(1, 8192, 8192, 8192))
    assert f32(lib, 0, 1024, 1024, 1024)[0] == am.amulet_shape_name(0, am.amulet_selected_shape(0, 1024, 1024, 1024))
    assert i8(lib, 8192, 8192, 4096)[0] == am.amulet_shape_name(100, am.amulet_selected_shape(100, 8192, 8192, 4096))
    assert f64(lib, 0, 1024, 1024, 1024)[0] == "mfma_f64_64x64_dma4" and f64(lib, 0, 4096, 4096, 256)[0] == "mfma_f64_128x128_dma4"


def test_the_identity_of_few_tiles_takes_pieces_where_they_are_ahead(lib):
    """us, fp32 kernels / pieces: 2643 x 384 x 576 14.1 / 15.4, 4288 x 422 x 768 29.5 / 33.7, 66 x 5248 x 704 12.4 / 14.4, 108 x 5120 x 6336 71 / 78;
    1024^3 20.7 / 18.5, 531 x 1600 x 3705 60 / 47, 1639 x 512 x 981 20.5 / 17.1."""
    for M, N, K in [(2643, 384, 576), (4288, 422, 768), (66, 5248, 704), (108, 5120, 6336), (3702, 452, 832), (2688, 384, 832)]:
        assert "tile_rows" not in f32(lib, 0, M, N, K)[1], (M, N, K)
    for M, N, K in [(1024, 1024, 1024), (531, 1600, 3705), (1327, 1472, 5120), (649, 1111, 4736)]:
        assert f32(lib, 0, M, N, K)[1].get("tile_rows") == 64, (M, N, K)


def test_a_named_shape_is_the_kernel_that_runs(lib):
    for shape in range(am.amulet_shape_count(1)):
        assert f32(lib, 1, 256, 256, 256, shape) == (am.amulet_shape_name(1, shape), {"rows": 256})
    for shape in range(am.amulet_f64_shape_count()):
        assert f64(lib, 3, 256, 256, 256, shape) == (am.amulet_f64_shape_name(shape), {"rows": 256})
    for shape in range(1, am.amulet_shape_count(100)):
        assert i8(lib, 256, 256, 256, shape) == (am.amulet_shape_name(100, shape), {"rows": 256})


def test_a_join_count_by_a_persistent_shape_names_the_kernel_that_ran(lib):
    """Four kernels share that shape id: the one that reads R during its K loop (by four or by eight values a lane), the
    one that reads it in its write-back, and, with too few whole tiles to walk, one workgroup to a tile."""
    for call, group in [((8192, 8192, 4096), 4), ((8192, 8192, 3392, 8), 4), ((8192, 8192, 3328, 8), 8), ((4096, 4096, 1856, 8), 8)]:
        got = i8(lib, *call)[1]
        assert got["workgroups"] == 256 and got["r_in_k_loop"] == group and got["r_bypass"] in (0, 1), (call, got)
    assert i8(lib, 8192, 8192, 1792, 8)[1] == {"rows": 8192, "workgroups": 256}
    assert i8(lib, 4096, 4096, 1792, 8)[1] == {"rows": 4096}
    # R written: nothing of it is read
    assert kernel(lib, lambda: lib.amulet_count_i8_assign(8, 8192, 8192, 4096, ptr(), 4096, ptr(), 8192, ptr(), 8192, None))[1] == {"rows": 8192, "workgroups": 256}


def test_a_join_count_that_fits_the_caches_writes_r_through_them(lib):
    """us repeated on the same matrices, the tile kernels / R around the caches / written through them: 4352 x 4096 x 3392 83 / 86 / 78,
    5120 x 4096 x 2560 72 / 75 / 70, 4608 x 4608 x 3072 77 / 80 / 74; 7168 x 8192 x 2432 with other matrices 161 (persistent) / 150 / 167."""
    for call in [(4352, 4096, 3392), (5120, 4096, 2560), (4608, 4608, 3072), (8448, 4096, 4096), (8192, 4096, 1856)]:
        assert i8(lib, *call)[1]["r_bypass"] == 0, call
    for call in [(7168, 8192, 2432), (4096, 4096, 4096), (6144, 8192, 4096), (8192, 8192, 1856), (8192, 8192, 4096)]:
        assert i8(lib, *call)[1]["r_bypass"] == 1, call


def test_a_tall_join_count_whose_rows_of_r_share_channels_keeps_the_phases(lib):
    """us, the persistent kernel / R read during the K loop: 16384 x 8192 x 2560 317 / 340, 24576 x 8192 x 2176 423 / 462, 16384^2 x 2176 570 / 599,
    28672 x 4096 x 2560 300 / 328; by a few rows or k less or more, or with rows of R at another pitch, the second is level or ahead."""
    def fields(M, N, K, ldr=None):
        return kernel(lib, lambda: lib.amulet_count_i8(M, N, K, ptr(), K, ptr(), N, ptr(), ldr or N, None))[1]
    for call in [(16384, 8192, 2560), (24576, 8192, 2176), (12288, 8192, 3328), (16384, 16384, 2176), (28672, 4096, 2560), (16384, 7936, 2560, 8192)]:
        assert fields(*call) == {"rows": call[0], "workgroups": 256}, call
    for call in [(16384, 8192, 2560, 8192 + 64), (12032, 8192, 2560), (16384, 8192, 3392), (16384, 16384, 2560), (24320, 4096, 2560), (12288, 12288, 2176),
                 (12288, 32768, 2176), (16384, 8192, 1984)]:
        assert "r_in_k_loop" in fields(*call), call


def test_stages_of_128_k_of_operands_across_k_want_rows_of_whole_lines(lib):
    """A transposed, B not, a short last stage: 128 k a stage where rows of A or B are multiples of 64 bytes apart, else 64
    (7000 x 300 x 5040 31.8 us by 64 k, 33.3 by 128).  K in whole stages, or an operand along k: 128 at any pitch."""
    def stage(tA, tB, M, N, K, lda, ldb):
        name, got = kernel(lib, lambda: lib.amulet_count_i8_general(tA, tB, M, N, K, ptr(), lda, ptr(), ldb, ptr(), N, ptr(), 1 << 30, None))
        assert name == "i8_tile_128x128" and got["parts"] == 1
        return got.get("stage_k", 64)
    for M, N, K in [(7000, 300, 5040), (300, 7000, 2500), (1500, 1500, 5040), (1200, 2600, 3564)]:
        assert stage(1, 0, M, N, K, M, N) == 64
        assert stage(1, 0, M, N, K, (M + 63) // 64 * 64, N) == 128 and stage(1, 0, M, N, K, M, (N + 63) // 64 * 64) == 128
        assert stage(1, 0, M, N, 4096, M, N) == 128
        assert stage(0, 0, M, N, K, K, N) == 128 and stage(1, 1, M, N, K, M, K) == 128
    assert stage(1, 0, 448, 5012, 5040, 448, 5012) == 128


def test_written_counts_have_k_in_parts_where_that_is_ahead(lib):
    """us, K in parts / whole: 470 x 512 x 3520 9.3 / 12.3, 282 x 5756 x 13692 81 / 101, 408 x 4604 x 12703 66 / 78, 192 x 6592 x 3072 24 / 28, 256 x 8644 x 14957 81 / 97;
    4677 x 960 x 15908 155 / 111, 6428 x 728 x 6272 115 / 100, 2048 x 2289 x 6528 84 / 67, 1024 x 1856 x 5120 29 / 23, 512 x 2368 x 3968 21 / 18."""
    def parts(M, N, K, at):
        return kernel(lib, lambda: lib.amulet_count_i8_assign(-1, M, N, K, ptr(at), K, ptr(at), N, ptr(), N, None))[1]["parts"]
    odd, even = (1 << 20) + 1, 1 << 20
    for M, N, K, at in [(470, 512, 3520, even), (282, 5756, 13692, odd), (408, 4604, 12703, even), (192, 6592, 3072, odd), (256, 8644, 14957, even), (2124, 1000, 19900, even)]:
        assert parts(M, N, K, at) > 1, (M, N, K)
    for M, N, K, at in [(4677, 960, 15908, even), (6428, 728, 6272, odd), (2048, 2289, 6528, even), (1024, 1856, 5120, even), (512, 2368, 3968, even), (64, 64, 256, even)]:
        assert parts(M, N, K, at) == 1, (M, N, K)


def test_named_phases_run_the_kernel_that_has_them(lib, monkeypatch):
    """AMULET_I8_PHASES is about the persistent kernel's write-backs: set, that kernel runs where the one without phases
    would, and where tile kernels were taken before that one they are; a value that is out of range is as if it were not set."""
    for phases, named in [("8,2,2,16", True), ("1,0,1,0", True), ("0,2,2,16", False), ("8,2", False)]:
        monkeypatch.setenv("AMULET_I8_PHASES", phases)
        for call in [(8192, 8192, 4096), (8192, 8192, 2048), (8192, 8192, 4096, 8)]:
            got = i8(lib, *call)[1]
            assert got["workgroups"] == 256 and ("r_in_k_loop" in got) == (not named), (phases, call, got)
        assert i8(lib, 4096, 4096, 4096)[0].startswith("i8_tile_") == named


def test_earlier_launches_stay_readable_and_are_the_threads_own(lib):
    import threading
    f32(lib, 1, 300, 256, 256)
    f32(lib, 1, 301, 256, 256, 3)
    assert am.amulet_recent_kernel(0) == "valu_32x512_k8 rows 301" and am.amulet_recent_kernel(1).split()[2] == "300"
    assert am.amulet_recent_kernel(-1) == "" and am.amulet_recent_kernel(16) == ""
    seen = []
    t = threading.Thread(target=lambda: seen.append(am.amulet_recent_kernel()))
    t.start()
    t.join()
    assert seen == [""]


def _wide_parts(f64_, task, M, N, K):
    """K parts of the wide kernels' own rule: none above 2048 waves or below 128 k; fp32 fills the chip to three
    waves per SIMD (four from 1024 waves on) with parts of at least 64 k, about 192 from K = 512; fp64 to four,
    with at least 64 k each, in whole stages."""
    if f64_:
        nw = 8 if task == 2 and 1024 ** 2 <= M * N <= 2048 ** 2 else 4
        rows, cols, unit = 4 * nw, 128, 16
    else:
        tiles = -(-M // 32) * -(-N // 256)
        nw = 8 if tiles >= 512 or (tiles >= 128 and K >= 8192) else 4
        rows, cols, unit = 4 * nw, 256, 64
    waves = -(-M // rows) * -(-N // cols) * nw
    if waves > 2048 or K < 128:
        return 1
    if f64_:
        want = min(4096 // waves, K // 64, 1024)
    else:
        want = max(1, min((4096 if waves >= 1024 else 3072) // waves, K // 64 if K < 512 else (K + 96) // 192, 1024))
    return -(-K // (-(-(-(-K // want)) // unit) * unit))


def test_tile_kernels_split_k_no_finer_than_the_wide_ones(lib):
    """Every part of a split K is one more rounding of each result, in an order that varies: the tile
    kernels' plans may not have more parts than the wide kernels they stand in for (64 x 64 x 1024 had
    32 for 4, 5018 x 590 x 6504 3 for none), and none in the deterministic mode."""
    import random
    rng = random.Random(3)
    sizes = [(64, 64, 1024), (64, 64, 2048), (5018, 590, 6504), (64, 64, 256), (16, 64, 8192), (73, 64, 832), (2880, 568, 6178)]
    sizes += [tuple(int(round(64 * 128 ** rng.random())) for _ in range(3)) for _ in range(150)]
    tiles = 0
    for call, is64 in ((f32, False), (f64, True)):
        for M, N, K in sizes:
            for task in (1, 2, 3):
                name, got = call(lib, task, M, N, K)
                if "tile" not in name:
                    continue
                tiles += 1
                assert got["parts"] <= _wide_parts(is64, task, M, N, K), (name, task, M, N, K, got)
                assert got["parts"] * got["kpart"] >= K > (got["parts"] - 1) * got["kpart"]
    assert tiles > 600
    was = am.amulet_get_deterministic()
    try:
        am.amulet_set_deterministic(True)
        assert f32(lib, 1, 64, 64, 1024)[1]["parts"] == 1 and f64(lib, 1, 64, 64, 1024)[1]["parts"] == 1
    finally:
        am.amulet_set_deterministic(was)
