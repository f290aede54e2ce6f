"""The compiled argument marshalling against the Python one: same results for ordinary arguments,
in every form and layout, on a side stream, on views and on single rows and columns; same errors for
the others."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def am():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_08872_amd as am
    am.load_library()
    from paper_2305_08872_amd import binding
    assert binding._marshal is not None, "the compiled marshalling is not built"
    return am


def _calls(am, M, N, K, tA, tB, form, stream):
    """(name, call on R, dtype of R) of each entry point that goes through it."""
    g = torch.Generator(device="cuda").manual_seed(1000 * M + N)

    def ints(dt, *shape):
        rows, cols = shape if len(shape) == 2 else (1, shape[0])
        t = torch.randint(-5, 6, (rows, cols + 3), generator=g, device="cuda").to(dt)[:, :cols]   # a view
        return t if len(shape) == 2 else t[0].contiguous()

    for dt in (torch.float32, torch.float64):
        A, B = ints(dt, K, M) if tA else ints(dt, M, K), ints(dt, N, K) if tB else ints(dt, K, N)
        th = ints(dt, *{0: (N,), 1: (M,), 2: (1,), 3: (M, N)}[form])
        dis = ints(dt, N) / 8
        fn = am.amulet_mmlike_f32_general if dt == torch.float32 else am.amulet_mmlike_f64
        for task in range(4):
            yield fn.__name__, lambda R, task=task, fn=fn, A=A, B=B, th=th, dis=dis: fn(
                task, A, B, th, dis, R, thres_form=form, trans_a=tA, trans_b=tB, stream=stream), dt
        if dt == torch.float32 and not tA and not tB and form == 0:
            for task, P in ((0, None), (1, torch.stack([th, dis])), (2, th), (3, th)):
                yield "amulet_mmlike_f32", lambda R, task=task, P=P, A=A, B=B: am.amulet_mmlike_f32(task, A, B, P, R, stream), dt
    A, B = ints(torch.int8, K, M) if tA else ints(torch.int8, M, K), ints(torch.int8, N, K) if tB else ints(torch.int8, K, N)
    ws = torch.empty(am.amulet_count_i8_repack_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    yield "amulet_count_i8_general", lambda R: am.amulet_count_i8_general(A, B, R, ws, trans_a=tA, trans_b=tB, stream=stream), torch.int32
    if not tA and not tB:
        yield "amulet_count_i8", lambda R: am.amulet_count_i8(A, B, R, stream), torch.int32
        yield "amulet_count_i8_assign", lambda R: am.amulet_count_i8_assign(A, B, R, stream=stream), torch.int32


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (1, 7, 70), (9, 1, 65), (33, 70, 20)])
@pytest.mark.parametrize("layout", [(False, False), (True, True), (False, True)])
def test_compiled_marshalling_reads_what_the_python_one_reads(am, monkeypatch, M, N, K, layout):
    from paper_2305_08872_amd import binding
    own = torch.cuda.Stream()
    for form in range(4):
        for stream in (None, own, own.cuda_stream):
            for name, call, dt in _calls(am, M, N, K, layout[0], layout[1], form, stream):
                print(name, M, N, K, layout, form, flush=True)
                out = []
                for compiled in (True, False):
                    R = torch.arange(M * (N + 1), device="cuda").to(dt).view(M, N + 1)[:, :N]
                    torch.cuda.synchronize()
                    with monkeypatch.context() as m:
                        if not compiled:
                            m.setattr(binding, "_marshal", None)
                        call(R)
                    torch.cuda.synchronize()
                    out.append(R.clone())
                assert torch.equal(out[0], out[1]), (name, form)


def test_what_the_compiled_marshalling_does_not_take_raises_as_before(am):
    x, y, z = torch.zeros(4, 4, device="cuda"), torch.zeros(5, 4, device="cuda"), torch.zeros(4, 4)
    for bad in (lambda: am.amulet_mmlike_f32(0, x, y, None, x), lambda: am.amulet_mmlike_f32(0, x.double(), x, None, x),
                lambda: am.amulet_mmlike_f32(0, z, x, None, x), lambda: am.amulet_mmlike_f32(2, x, x, z[0], x),
                lambda: am.amulet_mmlike_f32(0, x.t(), x, None, x), lambda: am.amulet_count_i8(x, x, x),
                lambda: am.amulet_mmlike_f32_general(2, x, x, y, None, x, thres_form=3),
                lambda: am.amulet_mmlike_f64(1, x.double(), x.double(), x.double()[0], None, x.double())):
        with pytest.raises(ValueError):
            bad()
    with pytest.raises(am.AmuletError):
        am.amulet_mmlike_f32(9, x, x, None, x)
    with pytest.raises(am.AmuletError):
        am.amulet_mmlike_f32(2, x, x, None, x)
