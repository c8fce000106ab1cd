"""The elementwise and the row actor at the edges of their tiles (GPU).

tanh: ROCm's tanhf, within 4 units in the last place.  Row sums: every order
of summation is within (cols + 8) 2^-24 of the sum of magnitudes (as many
roundings as additions); a chain's row sums of tanh add tanh's own 4 units.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 3), (3, 5), (1, 4096), (2, 4097), (5, 1023), (16, 256), (17, 255), (33, 4100),
          (257, 64), (1000, 1), (4099, 513), (3, 300001)]
ULP = 2.0 ** -23


@pytest.fixture(scope="module", params=["batched", "plain"])
def sysm(request):
    from paper_1505_07368_amd import binding as cg
    s = cg.System(mode=request.param, arena_bytes=256 << 20)
    yield s
    s.shutdown()


@pytest.mark.parametrize("offset", [0, 1])
def test_shapes(sysm, offset):
    """offset: the matrix starts that many floats into an allocation."""
    import torch
    from paper_1505_07368_amd import binding as cg
    th, rs = sysm.spawn(cg.BHV_TANH), sysm.spawn(cg.BHV_ROWSUM)
    fwd = sysm.spawn(cg.BHV_TANH, forward_to=rs)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    for rows, cols in SHAPES:
        whole = torch.randn(rows * cols + offset, generator=g, device="cuda") * 2
        x = whole[offset:]
        out = torch.full((rows * cols + offset,), 7.0, device="cuda")[offset:]
        torch.cuda.synchronize()
        a = cg.caf_shape_args(rows, cols)
        f = [sysm.request(th, a, inputs=[x], out=out), sysm.request(rs, a, inputs=[x]),
             sysm.request(fwd, a, inputs=[x])]
        got = [r.result() for r in f]
        assert [st for st, _ in got] == [cg.OK] * 3, (rows, cols)
        xd = x.double().view(rows, cols)
        t = torch.tanh(xd)
        assert ((out.double().view(rows, cols) - t).abs() <= 4 * ULP * t.abs()).all(), (rows, cols)
        mag = xd.abs().sum(1)
        assert ((got[1][1].double() - xd.sum(1)).abs() <= (cols + 8) * ULP / 2 * mag).all()
        mag = t.abs().sum(1)
        assert ((got[2][1].double() - t.sum(1)).abs() <= ((cols + 8) / 2 + 4) * ULP * mag).all()


def test_fused_chain_asks_whether_the_row_actor_lives():
    """A chain whose last actor quits while the messages wait is answered with
    an error, also where its last two stages run as one."""
    import torch
    from paper_1505_07368_amd import binding as cg
    with cg.System(mode="batched", arena_bytes=64 << 20) as s:
        rs = s.spawn(cg.BHV_ROWSUM)
        th = s.spawn(cg.BHV_TANH, forward_to=rs)
        gm = s.spawn(cg.BHV_GEMM, forward_to=th)
        A = torch.rand(64 * 64, device="cuda")
        torch.cuda.synchronize()
        assert s.hold(True) == cg.OK
        f = [s.request(gm, cg.caf_gemm_args(64, cg.F32), inputs=[A, A]) for _ in range(3)]
        s.quit(rs)
        assert s.hold(False) == cg.OK
        assert [r.result()[0] for r in f] == [cg.E_QUIT] * 3


@pytest.mark.parametrize("rows,cols", [(8191, 401), (5, 1048579), (2000003, 3), (4097, 4100)])
def test_matrices_of_several_tiles_per_claim(sysm, rows, cols):
    """Work tiles larger than the smallest: ragged last tiles, few long rows,
    many short ones."""
    import torch
    from paper_1505_07368_amd import binding as cg
    th, rs = sysm.spawn(cg.BHV_TANH), sysm.spawn(cg.BHV_ROWSUM)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn(rows * cols, generator=g, device="cuda")
    out = torch.full((rows * cols,), 7.0, device="cuda")
    torch.cuda.synchronize()
    a = cg.caf_shape_args(rows, cols)
    f = [sysm.request(th, a, inputs=[x], out=out), sysm.request(rs, a, inputs=[x])]
    got = [r.result() for r in f]
    assert [st for st, _ in got] == [cg.OK] * 2
    t = torch.tanh(x.double())
    assert ((out.double() - t).abs() <= 4 * ULP * t.abs()).all()
    xd = x.double().view(rows, cols)
    assert ((got[1][1].double() - xd.sum(1)).abs() <= (cols + 8) * ULP / 2 * xd.abs().sum(1)).all()


@pytest.mark.parametrize("mode", ["plain", "batched"])
def test_messages_of_too_many_tiles_are_refused(mode):
    """A message has at most 2^20 tiles, of 4096 elements, 16 rows or 1024
    pixels (512 in plain mode), whatever tiles it would be cut into.  (Their replies exceed the
    arena too, which is another refusal.)"""
    import torch
    from paper_1505_07368_amd import binding as cg
    few = torch.zeros(16, device="cuda")
    with cg.System(mode=mode, arena_bytes=16 << 20) as s:
        for bhv, rows, cols in ((cg.BHV_TANH, 65537, 65536), (cg.BHV_ROWSUM, (1 << 24) + 16, 1)):
            buf = cg.caf_buf(few.data_ptr(), rows * cols, cg.F32, 1)
            rc, f = s.request_raw(s.spawn(bhv), cg.caf_shape_args(rows, cols), inputs=[buf])
            assert rc == cg.E_INVALID and f is None, (bhv, rc)
        big = cg.caf_mandel_args(-2.0, -1.0, 1e-6, 1e-6, 1 << 20, 1025, 0, 1025, 10, cg.F32)
        rc, f = s.request_raw(s.spawn(cg.BHV_MANDELBROT), big)
        assert rc == cg.E_INVALID and f is None, rc


@pytest.mark.parametrize("gemm,wgs", [(False, 0), (True, 2), (True, 3)])
def test_tiles_follow_the_load_and_the_variant(gemm, wgs):
    """Work tiles grow with the messages out, and are cut for the drain
    variant that runs (a GEMM actor exists or not): the same matrices alone
    and behind a queue, whose last tiles are partial, of rows shorter than a
    vector, of few long rows."""
    import torch
    from paper_1505_07368_amd import binding as cg
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    with cg.System(mode="batched", arena_bytes=1 << 30, full_wgs_per_cu=wgs) as s:
        if gemm:
            s.spawn(cg.BHV_GEMM)
        th, rs = s.spawn(cg.BHV_TANH), s.spawn(cg.BHV_ROWSUM)
        cases = []
        for rows, cols in ((257, 1001), (13, 16384), (70001, 1), (5003, 63)):
            x = torch.rand(rows * cols, generator=g, device="cuda") * 4 - 2
            torch.cuda.synchronize()
            cases.append((rows, cols, x, x.double().view(rows, cols)))
        for copies in (1, 24):
            s.hold(True)
            futs = [(c, s.request(th, cg.caf_shape_args(*c[:2]), inputs=[c[2]]),
                     s.request(rs, cg.caf_shape_args(*c[:2]), inputs=[c[2]]))
                    for _ in range(copies) for c in cases]
            s.hold(False)
            for (rows, cols, _, ref), ft, fr in futs:
                (st, t), (sr, r) = ft.result(), fr.result()
                assert st == cg.OK and sr == cg.OK
                want = torch.tanh(ref)
                assert ((t.double().view(rows, cols) - want).abs() <= 4 * ULP * want.abs()).all()
                off = (r.double() - ref.sum(1)).abs()
                assert (off <= (cols + 8) * 2.0 ** -24 * ref.abs().sum(1)).all(), (rows, cols)
                ft.release()
                fr.release()
