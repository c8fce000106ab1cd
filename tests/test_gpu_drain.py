"""The drain pass and the completion path at their edges (GPU)."""
import numpy as np
import pytest

import oracle
from paper_1505_07368_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cg():
    from paper_1505_07368_amd import binding
    return binding


def _mandel(cg, s, a, rows, width=32):
    """A message of ceil(2 ceil(rows / 4) / 16) work tiles (1024 pixels each) over
    the boundary, and its reply from the oracle."""
    vp = gen.Viewport(-1.5, -1.0, 2.0 / width, 2.0 / rows, width, rows, 60)
    ref = oracle.mandelbrot(vp.re_min, vp.im_min, vp.step_re, vp.step_im, width, 0, rows, 60, "f32")
    return s.request(a, cg.mandel_args(vp)), ref


@pytest.mark.parametrize("rows", [[256, 257, 250, 4], [257], [2000, 256, 8, 8001, 257, 1],
                                  [300] * 40 + [8] * 40])
def test_tile_map_by_one_thread_and_by_the_workgroup(cg, rows):
    """Messages of 8 tiles (256 rows: one thread writes their map), 9 (257:
    the workgroup does) and more, alone and mixed in one drain pass."""
    with cg.System(mode="batched", arena_bytes=64 << 20, mandel_tile_px=1024) as s:
        a = s.spawn(cg.BHV_MANDELBROT)
        assert s.hold(True) == cg.OK
        sent = [_mandel(cg, s, a, r) for r in rows]
        assert s.hold(False) == cg.OK
        for (f, ref), r in zip(sent, rows):
            st, img = f.result()
            assert st == cg.OK
            got = img.cpu().numpy().reshape(r, 32)
            assert (got == ref).all(), (r, int((got != ref).sum()))
            f.release()


@pytest.mark.parametrize("fp", ["f32", "f64"])
@pytest.mark.parametrize("width,rows,max_iter", [(64, 64, 100), (67, 67, 110), (33, 125, 240),
                                                 (1, 1, 9), (5, 4097, 50), (129, 130, 700)])
def test_tiles_grow_with_the_load(cg, width, rows, max_iter, fp):
    """Counts are exact at every work-tile size that the load at submission
    chooses, from the first message (1024 pixels) to the last of many (4096
    where a tile is cheap)."""
    vp = gen.Viewport(-2.0, -1.25, 2.5 / width, 2.5 / rows, width, rows, max_iter)
    ref = oracle.mandelbrot(vp.re_min, vp.im_min, vp.step_re, vp.step_im, width, 0, rows,
                            max_iter, fp)
    with cg.System(mode="batched", arena_bytes=256 << 20) as s:
        a = s.spawn(cg.BHV_MANDELBROT)
        assert s.hold(True) == cg.OK
        args = cg.mandel_args(vp, fp=cg.F64 if fp == "f64" else cg.F32)
        sent = [s.request(a, args) for _ in range(400)]
        assert s.hold(False) == cg.OK
        for f in sent:
            st, img = f.result()
            assert st == cg.OK and (img.cpu().numpy().reshape(rows, width) == ref).all()
            f.release()
