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
