"""Replies: slots handed out again, several host threads on one system (GPU)."""
import threading

import numpy as np
import pytest

import oracle
from paper_1505_07368_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["batched", "persistent"])
@pytest.mark.parametrize("slots", [2, 8])
def test_a_slot_handed_out_again_starts_clean(mode, slots):
    """A completion record lets the host reuse the slot at once: the next
    message must find its tile count and status reset.  Messages of many
    tiles, failing ones and single ones in turn through few slots."""
    import torch
    from paper_1505_07368_amd import binding as cg
    vp = gen.tiny_viewport()
    rows = np.array([(vp.re_min, vp.im_min, vp.step_re, vp.step_im, 512, 512, r, 16, 100, cg.F32)
                     for r in range(0, 512, 16)], cg.NP_MANDEL)
    with cg.System(mode=mode, arena_bytes=16 << 20, ring_slots=slots, mandel_tile_px=256) as s:
        m, bad = s.spawn(cg.BHV_MANDELBROT), s.spawn(cg.BHV_FAULT)
        n = 30 * len(rows)
        out = torch.zeros((len(rows), 16, 512), dtype=torch.int16, device="cuda")
        msgs = np.zeros(n, cg.NP_MSG)
        k = np.arange(n)
        works = k % 3 != 1  # every third message fails
        at = k % len(rows)
        msgs["actor"] = np.where(works, m, bad)
        msgs["args"][works] = rows.ctypes.data + at[works].astype(np.uint64) * rows.itemsize
        msgs["args_bytes"][works] = rows.itemsize
        msgs["out"]["data"][works] = out.data_ptr() + at[works].astype(np.uint64) * (16 * 512 * 2)
        msgs["out"]["numel"][works] = 16 * 512
        msgs["out"]["dtype"][works] = cg.U16
        msgs["out"]["on_device"][works] = 1
        _, _, st, _ = cg.drive_array(s, msgs, (rows, out), window=slots)
        assert (st == np.where(works, cg.OK, cg.E_FAULT)).all(), np.unique(st)
        stats = s.stats()
        assert stats["completions"] == n and stats["duplicate_completions"] == 0
    ref = oracle.mandelbrot(vp.re_min, vp.im_min, vp.step_re, vp.step_im, 512, 0, 512, 100)
    assert (out.cpu().numpy().reshape(512, 512).view(np.uint16) == ref).all()
