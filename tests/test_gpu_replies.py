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


def _run_all(threads, limit=60):
    """Runs the functions, each in a thread; re-raises what one raised."""
    errors = []

    def guarded(f):
        try:
            f()
        except BaseException as e:  # noqa: BLE001 - handed to the test
            errors.append(e)
    ts = [threading.Thread(target=guarded, args=(f,), daemon=True) for f in threads]
    for t in ts:
        t.start()
    for t in ts:
        t.join(limit)
        assert not t.is_alive(), "a thread still waits"
    if errors:
        raise errors[0]


@pytest.mark.parametrize("mode", ["plain", "batched", "persistent"])
def test_waiters_pollers_and_drivers_on_one_system(mode):
    """The completion ring is read by whichever thread waits: three that wait
    for each reply, one that polls, one that waits with time-outs too short to
    be met, and two that drive windows.  Every reply arrives once, where it
    belongs."""
    from paper_1505_07368_amd import binding as cg
    with cg.System(mode=mode, arena_bytes=64 << 20, ring_slots=64) as s:
        echo = s.spawn(cg.BHV_NOOP)
        fault = s.spawn(cg.BHV_FAULT)
        rounds = 150

        def waits(base):
            def go():
                for i in range(rounds):
                    f = s.request(echo, inputs=[np.array([base, i], np.int32)])
                    st, v = f.result(30)
                    assert st == cg.OK and v.tolist() == [base, i]
                    f.release()
            return go

        def fails():
            for _ in range(rounds):
                f = s.request(fault)
                assert f.result(30)[0] == cg.E_FAULT
                f.release()

        def polls():
            for i in range(rounds):
                f = s.request(echo, inputs=[np.array([-i], np.int32)])
                got = f.poll()
                while not got[0]:
                    got = f.poll()
                assert got[1] == cg.OK and s.view(got[2]).tolist() == [-i]
                f.release()

        def gives_up():
            for i in range(rounds):
                f = s.request(echo, inputs=[np.array([i], np.int32)])
                try:
                    assert f.wait(1e-7)[0] == cg.OK
                except cg.CafError as e:
                    assert e.status == cg.E_TIMEOUT
                f.release()

        def drives(n):
            def go():
                xs = np.arange(2 * n, dtype=np.int32)
                bufs = np.zeros(n, cg.NP_BUF)
                bufs["data"] = xs.ctypes.data + np.arange(n, dtype=np.uint64) * 8
                bufs["numel"], bufs["dtype"] = 2, cg.I32
                msgs = np.zeros(n, cg.NP_MSG)
                msgs["actor"], msgs["n_in"] = echo, 1
                msgs["in_"] = bufs.ctypes.data + np.arange(n, dtype=np.uint64) * bufs.itemsize
                for _ in range(5):
                    rc, lat, st, _ = cg.drive_array(s, msgs, (xs, bufs), window=16)
                    assert rc == cg.OK and (st == cg.OK).all() and (lat > 0).all()
            return go

        _run_all([waits(1), waits(2), fails, polls, gives_up, drives(300), drives(70)])
        assert s.drain() == cg.OK
        stats = s.stats()
        assert stats["requests"] == stats["completions"] == 5 * rounds + 5 * 370
        assert stats["duplicate_completions"] == 0 and stats["outstanding"] == 0


@pytest.mark.parametrize("pause", [0.0, 0.01])
def test_shutdown_while_threads_wait(pause):
    """Threads inside a wait (pause: some of them past its first part) when
    the system goes: each gets CAF_E_QUIT and releases its future, beside the
    rest of the shutdown."""
    import time

    from paper_1505_07368_amd import binding as cg
    for _ in range(8):
        s = cg.System(mode="batched", arena_bytes=16 << 20, ring_slots=64)
        e = s.spawn(cg.BHV_NOOP)
        assert s.request(e, inputs=[np.array([5], np.int32)]).result()[0] == cg.OK
        assert s.drain() == cg.OK
        s.drain_kernel_ms()  # waits for the launch to end: a hold starts no other
        assert s.hold(True) == cg.OK
        futs = [s.request(e, inputs=[np.array([i], np.int32)]) for i in range(12)]
        started = threading.Barrier(5)

        def waits(mine):
            def go():
                started.wait()
                for f in mine:
                    assert f.wait(30.0)[0] == cg.E_QUIT
                    f.release()
            return go

        def ends():
            started.wait()
            time.sleep(pause)
            s.shutdown()

        _run_all([waits(futs[k::4]) for k in range(4)] + [ends])
