"""Performance cases: what a program does with the compute actors, over the
range of sizes, types and options in use.

A case names one kind of work.  ``prepare`` makes what the program holds
before the call (a running System, the messages, their inputs and reply
buffers in device memory), ``run`` is one pass through the public entry
points (the native driver, or a request and its future), ``work`` the bytes
and operations the pass cannot do without, ``exact`` the same replies from
float64.  Escape counts and colours are whole numbers and have no other
reference than themselves.

A program has one System and sends it many messages, so the System is kept
between states of one configuration.
"""
import math

import numpy as np
import torch

from paper_1505_07368_amd import binding as cg
from paper_1505_07368_amd import gen

F32, F64, BF16 = "f32", "f64", "bf16"
OPS_PER_ITER = 9  # 3 multiplies, 5 adds or subtracts, one compare
COST = {"image": 8 * 1920 * 1080 * 1000, "tiles": 4096 * 64 * 64 * 100, "gemm": 3.2e11,
        "gemm_bytes": 4.3e9, "chain": 4096 * 2 * 128 ** 3, "stage": 1 << 26}


def listed():
    return [
        # the smallest call: one int32 to an actor and back, waited for
        {"name": "echo_one", "kind": "echo", "count": 1, "len": 1},
        # many small messages: 64 x 64 tiles of the 512 x 512 viewport
        {"name": "tiles_64", "kind": "tiles", "count": 4096, "side": 64, "max_iter": 100,
         "window": 256},
        # the image batch: eight boundary viewports in row tiles of 64
        {"name": "image_f32", "kind": "image", "images": 8, "width": 1920, "height": 1080,
         "max_iter": 1000, "tile_rows": 64, "fp": F32, "colour": False, "view": 0,
         "mode": "batched"},
        # the same in double, for deep zooms
        {"name": "image_f64", "kind": "image", "images": 8, "width": 1920, "height": 1080,
         "max_iter": 1000, "tile_rows": 64, "fp": F64, "colour": False, "view": 0,
         "mode": "batched"},
        # one odd-sized colour picture as one message: a viewer's redraw
        {"name": "image_colour_odd", "kind": "image", "images": 1, "width": 1021, "height": 773,
         "max_iter": 300, "tile_rows": 773, "fp": F32, "colour": True, "view": 2,
         "mode": "batched"},
        # the grouped products: 4,096 requests of 64 to 512, both input types
        {"name": "gemm_f32_mix", "kind": "gemm", "dtype": F32, "sizes": "mix", "lo": 64, "hi": 512,
         "count": 4096, "tuned": True, "mode": "batched"},
        {"name": "gemm_bf16_mix", "kind": "gemm", "dtype": BF16, "sizes": "mix", "lo": 64,
         "hi": 512, "count": 4096, "tuned": True, "mode": "batched"},
        # products of any size, odd ones too, as a program's data gives them
        {"name": "gemm_f32_ragged", "kind": "gemm", "dtype": F32, "sizes": "ragged", "lo": 17,
         "hi": 500, "count": 512, "tuned": False, "mode": "batched"},
        # one large product
        {"name": "gemm_bf16_large", "kind": "gemm", "dtype": BF16, "sizes": "one", "lo": 4096,
         "hi": 4096, "count": 1, "tuned": False, "mode": "batched"},
        # product -> tanh -> row sums, forwarded on the device
        {"name": "chains_128", "kind": "chain", "n": 128, "count": 4096, "window": 1024},
        # the serving mix: 70 % escape-time squares, 30 % products
        {"name": "serving_mix", "kind": "mix", "count": 2000, "window": 1024, "view": 7},
        # a large matrix through the elementwise and the row actor
        {"name": "stages_large", "kind": "stage", "rows": 8192, "cols": 4100},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["echo", "tiles", "image", "image", "image", "gemm", "gemm", "gemm", "gemm",
                       "chain", "mix", "stage"])
    if kind == "echo":
        return {"kind": kind, "count": _log(rng, 1, 32), "len": rng.randint(1, 4)}
    if kind == "tiles":
        side, mi = _log(rng, 16, 128), _log(rng, 50, 400)
        most = max(16, int(COST["tiles"] / (side * side * mi)))
        return {"kind": kind, "count": _log(rng, 16, min(4096, most)), "side": side,
                "max_iter": mi, "window": rng.choice([64, 256, 1024])}
    if kind == "image":
        w, h, mi = _log(rng, 201, 1920), _log(rng, 150, 1080), _log(rng, 100, 2000)
        most = max(1, min(8, int(COST["image"] / (w * h * mi))))
        return {"kind": kind, "images": rng.randint(1, most), "width": w, "height": h,
                "max_iter": mi, "tile_rows": rng.choice([16, 33, 64, h]),
                "fp": rng.choice([F32, F32, F64]), "colour": rng.random() < 0.25,
                "view": rng.randrange(1000),
                "mode": rng.choice(["batched", "batched", "batched", "plain"])}
    if kind == "gemm":
        dtype, sizes = rng.choice([F32, BF16]), rng.choice(["mix", "one", "ragged"])
        if sizes == "mix":
            lo, hi = 64, 512
        elif sizes == "one":
            lo = hi = _log(rng, 32, 2048 if dtype == F32 else 4096)
        else:
            lo = _log(rng, 1, 100)
            hi = _log(rng, lo + 30, 600)
        top = max(1, min(4096, int(min(COST["gemm"] / (2 * hi ** 3), COST["gemm_bytes"] / (12 * hi * hi)))))
        return {"kind": kind, "dtype": dtype, "sizes": sizes, "lo": lo, "hi": hi,
                "count": _log(rng, min(top, 8 if hi <= 600 else 1), top),
                "tuned": rng.random() < 0.5, "mode": "batched"}
    if kind == "chain":
        n = _log(rng, 32, 512)
        top = max(8, min(4096, int(COST["chain"] / (2 * n ** 3))))
        return {"kind": kind, "n": n, "count": _log(rng, 8, top), "window": rng.choice([64, 1024])}
    if kind == "mix":
        return {"kind": kind, "count": _log(rng, 100, 2000), "window": rng.choice([256, 1024]),
                "view": rng.randrange(1000)}
    rows, cols = _log(rng, 64, 16384), _log(rng, 64, 16384)
    rows = max(1, min(rows, COST["stage"] // 2 // cols))
    return {"kind": kind, "rows": rows, "cols": cols}


# ---- the System a program keeps ------------------------------------------

_KEPT = {}


def _system(**cfg):
    """The System of this configuration: one at a time, as in a program."""
    key = tuple(sorted(cfg.items()))
    if key not in _KEPT:
        for s, _ in _KEPT.values():
            s.shutdown()
        _KEPT.clear()
        _KEPT[key] = (cg.System(**cfg), {})
    return _KEPT[key]


def _actor(kept, behavior, **kw):
    s, actors = kept
    key = (behavior,) + tuple(sorted(kw.items()))
    if key not in actors:
        actors[key] = s.spawn(behavior, **kw)
    return actors[key]


def _rand(seed, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand(n, generator=g, device="cuda") * 2 - 1


def _messages(args, actor):
    msgs = np.zeros(args.size, cg.NP_MSG)
    msgs["actor"] = actor
    msgs["args"] = args.ctypes.data + np.arange(args.size, dtype=np.uint64) * args.itemsize
    msgs["args_bytes"] = args.itemsize
    return msgs


def _inputs(msgs, ptrs, numel, dtype):
    """Device inputs: ptrs [messages, inputs]."""
    k = ptrs.shape[1]
    bufs = np.zeros(ptrs.size, cg.NP_BUF)
    bufs["data"] = ptrs.reshape(-1)
    bufs["numel"] = np.repeat(numel, k)
    bufs["dtype"] = dtype
    bufs["on_device"] = 1
    msgs["n_in"] = k
    msgs["in_"] = bufs.ctypes.data + np.arange(len(msgs), dtype=np.uint64) * (k * bufs.itemsize)
    return bufs


def _outputs(msgs, base, offs, numel, dtype, esz):
    msgs["out"]["data"] = base + offs.astype(np.uint64) * esz
    msgs["out"]["numel"] = numel
    msgs["out"]["dtype"] = dtype
    msgs["out"]["on_device"] = 1


def _offsets(numel):
    """Start of each buffer in one allocation, 128 elements apart or more, as
    an allocator aligns them."""
    room = (np.asarray(numel, np.int64) + 127) // 128 * 128
    return np.concatenate([[0], np.cumsum(room)[:-1]]).astype(np.int64)


def _total(numel):
    return int(_offsets(np.append(numel, 0))[-1])


# ---- escape-time geometry --------------------------------------------------

def _image_args(case, pan):
    rows = []
    for k in range(case["images"]):
        vp = gen.boundary_viewport(case["view"] + k, case["width"], case["height"],
                                   case["max_iter"])
        for r0, nr in gen.row_tiles(vp.height, case["tile_rows"]):
            rows.append((vp.re_min + pan[0] * vp.step_re, vp.im_min + pan[1] * vp.step_im,
                         vp.step_re, vp.step_im, vp.width, vp.height, r0, nr, vp.max_iter,
                         cg.F64 if case["fp"] == F64 else cg.F32))
    return np.array(rows, cg.NP_MANDEL)


def _tile_args(case, pan):
    side, c = case["side"], case["count"]
    st_re, st_im = 3.5 / (8 * side), 2.5 / (8 * side)
    i = np.arange(c)
    a = np.zeros(c, cg.NP_MANDEL)
    a["re_min"] = -2.5 + (side * (i % 8) + pan[0] + 0.37 * (i // 64)) * st_re
    a["im_min"] = -1.25 + pan[1] * st_im
    a["step_re"], a["step_im"] = st_re, st_im
    a["width"], a["height"], a["rows"] = side, 8 * side, side
    a["row0"] = side * ((i // 8) % 8)
    a["max_iter"], a["fp"] = case["max_iter"], cg.F32
    return a


def _mix(case, pan=(0.0, 0.0)):
    d = gen.serving_mix_arrays(case["view"], 1e5, 2 * case["count"] / 1e5 + 1e-3)
    d = {k: v[:case["count"]] for k, v in d.items()}
    a = np.zeros(len(d["side"]), cg.NP_MANDEL)
    a["re_min"], a["im_min"] = d["re_min"] + pan[0] * d["step"], d["im_min"] + pan[1] * d["step"]
    a["step_re"] = a["step_im"] = d["step"]
    a["width"] = a["height"] = a["rows"] = d["side"]
    a["max_iter"], a["fp"] = d["max_iter"], cg.F32
    return d, a


def _iterations(args, grid):
    """Escape iterations of these messages, from a coarse grid of each."""
    f = (np.arange(grid) + 0.5) / grid
    cr = args["re_min"][:, None] + args["step_re"][:, None] * args["width"][:, None] * f
    ci = args["im_min"][:, None] + args["step_im"][:, None] * (
        args["row0"][:, None] + args["rows"][:, None] * f)
    c = (cr[:, None, :] + 1j * ci[:, :, None]).reshape(-1)
    px = args["rows"].astype(np.float64) * args["width"] / (grid * grid)
    wt, lim = np.repeat(px, grid * grid), np.repeat(args["max_iter"], grid * grid)
    z, total = np.zeros_like(c), 0.0
    for it in range(int(args["max_iter"].max())):
        if it % 16 == 0:
            keep = (np.abs(z) <= 2) & (lim > it)
            z, c, wt, lim = z[keep], c[keep], wt[keep], lim[keep]
            total += 16 * float(wt.sum())
            if not len(z):
                break
        z = np.where(np.abs(z) <= 2, z * z + c, z)
    return total


# ---- the five things a case is asked for -----------------------------------

def _sizes(case):
    g = gen.rng(case["count"])
    if case["sizes"] == "mix":
        return gen.gemm_sizes(0, case["count"]).astype(np.int64)
    return g.integers(case["lo"], case["hi"] + 1, size=case["count"]).astype(np.int64)


def _gemm_inputs(sizes, seed, dtype):
    total = _total(sizes * sizes)
    A, B = _rand(seed, total), _rand(seed + 1000003, total)
    if dtype == BF16:
        A, B = A.to(torch.bfloat16), B.to(torch.bfloat16)
    return A, B


def _gemm_exact(sizes, A, B):
    nn = sizes * sizes
    offs = _offsets(nn)
    out = torch.zeros(_total(nn), dtype=torch.float64, device="cuda")
    for n, o, m in zip(sizes.tolist(), offs.tolist(), nn.tolist()):
        torch.mm(A[o:o + m].double().view(n, n), B[o:o + m].double().view(n, n),
                 out=out[o:o + m].view(n, n))
    return out


def _stage_input(case, seed):
    return 2 * _rand(seed, case["rows"] * case["cols"])


def prepare(case, seed):
    kind = case["kind"]
    g = gen.rng(seed)
    pan = g.uniform(-4.0, 4.0, size=2)
    if kind == "echo":
        kept = _system(mode="batched", arena_bytes=64 << 20)
        xs = [g.integers(-2 ** 31, 2 ** 31, size=case["len"]).astype(np.int32)
              for _ in range(case["count"])]
        return {"kind": kind, "s": kept[0], "actor": _actor(kept, cg.BHV_NOOP), "xs": xs}
    if kind in ("tiles", "image"):
        kept = _system(mode=case.get("mode", "batched"), arena_bytes=256 << 20)
        colour = case.get("colour", False)
        if colour:
            pal = (_rand(seed, 256) * 2 ** 31).to(torch.int32)
            actor = kept[0].spawn(cg.BHV_MANDELBROT, palette=pal)
        else:
            actor = _actor(kept, cg.BHV_MANDELBROT)
        args = (_tile_args if kind == "tiles" else _image_args)(case, pan)
        msgs = _messages(args, actor)
        px = args["rows"].astype(np.int64) * args["width"]
        out = torch.zeros(_total(px), dtype=torch.int32 if colour else torch.int16,
                          device="cuda")
        _outputs(msgs, out.data_ptr(), _offsets(px), px, cg.U32 if colour else cg.U16,
                 4 if colour else 2)
        return {"kind": kind, "keep": args, "out": out,
                "go": cg.PreparedDrive(kept[0], msgs, case.get("window", len(msgs)))}
    if kind == "gemm":
        tuned = case["tuned"]
        cls = (0, 0, 0, 0) if not tuned else (256,) * 4 if case["dtype"] == BF16 else (128,) * 4
        kept = _system(mode=case["mode"], arena_bytes=256 << 20, gemm_tile_class=cls)
        sizes = _sizes(case)
        A, B = _gemm_inputs(sizes, seed, case["dtype"])
        nn = sizes * sizes
        offs, esz = _offsets(nn), A.element_size()
        code = cg.BF16 if case["dtype"] == BF16 else cg.F32
        args = np.zeros(len(sizes), cg.NP_GEMM)
        args["n"], args["in_dtype"] = sizes, code
        msgs = _messages(args, _actor(kept, cg.BHV_GEMM))
        ptrs = np.stack([A.data_ptr() + offs * esz, B.data_ptr() + offs * esz], 1).astype(np.uint64)
        bufs = _inputs(msgs, ptrs, nn, code)
        out = torch.zeros(_total(nn), device="cuda")
        _outputs(msgs, out.data_ptr(), offs, nn, cg.F32, 4)
        return {"kind": kind, "keep": (args, bufs, A, B), "out": out,
                "go": cg.PreparedDrive(kept[0], msgs, len(msgs))}
    if kind == "chain":
        n, c = case["n"], case["count"]
        kept = _system(mode="batched", arena_bytes=4 << 30)
        rs = _actor(kept, cg.BHV_ROWSUM, n=n)
        th = _actor(kept, cg.BHV_TANH, n=n, forward_to=rs)
        sizes = np.full(c, n, np.int64)
        A, B = _gemm_inputs(sizes, seed, F32)
        offs = _offsets(sizes * sizes)
        args = np.zeros(c, cg.NP_GEMM)
        args["n"], args["in_dtype"] = n, cg.F32
        msgs = _messages(args, _actor(kept, cg.BHV_GEMM))
        ptrs = np.stack([A.data_ptr() + offs * 4, B.data_ptr() + offs * 4], 1).astype(np.uint64)
        bufs = _inputs(msgs, ptrs, sizes * sizes, cg.F32)
        msgs["forward_to"] = th
        out = torch.empty(c * n, device="cuda")
        _outputs(msgs, out.data_ptr(), np.arange(c) * n, n, cg.F32, 4)
        return {"kind": kind, "keep": (args, bufs, A, B), "out": out,
                "go": cg.PreparedDrive(kept[0], msgs, case["window"])}
    if kind == "mix":
        kept = _system(mode="persistent", arena_bytes=256 << 20, ring_slots=8192,
                       full_wgs_per_cu=3, idle_exit_us=2000)
        d, margs = _mix(case, pan)
        ism, sizes = d["is_mandel"], d["gemm_n"].astype(np.int64)
        numel = np.where(ism, d["side"].astype(np.int64) ** 2, sizes * sizes)
        moff, goff = _offsets(numel * ism), _offsets(numel * ~ism)  # the other kind: no room
        A, B = _gemm_inputs(sizes[~ism], seed, F32)
        counts = torch.zeros(_total(numel[ism]), dtype=torch.int16, device="cuda")
        products = torch.zeros(A.numel(), device="cuda")
        gargs = np.zeros(len(sizes), cg.NP_GEMM)
        gargs["n"], gargs["in_dtype"] = sizes, cg.F32
        idx = np.arange(len(sizes), dtype=np.uint64)
        msgs = np.zeros(len(sizes), cg.NP_MSG)
        ptrs = np.stack([A.data_ptr() + goff * 4, B.data_ptr() + goff * 4], 1).astype(np.uint64)
        bufs = _inputs(msgs, ptrs, numel, cg.F32)
        msgs["n_in"][ism], msgs["in_"][ism] = 0, 0
        msgs["actor"] = np.where(ism, _actor(kept, cg.BHV_MANDELBROT), _actor(kept, cg.BHV_GEMM))
        msgs["args"] = np.where(ism, margs.ctypes.data + idx * margs.itemsize,
                                gargs.ctypes.data + idx * gargs.itemsize)
        msgs["args_bytes"] = np.where(ism, margs.itemsize, gargs.itemsize)
        msgs["out"]["data"] = np.where(ism, counts.data_ptr() + moff * 2,
                                       products.data_ptr() + goff * 4).astype(np.uint64)
        msgs["out"]["numel"] = numel
        msgs["out"]["dtype"] = np.where(ism, cg.U16, cg.F32)
        msgs["out"]["on_device"] = 1
        return {"kind": kind, "keep": (margs, gargs, bufs, A, B), "counts": counts,
                "products": products, "go": cg.PreparedDrive(kept[0], msgs, case["window"])}
    kept = _system(mode="batched", arena_bytes=64 << 20)
    x = _stage_input(case, seed)
    th, rs = torch.empty_like(x), torch.empty(case["rows"], device="cuda")
    args = np.zeros(2, np.dtype([("rows", np.uint32), ("cols", np.uint32)]))
    args["rows"], args["cols"] = case["rows"], case["cols"]
    msgs = _messages(args, 0)
    msgs["actor"] = [_actor(kept, cg.BHV_TANH), _actor(kept, cg.BHV_ROWSUM)]
    bufs = _inputs(msgs, np.full((2, 1), x.data_ptr(), np.uint64), np.full(2, x.numel()), cg.F32)
    msgs["out"]["data"] = [th.data_ptr(), rs.data_ptr()]
    msgs["out"]["numel"] = [x.numel(), case["rows"]]
    msgs["out"]["dtype"], msgs["out"]["on_device"] = cg.F32, 1
    return {"kind": kind, "keep": (args, bufs, x), "tanh": th, "rowsum": rs,
            "go": cg.PreparedDrive(kept[0], msgs, 2)}


def run(state):
    if state["kind"] == "echo":
        got = []
        for x in state["xs"]:
            f = state["s"].request(state["actor"], inputs=[x])
            status, v = f.result()
            f.release()
            if status != cg.OK:
                raise RuntimeError(cg.strerror(status))
            got.append(v)
        return np.concatenate(got)
    rc = state["go"]()
    if rc != cg.OK or state["go"].st.any():
        raise RuntimeError(f"drive: {rc}, {np.unique(state['go'].st)}")
    return {k: state[k] for k in ("out", "counts", "products", "tanh", "rowsum") if k in state}


def work(case):
    kind = case["kind"]
    if kind == "echo":
        return {"bytes": 8 * case["len"] * case["count"], "flops": 0}
    if kind in ("tiles", "image"):
        args = (_tile_args if kind == "tiles" else _image_args)(case, (0.0, 0.0))
        px = float((args["rows"].astype(np.float64) * args["width"]).sum())
        some = args[:: max(1, len(args) // 256)]
        it = _iterations(some, 8 if kind == "tiles" else 24)
        it *= px / float((some["rows"].astype(np.float64) * some["width"]).sum())
        return {"bytes": px * (4 if case.get("colour") else 2), "flops": OPS_PER_ITER * it}
    if kind == "gemm":
        n = _sizes(case).astype(np.float64)
        return {"bytes": float((n * n).sum()) * (8 if case["dtype"] == BF16 else 12),
                "flops": float((2 * n ** 3).sum())}
    if kind == "chain":
        n, c = case["n"], case["count"]
        return {"bytes": 4.0 * c * (2 * n * n + n), "flops": 2.0 * c * n ** 3}
    if kind == "mix":
        d, args = _mix(case)
        ism, n = d["is_mandel"], d["gemm_n"].astype(np.float64)[~d["is_mandel"]]
        px = float((d["side"].astype(np.float64)[ism] ** 2).sum())
        return {"bytes": 2 * px + float((12 * n * n).sum()),
                "flops": OPS_PER_ITER * _iterations(args[ism], 4) + float((2 * n ** 3).sum())}
    # the elementwise and the row actor are two messages: each reads the matrix
    m = float(case["rows"]) * case["cols"]
    return {"bytes": 4 * (3 * m + case["rows"]), "flops": 2 * m}


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        sizes = _sizes(case)
        return {"out": _gemm_exact(sizes, *_gemm_inputs(sizes, seed, case["dtype"]))}
    if kind == "chain":
        n = case["n"]
        sizes = np.full(case["count"], n, np.int64)
        C = _gemm_exact(sizes, *_gemm_inputs(sizes, seed, F32)).view(case["count"], -1)[:, :n * n]
        return {"out": torch.tanh(C).reshape(-1, n).sum(1)}
    if kind == "mix":
        d, _ = _mix(case)
        sizes = d["gemm_n"].astype(np.int64)[~d["is_mandel"]]
        return {"counts": None, "products": _gemm_exact(sizes, *_gemm_inputs(sizes, seed, F32))}
    if kind == "stage":
        x = _stage_input(case, seed).double()
        return {"tanh": torch.tanh(x), "rowsum": x.view(case["rows"], case["cols"]).sum(1)}
    return None
