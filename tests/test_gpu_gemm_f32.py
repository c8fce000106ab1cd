"""fp32 products at the edges of their tiles and of the number range (GPU).

The bound is the one every summation order keeps: each output is off by at
most (n + 8) 2^-24 times the sum of |a b| (n roundings of the running sum, and
a few of its terms), plus what underflow may take, n 2^-126 (a product of
numbers near the smallest normal one).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NS = [1, 2, 3, 4, 5, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 130, 131, 200, 257]


@pytest.fixture(scope="module", params=[(64, 2, 0), (128, 2, 0), (128, 3, 0), (128, 2, 256), (0, 2, 0)])
def sysm(request):
    """Tile edge, workgroups per CU, and the wide variant (square tiles as
    calls)."""
    from paper_1505_07368_amd import binding as cg
    te, wgs, cls = request.param
    s = cg.System(mode="batched", arena_bytes=64 << 20, gemm_tile=te, full_wgs_per_cu=wgs,
                  gemm_tile_class=(cls,) * 4)
    yield s, s.spawn(cg.BHV_GEMM)
    s.shutdown()


def _product(sysm, A, B):
    import torch
    from paper_1505_07368_amd import binding as cg
    s, a = sysm
    n = A.shape[0]
    At, Bt = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    torch.cuda.synchronize()
    st, C = s.request(a, cg.caf_gemm_args(n, cg.F32), inputs=[At, Bt]).result()
    assert st == cg.OK
    return C.cpu().numpy().reshape(n, n)


def _range(kind, n, g):
    A, B = g.standard_normal((n, n)), g.standard_normal((n, n))
    if kind == "zeros":  # an operand of zeros, and zeros among the numbers
        return np.maximum(A, 0), 0 * B
    if kind == "tiny":  # products near the smallest normal number
        return A * 1e-25, B * 1e-12
    if kind == "denormal":
        return A * 1e-40, B
    if kind == "huge":
        return A * 1e25, B * 1e10
    if kind == "rows":  # magnitudes from 2^-60 to 2^60, by row
        return A * np.exp2(g.uniform(-60, 60, (n, 1))), B
    return g.uniform(-1, 1, (n, n)), g.uniform(-1, 1, (n, n))


@pytest.mark.parametrize("kind", ["uniform", "zeros", "tiny", "denormal", "huge", "rows"])
def test_bound_over_sizes_and_ranges(sysm, kind):
    g = np.random.Generator(np.random.PCG64(11))
    for n in NS:
        A, B = (x.astype(np.float32) for x in _range(kind, n, g))
        C = _product(sysm, A, B).astype(np.float64)
        A, B = A.astype(np.float64), B.astype(np.float64)
        bound = (n + 8) * 2.0 ** -24 * (np.abs(A) @ np.abs(B)) + n * 2.0 ** -126
        off = np.abs(C - A @ B)
        assert (off <= bound).all(), (kind, n, float((off / bound).max()))


@pytest.mark.parametrize("n", [5, 64, 130, 257])
def test_infinities_and_nans_stay_in_their_rows_and_columns(sysm, n):
    g = np.random.Generator(np.random.PCG64(n))
    A = g.uniform(0.5, 1, (n, n)).astype(np.float32)
    B = g.uniform(0.5, 1, (n, n)).astype(np.float32)
    A[n // 2, n - 1] = np.inf
    B[n // 3, 1] = np.nan
    A[0, 0] = 3.4e38  # overflows in its row
    B[0, 2] = 3.4e38
    C = _product(sysm, A, B)
    with np.errstate(all="ignore"):
        R = (A.astype(np.float64) @ B.astype(np.float64)).astype(np.float32)
    near = np.abs(R) > 3.3e38  # either side of the largest number
    assert (np.isnan(C) == np.isnan(R)).all()
    assert ((np.isinf(C) == np.isinf(R)) | near).all()
    ok = np.isfinite(R) & ~near
    assert np.allclose(C[ok], R[ok], rtol=(n + 8) * 2.0 ** -24, atol=0)


@pytest.mark.parametrize("n", [5, 32, 33, 64, 130, 257])
@pytest.mark.parametrize("at", [0, 100])
def test_sums_of_one_term_are_rounded_once(sysm, n, at):
    """A diagonal factor: each output is one product.  Its largest part is
    exact; what is added to it has at most eight roundings of 2^-24 of 2^-8 of
    the product, 2^-5 of the last place, and the sum rounds once more.  at:
    the factor's magnitudes are from 2^-109 on, where its last bits are
    numbers smaller than the smallest normal one."""
    g = np.random.Generator(np.random.PCG64(n))
    A = np.diag(g.uniform(1, 2, n) * 2.0 ** (-109 if at else 0)).astype(np.float32)
    B = (g.uniform(1, 2, (n, n)) * np.exp2(g.integers(-4, 4, (n, n)) + (60 if at else 0)))
    B = B.astype(np.float32)
    C = _product(sysm, A, B).astype(np.float64)
    R = A.astype(np.float64) @ B.astype(np.float64)
    ulp = np.exp2(np.floor(np.log2(np.abs(R))) - 23)
    assert (np.abs(C - R) <= (0.5 + 2.0 ** -5) * ulp).all(), float((np.abs(C - R) / ulp).max())


@pytest.mark.parametrize("n", [65, 129, 257])
def test_spread_magnitudes_are_no_further_off_than_one_rounding_per_term(sysm, n):
    """Magnitudes from 2^-20 to 2^20: the root mean square error is at most
    that of a fused multiply-add per term, in fp32."""
    g = np.random.Generator(np.random.PCG64(n))
    A, B = ((g.standard_normal((n, n)) * np.exp2(g.uniform(-20, 20, (n, n)))).astype(np.float32)
            for _ in range(2))
    C = _product(sysm, A, B).astype(np.float64)
    A, B = A.astype(np.float64), B.astype(np.float64)
    chain = np.zeros((n, n), np.float32)
    for k in range(n):
        chain = (chain + np.outer(A[:, k], B[k])).astype(np.float32)
    R, size = A @ B, np.abs(A) @ np.abs(B)
    rms = lambda x: float(np.sqrt((((x - R) / size) ** 2).mean()))
    assert rms(C) <= rms(chain.astype(np.float64)), (rms(C), rms(chain.astype(np.float64)))


def _special(kind, n, g):
    A, B = g.standard_normal((n, n)), g.standard_normal((n, n))
    if kind == "one_tiny":  # one number in the subnormal range in each operand
        A[n // 2, n // 3], B[n // 3, n // 2] = 1e-39, 1e-41
    if kind == "softmax":  # tiny numbers next to ordinary ones, and rows of zeros
        e = np.exp(40 * A)
        A = e / e.sum(1, keepdims=True)
        A[n // 2:n // 2 + 3] = 0
    if kind == "products":  # outputs near the smallest normal number
        A, B = A * 2.0 ** -60, B * 2.0 ** -60
    if kind == "infinite":
        A[n // 2, n // 3], B[n // 4, n // 5], A[0, 0] = np.inf, np.nan, 3.4e38
    return A.astype(np.float32), B.astype(np.float32)


KINDS = ["one_tiny", "softmax", "products", "infinite"]


@pytest.mark.parametrize("kind", KINDS)
def test_bits_do_not_depend_on_the_tile_edge_or_the_load(kind):
    """The tile edge follows the load, and work tiles of several output tiles
    run as one stream: neither may show in the product."""
    import torch
    from paper_1505_07368_amd import binding as cg
    g = np.random.Generator(np.random.PCG64(5))
    ins = {}
    for n in (33, 65, 129, 130, 200, 257, 300):
        A, B = _special(kind, n, g)
        t = [torch.zeros(n * n + 1, device="cuda") for _ in range(2)]  # odd addresses
        for x, v in zip(t, (A, B)):
            x[1:] = torch.from_numpy(v).cuda().view(-1)
        ins[n] = (A, B, t, [cg.caf_buf(x.data_ptr() + 4, n * n, cg.F32, 1) for x in t])
    torch.cuda.synchronize()
    first = {}
    for kw in ({"gemm_tile": 64}, {"gemm_tile": 128}, {}, {"full_wgs_per_cu": 3},
               {"mode": "plain"}):
        with cg.System(**{"mode": "batched", "arena_bytes": 256 << 20, **kw}) as s:
            a = s.spawn(cg.BHV_GEMM)
            req = lambda n: s.request(a, cg.caf_gemm_args(n, cg.F32), inputs=ins[n][3])
            got = [(n, req(n)) for n in ins]
            if not kw:  # the same ones behind a queue, thirty times each
                s.drain()
                s.hold(True)
                got += [(n, req(n)) for _ in range(30) for n in ins]
                s.hold(False)
            for n, f in got:
                st, C = f.result()
                assert st == cg.OK
                bits = C.view(torch.int32).masked_fill(C.isnan(), 0x7FC00000)
                if n not in first:
                    first[n] = bits.clone()
                    A, B = (x.astype(np.float64) for x in ins[n][:2])
                    with np.errstate(all="ignore"):
                        R, size = A @ B, np.abs(A) @ np.abs(B)
                        off = np.abs(C.cpu().numpy().reshape(n, n).astype(np.float64) - R)
                    ok = np.isfinite(R) & (np.abs(R) < 3.3e38)
                    assert (off <= (n + 8) * 2.0 ** -24 * size + n * 2.0 ** -126)[ok].all(), (kind, n)
                assert torch.equal(bits, first[n]), (kind, n, kw)
                f.release()


@pytest.mark.parametrize("kind", ["softmax", "tiny"])
def test_small_numbers_take_no_longer(kind):
    """Products of a softmax matrix, whose smallest entries are far below the
    ordinary ones, and of numbers about 1e-20 and 1e-14, at the speed of others
    (twice their time allowed)."""
    import time

    import torch
    from paper_1505_07368_amd import binding as cg
    n, count = 512, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    B = torch.randn(count, n, n, generator=g, device="cuda")
    logits = 8 * torch.randn(count, n, n, generator=g, device="cuda")
    out = torch.zeros(count, n * n, device="cuda")
    with cg.System(mode="batched", arena_bytes=64 << 20) as s:
        a = s.spawn(cg.BHV_GEMM)
        args = np.zeros(1, cg.NP_GEMM)
        args["n"], args["in_dtype"] = n, cg.F32

        def took(A):
            bufs = np.zeros((count, 2), cg.NP_BUF)
            bufs["data"][:, 0] = A.data_ptr() + np.arange(count) * n * n * 4
            bufs["data"][:, 1] = B.data_ptr() + np.arange(count) * n * n * 4
            bufs["numel"], bufs["dtype"], bufs["on_device"] = n * n, cg.F32, 1
            msgs = np.zeros(count, cg.NP_MSG)
            msgs["actor"], msgs["n_in"] = a, 2
            msgs["args"], msgs["args_bytes"] = args.ctypes.data, args.itemsize
            msgs["in_"] = bufs.ctypes.data + np.arange(count, dtype=np.uint64) * bufs[0].nbytes
            msgs["out"]["data"] = out.data_ptr() + np.arange(count) * n * n * 4
            msgs["out"]["numel"], msgs["out"]["dtype"], msgs["out"]["on_device"] = n * n, cg.F32, 1
            go, times = cg.PreparedDrive(s, msgs, count), []
            torch.cuda.synchronize()
            for _ in range(9):
                t = time.perf_counter()
                assert go() == cg.OK and not go.st.any()
                times.append(time.perf_counter() - t)
            return sorted(times)[4]

        ordinary = took(torch.rand(count, n, n, generator=g, device="cuda") - 0.5)
        if kind == "softmax":
            A = torch.softmax(logits, 2)
        else:
            A, B = logits * 1e-20, B * 1e-14
        assert took(A) <= 2 * ordinary


@pytest.mark.parametrize("n", [33, 130, 257])
@pytest.mark.parametrize("e", [50, 54, 56, 58, 60, 62])
def test_outputs_near_the_smallest_numbers(sysm, n, e):
    """Operands about 2^-e: outputs from 2^-96 down to 2^-124, on both sides of
    the line below which blocks are redone.  What the split may lose there is
    2^-146 per k."""
    g = np.random.Generator(np.random.PCG64(n + e))
    A, B = ((g.standard_normal((n, n)) * 2.0 ** -e).astype(np.float32) for _ in range(2))
    C = _product(sysm, A, B).astype(np.float64)
    A, B = A.astype(np.float64), B.astype(np.float64)
    bound = (n + 8) * 2.0 ** -24 * (np.abs(A) @ np.abs(B)) + n * 2.0 ** -146
    off = np.abs(C - A @ B)
    assert (off <= bound).all(), float((off / bound).max())


@pytest.mark.parametrize("te,wgs", [(0, 2), (64, 2), (128, 2), (0, 3), (128, 3)])
def test_streams_of_many_tiles(te, wgs):
    """Many products in one launch, so that a claim holds several tiles: the
    sizes' remainders at tile boundaries inside a stream, inputs one element
    into an allocation, and numbers in some tiles that leave the others' way
    (outputs that are not finite, operands of the subnormal range)."""
    import torch
    from paper_1505_07368_amd import binding as cg, gen
    with cg.System(mode="batched", arena_bytes=1 << 30, gemm_tile=te, full_wgs_per_cu=wgs) as s:
        a = s.spawn(cg.BHV_GEMM)
        for code in (cg.F32, cg.BF16):
            esz, keep, got = (4, 2)[code == cg.BF16], [], []
            s.hold(True)
            for n in (129, 200, 257, 300, 511):
                g = np.random.Generator(np.random.PCG64(n))
                A, B = (g.uniform(-1, 1, (n, n)).astype(np.float32) for _ in range(2))
                if code == cg.BF16:
                    A, B = (torch.from_numpy(x).bfloat16() for x in (A, B))
                else:
                    A[3, n - 1], A[n - 1, 0], B[5, n // 2] = np.inf, 1e-40, np.nan
                    A[70] *= np.float32(1e-38)
                    A, B = torch.from_numpy(A), torch.from_numpy(B)
                bufs = []
                for x in (A, B):
                    t = torch.zeros(n * n + 1, dtype=x.dtype, device="cuda")
                    t[1:] = x.cuda().view(-1)
                    bufs.append(t)
                torch.cuda.synchronize()
                ins = [cg.caf_buf(t.data_ptr() + esz, n * n, code, 1) for t in bufs]
                A, B = A.double(), B.double()
                keep.append(bufs)
                for _ in range(25):
                    f = s.request(a, cg.caf_gemm_args(n, code), inputs=ins)
                    got.append((n, f, A @ B, A.abs() @ B.abs()) if _ == 0 else (n, f, None, None))
            s.hold(False)
            for n, f, R, size in got:
                st, C = f.result()
                assert st == cg.OK
                C = C.cpu().double().view(n, n)
                if R is not None:
                    first = C
                    fin = torch.isfinite(R)
                    off = (C - R).abs()
                    assert (off <= (n + 8) * 2.0 ** -24 * size + n * 2.0 ** -126)[fin].all(), n
                    assert (torch.isnan(C) == torch.isnan(R)).all(), n
                assert torch.equal(C.nan_to_num(7.0), first.nan_to_num(7.0)), n
                f.release()
