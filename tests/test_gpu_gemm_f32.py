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
