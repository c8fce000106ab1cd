"""bf16 products of every remainder of n and at odd addresses (GPU).

Products of bf16 numbers are exact in fp32, so an output is off by at most its
n roundings: n 2^-24 times the sum of |a b| (n + 2 allowed), in any order.
"""
import numpy as np
import pytest

from paper_1505_07368_amd import gen

pytestmark = pytest.mark.gpu

NS = [1, 2, 3, 4, 7, 8, 9, 31, 33, 63, 64, 65, 66, 68, 72, 127, 129, 130, 136, 191, 200, 257, 300]


@pytest.mark.parametrize("te,wgs", [(64, 2), (128, 2), (64, 3), (128, 3), (0, 2)])
@pytest.mark.parametrize("offset", [0, 1])
def test_bound_over_sizes(te, wgs, offset):
    """offset: the inputs start that many elements into an allocation (2-byte
    alignment); tile edges and both occupancies."""
    import torch
    from paper_1505_07368_amd import binding as cg
    with cg.System(mode="batched", arena_bytes=64 << 20, gemm_tile=te, full_wgs_per_cu=wgs) as s:
        a = s.spawn(cg.BHV_GEMM)
        for n in NS:
            A, B = gen.gemm_pair(n, n, "bf16")
            bufs = []
            for x in (A, B):
                t = torch.zeros(n * n + 8, dtype=torch.int16, device="cuda")
                t[offset:offset + n * n] = torch.from_numpy(x.view(np.int16)).cuda().view(-1)
                bufs.append(t)
            torch.cuda.synchronize()
            ins = [cg.caf_buf(t.data_ptr() + 2 * offset, n * n, cg.BF16, 1) for t in bufs]
            st, C = s.request(a, cg.caf_gemm_args(n, cg.BF16), inputs=ins).result()
            assert st == cg.OK, n
            C = C.cpu().numpy().reshape(n, n).astype(np.float64)
            Af, Bf = (gen.bf16_bits_to_f32(x).astype(np.float64).reshape(n, n) for x in (A, B))
            off = np.abs(C - Af @ Bf)
            bound = (n + 2) * 2.0 ** -24 * (np.abs(Af) @ np.abs(Bf))
            assert (off <= bound).all(), (n, float((off / bound).max()))


def test_bits_do_not_depend_on_the_tile():
    """The tile follows the load (64, 128 or 128 x 256, with 64- or 32-deep
    slices): magnitudes spread over 2^-20 to 2^20 have the same sums in all."""
    import torch
    from paper_1505_07368_amd import binding as cg
    g = torch.Generator(device="cuda")
    first = {}
    for kw in ({"gemm_tile": 64}, {"gemm_tile": 128}, {"gemm_tile": 256}, {"full_wgs_per_cu": 3},
               {"mode": "plain"}):
        with cg.System(**{"mode": "batched", "arena_bytes": 64 << 20, **kw}) as s:
            a = s.spawn(cg.BHV_GEMM)
            for n in (64, 96, 130, 160, 257, 512):
                g.manual_seed(n)
                A, B = ((torch.randn(n * n, generator=g, device="cuda") * torch.exp2(
                    40 * torch.rand(n * n, generator=g, device="cuda") - 20)).bfloat16()
                    for _ in range(2))
                torch.cuda.synchronize()
                f = s.request(a, cg.caf_gemm_args(n, cg.BF16), inputs=[A, B])
                st, C = f.result()
                assert st == cg.OK
                bits = C.view(torch.int32)
                assert torch.equal(bits, first.setdefault(n, bits.clone())), (kw, n)
                f.release()
