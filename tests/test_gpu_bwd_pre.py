"""bwd_pre's row loop: calls on both sides of the line between one and four rows
per thread (4096 workgroups of 256 threads, d / 8 threads a row), whose rows do
not fill the last wave."""
import pytest
import torch

from gpu_util import REL_FROB, REL_MAX, run_bwd, run_fwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("N", [1, 37, 129])
def test_rows_per_thread(N, d):
    """A head's gradients are the same bits whichever loop its call takes, and
    right for the first and last head of each."""
    line = 4096 * 256 // (d // 8)  # rows at which the loop changes
    few, many = (line - 257) // N, -(-line // N) + 1
    assert few * N + 256 < line <= many * N
    g = torch.Generator(device="cuda")
    g.manual_seed(N + d)
    q, k, v, do = [torch.randn((1, many, N, d), generator=g, device="cuda").bfloat16() for _ in range(4)]
    o, lse = run_fwd(q, k, v, False)
    got = run_bwd(q, k, v, o, do, lse, False, "naive")
    cut = [t[:, :few].contiguous() for t in (q, k, v, o, do, lse)]
    for a, b in zip(got, run_bwd(*cut, False, "naive")):
        assert torch.equal(a[:, :few].view(torch.int16), b.view(torch.int16))
    # the definitions in float64.  One key: P = 1, O = V and dS = dP - D is 0 up
    # to the order of two fp32 sums; |dS| <= 2^-8 |dO| |V| bounds that amply
    for h in (0, few - 1, many - 1):
        qh, kh, vh, doh = (t[0, h].double() for t in (q, k, v, do))
        p = torch.softmax(qh @ kh.t().contiguous() * d ** -0.5, -1)
        ds = p * (doh @ vh.t().contiguous() - (doh * (p @ vh)).sum(-1, keepdim=True)) * d ** -0.5
        ref = (ds @ kh, ds.t().contiguous() @ qh, p.t().contiguous() @ doh)
        for name, a, r in zip(("dQ", "dK", "dV"), got, ref):
            e = (a[0, h].double() - r).abs()
            assert bool(e.isfinite().all()), name
            if N == 1 and name != "dV":
                bound = float(doh.norm() * vh.norm()) * 2.0 ** -8 * d ** -0.5 * float(max(qh.abs().max(), kh.abs().max()))
                assert float(e.max()) <= bound, name
            else:
                assert float(e.norm() / r.norm()) <= REL_FROB and float(e.max() / r.abs().max()) <= REL_MAX, name

