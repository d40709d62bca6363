"""Wide KV tiles at head dims 128 (256 rows) and 256 (128 rows): the sub-step
pipeline at the edges of its tiles (blocks whose second 32 rows lie past N,
tiles with few or no rows, chains of one block, Symmetric Shift's tile switch),
every mode, and the order of the sums.  Shapes have the fewest heads at which every
ordered schedule takes the wide tile."""
import numpy as np
import pytest
import torch

from gpu_util import REL_FROB, REL_MAX, run_bwd, run_fwd
from oracle import schedule as osched
from paper_2601_21824_amd import binding as dash

pytestmark = pytest.mark.gpu


def wide_heads(N, d, causal):
    for heads in range(2, 2049):
        if all(dash.dash_schedule_table(s, N, d, causal, heads=heads)["bc"] == (256 if d == 128 else 128)
               for s in scheds(d, causal)):
            return heads


def make(heads, N, d, seed=3, sigma=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + N + d)
    return [(torch.randn((1, heads, N, d), generator=g, device="cuda") * sigma).bfloat16() for _ in range(4)]


def reference(q, k, v, do, causal):
    """dQ, dK, dV of the given heads from the definitions in float64."""
    q, k, v, do = (t.double() for t in (q, k, v, do))
    scale = q.shape[-1] ** -0.5
    s = (q @ k.transpose(1, 2).contiguous()) * scale
    if causal:
        n = q.shape[1]
        s.masked_fill_(torch.ones((n, n), dtype=torch.bool, device=q.device).triu(1), float("-inf"))
    p = torch.softmax(s, -1)
    dp = do @ v.transpose(1, 2).contiguous()
    ds = p * (dp - (do * (p @ v)).sum(-1, keepdim=True)) * scale
    return ds @ k, ds.transpose(1, 2).contiguous() @ q, p.transpose(1, 2).contiguous() @ do


def scheds(d, causal):
    s = ("symshift", "descending", "naive") if causal else ("shift", "descending", "naive")
    return s + (("partials",) if d == 128 else ())


@pytest.mark.parametrize("d", [128, 256])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N", [65, 97, 129, 200, 257, 290, 400, 512, 513, 545, 700])
def test_wide_tiles_match_float64(N, causal, d):
    heads = wide_heads(N, d, causal)
    if heads is None:
        pytest.skip("no number of heads takes wide tiles under every schedule")
    assert dash.dash_schedule_table("naive", N, d, causal, heads=heads)["bc"] == (256 if d == 128 else 128)
    q, k, v, do = make(heads, N, d)
    o, lse = run_fwd(q, k, v, causal)
    some = [0, heads // 2, heads - 1]
    ref = reference(*(t[0, some] for t in (q, k, v, do)), causal)
    first = {}
    for s in scheds(d, causal):
        print(f"[wide] N={N} d={d} causal={causal} heads={heads} {s}", flush=True)
        ws = dash.new_workspace(1, heads, N, d, s)
        got = run_bwd(q, k, v, o, do, lse, causal, s, workspace=ws)
        assert dash.dash_bwd_check(ws) == dash.DASH_OK
        for name, a, r in zip(("dQ", "dK", "dV"), got, ref):
            e = (a[0, some].double() - r).abs()
            assert bool(e.isfinite().all()), name
            # the repository's tolerance: bf16 P and dS, fp32 sums, bf16 outputs
            assert float(e.norm() / r.norm()) <= REL_FROB and float(e.max() / r.abs().max()) <= REL_MAX, (s, name)
        first[s] = got
        for _ in range(3):
            again = run_bwd(q, k, v, o, do, lse, causal, s, workspace=ws)
            for a, b in zip(got, again):
                assert torch.equal(a.view(torch.int16), b.view(torch.int16)), s
    for s in ("descending",) + (("partials",) if d == 128 else ()):  # the same partials in the same order
        assert torch.equal(first["naive"][0].view(torch.int16), first[s][0].view(torch.int16)), s


ORDER = [(128, False, "shift"), (128, True, "symshift"), (128, True, "naive"), (256, False, "shift"), (256, True, "symshift"),
         (256, False, "descending")]


@pytest.mark.parametrize("d,causal,sched", ORDER)
def test_wide_tiles_order_and_replay(d, causal, sched):
    """The witnessed order is the schedule's; the exported partials summed in that
    order in fp32 are the accumulator, bit for bit; XCD-local placement and a
    grid of a few workgroups give the same bits."""
    N = 1100 if d == 128 else 600
    heads = wide_heads(N, d, causal)
    q, k, v, do = make(heads, N, d, seed=9)
    o, lse = run_fwd(q, k, v, causal)
    tab = dash.dash_schedule_table(sched, N, d, causal, heads=heads)
    bc, tc, nblk = tab["bc"], -(-N // tab["bc"]), -(-N // 64)
    assert bc == (256 if d == 128 else 128)
    witness = torch.full((heads, nblk, tc), -1, dtype=torch.int32, device="cuda")
    partials = torch.zeros((heads, tc, N, d), dtype=torch.float32, device="cuda")
    acc = torch.zeros((heads, N, d), dtype=torch.float32, device="cuda")
    ws = dash.new_workspace(1, heads, N, d, sched)
    opts = dash.dash_bwd_options_t(0, 0, witness.data_ptr(), partials.data_ptr(), acc.data_ptr())
    ref = run_bwd(q, k, v, o, do, lse, causal, sched, options=opts, workspace=ws)
    assert dash.dash_bwd_check(ws) == dash.DASH_OK
    kind = {"shift": osched.SHIFT, "symshift": osched.SYMSHIFT, "naive": osched.NAIVE, "descending": osched.DESCENDING}[sched]
    order = osched.build(kind, tab["t_r"], tab["t_c"], causal, tab["br"], bc, group=tab["group"] if kind == osched.SHIFT else None).order
    W = witness.cpu().numpy()
    nsub = tab["br"] // 64
    for h in (0, heads - 1):
        P, A = partials[h].cpu().numpy(), acc[h].cpu().numpy()
        for pb in range(nblk):
            js = [j for j in order[pb // nsub] if j < tc]
            assert W[h, pb, :len(js)].tolist() == js, (h, pb)
            rows = slice(64 * pb, min(N, 64 * pb + 64))
            total = P[js[0], rows].copy()
            for j in js[1:]:
                total = total + P[j, rows]
            np.testing.assert_array_equal(total, A[rows])
    xcd = dash.dash_bwd_options_t(0, 0, None, None, None, None, None, 0, 0, dash.DASH_PLACEMENT_XCD)
    few = dash.dash_bwd_options_t(0, 0, None, None, None, None, None, max(8, tab["group"]))
    for opt in (None, xcd, few):
        got = run_bwd(q, k, v, o, do, lse, causal, sched, options=opt, workspace=ws)
        assert dash.dash_bwd_check(ws) == dash.DASH_OK
        for a, b in zip(ref, got):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("d", [128, 256])
def test_wide_tiles_watchdog(d):
    """Poisoned counters: every wait gives up, the call reports the timeout, and the
    next call is right."""
    N = 300
    heads = wide_heads(N, d, False)
    q, k, v, do = make(heads, N, d)
    o, lse = run_fwd(q, k, v, False)
    ws = dash.new_workspace(1, heads, N, d)
    good = run_bwd(q, k, v, o, do, lse, False, "shift", workspace=ws)
    bad = dash.dash_bwd_options_t(64, dash.DASH_FLAG_POISON_COUNTERS)
    run_bwd(q, k, v, o, do, lse, False, "shift", options=bad, workspace=ws)
    assert dash.dash_bwd_check(ws) == dash.DASH_ERR_TIMEOUT
    again = run_bwd(q, k, v, o, do, lse, False, "shift", workspace=ws)
    assert dash.dash_bwd_check(ws) == dash.DASH_OK
    for a, b in zip(good, again):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
