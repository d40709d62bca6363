"""The forward at the edges of its tiles: 32-key units, 32-, 64- and 128-row
query groups, 64- and 32-row K/V tiles, the last unit of a wave at either place
in its pair, waves past N, workgroup-to-XCD runs that end inside a head, and
both workgroup sizes at d = 64.  Against the definition in float64."""
import math

import pytest
import torch

from gpu_util import REL_FROB, REL_MAX
from paper_2601_21824_amd import binding as dash

pytestmark = pytest.mark.gpu

LENGTHS = (1, 31, 32, 33, 63, 64, 65, 96, 127, 129, 255, 257, 300, 513)
# (heads, N, d, causal): every length at a head count that the XCD count does
# not divide and one that it does; then d = 64 full calls at the two-group rule (N > 128 and 512 workgroups of 256 rows)
CASES = [(h, n, d, c) for d in (64, 128, 256) for c in (False, True) for n in LENGTHS for h in (3, 8)]
CASES += [(512, 100, 64, False), (512, 128, 64, False), (512, 129, 64, False), (511, 250, 64, False), (171, 520, 64, False), (170, 520, 64, False), (520, 33, 64, True)]


@pytest.mark.parametrize("heads,N,d,causal", CASES)
def test_forward_tile_edges(heads, N, d, causal):
    g = torch.Generator(device="cuda")
    g.manual_seed(7 * N + d + heads)
    q, k, v = (torch.randn((1, heads, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    q[..., N // 2:, :] *= 4  # a wide range of scores: the running maximum keeps moving
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, heads, N), float("nan"), device="cuda")
    dash.dash_attn_fwd(q, k, v, o, lse, causal)
    o2, lse2 = dash.attn_fwd(q, k, v, causal)
    s = q[0].double() @ k[0].double().transpose(1, 2).contiguous() / math.sqrt(d)
    if causal:
        s.masked_fill_(torch.ones((N, N), dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    ro, rl = torch.softmax(s, -1) @ v[0].double(), torch.logsumexp(s, -1)
    err = (o[0].double() - ro).abs()
    # bf16 P and O: two roundings of at most 2^-9 of the terms (the repository's tolerance)
    assert float(err.norm() / ro.norm()) <= REL_FROB
    assert float(err.max() / ro.abs().max()) <= REL_MAX
    assert float((lse[0].double() - rl).abs().max()) <= 2e-5 * max(1.0, float(rl.abs().max()))
    assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, lse2)


def test_a_rows_bits_do_not_depend_on_the_grouping():
    """One head's rows alone (one query group per wave) and among 512 heads
    (two groups per wave): the same bits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q, k, v = (torch.randn((1, 512, 300, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    o, lse = dash.attn_fwd(q, k, v, False)
    o1, lse1 = dash.attn_fwd(*(t[:, 5:6].contiguous() for t in (q, k, v)), False)
    assert torch.equal(o[:, 5:6].view(torch.int16), o1.view(torch.int16)) and torch.equal(lse[:, 5:6], lse1)


def test_nan_keys_reach_only_rows_that_see_them():
    """A NaN key: NaN in the causal rows at and after it, nowhere before."""
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    q, k, v = (torch.randn((1, 2, 200, 128), generator=g, device="cuda").bfloat16() for _ in range(3))
    k[0, 1, 100] = float("nan")
    o, lse = dash.attn_fwd(q, k, v, True)
    assert not o[0, 0].isnan().any() and not o[0, 1, :100].isnan().any() and not lse[0, 1, :100].isnan().any()
    assert o[0, 1, 100:].isnan().all() and lse[0, 1, 100:].isnan().all()


# (leading keys, what is added to their scores / sqrt(d)): rows of a full mask see
# other keys after them; causal rows before them see no other
FAR = [(n, s) for n in (20, 32, 40, 64, 130) for s in (-1e4, -3e9, -1e30, float("-inf"))]


@pytest.mark.parametrize("lead,shift", FAR)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,d", [(2, 64), (512, 64), (2, 128), (2, 256)])
def test_leading_keys_far_below_the_others(heads, d, causal, lead, shift):
    """Keys taken out of the softmax by a large negative score (left padding by an
    extra channel) ahead of those that count: whole units of 32 keys, and half
    ones, whose row maximum is that score.  Against the definition in float64 where it
    is defined (a causal row whose keys all score -inf has none: O is NaN)."""
    N = 200
    g = torch.Generator(device="cuda")
    g.manual_seed(lead + d)
    q, k, v = (torch.randn((1, heads, N, d), generator=g, device="cuda").bfloat16() for _ in range(3))
    q[..., 0] = 1
    k[:, :, :lead, 0] = shift
    o, lse = dash.attn_fwd(q, k, v, causal)
    some = [0, heads - 1]
    s = q[0, some].double() @ k[0, some].double().transpose(1, 2).contiguous() / math.sqrt(d)
    if causal:
        s.masked_fill_(torch.ones((N, N), dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    ro, rl = torch.softmax(s, -1) @ v[0, some].double(), torch.logsumexp(s, -1)
    o, lse = o[0, some].double(), lse[0, some].double()
    ok = ro.isfinite().all(-1)
    assert int(ok.sum()) == (2 * (N - lead) if causal and math.isinf(shift) else 2 * N)
    assert o[~ok].isnan().all()
    # rows that see only shifted keys: their scores are shift + O(1) in fp32, whose
    # spacing beside shift (2^-23 |shift|) is the error of a score
    if causal and shift == -3e9:
        ok &= torch.arange(N, device="cuda") >= lead
    err = (o[ok] - ro[ok]).abs()
    assert float(err.norm() / ro[ok].norm()) <= REL_FROB
    assert float(err.max() / ro[ok].abs().max()) <= REL_MAX
    assert o.isfinite().all(-1).equal(ro.isfinite().all(-1))
    assert bool(((lse[ok] - rl[ok]).abs() <= 2e-5 * rl[ok].abs().clamp(min=1)).all())
