"""What the framework's speed is measured on: attention forward and backward calls.

Every case is one call (or one forward and backward in a row) on tensors that
are already on the GPU, through the binding a training program uses, with
caller-owned outputs and workspace.  A case is

  op        "fwd", "bwd" or "step" (forward, then backward on its O and L)
  entry     the backward's form: "workspace" (dash_attn_bwd with an explicit
            workspace) or "noalloc" (dash_attn_bwd_noalloc)
  B H N d   batch, heads, sequence length, head dim
  causal    mask
  schedule  the backward's schedule

Inputs are bf16 ~ N(0, sigma^2): sigma = 1, and 0.5 at d = 256 (the scores
of longer head dims are larger before scaling).
"""
import math

import torch

from paper_2601_21824_amd import binding as dash


def _case(name, op, B, H, N, d, causal, schedule="auto", entry="workspace"):
    return {"name": name, "op": op, "entry": entry, "B": B, "H": H, "N": N, "d": d, "causal": causal,
            "schedule": schedule}


def listed():
    return [
        # the smallest calls: one head of one short sequence (a unit test, a
        # probe, a serving-side fine-tune of one sample); launches count
        _case("bwd-1head-n256-d64", "bwd", 1, 1, 256, 64, False),
        # a small model's layer at a usual context: 4 sequences of 1024
        _case("bwd-n1024-d64-causal", "bwd", 4, 16, 1024, 64, True),
        # many short sequences, 16384 tokens in all (the short end of the sweep)
        _case("bwd-n512-d128-causal", "bwd", 32, 32, 512, 128, True),
        # the benchmark: 16384 tokens, hidden 2048, full mask, Shift
        _case("bwd-n8192-d128-full", "bwd", 2, 16, 8192, 128, False, "shift"),
        # pretraining at a long context, causal
        _case("bwd-n8192-d128-causal", "bwd", 2, 32, 8192, 128, True),
        # the same tokens at head dim 64, full mask (an encoder)
        _case("bwd-n8192-d64-full", "bwd", 2, 32, 8192, 64, False),
        # the longest sequence the backward takes, at the largest head dim
        _case("bwd-n32768-d256-causal", "bwd", 1, 8, 32768, 256, True),
        # a ragged length under graph-capture rules: no allocation, Descending
        _case("bwd-n3001-d128-noalloc", "bwd", 1, 16, 3001, 128, True, "descending", "noalloc"),
        # the forward, small and ragged
        _case("fwd-n200-d64-causal", "fwd", 2, 3, 200, 64, True),
        # the forward of the causal pretraining shape
        _case("fwd-n8192-d128-causal", "fwd", 2, 32, 8192, 128, True),
        # the forward of a long sequence at the largest head dim
        _case("fwd-n16384-d256-full", "fwd", 1, 8, 16384, 256, False),
        # a training step of one attention layer, ragged length, d = 64
        _case("step-n2100-d64-causal", "step", 1, 128, 2100, 64, True),
    ]


_MAX_FLOPS = 4e12  # of one drawn call; the largest listed case has 1.1e13


def draw(rng):
    while True:
        op = rng.choice(["bwd", "bwd", "bwd", "fwd", "step"])
        d = rng.choice([64, 128, 128, 256])
        causal = rng.random() < 0.5
        N = int(round(math.exp(rng.uniform(math.log(128), math.log(16384)))))
        if rng.random() < 0.4:
            N = max(128, N // 128 * 128)  # whole tiles
        heads = int(round(math.exp(rng.uniform(0.0, math.log(512)))))
        B = rng.choice([1, 1, 2, 4])
        H = max(1, heads // B)
        schedule = rng.choice(["auto", "auto", "auto", "shift", "descending"])
        entry = "workspace"
        if op != "fwd" and rng.random() < 0.2 and dash.dash_bwd_workspace_size(B, H, N, d) <= 256 << 20:
            entry = "noalloc"
        c = _case("", op, B, H, N, d, causal, schedule, entry)
        del c["name"]
        # work between a small call's and the cap; at most 2^18 rows
        if work(c)["flops"] <= _MAX_FLOPS and B * H * N <= 1 << 18:
            return c


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    sigma = 0.5 if case["d"] == 256 else 1.0
    shape = (case["B"], case["H"], case["N"], case["d"])
    n = 3 if case["op"] == "fwd" else 4
    return [(torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * sigma).to(torch.bfloat16)
            for _ in range(n)]


def prepare(case, seed):
    t = _inputs(case, seed)
    q, k, v = t[:3]
    B, H, N, d = q.shape
    st = dict(case=case, q=q, k=k, v=v, o=torch.empty_like(q),
              lse=torch.empty((B, H, N), dtype=torch.float32, device="cuda"))
    if case["op"] != "fwd":
        st["dO"] = t[3]
        st["dq"], st["dk"], st["dv"] = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        if case["entry"] == "workspace":
            st["ws"] = dash.new_workspace(B, H, N, d, case["schedule"])
        if case["op"] == "bwd":  # the forward's O and L are in hand
            dash.dash_attn_fwd(q, k, v, st["o"], st["lse"], case["causal"])
    return st


def run(state):
    s, c = state, state["case"]
    if c["op"] != "bwd":
        dash.dash_attn_fwd(s["q"], s["k"], s["v"], s["o"], s["lse"], c["causal"])
        if c["op"] == "fwd":
            return {"o": s["o"], "lse": s["lse"]}
    if c["entry"] == "noalloc":
        dash.dash_attn_bwd_noalloc(s["q"], s["k"], s["v"], s["o"], s["dO"], s["lse"], s["dq"], s["dk"], s["dv"],
                                   c["causal"], c["schedule"])
    else:
        dash.dash_attn_bwd(s["q"], s["k"], s["v"], s["o"], s["dO"], s["lse"], s["dq"], s["dk"], s["dv"],
                           c["causal"], c["schedule"], workspace=s["ws"])
    out = {"dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}
    if c["op"] == "step":
        out["o"], out["lse"] = s["o"], s["lse"]
    return out


def work(case):
    """Inputs read once, outputs written once; two matrix products forward and
    five backward over the keys a query sees."""
    rows = case["B"] * case["H"] * case["N"]
    N, d = case["N"], case["d"]
    pairs = rows * ((N + 1) / 2 if case["causal"] else N)
    t = rows * d * 2.0
    nb = nf = 0.0
    if case["op"] != "bwd":
        nb += 4 * t + 4.0 * rows
        nf += 4.0 * pairs * d
    if case["op"] != "fwd":
        nb += 8 * t + 4.0 * rows
        nf += 10.0 * pairs * d
    return {"bytes": nb, "flops": nf}


def tolerance(case):
    """Outputs are bf16 sums over products of bf16-rounded probabilities: 1.9e-3
    to 2.5e-3 against 64 bits at every listed case, so four times that between
    two such paths.  "max" is over the larger of the value and the output's
    root mean square: measured 0.02 with a full mask, and up to 0.18 with a
    causal one, whose first rows see few keys and are many times the typical row."""
    return {"rel": 1e-2, "max": 0.7 if case["causal"] else 0.1}


def exact(case, seed):
    """The same outputs in 64 bits, from the definitions, on blocks of query rows."""
    t = [x.double() for x in _inputs(case, seed)]
    q, k, v = t[:3]
    B, H, N, d = q.shape
    scale = 1.0 / math.sqrt(d)
    bwd, fwd = case["op"] != "fwd", case["op"] != "bwd"
    out = {}
    if fwd:
        out["o"] = torch.empty_like(q)
        out["lse"] = torch.empty((B, H, N), dtype=torch.float64, device=q.device)
    if bwd:
        for name in ("dq", "dk", "dv"):
            out[name] = torch.zeros_like(q)
    step = max(1, min(N, (1 << 26) // N))
    cols = torch.arange(N, device=q.device)
    for b in range(B):
        for h in range(H):
            kh, vh = k[b, h], v[b, h]
            kt, vt = kh.t().contiguous(), vh.t().contiguous()
            for r in range(0, N, step):
                e = min(N, r + step)
                m = e if case["causal"] else N  # keys past the block's last row are masked
                s = (q[b, h, r:e] @ kt[:, :m].contiguous()) * scale
                if case["causal"]:
                    s.masked_fill_(cols[None, :m] > cols[r:e, None], float("-inf"))
                lse = torch.logsumexp(s, dim=1)
                p = torch.exp_(s.sub_(lse[:, None]))
                o = p @ vh[:m]
                if fwd:
                    out["o"][b, h, r:e] = o
                    out["lse"][b, h, r:e] = lse
                if bwd:
                    do = t[3][b, h, r:e]
                    out["dv"][b, h, :m] += p.t().contiguous() @ do
                    ds = (do @ vt[:, :m].contiguous()).sub_((do * o).sum(1, keepdim=True)).mul_(p).mul_(scale)
                    out["dq"][b, h, r:e] = ds @ kh[:m]
                    out["dk"][b, h, :m] += ds.t().contiguous() @ q[b, h, r:e]
    return out
