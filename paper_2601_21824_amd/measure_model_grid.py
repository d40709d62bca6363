"""Measure the ordered schedules over a grid of shapes on the GPU: the data
behind the block-step times of the DAG model that picks DASH_SCHED_AUTO.

For d in (64, 128, 256), both masks, N from 512 (d = 128 and 256: from 64) to 16384
(d = 256: 32768) and B*H from 1 to 1024 heads (see shapes; at most 2^21 tokens and
6e13 FLOPs per call), every candidate deterministic schedule is timed over
back-to-back calls between two events, after 3 checked warm-up calls, at least
10 ms of work per timing and up to 400 calls, four times in alternating order; the
best is kept.  One JSON line per shape on stdout, in the format of
``bench.py --sweep``:

    python -m paper_2601_21824_amd.measure_model_grid > paper_2601_21824_amd/model_grid.jsonl

(Head dims as arguments measure only those, e.g. ``... measure_model_grid 64``;
``--heads 32,128`` only those head counts, ``--mask causal`` only that mask.)
"""
from __future__ import annotations

import json
import sys

HEADS = (1, 2, 4, 5, 8, 10, 16, 20, 32, 40, 64, 80, 128, 160, 256, 320, 512, 640, 1024)


def shapes(dims=(64, 128, 256), heads=HEADS, masks=(False, True)):
    for d in dims:
        # (192 to 768: there most calls change their tile, which cuts a line between two lengths short)
        lengths = (64, 128, 192, 256, 384, 512, 768, 1024, 2048, 4096, 8192, 16384, 32768)[:13 if d == 256 else 12]
        if d == 64:
            lengths = (512, 1024, 2048, 4096, 8192, 16384)
        for causal in masks:
            grid = [(n, bh) for n in lengths for bh in heads]
            if d != 64 and not causal:  # one round of 128-row tiles and a few more, which the grid passes over
                grid += [(n, 36864 // n) for n in (384, 768, 1536, 3072, 6144, 12288)]
            for n, bh in grid:
                flops = 4.0 * bh * n * n * d * 2.5 / (2 if causal else 1)
                if bh * n <= (1 << 21) and flops <= 6e13:
                    yield d, causal, n, bh


def main(*dims):
    import torch

    from paper_2601_21824_amd import binding as dash

    heads = HEADS
    if "--heads" in dims:
        i = dims.index("--heads")
        heads = tuple(int(x) for x in dims[i + 1].split(","))
        dims = dims[:i] + dims[i + 2:]
    masks = (False, True)
    if "--mask" in dims:
        i = dims.index("--mask")
        masks = (dims[i + 1] == "causal",)
        dims = dims[:i] + dims[i + 2:]
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for d, causal, N, bh in shapes(tuple(int(x) for x in dims) or (64, 128, 256), heads, masks):
        g = torch.Generator(device="cuda")
        g.manual_seed(N + d + bh)
        q, k, v, do = (torch.randn((1, bh, N, d), generator=g, device="cuda", dtype=torch.bfloat16) * (0.5 if d == 256 else 1.0)
                       for _ in range(4))
        o, lse = dash.attn_fwd(q, k, v, causal)
        dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        ws = dash.new_workspace(1, bh, N, d, "shift")

        def ms(sched, calls):
            begin.record()
            for _ in range(calls):
                dash.dash_attn_bwd(q, k, v, o, do, lse, dq, dk, dv, causal, sched, workspace=ws)
            end.record()
            end.synchronize()
            if dash.dash_bwd_check(ws) != dash.DASH_OK:
                raise RuntimeError(f"{sched}: ordering wait timed out")
            return begin.elapsed_time(end) / calls

        scheds = ["descending", "symshift", "naive"] if causal else ["shift", "descending", "naive"]
        calls = {s: max(2, min(400, int(10.0 / min(ms(s, 1) for _ in range(3))))) for s in scheds}
        best = {}
        for order in (scheds, scheds[::-1]) * 2:
            for s in order:
                best[s] = min(best.get(s, 1e30), ms(s, calls[s]))
        flops = 4.0 * bh * N * N * d * 2.5 / (2 if causal else 1)
        row = {"B": 1, "H": bh, "N": N, "d": d, "mask": "causal" if causal else "full"}
        row.update({s: float(f"{flops / (best[s] * 1e-3) / 1e12:.4g}") for s in scheds})
        print(json.dumps(row), flush=True)
        del q, k, v, do, o, lse, dq, dk, dv, ws
        torch.cuda.empty_cache()
    return 0


if __name__ == "__main__":
    sys.exit(main(*sys.argv[1:]))
