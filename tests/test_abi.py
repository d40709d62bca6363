"""C-ABI checks that need no GPU: the library loads and exports every symbol
the header declares, argument errors are reported before any device work, and
the schedule the kernels follow equals the oracle's independent enumeration
(bit-exact integer tables)."""
import ctypes
import os
import re

import numpy as np
import pytest

from oracle import schedule as osched
from paper_2601_21824_amd import binding as b

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    text = open(os.path.join(ROOT, "include", "dash.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dash_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = b.load()
    names = header_functions()
    assert set(names) == set(b.EXPORTS)
    for n in names:
        assert hasattr(lib, n), n


def call_bwd(lib, ptr, B=1, H=1, N=128, d=64, causal=0, sched=1):
    p = [ctypes.c_void_p(ptr)] * 9
    return lib.dash_attn_bwd(*p, B, H, N, d, causal, sched)


def test_argument_errors_without_device():
    lib = b.load()
    assert call_bwd(lib, 0) == b.DASH_ERR_INVALID_ARG  # null pointers
    assert call_bwd(lib, 4096, d=96) == b.DASH_ERR_INVALID_ARG
    assert call_bwd(lib, 4096, N=-1) == b.DASH_ERR_INVALID_ARG
    assert call_bwd(lib, 4096, B=1 << 14, H=1 << 6, N=1 << 10) == b.DASH_ERR_INVALID_ARG  # 2^30 rows
    assert call_bwd(lib, 4096, sched=9) == b.DASH_ERR_INVALID_ARG
    assert call_bwd(lib, 4096, sched=b.DASH_SCHED_SYMSHIFT, causal=0) == b.DASH_ERR_UNSUPPORTED
    assert "symmetric shift" in b.dash_last_error()
    # empty problems are successful no-ops, even with null pointers
    assert call_bwd(lib, 0, N=0) == b.DASH_OK
    assert call_bwd(lib, 0, B=0) == b.DASH_OK
    assert lib.dash_attn_fwd(*([ctypes.c_void_p(0)] * 5), 1, 1, 0, 64, 0) == b.DASH_OK
    assert lib.dash_attn_fwd(*([ctypes.c_void_p(0)] * 5), 1, 1, 8, 64, 0) == b.DASH_ERR_INVALID_ARG
    assert b.dash_bwd_workspace_size(1, 1, 100, 96) == 0
    assert b.dash_bwd_workspace_size(1, 1, 100, 64, 9) == 0
    assert b.dash_bwd_workspace_size(2, 16, 8192, 128) >= 2 * 16 * 8192 * 128 * 4
    # the partials comparison variant keeps one accumulator-sized buffer per KV tile
    base = b.dash_bwd_workspace_size(2, 16, 8192, 128, "naive")
    assert b.dash_bwd_workspace_size(2, 16, 8192, 128, "partials") >= base + 63 * 2 * 16 * 8192 * 128 * 4
    assert call_bwd(lib, 4096, d=256, sched=b.DASH_SCHED_PARTIALS) == b.DASH_ERR_UNSUPPORTED
    assert call_bwd(lib, 4096, d=256, sched=b.DASH_SCHED_SPLIT) == b.DASH_ERR_UNSUPPORTED
    assert call_bwd(lib, 4096, sched=8) == b.DASH_ERR_INVALID_ARG
    assert lib.dash_bwd_check(ctypes.c_void_p(0), ctypes.c_void_p(0)) == b.DASH_ERR_INVALID_ARG
    # explicit-workspace form: too small a workspace is an argument error
    opts = b.dash_bwd_options_t(0, 0, None, None, None, None, None)
    p = [ctypes.c_void_p(4096)] * 9
    rc = lib.dash_attn_bwd_ex(*p, 1, 1, 128, 64, 0, 1, ctypes.c_float(0.125), ctypes.c_void_p(4096),
                              16, ctypes.byref(opts), None)
    assert rc == b.DASH_ERR_INVALID_ARG
    # an unknown ticket order is an argument error (checked before any device call)
    opts = b.dash_bwd_options_t(0, 0, None, None, None, None, None, 0, 3)
    rc = lib.dash_attn_bwd_ex(*p, 1, 1, 128, 64, 0, 1, ctypes.c_float(0.125), ctypes.c_void_p(4096),
                              1 << 40, ctypes.byref(opts), None)
    assert rc == b.DASH_ERR_INVALID_ARG and "ticket_order" in b.dash_last_error()
    # ... and so is an unknown placement
    opts = b.dash_bwd_options_t(0, 0, None, None, None, None, None, 0, 0, 3)
    rc = lib.dash_attn_bwd_ex(*p, 1, 1, 128, 64, 0, 1, ctypes.c_float(0.125), ctypes.c_void_p(4096),
                              1 << 40, ctypes.byref(opts), None)
    assert rc == b.DASH_ERR_INVALID_ARG and "placement" in b.dash_last_error()
    assert lib.dash_schedule_table(1, 1, 128, 64, 0, 0, None, None, None, None, None) == b.DASH_ERR_INVALID_ARG
    assert lib.dash_schedule_table(1, 0, 128, 64, 0, b.DASH_PLACEMENT_GLOBAL, None, None, None, None, None) == \
        b.DASH_ERR_INVALID_ARG
    # the MFMA peak measurement checks its arguments before touching the device
    assert lib.dash_mfma_peak(0, None) == b.DASH_ERR_INVALID_ARG
    out = ctypes.c_double(0.0)
    assert lib.dash_mfma_peak(-1, ctypes.byref(out)) == b.DASH_ERR_INVALID_ARG


def test_schedule_resolution():
    assert b.dash_resolve_schedule("auto", 128, False) == b.DASH_SCHED_SHIFT
    assert b.dash_resolve_schedule("auto", 128, True) == b.DASH_SCHED_DESCENDING
    assert b.dash_resolve_schedule("auto", 64, True) == b.DASH_SCHED_DESCENDING
    assert b.dash_resolve_schedule("auto", 256, True) == b.DASH_SCHED_DESCENDING
    assert b.dash_resolve_schedule("auto", 256, False) == b.DASH_SCHED_SHIFT
    assert b.dash_resolve_schedule("shift", 64, True) == b.DASH_SCHED_SYMSHIFT
    assert b.dash_resolve_schedule("naive", 64, True) == b.DASH_SCHED_NAIVE


KINDS = {b.DASH_SCHED_NAIVE: osched.NAIVE, b.DASH_SCHED_DESCENDING: osched.DESCENDING,
         b.DASH_SCHED_SHIFT: osched.SHIFT, b.DASH_SCHED_SYMSHIFT: osched.SYMSHIFT,
         b.DASH_SCHED_ATOMIC: osched.NAIVE, b.DASH_SCHED_PARTIALS: osched.NAIVE,
         b.DASH_SCHED_SPLIT: osched.NAIVE}


def tile_rows(sched, d, causal, N, heads):
    """KV tile rows: narrow (128; 64 at d = 256), or twice that when the call has
    tiles enough for 256 workgroups and, at d = 128 and below N = 512 at d = 256, the
    narrow ones take enough more rounds of 256 chains."""
    bc = 64 if d == 256 else 128
    if d != 64 and sched in (b.DASH_SCHED_ATOMIC, b.DASH_SCHED_SPLIT):
        return bc
    tiles = heads * -(-N // (2 * bc))
    if tiles < {64: (256, 512), 128: (160, 384), 256: (128, 192)}[d][causal]:
        return bc
    if causal and N < {64: 1024, 128: 257, 256: 0}[d] or d == 256 and heads == 1:
        return bc
    if d == 64 or d == 256 and N >= 512 or d == 128 and sched == b.DASH_SCHED_SYMSHIFT and N > 8192:
        return 2 * bc

    even = not causal or sched == b.DASH_SCHED_SYMSHIFT
    fill, start = (0.5, 1.0) if d == 128 else (0.25, 0.0)

    def time(rows, step, start):
        chains = [-(-N // 64) - (j * rows // 64 if causal else 0) for j in range(-(-N // rows))]
        if sched == b.DASH_SCHED_SYMSHIFT:
            chains = [sum(chains) / -(-len(chains) // 2)] * -(-len(chains) // 2)
        n = heads * len(chains)
        rounds, mean = -(-n // 256), sum(chains) / len(chains)
        if even:
            return step * rounds * mean
        return max(step * (fill * rounds + (1 - fill) * n / 256) * (mean + start), chains[0] + start)

    step = 1.45 if not even else 1.5 if d == 128 else 1.2
    return 2 * bc if time(bc, 1.0, start / 2) > time(2 * bc, step, start) else bc


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("causal", [False, True])
def test_tile_rows_of_many_calls(d, causal):
    """The tile size of the library's tables over heads and lengths of every kind."""
    rng = np.random.default_rng(d + causal)
    seen = set()
    for _ in range(400):
        N, heads = int(2 ** rng.uniform(4, 13)), int(2 ** rng.uniform(0, 11))
        for s in (0, 1, 2, 4 if causal else 3, 6, 7):
            bc = b.dash_schedule_table(s, N, d, causal, heads=heads)["bc"]
            assert bc == tile_rows(s, d, causal, N, heads), (s, N, heads)
            seen.add(bc)
    assert len(seen) == 2


# (schedule, heads, N, d, causal, rows): the faster tile, both measured.  Short heads and
# a last round that few wide tiles begin: narrow (the wide one took 1.06-1.6 times as long)
FASTER = [("shift", 264, 64, 128, False, 128), ("shift", 264, 128, 128, False, 128), ("naive", 264, 200, 128, False, 128),
          ("shift", 132, 300, 128, False, 128), ("shift", 9, 8192, 128, False, 128), ("shift", 20, 4096, 128, False, 128),
          ("descending", 200, 300, 128, True, 128), ("symshift", 37, 3328, 128, True, 128), ("symshift", 162, 960, 128, True, 128),
          ("shift", 1024, 64, 256, False, 64), ("shift", 128, 128, 256, False, 64), ("symshift", 264, 64, 256, True, 64),
          ("descending", 264, 97, 256, True, 64),
          ("shift", 32, 8192, 128, False, 256), ("symshift", 64, 8192, 128, True, 256), ("descending", 64, 8192, 128, True, 256),
          ("shift", 256, 256, 128, False, 256), ("descending", 1024, 512, 128, True, 256), ("descending", 8, 32768, 256, True, 128),
          ("symshift", 8, 32768, 256, True, 128), ("symshift", 18, 9674, 128, True, 256), ("descending", 72, 387, 256, True, 128), ("shift", 33, 900, 256, False, 128), ("descending", 25, 1280, 256, True, 128)]


@pytest.mark.parametrize("sched,heads,N,d,causal,rows", FASTER)
def test_calls_take_the_faster_tile(sched, heads, N, d, causal, rows):
    assert b.dash_schedule_table(sched, N, d, causal, heads=heads)["bc"] == rows


@pytest.mark.parametrize("placement", [b.DASH_PLACEMENT_GLOBAL, b.DASH_PLACEMENT_XCD])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("N", [64, 200, 256, 1000, 1024, 4096, 4224, 8192, 16384, 32768])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("sched", [0, 1, 2, 3, 4, 6, 7])
@pytest.mark.parametrize("heads", [1, 64])
def test_schedule_table_matches_oracle(heads, sched, causal, N, d, placement):
    if sched == b.DASH_SCHED_SYMSHIFT and not causal:
        pytest.skip("symshift is causal-only")
    tab = b.dash_schedule_table(sched, N, d, causal, placement, heads=heads)
    concrete = b.dash_resolve_schedule(sched, d, causal)
    kind = KINDS[concrete]
    t_r, t_c, br, bc, grp = tab["t_r"], tab["t_c"], tab["br"], tab["bc"], tab["group"]
    # Q tiles of 64 rows (full) or KV-tile rows (causal); Shift groups of at
    # most 256 chains, 32 when every chain of a head runs on one XCD
    assert bc == tile_rows(concrete, d, causal, N, heads)
    assert br == (bc if causal else 64) and t_r * br == t_c * bc
    most = 32 if placement == b.DASH_PLACEMENT_XCD else 256
    assert grp == (min(t_c, most) if kind == osched.SHIFT else tab["chains"])
    ref = osched.build(kind, t_r, t_c, causal, br, bc, group=grp if kind == osched.SHIFT else None)
    assert tab["chains"] == len(ref.chains)
    for w, ch in enumerate(ref.chains):
        n = tab["chain_len"][w]
        assert n == len(ch)
        got = list(zip(tab["task_kv"][w][:n].tolist(), tab["task_q"][w][:n].tolist()))
        assert got == ch, (w, got, ch)
    want = np.full((t_r, t_c), -1)
    for i, js in ref.order.items():
        for r, j in enumerate(js):
            want[i, j] = r
    np.testing.assert_array_equal(tab["rank"], want)
    if kind in (osched.SHIFT, osched.SYMSHIFT):
        props = osched.check(ref, t_r, t_c, causal, br, bc, group=grp if kind == osched.SHIFT else None)
        assert props["coverage"] and props["conflict_free"] and props["monotone"]


def test_missing_library_raises_instead_of_falling_back():
    """With no built library every entry point raises, and CPU tensors are
    refused rather than computed on: there is no CPU fallback."""
    import subprocess
    import sys
    code = (
        "import sys, torch\n"
        f"sys.path.insert(0, {ROOT!r})\n"
        "from paper_2601_21824_amd import binding as b\n"
        "b.LIB_PATH = '/nonexistent/libdash.so'\n"
        "for call in (b.load, lambda: b.dash_resolve_schedule('auto', 128, False),\n"
        "             lambda: b.dash_bwd_workspace_size(1, 1, 64, 64)):\n"
        "    try:\n"
        "        call()\n"
        "        sys.exit(1)\n"
        "    except b.DashError as e:\n"
        "        assert 'is not built' in str(e), e\n"
        "q = torch.zeros(1, 1, 64, 64, dtype=torch.bfloat16)\n"
        "try:\n"
        "    b.attn_bwd(q, q, q, q, q, torch.zeros(1, 1, 64), False, 'shift')\n"
        "    sys.exit(1)\n"
        "except b.DashError as e:\n"
        "    assert 'device tensors' in str(e), e\n"
        "print('ok')\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("N,d", [(8000, 128), (8192, 128), (1000, 64), (32704, 256), (32768, 256), (333, 256)])
@pytest.mark.parametrize("sized_for", ["shift", "auto", "naive", "descending", "atomic", "split"])
def test_workspace_size_serves_every_schedule_and_mask(N, d, sized_for):
    """A workspace of dash_bwd_workspace_size(..., s) bytes passes the size
    check of dash_attn_bwd_ex for every schedule but PARTIALS under both masks
    -- including causal SHIFT, which runs as Symmetric Shift with T_c padded to
    even (odd T_c at N = 8000, d = 128 and N = 32704, d = 256).  The call is
    stopped right after the size check by an invalid option, so no device is
    touched; one byte less is reported as a workspace error."""
    lib = b.load()
    B, H = 2, 3
    ws = b.dash_bwd_workspace_size(B, H, N, d, sized_for)
    assert ws > 0
    p = [ctypes.c_void_p(1 << 20)] * 9
    bad_opts = b.dash_bwd_options_t(-1)  # spin_limit < 0: checked right after the workspace
    for causal in (0, 1):
        for sched in ("atomic", "naive", "descending", "shift", "symshift", "auto", "split"):
            if sched == "symshift" and not causal:
                continue
            if sched == "split" and d > 128:
                continue
            args = (*p, B, H, N, d, causal, b.SCHEDULES[sched], ctypes.c_float(0.125), ctypes.c_void_p(1 << 20))
            rc = lib.dash_attn_bwd_ex(*args, ws, ctypes.byref(bad_opts), None)
            assert rc == b.DASH_ERR_INVALID_ARG and "spin_limit" in b.dash_last_error(), (sched, causal)
            need = b.dash_bwd_workspace_size(B, H, N, d, sched)
            rc = lib.dash_attn_bwd_ex(*args[:-1], ctypes.c_void_p(1 << 20), need - 1, ctypes.byref(bad_opts), None)
            assert rc == b.DASH_ERR_INVALID_ARG and "workspace" in b.dash_last_error(), (sched, causal)
