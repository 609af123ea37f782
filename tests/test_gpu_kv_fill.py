"""Row shares that fill the rounds of the suffix backward's key-outer-only
launch: prefix key tiles cut into R shares come first, the suffix key tiles,
whole, last.  The choice is pinned on the CPU through the workspace sizes (R
partials of dK and dV for R > 1), then whole packed schedules with R = 1 (order
only), 2 and 4 are checked on sampled rows and keys, bitwise rerun, against the
padded layout, and with a workspace that only holds the shared launch."""
import numpy as np
import pytest

from sampled_checks import sampled_errors
from synthetic import GroupShape, make_group
from test_row_share_rule import _suffix_ws

TOL = 2e-2
CASES = [  # shape, shares of the prefix key tiles
    (GroupShape(32, 4, 128, 5200, (760, 333, 800, 601, 640, 700), "bf16"), 2),
    (GroupShape(32, 4, 64, 2900, (900, 899, 811, 900, 847, 880, 900, 840, 850, 833), "bf16"), 4),
    (GroupShape(32, 4, 128, 10000, (1500, 1311, 1402), "bf16"), 1),
]
IDS = ["r2_d128", "r4_d64", "r1_d128"]


def _sizes(shape):
    from paper_2606_01143_amd import binding as B
    dims = B.make_dims(shape.num_q_heads, shape.num_kv_heads, shape.head_dim, shape.prefix_len, "bf16")
    n, ml, T = shape.n, max(shape.suffix_lens), shape.total_suffix
    return B, dims, n, ml, T


def _fixed_bytes(shape):
    """row statistic and log2 LSE, and the query-outer key splits' dQ"""
    n, ml, T, hq = shape.n, max(shape.suffix_lens), shape.total_suffix, shape.num_q_heads
    up = lambda x: -(-x // 256) * 256
    nrb, nkt = -(-ml // 128) * hq * n, -(-shape.prefix_len // 64) + -(-ml // 64)
    ns = 1 if nrb >= 512 else max(1, min(nkt // 16, -(-512 // nrb), 8))
    return 2 * up(hq * T * 4) + (up(ns * T * hq * shape.head_dim * 4) if ns > 1 else 0)


@pytest.mark.parametrize("shape,r", CASES, ids=IDS)
def test_rule(shape, r):
    B, dims, n, ml, T = _sizes(shape)
    part = (shape.prefix_len + T) * shape.num_kv_heads * shape.head_dim * 4
    want = _fixed_bytes(shape) + (2 * -(-r * part // 256) * 256 if r > 1 else 0)
    assert B.workspace_size(B.OP_SUFFIX_BWD, dims, n, ml, T) == want


@pytest.mark.gpu
@pytest.mark.parametrize("shape,r", CASES, ids=IDS)
def test_filled_rounds_match_oracle(gpu, shape, r):
    import torch
    from paper_2606_01143_amd.group import DeviceGroup
    print(f"\n[gpu kv fill] {shape} shares={r}", flush=True)
    inp = make_group(shape, seed=6)
    mbs = [(0, shape.n)]
    grp = DeviceGroup(inp, dense=False)
    grp.run_schedule(mbs)
    got = grp.fetch("schedule")
    errs = sampled_errors(inp, got, np.random.default_rng(0))
    assert all(v <= TOL for v in errs.values()), errs
    grp.run_schedule(mbs)
    again = grp.fetch("schedule")
    assert all(np.array_equal(got[k], again[k]) for k in got)
    B, dims, n, ml, T = _sizes(shape)
    assert _key_outer_launches(B, grp, 0, n) == 2
    if r > 1:
        # the shared launch, in a workspace that holds no more than it needs
        base = _suffix_ws(shape.num_q_heads, shape.num_kv_heads, shape.head_dim, shape.prefix_len, n, ml, T, False)[0]
        assert base < B.workspace_size(B.OP_SUFFIX_BWD, dims, n, ml, T)
        full, grp.ws = grp.ws, torch.empty(base, dtype=torch.uint8, device="cuda")
        B.gkv_cache_zero(dims, grp.gk, grp.gv)
        assert _key_outer_launches(B, grp, 0, n) == 1
        grp.ws = full
        grp._prefix_bwd(True, None)
        small = sampled_errors(inp, grp.fetch("schedule"), np.random.default_rng(0))
        assert all(v <= TOL for v in small.values()), small
    del grp
    pad = DeviceGroup(inp, dense=False, layout="padded")
    pad.run_schedule(mbs)
    pad.gather_padded_outputs()
    padded = pad.fetch("schedule")
    assert all(np.array_equal(got[k], padded[k]) for k in got)


def _key_outer_launches(B, grp, a, b):
    """launches of both roles that the suffix backward of [a, b) makes"""
    B.profile_enable(True, "bwd_bf16")
    try:
        B.profile_reset()
        grp._suffix_bwd(a, b, None)
        return B.profile_query("bwd_bf16")[1]
    finally:
        B.profile_enable(False)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,taken", [(GroupShape(32, 4, 128, 8737, (500, 333), "bf16"), (True, False)),
                                         (GroupShape(32, 8, 128, 4957, (385, 512, 352), "bf16"), (True, True, False)),
                                         (GroupShape(32, 8, 128, 3700, (385, 512), "bf16"), (False, False))],
                         ids=["hkv4", "hkv8", "shared"])
def test_one_suffix_that_fills_a_round_matches_oracle(gpu, shape, taken):
    """One suffix per microbatch, its prefix and suffix key tiles filling one
    round of the key-outer-only launch to 70%, partial tiles at both ends; the
    launch is taken for the sizes it gains at, and for 48 steps (352 has 44)."""
    from paper_2606_01143_amd import binding as B
    from paper_2606_01143_amd.group import DeviceGroup
    print(f"\n[gpu kv fill] lone {shape}", flush=True)
    for s in shape.suffix_lens:
        blocks = (-(-shape.prefix_len // 192) + -(-s // 192)) * shape.num_kv_heads
        assert 0.7 * 256 <= blocks <= 256
    inp = make_group(shape, seed=7)
    grp = DeviceGroup(inp, dense=False)
    grp.run_schedule()
    assert tuple(_key_outer_launches(B, grp, i, i + 1) == 2 for i in range(shape.n)) == taken
    grp.run_schedule()
    errs = sampled_errors(inp, grp.fetch("schedule"), np.random.default_rng(0))
    assert all(v <= TOL for v in errs.values()), errs
