"""When the suffix backward runs its key-outer role in a launch of its own
whose rounds the prefix tiles' row shares fill.  The rule is restated here
from its description; its share count is compared with the library's through
the workspace sizes, its decision with the launches the library makes (GPU),
and its claim - the launch keeps its 256 slots busy whatever the lengths - by
replaying the launch with the true lengths as a list schedule.  One suffix per
microbatch: uncut, by an estimate of both ways' times, which is restated and
checked the same way."""
import heapq
import sys

import numpy as np
import pytest

from test_row_share_rule import _causal, _suffix_r, _suffix_ws, _tiles, _wide

SLOTS, TILE_COST, SHARE_STEPS = 256, 8, 128


def _shares(hq, hkv, P, n, ml, d=128):
    """R for suffixes of equal length, 0: not this form"""
    g = hq // hkv
    steps, longest = g * _tiles(n * ml, 32), g * _tiles(ml, 32)
    wide = _tiles(P, 192) * steps + n * _causal(ml, g, 192)
    nt = _tiles(P, 192) * hkv
    if not _wide(wide, hkv, False) or P == 0 or nt * 100 >= 85 * SLOTS * _tiles(nt, SLOTS):
        return 0
    sfx = n * _causal(ml, g, 192) * hkv
    work, even = sfx + n * _tiles(ml, 192) * hkv * TILE_COST, (nt * steps + sfx) // SLOTS
    best = None
    for r in range(1, 9):
        if steps // r < SHARE_STEPS or 10 * (steps // r) < 9 * longest:
            break
        share = _tiles(steps, r) + TILE_COST
        full, last = divmod(nt * r, SLOTS)
        rest = (last * share + work) // SLOTS
        t = full * share + (max(share, rest) if last else rest)
        if best is None or t < best[0]:
            best = (t, r)
    return best[1] if best and 100 * best[0] <= 117 * even and _pays(hq, hkv, P, n, ml, n * ml, best[1], d) else 0


def _pays(hq, hkv, P, n, ml, rows, r, d=128):
    g = hq // hkv
    nt, steps, longest = _tiles(P, 192) * hkv, g * _tiles(rows, 32), g * _tiles(ml, 32)
    sfx = _causal(ml, g, 192) * (256 * rows // ml) // 256 * hkv
    work = sfx + (rows // 192 + n) * hkv * TILE_COST
    share, whole = _tiles(steps, r) + TILE_COST, steps // r
    full, last = divmod(nt * r, SLOTS)
    rest = (last * share + work) // SLOTS
    t = max(full * share + (max(share, rest) if last else rest), full * share + longest + TILE_COST,
            (nt * r * share + work) // SLOTS + (longest + TILE_COST) // 2)
    useful = nt * steps + sfx
    limit = 125
    if rows == n * ml or _tiles(P, 192) <= 13:
        limit = 160 if rows == n * ml or _tiles(P, 192) <= 6 else 144
    if rows != n * ml and d == 64:
        limit = 180
    return whole >= 100 and 100 * t * SLOTS <= limit * useful


def _utilisation(hq, hkv, P, lens, r):
    """of the launch's slots, its blocks started in order on the first free one"""
    g = hq // hkv
    jobs = [_tiles(g * _tiles(sum(lens), 32), r) + TILE_COST] * (_tiles(P, 192) * hkv * r)
    for n in lens:
        jobs += [g * _tiles(n - k, 32) + TILE_COST for k in range(0, n, 192) for _ in range(hkv)]
    slots = [0] * SLOTS
    for j in jobs:
        heapq.heappush(slots, heapq.heappop(slots) + j)
    return sum(jobs) / SLOTS / max(slots)


def _random_groups(rng, count):
    log = lambda lo, hi: int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))
    for i in range(count):
        hq, hkv = ((32, 8), (32, 8), (32, 4), (16, 8), (8, 8))[rng.integers(5)]
        P, n = log(500, 20000), int(rng.integers(2, 17))
        if i % 4 == 0:    # one long suffix among short ones
            lens = [log(50, 400) for _ in range(n - 1)] + [log(800, 2048)]
        elif i % 4 == 1:  # within a factor of five
            m = log(150, 2048)
            lens = [max(1, int(m * rng.uniform(0.2, 1))) for _ in range(n)]
        else:
            lens = [log(100, 2048) for _ in range(n)]
        yield hq, hkv, P, [lens[k] for k in rng.permutation(n)]


def test_share_counts_follow_the_rule():
    from paper_2606_01143_amd import binding as B
    up = lambda x: -(-x // 256) * 256
    seen = set()
    for i, (hq, hkv, P, lens) in enumerate(_random_groups(np.random.default_rng(1), 600)):
        n, ml, T, d = len(lens), max(lens), sum(lens), (128, 64)[i % 2]
        r = _shares(hq, hkv, P, n, ml, d)
        base, rb = _suffix_ws(hq, hkv, d, P, n, ml, T, False)
        fixed = base - (2 * up(rb * (P + T) * hkv * d * 4) if rb > 1 else 0)
        want = fixed + (2 * up(r * (P + T) * hkv * d * 4) if r > 1 else 0) if r else base
        assert B.workspace_size(B.OP_SUFFIX_BWD, B.make_dims(hq, hkv, d, P, "bf16"), n, ml, T) == max(want, base)
        seen.add(r)
    assert {0, 1, 2, 3, 4} <= seen


def test_the_form_keeps_its_slots_busy():
    for d, long, bound in ((128, True, 0.70), (128, False, 0.58), (64, True, 0.49), (64, False, 0.49)):
        taken, refused = [], []
        for hq, hkv, P, lens in _random_groups(np.random.default_rng(2), 2500):
            n, ml = len(lens), max(lens)
            r = _shares(hq, hkv, P, n, ml, d)
            if r and (P > 13 * 192) == long:
                u = _utilisation(hq, hkv, P, lens, r)
                (taken if _pays(hq, hkv, P, n, ml, sum(lens), r, d) else refused).append(u)
        assert len(taken) > 100 and min(taken) >= bound, (d, long, len(taken), min(taken))
        assert len(refused) > 100 and min(refused) < 0.5  # what the equal-length choice alone would run


MANY = tuple(2 + 7 * i % 29 for i in range(1100))  # more lengths than a gather block adds up
PACKED = [  # hq, hkv, d, P, lens: taken?
    (32, 4, 128, 5200, (760, 333, 800, 601, 640, 700), True),
    (32, 4, 128, 10000, (1500, 1311, 1402), True),
    (32, 8, 64, 1418, (600, 1000, 900, 800, 700, 950, 600, 1000, 900, 800, 700, 950), True),
    (32, 4, 64, 687, (105, 1992, 538, 163, 658, 341), False),
    (32, 4, 128, 1306, (428, 410, 2046, 228, 323), False),
    (32, 8, 64, 1462, (1595, 319, 329, 374, 146, 164), True),
    (32, 8, 64, 1608, (214, 135, 1588, 1744, 371, 147), True),
    (32, 8, 128, 1846, (166, 1882, 1309, 136, 1420, 603), True),
    (32, 8, 128, 1075, (154, 2003, 121, 56, 63), False),
    (32, 8, 128, 2048, (1024,) * 4, True),
    (32, 4, 64, 1800, MANY, True),
    (16, 4, 64, 1600, (1, 2) * 550 + (40,), False),
]


def test_the_listed_groups_take_the_form_or_not():
    refused = 0
    for hq, hkv, d, P, lens, taken in PACKED:
        n, ml = len(lens), max(lens)
        r = _shares(hq, hkv, P, n, ml, d)
        assert (r > 0 and _pays(hq, hkv, P, n, ml, sum(lens), r, d)) == taken, (P, lens)
        refused += r > 0 and not taken
    assert refused >= 3  # a choice that padded calls make on the device


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d,P,lens,taken", PACKED, ids=[f"hkv{c[1]}_d{c[2]}_p{c[3]}" for c in PACKED])
def test_launches_and_bits(gpu, hq, hkv, d, P, lens, taken):
    """The launches the suffix backward makes, its outputs on sampled rows and
    keys, and the padded call's bits, whose choice is made on the device."""
    from paper_2606_01143_amd import binding as B
    from paper_2606_01143_amd.group import DeviceGroup
    from sampled_checks import sampled_errors
    from synthetic import GroupShape, make_group
    shape = GroupShape(hq, hkv, d, P, lens, "bf16")
    sys.stderr.write(f"\n[gpu-case] fill rule {shape}\n")
    sys.stderr.flush()
    inp = make_group(shape, seed=6)
    got = {}
    for layout in ("packed", "padded"):
        grp = DeviceGroup(inp, dense=False, layout=layout)
        grp.run_schedule([(0, shape.n)])
        if layout == "packed":
            B.gkv_cache_zero(grp.dims, grp.gk, grp.gv)
            B.profile_enable(True, "bwd_bf16")
            try:
                B.profile_reset()
                grp._suffix_bwd(0, shape.n, None)
                assert B.profile_query("bwd_bf16")[1] == (2 if taken else 1)
            finally:
                B.profile_enable(False)
            grp.run_schedule([(0, shape.n)])
        else:
            grp.gather_padded_outputs()
        got[layout] = grp.fetch("schedule")
        del grp
    if P < 2000 and len(lens) < 100:
        errs = sampled_errors(inp, got["packed"], np.random.default_rng(0))
        assert all(v <= 2e-2 for v in errs.values()), errs
    assert all(np.array_equal(got["packed"][k], got["padded"][k]) for k in got["packed"])


def _lone(hq, hkv, P, S):
    """one suffix: estimated gain of the key-outer-only launch, 0 outside its range"""
    g = hq // hkv
    pre, sfx, steps = _tiles(P, 192) * hkv, _tiles(S, 192) * hkv, g * _tiles(S, 32)
    rounds = _tiles(pre + sfx, SLOTS)
    if steps < 48 or (pre + sfx) * 100 < (70 if rounds == 1 else 85) * SLOTS * rounds:
        return 0
    sweep, work = steps + TILE_COST, _causal(S, g, 192) * hkv + sfx * TILE_COST
    full, last = divmod(pre, SLOTS)
    key = (full + 1) * sweep
    if last + sfx > SLOTS:
        key = max(key, full * sweep + (last * sweep + work) / SLOTS, (pre * sweep + work) / SLOTS + sweep / 2)
    pt, st, blocks = _tiles(P, 64), _tiles(S, 64), _tiles(S, 128) * hq
    ns = 1 if blocks >= 512 else max(1, min((pt + st) // 16, _tiles(512, blocks), 8))
    query = _tiles(blocks * ns, 512) * ((pt + (st + 2) / 2) / ns + 2)
    shared = 33.5 + 1.35 * (pt * steps + _causal(S, g)) * hkv / 512 + 2.71 * blocks * (pt + (st + 1) / 2) / 512
    return shared / (24 + 1.62 * key + 1.55 * query)


LONE = [  # hq, hkv, P, S: taken?
    (32, 8, 4060, 512, True),     # one 64-key tile of prefix past the line
    (32, 8, 4032, 512, False),
    (32, 4, 8737, 161, True),     # 48 steps
    (32, 4, 8737, 160, False),    # 40
    (16, 8, 10236, 964, True),    # two rounds
    (8, 8, 2403, 1890, False),    # 72% of a round by count, half of it by work
    (32, 8, 2685, 1592, False),
    (32, 8, 3700, 512, False),
]


def test_one_suffix_fills_its_launch_or_shares():
    for hq, hkv, P, S, taken in LONE:
        assert (_lone(hq, hkv, P, S) >= 1.01) == taken, (hq, hkv, P, S)
    rng = np.random.default_rng(3)
    log = lambda lo, hi: int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))
    taken, refused = [], []
    for _ in range(4000):
        hq, hkv = ((32, 8), (32, 8), (32, 4), (16, 8), (8, 8))[rng.integers(5)]
        P, S = log(500, 20000), log(100, 2048)
        gain = _lone(hq, hkv, P, S)
        if gain:
            (taken if gain >= 1.01 else refused).append(_utilisation(hq, hkv, P, [S], 1))
    assert len(taken) > 200 and min(taken) >= 0.70, (len(taken), min(taken))
    assert len(refused) > 100 and min(refused) < 0.6  # what the count of tiles alone would run


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,P,S,taken", LONE)
def test_one_suffix_launches(gpu, hq, hkv, P, S, taken):
    """The launches of the call; both forms' outputs are checked elsewhere."""
    import torch
    from paper_2606_01143_amd import binding as B
    sys.stderr.write(f"\n[gpu-case] fill rule, one suffix {hq, hkv, P, S}\n")
    sys.stderr.flush()
    d, dims = 128, B.make_dims(hq, hkv, 128, P, "bf16")
    bf = lambda *shape: torch.zeros(*shape, dtype=torch.bfloat16, device="cuda")
    f32 = lambda *shape: torch.zeros(*shape, dtype=torch.float32, device="cuda")
    kp, vp, gk, gv = bf(P, hkv, d), bf(P, hkv, d), f32(P, hkv, d), f32(P, hkv, d)
    q, k, v, o, do = bf(S, hq, d), bf(S, hkv, d), bf(S, hkv, d), bf(S, hq, d), bf(S, hq, d)
    cu = torch.tensor([0, S], dtype=torch.int32, device="cuda")
    ws = torch.empty(B.workspace_size(B.OP_SUFFIX_BWD, dims, 1, S, S), dtype=torch.uint8, device="cuda")
    B.profile_enable(True, "bwd_bf16")
    try:
        B.profile_reset()
        B.suffix_attn_bwd_accum(dims, kp, vp, q, k, v, o, f32(S, hq), do, cu, 1, S, S, torch.empty_like(q),
                                torch.empty_like(k), torch.empty_like(v), gk, gv, ws)
        assert B.profile_query("bwd_bf16")[1] == (2 if taken else 1)
    finally:
        B.profile_enable(False)
