"""Infinite and NaN inputs stay where the equations put them: an output is
non-finite only if it sums over the pair that holds the value, and an infinite
value with a positive weight gives an infinity, not a NaN."""
import sys

import numpy as np
import pytest

from synthetic import GroupShape, make_group

pytestmark = pytest.mark.gpu


def _say(*what):
    sys.stderr.write("\n[gpu-case] " + " ".join(map(str, what)) + "\n")
    sys.stderr.flush()


@pytest.mark.parametrize("lens,P", [((24, 7), 2048), ((128,), 1792)], ids=["packed_rows_9_splits", "one_head_7_splits"])
def test_infinite_value_in_the_last_key_split(gpu, lens, P):
    """The merge of key splits, whose number is no multiple of the four it
    loads together: V = +Inf at one key of the last split, which every row
    sees, gives +Inf in that column and finite values elsewhere."""
    from paper_2606_01143_amd import binding as B
    from paper_2606_01143_amd.group import DeviceGroup
    shape = GroupShape(8, 2, 128, P, lens, "bf16")
    _say("infinite V", shape)
    n, ml, T = shape.n, max(lens), shape.total_suffix
    up = lambda x: -(-x // 256) * 256
    splits = 9 if P == 2048 else 7
    assert B.workspace_size(B.OP_SUFFIX_FWD, B.make_dims(8, 2, 128, P, "bf16"), n, ml, T) == \
        up(splits * T * 8 * 128 * 4) + up(splits * T * 8 * 4)
    inp = make_group(shape, seed=2)
    if n > 1:  # the suffixes' own keys are the last split
        inp["v_s"][np.asarray(inp["cu_seqlens"][:-1]), :, 5] = np.inf
    else:      # the last split ends the prefix
        inp["v_p"][P - 1, :, 5] = np.inf
    grp = DeviceGroup(inp, dense=False)
    grp._suffix_fwd(0, n, grp.ws, None)
    o = grp.out["o_s"].float().cpu().numpy()
    assert np.all(np.isposinf(o[..., 5]))
    assert np.all(np.isfinite(np.delete(o, 5, axis=-1)))


def _visible(P, lens):
    """[rows, keys] over prefix rows then suffix rows, and the same for keys."""
    T = sum(lens)
    vis = np.zeros((P + T, P + T), bool)
    vis[:P, :P] = np.tril(np.ones((P, P), bool))
    r = P
    for n in lens:
        vis[r:r + n, :P] = True
        vis[r:r + n, r:r + n] = np.tril(np.ones((n, n), bool))
        r += n
    return vis


def _reached(what, at, vis, heads, hkv):
    """Which (row, q head) and (key, kv head) a NaN of tensor `what` at row or
    key `at` (q heads `heads`) reaches: o, lse, dq, dk, dv."""
    rows, hq = vis.shape[0], 4
    g = hq // hkv
    o, lse, dq = (np.zeros((rows, hq), bool) for _ in range(3))
    dk, dv = (np.zeros((rows, hkv), bool) for _ in range(2))
    for h in heads:
        hit = np.zeros(rows, bool)  # rows whose scores, or dS, hold a NaN
        if what in ("q", "do"):
            hit[at] = True
        else:
            hit = vis[:, at].copy()
        keys = vis[hit].any(0)
        dq[:, h] |= hit
        dk[:, h // g] |= keys
        if what in ("q", "k"):
            lse[:, h] |= hit
        if what != "do":
            o[:, h] |= hit
        if what != "v":
            dv[:, h // g] |= keys
    return dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)


@pytest.mark.parametrize("P,lens,d,packed", [(45, (20, 37), 64, False), (45, (20, 37), 128, True),
                                             (150, (70, 33), 128, True)], ids=["d64", "d128_packed", "two_tiles"])
def test_f32_nan_reaches_only_visible_pairs(gpu, P, lens, d, packed):
    """fp32 storage, forward and backward: the matrix instruction multiplies a
    hidden pair's zero by whatever the tile holds, so hidden pairs of diagonal
    and partial tiles have to be kept out of it."""
    from paper_2606_01143_amd.group import DeviceGroup
    hkv = 2
    shape = GroupShape(4, hkv, d, P, lens, "f32")
    _say("f32 NaN", shape)
    vis = _visible(P, lens)
    clean = None
    for what, at in [(None, 0)] + [(w, x) for w in ("q", "k", "v", "do") for x in (19, P - 1, P + lens[0] + 10)]:
        inp = make_group(shape, seed=3)
        heads = (0, 1) if what in ("k", "v") else (1,)
        if what:
            name = {"do": ("g_y", "do_s")}.get(what, (what + "_p", what + "_s"))[at >= P]
            inp[name][at - (P if at >= P else 0), 0 if what in ("k", "v") else 1, 7] = np.nan
        grp = DeviceGroup(inp, dense=False)
        grp.run_schedule([(0, shape.n)] if packed else None)
        got = grp.fetch("schedule")
        cat = {k: np.concatenate([got[k + "_p"], got[k + "_s"]]) for k in ("o", "lse", "dq", "dk", "dv")}
        if clean is None:
            clean = cat
            continue
        for k, want in _reached(what, at, vis, heads, hkv).items():
            bad = ~np.isfinite(cat[k] if k == "lse" else cat[k].sum(-1))
            assert np.array_equal(bad, want), (what, at, k, np.argwhere(bad != want)[:5])
            # the others are what they are without the NaN
            assert np.allclose(cat[k][~want], clean[k][~want], rtol=1e-4, atol=1e-4), (what, at, k)


def test_f32_infinite_value_at_the_last_key(gpu):
    """Tiles that end past the last key repeat it: the repeats' zero weights
    must not turn its infinity into a NaN."""
    from paper_2606_01143_amd.group import DeviceGroup
    P, lens = 45, (20, 37)
    inp = make_group(GroupShape(4, 2, 64, P, lens, "f32"), seed=3)
    _say("f32 Inf at the last prefix key")
    inp["v_p"][P - 1, :, 3] = np.inf
    grp = DeviceGroup(inp, dense=False)
    grp.run_schedule()
    got = grp.fetch("schedule")
    assert np.all(np.isposinf(got["o_s"][..., 3])) and np.all(np.isposinf(got["o_p"][P - 1, :, 3]))
    assert np.all(np.isfinite(got["o_p"][:P - 1])) and np.all(np.isfinite(np.delete(got["o_s"], 3, axis=-1)))


@pytest.mark.parametrize("dtype,hq", [("f32", 4), ("f32", 64), ("bf16", 4)], ids=["f32_key_halves", "f32", "bf16"])
def test_rows_whose_scores_are_all_minus_infinity(gpu, dtype, hq):
    """log 0: LSE is -Inf for a row without any finite score, in every form."""
    from paper_2606_01143_amd.group import DeviceGroup
    shape = GroupShape(hq, 2, 64, 1030, (20, 37), dtype)
    inp = make_group(shape, seed=3)
    _say("all scores -Inf", shape)
    for k in ("k_p", "k_s"):
        inp[k][...] = -1.0
    for k in ("q_p", "q_s"):
        inp[k][:, 1] = 2.0 ** 127
    grp = DeviceGroup(inp, dense=False)
    grp.run_schedule()
    got = grp.fetch("schedule")
    for k in ("lse_p", "lse_s"):
        assert np.all(np.isneginf(got[k][:, 1])), k
        assert not np.any(np.isneginf(np.delete(got[k], 1, axis=1))), k
