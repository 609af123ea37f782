"""fp32 storage holds what fp32 holds: softmax weights below 2^-126 keep their
value (fp32 denormals, not zeros).  The tolerance is the spacing of denormals,
2^-149, relative to the weight, plus fp32 rounding of the products."""
import sys

import numpy as np
import pytest

from synthetic import GroupShape, make_group

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq", [2, 64], ids=["key_halves", "one_wave_per_row"])
@pytest.mark.parametrize("d", [64, 128])
def test_weights_below_the_normal_range(gpu, d, hq):
    """Every row sees key 0 with weight 1 and value 0, and other keys with
    weight 2^-130 (log2 scores 0 and -130) and value 2^100: O is their number
    times 2^-30.  Backward of dO = 2^100: dV of those keys is 2^-30 per row."""
    from paper_2606_01143_amd.group import DeviceGroup
    P, lens = 1030, (20, 37)
    shape = GroupShape(hq, hq, d, P, lens, "f32")
    sys.stderr.write(f"\n[gpu-case] f32 weights below 2^-126 {shape}\n")
    sys.stderr.flush()
    inp = make_group(shape, seed=3)
    for k in ("q_p", "q_s", "k_p", "k_s", "v_p", "v_s", "g_y", "do_s"):
        inp[k] = np.zeros_like(inp[k])
    for k in ("q_p", "q_s"):
        inp[k][..., 0] = 1.0
    s = -130.0 * np.log(2.0) * np.sqrt(d)  # log2 weight -130 after 1/sqrt(d) and log2(e)
    for k, v in (("k_p", "v_p"), ("k_s", "v_s")):
        inp[k][..., 0] = s
        inp[v][..., 1] = 2.0 ** 100
    inp["k_p"][0, :, 0] = 0.0
    inp["v_p"][0] = 0.0
    inp["do_s"][..., 2] = 2.0 ** 100
    grp = DeviceGroup(inp, dense=False)
    grp.run_schedule()
    got = grp.fetch("schedule")
    tol = 2.0 ** -18  # 2^-149 / 2^-130, and the score's own rounding 130 * 2^-24
    rows = np.arange(P)  # prefix row r sees r such keys; suffix row t P - 1 + t + 1
    np.testing.assert_allclose(got["o_p"][:, 0, 1], rows * 2.0 ** -30, rtol=tol)
    cu = np.concatenate([[0], np.cumsum(lens)])
    for i, n in enumerate(lens):
        np.testing.assert_allclose(got["o_s"][cu[i]:cu[i + 1], -1, 1], (P + np.arange(n)) * 2.0 ** -30, rtol=tol)
        np.testing.assert_allclose(got["dv_s"][cu[i]:cu[i + 1], 0, 2], (n - np.arange(n)) * 2.0 ** -30, rtol=tol)
    np.testing.assert_allclose(got["g_v"][1:, 0, 2], sum(lens) * 2.0 ** -30, rtol=tol)


@pytest.mark.parametrize("hq", [2, 64], ids=["key_halves", "one_wave_per_row"])
def test_scores_beyond_the_fused_products_range(gpu, hq):
    """Scores of the order of 2^43: products of small integers, exact in fp32,
    so the softmax picks a row's largest ones (equally where several tie).
    Tolerance: one rounding of O and of the LSE."""
    from paper_2606_01143_amd.group import DeviceGroup
    P, lens = 1030, (20, 37)
    shape = GroupShape(hq, hq, 64, P, lens, "f32")
    sys.stderr.write(f"\n[gpu-case] f32 scores of 2^43 {shape}\n")
    sys.stderr.flush()
    inp = make_group(shape, seed=3)
    rng = np.random.default_rng(1)
    for k in ("q_p", "q_s", "k_p", "k_s"):
        inp[k] = (rng.integers(-3, 4, inp[k].shape) * 2.0 ** 20).astype(np.float32)
    grp = DeviceGroup(inp, dense=False)
    grp._suffix_fwd(0, 2, grp.ws, None)
    from paper_2606_01143_amd import binding as B
    B.prefix_fwd(grp.dims, grp.q_p, grp.k_p, grp.v_p, grp.out["o_p"], grp.out["lse_p"])
    got = {k: grp.out[k].cpu().numpy().astype(np.float64) for k in ("o_p", "lse_p", "o_s", "lse_s")}
    cu = [0, lens[0], sum(lens)]
    for h in (0, hq - 1):
        f = lambda k: inp[k][:, h].astype(np.float64)
        seqs = [("p", slice(0, P), f("k_p"), f("v_p"), 0)] + [
            ("s", slice(cu[i], cu[i + 1]), np.concatenate([f("k_p"), f("k_s")[cu[i]:cu[i + 1]]]),
             np.concatenate([f("v_p"), f("v_s")[cu[i]:cu[i + 1]]]), P) for i in (0, 1)]
        for x, rows, k, v, free in seqs:
            s = f("q_" + x)[rows] @ k.T
            s[np.arange(s.shape[1])[None] > free + np.arange(s.shape[0])[:, None]] = -np.inf
            top = s.max(1, keepdims=True)
            w = (s == top) / (s == top).sum(1, keepdims=True)
            np.testing.assert_allclose(got["o_" + x][rows, h], w @ v, rtol=1e-6, atol=1e-6)
            np.testing.assert_allclose(got["lse_" + x][rows, h], top[:, 0] / 8, rtol=3e-7)
