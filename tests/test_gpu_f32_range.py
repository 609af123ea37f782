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
