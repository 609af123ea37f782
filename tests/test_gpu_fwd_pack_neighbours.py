"""Packed-row suffix forward: a suffix's O and LSE bits do not depend on the
suffixes that share its waves, nor on its place among them.  The neighbours'
scores grow by far more than 2^8 along the prefix, so their softmax references
move in tiles where the suffix's own need not."""
import sys

import numpy as np
import pytest

from synthetic import GroupShape, make_group

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,P", [(8, 2, 128, 2100), (6, 2, 64, 700), (8, 1, 128, 200)],
                         ids=["ranges_g4", "ranges_g3", "one_split_g8"])
def test_bits_do_not_follow_the_neighbours(gpu, hq, hkv, d, P):
    from paper_2606_01143_amd.group import DeviceGroup
    own, others = 7, (24, 9, 13)
    got = []
    for place in (0, 1, 3):
        lens = list(others)
        lens.insert(place, own)
        shape = GroupShape(hq, hkv, d, P, tuple(lens), "bf16")
        sys.stderr.write(f"\n[gpu-case] packed-row neighbours {shape}\n")
        sys.stderr.flush()
        inp = make_group(shape, seed=5)  # the same prefix whatever the suffixes
        rng = np.random.default_rng(8)
        r0 = int(inp["cu_seqlens"][place])
        for k in ("q_s", "k_s", "v_s"):
            inp[k][r0:r0 + own] = rng.integers(-8, 9, (own,) + inp[k].shape[1:]) / 4.0
        inp["k_p"] = (np.random.default_rng(9).integers(-8, 9, inp["k_p"].shape) / 4.0 *
                      2.0 ** np.floor(6 * np.arange(P) / P)[:, None, None]).astype(np.float32)
        inp["v_p"] = (np.random.default_rng(10).integers(-8, 9, inp["v_p"].shape) / 4.0).astype(np.float32)
        out = np.ones(shape.total_suffix, bool)
        out[r0:r0 + own] = False
        inp["q_s"][out] *= 16.0
        inp["q_s"][~out] /= 64.0
        grp = DeviceGroup(inp, dense=False)
        grp._suffix_fwd(0, shape.n, grp.ws, None)
        o, lse = (grp.out[k][r0:r0 + own].float().cpu().numpy() for k in ("o_s", "lse_s"))
        assert np.all(np.isfinite(o))
        got.append((o, lse))
    for o, lse in got[1:]:
        assert np.array_equal(o, got[0][0]) and np.array_equal(lse, got[0][1])
