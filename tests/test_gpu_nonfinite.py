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
