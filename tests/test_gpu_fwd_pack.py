"""The suffix forward's packed-row form: the 128 rows of a workgroup are
consecutive (token, q head) pairs of one kv head, taken where the one-head
form would need at least 4/3 of the row tiles (short suffixes, or lengths just
past a multiple of 128).  With few tiles and a prefix, key ranges of the prefix
are swept for the rows of all suffixes together, the suffixes' own keys apart.

O and LSE of every suffix row against the oracle, at one row, tiles that end
inside a token's heads, suffixes of one and of several tiles, with and without a prefix, split and unsplit, three and eight q
heads per kv head; the padded call stays bitwise equal.  bf16 rounds P and O
once each: the repository's 2e-2 gate for max-abs-relative error."""
import sys

import numpy as np
import pytest

from oracle import max_abs_rel, three_phase_reference
from synthetic import GroupShape, make_group

CASES = [
    GroupShape(8, 2, 128, 2100, (1, 24, 7, 16), "bf16"),
    GroupShape(6, 2, 64, 700, (33, 5, 1, 40), "bf16"),
    GroupShape(8, 1, 128, 300, (1,), "bf16"),
    GroupShape(4, 1, 128, 0, (17, 90, 3), "bf16"),
    GroupShape(4, 2, 128, 520, (130, 190, 129), "bf16"),
    GroupShape(8, 2, 64, 64, tuple(range(1, 71)), "bf16"),
]


def _packs(hq, hkv, ml):
    g = hq // hkv
    return 4 * -(-(ml * g) // 128) <= 3 * -(-ml // 128) * g


def test_rule_picks_the_packed_form():
    assert all(_packs(s.num_q_heads, s.num_kv_heads, max(s.suffix_lens)) for s in CASES)
    for s in (128, 512, 1024):  # whole row tiles stay in the one-head form
        assert not _packs(32, 8, s)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", CASES, ids=lambda s: f"hq{s.num_q_heads}_hkv{s.num_kv_heads}_d{s.head_dim}"
                                                       f"_p{s.prefix_len}_n{s.n}_max{max(s.suffix_lens)}")
def test_packed_rows_match_oracle(gpu, shape):
    from paper_2606_01143_amd.group import DeviceGroup
    sys.stderr.write(f"\n[gpu-case] packed-row forward {shape}\n")
    sys.stderr.flush()
    inp = make_group(shape, seed=3)
    ref = three_phase_reference(inp)
    outs = {}
    for layout in ("packed", "padded"):
        grp = DeviceGroup(inp, dense=False, layout=layout)
        grp.run_schedule([(0, shape.n)])
        if layout == "padded":
            grp.gather_padded_outputs()
        outs[layout] = {k: grp.out[k].float().cpu().numpy().astype(np.float64) for k in ("o_s", "lse_s")}
    for k in ("o_s", "lse_s"):
        want = ref[k].T if k == "lse_s" else ref[k]
        assert max_abs_rel(outs["packed"][k], want) <= 2e-2, k
        # element by element too: a row of another suffix or head is far off
        assert np.max(np.abs(outs["packed"][k] - want) / (1 + np.abs(want))) <= 2e-2, k
        assert np.array_equal(outs["packed"][k], outs["padded"][k]), k
