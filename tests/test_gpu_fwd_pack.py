"""The suffix forward's packed-row form: the 128 rows of a workgroup are
consecutive (token, q head) pairs of one kv head, taken where the one-head
form would need at least 4/3 of the row tiles (short suffixes, or lengths just
past a multiple of 128) and is not the faster one.  With few tiles and a
prefix, key ranges of the prefix are swept for the rows of all suffixes
together, the suffixes' own keys apart.

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


@pytest.mark.parametrize("hq,hkv,d,P,n,ml,splits", [
    (32, 8, 128, 8191, 4, 24, 17),    # 24 blocks a range: 16 ranges of eight tiles, not 21
    (32, 8, 128, 16000, 4, 24, 22),   # ranges past eight tiles: two workgroups per CU
    (32, 8, 128, 16000, 1, 60, 32),   # 16 blocks: 31 ranges of eight tiles, not 32
    (32, 4, 64, 6000, 3, 24, 20),     # 20 blocks: 19
    (32, 4, 128, 8000, 6, 60, 6),     # 92 blocks: fewer than 16 ranges keep two per CU
    (32, 8, 128, 1024, 2, 4, 5),      # ranges of four tiles at least
])
def test_split_counts(hq, hkv, d, P, n, ml, splits):
    """The reported workspace is the partials of the expected splits (outputs, then LSE,
    each rounded up to 256 bytes)."""
    from paper_2606_01143_amd import binding as B
    up = lambda x: -(-x // 256) * 256
    T = n * ml
    got = B.workspace_size(B.OP_SUFFIX_FWD, B.make_dims(hq, hkv, d, P, "bf16"), n, ml, T)
    assert got == up(splits * T * hq * d * 4) + up(splits * T * hq * 4)



@pytest.mark.parametrize("hq,hkv,d,P,n,ml,splits", [
    (32, 8, 64, 500, 3, 156, 1),      # one range would only add a merge
    (32, 8, 128, 282, 5, 192, 1),
    (32, 8, 128, 908, 6, 262, 1),
    (32, 4, 128, 2136, 4, 267, 3),    # from 1536 keys on there are two
    (32, 4, 128, 2136, 5, 280, 2),    # (three splits would not fit the static scratch)
    (32, 8, 128, 1113, 2, 38, 4),     # the one-head form's splits: as short, a CU each
    (32, 8, 128, 1038, 4, 48, 5),     # two of its workgroups per CU: packed
    (32, 4, 64, 2210, 1, 181, 8),     # as many, its row tiles 70% full
    (16, 8, 128, 2558, 1, 150, 10),   # 59% full: packed
    (32, 8, 64, 1799, 6, 63, 6),
    (32, 8, 64, 1662, 2, 162, 5),     # five ranges and the own keys would need a second round
])
def test_split_counts_of_short_prefixes(hq, hkv, d, P, n, ml, splits):
    from paper_2606_01143_amd import binding as B
    up = lambda x: -(-x // 256) * 256
    T = n * ml
    got = B.workspace_size(B.OP_SUFFIX_FWD, B.make_dims(hq, hkv, d, P, "bf16"), n, ml, T)
    assert got == (up(splits * T * hq * d * 4) + up(splits * T * hq * 4) if splits > 1 else 0)


SHORT_PREFIX = [
    GroupShape(32, 8, 128, 282, (192, 150, 130, 70, 69), "bf16"),  # packed, unsplit
    GroupShape(32, 8, 64, 500, (156, 120, 132), "bf16"),           # one-head
    GroupShape(32, 8, 128, 1113, (38, 2), "bf16"),                 # one-head, split
    GroupShape(32, 8, 64, 1662, (162, 80), "bf16"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", CASES + SHORT_PREFIX, ids=lambda s: f"hq{s.num_q_heads}_hkv{s.num_kv_heads}_d{s.head_dim}"
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


def _one_head_bytes(shape):
    """workspace of the one-head form: its key splits' fp32 partials"""
    n, ml, T = shape.n, max(shape.suffix_lens), shape.total_suffix
    nrb = -(-ml // 128) * shape.num_q_heads * n
    ns = max(1, min(-(-512 // nrb), max(1, shape.prefix_len // 256), 16))
    up = lambda x: -(-x // 256) * 256
    return 0 if ns == 1 else up(ns * T * shape.num_q_heads * shape.head_dim * 4) + up(ns * T * shape.num_q_heads * 4)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [CASES[0], CASES[1], GroupShape(32, 8, 64, 900, (20,) * 16, "bf16")],
                         ids=["split", "split_d64", "none_needed"])
def test_packed_rows_take_a_smaller_workspace(gpu, shape):
    """A workspace of the one-head form's size (sized for other lengths) still
    serves, with fewer key splits; a byte less is refused as it was there."""
    import torch
    from paper_2606_01143_amd import binding as B
    from paper_2606_01143_amd.group import DeviceGroup
    sys.stderr.write(f"\n[gpu-case] packed-row forward, small workspace {shape}\n")
    sys.stderr.flush()
    inp = make_group(shape, seed=4)
    grp = DeviceGroup(inp, dense=False)
    n, ml, T = shape.n, max(shape.suffix_lens), shape.total_suffix
    need = _one_head_bytes(shape)
    assert need < B.workspace_size(B.OP_SUFFIX_FWD, grp.dims, n, ml, T)
    o, lse = torch.full_like(grp.out["o_s"], float("nan")), torch.full_like(grp.out["lse_s"], float("nan"))

    def call(nbytes):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
        B.suffix_attn_fwd(grp.dims, grp.k_p, grp.v_p, grp.q_s, grp.k_s, grp.v_s, grp._mb_cu(0, n), n, ml, T, o, lse, ws)

    if need:
        with pytest.raises(B.SprError, match="SPR_ERR_WORKSPACE"):
            call(need - 1)
    ref = three_phase_reference(inp)
    for nbytes in (need, need + need // 3 + 4096):
        call(nbytes)
        torch.cuda.synchronize()
        assert max_abs_rel(o.float().cpu().numpy().astype(np.float64), ref["o_s"]) <= 2e-2
        assert max_abs_rel(lse.cpu().numpy().astype(np.float64), ref["lse_s"].T) <= 2e-2
