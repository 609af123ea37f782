"""fp32 storage at the edges of its tiles: 16-row wave blocks, 32-row LDS
tiles and key blocks, 64-row workgroups, both head dims, no prefix, one row.

Tolerance: an output is a sum of at most `terms` fp32 products whose factors
were themselves summed over d, so its error stays below 2 (d + terms) 2^-24
of the largest value, with `terms` the most rows (times the q heads of a kv
head) or keys any output sums over.  The value is taken as at least 1: dS is
P (dP - D), a difference of two sums of d products of N(0, 1) values, scaled
by 1/sqrt(d) into dQ, so that is the size its rounding is relative to where
the difference itself vanishes (a lone prefix row's dQ is exactly zero).
"""
import sys

import pytest

from oracle import max_abs_rel, three_phase_reference
from synthetic import GroupShape, make_group

pytestmark = pytest.mark.gpu

KEYS = ["o_p", "lse_p", "o_s", "lse_s", "dq_p", "dk_p", "dv_p", "dq_s", "dk_s", "dv_s", "g_k", "g_v"]
SHAPES = [
    GroupShape(4, 2, 128, 63, (15, 17, 1), "f32"),
    GroupShape(4, 1, 64, 65, (16, 31, 33), "f32"),
    GroupShape(2, 2, 128, 1, (64, 2), "f32"),
    GroupShape(6, 3, 64, 32, (65, 49), "f32"),
    GroupShape(4, 4, 128, 0, (48, 97), "f32"),
    GroupShape(8, 1, 128, 300, (130,), "f32"),
]


@pytest.mark.parametrize("packed", [False, True], ids=["per_suffix", "packed"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"hq{s.num_q_heads}_hkv{s.num_kv_heads}_d{s.head_dim}"
                                                        f"_p{s.prefix_len}_{'_'.join(map(str, s.suffix_lens))}")
def test_f32_schedule_at_tile_edges(gpu, shape, packed):
    from paper_2606_01143_amd.group import DeviceGroup
    sys.stderr.write(f"\n[gpu-case] f32 tiles {shape} packed={packed}\n")
    sys.stderr.flush()
    inp = make_group(shape, seed=5)
    grp = DeviceGroup(inp)
    grp.run_schedule([(0, shape.n)] if packed else None)
    got, ref = grp.fetch("schedule"), three_phase_reference(inp)
    terms = shape.group * (shape.prefix_len + shape.total_suffix)
    tol = 2 * (shape.head_dim + terms) * 2.0 ** -24
    errs = {k: max_abs_rel(got[k], ref[k].T if k.startswith("lse") else ref[k], floor=1.0)
            for k in KEYS if ref[k].size}
    assert all(v <= tol for v in errs.values()), (tol, errs)
