"""The suffix forward without a workspace takes the key splits of the call
with the reported workspace, or refuses: packed-row partials always fit the
64 MiB static scratch.  The sizes are checked on the CPU over a range, the
bits on the GPU at sizes where two splits would not fit."""
import sys

import numpy as np
import pytest

SCRATCH = 64 << 20


def _up(x):
    return -(-x // 256) * 256


def _one_head_bytes(hq, d, P, n, ml, T):
    """workspace of the one-head form: its key splits' fp32 partials"""
    nrb = -(-ml // 128) * hq * n
    ns = max(1, min(-(-512 // nrb), max(1, P // 256), 16))
    return 0 if ns == 1 else _up(ns * T * hq * d * 4) + _up(ns * T * hq * 4)


def test_reported_bytes_beyond_the_scratch_are_the_one_head_forms():
    from paper_2606_01143_amd import binding as B
    assert B.STATIC_SCRATCH_BYTES == SCRATCH
    rng = np.random.default_rng(0)
    sizes = [(hkv * g, hkv, 128, 1024, 511 // hkv // (ml * g // 128), ml)  # 509 to 511 full packed tiles
             for hkv in (1, 2) for g in (16, 32) for ml in (8, 24, 56)]
    for _ in range(2000):
        hkv = int(rng.choice([1, 2, 4, 8]))
        sizes.append((hkv * int(rng.choice([2, 3, 4, 8, 16])), hkv, int(rng.choice([64, 128])),
                      *(int(2 ** rng.uniform(a, b)) for a, b in ((6, 14), (0, 9), (0, 8)))))
    for hq, hkv, d, P, n, ml in sizes:
        T = n * ml
        got = B.workspace_size(B.OP_SUFFIX_FWD, B.make_dims(hq, hkv, d, P, "bf16"), n, ml, T)
        one = _one_head_bytes(hq, d, P, n, ml, T)
        assert one <= got <= max(one, SCRATCH), (hq, hkv, d, P, n, ml)


@pytest.mark.gpu
def test_same_bits_where_two_splits_do_not_fit(gpu):
    import torch
    from paper_2606_01143_amd import binding as B
    from paper_2606_01143_amd.group import DeviceGroup
    from synthetic import GroupShape, make_group
    shape = GroupShape(16, 1, 128, 1024, (56,) * 73, "bf16")
    sys.stderr.write(f"\n[gpu-case] no-alloc at the scratch's edge {shape}\n")
    sys.stderr.flush()
    grp = DeviceGroup(make_group(shape, seed=4), dense=False)
    n, ml, T = shape.n, 56, shape.total_suffix
    outs = []
    for noalloc in (False, True):
        o, lse = torch.full_like(grp.out["o_s"], float("nan")), torch.full_like(grp.out["lse_s"], float("nan"))
        args = (grp.dims, grp.k_p, grp.v_p, grp.q_s, grp.k_s, grp.v_s, grp._mb_cu(0, n), n, ml, T, o, lse)
        if noalloc:
            B.suffix_attn_fwd_noalloc(*args)
        else:
            need = B.workspace_size(B.OP_SUFFIX_FWD, grp.dims, n, ml, T)
            B.suffix_attn_fwd(*args, torch.empty(need, dtype=torch.uint8, device="cuda") if need else None)
        outs.append((o, lse))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*outs)) and not torch.isnan(outs[0][0]).any()
