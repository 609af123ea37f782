"""MoE accounting on both sides of its launch rule (one launch up to 16384
tokens and 262144 selected ids, block partials and a reduction beyond), at the
edges of its blocks: one token, 512 rows, eight rounds of rows, counting blocks
that end inside a token's ids, expert counts that are no multiple of 32,
per-token multiplicities, ids out of range, a second accumulation on top.

Counts, totals and invalid ids are exact.  The mass is a sum of n products of
an int and an fp32 value in fp64: n 2^-53 of the sum bounds its error."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [(1, 4, 1), (206, 128, 8), (511, 60, 3), (513, 8, 8), (4097, 128, 2), (16384, 64, 4), (16385, 64, 4),
         (700, 1024, 375), (698, 1024, 375)]


@pytest.mark.parametrize("weighted", [False, True], ids=["scalar", "per_token"])
@pytest.mark.parametrize("n,E,k", CASES)
def test_accumulate_forms(gpu, n, E, k, weighted):
    import torch
    from paper_2606_01143_amd import binding as B
    sys.stderr.write(f"\n[gpu-case] moe n={n} E={E} k={k} weighted={weighted}\n")
    sys.stderr.flush()
    rng = np.random.default_rng(n + k)
    p = rng.random((n, E), dtype=np.float32)
    r = rng.integers(0, E, size=(n, k), dtype=np.int32)
    r[n // 2, k // 2], r[0, 0] = -1, E
    mu = rng.integers(0, 9, size=n, dtype=np.int32) if weighted else np.full(n, 5, np.int32)
    dev = lambda x: torch.from_numpy(x).cuda()
    stats = torch.empty(B.moe_stats_bytes(E), dtype=torch.uint8, device="cuda")
    ws = torch.empty(max(16, B.moe_aux_workspace_size(E, n)), dtype=torch.uint8, device="cuda")
    B.moe_stats_zero(E, stats)
    for _ in range(2):
        B.moe_aux_accumulate(E, k, dev(p), dev(r), stats, multiplicity=5,
                             token_multiplicity=dev(mu) if weighted else None, ws=ws)
    torch.cuda.synchronize()
    got = stats.cpu().numpy()
    ok = (r >= 0) & (r < E)
    count = np.zeros(E, np.int64)
    np.add.at(count, r[ok], np.broadcast_to(mu[:, None], r.shape)[ok].astype(np.int64))
    assert np.array_equal(got[:8 * E].view(np.int64), 2 * count)
    assert got[16 * E:].view(np.int64).tolist() == [2 * int(mu.sum()), 2 * int((~ok).sum())]
    mass = 2 * (mu[:, None].astype(np.longdouble) * p).sum(0)
    err = np.abs(got[8 * E:16 * E].view(np.float64) - mass)
    assert bool((err <= 2 * n * 2.0 ** -53 * mass).all())
