"""The calls whose speed matters in this framework, as measurable cases.

A case is a dict of plain values.  ``listed()`` holds fixed ones, ``draw(rng)``
makes more of the same ranges.  ``prepare`` builds what a program holds before
the call (tensors, group, layer), ``run`` is one pass through the public entry
points, ``work`` the bytes and floating-point operations the pass cannot do
without, ``exact`` the same outputs in 64 bits from plain torch, and
``tolerance`` how far two correct implementations may differ.

Kinds:
  group   one prompt group through the three-phase schedule
          (``DeviceGroup.run_schedule``): Phase A, the suffix microbatches'
          forward and backward, Phase C
  prefix  the prefix calls alone: forward, then the backward's two halves
  suffix  one short suffix microbatch's forward without a workspace
          (``suffix_attn_fwd_noalloc``), as a serving loop calls it
  padded  one batch-plus-padding microbatch's forward and backward
  moe     the router's auxiliary-loss accounting of one prompt group
  tokens  the decoder layer's token-wise operations, forward and backward
  layer   a whole decoder layer through the schedule (``DecoderLayer``)
"""
from __future__ import annotations

from collections import namedtuple
from types import SimpleNamespace

import math

import numpy as np
import torch

from paper_2606_01143_amd import binding as B
from paper_2606_01143_amd.group import DeviceGroup, plan_suffix_waves
from paper_2606_01143_amd.layer import DecoderLayer

DEV = "cuda:0"


class Shape(namedtuple("Shape", "num_q_heads num_kv_heads head_dim prefix_len suffix_lens dtype")):
    """The group shape DeviceGroup reads."""

    n = property(lambda s: len(s.suffix_lens))
    total_suffix = property(lambda s: sum(s.suffix_lens))


class LayerShape(namedtuple("LayerShape", "hidden num_q_heads num_kv_heads head_dim intermediate prefix_len "
                                          "suffix_lens dtype rope_theta norm_eps")):
    """The layer shape DecoderLayer reads."""

    n = property(lambda s: len(s.suffix_lens))


def _lens(case):
    return tuple(int(x) for x in case["lens"].split(","))


def _text(lens):
    return ",".join(str(x) for x in lens)


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest group: two heads in full precision, as a correctness
        # run of a trainer's port uses it; latency and launches count
        dict(name="tiny_fp32_group", kind="group", hq=2, hkv=2, d=64, P=128, lens="32,32,32,32", dtype="f32",
             waves=0),
        # a model-shaped group in full precision with odd lengths (numerics
        # runs beside the bf16 ones)
        dict(name="fp32_group_ragged", kind="group", hq=32, hkv=8, d=128, P=1000, lens="100,257,64,180",
             dtype="f32", waves=0),
        # short prefix, long suffixes: Phase B is nearly everything
        dict(name="qwen3_8b_p2048_n4_s1024", kind="group", hq=32, hkv=8, d=128, P=2048, lens="1024,1024,1024,1024",
             dtype="bf16", waves=0),
        # the Llama3-8B group, one suffix per microbatch
        dict(name="llama3_8b_p4096_n8_s512", kind="group", hq=32, hkv=8, d=128, P=4096,
             lens=_text((512,) * 8), dtype="bf16", waves=0),
        # the ragged mixture-of-experts group, all suffixes as one packed
        # microbatch
        dict(name="qwen3_moe_p8192_n16_ragged", kind="group", hq=32, hkv=4, d=128, P=8192,
             lens="1762,1350,1109,646,719,206,273,160,465,1691,1368,1881,1099,1299,2045,1470", dtype="bf16",
             waves=1 << 20),
        # the long-context group, the largest listed
        dict(name="llama3_8b_p28672_n8_s128", kind="group", hq=32, hkv=8, d=128, P=28672, lens=_text((128,) * 8),
             dtype="bf16", waves=0),
        # prefix calls with 64-wide heads, eight q heads per kv head and a
        # length that fills no tile
        dict(name="prefix_d64_p6001", kind="prefix", hq=32, hkv=4, d=64, P=6001, dtype="bf16"),
        # a serving loop scoring a few short continuations of one prompt
        dict(name="serving_p8191_short", kind="suffix", hq=32, hkv=8, d=128, P=8191, lens="1,24,7,16", dtype="bf16"),
        # a padded suffix batch of unequal lengths
        dict(name="padded_p4096_n6_ragged", kind="padded", hq=32, hkv=8, d=128, P=4096,
             lens="512,131,388,77,256,305", s_max=512, dtype="bf16"),
        # router accounting of the ragged mixture-of-experts group, one
        # suffix per microbatch
        dict(name="moe_router_p8192_n16_ragged", kind="moe", experts=128, top_k=8, P=8192,
             lens="1762,1350,1109,646,719,206,273,160,465,1691,1368,1881,1099,1299,2045,1470"),
        # the token-wise operations of a Llama3-8B layer on one prefix
        dict(name="token_ops_t4096", kind="tokens", hidden=4096, hq=32, hkv=8, d=128, inter=14336, T=4096),
        # a whole Llama3-8B layer over the P = 4096 group's lengths
        dict(name="llama3_8b_layer_p4096_n4_s512", kind="layer", hidden=4096, hq=32, hkv=8, d=128, inter=14336,
             P=4096, lens="512,512,512,512"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("group", "group", "group", "group_fp32", "prefix", "suffix", "padded", "moe", "tokens",
                       "layer"))
    hq, hkv = rng.choice(((32, 8), (32, 8), (32, 4), (16, 8), (8, 8)))
    d = rng.choice((128, 128, 64))
    if kind == "group":
        while True:
            c = dict(kind="group", hq=hq, hkv=hkv, d=d, P=_log(rng, 500, 20000), dtype="bf16",
                     lens=_text([_log(rng, 100, 2048) for _ in range(rng.randint(1, 16))]),
                     waves=rng.choice((0, 0, 4096, 1 << 20)))
            if work(c)["flops"] < 1.5e13:
                return c
    if kind == "group_fp32":
        return dict(kind="group", hq=hq // 2, hkv=hkv // 2, d=d, P=_log(rng, 60, 1200), dtype="f32",
                    lens=_text([_log(rng, 10, 300) for _ in range(rng.randint(1, 5))]), waves=0)
    if kind == "prefix":
        return dict(kind="prefix", hq=hq, hkv=hkv, d=d, P=_log(rng, 300, 16000), dtype="bf16")
    if kind == "suffix":
        return dict(kind="suffix", hq=hq, hkv=hkv, d=d, P=_log(rng, 500, 16000), dtype="bf16",
                    lens=_text([_log(rng, 1, 64) for _ in range(rng.randint(1, 6))]))
    if kind == "padded":
        lens = [_log(rng, 30, 900) for _ in range(rng.randint(1, 8))]
        return dict(kind="padded", hq=hq, hkv=hkv, d=d, P=_log(rng, 500, 9000), dtype="bf16", lens=_text(lens),
                    s_max=max(lens))
    if kind == "moe":
        return dict(kind="moe", experts=rng.choice((8, 60, 64, 128, 256)), top_k=rng.choice((1, 2, 4, 8)),
                    P=_log(rng, 300, 16000), lens=_text([_log(rng, 100, 2048) for _ in range(rng.randint(1, 16))]))
    if kind == "tokens":
        return dict(kind="tokens", hidden=128 * rng.randint(8, 40), hq=hq, hkv=hkv, d=d,
                    inter=128 * rng.randint(16, 112), T=_log(rng, 100, 16000))
    return dict(kind="layer", hidden=4096, hq=32, hkv=8, d=128, inter=14336, P=_log(rng, 300, 4000),
                lens=_text([_log(rng, 60, 512) for _ in range(rng.randint(1, 4))]))


# ------------------------------------------------------------------ inputs
class _Draw:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed))
        self.dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]

    def __call__(self, *shape, scale=1.0):
        return (torch.randn(*shape, generator=self.g, device=DEV) * scale).to(self.dt)


def _group_inputs(case, seed):
    """Q, K, V and the upstream adjoints, all N(0, 1), on the GPU."""
    dr = _Draw(seed, case["dtype"])
    hq, hkv, d, P, T = case["hq"], case["hkv"], case["d"], case["P"], sum(_lens(case))
    return dict(q_p=dr(P, hq, d), k_p=dr(P, hkv, d), v_p=dr(P, hkv, d), q_s=dr(T, hq, d), k_s=dr(T, hkv, d),
                v_s=dr(T, hkv, d), do_s=dr(T, hq, d), g_y=dr(P, hq, d))


def _prefix_inputs(case, seed):
    dr = _Draw(seed, case["dtype"])
    hq, hkv, d, P = case["hq"], case["hkv"], case["d"], case["P"]
    f = torch.float32
    return dict(q_p=dr(P, hq, d), k_p=dr(P, hkv, d), v_p=dr(P, hkv, d), g_y=dr(P, hq, d),
                gk=dr(P, hkv, d).to(f), gv=dr(P, hkv, d).to(f))


def _moe_inputs(case, seed):
    """Router probabilities (softmax of N(0, 1) logits) and the top-k ids."""
    dr = _Draw(seed, "f32")
    E, k, P, T = case["experts"], min(case["top_k"], case["experts"]), case["P"], sum(_lens(case))
    out = {}
    for name, n in (("p", P), ("s", T)):
        logits = dr(n, E)
        out["p_" + name] = logits.double().softmax(1).float()
        out["r_" + name] = logits.topk(k, dim=1).indices.to(torch.int32)
    return out


def _token_inputs(case, seed):
    dr = _Draw(seed, "bf16")
    T, h, I, d = case["T"], case["hidden"], case["inter"], case["d"]
    return dict(x=dr(T, h), dy=dr(T, h), add=dr(T, h), q=dr(T, case["hq"], d), k=dr(T, case["hkv"], d),
                g=dr(T, I), u=dr(T, I), dm=dr(T, I))


def _layer_inputs(case, seed):
    """Weights N(0, 0.02), layer inputs and upstream adjoints N(0, 1)."""
    dr = _Draw(seed, "bf16")
    h, I, hd, kd = case["hidden"], case["inter"], case["hq"] * case["d"], case["hkv"] * case["d"]
    w = {k: dr(*s, scale=0.02) for k, s in dict(wq=(h, hd), wk=(h, kd), wv=(h, kd), wo=(hd, h), wg=(h, I),
                                                wu=(h, I), wd=(I, h)).items()}
    return dict(w=w, x_p=dr(case["P"], h), x_s=[dr(s, h) for s in _lens(case)],
                dy_s=[dr(s, h) for s in _lens(case)], g_y=dr(case["P"], h))


def _host(x):
    return x.float().cpu().numpy()


def _empty(*shape, dt=torch.bfloat16):
    return torch.empty(*shape, dtype=dt, device=DEV)


_F32 = torch.float32
_THETA = 500000.0


def prepare(case, seed):
    kind = case["kind"]
    s = SimpleNamespace(case=case, kind=kind)
    if kind == "group":
        lens = _lens(case)
        shape = Shape(case["hq"], case["hkv"], case["d"], case["P"], lens, case["dtype"])
        inp = {k: _host(v) for k, v in _group_inputs(case, seed).items()}
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        s.waves = plan_suffix_waves(lens, case["waves"]) if case["waves"] else [(i, i + 1) for i in range(len(lens))]
        s.group = DeviceGroup(dict(inp, shape=shape, suffix_lens=np.asarray(lens, np.int32), cu_seqlens=cu),
                              device=DEV, dense=False, microbatch_splits=[s.waves])
        s.group.prepare(s.waves)
        return s
    if kind == "layer":
        inp = _layer_inputs(case, seed)
        shape = LayerShape(case["hidden"], case["hq"], case["hkv"], case["d"], case["inter"], case["P"],
                           _lens(case), "bf16", _THETA, 1e-5)
        # one layer of a model: its weights on the GPU, the group's inputs
        s.layer = DecoderLayer.of_weights(shape, inp["w"], DEV)
        s.layer.x_p, s.layer.x_s, s.layer.dy_s = inp["x_p"], inp["x_s"], inp["dy_s"]
        s.layer.g_y = inp["g_y"]
        return s
    if kind == "prefix":
        s.__dict__.update(_prefix_inputs(case, seed))
        hq, hkv, d, P = case["hq"], case["hkv"], case["d"], case["P"]
        s.dims = B.make_dims(hq, hkv, d, P, "bf16")
        s.o, s.lse, s.dq = _empty(P, hq, d), _empty(P, hq, dt=_F32), _empty(P, hq, d)
        s.dk, s.dv = _empty(P, hkv, d), _empty(P, hkv, d)
        s.ws = _empty(max(256, B.workspace_size(B.OP_PREFIX_BWD, s.dims)), dt=torch.uint8)
        return s
    if kind in ("suffix", "padded"):
        lens, hq, hkv, d, P = _lens(case), case["hq"], case["hkv"], case["d"], case["P"]
        inp = _group_inputs(case, seed)
        s.k_p, s.v_p = inp["k_p"], inp["v_p"]
        s.dims = B.make_dims(hq, hkv, d, P, "bf16")
        s.n, s.mx, s.T = len(lens), max(lens), sum(lens)
        if kind == "suffix":
            s.q, s.k, s.v = inp["q_s"], inp["k_s"], inp["v_s"]
            s.cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)
            s.o, s.lse = _empty(s.T, hq, d), _empty(s.T, hq, dt=_F32)
            return s
        s.mx = case["s_max"]
        for name in ("q", "k", "v", "do"):
            setattr(s, name, _pad(inp[name + "_s"], lens, s.mx))
        s.lens = torch.tensor(lens, dtype=torch.int32, device=DEV)
        s.o, s.lse = _empty(s.n, s.mx, hq, d), _empty(s.n, s.mx, hq, dt=_F32)
        s.dq, s.dk, s.dv = _empty(s.n, s.mx, hq, d), _empty(s.n, s.mx, hkv, d), _empty(s.n, s.mx, hkv, d)
        s.gk, s.gv = _empty(P, hkv, d, dt=_F32), _empty(P, hkv, d, dt=_F32)
        s.ws = _empty(max(B.workspace_size(B.OP_SUFFIX_FWD_PADDED, s.dims, s.n, s.mx),
                          B.workspace_size(B.OP_SUFFIX_BWD_PADDED, s.dims, s.n, s.mx)), dt=torch.uint8)
        return s
    if kind == "moe":
        inp = _moe_inputs(case, seed)
        E, lens = case["experts"], _lens(case)
        s.E, s.k, s.n = E, min(case["top_k"], E), len(lens)
        cu = np.concatenate([[0], np.cumsum(lens)])
        s.sets = [(inp["p_p"], inp["r_p"], s.n)] + [(inp["p_s"][a:b], inp["r_s"][a:b], 1)
                                                    for a, b in zip(cu[:-1], cu[1:])]
        s.dp_p, s.dp_s = torch.empty_like(inp["p_p"]), torch.empty_like(inp["p_s"])
        s.dps = [s.dp_p] + [s.dp_s[a:b] for a, b in zip(cu[:-1], cu[1:])]
        s.stats = _empty(B.moe_stats_bytes(E), dt=torch.uint8)
        s.ws = _empty(max(B.moe_aux_workspace_size(E, p.shape[0]) for p, _, _ in s.sets), dt=torch.uint8)
        s.f, s.pe, s.loss = (_empty(n, dt=torch.float64) for n in (E, E, 1))
        return s
    # tokens
    s.__dict__.update(_token_inputs(case, seed))
    s.out = {n: torch.empty_like(getattr(s, src)) for n, src in dict(
        y="x", dx="x", qr="q", kr="k", dq="q", dk="k", m="g", dg="g", du="u").items()}
    s.rstd = _empty(case["T"], dt=_F32)
    return s


def _pad(x, lens, mx):
    y = torch.zeros(len(lens), mx, *x.shape[1:], dtype=x.dtype, device=x.device)
    r = 0
    for i, n in enumerate(lens):
        y[i, :n] = x[r:r + n]
        r += n
    return y


# --------------------------------------------------------------------- run
def run(s):
    kind = s.kind
    if kind == "group":
        g = s.group
        g.run_schedule(s.waves)
        return dict(g.out, gk=g.gk, gv=g.gv)
    if kind == "layer":
        return s.layer.run_schedule()
    if kind == "prefix":
        B.prefix_fwd(s.dims, s.q_p, s.k_p, s.v_p, s.o, s.lse)
        B.prefix_bwd_dq(s.dims, s.q_p, s.k_p, s.v_p, s.o, s.lse, s.g_y, s.dq, s.ws)
        B.prefix_bwd_dkv(s.dims, s.q_p, s.k_p, s.v_p, s.o, s.lse, s.g_y, s.gk, s.gv, s.dk, s.dv, s.ws)
        return dict(o=s.o, lse=s.lse, dq=s.dq, dk=s.dk, dv=s.dv)
    if kind == "suffix":
        B.suffix_attn_fwd_noalloc(s.dims, s.k_p, s.v_p, s.q, s.k, s.v, s.cu, s.n, s.mx, s.T, s.o, s.lse)
        return dict(o=s.o, lse=s.lse)
    if kind == "padded":
        B.gkv_cache_zero(s.dims, s.gk, s.gv)
        B.suffix_attn_fwd_padded(s.dims, s.k_p, s.v_p, s.q, s.k, s.v, s.lens, s.n, s.mx, s.o, s.lse, s.ws)
        B.suffix_attn_bwd_accum_padded(s.dims, s.k_p, s.v_p, s.q, s.k, s.v, s.o, s.lse, s.do, s.lens, s.n, s.mx,
                                       s.dq, s.dk, s.dv, s.gk, s.gv, s.ws)
        return dict(o=s.o, lse=s.lse, dq=s.dq, dk=s.dk, dv=s.dv, gk=s.gk, gv=s.gv)
    if kind == "moe":
        B.moe_stats_zero(s.E, s.stats)
        for p, r, m in s.sets:
            B.moe_aux_accumulate(s.E, s.k, p, r, s.stats, multiplicity=m, ws=s.ws)
        B.moe_aux_loss(s.E, s.k, 0.01, s.stats, s.f, s.pe, s.loss)
        for (_, _, m), dp in zip(s.sets, s.dps):
            B.moe_aux_grad(s.E, s.k, 0.01, 1.0, s.stats, dp, multiplicity=m)
        E = s.E
        return dict(count=s.stats[:8 * E].view(torch.int64), mass=s.stats[8 * E:16 * E].view(torch.float64),
                    total=s.stats[16 * E:].view(torch.int64), f=s.f, p=s.pe, loss=s.loss, dp_p=s.dp_p, dp_s=s.dp_s)
    o = s.out
    B.rmsnorm_fwd(s.x, o["y"], s.rstd)
    B.rope_fwd(s.q, o["qr"], 0, _THETA)
    B.rope_fwd(s.k, o["kr"], 0, _THETA)
    B.swiglu_fwd(s.g, s.u, o["m"])
    B.swiglu_bwd(s.g, s.u, s.dm, o["dg"], o["du"])
    B.rope_bwd(s.q, o["dq"], 0, _THETA)
    B.rope_bwd(s.k, o["dk"], 0, _THETA)
    B.rmsnorm_bwd(s.x, s.rstd, s.dy, o["dx"], add=s.add)
    return dict(o, rstd=s.rstd)


# -------------------------------------------------------------------- work
def _pairs(P, lens, prefix=True):
    """Visible (row, key) pairs of one head: prefix causal, suffixes."""
    return (P * (P + 1) // 2 if prefix else 0) + sum(n * P + n * (n + 1) // 2 for n in lens)


def work(case):
    kind = case["kind"]
    if kind == "tokens":
        T, h, I, qk = case["T"], case["hidden"], case["inter"], (case["hq"] + case["hkv"]) * case["d"]
        # x, y and the backward's x, dy, add, dx; rope both ways; swiglu 3 + 5 tensors
        return {"bytes": 2 * T * (6 * h + 4 * qk + 8 * I) + 8 * T, "flops": T * (12 * h + 6 * qk + 40 * I)}
    if kind == "moe":
        E, n = case["experts"], case["P"] + sum(_lens(case))
        return {"bytes": n * (8 * E + 4 * min(case["top_k"], E)), "flops": 3 * n * E}
    hq, hkv, d, P = case["hq"], case["hkv"], case["d"], case["P"]
    e = 4 if case.get("dtype") == "f32" else 2
    if kind == "prefix":
        # the backward's halves each need the scores: 4d + 6d + 8d per pair
        return {"bytes": P * (hq * d * e * 4 + hkv * d * (e * 4 + 8) + hq * 4),
                "flops": 18 * d * hq * _pairs(P, ())}
    lens = _lens(case)
    T = sum(lens)
    if kind == "suffix":
        return {"bytes": (P + T) * 2 * hkv * d * e + T * (2 * hq * d * e + 4 * hq),
                "flops": 4 * d * hq * _pairs(P, lens, False)}
    if kind == "padded":
        return {"bytes": (P + 2 * T) * 2 * hkv * d * e + P * 2 * hkv * d * 4 + T * (4 * hq * d * e + 4 * hq),
                "flops": 14 * d * hq * _pairs(P, lens, False)}
    attn = 14 * d * hq * _pairs(P, lens)
    rows = P + T
    if kind == "layer":
        h, I = case["hidden"], case["inter"]
        w = 2 * h * (hq + hkv) * d + 3 * h * I
        return {"bytes": w * (2 + 4) + rows * h * 2 * 4, "flops": 6 * rows * w + attn}
    return {"bytes": rows * (4 * hq * d * e + 4 * hkv * d * e + 4 * hq) + P * 2 * hkv * d * 4, "flops": attn}


def tolerance(case):
    """About four times the largest error against 64 bits measured over the
    listed and some drawn cases (per output: norm of the difference over the
    norm; largest difference over the value or the root mean square)."""
    if case["kind"] == "moe":     # fp64 statistics, fp32 gradient: 3e-8, 5e-8
        return {"rel": 1.2e-7, "max": 2.5e-7}
    if case["kind"] == "tokens":  # one bf16 rounding: 1.7e-3, 3.9e-3
        return {"rel": 7e-3, "max": 1.6e-2}
    if case["kind"] == "layer":   # bf16 through a whole layer: 1.1e-2, 8e-2
        return {"rel": 3e-2, "max": 0.33}
    if case["dtype"] == "f32":    # 1.2e-6, 2.7e-5
        return {"rel": 5e-6, "max": 1.1e-4}
    # bf16 P, dS and outputs: 3e-3; 3e-2 on suffix rows, 0.3 on the first
    # prefix rows, whose dQ nearly cancels (one or two visible keys)
    return {"rel": 1.2e-2, "max": 0.13 if case["kind"] in ("suffix", "padded") else 0.95}


# ------------------------------------------------------------------- exact
def _causal_rows(q, k, v, do, n_free, scale, chunk):
    """Attention of rows q [G, R, d] over keys k/v [N, d]: row t sees the
    first n_free + t + 1 keys.  Returns o, lse, and with do also dq, dk, dv
    (dk, dv summed over the G heads)."""
    G, R, d = q.shape
    o, lse = torch.zeros_like(q), q.new_zeros(G, R)
    dq = torch.zeros_like(q) if do is not None else None
    dk, dv = (torch.zeros_like(k), torch.zeros_like(v)) if do is not None else (None, None)
    for a in range(0, R, chunk):
        b = min(R, a + chunk)
        n = n_free + b
        kk, vv = k[:n], v[:n]
        z = torch.matmul(q[:, a:b], kk.t()) * scale
        hide = torch.arange(n, device=q.device)[None, :] > n_free + torch.arange(a, b, device=q.device)[:, None]
        z.masked_fill_(hide, -math.inf)
        L = torch.logsumexp(z, -1)
        p = torch.exp(z - L[..., None])
        del z
        ob = torch.matmul(p, vv)
        o[:, a:b], lse[:, a:b] = ob, L
        if do is None:
            continue
        g = do[:, a:b]
        dv[:n] += torch.matmul(p.reshape(-1, n).t(), g.reshape(-1, d))
        ds = torch.matmul(g, vv.t())
        ds -= (g * ob).sum(-1, keepdim=True)
        ds *= p
        del p
        dq[:, a:b] = torch.matmul(ds, kk) * scale
        dk[:n] += torch.matmul(ds.reshape(-1, n).t(), q[:, a:b].reshape(-1, d)) * scale
        del ds
    return o, lse, dq, dk, dv


def _group_exact(inp, lens, hq, hkv, d, prefix=True, backward=True):
    """Outputs of a group in float64, one kv head at a time."""
    G, scale = hq // hkv, 1.0 / math.sqrt(d)
    names_q = ("o_s", "lse_s") + (("dq_s",) if backward else ())
    P, T = inp["k_p"].shape[0], sum(lens)
    z = lambda *s: torch.zeros(*s, dtype=torch.float64, device=DEV)
    out = {"o_s": z(T, hq, d), "lse_s": z(T, hq)}
    if backward:
        out.update(dq_s=z(T, hq, d), dk_s=z(T, hkv, d), dv_s=z(T, hkv, d), gk=z(P, hkv, d), gv=z(P, hkv, d))
    if prefix:
        out.update(o_p=z(P, hq, d), lse_p=z(P, hq), dq_p=z(P, hq, d), dk_p=z(P, hkv, d), dv_p=z(P, hkv, d))
    chunk = max(64, int(1.5e8 // (G * (P + max(lens)))))
    for hk in range(hkv):
        hs = slice(hk * G, hk * G + G)
        rows = lambda x, a, b: x[a:b, hs].double().transpose(0, 1).contiguous()
        kp, vp = inp["k_p"][:, hk].double(), inp["v_p"][:, hk].double()
        r = 0
        for n in lens:
            k = torch.cat([kp, inp["k_s"][r:r + n, hk].double()])
            v = torch.cat([vp, inp["v_s"][r:r + n, hk].double()])
            do = rows(inp["do_s"], r, r + n) if backward else None
            got = _causal_rows(rows(inp["q_s"], r, r + n), k, v, do, P, scale, chunk)
            for name, x in zip(names_q, got):
                out[name][r:r + n, hs] = x.transpose(0, 1)
            if backward:
                out["dk_s"][r:r + n, hk], out["dv_s"][r:r + n, hk] = got[3][P:], got[4][P:]
                out["gk"][:, hk] += got[3][:P]
                out["gv"][:, hk] += got[4][:P]
            r += n
        if prefix:
            o, lse, dq, dk, dv = _causal_rows(rows(inp["q_p"], 0, P), kp, vp, rows(inp["g_y"], 0, P), 0, scale, chunk)
            for name, x in (("o_p", o), ("lse_p", lse), ("dq_p", dq)):
                out[name][:, hs] = x.transpose(0, 1)
            out["dk_p"][:, hk], out["dv_p"][:, hk] = dk + out["gk"][:, hk], dv + out["gv"][:, hk]
    return out


def _rope(x, pos0, sign=1.0):
    T, d = x.shape[0], x.shape[-1]
    pos = torch.arange(pos0, pos0 + T, dtype=torch.float64, device=x.device)
    ang = pos[:, None] * _THETA ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    c, s = torch.cos(ang)[:, None], sign * torch.sin(ang)[:, None]
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _rms(x):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5)


def _layer_attention(q, k, v, n_free, scale):
    """q [R, Hq, d] over k/v [N, Hkv, d], row t seeing n_free + t + 1 keys."""
    R, hq, d = q.shape
    hkv = k.shape[1]
    hide = torch.arange(k.shape[0], device=q.device)[None, :] > n_free + torch.arange(R, device=q.device)[:, None]
    o = []
    for hk in range(hkv):
        qq = q[:, hk * (hq // hkv):(hk + 1) * (hq // hkv)].transpose(0, 1)
        z = (torch.matmul(qq, k[:, hk].t()) * scale).masked_fill(hide, -math.inf)
        o.append(torch.matmul(z.softmax(-1), v[:, hk]).transpose(0, 1))
    return torch.cat(o, 1)


def _layer_exact(case, inp):
    hq, hkv, d, P = case["hq"], case["hkv"], case["d"], case["P"]
    leaf = lambda x: x.double().requires_grad_()
    w = {k: leaf(v) for k, v in inp["w"].items()}
    x_p, x_s = leaf(inp["x_p"]), [leaf(x) for x in inp["x_s"]]
    scale = 1.0 / math.sqrt(d)

    def layer(x, pos0, past):
        n1 = _rms(x)
        q = _rope((n1 @ w["wq"]).view(-1, hq, d), pos0)
        k = _rope((n1 @ w["wk"]).view(-1, hkv, d), pos0)
        v = (n1 @ w["wv"]).view(-1, hkv, d)
        kk, vv = (k, v) if past is None else (torch.cat([past[0], k]), torch.cat([past[1], v]))
        o = _layer_attention(q, kk, vv, 0 if past is None else P, scale)
        h = x + o.reshape(x.shape[0], -1) @ w["wo"]
        n2 = _rms(h)
        return h + (torch.nn.functional.silu(n2 @ w["wg"]) * (n2 @ w["wu"])) @ w["wd"], (k, v)

    y_p, past = layer(x_p, 0, None)
    y_s = [layer(x, P, past)[0] for x in x_s]
    loss = (y_p * inp["g_y"].double()).sum() + sum((y * g.double()).sum() for y, g in zip(y_s, inp["dy_s"]))
    loss.backward()
    return {"y_p": y_p.detach(), "y_s": [y.detach() for y in y_s], "dx_p": x_p.grad, "dx_s": [x.grad for x in x_s],
            "dw": {k: v.grad for k, v in w.items()}}


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        return _layer_exact(case, _layer_inputs(case, seed))
    if kind == "moe":
        inp = _moe_inputs(case, seed)
        E, n = case["experts"], len(_lens(case))
        k = inp["r_p"].shape[1]
        hist = lambda r: torch.bincount(r.reshape(-1).long(), minlength=E)
        count = n * hist(inp["r_p"]) + hist(inp["r_s"])
        mass = n * inp["p_p"].double().sum(0) + inp["p_s"].double().sum(0)
        total = n * case["P"] + inp["p_s"].shape[0]
        f, p = count.double() / (k * total), mass / total
        g = 0.01 * E * f / total
        return dict(count=count, mass=mass, total=torch.tensor([total, 0], device=DEV), f=f, p=p,
                    loss=(0.01 * E * (f * p).sum()).reshape(1), dp_p=(n * g).expand(case["P"], E),
                    dp_s=g.expand(inp["p_s"].shape[0], E))
    if kind == "tokens":
        i = {k: v.double() for k, v in _token_inputs(case, seed).items()}
        r = torch.rsqrt(i["x"].square().mean(-1, keepdim=True) + 1e-5)
        sg = torch.sigmoid(i["g"])
        silu = i["g"] * sg
        return dict(y=i["x"] * r, rstd=r[:, 0], qr=_rope(i["q"], 0), kr=_rope(i["k"], 0),
                    dq=_rope(i["q"], 0, -1.0), dk=_rope(i["k"], 0, -1.0), m=silu * i["u"],
                    dg=i["dm"] * i["u"] * sg * (1 + i["g"] * (1 - sg)), du=i["dm"] * silu,
                    dx=r * i["dy"] - r ** 3 * i["x"] * (i["dy"] * i["x"]).mean(-1, keepdim=True) + i["add"])
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    if kind == "prefix":
        i = _prefix_inputs(case, seed)
        none = i["q_p"][:0]
        e = _group_exact(dict(i, q_s=none, do_s=none, k_s=i["k_p"][:0], v_s=i["v_p"][:0]), (0,), hq, hkv, d)
        return dict(o=e["o_p"], lse=e["lse_p"], dq=e["dq_p"], dk=e["dk_p"] + i["gk"].double(),
                    dv=e["dv_p"] + i["gv"].double())
    lens = _lens(case)
    inp = _group_inputs(case, seed)
    if kind == "suffix":
        e = _group_exact(inp, lens, hq, hkv, d, prefix=False, backward=False)
        return dict(o=e["o_s"], lse=e["lse_s"])
    if kind == "padded":
        e = _group_exact(inp, lens, hq, hkv, d, prefix=False)
        out = {n: _pad(e[n + "_s"], lens, case["s_max"]) for n in ("o", "lse", "dq", "dk", "dv")}
        return dict(out, gk=e["gk"], gv=e["gv"])
    return _group_exact(inp, lens, hq, hkv, d)
