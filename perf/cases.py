"""Measured cases: what a serving program has this library do, through its public entry points.

One layer of a prefix-reuse prefill step (append the new tokens' K/V, causal attention
over cached prefix and new tokens), decode steps, prefill and decode rows in one launch,
reading tokens back out of the pool, and the layer pipeline with loads from and offloads
to pinned host memory. `listed()` names the fixed cases and `draw()` makes more of the
same ranges. Every value is made from the seed alone: bf16 standard normals for Q, K and
V, distinct random pool blocks for the block tables.

A case is a dict of plain values; ragged lengths follow from its numbers (`_lens`).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_23049_amd import pcr

BS = 16   # tokens per pool block


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # The smallest step: one sequence of 256 cached and 64 new tokens, 8 heads of 64 dims
        # (a small model, or one GPU's heads of a larger one), append and attention.
        # Launches and latency are all there is.
        dict(name="step_tiny", kind="step", B=1, Hq=8, Hkv=8, D=64, p=256, p_min=256, s=64, s_min=64, lens=0),
        # One chat turn on a long cached conversation: an odd-sized short message (43 new
        # tokens) after 7985 cached ones, the 8B model's heads. The prefix hit is nearly all
        # of the context, which is what prefix reuse is for.
        dict(name="turn_8b", kind="step", B=1, Hq=32, Hkv=8, D=128, p=7985, p_min=7985, s=43, s_min=43, lens=0),
        # The 8B model's layer: 4 sequences, 4096 cached and 256 new tokens each.
        dict(name="layer_8b", kind="attn", B=4, Hq=32, Hkv=8, D=128, p=4096, p_min=4096, s=256, s_min=256, lens=0),
        # A retrieval batch: 16 ragged requests of 1.5-5k tokens, about a fifth of them cached.
        dict(name="rag_mix", kind="attn", B=16, Hq=32, Hkv=8, D=128, p=1280, p_min=16, s=4096, s_min=1056, lens=4),
        # The 70B model's layer at a 16k context, 1024 new tokens of each of two sequences.
        dict(name="layer_70b", kind="attn", B=2, Hq=64, Hkv=8, D=128, p=15360, p_min=15360, s=1024, s_min=1024,
             lens=0),
        # One GPU's share of that layer under 8-way tensor parallelism: 8 query heads, 1 kv head.
        dict(name="tp8_70b", kind="attn", B=2, Hq=8, Hkv=1, D=128, p=15360, p_min=15360, s=1024, s_min=1024, lens=0),
        # Continuous batching: two prefill chunks beside 48 sequences that decode one token
        # each, in one launch of the prefill entry point.
        dict(name="mixed", kind="mixed", B=2, Hq=32, Hkv=8, D=128, p=4096, p_min=1000, s=2048, s_min=1500, lens=7,
             rows=48, ctx=6000, ctx_min=700),
        # A full decode batch: 64 sequences of 4352 tokens, the 8B model's heads.
        dict(name="decode_64", kind="decode", B=64, Hq=32, Hkv=8, D=128, ctx=4352, ctx_min=4352, lens=0),
        # A small decode step: 12 sequences of 1k-8k tokens, append of the new token and attention.
        dict(name="decode_12_ragged", kind="decode_step", B=12, Hq=32, Hkv=8, D=128, ctx=8000, ctx_min=1000, lens=9),
        # The K/V of a batch's new tokens written into the pool: 60 ragged sequences.
        dict(name="append_ragged", kind="append", B=60, Hq=32, Hkv=8, D=128, p=700, p_min=3, s=600, s_min=70, lens=11),
        # Tokens read back out of the pool in logical order (staging for an offload).
        dict(name="gather_ragged", kind="gather", B=24, Hq=32, Hkv=8, D=128, p=300, p_min=1, s=1400, s_min=100,
             lens=12),
        # The layer pipeline: every layer's prefix blocks loaded from pinned host memory,
        # append and attention behind the loads, the computed chunks offloaded back.
        dict(name="pipeline_8b", kind="pipeline", B=2, Hq=32, Hkv=8, D=128, p=1024, p_min=1024, s=512, s_min=512,
             lens=0, layers=4),
    ]


HEADS = [(8, 8, 64), (32, 8, 128), (32, 8, 128), (64, 8, 128), (8, 1, 128), (16, 2, 128), (16, 4, 64), (28, 4, 128)]
MAX_FLOPS = 1.0e12     # a drawn case costs no more than the 70B layer


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "attn", "attn", "attn", "mixed", "decode", "decode", "decode_step", "append",
                       "gather", "pipeline"])
    Hq, Hkv, D = rng.choice(HEADS)
    c = dict(kind=kind, Hq=Hq, Hkv=Hkv, D=D, lens=rng.randrange(1, 1 << 30))
    if kind in ("step", "attn"):
        # chat turns (few new tokens on a long prefix) to whole prompts, one sequence to a batch
        c["B"] = _log(rng, 1, 16)
        c["s"] = _log(rng, 2, 4096)
        c["p"] = _log(rng, 16, 16384) if rng.random() < 0.85 else 0     # 0: nothing cached
    elif kind == "mixed":
        c["B"] = _log(rng, 1, 6)
        c["s"] = _log(rng, 64, 3000)
        c["p"] = _log(rng, 16, 8192)
        c["rows"] = _log(rng, 1, 64)
        c["ctx"] = _log(rng, 64, 8192)
        c["ctx_min"] = max(1, int(c["ctx"] * rng.choice([1.0, 0.5, 0.1])))
    elif kind in ("decode", "decode_step"):
        c["B"] = _log(rng, 1, 64)
        c["ctx"] = _log(rng, 100, min(32768, 400000 // c["B"]))
        c["ctx_min"] = max(1, int(c["ctx"] * rng.choice([1.0, 0.5, 0.1])))
        return c
    elif kind in ("append", "gather"):
        c["B"] = _log(rng, 1, 64)
        c["s"] = _log(rng, 1, 32768 // c["B"])
        c["p"] = _log(rng, 1, 1024)
    else:
        c["B"] = _log(rng, 1, 4)
        c["s"] = _log(rng, 16, 600)
        c["p"] = _log(rng, 64, 3000)
        c["layers"] = rng.randrange(2, 5)
    c["p_min"] = max(min(1, c["p"]), int(c["p"] * rng.choice([1.0, 0.5, 0.1])))
    c["s_min"] = max(1, int(c["s"] * rng.choice([1.0, 0.5, 0.1])))
    while work(c)["flops"] > MAX_FLOPS and c["B"] > 1:
        c["B"] = max(1, c["B"] // 2)
    while work(c)["flops"] > MAX_FLOPS:
        c["s"] = max(1, c["s"] // 2)
        c["s_min"] = min(c["s"], c["s_min"])
    return c


def _spread(rng, lo, hi, n):
    return [hi] * n if lo >= hi else [int(x) for x in rng.integers(lo, hi + 1, size=n)]


def _lens(c):
    """(prefix lengths, suffix lengths): a decode row is a suffix of one token."""
    rng = np.random.Generator(np.random.PCG64(c["lens"]))
    if c["kind"] in ("decode", "decode_step"):
        ctx = _spread(rng, c["ctx_min"], c["ctx"], c["B"])
        return [n - 1 for n in ctx], [1] * c["B"]
    p = _spread(rng, c["p_min"], c["p"], c["B"])
    s = _spread(rng, c["s_min"], c["s"], c["B"])
    if c["kind"] == "mixed":
        ctx = _spread(rng, c["ctx_min"], c["ctx"], c["rows"])
        p, s = p + [n - 1 for n in ctx], s + [1] * c["rows"]
    return p, s


def work(c):
    p, s = _lens(c)
    T, D, Hq, Hkv, kind = sum(s), c["D"], c["Hq"], c["Hkv"], c["kind"]
    row = Hkv * D * 2 * 2                                   # K and V of one token
    keys = sum(p) + T
    flops = sum(4 * D * Hq * (si * pi + si * (si + 1) // 2) for pi, si in zip(p, s))
    attn = keys * row + 2 * T * Hq * D * 2                  # K/V once, Q once, out once
    if kind in ("append", "gather"):
        return {"bytes": 2 * T * row, "flops": 0}
    if kind in ("step", "decode_step"):
        return {"bytes": attn + 2 * T * row, "flops": flops}
    if kind == "pipeline":
        n_off = _chunks(p, s) * 16
        return {"bytes": c["layers"] * (attn + 2 * T * row + 2 * (sum(p) + n_off * BS) * row),
                "flops": c["layers"] * flops}
    return {"bytes": attn, "flops": flops}


def _chunks(p, s, chunk=256):
    """Whole chunks inside the computed ranges (what is offloaded)."""
    return sum(max(0, (pi + si) // chunk - -(-pi // chunk)) for pi, si in zip(p, s))


def tolerance(c):
    # append and gather move bits. Attention: bf16 inputs, fp32 sums, bf16 probabilities
    # and output. Against 64 bits the relative error measured 2.1e-3 to 2.4e-3 (the output's
    # own rounding alone is 1.7e-3); "rel" is about four times that, and "max" the same for
    # the largest difference (half an ulp of a value four times the root mean square is
    # 8e-3 of it, the probabilities' rounding adds as much).
    if c["kind"] in ("append", "gather"):
        return "exact"
    return {"rel": 1e-2, "max": 5e-2}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _layout(c, seed):
    """Block table (numpy [B][max_blocks]), slot of every new token, pool blocks."""
    p, s = _lens(c)
    rng = np.random.Generator(np.random.PCG64(seed))
    need = [-(-(pi + si) // BS) for pi, si in zip(p, s)]
    nb = sum(need) + max(8, sum(need) // 16)
    perm = rng.permutation(nb).astype(np.int32)
    bt = np.full((len(p), max(need)), -1, np.int32)
    slots, off = [], 0
    for b, n in enumerate(need):
        bt[b, :n] = perm[off:off + n]
        off += n
        t = np.arange(p[b], p[b] + s[b])
        slots.append(bt[b][t // BS].astype(np.int64) * BS + t % BS)
    return p, s, bt, np.concatenate(slots).astype(np.int32), nb


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _inputs(c, seed, layer=0):
    """One layer's pool K/V, Q and new K/V, from the seed."""
    p, s, bt, slots, nb = _layout(c, seed)
    T, D, Hq, Hkv = sum(s), c["D"], c["Hq"], c["Hkv"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 64 + layer)
    return dict(pool_k=_normal(gen, nb, Hkv, BS * D), pool_v=_normal(gen, nb, Hkv, BS * D),
                q=_normal(gen, T, Hq, D), k_new=_normal(gen, T, Hkv, D), v_new=_normal(gen, T, Hkv, D))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(c, seed):
    if c["kind"] == "pipeline":
        return _prepare_pipeline(c, seed)
    p, s, bt, slots, nb = _layout(c, seed)
    x = _inputs(c, seed)
    st = dict(case=c, kind=c["kind"], Hq=c["Hq"], pool=pcr.KVPool(x["pool_k"], x["pool_v"], c["Hkv"], c["D"]),
              bt=_dev(bt), q=x["q"], k_new=x["k_new"], v_new=x["v_new"], slots=_dev(slots))
    if c["kind"] in ("append", "gather"):
        T, Hkv, D = sum(s), c["Hkv"], c["D"]
        cu = np.concatenate([[0], np.cumsum(s)]).astype(np.int32)
        st.update(T=T, starts=_dev(np.asarray(p, np.int32)), cu=_dev(cu),
                  k_out=torch.zeros(T, Hkv, D, dtype=torch.bfloat16, device="cuda"),
                  v_out=torch.zeros(T, Hkv, D, dtype=torch.bfloat16, device="cuda"))
        return st
    st["out"] = torch.zeros_like(x["q"])
    if c["kind"] in ("decode", "decode_step"):
        ctx = (np.asarray(p) + np.asarray(s)).astype(np.int32)
        n = pcr.decode_attn_workspace_bytes(len(p), c["Hq"], c["Hkv"], c["D"], int(ctx.max()))
        st.update(h_ctx=ctx, ctx=_dev(ctx),
                  ws=torch.empty(max(n, 16), dtype=torch.uint8, device="cuda"))   # kept by the serving loop
        return st
    h_pl = np.asarray(p, np.int32)
    h_cu = np.concatenate([[0], np.cumsum(s)]).astype(np.int32)
    st.update(h_pl=h_pl, h_cu=h_cu, pl=_dev(h_pl), cu=_dev(h_cu))
    return st


def _prepare_pipeline(c, seed):
    p, s, bt, _, nb = _layout(c, seed)
    Hkv, D = c["Hkv"], c["D"]
    n_host = [-(-pi // BS) for pi in p]
    hb = np.full((len(p), max(n_host)), -1, np.int32)
    off = 0
    for b, n in enumerate(n_host):     # a sequence's cached prefix is one run of host blocks
        hb[b, :n] = np.arange(off, off + n)
        off += n
    src, dst, slots, cu = pcr.plan(p, s, bt, hb)
    off_src, off_dst = pcr.plan_offload(p, s, bt)
    layers, offs = [], []

    def pin(t):
        h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
        h.copy_(t)
        return h

    for i in range(c["layers"]):
        x = _inputs(c, seed, i)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed * 64 + 32 + i)
        host = pcr.HostKV(pin(_normal(gen, off, Hkv, BS * D)), pin(_normal(gen, off, Hkv, BS * D)), Hkv, D)
        layers.append(pcr.Layer(host, pcr.KVPool(x["pool_k"], x["pool_v"], Hkv, D), x["q"], x["k_new"], x["v_new"],
                                torch.zeros_like(x["q"])))
        shape = (max(1, len(off_dst)), Hkv, BS * D)
        offs.append(pcr.HostKV(pin(torch.zeros(shape, dtype=torch.bfloat16)),
                               pin(torch.zeros(shape, dtype=torch.bfloat16)), Hkv, D))
    h_pl = np.asarray(p, np.int32)
    batch = pcr.BatchPlan(src, dst, _dev(slots), _dev(bt), _dev(h_pl), _dev(cu), h_pl, cu, c["Hq"], D ** -0.5)
    ws = torch.empty(max(16, pcr.staged_workspace_bytes(len(off_src), Hkv, D)), dtype=torch.uint8, device="cuda")
    return dict(case=c, kind="pipeline", layers=layers, offs=offs, batch=batch, off_src=off_src, off_dst=off_dst,
                ws=ws, streams=[torch.cuda.Stream(), torch.cuda.Stream()])


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(st):
    kind = st["kind"]
    if kind == "pipeline":
        compute = torch.cuda.current_stream()
        copy, offload = st["streams"]
        pcr.pipeline_run_offload(st["layers"], st["offs"], st["batch"], st["off_src"], st["off_dst"], copy, compute,
                                 offload, offload_method="dma_staged" if len(st["off_src"]) else "auto",
                                 workspace=st["ws"])
        compute.wait_stream(offload)
        return [[L.out for L in st["layers"]], [L.pool.k for L in st["layers"]], [L.pool.v for L in st["layers"]],
                [h.k for h in st["offs"]], [h.v for h in st["offs"]]]
    pool = st["pool"]
    if kind == "append":
        pcr.append_kv(pool, st["k_new"], st["v_new"], st["slots"])
        return [pool.k, pool.v]
    if kind == "gather":
        pcr.gather_kv(pool, st["bt"], st["starts"], st["cu"], st["T"], st["k_out"], st["v_out"])
        return [st["k_out"], st["v_out"]]
    if kind in ("step", "decode_step"):
        pcr.append_kv(pool, st["k_new"], st["v_new"], st["slots"])
    if kind in ("decode", "decode_step"):
        pcr.decode_attn(st["q"], pool, st["bt"], st["ctx"], st["h_ctx"], st["Hq"], st["out"], workspace=st["ws"])
    else:
        pcr.prefix_prefill_attn(st["q"], pool, st["bt"], st["pl"], st["cu"], st["h_pl"], st["h_cu"], st["Hq"],
                                st["out"])
    return [st["out"], pool.k, pool.v] if kind in ("step", "decode_step") else [st["out"]]


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _attention64(c, p, s, bt, pool_k, pool_v, q):
    """Causal attention of the new rows in 64 bits, one (sequence, kv head) at a time."""
    D, Hq, Hkv = c["D"], c["Hq"], c["Hkv"]
    G = Hq // Hkv
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    t0 = 0
    for b in range(len(p)):
        n, sb = p[b] + s[b], s[b]
        blocks = _dev(bt[b][:-(-n // BS)].astype(np.int64))
        for g in range(Hkv):
            k = pool_k[blocks, g].reshape(-1, D)[:n].double()
            v = pool_v[blocks, g].reshape(-1, D, BS).transpose(1, 2).reshape(-1, D)[:n].double()
            qq = q[t0:t0 + sb, g * G:(g + 1) * G].reshape(sb * G, D).double()
            pos = p[b] + torch.arange(sb, device=q.device).repeat_interleave(G)
            res = torch.empty(sb * G, D, dtype=torch.float64, device=q.device)
            step = max(1, (1 << 27) // n)
            for r in range(0, sb * G, step):
                sc = (qq[r:r + step] @ k.t()) * D ** -0.5
                sc.masked_fill_(torch.arange(n, device=q.device)[None, :] > pos[r:r + step, None], float("-inf"))
                res[r:r + step] = torch.softmax(sc, dim=1) @ v
            out[t0:t0 + sb, g * G:(g + 1) * G] = res.reshape(sb, G, D)
        t0 += sb
    return out


def _append(c, slots, x):
    """The pool with the new tokens' rows written (plain indexing)."""
    D, Hkv = c["D"], c["Hkv"]
    sl = _dev(slots.astype(np.int64))
    k = x["pool_k"].view(-1, Hkv, BS, D)
    v = x["pool_v"].view(-1, Hkv, D, BS)
    k[sl // BS, :, sl % BS] = x["k_new"]
    v[sl // BS, :, :, sl % BS] = x["v_new"]
    return x["pool_k"], x["pool_v"]


def exact(c, seed):
    kind = c["kind"]
    if kind in ("append", "gather"):
        return None                      # bits moved, nothing computed
    p, s, bt, slots, nb = _layout(c, seed)
    if kind == "pipeline":
        outs = []
        for i in range(c["layers"]):
            x = _inputs(c, seed, i)
            gen = torch.Generator(device="cuda")
            gen.manual_seed(seed * 64 + 32 + i)
            n_host = [-(-pi // BS) for pi in p]
            hk, hv = (_normal(gen, sum(n_host), c["Hkv"], BS * c["D"]) for _ in range(2))
            at = 0
            for b, n in enumerate(n_host):
                blocks = _dev(bt[b][:n].astype(np.int64))
                x["pool_k"][blocks] = hk[at:at + n]
                x["pool_v"][blocks] = hv[at:at + n]
                at += n
            pk, pv = _append(c, slots, x)
            outs.append(_attention64(c, p, s, bt, pk, pv, x["q"]))
        none = [None] * c["layers"]
        return [outs, none, list(none), list(none), list(none)]
    x = _inputs(c, seed)
    if kind in ("step", "decode_step"):
        pk, pv = _append(c, slots, x)
        return [_attention64(c, p, s, bt, pk, pv, x["q"]), None, None]
    return [_attention64(c, p, s, bt, x["pool_k"], x["pool_v"], x["q"])]
