"""GPU: decode rows where whole 32-key steps have no finite score (products of the queries
with their keys overflow to -inf), against the fp64 oracle: such keys weigh nothing,
wherever they lie in the range a wave walks, and however the waves' parts are merged."""
import numpy as np
import pytest
import torch

from oracle import attention as oattn
from paper_2603_23049_amd import pcr, synth
from gpuio import MAX_ABS, MEAN_ABS, attn_schedule, dev, error_stats, say, u16

pytestmark = pytest.mark.gpu
BS = 16
LOW = np.uint16(0xFF62)     # bf16 -3.0e38

# keys without a finite score, of a row that sees n keys
PATTERNS = {
    "even steps": lambda t, n: t // 32 % 2 == 0,
    "odd steps": lambda t, n: t // 32 % 2 == 1,
    "first half": lambda t, n: t < n // 2,
    "second half": lambda t, n: t >= (n + 1) // 2,
    "all but the last": lambda t, n: t < n - 1,
    "all but the first": lambda t, n: t > 0,
}


def _inputs(ctx, Hq, Hkv, d, seed):
    """Non-negative queries, one per context; pool and block tables as bf16 bits."""
    rng = np.random.Generator(np.random.PCG64(seed))
    need = [-(-n // BS) for n in ctx]
    nb = sum(need) + 2
    perm = rng.permutation(nb).astype(np.int32)
    bt = np.full((len(ctx), max(need)), -1, np.int32)
    off = 0
    for b, n in enumerate(need):
        bt[b, :n] = perm[off:off + n]
        off += n
    shape = (nb, Hkv, BS * d)
    q = synth.normal_bf16(rng, (len(ctx), Hq, d)) & 0x7FFF
    return q, synth.normal_bf16(rng, shape), synth.normal_bf16(rng, shape), bt


def _lower(pk, bt, ctx, Hkv, d, pattern):
    pk = pk.copy()
    rows = pk.reshape(-1, Hkv, BS, d)
    for b, n in enumerate(ctx):
        t = np.arange(n)
        t = t[PATTERNS[pattern](t, n)]
        rows[bt[b][t // BS], :, t % BS] = LOW
    return pk


def _check(out, want, label):
    got = synth.bf16_bits_to_f32(u16(out)).astype(np.float64)
    assert np.all(np.isfinite(got)), f"{label}: rows without a value"
    mx, mean = error_stats(got, want)
    say(f"    {label}: max_abs={mx:.3e} mean_abs={mean:.3e}")
    assert mx <= MAX_ABS and mean <= MEAN_ABS, (label, mx, mean)


SHAPES = [
    # one wave (one chunk a sequence); chunks that merge in LDS, through the workspace, and
    # shared by two and by four waves each
    ([33, 64, 200, 70] * 70, 32, 8, 128), ([1100] * 32, 32, 8, 128),
    ([1000, 2000, 4100, 3333] * 4, 32, 8, 128), ([8192] * 2, 64, 4, 64),
    ([4000], 32, 8, 128), ([2600, 64, 1300], 8, 8, 64), ([16001], 16, 1, 128),
]


@pytest.mark.parametrize("ctx,Hq,Hkv,d", SHAPES)
def test_decode_steps_without_a_finite_score(ctx, Hq, Hkv, d):
    q, pk0, pv, bt = _inputs(ctx, Hq, Hkv, d, seed=len(ctx) + Hq + d)
    cl = np.asarray(ctx, np.int32)
    cu = np.arange(len(ctx) + 1, dtype=np.int32)
    say(f"[gpu] decode, steps without a score: B={len(ctx)} max={max(ctx)} Hq={Hq} Hkv={Hkv} d={d}")
    ws = torch.empty(max(16, pcr.decode_attn_workspace_bytes(len(ctx), Hq, Hkv, d, max(ctx))), dtype=torch.uint8,
                     device="cuda")
    for pattern in PATTERNS:
        pk = _lower(pk0, bt, ctx, Hkv, d, pattern)
        want = oattn.attention(q, pk, pv, bt, cl - 1, cu, Hkv, BS)
        pool = pcr.KVPool(dev(pk), dev(pv), Hkv, d)
        for how in ("workspace", "one-byte workspace", "noalloc"):
            out = torch.full((len(ctx), Hq, d), -1, dtype=torch.int16, device="cuda")
            if how == "noalloc":
                pcr.decode_attn_noalloc(dev(q), pool, dev(bt), dev(cl), cl, Hq, out)
            elif how == "workspace" or max(ctx) <= 1100:     # (a plan that merges in LDS needs none)
                pcr.decode_attn(dev(q), pool, dev(bt), dev(cl), cl, Hq, out,
                                workspace=ws if how == "workspace" else ws[:1])
            else:
                continue
            torch.cuda.synchronize()
            _check(out, want, f"{pattern}, {how}")


@pytest.mark.parametrize("pl,sl,G,Hkv,d", [
    ([3999], [1], 4, 8, 128), ([9000], [1], 5, 1, 64), ([3000, 3100, 64, 2600], [1, 1, 1, 1], 8, 8, 64),
    ([4000, 2999, 64], [20, 1, 1], 4, 4, 128),
])
def test_prefill_launch_decode_rows_without_a_finite_score(pl, sl, G, Hkv, d):
    """One-token rows of the prefill entry point, in launches that cut the keys into chunks
    (the default for these lengths) and whole."""
    ctx = [p + s for p, s in zip(pl, sl)]
    q, pk0, pv, bt = _inputs(ctx, G * Hkv, Hkv, d, seed=G + d + sum(sl))
    T = sum(sl)
    q = np.repeat(q, sl, axis=0)
    cu = np.concatenate([[0], np.cumsum(sl)]).astype(np.int32)
    pln = np.asarray(pl, np.int32)
    say(f"[gpu] prefill launch, decode rows without a score: p={pl} s={sl} G={G} Hkv={Hkv} d={d}")
    for pattern in PATTERNS:
        if pattern == "all but the last" and max(sl) > 1:
            continue                         # (no finite score for the rows before the last)
        pk = _lower(pk0, bt, ctx, Hkv, d, pattern)
        want = oattn.attention(q, pk, pv, bt, pln, cu, Hkv, BS)
        pool = pcr.KVPool(dev(pk), dev(pv), Hkv, d)
        for schedule in ("auto", "key_halves", "row_halves"):
            out = torch.full((T, G * Hkv, d), -1, dtype=torch.int16, device="cuda")
            with attn_schedule(schedule):
                pcr.prefix_prefill_attn(dev(q), pool, dev(bt), dev(pln), dev(cu), pln, cu, G * Hkv, out)
            torch.cuda.synchronize()
            _check(out, want, f"{pattern}, {schedule}")
