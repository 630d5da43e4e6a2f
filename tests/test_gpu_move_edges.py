"""GPU: gather and append against plain numpy indexing, bit for bit, where their tiles of 32 tokens and
chunks of 8 slots can go wrong: ranges that start and end inside chunks and blocks, empty
and one-token sequences, rows whose block is missing, sizes on both sides of the
non-temporal loads."""
import numpy as np
import pytest
import torch

from paper_2603_23049_amd import pcr, synth
from gpuio import dev, say, u16

pytestmark = pytest.mark.gpu
BS = 16


def _pool(rng, nb, Hkv, d):
    shape = (nb, Hkv, BS * d)
    return synth.normal_bf16(rng, shape), synth.normal_bf16(rng, shape)


def _gather_case(starts, lens, Hkv, d, seed, missing=0):
    rng = np.random.Generator(np.random.PCG64(seed))
    need = [-(-(max(0, a) + n) // BS) for a, n in zip(starts, lens)]
    nb = sum(need) + 2
    pk, pv = _pool(rng, nb, Hkv, d)
    perm = rng.permutation(nb).astype(np.int32)
    bt = np.full((len(lens), max(max(need), 1)), -1, np.int32)
    off = 0
    for b, n in enumerate(need):
        bt[b, :n] = perm[off:off + n]
        off += n
    for _ in range(missing):                       # ids outside the pool: their rows come back as zeros
        b = int(rng.integers(len(need)))
        if need[b]:
            bt[b, int(rng.integers(need[b]))] = rng.choice([-1, nb, 2**31 - 1])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(cu[-1])
    k_out = torch.full((total, Hkv, d), -1, dtype=torch.int16, device="cuda")
    v_out = torch.full_like(k_out, -1)
    pool = pcr.KVPool(dev(pk), dev(pv), Hkv, d)
    pcr.gather_kv(pool, dev(bt), dev(np.asarray(starts, np.int32)), dev(cu), total, k_out, v_out)
    torch.cuda.synchronize()
    t = np.concatenate([np.arange(a, a + n) for a, n in zip(starts, lens)]).astype(np.int64)
    b = np.repeat(np.arange(len(lens)), lens)
    inside = (t >= 0) & (t // BS < bt.shape[1])
    blk = np.where(inside, bt[b, np.clip(t // BS, 0, bt.shape[1] - 1)], -1).astype(np.int64)
    ok = (blk >= 0) & (blk < nb)
    blk0, o = np.where(ok, blk, 0), t % BS
    wk = pk.reshape(nb, Hkv, BS, d)[blk0, :, o]
    wv = pv.reshape(nb, Hkv, d, BS)[blk0, :, :, o]
    wk[~ok], wv[~ok] = 0, 0
    assert np.array_equal(u16(k_out), wk) and np.array_equal(u16(v_out), wv)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hkv", [1, 3, 8])
def test_gather_edges(d, Hkv):
    say(f"[gpu] gather edges d={d} Hkv={Hkv}")
    _gather_case([0], [1], Hkv, d, 1)
    _gather_case([7], [1], Hkv, d, 2)
    for i, (a, n) in enumerate([(0, 32), (1, 31), (8, 33), (15, 64), (16, 65), (5, 96), (31, 7)]):
        _gather_case([a], [n], Hkv, d, 10 + i)
    _gather_case([3, 0, 40, 9, 0, 15, 2], [0, 17, 1, 0, 33, 8, 9], Hkv, d, 30)
    _gather_case(list(range(70)), [1, 2, 3, 5, 7, 9, 0] * 10, Hkv, d, 31, missing=12)
    _gather_case([-5, 3], [20, 40], Hkv, d, 32)    # a start before the sequence: zero rows


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hkv", [1, 3, 8])
def test_gather_edges_in_tiles(d, Hkv):
    """The edges above in calls of more than 4 MiB of output, which tiles of 32 rows take (and
    the last call that goes row by row); a first sequence shifts them against the tiles."""
    most = (4 << 20) // (4 * Hkv * d)                  # rows of the last call that goes row by row
    say(f"[gpu] gather edges in tiles d={d} Hkv={Hkv}, from {most + 1} rows on")
    _gather_case([3], [most], Hkv, d, 40)
    _gather_case([3], [most + 1], Hkv, d, 41)
    small = [1, 31, 33, 64, 65, 96, 7, 0, 17, 1, 0, 33, 8, 9] + [1, 2, 3, 5, 7, 9, 0] * 10
    starts = [7, 1, 8, 15, 16, 5, 31, 3, 0, 40, 9, 0, 15, 2] + list(range(70))
    for shift in (0, 1, 15, 30):
        _gather_case([9] + starts, [most + shift] + small, Hkv, d, 50 + shift, missing=20)
    _gather_case([-5, 3], [most, 40], Hkv, d, 60)      # a start before the sequence: zero rows


@pytest.mark.parametrize("Hkv,d", [(8, 128), (15, 64)])
def test_gather_large_with_nontemporal_loads(Hkv, d):
    rng = np.random.Generator(np.random.PCG64(5))
    lens = [int(x) for x in rng.integers(900, 1200, size=18)]
    starts = [int(x) for x in rng.integers(0, 50, size=18)]
    assert sum(lens) * Hkv * d * 4 > 64 << 20
    say(f"[gpu] gather large: {sum(lens)} tokens, Hkv={Hkv} d={d}")
    _gather_case(starts, lens, Hkv, d, 6, missing=3)


def _append_case(slots, nb, Hkv, d, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    T = len(slots)
    slots = np.asarray(slots, np.int32)
    pk, pv = _pool(rng, nb, Hkv, d)
    k_new, v_new = synth.normal_bf16(rng, (T, Hkv, d)), synth.normal_bf16(rng, (T, Hkv, d))
    pool = pcr.KVPool(dev(pk), dev(pv), Hkv, d)
    pcr.append_kv(pool, dev(k_new), dev(v_new), dev(slots))
    torch.cuda.synchronize()
    ok = (slots >= 0) & (slots // BS < nb)
    sl = slots[ok].astype(np.int64)
    pk.reshape(nb, Hkv, BS, d)[sl // BS, :, sl % BS] = k_new[ok]
    pv.reshape(nb, Hkv, d, BS)[sl // BS, :, :, sl % BS] = v_new[ok]
    assert np.array_equal(u16(pool.k), pk), "K pool"
    assert np.array_equal(u16(pool.v), pv), "V pool"


def _segments(rng, n, nb):
    """A slot list of n runs of consecutive slots, each from anywhere in blocks of its own."""
    blocks = iter(rng.permutation(nb // 4) * 4)
    out = []
    for _ in range(n):
        base = int(next(blocks)) * BS + int(rng.integers(0, BS))
        out += range(base, base + int(rng.integers(1, 48)))
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hkv", [1, 3, 8])
def test_append_edges(d, Hkv):
    """Runs that cross tile edges (multiples of 32 tokens) inside blocks and chunks, at
    every offset; slots that are skipped in the middle of a run; runs in falling order."""
    say(f"[gpu] append edges d={d} Hkv={Hkv}")
    rng = np.random.Generator(np.random.PCG64(d + Hkv))
    for T in (1, 15, 16, 31, 32, 33, 47, 48, 49, 64, 100):
        for first in (0, 1, 7, 8, 15):
            _append_case(range(first, first + T), 8, Hkv, d, 100 + T + first)
    seg = _segments(rng, 40, 400)
    _append_case(seg, 400, Hkv, d, 7)
    holes = np.asarray(seg)
    holes[rng.integers(0, len(seg), size=60)] = rng.choice([-1, 400 * BS, 2**31 - 1], size=60)
    _append_case(holes, 400, Hkv, d, 8)
    _append_case(seg[::-1], 400, Hkv, d, 9)
    _append_case(rng.permutation(400 * BS)[:777], 400, Hkv, d, 10)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hkv", [1, 3, 8])
def test_append_edges_of_many_workgroups(d, Hkv):
    """From 257 workgroups on a tile asks for the rows after it only once it knows its slots;
    the last call below does so at once."""
    rng = np.random.Generator(np.random.PCG64(20 + d + Hkv))
    most = 256 // Hkv * 32                             # tokens of 256 workgroups
    nb = 4 * (most // 16)
    seg = _segments(rng, nb // 4, nb)[:most + 40]
    assert len(seg) == most + 40
    say(f"[gpu] append edges of many workgroups d={d} Hkv={Hkv}: {len(seg)} tokens")
    _append_case(seg[:most], nb, Hkv, d, 21)
    _append_case(seg, nb, Hkv, d, 22)
    _append_case(range(5, 5 + most + 33), nb, Hkv, d, 23)
    holes = np.asarray(seg)
    holes[rng.integers(0, len(seg), size=90)] = rng.choice([-1, nb * BS, 2**31 - 1], size=90)
    _append_case(holes, nb, Hkv, d, 24)
    _append_case(seg[::-1], nb, Hkv, d, 25)


@pytest.mark.parametrize("Hkv,d", [(8, 128), (15, 64)])
def test_append_large_ragged_with_nontemporal_loads(Hkv, d):
    rng = np.random.Generator(np.random.PCG64(11))
    nb = 4 * 800
    seg = _segments(rng, 790, nb)
    assert len(seg) * Hkv * d * 4 > 64 << 20
    say(f"[gpu] append large ragged: {len(seg)} tokens, Hkv={Hkv} d={d}")
    _append_case(seg, nb, Hkv, d, 12)
