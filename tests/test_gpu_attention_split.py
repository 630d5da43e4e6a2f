"""GPU: prefill launches of few workgroups, whose row tiles' keys are cut into chunks and
merged by a second kernel (the default schedule's choice for a short suffix on a long
prefix), against the fp64 oracle; from captured graphs; on many streams at once; and not
taken for an output that is the query buffer."""
import numpy as np
import pytest
import torch

from oracle import attention as oattn
from oracle import datamove as odm
from paper_2603_23049_amd import pcr, synth
from gpuio import GpuLayer, MAX_ABS, MEAN_ABS, attn_schedule, error_stats, say, u16

pytestmark = pytest.mark.gpu
BS = 16


def _layer(pl, sl, G, Hkv, d, seed):
    nb = sum(-(-(p + s) // BS) for p, s in zip(pl, sl)) + 3
    b = synth.ragged_batch("split", Hq=Hkv * G, Hkv=Hkv, d=d, prefix_lens=pl, suffix_lens=sl, pool_blocks=nb, seed=seed)
    data = synth.make_layer(b)
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    shape = (nb, Hkv, BS * d)
    # (the slots no token fills hold NaN patterns: nothing past a sequence may reach the result)
    pk0, pv0 = np.full(shape, 0xFFFF, np.uint16), np.full(shape, 0xFFFF, np.uint16)
    L = GpuLayer(b, data, pk0, pv0)
    L.load("kernel_pull")
    L.append()
    torch.cuda.synchronize()
    # a partial last prefix block is loaded whole; the tokens past the sequence get the NaN back
    plan = odm.plan(b.prefix_lens, b.suffix_lens, b.block_tables, b.host_blocks, BS)
    pk, pv = odm.pool_after_layer(pk0, pv0, data.host_k, data.host_v, plan, data.k_new, data.v_new, BS)
    flat = np.arange(0, b.T * b.num_q_heads, max(1, b.T * b.num_q_heads // 1500))
    rows = np.stack([flat // b.num_q_heads, flat % b.num_q_heads], 1).astype(np.int32)
    want = oattn.attention(data.q, pk, pv, b.block_tables, np.asarray(pl, np.int32), plan[3], Hkv, BS, rows=rows)
    return L, rows, want


def _check(L, rows, want, label):
    got = L.out_f64()
    assert np.all(np.isfinite(got)), label
    mx, mean = error_stats(got[rows[:, 0], rows[:, 1]], want)
    say(f"    {label}: max_abs={mx:.3e} mean_abs={mean:.3e}")
    assert mx <= MAX_ABS and mean <= MEAN_ABS, f"{label}: max {mx} mean {mean}"


CASES = [
    # one row tile, partly filled; last chunk of one key past a tile, a full one, one short of it
    ([1985], [15], 4, 8, 128), ([1984], [64], 1, 8, 128), ([2031], [1], 4, 8, 128), ([4095], [1], 16, 2, 64),
    # many chunks: more than one pass of the combine
    ([9000], [3], 4, 1, 128), ([9000], [1], 5, 1, 64),
    # row tiles that end chunks before the last one (no prefix), rows past the end of a tile
    ([0], [2000], 2, 2, 128), ([5], [1999], 1, 3, 64),
    # a token's heads cut by row tiles; more than 16 heads per kv head: one-token rows on tiles
    ([3000, 2500], [33, 70], 5, 2, 128), ([3000, 4000], [1, 9], 20, 1, 128),
    # ragged: sequences of one chunk, of many, decode rows beside them, none new in one
    ([4000, 100, 2999, 0, 5000, 17], [40, 30, 1, 64, 1, 0], 4, 4, 128),
    ([3000, 3100, 10, 2600], [1, 1, 1, 1], 8, 8, 64),
]


# Few workgroups, but keys too short to gain by it: 14 us whole, 17 us cut.
WHOLE = [([2047], [1], 16, 2, 64)]


@pytest.mark.parametrize("pl,sl,G,Hkv,d", CASES + WHOLE)
def test_split_launch_against_oracle(pl, sl, G, Hkv, d):
    say(f"[gpu] key split p={pl} s={sl} G={G} Hkv={Hkv} d={d}")
    L, rows, want = _layer(pl, sl, G, Hkv, d, seed=300 + len(pl) + G + sl[0])
    L.attn()
    torch.cuda.synchronize()
    _check(L, rows, want, "split")
    first = L.out.clone()
    L.out.fill_(-1)
    L.attn()
    torch.cuda.synchronize()
    assert torch.equal(L.out, first), "a repeated call differs"
    with attn_schedule("key_halves"):
        L.attn()
    torch.cuda.synchronize()
    assert torch.equal(L.out, first) == ((pl, sl, G, Hkv, d) in WHOLE), "the default schedule's choice for these keys"


def test_split_launch_replayed_from_a_graph_beside_eager_calls():
    L, rows, want = _layer([3000], [20], 4, 8, 128, seed=41)
    say("[gpu] key split from a graph")
    L.attn()
    torch.cuda.synchronize()
    eager = L.out.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.attn()
    for _ in range(4):
        L.out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(L.out, eager)
        L.attn()
        torch.cuda.synchronize()
        assert torch.equal(L.out, eager)
    _check(L, rows, want, "graph")


def test_split_launches_on_many_streams():
    """Claims and reuse of the scratch by launches that overlap (as many as the hardware
    queues run at once): every output is right, and the scratch is whole again afterwards."""
    L, rows, want = _layer([5000], [24], 4, 8, 128, seed=43)
    say("[gpu] key split on 12 streams")
    L.attn()
    torch.cuda.synchronize()
    eager = L.out.clone()
    streams = [torch.cuda.Stream() for _ in range(12)]
    outs = [torch.full_like(L.out, -1) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(6):
        for s, o in zip(streams, outs):
            pcr.prefix_prefill_attn(L.q, L.pool, L.bt, L.pl, L.cu, L.pl_np, L.cu_np, L.batch.num_q_heads, o,
                                    sm_scale=L.sm_scale, stream=s)
    torch.cuda.synchronize()
    for o in outs:
        L.out.copy_(o)
        _check(L, rows, want, "stream")
    L.attn()
    torch.cuda.synchronize()
    assert torch.equal(L.out, eager)
    assert pcr.prefill_attn_hold_scratch(0) == 64


@pytest.mark.parametrize("pl,sl,G,Hkv,d", [
    ([3000], [20], 4, 8, 128), ([2500], [70], 5, 3, 64), ([4000], [1], 4, 8, 128),
    ([3000, 2000, 10], [1, 33, 1], 8, 2, 64),
])
def test_launch_that_finds_the_scratch_taken_runs_whole(pl, sl, G, Hkv, d):
    """With every part of the scratch held, a call and a replay of a captured call take every
    key in one piece (the bits of key halves, tile rows and one-token rows); with one part
    free, and after all are, they cut the keys again."""
    say(f"[gpu] key split, scratch held: p={pl} s={sl} G={G} Hkv={Hkv} d={d}")
    L, rows, want = _layer(pl, sl, G, Hkv, d, seed=48 + G)

    def both():
        outs = []
        for call in (L.attn, g.replay):
            L.out.fill_(-1)
            call()
            torch.cuda.synchronize()
            outs.append(L.out.clone())
        assert torch.equal(*outs), "replay and call differ"
        return outs[0]

    with attn_schedule("key_halves"):
        L.attn()
    torch.cuda.synchronize()
    whole = L.out.clone()
    L.attn()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.attn()
    cut = both()
    assert not torch.equal(cut, whole)
    try:
        assert pcr.prefill_attn_hold_scratch(8) == 56
        assert torch.equal(both(), whole)
        assert torch.equal(both(), whole)
        assert pcr.prefill_attn_hold_scratch(7) == 57
        assert torch.equal(both(), cut)
    finally:
        free = pcr.prefill_attn_hold_scratch(0)
    assert free == 64
    assert torch.equal(both(), cut)
    _check(L, rows, want, "cut")


def test_overlapping_calls_with_one_output_keep_the_scratch_whole():
    """Equal calls on several streams write one output: each has scratch of its own, the
    bits are those of one call, and every part of the scratch is free afterwards. So do
    replays of one captured call, which share theirs."""
    L, _, _ = _layer([5000], [24], 4, 8, 128, seed=44)
    say("[gpu] key split, one output on 6 streams")
    L.attn()
    torch.cuda.synchronize()
    eager = L.out.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.attn()
    streams = [torch.cuda.Stream() for _ in range(6)]
    for replay in (False, True):
        for _ in range(5):
            L.out.fill_(-1)
            torch.cuda.synchronize()
            for _ in range(4):
                for s in streams:
                    if replay:
                        with torch.cuda.stream(s):
                            g.replay()
                    else:
                        L.attn(stream=s)
            torch.cuda.synchronize()
            assert torch.equal(L.out, eager)
    assert pcr.prefill_attn_hold_scratch(0) == 64


def test_output_in_place_of_the_queries_is_not_split():
    """Chunks of one row tile read its queries after others have been written out, so an
    output that overlaps q takes the launch without chunks."""
    L, rows, want = _layer([3000], [20], 4, 8, 128, seed=47)
    with attn_schedule("key_halves"):
        L.attn()
    torch.cuda.synchronize()
    whole = L.out.clone()
    q = L.q.clone()
    pcr.prefix_prefill_attn(q, L.pool, L.bt, L.pl, L.cu, L.pl_np, L.cu_np, L.batch.num_q_heads, q, sm_scale=L.sm_scale)
    torch.cuda.synchronize()
    assert torch.equal(q.view(torch.int16), whole)


@pytest.mark.parametrize("low", [100, 6000])
def test_keys_whose_products_overflow_weigh_nothing(low):
    """The first keys' products overflow to -inf: whole chunks, and a whole pass of the
    merge, carry no weight, and the rows come from the other keys (as without chunks)."""
    L, _, _ = _layer([9000], [3], 4, 1, 128, seed=51)
    say(f"[gpu] key split, {low} keys at -inf")
    L.q.copy_(L.q.view(torch.bfloat16).abs().view(L.q.dtype))
    k = L.pool.k.view(torch.bfloat16).view(-1, 1, BS, 128)
    for t in range(0, low, BS):
        k[L.bt[0, t // BS].long(), 0, :min(BS, low - t)] = -3e38
    L.attn()
    torch.cuda.synchronize()
    got = L.out_f64()
    assert np.all(np.isfinite(got))
    with attn_schedule("key_halves"):
        L.attn()
    torch.cuda.synchronize()
    mx, mean = error_stats(got, L.out_f64())
    assert mx <= MAX_ABS and mean <= MEAN_ABS, f"max {mx} mean {mean}"


@pytest.mark.parametrize("pl,sl,G,Hkv,d", [
    ([300] * 64, [20] * 64, 4, 8, 128),            # suffixes shorter than a tile: key halves
    ([700], [1280], 4, 8, 128), ([40] * 5, [700] * 5, 4, 8, 64),
    ([1000], [3600], 2, 8, 128), ([0, 5, 900], [1700, 1, 900], 7, 4, 128),
])
def test_default_schedule_of_one_to_four_rounds(pl, sl, G, Hkv, d):
    """More items than compute units: the default takes one of the two schedules, whole."""
    say(f"[gpu] default schedule B={len(pl)} s={sl[0]} G={G} Hkv={Hkv} d={d}")
    L, rows, want = _layer(pl, sl, G, Hkv, d, seed=500 + len(pl) + G)
    L.attn()
    torch.cuda.synchronize()
    _check(L, rows, want, "default")
    got = L.out.clone()
    same = []
    for name in ("key_halves", "row_halves"):
        with attn_schedule(name):
            L.attn()
        torch.cuda.synchronize()
        same.append(torch.equal(L.out, got))
    assert any(same)


@pytest.mark.parametrize("pl,sl,G,Hkv,d,faster", [
    # few workgroups, but keys too short to cut: 14 us whole and 17 us cut, 11 and 17, 20 and 25
    ([1899] * 7, [1] * 7, 4, 4, 64, "key_halves"), ([1270], [1], 16, 4, 64, "key_halves"),
    ([1200], [78], 8, 8, 128, "key_halves"),
    # triangular items of 2 to 34 key tiles: 79 us with key halves, 103 with row halves
    ([98, 74], [2117, 2082], 7, 4, 128, "key_halves"),
    # 1.09 row-halves items per compute unit: 47 and 52 us
    ([717] * 5, [315] * 5, 5, 8, 128, "key_halves"),
    # 2.66, 64 dims: 717 and 655 us; 3.75: 468 and 423
    ([12972] * 5, [541] * 5, 16, 4, 64, "row_halves"), ([4683] * 3, [2544] * 3, 4, 8, 64, "row_halves"),
    # one row-halves item each for suffixes of half a tile: 154 and 200 us
    ([3000] * 64, [32] * 64, 4, 8, 128, "key_halves"),
])
def test_default_schedule_is_the_faster_one(pl, sl, G, Hkv, d, faster):
    """Where the two schedules differ in time the default takes the faster: its bits."""
    say(f"[gpu] default schedule B={len(pl)} s={sl[0]} p={pl[0]} G={G} Hkv={Hkv} d={d}: {faster}")
    need = [-(-(p + n) // BS) for p, n in zip(pl, sl)]
    nb, T = sum(need), sum(sl)
    bt = np.full((len(pl), max(need)), -1, np.int32)
    off = 0
    for b, n in enumerate(need):
        bt[b, :n] = np.arange(off, off + n)
        off += n
    gen = torch.Generator(device="cuda")
    gen.manual_seed(G + T)
    k, v = (torch.randn(nb, Hkv, BS * d, device="cuda", generator=gen).bfloat16() for _ in range(2))
    q = torch.randn(T, G * Hkv, d, device="cuda", generator=gen).bfloat16()
    hp, hc = np.asarray(pl, np.int32), np.concatenate([[0], np.cumsum(sl)]).astype(np.int32)
    bt, pl_d, cu_d = (torch.from_numpy(x).cuda() for x in (bt, hp, hc))
    outs = {}
    for name in ("auto", "key_halves", "row_halves"):
        outs[name] = torch.zeros_like(q)
        with attn_schedule(name):
            pcr.prefix_prefill_attn(q, pcr.KVPool(k, v, Hkv, d), bt, pl_d, cu_d, hp, hc, G * Hkv, outs[name])
        torch.cuda.synchronize()
    if len(set(sl)) > 1 or sl[0] > 1:        # (one-token rows are the same in both)
        assert not torch.equal(outs["key_halves"], outs["row_halves"])
    assert torch.equal(outs["auto"], outs[faster])
