"""Decode batches and appends at the sizes where the short-batch paths change: the rounds of the
append's sequence search (16 offsets each), the pieces KV ranges are cut into, the merge's early
rows and its records beyond the first 64."""
import numpy as np
import pytest

import mc_inputs as mi
import paper_2412_12488_amd as mc
from test_gpu_parity import (LSE_TOL, O_TOL, canary, check_attention, fill_both, forked_decode_workload,
                             plan_header, small_workload)
from gpu_harness import DEV, DevBatch, DevPool, bits, dev, gpu_append

import oracle
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2, 16, 17, 31, 256, 257, 300])
@pytest.mark.parametrize("Hkv", [1, 8, 16])
def test_append_finds_every_sequence(batch, Hkv):
    # one to three new tokens a sequence, every fifth sequence (the last included) with none
    rng = mi.rng_for(900 + batch)
    begins = [int(x) for x in rng.integers(0, 40, size=batch)]
    new = [0 if batch > 1 and (batch - 1 - i) % 5 == 0 else 1 + i % 3 for i in range(batch)]
    lens = [max(b + n, 1) for b, n in zip(begins, new)]
    w = small_workload(900 + batch, mi.BF16, Hkv, Hkv, lens, begins)
    init = canary(3, DevPool(w).elems)
    pool, opool, db = DevPool(w, fill=init), init.copy(), DevBatch(w)
    ks, vs = [], []
    for s in range(w.batch):
        k, v = w.kv(s, 0)
        k, v = k[w.b[s]:], v[w.b[s]:]
        ks.append(k), vs.append(v)
        if len(k):
            oracle.append(opool, pool.shape, 0, k, v, int(w.b[s]), w.page_tables[s])
    gpu_append(pool, 0, dev(np.concatenate(ks)), dev(np.concatenate(vs)), db)
    torch.cuda.synchronize()
    assert np.array_equal(bits(pool.t), opool)


@pytest.mark.parametrize("batch", [1, 17, 257])
@pytest.mark.parametrize("Hkv", [1, 3, 8, 16])
def test_append_send_finds_every_sequence(batch, Hkv):
    # heads below, at and above what a lane loads at once, every round of the sequence search; each
    # sequence marks another range: its new tokens, from or up to one inside them, beyond them, none
    rng = mi.rng_for(930 + batch)
    begins = [int(x) for x in rng.integers(0, 40, size=batch)]
    new = [0 if batch > 1 and (batch - 1 - i) % 5 == 0 else 1 + i % 3 for i in range(batch)]
    lens = [max(b + n, 1) for b, n in zip(begins, new)]
    new = [n - b for n, b in zip(lens, begins)]
    marks = [[(b, b + n), (b + 1, b + n + 2), (max(b - 2, 0), b + 1), (b + n, b + n + 3), (b, b)][i % 5]
             for i, (b, n) in enumerate(zip(begins, new))]
    w = small_workload(930 + batch, mi.BF16, Hkv, Hkv, lens, begins)
    init = canary(4, DevPool(w).elems)
    pool, opool, db = DevPool(w, fill=init), init.copy(), DevBatch(w)
    row = Hkv * 128
    offs = np.concatenate([[0], np.cumsum([2 * (e - s) * row + 64 for s, e in marks])]) + 64
    raw = canary(5, int(offs[-1]))
    send, expect = dev(raw), raw.copy()
    ks, vs = [], []
    for i in range(batch):
        k, v = (x[begins[i]:] if new[i] else x[:0] for x in w.kv(i, 0))
        ks.append(k), vs.append(v)
        if new[i]:
            oracle.append(opool, pool.shape, 0, k, v, begins[i], w.page_tables[i])
        s0, s1 = marks[i]
        for h, x in enumerate((k, v)):                    # [K|V][token - s0][head][D]
            for t in range(max(s0, begins[i]), min(s1, begins[i] + new[i])):
                at = int(offs[i]) + (h * (s1 - s0) + t - s0) * row
                expect[at:at + row] = np.ascontiguousarray(x[t - begins[i]]).reshape(-1).view(np.uint16)
    mc.mc_kv_append_send(pool.desc, 0, dev(np.concatenate(ks)), dev(np.concatenate(vs)), db.batch, db.total_q,
                         db.cu_q, db.begin, db.page_table, db.cu_pages, 0,
                         dev(np.array([m[0] for m in marks], np.int32)),
                         dev(np.array([m[1] for m in marks], np.int32)),
                         torch.tensor([2 * int(o) for o in offs[:-1]], dtype=torch.int64, device=DEV), send)
    torch.cuda.synchronize()
    assert np.array_equal(bits(pool.t), opool)
    assert np.array_equal(bits(send), expect)             # marked rows, holes and guards


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("lens,chunk", [
    ([128], 0),                       # two tiles: nothing to cut
    ([129], 2), ([1024], 2),          # up to 16 tiles: pieces of two tiles, at most eight
    ([1025], 4), ([2048, 700, 1], 4), # longer: pieces of four
    ([4097], 4),                      # more pieces than rows requested early
    ([200] * 65, 2),                  # more merge records than lanes
])
def test_decode_pieces(dtype, lens, chunk):
    Hq, Hkv = (8, 1) if len(lens) > 3 else (32, 8)
    w = small_workload(950 + len(lens) + lens[0], dtype, Hq, Hkv, lens, [n - 1 for n in lens])
    assert plan_header(w)["chunk_tiles"] == chunk
    check_attention(w)


@pytest.mark.parametrize("lens,begins,chunk", [
    ([1280] + [16] * 255, [1024] + [16] * 255, 8),    # one range among idle sequences: no decode step
    ([16] * 255 + [700], [16] * 255 + [699], 2),      # one decode row among idle sequences
    ([16] * 40 + [1300] * 2, [16] * 40 + [1299] * 2, 4),
    ([900] * 63 + [902], [899] * 63 + [900], 8),      # one row of two new tokens: a range
])
def test_decode_pieces_are_for_single_new_tokens(lens, begins, chunk):
    w = small_workload(970 + chunk, mi.BF16, 8, 1, lens, begins)
    assert plan_header(w)["chunk_tiles"] == chunk
    check_attention(w)


# per line: both sides of one bound, as it lies with 512 workgroup slots
@pytest.mark.parametrize("Hq,Hkv,lens,chunk", [
    (8, 2, [800] * 38, 2), (8, 2, [800] * 39, 4),           # pieces of two in one turn, or of four
    (8, 2, [900] * 80, 6), (8, 2, [900] * 100, 8),          # pieces of six, or of eight
    (32, 8, [1150] * 14, 4), (32, 8, [960] * 17, 8),        # pieces of four, or of eight
    (8, 2, [6000] * 8, 4), (8, 2, [7000] * 8, 8),           # 24 pieces a row, or more
    (32, 8, [2600] * 8, 6), (32, 8, [2300] * 8, 8),         # six fill the slots, or not
    (32, 8, [500] * 24, 4), (32, 8, [500] * 32, 0),         # whole ranges: few to read at once, or many
    (8, 1, [500] * 144, 4), (8, 1, [500] * 145, 0),
    (8, 1, [300] * 64, 2), (8, 1, [300] * 65, 2), (8, 1, [300] * 130, 0),
])
def test_short_pieces_only_where_they_pay(Hq, Hkv, lens, chunk):
    w = small_workload(960 + len(lens), mi.BF16, Hq, Hkv, lens, [n - 1 for n in lens])
    assert plan_header(w)["chunk_tiles"] == chunk
    check_attention(w)


@pytest.mark.parametrize("forks,chunk", [(64, 4), (128, 8)])
def test_short_pieces_of_groups_whose_merges_are_small(forks, chunk):
    w = forked_decode_workload(990, 8, 1, mi.BF16, [[(4400, 0)] + [(4390, 4096)] * (forks - 1)])
    h = plan_header(w)
    assert h["chunk_tiles"] == chunk and h["num_groups_rows"] == forks * 64 // chunk, h


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("start", [[1500, 2100, 900], [1000, 640, 129]])
def test_pieces_that_are_not_computed_leave_nothing_behind(dtype, start):
    """A begin below the planned one leaves the last pieces of a row without a key.  The merge gives
    them no weight whatever their partial rows held: here, and in any recycled memory, NaN."""
    Hq, Hkv, B = 32, 8, 3
    w = small_workload(980, dtype, Hq, Hkv, [n + 1 for n in start], start)
    pool = DevPool(w)
    opool = oracle.new_pool(pool.shape)
    fill_both(w, pool, opool)
    db = DevBatch(w)
    ws_bytes = mc.mc_attn_workspace_size(B, B, Hq, Hkv)
    ws = torch.full((ws_bytes,), 0xff, dtype=torch.uint8, device=DEV)
    mc.mc_attn_plan(pool.desc, Hq, B, B, db.cu_q, db.begin, db.page_table, db.cu_pages, ws, ws_bytes)
    mc.mc_attn_plan_check(ws)
    assert int(ws[:64].view(torch.int32)[6]) == B           # every row is cut
    q = np.concatenate([w.q(s) for s in range(B)])
    out = torch.full((B, Hq, 128), 0x7fc1, dtype=torch.int16, device=DEV)
    lse = torch.full((B, Hq), float("nan"), dtype=torch.float32, device=DEV)
    at = [3, start[1] - 300, start[2]]          # far below the plan, some pieces below it, as planned
    mc.mc_prefix_prefill_attn(pool.desc, 0, dev(q), Hq, B, B, db.cu_q, dev(np.array(at, dtype=np.int32)),
                              db.page_table, db.cu_pages, 0.0, out, lse, ws, ws_bytes)
    torch.cuda.synchronize()
    for s in range(B):
        ro, rl = oracle.attention(opool, pool.shape, 0, w.page_tables[s], w.q(s), Hq, at[s], at[s] + 1)
        assert np.max(np.abs(oracle.decode(bits(out[s:s + 1]), dtype) - ro)) <= O_TOL, s
        assert np.max(np.abs(lse[s:s + 1].cpu().numpy() - rl)) <= LSE_TOL, s


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (32, 8), (8, 1)])
def test_short_pieces_inside_a_shared_prefix(dtype, Hq, Hkv):
    # forks of at most 16 tiles: the prefix they share and their own parts in pieces of two tiles
    w = forked_decode_workload(985, Hq, Hkv, dtype, [
        [(600, 0), (1024, 528), (640, 528), (577, 528)],      # prefix of 8 tiles: 4 pieces
        [(1000, 0), (1010, 992), (1024, 992)]])               # prefix of 14 tiles: 7 pieces
    h = plan_header(w)
    assert h["chunk_tiles"] == 2 and h["num_groups_rows"] == 4 * 4 + 7 * 3, h
    check_attention(w)


# tables of fewer entries than a lane looks at, of one trip and several, mostly or partly not needed
@pytest.mark.parametrize("need,slack", [([1], 0), ([3], 2), ([5, 0, 70], 1), ([1100], 0), ([40] * 17, 3),
                                        ([9] * 40, 30), ([270] * 256, 1)])
def test_page_ids_are_checked_where_a_token_needs_them(need, slack):
    num_pages, B = 50, len(need)
    rng = mi.rng_for(995 + B)
    cu_pages = np.concatenate([[0], np.cumsum([n + slack for n in need])]).astype(np.int32)
    table = np.where(np.arange(cu_pages[-1]) % 2, -1, num_pages).astype(np.int32)      # what no token needs
    for s, n in enumerate(need):
        table[cu_pages[s]:cu_pages[s] + n] = rng.integers(0, num_pages, n)
    new = [int(n > 0) for n in need]
    cu_q = dev(np.concatenate([[0], np.cumsum(new)]).astype(np.int32))
    begin = dev(np.array([16 * n - 1 if n else 0 for n in need], np.int32))
    pool = torch.zeros(num_pages * 2 * 8 * 16 * 128, dtype=torch.int16, device=DEV)
    desc = mc.pool_desc(pool, 1, num_pages, 8, mc.MC_BF16)
    size = mc.mc_attn_workspace_size(B, sum(new), 32, 8)
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)

    def plan(t):
        mc.mc_attn_plan(desc, 32, B, sum(new), cu_q, begin, dev(t), dev(cu_pages), ws, size)
        mc.mc_attn_plan_check(ws)

    plan(table)
    for s, e in [(0, 0), (0, need[0] - 1), (B // 2, need[B // 2] // 2), (B - 1, need[-1] - 1)]:
        if need[s] == 0:
            continue
        for bad in (-1, num_pages):
            t = table.copy()
            t[cu_pages[s] + e] = bad
            with pytest.raises(mc.McError) as err:
                plan(t)
            assert err.value.status == mc.MC_ERR_RANGE, (s, e, bad)


# every id is in range but one, so the look at the table as it lies has to find it: entries that are requested early (16 of
# 256 threads, 4 of 1024), in later trips of as many, in the last four, and behind a trip's edges
@pytest.mark.parametrize("need,slack,shared", [([9000], 0, 0), ([4097], 0, 0), ([33000, 7], 0, 0), ([1000] * 17, 0, 0),
                                               ([600] * 20, 2, 0), ([150, 0, 90] * 30, 0, 0), ([130] * 255 + [4099], 0, 0),
                                               ([700] * 16, 0, 600), ([300] * 40 + [9, 0] * 5 + [2500] * 4, 0, 250)])
def test_a_single_page_id_out_of_range_is_found(need, slack, shared):
    plan, table, cu_pages, num_pages = planned_tables(need, slack)
    for s, n in enumerate(need):          # forks: found by their tables before the items are counted
        if n >= shared:
            table[cu_pages[s]:cu_pages[s] + shared] = table[:shared]
    plan(table)
    early = 4096                          # 4 entries x 4 x 256 threads, x 1 x 1024
    edges = [0, 1, 3, 4, 1023, 1024, early - 1, early, early + 1]
    trip = 4 * 4 * (256 if len(need) <= 16 else 1024)
    edges += [early + k * trip + d for k in (1, 2) for d in (-4, -1, 0)]
    last = len(table) - slack
    edges += [last - 1, last - 2, last - 3, last - 4, last - 5, last // 2]
    needed = np.concatenate([np.arange(cu_pages[s], cu_pages[s] + n) for s, n in enumerate(need)])
    for at in sorted(set(edges) & set(needed.tolist())):
        refused(plan, table, at, (-1, num_pages)[at % 2])


def refused(plan, table, at, bad):
    t = table.copy()
    t[at] = bad
    with pytest.raises(mc.McError) as err:
        plan(t)
    assert err.value.status == mc.MC_ERR_RANGE, (at, bad)


def planned_tables(need, slack):
    """plan(table) for one decode row over all entries a sequence needs, such a table with slack more entries a
    sequence, all in range, its cu_pages, and the pool's pages."""
    num_pages, B = 50, len(need)
    rng = mi.rng_for(997 + B)
    cu_pages = np.concatenate([[0], np.cumsum([n + slack for n in need])]).astype(np.int32)
    table = rng.integers(0, num_pages, cu_pages[-1]).astype(np.int32)
    new = [int(n > 0) for n in need]
    cu_q = dev(np.concatenate([[0], np.cumsum(new)]).astype(np.int32))
    begin = dev(np.array([16 * n - 1 if n else 0 for n in need], np.int32))
    pool = torch.zeros(num_pages * 2 * 8 * 16 * 128, dtype=torch.int16, device=DEV)
    desc = mc.pool_desc(pool, 1, num_pages, 8, mc.MC_BF16)
    size = mc.mc_attn_workspace_size(B, sum(new), 32, 8)
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)

    def plan(t):
        mc.mc_attn_plan(desc, 32, B, sum(new), cu_q, begin, dev(t), dev(cu_pages), ws, size)
        mc.mc_attn_plan_check(ws)

    return plan, table, cu_pages, num_pages
