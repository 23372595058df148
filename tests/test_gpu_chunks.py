"""Chunks of a cut KV range are combined inside the attention launch - rows that are counted (up to 16
a q tile and kv head, 32 of narrow q tiles), trees over two to many chunks, groups of both kinds, at the
row counts where one becomes the other - or in a launch behind it.  Launch after launch on one plan (the
arrival words wrap), every launch the same bits whichever chunk comes last, and the oracle's result."""
import numpy as np
import pytest

import mc_inputs as mi
import oracle
import paper_2412_12488_amd as mc
import torch
from gpu_harness import DEV, DevBatch, DevPool, bits, dev, oracle_rows
from test_gpu_parity import LSE_TOL, O_TOL, fill_both, forked_decode_workload, small_workload

pytestmark = pytest.mark.gpu


def launches(w, n=6, q=None, begin=(), blank=(0x7fc1, float("nan"))):
    """(out bits, lse) of n launches on one plan, the plan's header, and the oracle's pool.  The launches
    take other q if given, the first ones other begins, and find blank in out and lse."""
    pool = DevPool(w)
    pool.t.fill_(0x7fc1)
    opool = np.full(pool.elems, 0x7fc1, dtype=np.uint16)
    fill_both(w, pool, opool)
    db, Hq, Hkv = DevBatch(w), w.num_q_heads, w.num_kv_heads
    size = mc.mc_attn_workspace_size(db.batch, db.total_q, Hq, Hkv)
    ws = torch.full((size,), 0xff, dtype=torch.uint8, device=DEV)     # NaN wherever nothing is written
    mc.mc_attn_plan(pool.desc, Hq, db.batch, db.total_q, db.cu_q, db.begin, db.page_table, db.cu_pages, ws, size)
    mc.mc_attn_plan_check(ws)
    q = dev(np.concatenate([w.q(s) for s in range(w.batch)]) if q is None else q)
    got = []
    for i in range(n):
        b = dev(np.array(begin[i], np.int32)) if i < len(begin) else db.begin
        out = torch.full((db.total_q, Hq, 128), blank[0], dtype=torch.int16, device=DEV)
        lse = torch.full((db.total_q, Hq), blank[1], dtype=torch.float32, device=DEV)
        mc.mc_prefix_prefill_attn(pool.desc, 0, q, Hq, db.batch, db.total_q, db.cu_q, b, db.page_table,
                                  db.cu_pages, 0.0, out, lse, ws, size)
        got.append((out, lse))
    torch.cuda.synchronize()
    return got, ws[:64].view(torch.int32).cpu().numpy(), pool, opool


def check(w, n=6, rows=0):
    """The plan's header, once all launches agree with each other and with the oracle (rows > 0: on as many
    rows a sequence, any head)."""
    got, h, pool, opool = launches(w, n)
    out, lse = bits(got[0][0]), got[0][1].cpu().numpy()
    for o, l in got[1:]:
        assert np.array_equal(bits(o), out) and np.array_equal(l.cpu().numpy(), lse)
    for s in range(w.batch):
        at, q_len = int(w.cu_q[s]), int(w.n[s] - w.b[s])
        if q_len == 0:
            continue
        o, l = out[at:at + q_len], lse[at:at + q_len]
        rr = hh = None
        if rows:
            rng = mi.rng_for(w.seed, s)
            rr, hh = rng.integers(0, q_len, rows), rng.integers(0, w.num_q_heads, rows)
            o, l = o[rr, hh], l[rr, hh]
        ro, rl = oracle_rows(w, opool, pool.shape, 0, s, w.q(s), rr, hh)
        assert np.max(np.abs(oracle.decode(o, w.dtype) - ro)) <= O_TOL, s
        assert np.max(np.abs(l - rl)) <= LSE_TOL, s
    return h


# per line: the tokens of a q tile, and how many of them are cut, with 512 workgroup slots
@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,new,keys,tokens,cut", [
    # whole q tiles: 16 rows, counted (G = 4, 8, 1); a tree of more chunks than one word of arrivals has nodes
    (32, 8, 4, 2100, 32, 1), (64, 8, 2, 1100, 16, 1), (8, 8, 16, 2700, 128, 1), (8, 1, 130, 40000, 16, 9),
    # narrow ones of 16 rows, the last of 4 rows or 8, a row, as many as the others; many pieces a tile
    (32, 8, 5, 2100, 4, 2), (64, 8, 3, 1600, 2, 2), (8, 8, 17, 2700, 16, 2), (8, 8, 128, 3200, 16, 8),
    (32, 8, 33, 1000, 4, 9), (32, 8, 36, 2100, 4, 9), (32, 8, 37, 2100, 4, 10), (64, 8, 18, 1600, 2, 9),
    (64, 8, 19, 2600, 2, 10), (8, 8, 144, 2700, 16, 9), (8, 8, 145, 3300, 16, 10), (8, 1, 128, 1300, 2, 64),
    (8, 1, 129, 1300, 2, 65),
    # of 32 rows: the last of one row, of two; uncut; many pieces
    (8, 8, 129, 4300, 32, 5), (16, 8, 81, 4500, 16, 6), (16, 8, 40, 700, 8, 0), (8, 1, 20, 40000, 4, 5),
])
def test_ranges_of_few_and_many_rows(dtype, Hq, Hkv, new, keys, tokens, cut):
    w = small_workload(1200 + new, dtype, Hq, Hkv, [keys], [keys - new])
    h = check(w, rows=0 if new * keys < 1 << 20 else 512)
    assert (h[3], h[6]) == (tokens, cut) and (h[7] > 0) == (cut > 0), h[:9]


def beside_others(Hq, lens, begins):
    """lens and begins with three short ranges behind, too many tokens in all for narrow q tiles."""
    n = {8: 400, 16: 180, 32: 90, 64: 45}[Hq]
    return lens + [n + 60, n + 7, n], begins + [60, 7, 0]


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,new,keys", [
    # one tile for each of eight kv heads, or fewer: 16 rows are counted, more go up a tree
    (32, 8, 4, 2100), (32, 8, 5, 2100),       # 16 rows; 20 (G = 4)
    (64, 8, 2, 1100), (64, 8, 3, 1600),       # 16 rows, 24 (G = 8): two chunks, three
    (8, 8, 16, 2700), (8, 8, 17, 2700),       # 16 rows, 17 (G = 1): five chunks
    (8, 8, 128, 3200), (16, 8, 40, 700),      # a full tile; two chunks (G = 2)
    (8, 1, 20, 40000), (8, 1, 128, 1300),     # many chunks; eight tiles of one kv head
    # more tiles: trees, a tile of 16 rows or fewer counted
    (32, 8, 33, 1000), (32, 8, 36, 2100), (32, 8, 37, 2100),      # a tile and 4 rows, 16, 20
    (64, 8, 18, 1600), (64, 8, 19, 2600),     # 16 rows, 24
    (8, 8, 129, 4300), (8, 8, 144, 2700), (8, 8, 145, 3300),      # one row, 16, 17
    (8, 1, 129, 1300), (16, 8, 81, 4500),     # nine tiles, the last of 8 rows; 17 tokens of two rows
    (8, 1, 130, 40000),                       # more chunks than one word of arrivals has nodes
])
def test_whole_tiles_of_few_and_many_rows(dtype, Hq, Hkv, new, keys):
    lens, begins = beside_others(Hq, [keys], [keys - new])
    w = small_workload(1400 + new, dtype, Hq, Hkv, lens, begins)
    h = check(w, rows=256)
    tokens = 128 * Hkv // Hq
    assert (h[3], h[6]) == (tokens, -(-new // tokens)) and h[7] >= 8, h[:9]     # every tile of the first is cut


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (8, 8), (64, 8)])
def test_many_rounds_of_chunks(Hq, Hkv):
    # more items than run at once, decode rows beside ranges of several tiles
    w = small_workload(1230, mi.BF16, Hq, Hkv, [5000, 3000, 4100, 1800, 2600, 900], [4900, 2999, 4000, 1790, 2580, 899])
    assert check(w)[6] >= 5


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,members", [
    (32, 8, 4), (32, 8, 5), (8, 8, 16), (8, 8, 17), (64, 8, 2), (64, 8, 3),    # 16 rows of a prefix, more
    (32, 8, 40), (8, 1, 12),
])
def test_prefixes_of_few_and_many_rows(dtype, Hq, Hkv, members):
    # own parts from one token to several chunks: the prefix or the member's own chunks come last
    own = [1, 700, 40, 1500, 64, 3000, 300]
    w = forked_decode_workload(1240 + members, Hq, Hkv, dtype,
                               [[(1600 + own[i % 7], 1600 if i else 0) for i in range(members)]])
    assert check(w)[8] > 0


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
def test_members_with_trees_of_their_own(dtype):
    # forks that bring 5..8 new tokens (20..32 rows of a kv head) over own middle parts of up to five
    # chunks: these and the prefix's are combined in the launch behind it (a member's tree beside a prefix:
    # test_trees_of_members_in_larger_batches)
    begins, new = [2048, 2300, 4700, 2048, 3300], [5, 6, 8, 4, 7]
    w = small_workload(1260, dtype, 32, 8, [b + n for b, n in zip(begins, new)], begins)
    for s in range(1, 5):
        w.share_prefix(s, 0, 2048)
    assert check(w)[8] > 0


# per line: where the chunks of the row of NaN come together; the tokens of a q tile, how many are cut
@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,lens,new,shared,tokens,cut", [
    (32, 8, [1500, 900], [1, 1], 0, 32, 2),                                    # counted
    (32, 8, [2100, 1600], [5, 7], 0, 4, 4),                                    # counted, narrow tiles of 16 rows
    (32, 8, [2100, 1600], [40, 37], 0, 8, 10),                                 # and of 32
    (32, 8, [2100, 1600, 400, 90, 300], [5, 7, 90, 90, 90], 0, 32, 2),         # trees of 20 and 28 rows
    (32, 8, [2100, 1600, 400, 90, 300], [40, 37, 90, 90, 90], 0, 32, 4),       # of 128 and 32, and of 20
    (32, 8, [2300, 2200, 2150], [1, 1, 1], 2048, 32, 3),                       # a prefix, combined in the launch
    (32, 8, [2100 + 10 * i for i in range(12)], [1] * 12, 2048, 32, 12),       # and behind it
    (32, 8, [2100, 2600, 3100], [5, 6, 8], 2048, 32, 3),                       # members of more rows, behind it
    (32, 8, [2100 + 300 * i for i in range(11)], [15] * 11, 2048, 32, 11),     # trees of members, read behind it
])
def test_a_row_that_is_not_a_number_is_written_as_such(dtype, Hq, Hkv, lens, new, shared, tokens, cut):
    w = small_workload(1280, dtype, Hq, Hkv, lens, [n - k for n, k in zip(lens, new)])
    for s in range(1, len(lens) if shared else 0):
        w.share_prefix(s, 0, shared)
    q = np.concatenate([w.q(s) for s in range(w.batch)])
    token, head = int(w.cu_q[1]), 9
    q[token, head] = 0x7fc1
    got, h, pool, opool = launches(w, 3, q=q, blank=(0x1111, 7.0))
    assert (h[3], h[6]) == (tokens, cut) and (h[8] > 0) == (shared > 0), h[:9]
    for out, lse in got:
        o, l = oracle.decode(bits(out), dtype), lse.cpu().numpy()
        assert np.isnan(o[token, head]).all() and np.isnan(l[token, head])
        o[token, head], l[token, head] = 0, 0
        for s in range(w.batch):
            at, n = int(w.cu_q[s]), new[s]
            ro, rl = oracle.attention(opool, pool.shape, 0, w.page_tables[s], w.q(s), Hq, lens[s] - n, lens[s])
            if s == 1:
                ro[0, head], rl[0, head] = 0, 0
            assert np.max(np.abs(o[at:at + n] - ro)) <= O_TOL, s
            assert np.max(np.abs(l[at:at + n] - rl)) <= LSE_TOL, s


# per line: narrow tiles of 32 rows, counted; trees
@pytest.mark.parametrize("others,tokens,cut", [(False, 8, 10), (True, 32, 4)])
def test_a_row_that_is_not_a_number_beside_chunks_without_a_key(others, tokens, cut):
    # the last chunks of both ranges hold no key (a begin below the planned one), whichever of two comes first
    lens, begins = [4100, 4100], [4060, 4060]
    if others:
        lens, begins = beside_others(32, lens, begins)
    w = small_workload(1290, mi.BF16, 32, 8, lens, begins)
    q = np.concatenate([w.q(s) for s in range(w.batch)])
    q[41, 9] = 0x7fc1
    got, h, _, _ = launches(w, 6, q=q, begin=[[700, 1900] + begins[2:]] * 6, blank=(0x1111, 7.0))
    assert (h[3], h[6]) == (tokens, cut), h[:9]
    for out, lse in got:
        o, l = oracle.decode(bits(out), mi.BF16), lse.cpu().numpy()
        assert np.isnan(o[41, 9]).all() and np.isnan(l[41, 9])
        assert np.isnan(o).sum() == 128 and np.isnan(l).sum() == 1


def forks(seed, dtype, Hq, Hkv, shared, own, new):
    """One workload of forks: own[i] tokens of sequence i lie between the prefix and its new[i]."""
    begins = [shared + o for o in own]
    w = small_workload(seed, dtype, Hq, Hkv, [b + n for b, n in zip(begins, new)], begins)
    for s in range(1, len(own)):
        w.share_prefix(s, 0, shared)
    return w


# up to 8 sequences with no more new tokens than those: combined in the launch, prefix items of members
# whose first tokens lie in the same 16 rows; with more new tokens: behind it
@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,new", [
    (32, 8, [1] * 8), (64, 8, [1] * 8), (8, 8, [1] * 7),        # 4, 2, 16 tokens an item
    (64, 8, [2, 1, 1, 1, 1, 1, 1, 0]),                          # an idle sequence, a member of two tokens
    (64, 8, [3, 1, 1, 1, 1, 0, 1]), (64, 8, [1, 3, 1, 1, 0, 0]),    # of three: 24 rows an item, 32; two groups
    (32, 8, [7, 1, 0, 0, 0, 0, 0, 0]),                          # 32 rows, members by a tree
    (32, 8, [2, 1]), (32, 8, [2, 2, 2, 2]), (64, 8, [5, 8, 3]), (8, 8, [17, 30, 2, 1, 9]),
])
def test_small_batches_that_share_a_prefix(dtype, Hq, Hkv, new):
    own = [5, 300, 64, 1200, 17, 40, 700, 2][:len(new)]
    h = check(forks(1300 + len(new), dtype, Hq, Hkv, 1600, own, new))
    assert h[8] > 0, h[:9]


@pytest.mark.parametrize("tiles,chunk", [(44, 4), (46, 6), (64, 6), (68, 8), (130, 12), (140, 12)])
def test_pieces_of_a_prefix_combined_in_the_launch(tiles, chunk):
    # no more than eleven beside the member's own, up to pieces of twelve tiles
    w = forks(1320, mi.BF16, 8, 1, 64 * tiles, [9, 70, 30], [1, 1, 1])
    assert check(w, 2)[7] == chunk


@pytest.mark.parametrize("new", [6, 15])
def test_trees_of_members_in_larger_batches(new):
    # own middle parts of up to five chunks: combined in a tree, read by the launch behind it, or all there
    own = [0, 300, 2700, 40, 1300, 700, 90, 2000, 10, 550, 64]
    w = forks(1330 + new, mi.BF16, 32, 8, 1600, own, [new + i % 2 for i in range(len(own))])
    assert check(w)[8] > 0


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("new,tokens,cut", [(8, 4, 2), (40, 8, 5), (500, 32, 16), (513, 32, 17)])
def test_chunks_without_a_key_and_the_plan_used_again(dtype, new, tokens, cut):
    # a begin so far below the planned one that the last chunks hold no key (counted, of narrow tiles of 16 rows
    # and 32; trees in the kernel without short tiles); then the planned begin on the same plan, whose arrival
    # words have wrapped (whole tiles are of 32 tokens: begins are a multiple of that many)
    w = small_workload(1340 + new, dtype, 32, 8, [4500 + new], [4500])
    low = [[896], [2496], [32]]
    got, h, pool, opool = launches(w, 5, begin=low)
    assert (h[3], h[6]) == (tokens, cut) and h[7] > 0, h[:9]
    rng = mi.rng_for(1340, new)
    rr, hh = rng.integers(0, new, 256), rng.integers(0, 32, 256)
    for (out, lse), (b,) in zip(got, low + [[4500]] * 2):
        ro, rl = oracle.attention(opool, pool.shape, 0, w.page_tables[0], w.q(0), 32, b, b + new, sel_rows=rr,
                                  sel_heads=hh)
        assert np.max(np.abs(oracle.decode(bits(out)[rr, hh], dtype) - ro)) <= O_TOL, b
        assert np.max(np.abs(lse.cpu().numpy()[rr, hh] - rl)) <= LSE_TOL, b


@pytest.mark.parametrize("Hq,Hkv,new,keys", [(32, 8, 500, 5000), (32, 8, 513, 5013), (64, 8, 130, 3000),
                                             (8, 8, 1025, 9000), (16, 8, 700, 2200)])
def test_long_ranges_launch_after_launch(Hq, Hkv, new, keys):
    # the kernel without short tiles: full tiles in trees, the last one counted where it has 16 rows or fewer
    w = small_workload(1350 + new, mi.BF16, Hq, Hkv, [keys], [keys - new])
    h = check(w, rows=512)
    assert h[6] == -(-new // (128 * Hkv // Hq)), h[:9]


@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
def test_the_remainder_round_launch_after_launch(dtype):
    # 560 similar items for 512 slots: the 48 shortest are cut, three chunks each
    w = small_workload(1360, dtype, 8, 1, [1280] * 35, [1024] * 35)
    h = check(w, rows=16)
    assert h[7] == 0 and h[9] > 1 and h[6] == 48, h[:10]


# per line: the tokens of a q tile that the planner takes, on both sides of each bound with 512 workgroup slots
@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,new,cached,tokens", [
    (8, 8, [256], [256], 16), (32, 8, [128], [1024], 4), (32, 8, [128], [1025], 8),  # 18 KV tiles; 19, not to be cut
    (32, 8, [129], [64], 8), (32, 8, [256], [512], 8), (32, 8, [257], [512], 32),    # 256 workgroups, or more
    (64, 8, [3], [6000], 2), (8, 1, [130], [1100], 2), (16, 8, [40], [650], 8),      # 16 rows, cut and uncut
    (64, 8, [8], [8100], 2), (64, 8, [8], [8300], 4),                                # 16 tiles a unit, or more
    (32, 8, [64], [6000], 8), (32, 8, [64], [6200], 32), (32, 8, [20], [17000], 8),  # 24, or more, or few pairs
    (32, 8, [5, 17, 64, 1, 0, 33], [100, 3000, 200, 2000, 70, 0], 8),                # ragged
    (8, 8, [17, 3, 31, 32, 1], [0, 15, 700, 2500, 5], 16),
    (64, 8, [3] * 16, [40 * i for i in range(16)], 2), (64, 8, [3] * 17, [40 * i for i in range(17)], 16),
    # whole tiles sooner done, or narrow ones: one range; ranges beside longer decode rows
    (32, 8, [128], [2300], 8), (32, 8, [128], [2700], 32), (32, 8, [256], [1100], 8), (32, 8, [256], [1500], 32),
    (32, 8, [1] * 8 + [100], [4000] * 8 + [900], 32), (8, 2, [1] * 15 + [800], [500 + 240 * i for i in range(15)] + [0], 32),
    (32, 8, [1] * 4 + [200], [300, 600, 900, 1100, 0], 32), (32, 8, [1] * 4 + [100], [600, 900, 1200, 1500, 0], 8),
    (8, 1, [1] * 4 + [300], [2100, 2300, 2400, 2600, 0], 4),
])
def test_narrow_q_tiles(dtype, Hq, Hkv, new, cached, tokens):
    w = small_workload(1370 + sum(new), dtype, Hq, Hkv, [n + c for n, c in zip(new, cached)], cached)
    assert check(w, 3, rows=0 if max(cached) < 4000 else 64)[3] == tokens


@pytest.mark.parametrize("Hq,Hkv,new,cached,tiles", [
    (32, 8, 32, 16000, 32), (32, 8, 20, 9000, 18), (32, 8, 24, 12000, 20),     # eight pieces; not nine; ten
    (8, 1, 16, 32000, 32), (8, 1, 8, 32000, 16),                               # 16 at most; 32 of few tiles of 16 rows
    (32, 8, 64, 4700, 20), (32, 8, 37, 600, 0),                                # four; uncut
])
def test_pieces_of_narrow_q_tiles(Hq, Hkv, new, cached, tiles):
    w = small_workload(1390 + new, mi.BF16, Hq, Hkv, [new + cached], [cached])
    h = check(w, 3, rows=64)
    assert h[3] < 128 * Hkv // Hq and h[7] == tiles, h[:9]


# batches that may have narrow q tiles and keep whole ones: decode rows counted, 17 to 32 rows and more in trees, wavefronts
# without a row; a shared prefix, whose members are combined behind the launch
@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,new,cached,shared", [
    (16, 8, [16, 3, 9, 14, 1, 16, 11, 16, 8, 2, 16, 16, 12, 16, 0, 16], 4000, 0),     # 2 to 32 rows
    (64, 8, [5, 1, 4, 2, 8, 5, 7, 3, 5, 6, 1, 5, 5, 5, 5, 5], 4000, 0),               # 8 to 64
    (8, 8, [40, 60, 96, 17, 33, 128, 1, 16], 6000, 0),                                # one to four wavefronts
    (32, 8, [1] * 8 + [100], 1100, 1024), (32, 8, [5, 4, 1, 8, 3], 1100, 1024),       # 32 rows of the prefix; 84
    (64, 8, [1, 1, 1, 1, 30], 1100, 1024), (8, 8, [17, 8, 1, 5, 200], 1100, 1024), (16, 8, [1] * 9 + [100], 1100, 1024),
])
def test_whole_tiles_where_narrow_ones_are_possible(dtype, Hq, Hkv, new, cached, shared):
    cached = [cached + 70 * i for i in range(len(new))]
    w = small_workload(1500 + sum(new), dtype, Hq, Hkv, [n + c for n, c in zip(new, cached)], cached)
    for s in range(1, len(new) if shared else 0):
        w.share_prefix(s, 0, shared)
    assert sum(new) * Hq <= 32 * 256
    h = check(w, 3, rows=32)
    assert h[3] == 128 * Hkv // Hq and h[6] >= len(new) - 2 and (h[8] > 0) == (shared > 0), h[:9]


# a plan made ahead: per line the tile's tokens, and whether it is cut.  The ranges step over the end of a 64-key tile, so
# that a last piece (a last KV tile) holds no key at first and some later
@pytest.mark.parametrize("dtype", [mi.BF16, mi.F16])
@pytest.mark.parametrize("Hq,Hkv,new,cached,tokens,cut", [
    (32, 8, [9], [1020], 4, True), (32, 8, [40], [250], 4, False),          # 16 rows
    (32, 8, [128], [2040], 8, True), (32, 8, [200], [500], 8, False),       # 32
    (64, 8, [3, 8, 1, 5], [700, 1275, 2000, 60], 2, True),                  # ragged
])
def test_narrow_q_tiles_planned_ahead(dtype, Hq, Hkv, new, cached, tokens, cut):
    ahead, B, tq = 70, len(new), sum(new)
    final = [n + c + ahead for n, c in zip(new, cached)]
    w = small_workload(1600 + tq, dtype, Hq, Hkv, final, cached)
    pool = DevPool(w)
    pool.t.fill_(0x7fc1)
    opool = np.full(pool.elems, 0x7fc1, dtype=np.uint16)
    fill_both(w, pool, opool)
    cu_q = dev(np.concatenate([[0], np.cumsum(new)]).astype(np.int32))
    db = DevBatch(w)
    size = mc.mc_attn_workspace_size(B, tq, Hq, Hkv)
    ws = torch.full((size,), 0xff, dtype=torch.uint8, device=DEV)
    mc.mc_attn_plan_ahead(pool.desc, Hq, B, tq, cu_q, db.begin, db.page_table, db.cu_pages, ahead, ws, size)
    mc.mc_attn_plan_check(ws)
    h = ws[:64].view(torch.int32).cpu().numpy()
    assert h[3] == tokens and (h[7] > 0) == cut, h[:9]
    q = np.concatenate([w.q(s)[:n] for s, n in enumerate(new)])
    for step in (0, 1, 27, 63, 64, ahead):
        begin = [c + step for c in cached]
        out = torch.full((tq, Hq, 128), 0x7fc1, dtype=torch.int16, device=DEV)
        lse = torch.full((tq, Hq), float("nan"), dtype=torch.float32, device=DEV)
        mc.mc_prefix_prefill_attn(pool.desc, 0, dev(q), Hq, B, tq, cu_q, dev(np.array(begin, np.int32)), db.page_table,
                                  db.cu_pages, 0.0, out, lse, ws, size)
        torch.cuda.synchronize()
        at = 0
        for s, (n, b) in enumerate(zip(new, begin)):
            ro, rl = oracle.attention(opool, pool.shape, 0, w.page_tables[s], q[at:at + n], Hq, b, b + n)
            assert np.max(np.abs(oracle.decode(bits(out[at:at + n]), dtype) - ro)) <= O_TOL, (step, s)
            assert np.max(np.abs(lse[at:at + n].cpu().numpy() - rl)) <= LSE_TOL, (step, s)
            at += n
