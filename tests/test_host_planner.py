"""CPU-only checks of the C-ABI library: it loads, exports what the header declares, validates
its inputs, and the planner's work items cover every decode token and every visible prefill
(row, key) pair exactly once."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2508_15919_amd import binding as hb
from paper_2508_15919_amd import synth
from paper_2508_15919_amd.synth import DECODE, PREFILL

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(hb.LIB_PATH):
        from paper_2508_15919_amd import build
        build.build()
    return hb.load()


def test_library_exports_every_declared_symbol(lib):
    header = open(os.path.join(ROOT, "include", "hfxattn.h")).read()
    declared = set(re.findall(r"\b(hfx_[a-z_]+)\s*\(", header))
    assert declared == set(hb.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name
    assert hb.hfx_status_string(0) == "ok" and "page id" in hb.hfx_status_string(hb.HFX_ERR_PAGE_ID)
    assert hb.hfx_version()[1] >= 1


def fill(b, scale=0.0):
    shape = hb.make_shape(b.num_q_heads, b.num_kv_heads, b.head_dim, b.num_pages, scale)
    hbts, dbts, wbts = hb.hfx_batch_desc_sizes(shape, b.kind, b.q_len, b.ctx_len)
    host = np.zeros(hbts, np.uint8)
    hb.hfx_fill_batch_desc(shape, b.kind, b.q_len, b.ctx_len, b.bt_indptr, b.bt_pages, host)
    d = hb.parse_desc(host)
    assert d["header"].total_bytes == hbts == dbts and d["header"].workspace_bytes == wbts
    return d


def lengths_only(Hq, Hkv, D, kind, q_len, ctx_len):
    """A step with a block table but a one-page dummy pool (the planner never reads the pool)."""
    kind, q_len, ctx_len = (np.asarray(a, np.int32) for a in (kind, q_len, ctx_len))
    npg = (ctx_len.astype(np.int64) + 15) // 16
    indptr = np.zeros(len(kind) + 1, np.int32)
    indptr[1:] = np.cumsum(npg)
    pages = np.arange(int(npg.sum()), dtype=np.int32)[::-1].copy()
    return synth.StepBatch(Hq, Hkv, D, max(1, int(npg.sum())), kind, q_len, ctx_len, indptr, pages,
                           np.zeros((int(q_len.sum()), Hq, D), np.uint16), np.zeros((1, Hkv, 2, 16 * D), np.uint16))


def check_class_order(b, items):
    """Queue of a prefill-dominated step: 8 position classes (position mod 8), one per die.

    The prefill items that read the same piece of the keys of one (request, kv-head), i.e. the same
    split index over row tiles and head blocks, form a unit; the planner may cut a unit into sub-units
    of consecutive row tiles.  A decode item is a unit of its own.  Checked here: the items of one
    (unit, row tile) share a home class; class loads differ by no more than the largest total a unit
    has in one class; the list of a class (its own items in position order, then what other classes
    took off its tail) is in descending cost; a class's positions hold foreign items only behind its
    own."""
    G = b.num_q_heads // b.num_kv_heads
    n = len(items)
    cost, home_of = items["cost"].astype(np.int64), items["home"]
    unit = {}
    by_tile = {}
    for i, it in enumerate(items):
        if it["type"] == 1:
            by_tile.setdefault((int(it["req"]), int(it["row0"]), int(it["h0"])), []).append((int(it["kb"]), i))
        else:
            unit[i] = ("d", i)
    for (req, row0, h0), lst in by_tile.items():
        for s, (_, i) in enumerate(sorted(lst)):
            unit[i] = ("p", req, h0 // G, s)
    home = {}
    for i, it in enumerate(items):
        assert 0 <= int(home_of[i]) < 8
        k = unit[i] + (int(it["row0"]),)
        assert home.setdefault(k, int(home_of[i])) == int(home_of[i]), "one home per unit and row tile"
    loads, unit_total = [], {}
    for c in range(8):
        seq = list(range(c, n, 8))
        own = [i for i in seq if int(home_of[i]) == c]
        assert seq[:len(own)] == own, "foreign items only behind the class's own"
        taken = [i for i in range(n) if int(home_of[i]) == c and i % 8 != c]
        full = own + taken[::-1]                    # taken off the tail, last first
        loads.append(int(cost[full].sum()))
        assert np.all(np.diff(cost[full]) <= 0), "a class's list is in descending cost"
        for i in full:
            unit_total[(c, unit[i])] = unit_total.get((c, unit[i]), 0) + int(cost[i])
    assert max(loads) - min(loads) <= max(unit_total.values()), (loads, max(unit_total.values()))


def check_coverage(b, d):
    h, items, reqs, groups = d["header"], d["items"], d["reqs"], d["groups"]
    Hq, Hkv = b.num_q_heads, b.num_kv_heads
    G = Hq // Hkv
    assert h.n_items == len(items) == h.n_decode_items + h.n_prefill_items
    ty = items["type"]
    n_dec, n_pre = int((ty == 0).sum()), int((ty == 1).sum())
    if np.all(items["home"] >= 0):
        assert h.queue_classes == 8
        check_class_order(b, items)
    else:
        assert np.all(items["home"] == -1) and h.queue_classes == 1
        for k in (0, 1):
            assert np.all(np.diff(items["cost"][ty == k]) <= 0), "each kind in descending modelled cost"
        if n_pre == 0 or n_dec == 0 or np.all(np.diff(items["cost"]) <= 0):
            pass                                   # one kind only, or plain descending order
        else:
            # decode-dominated mixed step: over the first two rounds of 512 positions the prefill items sit
            # at the positions of the workgroups of the first ceil(n_pre / 4) CUs (position mod 256), at
            # most 128 of them; behind that, blocks of 256, decode first, as long as both kinds last
            pair_cus = min((n_pre + 3) // 4, 128)
            want = []
            for pos in range(min(1024, n_dec + n_pre)):
                slot = (pos % 512) % 256 < pair_cus
                if (slot and n_pre) or not n_dec:
                    want.append(1); n_pre -= 1
                else:
                    want.append(0); n_dec -= 1
            while n_dec or n_pre:
                k = min(256, n_dec); want += [0] * k; n_dec -= k
                k = min(256, n_pre); want += [1] * k; n_pre -= k
            assert ty.tolist() == want
    assert np.all(d["ctrl"] == 0)
    # stored block table: exactly the needed pages, in order
    for r in range(b.num_requests):
        n = int(reqs["n_pages"][r])
        assert n == (int(b.ctx_len[r]) + 15) // 16
        assert np.array_equal(d["bt"][reqs["bt_start"][r]:reqs["bt_start"][r] + n],
                              b.bt_pages[b.bt_indptr[r]:b.bt_indptr[r] + n])
        # stored quad-aligned, with the last page repeated behind it
        m = int(reqs["bt_len"][r])
        assert reqs["bt_start"][r] % 4 == 0 and m == (n + 3) // 4 * 4 + 16
        assert np.all(d["bt"][reqs["bt_start"][r] + n:reqs["bt_start"][r] + m] == b.bt_pages[b.bt_indptr[r] + n - 1])
    qi = b.q_indptr()
    assert np.array_equal(reqs["q_start"], qi[:-1])
    # append runs: every new token exactly once, in its page and slot, never across a page boundary
    where = {}
    for row0, n, page, slot0 in d["runs"]:
        assert 1 <= n <= 16 and 0 <= slot0 and slot0 + n <= 16
        for k in range(n):
            assert row0 + k not in where
            where[row0 + k] = (page, slot0 + k)
    assert len(where) == h.total_q
    for r in range(b.num_requests):
        for i in range(int(b.q_len[r])):
            t = int(b.ctx_len[r]) - int(b.q_len[r]) + i
            assert where[qi[r] + i] == (int(b.bt_pages[b.bt_indptr[r] + t // 16]), t % 16)
    slot_owner = np.zeros(max(1, h.n_partial_rows), np.int32)
    group_count = np.zeros(max(1, h.n_groups), np.int32)
    for r in range(b.num_requests):
        mine = items[items["req"] == r]
        c, ql = int(b.ctx_len[r]), int(b.q_len[r])
        if b.kind[r] == DECODE:
            assert np.all(mine["type"] == 0)
            cover = np.zeros((Hkv, (c + 15) // 16), np.int32)
            for it in mine:
                assert it["hn"] in (1, 2, 4) and 0 <= it["kb"] < it["ke"] <= (c + 15) // 16 and it["kb"] % 2 == 0
                cover[it["h0"]:it["h0"] + it["hn"], it["kb"]:it["ke"]] += 1
            assert np.all(cover == 1)
        else:
            assert np.all(mine["type"] == 1)
            p = c - ql
            cover = np.zeros((Hq, ql, c), np.int16)
            for it in mine:
                assert it["hn"] in (1, 2, 4) and it["nrows"] == 32 * 4 // it["hn"] and it["kb"] % 64 == 0
                assert it["h0"] // G == (it["h0"] + it["hn"] - 1) // G, "an item stays inside one kv group"
                r1 = min(ql, it["row0"] + it["nrows"])
                assert it["ke"] <= p + r1
                cover[it["h0"]:it["h0"] + it["hn"], it["row0"]:r1, it["kb"]:it["ke"]] += 1
                # modelled cost: a workgroup's time, 4*D flops per key for each of its 128 rows at 2000 flops/ns (1400
                # where heads are 64 wide) however many of the rows exist, plus a fixed 3000 ns
                rate = 1400.0 if b.head_dim == 64 else 2000.0
                assert it["cost"] == int(4.0 * b.head_dim * 128 * int(it["ke"] - it["kb"]) / rate + 3000.0)
            visible = (np.arange(c)[None, :] <= (p + np.arange(ql))[:, None])
            assert np.all(cover[:, visible] == 1), "every visible pair exactly once"
        for f in ("kind", "q_len", "ctx_len", "q_start", "bt_start", "n_pages", "bt_len"):
            assert np.all(mine["rq_" + f] == reqs[f][r]), "an item carries a copy of its request record"
        for it in mine:
            if it["group"] >= 0:
                g = groups[it["group"]]
                rows = g["rows_per_split"]
                assert rows == (it["hn"] * G if it["type"] == 0 else 128)
                s = (it["slot_row"] - g["base_row"]) // rows
                assert 0 <= s < g["nsplit"] and it["slot_row"] == g["base_row"] + s * rows
                slot_owner[it["slot_row"]:it["slot_row"] + rows] += 1
                group_count[it["group"]] += 1
            else:
                assert it["slot_row"] == -1
    if h.n_groups:
        assert np.array_equal(group_count[:h.n_groups], groups["nsplit"]) and np.all(groups["nsplit"] > 1)
        # merge units: every row of every group belongs to exactly one unit
        seen = [np.zeros(g["rows_per_split"], np.int32) for g in groups]
        for gi, chunk in d["units"]:
            per = 1 if groups[gi]["nsplit"] > 8 else 8
            seen[gi][chunk * per:(chunk + 1) * per] += 1
        assert all(np.all(x == 1) for x in seen) and h.n_units == len(d["units"])
        assert np.all(slot_owner[:h.n_partial_rows] == 1)
        assert h.workspace_bytes >= h.ws_off_ml + 8 * h.n_partial_rows >= 4 * h.n_partial_rows * b.head_dim
    else:
        assert h.workspace_bytes == 0


@pytest.mark.parametrize("idx,scale", [(1, 1.0), (2, 0.25), (3, 0.1), (4, 0.12), (5, 0.05)])
def test_planner_covers_scaled_configs(lib, idx, scale):
    b = synth.config(idx, scale)
    check_coverage(b, fill(b))


@pytest.mark.parametrize("Hq,Hkv,D,n,lo,hi,dealt", [
    (32, 8, 128, 165, 300, 6000, True), (32, 4, 64, 288, 300, 9000, True), (8, 8, 128, 400, 200, 4000, True),
    (32, 8, 128, 288, 300, 9000, False),       # a workgroup would stream for more than 600 us
    (32, 8, 64, 288, 4000, 4011, False),       # equal contexts: whole, or in more pieces than are dealt
    (32, 8, 128, 600, 2000, 2001, False)])     # more contexts than are dealt
def test_decodes_alone_are_dealt_whole_rounds(lib, Hq, Hkv, D, n, lo, hi, dealt):
    """Decode pieces of a step without prefills are lengthened until the two dealt rounds hold them all, where these are then filled."""
    c = np.random.default_rng(5).integers(lo, hi, n)
    b = lengths_only(Hq, Hkv, D, [DECODE] * n, [1] * n, c)
    d = fill(b)
    check_coverage(b, d)
    items = d["header"].n_items
    assert 2 * 1024 // 3 <= items <= 1024 if dealt else items > 1024


def test_planner_covers_full_size_lengths(lib):
    # full-size length mixes without materialising pools
    g = np.random.default_rng(0)
    c3 = g.integers(2048, 16385, 256)
    b = lengths_only(32, 8, 128, [DECODE] * 256, [1] * 256, c3)
    d = fill(b)
    check_coverage(b, d)
    assert d["header"].n_items >= 4 * 512, "enough items to balance 512 resident workgroups"
    b = lengths_only(8, 1, 128, [DECODE] * 4 + [PREFILL], [1] * 4 + [4096], [131072, 32768, 70001, 99999, 8192])
    d = fill(b)
    check_coverage(b, d)
    assert d["groups"]["nsplit"].max() <= 64


def test_queue_per_die_and_whole_rounds(lib):
    """Long prefill-dominated steps of four to eight items per workgroup get one queue class per die;
    steps of few prefill items per workgroup are cut so that the prefill items fill whole rounds of 512."""
    # four prompts' chunks of 2048 tokens at different depths plus 32 decodes (the prefill-heavy mixed shape)
    g = np.random.default_rng(1)
    dec = g.integers(512, 4097, 32).tolist()
    b = lengths_only(32, 8, 128, [PREFILL] * 4 + [DECODE] * 32, [2048] * 4 + [1] * 32,
                     [2048, 6144, 10240, 14336] + dec)
    d = fill(b)
    assert d["header"].queue_classes == 8 and 3 * 512 <= d["header"].n_items <= 8 * 512
    check_coverage(b, d)
    # one long prompt on one kv-head, with and without decodes beside it
    b = lengths_only(8, 1, 128, [PREFILL] + [DECODE] * 16, [4096] + [1] * 16, [65536] + [90000] * 16)
    d = fill(b)
    assert d["header"].queue_classes == 8
    check_coverage(b, d)
    b = lengths_only(8, 1, 128, [PREFILL], [4096], [65536])
    d = fill(b)
    assert d["header"].n_prefill_items == 1024 and d["header"].queue_classes == 1
    check_coverage(b, d)
    # many short prompts, a decode-only step and a small step keep the single queue
    b = lengths_only(32, 8, 128, [PREFILL] * 256, [256] * 256, [256] * 256)
    assert fill(b)["header"].queue_classes == 1
    b = lengths_only(32, 8, 128, [DECODE] * 64, [1] * 64, [4096] * 64)
    assert fill(b)["header"].queue_classes == 1
    b = lengths_only(32, 8, 128, [PREFILL] * 2, [512] * 2, [512, 2048])
    assert fill(b)["header"].queue_classes == 1


@pytest.mark.parametrize("Hq,Hkv,D,chunks", [
    (32, 8, 128, [(9000, 0)]), (32, 8, 128, [(2048, 0), (2048, 256), (2048, 512), (2148, 100)]), (24, 8, 128, [(6000, 144), (5743, 3040)]),
    (32, 8, 64, [(7993, 1035), (4771, 142), (706, 1961)]), (32, 4, 64, [(6336, 8000), (6214, 9000)])])
def test_one_queue_where_the_dies_would_end_apart(lib, Hq, Hkv, D, chunks):
    """Four to eight rounds of prompt tiles in less than 800 us, or of 64-wide heads, are done sooner from one queue."""
    h = fill(lengths_only(Hq, Hkv, D, [PREFILL] * len(chunks), [q for q, _ in chunks], [q + p for q, p in chunks]))["header"]
    assert 4 * 512 <= h.n_items <= 8 * 512 and h.queue_classes == 1


@pytest.mark.parametrize("Hq,Hkv,D,n,q,prior,classes", [
    (24, 8, 128, 134, 2, 22937, 8), (24, 8, 128, 97, 1, 12208, 8), (12, 4, 128, 273, 4, 5267, 8), (24, 8, 128, 68, 4, 2396, 8), (24, 8, 128, 60, 1, 30000, 1),
    (24, 8, 128, 99, 4, 2091, 1), (32, 8, 128, 200, 1, 30000, 1), (32, 4, 128, 180, 33, 1785, 1), (24, 8, 64, 68, 4, 5198, 1),
    (24, 8, 64, 105, 64, 16000, 8), (32, 4, 64, 200, 64, 12000, 8), (32, 8, 128, 260, 32, 5500, 1)])
def test_queue_per_die_where_few_row_tiles_read_the_same_keys(lib, Hq, Hkv, D, n, q, prior, classes):
    """Chunks of a few rows behind long contexts, several head blocks to a kv-head: one die per kv-head's keys from three rounds
    on.  Not with fewer or shorter items, where no two items share keys, or where the tiles are bound by the matrix cores, unless
    there are a great many keys."""
    b = lengths_only(Hq, Hkv, D, [PREFILL] * n, [q] * n, [q + prior] * n)
    d = fill(b)
    assert d["header"].queue_classes == classes
    if classes > 1:
        check_class_order(b, d["items"])


@pytest.mark.parametrize("Hq,Hkv,n,longer,items,per_die", [
    (32, 8, 87, 0, 1392, False), (32, 8, 88, 0, 1408, True), (8, 8, 44, 0, 1056, False), (16, 16, 87, 0, 4176, True), (32, 8, 80, 400, 1384, False), (32, 8, 89, 400, 1528, False),
    (32, 8, 90, 400, 1544, True), (16, 4, 160, 0, 1280, True), (16, 4, 129, 0, 1032, True), (8, 2, 260, 0, 1040, True)])
def test_queue_per_die_starts_where_there_is_something_behind_the_dealt_items(lib, Hq, Hkv, n, longer, items, per_die):
    """Prompts of two row tiles or more, alone (a share of more than 1.5 of the longest item) or beside a longer one (less): with a multiple of 8 kv-heads from 2.75 and 3
    rounds on, because dealt items of a stream meet on a die as they are; with fewer kv-heads whenever items are left for the counters."""
    q = [64 if Hq > Hkv else 257 if Hq == 8 else 300] * n + ([longer] if longer else [])
    b = lengths_only(Hq, Hkv, 128, [PREFILL] * len(q), q, q)
    d = fill(b)
    assert d["header"].n_items == items
    assert (d["queue"] is not None) == per_die
    check_coverage(b, d)


@pytest.mark.parametrize("D,n,q,per_die", [(64, 8, 1536, False), (64, 19, 800, False), (64, 20, 800, True), (128, 8, 1536, True), (128, 19, 800, True)])
def test_queue_per_die_of_64_wide_heads_needs_more_streams(lib, D, n, q, per_die):
    """Prompts on 4 kv-heads: 32 streams are enough where heads are 128 wide, 80 are needed where they are 64 wide."""
    b = lengths_only(16, 4, D, [PREFILL] * n, [q] * n, [q] * n)
    d = fill(b)
    assert d["header"].n_items > 1408 and (d["queue"] is not None) == per_die
    check_coverage(b, d)


@pytest.mark.parametrize("Hq,Hkv,D,n,lo,hi,decodes,per_die", [
    (32, 8, 128, 64, 20, 700, 0, True), (32, 4, 64, 60, 100, 900, 20, True), (24, 8, 128, 20, 500, 3000, 0, True), (8, 8, 128, 120, 50, 600, 5, True),
    (8, 1, 128, 170, 20, 500, 0, True), (32, 8, 128, 4, 1500, 2500, 0, True), (32, 8, 128, 3, 2500, 2500, 0, False), (8, 1, 128, 25, 1000, 2000, 0, False),
    (32, 8, 128, 100, 1, 32, 0, False), (32, 8, 128, 24, 30, 1200, 0, True), (8, 8, 128, 130, 50, 600, 400, False)])
def test_order_of_a_queue_per_die(lib, Hq, Hkv, D, n, lo, hi, decodes, per_die):
    """Steps of many prompts list the order in which their items are taken: every item once, position p for die p % 8 up to a
    multiple of 8 behind which little is left for all; the tiles of a (request, kv-head) on as few dies as its share of the step allows, one behind the
    other, and the dies about equally loaded.  Not where few prompts share the chip, items are few, no two items share keys or decodes weigh much."""
    g = np.random.default_rng(n)
    q = g.integers(lo, hi + 1, n).tolist()
    b = lengths_only(Hq, Hkv, D, [PREFILL] * n + [DECODE] * decodes, q + [1] * decodes, q + g.integers(100, 2000, decodes).tolist())
    d = fill(b)
    h, items, queue = d["header"], d["items"], d["queue"]
    assert (queue is not None) == per_die and (h.die_items > 0) == per_die
    assert h.queue_classes == 1 and np.all(items["home"] == -1)
    check_coverage(b, d)
    if not per_die:
        return
    assert np.array_equal(np.sort(queue), np.arange(h.n_items))
    cost = items["cost"].astype(np.float64)[queue]
    assert h.die_items % 8 == 0 and h.die_items <= h.n_items
    assert cost[h.die_items:].sum() <= 0.07 * cost.sum() + 8 * cost.max()
    die = np.arange(h.n_items) % 8
    load = np.array([cost[die == c].sum() for c in range(8)])
    G = Hq // Hkv
    unit = np.where(items["type"] == 1, items["req"] * Hkv + items["h0"] // G, -1 - np.arange(h.n_items))[queue]
    share = cost.sum() / 256                    # of a die's 32nd part
    largest = max(cost[unit == u].sum() for u in np.unique(unit))
    assert load.max() - load.min() <= min(largest, share) + 2 * cost.max()
    front = 8 * min(int((die[:h.die_items] == c).sum()) for c in range(8))
    for u in np.unique(unit[unit >= 0])[:40]:
        at = np.flatnonzero(unit[:front] == u)
        pieces = int(np.ceil(1.1 * cost[unit == u].sum() / share))
        runs = sum(int(np.count_nonzero(np.diff(at[at % 8 == c]) != 8) + 1) for c in np.unique(at % 8)) if len(at) else 0
        # (where a die's list ends early, items from the end of a longer one stand in for it)
        assert runs <= pieces + 8, (u, runs, pieces)


@pytest.mark.parametrize("Hq,Hkv,D", [(32, 8, 128), (8, 1, 128), (24, 8, 128), (32, 4, 64), (16, 16, 128)])
@pytest.mark.parametrize("q,prior", [(5, 20000), (100, 8000), (777, 0), (500, 3000), (1500, 0), (992, 2000), (4096, 0)])
def test_cut_of_a_single_prompt(lib, Hq, Hkv, D, q, prior):
    """The cut of a prompt's row tiles along the keys (whole where tiles fill the CUs, pieces where there are
    fewer): every pair covered once, and bounded partials."""
    b = lengths_only(Hq, Hkv, D, [PREFILL, PREFILL], [q, 40], [q + prior, 40])
    d = fill(b)
    check_coverage(b, d)
    assert d["header"].deal_balanced == 1 and d["header"].workspace_bytes <= 48 << 20


def workspace_of_cut_by_pairs(Hq, Hkv, D, kind, q_len, ctx_len, decode_rows):
    """Workspace of a step whose prefill tiles are cut by the (row, key) pairs they work on: pieces of half a workgroup's
    share of the step (0.6 of one where decodes outweigh prefills), at least 32 us, in whole rounds of 512."""
    G = Hq // Hkv
    hpw = 4 if G % 4 == 0 else 2 if G % 2 == 0 else 1
    rows_wg, mult = 128 // hpw, Hkv * (G // hpw)
    pre = kind == PREFILL
    q, c = q_len[pre].astype(np.int64), ctx_len[pre].astype(np.int64)
    dec_ns = float(ctx_len[~pre].sum()) * Hkv * D * 4 / 12.0
    pre_ns = 4.0 * D * Hq * float((q * (c - q) + q * (q + 1) // 2).sum()) / 2000.0
    n_rt = -(-q // rows_wg)
    p = np.repeat(c - q, n_rt)
    r0 = (np.arange(n_rt.sum()) - np.repeat(np.cumsum(n_rt) - n_rt, n_rt)) * rows_wg
    r1 = np.minimum(np.repeat(q, n_rt), r0 + rows_wg)
    ns = 4.0 * D * hpw * ((r1 - r0) * (p + 1) + (r0 + r1 - 1) * (r1 - r0) // 2) / 2000.0

    def pieces(cap):
        tiles = (p + r1 + 63) // 64
        n = np.clip(np.ceil(ns / cap), 1, 64).astype(np.int64)
        n = -(-tiles // np.maximum(-(-tiles // n), 4))
        return int(n.sum()) * mult, int(n[n > 1].sum()) * mult

    cap = max((dec_ns + pre_ns) / 1024, 32000.0)
    if dec_ns > pre_ns:
        cap = max(cap, 0.6 * (dec_ns + pre_ns) / 512)
    whole = pieces(cap)[0] // 512 * 512
    if pre_ns > dec_ns and 512 <= whole < pieces(cap)[0] < 6 * 512 and pieces(1.5 * cap)[0] <= whole:
        lo, cap = cap, 1.5 * cap
        for _ in range(12):
            mid = 0.5 * (lo + cap)
            if pieces(mid)[0] <= whole:
                cap = mid
            else:
                lo = mid
    rows = decode_rows + 128 * pieces(cap)[1]
    return -(-rows * D * 4 // 256) * 256 + -(-rows * 8 // 256) * 256


def check_workspace(Hq, Hkv, D, kind, q_len, ctx_len):
    kind, q_len, ctx_len = (np.asarray(a, np.int32) for a in (kind, q_len, ctx_len))
    shape = hb.make_shape(Hq, Hkv, D, 1 << 30)
    ws = hb.hfx_batch_desc_sizes(shape, kind, q_len, ctx_len)[2]
    if ws <= FIXED_WORKSPACE:
        return ws
    d = fill(lengths_only(Hq, Hkv, D, kind, q_len, ctx_len))
    decode_rows = int(sum(g["nsplit"] * g["rows_per_split"] for g in d["groups"] if g["type"] == 0))
    assert ws <= workspace_of_cut_by_pairs(Hq, Hkv, D, kind, q_len, ctx_len, decode_rows)
    return ws


FIXED_WORKSPACE = 64 << 20


@pytest.mark.parametrize("Hq,Hkv,D,chunks", [
    (32, 8, 128, [(32, 1, 64000)]), (8, 1, 128, [(64, 2, 64000)]), (32, 8, 128, [(40, 40, 20000), (4, 2048, 2048)]),
    (8, 8, 128, [(77, 2, 13424)]), (2, 2, 128, [(272, 2, 9000)]), (12, 4, 128, [(17, 300, 40000)]), (24, 8, 128, [(89, 4, 6000)])])
def test_steps_of_few_row_chunks_fit_the_fixed_workspace(lib, Hq, Hkv, D, chunks):
    """Tiles of few rows are cut like full ones, each piece with as many partial rows: a caller of the entry point with the
    fixed workspace must not be refused for it."""
    q = [n_q for n, n_q, _ in chunks for _ in range(n)]
    c = [n_c for n, _, n_c in chunks for _ in range(n)]
    assert check_workspace(Hq, Hkv, D, [PREFILL] * len(q), q, c) <= FIXED_WORKSPACE
    check_coverage_of_groups(fill(lengths_only(Hq, Hkv, D, [PREFILL] * len(q), q, c)))


@pytest.mark.parametrize("Hq,Hkv,D,chunks", [
    (8, 1, 128, [(2048, 564)] * 17 + [(2048, 43732)] * 3 + [(2, 3543)]),
    (16, 1, 128, [(3612, 19), (5891, 20), (774, 869), (1440, 517), (1125, 43), (3461, 331), (1151, 2), (2048, 50257), (2048, 50257),
                  (6774, 105), (6948, 16), (756, 9729)])])
def test_long_steps_are_cut_only_where_it_gains(lib, Hq, Hkv, D, chunks):
    """Long steps of a few long tiles and many short ones, where whole tiles are as good as pieces: no workspace is taken."""
    q = [n for n, _ in chunks]
    assert check_workspace(Hq, Hkv, D, [PREFILL] * len(q), q, [n + p for n, p in chunks]) == 0


@pytest.mark.parametrize("Hq,Hkv,D", [(32, 8, 128), (8, 1, 128), (8, 2, 64), (24, 8, 128), (16, 16, 128), (12, 4, 64)])
@pytest.mark.parametrize("n,lo,hi,prompt", [(1, 1, 1, 0), (1, 31, 33, 0), (1, 130000, 131000, 0), (3, 37, 129, 32), (5, 1, 2500, 0), (31, 200, 900, 0),
                                            (64, 1000, 1000, 0), (65, 3, 5000, 0), (128, 40, 400, 0), (129, 40, 400, 0), (6, 100, 900, 40), (6, 500, 5000, 777),
                                            (512, 16, 17, 0), (600, 1, 40, 0), (64, 16, 8192, 0)])
def test_decodes_of_steps_that_fit_the_chip_at_once(lib, Hq, Hkv, D, n, lo, hi, prompt):
    """Decode items of one, two or four kv-heads and pieces of any number of page pairs: everything covered once; alone, decodes that
    can be on the chip at once are, and have nothing to merge where their contexts are short."""
    rng = np.random.default_rng(n + hi)
    c = rng.integers(lo, hi + 1, n).tolist()
    b = lengths_only(Hq, Hkv, D, [DECODE] * n + [PREFILL] * bool(prompt), [1] * n + [prompt] * bool(prompt), c + [prompt] * bool(prompt))
    d = fill(b)
    check_coverage(b, d)
    heads = next((h for h in (1, 2) if Hkv % h == 0 and n * (Hkv // h) <= 512), 0)
    if heads and not prompt:
        share = sum(c) * Hkv // heads // 512               # tokens of an item's heads, spread evenly over 512 items
        if max(c) <= 3 * max(256 // heads, share) // 32 * 32:        # no context is far longer than that
            assert d["header"].n_items <= 512 and np.all(d["items"]["hn"] == heads)
        if max(c) <= 1024 // heads and share * heads <= 512:
            assert d["header"].n_groups == 0 and d["header"].workspace_bytes == 0


def decode_items_by_time(b):
    """Decode items where pieces go by time alone: four kv-heads an item, whole rounds of 512 pieces of at least 32 us at 12 bytes a ns."""
    heads = 4 if b.num_kv_heads % 4 == 0 else 2 if b.num_kv_heads % 2 == 0 else 1
    ctx = b.ctx_len[b.kind == DECODE].astype(np.int64)
    ns = float(ctx.sum()) * b.num_kv_heads * b.head_dim * 4 / 12
    rounds = min(max(ns // (512 * 32000), 1), 4)
    tokens = max(int(max(ns / (512 * rounds), 32000) / (heads * b.head_dim * 4 / 12)), 128)
    pairs, piece = (ctx + 31) // 32, (tokens + 31) // 32
    piece = np.maximum(piece, (pairs + 63) // 64)
    return int(((pairs + piece - 1) // piece).sum()) * (b.num_kv_heads // heads)


def mixed_step_is_dealt_whole(b):
    """Whether the decode pieces of a step that decodes outweigh were lengthened until two rounds of 512 hold all items: where
    pieces by time would make one to two times as many, and only there."""
    d = fill(b)
    h = d["header"]
    check_coverage(b, d)
    assert h.deal_balanced == 0 and h.n_prefill_items < 512
    by_time = decode_items_by_time(b) + h.n_prefill_items
    lengthened = 1024 < by_time <= 2048
    assert h.n_items <= 1024 if lengthened else h.n_items == by_time, (h.n_items, by_time)
    return lengthened


@pytest.mark.parametrize("seed", range(6))
def test_mixed_steps_of_a_little_more_than_two_rounds_are_dealt_whole(lib, seed):
    """Decodes that outweigh the prefills beside them: a step of up to twice the 1024 items of two rounds has longer decode pieces, one of more
    has not, and everything is covered once."""
    rng = np.random.default_rng(seed)
    dealt = 0
    for _ in range(8):
        n = int(rng.integers(30, 60))
        c = rng.integers(100, 5000, n).tolist()
        q = [int(x) for x in rng.integers(30, 400, rng.integers(1, 4))]
        p = [int(x) for x in rng.integers(0, 1000, len(q))]
        b = lengths_only(32, 8, 128, [DECODE] * n + [PREFILL] * len(q), [1] * n + q, c + [x + y for x, y in zip(q, p)])
        dealt += mixed_step_is_dealt_whole(b)
    assert dealt > 0


@pytest.mark.parametrize("Hq,Hkv,D,n,lo,hi,chunks,dealt", [
    (32, 8, 128, 64, 100, 8192, [(512, 0), (512, 1536)], True),                     # 1.1 to 1.9 times 1024 items by time
    (8, 8, 128, 96, 500, 10000, [(20, 80), (150, 117)], True), (32, 8, 64, 118, 2500, 3900, [(566, 0), (96, 0), (266, 628)], True),
    (16, 4, 128, 83, 800, 21000, [(76, 35), (187, 0), (30, 0)], True), (16, 16, 128, 13, 7300, 10200, [(185, 0), (103, 587)], True),
    (32, 8, 128, 200, 1000, 12000, [(134, 46), (668, 661)], False)])                # 2.4
def test_mixed_steps_dealt_whole_on_other_layouts(lib, Hq, Hkv, D, n, lo, hi, chunks, dealt):
    c = np.rint(np.exp(np.random.default_rng(n).uniform(np.log(lo), np.log(hi), n))).astype(int).tolist()
    b = lengths_only(Hq, Hkv, D, [DECODE] * n + [PREFILL] * len(chunks), [1] * n + [q for q, _ in chunks], c + [q + p for q, p in chunks])
    assert mixed_step_is_dealt_whole(b) == dealt


def test_decode_pieces_are_not_lengthened_where_two_rounds_are_out_of_reach(lib):
    """480 prefill items leave 544 of two rounds' places to decodes that have 494 items when uncut and two contexts of many
    pieces: pieces four times as long would not be enough, and pieces stay as they are by time."""
    c = [150] * 245 + [20000] * 2
    q = [32] * 60
    b = lengths_only(32, 8, 128, [DECODE] * len(c) + [PREFILL] * len(q), [1] * len(c) + q, c + q)
    d = fill(b)
    h = d["header"]
    check_coverage(b, d)
    assert h.deal_balanced == 0 and h.n_prefill_items == 480
    assert 1024 < h.n_items == decode_items_by_time(b) + 480 < 1331


def check_coverage_of_groups(d):
    """What check_coverage says of partial rows, for steps whose (row, key) pairs are too many to list."""
    rows = np.zeros(d["header"].n_partial_rows, np.int32)
    for it in d["items"][d["items"]["group"] >= 0]:
        rows[it["slot_row"]:it["slot_row"] + d["groups"][it["group"]]["rows_per_split"]] += 1
    assert np.all(rows == 1)


@pytest.mark.parametrize("seed", range(4))
def test_workspace_beyond_the_fixed_one_only_where_the_work_asks_for_it(lib, seed):
    """Random steps: workspace above the fixed 64 MiB is no more than cutting by visible pairs takes, so that whatever
    that cut lets the entry point with the fixed workspace accept, it accepts."""
    rng = np.random.default_rng(seed)

    def log_int(lo, hi):
        return int(np.rint(np.exp(rng.uniform(np.log(lo), np.log(hi)))))

    largest = 0
    for _ in range(150):
        Hq, Hkv, D = [(32, 8, 128), (8, 1, 128), (8, 2, 128), (24, 8, 128), (8, 8, 128), (12, 4, 128), (2, 2, 128),
                      (16, 1, 64), (32, 8, 64)][rng.integers(9)]
        kind, q, c = [], [], []
        for _ in range(rng.integers(1, 4)):
            rows, ctx, same = [(1, 8), (1, 64), (20, 500), (500, 5000)][rng.integers(4)], log_int(1000, 70000), rng.random() < 0.5
            for _ in range(log_int(1, 100) if rows[1] < 5000 else rng.integers(1, 6)):
                n = rows[1] // 3 if same else log_int(*rows)
                kind.append(PREFILL); q.append(n); c.append(n + (ctx if same else log_int(1, ctx)))
        if rng.random() < 0.5:
            for _ in range(log_int(1, 200)):
                kind.append(DECODE); q.append(1); c.append(log_int(20, 50000))
        largest = max(largest, check_workspace(Hq, Hkv, D, kind, q, c))
    assert largest > FIXED_WORKSPACE // 2


def test_partials_stay_bounded_where_tiles_are_nearly_empty(lib):
    """Chunks of one row behind long contexts take the time of full tiles: the caps follow that time, or such
    a step would be cut into pieces without number."""
    for decodes in (0, 400):
        b = lengths_only(32, 8, 128, [PREFILL] * 200 + [DECODE] * decodes, [1] * (200 + decodes), [30000] * 200 + [9000] * decodes)
        d = fill(b)
        assert d["header"].n_prefill_items <= 200 * 8 + 2048
        assert d["header"].workspace_bytes <= FIXED_WORKSPACE


@pytest.mark.parametrize("Hq,Hkv,D,chunks", [
    (32, 8, 128, [(2500, 0)]), (32, 8, 128, [(4097, 0)]), (32, 8, 128, [(2049, 0)]), (32, 8, 128, [(777, 0)]), (24, 8, 128, [(1025, 0)]),
    (32, 8, 64, [(301, 0), (1029, 700), (130, 63)]), (8, 1, 128, [(33, 900), (65, 300)])])
def test_longest_items_come_first(lib, Hq, Hkv, D, chunks):
    """The last tile of a prompt of 32 k + 1 tokens holds one row and sees the most keys: it takes longest, so it may not be
    queued behind tiles that see fewer."""
    items = fill(lengths_only(Hq, Hkv, D, [PREFILL] * len(chunks), [q for q, _ in chunks], [q + p for q, p in chunks]))["items"]
    assert np.all(np.diff(items["ke"] - items["kb"]) <= 0)


@pytest.mark.parametrize("Hq,Hkv,D,n,q,prior,whole", [
    (8, 8, 128, 36, 4, 17273, True), (12, 4, 128, 23, 4, 8015, True), (16, 16, 128, 27, 4, 18490, True), (8, 8, 64, 42, 4, 5321, True),
    (16, 8, 128, 33, 1, 12028, True), (8, 8, 128, 2, 4, 18671, False), (24, 8, 128, 3, 3, 20051, False)])
def test_tiles_with_idle_wavefronts_stay_whole_where_they_all_start_at_once(lib, Hq, Hkv, D, n, q, prior, whole):
    """Between 256 and 512 tiles of a few rows, one to a workgroup, do not slow each other like full ones and last as long as
    their keys take to stream: cutting them only adds partials.  Fewer tiles than CUs are cut."""
    h = fill(lengths_only(Hq, Hkv, D, [PREFILL] * n, [q] * n, [q + prior] * n))["header"]
    assert (h.n_groups == 0) == whole, (h.n_items, h.n_groups)


@pytest.mark.parametrize("rows", [1, 8, 32])
def test_cut_goes_by_the_time_of_a_tile_not_by_its_rows(lib, rows):
    """A tile of few rows takes as long as a full one: it is cut into as many pieces."""
    b = lengths_only(32, 8, 128, [PREFILL], [rows], [rows + 12968])
    assert fill(b)["header"].n_prefill_items == fill(lengths_only(32, 8, 128, [PREFILL], [32], [13000]))["header"].n_prefill_items


def test_planning_time_per_item_does_not_depend_on_the_head_layout(lib):
    """The trial of cuts looks at every row tile that differs: one of eight items on 8 kv-heads, every one or two on a single
    kv-head.  Time per descriptor byte of two steps of about 8000 items, best of twenty."""
    import time
    g = np.random.default_rng(5)
    q = np.rint(np.exp(g.uniform(np.log(100), np.log(3000), 120))).astype(np.int32)
    c = q + np.rint(np.exp(g.uniform(0, np.log(40000), 120))).astype(np.int32)

    def seconds_per_byte(Hq, Hkv, every):
        args = hb.make_shape(Hq, Hkv, 128, 1 << 30), np.full(len(q[::every]), PREFILL, np.int32), q[::every], c[::every]
        best = np.inf
        for _ in range(20):
            t = time.perf_counter()
            size = hb.hfx_batch_desc_sizes(*args)[0]
            best = min(best, time.perf_counter() - t)
        return best / size

    assert seconds_per_byte(8, 1, 1) < 3.5 * seconds_per_byte(32, 8, 4)      # 1.6 to 2.3; 4.6 to 5.6 with a general sort and heap


def test_dealing_is_straight_where_the_layout_is_by_workgroup(lib):
    b = lengths_only(32, 8, 128, [DECODE] * 64 + [PREFILL], [1] * 64 + [256], [3000] * 64 + [256])
    assert fill(b)["header"].deal_balanced == 0
    b = lengths_only(32, 8, 128, [DECODE] * 64, [1] * 64, [3000] * 64)
    assert fill(b)["header"].deal_balanced == 1


def test_decodes_outweigh_prefills_by_time(lib):
    """48 chunks of one row take the time of full tiles: four decodes beside them do not make a decode step of it."""
    h = fill(lengths_only(8, 8, 64, [DECODE] * 4 + [PREFILL] * 48, [1] * 52, [2000] * 4 + [3270] * 48))["header"]
    assert h.deal_balanced == 1 and h.n_prefill_items == 48 * 8
    h = fill(lengths_only(8, 8, 64, [DECODE] * 400 + [PREFILL] * 8, [1] * 408, [2000] * 400 + [3270] * 8))["header"]
    assert h.deal_balanced == 0


@pytest.mark.parametrize("Hq,Hkv,D", [(4, 4, 64), (2, 2, 128), (16, 1, 64), (12, 4, 128), (6, 2, 64)])
def test_planner_head_layouts_and_ragged_chunks(lib, Hq, Hkv, D):
    b = lengths_only(Hq, Hkv, D, [PREFILL, DECODE, PREFILL, DECODE, PREFILL], [1, 1, 33, 1, 130],
                     [1, 1, 33, 500, 700])
    check_coverage(b, fill(b))


def test_planner_is_a_function_of_lengths_only(lib):
    b = synth.config(2, 0.25)
    p = synth.permute_pages(b, 5)
    d0, d1 = fill(b), fill(p)
    assert np.array_equal(d0["items"], d1["items"]) and np.array_equal(d0["groups"], d1["groups"])
    assert not np.array_equal(d0["bt"], d1["bt"])


def test_validation_errors(lib):
    b = synth.config(1)
    shape = hb.make_shape(4, 2, 64, b.num_pages)
    host = np.zeros(1 << 16, np.uint8)

    def code(fn, *a):
        with pytest.raises(hb.HfxError) as e:
            fn(*a)
        return e.value.code

    ok = (b.kind, b.q_len, b.ctx_len, b.bt_indptr, b.bt_pages)
    hb.hfx_fill_batch_desc(shape, *ok, host)
    for bad_shape in [hb.make_shape(4, 3, 64, 8), hb.make_shape(4, 2, 96, 8), hb.make_shape(4, 2, 64, 8, page_size=32),
                      hb.make_shape(4, 2, 64, 0), hb.make_shape(64, 2, 64, 8), hb.make_shape(12, 6, 64, 8)]:
        assert code(hb.hfx_fill_batch_desc, bad_shape, *ok, host) == hb.HFX_ERR_SHAPE
    k = b.kind.copy(); k[0] = 2
    assert code(hb.hfx_fill_batch_desc, shape, k, *ok[1:], host) == hb.HFX_ERR_KIND
    q = b.q_len.copy(); q[0] = 2                          # decode with q_len != 1
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, q, *ok[2:], host) == hb.HFX_ERR_LEN
    c = b.ctx_len.copy(); c[3] = 31                       # context shorter than the chunk
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, b.q_len, c, *ok[3:], host) == hb.HFX_ERR_LEN
    q = b.q_len.copy(); q[3] = 0
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, q, *ok[2:], host) == hb.HFX_ERR_LEN
    ip = b.bt_indptr.copy(); ip[1] = 2                    # request 0 needs 3 pages, gets 2
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, b.q_len, b.ctx_len, ip, b.bt_pages, host) == hb.HFX_ERR_PAGES
    ip = b.bt_indptr.copy(); ip[0] = 1
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, b.q_len, b.ctx_len, ip, b.bt_pages, host) == hb.HFX_ERR_PAGES
    pg = b.bt_pages.copy(); pg[4] = b.num_pages
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, b.q_len, b.ctx_len, b.bt_indptr, pg, host) == hb.HFX_ERR_PAGE_ID
    pg = b.bt_pages.copy(); pg[0] = -1
    assert code(hb.hfx_fill_batch_desc, shape, b.kind, b.q_len, b.ctx_len, b.bt_indptr, pg, host) == hb.HFX_ERR_PAGE_ID
    assert code(hb.hfx_fill_batch_desc, shape, *ok, np.zeros(64, np.uint8)) == hb.HFX_ERR_BUFSIZE
    # null pointers, through the raw ABI
    sz = ctypes.c_size_t()
    assert lib.hfx_batch_desc_sizes(ctypes.byref(shape), 4, None, None, None, ctypes.byref(sz), ctypes.byref(sz),
                                    ctypes.byref(sz)) == hb.HFX_ERR_NULL
    assert lib.hfx_batch_desc_sizes(None, 4, None, None, None, None, None, None) == hb.HFX_ERR_NULL
    assert lib.hfx_mixed_paged_attention(ctypes.byref(shape), None, None, None, None, None, 0, None, None) == hb.HFX_ERR_NULL
    # a blob that is not a descriptor
    junk = np.zeros(4096, np.uint8)
    assert lib.hfx_mixed_paged_attention(ctypes.byref(shape), 16, 16, junk.ctypes.data, 16, None, 0, 16, None) == hb.HFX_ERR_DESC
    # shape that differs from the descriptor's
    other = hb.make_shape(4, 2, 64, b.num_pages + 1)
    assert lib.hfx_mixed_paged_attention(ctypes.byref(other), 16, 16, host.ctypes.data, 16, None, 0, 16, None) == hb.HFX_ERR_SHAPE
    # misaligned device pointer
    assert lib.hfx_mixed_paged_attention(ctypes.byref(shape), 8, 16, host.ctypes.data, 16, None, 0, 16, None) == hb.HFX_ERR_ALIGN
    # the other calls that take their geometry from the staging buffer's header refuse the same blobs
    sh, oth = ctypes.byref(shape), ctypes.byref(other)
    assert lib.hfx_mixed_paged_attention_static(sh, 16, 16, junk.ctypes.data, 16, 16, None) == hb.HFX_ERR_DESC
    assert lib.hfx_mixed_paged_attention_static(oth, 16, 16, host.ctypes.data, 16, 16, None) == hb.HFX_ERR_SHAPE
    assert lib.hfx_gather_kv(sh, 16, junk.ctypes.data, 16, 0, 16, 16, None) == hb.HFX_ERR_DESC
    assert lib.hfx_gather_kv(oth, 16, host.ctypes.data, 16, 0, 16, 16, None) == hb.HFX_ERR_SHAPE
    assert lib.hfx_gather_kv(sh, 16, host.ctypes.data, 16, 4, 16, 16, None) == hb.HFX_ERR_LEN      # request out of range
    assert lib.hfx_append_kv(sh, 16, 16, 16, junk.ctypes.data, 16, None) == hb.HFX_ERR_DESC
    assert lib.hfx_append_kv(oth, 16, 16, 16, host.ctypes.data, 16, None) == hb.HFX_ERR_SHAPE
    stale = host.copy()
    stale[4] ^= 1                                         # a descriptor of another layout version
    assert lib.hfx_mixed_paged_attention(sh, 16, 16, stale.ctypes.data, 16, None, 0, 16, None) == hb.HFX_ERR_DESC
    # a header whose count of queue classes is neither 1 nor 8 (the kernel would index the counters with it)
    bent = host.copy()
    off = hb.DescHeader.queue_classes.offset
    bent[off:off + 4] = np.frombuffer(np.uint32(5).tobytes(), np.uint8)
    ws = 16 if hb.parse_desc(host)["header"].workspace_bytes else None
    assert lib.hfx_mixed_paged_attention(sh, 16, 16, bent.ctypes.data, 16, ws, 1 << 40, 16, None) == hb.HFX_ERR_DESC


def test_a_header_with_impossible_die_positions_is_refused(lib):
    """die_items says which queue positions are handed out by die: a multiple of 8, and none past the end of the queue."""
    b = lengths_only(8, 1, 128, [PREFILL] * 170, [300] * 170, [300] * 170)
    shape = hb.make_shape(8, 1, 128, b.num_pages)
    size, _, ws = hb.hfx_batch_desc_sizes(shape, b.kind, b.q_len, b.ctx_len)
    host = np.zeros(size, np.uint8)
    hb.hfx_fill_batch_desc(shape, b.kind, b.q_len, b.ctx_len, b.bt_indptr, b.bt_pages, host)
    h = hb.parse_desc(host)["header"]
    assert 0 < h.die_items < h.n_items
    off = hb.DescHeader.die_items.offset
    for wrong in (h.die_items + 1, (h.n_items + 8) // 8 * 8, 0xfffffff8):
        bent = host.copy()
        bent[off:off + 4] = np.frombuffer(np.uint32(wrong).tobytes(), np.uint8)
        assert lib.hfx_mixed_paged_attention(ctypes.byref(shape), 16, 16, bent.ctypes.data, 16, 16, ws, 16, None) == hb.HFX_ERR_DESC, wrong


def test_page_ids_that_change_meanwhile_are_refused(lib):
    """The ids that go into the descriptor are the ones that have been checked.  Here the list lies where the descriptor's header is written, so that it
    changes between the two."""
    shape = hb.make_shape(4, 2, 64, 16)
    size = hb.hfx_batch_desc_sizes(shape, [0], [1], [200])[0]
    host = np.zeros(size, np.uint8)
    pages = host[:52].view(np.int32)
    pages[:] = np.arange(13)
    with pytest.raises(hb.HfxError) as e:
        lib_fill(lib, shape, [0], [1], [200], [0, 13], pages, host)
    assert e.value.code == hb.HFX_ERR_PAGE_ID
    assert lib.hfx_mixed_paged_attention(ctypes.byref(shape), 16, 16, host.ctypes.data, 16, 16, 1 << 30, 16, None) == hb.HFX_ERR_DESC


def lib_fill(lib, shape, kind, q_len, ctx_len, indptr, pages, host):
    a = [np.array(v, np.int32) for v in (kind, q_len, ctx_len, indptr)]
    rc = lib.hfx_fill_batch_desc(ctypes.byref(shape), 1, *(v.ctypes.data for v in a), pages.ctypes.data, host.ctypes.data, host.nbytes)
    if rc != hb.HFX_OK:
        raise hb.HfxError(rc, "hfx_fill_batch_desc")


def test_extra_reserved_pages_are_ignored(lib):
    b = synth.make_batch(4, 2, 64, [DECODE, PREFILL], [1, 20], [37, 50], 3, extra_pages_per_request=3)
    d = fill(b)
    assert d["header"].n_bt == (4 + 16) + (4 + 16)      # stored: rounded up to 4 entries, plus the padding
    check_coverage(b, d)


def test_copy_pages_validation(lib):
    # every check below fails on the host before anything is enqueued, so dummy device addresses do
    shape = hb.make_shape(8, 2, 64, 10, 0.0)
    stage = np.zeros(64, np.uint8)
    src, dst = 0x10000, 0x20000

    def call(s_ids, d_ids, src_pool=src, dst_pool=dst, dst_pages=6, host=stage, dev=0x30000):
        hb.hfx_copy_pages(shape, src_pool, dst_pool, dst_pages, s_ids, d_ids, host, dev, stage_bytes=64)

    call([], [])                                           # nothing to do
    for s_ids, d_ids, kw, code in [
            ([10], [0], {}, hb.HFX_ERR_PAGE_ID), ([-1], [0], {}, hb.HFX_ERR_PAGE_ID),
            ([0], [6], {}, hb.HFX_ERR_PAGE_ID), ([0, 1], [3, 3], {}, hb.HFX_ERR_PAGES),
            ([0, 1], [2, 0], {"dst_pool": src, "dst_pages": 10}, hb.HFX_ERR_PAGES),
            ([0], [1], {"src_pool": 0x10008}, hb.HFX_ERR_ALIGN),
            (list(range(9)), list(range(9)), {"dst_pages": 10}, hb.HFX_ERR_BUFSIZE),
            ([0], [1], {"dst_pages": 0}, hb.HFX_ERR_SHAPE)]:
        with pytest.raises(hb.HfxError) as e:
            call(s_ids, d_ids, **kw)
        assert e.value.code == code, (s_ids, d_ids, kw)


def test_header_is_plain_c_and_cpp(tmp_path):
    """The boundary is a C ABI: the header must compile on its own as C99 and as C++."""
    import shutil
    import subprocess
    hdr = os.path.join(ROOT, "include", "hfxattn.h")
    for compiler, flags, ext in (("gcc", ["-std=c99", "-pedantic", "-Wall", "-Werror"], "c"),
                                 ("g++", ["-std=c++11", "-Wall", "-Werror"], "cpp")):
        if shutil.which(compiler) is None:
            pytest.skip(f"{compiler} not available")
        src = tmp_path / f"use.{ext}"
        src.write_text('#include "hfxattn.h"\nint main(void) { hfx_shape s; hfx_decision d; (void)s; (void)d; return HFX_OK; }\n')
        subprocess.run([compiler, *flags, "-fsyntax-only", "-I", os.path.dirname(hdr), str(src)], check=True)


def test_inline_assembly_declares_the_registers_it_writes():
    """An asm statement that writes m0 says so: the compiler keeps values of its own there otherwise."""
    src = open(os.path.join(ROOT, "paper_2508_15919_amd", "csrc", "hfx_kernels.hip")).read()
    writes = 0
    for stmt in re.findall(r"\basm\s+volatile\s*\((.*?)\)\s*;", src, re.S):
        if not re.search(r"\bs_mov_b32 m0\b", stmt):
            continue
        writes += 1
        assert '"m0"' in stmt.rsplit(":", 1)[1], stmt
    assert writes == 2           # one per head dimension
