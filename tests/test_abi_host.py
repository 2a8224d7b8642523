"""Host-side checks of the C ABI that need no GPU: the library loads and exports every
symbol include/tc.h declares, descriptor validation returns the documented status codes,
and the planner's work list covers the batch exactly."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def tc():
    import paper_2508_01989_amd as tc
    if not os.path.exists(tc.LIB_PATH):
        from paper_2508_01989_amd.build import build
        build()
    tc.lib()
    return tc


def test_header_compiles_as_c99(tmp_path):
    src = tmp_path / "t.c"
    src.write_text('#include "tc.h"\nint main(void){ tc_plan_info i; (void)i; return TC_OK; }\n')
    rc = os.system(f"gcc -std=c99 -Wall -Werror -pedantic -I {ROOT}/include -c {src} -o {tmp_path}/t.o")
    assert rc == 0


def test_library_exports_every_declared_symbol(tc):
    header = open(os.path.join(ROOT, "include", "tc.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(tc_[a-z_]+)\s*\(", header))
    assert declared == set(tc.EXPORTS)
    L = C.CDLL(tc.LIB_PATH)
    for name in declared:
        assert hasattr(L, name), name
    assert tc.tc_version() >= 1
    assert tc.status_str(tc.TC_ERR_BLOCK) == "TC_ERR_BLOCK"


def _plan(tc, Hq=8, Hkv=2, D=128, q_len=(5, 1), ctx=(3, 40), nb=32, table=None, **kw):
    sp = W.custom_spec("x", Hq, Hkv, D, q_len, ctx)
    if table is None:
        table, mb, _ = W.make_tables(W.custom_spec("x", Hq, Hkv, D, q_len, ctx, num_blocks=nb), np.random.default_rng(0))
    qs = np.zeros(len(q_len) + 1, np.int32)
    qs[1:] = np.cumsum(q_len)
    pool = tc.make_pool(Hq, Hkv, D, nb, **kw)
    return tc.Plan(pool, qs, np.asarray(ctx, np.int32), table, host_only=True)


def _status(tc, fn):
    with pytest.raises(tc.TcError) as e:
        fn()
    assert tc.last_error() != ""
    return e.value.status


def test_validation_status_codes(tc):
    assert _status(tc, lambda: _plan(tc, D=96)) == tc.TC_ERR_SHAPE
    assert _status(tc, lambda: _plan(tc, Hq=7, Hkv=2)) == tc.TC_ERR_SHAPE
    assert _status(tc, lambda: _plan(tc, Hq=34, Hkv=2)) == tc.TC_ERR_SHAPE       # G = 17
    assert _status(tc, lambda: _plan(tc, block_size=32)) == tc.TC_ERR_SHAPE
    assert _status(tc, lambda: _plan(tc, dtype=0)) == tc.TC_ERR_SHAPE
    assert _status(tc, lambda: _plan(tc, ctx=(-1, 40))) == tc.TC_ERR_SPAN
    good = _plan(tc)
    assert good.info.num_seqs == 2
    table = np.zeros((2, 3), np.int32)
    assert _status(tc, lambda: _plan(tc, table=np.zeros((2, 2), np.int32))) == tc.TC_ERR_BLOCK   # 41 tokens need 3 pages
    bad = table.copy(); bad[1, 2] = 32
    assert _status(tc, lambda: _plan(tc, table=bad)) == tc.TC_ERR_BLOCK
    bad = table.copy(); bad[0, 0] = -1
    assert _status(tc, lambda: _plan(tc, table=bad)) == tc.TC_ERR_BLOCK
    # entries past the used prefix are never looked at
    ok = np.full((2, 9), W.TABLE_SENTINEL, np.int32); ok[0, :1] = 1; ok[1, :3] = [2, 3, 4]
    assert _plan(tc, table=ok).info.total_pages == 4
    # spans: zero-length sequence, q_start[0] != 0
    pool = tc.make_pool(8, 2, 128, 32)
    z = np.zeros(2, np.int32)
    assert _status(tc, lambda: tc.Plan(pool, np.array([0, 2, 2], np.int32), z, table, host_only=True)) == tc.TC_ERR_SPAN
    assert _status(tc, lambda: tc.Plan(pool, np.array([1, 2, 3], np.int32), z, table, host_only=True)) == tc.TC_ERR_SPAN
    # NULL arguments
    L = tc.lib()
    h = C.c_void_p()
    assert L.tc_plan_create_host(None, None, C.byref(h)) == tc.TC_ERR_NULL
    assert L.tc_plan_get_info(None, None) == tc.TC_ERR_NULL
    assert L.tc_plan_workspace_bytes(None) == 0
    L.tc_plan_destroy(None)


def test_element_type_is_part_of_the_plan(tc):
    p16 = _plan(tc, dtype=tc.TC_FP16)
    pool_bf = tc.make_pool(8, 2, 128, 32, k_pool=4096, v_pool=4096)
    pool_16 = tc.make_pool(8, 2, 128, 32, k_pool=4096, v_pool=4096, dtype=tc.TC_FP16)
    assert _status(tc, lambda: tc.tc_kv_append(p16, pool_bf, 4096, 4096)) == tc.TC_ERR_SHAPE   # plan is fp16, pool says bf16
    assert _status(tc, lambda: tc.tc_kv_append(p16, pool_16, 4096, 4096)) == tc.TC_ERR_ARG     # matches; host-only plan
    with pytest.raises(tc.TcError) as e:
        _plan(tc, dtype=3)
    assert e.value.status == tc.TC_ERR_SHAPE


def test_host_only_plan_cannot_be_launched(tc):
    p = _plan(tc)
    pool = tc.make_pool(8, 2, 128, 32, k_pool=4096, v_pool=4096)
    assert _status(tc, lambda: tc.tc_kv_append(p, pool, 4096, 4096)) == tc.TC_ERR_ARG
    pool2 = tc.make_pool(8, 2, 128, 33, k_pool=4096, v_pool=4096)
    assert _status(tc, lambda: tc.tc_kv_append(p, pool2, 4096, 4096)) == tc.TC_ERR_SHAPE
    pool3 = tc.make_pool(8, 2, 128, 32)
    assert _status(tc, lambda: tc.tc_kv_append(p, pool3, 4096, 4096)) == tc.TC_ERR_NULL


def test_migration_argument_checks_and_buffer_size(tc):
    p = _plan(tc)  # sequences of 8 and 41 tokens: 1 and 3 pages; Hkv=2, D=128 -> 8 KiB per block per pool
    per_page = 2 * 2 * 16 * 128 * 2
    assert tc.tc_kv_transfer_bytes(p, 0, 1) == 1 * per_page
    assert tc.tc_kv_transfer_bytes(p, 1, 5) == 5 * 3 * per_page
    assert tc.tc_kv_transfer_bytes(p, -1, 2) == 2 * 4 * per_page
    assert tc.tc_kv_transfer_bytes(p, 2, 1) == 0 and tc.tc_kv_transfer_bytes(p, -2, 1) == 0
    assert tc.tc_kv_transfer_bytes(p, 0, 0) == 0 and tc.tc_kv_transfer_bytes(p, 0, 4097) == 0
    pool = tc.make_pool(8, 2, 128, 32)
    # a host-only plan cannot be launched; shape mismatches are reported first
    assert _status(tc, lambda: tc.tc_kv_export(p, pool, 0, [4096], [4096], 4096)) == tc.TC_ERR_ARG
    assert _status(tc, lambda: tc.tc_kv_import(p, pool, 0, [4096], [4096], 4096)) == tc.TC_ERR_ARG
    pool2 = tc.make_pool(8, 2, 128, 33)
    assert _status(tc, lambda: tc.tc_kv_export(p, pool2, 0, [4096], [4096], 4096)) == tc.TC_ERR_SHAPE


def test_empty_batch_is_a_valid_plan(tc):
    pool = tc.make_pool(8, 2, 128, 4)
    p = tc.Plan(pool, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros((0, 1), np.int32), host_only=True)
    assert p.info.grid_blocks == 0 and p.workspace_bytes == 0


def check_work_list(tc, sp, table, nb):
    qs = np.zeros(sp.num_seqs + 1, np.int32)
    qs[1:] = np.cumsum(sp.q_len)
    pool = tc.make_pool(sp.num_q_heads, sp.num_kv_heads, sp.head_dim, nb)
    p = tc.Plan(pool, qs, sp.ctx_len, table, host_only=True)
    info, G, Hkv = p.info, sp.num_q_heads // sp.num_kv_heads, sp.num_kv_heads
    pf, dc, mg, pc = p.items(0), p.items(1), p.items(2), p.items(3)
    # prefill: every (sequence, KV head) has its positions covered once, in tiles of <= rows_per_prefill_item/G positions
    for s in np.flatnonzero(sp.q_len > 1):
        for h in range(Hkv):
            it = pf[(pf[:, 0] == s) & (pf[:, 1] == h)]
            it = it[np.argsort(it[:, 2])]
            assert it[0, 2] == 0 and np.all(it[1:, 2] == it[:-1, 2] + it[:-1, 3])
            assert it[-1, 2] + it[-1, 3] == sp.q_len[s] and np.all(it[:, 3] * G <= info.rows_per_prefill_item)
            assert np.all(it[:, 4] == qs[s]) and np.all(it[:, 5] == sp.ctx_len[s])
            assert np.all(it[:, 7] == (sp.kv_len[s] + 15) // 16)
    assert len(pf) == sum(-(-int(q) // (info.rows_per_prefill_item // G)) for q in sp.q_len[sp.q_len > 1]) * Hkv
    # heaviest prefill tiles first; KV head is the fastest index
    cost = pf[:, 5] + pf[:, 2] + pf[:, 3]
    assert np.all(np.diff(cost[::Hkv]) <= 0) and np.all(pf[:, 1] == np.arange(len(pf)) % Hkv)
    # pieces: the 64-token KV tiles of every item are covered once, by 1 piece (writes out) or by k pieces
    # (piece regions slot0 + c, one arrival counter per cut item)
    assert len(pc) == info.num_prefill_pieces
    slots = []
    regions = []
    counters = []
    merge_expected = []
    for i, item in enumerate(pf):
        mine = pc[pc[:, 0] == i]
        mine = mine[np.argsort(mine[:, 1])]
        n_tiles = (int(cost[i]) - 1) // 64 + 1
        k = len(mine)
        assert mine[0, 1] == 0 and mine[-1, 2] == n_tiles and np.all(mine[1:, 1] == mine[:-1, 2])
        assert np.all(mine[:, 2] > mine[:, 1]) and np.all(mine[:, 4] == k)
        assert mine[:, 5].tolist() == list(range(k))
        if k == 1:
            assert mine[0, 3] == -1 and mine[0, 6] == -1
        else:
            base = int(mine[0, 3])
            assert np.all(mine[:, 3] == base) and np.all(mine[:, 6] == mine[0, 6]) and mine[0, 6] >= 0
            counters.append(int(mine[0, 6]))
            regions += [base + c for c in range(k)]
            merge_expected.append((int(item[0]), int(item[1]), int(item[4] + item[2]), base, k, int(mine[0, 6]), int(item[3]), i))
    # prefill workgroups: each runs a run of consecutive pieces, the last one marked; together they hold every piece once
    wg = p.items(4)
    n_wg = info.num_prefill_workgroups
    assert len(wg) == n_wg and (n_wg > 0) == (len(pc) > 0)
    if n_wg:
        assert wg[0] == 0 and np.all(np.diff(wg) > 0)
        ends = np.flatnonzero(pc[:, 7] == 1)
        assert np.array_equal(ends, np.append(wg[1:], len(pc)) - 1) and set(np.unique(pc[:, 7])) <= {0, 1}
        # one KV head per workgroup; with a KV-head count that divides the compute units, workgroup id mod Hkv names it
        wg_of_piece = np.searchsorted(wg, np.arange(len(pc)), side="right") - 1
        heads = pf[pc[:, 0], 1]
        for w_ in range(n_wg):
            assert len(set(heads[wg_of_piece == w_])) == 1
        if 256 % Hkv == 0:
            assert np.all(heads == wg_of_piece % Hkv)
        tiles_of_wg = np.bincount(wg_of_piece, weights=(pc[:, 2] - pc[:, 1]), minlength=n_wg)
        levelled = 256 < 4 * len(pf) and len(pc) > len(pf)   # (up to a quarter of the compute units items are cut evenly)
        if not levelled:      # one piece per workgroup, most tiles first (uncut items, or few items whose KV ranges are cut)
            tiles_of_record = tiles_of_wg[::Hkv].copy()
            if len(pf) == len(pc) and info.block_threads == 256 and n_wg <= 256 * (2 if sp.head_dim == 128 else 3):
                row = max(1, 256 // Hkv)
                for first in range(row, n_wg // Hkv, 2 * row):  # workgroups of four waves that all run at once: every other row of 256 turned round
                    tiles_of_record[first:first + row] = tiles_of_record[first:first + row][::-1].copy()
            assert n_wg == len(pc) and np.all(np.diff(tiles_of_record) <= 0)
        else:                 # every KV head has the same runs, of nearly equal cost (tiles + 3 per piece)
            assert n_wg % Hkv == 0 and n_wg <= 256
            cost_of_wg = tiles_of_wg + 3 * np.bincount(wg_of_piece, minlength=n_wg)
            per_head = cost_of_wg.reshape(-1, Hkv)
            assert np.all(per_head == per_head[:, :1])
            assert per_head[:, 0].max() <= per_head[:, 0].mean() * 1.15 + 8
    # decode: the items fill whole workgroups of W waves; padding items hold no tokens
    W_ = info.block_threads // (64 * info.waves_per_item)
    assert len(dc) % W_ == 0 and len(dc) == info.num_decode_items
    real = dc[dc[:, 3] > dc[:, 2]]
    pad = dc[dc[:, 3] == dc[:, 2]]
    assert np.all(pad[:, 0] == -1) and np.all(pad[:, 7] == 1) and len(pad) < 32 * W_
    team_n, team_pos, tail, merge_idx = dc[:, 7] & 15, (dc[:, 7] >> 4) & 7, (dc[:, 7] >> 7) & 1, (dc[:, 7] >> 8) - 1
    # splits tile [0, kv_len) page-aligned, <= 64 pages each, for every KV head
    for s in np.flatnonzero(sp.q_len == 1):
        for h in range(Hkv):
            it = real[(real[:, 0] == s) & (real[:, 1] == h)]
            it = it[np.argsort(it[:, 2])]
            assert it[0, 2] == 0 and np.all(it[1:, 2] == it[:-1, 3]) and it[-1, 3] == sp.kv_len[s]
            assert np.all(it[:, 2] % 16 == 0) and np.all(it[:, 3] - it[:, 2] <= 1024)
            assert np.all(it[:, 4] == qs[s])
            # splits of at most split_tokens; beyond that a sequence that one workgroup covers has W of them, and one that takes several where the others'
            # splits were shortened (a chunk's workgroups of eight single waves, 2000 tokens on the mean)
            within = np.all(it[:, 3] - it[:, 2] <= info.split_tokens)
            shortened = len(pf) > 0 and info.block_threads == 512 and info.waves_per_item == 1 and np.mean(sp.kv_len[sp.q_len == 1]) >= 2000
            assert within or (len(it) == W_ if sp.kv_len[s] <= W_ * 1024 else shortened)
            # 1, 2, 4 .. W splits (one team), or a multiple of W when W splits of 1024 tokens cannot cover the sequence
            n_teams = int(np.sum((it[:, 7] >> 4) & 7 == 0))
            # exactly the split that ends the sequence is marked as holding the newest token
            assert np.array_equal((it[:, 7] >> 7) & 1, (it[:, 3] == sp.kv_len[s]).astype(int))
            assert len(it) in (1, 2, 4, 8)[:W_.bit_length()] if sp.kv_len[s] <= W_ * 1024 else len(it) % W_ == 0
            assert n_teams == -(-len(it) // W_)
            # a partial slot exactly when the splits are in more than one team (then one slot per team)
            assert np.all((it[:, 5] >= 0) == (n_teams > 1))
    # teams: consecutive waves of one workgroup, positions 0..n-1, consecutive splits of one (sequence, KV head), one slot
    i = 0
    leaders = []
    while i < len(dc):
        n, pos = int(team_n[i]), int(team_pos[i])
        assert pos == 0 and 1 <= n <= W_ and i // W_ == (i + n - 1) // W_
        team = dc[i:i + n]
        assert np.all(team_n[i:i + n] == n) and np.array_equal(team_pos[i:i + n], np.arange(n))
        assert np.all(merge_idx[i:i + n] == merge_idx[i])
        if team[0, 3] > team[0, 2]:
            assert np.all(team[:, 0] == team[0, 0]) and np.all(team[:, 1] == team[0, 1]) and np.all(team[:, 5] == team[0, 5])
            assert np.all(team[1:, 2] == team[:-1, 3])
            leaders.append(team[0])
        else:
            assert n == 1
        i += n
    leaders = np.array(leaders).reshape(-1, 8)
    # partial slots of decode teams and piece regions of cut prefill items: each unique and dense
    slots += leaders[leaders[:, 5] >= 0, 5].tolist()
    assert len(slots) == info.num_partials and sorted(slots) == list(range(info.num_partials))
    assert len(regions) == info.num_piece_partials and sorted(regions) == list(range(info.num_piece_partials))
    # merge items name exactly the slots of their teams / pieces, and every team points at its pair's merge item
    for s in np.flatnonzero(sp.q_len == 1):
        for h in range(Hkv):
            mine = leaders[(leaders[:, 0] == s) & (leaders[:, 1] == h)]
            m_idx = (mine[:, 7] >> 8) - 1
            if len(mine) > 1:
                assert np.all(m_idx == m_idx[0]) and m_idx[0] >= 0
                item = mg[m_idx[0]]
                assert (item[0], item[1], item[2], item[3], item[4]) == (s, h, qs[s], mine[:, 5].min(), len(mine))
                counters.append(int(item[5]))
                merge_expected.append((int(s), h, int(qs[s]), int(mine[:, 5].min()), len(mine), int(item[5]), 1, -1))
                assert sorted(mine[:, 5].tolist()) == list(range(mine[:, 5].min(), mine[:, 5].min() + len(mine)))
            else:
                assert np.all(m_idx == -1)
    assert sorted(merge_expected) == sorted(tuple(int(x) for x in m[:8]) for m in mg)
    n_cut = sum(1 for m in mg if m[7] >= 0)
    assert all(m[7] >= 0 for m in mg[:n_cut]) and all(m[7] < 0 for m in mg[n_cut:])   # those of cut prefill items come first
    # arrival counters: one per split pair, dense
    assert info.num_counters == len(counters) and sorted(counters) == list(range(len(counters)))
    assert p.workspace_bytes == (info.num_partials * G + info.num_piece_partials * 256) * (sp.head_dim + 2) * 4
    units = -(-info.num_decode_items // W_)
    if info.decode_queue:   # no more workgroups than compute units; the decode items are drawn from a queue
        assert 0 < info.num_prefill_workgroups <= 256 and units > 0
        assert info.grid_blocks == info.num_prefill_workgroups + min(units, 256 - info.num_prefill_workgroups) <= 256
    else:
        assert info.grid_blocks == info.num_prefill_workgroups + units
    return info


@pytest.mark.parametrize("idx", [0, 1, 2, 3, 4])
def test_work_list_covers_the_batch_exactly(tc, idx):
    sp = W.config_spec(idx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(3))
    info = check_work_list(tc, sp, table, nb)
    if idx == 1:
        # 256 row blocks for 256 compute units and about as much decode work as their uneven sweeps leave idle time:
        # one uncut row block per workgroup, the decode items drawn from the queue by the workgroups that finish early
        assert info.num_prefill_workgroups == info.num_prefill_pieces == info.num_prefill_items == 256
        assert info.decode_queue == 1 and info.grid_blocks == 256 and info.num_piece_partials == 0
    elif idx == 2:
        # 32 row blocks beside a long decode phase: neither cut nor levelled
        assert info.num_prefill_pieces == info.num_prefill_items == info.num_prefill_workgroups
    else:
        assert info.num_prefill_pieces == info.num_prefill_items == info.num_prefill_workgroups


@pytest.mark.parametrize("name,Hq,Hkv,q_len,ctx,cut", [
    ("small chunk, few short decodes", 32, 8, [128] + [1] * 16, [2048] + [300] * 16, True),
    ("small chunk alone", 32, 8, [256], [4000], True),
    ("ragged chunk, G=5", 10, 2, [77, 1], [1500, 40], True),
    ("small chunk under a long decode phase", 32, 8, [128] + [1] * 256, [2048] + [3000] * 256, False),
    ("short context", 32, 8, [128], [100], False),
    ("mid-sized chunk alone: levelled", 32, 8, [1024], [4096], True),
    ("mid-sized chunk, few decodes: levelled, decode queue", 32, 8, [1024] + [1] * 4, [4096] + [900] * 4, True),
    ("mid-sized chunk, many decodes: uncut, decode queue", 32, 8, [1024] + [1] * 64, [4096] + [2300] * 64, False),
    ("chunk that fills the chip, alone: uncut", 32, 8, [2048], [4096], False),
    ("chunk that fills the chip, decodes: uncut, decode queue", 32, 8, [1800] + [1] * 40, [4096] + [900] * 40, False),
])
def test_small_prefill_batches_are_cut_into_kv_pieces(tc, name, Hq, Hkv, q_len, ctx, cut):
    sp = W.custom_spec(name, Hq, Hkv, 128, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(5))
    info = check_work_list(tc, sp, table, nb)
    assert (info.num_prefill_pieces > info.num_prefill_items) == cut
    assert info.num_prefill_pieces <= 8 * info.num_prefill_items


@pytest.mark.parametrize("seed", range(25))
def test_work_list_invariants_on_random_batches(tc, seed):
    """Random mixes of prefill chunks and decodes, random head shapes: the same coverage checks."""
    rng = np.random.default_rng(4000 + seed)
    Hkv = int(rng.choice([1, 2, 4, 8]))
    G = int(rng.choice([1, 2, 3, 4, 5, 8, 16]))
    n_pf, n_dec = int(rng.integers(0, 4)), int(rng.integers(0, 40))
    if n_pf + n_dec == 0:
        n_dec = 1
    q_len = [int(rng.integers(2, 700)) for _ in range(n_pf)] + [1] * n_dec
    ctx = [int(rng.integers(0, 6000)) for _ in range(n_pf)] + [int(rng.integers(0, 9000)) for _ in range(n_dec)]
    order = rng.permutation(len(q_len))
    sp = W.custom_spec(f"rand{seed}", Hkv * G, Hkv, int(rng.choice([64, 128])), [q_len[i] for i in order], [ctx[i] for i in order])
    table, mb, nb = W.make_tables(sp, rng)
    check_work_list(tc, sp, table, nb)


def test_plan_update_gives_the_work_lists_of_fresh_plans(tc):
    """Two successive batches through one plan object (tc_plan_update) give the same work lists as fresh plans,
    whatever was planned before; a failed update leaves an empty plan."""
    shapes = [(32, 8, [2048] + [1] * 64, [4096] + [900] * 64), (32, 8, [1] * 40, [3000] * 40), (32, 8, [256, 1], [100, 70000]),
              (32, 8, [5], [0])]
    pool = tc.make_pool(32, 8, 128, 1 << 16)
    reused = None
    for Hq, Hkv, q_len, ctx in shapes + shapes[::-1]:
        sp = W.custom_spec("u", Hq, Hkv, 128, q_len, ctx, num_blocks=1 << 16)
        table, mb, nb = W.make_tables(sp, np.random.default_rng(len(q_len)))
        qs = np.zeros(len(q_len) + 1, np.int32)
        qs[1:] = np.cumsum(q_len)
        fresh = tc.Plan(pool, qs, sp.ctx_len, table, host_only=True)
        if reused is None:
            reused = tc.Plan(pool, qs, sp.ctx_len, table, host_only=True)
        else:
            reused.update(pool, qs, sp.ctx_len, table)
        for f in ("num_seqs", "total_q", "num_prefill_items", "num_decode_items", "num_merge_items", "num_partials", "split_tokens",
                  "grid_blocks", "block_threads", "total_pages", "num_prefill_pieces", "num_prefill_workgroups", "num_counters", "num_piece_partials",
                  "decode_queue"):
            assert getattr(fresh.info, f) == getattr(reused.info, f), f
        for kind in range(5):
            assert np.array_equal(fresh.items(kind), reused.items(kind)), kind
        assert fresh.workspace_bytes == reused.workspace_bytes
    with pytest.raises(tc.TcError) as e:
        reused.update(pool, np.array([0, 0], np.int32), np.zeros(1, np.int32), np.zeros((1, 1), np.int32))
    assert e.value.status == tc.TC_ERR_SPAN
    assert reused.info.num_seqs == 0 and reused.info.grid_blocks == 0 and reused.workspace_bytes == 0


@pytest.mark.parametrize("name,Hq,Hkv,D,q_len,ctx,waves,rows", [
    ("few decodes: a split per workgroup", 32, 8, 128, [1] * 8, [900, 64, 3000, 1023, 1024, 1025, 7, 0], 4, 256),
    ("one decode over 200k tokens", 8, 2, 128, [1], [200000], 4, 256),
    ("even decodes under 4096 tokens: a split per wave", 8, 2, 64, [1] * 200, [1400 + i for i in range(200)], 1, 256),
    ("many decodes: a split per wave", 32, 8, 128, [1] * 120, [1000] * 120, 1, 256),
    ("few long decodes beside a first chunk", 40, 8, 128, [300] + [1] * 4, [0, 6000, 2000, 12000, 30], 8, 256),  # 16 us of K/V, 9 of sweep
    ("one long decode beside a first chunk", 40, 8, 128, [300, 1, 1], [0, 3000, 30], 8, 128),
    ("few long decodes beside a chunk that fills the chip", 16, 4, 64, [4000] + [1] * 3, [0, 8000, 7000, 100], 1, 256),
    ("short decodes beside a first chunk", 8, 8, 64, [64] + [1] * 4, [0, 36, 63, 99, 127], 1, 128),
    ("small chunk over a long context: cut", 16, 1, 128, [20], [30000], 1, 128),
    ("first chunk beside a heavy decode branch", 32, 8, 128, [64] + [1] * 40, [0] + [1500] * 40, 1, 256),
])
def test_work_lists_of_the_launch_forms(tc, name, Hq, Hkv, D, q_len, ctx, waves, rows):
    """Every rule that chooses a launch form: the work list still covers the batch exactly, and the form is the one expected."""
    sp = W.custom_spec(name, Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(6))
    info = check_work_list(tc, sp, table, nb)
    assert (info.waves_per_item, info.rows_per_prefill_item) == (waves, rows)
    assert info.block_threads == (512 if info.num_prefill_items else 256)   # the launch's, whatever the decode items are


def _longest_sweep(p):
    """Tiles the busiest prefill workgroup sweeps."""
    pc, wg = p.items(3), p.items(4)
    tiles = pc[:, 2] - pc[:, 1]
    return max(int(tiles[a:b].sum()) for a, b in zip(wg, list(wg[1:]) + [len(pc)]))


@pytest.mark.parametrize("G", range(1, 17))
@pytest.mark.parametrize("D,us,overhead", [(128, {256: 1.8, 128: 1.1}, 12.0), (64, {256: 0.9, 128: 0.62}, 6.0)])
def test_small_items_never_make_the_longest_sweep_slower(tc, G, D, us, overhead):
    """Items of 128 rows hold 128 // G positions, less than half of 256 // G where that is odd: however a chunk's length falls on
    the two, the longest sweep, in microseconds at the rate of its item size, is not above that of 256-row items whose KV range is
    cut to fill the chip, but for what starting and combining twice as many pieces per item costs."""
    Hkv, whole, half = 8, 256 // G, 128 // G
    lengths = sorted({n for m in (1, 2, 3, 4) for n in (m * whole - 1, m * whole, m * whole + 1, m * half, m * half + 1, m * (half * 2 + 1)) if n >= 2})
    pool = tc.make_pool(G * Hkv, Hkv, D, 1 << 12)
    for n in lengths:
        for ctx in (2000, 8000, 30000):
            tiles = (ctx + n + 63) // 64
            items = -(-n // whole) * Hkv
            if items * 4 > 256:
                continue
            p = tc.Plan(pool, np.array([0, n], np.int32), np.array([ctx], np.int32), np.zeros((1, (ctx + n + 15) // 16), np.int32), host_only=True)
            k = max(1, min(8, 256 // items, tiles // 8))
            bound = -(-tiles // k) * us[256] + overhead
            got = _longest_sweep(p) * us[p.info.rows_per_prefill_item]
            assert got <= bound, (n, ctx, p.info.rows_per_prefill_item, p.info.num_prefill_pieces, got, bound)


@pytest.mark.parametrize("Hq,Hkv,D,q_len,ctx,rows", [
    (40, 8, 128, [204], [20000], 256),                          # 72 items of 128 rows could not be cut
    (40, 8, 128, [102, 102], [20000, 15000], 256),
    (24, 8, 128, [340], [24576], 256),
    (32, 8, 128, [64], [20000], 128),                           # 256-row items cut in eight leave units empty
    (32, 8, 128, [256], [20000], 256),                          # a full chip either way
    (40, 8, 128, [801], [0], 128),                              # 264 short items
    (40, 8, 128, [400, 405] + [1] * 16, [0, 0] + [500] * 16, 256),  # they leave no units for the decodes
    (40, 8, 128, [51] * 16 + [1] * 4, [0] * 16 + [500] * 4, 256),   # 384 items of one tile
    (32, 8, 128, [300] + [1] * 4, [0] + [500] * 4, 128),
    (8, 8, 64, [455] + [1] * 37, [9062] + [1400] * 37, 256),    # pieces of both sizes are as long, halves take all units
    (32, 8, 64, [128] + [1] * 8, [8000] + [500] * 8, 128),
    (32, 8, 128, [256] + [1] * 32, [2048] + [2270] * 32, 128),  # neither size is worth cutting more than once under the decodes
])
def test_rows_per_item(tc, Hq, Hkv, D, q_len, ctx, rows):
    sp = W.custom_spec("rows", Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(8))
    assert check_work_list(tc, sp, table, nb).rows_per_prefill_item == rows


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n,items,queue", [(270, 72, 0), (400, 104, 0), (500, 128, 0), (516, 136, 1), (800, 200, 1)])
def test_small_items_draw_decodes_from_a_queue_from_half_of_the_units_on(tc, D, n, items, queue):
    sp = W.custom_spec("queue", 32, 8, D, [n] + [1] * 3, [0] + [200] * 3)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(9))
    info = check_work_list(tc, sp, table, nb)
    assert (info.rows_per_prefill_item, info.num_prefill_workgroups, info.decode_queue) == (128, items, queue)


@pytest.mark.parametrize("Hq,Hkv,D,ctx,waves", [
    (32, 8, 128, [65] * 64, 4),                     # 512 pairs: two workgroups per compute unit
    (32, 8, 128, [65] * 96, 4),                     # 768, the line
    (32, 8, 128, [65] * 97, 1),
    (32, 32, 128, [65] * 25, 1),                    # the same with more KV heads
    (32, 8, 64, [65] * 192, 4),                     # twice as many at head_dim 64
    (32, 8, 64, [65] * 193, 1),
    (32, 8, 128, [7] * 512, 1),
    (8, 2, 64, [12] * 2000, 1),
    (32, 8, 128, [286] * 200, 1),                   # 287 tokens with the new one
    (32, 8, 128, [287] * 200, 4),
    (32, 32, 128, [2100] + [30] * 29, 4),           # one sequence keeps single waves busy for 33 pages
    (32, 8, 128, [900] + [30] * 120, 1),            # and for 15
])
def test_many_short_decodes_are_run_by_single_waves(tc, Hq, Hkv, D, ctx, waves):
    sp = W.custom_spec("short", Hq, Hkv, D, [1] * len(ctx), ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(10))
    assert check_work_list(tc, sp, table, nb).waves_per_item == waves


@pytest.mark.parametrize("Hkv,D,ctx,waves", [
    (8, 128, [260, 310, 429, 539, 576, 595, 617, 665, 784, 851, 870, 922, 928, 943, 1046, 1127, 1149, 1162, 1173, 1240, 1259, 1306, 1353, 1365, 1431], 1),
    (8, 64, [260, 310, 429, 539, 576, 595, 617, 665, 784, 851, 870, 922, 928, 943, 1046, 1127, 1149, 1162, 1173, 1240, 1259, 1306, 1353, 1365, 1431], 4),
    (8, 128, [260, 310, 429, 539, 576, 595, 617, 665, 784, 851, 870, 922, 928, 943, 1046, 1127], 4),  # a unit each
])
def test_decodes_that_would_double_a_few_units_are_run_by_single_waves(tc, Hkv, D, ctx, waves):
    sp = W.custom_spec("doubled", Hkv, Hkv, D, [1] * len(ctx), ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(11))
    assert check_work_list(tc, sp, table, nb).waves_per_item == waves


@pytest.mark.parametrize("Hq,rows,n,decodes,waves", [
    (40, 128, 320, [157, 205, 214, 351, 267, 260, 184, 234, 368, 460, 231, 438, 149, 475], 8),
    (64, 128, 438, [252, 24, 190, 374, 399, 465, 245, 341, 197, 199, 86, 380, 159], 8),
    (32, 256, 2200, [465] * 10, 1),   # sweeps of 35 tiles at 256 rows
])
def test_sweeps_of_small_items_are_taken_at_their_own_rate(tc, Hq, rows, n, decodes, waves):
    """Whether few long decodes are run by whole workgroups depends on what else the launch waits for."""
    sp = W.custom_spec("rate", Hq, 8, 128, [n] + [1] * len(decodes), [0] + decodes)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(12))
    info = check_work_list(tc, sp, table, nb)
    assert (info.rows_per_prefill_item, info.waves_per_item) == (rows, waves)


@pytest.mark.parametrize("Hq,Hkv,D,chunks,long,n_short,waves", [
    (32, 32, 128, [128], [8000] * 4, 128, 1),     # 5120 workgroups
    (32, 32, 128, [128], [6000], 64, 8),          # 2240, and nothing else to wait for
    (32, 8, 64, [701, 333, 45], [6000], 400, 1),  # 3248 units of the queue
    (32, 8, 64, [701, 333, 45], [6000], 128, 8),
    (32, 8, 128, [128], [6000], 400, 8),          # 3248, half as long as the long one
])
def test_one_long_decode_beside_a_chunk_does_not_take_many_short_ones_along(tc, Hq, Hkv, D, chunks, long, n_short, waves):
    sp = W.custom_spec("along", Hq, Hkv, D, chunks + [1] * (len(long) + n_short), [0] * len(chunks) + long + [40 + i % 41 for i in range(n_short)])
    table, mb, nb = W.make_tables(sp, np.random.default_rng(13))
    assert check_work_list(tc, sp, table, nb).waves_per_item == waves


STATIC_SCRATCH = 64 << 20  # what tc_mixed_attention_static has


@pytest.mark.parametrize("Hq,Hkv,q_len,ctx,levelled", [
    (16, 2, [8709], [20000], True),                             # runs whose cuts all leave two regions: 508 of 133 KB
    (16, 1, [4116], [20000], True),
    (4, 1, [20608], [40000], True),
    (8, 2, [8410] * 3, [13417, 56851, 0], True),
    (128, 8, [556] + [1] * 6, [20000] + [15000] * 6, True),     # beside the decodes' own partial results
    (128, 8, [520] + [1] * 8, [30000] + [9000] * 8, True),
    (32, 2, [2143] + [1] * 5, [51899] + [57495] * 5, True),
    (128, 8, [639] + [1] * 15, [79919] + [9701] * 15, False),   # too few runs would fit
])
def test_chunks_cut_into_runs_fit_the_static_scratch(tc, Hq, Hkv, q_len, ctx, levelled):
    """Whole items need no workspace: a chunk of more items than three quarters of the compute units (which ran whole at first)
    must not be refused by tc_mixed_attention_static for the sake of a level load."""
    sp = W.custom_spec("static", Hq, Hkv, 128, q_len, ctx)
    mb = int((sp.kv_len.max() + 15) // 16)
    qs = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    p = tc.Plan(tc.make_pool(Hq, Hkv, 128, 16), qs, sp.ctx_len, np.zeros((len(q_len), mb), np.int32), host_only=True)
    assert 4 * p.info.num_prefill_items > 3 * 256
    assert (p.info.num_prefill_workgroups < p.info.num_prefill_pieces) == levelled
    assert p.workspace_bytes <= STATIC_SCRATCH


@pytest.mark.parametrize("Hq,Hkv,D,q_len,ctx,levelled", [
    (40, 8, 128, [1115] + [1] * 4, [2091] + [1200] * 4, True),
    (64, 8, 64, [609] + [1] * 69, [4975] + [495] * 69, True),
    (32, 8, 128, [1408] + [1] * 3, [0] + [2000] * 3, True),
    (16, 2, 64, [1424] + [1] * 8, [0] + [2000] * 8, True),
    (32, 8, 128, [2048], [0], False),                         # small workgroups, without decodes
    (32, 32, 128, [1136, 1], [174, 1000], False),             # seven runs per KV head: whole items
])
def test_runs_where_small_workgroups_are_out_of_the_question(tc, Hq, Hkv, D, q_len, ctx, levelled):
    """Beside decodes that small workgroups do not serve, the choice is between whole items and runs, whatever small ones would take."""
    sp = W.custom_spec("runs", Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(14))
    info = check_work_list(tc, sp, table, nb)
    assert (info.num_prefill_workgroups < info.num_prefill_pieces) == levelled
    assert info.block_threads == (512 if 1 in q_len else 256)


@pytest.mark.parametrize("Hq,Hkv,D,chunk,offset,decodes,waves", [
    (40, 8, 128, 2664, 0, [3000 + 250 * i for i in range(29)], 1),    # 155 us of K/V: the longest sequences are a part of that
    (32, 8, 64, 3300, 0, [1500 + 180 * i for i in range(36)], 1),
    (32, 8, 128, 3648, 0, [2264 + 25 * i for i in range(62)], 1),
    (40, 8, 128, 2664, 0, [3000, 5000, 7000], 8),
    (32, 8, 128, 8190, 0, [3000] * 8, 8),                             # 1024 sweeps, four for every unit
    (32, 8, 128, 8224, 0, [3000] * 8, 8),                             # and 1032
    (128, 8, 128, 2480, 0, [2546], 8),
    (64, 8, 128, 8192, 24576, [16000] * 32, 1),
])
def test_decodes_behind_many_sweeps(tc, Hq, Hkv, D, chunk, offset, decodes, waves):
    """Whole workgroups for decodes that start when the last sweeps have: however many sweeps there are, where the longest sequence
    takes more than half of the time of the decodes' stream."""
    sp = W.custom_spec("late", Hq, Hkv, D, [chunk] + [1] * len(decodes), [offset] + decodes)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(15))
    info = check_work_list(tc, sp, table, nb)
    assert info.num_prefill_workgroups > 256 and info.decode_queue == 0
    assert (info.block_threads, info.waves_per_item) == (512, waves)


@pytest.mark.parametrize("Hq,Hkv,D,q_len,ctx,threads,levelled", [
    (32, 8, 128, [1200, 1200], [3400, 0], 512, False),           # 304 long small items for 256 units: whole ones
    (64, 8, 128, [600, 600], [3400, 0], 512, False),
    (64, 8, 64, [685, 830, 1, 1], [12873, 0, 900, 200], 512, False),
    (16, 2, 128, [2652, 2355] + [1] * 5, [11274, 0] + [600] * 5, 512, False),
    (40, 8, 64, [1204], [4097], 512, True),                      # 392 long ones, from 192 items of 256 rows: runs
    (32, 8, 128, [2048], [0], 256, False),                       # every long one with a short one beside it
    (16, 2, 128, [4624], [0], 256, False),
    (32, 8, 64, [1500, 900], [3400, 0], 256, False),             # three to a unit
    (128, 8, 128, [169, 104], [0, 0], 256, False),               # short sweeps
])
def test_small_workgroups_where_no_unit_has_two_long_sweeps(tc, Hq, Hkv, D, q_len, ctx, threads, levelled):
    sp = W.custom_spec("crowded", Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(18))
    info = check_work_list(tc, sp, table, nb)
    assert (info.block_threads, info.num_prefill_workgroups < info.num_prefill_pieces) == (threads, levelled)


@pytest.mark.parametrize("Hq,Hkv,D,ctx,waves", [
    (32, 32, 64, [2281, 639, 1722, 2003], 8),           # halves of up to 63 pages, eight waves on 40 of the second round
    (40, 8, 64, [952, 623, 1571, 1056, 1556, 1411, 365, 401, 1752, 1946, 1151, 2093, 1822, 741, 430, 1267, 713, 1861, 2074, 480, 1095], 8),
    (32, 8, 128, [2500, 5000, 4000, 9000, 7000, 8000], 4),   # long ones: halves as short as it takes
    (32, 8, 128, [1900] * 16, 4),                       # the second round's splits are as long as the first's
])
def test_two_splits_to_a_workgroup_where_halves_are_not_long(tc, Hq, Hkv, D, ctx, waves):
    sp = W.custom_spec("halves", Hq, Hkv, D, [4] + [1] * len(ctx), [2] + ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(17))
    info = check_work_list(tc, sp, table, nb)
    assert (info.block_threads, info.waves_per_item) == (512, waves)


def _build_ratio(tc, Hq, Hkv, first, second):
    """Host time of building one work list over that of another: the least of many, in turn, which other load does not reach."""
    pool, batches = tc.make_pool(Hq, Hkv, 128, 16), []
    for q_len, ctx in (first, second):
        sp = W.custom_spec("time", Hq, Hkv, 128, q_len, ctx)
        qs = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
        table = np.zeros((len(q_len), int((sp.kv_len.max() + 15) // 16)), np.int32)
        batches.append((tc.Plan(pool, qs, sp.ctx_len, table, host_only=True), qs, sp.ctx_len, table, []))
    for _ in range(300):
        for p, qs, ctx_len, table, ns in batches:
            p.update(pool, qs, ctx_len, table)
            ns.append(p.info.build_ns)
    return min(batches[0][4]) / min(batches[1][4])


def test_estimating_the_forms_of_a_chunk_is_a_small_part_of_planning(tc):
    """A plan is made every iteration.  1000 items, whose forms are estimated, against 1032, which run whole without a look at it."""
    assert _build_ratio(tc, 32, 8, ([8000], [0]), ([8256], [0])) < 1.4


def test_looking_for_two_splits_to_a_workgroup_is_a_small_part_of_planning(tc):
    """499 short decodes and a long one, where the length of two splits is looked for, against 1099 and one, where it is not."""
    batch = lambda n: ([128] + [1] * n, [1000, 8000] + [100] * (n - 1))
    assert _build_ratio(tc, 8, 1, batch(500), batch(1100)) < 0.7


RECORDS = """
#include <cstdio>
#include <vector>
#include "tc_internal.h"
int main(int, char **argv) {  // {heads, KV heads, head_dim, blocks, sequences, table columns, q_start, ctx_len, table} -> {records, the image's counters, stride}
    FILE *in = fopen(argv[1], "rb"), *out = fopen(argv[2], "wb");
    int32_t h[6];
    if (!in || !out || fread(h, 4, 6, in) != 6) return 1;
    std::vector<int32_t> a((size_t)(h[4] + 1) + h[4] + (size_t)h[4] * h[5]);
    if (fread(a.data(), 4, a.size(), in) != a.size()) return 1;
    tc_kv_pool pool = {};
    pool.num_q_heads = h[0]; pool.num_kv_heads = h[1]; pool.head_dim = h[2]; pool.block_size = 16; pool.dtype = TC_BF16; pool.num_blocks = h[3];
    tc_batch b = {h[4], a.data(), a.data() + h[4] + 1, a.data() + 2 * h[4] + 1, h[5]};
    tc_plan *p = nullptr;
    if (tc_plan_create_host(&pool, &b, &p)) return 1;
    if (p->off_records % tc::kRecordInts) return 1;
    const int32_t n[2] = {p->n_counters, p->counter_stride};
    fwrite(n, 4, 2, out);
    fwrite(p->host + p->off_records, 4, (size_t)p->n_pieces / h[1] * tc::kRecordInts, out);
    tc_plan_destroy(p);
    return fclose(out);
}
"""


@pytest.fixture(scope="module")
def records_of(tc, tmp_path_factory):
    """The records of a plan as the kernels read them (the image that is uploaded), [record][32]."""
    d = tmp_path_factory.mktemp("records")
    src, exe, lib_dir = d / "t.cpp", d / "t", os.path.dirname(tc.LIB_PATH)
    src.write_text(RECORDS)
    assert os.system(f"g++ -std=c++17 -I {ROOT}/include -I {lib_dir}/csrc {src} {tc.LIB_PATH} -Wl,-rpath,{lib_dir} -Wl,-rpath-link,/opt/rocm/lib -o {exe}") == 0

    def run(sp, table, nb):
        qs = np.concatenate([[0], np.cumsum(sp.q_len)])
        head = [sp.num_q_heads, sp.num_kv_heads, sp.head_dim, nb, sp.num_seqs, table.shape[1]]
        np.concatenate([head, qs, sp.ctx_len, table.ravel()]).astype(np.int32).tofile(d / "in")
        assert os.system(f"LD_LIBRARY_PATH=/opt/rocm/lib {exe} {d}/in {d}/out") == 0
        out = np.fromfile(d / "out", np.int32)
        return out[:2], out[2:].reshape(-1, 32)
    return run


CHUNK_FORMS = [
    # Hq, Hkv, D, q_len, ctx, (block_threads, rows per item, waves per decode item, queue, several pieces to a workgroup)
    (32, 8, 128, [1024], [4096], (512, 256, 1, 0, True)),                                    # 128 items
    (8, 8, 128, [7760], [0], (512, 256, 1, 0, True)),                                        # 248
    (64, 8, 64, [1055], [13870], (512, 256, 1, 0, True)),                                    # 264
    (16, 1, 128, [4116], [20000], (512, 256, 1, 0, True)),                                   # 258, as many runs as fit the static scratch
    (16, 2, 64, [1270] + [1] * 3, [18176] + [7000, 2000, 300], (512, 256, 1, 1, True)),
    (32, 2, 128, [2143] + [1] * 5, [51899] + [57495] * 5, (512, 256, 1, 1, True)),           # 268, with partial results of the decodes
    (16, 2, 64, [1424] + [1] * 8, [0] + [2000] * 8, (512, 256, 8, 1, True)),
    (32, 8, 128, [2048], [0], (256, 128, 1, 0, False)),                                      # small workgroups: two full rows of 256
    (40, 8, 128, [1000], [0], (256, 128, 1, 0, False)),                                      # one and a part
    (32, 8, 64, [2048, 300], [0, 5], (256, 128, 1, 0, False)),                               # two and a part
    (48, 3, 128, [904], [0], (256, 128, 1, 0, False)),                                       # rows of 85 workgroups per KV head
    (64, 8, 64, [2544], [0], (256, 128, 1, 0, False)),                                       # more than the chip takes at once: not turned
    (32, 8, 128, [2048, 1], [0, 2500], (256, 128, 4, 0, False)),                             # decodes by whole workgroups of four waves
    (15, 3, 128, [1092, 1, 1], [0, 597, 1329], (256, 128, 4, 0, False)),                     # with partial results
    (105, 7, 64, [387, 1, 1], [0, 24, 1038], (256, 128, 4, 0, False)),
    (30, 2, 128, [841, 1, 1], [213, 17, 4613], (256, 128, 1, 0, False)),                     # by single waves, five teams and one
    (32, 8, 128, [256], [3000], (512, 128, 1, 0, False)),                                    # few items: cut evenly
    (12, 4, 128, [837, 1], [830, 29], (512, 256, 1, 0, False)),
]


@pytest.mark.parametrize("Hq,Hkv,D,q_len,ctx,form", CHUNK_FORMS)
def test_records_that_the_kernels_read(tc, records_of, Hq, Hkv, D, q_len, ctx, form):
    """Every form of a chunk: the work list covers the batch, and the records name its items, pieces, regions, counters and pages."""
    sp = W.custom_spec("records", Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(16))
    info = check_work_list(tc, sp, table, nb)
    levelled = info.num_prefill_workgroups < info.num_prefill_pieces
    assert (info.block_threads, info.rows_per_prefill_item, info.waves_per_item, info.decode_queue, levelled) == form
    qs = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    p = tc.Plan(tc.make_pool(Hq, Hkv, D, nb), qs, sp.ctx_len, table, host_only=True)
    items, pieces, first = p.items(0), p.items(3), p.items(4)
    (n_counters, stride), rec = records_of(sp, table, nb)
    assert n_counters == info.num_counters and len(rec) * Hkv == info.num_prefill_pieces
    t0, t1, k, c, region, counter, cstride, nxt, pos0, npos, qrow0, ctx_, pageoff, n_pages, block = rec[:, :15].T
    # chains: from the record of every workgroup to the one marked last, each record once
    n_wg, seen = info.num_prefill_workgroups // Hkv, []
    chains = []
    for i in range(n_wg):
        chain = []
        while i >= 0:
            assert i < len(rec) and len(chain) <= len(rec)
            chain.append(i)
            i = int(nxt[i])
        chains.append(chain)
    assert sorted(sum(chains, [])) == list(range(len(rec)))
    # what tc_plan_copy_items says is in these chains, in the order of the launch
    assert first.tolist() == list(np.cumsum([0] + [len(chains[w // Hkv]) for w in range(n_wg * Hkv)])[:-1])
    order = np.array([i * Hkv + h for chain in chains for h in range(Hkv) for i in chain])
    i, h = order // Hkv, order % Hkv
    assert np.array_equal(pieces[:, 0], block[i] * Hkv + h) and np.array_equal(pieces[:, 1:3], np.stack([t0[i], t1[i]], 1))
    cut = k > 1
    assert np.array_equal(pieces[:, 3], np.where(cut[i], region[i] + h * k[i], -1)) and np.array_equal(pieces[:, 4:6], np.stack([k[i], c[i]], 1))
    assert np.all((region >= 0) == cut) and np.all(cstride == stride) and np.all(counter % stride == 0)
    assert np.array_equal(pieces[:, 6], np.where(cut[i], counter[i] // stride + h, -1))
    # the item's own fields, and the page ids of the first four tiles (past the end: the last page)
    mine = items[block * Hkv]
    assert np.array_equal(np.stack([pos0, npos, qrow0, ctx_, pageoff, n_pages], 1), mine[:, 2:8])
    for r in range(len(rec)):
        row = table[mine[r, 0]]
        assert np.array_equal(rec[r, 16:], row[np.minimum(t0[r] * 4 + np.arange(16), n_pages[r] - 1)]), r


COUNTER_IMAGE = """
#include <cstdio>
#include <cstdlib>
#include "tc_internal.h"
int main(int argc, char **argv) {
    const int seqs = atoi(argv[1]), ctx = atoi(argv[2]), heads = atoi(argv[3]);
    tc_kv_pool pool = {};
    pool.num_q_heads = pool.num_kv_heads = heads; pool.head_dim = 64; pool.block_size = 16; pool.dtype = TC_BF16; pool.num_blocks = 1;
    std::vector<int32_t> q_start(seqs + 1), ctx_len(seqs, ctx), table((size_t)seqs * (ctx / 16 + 1), 0);
    for (int s = 0; s <= seqs; s++) q_start[s] = s;
    tc_batch b = {seqs, q_start.data(), ctx_len.data(), table.data(), ctx / 16 + 1};
    tc_plan *p = nullptr;
    if (tc_plan_create_host(&pool, &b, &p)) return 1;
    printf("%d %d %zu\\n", p->n_counters, p->counter_stride, (p->host_n - p->off_counters) * sizeof(int32_t));
    tc_plan_destroy(p);
}
"""


def test_arrival_counters_take_a_bounded_share_of_the_uploaded_image(tc, tmp_path):
    """A line each for the pairs of few long decodes; closer together when there are many, so that clearing and uploading
    them stays a small part of a plan update (32 KiB, or 4 bytes each beyond 8192 pairs)."""
    src, exe, lib_dir = tmp_path / "t.cpp", tmp_path / "t", os.path.dirname(tc.LIB_PATH)
    src.write_text(COUNTER_IMAGE)
    cmd = f"g++ -std=c++17 -I {ROOT}/include -I {lib_dir}/csrc {src} {tc.LIB_PATH} -Wl,-rpath,{lib_dir} -Wl,-rpath-link,/opt/rocm/lib -o {exe}"
    assert os.system(cmd) == 0
    for seqs, pairs, stride, size in [(1, 8, 32, 1024), (32, 256, 32, 32768), (33, 264, 16, 16896), (512, 4096, 2, 32768), (2000, 16000, 1, 64000)]:
        out = os.popen(f"LD_LIBRARY_PATH=/opt/rocm/lib {exe} {seqs} 20000 8").read().split()
        assert [int(x) for x in out] == [pairs, stride, size], seqs


@pytest.mark.parametrize("Hq,Hkv,D,chunk,offset,decodes,queue,split", [
    (32, 8, 128, 256, 1234, [2000] * 256, 1, 256),         # long sequences, eight rounds of shorter splits
    (32, 8, 128, 256, 1234, [1998] * 256, 0, 1024),        # 1999 tokens on the mean: as long as they are, and 2.3 rounds of them
    (32, 8, 64, 256, 1234, [2600] * 256, 1, 512),          # at head_dim 64 no shorter than the same bytes
    (32, 8, 128, 256, 1234, [2300] * 128 + [9000], 1, 256),  # a sequence that takes two workgroups keeps its splits
    (32, 8, 128, 256, 1234, [1023] * 74, 1, 128),          # 310 MB
    (32, 8, 128, 256, 1234, [1023] * 71, 0, 128),          # and 298
    (32, 8, 128, 256, 1234, [1800] * 66, 0, 256),          # 2.36 rounds of the units that the chunk leaves free
    (32, 8, 128, 256, 1234, [1800] * 68, 1, 256),          # and 2.43
    (32, 8, 128, 256, 1234, [2000] * 84 + [9000], 0, 256),   # with partial results 3.18 rounds of 730 MB
    (32, 8, 128, 256, 1234, [2000] * 85 + [9000], 1, 256),   # and 3.21
    (32, 8, 128, 256, 1234, [2600] * 71 + [9000], 0, 256),   # 2.7 rounds of 794 MB
    (32, 8, 128, 256, 1234, [2600] * 72 + [9000], 1, 256),   # and 805
])
def test_long_decode_streams_beside_a_few_sweeps_are_drawn(tc, Hq, Hkv, D, chunk, offset, decodes, queue, split):
    sp = W.custom_spec("few", Hq, Hkv, D, [chunk] + [1] * len(decodes), [offset] + decodes)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(19))
    info = check_work_list(tc, sp, table, nb)
    assert 0 < info.num_prefill_workgroups <= 64 and info.waves_per_item == 1, info.waves_per_item
    assert (info.decode_queue, info.split_tokens) == (queue, split)


DEALT = """
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <vector>
#include "tc_internal.h"
int main(int argc, char **argv) {  // heads, KV heads, head_dim, then q_len ctx_len of every sequence -> units dealt, prefill and decode workgroups, units, drawers
    std::vector<int32_t> q_start(1, 0), ctx;
    int most = 1;
    for (int i = 4; i + 1 < argc; i += 2) {
        q_start.push_back(q_start.back() + atoi(argv[i]));
        ctx.push_back(atoi(argv[i + 1]));
        most = std::max(most, (atoi(argv[i]) + atoi(argv[i + 1])) / 16 + 1);
    }
    std::vector<int32_t> table(ctx.size() * most, 0);
    tc_kv_pool pool = {};
    pool.num_q_heads = atoi(argv[1]); pool.num_kv_heads = atoi(argv[2]); pool.head_dim = atoi(argv[3]); pool.block_size = 16; pool.dtype = TC_BF16; pool.num_blocks = 1;
    tc_batch b = {(int32_t)ctx.size(), q_start.data(), ctx.data(), table.data(), most};
    tc_plan *p = nullptr;
    if (tc_plan_create_host(&pool, &b, &p)) return 1;
    printf("%d %d %d %d %d\\n", p->n_dealt, p->n_prefill_wg, p->n_decode_wg, p->n_decode / p->items_per_wg, p->n_drawers);
    tc_plan_destroy(p);
}
"""


@pytest.fixture(scope="module")
def launch_of(tc, tmp_path_factory):
    d = tmp_path_factory.mktemp("dealt")
    src, exe, lib_dir = d / "t.cpp", d / "t", os.path.dirname(tc.LIB_PATH)
    src.write_text(DEALT)
    assert os.system(f"g++ -std=c++17 -I {ROOT}/include -I {lib_dir}/csrc {src} {tc.LIB_PATH} -Wl,-rpath,{lib_dir} -Wl,-rpath-link,/opt/rocm/lib -o {exe}") == 0

    def run(Hq, Hkv, D, q_len, ctx):
        args = " ".join(f"{q} {c}" for q, c in zip(q_len, ctx))
        return tuple(int(x) for x in os.popen(f"LD_LIBRARY_PATH=/opt/rocm/lib {exe} {Hq} {Hkv} {D} {args}").read().split())
    return run


@pytest.fixture(scope="module")
def dealt_units(launch_of):
    return lambda *batch: launch_of(*batch)[:4]


@pytest.mark.parametrize("Hq,Hkv,D,q_len,ctx,expected", [
    # units dealt, prefill workgroups, decode workgroups, units
    (32, 8, 128, [2048] + [1] * 64, [4096] + [1000] * 64, (128, 256, 0, 512)),                   # half of the compute units
    (40, 8, 128, [701, 333, 45] + [1] * 16, [0, 0, 0] + [1000] * 16, (104, 176, 80, 128)),       # three blocks of light sweeps
    (16, 2, 64, [1000, 800] + [1] * 30, [0, 100] + [700] * 30, (60, 226, 30, 60)),               # all there are
    (16, 1, 128, [1500] + [1] * 40, [0] + [900] * 40, (40, 144, 40, 40)),                        # own workgroups for all of them
    (32, 8, 128, [1024] + [1] * 4, [4096] + [900] * 4, (8, 248, 8, 32)),                         # level runs have no light ones
    (128, 8, 64, [135, 1, 1], [2105, 4662, 2698], (40, 216, 40, 64)),                            # nor where each of them is a piece
    (64, 8, 64, [279] + [1] * 173, [1392] + [133] * 173, (112, 144, 112, 346)),
    (8, 8, 128, [30, 1649, 8, 1, 1], [3957, 319, 2863, 2877, 2940], (40, 216, 40, 64)),
    (32, 8, 128, [256] + [1] * 74, [1234] + [1023] * 74, (224, 32, 224, 592)),                   # more own workgroups than half of the units
])
def test_decode_units_that_workgroups_begin_with(dealt_units, Hq, Hkv, D, q_len, ctx, expected):
    assert dealt_units(Hq, Hkv, D, q_len, ctx) == expected


@pytest.mark.parametrize("Hq,Hkv,D,chunk,offset,decodes,threads", [
    (32, 8, 128, 20, 0, [200] * 16, 256),         # 128 pairs
    (32, 8, 128, 20, 0, [200] * 15, 512),         # and 120
    (32, 8, 128, 300, 0, [767] * 60, 256),
    (32, 8, 128, 300, 0, [768] + [767] * 59, 512),  # a longer decode
    (8, 8, 64, 24, 744, [100] * 40, 256),         # 12 tiles
    (8, 8, 64, 24, 745, [100] * 40, 512),         # and 13
    (32, 32, 128, 100, 0, [500] * 73, 256),       # 599 MB
    (32, 32, 128, 100, 0, [500] * 74, 512),       # and 607
    (32, 32, 64, 256, 0, [50] * 30, 256),
    (32, 32, 64, 512, 0, [50] * 30, 512),         # 128 items
    (16, 2, 128, 5, 3, [100] * 64, 256),
])
def test_short_decodes_beside_few_sweeps_run_in_small_workgroups(tc, Hq, Hkv, D, chunk, offset, decodes, threads):
    sp = W.custom_spec("short", Hq, Hkv, D, [chunk] + [1] * len(decodes), [offset] + decodes)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(20))
    info = check_work_list(tc, sp, table, nb)
    assert info.block_threads == threads


@pytest.mark.parametrize("Hq,Hkv,D,q_len,ctx", [
    (255, 255, 64, [600, 1, 1], [3000, 100, 200]),                      # a run to every unit but one
    (256, 256, 64, [69, 20, 1, 1], [8000, 0, 101, 501]),
    (257, 257, 64, [109, 7, 1], [3160, 0, 69]),                         # one KV head more than there are units
    (257, 257, 128, [200, 1, 1], [4000, 100, 200]),
    (280, 280, 64, [25, 58, 1, 1, 1], [0, 3306, 25, 129, 17]),
    (300, 300, 64, [69, 1, 1, 1], [8000, 101, 501, 41]),
    (300, 300, 128, [600, 1, 1], [3000, 400, 900]),
    (600, 300, 64, [99, 86, 1], [0, 8651, 228]),
    (514, 257, 64, [138, 1, 1], [21684, 23, 111]),                      # workgroups of four waves
    (2080, 260, 128, [3, 12] + [1] * 6, [0, 25912, 296, 545, 18, 975, 1885, 114]),
    (512, 512, 128, [300, 1, 1], [100, 900, 41]),
    (1024, 1024, 64, [2, 1], [5, 3000]),
    (1024, 1024, 128, [70, 30, 1, 1], [0, 900, 8, 64]),
])
def test_every_decode_unit_has_a_workgroup_that_runs_it(tc, launch_of, Hq, Hkv, D, q_len, ctx):
    """More KV heads than compute units, and about as many: a unit has a workgroup of its own, or there are workgroups that draw."""
    sp = W.custom_spec("many_heads", Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(21))
    info = check_work_list(tc, sp, table, nb)
    dealt, n_prefill, n_decode, units, drawers = launch_of(Hq, Hkv, D, q_len, ctx)
    assert info.grid_blocks == n_prefill + n_decode and units > 0
    if drawers == 0:                                     # a workgroup for every unit
        assert n_decode == units and dealt == 0 and info.decode_queue == 0
    elif info.decode_queue:                              # everybody draws, and runs from the start
        assert drawers == n_prefill + n_decode <= 256 and n_decode <= dealt <= units
    else:                                                # the decode workgroups draw, behind more sweeps than the chip takes at once
        assert drawers == n_decode == units and dealt == 0 and n_prefill > 256


@pytest.mark.parametrize("Hq,Hkv,D,chunk,offset,decodes,waves,drawn", [
    (64, 8, 128, 1500, 255, [3000] + [400] * 120, 1, False),   # 23.5 tiles a unit
    (64, 8, 128, 1500, 272, [3000] + [400] * 120, 1, True),    # and 24.6
    (64, 8, 128, 2000, 255, [2500] * 10, 8, False),            # whole workgroups: 39.8
    (64, 8, 128, 2000, 272, [2500] * 10, 8, True),             # and 40.8
    (128, 8, 128, 1584, 280, [600] * 100 + [5000] * 3, 8, False),  # 3.6 times as many units as compute units: 53.5
    (128, 8, 128, 1584, 304, [600] * 100 + [5000] * 3, 8, True),   # and 54.5
    (64, 8, 64, 2000, 3440, [3000, 100], 1, False),            # 139
    (64, 8, 64, 2000, 3504, [3000, 100], 1, True),             # and 140.3
    (64, 8, 64, 2000, 4980, [700] * 200, 1, False),            # 3.1 times as many units: 187
    (64, 8, 64, 2000, 5040, [700] * 200, 1, True),             # and 187.5
])
def test_decodes_behind_long_sweeps_are_drawn_by_their_own_workgroups(tc, launch_of, Hq, Hkv, D, chunk, offset, decodes, waves, drawn):
    """More sweeps than units.  tc_plan_info.decode_queue says 0 for both: no prefill workgroup draws."""
    q_len, ctx = [chunk] + [1] * len(decodes), [offset] + decodes
    sp = W.custom_spec("late", Hq, Hkv, D, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(22))
    info = check_work_list(tc, sp, table, nb)
    dealt, n_prefill, n_decode, units, drawers = launch_of(Hq, Hkv, D, q_len, ctx)
    assert n_prefill > 256 and n_decode == units > 0 and dealt == 0
    assert (info.block_threads, info.waves_per_item, info.decode_queue) == (512, waves, 0) and drawers == (units if drawn else 0)
    assert drawn == (sum(-(-(offset + min(chunk, a + 256 * Hkv // Hq)) // 64) for a in range(0, chunk, 256 * Hkv // Hq)) * Hkv
                     >= max({(128, 1): 24, (128, 8): 40, (64, 1): 140}[D, waves] * 256, {(128, 1): 0, (128, 8): 15, (64, 1): 60}[D, waves] * units))


@pytest.mark.parametrize("name", ["waves", "waves_d64", "whole"])
def test_queue_of_the_decode_workgroups_in_the_gpu_tests(launch_of, name):
    """The batches that the GPU tests launch several times do have that queue, and draw more units than one."""
    from test_gpu_parity import LATE_QUEUE
    Hq, Hkv, D, q_len, ctx, dtype, waves = LATE_QUEUE[name]
    dealt, n_prefill, n_decode, units, drawers = launch_of(Hq, Hkv, D, q_len, ctx)
    assert n_prefill > 256 and dealt == 0 and drawers == n_decode == units > 1


def test_split_tokens_bounds_all_but_the_long_sequences_of_a_shortened_stream(tc):
    """128 decodes of 2300 tokens in splits of at most 256 (a workgroup covers them: eight splits, of 18 pages) and one of 9000 in longer ones."""
    q_len, ctx = [256] + [1] * 129, [1234] + [2300] * 128 + [9000]
    sp = W.custom_spec("splits", 32, 8, 128, q_len, ctx)
    table, mb, nb = W.make_tables(sp, np.random.default_rng(23))
    info = check_work_list(tc, sp, table, nb)
    qs = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    dc = tc.Plan(tc.make_pool(32, 8, 128, nb), qs, sp.ctx_len, table, host_only=True).items(1)
    longest = lambda seqs: int((dc[:, 3] - dc[:, 2])[np.isin(dc[:, 0], seqs)].max())
    assert (info.split_tokens, longest(range(1, 129)), longest([129])) == (256, 288, 384)
