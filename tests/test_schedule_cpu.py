"""The host planner against the block mask: the work items of a call cover exactly the visible
(query token, key token) pairs of the Block-attention mask (Section 2.1, 2.4, 2.5), none twice, and no
item walks a key tile in which none of its rows sees anything.  Host only: the items come from the
code the calls themselves plan with, and the key-range arithmetic of a split is the kernel's."""
import numpy as np
import pytest

import oracle
from paper_2409_15355_amd import binding as ba


@pytest.fixture(scope="module", autouse=True)
def lib():
    import os
    if not os.path.exists(ba.LIB_PATH):
        from paper_2409_15355_amd import build
        build.build()
    return ba.load()


def coverage_of(items, G, problem_rows):
    """count[problem][token, key] over the items; keys = (context keys..., own tokens...).
    problem_rows: {problem: (n_ctx_keys, n_tokens)}.  Also checks the per-item invariants.
    Items that name their KV head (splits sized by XCD speed) are checked head by head: every head's
    items must give the same, complete coverage."""
    heads_named = sorted({w.kv_head for w in items})
    if heads_named and heads_named != [-1]:
        assert -1 not in heads_named
        covs = [_coverage_of([w for w in items if w.kv_head == h], G, problem_rows) for h in heads_named]
        for c in covs[1:]:
            assert all(np.array_equal(c[p], covs[0][p]) for p in c)
        return covs[0]
    return _coverage_of(items, G, problem_rows)


def _coverage_of(items, G, problem_rows):
    cov = {p: np.zeros((lq, tc + lq), dtype=np.int32) for p, (tc, lq) in problem_rows.items()}
    seen_rows = {p: np.zeros(lq * G, dtype=np.int32) for p, (tc, lq) in problem_rows.items()}
    for w in items:
        tc, lq = problem_rows[w.problem]
        assert 0 <= w.row_begin < w.row_end <= lq * G and w.row_end - w.row_begin <= w.tile_rows
        assert w.row_begin % w.tile_rows == 0
        assert 0 <= w.ctx_begin <= w.ctx_end <= tc and 0 <= w.self_begin <= w.self_end <= lq
        # whole key tiles, cut at the end of a segment
        assert w.ctx_begin % w.tile_keys == 0 or w.ctx_begin == tc
        assert w.self_begin % w.tile_keys == 0 or w.self_begin == lq
        toks = np.arange(w.row_begin, w.row_end) // G
        last_tok = int(toks[-1])
        # no fully masked tile: every tile of the causal range starts at or before the last row's token
        if w.self_end > w.self_begin:
            last_tile_key0 = (w.self_end - 1) // w.tile_keys * w.tile_keys
            assert last_tile_key0 <= last_tok, (w.problem, w.row_begin, w.self_begin, w.self_end)
        if w.split == 0:
            seen_rows[w.problem][w.row_begin:w.row_end] += 1
        for t in np.unique(toks):
            heads_here = int((toks == t).sum())  # every head of the group is a row: count a pair once per row
            cov[w.problem][t, w.ctx_begin:w.ctx_end] += heads_here
            hi = min(w.self_end, t + 1)
            if hi > w.self_begin:
                cov[w.problem][t, tc + w.self_begin:tc + hi] += heads_here
    for p, rows in seen_rows.items():
        assert (rows == 1).all(), f"problem {p}: rows not covered exactly once per split"
    return cov


def expected_final(tc, lq, G):
    """The mask of Section 2.5 for one prompt, from the oracle's block mask: context = one block
    per... any earlier blocks (all of them visible to the last block), then the final block."""
    m = oracle.block_mask([0, tc, tc + lq]) if tc else oracle.block_mask([0, lq])
    return m[tc:, :].astype(np.int32) * G


@pytest.mark.parametrize("hq,hkv", [(32, 8), (4, 4), (8, 1)])
@pytest.mark.parametrize("n_cu", [256, 8, 1])
def test_final_block_items_cover_the_mask_exactly(hq, hkv, n_cu):
    rng = np.random.default_rng(7 + hq + n_cu)
    h = ba.Heads(hq, hkv, 128, 500000.0)
    G = hq // hkv
    for case in range(12):
        n_prompts = int(rng.integers(1, 5))
        lqs = [int(rng.choice([1, 17, 64, 65, 130, 256])) for _ in range(n_prompts)]
        tcs = [int(rng.choice([0, 1, 63, 64, 700, 3001, 9000])) for _ in range(n_prompts)]
        cu_q, cu_ctx = np.concatenate([[0], np.cumsum(lqs)]), np.concatenate([[0], np.cumsum(tcs)])
        items = ba.ba_schedule_final_block(h, cu_q, cu_ctx, n_cu)
        assert len({w.n_splits for w in items}) == 1
        cov = coverage_of(items, G, {p: (tcs[p], lqs[p]) for p in range(n_prompts)})
        for p in range(n_prompts):
            assert np.array_equal(cov[p], expected_final(tcs[p], lqs[p], G)), (case, p, lqs, tcs)
        assert all(w.first_token == cu_q[w.problem] for w in items)


def test_config5_schedule_is_the_one_the_design_states():
    h = ba.Heads(32, 8, 128, 500000.0)
    items = ba.ba_schedule_final_block(h, [0, 256], [0, 31744], 256)
    assert len(items) == 8 * 4 and {w.n_splits for w in items} == {8}   # x 8 KV heads = 256 workgroups
    tiles = lambda w: (w.ctx_end - w.ctx_begin + w.self_end - w.self_begin) // 64
    per_split = sorted({(w.split, tiles(w)) for w in items if w.row_begin == 0})
    # equal shares, except that the split with the causal tiles gets fewer
    assert [t for _, t in per_split][:-1] == [62] * 6 + [63] or max(t for _, t in per_split) - min(t for _, t in per_split) <= 4
    assert per_split[-1][1] < per_split[0][1]


@pytest.mark.parametrize("hq,hkv", [(32, 8), (4, 4), (2, 1)])
def test_encode_items_cover_the_block_diagonal_mask_exactly(hq, hkv):
    rng = np.random.default_rng(11 + hq)
    h = ba.Heads(hq, hkv, 64, 10000.0)
    G = hq // hkv
    for case in range(8):
        lens = [int(x) for x in rng.choice([0, 1, 31, 32, 33, 100, 257, 300], size=int(rng.integers(1, 9)))]
        if case == 0:
            lens = [7000, 5, 0, 6144, 6145]   # both schedules in one call (the long-block core beyond 6144 tokens)
        offs = np.concatenate([[0], np.cumsum(lens)])
        items = ba.ba_schedule_encode_blocks(h, offs)
        live = {b: (0, lens[b]) for b in range(len(lens)) if lens[b] > 0}
        assert {w.problem for w in items} == set(live)
        cov = coverage_of(items, G, live)
        mask = oracle.block_mask(np.concatenate([offs, [offs[-1]]]))  # (a trailing empty block: no block is "last")
        for b, (_, L) in live.items():
            want = mask[offs[b]:offs[b] + L, offs[b]:offs[b] + L].astype(np.int32) * G
            assert np.array_equal(cov[b], want), (case, b, lens)
            assert not mask[offs[b]:offs[b] + L, :offs[b]].any()
        if case == 0 and G >= 4:
            assert {w.tile_rows for w in items if w.problem in (0, 4)} == {256}
            assert {w.tile_rows for w in items if w.problem in (1, 3)} == {128}


@pytest.mark.parametrize("d", [64, 128])
def test_small_groups_encode_on_the_main_core_where_few_long_blocks_leave_compute_units_idle(d):
    """Fewer than four query heads per KV head: small workgroups up to 512 tokens a block, and above where there
    is enough work for them; a few long blocks keep the main core.  One schedule for all of a call's blocks."""
    tile_rows = lambda hq, hkv, lens: {w.tile_rows for w in ba.ba_schedule_encode_blocks(
        ba.Heads(hq, hkv, d, 10000.0), np.concatenate([[0], np.cumsum(lens)]))}
    for g in (1, 2, 3):
        assert tile_rows(8 * g, 8, [128]) == tile_rows(8 * g, 8, [512]) == {128}
        assert tile_rows(8 * g, 8, [512, 1, 300]) == {128}
        assert tile_rows(8 * g, 8, [513]) == tile_rows(8 * g, 8, [2048]) == {256}
        assert tile_rows(2 * g, 2, [6144]) == tile_rows(2 * g, 2, [6000] + [200] * 40) == {256}
        assert tile_rows(8 * g, 8, [1000] * 33) == {128}
    assert tile_rows(16, 8, [6000] + [200] * 160) == tile_rows(8, 8, [6144, 6144]) == {128}
    assert tile_rows(8, 8, [6144]) == tile_rows(16, 8, [2048, 2048]) == {256}
    for g in (4, 8):  # (from four on by a block's own length)
        assert tile_rows(8 * g, 8, [6144]) == tile_rows(g, 1, [513]) == {128}
        assert tile_rows(g, 1, [6145, 5]) == {128, 256}


@pytest.mark.parametrize("hq,hkv", [(32, 8), (8, 2)])
def test_whole_prompt_items_cover_the_mask_of_section_2_4_exactly(hq, hkv):
    rng = np.random.default_rng(13 + hq)
    h = ba.Heads(hq, hkv, 128, 500000.0)
    G = hq // hkv
    for case in range(8):
        n_prompts = int(rng.integers(1, 4))
        cu_blk, lens = [0], []
        for _ in range(n_prompts):
            nb = int(rng.integers(1, 6))
            lens += [int(x) for x in rng.choice([0, 1, 31, 33, 100, 257], size=nb - 1)] + [int(rng.choice([1, 32, 70]))]
            cu_blk.append(len(lens))
        offs = np.concatenate([[0], np.cumsum(lens)])
        items = ba.ba_schedule_prompts(h, cu_blk, offs)
        T = int(offs[-1])
        count = np.zeros((T, T), dtype=np.int32)
        rows_seen = np.zeros(T * G, dtype=np.int32)
        for w in items:
            p0 = int(offs[cu_blk[w.problem]])          # first token of the prompt
            blk_len = None
            b = int(np.searchsorted(offs, w.first_token, side="right") - 1)
            while lens[b] == 0:
                b += 1
            assert offs[b] == w.first_token
            blk_len = lens[b]
            is_last = b == cu_blk[w.problem + 1] - 1
            dq = w.first_token - p0 if is_last else 0
            assert w.ctx_begin == 0 and w.ctx_end <= dq
            toks = np.arange(w.row_begin, w.row_end) // G
            assert toks[-1] < blk_len
            rows_seen[w.first_token * G + w.row_begin:w.first_token * G + w.row_end] += 1
            for t in np.unique(toks):
                nh = int((toks == t).sum())
                count[w.first_token + t, p0:p0 + w.ctx_end] += nh
                hi = min(w.self_end, t + 1)
                count[w.first_token + t, w.first_token:w.first_token + hi] += nh
            # the walk reaches the last row's own token, and its last key tile is not fully masked
            walked = w.ctx_end + w.self_end
            assert walked >= min(dq + toks[-1] + 1, dq + blk_len) and (walked - 1) // 32 * 32 <= dq + toks[-1]
        assert (rows_seen == 1).all()
        want = np.zeros((T, T), dtype=np.int32)
        for n in range(n_prompts):
            o = offs[cu_blk[n]:cu_blk[n + 1] + 1]
            m = oracle.block_mask(o - o[0])
            want[o[0]:o[-1], o[0]:o[-1]] = m.astype(np.int32) * G
        assert np.array_equal(count, want), (case, lens, cu_blk)


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (8, 2, 64), (32, 8, 128), (6, 2, 128)])
def test_shared_walks_of_whole_prompts_cover_the_mask_once(hq, hkv, d):
    """Last blocks behind long prompts: the splits of a row tile partition its walk, in order, and every visible
    pair belongs to exactly one work item; prompts at the edge of the rule are left alone."""
    G = hq // hkv
    h = ba.Heads(hq, hkv, d, 10000.0)
    seen = set()
    for lens_of in ([[1152]], [[1120, 32]], [[1121, 32]], [[700, 0, 800, 33]], [[3000, 2500, 1]], [[5000, 70], [40, 7], [1300, 300]]):
        cu_blk = np.concatenate([[0], np.cumsum([len(p) for p in lens_of])])
        offs = np.concatenate([[0], np.cumsum([n for p in lens_of for n in p])])
        items = ba.ba_schedule_prompts(h, cu_blk, offs)
        for n, p in enumerate(lens_of):
            p0, last, lq = int(offs[cu_blk[n]]), int(offs[cu_blk[n + 1] - 1]), p[-1]
            ctx = last - p0
            tiles = {}
            for w in items:
                if w.problem == n and w.first_token == last:
                    tiles.setdefault(w.row_begin, []).append(w)
            assert sorted(tiles) == list(range(0, lq * G, 128))
            for ws in tiles.values():
                ws.sort(key=lambda w: w.split)
                seen.add(ws[0].n_splits)
                # (by the block's own walk, and row tiles times KV heads of up to half of 24)
                shared = ctx > 0 and (ctx + lq - 1) // 32 + 1 > 36 and len(tiles) * hkv <= 12
                assert (ws[0].n_splits > 1) == shared
                assert [w.split for w in ws] == list(range(ws[0].n_splits))
                at = 0
                for w in ws:
                    begin, end = w.ctx_begin + w.self_begin, w.ctx_end + w.self_end
                    assert begin == at and end >= begin
                    at = end
                last_tok = (ws[0].row_end - 1) // G
                assert at == min(ctx + lq, ((ctx + last_tok) // 32 + 1) * 32)
    assert 1 in seen and max(seen) >= (4 if hq <= 6 else 2)


@pytest.mark.parametrize("hq,hkv,d,prompt,parts", [
    (32, 8, 128, [880, 860, 51], 3), (32, 8, 128, [880, 861, 51], 3), (32, 8, 128, [880, 828, 51], 1),  # 56, 56 and 55 key tiles
    (8, 1, 64, [1600, 192], 2), (8, 1, 64, [1600, 193], 4),                           # 12 row tiles times KV heads, 13
    (32, 8, 128, [1500, 1500, 1500, 260], 2), (32, 8, 128, [1500, 1500, 1500, 400], 1),  # 72 and 104: at most 192 workgroups
    (4, 4, 64, [2000, 2000, 1700], 3), (16, 16, 64, [1500, 1500, 100], 1)])
def test_walks_of_many_row_tiles_are_shared_from_56_key_tiles_on(hq, hkv, d, prompt, parts):
    """More than twelve row tiles times KV heads: parts of 24 key tiles (16 at head_dim 64), at most 192 workgroups, at most twelve KV heads; the
    parts of a row tile partition its walk."""
    h, G = ba.Heads(hq, hkv, d, 10000.0), hq // hkv
    offs = np.concatenate([[0], np.cumsum(prompt)])
    last = int(offs[-2])
    tiles = {}
    for w in ba.ba_schedule_prompts(h, [0, len(prompt)], offs):
        if w.first_token == last:
            tiles.setdefault(w.row_begin, []).append(w)
    assert sorted(tiles) == list(range(0, prompt[-1] * G, 128))
    for ws in tiles.values():
        ws.sort(key=lambda w: w.split)
        assert [w.split for w in ws] == list(range(parts)) and {w.n_splits for w in ws} == {parts}
        at = 0
        for w in ws:
            assert w.ctx_begin + w.self_begin == at
            at = w.ctx_end + w.self_end
        last_tok = (ws[0].row_end - 1) // G
        assert at == min(last + prompt[-1], ((last + last_tok) // 32 + 1) * 32)


@pytest.mark.parametrize("hkv", [8, 9, 12, 13, 16, 32])
@pytest.mark.parametrize("d", [64, 128])
def test_walks_are_shared_up_to_twelve_kv_heads(hkv, d):
    """... whatever the last block: with more a prompt is computed the same way in every batch.  With up to twelve, blocks of many row tiles
    as well as few."""
    for group, last in ((4, 64), (2, 200), (4, 20), (1, 50)):
        h, prompt = ba.Heads(hkv * group, hkv, d, 10000.0), [200] * 20 + [last]
        offs = np.concatenate([[0], np.cumsum(prompt)])
        assert (max(w.n_splits for w in ba.ba_schedule_prompts(h, [0, 21], offs)) > 1) == (hkv <= 12), (group, last)


@pytest.mark.parametrize("hq,hkv,d,prompt,most", [
    # groups of four: from 0.7 of the load on at head_dim 128, 0.8 at 64 (the forward pass: 0.64)
    (32, 8, 128, [200] * 20 + [64], 4), (32, 8, 64, [200] * 20 + [64], 3),
    # of one and two from 0.86 and from 1.1 on, of eight as the forward pass
    (16, 8, 128, [200] * 20 + [100], 4), (8, 8, 64, [115] * 28 + [268], 6), (16, 2, 64, [200] * 20 + [150], 7),
    # up to twelve KV heads
    (48, 12, 128, [200] * 20 + [64], 2), (52, 13, 128, [200] * 20 + [64], 0), (64, 16, 64, [200] * 20 + [64], 0)])
def test_the_dq_kernel_shares_walks_of_many_row_tiles_by_a_line_of_its_own(hq, hkv, d, prompt, most):
    """Of up to how many such prompts a backward call shares the walks: what its query names beyond what the call cannot do without is the
    partial results (the dk/dv kernel alone asks for none in calls of these prompts)."""
    up = lambda n: (n + 255) // 256 * 256

    def least(T):
        padded, g = 0, hq // hkv
        if g < 4:
            padded, g = 4 * up(T * hkv * 4 * d * 2) + up(T * hkv * 16), 4
        return padded + up(T * hkv * g * d * 2) + up(T * hkv * d * 2) + up(T * d * 4) + up(T * hkv * ((g + 3) // 4 * 4) * 8 + 16)

    for n in range(1, 11):
        offs = np.concatenate([[0], np.cumsum(prompt * n)])
        size = ba.ba_block_attention_prompts_backward_workspace_bytes(ba.Heads(hq, hkv, d, 10000.0), np.arange(n + 1) * len(prompt), offs)
        assert (size > least(int(offs[-1]))) == (n <= most), n


@pytest.mark.parametrize("hq,hkv,d,prompt,parts", [
    # a passage nearly as long as the whole prompt, whose walk stays: shared only from a quarter more on ...
    (8, 1, 128, [5000, 900], 1), (8, 1, 128, [4000, 1200], 2), (14, 2, 64, [5150, 268], 1), (16, 8, 128, [3450, 105], 1), (14, 2, 64, [2500, 2500, 268], 6),
    # ... or where the chip has little else to do
    (8, 2, 64, [1600, 200], 4), (8, 1, 128, [2000, 400], 4)])
def test_walks_of_many_row_tiles_are_shared_where_no_passage_is_nearly_as_long(hq, hkv, d, prompt, parts):
    offs = np.concatenate([[0], np.cumsum(prompt)])
    assert max(w.n_splits for w in ba.ba_schedule_prompts(ba.Heads(hq, hkv, d, 10000.0), [0, len(prompt)], offs)) == parts


@pytest.mark.parametrize("hq,hkv,d,prompt,below,above", [(32, 8, 128, [200] * 6 + [20], 4, 5), (16, 8, 128, [200] * 20 + [64], 8, 9),
                                                         (4, 4, 64, [200] * 6 + [20], 24, 32)])
def test_walks_are_shared_only_where_the_call_leaves_the_chip_idle(hq, hkv, d, prompt, below, above):
    """The longest shared walk against 0.64 of what every compute unit has to do: one more prompt than the line allows
    and no walk of the call is shared.  Into how many parts a walk is cut does not depend on the batch."""
    h = ba.Heads(hq, hkv, d, 10000.0)
    G = hq // hkv

    def splits(n_prompts):
        offs = np.concatenate([[0], np.cumsum(prompt * n_prompts)])
        cu_blk = np.arange(n_prompts + 1) * len(prompt)
        return {w.n_splits for w in ba.ba_schedule_prompts(h, cu_blk, offs) if w.first_token == offs[cu_blk[w.problem + 1] - 1]}

    def load(n_prompts):  # key tiles of 32 per compute unit, four for what a workgroup does besides
        ctx = sum(prompt[:-1])
        tiles = [-(-n * G // 128) * (0.5 * n / 32 + 4.5) for n in prompt[:-1]] + [-(-prompt[-1] * G // 128) * ((ctx + 0.5 * prompt[-1]) / 32 + 4.5)]
        # (head_dim 128: 24 more for every part beyond a walk's first)
        parts = 2 * -(-prompt[-1] * G // 128) * (24 if d == 128 else 0)
        return n_prompts * (sum(tiles) + parts) * hkv / 256

    walk = (sum(prompt) - 1) // 32 + 1
    assert splits(1) == splits(below) == {3} and walk >= 0.64 * load(below)
    assert splits(above) == splits(64) == {1} and walk < 0.64 * load(above)


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (8, 2, 64), (4, 1, 128)])
def test_walks_are_shared_only_where_no_other_walk_is_as_long(hq, hkv, d):
    """A passage, or a last block of too many row tiles to share, whose walk is as long as the longest that could be cut
    (to a hundredth): the launch would be no shorter.  One key tile less and the walks are cut."""
    h = ba.Heads(hq, hkv, d, 10000.0)
    long_last = [400, 832, 500]  # 55 key tiles; 4, 16 and 16 row tiles times 4, 2 and 1 KV heads
    for prompts, shared in (([[1700, 32], [1500], [1700]], True), ([[1700, 32], [1500], [1732]], False),
                            ([[1200, 532, 28], [1600, 132, 28]], True), ([[1200, 528, 32], long_last, [1600]], False),
                            ([[1200, 560, 32], long_last, [1600]], True)):
        cu_blk = np.concatenate([[0], np.cumsum([len(p) for p in prompts])])
        offs = np.concatenate([[0], np.cumsum([n for p in prompts for n in p])])
        assert (max(w.n_splits for w in ba.ba_schedule_prompts(h, cu_blk, offs)) > 1) == shared, prompts


def test_split_range_arithmetic_partitions_every_walk():
    """split_tile_range through the final-block query: over split counts of 1 to 32 (eight KV heads, by varying the
    compute-unit count; more splits: below), the splits of a row tile partition its walk."""
    h = ba.Heads(8, 8, 64, 10000.0)
    seen_splits = set()
    for n_cu in (1, 2, 3, 5, 8, 13, 16, 24, 32, 64, 100, 256, 1000):
        for tc in (0, 5, 64, 1000, 4097, 20000):
            for lq in (1, 64, 200):
                items = ba.ba_schedule_final_block(h, [0, lq], [0, tc], n_cu)
                seen_splits.add(items[0].n_splits)
                by_tile = {}
                for w in items:
                    by_tile.setdefault(w.row_begin, []).append(w)
                for ws in by_tile.values():
                    ws.sort(key=lambda w: w.split)
                    assert [w.split for w in ws] == list(range(ws[0].n_splits))
                    at_ctx, at_self = 0, 0
                    for w in ws:   # contiguous, in order, nothing skipped
                        if w.ctx_end > w.ctx_begin:
                            assert w.ctx_begin == at_ctx
                            at_ctx = w.ctx_end
                        if w.self_end > w.self_begin:
                            assert w.self_begin == at_self and at_ctx == tc
                            at_self = w.self_end
                    assert at_ctx == tc and at_self == min(lq, ((ws[0].row_end - 1) // 64 + 1) * 64)  # (one head per group: row = token)
    assert len(seen_splits) >= 6 and max(seen_splits) >= 16


def test_more_than_32_splits_only_where_they_were_measured_to_pay():
    """Workgroups per split x head_dim decide: up to four of head_dim 128 and up to seven of 64 take up to 64 splits;
    five of 128 only over contexts long enough for the merge; six and seven of 128 stay at 32."""
    splits = lambda hkv, d, lq, tc: ba.ba_schedule_final_block(ba.Heads(4 * hkv, hkv, d, 500000.0), [0, lq], [0, tc])[0].n_splits
    for tc in (16000, 31950, 64000, 128000):
        assert splits(4, 128, 60, tc) > 32 and splits(1, 128, 60, tc) > 32
        assert splits(6, 128, 60, tc) <= 32 and splits(7, 128, 60, tc) <= 32 and splits(3, 128, 128, tc) <= 32
    for hkv in range(1, 8):
        assert splits(hkv, 64, 50, 64000) > 32
    assert splits(5, 128, 60, 16000) <= 32 < splits(5, 128, 60, 64000)


def test_splits_of_very_long_contexts_stay_within_the_static_scratch():
    """From eight workgroups per split on (row tiles x KV heads) never more than 32 splits, whatever the context, so
    that the partials of such a call do not outgrow the scratch of ba_final_block_attention_static with its
    length, and with measured XCD speeds its splits are still sized by them; fewer workgroups, up to 64, fit too."""
    static = ba.STATIC_SCRATCH_BYTES
    speeds = [1.03, 0.97, 1.02, 0.97, 1.03, 1.0, 1.02, 0.95]
    for hkv, tiles in [(1, 8), (1, 10), (1, 13), (1, 19), (1, 25), (2, 5), (2, 14), (8, 1), (1, 31), (2, 31), (4, 31)]:
        for tc in (430000, 600000, 900000, 1600000):
            cu_q, cu_ctx = [0, 8 * tiles], [0, tc]
            for speed in (None, speeds):
                h = ba.Heads(32 * hkv, hkv, 128, 500000.0, xcd_speed=speed)
                items = ba.ba_schedule_final_block(h, cu_q, cu_ctx)
                assert items[0].n_splits <= 32, (hkv, tiles, tc)
                if speed and items[0].n_splits > 1:
                    assert items[0].kv_head >= 0, (hkv, tiles, tc)   # (a KV head's own shares)
            assert ba.ba_final_block_attention_workspace_bytes(h, cu_q, cu_ctx) <= static, (hkv, tiles, tc)
    for base in range(1, 8):
        for g, hkv, lq in ([(32, 1, 8 * base), (1, base, 256), (32, base, 8)]):
            for tc in (8000, 31950, 128000, 1600000):
                h = ba.Heads(g * hkv, hkv, 128, 500000.0)
                assert ba.ba_final_block_attention_workspace_bytes(h, [0, lq], [0, tc]) <= static, (base, g, hkv, tc)


@pytest.mark.parametrize("hkv,d", [(1, 64), (2, 64), (4, 64), (1, 128), (2, 128), (4, 128)])
def test_walks_cut_into_more_than_32_splits_are_partitioned(hkv, d):
    """33 to 64 splits (few KV heads, contexts of 8,000 to 60,000 tokens): contiguous, in order, nothing skipped, four
    key tiles or more on average; with XCD speeds the same equal splits, the speeds' shares hold 32 at most."""
    speeds = [1.03, 0.97, 1.02, 0.97, 1.03, 1.0, 1.02, 0.95]
    seen = set()
    for tc in (8000, 8191, 12345, 16000, 31950, 47777, 60000):
        for lq in (1, 50, 64):
            plain, sized = (ba.ba_schedule_final_block(ba.Heads(hkv, hkv, d, 10000.0, xcd_speed=s), [0, lq], [0, tc], 256)
                            for s in (None, speeds))
            n = plain[0].n_splits
            seen.add(n)
            if n > 32:
                assert [(w.split, w.ctx_begin, w.ctx_end, w.self_begin, w.self_end) for w in plain] == \
                    [(w.split, w.ctx_begin, w.ctx_end, w.self_begin, w.self_end) for w in sized]
            assert n * 4 <= -(-tc // 64) + 1
            at_ctx = at_self = 0
            for w in sorted(plain, key=lambda w: w.split):  # (one row tile: 64 rows at most)
                if w.ctx_end > w.ctx_begin:
                    assert w.ctx_begin == at_ctx
                    at_ctx = w.ctx_end
                if w.self_end > w.self_begin:
                    assert w.self_begin == at_self and at_ctx == tc
                    at_self = w.self_end
            assert at_ctx == tc and at_self == lq
    assert max(seen) > 32, seen


@pytest.mark.parametrize("speeds", [[1.0] * 8, [0.92, 1.0, 1.08, 1.0, 0.95, 1.05, 1.0, 1.0], [0.5, 2.0, 0.5, 2.0, 1.0, 1.0, 1.0, 1.0]])
def test_splits_sized_by_xcd_speed_still_cover_the_mask_exactly(speeds):
    """ba_heads.xcd_speed moves the boundaries between KV splits (faster XCDs get more key tiles); the
    work items must still cover every visible pair exactly once."""
    rng = np.random.default_rng(5)
    h = ba.Heads(32, 8, 128, 500000.0, xcd_speed=speeds)
    for case in range(6):
        n_prompts = int(rng.integers(1, 4))
        lqs = [int(rng.choice([1, 64, 130, 256])) for _ in range(n_prompts)]
        tcs = [int(rng.choice([0, 700, 3001, 9000, 31744])) for _ in range(n_prompts)]
        if case == 0:
            n_prompts, lqs, tcs = 1, [256], [31744]
        cu_q, cu_ctx = np.concatenate([[0], np.cumsum(lqs)]), np.concatenate([[0], np.cumsum(tcs)])
        items = ba.ba_schedule_final_block(h, cu_q, cu_ctx, 256)
        cov = coverage_of(items, 4, {p: (tcs[p], lqs[p]) for p in range(n_prompts)})
        for p in range(n_prompts):
            assert np.array_equal(cov[p], expected_final(tcs[p], lqs[p], 4)), (case, p, lqs, tcs)
        if case == 0:
            # config 5: 256 workgroups; a split's share of its KV head's key tiles follows the speed of the XCD
            # that runs it (which XCDs a KV head's splits lie on is the planner's choice)
            assert sorted({w.kv_head for w in items}) == list(range(8))
            for kvh in range(8):
                mine = [w for w in items if w.kv_head == kvh and w.row_begin == 0]
                assert [w.split for w in sorted(mine, key=lambda w: w.split)] == list(range(8))
                if len(set(speeds)) == 1:
                    assert {w.xcd for w in mine} == {kvh}   # nothing to balance: an XCD fetches one KV head's query rows
                else:
                    assert len({w.xcd for w in mine}) >= 2  # a KV head's splits lie on XCDs that can be balanced against each other
                tiles = {w.split: (w.ctx_end - w.ctx_begin + w.self_end - w.self_begin) // 64 for w in mine}
                sp = {w.split: speeds[w.xcd] for w in mine}
                if len(set(speeds)) == 1:
                    assert max(tiles[s] for s in range(7)) - min(tiles[s] for s in range(7)) <= 1
                else:
                    share = np.array([tiles[s] / sp[s] for s in range(7)])
                    assert share.max() / share.min() < 1.06   # equal time per split, to a tile
                    if sp[0] != sp[4]:
                        assert (tiles[0] < tiles[4]) == (sp[0] < sp[4])
            # every row tile of a (KV head, split) runs on the same XCD: they share its K/V tiles
            for kvh in range(8):
                for s_ in range(8):
                    assert len({w.xcd for w in items if w.kv_head == kvh and w.split == s_}) == 1


@pytest.mark.parametrize("speeds", [[1.0608, 0.9721, 1.0293, 0.9882, 1.0236, 0.9837, 1.0255, 0.9167],
                                    [1.0393, 0.9966, 0.9955, 0.9547, 1.0547, 0.9905, 1.0048, 0.9638],
                                    [0.93, 0.94, 0.95, 0.96, 1.04, 1.05, 1.06, 1.07]])
def test_xcds_are_dealt_to_kv_head_groups_by_speed(speeds):
    """With measured speeds the planner also chooses which XCD runs which stretch of the work items: XCDs
    that share KV heads can be balanced against each other, so slow ones are put with fast ones.  Every
    XCD still runs an eighth of the launch, and the launch is expected to end within 3 % of the time a
    perfect balance would give (speeds as measured on two devices, and a set sorted the worst way)."""
    h = ba.Heads(32, 8, 128, 500000.0, xcd_speed=speeds)
    items = ba.ba_schedule_final_block(h, [0, 256], [0, 31744], 256)
    assert len(items) == 256
    tiles = lambda w: -(-(w.ctx_end - w.ctx_begin) // 64) - (-(w.self_end - w.self_begin) // 64)
    per_xcd = {x: [w for w in items if w.xcd == x] for x in range(8)}
    assert all(len(v) == 32 for v in per_xcd.values())
    ends = [max(tiles(w) for w in per_xcd[x]) / speeds[x] for x in range(8)]
    ideal = sum(tiles(w) for w in items) / 32.0 / sum(speeds)
    assert max(ends) <= 1.03 * ideal, (ends, ideal)
    hosted = {x: frozenset(w.kv_head for w in per_xcd[x]) for x in range(8)}
    if 1 < len(hosted[0]) < 8:
        # groups of XCDs share KV heads; the slowest XCD sits in a group with the fastest
        assert hosted[int(np.argmin(speeds))] == hosted[int(np.argmax(speeds))]
        groups = {}
        for x in range(8):
            groups.setdefault(hosted[x], []).append(speeds[x])
        means = [np.mean(v) for v in groups.values()]
        assert max(means) - min(means) < 0.02, groups


def test_every_xcd_runs_its_share_whatever_the_speeds():
    """Drawn speeds and shapes: the work items of a launch are dealt to the XCDs in equal numbers (to
    within one), each (KV head, split, row tile) exactly once, whichever XCD runs which stretch."""
    rng = np.random.default_rng(77)
    for case in range(40):
        hkv = int(rng.choice([1, 2, 4, 8]))
        g = int(rng.choice([1, 4, 8]))
        speeds = [float(x) for x in rng.uniform(0.8, 1.25, 8)]
        h = ba.Heads(hkv * g, hkv, 128, 500000.0, xcd_speed=speeds)
        lq, tc = int(rng.choice([1, 50, 64, 256, 700])), int(rng.choice([0, 900, 8000, 31744, 100000]))
        items = ba.ba_schedule_final_block(h, [0, lq], [0, tc], 256)
        if not items or items[0].xcd < 0:
            continue  # equal splits (one split, or nothing to size): no XCDs in the answer
        seen = {(w.kv_head, w.split, w.row_begin) for w in items}
        assert len(seen) == len(items), (case, hkv, g, lq, tc)
        counts = np.bincount([w.xcd for w in items], minlength=8)
        assert counts.max() - counts.min() <= 1, (case, counts)


def test_bad_xcd_speeds_are_rejected():
    h = ba.Heads(32, 8, 128, 500000.0, xcd_speed=[1, 1, 1, 0.1, 1, 1, 1, 1])
    with pytest.raises(ba.BaError):
        ba.ba_schedule_final_block(h, [0, 256], [0, 31744], 256)
    h = ba.Heads(32, 8, 128, 500000.0, xcd_speed=[1, 1, 1, float("nan"), 1, 1, 1, 1])
    with pytest.raises(ba.BaError):
        ba.ba_schedule_final_block(h, [0, 256], [0, 31744], 256)
    with pytest.raises(ValueError):
        ba.Heads(32, 8, 128, xcd_speed=[1.0] * 7)


KV_PLAN = r'''
// Prints the dk/dv kernel's work of a call: "shares n_split items part_slots counters", then per launch and table entry
// "launch block key_tile split n_splits begin end walk".
#include <cstdio>
#include <cstdlib>
#include "ba_plan.h"
#include "ba_schedule.h"
int main(int, char **a) {  // n_q_heads n_kv_heads head_dim n_prompts {n_blocks {len}}
  ba_heads h = {};
  h.n_q_heads = atoi(a[1]), h.n_kv_heads = atoi(a[2]), h.head_dim = atoi(a[3]);
  std::vector<int32_t> cu(1, 0), offs(1, 0);
  const int n_prompts = atoi(a[4]);
  a += 5;
  for (int n = 0; n < n_prompts; ++n) {
    const int nb = atoi(*a++);
    cu.push_back(cu.back() + nb);
    for (int b = 0; b < nb; ++b) offs.push_back(offs.back() + atoi(*a++));
  }
  const int G = h.n_q_heads / h.n_kv_heads;
  const ba::WalkShares s = ba::plan_kv_shares(&h, n_prompts, cu.data(), offs.data());
  printf("shares %d %lld %zu %zu\n", s.n_split, (long long)s.items, s.part_bytes / (32 * 4 * (size_t)h.head_dim), s.count_bytes / 4);
  std::vector<ba::PromptBlock> blks = ba::list_prompt_blocks(n_prompts, cu.data(), offs.data());
  ba::sort_by_query_rows(&blks, G, s);
  int launch = 0;
  for (size_t b0 = 0; b0 < blks.size(); b0 += ba::kEncMaxBlocks, ++launch) {
    const int n = (int)std::min<size_t>(ba::kEncMaxBlocks, blks.size() - b0);
    ba::BwdKvMeta m;
    const int64_t tiles = ba::build_kv_meta(blks, b0, n, G, s, &m);
    for (int e = 0; e < tiles; ++e) {  // (the kernel's own arithmetic, from its entry on)
      int b = 0;
      while (m.tile_start[b + 1] <= e) ++b;
      int split = 0, jt = e - m.tile_start[b], n_splits = 1;
      const bool shared = b < m.n_split;
      if (shared) {
        const int n_kt = (m.len[b] + ba::kBwdTileKeys - 1) / ba::kBwdTileKeys;
        split = jt / n_kt;
        jt -= split * n_kt;
      }
      const int rows_a = m.len[b] * G, rows_f = m.fin_len[b] * G, R = ba::kKvTileRows;
      ba::TileRange w = {0, (rows_f + R - 1) / R + (rows_a + R - 1) / R - jt * ba::kBwdTileKeys * G / R};
      const int walk = w.end;
      if (shared) {
        n_splits = ba::walk_splits(walk, m.chunk);
        if (split >= n_splits) continue;
        w = ba::walk_split_range(walk, n_splits, split);
      }
      printf("%d %d %d %d %d %d %d %d %d\n", launch, m.start[b], jt, split, n_splits, w.begin, w.end, walk, shared ? e : -1);
    }
  }
}
'''


@pytest.fixture(scope="module")
def kv_plan(tmp_path_factory):
    import os
    import shutil
    import subprocess
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler here")
    csrc = os.path.join(os.path.dirname(ba.LIB_PATH), "csrc")
    d = tmp_path_factory.mktemp("kv_plan")
    (d / "kv_plan.cpp").write_text("#include <algorithm>\n#include <vector>\n" + KV_PLAN)
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", csrc, str(d / "kv_plan.cpp"),
                    os.path.join(csrc, "ba_plan.cpp"), "-o", str(d / "kv_plan")], check=True)

    def plan(hq, hkv, d_, prompts):
        args = [hq, hkv, d_, len(prompts)]
        for p in prompts:
            args += [len(p), *p]
        out = subprocess.run([str(d / "kv_plan"), *map(str, args)], check=True, capture_output=True, text=True).stdout.splitlines()
        return [int(x) for x in out[0].split()[1:]], [tuple(int(x) for x in l.split()) for l in out[1:]]

    return plan


def test_shared_walks_of_key_tiles_cover_every_row_tile_once(kv_plan):
    """The dk/dv kernel's plan: the splits of a key tile partition the row tiles that see it, none of them empty, whether
    the block is shared or not; a shared entry's partial results and counter lie inside the memory planned for them.
    Drawn calls, and the ones whose gradients the GPU tests compare: their walks are shared."""
    gpu_cases = [(2, 2, 64, [[1150, 37], [40, 9]]), (6, 2, 128, [[700, 420, 50]]), (8, 2, 128, [[30, 5], [1300, 33]]),
                 (4, 1, 64, [[1, 1500, 1]]), (8, 2, 128, [[64, 9], [900, 380, 33]]), (4, 1, 64, [[200, *[6] * 180, 24]] * 2),
                 (8, 2, 64, [[1200, 10]]), (8, 2, 64, [[800, 420, 30], [64, 9]])]
    rng = np.random.default_rng(5)
    drawn = []
    for _ in range(60):
        hq, hkv, d = [(4, 4, 64), (8, 2, 64), (32, 8, 128), (16, 8, 128), (6, 2, 128), (1, 1, 64)][int(rng.integers(6))]
        hi = int(rng.choice([60, 300, 2000]))
        drawn.append((hq, hkv, d, [[*rng.integers(0, hi, int(rng.integers(0, 9))).tolist(), int(rng.integers(0, 300))] for _ in range(int(rng.integers(1, 9)))]))
    seen = set()
    for i, (hq, hkv, d, prompts) in enumerate(gpu_cases + drawn):
        G = hq // hkv
        (n_split, items, slots, counters), entries = kv_plan(hq, hkv, d, prompts)
        seen.add(n_split > 0)
        assert i >= len(gpu_cases) or n_split > 0
        assert slots == items * hkv * 4 and counters == items * hkv
        tiles = {}
        for launch, start, jt, split, n_splits, begin, end, walk, entry in entries:
            assert begin < end and (n_splits == 1 or launch == 0) and entry < items
            tiles.setdefault((start, jt), []).append((split, n_splits, begin, end, walk))
        t0, want = 0, {}
        for p in prompts:
            for b, n in enumerate(p):
                fin = p[-1] if b < len(p) - 1 else 0
                for jt in range(-(-n // 64)):
                    want[t0, jt] = -(-fin * G // 32) + -(-n * G // 32) - jt * 64 * G // 32
                t0 += n
        assert {k: v[0][4] for k, v in tiles.items()} == want
        for k, parts in tiles.items():
            parts.sort()
            assert [x[0] for x in parts] == list(range(parts[0][1]))
            assert [x[2] for x in parts] + [want[k]] == [0] + [x[3] for x in parts]
    assert seen == {True, False}


@pytest.mark.parametrize("hq,hkv,d,prompts,shared", [
    (64, 8, 128, [[90] * 4 + [5]] * 10, False), (64, 8, 128, [[90] * 4 + [5]], True), (32, 8, 128, [[166] * 5 + [12]] * 3, False),
    (32, 8, 128, [[290, 290, 3]] * 5, True), (16, 8, 128, [[418] * 4 + [36]] * 2, True), (8, 2, 64, [[300] * 6 + [20]] * 8, True)])
def test_walks_of_key_tiles_are_shared_only_where_the_launch_gets_shorter(kv_plan, hq, hkv, d, prompts, shared):
    """Groups of four and more at head_dim 128 whose launch is hardly longer than its load or than the walks that stay;
    the same prompt alone, longer walks, smaller groups and head_dim 64 are shared as ever."""
    assert (kv_plan(hq, hkv, d, prompts)[0][0] > 0) == shared
