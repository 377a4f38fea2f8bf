"""The library's own planner on the CPU (no GPU): validation, page bookkeeping, rotary positions,
write targets and attention work lists of hat_mid_forward, through a host-only handle.

Integer work: everything is compared exactly -- pages, lengths and write targets against the
independent page model of oracle/, positions against the definition (start + row, or start + depth
for a tree), and the work lists against what the kernels assume of them."""
import numpy as np
import pytest

import hat_inputs as hi
from oracle.page_model import PageModel, PageModelError
from paper_2503_18989_amd import HatError, HatPlanner

SHAPE = dict(hi.MID7B)        # only the head count and head size matter to the planner


def both(n_pages, **kw):
    return HatPlanner(SHAPE, n_pages, **kw), PageModel(n_pages, 16, kw.get("max_devices", 64), kw.get("max_step_tokens", 8192),
                                                       kw.get("max_pos", 16384))


def check_items(plan, segs, part_rows_seen):
    """Properties the attention kernels rely on."""
    tok0 = np.cumsum([0] + [sg[3] for sg in segs])
    by_seg_c, by_seg_v = {}, {}
    for it in plan["chunk_items"]:
        by_seg_c.setdefault((it["seg"], it["q0"]), []).append(it)
    for it in plan["verify_items"]:
        by_seg_v.setdefault(it["seg"], []).append(it)
    merges = {m["row0"]: m for m in plan["merge_items"]}
    for i, sg in enumerate(segs):
        dev, kind, start, n = sg[:4]
        if kind == hi.CHUNK:
            assert i not in by_seg_v
            for q0 in range(0, n, 256):
                nq = min(256, n - q0)
                items = sorted(by_seg_c[(i, q0)], key=lambda it: it["kv_begin"])
                need = start + q0 + nq
                assert items[0]["kv_begin"] == 0 and items[-1]["kv_end"] == need
                for a, b in zip(items, items[1:]):
                    assert a["kv_end"] == b["kv_begin"]
                for k, it in enumerate(items):
                    assert it["kv_begin"] % 64 == 0 and it["kv_begin"] < it["kv_end"]
                    assert (it["nq"], it["start"], it["tok0"], it["kv_len"]) == (nq, start, tok0[i], start + n)
                    if len(items) == 1:
                        assert it["part_row"] == -1
                    else:
                        assert it["part_row"] == items[0]["part_row"] + k * nq
                        part_rows_seen.append((it["part_row"], nq))
                if len(items) > 1:
                    covered = 0
                    for g0 in range(0, nq, 16):           # merged in groups of at most 16 rows
                        m = merges[tok0[i] + q0 + g0]
                        assert (m["nsplit"], m["stride"], m["part_row"]) == (len(items), nq, items[0]["part_row"] + g0)
                        covered += m["nrows"]
                    assert covered == nq
        else:
            assert not any(s_ == i for s_, _ in by_seg_c)
            items = sorted(by_seg_v[i], key=lambda it: it["kv_begin"])
            ln = start + n
            assert items[0]["kv_begin"] == 0 and items[-1]["kv_end"] == ln
            for a, b in zip(items, items[1:]):
                assert a["kv_end"] == b["kv_begin"]
            masks = sg[4] if len(sg) > 4 and sg[4] is not None else [(2 << r) - 1 for r in range(n)]
            for k, it in enumerate(items):
                assert it["kv_begin"] % 64 == 0 and it["kv_begin"] < it["kv_end"] and it["q0"] == 0
                assert (it["nq"], it["start"], it["tok0"], it["kv_len"]) == (n, start, tok0[i], ln)
                vis = it["vis_lo"] | (it["vis_hi"] << 32)
                assert [(vis >> (8 * r)) & 0xFF for r in range(n)] == list(masks) and vis >> (8 * n) == 0
                if len(items) == 1:
                    assert it["part_row"] == -1
                else:
                    assert it["part_row"] == items[0]["part_row"] + k * n
                    part_rows_seen.append((it["part_row"], n))
            if len(items) > 1:
                m = merges[tok0[i]]
                assert (m["nrows"], m["nsplit"], m["stride"], m["part_row"]) == (n, len(items), n, items[0]["part_row"])


def disjoint(part_rows):
    spans = sorted(part_rows)
    for (a, na), (b, _) in zip(spans, spans[1:]):
        assert a + na <= b, "partial rows overlap"


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_traffic_pages_targets_positions_and_work_lists(seed):
    rng = np.random.default_rng(seed)
    ndev, max_pos, max_step = 12, 6000, 4096
    lib, pm = both(ndev * max_pos // 16 // 2, max_devices=ndev, max_step_tokens=max_step, max_pos=max_pos)
    ln = [0] * ndev
    for step in range(120):
        segs, trees, rows = [], {}, 0
        for d in map(int, rng.permutation(ndev)):
            r = rng.random()
            if r < 0.3:
                continue
            if (r < 0.36 and ln[d] > 0) or ln[d] + 1100 > max_pos:
                lib.release(d); pm.release(d); ln[d] = 0
                continue
            if ln[d] == 0 or r < 0.55:
                n = int(min(rng.choice([1, 15, 16, 17, 100, 255, 256, 257, 512, 700, 1024]), max_step - rows))
                if n <= 0:
                    continue
                segs.append((d, hi.CHUNK, ln[d], n)); ln[d] += n
            elif r < 0.8:
                back = int(min(rng.integers(0, 6), ln[d]))
                n = int(min(rng.integers(1, 9), max_step - rows))
                if n <= 0:
                    continue
                segs.append((d, hi.VERIFY, ln[d] - back, n)); ln[d] += n - back
            else:
                n = int(min(rng.integers(1, 9), max_step - rows))
                if n <= 0:
                    continue
                trees[d] = hi.random_tree(seed, n, step, d)
                segs.append((d, hi.VERIFY, ln[d], n, hi.tree_masks(trees[d])))
            rows += segs[-1][3]
        if not segs:
            continue
        plan = lib.plan(segs)
        targets = pm.step([tuple(sg[:4]) for sg in segs])
        want_dst = [pg * 16 + slot for tg in targets for pg, slot in tg]
        assert plan["kv_dst"] == want_dst
        want_pos = []
        for sg in segs:
            if len(sg) > 4:
                want_pos += [sg[2] + bin(m).count("1") - 1 for m in sg[4]]
            else:
                want_pos += list(range(sg[2], sg[2] + sg[3]))
        assert plan["pos"] == want_pos
        part_rows = []
        check_items(plan, segs, part_rows)
        disjoint(part_rows)
        for d, parents in trees.items():
            node = int(rng.integers(-1, len(parents)))
            keep = hi.tree_path(parents, node) if node >= 0 else []
            lib.kv_compact(d, ln[d], keep); pm.compact(d, ln[d], keep); ln[d] += len(keep)
        for d in range(ndev):
            assert lib.kv_query(d) == pm.query(d), (step, d)
    lib.close()


def test_errors_match_the_page_model_and_change_nothing():
    lib, pm = both(4, max_devices=4, max_step_tokens=64, max_pos=100)
    lib.plan([(0, 0, 0, 20)]); pm.step([(0, 0, 0, 20)])
    snap = [lib.kv_query(d) for d in range(4)]
    cases = [[(0, 0, 21, 4)], [(1, 0, 1, 4)], [(0, 0, 20, 4), (0, 0, 24, 4)], [(4, 0, 0, 4)], [(-1, 0, 0, 4)],
             [(1, 1, 0, 9)], [(1, 0, 0, 65)], [(0, 0, 20, 81)], [(0, 0, 10, 4), (1, 0, 0, 49)], [(1, 2, 0, 4)], [(1, 0, 0, 0)]]
    for segs in cases:
        with pytest.raises(HatError) as e:
            lib.plan(segs)
        with pytest.raises(PageModelError) as e2:
            pm.step(segs)
        assert e.value.code == e2.value.code, segs
        assert [lib.kv_query(d) for d in range(4)] == snap
    for masks in ([0], [3], [1, 2, 7], [1, 3, 6], [1, 1]):
        with pytest.raises(HatError) as e:
            lib.plan([(1, 1, 0, len(masks), masks)])
        assert e.value.code == -1 and [lib.kv_query(d) for d in range(4)] == snap
    with pytest.raises(HatError) as e:
        lib.plan([(1, 0, 0, 2, [1, 3])])          # a tree on a chunk segment
    assert e.value.code == -1
    plan = lib.plan([(0, 0, 10, 4), (1, 0, 0, 48)]); pm.step([(0, 0, 10, 4), (1, 0, 0, 48)])   # exactly fills the pool
    assert [lib.kv_query(d) for d in range(4)] == [pm.query(d) for d in range(4)]
    assert lib.plan([]) == dict(pos=[], kv_dst=[], chunk_items=[], verify_items=[], merge_items=[])
    lib.close()


@pytest.mark.parametrize("which", ["mixed", "verify", "sweep"])
def test_benchmark_shaped_steps_fit_every_capacity(which):
    # the largest steps the benchmark configurations produce: the plan must fit its buffers (a plan
    # that did not would be rejected with an internal error) and obey the work-list properties
    if which == "mixed":
        pref = hi.mixed_prefixes(3003)
        segs = [(d, k, p, n) for (d, k, p, n) in hi.mixed_step(3003, 0, pref)]
        pre = [(d, hi.CHUNK, 0, p) for d, p in enumerate(pref)]
        lib, pm = both(sum((p + 600) // 16 + 1 for p in pref) + 64, max_devices=32, max_step_tokens=8192, max_pos=8192)
    elif which == "verify":
        lengths = hi.verify_lengths(4004)
        pre = [(d, hi.CHUNK, 0, ln) for d, ln in enumerate(lengths)]
        segs = [(d, hi.VERIFY, ln, 8, hi.tree_masks(hi.MEDUSA_LIKE_TREE)) for d, ln in enumerate(lengths)]
        lib, pm = both(sum((ln + 8) // 16 + 1 for ln in lengths) + 64, max_devices=32, max_step_tokens=8192, max_pos=8192 + 64)
    else:
        pre = [(d, hi.CHUNK, 0, 7168) for d in range(8)]
        segs = [(d, hi.CHUNK, 7168, 1024) for d in range(8)]
        lib, pm = both(8 * 8192 // 16 + 8, max_devices=8, max_step_tokens=8192, max_pos=8192)
    for sg in pre:                                   # prefixes, one device per step (each fits max_step_tokens)
        lib.plan([sg]); pm.step([sg])
    plan = lib.plan(segs); pm.step([tuple(sg[:4]) for sg in segs])
    part_rows = []
    check_items(plan, segs, part_rows)
    disjoint(part_rows)
    assert [lib.kv_query(sg[0]) for sg in segs] == [pm.query(sg[0]) for sg in segs]
    lib.close()


def test_plan_capacity_failure_undoes_the_page_movements():
    # the "plan exceeds capacity" failure is only found after the step's rollbacks and allocations have
    # been made: every length, page list and the free set must come back exactly, and the handle must
    # carry on as if the failed call had never happened (compared with a planner that never saw it)
    a, pm = both(64, max_devices=4, max_step_tokens=256, max_pos=512)
    b = HatPlanner(SHAPE, 64, max_devices=4, max_step_tokens=256, max_pos=512)
    first = [(0, hi.CHUNK, 0, 100), (1, hi.CHUNK, 0, 40), (2, hi.CHUNK, 0, 33)]
    for h in (a, b):
        h.plan(first)
    pm.step(first)
    snap = [a.kv_query(d) for d in range(4)]
    # rolls device 0 back over three pages, extends device 1, restarts device 2, admits device 3
    step = [(0, hi.VERIFY, 60, 5), (1, hi.CHUNK, 40, 100), (2, hi.CHUNK, 0, 20), (3, hi.CHUNK, 0, 50)]
    a.limit_plan(8)
    with pytest.raises(HatError) as e:
        a.plan(step)
    assert e.value.code == -1 and "capacity" in str(e.value)
    assert [a.kv_query(d) for d in range(4)] == snap
    a.limit_plan(0)
    pa, pb = a.plan(step), b.plan(step)
    pm.step(step)
    assert pa == pb
    for d in range(4):
        assert a.kv_query(d) == b.kv_query(d) == pm.query(d)
    # the free set is intact as well: the next allocations take the same lowest ids on both
    nxt = [(3, hi.CHUNK, 50, 200), (0, hi.VERIFY, 65, 8)]
    assert a.plan(nxt) == b.plan(nxt)
    pm.step(nxt)
    for d in range(4):
        assert a.kv_query(d) == b.kv_query(d) == pm.query(d)
    a.close(); b.close()


@pytest.mark.parametrize("case", ["equal", "skewed", "one", "many short", "with a wide one"])
def test_partial_rows_of_narrow_chunks_fit_their_own_buffer(case):
    # chunk items of at most 32 rows are cut into key ranges of about equal size whose fp32 partial rows have a buffer
    # sized for the ranges wanted: no mix of cache lengths may run out of it (an item would then stay whole)
    rng = np.random.default_rng(5)
    lens = {"equal": [4096] * 20, "skewed": [6000] * 3 + [300] * 17, "one": [5900], "many short": list(rng.integers(257, 700, 24)),
            "with a wide one": [3000, 1024, 5000]}[case]
    rows = [int(r) for r in rng.integers(1, 33, len(lens))]
    lib, pm = both(sum(int(n) // 16 + 50 for n in lens), max_devices=24, max_step_tokens=8192, max_pos=6500)
    for d, n in enumerate(lens):
        lib.plan([(d, hi.CHUNK, 0, int(n))])
    segs = [(d, hi.CHUNK, int(n), r) for d, (n, r) in enumerate(zip(lens, rows))]
    if case == "with a wide one":
        segs[1] = (1, hi.CHUNK, 1024, 300)          # items of 256 and 44 rows
    plan = lib.plan(segs)
    part_rows = []
    check_items(plan, segs, part_rows)
    disjoint(part_rows)
    n_wide = len(plan["chunk_items"]) - lib.narrow_items()
    wide, narrow = plan["chunk_items"][:n_wide], plan["chunk_items"][n_wide:]
    assert all(it["nq"] > 32 for it in wide) and narrow and all(it["nq"] <= 32 for it in narrow)
    wanted = -(-2048 // SHAPE["n_heads"]) * 3 // 8
    keys = sum(n + r for d, _, n, r in segs if r <= 32)
    step = max(256, -(-(keys // wanted) // 128) * 128)
    assert max(it["kv_end"] - it["kv_begin"] for it in narrow) <= max(step + 64, 511)
    first_narrow = min([it["part_row"] for it in narrow if it["part_row"] >= 0], default=None)
    assert first_narrow is None or all(it["part_row"] < first_narrow for it in wide)
    lib.close()


def test_narrow_chunks_next_to_larger_ones_stream_only_when_long():
    lib, _ = both(400, max_devices=4, max_step_tokens=4096, max_pos=4096)
    for d in (0, 1):
        lib.plan([(d, hi.CHUNK, 0, 2000)])
    for start, n, want in [(1503, 32, 0), (1504, 32, 1), (1700, 33, 0), (1535, 1, 1), (1534, 1, 0)]:
        plan = lib.plan([(0, hi.CHUNK, 300, 200), (1, hi.CHUNK, start, n)])
        count = lib.narrow_items()
        assert (count > 0) == bool(want), (start, n)
        assert all((it["seg"] == 1) == (k >= len(plan["chunk_items"]) - count) for k, it in enumerate(plan["chunk_items"]) if count)
        lib.plan([(1, hi.CHUNK, start, 2000 - start)])
    lib.plan([(1, hi.CHUNK, 100, 32)])
    assert lib.narrow_items() == 1                   # alone: always
    lib.plan([(1, hi.VERIFY, 100, 8)])
    assert lib.narrow_items() == 0
    lib.close()


def check_blocks(lib, plan):
    """Streamed chunk items reach the launch as blocks of at most 32 rows: every row of every key range once, no empty block, the
    blocks of a key range side by side with the one that sees most keys first."""
    blocks = lib.blocks()
    items = plan["chunk_items"][:len(plan["chunk_items"]) - lib.narrow_items()]
    want = []
    for it in items:
        for r0 in reversed(range(0, it["nq"], 32)):
            b = {k: it[k] for k in ("seg", "kv_begin", "kv_end", "start", "tok0", "kv_len", "pt_off")}
            want.append(dict(b, q0=it["q0"] + r0, nq=min(32, it["nq"] - r0), part_row=it["part_row"] + r0 if it["part_row"] >= 0 else -1))
    assert blocks == want
    return len(blocks)


@pytest.mark.parametrize("rows,start", [([33], 200), ([130, 64], 300), ([256] + [64] * 9, 500), ([257, 40, 7], 90), ([300], 1500), ([40, 17], 1700)])
def test_streamed_chunks_are_listed_in_blocks_of_rows(rows, start):
    lib, _ = both(3000, max_devices=16, max_step_tokens=2048, max_pos=2048)
    if start:
        for d in range(len(rows)):
            lib.plan([(d, hi.CHUNK, 0, start)])
    plan = lib.plan([(d, hi.CHUNK, start, n) for d, n in enumerate(rows)])
    n = check_blocks(lib, plan)
    ranges = sum(-(-it["nq"] // 32) for it in plan["chunk_items"][:len(plan["chunk_items"]) - lib.narrow_items()])
    with pytest.raises(HatError):
        lib.blocks(cap=n - 1)
    assert n == ranges > 0                           # 26 blocks for 256 + 9 x 64 rows, where ten times the longest item's would be 80
    lib.set_attn_targets(4096, 2048)                 # many key ranges: staged
    plan = lib.plan([(d, hi.CHUNK, start, n) for d, n in enumerate(rows)])
    assert lib.blocks() == []
    lib.plan([(0, hi.VERIFY, start, 5)])
    assert lib.blocks() == []
    lib.close()


@pytest.mark.parametrize("rows,start,waves", [([64], 900, 8), ([256], 900, 8),                # a workgroup per CU at most
                                              ([120, 70, 90, 150, 160], 400, 4),              # 672: two rounds of short ones with one workgroup per CU
                                              ([512], 1000, 4), ([512] * 4, 100, 4)])         # 512 and more
def test_waves_of_a_row_block(rows, start, waves):
    lib, _ = both(3000, max_devices=16, max_step_tokens=2048, max_pos=2048)
    for d in range(len(rows)):
        lib.plan([(d, hi.CHUNK, 0, start)])
    plan = lib.plan([(d, hi.CHUNK, start, n) for d, n in enumerate(rows)])
    assert check_blocks(lib, plan) and lib.block_waves() == waves
    lib.plan([(0, hi.VERIFY, start, 5)])
    assert lib.block_waves() == 0
    lib.close()


def test_chunks_stream_where_that_is_faster():
    # measured (7B-shaped heads), staged against streamed in us: 30.8 | 20.4, 90 | 76, 75 | 58; 265 | 284 for 4096 rows
    def plan(rows, start, target=256):
        lib, _ = both(4000, max_devices=16, max_step_tokens=4096, max_pos=8192)
        lib.set_attn_targets(target, 2048)
        for d in range(len(rows) if start else 0):
            for q in range(0, start, 4096):
                lib.plan([(d, hi.CHUNK, q, min(4096, start - q))])
        p = lib.plan([(d, hi.CHUNK, start, n) for d, n in enumerate(rows)])
        n = check_blocks(lib, p) if lib.blocks() else 0
        assert (n > 0) == (lib.block_waves() > 0)
        lib.close()
        return n
    for rows, start in [([256], 1000), ([512] * 4, 500), ([256] + [64] * 9, 1000)]:
        assert plan(rows, start), (rows, start)
        for target in (64, 255, 257, 4096):          # a wish for the staged kernel's key ranges
            assert not plan(rows, start, target), (rows, start, target)
    for rows, start in [([512] * 8, 2000), ([4096], 0), ([230] * 9, 30)]:
        assert not plan(rows, start), (rows, start)


@pytest.mark.parametrize("rows,start,ranges", [([64], 600, 1), ([64], 1000, 1), ([64], 4000, 4), ([33], 6000, 4),        # measured: whole at 1000, four at 4000
                                               ([256], 4000, 1),                                        # a workgroup per CU: none to spare
                                               ([64, 20], 1600, 1)])                                    # next to a narrow item
def test_key_ranges_of_streamed_chunks(rows, start, ranges):
    lib, _ = both(3000, max_devices=2, max_step_tokens=4096, max_pos=8192)
    for d in range(len(rows)):
        for q in range(0, start, 2048):
            lib.plan([(d, hi.CHUNK, q, min(2048, start - q))])
    plan = lib.plan([(d, hi.CHUNK, start, n) for d, n in enumerate(rows)])
    check_items(plan, [(d, hi.CHUNK, start, n) for d, n in enumerate(rows)], [])
    assert check_blocks(lib, plan) == ranges * -(-rows[0] // 32)
    wide = [it for it in plan["chunk_items"] if it["nq"] > 32]
    assert len(wide) == ranges and all((it["part_row"] < 0) == (ranges == 1) for it in wide)
    lib.close()


def test_partial_rows_of_staged_and_narrow_chunks_are_apart():
    # a wide item that is staged in several key ranges (fp16 partial rows) next to a narrow one in several (fp32, numbered after them)
    lib, _ = both(3000, max_devices=2, max_step_tokens=4096, max_pos=8192)
    lib.set_attn_targets(257, 2048)                  # staged
    for d in (0, 1):
        lib.plan([(d, hi.CHUNK, 0, 4000)])
    plan = lib.plan([(0, hi.CHUNK, 4000, 64), (1, hi.CHUNK, 4000, 20)])
    part_rows = []
    check_items(plan, [(0, hi.CHUNK, 4000, 64), (1, hi.CHUNK, 4000, 20)], part_rows)
    disjoint(part_rows)
    n = lib.narrow_items()
    wide, narrow = plan["chunk_items"][:-n], plan["chunk_items"][-n:]
    assert lib.blocks() == [] and len(wide) > 1 and len(narrow) > 1
    assert 0 <= min(it["part_row"] for it in wide)
    assert max(it["part_row"] + it["nq"] for it in wide) <= min(it["part_row"] for it in narrow)
    lib.close()


@pytest.mark.parametrize("rows,start,millions", [([128], 4000, 17), ([256], 6000, 51), ([256, 40], 4500, 46), ([512], 3000, 53)])
def test_small_steps_hold_no_partial_results_in_fp16(rows, start, millions):
    # staged items hold the results of their key ranges in fp16, streamed ones in fp32 (numbered after the others): up to 95 M rows x
    # keys x heads a step is staged only if no item is cut, however much faster that may be
    lib, _ = both(4000, max_devices=8, max_step_tokens=4096, max_pos=8192)
    for d in range(len(rows)):
        for q in range(0, start, 2048):
            lib.plan([(d, hi.CHUNK, q, min(2048, start - q))])
    segs = [(d, hi.CHUNK, start, n) for d, n in enumerate(rows)]
    lib.set_attn_targets(257, 2048)
    fp16_rows = max(it["part_row"] for it in lib.plan(segs)["chunk_items"])
    lib.set_attn_targets(256, 2048)
    plan = lib.plan(segs)
    assert fp16_rows >= 0                            # staged, these steps would be cut
    assert lib.blocks() or not plan["merge_items"]
    assert sum(-(-n // 32) * 32 * (start + n / 2) for n in rows) * SHAPE["n_heads"] / 1e6 == pytest.approx(millions, abs=2)
    lib.close()


@pytest.mark.parametrize("chunks,drafts,n,hd,along", [([(64, 900)], 200, 8, 128, True), ([(64, 900)], 200, 9, 128, False),        # eight waves: 256 items x heads
                                                      ([(512, 1000)], 3500, 30, 128, True),                                      # four waves
                                                      ([(20, 500)], 3500, 25, 128, True), ([(20, 500)], 3500, 30, 128, False),   # narrow alone: 1.4, 1.7 GB of drafts
                                                      ([(20, 500)], 3500, 60, 64, True),                                         # (the same bytes at head dim 64)
                                                      ([(512, 2000)] * 8, 200, 8, 128, False),                                   # staged
                                                      ([(512, 2000)] * 8 + [(20, 1600)], 200, 8, 128, True),                     # staged, and a narrow launch
                                                      ([(64, 900)], 0, 0, 128, False), ([], 500, 4, 128, False)])
def test_verify_items_that_go_along(chunks, drafts, n, hd, along):
    lib = HatPlanner(dict(SHAPE, head_dim=hd, d_model=hd * SHAPE["n_heads"]), 20000, max_devices=64, max_step_tokens=8192, max_pos=8192)
    for d, (_, start) in enumerate(chunks):
        lib.plan([(d, hi.CHUNK, 0, start)])
    for d in range(n):
        lib.plan([(len(chunks) + d, hi.CHUNK, 0, drafts)])
    lib.plan([(d, hi.CHUNK, start, rows) for d, (rows, start) in enumerate(chunks)] + [(len(chunks) + d, hi.VERIFY, drafts, 5) for d in range(n)])
    assert lib.verify_along() == along
    lib.plan([])
    assert not lib.verify_along()                     # (of the last plan)
    lib.close()
