"""CPU model of how an attention launch's work is cut (delta_api.cpp plan_split, attn_kernel.hip
balanced decomposition), checked for the properties the kernel's buffers rely on.  Sparse layers
are cut by the shape alone.

Every (sequence, KV head) pair is COST units of work followed by its 16-row groups; the pairs, in
(sequence, KV head) order, are cut into runs of equal length, run w for workgroup w.  A pair is
combined from the pieces that the run boundaries cut its groups into.  The cut is taken when a
run's length plus COST is at most 19/20 of the static pieces a CU takes one after another.  For
many random batches (dense layers from one sequence on, sparse layers with selections shorter than
the budget, host bounds far above the lengths): every group of every pair belongs to exactly one
piece, a pair's partial slots are exactly 0 .. n-1 and within the workspace's, and no workgroup
carries more than its run and the cost of the piece that the run begins in.  The partial slots and
the splits behind them are the library's: its workspace sizes say so.
"""
import random

import balanced_cases as BC
from paper_2510_09883_amd import delta as D

COST, KMAX_SPLITS, BAL_MAX_BATCH, TARGET, MIN_GPS, LIST = 8, 64, 64, 256, 8, 1024


def cdiv(a, b):
    return (a + b - 1) // b


def host_plan(B, Hkv, N, dense=None, tokens=False):
    """`dense`: the plan of the dense layers, for a sparse layer's plan (of single tokens)."""
    pairs = B * Hkv
    cap = 32 if pairs < 32 else 16
    want = cdiv(TARGET, pairs)
    if dense is not None:
        want = max(1, (2 if tokens and 32 < pairs < TARGET else 1) * TARGET // pairs)
        if TARGET < pairs and 3 * pairs <= 4 * TARGET and N >= 96:
            want = 3
        want = min(want, max(dense["slots"], cdiv(TARGET, pairs)))
    n = min(want, max(1, cdiv(N, MIN_GPS)), cap)
    n_split = cdiv(N, cdiv(N, n))
    p = dict(n_split=n_split, gps=cdiv(N, n_split), slots=n_split, n_runs=0,
             rounds=cdiv(n_split * pairs, TARGET))
    work = pairs * (N + COST)
    if dense is not None or B > BAL_MAX_BATCH or work >= 1 << 26 or (B == 1 and pairs >= 32):
        return p
    slots = max(n_split, cdiv(N, max(MIN_GPS, cdiv(N, cap))) + 1)
    if slots >= 2:
        p.update(slots=slots, n_runs=min(n_split * pairs, TARGET))
    return p


def cut(groups, Hkv, N, plan):
    """Per workgroup: the pieces (b, g, g0, n, slot, n_valid), and the balanced cut's run length (0:
    static pieces).  groups: each sequence's 16-row groups (0: an empty sequence)."""
    groups = [min(max(x, 0), N) for x in groups]
    B = len(groups)
    units = [max(1, x) + COST for x in groups]
    before = [sum(units[:b]) for b in range(B)]
    W, longest = Hkv * sum(units), max(units) - COST
    balanced = False
    if plan["n_runs"] and (B > 1 or 10 * groups[0] < 9 * N):
        chunk = max(cdiv(W, plan["n_runs"]), MIN_GPS, cdiv(longest, plan["slots"] - 1))
        balanced = 20 * (chunk + COST) <= 19 * (min(plan["gps"], longest) + COST) * plan["rounds"]
    out = []
    if balanced:
        for w in range(plan["n_runs"]):
            x, xe, segs = min(w * chunk, W), min((w + 1) * chunk, W), []
            while x < xe:
                b = sum(1 for v in before if Hkv * v <= x) - 1
                g = (x - Hkv * before[b]) // units[b]
                off = Hkv * before[b] + g * units[b] + COST
                end = off + units[b] - COST
                if off >= xe:
                    break
                y = max(x, off)
                first = off // chunk
                n_valid = (end - 1) // chunk - first + 1
                segs.append((b, g, y - off, min(xe, end) - y, w - first, n_valid))
                x = min(xe, end)
            out.append(segs)
    else:
        for b in range(B):
            for g in range(Hkv):
                n_valid = max(1, cdiv(groups[b], plan["gps"]))
                for s in range(n_valid):
                    g0 = s * plan["gps"]
                    out.append([(b, g, g0, min(plan["gps"], max(1, groups[b]) - g0), s, n_valid)])
    return out, chunk if balanced else 0


def check(groups, Hkv, N, dense=None, tokens=False):
    plan = host_plan(len(groups), Hkv, N, dense, tokens)
    out, balanced = cut(groups, Hkv, N, plan)
    seen, slots = {}, {}
    for segs in out:
        for b, g, g0, n, slot, n_valid in segs:
            assert n >= 1 and 0 <= slot < n_valid <= plan["slots"] <= KMAX_SPLITS
            slots.setdefault((b, g), []).append((slot, n_valid))
            seen.setdefault((b, g), []).append((g0, g0 + n))
    for b, x in enumerate(groups):
        for g in range(Hkv):
            spans, at = sorted(seen[(b, g)]), 0
            for lo, hi in spans:
                assert lo == at
                at = hi
            assert at == max(1, min(x, N))
            got = sorted(slots[(b, g)])
            assert [s for s, _ in got] == list(range(len(got))) and got[0][1] == len(got)
    if balanced:
        assert max(sum(seg[3] + COST for seg in segs) for segs in out) <= balanced + COST
    return plan, balanced


def test_random_batches_cover_every_group_once():
    rng, taken = random.Random(7), 0
    for _ in range(600):
        B, Hkv, N = rng.randint(1, 70), rng.choice([1, 2, 3, 4, 8]), rng.randint(1, 400)
        kind = rng.random()
        if kind < 0.3:
            groups = [rng.randint(1, N) for _ in range(B)]
        elif kind < 0.5:
            groups = [N] * B
        elif kind < 0.7:   # the host's bound is for a longer generation
            groups = [rng.randint(1, max(1, N // 4)) for _ in range(B)]
        else:
            groups = [rng.choice([0, 1, N, rng.randint(1, N)]) for _ in range(B)]
        dense = host_plan(B, Hkv, rng.randint(1, 400)) if rng.random() < 0.4 else None
        taken += check(groups, Hkv, N, dense, rng.random() < 0.5)[1] > 0
    assert taken > 150


def test_sparse_layers_are_cut_by_the_shape():
    """Every sequence gets the pieces that it would get alone among full selections, and no CU two
    pieces of pages while another has none (up to one pair per CU)."""
    rng = random.Random(3)
    for _ in range(300):
        B, Hkv, N = rng.randint(1, 70), rng.choice([1, 2, 4, 8]), rng.randint(1, 300)
        dense = host_plan(B, Hkv, rng.randint(1, 2000))
        groups = [rng.choice([N, N, rng.randint(0, N)]) for _ in range(B)]
        plan, balanced = check(groups, Hkv, N, dense)
        assert not balanced
        assert plan["n_split"] * B * Hkv <= TARGET or B * Hkv > TARGET
        full, _ = cut([N] * B, Hkv, N, plan)
        mine, _ = cut(groups, Hkv, N, plan)
        for b in (b for b in range(B) if groups[b] == N):
            assert [s for s in full if s[0][0] == b] == [s for s in mine if s[0][0] == b]


def _align(n):
    return -(-n // 256) * 256


def test_slots_are_the_library_s():
    """delta_workspace_bytes() from the model's partial slots: the status word, a 256-byte arrival
    counter per pair and the partials (largest of the dense and sparse layers' slots and the fused
    kernel's 64-page chunks), then a selection's buffers."""
    rng = random.Random(5)
    for _ in range(400):
        B, Hkv, G, d = rng.randint(1, 90), rng.choice([1, 2, 3, 4, 8, 31]), rng.randint(1, 8), rng.choice([64, 128])
        N, unit = rng.randint(1, rng.choice([60, 500, 3000])), rng.choice([None, 16, 16, 1])
        if unit == 1:
            N = min(N, 500)
        pairs, dense = B * Hkv, host_plan(B, Hkv, N)
        slots, extra = dense["slots"], 0
        sel = None
        if unit:
            K = rng.randint(1, 300)
            budget = 16 * K
            sel = D.make_select(budget, 0, unit)
            sparse = host_plan(B, Hkv, K, dense, unit == 1)
            chunks = cdiv(N, 64)
            slots = max(slots, sparse["slots"], chunks)
            extra = (_align(4 * B * N * Hkv * G * 16) + _align(4 * B * Hkv * G) + _align(4 * B * 16 * N // unit)
                     + _align(4 * B * budget // unit) + _align(256 * B) + _align(4 * B * chunks))
        want = 256 + 256 * pairs + _align(8 * pairs * slots * G) + _align(4 * pairs * slots * G * d) + extra
        assert D.delta_workspace_bytes(D.make_shape(B, Hkv * G, Hkv, d, N, 16 * N), sel) == want, (B, Hkv, G, d, N, unit)


def test_even_batches_keep_the_static_pieces_and_uneven_ones_do_not():
    for B, Hkv, N in [(16, 8, 2048), (8, 4, 2048), (64, 2, 1152), (64, 2, 65), (1, 8, 512), (32, 8, 2048)]:
        assert not check([N] * B, Hkv, N)[1]
    assert not check([65, 66] * 32, 2, 66)[1]
    # 32 ragged sequences, 8 KV heads: at most three quarters of the longest one a run
    rng = random.Random(5000)
    assert 0 < check([rng.randint(1024, 2048) for _ in range(32)], 8, 2048)[1] <= 1600
    # 160 pairs in two splits are 320 workgroups on 256 CUs; a bound of twice the length
    assert check([769] * 20, 8, 769)[1]
    assert check([512], 8, 1024)[1]


def test_gpu_balanced_batches_take_the_cut():
    for _, hkv, lens in BC.RAGGED:
        groups = [cdiv(s, 16) for s in lens]
        assert check(groups, hkv, max(groups))[1], lens
    for _, seed in BC.RANDOM:
        hkv, _, lens = BC.random_case(seed)
        groups = [cdiv(s, 16) for s in lens]
        assert check(groups, hkv, max(groups))[1], seed
    for B in BC.BATCH_LIMIT:
        groups = [cdiv(s, 16) for s in BC.batch_limit_lens(B)]
        assert bool(check(groups, BC.BATCH_LIMIT_KV_HEADS, max(groups))[1]) == (B <= BAL_MAX_BATCH), B


def test_gpu_short_pieces_fill_runs_of_three():
    groups = [cdiv(s, 16) for s in BC.SHORT_PIECES]
    out, taken = cut(groups, 8, max(groups), host_plan(len(groups), 8, max(groups)))
    assert taken and max(len(segs) for segs in out) == 3


def test_gpu_long_pieces_are_longer_than_the_list():
    for hkv, lens, balanced, _ in BC.LONG_PIECES:
        groups = [cdiv(s, 16) for s in lens]
        plan, taken = check(groups, hkv, max(groups))
        out, _ = cut(groups, hkv, max(groups), plan)
        assert bool(taken) == balanced and max(seg[3] for segs in out for seg in segs) > LIST
    for B, hkv, budget, _, longest in BC.LONG_TOKEN_PIECES:
        N = budget // 16
        plan, _ = check([N] * B, hkv, N, host_plan(B, hkv, cdiv(budget + 100, 16)), tokens=True)
        assert plan["gps"] == longest > LIST // 16


def test_gpu_sparse_splits_are_the_rule_s():
    for B, hkv, budget, unit, n_split in BC.SPARSE_SPLITS:
        N, dense = budget // 16, host_plan(B, hkv, cdiv(budget + 100, 16))
        plan, _ = check([N] * B, hkv, N, dense, tokens=unit == 1)
        assert plan["n_split"] == n_split, (B, hkv, budget, unit, plan)
