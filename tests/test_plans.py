"""What the launch plans promise, over the shapes they accept (host functions: nothing is launched)."""
import ctypes
import itertools
import os
import random
import subprocess

import numpy as np
import pytest
from scipy import stats

import fused_rows
import long_rows
import paper_2510_05485_amd as tb
from paper_2510_05485_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
LDS = 160 * 1024


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if not os.path.exists(build.LIB):
        build.build(verbose=False)
    so = str(tmp_path_factory.mktemp("plans") / "plans.so")
    subprocess.check_call([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-shared", "-fPIC",
                           "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "plans.cpp"),
                           "-o", so, "-L", build.PKG, "-ltensorbleu", "-Wl,-rpath," + build.PKG])
    tb.load_library()
    lib = ctypes.CDLL(so)
    i64, i32, flag = ctypes.c_int64, ctypes.c_int, ctypes.c_bool
    lib.runs_plan.restype = flag
    lib.runs_plan.argtypes = [i64, i64, i64, i32, i32, i32, flag, flag, ctypes.POINTER(i64)]
    lib.deal_plan.restype = flag
    lib.deal_plan.argtypes = [i64, i64, i64, i32, i32, i32, flag, flag, ctypes.POINTER(i64)]
    lib.fused_plan.restype = lib.fused_path.restype = flag
    lib.fused_plan.argtypes = [i64, i64, i64, i32, i32, i32, flag, ctypes.POINTER(i64)]
    lib.fused_path.argtypes = [i64, i64, i32, i32]
    lib.route.argtypes = [i32, i32, i64, i64, i32, i32, flag, flag]
    lib.runs_shape.restype = flag
    lib.runs_shape.argtypes = [i64, i64, i64, i32, i32, i32, flag, ctypes.POINTER(i32)]
    lib.first_free_slot.restype = ctypes.c_uint32
    lib.first_free_slot.argtypes = [ctypes.c_uint32] * 3
    return lib


def test_sorted_runs_leave_their_tables_room(plans):
    # Every table (where n-grams have more than 64 bits: every part of one) receives a binomial share
    # of the distinct n-grams, at most one per position.  That a share outgrows its table has to stay
    # below exp(-40) each.
    out = (ctypes.c_int64 * 5)()
    shapes, entries, tables, slots = [], [], [], []
    for R, cs, of, N, bits in itertools.product(
            (1, 2, 3, 4, 6, 8, 12, 16, 31, 62),
            (100, 1000, 3000, 4096, 8192, 12000, 30000, 65536, 131072, 262144, 1000000),
            (0.01, 0.5, 1.0, 2.0), (1, 3, 4, 8), (1, 8, 13, 14, 16, 17, 18, 19, 22, 23, 24, 25, 31)):
        rs = max(int(of * cs), 1)
        cap = cs + R * rs
        if not 12288 < cap <= 2097152:
            continue
        for B, (rouge, sizes) in itertools.product((1, 50), ((False, False), (False, True), (True, False))):
            if plans.runs_plan(B, cs, rs, R, N, bits, rouge, sizes, out):
                shapes.append((B, cs, rs, R, N, bits, rouge, sizes))
                entries.append(cap if sizes else cs)
                tables.append(out[0])
                slots.append(out[1])
                assert out[2] <= 512 and out[3] * out[2] <= cap and out[4] + 1024 <= LDS, shapes[-1]
    assert len(shapes) > 10000
    assert (8192, 8192, 16, 4, 18) in {s[1:6] for s in shapes}
    chance = stats.binom.logsf(slots, entries, 1.0 / np.array(tables, dtype=np.float64))
    worst = int(np.argmax(chance))
    assert chance[worst] <= -40.0, (shapes[worst], tables[worst], slots[worst], chance[worst])


def test_dealt_partitions_leave_their_tables_room(plans):
    # tables of tokens and of pairs: as the sorted runs'; ids never fill their table (a search ends at a free
    # slot); two workgroups on a unit; runs' places fit their part of the workspace
    out = (ctypes.c_int64 * 14)()
    rng, shapes, mean, tables, slots = random.Random(31), 0, [], [], []
    for _ in range(60000):
        R, N = rng.choice((1, 1, 2, 3, 5, 8, 16, 40, 61)), rng.randint(1, 4)
        rouge, sizes = rng.choice(((False, False), (False, True), (True, False)))
        cs = int(2 ** (20.5 * rng.random()))
        rs = max(1, min(int(2097152 / R), int(cs * 4 ** rng.uniform(-3, 1.5))))
        B, vocab = int(2 ** (8 * rng.random())), rng.choice((2, 1000, 65536, (1 << 20) - 2))
        cap = cs + R * rs
        if not 12288 < cap <= 2097152 or not plans.deal_plan(B, cs, rs, R, N, vocab, rouge, sizes, out):
            continue
        shapes += 1
        first, kinds = out[13], out[0]
        assert kinds == min(N, 3) and first == (N - 1 if rouge else 0) and (not rouge or N <= 2)
        assert out[10] == sum(out[1 + first:1 + kinds]) <= 2048
        assert out[12] <= LDS // 2 and out[11] <= 1024 and out[11] * out[10] <= (kinds - first) * cap
        assert out[9] % 64 == 0 and 4 * out[7] <= 3 * out[6] and out[7] <= out[8] and out[7] % 8 == 0
        assert out[8] <= 1 << 20             # (id, order and at least eleven bits of the hash in a word)
        for kind in range(first, min(kinds, 2)):
            mean.append(cap if sizes else cs)
            tables.append(out[1 + kind])
            slots.append(out[4 + kind])
    assert shapes > 10000
    assert not plans.deal_plan(4, 20000, 20000, 1, 4, (1 << 20) - 1, False, False, out)
    assert not plans.deal_plan(4, 20000, 20000, 1, 5, 1000, False, False, out)
    chance = stats.binom.logsf(slots, mean, 1.0 / np.array(tables, dtype=np.float64))
    assert chance.max() <= -40.0


def test_long_shapes_reach_their_kernels(plans):
    dealt, runs = 1, 2
    for (B, R, L, Lr, vocab, N), calls in long_rows.DEALT.items():
        for call, (n, rouge, sizes) in {"b": (N, False, False), "d": (N, False, True), "1": (1, True, False),
                                        "2": (2, True, False)}.items():
            assert (plans.route(B, R, L, Lr, n, vocab, rouge, sizes) == dealt) == (call in calls), (B, R, L, Lr, call)
    for B, R, L, N in long_rows.FEW_TOKENS + [(*row[:3], 4) for row in long_rows.CROWDED]:
        assert plans.route(B, R, L, L, N, 50257, False, False) == dealt, (B, R, L)
    # one order, many positions: with one reference only
    assert plans.route(12, 2, 48662, 50090, 1, 300, False, False) == runs
    assert plans.route(10, 2, 48662, 50090, 1, 300, False, False) == dealt
    assert plans.route(51, 1, 25511, 26000, 1, 300, False, False) == dealt
    out = (ctypes.c_int32 * 4)()
    for (B, R, L, Lr, vocab, N), (items, words, wide) in long_rows.RUNS.items():
        bits = (vocab - 1).bit_length()
        for sizes in (False, True):
            assert plans.route(B, R, L, Lr, N, vocab, False, sizes) == runs, (B, R, L, Lr, sizes)
            assert plans.runs_shape(B, L, Lr, R, N, bits, sizes, out)
            assert list(out[:3]) == [items, words, wide] and (out[3] > 0) == (vocab == 262144), (B, R, L, Lr)


def fused_table(plans, *shape):
    """Share of the table's slots that are taken if no n-gram repeats, and bits of an entry's probe
    count (what the remainder of the key and the id leave of 32); None: no such plan."""
    out = (ctypes.c_int64 * 9)()
    if not plans.fused_plan(*shape, out):
        return None
    lg, id_bits, key_bits, _, lds = out[:5]
    assert lds <= LDS, shape
    # (however many orders share the table: test_a_table_holds_no_more_than_the_candidate)
    load = shape[1] / 2 ** lg
    return load, min(32 - key_bits + lg - 2, 32) - id_bits


def test_shared_units_keep_their_registers(plans):
    # more than 16 blocks a wavefront need scratch where workgroups share a unit, and are for workgroups of 16
    # wavefronts and, up to order 2, of 8 only; no kernel of one block is built for these units
    out = (ctypes.c_int64 * 9)()
    rng, seen = random.Random(29), {}
    for _ in range(40000):
        R, N, rouge = rng.choice((1, 2, 3, 5, 8, 16, 40, 62)), rng.randint(1, 8), rng.random() < 0.3
        cs = int(8192 ** rng.random())
        rs = int(max(24000 - cs, R) / R * rng.random()) + 1
        if not plans.fused_plan(int(257 * 40 ** rng.random()), cs, rs, R, N, 16, rouge, out) or out[8]:
            continue
        waves, blocks = out[5:7]
        assert blocks >= 2 and (blocks <= 16 or waves == 16 or (waves == 8 and N <= 2)), (cs, rs, R, N, rouge, list(out))
        seen[waves] = max(seen.get(waves, 0), blocks)
    assert seen[16] > 16 and min(seen[w] for w in (1, 2, 4, 8)) > 8, seen


def test_many_counters_get_a_table_for_each_stretch(plans):
    # five orders and more with three references or more: no single table (bit 1 of pass_ends) where fewer
    # workgroups would be on a unit for it
    out = (ctypes.c_int64 * 9)()
    for B, R, cs, rs, N, bits in ((3615, 16, 26, 16, 8, 7), (3711, 16, 42, 50, 5, 16), (2636, 3, 319, 330, 8, 9),
                                  (5013, 3, 84, 85, 8, 10), (1184, 16, 280, 91, 5, 7)):
        assert plans.fused_plan(B, cs, rs, R, N, bits, False, out)
        workgroups = min((B + 255) // 256, 32 // out[5])
        assert not out[3] & 2 or out[4] * workgroups <= LDS, (B, R, N)


def way_of(pass_ends, orders):
    ends = [pass_ends >> 4 * n & 15 for n in range(1, orders)]  # of the stretches that begin with 2, 3, ...
    if ends[0] == 2 and orders > 2:
        return "single" if ends[1] == 3 else "pairs"
    return ("together" if pass_ends & 2 else "stretches") + (" apart" if pass_ends & 1 else "")


def test_the_rows_reach_what_they_name(plans):
    out = (ctypes.c_int64 * 9)()
    kernels = (1, 2, 3, 4, 5, 6, 8, 12, 16, 24)

    def planned(mode, B, R, cs, rs, N):
        assert R in {"one": (1,), "two": (2,), "more": range(3, 63), "rouge": range(1, 63)}[mode]
        assert plans.fused_plan(B, cs, rs, R, N, fused_rows.BITS, mode == "rouge", out)
        # (longer shapes than the path's own go there from some tens of groups on)
        assert B >= 100 or plans.fused_path(cs, rs, R, fused_rows.BITS)
        return out

    for (alone, keep, mode), rows in fused_rows.KERNELS.items():
        assert sorted(rows) == list(kernels[0 if alone else 1:])
        for blocks, shape in rows.items():
            plan = planned(mode, *shape)
            assert (plan[8], plan[7]) == (alone, keep), (shape, list(plan))
            assert blocks == min(k for k in kernels if k >= plan[6]), (shape, list(plan))
    for way, rows in fused_rows.PASSES.items():
        for alone, mode, shape in rows:
            plan = planned(mode, *shape)
            assert (plan[8], way_of(plan[3], shape[4])) == (alone, way), (shape, list(plan))
    assert len(fused_rows.KERNELS) == 16


def test_rouge_shapes_reach_their_kernels(plans):
    out = (ctypes.c_int64 * 9)()
    kernels = (1, 2, 3, 4, 5, 6, 8, 12, 16, 24)
    for alone, rows in fused_rows.ROUGE.items():
        assert sorted(rows) == list(kernels[0 if alone else 1:])
        for blocks, (B, R, cs, rs) in rows.items():
            for N in (1, 2, 3):
                assert plans.fused_plan(B, cs, rs, R, N, fused_rows.BITS, True, out)
                assert B >= 100 or plans.fused_path(cs, rs, R, fused_rows.BITS)
                assert (out[8], out[7]) == (alone, 0)
                assert blocks == min(k for k in kernels if k >= out[6])
    # ids are kept between passes from order 3 on only: ROUGE-1 and -2 need no kernels that keep them
    rng = random.Random(41)
    for _ in range(20000):
        B, R, N = int(2 ** (13 * rng.random())), rng.choice((1, 2, 3, 8, 40, 62)), rng.randint(1, 2)
        cs, rs = int(2 ** (13.6 * rng.random())), int(2 ** (14 * rng.random()))
        if plans.fused_plan(B, cs, rs, R, N, rng.choice((1, 8, 16, 31)), True, out):
            assert not out[7]


def test_colliding_ids_walk_further_than_an_entry_counts(plans):
    # order 1 of the batch of test_gpu_fused.py: so many of the ids have the same bucket and the same step that
    # they fill more buckets than an entry can count
    out = (ctypes.c_int64 * 9)()
    ids = fused_rows.colliding_ids()[0].astype(np.uint64)
    word = np.uint64(0xFFFFFFFF)
    for R, N, rouge in itertools.product((1, 2, 3), (1, 2, 4), (False, True)):
        assert plans.fused_plan(6, 400, 400, R, N, 31, rouge, out)
        lg, id_bits, key_bits = out[:3]
        h = ids * np.uint64(0x9E3779B1 << 32 - key_bits) & word
        remainder = h << np.uint64(lg - 2) & word
        walks = list(zip(h >> np.uint64(34 - lg), remainder >> np.uint64(21)))
        longest = 2 ** (min(32 - key_bits + lg - 2, 32) - id_bits) - 1
        assert max(walks.count(walk) for walk in set(walks)) > 4 * longest, (R, N, rouge, list(out))


def entries(tokens, first, last, rng):
    """Entries that the orders first..last of a candidate make in the fused kernel's table, and the ids
    of the last order's n-grams: an n-gram that goes on as the candidate does at its prefix's id needs
    none, the others are entered once, by whichever position comes first."""
    made, ids = 0, list(range(len(tokens)))
    for n in range(1, last + 1):
        table, new = {}, {}
        where = list(range(len(tokens) - n + 1))
        rng.shuffle(where)
        for i in where:
            key = (ids[i] if n > 1 else -1, tokens[i + n - 1])
            at = ids[i] + n - 1
            if n > 1 and at < len(tokens) and tokens[at] == tokens[i + n - 1]:
                new[i] = ids[i]
            else:
                new[i] = table.setdefault(key, i)
        ids = [new[i] for i in range(len(tokens) - n + 1)]
        made += len(table) if first <= n else 0
    return made, ids


def test_a_table_holds_no_more_than_the_candidate():
    # Order n makes at most d(n) - d(n - 1) + 1 entries, d(n) being the number of distinct n-grams: every
    # (n-1)-gram but perhaps the last window's has one continuation that needs none.  d(N) is at most
    # len - N + 1, so orders first..last make at most len - first + 1 together.
    rng = random.Random(17)
    for length, vocab in itertools.product((1, 2, 3, 7, 8, 9, 60, 300), (1, 2, 3, 20, 1000)):
        for _ in range(4):
            tokens = [rng.randrange(vocab) for _ in range(length)]
            for first, last in ((1, 1), (1, 2), (1, 4), (2, 4), (3, 4), (1, 8), (2, 8), (4, 4), (7, 8)):
                made, ids = entries(tokens, first, last, rng)
                assert made <= max(length - first + 1, 0)
                grams = [tuple(tokens[i:i + last]) for i in range(length - last + 1)]
                assert len(set(ids)) == len(set(grams)) == len(set(zip(ids, grams)))


def test_fused_tables_count_far_enough(plans):
    # A probe sequence of ordinary tokens must not reach the largest count of an entry.  The share of
    # the sequences that go one bucket further is an eighth at half load and 0.43 at three quarters.
    seen = {False: 0, True: 0}
    for R, cs, of, (N, bits), B in itertools.product(
            (1, 2, 3, 4, 5, 7, 8, 12, 16, 31, 62), list(range(1024, 8193, 128)) + [1, 5, 60, 500, 5600],
            (0.1, 0.3, 0.8, 1.0, 1.2), ((1, 8), (2, 14), (4, 16), (4, 23), (8, 12)), (1, 40, 700, 4096)):
        for rouge in (False, True):
            shape = (B, cs, max(int(of * cs), 1), R, N, bits, rouge)
            table = fused_table(plans, *shape)
            if table:
                load, count_bits = table
                assert load <= 0.75 and count_bits >= (4 if load <= 0.5 else 6), (shape, table)
                seen[load > 0.5] += 1
    assert min(seen.values()) > 10, seen


def test_the_fused_plan_takes_what_the_path_accepts(plans):
    # an AUTO or forced FUSED call on a shape that the layout calls fused must not be refused later
    accepted = 0
    strides = sorted({1, 2, 3, 63, 64, 65, 100, 255, 256, 300, 700, 1000, 1024, 1500, 2048, 3000, 3072, 4000,
                      4095, 4096})
    for R, cs, rs, bits in itertools.product((1, 2, 3, 4, 7, 12, 20, 40, 62, 63), strides,
                                             strides + [8000, 11000], (1, 6, 8, 15, 16, 18, 20, 22, 26, 31)):
        if plans.fused_path(cs, rs, R, bits):
            accepted += 1
            for N, B, rouge in ((1, 1, False), (4, 1, False), (8, 300, False), (4, 2400, False), (3, 9000, True)):
                assert fused_table(plans, B, cs, rs, R, N, bits, rouge), (B, cs, rs, R, N, bits, rouge)
    assert accepted > 5000


def test_an_insertion_skips_no_slot_it_saw_free(plans):
    # `before` and `after`: how many slots of the bucket are taken, front to back, when a 16-byte read
    # of it begins and ends.  Each word comes from some moment in between.  The key may be in any slot
    # that was filled meanwhile, so the insertion has to begin at or before the first slot seen free.
    for before in range(5):
        for after in range(before, 5):
            for seen in itertools.product((0, 7), repeat=4):
                if all(seen[:before]) and not any(seen[after:]):
                    free = [k for k in range(4) if not seen[k]]
                    at = plans.first_free_slot(*seen[:3])
                    assert at == 4 * (free[0] if free else 3), (before, after, seen)
