"""The fused kernel at the edges of its blocks of 64 positions, of its plans (how many orders share
a table, how many workgroups share a compute unit) and of its table, against the CPU oracle."""
import numpy as np
import pytest
import torch

import fused_rows
import oracle
import paper_2510_05485_amd as tb
import synth_inputs as syn
from rouge_validity import check_rouge

pytestmark = pytest.mark.gpu
TOL = 1e-5
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def check(w, N, int64=False, rouge=True, rouge_n=2):
    cand, refs = dev(w.cand), dev(w.refs)
    if int64:
        cand, refs = cand.long(), refs.long()
    cl, rl = dev(w.cand_len), dev(w.ref_len)
    ref = oracle.bleu(w.cand, w.cand_len, w.refs, w.ref_len, max_n=N, smoothing="exp", threads=8)
    cfg = tb.make_config(max_n=N, smoothing="exp", vocab_size=w.vocab)
    stats = tb.Stats.allocate(w.B, N, DEV)
    stats.group_distinct = None  # (asking for it keeps long shapes on the staged kernels)
    out = tb.tensorbleu_sentence(cand, cl, refs, rl, cfg, stats=stats)
    torch.cuda.synchronize()
    assert stats.device_status.item() == 0
    np.testing.assert_array_equal(stats.clipped.cpu().numpy(), ref.clipped)
    np.testing.assert_array_equal(stats.total.cpu().numpy(), ref.total)
    np.testing.assert_array_equal(stats.closest_ref_len.cpu().numpy(), ref.closest_ref_len)
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref.bleu).max() <= TOL
    if rouge:
        n = min(N, rouge_n)
        want = oracle.rouge_n(w.cand, w.cand_len, w.refs, w.ref_len, n=n)
        prf, overlap, best = tb.tensorrouge_n(cand, cl, refs, rl, n=n, vocab_size=w.vocab,
                                              want_overlap=True, want_best=True)
        check_rouge(want, overlap.cpu().numpy(), best.cpu().numpy(), prf.cpu().numpy(), TOL)


@pytest.mark.parametrize("N", [1, 2, 4, 8])
@pytest.mark.parametrize("L,Lr", [(1, 1), (3, 2), (63, 65), (64, 64), (65, 63), (128, 191)])
def test_block_edges(N, L, Lr):
    # rows of every length around a block's end, short of the order, and empty
    w = syn.random_small(601 + L, B=24, R=3, vocab=5, max_len=min(L, Lr), cand_stride=L,
                         ref_stride=Lr)
    for i in range(0, w.B, 2):
        w.cand_len[i], w.ref_len[i] = max(L - i // 4, 0), max(Lr - i // 8, 0)
        w.cand[i, :w.cand_len[i]] = (np.arange(w.cand_len[i]) * 7 + i) % 5
        w.refs[i, :, :max(Lr - i // 8, 0)] = (np.arange(max(Lr - i // 8, 0)) * 7 + i + i // 6) % 5
    check(w, N, int64=L % 2 == 1)


@pytest.mark.parametrize("B,R,L,vocab,N", [
    (300, 1, 90, 40, 4),        # two workgroups on a unit
    (1300, 1, 1000, 300, 4),    # six
    (1300, 4, 300, 50, 4),
    (2300, 2, 200, 500, 4),     # nine
    (1600, 3, 280, 3000, 4),    # seven
    (9000, 1, 40, 30, 4),       # as many workgroups as a unit takes
    (40, 2, 2700, 50257, 4),    # a unit for each, nine blocks a wavefront
    (600, 1, 4096, 2, 3),       # long runs: counters near their limit
    (70, 1, 7000, 50257, 4),    # longer than the path's own shapes
    (33, 1, 8192, 3, 8),
])
def test_plans(B, R, L, vocab, N):
    check(syn.random_small(B + L, B=B, R=R, vocab=vocab, max_len=L, min_len=L // 3), N)


@pytest.mark.parametrize("B", [256, 257])   # a unit for each workgroup, and one shared
@pytest.mark.parametrize("R,L,vocab,N", [
    (1, 100, 40, 4),
    (2, 4000, 3000, 2),
    (3, 2500, 300, 2),
    (62, 190, 50, 2),
    (2, 6200, 3000, 3),         # 24 blocks a wavefront, all of LDS: alone on the unit either way
    (3, 5000, 3000, 4),
    (62, 300, 50, 4),
])
def test_alone_on_a_unit(B, R, L, vocab, N):
    w = syn.random_small(680 + R, B=B, R=R, vocab=vocab, max_len=L, min_len=L // 2)
    check(w, N, rouge=R != 2)


@pytest.mark.parametrize("B,R,L,Lr,vocab,N", [
    (30, 16, 2984, 895, 1 << 23, 4),   # a table of 4096 slots 0.73 full, six bits for the probe count
    (12, 62, 1059, 105, 2000, 4),      # of 2048 slots 0.52 full
    (30, 4, 6144, 2000, 50257, 4),     # would be 0.75 full with four bits: not for this kernel
    (28, 3, 6144, 6144, 50257, 4),
])
def test_full_tables(B, R, L, Lr, vocab, N):
    w = syn.random_small(641 + L, B=B, R=R, vocab=vocab, max_len=min(L, Lr), min_len=min(L, Lr),
                         cand_stride=L, ref_stride=Lr)
    rng = np.random.default_rng(641)
    for i in range(B):
        w.cand[i], w.cand_len[i] = rng.integers(0, vocab, L), L
        for j in range(R):
            w.refs[i, j] = np.where(rng.random(Lr) < 0.2, w.refs[i, j], w.cand[i, j:j + Lr] if L >= j + Lr
                                    else w.cand[i, :Lr])
    check(w, N)


@pytest.mark.parametrize("N", [1, 4])
@pytest.mark.parametrize("R", [1, 2, 3])
def test_tokens_chosen_to_collide(R, N):
    # tokens that walk the same sequence of buckets, further than an entry can count (test_plans.py):
    # the loop that needs no table, for each way of counting matches
    ids, vocab = fused_rows.colliding_ids()
    w = syn.random_small(631, B=6, R=R, vocab=len(ids), max_len=400, min_len=300)
    w.cand, w.refs, w.vocab = ids[w.cand], ids[w.refs], vocab
    check(w, N)


def drawn(seed, B, R, cs, rs):
    """Every eighth row full, the others up to an eighth of it; between 3 and 100 different tokens a group,
    references that share three quarters of them with the candidate."""
    rng = np.random.default_rng(seed)
    full = (np.arange(B) % 8 == seed % 8) | (np.arange(B) < 2)
    cl = np.where(full, cs, rng.integers(0, cs // 8 + 2, B)).astype(np.int32)
    rl = np.where(full[:, None], rs, rng.integers(0, rs // 8 + 2, (B, R))).astype(np.int32)
    cl, rl = np.minimum(cl, cs), np.minimum(rl, rs)
    kinds = rng.choice([3, 20, 100], B).astype(np.int32)
    base = rng.integers(0, 1 << 30, (B, max(cs, rs)), dtype=np.int32) % kinds[:, None]

    def varied(rows, length):
        other = rng.integers(0, 100, rows.shape, dtype=np.int32)
        rows = np.where(rng.random(rows.shape, dtype=np.float32) < 0.25, other, rows)
        return np.where(np.arange(rows.shape[-1]) < length[..., None], rows, 0).astype(np.int32)

    cand = varied(base[:, :cs], cl)
    refs = varied(np.broadcast_to(base[:, None, :rs], (B, R, rs)), rl)
    return syn.Workload("drawn", 100, cand, cl, refs, rl)


def check_row(seed, mode, shape):
    B, R, cs, rs, N = shape
    w = drawn(seed, B, R, cs, rs)
    print(mode, shape, flush=True)
    if mode != "rouge":
        check(w, N, int64=seed % 2 == 1, rouge=False)
        return
    want = oracle.rouge_n(w.cand, w.cand_len, w.refs, w.ref_len, n=N)
    prf, overlap, best = tb.tensorrouge_n(dev(w.cand), dev(w.cand_len), dev(w.refs), dev(w.ref_len), n=N,
                                          vocab_size=w.vocab, want_overlap=True, want_best=True)
    check_rouge(want, overlap.cpu().numpy(), best.cpu().numpy(), prf.cpu().numpy(), TOL)


@pytest.mark.parametrize("kernel", list(fused_rows.KERNELS), ids=str)
def test_every_kernel(kernel):
    for blocks, shape in fused_rows.KERNELS[kernel].items():
        check_row(690 + blocks, kernel[2], shape)


@pytest.mark.parametrize("N", [1, 2, 3])
@pytest.mark.parametrize("alone", [False, True])
def test_rouge_kernels(alone, N):
    # ROUGE-1 and -2 on kernels without what longer orders need, every number of blocks; ROUGE-3 beside them
    for blocks, shape in fused_rows.ROUGE[alone].items():
        check_row(740 + blocks, "rouge", (*shape, N))


@pytest.mark.parametrize("way", list(fused_rows.PASSES))
def test_every_way_to_divide_the_orders(way):
    for i, (alone, mode, shape) in enumerate(fused_rows.PASSES[way]):
        check_row(720 + i, mode, shape)


@pytest.mark.parametrize("N", [5, 6, 7, 8])
@pytest.mark.parametrize("B,R", [(20, 1), (300, 1), (20, 2), (300, 2), (300, 3), (20, 4), (300, 6)])
def test_orders_beyond_four(B, R, N):
    # several stretches of orders with one table and one set of counters, workgroups alone on a unit and
    # not; short cycles, so that the upper orders have matches
    w = syn.random_small(671 + R, B=B, R=R, vocab=4, max_len=150, min_len=3)
    for i in range(0, w.B, 2):
        w.cand[i] = np.arange(w.cand.shape[1]) % (2 + i % 11)
        w.refs[i] = np.arange(w.refs.shape[2]) % (2 + i % 13)
    w.vocab = 16
    check(w, N, int64=N == 7, rouge_n=N)


@pytest.mark.parametrize("N", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("R", [1, 2, 3, 4, 7])
def test_counters(R, N):
    # Counters of one, two and more references, an odd and an even number of orders in a pass, several
    # passes: short cycles of tokens, so that counts are large and either side has more of an n-gram
    # (differences below zero), with fewer references in use than there are rows.
    w = syn.random_small(661 + R, B=40, R=R, vocab=3, max_len=200, min_len=1)
    rng = np.random.default_rng(661 + 10 * R + N)
    for i in range(0, w.B, 2):
        n = int(rng.integers(1, 4))
        w.cand[i] = np.arange(w.cand.shape[1]) % n
        w.refs[i] = (np.arange(w.refs.shape[2]) // int(rng.integers(1, 5)) + i) % 3
    used = rng.integers(1, R + 1, w.B).astype(np.int32)
    ref = oracle.bleu(w.cand, w.cand_len, w.refs, w.ref_len, max_n=N, smoothing="exp", threads=8,
                      ref_count=used)
    stats = tb.Stats.allocate(w.B, N, DEV)
    cfg = tb.make_config(max_n=N, smoothing="exp", vocab_size=w.vocab, ref_count=dev(used))
    out = tb.tensorbleu_sentence(dev(w.cand), dev(w.cand_len), dev(w.refs), dev(w.ref_len), cfg, stats=stats)
    np.testing.assert_array_equal(stats.clipped.cpu().numpy(), ref.clipped)
    np.testing.assert_array_equal(stats.total.cpu().numpy(), ref.total)
    np.testing.assert_array_equal(stats.closest_ref_len.cpu().numpy(), ref.closest_ref_len)
    np.testing.assert_array_equal(stats.group_distinct.cpu().numpy(), ref.cand_distinct)
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref.bleu).max() <= TOL
    check(w, N)
