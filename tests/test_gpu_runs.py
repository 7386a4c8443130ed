"""The sorted-run kernels (whole calls on groups beyond one LDS table) against the CPU oracle: edges of
their chunks, short and empty rows, n-grams of more than 64 bits, counters of 16 and 32 bits, one and
several words of them, reference lists, with and without the dictionary sizes."""
import numpy as np
import pytest
import torch

import long_rows
import oracle
import paper_2510_05485_amd as tb
import synth_inputs as syn
from rouge_validity import check_rouge

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-5     # scores; whole numbers are exact


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def check(w, N, int64=False, rouge_n=2, lists=None, counts=None):
    cand, cl = dev(w.cand), dev(w.cand_len)
    rows, lens = (w.refs, w.ref_len) if lists is None else lists[:2]
    refs, rl = dev(rows), dev(lens)
    if int64:
        cand, refs = cand.long(), refs.long()
    extra, host = {}, {}
    if lists is not None:
        extra = dict(ref_offsets=dev(lists[2]), max_refs=w.R)
        host = dict(ref_offsets=lists[2])
    if counts is not None:
        extra, host = dict(ref_count=dev(counts)), dict(ref_count=counts)
    ref = oracle.bleu(w.cand, w.cand_len, rows, lens, max_n=N, smoothing="exp", threads=8, **host)
    for fn in (tb.tensorbleu_sentence, tb.tensorbleu_corpus):
        for sizes in (True, False):
            cfg = tb.make_config(max_n=N, smoothing="exp", vocab_size=w.vocab, **extra)
            st = tb.Stats.allocate(w.B, N, DEV)
            if not sizes:
                st.group_distinct = None
            out = fn(cand, cl, refs, rl, cfg, stats=st).cpu().numpy().astype(np.float64)
            assert st.device_status.item() == 0
            np.testing.assert_array_equal(st.clipped.cpu().numpy(), ref.clipped)
            np.testing.assert_array_equal(st.total.cpu().numpy(), ref.total)
            np.testing.assert_array_equal(st.closest_ref_len.cpu().numpy(), ref.closest_ref_len)
            np.testing.assert_array_equal(st.corpus_stats.cpu().numpy(), ref.corpus_stats)
            if sizes:
                np.testing.assert_array_equal(st.group_distinct.cpu().numpy(), ref.group_distinct)
            if fn is tb.tensorbleu_corpus:
                assert abs(out[0] - ref.corpus_bleu) <= TOL
            else:
                assert np.abs(out - ref.bleu).max() <= TOL
    n = min(N, rouge_n)
    want = oracle.rouge_n(w.cand, w.cand_len, rows, lens, n=n, **host)
    prf, overlap, best = tb.tensorrouge_n(cand, cl, refs, rl, n=n, vocab_size=w.vocab,
                                          want_overlap=True, want_best=True, **extra)
    check_rouge(want, overlap.cpu().numpy(), best.cpu().numpy(), prf.cpu().numpy(), TOL)


@pytest.mark.parametrize("B,R,L,Lr,vocab,N", [
    (1, 1, 7000, 7000, 50257, 4),      # 1024 positions a chunk
    (2, 1, 8192, 8193, 300, 4),        # rows that end with a chunk and one behind it
    (20, 1, 9000, 8000, 50257, 4),     # 2048 a chunk
    (25, 3, 6000, 6100, 3000, 4),      # 4096 a chunk, two counter words
    (3, 8, 4096, 4097, 400, 4),        # five counter words
    (2, 20, 700, 700, 12, 3),          # many short references
    (2, 1, 9000, 4000, 10000, 5),      # 70 bits at order 5: partition takes the rest
    (4, 1, 9000, 9000, 262144, 4),     # 72 bits: part of the table, too
    (1, 1, 40000, 100, 262144, 4),
    (1, 1, 70000, 66000, 2, 4),        # 32-bit counters
    (2, 1, 7000, 7000, 200, 8),        # orders up to eight of exactly 64 bits
    (1, 1, 100, 30000, 50, 2),         # candidate much shorter than the reference
])
def test_shapes(B, R, L, Lr, vocab, N):
    w = syn.random_small(811 + L, B=B, R=R, vocab=vocab, max_len=min(L, Lr), min_len=min(L, Lr) // 2,
                         cand_stride=L, ref_stride=Lr)
    if B > 1:                          # empty rows, and rows shorter than an n-gram
        w.cand_len[0], w.ref_len[1, 0] = 2, 0
    check(w, N, int64=B % 2 == 0, rouge_n=N if vocab == 10000 else 2)


@pytest.mark.parametrize("B,R,L,Lr,vocab,N", list(long_rows.RUNS))
def test_shapes_that_are_not_dealt(B, R, L, Lr, vocab, N):
    # (many of the shapes above go to the kernels for dealt positions on AUTO)
    w = syn.random_small(815 + L, B=B, R=R, vocab=vocab, max_len=min(L, Lr), min_len=min(L, Lr) // 2,
                         cand_stride=L, ref_stride=Lr)
    if B > 1:
        w.cand_len[0], w.ref_len[1, 0] = 2, 0
    check(w, N, int64=B % 2 == 0)


def test_frequent_tokens_of_five_orders():
    check(syn.long_form(B=1, L=100000, vocab=9000), 5)


@pytest.mark.parametrize("B,R,L,Lr,vocab,N", [
    (2, 16, 4096, 700, 262144, 4),     # parts of 64 slots, the smallest
    (1, 16, 8192, 1000, 262144, 4),    # of 128
])
def test_parts_of_a_table(B, R, L, Lr, vocab, N):
    # every n-gram another one: the table's parts as full as the plan reckons with
    w = syn.random_small(871, B=B, R=R, vocab=vocab, max_len=min(L, Lr), min_len=min(L, Lr),
                         cand_stride=L, ref_stride=Lr)
    rng = np.random.default_rng(871)
    for i in range(B):
        w.cand[i], w.cand_len[i] = rng.permutation(vocab)[:L], L
        for j in range(R):
            w.refs[i, j] = w.cand[i, 64 * j:64 * j + Lr]
    check(w, N)


@pytest.mark.parametrize("length", [1024, 1025, 4095, 8192])
def test_chunk_edges(length):
    # the length ends a chunk, starts one, or leaves fewer positions than an n-gram has
    w = syn.random_small(821, B=3, R=1, vocab=900, max_len=8192, min_len=8192)
    for i in range(3):
        w.cand_len[i], w.ref_len[i, 0] = length + i, length + 3 - i
    w.cand_len, w.ref_len = np.minimum(w.cand_len, 8192), np.minimum(w.ref_len, 8192)
    check(w, 4)


def test_one_text_of_many_chunks_with_frequent_tokens():
    w = syn.long_form(B=1, L=100000, vocab=50257)
    check(w, 4)


def test_all_ones_keys():
    # 4-grams of 64 set bits look like a free table slot; they are the most frequent ones here
    w = syn.random_small(831, B=2, R=2, vocab=65536, max_len=6500, min_len=6000)
    w.cand[:, 100:4000] = 65535
    w.refs[:, :, 3000:5000] = 65535
    check(w, 4)
    w = syn.random_small(832, B=2, R=1, vocab=131072, max_len=9000, min_len=8000)  # 68 bits
    w.cand[:, 100:4000] = 131071
    w.cand[:, 4000:4003], w.refs[:, 0, 10:13] = 131071, 131071
    w.refs[:, :, 3000:5000] = 131071
    check(w, 4)


def test_lists_and_counts():
    w = syn.random_small(841, B=10, R=6, vocab=5000, max_len=3000, min_len=2000)
    counts = syn.ref_counts(841, w.B, w.R)
    check(w, 4, counts=counts)
    check(w, 4, lists=syn.pack_reference_lists(w.refs, w.ref_len, counts))


def test_replays_of_a_captured_call():
    ws = [syn.random_small(s, B=3, R=1, vocab=50257, max_len=7000, min_len=6500) for s in (851, 852)]
    scorer = tb.BleuScorer(3, 1, 7000, 7000, vocab_size=50257, smoothing="exp", device=DEV)
    held = [dev(a) for a in (ws[0].cand, ws[0].cand_len, ws[0].refs, ws[0].ref_len)]
    scorer(*held)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = scorer(*held)
    for w in (ws[0], ws[1], ws[0]):
        for t, a in zip(held, (w.cand, w.cand_len, w.refs, w.ref_len)):
            t.copy_(dev(a))
        graph.replay()
        torch.cuda.synchronize()
        ref = oracle.bleu(w.cand, w.cand_len, w.refs, w.ref_len, smoothing="exp")
        assert np.abs(out.cpu().numpy() - ref.bleu).max() <= TOL


def test_tokens_chosen_to_collide_are_reported():
    # tokens of one hash partition, however many partitions there are: more than its table holds
    M = 1 << 32
    tokens = np.arange(1 << 22, dtype=np.uint64)
    h = (tokens * 0x9E3779B1) % M
    h = ((h ^ (h >> 15)) * 0x85EBCA6B + 0x27D4EB2F) % M
    ids = tokens[h >> 23 == 0][:7000].astype(np.int32)
    assert len(ids) == 7000
    w = syn.random_small(861, B=2, R=1, vocab=1 << 22, max_len=7000, min_len=7000)
    w.cand[0], w.refs[0, 0] = ids, ids[::-1]
    cfg = tb.make_config(vocab_size=w.vocab, max_n=1)
    st = tb.Stats.allocate(2, 1, DEV)
    out = tb.tensorbleu_sentence(dev(w.cand), dev(w.cand_len), dev(w.refs), dev(w.ref_len), cfg,
                                 stats=st)
    assert st.device_status.item() == tb.TB_DEV_TABLE_OVERFLOW
    ref = oracle.bleu(w.cand, w.cand_len, w.refs, w.ref_len, max_n=1)
    got = out.cpu().numpy()
    assert np.isnan(got[0]) and abs(got[1] - ref.bleu[1]) <= TOL
