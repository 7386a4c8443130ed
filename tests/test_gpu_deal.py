"""The kernels that deal every position of a long group out once, against the CPU oracle: edges of their chunks,
short and empty rows, one to four orders, counters of 32 and 16 bits, several windows of members, reference
lists, 4-grams that need more ids than a partition has; with and without dictionary sizes, and ROUGE-1 and -2."""
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


def check(w, N, int64=False, lists=None, counts=None):
    # (the kernels are for so many positions in all, and for rows beyond the fused kernel's)
    assert w.B * (w.cand.shape[1] + w.R * w.refs.shape[2]) >= (98304 if w.R <= 4 else 262144)
    cand, cl = dev(w.cand), dev(w.cand_len)
    rows, lens = (w.refs, w.ref_len) if lists is None else lists[:2]
    refs, rl = dev(rows), dev(lens)
    if int64:
        cand, refs = cand.long(), refs.long()
    extra, host = {}, {}
    if lists is not None:
        extra, host = dict(ref_offsets=dev(lists[2]), max_refs=w.R), dict(ref_offsets=lists[2])
    if counts is not None:
        extra, host = dict(ref_count=dev(counts)), dict(ref_count=counts)
    ref = oracle.bleu(w.cand, w.cand_len, rows, lens, max_n=N, smoothing="exp", threads=8, **host)
    cfg = tb.make_config(max_n=N, smoothing="exp", vocab_size=w.vocab, **extra)
    for fn, sizes in ((tb.tensorbleu_sentence, False), (tb.tensorbleu_sentence, True), (tb.tensorbleu_corpus, False)):
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
    for n in (1, 2):
        want = oracle.rouge_n(w.cand, w.cand_len, rows, lens, n=n, **host)
        prf, overlap, best = tb.tensorrouge_n(cand, cl, refs, rl, n=n, vocab_size=w.vocab,
                                              want_overlap=True, want_best=True, **extra)
        check_rouge(want, overlap.cpu().numpy(), best.cpu().numpy(), prf.cpu().numpy(), TOL)


@pytest.mark.parametrize("B,R,L,Lr,vocab,N", list(long_rows.DEALT))
def test_shapes(B, R, L, Lr, vocab, N):
    w = syn.random_small(911 + L, B=B, R=R, vocab=vocab, max_len=min(L, Lr), min_len=min(L, Lr) // 2,
                         cand_stride=L, ref_stride=Lr)
    if B > 1:                                # empty rows, and rows shorter than an n-gram
        w.cand_len[0], w.ref_len[1, 0] = 2, 0
    check(w, N, int64=B % 2 == 0)


@pytest.mark.parametrize("length", [1023, 1024, 1026, 2047, 2048, 2050, 4096, 13000])
def test_chunk_edges(length):
    # the length ends a chunk, starts one, or leaves fewer positions than an n-gram has
    for B in (4, 24):                        # 1024 and 2048 positions a chunk
        w = syn.random_small(921, B=B, R=1, vocab=900, max_len=13000, min_len=13000)
        for i in range(B):
            w.cand_len[i], w.ref_len[i, 0] = length + i % 4, length + 3 - i % 4
        w.cand_len, w.ref_len = np.minimum(w.cand_len, 13000), np.minimum(w.ref_len, 13000)
        check(w, 4)


def test_frequent_tokens():
    w = syn.long_form(B=2, L=100000, vocab=50257)
    check(w, 4)


def test_repetition():
    # one token, and a few of them: a partition receives whole chunks, merged
    w = syn.random_small(931, B=4, R=1, vocab=50257, max_len=40000, min_len=39000)
    w.cand[0], w.refs[0] = 7, 7
    w.cand[1, 100:30000] = 9
    w.refs[2, 0, 500:39000] = np.resize(np.arange(11), 38500)
    w.cand[2, 1000:20000] = np.resize(np.arange(11), 19000)
    check(w, 4)


@pytest.mark.parametrize("vocab", [2, 4, 13])
@pytest.mark.parametrize("B,R,L,N", long_rows.FEW_TOKENS)
def test_few_different_tokens(B, R, L, N, vocab):
    # all lanes enter the same n-grams at once: ids are taken in vain, given back and used again
    check(syn.random_small(991 + R, B=B, R=R, vocab=vocab, max_len=L, min_len=L - 100), N)


@pytest.mark.parametrize("N", [3, 4])
def test_equal_beginnings(N):
    # n-grams that are merged by three tokens, but not by four, and those at the ends of rows
    w = syn.random_small(996, B=12, R=1, vocab=900, max_len=6000, min_len=5000)
    w.cand[:, ::4], w.cand[:, 1::4], w.cand[:, 2::4] = 3, 4, 5
    w.refs[:, :, ::4], w.refs[:, :, 1::4], w.refs[:, :, 2::4] = 3, 4, 5
    for i in range(12):
        w.cand_len[i], w.ref_len[i, 0] = (1026, 2050, 4098)[i % 3] + i // 3, (2050, 4097)[i % 2] + i // 4
    check(w, N)


@pytest.mark.parametrize("R,N", [(1, 4), (2, 4), (1, 3), (3, 4)])
def test_more_ids_than_a_partition_has(R, N):
    # 4-grams of one beginning, a quarter of the text: counted in shares (with three orders the beginnings are merged,
    # and there are enough ids)
    w = syn.random_small(941, B=2, R=R, vocab=50257, max_len=30000, min_len=29000)
    rng = np.random.default_rng(941)
    for i in range(2):
        text = np.full(30000, 5, dtype=np.int32)
        text[3::4] = rng.permutation(50000)[:7500] + 100
        w.cand[i] = text
        for j in range(R):
            other = text.copy()
            other[3 + 4 * j:20000:8] = 17
            w.refs[i, j] = other
    check(w, N)


# What chooses a 4-gram's partition (of its first three tokens) and, where order 4 is counted in shares, its share.
def hashes(t0, t1, t2, t3):
    M = np.uint64(0xFFFFFFFF)
    mul = lambda x, c: (np.asarray(x, dtype=np.uint64) * np.uint64(c)) & M
    mix = lambda h: mul(h ^ (h >> np.uint64(15)), 0xC2B2AE3D)
    h3 = mix((mul(t0, 0x9E3779B1) + mul(t1, 0x85EBCA6B) + mul(t2, 0x27D4EB2F)) & M)
    return h3, mul(mix((h3 + mul(t3, 0x165667B1)) & M), 0x9E3779B1)


def behind_beginnings(seed, B, R, L, vocab, each, beginnings, ids=None):
    """Texts with `each` 4-grams behind each of the beginnings (b, b, b), another token behind it every time, a half of
    them in the references, too; the rest random."""
    w = syn.random_small(seed, B=B, R=R, vocab=vocab, max_len=L, min_len=L - 50)
    rng = np.random.default_rng(seed)
    for i in range(B):
        at = 4 * rng.permutation(L // 4)[:each * beginnings]
        x = rng.permutation(vocab if ids is None else ids)[:each]
        for k in range(3):
            w.cand[i, at + k] = 1 + np.repeat(np.arange(beginnings), each)
        w.cand[i, at + 3] = np.resize(x, len(at))
        for j in range(R):
            w.refs[i, j] = np.where(rng.random(L) < 0.5, w.cand[i], w.refs[i, j])
            some = at[rng.random(len(at)) < 0.5]
            for k in range(4):
                w.refs[i, j, some + k] = w.cand[i, some + k]
    return w


@pytest.mark.parametrize("B,R,L,each,beginnings", long_rows.CROWDED)
def test_crowded_partitions(B, R, L, each, beginnings):
    check(behind_beginnings(1001 + L + each, B, R, L, 50257, each, beginnings), 4)


@pytest.mark.parametrize("part,each", [(16, 900), (100, 1200)])
def test_shares_of_uneven_size(part, each):
    # all 4-grams of the beginning in the first sixteenth or hundredth of the hashes: shares are divided several times,
    # in the end one lane of a wavefront goes after the other
    vocab = (1 << 20) - 2
    x = np.arange(10, vocab)
    ids = x[hashes(1, 1, 1, x)[1] < (1 << 32) // part].astype(np.int32)
    check(behind_beginnings(1011, 2, 1, 30000, vocab, each, 1, ids), 4)


def test_members_beyond_a_window():
    # pairs and 4-grams of few tokens: unmerged in part, far more of them in a partition than its share
    w = syn.random_small(951, B=2, R=1, vocab=13, max_len=60000, min_len=60000)
    check(w, 4)
    w = syn.random_small(952, B=4, R=3, vocab=40, max_len=20000, min_len=18000)
    check(w, 4)


def test_lists_and_counts():
    for R, L in ((6, 6000), (3, 12500)):
        w = syn.random_small(961, B=10, R=R, vocab=5000, max_len=L, min_len=L - 1000)
        counts = syn.ref_counts(961, w.B, w.R)
        counts[0], counts[1] = R, 1
        check(w, 4, counts=counts)
        check(w, 4, lists=syn.pack_reference_lists(w.refs, w.ref_len, counts))


def test_tokens_outside_the_vocabulary_are_reported():
    w = syn.random_small(971, B=4, R=1, vocab=3000, max_len=20000, min_len=20000)
    for bad, where in ((3000, 0), (-1, 19999), (1 << 33, 2048)):
        cand, refs = dev(w.cand).long(), dev(w.refs).long()
        cand[3, where] = bad
        w.cand[3, where] = 0
        st = tb.Stats.allocate(4, 4, DEV)
        st.group_distinct = None
        cfg = tb.make_config(vocab_size=3000, smoothing="exp")
        tb.tensorbleu_sentence(cand, dev(w.cand_len), refs, dev(w.ref_len), cfg, stats=st)
        assert st.device_status.item() == tb.TB_DEV_TOKEN_RANGE
        ref = oracle.bleu(w.cand, w.cand_len, w.refs, w.ref_len, smoothing="exp", threads=4)
        np.testing.assert_array_equal(st.clipped.cpu().numpy(), ref.clipped)


@pytest.mark.parametrize("R", [1, 2])
def test_scores_are_those_of_the_stages(R):
    # bit by bit: of the same whole numbers, by the same steps
    w = syn.random_small(1021, B=20, R=R, vocab=900, max_len=12000, min_len=6000)
    args = [dev(a) for a in (w.cand, w.cand_len, w.refs, w.ref_len)]
    for smoothing, param in (("none", 0.0), ("floor", 0.1), ("add-k", 1.0), ("exp", 0.0)):
        for fn in (tb.tensorbleu_sentence, tb.tensorbleu_corpus):
            here, there = (fn(*args, tb.make_config(vocab_size=w.vocab, smoothing=smoothing, smooth_param=param, path=path))
                           for path in ("auto", "global"))
            assert torch.equal(here.view(torch.int32), there.view(torch.int32))


def test_a_table_that_tokens_fill_is_reported():
    # 5000 tokens of one partition, whose table has 4096 slots: reported, that sentence scored NaN, and the corpus
    vocab = (1 << 20) - 2
    tokens = np.arange(vocab, dtype=np.uint64)
    ids = tokens[((tokens * np.uint64(0x9E3779B1) + np.uint64(0x6A09E667)) & np.uint64(0xFFFFFFFF)) < (1 << 32) // 16]
    w = syn.random_small(1031, B=4, R=1, vocab=vocab, max_len=20000, min_len=20000)
    w.cand[2, 100:5100] = ids[:5000]
    args = [dev(a) for a in (w.cand, w.cand_len, w.refs, w.ref_len)]
    ref = oracle.bleu(w.cand, w.cand_len, w.refs, w.ref_len, max_n=1)
    for fn in (tb.tensorbleu_sentence, tb.tensorbleu_corpus):
        st = tb.Stats.allocate(4, 1, DEV)
        st.group_distinct = None
        out = fn(*args, tb.make_config(max_n=1, vocab_size=vocab), stats=st).cpu().numpy()
        assert st.device_status.item() == tb.TB_DEV_TABLE_OVERFLOW
        if fn is tb.tensorbleu_corpus:
            assert np.isnan(out[0])
        else:
            assert np.isnan(out[2]) and np.abs(np.delete(out - ref.bleu, 2)).max() <= TOL
    cfg = tb.make_config(max_n=1, vocab_size=vocab)
    cfg.workspace_tables = 1                 # the way to re-issue the call
    assert abs(tb.tensorbleu_sentence(*args, cfg).cpu().numpy()[2] - ref.bleu[2]) <= TOL


def test_replays_of_a_captured_call():
    ws = [syn.random_small(s, B=3, R=1, vocab=50257, max_len=20000, min_len=19000) for s in (981, 982)]
    scorer = tb.BleuScorer(3, 1, 20000, 20000, vocab_size=50257, smoothing="exp", device=DEV)
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
