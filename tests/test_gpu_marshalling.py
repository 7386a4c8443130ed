"""Calls that the native marshalling takes and calls that it leaves to the general way give the same
results; what it must not take raises."""
import threading

import numpy as np
import pytest
import torch

import paper_2510_05485_amd as tb
import synth_inputs as syn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def batch(seed, B=21, R=2, L=70):
    w = syn.random_small(seed, B=B, R=R, vocab=60, max_len=L, min_len=1)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    return [to(w.cand), to(w.cand_len), to(w.refs), to(w.ref_len)], w


def other_forms(a):
    """The same batch in forms that the general way converts."""
    cand, cl, refs, rl = a
    wide = torch.zeros(cand.shape[0], 2 * cand.shape[1], dtype=cand.dtype, device=DEV)
    wide[:, ::2] = cand
    yield [wide[:, ::2], cl, refs, rl]                      # not contiguous
    yield [cand, cl.long(), refs, rl.long()]                # int64 lengths
    yield [cand, cl, list(refs.unbind(1)), rl]              # a list of references
    yield [cand.long(), cl, refs.long(), rl]                # int64 ids: natively, too


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("counts", [False, True])
def test_both_ways_agree(dtype, counts):
    a, w = batch(711)
    count = torch.arange(w.B, device=DEV, dtype=torch.int32) % w.R + 1 if counts else None
    mk = lambda: tb.BleuScorer(w.B, w.R, w.cand.shape[1], w.refs.shape[2], vocab_size=60,
                               smoothing="exp", score_dtype=dtype, want_stats=True)
    s = mk()
    want, clipped = s(*a, count).clone(), s.stats.clipped.clone()
    corpus = s.corpus(*a, count).clone()
    kw = dict(vocab_size=60, smoothing="exp", score_dtype=dtype)
    rouge = tb.rouge_n(*a, vocab_size=60, ref_count=count, score_dtype=dtype)
    for form in other_forms(a):
        t = mk()
        assert torch.equal(t(*form, None if count is None else count.long()), want)
        assert torch.equal(t.stats.clipped, clipped)
        assert torch.equal(t.corpus(*form, count), corpus)
        assert torch.equal(tb.rouge_n(*form, vocab_size=60, ref_count=count, score_dtype=dtype), rouge)
        if count is None:
            assert torch.equal(tb.sentence_bleu(*form, **kw), want)
            assert torch.equal(tb.corpus_bleu(*form, **kw), corpus)
            assert torch.equal(tb.corpus_bleu(*form, weights=[0.25] * 4, **kw), corpus)
    assert torch.equal(s(*a), mk()(*a))                     # ref_count of an earlier call is gone


def test_streams_and_threads():
    jobs = [batch(720 + i) for i in range(4)]
    scorers = [tb.BleuScorer(w.B, w.R, w.cand.shape[1], w.refs.shape[2], vocab_size=60)
               for _, w in jobs]
    want = [s(*a).clone() for s, (a, _) in zip(scorers, jobs)]
    torch.cuda.synchronize()
    got = [None] * len(jobs)

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(20):
                scorers[i].out.zero_()
                got[i] = scorers[i](*jobs[i][0]).clone()
        stream.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for g, x in zip(got, want):
        assert torch.equal(g, x)


def test_errors_are_raised():
    a, w = batch(731)
    s = tb.BleuScorer(w.B, w.R, w.cand.shape[1], w.refs.shape[2], vocab_size=60)
    cases = [
        lambda: s(a[0][:-1], a[1][:-1], a[2][:-1], a[3][:-1]),
        lambda: s(a[0].float(), *a[1:]),
        lambda: s(a[0].cpu(), *a[1:]),
        lambda: s(*a, a[1][:-1]),
        lambda: tb.rouge_n(*a, n=9, vocab_size=60),
        lambda: tb.corpus_bleu(*a, vocab_size=0),
        lambda: tb.tensorbleu_sentence(*a, tb.make_config(vocab_size=60),
                                       workspace=torch.empty(16, dtype=torch.uint8, device=DEV)),
        lambda: tb.tensorbleu_sentence(*a, tb.make_config(vocab_size=60),
                                       out=torch.empty(w.B + 1, device=DEV)),
    ]
    for f in cases:
        with pytest.raises(tb.TensorBLEUError):
            f()
