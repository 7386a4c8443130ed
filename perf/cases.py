"""The work that users of this framework have it do, as cases to be timed.

A case is one call of a public entry point on a batch of token-ID sequences that already lives on
the GPU, together with the plan (scorer, workspace) that a user's program keeps between calls.
`listed()` names twelve of them, `draw()` gives more of the same ranges.

Fields of a case
  entry    "scorer"   BleuScorer.__call__: one score per candidate (a reward function)
           "corpus"   BleuScorer.corpus: one score for the batch (an evaluation loop)
           "oneshot"  corpus_bleu: the same without a scorer kept (an evaluation script)
           "lists"    tensorbleu_sentence with reference lists in CSR form
           "rouge"    rouge_n of order max_n
  B, R     candidates, and the largest number of references of one
  L, Lr    row length of candidates and references
  low      lengths are uniform in [low * L, L] (references: of Lr); 1.0: every row is full
  vocab    token ids are Zipf(1.1) ranks below it, or uniform where it is at most 256
  sub      share of the candidate's tokens that differ from the text it shares with its references
  ids      token dtype; scores: score dtype; stats: the integer statistics are asked for, too
  counts   candidates use 1..R of their references (ref_count)
"""
import torch

import paper_2510_05485_amd as tb

DEVICE = "cuda:0"
REF_SUB = 0.3           # share of a reference's tokens that differ from the shared text

DEFAULTS = dict(entry="scorer", B=16, R=1, L=256, Lr=256, low=1.0, vocab=32000, sub=0.3,
                ids="int32", scores="float32", stats=False, counts=False, max_n=4,
                smoothing="none", param=0.0)


def _case(name=None, **kw):
    case = dict(DEFAULTS, **kw)
    if "Lr" not in kw:
        case["Lr"] = case["L"]
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: one prompt's rollouts in a reward loop (benchmark configuration 1)
        _case("reward_16x256", B=16, L=256, smoothing="add-k", param=1.0),
        # a training batch with ragged rows; the trainer keeps rewards in bfloat16 (configuration 2)
        _case("reward_256x1024_bf16", B=256, L=1088, Lr=1024, low=0.9, vocab=50257,
              smoothing="floor", param=0.1, scores="bfloat16"),
        # the headline configuration: four references of different lengths (configuration 3)
        _case("reward_512x1024_r4", B=512, R=4, L=1024, Lr=1280, low=0.6, vocab=50257, sub=0.4,
              smoothing="exp"),
        # large vocabulary, corpus score and every statistic (configuration 4)
        _case("corpus_1024x2048_v262144", entry="corpus", B=1024, L=2048, vocab=262144, sub=0.25,
              smoothing="add-k", param=1.0, stats=True),
        # many short ragged rows over a tiny vocabulary: heavy repetition (configuration 5)
        _case("ragged_4096x512_v64", B=4096, R=2, L=512, Lr=640, low=0.06, vocab=64, sub=0.5,
              smoothing="floor", param=0.1, stats=True),
        # the largest: a whole rollout of a policy, ids as the tokenizer gives them (int64)
        _case("rollout_4096x2048_r2_int64", B=4096, R=2, L=2048, low=0.25, vocab=50257,
              ids="int64", smoothing="exp"),
        # ROUGE-2 of summaries against three references with unequal numbers in use
        _case("rouge2_512x512_r3", entry="rouge", B=512, R=3, L=512, low=0.3, vocab=50257,
              counts=True, max_n=2),
        # corpus BLEU of a translation test set by the one-shot function
        _case("testset_2000x64_int64", entry="oneshot", B=2000, L=64, low=0.12, vocab=32000,
              ids="int64", smoothing="none"),
        # captions with up to eight references each, packed without padding rows
        _case("lists_1000x96_r8", entry="lists", B=1000, R=8, L=96, low=0.2, vocab=32000,
              smoothing="floor", param=0.1),
        # document translation: rows beyond the length limits of the one-kernel path
        _case("documents_128x5000", B=128, L=5000, low=0.8, vocab=50257, ids="int64",
              smoothing="exp"),
        # long generations (the benchmark's long workload)
        _case("long_128x8192", B=128, L=8192, low=0.9, vocab=50257, smoothing="exp"),
        # one book-length text against its reference
        _case("book_1x262144", B=1, L=262144, low=0.9, vocab=50257, smoothing="exp"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["scorer", "scorer", "scorer", "corpus", "oneshot", "lists", "rouge",
                       "rouge", "long", "long", "long"])
    case = _case(entry="scorer" if kind == "long" else kind)
    if kind == "long":
        case["R"] = rng.choice([1, 1, 1, 2, 3])
        case["L"] = min(_log_int(rng, 4097, 262144), 524288 // (1 + case["R"]))
        case["entry"] = rng.choice(["scorer", "scorer", "corpus", "rouge"])
        case["vocab"] = _log_int(rng, 8000, 262144)
        tokens = 2_000_000
    else:
        case["L"] = _log_int(rng, 64 if kind == "scorer" else 16, 4096)
        case["R"] = rng.choice([1, 1, 1, 2, 3, 4, 8])
        case["vocab"] = _log_int(rng, 64, 262144)
        tokens = 12_000_000
    case["Lr"] = max(16, int(case["L"] * rng.uniform(0.8, 1.2)))
    if case["entry"] == "lists":
        case["R"] = rng.choice([2, 5, 8, 16])
        case["L"] = min(case["L"], 512)
        case["Lr"] = min(case["Lr"], 640)
    group = case["L"] + case["R"] * case["Lr"]
    case["B"] = _log_int(rng, 1, max(1, min(4096, tokens // group)))
    case["low"] = rng.choice([1.0, 0.9, 0.5, 0.1])
    case["sub"] = round(rng.uniform(0.1, 0.6), 3)
    case["ids"] = rng.choice(["int32", "int64"])
    case["smoothing"], case["param"] = rng.choice([("none", 0.0), ("floor", 0.1), ("add-k", 1.0),
                                                   ("exp", 0.0)])
    case["counts"] = case["R"] > 1 and case["entry"] in ("scorer", "rouge") and rng.random() < 0.3
    if case["entry"] == "rouge":
        case["max_n"] = rng.choice([1, 2, 2])
        case["smoothing"], case["param"] = "none", 0.0
    else:
        case["max_n"] = rng.choice([4, 4, 4, 2])
    if case["entry"] in ("scorer", "corpus"):
        case["stats"] = rng.random() < 0.3
    if case["entry"] == "scorer":
        case["scores"] = rng.choice(["float32", "float32", "bfloat16"])
    return case


class _Draw:
    """Seeded inputs, made on the GPU."""

    def __init__(self, case, seed):
        self.case = case
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(int(seed) * 1_000_003 + 17)
        self.cdf = None
        if case["vocab"] > 256:
            w = torch.arange(1, case["vocab"] + 1, dtype=torch.float64, device=DEVICE) ** -1.1
            cdf = torch.cumsum(w, 0)
            self.cdf = (cdf / cdf[-1]).to(torch.float32)

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.gen, device=DEVICE)

    def tokens(self, *shape):
        v = self.case["vocab"]
        if self.cdf is None:
            return torch.randint(0, v, shape, generator=self.gen, device=DEVICE, dtype=torch.int32)
        ranks = torch.searchsorted(self.cdf, self.uniform(*shape), right=True, out_int32=True)
        return ranks.clamp_(max=v - 1)

    def lengths(self, stride, *shape):
        lo = max(1, int(self.case["low"] * stride))
        return torch.randint(lo, stride + 1, shape, generator=self.gen, device=DEVICE,
                             dtype=torch.int32)

    def varied(self, base, share):
        """`base` with each token replaced by a fresh one with probability `share`."""
        return torch.where(self.uniform(*base.shape) < share, self.tokens(*base.shape), base)

    def padded(self, rows, lengths):
        """Rows cut at their lengths, padded with id 0, in the case's token dtype."""
        pos = torch.arange(rows.shape[-1], device=DEVICE, dtype=torch.int32)
        cut = torch.where(pos < lengths.unsqueeze(-1), rows, torch.zeros_like(rows))
        return cut.to(getattr(torch, self.case["ids"])).contiguous()


def prepare(case, seed):
    d = _Draw(case, seed)
    B, R, L, Lr = case["B"], case["R"], case["L"], case["Lr"]
    base = d.tokens(B, max(L, Lr))
    s = {"case": case}
    cand_len = d.lengths(L, B)
    s["cand"], s["cand_len"] = d.padded(d.varied(base[:, :L], case["sub"]), cand_len), cand_len
    if case["entry"] == "lists":
        counts = torch.randint(1, R + 1, (B,), generator=d.gen, device=DEVICE, dtype=torch.int32)
        offsets = torch.zeros(B + 1, dtype=torch.int32, device=DEVICE)
        offsets[1:] = torch.cumsum(counts, 0)
        owner = torch.repeat_interleave(torch.arange(B, device=DEVICE), counts.long())
        ref_len = d.lengths(Lr, owner.numel())
        s["refs"] = d.padded(d.varied(base[owner, :Lr], REF_SUB), ref_len)
        s["ref_len"] = ref_len
        s["cfg"] = tb.make_config(max_n=case["max_n"], smoothing=case["smoothing"],
                                  smooth_param=case["param"], vocab_size=case["vocab"],
                                  ref_offsets=offsets, max_refs=R)
        s["cfg"].token_bytes = 8 if case["ids"] == "int64" else 4
        s["workspace"] = tb.allocate_workspace(B, R, L, Lr, s["cfg"], DEVICE)
        s["out"] = torch.empty(B, dtype=torch.float32, device=DEVICE)
        return s
    ref_len = d.lengths(Lr, B, R)
    shared = base[:, :Lr].unsqueeze(1).expand(B, R, Lr)
    s["refs"], s["ref_len"] = d.padded(d.varied(shared, REF_SUB), ref_len), ref_len
    s["ref_count"] = None
    if case["counts"]:
        s["ref_count"] = torch.randint(1, R + 1, (B,), generator=d.gen, device=DEVICE,
                                       dtype=torch.int32)
    if case["entry"] in ("scorer", "corpus"):
        s["scorer"] = tb.BleuScorer(B, R, L, Lr, vocab_size=case["vocab"], max_n=case["max_n"],
                                    smoothing=case["smoothing"], smooth_param=case["param"],
                                    device=DEVICE, want_stats=case["stats"],
                                    score_dtype=getattr(torch, case["scores"]))
    return s


def run(state):
    s, case = state, state["case"]
    if case["entry"] == "lists":
        return tb.tensorbleu_sentence(s["cand"], s["cand_len"], s["refs"], s["ref_len"], s["cfg"],
                                      out=s["out"], workspace=s["workspace"])
    if case["entry"] == "rouge":
        return tb.rouge_n(s["cand"], s["cand_len"], s["refs"], s["ref_len"], n=case["max_n"],
                          vocab_size=case["vocab"], ref_count=s["ref_count"])
    if case["entry"] == "oneshot":
        return tb.corpus_bleu(s["cand"], s["cand_len"], s["refs"], s["ref_len"],
                              vocab_size=case["vocab"], max_n=case["max_n"],
                              smoothing=case["smoothing"], smooth_param=case["param"])
    call = s["scorer"].corpus if case["entry"] == "corpus" else s["scorer"]
    score = call(s["cand"], s["cand_len"], s["refs"], s["ref_len"], s["ref_count"])
    if not case["stats"]:
        return score
    st = s["scorer"].stats
    return {"score": score, "clipped": st.clipped, "total": st.total,
            "closest_ref_len": st.closest_ref_len, "group_distinct": st.group_distinct,
            "corpus_stats": st.corpus_stats}


def work(case):
    """Every token inside the lengths read once (expected lengths), every result written once.
    There is no arithmetic to speak of: a few dozen operations a score."""
    B, R, N = case["B"], case["R"], case["max_n"]

    def mean(stride):
        return (max(1, int(case["low"] * stride)) + stride) / 2

    refs = (R + 1) / 2 if case["counts"] or case["entry"] == "lists" else R
    tokens = B * (mean(case["L"]) + refs * mean(case["Lr"]))
    bytes_ = tokens * (8 if case["ids"] == "int64" else 4) + 4 * B * (1 + refs)
    if case["entry"] == "rouge":
        bytes_ += 12 * B
    else:
        bytes_ += 4 if case["entry"] in ("corpus", "oneshot") else \
            B * (2 if case["scores"] == "bfloat16" else 4)
    if case["stats"]:
        bytes_ += B * (12 * N + 4) + 8 * (2 * N + 2)
    return {"bytes": bytes_, "flops": 30 * B * N}


def tolerance(case):
    """Whole numbers are exact.  Scores are formed in float32; a bfloat16 score may be rounded
    to its neighbour.  ROUGE takes the best reference by a float32 quotient: near-ties between
    references may go either way."""
    if case["scores"] == "bfloat16":
        return {"rel": 5e-3, "max": 2e-2}
    if case["entry"] == "rouge":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-5, "max": 1e-4}
