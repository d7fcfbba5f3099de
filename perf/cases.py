"""Workloads for timing this framework: what its users have it do, through its public entry points.

The framework translates sets of sentences (token ids in, token ids out) with the student Transformer and its
relatives.  A program loads a model once, with an arena for its largest batches, and then calls

    translate_batch       host arrays in and out, batching inside (the usual call);
    translate_batch_eos   the same, a sentence ending at its end symbol;
    encode + decode_greedy   one padded batch that is already on the GPU, for callers that batch themselves.

Models and sizes are those of the repository's own configurations: the one-head student without FFN (with the fp16 and
with the 8-bit output layer), the tiny student, the ablation student (8 heads, FFN everywhere), the 30 + 6 layer
teacher with relative positions, and the submitted student (8-head encoder with FFN, one-head decoder with a narrow
one).  Sentences have lognormal lengths and Zipf token ids.
"""
import math

import numpy as np
import torch

import paper_2109_08003_amd as nt

EOS = 2
FIRST_ID = 4     # 0 .. 3 are the special symbols

_STUDENT = dict(n_enc=6, n_dec=1, d_model=512, n_heads=1, d_ffn=0, vocab=32000, max_len=256, rpr_clip=0, tie_output=0,
                bos_id=1, pad_id=0, ln_eps=1e-5, dec_n_heads=0, dec_d_ffn=0, ln_l1=0, q8_output=0)
MODELS = {
    "tiny": dict(_STUDENT, d_model=256, vocab=4000),
    "student": dict(_STUDENT),
    "ablation": dict(_STUDENT, n_heads=8, d_ffn=2048),
    "teacher": dict(_STUDENT, n_enc=30, n_dec=6, n_heads=8, d_ffn=2048, rpr_clip=8),
    "submitted": dict(_STUDENT, n_enc=3, n_heads=8, d_ffn=2048, dec_n_heads=1, dec_d_ffn=512),
}
ARENA = {"tiny": 16384, "student": 65536, "ablation": 65536, "teacher": 16384, "submitted": 65536}  # largest batch, tokens
MAX_LENGTH = 200  # longest source sentence

# A case:
#   model, q8 (8-bit output layer), l1 (L1-norm layer normalisation)
#   call        "translate", "eos" or "batch" (encode + decode_greedy)
#   sentences   how many
#   median, sigma   lengths are median * exp(sigma * N(0, 1)), rounded, in [1, 200]
#   budget, max_rows   caps of a batch: padded tokens, and rows (0 = none); unused for "batch"
_CASE = dict(model="student", q8=False, l1=False, call="translate", sentences=1, median=22, sigma=0.5, budget=4096, max_rows=0)


def listed():
    return [
        # one sentence of an interactive session: every launch of the path at one row, nothing but latency
        dict(_CASE, name="one sentence"),
        # the parity configuration: eight short sentences, narrow model
        dict(_CASE, name="tiny model", model="tiny", sentences=8, median=16, budget=256),
        # a page of text as one request
        dict(_CASE, name="page", sentences=45),
        # the paper-shaped configuration at its own small budget: batches of 30 to 350 rows
        dict(_CASE, name="4k budget", sentences=4096),
        # the middle of the budget sweep
        dict(_CASE, name="16k budget", sentences=16384, budget=16384),
        # the throughput configuration: 200,000 sentences at the best budget
        dict(_CASE, name="64k budget", sentences=200000, budget=65536),
        # long sentences, batched by the caller and resident on the GPU: 128 keys and more in every attention
        dict(_CASE, name="long sentences, on the GPU", call="batch", sentences=320, median=150, sigma=0.15),
        # sentences that end at their end symbol, under the paper's own caps (64,000 tokens, 3,072 sentences)
        dict(_CASE, name="end symbol", call="eos", sentences=32768, budget=64000, max_rows=3072),
        # the 8-bit output layer
        dict(_CASE, name="8-bit output", q8=True, sentences=32768, budget=65536),
        # 8 heads and FFN 2,048 in every layer
        dict(_CASE, name="ablation model", model="ablation", sentences=16384, budget=16384),
        # the deep teacher with relative positions
        dict(_CASE, name="teacher model", model="teacher", sentences=2048, budget=8192),
        # the submitted student, with the L1-norm the paper's GPU systems use
        dict(_CASE, name="submitted student", model="submitted", l1=True, sentences=32768, budget=65536),
    ]


def draw(rng):
    def between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    model = rng.choice(["student"] * 5 + ["tiny", "ablation", "teacher", "submitted", "submitted"])
    c = dict(_CASE, model=model, call=rng.choice(["translate"] * 3 + ["eos", "batch"]), median=between(8, 60),
             sigma=round(rng.uniform(0.2, 0.6), 2))
    c["q8"] = model == "student" and c["call"] != "batch" and rng.random() < 0.25
    c["l1"] = model == "submitted" or rng.random() < 0.1
    mean = c["median"] * math.exp(c["sigma"] ** 2 / 2)
    if c["call"] == "batch":
        c["median"], c["sigma"] = between(8, 150), round(rng.uniform(0.0, 0.2), 2)
        longest = min(MAX_LENGTH, c["median"] * math.exp(4 * c["sigma"]) + 1)
        c["sentences"] = between(1, min(4096, int(ARENA[model] / longest)))
        return c
    c["budget"] = between(1024, ARENA[model])
    c["max_rows"] = between(16, 4096) if rng.random() < 0.25 else 0
    # as many tokens as that model's own workload has, and no more decode steps than take a few tenths of a second
    most = {"tiny": 2e5, "student": 2.5e6, "ablation": 4e5, "teacher": 5e4, "submitted": 8e5}[model]
    steps = {"teacher": 500, "ablation": 2000}.get(model, 4000)
    rows = c["budget"] / mean if not c["max_rows"] else min(c["budget"] / mean, c["max_rows"])
    c["sentences"] = between(1, max(8, min(most / mean, rows * steps / (1.2 * mean + 2))))
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------

def _lengths(case):
    """One length for each of n equal slices of the distribution, so that every seed gives the same amount of work."""
    n = case["sentences"]
    q = (torch.arange(n, dtype=torch.float64) + 0.5) / n
    return torch.exp(math.log(case["median"]) + case["sigma"] * torch.special.ndtri(q)).round().clamp(1, MAX_LENGTH).to(torch.int64)


def _sentences(case, seed):
    """(token ids int32 [sum of lengths], offsets int64 [n + 1]), host arrays."""
    g = torch.Generator().manual_seed(seed)
    n, vocab = case["sentences"], MODELS[case["model"]]["vocab"]
    lens = _lengths(case)[torch.randperm(n, generator=g)]
    if case["call"] == "batch":
        lens = lens.sort(descending=True).values  # a caller that batches itself hands its rows over longest first
    offsets = torch.zeros(n + 1, dtype=torch.int64)
    torch.cumsum(lens, 0, out=offsets[1:])
    ranks = torch.arange(1, vocab - FIRST_ID + 1, dtype=torch.float64, device="cuda")
    cdf = torch.cumsum(ranks ** -1.1, 0)
    u = torch.rand(int(offsets[-1]), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(seed))
    ids = torch.searchsorted(cdf / cdf[-1], u).clamp_(max=vocab - FIRST_ID - 1) + FIRST_ID
    return ids.to(torch.int32).cpu().numpy(), offsets.numpy()


def _config(case):
    return dict(MODELS[case["model"]], ln_l1=int(case["l1"]), q8_output=int(case["q8"]))


def _norm_spans(cfg):
    """(offset, kind) of every layer-normalisation vector in the weight blob; the rest is matrices, biases, tables."""
    d, c = cfg["d_model"], cfg["rpr_clip"]
    at = cfg["vocab"] * d * (1 if cfg["tie_output"] else 2)
    spans = []

    def norm():
        nonlocal at
        spans.extend([(at, 1.0), (at + d, 0.0)])
        at += 2 * d

    def attention(heads, relative):
        nonlocal at
        at += 4 * (d * d + d) + ((2 * c + 1) * (d // heads) if relative and c else 0)

    def ffn(width):
        nonlocal at
        if width > 0:
            norm()
            at += 2 * d * width + width + d

    heads, width = cfg["dec_n_heads"] or cfg["n_heads"], cfg["dec_d_ffn"] or cfg["d_ffn"]
    for _ in range(cfg["n_enc"]):
        norm(), attention(cfg["n_heads"], True), ffn(cfg["d_ffn"])
    norm()
    for _ in range(cfg["n_dec"]):
        norm(), attention(heads, True), norm(), attention(heads, False), ffn(width)
    norm()
    assert at == nt.param_count(cfg)
    return spans


def _weights(cfg, ends_early):
    """fp16 weight blob: N(0, 1/d) entries, layer normalisations at gain 1 and offset 0.  ends_early scales the end
    symbol's row of the output matrix, so that sentences end at varied steps (random weights alone never emit it)."""
    d = cfg["d_model"]
    w = torch.randn(nt.param_count(cfg), device="cuda", generator=torch.Generator("cuda").manual_seed(7)) * d ** -0.5
    for at, value in _norm_spans(cfg):
        w[at:at + d] = value
    if ends_early:
        row = (cfg["vocab"] + EOS) * d
        w[row:row + d] *= 1.6
    return w.half().cpu().numpy()


_loaded = {}  # a program keeps the models it has loaded


def _model(case):
    cfg, ends_early = _config(case), case["call"] == "eos"
    key = (tuple(sorted(cfg.items())), ends_early)
    if key not in _loaded:
        if len(_loaded) >= 3:
            _loaded.pop(next(iter(_loaded)))  # freed once no state holds it
        _loaded[key] = nt.Model(cfg, _weights(cfg, ends_early), max_batch_tokens=ARENA[case["model"]])
    return _loaded[key]


def prepare(case, seed):
    tokens, offsets = _sentences(case, seed)
    state = dict(case=case, model=_model(case), tokens=tokens, offsets=offsets)
    if case["call"] == "batch":
        lens = np.diff(offsets).astype(np.int32)
        rows, longest = len(lens), int(lens[0])
        ids = np.zeros((rows, longest), dtype=np.int32)
        ids[np.arange(longest)[None, :] < lens[:, None]] = tokens
        steps = np.array([nt.n_steps(int(n)) for n in lens], dtype=np.int32)
        state.update(steps=steps, ids=torch.from_numpy(ids).cuda(), lens=torch.from_numpy(lens).cuda(),
                     out=torch.empty((rows, int(steps[0])), dtype=torch.int32, device="cuda"))
    return state


def run(state):
    case, model = state["case"], state["model"]
    if case["call"] == "translate":
        return model.translate_batch(state["tokens"], state["offsets"], case["budget"], max_rows=case["max_rows"])
    if case["call"] == "eos":
        return model.translate_batch_eos(state["tokens"], state["offsets"], case["budget"], EOS, max_rows=case["max_rows"])
    rows, steps = state["out"].shape
    model.encode(state["ids"], state["lens"])
    model.decode_greedy(rows, steps, state["out"], row_steps=state["steps"])
    return state["out"]


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def work(case):
    """Bytes: weights and source ids in, target ids out.  Flops: the matrix products and attentions of every real token."""
    cfg = _config(case)
    d, V, F = cfg["d_model"], cfg["vocab"], cfg["d_ffn"]
    Fd = cfg["dec_d_ffn"] or F
    L = _lengths(case).double()
    T = torch.ceil(1.2 * L) + 2
    if case["call"] == "eos":
        T = 0.76 * T  # share of the capped steps that these weights emit
    enc = cfg["n_enc"] * (L * (8 * d * d + 4 * d * F) + 4 * d * L * L)
    dec = cfg["n_dec"] * (L * 4 * d * d + T * (12 * d * d + 4 * d * Fd) + 4 * d * (T * L + T * T / 2))
    matrix_bytes = 2 * nt.param_count(cfg) - (V * d if case["q8"] else 0)
    return {"bytes": float(matrix_bytes + 4 * L.sum() + 4 * T.sum()), "flops": float((enc + dec + 2 * V * d * T).sum())}


def tolerance(case):
    """Token ids.  A step's arg-max is decided by logit gaps that are often below 1e-3, and a sentence that takes the other
    side of one differs from there on: about one in a thousand, for sums in another order; more where the state is
    rounded to 8 bits before the output layer."""
    return {"rel": 0.0, "differ": 0.01 if case["q8"] else 0.005}
