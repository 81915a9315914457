"""What a program that decodes speech tokens with this framework asks of it, as cases to be timed.

A pass is one request (or one batch of requests) taken through the public binding from its prompt: `prefill`, a
number of speculative steps, the tokens back on the host, and the logits of the last step.  Every pass starts
from the prompt again, so a pass does not depend on the passes before it.  The number of steps is short of a
whole utterance (a pass would take a second); prompt lengths stand for the place in the utterance that the steps are taken at.

The models have the shapes of the framework's own workload presets and seeded weights.  Purely random weights
would give logits without a clear winner, so that a rounding decides which token comes next, and draft heads that are never
right.  Here the weights carry, besides their random part, what a trained model has: a next token that stands out,
and draft lists that are graded and right about as often as the method's authors report (some three tokens per step).
For that, a few dimensions of the residual stream hold the token's class: the embedding writes them and no layer does;
the vocabulary maps read them beside everything else.  All linear maps, attention and LayerNorms work on
full-width random values as before, and most of a logit row is what the layers computed.
"""
import numpy as np
import torch

from paper_2410_21951_amd import Vadusa, TreeArrays, build_tree
from paper_2410_21951_amd.vadusa import DBG

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
# layers, d, ffn, draft heads (of the model); vocab: speech tokens; positions: rows of the cache; dtype
FULL = dict(layers=12, d=1024, ffn=4096, heads=4, vocab=1024, positions=1280, dtype="bf16")
TINY = dict(layers=2, d=256, ffn=1024, heads=3, vocab=512, positions=512, dtype="fp32")
# batch; text and prompt tokens per sequence (drawn between lo and hi); nodes of the tree; tau; steps after the prompt;
# stream: every step's tokens are fetched as it ends (else all of them after the last step); chunk: rows of a
# sequence per prefill pass (0: the tree's size); sampled: the stochastic rule with temperature and top_p
CALL = dict(batch=1, text_lo=64, text_hi=64, prompt_lo=225, prompt_hi=225, nodes=64, tau=1, steps=16, stream=True, chunk=0,
            sampled=False, temperature=1.0, top_p=1.0)


def _case(name, model, **kw):
    return dict(dict(CALL, **model), **dict(kw, name=name))


def listed():
    return [
        # the smallest model in fp32, streamed token by token: latency and launches
        _case("tiny_fp32", TINY, text_lo=32, text_hi=32, prompt_lo=75, prompt_hi=75, nodes=16, steps=24),
        # plain auto-regressive decoding, one row per step: what speculative decoding is compared with
        _case("ar_b1", FULL, nodes=1, steps=24, chunk=512),
        # one listener, 64-node tree, each step's tokens go on to the vocoder at once: the ordinary call
        _case("stream_b1", FULL, steps=32, chunk=512),
        # the same by the stochastic rule (temperature and nucleus), tokens fetched at the end
        _case("sampled_b1", FULL, steps=16, tau=3, stream=False, chunk=512, sampled=True, temperature=0.9, top_p=0.9),
        # long-form speech late in the utterance: five draft heads, 128-node tree, some 2000 committed rows
        _case("longform_b1", dict(FULL, heads=5, positions=3328), prompt_lo=1964, prompt_hi=1964, nodes=128, steps=16,
              stream=False, chunk=1024),
        # large speech vocabulary (16 000 units)
        _case("vocab16k_b1", dict(FULL, vocab=16000), steps=16, chunk=512),
        # a few listeners at once with prompts of different lengths and a small odd tree
        _case("small_batch", FULL, batch=5, text_lo=20, text_hi=80, prompt_lo=75, prompt_hi=225, nodes=27, tau=2, steps=16),
        # 16 ragged sequences, 2048 units, tau 3
        _case("hubert_b16", dict(FULL, vocab=2048, positions=1024), batch=16, text_lo=20, text_hi=80, prompt_lo=100,
              prompt_hi=200, tau=3, steps=12, chunk=128),
        # offline synthesis of 64 sequences: throughput
        _case("throughput_b64", dict(FULL, positions=1200), batch=64, nodes=32, steps=10, stream=False),
        # time to the first tokens: a prompt and one step
        _case("first_tokens_b1", FULL, steps=1, chunk=512),
        # a long prompt (an earlier part of the text as context)
        _case("long_prompt_b1", dict(FULL, heads=5, positions=3328), prompt_lo=1500, prompt_hi=1500, nodes=128, steps=1, chunk=1024),
        # a ragged batch of prompts
        _case("prompts_b16", dict(FULL, vocab=2048, positions=1024), batch=16, text_lo=20, text_hi=80, prompt_lo=100,
              prompt_hi=200, steps=1, chunk=512),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """Ranges: batch 1 to 64, trees of 1 to 128 nodes, up to 2048 rows per step, prompts of 20 to 2000 tokens, models
    of 2 to 12 layers and d 256 to 1024 (fp32 only for the small ones), 200 to 16 000 units, 1 to 16 steps."""
    small = rng.random() < 0.15
    model = dict(TINY if small else FULL)
    if small:
        model.update(layers=rng.randint(1, 4), d=64 * rng.randint(2, 6), vocab=_log(rng, 200, 2048))
        model.update(ffn=4 * model["d"], positions=1024, heads=rng.randint(1, 4))
    else:
        if rng.random() < 0.3:
            model.update(layers=rng.randint(2, 12), d=64 * rng.randint(4, 16))
            model.update(ffn=64 * rng.randint(model["d"] // 32, model["d"] // 16))
        model.update(heads=rng.randint(3, 6), vocab=_log(rng, 500, 16000) if rng.random() < 0.3 else rng.choice((1024, 2048)), positions=3328)
    batch = _log(rng, 1, 64) if not small and rng.random() < 0.6 else rng.choice((1, 1, 2, 3))
    nodes = max(1, min(_log(rng, 1, 128) if rng.random() < 0.4 else rng.randint(16, 128), 2048 // batch, 64 if small else 128))
    longest = min(2000, 18000 // batch, 300 if small else 2000)
    hi = _log(rng, 40, longest)
    lo = hi if batch == 1 else max(20, hi // rng.randint(1, 3))
    steps = 1 if rng.random() < 0.25 else rng.randint(4, 16)
    sampled = rng.random() < 0.2 and batch * nodes * model["vocab"] < 1.2e6
    return dict(dict(CALL, **model), batch=batch, text_lo=16, text_hi=rng.randint(16, 80), prompt_lo=lo, prompt_hi=hi, nodes=nodes,
                tau=rng.choice((1, 1, 2, 3, 4)), steps=steps, stream=rng.random() < 0.6,
                chunk=0 if rng.random() < 0.4 else max(nodes, min(rng.choice((128, 256, 512, 1024)), 16384 // batch)),
                sampled=sampled, temperature=rng.choice((0.9, 1.0)) if sampled else 1.0, top_p=rng.choice((0.9, 0.95, 1.0)) if sampled else 1.0)


# ---------------------------------------------------------------------------
# model
# ---------------------------------------------------------------------------
TEXT_VOCAB = 512
CLASS_AMP = 16.0                    # the class dimension's value in the residual stream
NEXT = (11.0, 5.0, 4.5, 4.0)        # logits of the next token and of its alternatives, over a background of spread 1
RIGHT_AT = (0.62, 0.12, 0.06, 0.04)  # how often a draft head's list holds the token that comes at rank 0, 1, 2, 3


def _model(c):
    return dict(n_layers=c["layers"], d_model=c["d"], n_heads=c["d"] // 64, head_dim=64, d_ffn=c["ffn"], speech_vocab=c["vocab"],
                text_vocab=TEXT_VOCAB, n_draft_heads=c["heads"], max_positions=c["positions"], dtype=c["dtype"])


def _weights(c, seed):
    """The fp32 weight blob on the GPU, in the order of vadusa_load_weights."""
    d, F, V, V1, Hh, Ly = c["d"], c["ffn"], c["vocab"], c["vocab"] + 1, c["heads"], c["layers"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng([seed, 1])
    shapes = [(TEXT_VOCAB, d), (V1, d), (c["positions"], d)]
    for _ in range(Ly):
        shapes += [(d,), (d,), (3 * d, d), (3 * d,), (d, d), (d,), (d,), (d,), (F, d), (F,), (d, F), (d,)]
    shapes += [(d,), (d,), (V1, d)]
    for _ in range(Hh):
        shapes += [(d, d), (d,), (V1, d)]
    blob = torch.empty(sum(int(np.prod(s)) for s in shapes), device="cuda")
    blob.normal_(0.0, 0.02, generator=gen)
    views, at = [], 0
    for s in shapes:
        n = int(np.prod(s))
        views.append(blob[at:at + n].view(s))
        at += n
    C = max(8, d // 32)             # classes, one dimension each: dimensions 0 .. C - 1
    # what the class dimension is after the final LayerNorm (the layers' own contribution to the variance, roughly)
    h_c = CLASS_AMP * (d / (CLASS_AMP ** 2 + d * (0.3 + 0.26 * Ly * (d / 1024) * (F / 4096)))) ** 0.5
    E_text, E_speech, P = views[:3]
    for E, n in ((E_text, TEXT_VOCAB), (E_speech, V1)):
        E.mul_(25.0)                # token identity on the scale of the residual stream
        E[:, :C] = 0.0
        E[torch.arange(n, device="cuda"), torch.arange(n, device="cuda") % C] = CLASS_AMP
    P.mul_(12.0)
    P[:, :C] = 0.0
    for l in range(Ly):
        g1, b1, _, _, Wo, bo, g2, b2, _, _, W2, bf = views[3 + 12 * l:15 + 12 * l]
        for g in (g1, g2):
            g.add_(1.0)
        for m in (Wo, bo, W2, bf):
            m[:C] = 0.0             # no layer writes the class dimensions
    at = 3 + 12 * Ly
    views[at].fill_(1.0)
    views[at + 1].zero_()
    W_out = views[at + 2]
    W_out.mul_(50.0 / d ** 0.5)
    W_out[:, :C] = 0.0
    # class k is followed by a token of class k + 1
    follow = (np.arange(1, C + 1) % C + C * rng.integers(0, V // C - 1, C)).astype(np.int64)
    table = torch.zeros(V1, C)
    for k in range(C):
        others = rng.permutation(V)[:len(NEXT)]
        for j, value in enumerate(NEXT):
            table[follow[k] if j == 0 else int(others[j]), k] = value / h_c
        table[follow[k], k] = NEXT[0] / h_c
    W_out[:, :C] = table.cuda()
    for i in range(Hh):
        D1, db, D2 = views[at + 3 + 3 * i:at + 6 + 3 * i]
        D1[:C] = 0.0
        db[:C] = 0.0
        D2.mul_(5.0 / d ** 0.5)
        table = torch.zeros(V1, C)
        for k in range(C):
            true = int(follow[(k + 1 + i) % C])
            ids = [int(t) for t in rng.permutation(V)[:18] if t != true][:16]
            u, r = rng.random(), 0
            while r < len(RIGHT_AT) and u >= RIGHT_AT[r]:
                u -= RIGHT_AT[r]
                r += 1
            if r < len(RIGHT_AT):
                ids[r] = true
            for r, t in enumerate(ids):
                table[t, k] = (16 - r) / h_c
        D2[:, :C] = table.cuda()
    return blob


def prepare(case, seed):
    c = case
    rng = np.random.default_rng([seed, 2])
    dev = Vadusa(_model(c), max_batch=c["batch"], max_tree_nodes=c["nodes"], prefill_chunk=c["chunk"])
    dev.load_blob_device(_weights(c, seed))
    text = [rng.integers(0, TEXT_VOCAB, int(rng.integers(c["text_lo"], c["text_hi"] + 1))).astype(np.int32) for _ in range(c["batch"])]
    prompt = [rng.integers(0, c["vocab"], int(rng.integers(c["prompt_lo"], c["prompt_hi"] + 1))).astype(np.int32) for _ in range(c["batch"])]
    if c["nodes"] == 1:
        tree = TreeArrays([-1], [0])
    else:   # the acceptance probabilities of the presets' trees: ranks fall off by 0.6, depths by 0.85
        fall = 0.6 ** np.arange(10)
        acc = 0.75 * 0.85 ** np.arange(c["heads"])[:, None] * (fall / fall.sum())[None]
        tree = build_tree(acc, c["nodes"])
    uniforms = None
    if c["sampled"]:
        gen = torch.Generator(device="cuda").manual_seed(seed + 1)
        n = c["batch"] * tree.n_nodes * (c["vocab"] + 1)
        uniforms = [torch.rand(n, device="cuda", generator=gen).clamp_(2.0 ** -24, 1.0 - 2.0 ** -24) for _ in range(c["steps"])]
    return dict(case=c, dev=dev, text=text, prompt=prompt, tree=tree, uniforms=uniforms)


def run(state):
    c, dev, tree = state["case"], state["dev"], state["tree"]
    roots = dev.prefill(state["text"], state["prompt"])
    tokens = [[] for _ in range(c["batch"])]
    for i in range(c["steps"]):
        sample = (c["temperature"], c["top_p"], state["uniforms"][i]) if c["sampled"] else None
        accepted = dev.step(tree, c["tau"], sync=c["stream"], sample=sample)
        if c["stream"]:
            for mine, new in zip(tokens, accepted):
                mine.extend(new)
    if not c["stream"]:
        tokens = [dev.read_output(b) for b in range(c["batch"])]
    out = np.full((c["batch"], c["steps"] * (c["heads"] + 1)), -1, np.int32)
    for row, mine in zip(out, tokens):
        row[:len(mine)] = mine
    return {"roots": roots, "tokens": out, "logits": dev.debug(DBG.LOGITS)}


def work(case):
    """Weights once per prefill pass that the prompt needs (one, when the caller's chunk holds it) and once per step; the
    committed cache rows once per step, the tree's rows written once; the logits once.  About three tokens a step."""
    c = case
    s = 2 if c["dtype"] == "bf16" else 4
    d, F, Ly, V1, Hh, B, M = c["d"], c["ffn"], c["layers"], c["vocab"] + 1, c["heads"], c["batch"], c["nodes"]
    layers = Ly * (4 * d * d + 2 * d * F)
    heads = Hh * (d * d + V1 * d)
    row = Ly * 2 * d                                    # K and V values of one position
    n = (c["text_lo"] + c["text_hi"] + c["prompt_lo"] + c["prompt_hi"]) / 2.0
    chunk = c["chunk"] or M
    passes = -(-int(n) // chunk)
    gain = 1.0 if M == 1 else min(3.0, Hh + 1)
    by = (passes * layers + V1 * d + heads + B * n * row) * s
    fl = 2.0 * B * n * layers + 2.0 * B * (V1 * d + heads) + 2.0 * B * n * n * d * Ly
    for i in range(c["steps"]):
        L = n + gain * i
        by += (layers + V1 * d + heads + B * (L + M) * row) * s
        fl += 2.0 * B * M * (layers + V1 * d) + 2.0 * B * heads + 4.0 * B * M * (L + M / 2.0) * d * Ly
    by += B * M * V1 * 4
    if c["sampled"]:
        by += c["steps"] * B * M * V1 * 4
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    """Tokens are the same (the margins are wide).  Logits: in bf16, two ways through the same prompt (passes of another
    length, hence other kernels and other orders of summation) differ by 3.4e-3 to 3.8e-3 and at most by 0.023 of the
    row's spread; against 64-bit arithmetic on the same weights they are off by 5e-3.  In fp32 they are off by 1e-7
    (models of more layers and wider ones: more)."""
    return {"rel": 1.4e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 5e-6, "max": 5e-5}
