"""The kernels of the decoder layers at the sizes where they can go wrong: remainders of row and column tiles, reductions
whose stages leave a remainder, the change from one tile shape to the next, an odd number of query tiles, and
the row statistics of the fp32 maps on both sides of what they keep in registers.  Against the CPU oracle, with the
tolerances of tests/parity.py (logits relative L2: 1e-4 in fp32, 1e-2 in bf16)."""
import numpy as np
import pytest

from synth import ModelConfig, make_weights, make_tree
from test_gpu_parity import rand_tokens

pytestmark = pytest.mark.gpu

# Weight scale.  The harness takes a decision for an error when its margin exceeds 1e-2, an absolute logit gap stated for a
# logit spread of 0.57 to 0.64 (weight std x sqrt(d)).  bf16 logits are off by some 5e-3 of their spread, so the gap of two by
# 7e-3: a spread of 0.9 (std 0.05 at d = 320) has gaps of 1.5e-2 decided either way.  The scale keeps the spread at 0.57.
def _std(cfg):
    return 0.08 if cfg.dtype == "fp32" else 0.57 / cfg.d_model ** 0.5


def _run(cfg, batch, nodes, caps, taus, seed, prompt_lo, prompt_hi, compared=1):
    from parity import Lockstep
    W = make_weights(cfg, seed, std=_std(cfg), ln_jitter=0.1)
    rng = np.random.default_rng(seed)
    text, prompt = rand_tokens(cfg, rng, batch, (2, 6), (prompt_lo, prompt_hi))
    ls = Lockstep(cfg, W, text, prompt, nodes)
    tree = make_tree(nodes, caps)
    for tau in taus:
        ls.step(tree, tau)
    ls.check_kv(layers=[0, cfg.n_layers - 1])
    s = ls.stats
    print(f"d {cfg.d_model} rows {batch * nodes}: compared {s.compared}/{s.steps} logit err {s.max_logit_err:.2e}", flush=True)
    assert s.compared >= compared


def _cfg(dtype, d, V, layers=2, heads=2, ffn=None, maxpos=192):
    return ModelConfig(n_layers=layers, d_model=d, n_heads=d // 64, head_dim=64, d_ffn=ffn or 3 * d, speech_vocab=V, text_vocab=40,
                       n_draft_heads=heads, max_positions=maxpos, dtype=dtype)


# d: one, three, five and eight stages of 64; rows just below, at and above a 64-row tile; V + 1 logits: ragged column tiles
@pytest.mark.parametrize("d,nodes,batch,V", [(64, 63, 1, 127), (192, 32, 2, 128), (320, 65, 1, 257), (512, 43, 3, 300)])
def test_many_row_tiles_at_their_edges(monkeypatch, d, nodes, batch, V):
    monkeypatch.setenv("VADUSA_BIG_MIN_UNITS", "1")
    _run(_cfg("bf16", d, V), batch, nodes, (9, 9), (2, 1), 300 + d, 20, 70)


# Both shapes of k_tile (256 x 128 and 128 x 64 outputs) for every map: fewer stages than the ring has and more, an odd number of them,
# a last stage that is half empty (K = 64, 192, 320), rows and columns that end inside a tile or leave whole blocks of it
# empty, row statistics of 16, 32 and 64 columns, values whose rows share a piece of the cache with those of no, one or two passes
@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("d,nodes,batch,V", [(64, 65, 1, 127), (192, 43, 3, 300), (320, 126, 2, 257), (512, 64, 5, 128), (128, 5, 61, 90)])
def test_many_row_tile_shapes(monkeypatch, shape, d, nodes, batch, V):
    monkeypatch.setenv("VADUSA_BIG_MIN_UNITS", str(-shape))
    _run(_cfg("bf16", d, V), batch, nodes, (4, 3) if nodes == 5 else (11, 11), (2, 1), 800 + d, 20, 70)


# By the rule one model mixes the kernels, and with them statistics of 16 and of 32 columns (tests/test_emulated_kernel.py holds the
# rule to this: QKV, out-projection, FFN1, FFN2)
MIXED = [(256, 4096, 100, 4, "lin lin big lin"), (256, 4096, 127, 5, "big lin big lin"), (128, 16384, 127, 4, "lin lin tile256 lin"),
         (128, 1024, 77, 27, "tile128 big big tile128")]


@pytest.mark.parametrize("d,ffn,nodes,batch,kernels", MIXED)
def test_kernels_mixed_by_the_rule(d, ffn, nodes, batch, kernels):
    _run(_cfg("bf16", d, 90, layers=1, ffn=ffn, maxpos=192), batch, nodes, (11, 11), (2, 1), 830 + batch, 4, 40)


# rows below, at and above whole tiles; at this width all maps run in tiles of one or two by one or two
@pytest.mark.parametrize("rows", [1, 16, 17, 33, 64, 97, 128, 193])
def test_small_tile_shapes(rows):
    batch = 1 if rows <= 100 else 2 if rows % 2 == 0 else 1
    nodes = rows // batch if rows // batch <= 128 else 0
    if not nodes:
        batch, nodes = 2, 97    # 194 rows
    caps = () if nodes == 1 else (10, 10, 10)
    _run(_cfg("bf16", 256, 301, heads=3, maxpos=224), batch, nodes, caps, (1, 2), 400 + rows, 30, 80)


# Every tile shape of k_lin with a ragged last row tile (and, in the vocabulary map, a ragged last column tile and a column
# count that the shape does not divide): d, ffn, nodes, batch, V, and the shapes (row tiles x column tiles) that the rule picks
# for QKV, out-projection and FFN2, FFN1, vocabulary map.  tests/test_emulated_kernel.py holds the rule to this table.
TILE_SHAPES = [
    (64, 4096, 17, 1, 1349, "1x1 1x1 1x2 1x1"),
    (64, 4096, 33, 1, 2060, "1x1 1x1 2x2 1x2"),
    (64, 4096, 65, 1, 4110, "1x1 1x1 2x4 2x4"),
    (64, 4096, 43, 3, 1610, "1x1 1x1 3x4 2x2"),
    (64, 4096, 97, 2, 300, "1x1 1x1 4x4 1x1"),
    (64, 256, 85, 1, 1349, "1x1 1x1 1x1 2x1"),
    (64, 256, 17, 17, 1610, "1x1 1x1 1x2 4x2"),
    (64, 64, 33, 1, 8205, "1x1 1x1 1x1 3x4"),
    (64, 64, 49, 1, 8300, "1x1 1x1 1x1 4x4"),
    (64, 128, 26, 13, 77, "1x2 1x1 1x1 1x1"),
    (64, 128, 27, 25, 300, "2x2 1x1 1x2 2x2"),
    (128, 128, 27, 25, 77, "2x4 1x2 1x2 1x1"),
    (192, 192, 23, 39, 77, "3x4 2x2 2x2 1x2"),
    (512, 512, 27, 19, 77, "4x4 2x4 2x4 1x1"),
    (512, 512, 41, 25, 77, "4x4 3x4 3x4 1x2"),
    (512, 512, 53, 29, 77, "4x4 4x4 4x4 2x1"),
    (512, 2048, 27, 5, 77, "2x2 1x2 2x4 1x1"),     # a reduction of 2048: eight waves in FFN2
    (512, 2048, 41, 7, 77, "2x4 2x2 3x4 1x1"),
    (512, 2048, 53, 12, 77, "4x4 2x4 3x4 1x1"),
]


@pytest.mark.parametrize("d,ffn,nodes,batch,V,shapes", TILE_SHAPES)
def test_every_small_tile_shape(monkeypatch, d, ffn, nodes, batch, V, shapes):
    monkeypatch.setenv("VADUSA_BIG_MIN_UNITS", "1000000")   # k_big never
    _run(_cfg("bf16", d, V, layers=1, ffn=ffn, maxpos=160), batch, nodes, (16, 16), (2,), 700 + d + nodes, 4, 20)


def test_two_query_tiles_per_workgroup_with_an_odd_number_of_tiles():
    # by the rule: 32 sequences x 8 heads x two workgroups.  40 nodes: three tiles of 16 queries, the last one ragged
    _run(_cfg("bf16", 512, 90, layers=1, ffn=256, maxpos=128), 32, 40, (7, 7), (2,), 511, 10, 60)


# Prompt passes have the rows of the tokens they hold: sequences without rows in the first passes, of one token, that end at and beside
# a tile of 16; a pass whose sequences have a row each; behind the last layer's attention only the sequences' last rows (a
# hidden layer of 64 leaves no room for that with fewer than 16 rows per sequence); one sequence alone; every kernel of the maps
@pytest.mark.parametrize("big_min", [0, 1, -1, -2])
@pytest.mark.parametrize("lens,chunk,d,ffn", [((1, 17, 70), 16, 128, 256), ((33, 1, 1, 2, 16), 0, 192, 64), ((5, 9, 3), 0, 512, 64), ((97,), 32, 64, 128),
                                              ((1, 1), 64, 128, 128), ((129, 64, 100, 31), 64, 256, 512)])
def test_ragged_prompt_passes(monkeypatch, big_min, lens, chunk, d, ffn):
    from parity import Lockstep
    monkeypatch.setenv("VADUSA_BIG_MIN_UNITS", str(big_min))
    cfg = _cfg("bf16", d, 90, ffn=ffn, maxpos=192)
    W = make_weights(cfg, 940 + d, std=_std(cfg), ln_jitter=0.1)
    rng = np.random.default_rng(940 + len(lens))
    text = [rng.integers(0, cfg.text_vocab, n // 3).astype(np.int32) for n in lens]
    tokens = [rng.integers(0, cfg.speech_vocab, n - n // 3).astype(np.int32) for n in lens]
    ls = Lockstep(cfg, W, text, tokens, 16, prefill_chunk=chunk)
    ls.check_kv(layers=[0, 1])    # beside the draft lists' logits and the first root, which the harness compares
    tree = make_tree(16, (4, 4))
    for tau in (2, 1):
        ls.step(tree, tau)
    print(f"{lens}: compared {ls.stats.compared}/{ls.stats.steps} logit err {ls.stats.max_logit_err:.2e} kv {ls.stats.max_kv_err:.2e}", flush=True)
    assert ls.stats.compared >= 1


# Attention: one query tile with four and with eight waves, two with four; 9 to 34 blocks of keys, so that some waves take one more than
# others and the last block is ragged; prompts in one pass and in passes of the tree's rows; the keys' bound moves with the steps.  The
# last column: query tiles x waves of the prompt's passes, then of the steps (tests/test_emulated_kernel.py holds the rule to it); big_min 1:
# two tiles wherever there are two.
ATTENTION = [
    (128, 1, 40, 520, 0, 0, "1x4 1x8, 1x8"),
    (64, 2, 17, 590, 0, 0, "1x4 1x8, 1x8"),
    (128, 3, 33, 300, 0, 0, "1x4 1x8, 1x8"),
    (512, 32, 40, 240, 0, 0, "2x4, 2x4"),
    (64, 1, 1, 511, 0, 0, "1x4 1x8, 1x8"),
    (128, 2, 24, 560, 576, 0, "1x8, 1x8"),
    (128, 1, 33, 1010, 1024, 0, "1x8, 1x8"),
    (128, 1, 33, 1010, 1024, 1, "2x4, 2x4"),
    (64, 3, 16, 250, 0, 0, "1x4 1x8, 1x4"),
]


@pytest.mark.parametrize("d,batch,nodes,prompt,chunk,big_min,shapes", ATTENTION)
def test_attention_waves(monkeypatch, d, batch, nodes, prompt, chunk, big_min, shapes):
    from parity import Lockstep
    monkeypatch.setenv("VADUSA_BIG_MIN_UNITS", str(big_min))
    cfg = _cfg("bf16", d, 90, layers=1, ffn=128, maxpos=1104 if prompt > 700 else 704)
    W = make_weights(cfg, 900 + d, std=_std(cfg), ln_jitter=0.1)
    rng = np.random.default_rng(900 + prompt)
    text, tokens = rand_tokens(cfg, rng, batch, (2, 6), (prompt, prompt + 9))
    ls = Lockstep(cfg, W, text, tokens, nodes, prefill_chunk=chunk)
    tree = make_tree(nodes, () if nodes == 1 else (7, 7))
    for tau in (2, 1):
        ls.step(tree, tau)
    ls.check_kv(layers=[0])
    print(f"keys {prompt}: compared {ls.stats.compared}/{ls.stats.steps} logit err {ls.stats.max_logit_err:.2e}", flush=True)
    assert ls.stats.compared >= 1


@pytest.mark.parametrize("nodes,caps", [(40, (7, 7)), (17, (5, 4))])
def test_two_query_tiles_beside_a_finished_sequence(monkeypatch, nodes, caps):
    """Forced on for three sequences: an odd number of query tiles (three), or two with one query in the second; the
    prompt's passes likewise; after the first step sequence 0 has ended with EOS and has no rows."""
    from parity import Lockstep
    from oracle import vadusa_oracle as O
    monkeypatch.setenv("VADUSA_BIG_MIN_UNITS", "1")
    cfg = _cfg("bf16", 128, 90)
    W = make_weights(cfg, 521, std=_std(cfg), ln_jitter=0.1)
    W["W_out"] = W["W_out"].copy()
    W["W_out"][cfg.speech_vocab] = 0    # EOS (logit 0, the largest of the other 90 is near 2.4 standard deviations) comes from the plan alone
    rng = np.random.default_rng(521)
    text, prompt = rand_tokens(cfg, rng, 3, (2, 6), (30, 60))
    ls = Lockstep(cfg, W, text, prompt, nodes, ignore_eos=False)
    tree = make_tree(nodes, caps)
    need = O.topk_needed(tree.depth, tree.rank, cfg.n_draft_heads)
    lists = [[rng.permutation(cfg.speech_vocab)[:k] for k in need] for _ in range(3)]
    lists[0][0][0] = cfg.speech_vocab
    for _ in range(2):    # every edge passes (tau above the vocabulary): the paths are the planted ones
        r = ls.step(tree, cfg.n_logits, override=lists)
        assert ls.sts[0].finished and not ls.sts[1].finished and not ls.sts[2].finished
    assert [len(x["accepted"]) for x in r] == [0, 3, 3]
    ls.check_kv(layers=[0, 1])
    print(f"{nodes} nodes: compared {ls.stats.compared}/{ls.stats.steps} logit err {ls.stats.max_logit_err:.2e}", flush=True)
    assert ls.stats.compared == 2


# 384 values of a row stay in registers, more are read again; 15 and 17 rows: one row tile, two
@pytest.mark.parametrize("d,nodes,V", [(64, 15, 70), (384, 17, 200), (448, 33, 129)])
def test_fp32_maps_at_their_edges(d, nodes, V):
    _run(_cfg("fp32", d, V), 2, nodes, (6, 6), (1, 3), 600 + d, 20, 60)


# The lists, the edges and the roots of long rows, from the kernels' own logits: whole numbers, so the same.  V + 1 logits: the first row
# beyond 4096; one slice of 16 384 full, and one entry in the next; four slices full, and beyond them (one entry per round);
# odd ones between.  equal: all logits the same, more candidates than the list of them holds.
@pytest.mark.parametrize("V,equal", [(4096, False), (8702, False), (16383, False), (16384, False), (40001, False), (65535, False), (65536, False), (5000, True), (20000, True)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_long_rows_are_ranked_as_by_sorting(V, equal, dtype):
    from paper_2410_21951_amd import TreeArrays, Vadusa
    from paper_2410_21951_amd.vadusa import DBG
    cfg = _cfg(dtype, 64, V, layers=1, ffn=64, maxpos=96)
    W = make_weights(cfg, 77, std=_std(cfg), ln_jitter=0.1)
    if equal:
        for name in ("W_out", "D0.W2", "D1.W2"):
            W[name] = np.zeros_like(W[name])
    rng = np.random.default_rng(V)
    text, prompt = rand_tokens(cfg, rng, 2, (2, 6), (20, 30))
    tree = make_tree(23, (8, 8))
    dev = Vadusa(cfg, max_batch=2, max_tree_nodes=23)
    dev.load_weights(W)
    dev.prefill(text, prompt)

    def lists_are_sorted():
        z, got = dev.debug(DBG.DRAFT_LOGITS), dev.debug(DBG.DRAFT_TOPK)
        for b in range(2):
            for i in range(2):
                want = np.argsort(-z[b, i], kind="stable")[:got.shape[2]]
                assert np.array_equal(got[b, i], want), (V, b, i)

    lists_are_sorted()
    for tau in (1, V // 8, V // 3):
        print(f"{V + 1} logits, {dtype}, tau {tau}", flush=True)
        accepted = dev.step(TreeArrays(tree.parent, tree.rank), tau)
        z, tok, ok, root = dev.debug(DBG.LOGITS), dev.debug(DBG.TREE_TOK), dev.debug(DBG.EDGE_OK), dev.debug(DBG.ROOT)
        for b in range(2):
            for n in range(1, 23):
                row, t = z[b, tree.parent[n]], tok[b, n]
                ahead = int((row > row[t]).sum() + (row[:t] == row[t]).sum())
                assert ok[b, n] == (ahead < tau), (V, tau, b, n)
            good = [True]
            for n in range(1, 23):
                good.append(bool(ok[b, n]) and good[tree.parent[n]])
            last = max((n for n in range(23) if good[n]), key=lambda n: (tree.depth[n], -n))
            assert len(accepted[b]) == tree.depth[last] + 1
            assert root[b] == int(np.argmax(z[b, last])), (V, tau, b)
        lists_are_sorted()
    dev.close()


# Scores of the stochastic rule against 64 bits from the kernel's own logits, around the sizes where its kernels change (4096 and 8192
# logits) and end (16 384).  A token may be kept or not where the mass above it is within 1e-5 of top_p: sums of 16 384 masses in
# trees of some 30 additions (2e-6) of exponentials good to 1e-6.  Scores: two logarithms and a quotient, a few 2^-24 of each.
@pytest.mark.parametrize("V1", [4096, 4097, 6000, 8192, 8193, 16001, 16384])
def test_scores_of_long_rows(V1):
    from paper_2410_21951_amd import TreeArrays, Vadusa
    from paper_2410_21951_amd.vadusa import DBG
    from synth import make_uniforms
    cfg = _cfg("bf16", 64, V1 - 1, layers=1, ffn=64, maxpos=96)
    W = make_weights(cfg, 78, std=_std(cfg), ln_jitter=0.1)
    W["W_out"] = W["W_out"].copy() * 4     # logits of spread 2.3
    W["W_out"][V1 - 9:] = W["W_out"][7]    # nine equal logits
    rng = np.random.default_rng(V1)
    text, prompt = rand_tokens(cfg, rng, 2, (2, 6), (20, 30))
    tree = make_tree(13, (6, 6))
    dev = Vadusa(cfg, max_batch=2, max_tree_nodes=13)
    dev.load_weights(W)
    dev.prefill(text, prompt)
    for i, (tau, T, top_p) in enumerate([(1, 0.9, 0.9), (3, 1.0, 0.5), (40, 0.5, 1e-4), (1, 1.0, 1.0), (V1, 1.0, 0.3), (2, 0.7, 0.999)]):
        print(f"{V1} logits, tau {tau}, temperature {T}, top_p {top_p}", flush=True)
        u = make_uniforms(91, i, 2, 13, V1)
        dev.step(TreeArrays(tree.parent, tree.rank), tau, sample=(T, top_p, u))
        z, got = dev.debug(DBG.LOGITS).reshape(26, V1), dev.debug(DBG.SCORES).reshape(26, V1)
        for row, y, ur in zip(z, got, np.asarray(u, np.float64).reshape(26, V1)):
            s32 = row / np.float32(T)
            s = s32.astype(np.float64)
            of = np.unique(-s32, return_inverse=True)[1]     # rank of the value, largest first
            count = np.bincount(of)
            mass = np.bincount(of, np.exp(s - s.max()))
            above, ahead = (np.cumsum(mass) - mass)[of] / mass.sum(), (np.cumsum(count) - count)[of]
            kept = np.isfinite(y)
            sure = (np.abs(above - top_p) > 1e-5) | (ahead < tau) | (top_p >= 1)
            want = (above < top_p) | (ahead < tau) | (top_p >= 1)
            assert np.array_equal(kept[sure], want[sure]), (V1, tau, top_p)
            score = s - np.log(-np.log(ur))
            assert np.allclose(y[kept], score[kept], rtol=1e-6, atol=1e-5)
    dev.close()
