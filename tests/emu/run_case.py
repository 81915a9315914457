"""Child process of tests/test_emulated_kernel.py: one lockstep run of the emulated kernels
against the oracle.  usage: run_case.py <libvadusa_emu.so> <case of tests/test_emulated_kernel.py>"""
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)
sys.path.insert(0, os.path.dirname(HERE))
import emulate
# nanfill: the arena arrives holding NaN bits (0xFFFF is a NaN in bf16, 0xFFFFFFFF in fp32)
emulate.install(sys.argv[1], fill=0xFF if sys.argv[2].endswith("-nanfill") else 0xAB)
import numpy as np
from synth import ModelConfig, make_weights, make_tree, make_uniforms
from parity import Lockstep

dtype = sys.argv[2]
if dtype == "bf16-40rows":
    # 40 rows: three row tiles and three query tiles, the last of each ragged, masks of two words; two layers.
    cfg = ModelConfig(n_layers=2, d_model=64, n_heads=1, head_dim=64, d_ffn=192, speech_vocab=71, text_vocab=20,
                      n_draft_heads=2, max_positions=192, dtype="bf16")
    W = make_weights(cfg, 71, std=0.05)
    rng = np.random.default_rng(72)
    text = [rng.integers(0, cfg.text_vocab, 2).astype(np.int32)]
    prompt = [rng.integers(0, cfg.speech_vocab, 45).astype(np.int32)]
    tree = make_tree(40, (10, 10))
    t0 = time.time()
    ls = Lockstep(cfg, W, text, prompt, 40)
    ls.step(tree, 2)
    ls.step(tree, 1)
    ls.check_kv(layers=[0, 1])
    s = ls.stats
    print(f"emulated {dtype}: compared {s.compared}/{s.steps} logit err {s.max_logit_err:.2e} "
          f"ties {s.tie_root}/{s.tie_list}/{s.tie_edge} in {time.time() - t0:.0f} s", flush=True)
    assert s.compared >= 1
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-72rows":
    # 72 rows: five row tiles, the last ragged, masks of three words.  The prompt's 70 tokens are one causal pass of 70 rows.
    cfg = ModelConfig(n_layers=2, d_model=64, n_heads=1, head_dim=64, d_ffn=192, speech_vocab=71, text_vocab=20,
                      n_draft_heads=3, max_positions=224, dtype="bf16")
    W = make_weights(cfg, 81, std=0.05)
    rng = np.random.default_rng(82)
    text = [rng.integers(0, cfg.text_vocab, 3).astype(np.int32)]
    prompt = [rng.integers(0, cfg.speech_vocab, 67).astype(np.int32)]
    tree = make_tree(72, (10, 10, 10))
    t0 = time.time()
    ls = Lockstep(cfg, W, text, prompt, 72)
    ls.step(tree, 2)
    ls.check_kv(layers=[0, 1])
    s = ls.stats
    print(f"emulated {dtype}: compared {s.compared}/{s.steps} logit err {s.max_logit_err:.2e} "
          f"ties {s.tie_root}/{s.tie_list}/{s.tie_edge} in {time.time() - t0:.0f} s", flush=True)
    assert s.compared >= 1
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-256rows":
    # 256 rows (8 sequences x 32 nodes) with the many-row kernels forced on for these small maps: 64 x 128 tiles (192 and
    # 72 columns: the last column group partial), attention with two query tiles per workgroup, tree and causal.
    os.environ["VADUSA_BIG_MIN_UNITS"] = "1"
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=192, speech_vocab=71, text_vocab=20,
                      n_draft_heads=2, max_positions=64, dtype="bf16")
    W = make_weights(cfg, 91, std=0.05)
    rng = np.random.default_rng(92)
    text = [rng.integers(0, cfg.text_vocab, int(rng.integers(1, 4))).astype(np.int32) for _ in range(8)]
    prompt = [rng.integers(0, cfg.speech_vocab, int(rng.integers(3, 12))).astype(np.int32) for _ in range(8)]
    tree = make_tree(32, (6, 6))
    t0 = time.time()
    ls = Lockstep(cfg, W, text, prompt, 32)
    ls.step(tree, 2)
    ls.check_kv(layers=[0])
    s = ls.stats
    print(f"emulated {dtype}: compared {s.compared}/{s.steps} logit err {s.max_logit_err:.2e} "
          f"ties {s.tie_root}/{s.tie_list}/{s.tie_edge} in {time.time() - t0:.0f} s", flush=True)
    assert s.compared >= 1
    sys.stdout.flush()
    os._exit(0)
if dtype in ("bf16-tile256", "bf16-tile128", "bf16-long-ffn", "bf16-long-keys"):
    # tile256, tile128: every map by k_tile of 256 x 128 or 128 x 64 outputs (81 rows, 192 and 72 columns: blocks of a tile that are empty, a
    # last stage that is half empty); long-ffn: a reduction of 2048 by eight waves; long-keys: 318 keys and more, eight waves per query tile.
    long_ffn, long_keys = dtype == "bf16-long-ffn", dtype == "bf16-long-keys"
    os.environ["VADUSA_BIG_MIN_UNITS"] = {"bf16-tile256": "-1", "bf16-tile128": "-2"}.get(dtype, "0")
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=2048 if long_ffn else 64 if long_keys else 192,
                      speech_vocab=71, text_vocab=20, n_draft_heads=2, max_positions=392 if long_keys else 96, dtype="bf16")
    W = make_weights(cfg, 95, std=0.05)
    rng = np.random.default_rng(96)
    B, M = (1, 17) if long_ffn or long_keys else (3, 27)
    text = [rng.integers(0, cfg.text_vocab, 2 + b).astype(np.int32) for b in range(B)]
    prompt = [rng.integers(0, cfg.speech_vocab, 315 if long_keys else 20 - 7 * b).astype(np.int32) for b in range(B)]
    t0 = time.time()
    ls = Lockstep(cfg, W, text, prompt, M, prefill_chunk=160 if long_keys else 0)
    ls.step(make_tree(M, (6, 6)), 2)
    ls.check_kv(layers=[0, cfg.n_layers - 1])
    s = ls.stats
    print(f"emulated {dtype}: compared {s.compared}/{s.steps} logit err {s.max_logit_err:.2e} in {time.time() - t0:.0f} s", flush=True)
    assert s.compared >= 1
    sys.stdout.flush()
    os._exit(0)
if dtype == "long-rows":
    # The kernels of rows of more than 4096 logits alone, their rows up against the guard page: draft lists, edges and perturbed scores against sorting,
    # counting and 64-bit sums.  Sizes where they change: one slice of 16 384 and the next entry, four slices and the next entry (one list entry per
    # round, as with more than 256 equal candidates), 8192 and 16 384 values of a row in registers.  Rows of NaN stay inside the row.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    lib, f32, i32 = V._lib, np.float32, np.int32

    def guarded(a):
        p = lib.emu_alloc(a.nbytes, 0xAB)
        v = np.frombuffer((C.c_char * a.nbytes).from_address(p), a.dtype).reshape(a.shape)
        v[...] = a
        return v
    ptr = lambda a: C.c_void_p(a.ctypes.data)
    rng = np.random.default_rng(97)
    for V1, kind in ((4097, ""), (16384, ""), (16385, ""), (40001, ""), (65536, ""), (65537, ""), (5001, "equal"), (4999, "nan"), (6001, "some nan"), (4098, "-inf")):
        z = rng.standard_normal((2, V1)).astype(f32)
        z[:, V1 - 5:] = z[:, :5]                                   # equal values at both ends
        if kind == "equal": z[:] = 1.5
        if kind == "nan": z[:] = np.nan
        if kind == "some nan": z[:, ::7] = np.nan
        if kind == "-inf": z[:, 10:] = -np.inf
        lists = guarded(np.full((2, 16), -1, i32))
        lib.emu_topk(ptr(guarded(z)), V1, 2, ptr(lists))
        print(f"lists of {V1} logits {kind}", flush=True)
        assert ((lists >= 0) & (lists < V1)).all()
        if "nan" not in kind:
            for row, got in zip(z, lists):
                assert np.array_equal(got, np.argsort(-row, kind="stable")[:16]), (V1, kind)
    for V1 in (4097, 16001):
        B, M = 2, 4
        parent, finished = guarded(np.array([-1, 0, 0, 1], i32)), guarded(np.array([0, 1], i32))
        z, tok = rng.standard_normal((B, M, V1)).astype(f32), rng.integers(0, V1, (B, M)).astype(i32)
        tok[0, 1] = V1 - 1
        z[0, 0, 5:50] = z[0, 0, tok[0, 1]]
        for tau in (1, V1 // 3, V1):
            ok = guarded(np.full((B, M), -1, i32))
            lib.emu_edges(ptr(guarded(z)), B, M, V1, ptr(parent), ptr(guarded(tok)), ptr(finished), tau, ptr(ok))
            print(f"edges of {V1} logits, tau {tau}", flush=True)
            for n in range(M):
                row, t = z[0, max(parent[n], 0)], tok[0, n]
                ahead = int((row > row[t]).sum() + (row[:t] == row[t]).sum())
                assert ok[0, n] == (n == 0 or ahead < tau), (V1, tau, n)
            assert not ok[1].any()
    for V1, tau, T, top_p in ((4097, 1, 0.9, 0.9), (8192, 3, 1.0, 0.5), (8193, 40, 0.5, 1e-4), (16384, 2, 0.7, 0.999), (4100, 1, 1.0, 1.0)):
        z, u = (2.3 * rng.standard_normal((1, V1))).astype(f32), np.clip(rng.random((1, V1)), 2.0 ** -24, 1 - 2.0 ** -24).astype(f32)
        z[0, V1 - 9:] = z[0, 7]
        y = guarded(np.zeros((1, V1), f32))
        lib.emu_perturb(ptr(guarded(z)), ptr(guarded(u)), ptr(y), 1, V1, C.c_float(T), C.c_float(top_p), tau)
        print(f"scores of {V1} logits", flush=True)
        s = (z[0] / f32(T)).astype(np.float64)
        of = np.unique(-s, return_inverse=True)[1]
        count, mass = np.bincount(of), np.bincount(of, np.exp(s - s.max()))
        above, ahead = (np.cumsum(mass) - mass)[of] / mass.sum(), (np.cumsum(count) - count)[of]
        kept = np.isfinite(y[0])
        sure = (np.abs(above - top_p) > 1e-5) | (ahead < tau) | (top_p >= 1)     # (fp32 sums of the masses)
        assert np.array_equal(kept[sure], ((above < top_p) | (ahead < tau) | (top_p >= 1))[sure]), V1
        assert np.allclose(y[0][kept], (s - np.log(-np.log(u[0].astype(np.float64))))[kept], rtol=1e-6, atol=1e-5)
    z = np.full((1, 4500), np.nan, f32)
    lib.emu_perturb(ptr(guarded(z)), ptr(guarded(np.full((1, 4500), 0.5, f32))), ptr(guarded(z.copy())), 1, 4500, C.c_float(1.0), C.c_float(0.9), 2)
    print("emulated long rows: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-attn-bound":
    # The tree attention with several query tiles: results are right and the same bits whatever upper bound of the keys the host has (exact, a block
    # too long, the whole cache) and whichever sequences lie beside a sequence; four and eight waves, one and two query tiles per workgroup.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    lib, f32 = V._lib, np.float32
    p = lambda a: a.ctypes.data_as(C.c_void_p)

    def bf16(a):
        u = a.astype(f32).view(np.uint32)
        return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(f32)
    rng = np.random.default_rng(98)
    for M, lengths, maxpos, big_min in ((33, (61, 159), 256, 0), (49, (78, 130), 256, 0), (96, (31, 100), 264, 1), (40, (350, 470), 560, 0)):
        B, nH, cap = 2, 1, (maxpos + 31) // 32 * 32
        q, K, Vv = bf16(3 * rng.standard_normal((B * M, nH * 64))), bf16(rng.standard_normal((B, nH, cap, 64))), bf16(rng.standard_normal((B, nH, cap, 64)))
        tree = make_tree(M, (10, 10, 10))
        see = np.zeros((M, 128), bool)
        for n in range(M):
            m = n
            while m >= 0:
                see[n, m] = True
                m = tree.parent[m]
        mask = np.packbits(see, axis=1, bitorder="little").view(np.uint32).copy()
        L = np.array(lengths, np.int32)

        def run(sel, keys):
            out = np.zeros((len(sel) * M, nH * 64), f32)
            rows = np.concatenate([q[b * M:(b + 1) * M] for b in sel])
            lib.emu_attn(p(rows), p(np.ascontiguousarray(K[sel])), p(np.ascontiguousarray(Vv[sel])), p(L[sel].copy()), len(sel), M, nH, maxpos, p(mask), keys, big_min, p(out))
            return out
        own = np.concatenate([run([b], int(L[b]) + M) for b in range(B)])
        for b in range(B):
            T = L[b] + M
            sc = q[b * M:(b + 1) * M].astype(np.float64) @ K[b, 0, :T].astype(np.float64).T / 8
            sc[:, L[b]:][~see[:, :M]] = -np.inf
            w = np.exp(sc - sc.max(1, keepdims=True))
            want = w @ Vv[b, 0, :T].astype(np.float64) / w.sum(1, keepdims=True)
            err = np.abs(own[b * M:(b + 1) * M] - want).max()
            # weights and result each rounded to bf16: 2^-9 of the largest value each, and a tenth for the fp32 sums
            assert err < 1.1 * 2.0 ** -8 * np.abs(Vv[b]).max(), (M, b, err)
        for keys in (int(L.max()) + M, int(L.max()) + M + 32, maxpos):
            assert np.array_equal(run([0, 1], keys), own), (M, lengths, keys)
        print(f"attention of {M} nodes: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-unfetched":
    # Steps whose tokens are fetched and steps whose tokens are not (the host's bound of the length grows by the longest path) leave the same bits: three
    # query tiles, lengths at which the bound is a block longer than the sequence.
    from paper_2410_21951_amd import Vadusa, TreeArrays, DBG
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=64, speech_vocab=71, text_vocab=20,
                      n_draft_heads=4, max_positions=256, dtype="bf16")
    W = make_weights(cfg, 85, std=0.08)
    rng = np.random.default_rng(86)
    text, prompt = [rng.integers(0, cfg.text_vocab, 2).astype(np.int32)], [rng.integers(0, cfg.speech_vocab, 134).astype(np.int32)]
    t = make_tree(48, (10, 10, 10, 10))
    tree = TreeArrays(t.parent, t.rank)
    got = []
    for mode in ("fetched", "unfetched"):
        dev = Vadusa(cfg, max_batch=1, max_tree_nodes=48, ignore_eos=True, prefill_chunk=144)
        dev.load_weights(W)
        dev.prefill(text, prompt)
        lengths = []
        for i in range(3):
            dev.step(tree, 1, sync=mode == "fetched")
            if mode == "fetched":
                lengths.append(136 + len(dev.read_output(0)))
        got.append((dev.read_output(0).tolist(), dev.debug(DBG.LOGITS).copy()))
        if mode == "fetched":
            # the third step's bound without fetching: five rows more per step
            assert -(-(136 + 2 * 5 + 48) // 32) > -(-(lengths[1] + 48) // 32), lengths
    assert got[1][0] == got[0][0] and np.array_equal(got[1][1], got[0][1])
    print("emulated unfetched steps: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-lin-turns":
    # Maps behind which the residual stream is written: a row block's workgroups go through a wave's k-steps from rb / row blocks of them on, also where the
    # k-steps are no whole number of chunks.  So a row block gives the bits that it gives as the first one (which starts at the first
    # k-step) on operands whose k-steps are moved around by that much.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    lib, f32 = V._lib, np.float32
    p = lambda a: C.c_void_p(a.ctypes.data)

    def bf16(a):
        return (a.astype(f32).view(np.uint32) & 0xffff0000).view(f32)

    def run(X, W):
        out = np.zeros((len(X), len(W)), f32)
        return out, lib.emu_lin_resid(p(X), p(W), len(X), len(W), X.shape[1], p(out))
    rng = np.random.default_rng(99)
    # one chunk and less per wave, several and a rest, whole ones; four and eight waves; one and two row tiles, a ragged last block
    for R, N, K in ((64, 16, 192), (40, 16, 768), (64, 32, 1024), (64, 16, 2048), (48, 32, 2240), (130, 1024, 384)):
        X, W = bf16(rng.standard_normal((R, K))), bf16(rng.standard_normal((N, K)))
        out, shape = run(X, W)
        rows, nks = shape // 16 * 16, K // 32
        want = X.astype(np.float64) @ W.astype(np.float64).T
        assert np.abs(out - want).max() < 1e-4 * np.sqrt(K), (R, N, K)
        nw, blocks = 8 if nks >= 64 else 4, -(-R // rows)
        moved = 0
        for rb in range(1, blocks) if N < 1024 else (blocks - 1,):
            order = []
            for w in range(nw):
                lo, hi = nks * w // nw, nks * (w + 1) // nw
                turn = (hi - lo) * rb * (65536 // blocks) >> 16
                moved += turn > 0
                order += [lo + (i + turn) % (hi - lo) for i in range(hi - lo)]
            at = (np.array(order)[:, None] * 32 + np.arange(32)).ravel()
            mine = X[rb * rows:(rb + 1) * rows]
            first = np.concatenate([mine, X])[:R]
            got, _ = run(np.ascontiguousarray(first[:, at]), np.ascontiguousarray(W[:, at]))
            assert np.array_equal(got[:len(mine)], out[rb * rows:rb * rows + len(mine)]), (R, N, K, rb)
        assert moved
        print(f"turns of {R} x {N} x {K}: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
def taken_events():
    """(launch, what, address, x, y) of everything since the last call (see tests/emu/emu_rt.cpp)."""
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    f = V._lib.emu_take_events
    f.restype, f.argtypes = C.c_size_t, [C.c_void_p, C.c_size_t]
    a = np.zeros((f(None, 0), 5), np.uint64)
    f(a.ctypes.data_as(C.c_void_p), len(a))
    return a.astype(np.int64)


if dtype == "bf16-touched":
    # What idle workgroups touch over a prompt of three passes and a step: lines of the weights of a map that a later launch of the same pass reads, each
    # once a pass.  Two layers of several column groups each, more pieces than one launch may touch.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    from paper_2410_21951_amd import Vadusa, TreeArrays
    cfg = ModelConfig(n_layers=2, d_model=192, n_heads=3, head_dim=64, d_ffn=384, speech_vocab=71, text_vocab=20,
                      n_draft_heads=3, max_positions=96, dtype="bf16")
    d, F = cfg.d_model, cfg.d_ffn
    W = make_weights(cfg, 71, std=0.05)
    rng = np.random.default_rng(87)
    t = make_tree(8, (3, 2))
    dev = Vadusa(cfg, max_batch=1, max_tree_nodes=8, ignore_eos=True, prefill_chunk=16)
    dev.load_weights(W)
    C.c_int.in_dll(V._lib, "emu_logging").value = 1
    dev.prefill([rng.integers(0, cfg.text_vocab, 3).astype(np.int32)], [rng.integers(0, cfg.speech_vocab, 37).astype(np.int32)])
    dev.step(TreeArrays(t.parent, t.rank), 1)
    ev = taken_events()
    maps, lines = ev[ev[:, 1] == 1], ev[ev[:, 1] == 0]
    # the step's maps in the order of their launches: all that there are
    layer = [3 * d * d, d * d, F * d, d * F]
    size = [2 * n for n in layer * 2 + [80 * d, d * d, 80 * d]]
    step = maps[-len(size):]
    start = list(step[:, 2])
    assert len(set(start)) == len(size) and list(step[:, 4]) == [1] * 9 + [3, 3]
    passes = np.flatnonzero(maps[:, 2] == start[0])              # the first map of each pass
    assert [len(p) for p in np.split(maps, passes[1:])] == [5, 5, 11, 11]   # earlier prompt passes end behind the last layer's QKV
    bounds = [(a + z * int(m[3]), a + z * int(m[3]) + n, i) for i, (a, n, m) in enumerate(zip(start, size, step)) for z in range(int(m[4]))]
    touched = set()
    seen = {}
    for launch, _, at, x, y in lines:
        inside = [i for lo, hi, i in bounds if lo <= at and at + 4 <= hi]
        assert len(inside) == 1, f"line {at:x} touched by launch {launch} is not of one map"
        i = inside[0]
        after = maps[maps[:, 0] > launch]
        read = after[after[:, 2] == start[i]]
        assert len(read), f"map {i} touched by launch {launch} is not read any more"
        again = after[after[:, 2] == start[0]]                   # the next pass
        assert i == 0 or not len(again) or read[0, 0] < again[0, 0], f"map {i} touched by launch {launch} is not read in its pass"
        assert (at - start[i] if i < 9 else at - min(lo for lo, hi, k in bounds if k == i and lo <= at < hi)) % 128 == 0
        n_pass = int((maps[passes, 0] <= launch).sum())
        key = (n_pass, int(at))
        assert seen.setdefault(key, (launch, x, y)) == (launch, x, y), f"line {at:x} touched again by launch {launch}"
        touched.add(i)
    print(f"touched {len(seen)} lines of maps {sorted(touched)}", flush=True)
    assert touched == set(range(1, 11))                          # (nothing is idle ahead of a pass's first map)
    print("emulated touched weights: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-touch-grid":
    # The pieces that idle workgroups share out: every line of a piece by exactly one lane, on the XCD whose workgroups read its group, from buffers that end at
    # a guard page.  Four and eight waves, several rows of the grid, a first column that is no multiple of eight, several maps of one
    # shape, fewer workgroups than pieces and more.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    lib = V._lib
    C.c_int.in_dll(lib, "emu_logging").value = 1
    for waves, first, columns, rows, nz, maps in (
            (4, 16, 8, 1, 1, [(1, 6, 12, 0, 1000)]), (8, 8, 16, 3, 1, [(2, 6, 40, 0, 1000), (1, 20, 9, 1, 1000)]), (4, 1, 24, 1, 3, [(1, 6, 12, 0, 1000), (1, 6, 5, 0, 1000)]),
            (4, 5, 8, 1, 4, [(1, 10, 17, 0, 34), (1, 10, 3, 0, 3)]), (8, 24, 8, 2, 2, [(4, 6, 32, 2, 7), (1, 2, 1, 0, 9)]), (4, 64, 192, 1, 1, [(1, 4, 3, 0, 100)])):
        n = len(maps)
        one = [NT * nks * 1024 for _, nks, NT, _, _ in maps]
        base = [lib.emu_alloc(nz * b, 0) for b in one]           # (sizes are multiples of 256: the last map ends at the guard page)
        ints = lambda k: (C.c_int * n)(*(m[k] for m in maps))
        lib.emu_touch_grid(waves, first, columns, rows, nz, n, (C.c_void_p * n)(*base), ints(0), ints(1), ints(2), ints(3), ints(4), (C.c_size_t * n)(*one))
        ev = taken_events()
        got = sorted((int(at), int(x) % 8) for _, _, at, x, y in ev)
        assert all(first <= x < first + columns and y < rows for _, _, _, x, y in ev)
        want = []
        for (ct, nks, NT, start, pieces), b, bytes_ in zip(maps, base, one):
            group, groups = ct * nks * 1024, NT // ct
            take = max(min(-(-group // 8192) - start, pieces // groups), 0)
            want += [(b + z * bytes_ + g * group + min((start + i) * 8192 + lane * 128, group - 128), g % 8)
                     for z in range(nz) for g in range(groups) for i in range(take) for lane in range(64)]
        assert got == sorted(want), (waves, first, columns, rows, nz, maps)
        assert want
        print(f"{len(want)} lines by {columns} x {rows} workgroups of {waves} waves: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-row-stats":
    # The row statistics that a map with a folded LayerNorm merges: the same bits as in this order, lane by lane, with one of a pair's squares
    # unrounded where the other is added to it.  The map is of zeros with column sums of -1, so an output is the row's 1 / standard deviation times its mean.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    lib, f32 = V._lib, np.float32
    p = lambda a: C.c_void_p(a.ctypes.data)
    rng = np.random.default_rng(101)
    for rt, big, nks in ((1, False, 32), (2, False, 32), (4, False, 32), (4, True, 32), (2, False, 6), (4, False, 20), (4, True, 40)):
        R, tiles = 16 * rt, 2 * nks
        N = 128 if big else R
        X, W = np.zeros(R * nks * 32, np.uint16), np.zeros(N * nks * 32, np.uint16)
        bias, cs, out = np.zeros(N, f32), np.full(N, -1, f32), np.zeros((R, N), f32)
        st = np.stack([rng.standard_normal((R, tiles)) + 3, rng.random((R, tiles)) * 16], axis=2).astype(f32)
        if big:
            lib.emu_big_logits(p(X), p(W), p(bias), p(cs), p(st), p(out), nks, N // 16, R, C.c_uint(0))
        else:
            lib.emu_lin_logits(p(X), p(W), p(bias), p(cs), p(st), p(out), nks, R, rt)
        lanes = 8 if rt > 1 else 16                              # neighbouring lanes of a row, 32 / lanes pairs each, the rest behind them
        first = 32 // lanes
        want = np.zeros(R, f32)
        for r in range(R):
            c0 = st[r, 0, 0]
            s = np.zeros((lanes, 3), f32)
            for part in range(lanes):
                for j in range(-(-tiles // (2 * lanes))):
                    t = 2 * (part + j * lanes)
                    if t >= tiles:
                        continue
                    d0, d1 = st[r, t, 0] - c0, st[r, t + 1, 0] - c0
                    # workgroups of 64 rows, the first half of them: the second square stays unrounded in piece 1 (k_lin's vocabulary map: 1 and 2)
                    if rt == 4 and r < 32 and j < first and 0 < j <= (1 if big else 2):
                        d0, d1 = d1, d0
                    pair = f32(np.float64(d0) * np.float64(d0) + np.float64(d1 * d1))     # (53 bits hold both: rounded once, but for ties)
                    s[part] += np.array([d0 + d1, st[r, t, 1] + st[r, t + 1, 1], pair], f32)
            for mask in (1, 2, 7, 15)[:3 if lanes == 8 else 4]:
                s = s + s[np.arange(lanes) ^ mask]
            s1, s2, s3 = s[0]
            m2 = s2 + f32(16) * max(s3 - s1 * s1 / f32(tiles), f32(0))
            want[r] = (c0 + s1 / f32(tiles)) * (f32(1) / np.sqrt(m2 / f32(nks * 32) + f32(1e-5)))
        assert (out == out[:, :1]).all()
        same = out[:, 0] == want
        print(f"statistics of {R} rows of {tiles} tiles, {'k_big' if big else 'k_lin'}: {int(same.sum())} of {R} the same bits", flush=True)
        assert same.all(), np.flatnonzero(~same)
    print("emulated row statistics: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-giveup":
    # the error word, raised from the host: the next synchronising call reports it, later calls refuse, a prefill
    # recovers and decodes the same tokens
    from paper_2410_21951_amd import Vadusa, TreeArrays, VadusaError, DBG
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                      n_draft_heads=2, max_positions=64, dtype="bf16")
    W = make_weights(cfg, 71, std=0.08)
    rng = np.random.default_rng(73)
    text = [rng.integers(0, cfg.text_vocab, 3).astype(np.int32)]
    prompt = [rng.integers(0, cfg.speech_vocab, 9).astype(np.int32)]
    t = make_tree(8, (3, 2))
    tree = TreeArrays(t.parent, t.rank)
    dev = Vadusa(cfg, max_batch=1, max_tree_nodes=8, ignore_eos=True)
    dev.load_weights(W)

    def run():
        dev.prefill(text, prompt)
        return [dev.step(tree, 1 + i % 2) for i in range(3)]
    want = run()
    dev.debug_raise_error()
    codes = []
    for call in (lambda: dev.step(tree, 1), lambda: dev.debug(DBG.ROOT), lambda: dev.step(tree, 1)):
        try:
            call()
            codes.append(0)
        except VadusaError as e:
            codes.append(e.code)
    assert codes == [-5, -4, -4], codes
    assert run() == want
    print("emulated error word: reported, refused, recovered", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype.endswith("-pinned"):
    # The blocks that results arrive in: one per context, handed on by vadusa_destroy, and those that a create does not take
    # are given back by it; without pinned memory the results are the same.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    from paper_2410_21951_amd import Vadusa, TreeArrays
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                      n_draft_heads=2, max_positions=64, dtype=dtype[:4])
    blocks = C.c_int.in_dll(V._lib, "emu_host_blocks")
    new = lambda batch=1: Vadusa(cfg, max_batch=batch, max_tree_nodes=8, ignore_eos=True)
    several = [new(b) for b in (1, 300, 1, 2)]
    assert blocks.value == 4
    for v in several:
        v.close()
    assert blocks.value == 4                       # vadusa_destroy makes no HIP call
    dev = new()
    assert blocks.value == 1
    other = new(300)                               # (its results do not fit a block of the smallest size)
    assert blocks.value == 2
    other.close()
    W = make_weights(cfg, 71, std=0.08)
    text, prompt = [np.arange(3, dtype=np.int32)], [np.arange(5, dtype=np.int32)]
    t = make_tree(8, (3, 2))
    tree = TreeArrays(t.parent, t.rank)

    def run(v):
        v.load_weights(W)
        return v.prefill(text, prompt).tolist(), v.step(tree, 1), v.read_output(0).tolist()
    want = run(dev)
    dev.close()
    blocks.value = -1
    several = [new(), new()]                       # the first takes the block that is left
    assert run(several[1]) == want
    print("emulated results: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype.endswith("-errors"):
    # An error that another library's HIP call left behind is not this library's: every call works as without it.  A launch
    # of its own that is refused is reported by the call that made it, and by no later one.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    from paper_2410_21951_amd import Vadusa, TreeArrays, VadusaError, DBG
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                      n_draft_heads=2, max_positions=64, dtype=dtype[:4])
    W = make_weights(cfg, 71, std=0.08)
    text, prompt = [np.arange(3, dtype=np.int32)], [np.arange(5, dtype=np.int32)]
    t = make_tree(8, (3, 2))
    tree = TreeArrays(t.parent, t.rank)
    dev = Vadusa(cfg, max_batch=1, max_tree_nodes=8, ignore_eos=True)
    left, refuse = C.c_int.in_dll(V._lib, "emu_last_error"), C.c_int.in_dll(V._lib, "emu_fail_launch")
    calls = [lambda: dev.load_weights(W), lambda: dev.prefill(text, prompt), lambda: dev.step(tree, 1), lambda: dev.read_output(0),
             lambda: dev.debug(DBG.H_NODES), lambda: dev.read_kv(0, 0, 0, 0, 4), lambda: dev.read_kv(0, 0, 0, 0, 4, static=True)]
    for call in calls:
        left.value = 101
        call()
    left.value = 0
    for i in (1, 2, 3, 4, 5, 6, 0):
        refuse.value = 1
        try:
            calls[i]()
            raise AssertionError(f"call {i}: a refused launch went unreported")
        except VadusaError as e:
            assert e.code == -5, (i, e)
        if i in (1, 2):
            calls[1]()                            # a prefill starts the sequences again
    print("emulated errors: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype.endswith("-partial"):
    # kv_compact of one sequence of two with planted lists: the other one's verification is still pending, and its
    # lists stay the planted ones until its own compaction.
    from paper_2410_21951_amd import Vadusa, TreeArrays, DBG
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                      n_draft_heads=2, max_positions=64, dtype=dtype[:4])
    W = make_weights(cfg, 71, std=0.08)
    rng = np.random.default_rng(76)
    text = [rng.integers(0, cfg.text_vocab, 3).astype(np.int32) for _ in range(2)]
    prompt = [rng.integers(0, cfg.speech_vocab, 5).astype(np.int32) for _ in range(2)]
    t = make_tree(8, (3, 2))
    dev = Vadusa(cfg, max_batch=2, max_tree_nodes=8, ignore_eos=True)
    dev.load_weights(W)
    dev.prefill(text, prompt)
    planted = np.stack([[rng.permutation(70)[:16] for _ in range(2)] for _ in range(2)]).astype(np.int32)
    dev.verify(TreeArrays(t.parent, t.rank), 1, override=planted)
    dev.kv_compact(0)
    lists = dev.debug(DBG.DRAFT_TOPK)
    assert np.array_equal(lists[1], planted[1]) and not np.array_equal(lists[0], planted[0]), lists
    dev.kv_compact(1)
    lists = dev.debug(DBG.DRAFT_TOPK)
    z = dev.debug(DBG.DRAFT_LOGITS)
    for b in range(2):
        for i in range(2):
            assert np.array_equal(lists[b, i], np.lexsort((np.arange(71), -z[b, i]))[:16]), (b, i)
    print("emulated partial compaction: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "fp32-sums":
    # The linear map of the fp32 model against 64-bit arithmetic: no further off than 64 partial sums of K / 64 products each
    # (fused multiply-add), added pairwise, are on the same operands.
    import ctypes as C
    import paper_2410_21951_amd.vadusa as V
    rng = np.random.default_rng(77)
    f = np.float32
    for K in (64, 256, 320, 1024):
        X, Wm = rng.standard_normal((16, K)).astype(f), rng.standard_normal((48, K)).astype(f)
        out = np.zeros((16, 48), f)
        p = lambda a: a.ctypes.data_as(C.c_void_p)
        V._lib.emu_lin32(p(X), p(Wm), p(out), 16, K, 48)
        prod = X.astype(np.float64)[:, None, :] * Wm.astype(np.float64)[None]      # exact
        part = np.zeros((16, 48, 64), f)
        for k in range(0, K, 64):
            part = (part + prod[:, :, k:k + 64]).astype(f)
        while part.shape[2] > 1:
            part = (part[:, :, ::2] + part[:, :, 1::2]).astype(f)
        want = prod.sum(axis=2)
        err = lambda a: float(np.sqrt(np.mean((a - want) ** 2) / np.mean(want ** 2)))
        print(f"K {K}: kernel {err(out):.2e}, pairwise sums {err(part[:, :, 0]):.2e}", flush=True)
        assert err(out) < 1.1 * err(part[:, :, 0]), K       # (768 results: the two root mean squares scatter by some 4 % each)
    print("emulated fp32 sums: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype == "bf16-4gib-map":
    # One linear map of more than 4 GiB (K = 4096): 64 x 128 workgroups at its start and on both sides of the 4 GiB mark.
    # The weights are address space that is never touched but for the tiles of these workgroups, all values of tile t
    # being t's value; X is all ones, its statistics mean 0 and variance 1.
    import ctypes as C
    import mmap
    import paper_2410_21951_amd.vadusa as V
    nks, R = 128, 2
    tile = nks * 1024                                     # bytes of a column tile
    first = (1 << 32) // tile                             # first tile behind the mark
    NT = first + 8
    space = mmap.mmap(-1, NT * tile, flags=mmap.MAP_PRIVATE | mmap.MAP_ANONYMOUS | 0x4000)   # MAP_NORESERVE
    Wt = np.frombuffer(space, np.uint16)
    value = lambda t: 0x3c00 + (t % 8) * 8 + (256 if t >= first else 128 if t >= 8 else 0)   # bits of a bf16
    groups = (0, first // 8 - 1, first // 8)
    for g in groups:
        for t in range(8 * g, 8 * g + 8):
            Wt[t * tile // 2:(t + 1) * tile // 2] = value(t)
    X = np.full(nks * 512, 0x3f80, np.uint16)
    zero = np.zeros(NT * 16, np.float32)
    stats = np.tile(np.array([0, 16], np.float32), R * nks * 2)
    out = np.full((R, NT * 16), np.nan, np.float32)
    p = lambda a: a.ctypes.data_as(C.c_void_p)
    for g in groups:
        V._lib.emu_big_logits(p(X), p(Wt), p(zero), p(zero), p(stats), p(out), nks, NT, R, C.c_uint(g))
        for t in range(8 * g, 8 * g + 8):
            want = 32 * nks * np.array([value(t) << 16], np.uint32).view(np.float32)[0] / np.sqrt(1 + 1e-5)
            got = out[:, 16 * t:16 * t + 16]
            assert np.abs(got / want - 1).max() < 1e-5, (g, t, got[0, 0], want)   # (4096 equal terms: sums exact but for a few roundings)
    print("emulated 4 GiB map: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype.endswith("-nanfill"):
    # A cache of 40 positions is stored as 64 (whole blocks of 32 keys), and a masked or unwritten key enters the
    # attention as 0 x its value: whatever the caller's memory held, a context starts with zeros in all of it.
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                      n_draft_heads=2, max_positions=40, dtype=dtype[:4])
    W = make_weights(cfg, 71, std=0.08)
    rng = np.random.default_rng(75)
    text = [rng.integers(0, cfg.text_vocab, 2 + b).astype(np.int32) for b in range(2)]
    prompt = [rng.integers(0, cfg.speech_vocab, 9 - b).astype(np.int32) for b in range(2)]
    Lockstep(cfg, W, text, prompt, 8)              # compares the prompt's cache and the draft heads' logits
    print(f"emulated {dtype}: compared", flush=True)
    sys.stdout.flush()
    os._exit(0)
if dtype in ("bf16-nan", "fp32-nan"):
    # A model whose logits are all NaN (a NaN in the final LayerNorm's scale): no row has a largest entry, so the
    # arg-max and the draft lists have nothing to return.  The step must still stay inside its buffers (the arena sits
    # between guard pages) and hand back token ids of the vocabulary.
    from paper_2410_21951_amd import Vadusa, TreeArrays
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                      n_draft_heads=2, max_positions=64, dtype=dtype[:4])
    W = make_weights(cfg, 71, std=0.08)
    W["lnf_g"] = W["lnf_g"].copy()
    W["lnf_g"][3] = np.nan
    rng = np.random.default_rng(74)
    text = [rng.integers(0, cfg.text_vocab, 3).astype(np.int32)]
    prompt = [rng.integers(0, cfg.speech_vocab, 9).astype(np.int32)]
    t = make_tree(8, (3, 2))
    tree = TreeArrays(t.parent, t.rank)
    dev = Vadusa(cfg, max_batch=1, max_tree_nodes=8, ignore_eos=True)
    dev.load_weights(W)
    dev.prefill(text, prompt)
    for i in range(3):
        out = dev.step(tree, 1 + i % 2)
        for toks in out:
            assert all(0 <= int(v) <= cfg.speech_vocab for v in toks), toks
    print("emulated NaN logits: stayed in bounds", flush=True)
    sys.stdout.flush()
    os._exit(0)
cfg = ModelConfig(n_layers=1, d_model=64, n_heads=1, head_dim=64, d_ffn=128, speech_vocab=70, text_vocab=20,
                  n_draft_heads=2, max_positions=64, dtype=dtype)
W = make_weights(cfg, 71, std=0.08)
rng = np.random.default_rng(72)
text = [rng.integers(0, cfg.text_vocab, 2).astype(np.int32), rng.integers(0, cfg.text_vocab, 3).astype(np.int32)]
prompt = [rng.integers(0, cfg.speech_vocab, 9).astype(np.int32), rng.integers(0, cfg.speech_vocab, 5).astype(np.int32)]
tree = make_tree(8, (3, 2))
t0 = time.time()
ls = Lockstep(cfg, W, text, prompt, 8)
for tau in (1, 3):
    ls.step(tree, tau)
# the stochastic rule on a 4-node tree (its kernel does not depend on the model's dtype, so the
# search regimes run once): every token kept for the bf16 model; a nucleus cut and a nucleus smaller than tau for the fp32 model
small = make_tree(4, (2, 1))
regimes = ((2, 0.9, 1.0),) if dtype == "bf16" else ((3, 1.0, 0.7), (4, 0.5, 0.02))
for i, (tau, T, top_p) in enumerate(regimes):
    ls.step(small, tau, sample=(T, top_p, make_uniforms(73, i, 2, small.n_nodes, cfg.speech_vocab + 1)))
ls.step(tree, 1)
ls.check_kv(layers=[0])
s = ls.stats
print(f"emulated {dtype}: compared {s.compared}/{s.steps} logit err {s.max_logit_err:.2e} score err "
      f"{s.max_score_err:.2e} nucleus sizes {[round(x, 1) for x in s.nucleus_sizes]} ties {s.tie_root}/{s.tie_list}/{s.tie_edge} in {time.time() - t0:.0f} s", flush=True)
assert s.compared >= 1
sys.stdout.flush()
os._exit(0)   # the emulation's worker threads never end
