"""The HIP kernel sources compiled for the host and run on a CPU emulation of the GPU's
execution model (tests/emu), in lockstep with the oracle: checks index arithmetic, control
flow and bounds (the arena sits between guard pages and starts out filled with garbage)
without a GPU.  The smallest legal model (d = 64, one head), where two of a workgroup's four
waves have no k-steps of a linear map at all; 40, 72 and 256 rows (ragged tiles, masks of several words, the many-row
kernels); both shapes of k_tile; eight waves on a reduction of 2048 and on more than 288 keys; lists, edges and scores of rows of more than 4096 logits; the error word raised from the host; models whose logits are all NaN (no arg-max, no draft lists: the
step must stay inside its buffers); an arena that arrives full of NaN bits; one linear map of more than 4 GiB; compaction of one
sequence beside a pending one; left-over errors of other HIP calls and refused launches; the pinned result blocks; the order of sums: row
statistics, the k-steps of row blocks, the attention under other bounds of its keys; what idle workgroups touch."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "emu"))

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/llvm/bin/clang++"), reason="needs ROCm's clang++")


@pytest.fixture(scope="module")
def emu_lib(tmp_path_factory):
    import emulate
    out = tmp_path_factory.mktemp("emu")
    lib = emulate.build(str(out))
    yield lib
    shutil.rmtree(str(out), ignore_errors=True)


@pytest.mark.parametrize("dtype", ["bf16", "fp32", "bf16-40rows", "bf16-72rows", "bf16-256rows", "bf16-tile256", "bf16-tile128", "bf16-long-ffn", "bf16-long-keys", "long-rows", "bf16-giveup", "bf16-nan", "fp32-nan", "bf16-nanfill", "bf16-4gib-map", "bf16-partial", "fp32-partial", "bf16-errors", "bf16-pinned", "fp32-sums"])
def test_emulated_step_matches_oracle(emu_lib, dtype):
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_case.py"), emu_lib, dtype],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=600, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    assert ("recovered" if dtype == "bf16-giveup" else "stayed in bounds" if dtype.endswith("-nan") else "compared") in r.stdout


def test_row_statistics_are_added_in_one_order(emu_lib):
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_case.py"), emu_lib, "bf16-row-stats"],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=600, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "compared" in r.stdout


@pytest.mark.parametrize("case", ["bf16-attn-bound", "bf16-unfetched"])
def test_results_do_not_depend_on_the_hosts_bound(emu_lib, case):
    """The attention's sums follow from a sequence's own length, not from the upper bound that the host has of the longest one."""
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_case.py"), emu_lib, case],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=600, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "compared" in r.stdout


@pytest.mark.parametrize("case", ["bf16-touched", "bf16-touch-grid"])
def test_weights_touched_ahead(emu_lib, case):
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_case.py"), emu_lib, case],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=600, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "compared" in r.stdout


def test_what_is_touched_is_what_is_read_next(emu_lib):
    """A launch touches, from where the last one stopped, the maps behind the one that is being read, in their order, up to three of them and within what it
    may; a map is left behind once it is read, and one that k_lin does not take is passed over."""
    f = C.CDLL(emu_lib).emu_ahead
    rng = np.random.default_rng(11)
    ints = lambda a: (C.c_int * len(a))(*map(int, a))
    stopped = finished = 0
    for _ in range(300):
        n = int(rng.integers(1, 14))
        groups = np.where(rng.random(n) < 0.2, 0, rng.integers(1, 200, n))
        size = 1024 * rng.integers(1, 129, n)
        reading, workgroups = [], []
        for m in range(n):                                       # launches without a map of their own between the maps'
            if rng.random() < 0.5:
                reading.append(-1)
                workgroups.append(0 if rng.random() < 0.4 else 8 * int(rng.integers(1, 31)))
            reading.append(m)
            workgroups.append(0 if rng.random() < 0.4 else 8 * int(rng.integers(1, 31)))
        kib, most = rng.integers(8, 161, len(reading)), rng.integers(100, 25000, len(reading))
        out = np.zeros((len(reading), 3, 4), np.int32)
        f(n, ints(groups), ints(size), len(reading), ints(reading), ints(workgroups), ints(kib), ints(most), out.ctypes.data_as(C.c_void_p))
        at = [0] * n                                             # pieces of each group that have been touched
        now = -1
        for k, mine in enumerate(out):
            now = max(now, reading[k])
            took = [tuple(t) for t in mine if t[0] >= 0]
            budget = min(workgroups[k] * int(kib[k]), int(most[k])) // 8 if workgroups[k] else 0
            nxt = [m for m in range(now + 1, n) if groups[m] and at[m] * 8192 < size[m]]
            want = []
            while budget and nxt and len(want) < 3:
                m = nxt.pop(0)
                take = min(-(-int(size[m]) // 8192) - at[m], budget // int(groups[m]))
                if not take:
                    stopped += 1
                    break
                want.append((m, at[m], take, int(groups[m])))
                budget -= take * int(groups[m])
                at[m] += take
                if at[m] * 8192 < size[m]:
                    stopped += 1
                    break
                finished += 1
            assert took == want, (k, took, want)
    assert stopped > 100 and finished > 100


def test_row_blocks_start_at_different_k_steps(emu_lib):
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_case.py"), emu_lib, "bf16-lin-turns"],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=600, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "compared" in r.stdout


def test_workgroups_of_a_head_start_apart(emu_lib):
    """The key block at which each query tile's workgroup starts is blocks * y / tiles, rounded down, without a division."""
    f = C.CDLL(emu_lib).emu_turns
    out = np.zeros(64, np.int32)
    for tiles in range(1, 65):
        for blocks in [*range(1, 140), 1000, 3328, 16384, (1 << 20) - 1]:
            f(blocks, tiles, out.ctypes.data_as(C.c_void_p))
            assert np.array_equal(out[:tiles], blocks * np.arange(tiles) // tiles), (blocks, tiles)


def test_tile_shapes_of_the_gpu_tests(emu_lib):
    """The shapes that the GPU tests of k_lin name are those that the library picks, and each shape is among them."""
    import ctypes as C
    from test_gpu_layer_kernels import TILE_SHAPES
    pick = C.CDLL(emu_lib).emu_lin_shape
    seen = set()
    for d, ffn, nodes, batch, V, shapes in TILE_SHAPES:
        rows = nodes * batch
        assert rows % 16, "the last row tile is ragged"
        got = [pick(rows, -(-n // 16)) for n in (3 * d, d, ffn, V + 1)]
        assert " ".join(f"{s // 16}x{s % 16}" for s in got) == shapes, (d, ffn, rows, V)
        seen |= {(kind, s) for kind, s in zip(("qkv", "residual", "ffn1", "logits"), shapes.split())}
    every = ("1x1", "1x2", "2x2", "2x4", "3x4", "4x4")
    assert seen == {(kind, s) for kind in ("qkv", "residual", "ffn1", "logits") for s in every} | {("logits", "2x1"), ("logits", "4x2")}
    # maps whose columns are a multiple of 64 never pick 2x1 or 4x2, which are built for the vocabulary map alone
    assert {pick(16 * rt, nt) for rt in range(1, 129) for nt in range(4, 1025, 4)} <= {16 * int(s[0]) + int(s[2]) for s in every}


def test_kernels_of_the_mixed_gpu_tests(emu_lib):
    """The kernels that the GPU test of mixed maps names are those that the rule picks."""
    import ctypes as C
    sys.path.insert(0, HERE)
    from test_gpu_layer_kernels import MIXED
    pick = C.CDLL(emu_lib).emu_map_kernel
    names = ("lin", "big", "tile256", "tile128")
    for d, ffn, nodes, batch, kernels in MIXED:
        rows = nodes * batch
        got = [pick(rows, n // 16, k // 32, epi) for n, k, epi in ((3 * d, d, 0), (d, d, 3), (ffn, d, 1), (d, ffn, 3))]
        assert " ".join(names[g] for g in got) == kernels, (d, ffn, rows)


# us per launch on an MI355X, in steps whose maps all ran in k_lin, k_big, k_tile 256 x 128, k_tile 128 x 64
# map (0 QKV, 1 FFN1, 2 vocabulary, 3 out-projection and FFN2), rows, columns, reduction
MEASURED = [
    (3, 16384, 64, 64, 27.4, 7.3, 10.2, 6.5), (3, 8192, 64, 256, 22.4, 7.1, 11.5, 6.4), (3, 4096, 128, 128, 12.0, 6.0, 11.7, 6.3),
    (0, 2048, 576, 192, 14.8, 6.5, 14.4, 7.3), (1, 1536, 768, 192, 11.0, 5.9, 11.6, 7.9), (3, 6144, 256, 256, 18.0, 8.9, 14.4, 8.2),
    (0, 896, 768, 256, 11.5, 6.9, 14.6, 7.0), (0, 1536, 768, 256, 11.0, 7.0, 14.9, 8.2), (1, 1280, 1024, 256, 11.3, 6.9, 12.3, 8.2),
    (3, 4096, 256, 256, 11.1, 8.5, 15.1, 8.8), (3, 4096, 256, 1024, 19.0, 11.8, 22.0, 11.7), (1, 1024, 1280, 320, 13.4, 8.3, 14.2, 9.7),
    (0, 768, 1152, 384, 12.2, 7.5, 16.0, 8.7), (0, 512, 1152, 384, 9.5, 7.4, 15.8, 8.5), (0, 4096, 1536, 512, 35.4, 25.8, 21.0, 26.8),
    (2, 16384, 1025, 512, 111.8, 106.1, 73.6, 94.4), (3, 896, 640, 640, 12.5, 9.2, 17.8, 9.4), (0, 320, 2304, 768, 12.8, 9.7, 19.5, 10.4),
    (0, 1536, 2304, 768, 26.0, 19.5, 22.1, 20.6), (1, 2048, 3840, 960, 51.6, 27.2, 26.6, 39.5), (2, 8192, 1025, 1024, 73.9, 76.6, 55.0, 61.8),
    (0, 64, 3072, 1024, 5.9, 12.8, 17.1, 11.2), (1, 320, 4096, 1024, 14.0, 12.0, 19.5, 11.7), (3, 320, 1024, 4096, 12.0, 32.1, 49.5, 24.7),
    (3, 1024, 1024, 4096, 19.2, 33.1, 53.0, 27.9), (1, 2048, 4096, 1024, 51.3, 28.0, 25.5, 39.6), (3, 2048, 1024, 4096, 34.4, 35.6, 54.2, 30.3),
    (3, 3200, 1024, 4096, 60.6, 44.1, 54.0, 49.1), (0, 1024, 3072, 1024, 23.9, 17.7, 25.0, 23.2), (2, 64, 16001, 1024, 13.8, 16.5, 19.9, 14.6),
    (2, 1024, 16001, 1024, 134.0, 94.7, 83.1, 114.3),
]


def test_kernels_at_measured_maps(emu_lib):
    """Widths from 64 to 1024: the kernel that the rule takes is within 15 % of the fastest (a launch's time repeats within 5 %; two kernels
    may be close)."""
    import ctypes as C
    pick = C.CDLL(emu_lib).emu_map_kernel
    for epi, R, N, K, *us in MEASURED:
        took = us[pick(R, -(-N // 16), K // 32, epi)]
        assert took <= 1.15 * min(us), (epi, R, N, K, took, us)


def test_attention_shapes(emu_lib):
    """The attention's tiles and waves that the GPU test names are those that the rule picks; and no shape is taken at one number of
    workgroups only: what 512 workgroups of two tiles take, 528 take too, and 16 heads fewer take what 256 and 512 of one tile take."""
    import ctypes as C
    sys.path.insert(0, HERE)
    from test_gpu_layer_kernels import ATTENTION
    pick = C.CDLL(emu_lib).emu_attn_shape
    seen = set()
    for d, batch, nodes, prompt, chunk, big_min, shapes in ATTENTION:
        heads, lo, hi = batch * d // 64, prompt + 2, prompt + 16      # lengths of the prompts
        name = lambda rows, keys: "{}x{}".format(*divmod(pick(heads, -(-rows // 16), keys, big_min), 16))
        step = {name(nodes, n + nodes + 4 * i) for n in (lo, hi) for i in (0, 1)}
        per = min(chunk or max(nodes, min(128, max(1, 2048 // batch) // 16 * 16)), -(-hi // 16) * 16)
        # all passes but the first are full; the last layer's attention of the last pass has one tile
        passes = sorted({name(min(per, n), min((i + 1) * per, 704 if prompt < 700 else 1104)) for n in (lo, hi) for i in range(-(-n // per))})
        assert (" ".join(passes) + ", " + " ".join(sorted(step))) == shapes, (d, batch, nodes, prompt)
        seen |= set(passes) | step
    assert seen == {"1x4", "1x8", "2x4"}
    for keys in range(32, 3328, 32):
        for qt in (2, 4, 8, 64):
            for heads, beside in ((512 // (qt // 2), 528 // (qt // 2)), (256 // qt, 240 // qt), (512 // qt, 496 // qt)):
                if heads and beside:
                    assert pick(heads, qt, keys, 0) == pick(beside, qt, keys, 0), (heads, qt, keys)


@pytest.mark.parametrize("ct,nks,NT,start,pieces", [(1, 32, 64, 0, 10000), (2, 32, 192, 0, 10000), (4, 32, 65, 0, 10000), (1, 128, 64, 0, 400), (1, 128, 64, 6, 10000),
                                                    (1, 2, 3, 0, 10000), (2, 18, 7, 0, 10000), (3, 6, 40, 1, 30), (1, 32, 64, 0, 63), (4, 2, 3, 0, 10000)])
def test_touched_lines(emu_lib, ct, nks, NT, start, pieces):
    """Weights touched ahead: from piece `start` of 64 lines of each group of column tiles on, as many as `pieces` allows, every line in its group, by
    the XCD whose workgroups read the group, and none outside the map."""
    f = C.CDLL(emu_lib).emu_touch_lines
    group, groups = ct * nks * 1024, NT // ct
    lines, xcds = np.zeros((20000, 64), np.int64), np.zeros(20000, np.int32)
    n = f(ct, nks, NT, start, pieces, lines.ctypes.data_as(C.c_void_p), xcds.ctypes.data_as(C.c_void_p))
    take = min(-(-group // 8192) - start, pieces // groups) if groups else 0
    want = {(g, line) for g in range(groups) for line in range(start * 64, min((start + take) * 64, group // 128))}
    got = set()
    for row, x in zip(lines[:n], xcds[:n]):
        for at in row:
            g, off = divmod(int(at), group)
            assert g % 8 == x and off % 128 == 0 and 0 <= g < groups
            got.add((g, off // 128))
    assert got == want
    assert n == take * groups


@pytest.mark.parametrize("R,NT,rows,ct", [(2048, 256, 256, 8), (1024, 64, 64, 8), (3200, 64, 128, 4), (300, 65, 64, 8), (65, 1, 64, 8), (64, 1001, 64, 8), (577, 36, 128, 4), (2000, 24, 256, 8)])
@pytest.mark.parametrize("exact", [1, 0])
def test_every_tile_is_taken_once(emu_lib, R, NT, rows, ct, exact):
    """The tiles of the many-row maps in blocks per XCD, by multiplications and by the divisions that stand in for them in very large grids."""
    out = np.full((20000, 2), -1, np.int32)
    n = C.CDLL(emu_lib).emu_tiles(R, NT, rows, ct, exact, out.ctypes.data_as(C.c_void_p))
    got = [tuple(t) for t in out[:n] if t[0] >= 0]
    assert sorted(got) == [(r, c) for r in range(-(-R // rows)) for c in range(-(-NT // ct))]
