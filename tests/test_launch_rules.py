"""The rules by which work is cut into workgroups, compiled on the host on their own: that what they choose stays inside the
scratch and grid limits the kernels assume, and is the best or near the best of what was measured on the device."""
import pathlib
import random
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = tmp_path_factory.mktemp("rules") / "driver"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2511_14450_amd/csrc'}", str(ROOT / "tests/rules/rules_driver.cpp"),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(lines):
        r = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]
    return run


# ---------------------------------------------------------------- decode attention of generic stages
# bytes an element, features of a head, (request, head group) pairs, longest context, us a block with 1, 2, 4, 8 shares
ATTENTION = [
    (2, 160, 8, 570, (42.49, 34.91, 31.10, 26.99)), (2, 160, 64, 770, (54.21, 43.27, 38.32, 40.62)),
    (2, 256, 2, 370, (38.33, 34.29, 29.30, 25.21)), (2, 256, 8, 320, (36.28, 32.80, 30.42, 25.55)),
    (2, 256, 8, 570, (46.56, 38.06, 32.97, 28.51)), (2, 256, 64, 370, (42.72, 39.26, 35.21, 37.68)),
    (2, 256, 64, 1570, (96.72, 66.59, 53.37, 58.06)), (2, 256, 8, 4070, (206.10, 116.32, 70.18, 47.32)),
    (4, 160, 8, 570, (58.30, 45.26, 38.53, 33.92)), (4, 256, 64, 770, (97.10, 73.19, 63.36, 71.34)),
    (4, 256, 64, 1570, (171.36, 114.10, 89.77, 97.68)), (4, 128, 8, 4070, (61.67, 45.38, 37.17, 32.85)),
    (4, 128, 64, 370, (36.74, 39.25, 38.95, 44.04)), (4, 128, 64, 770, (39.89, 41.03, 42.09, 45.11)),
    (2, 128, 64, 1570, (36.25, 34.22, 33.99, 36.19)), (2, 128, 16, 2070, (36.51, 32.86, 29.08, 25.35)),
    (2, 64, 32, 2070, (31.89, 30.32, 28.13, 25.19)), (4, 64, 128, 770, (36.43, 39.37, 41.18, 37.04)),
]


def test_attention_split_is_near_the_best_measured(ask):
    got = ask([f"attn {e} {d} {pairs} {longest}" for e, d, pairs, longest, _ in ATTENTION])
    for (split,), case in zip(got, ATTENTION):
        times = dict(zip((1, 2, 4, 8), case[4]))
        assert times[split] <= 1.05 * min(times.values()), (case, split)


def test_attention_split_stays_inside_its_scratch(ask):
    rng = random.Random(1)
    cases = [(rng.choice((2, 4)), 2 * rng.randint(1, 128), int(2 ** rng.uniform(0, 16)), int(2 ** rng.uniform(0, 20)) - 1) for _ in range(2000)]
    for (split,), (e, d, pairs, longest) in zip(ask([f"attn {e} {d} {p} {n}" for e, d, p, n in cases]), cases):
        assert split in (1, 2, 4, 8) and (split == 1 or pairs * split <= 512), (e, d, pairs, longest, split)


# ---------------------------------------------------------------- skinny GEMMs of a decode step
QKV, O, GATEUP, DOWN = 6, 9, 10, 12  # HYP_K_GEMV_*
# rows, K, batch: us a block with QKV in (32-row blocks, waves) to a workgroup, unsplit
QKV_PLANS = [
    (12288, 8192, 1, {(1, 4): 92.5, (1, 8): 91.8, (2, 8): 87.8}), (12288, 8192, 32, {(1, 4): 123.7, (1, 8): 121.1, (2, 8): 112.2}),
    (12288, 4096, 1, {(1, 4): 55.3, (1, 8): 58.2, (2, 8): 54.2}), (12288, 4096, 32, {(1, 4): 84.0, (1, 8): 84.7, (2, 8): 79.1}),
    (9216, 3072, 8, {(1, 4): 47.8, (1, 8): 48.1, (2, 8): 45.8}), (12288, 1024, 8, {(1, 4): 41.6, (1, 8): 42.0, (2, 8): 41.5}),
    (15360, 5120, 32, {(1, 4): 99.0, (1, 8): 99.2, (2, 8): 92.0}), (7168, 5120, 8, {(1, 4): 52.0, (1, 8): 51.8, (2, 8): 56.2}),
    (7168, 5120, 32, {(1, 4): 72.1, (1, 8): 72.4, (2, 8): 78.9}), (6144, 4096, 1, {(1, 4): 47.0, (1, 8): 48.5, (2, 8): 51.1}),
    (6144, 8192, 1, {(1, 4): 63.7, (1, 8): 61.5, (2, 8): 69.7}), (6144, 8192, 32, {(1, 4): 86.0, (1, 8): 84.1, (2, 8): 93.4}),
    (1536, 8192, 8, {(1, 4): 56.0, (1, 8): 53.5, (2, 8): 62.5}), (1536, 512, 8, {(1, 4): 22.6, (1, 8): 22.6, (2, 8): 23.1}),
    (6144, 7168, 16, {(1, 4): 64.4, (1, 8): 63.7, (2, 8): 71.8}), (6144, 2048, 1, {(1, 4): 36.7, (1, 8): 36.8, (2, 8): 38.7}),
]


def test_qkv_plans_are_near_the_best_measured(ask):
    for (fbw, nw, ksplit, tail), (N, K, batch, times) in zip(ask([f"gemv {QKV} {N} {K} {b}" for N, K, b, _ in QKV_PLANS]), QKV_PLANS):
        assert (ksplit, tail) == (1, 1)
        assert times[fbw, nw] <= 1.01 * min(times.values()), (N, K, batch, fbw, nw)


def test_plans_deal_all_of_k_and_all_rows(ask):
    rng = random.Random(2)
    cases = [(rng.choice((QKV, O, GATEUP, DOWN)), 256 * rng.randint(1, 150), 256 * rng.randint(1, 80), rng.randint(1, 32)) for _ in range(3000)]
    built = {QKV: {(1, 4), (1, 8), (2, 8)}, O: {(1, 4), (2, 8)}, GATEUP: {(2, 8)}, DOWN: {(1, 4), (2, 8)}}
    for (fbw, nw, ksplit, tail), (cls, N, K, batch) in zip(ask([f"gemv {c} {n} {k} {b}" for c, n, k, b in cases]), cases):
        assert (fbw, nw) in built[cls], (cls, N, K, batch, fbw, nw)
        assert N % (32 * fbw) == 0 and K // 16 % (nw * ksplit) == 0 and K // 16 // (nw * ksplit) % tail == 0, (cls, N, K, batch)


# ---------------------------------------------------------------- chunks of decode attention
def test_chunks_fill_the_chip_with_whole_rounds(ask):
    got = ask([f"chunk {n} {pairs} {even}" for n, pairs, even, _ in CHUNKS])
    assert [c for c, in got] == [c for *_, c in CHUNKS]
    rng = random.Random(4)
    cases = [(int(2 ** rng.uniform(0, 17.5)), 2 * rng.randint(1, 640)) for _ in range(3000)]
    for (plain,), (even,), (n, pairs) in zip(ask([f"chunk {n} {p} 0" for n, p in cases]), ask([f"chunk {n} {p} 1" for n, p in cases]), cases):
        for c in (plain, even):
            assert c % 128 == 0 and c & (c - 1) == 0 and -(-n // c) <= 64, (n, pairs, c)
        one_to_two = 1024 < pairs * -(-n // 1024) < 2048  # waves of 1024-key chunks: some SIMDs with two
        assert even == (plain // 2 if one_to_two and n <= 64 * 512 else plain), (n, pairs, plain, even)
        assert plain == 1024 or n > 64 * 1024 or pairs * -(-n // (2 * plain)) < 512, (n, pairs, plain)


# room for keys, (request, KV head) pairs, even: keys a chunk
CHUNKS = [(2048, 80, 1, 256), (9216, 80, 1, 1024), (1024, 320, 1, 512), (1025, 320, 1, 1024), (3072, 320, 1, 1024), (3073, 320, 1, 512),
          (6144, 320, 1, 512), (6145, 320, 1, 1024), (4000, 320, 0, 1024), (100, 2, 1, 128), (100000, 2, 1, 2048), (64 * 128, 2, 1, 128)]


# class, rows, K: us of a step of one block (QKV: of the second of two) at batch 8 with that GEMV in one window and in several
WINDOWS = [
    (GATEUP, 8192, 1024, 29.3, 31.4), (GATEUP, 16384, 1024, 37.5, 38.7), (GATEUP, 16896, 1024, 37.3, 36.8), (GATEUP, 32768, 1024, 44.2, 42.8),
    (GATEUP, 16384, 512, 33.6, 35.0), (GATEUP, 24576, 512, 33.6, 33.0), (GATEUP, 49152, 512, 39.9, 37.9), (GATEUP, 20480, 768, 34.9, 34.4),
    (GATEUP, 18432, 1280, 41.1, 40.1), (GATEUP, 57344, 1280, 59.1, 56.7), (QKV, 18432, 512, 36.6, 34.9), (QKV, 24576, 512, 39.6, 37.3),
    (QKV, 18432, 1024, 39.3, 39.7), (QKV, 24576, 1024, 43.4, 43.6), (QKV, 24576, 1280, 47.1, 48.0), (QKV, 36864, 768, 45.4, 45.0),
]


def test_windows_are_near_the_best_measured(ask):
    for (one,), (cls, N, K, in_one, in_several) in zip(ask([f"window {c} {N} {K} 8" for c, N, K, _, _ in WINDOWS]), WINDOWS):
        assert (in_one if one else in_several) <= 1.02 * min(in_one, in_several), (cls, N, K, one)


def test_one_window_stays_with_the_forms_it_is_built_for(ask):
    cases = [(c, N, K, 1) for c in (QKV, O, GATEUP, DOWN) for N in range(256, 65536, 512) for K in range(256, 16384, 256)]
    plans, windows = ask([f"gemv {c} {n} {k} {b}" for c, n, k, b in cases]), ask([f"window {c} {n} {k} {b}" for c, n, k, b in cases])
    seen = {(case[0], fbw, nw) for case, (fbw, nw, _, _), (one,) in zip(cases, plans, windows) if one}
    assert seen == {(QKV, 1, 4), (QKV, 2, 8), (O, 1, 4), (GATEUP, 2, 8), (DOWN, 1, 4)}


# ---------------------------------------------------------------- decode steps, one by one or recorded
# weights of a block, blocks: us of a step launched one by one and replayed: a stage on its own stream, and a step of each of several
# stages that one thread feeds on as many streams (three of 512 and 1024 wide blocks, two Llama3-8B-shaped stages)
STEPS = [
    (4.98e6, 1, (20.4, 25.1), (64.2, 110.5)), (4.98e6, 2, (41.9, 44.3), (104.7, 114.0)), (4.98e6, 3, (66.6, 63.9), (142.8, 119.6)),
    (4.98e6, 4, (84.4, 84.2), (217.0, 120.5)), (4.98e6, 6, (127.8, 127.4), (298.2, 147.4)), (4.98e6, 8, (170.6, 171.0), (416.8, 194.0)),
    (31.5e6, 1, (28.5, 32.8), (65.6, 105.7)), (31.5e6, 2, (58.5, 63.3), (105.1, 112.0)), (31.5e6, 4, (116.4, 120.7), (214.2, 162.8)),
    (31.5e6, 8, (231.0, 234.9), (422.1, 332.4)), (436e6, 1, (85.4, 91.1), (142.7, 151.5)), (436e6, 3, (260.7, 265.9), (439.2, 447.8)),
    (436e6, 8, (695.6, 702.1), (1188.0, 1192.0)),
]


def test_steps_are_launched_one_by_one_only_where_no_thread_is_held_up(ask):
    for (direct,), (_, blocks, alone, several) in zip(ask([f"direct {n} {int(b)}" for b, n, _, _ in STEPS]), STEPS):
        for one_by_one, replayed in (alone, several):
            assert (one_by_one if direct else replayed) <= 1.05 * min(one_by_one, replayed), (blocks, direct)
    assert ask(["direct 9 1000000000", "direct 20 500000000"]) == [[0], [0]]


# ---------------------------------------------------------------- prefill GEMMs
# internal rows, N, K, gate/up: us of the GEMM in tiles of 128 x 64 (as the rule slices them) and in the wide form
FORMS = [
    (576, 1536, 512, 0, 12.8, 27.3), (576, 8192, 2048, 1, 47.2, 42.7), (704, 8192, 1024, 1, 29.1, 27.5), (2016, 3072, 1024, 0, 32.1, 35.2),
    (1600, 4096, 512, 1, 23.4, 20.6), (3520, 2560, 768, 1, 36.0, 24.7), (224, 2048, 2048, 0, 16.6, 20.7), (2720, 1024, 2048, 0, 28.7, 33.7),
    (1312, 4096, 1024, 0, 33.8, 36.5), (576, 4096, 4096, 1, 49.7, 39.5), (1600, 1536, 4096, 0, 46.1, 39.5), (416, 1024, 4096, 0, 18.4, 22.0),
    (2720, 4096, 4096, 1, 144.5, 84.5), (1312, 2560, 1536, 1, 38.8, 43.6), (3520, 512, 1024, 0, 16.2, 31.0), (288, 3072, 2048, 0, 22.2, 24.9),
]


def test_forms_are_near_the_best_measured(ask):
    got = ask([f"gemm {rows} {N} {K} {gu}" for rows, N, K, gu, _, _ in FORMS])
    for (form, *_), (rows, N, K, gu, short, wide) in zip(got, FORMS):
        assert (short if form == 64 else wide) <= 1.05 * min(short, wide), (rows, N, K, gu, form)


# internal rows, N, K: us of the GEMM in tiles of 128 x 64 by its slices
SLICES = [
    (128, 1024, 1792, {1: 20.27, 2: 15.86, 3: 14.10, 4: 13.49}), (128, 3072, 2048, {1: 23.78, 2: 20.17, 3: 17.86, 4: 17.34, 5: 17.89}),
    (96, 1024, 4096, {1: 35.06, 2: 24.06, 4: 16.99, 5: 15.99, 6: 15.01, 8: 14.23, 10: 14.76}), (576, 1024, 1024, {1: 14.53, 2: 15.60}),
    (128, 1536, 5120, {1: 47.05, 3: 25.19, 5: 20.90, 6: 20.01, 8: 19.26, 10: 20.26}), (576, 2048, 4096, {1: 35.55, 2: 31.79, 3: 27.53}),
    (320, 1024, 2048, {1: 21.53, 2: 17.76, 3: 15.79, 4: 15.37, 5: 14.01}), (800, 1024, 2048, {1: 21.40, 2: 18.46, 3: 18.70, 4: 18.18}),
    (320, 4096, 2048, {1: 22.13, 2: 26.04, 3: 24.20}), (800, 2048, 2048, {1: 23.30, 2: 24.57}), (96, 512, 1024, {1: 13.79, 2: 13.01}),
]


def test_slices_are_near_the_best_measured(ask):
    got = ask([f"gemm {rows} {N} {K} 0" for rows, N, K, _ in SLICES])
    for (form, _, _, _, ksplit, *_), (rows, N, K, times) in zip(got, SLICES):
        assert form == 64 and ksplit in times and times[ksplit] <= 1.05 * min(times.values()), (rows, N, K, form, ksplit)


def test_prefill_cuts_stay_inside_grid_and_scratch(ask):
    rng = random.Random(3)
    cases = [(32 * (1 + int(2 ** rng.uniform(0, 11.5))), 256 * rng.randint(1, 140), 256 * rng.randint(1, 72), rng.randint(0, 1)) for _ in range(6000)]
    feats, toks, lds = {64: 128, 128: 128, 256: 256}, {64: 64, 128: 128, 256: 256}, {64: 6, 128: 4, 256: 4}
    for got, (rows, N, K, gu) in zip(ask(["gemm %d %d %d %d" % c for c in cases]), cases):
        form, tiles_t, n_tiles, first, ksplit, finish, n_static, pool, first_grid, rest_grid = got
        where = (rows, N, K, gu, got)
        assert tiles_t == -(-rows // toks[form]) and n_tiles == tiles_t * (N // feats[form]), where
        assert 0 <= first <= n_tiles and (first == n_tiles) == (ksplit == 1), where
        if ksplit > 1:
            assert (n_tiles - first) * ksplit <= 512 and K // 32 // ksplit >= 2 * lds[form], where
            assert rest_grid % 8 == 0 and rest_grid >= (n_tiles - first) * ksplit, where
            assert finish or n_tiles <= 511, where  # arrival counters
        else:
            assert rest_grid == 0, where
        if pool:
            assert first == n_tiles and n_static % 256 == 0 and first_grid == n_static + pool and pool >= 2 * (n_tiles - n_static), where
        else:
            assert first_grid % 8 == 0 and first_grid >= first, where


def test_a_long_request_has_the_cut_of_its_batch(ask):
    # a request that fills two and a half rounds of wide tiles in every GEMM of its block is cut like any batch it is part of:
    # nothing is split (Phi-3 blocks from 7937 rows on: 640 tiles of the O projection)
    shapes = [(7168, 5120, 0), (5120, 5120, 0), (35840, 5120, 1), (5120, 17920, 0)]
    for rows in (7968, 8192, 16384, 65536):
        assert all(got[0] == 256 and got[4] == 1 for got in ask([f"gemm {rows} {N} {K} {gu}" for N, K, gu in shapes])), rows


def test_split_gemm_cases_take_the_paths_they_are_made_for(ask):
    from tests.test_gpu_split_gemms import CASES
    for name, ((hidden, nq, nkv, ffn), lens, paths) in CASES.items():
        rows = -(-sum(lens) // 32) * 32
        gemms = [((nq + 2 * nkv) * 128, hidden, 0), (hidden, nq * 128, 0), (2 * ffn, hidden, 1), (hidden, ffn, 0)]
        for got, path in zip(ask([f"gemm {rows} {N} {K} {gu}" for N, K, gu in gemms]), paths):
            form, _, n_tiles, first, ksplit, finish = got[:6]
            kind = "unsplit" if ksplit == 1 else "short" if form < 256 else "wide" if first == 0 else "rest"
            assert kind == path and finish, (name, path, got)


def test_split_decode_case_is_split(ask):
    # what test_gpu_mfma_parity.py and test_gpu_depth_parity.py say of hidden 5120, FFN 7680
    for batch in (3, 5, 17, 31):
        assert [g[2] for g in ask([f"gemv {GATEUP} 15360 5120 {batch}", f"gemv {DOWN} 5120 7680 {batch}"])] == [2, 3]
