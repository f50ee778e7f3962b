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
