"""Which form a prefill contraction of a generic stage takes (csrc/launch_rules.h): near the best of what was measured, on the host; and
the forms against the oracle at the edges of their tiles, on the device (the wide ones with every epilogue: test_gpu_plain_kernels.py)."""
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host
from tests.test_gpu_plain_kernels import WIDE_FORMS, WIDE_LENS, WIDE_SHAPES

ROOT = pathlib.Path(__file__).resolve().parents[1]
REGISTERS, SMALL, WIDE, MANY = range(4)
QKV, GATEUP, O, DOWN = range(4)
ASK = """#include <stdio.h>
#include "launch_rules.h"
int main() {
  int e, rows, N, K, epi;
  while (scanf("%d %d %d %d %d", &e, &rows, &N, &K, &epi) == 5) printf("%d\\n", hyp::plain_gemm_form(e, rows, N, K, epi == 0, epi == 1));
}
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = tmp_path_factory.mktemp("forms") / "ask"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2511_14450_amd/csrc'}",
                        "-x", "c++", "-", "-o", str(exe)], input=ASK, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def ask(cases):
        r = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True)
        return [int(v) for v in r.stdout.split()]
    return ask


# bytes an element, rows, N, K, contraction: us in 32 x 32 from registers, 64 x 64, 128 x 128 and, bf16, 128 x 128 in four waves
MEASURED = [
    (4, 800, 1024, 4096, DOWN, (89.3, 81.9, 252.3)), (4, 800, 1024, 1024, O, (27.0, 25.1, 71.3)), (4, 3800, 256, 488, QKV, (19.6, 18.2, 44.7)),
    (4, 400, 3072, 624, QKV, (27.0, 34.6, 53.6)), (4, 800, 2048, 1024, QKV, (47.0, 51.2, 78.8)), (4, 3800, 488, 1624, DOWN, (77.4, 75.4, 112.4)),
    (4, 2800, 816, 1448, DOWN, (82.5, 96.3, 104.1)), (4, 600, 5008, 792, GATEUP, (62.7, 68.3, 55.4)), (4, 2000, 2304, 2048, QKV, (203.4, 199.7, 268.0)),
    (4, 800, 8192, 1024, GATEUP, (164.7, 153.2, 143.5)), (4, 4000, 5120, 2560, O, (1076.8, 1056.6, 820.8)), (4, 400, 888, 3904, DOWN, (43.7, 78.1, 240.4)),
    (2, 800, 1152, 2592, DOWN, (18.4, 13.7, 39.0, 35.7)), (2, 1000, 1024, 4096, DOWN, (26.3, 17.2, 35.1, 47.1)), (2, 600, 904, 3960, DOWN, (26.5, 17.9, 33.0, 48.9)),
    (2, 600, 1920, 696, QKV, (13.3, 14.3, 21.9, 27.9)), (2, 1000, 1536, 1024, QKV, (17.8, 16.2, 22.7, 31.2)), (2, 400, 1000, 1480, DOWN, (7.3, 9.0, 18.7, 24.6)),
    (2, 600, 4256, 696, GATEUP, (19.3, 15.6, 11.8, 15.7)), (2, 1000, 8192, 1024, GATEUP, (57.1, 37.5, 23.4, 25.5)), (2, 2000, 2304, 2048, QKV, (65.9, 50.6, 56.4, 55.2)),
    (2, 4600, 4192, 664, GATEUP, (115.4, 67.6, 45.3, 42.0)), (2, 4000, 5120, 3200, O, (386.5, 225.3, 167.6, 179.0)), (2, 4000, 17920, 5120, GATEUP, (3025.9, 1633.7, 862.1, 879.2)),
]


def test_forms_are_near_the_best_measured(form):
    for got, (*case, times) in zip(form([c[:5] for c in MEASURED]), MEASURED):
        assert times[got] <= 1.12 * min(times), (case, got)


# hidden, query and KV heads, head size, FFN width; rows of two prompts; the forms of QKV, gate/up, O, down.  Rows, features and K
# off the tiles of 16 and 64 bytes, fewer tiles along K than stages in LDS, odd and even numbers of stages, one tile along K.
CASES = {
    "f32_small": ("f32", (1000, 15, 1, 66, 2100), (601, 270), (SMALL, WIDE, SMALL, SMALL)),
    "f32_small_many": ("f32", (180, 4, 2, 90, 7800), (500, 33), (REGISTERS, SMALL, REGISTERS, REGISTERS)),
    "f32_wide": ("f32", (180, 4, 2, 90, 5600), (500, 33), (REGISTERS, WIDE, REGISTERS, REGISTERS)),
    "f32_wide_k_of_a_tile": ("f32", (16, 2, 1, 8, 20000), (700, 111), (REGISTERS, WIDE, REGISTERS, REGISTERS)),
    "bf16_small": ("bf16", (1000, 14, 2, 66, 1100), (601, 270), (REGISTERS, SMALL, SMALL, SMALL)),
    "bf16_wide": ("bf16", (340, 4, 2, 90, 5600), (500, 33), (REGISTERS, WIDE, REGISTERS, REGISTERS)),
    "bf16_many": ("bf16", (520, 30, 2, 66, 6000), (1100, 33), (WIDE, MANY, SMALL, SMALL)),
    "bf16_many_k_of_a_tile": ("bf16", (24, 2, 1, 8, 9000), (1100, 33), (REGISTERS, MANY, REGISTERS, REGISTERS)),
}


def test_cases_take_the_forms_they_are_made_for(form):
    for name, (dtype, (H, nq, nkv, d, I), lens, forms) in CASES.items():
        e, rows = 4 if dtype == "f32" else 2, sum(lens)
        gemms = [((nq + 2 * nkv) * d, H), (2 * I, H), (H, nq * d), (H, I)]
        assert tuple(form([(e, rows, N, K, epi) for epi, (N, K) in enumerate(gemms)])) == forms, name


def test_wide_projections_take_the_forms_they_are_made_for(form):
    for (shape, dtype), forms in WIDE_FORMS.items():
        b, e, rows = WIDE_SHAPES[shape], 4 if dtype == "f32" else 2, sum(WIDE_LENS)
        H, q, kv, I = b["hidden"], b["n_q_heads"] * b["head_dim"], b["n_kv_heads"] * b["head_dim"], b["ffn_dim"]
        got = form([(e, rows, N, K, epi) for epi, (N, K) in enumerate([(q + 2 * kv, H), (2 * I, H), (H, q), (H, I)])])
        assert [("registers", "small", "wide", "many")[f] for f in got] == forms.split(), (shape, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("case", list(CASES))
def test_forms_against_oracle(case):
    from paper_2511_14450_amd import binding
    dtype, (H, nq, nkv, d, I), lens, _ = CASES[case]
    shape = synth.BlockShape(hidden=H, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn_dim=I, dtype=dtype)
    tol, T, B = 1e-4 if dtype == "f32" else 2e-2, sum(lens), len(lens)
    w = synth.layer_weights(shape, 0, 57_000, sigma=0.02 * (5120 / H) ** 0.5)
    x = synth.hidden_states(T, shape, 57_001)
    ost, gst = orc.Stage(shape, [w], B, max(lens), "f32"), make_gpu_stage(shape, [w], B, max(lens), T, flags=binding.HYP_FLAG_PLAIN_KERNELS)
    got, ref = to_host(gst.prefill(to_dev(x, dtype), list(lens))), ost.prefill(x, list(lens))
    # storing the output in bf16 costs the update half a unit in the last place of the output
    store = 2.0 ** -8 * np.abs(ref).max() / np.abs(ref - x).max() if dtype == "bf16" else 0.0
    assert rel_err(got, ref) <= tol and rel_err(got - x, ref - x) <= tol + store
    for b in range(B):
        k, v = gst.export_kv(0, b)
        assert rel_err(to_host(k), ost.K[0, b, :lens[b]]) <= tol
        assert rel_err(to_host(v), ost.V[0, b, :lens[b]]) <= tol
    gst.destroy()
