"""Prefill GEMMs of at most 128 internal rows (their forms of 64 and 128 tokens): row counts around the change of form,
widths whose tiles are split along K, left whole, and split beyond the first 256 only, against the oracle
(Sec. III-A block; Sec. V-A uses 64-token prompts)."""
import numpy as np
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


# ffn 256: 4 tiles of 128 gate/up rows; 2560: 40, K of the down projection splits; 17408: 272 tiles, 16 beyond the first 256
@pytest.mark.parametrize("ffn", [256, 2560, 17408])
@pytest.mark.parametrize("lens", [[64], [1], [63, 64], [128], [129], [65, 1]])
def test_short_prompts_against_oracle(lens, ffn):
    shape = synth.BlockShape(hidden=512, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=ffn, dtype="bf16")
    n_layers = 1 if ffn > 10000 else 2
    layers = [synth.layer_weights(shape, l, 43_000, sigma=0.05) for l in range(n_layers)]
    B, T = len(lens), sum(lens)
    x = synth.hidden_states(T, shape, 43_001)
    ost, gst = orc.Stage(shape, layers, B, max(lens) + 2, "f32"), make_gpu_stage(shape, layers, B, max(lens) + 2, T)
    for _ in range(2):  # the arrival counters of the first call must be clear for the second
        ref, got = ost.prefill(x, lens), to_host(gst.prefill(to_dev(x, "bf16"), lens))
        assert max(rel_err(got, ref), rel_err(got - x, ref - x)) <= TOL
    for b in range(B):
        k, v = gst.export_kv(n_layers - 1, b)
        assert rel_err(to_host(k), ost.K[n_layers - 1, b, :lens[b]]) <= TOL
        assert rel_err(to_host(v), ost.V[n_layers - 1, b, :lens[b]]) <= TOL
    gst.destroy()
