"""Prefill GEMMs of more than 128 rows whose K loop is split: all tiles of a small grid, or the ones beyond the last whole round
of 256 (gate/up of three token tiles: 264 tiles), in slices of unequal length, added up by the second kernel with every
epilogue, against the oracle (Sec. III-A block)."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("lens", [[600, 1], [129], [250, 7]])
def test_split_gemms_against_oracle(lens):
    shape = synth.BlockShape(hidden=1024, n_q_heads=14, n_kv_heads=14, head_dim=128, ffn_dim=11264, dtype="bf16")
    layers = [synth.layer_weights(shape, l, 53_000, sigma=0.04) for l in range(2)]
    B, T = len(lens), sum(lens)
    x = synth.hidden_states(T, shape, 53_001)
    ost, gst = orc.Stage(shape, layers, B, max(lens), "f32"), make_gpu_stage(shape, layers, B, max(lens), T)
    ref, first = ost.prefill(x, lens), to_host(gst.prefill(to_dev(x, "bf16"), lens))
    assert max(rel_err(first, ref), rel_err(first - x, ref - x)) <= TOL
    for b in range(B):
        k, v = gst.export_kv(1, b)
        assert rel_err(to_host(k), ost.K[1, b, :lens[b]]) <= TOL
        assert rel_err(to_host(v), ost.V[1, b, :lens[b]]) <= TOL
    assert (to_host(gst.prefill(to_dev(x, "bf16"), lens)) == first).all()  # the scratch of the call before leaves no trace
    gst.destroy()
