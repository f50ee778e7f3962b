"""Decode GEMVs on both sides of the number of workgroups up to which all tiles of a wave are requested in one window (256 of eight
waves), with fewer tiles than one of several windows holds, with one more and with two windows full: against the oracle (Sec. III-A block)."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


# gate/up of 256 and 264 workgroups, K = 256 (2 tiles a wave), 768 (6) and 1280 (10); QKV of 256 and 264 with 4 tiles a wave
@pytest.mark.parametrize("hidden,heads,kv,ffn", [(256, 4, 2, 8192), (256, 4, 2, 8448), (768, 4, 2, 8448), (1280, 4, 2, 8192), (1280, 4, 2, 8448),
                                                 (512, 64, 32, 256), (512, 88, 22, 256)])
def test_one_window_and_several(hidden, heads, kv, ffn):
    shape = synth.BlockShape(hidden=hidden, n_q_heads=heads, n_kv_heads=kv, head_dim=128, ffn_dim=ffn, dtype="bf16")
    # updates as large as those of weights N(0, 0.02^2) at hidden size 5120
    layers = [synth.layer_weights(shape, l, 65_000, sigma=0.02 * (5120 / hidden) ** 0.5) for l in range(2)]
    lens = [1, 30, 7]
    x = synth.hidden_states(sum(lens), shape, 65_001)
    ost, st = orc.Stage(shape, layers, 3, 40, "f32"), make_gpu_stage(shape, layers, 3, 40, sum(lens))
    ost.prefill(x, lens)
    st.prefill(to_dev(x, "bf16"), lens)
    for s in range(2):
        xd = synth.hidden_states(3, shape, 65_002 + s)
        got, ref = to_host(st.decode_step(to_dev(xd, "bf16"))), ost.decode_step(xd)
        assert max(rel_err(got, ref), rel_err(got - xd, ref - xd)) <= TOL, s
    st.destroy()
