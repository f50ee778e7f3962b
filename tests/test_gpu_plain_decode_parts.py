"""Generic decode attention whose heads are dealt to several workgroups by value features: on both sides of the batch at which
every workgroup has a CU of its own (128 pairs of 64 features in two parts, 64 of 128 in four), with two column groups of query
heads, one key to a request and more than a round of blocks.  Against the oracle (Sec. III-A block)."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch,heads,kv,d", [(64, 4, 2, 64), (65, 4, 2, 64), (64, 1, 1, 128), (65, 1, 1, 128), (2, 6, 1, 128), (3, 5, 1, 64)])
def test_parts_of_value_features_against_oracle(batch, heads, kv, d, dtype):
    from paper_2511_14450_amd import binding
    shp = synth.BlockShape(64, heads, kv, d, 96, dtype=dtype)
    lens = [1 + (b * 29) % 40 for b in range(batch)]
    lens[0], lens[-1] = 1, 16 * 8 + 15
    layers = [synth.layer_weights(shp, 0, 59_000, sigma=0.1)]
    x = synth.hidden_states(sum(lens), shp, 59_001)
    ost = orc.Stage(shp, layers, batch, max(lens) + 2, "f32")
    gst = make_gpu_stage(shp, layers, batch, max(lens) + 2, sum(lens), flags=binding.HYP_FLAG_PLAIN_KERNELS)
    ost.prefill(x, lens)
    gst.prefill(to_dev(x, dtype), lens)
    for s in range(2):
        xd = synth.hidden_states(batch, shp, 59_002 + s)
        got, ref = to_host(gst.decode_step(to_dev(xd, dtype))), ost.decode_step(xd)
        assert rel_err(got, ref) <= TOL[dtype], f"step {s}"
    gst.destroy()
