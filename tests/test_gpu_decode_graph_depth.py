"""Decode steps on either side of the depth at which a stage of narrow blocks replays a recorded graph (more than 2): against the oracle over
the forms that attention takes as contexts grow, with two output buffers and a prefill in between (Sec. V-A generation), and
the bits of the same kernels launched one by one."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("blocks", [2, 3, 8, 9])
def test_steps_of_deep_stages(blocks):
    import torch
    from paper_2511_14450_amd import binding
    shape = synth.BlockShape(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")
    # Weights of 0.05, as for the other stages of this width: the update (output - input) is then about as large as the input.  At
    # 0.02 it is 0.07 of it, and the rounding of the bf16 output alone, 2^-9 / sqrt(3) .. 2^-9 of the output, is 0.016 - 0.03 of the update.
    layers = [synth.layer_weights(shape, l, 63_000, sigma=0.05) for l in range(blocks)]
    a, b = (make_gpu_stage(shape, layers, 3, 700, 900, flags=f) for f in (0, binding.HYP_FLAG_NO_GRAPH))
    for lens in ([253, 9, 40], [509, 300], [253, 9, 40]):  # across the changes of form at 256 and 512 keys
        B = len(lens)
        x = synth.hidden_states(sum(lens), shape, 63_001)
        ost = orc.Stage(shape, layers, B, 700, "f32")
        ost.prefill(x, lens)
        for s in (a, b):
            s.prefill(to_dev(x, "bf16"), lens)
        outs = [torch.empty((B, shape.hidden), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        for s in range(7):
            xd = synth.hidden_states(B, shape, 63_002 + s)
            ref = ost.decode_step(xd)
            ya = a.decode_step(to_dev(xd, "bf16"), outs[s % 2]).clone()
            yb = b.decode_step(to_dev(xd, "bf16"))
            got = to_host(ya)
            assert max(rel_err(got, ref), rel_err(got - xd, ref - xd)) <= TOL, (lens, s)
            assert torch.equal(ya, yb), (lens, s)
    a.destroy(); b.destroy()
