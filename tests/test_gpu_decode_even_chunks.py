"""Decode steps of stages whose 1024-key chunks would give between one wave and two per SIMD (320 pairs, room for 3100 keys: 4
chunks a head), which halve them, and of one that does not because its temporaries would outgrow the static array: contexts that
end a block short of a chunk, with it and behind it, against the oracle (Sec. III-A attention); the same bits without allocation."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


# an FFN of 83968 features takes 25.6 MiB of the 32 MiB for partial sums and activations: with 4 chunks a head the rest fits, with 7 it does not
@pytest.mark.parametrize("ffn,lens", [(256, [511, 510, 479, 480, 542, 543, 1023, 1055]), (83968, [511, 30])])
def test_steps_across_chunks(ffn, lens):
    import torch
    shape = synth.BlockShape(hidden=256, n_q_heads=40, n_kv_heads=10, head_dim=128, ffn_dim=ffn, dtype="bf16")
    layers = [synth.layer_weights(shape, 0, 62_000, sigma=0.02)]
    lens = lens + [1 + b for b in range(32 - len(lens))]
    B, T, cap = len(lens), sum(lens), 3100
    x = synth.hidden_states(T, shape, 62_001)
    ost = orc.Stage(shape, layers, B, cap, "f32")
    ost.prefill(x, lens)
    st, same = (make_gpu_stage(shape, layers, B, cap, T) for _ in range(2))
    for s in (st, same):
        s.prefill(to_dev(x, "bf16"), lens)
    for s in range(3):
        xd = synth.hidden_states(B, shape, 62_002 + s)
        r = ost.decode_step(xd)
        hid = to_dev(xd, "bf16")
        out, out2 = torch.empty_like(hid), torch.empty_like(hid)
        st.decode_step(hid, out)
        same.decode_step_noalloc(hid, out2)
        y = to_host(out)
        assert max(rel_err(y, r), rel_err(y - xd, r - xd)) <= TOL, s
        assert torch.equal(out, out2), s
    st.destroy(); same.destroy()
