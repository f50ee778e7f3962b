"""Decode steps whose attention over short contexts reads the O projection's weights into L2 with workgroups of its own (stages
with an O projection of 16 MiB and more): whole row groups and the first part of them, one request and as many as there are, both
short forms and the change between them; against the oracle (Sec. III-A block), and the bits of a step that the caller records,
which does not read ahead."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


# O projections of 16 MiB (128 row groups of 128 KiB, read whole) and 40 MiB (128 groups of 320 KiB, 224 of them read)
@pytest.mark.parametrize("heads,kv,lens", [(16, 4, [255]), (16, 4, [3, 300, 510]), (16, 4, [5 + b for b in range(32)]), (40, 10, [254, 9])])
def test_steps_that_read_ahead(heads, kv, lens):
    import torch
    shape = synth.BlockShape(hidden=4096, n_q_heads=heads, n_kv_heads=kv, head_dim=128, ffn_dim=256, dtype="bf16")
    layers = [synth.layer_weights(shape, 0, 61_000, sigma=0.02)]
    B, T, cap = len(lens), sum(lens), 600
    x = synth.hidden_states(T, shape, 61_001)
    ost = orc.Stage(shape, layers, B, cap, "f32")
    ost.prefill(x, lens)
    xd = [synth.hidden_states(B, shape, 61_002 + s) for s in range(4)]
    ref = [ost.decode_step(d) for d in xd]
    got = []
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for recorded in (False, True):
            st = make_gpu_stage(shape, layers, B, cap, T)
            st.prefill(to_dev(x, "bf16"), lens)
            hid = to_dev(xd[0], "bf16")
            out = torch.empty_like(hid)
            stream.synchronize()
            if recorded:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=stream):
                    st.decode_step_noalloc(hid, out)
            for d in xd:
                hid.copy_(to_dev(d, "bf16"))
                if recorded:
                    graph.replay()
                else:
                    st.decode_step(hid, out)
                got.append(out.clone())
            stream.synchronize()
            st.destroy()
    for s, r in enumerate(ref):
        y = to_host(got[s])
        assert max(rel_err(y, r), rel_err(y - xd[s], r - xd[s])) <= TOL, s
        assert torch.equal(got[s], got[len(xd) + s]), s
