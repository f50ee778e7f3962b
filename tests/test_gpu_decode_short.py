"""Decode attention in one workgroup per (request, KV head): contexts around the edges of its block counts (32 keys a
wave, 256 and 512 keys a workgroup) and across the change to the chunked form, against the oracle (Sec. III-A
attention, Sec. V-A generation); a step recorded by the caller and replayed beyond those edges."""
import numpy as np
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("G", [1, 3, 4])
@pytest.mark.parametrize("lens", [[31, 1, 224], [255, 64], [511, 256, 509]])
def test_short_contexts_against_oracle(lens, G):
    shape = synth.BlockShape(hidden=256, n_q_heads=2 * G, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")
    layers = [synth.layer_weights(shape, l, 41_000, sigma=0.05) for l in range(2)]
    B, cap = len(lens), max(lens) + 600
    x = synth.hidden_states(sum(lens), shape, 41_001)
    ost, gst = orc.Stage(shape, layers, B, cap, "f32"), make_gpu_stage(shape, layers, B, cap, sum(lens))
    assert gst.uses_mfma()
    ost.prefill(x, lens)
    gst.prefill(to_dev(x, "bf16"), lens)
    for s in range(4):
        xd = synth.hidden_states(B, shape, 41_002 + s)
        ref, got = ost.decode_step(xd), to_host(gst.decode_step(to_dev(xd, "bf16")))
        assert max(rel_err(got, ref), rel_err(got - xd, ref - xd)) <= TOL, s
    gst.destroy()


def test_a_recorded_step_replayed_past_the_short_form():
    # the caller records one step at 508 cached keys and replays it to 520: as the steps launched one by one
    import torch
    shape = synth.BlockShape(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")
    layers = [synth.layer_weights(shape, 0, 42_000, sigma=0.05)]
    lens, cap = [508, 40], 900
    x = to_dev(synth.hidden_states(sum(lens), shape, 42_001), "bf16")
    xd = [to_dev(synth.hidden_states(2, shape, 42_002 + s), "bf16") for s in range(12)]
    eager = make_gpu_stage(shape, layers, 2, cap, sum(lens))
    eager.prefill(x, lens)
    want = [to_host(eager.decode_step(d)) for d in xd]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        rec = make_gpu_stage(shape, layers, 2, cap, sum(lens))
        rec.prefill(x, lens)
        hid, out = xd[0].clone(), torch.empty_like(xd[0])
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            rec.decode_step_noalloc(hid, out)
        for s, d in enumerate(xd):
            hid.copy_(d)
            graph.replay()
            stream.synchronize()
            got = to_host(out)
            assert rel_err(got, want[s]) <= TOL, s
    eager.destroy(); rec.destroy()
