"""Prefill rows packed without padding between requests: requests that start and end anywhere inside the 16 / 32 / 64-row
tiles against the oracle; values that an earlier prefill left behind a shorter request's end stay out of its results (Sec. III-A block, ragged batches)."""
import numpy as np
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("lens", [[1, 1, 1], [33, 31, 64, 1, 95], [5] * 27, [127, 3, 129, 65, 63], [300, 17, 40, 211]])
@pytest.mark.parametrize("G", [2, 3])
def test_ragged_batches_against_oracle(lens, paged, G):
    from paper_2511_14450_amd import binding
    shape = synth.BlockShape(hidden=256, n_q_heads=2 * G, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")
    layers = [synth.layer_weights(shape, l, 44_000, sigma=0.05) for l in range(2)]
    B, T, cap = len(lens), sum(lens), max(lens) + 3
    x = synth.hidden_states(T, shape, 44_001)
    ost = orc.Stage(shape, layers, B, cap, "f32")
    gst = make_gpu_stage(shape, layers, B, cap, T, flags=binding.HYP_FLAG_PAGED_KV if paged else 0)
    assert gst.uses_mfma()
    for _ in range(2):
        ref, got = ost.prefill(x, lens), to_host(gst.prefill(to_dev(x, "bf16"), lens))
        assert max(rel_err(got, ref), rel_err(got - x, ref - x)) <= TOL
    for s in range(3):
        xd = synth.hidden_states(B, shape, 44_002 + s)
        ref, got = ost.decode_step(xd), to_host(gst.decode_step(to_dev(xd, "bf16")))
        assert max(rel_err(got, ref), rel_err(got - xd, ref - xd)) <= TOL, s
    gst.destroy()


# (prompts after the longer one, decode steps): inside the last 64 keys of a prompt; a prompt that ends on their edge, so that
# the first step opens a block; steps across it; contexts of the chunked form (its last block, over two edges), alone and mixed
@pytest.mark.parametrize("lens,steps", [([31, 40], 4), ([64, 1], 2), ([31, 62], 40), ([640, 574], 70), ([600, 64], 3)])
@pytest.mark.parametrize("paged", [False, True])
def test_what_an_earlier_prefill_left_stays_out(lens, steps, paged):
    import torch
    from paper_2511_14450_amd import binding
    shape = synth.BlockShape(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")
    layers = [synth.layer_weights(shape, l, 45_000, sigma=0.05) for l in range(2)]
    longer, cap = [max(lens) + 120] * 2, max(lens) + 121
    x = synth.hidden_states(sum(longer), shape, 45_001)
    bad = x.copy()
    bad[30:] = np.nan
    flags = binding.HYP_FLAG_PAGED_KV if paged else 0
    used, fresh = (make_gpu_stage(shape, layers, 2, cap, sum(longer), flags=flags) for _ in range(2))
    used.prefill(to_dev(bad, "bf16"), longer)  # the caches hold NaN from key 30 on, and so does every scratch row
    xs = to_dev(x[:sum(lens)], "bf16")
    a, b = used.prefill(xs, lens), fresh.prefill(xs, lens)
    assert torch.equal(a, b) and bool(torch.isfinite(a).all())
    for s in range(steps):
        d = to_dev(synth.hidden_states(2, shape, 45_002 + s), "bf16")
        a, b = used.decode_step(d), fresh.decode_step(d)
        assert torch.equal(a, b) and bool(torch.isfinite(a).all()), s
    used.destroy(); fresh.destroy()
