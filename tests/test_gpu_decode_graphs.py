"""Recorded decode steps (Sec. V-A generation): a program that cycles through several output buffers and context lengths
finds its recordings again instead of making them anew on every step."""
import time

import pytest

from workloads import synth
from tests.helpers import make_gpu_stage, to_dev

pytestmark = pytest.mark.gpu


def test_four_output_buffers_over_short_and_long_contexts_are_recorded_once():
    import torch
    shape = synth.BlockShape(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=256, dtype="bf16")
    layer = synth.layer_weights(shape, 0, 46_000, sigma=0.02)
    st = make_gpu_stage(shape, [layer] * 40, 2, 1000, 1300)  # 200 kernels a step: a recording costs many replays
    x = to_dev(synth.hidden_states(1300, shape, 46_001), "bf16")
    xd = to_dev(synth.hidden_states(2, shape, 46_002), "bf16")
    outs = [torch.empty_like(xd) for _ in range(4)]
    host = []
    for visit in range(4):
        for lens in ([100, 90], [300, 90], [600, 90]):  # every form of attention
            st.prefill(x[:sum(lens)].contiguous(), lens)
            for o in outs:
                torch.cuda.synchronize()
                t = time.perf_counter()
                st.decode_step(xd, o)
                host.append((visit, time.perf_counter() - t))
    torch.cuda.synchronize()
    def median(v):
        return sorted(v)[len(v) // 2]
    first, later = median([t for v, t in host if v == 0]), median([t for v, t in host if v > 0])
    print(f"host time of a step: {first * 1e6:.0f} us recording, {later * 1e6:.0f} us replaying")
    assert later < first / 2
    st.destroy()
