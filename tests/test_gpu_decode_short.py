"""Decode attention of contexts up to 512 keys: contexts around the edges of its block counts (32 keys a wave, 256 keys a
round of waves) and across the change to the chunked form, against the oracle (Sec. III-A attention, Sec. V-A generation);
a step recorded by the caller and replayed beyond those edges, and steps called directly after such replays; the bits
of a step, which do not depend on how it is launched."""
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


class LateKeys:
    """One block without its feed-forward part, driven so that the newest keys decide the result: prompt tokens lie around
    -b, step tokens around b and from position 512 on around c, for fixed vectors b and c, so that the average of the values
    turns as steps are added.  (The norm takes the inputs' scale away; small ones keep bf16's rounding of the sum small.)"""
    SHAPE = synth.BlockShape(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")

    def __init__(self, seed):
        self.seed = seed
        w = synth.layer_weights(self.SHAPE, 0, seed, sigma=0.05)
        w["w_down"] = np.zeros_like(w["w_down"])
        self.layers = [w]
        self.b, self.c = 2 * synth.normal((2, self.SHAPE.hidden), seed, tag=77)

    def prompt(self, rows):
        return synth.round_bf16((synth.normal((rows, self.SHAPE.hidden), self.seed + 1) - self.b) / 4)

    def step(self, pos, batch):
        towards = self.b if pos < 512 else self.c
        return synth.round_bf16((synth.normal((batch, self.SHAPE.hidden), self.seed + 2 + pos) + towards) / 4)


def err_without_late_keys(ost, x, ref, keys):
    """Error of the update where request 0's step sees its first `keys` keys only."""
    part = orc.Stage(LateKeys.SHAPE, ost.layers_np, 1, ost.cap, "f32")
    part.K[:, 0], part.V[:, 0], part.lens = ost.K[:, 0], ost.V[:, 0], np.array([keys - 1], np.int32)
    return rel_err(part.decode_step(x[:1]) - x[:1], ref[:1] - x[:1])


# (prompt, replays): the host last saw up to 256 keys and the device holds up to 512; ... up to 512, and beyond
@pytest.mark.parametrize("prompt,replays", [(200, 120), (400, 300), (100, 600)])
@pytest.mark.parametrize("entry", ["decode_step", "decode_step_noalloc"])
def test_recorded_steps_replayed_past_the_short_form_and_direct_steps_after_them(prompt, replays, entry):
    import torch
    late, lens, cap = LateKeys(42_000), [prompt, 5], 900
    ost = orc.Stage(late.SHAPE, late.layers, 2, cap, "f32")
    ost.layers_np = late.layers
    x = late.prompt(sum(lens))
    ost.prefill(x, lens)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = make_gpu_stage(late.SHAPE, late.layers, 2, cap, sum(lens))
        st.prefill(to_dev(x, "bf16"), lens)
        hid = torch.empty((2, late.SHAPE.hidden), dtype=torch.bfloat16, device="cuda")
        out = torch.empty_like(hid)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            st.decode_step_noalloc(hid, out)
        for s in range(replays + 3):
            xd = late.step(prompt + s, 2)
            ref = ost.decode_step(xd)
            hid.copy_(to_dev(xd, "bf16"))
            if s < replays:
                graph.replay()
            elif entry == "decode_step":
                st.decode_step(hid, out)
            else:
                st.decode_step_noalloc(hid, out)
            if s < replays and s % 20 and prompt + s not in range(500, 520):
                continue
            got = to_host(out)
            assert rel_err(got - xd, ref - xd) <= TOL, s
            for keys in (256, 512):  # a form that ends there would show: 0.087 and more, 20 step tokens past the edge
                if prompt + s >= max(keys, prompt) + 20:
                    assert err_without_late_keys(ost, xd, ref, keys) > 4 * TOL, (s, keys)
    st.destroy()


def test_a_recorded_step_gives_the_bits_of_a_direct_one():
    import torch
    shape = synth.BlockShape(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=512, dtype="bf16")
    layers = [synth.layer_weights(shape, 0, 42_100, sigma=0.05)]
    lens, cap = [508, 40, 250, 700], 900
    x = to_dev(synth.hidden_states(sum(lens), shape, 42_101), "bf16")
    xd = [to_dev(synth.hidden_states(4, shape, 42_102 + s), "bf16") for s in range(12)]
    for some in ([0, 1, 2, 3], [0, 1, 2], [1, 2], [3]):  # long and short contexts; across the change of form; short; long
        ln = [lens[r] for r in some]
        at = [sum(lens[:r]) for r in some]
        xs = torch.cat([x[a:a + n] for a, n in zip(at, ln)])
        direct = make_gpu_stage(shape, layers, 4, cap, sum(lens))
        direct.prefill(xs, ln)
        want = [direct.decode_step(d[some].contiguous()).clone() for d in xd]
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            rec = make_gpu_stage(shape, layers, 4, cap, sum(lens))
            rec.prefill(xs, ln)
            hid, out = xd[0][some].contiguous(), torch.empty_like(xd[0][some])
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                rec.decode_step_noalloc(hid, out)
            for s, d in enumerate(xd):
                hid.copy_(d[some])
                graph.replay()
                stream.synchronize()
                assert torch.equal(out, want[s]), (some, s)
        direct.destroy(); rec.destroy()
