"""The device's conversion of float32 to bf16 against round-to-nearest-even on the bit patterns: a stage whose attention adds one
known product to each element of its input, so that the element it stores is the rounding of a known float32 - ties of either
parity, neighbours of ties, carries into the next power of two, cancellations."""
import numpy as np
import pytest

from workloads import synth
from tests.helpers import make_gpu_stage, to_dev, to_host

pytestmark = pytest.mark.gpu


def nearest_even(a):
    """bf16 value of every float32 of `a`, in integers"""
    u = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("plain", [False, True])
def test_stored_elements_are_rounded_to_nearest_even(plain):
    from paper_2511_14450_amd import binding
    H, d, batch = 512, 128, 9
    shape = synth.BlockShape(hidden=H, n_q_heads=4, n_kv_heads=2, head_dim=d, ffn_dim=256, rms_eps=0.0, dtype="bf16")
    rng = np.random.default_rng(7)
    # queries and keys are zero, so attention averages equal values: value feature j of a token is v[j] x[0], with x[0] = 1, and
    # the output projection adds w[i] v[i % d] to element i.  The rows are +-1: their RMS Norm is the identity.
    v = np.where(rng.random(d) < 0.5, 2.0 ** rng.integers(-4, 4, d), nearest_even(rng.uniform(0.5, 2.0, d))).astype(np.float32)
    unit = v[np.arange(H) % d]
    w = nearest_even(rng.standard_normal(H) * 2.0 ** rng.integers(-10, 3, H))
    exact = np.log2(unit) % 1 == 0
    ties = (2 * rng.integers(-300, 300, H) + 1) * 2.0 ** -8  # half a unit of 1.0: odd multiples, some past the next power of two
    w = np.where(exact & (np.abs(ties) < 1), nearest_even(ties / unit), w).astype(np.float32)
    near = exact & (rng.random(H) < 0.3)
    w = np.where(near, nearest_even(w * (1 + 2.0 ** -7)), w)  # a little beyond
    layers = [{"attn_norm_g": np.ones(H), "ffn_norm_g": np.ones(H), "wq": np.zeros((4 * d, H)), "wk": np.zeros((2 * d, H)),
               "wv": np.zeros((2 * d, H)), "wo": np.zeros((H, 4 * d)), "w_gate": np.zeros((256, H)), "w_up": np.zeros((256, H)),
               "w_down": np.zeros((H, 256))}]
    layers = [{k: a.astype(np.float32) for k, a in l.items()} for l in layers]
    layers[0]["wv"][:d, 0] = v
    layers[0]["wo"][np.arange(H), np.arange(H) % d] = w
    gst = make_gpu_stage(shape, layers, batch, 8, batch, flags=binding.HYP_FLAG_PLAIN_KERNELS if plain else 0)
    assert gst.uses_mfma() != plain
    seen = 0
    for step in range(4):
        x = rng.choice(np.float32([-1, 1]), (batch, H))
        x[:, 0] = 1
        got = to_host(gst.prefill(to_dev(x, "bf16"), [1] * batch) if step == 0 else gst.decode_step(to_dev(x, "bf16")))
        sums = (x + (w * unit)[None]).astype(np.float32)
        seen += int(((sums.view(np.uint32) & 0xffff) == 0x8000).sum())
        assert np.array_equal(got.view(np.uint32), nearest_even(sums).view(np.uint32)), step
    assert seen > 1000  # ties
    gst.destroy()


def test_nan_stays_nan():
    """Through the generic kernels with all projections zero, whose bf16 stores must not turn a NaN into a number or infinity."""
    import torch
    from paper_2511_14450_amd import binding
    shape = synth.BlockShape(hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=32, ffn_dim=32, dtype="bf16")
    layers = [{k: np.zeros_like(a) if k.startswith("w") else a for k, a in synth.layer_weights(shape, 0, 61).items()}]
    gst = make_gpu_stage(shape, layers, 3, 4, 3, flags=binding.HYP_FLAG_PLAIN_KERNELS)
    x = synth.hidden_states(3, shape, 62)
    for call in (lambda h: gst.prefill(h, [1, 1, 1]), gst.decode_step):
        h = to_dev(x, "bf16")
        h[1, 5] = torch.nan
        got = to_host(call(h))
        assert np.isnan(got[1]).all() and np.array_equal(got[[0, 2]], x[[0, 2]])
    gst.destroy()
