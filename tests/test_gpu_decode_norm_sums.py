"""The sums of squares that a decode step's residual epilogues leave for the next RMS Norm, bit for bit: a butterfly over the lanes of
a row group, the first addition fused with a lane's own square.  Block 0's projections are chosen so that what its residual
kernels add up is known exactly (two keys of equal weight, one product to a feature, an FFN of zeros), block 1's values so that they
show the norm factor; both are followed in float32 on the host (Sec. III-A block)."""
import numpy as np
import pytest

from workloads import synth
from tests.helpers import make_gpu_stage, to_dev, to_host

pytestmark = pytest.mark.gpu
F = np.float32
H, HEADS, KV, B, EPS, ROUNDS = 256, 32, 16, 32, 1e-5, 64


def picked(n_out, n_in, rng):
    """one product to an output: column n % n_in of row n, values of 8 bits"""
    w = np.zeros((n_out, n_in), F)
    w[np.arange(n_out), np.arange(n_out) % n_in] = synth.round_bf16(rng.uniform(0.5, 1.5, n_out).astype(F))
    return w


def lane_sums(x, fused):
    """[tokens, groups, lanes] -> [tokens, groups]"""
    half = x.shape[-1] // 2
    sq = x * x
    own, other = x[..., :half], sq[..., half:]
    v = (own.astype(np.float64) ** 2 + other).astype(F) if fused else sq[..., :half] + other
    while v.shape[-1] > 1:
        half = v.shape[-1] // 2
        v = v[..., :half] + v[..., half:]
    return v[..., 0]


def values(xn, gain, w, lanes, fused):
    """block 1's values of rows xn: W bf16(x g) / rms, the norm's row groups in order"""
    ss = np.zeros(len(xn), F)
    for g in lane_sums(xn.reshape(len(xn), -1, lanes), fused).T:
        ss = ss + g
    # the compiler fuses ss / H + eps; H is a power of two, so that changes nothing
    rstd = F(1) / np.sqrt(ss * F(1 / H) + F(EPS), dtype=F)
    y = synth.round_bf16(xn * gain)
    n = np.arange(len(w))
    return synth.round_bf16(w[n, n % H] * y[:, n % H] * rstd[:, None])


# an FFN of 7424 features: the down projection in 64-row workgroups, whose row groups take a whole wave
@pytest.mark.parametrize("ffn,lanes", [(512, 32), (7424, 64)])
def test_sums_of_squares_bit_for_bit(ffn, lanes):
    shape = synth.BlockShape(hidden=H, n_q_heads=HEADS, n_kv_heads=KV, head_dim=128, ffn_dim=ffn, dtype="bf16")
    rng = np.random.default_rng(64_000)
    zero = {"wq": (HEADS * 128, H), "wk": (KV * 128, H), "w_gate": (ffn, H), "w_up": (ffn, H), "w_down": (H, ffn)}
    layers = []
    for _ in range(2):
        w = {k: np.zeros(s, F) for k, s in zero.items()}
        w["wv"], w["wo"] = picked(KV * 128, H, rng), picked(H, HEADS * 128, rng)
        w["attn_norm_g"], w["ffn_norm_g"] = (synth.round_bf16(rng.normal(1.0, 0.1, H).astype(F)) for _ in range(2))
        layers.append(w)
    st = make_gpu_stage(shape, layers, B, 4, B)
    assert st.uses_mfma()
    told_apart = 0
    for s in range(ROUNDS):
        x, xd = synth.hidden_states(B, shape, 64_001 + 2 * s), synth.hidden_states(B, shape, 64_002 + 2 * s)
        st.prefill(to_dev(x, "bf16"), [1] * B)
        st.decode_step(to_dev(xd, "bf16"))
        v0, v1 = (np.stack([to_host(st.export_kv(l, r)[1]) for r in range(B)]) for l in range(2))
        v0, v1 = v0.reshape(B, 2, KV, 128), v1.reshape(B, 2, KV * 128)[:, 1]
        heads = synth.round_bf16((v0[:, 0] + v0[:, 1]) * F(0.5)).repeat(HEADS // KV, axis=1).reshape(B, HEADS * 128)
        n = np.arange(H)
        xn = xd + layers[0]["wo"][n, n] * heads[:, :H]
        fused, plain = (values(xn, layers[1]["attn_norm_g"], layers[1]["wv"], lanes, f) for f in (True, False))
        told_apart += int((fused != plain).sum())
        assert np.array_equal(v1, fused), (s, int((v1 != fused).sum()))
    assert told_apart > 0  # one value in 10^5 shows the order: about 13 of 10^6
    st.destroy()
