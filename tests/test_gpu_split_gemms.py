"""Prefill GEMMs whose K loop is split into slices that a second kernel adds up: in the wide form all tiles of a small grid or the
ones beyond the last whole round of 256 (gate/up of three token tiles: 264 tiles), in tiles of 128 x 64 over one token tile and
several, slices of unequal length among them, with every epilogue; in the second block the QKV and gate/up GEMMs then add up the
sums of squares themselves.  Against the oracle (Sec. III-A block).  Which path a GEMM takes is checked on the host
(test_launch_rules.py)."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2

# hidden, query and KV heads, FFN width; prompt lengths; what QKV, O, gate/up, down are made of: "wide" or "short" tiles, in
# slices as a whole, "rest": the tiles beyond a whole round of the wide form, "unsplit"
CASES = {
    "wide_rest": ((1024, 14, 14, 11264), [600, 1], ("unsplit", "short", "rest", "short")),
    "short_of_three_token_tiles": ((1024, 14, 14, 11264), [129], ("unsplit", "short", "unsplit", "short")),
    "short_of_five_token_tiles": ((1024, 14, 14, 11264), [250, 7], ("unsplit", "short", "unsplit", "short")),
    "wide_of_one_token_tile": ((5120, 24, 8, 7680), [150, 1], ("wide", "short", "wide", "wide")),
    "wide_of_two_token_tiles": ((5120, 24, 8, 7680), [33, 255], ("wide", "unsplit", "wide", "wide")),
    "wide_o": ((4096, 32, 8, 1024), [599], ("wide", "wide", "short", "unsplit")),
    "short_qkv_of_two_token_tiles": ((2048, 8, 2, 2048), [97, 3], ("short", "unsplit", "short", "short")),
    "short_all_of_three_token_tiles": ((2048, 16, 4, 2048), [60, 99], ("short", "short", "short", "short")),
}


@pytest.mark.parametrize("case", list(CASES))
def test_split_gemms_against_oracle(case):
    (hidden, nq, nkv, ffn), lens, _ = CASES[case]
    shape = synth.BlockShape(hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=128, ffn_dim=ffn, dtype="bf16")
    # scores of spread sigma^2 hidden: 1.6 at 1024, kept there for the wider ones
    layers = [synth.layer_weights(shape, l, 53_000, sigma=0.04 * (1024 / hidden) ** 0.5) for l in range(2)]
    B, T = len(lens), sum(lens)
    x = synth.hidden_states(T, shape, 53_001)
    ost, gst = orc.Stage(shape, layers, B, max(lens), "f32"), make_gpu_stage(shape, layers, B, max(lens), T)
    ref, first = ost.prefill(x, lens), to_host(gst.prefill(to_dev(x, "bf16"), lens))
    assert max(rel_err(first, ref), rel_err(first - x, ref - x)) <= TOL
    for b in range(B):
        k, v = gst.export_kv(1, b)
        assert rel_err(to_host(k), ost.K[1, b, :lens[b]]) <= TOL
        assert rel_err(to_host(v), ost.V[1, b, :lens[b]]) <= TOL
    assert (to_host(gst.prefill(to_dev(x, "bf16"), lens)) == first).all()  # the scratch of the call before leaves no trace
    gst.destroy()
