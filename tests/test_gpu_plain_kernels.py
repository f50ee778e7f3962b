"""Shape-generic kernels at the sizes where they can go wrong: rows around the 16-token tiles that
choose a GEMM form, widths off the 64-byte K tiles, head sizes and groups off the 16-wide blocks,
the wide form, and values that are not finite behind a query (Sec. III-A block against the oracle)."""
import numpy as np
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}

SHAPES = {
    "odd": dict(hidden=10, n_q_heads=3, n_kv_heads=3, head_dim=2, ffn_dim=5),
    "k_remainder": dict(hidden=72, n_q_heads=6, n_kv_heads=2, head_dim=10, ffn_dim=100),
    "head80": dict(hidden=168, n_q_heads=4, n_kv_heads=1, head_dim=80, ffn_dim=264),
    "head256": dict(hidden=96, n_q_heads=2, n_kv_heads=1, head_dim=256, ffn_dim=64),
    "group20": dict(hidden=64, n_q_heads=20, n_kv_heads=1, head_dim=18, ffn_dim=130),
    "wide": dict(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=16384),
}
# the narrowest blocks get wider weights: every sub-layer's update is then of the size of its input, and seen in bf16 too
SIGMA = {"odd": 0.5, "k_remainder": 0.1}
ROWS = {"tile": [16], "two": [1, 15, 16], "ragged": [17, 1, 33, 130], "wide": [130, 127, 9]}


def check(got, ref, x, dtype, what):
    """TOL on the output and on the update; narrow blocks add little to their input, so the update also gets the half
    unit in the last place that storing the output in bf16 costs: at most 2^-8 of the largest output (eight significant bits).
    That is kept below TOL: an update without the feed-forward part is off by 0.11 and more."""
    assert rel_err(got, ref) <= TOL[dtype], what
    store = 2.0 ** -8 * np.abs(ref).max() / np.abs(ref - x).max() if dtype == "bf16" else 0.0
    assert store <= 2e-2, what
    assert rel_err(got - x, ref - x) <= TOL[dtype] + store, what


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,rows", [("odd", "two"), ("odd", "ragged"), ("k_remainder", "tile"), ("k_remainder", "ragged"),
                                        ("head80", "two"), ("head80", "ragged"), ("head256", "ragged"), ("group20", "ragged"),
                                        ("wide", "wide")])
def test_generic_block_against_oracle(shape, rows, dtype):
    from paper_2511_14450_amd import binding
    shp = synth.BlockShape(dtype=dtype, **SHAPES[shape])
    lens, n_layers = ROWS[rows], 1 if shape == "wide" else 2
    B, T, cap = len(lens), sum(lens), max(lens) + 4
    layers = [synth.layer_weights(shp, l, 31_000, sigma=SIGMA.get(shape, 0.05)) for l in range(n_layers)]
    x = synth.hidden_states(T, shp, 31_001)
    ost = orc.Stage(shp, layers, B, cap, "f32")
    gst = make_gpu_stage(shp, layers, B, cap, T, flags=binding.HYP_FLAG_PLAIN_KERNELS)
    assert not gst.uses_mfma()
    tol = TOL[dtype]
    check(to_host(gst.prefill(to_dev(x, dtype), lens)), ost.prefill(x, lens), x, dtype, "prefill")
    for s in range(3):
        xd = synth.hidden_states(B, shp, 31_002 + s)
        check(to_host(gst.decode_step(to_dev(xd, dtype))), ost.decode_step(xd), xd, dtype, f"decode step {s}")
    for b in range(B):
        k, v = gst.export_kv(n_layers - 1, b)
        n = lens[b] + 3
        assert rel_err(to_host(k), ost.K[n_layers - 1, b, :n]) <= tol
        assert rel_err(to_host(v), ost.V[n_layers - 1, b, :n]) <= tol
    gst.destroy()


# 4090 rows, which end inside a tile: projections in tiles of 64 x 64, of 128 x 128 and, bf16, of 128 x 128 in four waves, each with a
# residual whose rows are read four features at a time and one whose are not (the forms they take: WIDE_FORMS, checked on the host)
WIDE_SHAPES = {"hidden2050": dict(hidden=2050, n_q_heads=24, n_kv_heads=4, head_dim=64, ffn_dim=72),
               "hidden2048": dict(hidden=2048, n_q_heads=21, n_kv_heads=3, head_dim=76, ffn_dim=72),
               "hidden2046": dict(hidden=2046, n_q_heads=24, n_kv_heads=4, head_dim=64, ffn_dim=72),
               "hidden3070": dict(hidden=3070, n_q_heads=96, n_kv_heads=4, head_dim=66, ffn_dim=6150),
               "hidden3072": dict(hidden=3072, n_q_heads=96, n_kv_heads=4, head_dim=66, ffn_dim=6150)}
WIDE_LENS = [1500, 1333, 1000, 257]
# the forms of QKV, gate/up, O, down: registers, 64 x 64 (small), 128 x 128 (wide), the same in four waves (many)
WIDE_FORMS = {("hidden2050", "f32"): "wide registers small registers", ("hidden2050", "bf16"): "wide small wide wide",
              ("hidden2048", "f32"): "small registers wide wide", ("hidden2048", "bf16"): "wide small wide wide",
              ("hidden2046", "f32"): "wide registers wide wide", ("hidden3070", "bf16"): "many many many many",
              ("hidden3072", "bf16"): "many many many many"}


@pytest.mark.parametrize("shape,dtype", list(WIDE_FORMS))
def test_wide_projections_against_oracle(shape, dtype):
    from paper_2511_14450_amd import binding
    shp, lens = synth.BlockShape(dtype=dtype, **WIDE_SHAPES[shape]), WIDE_LENS
    w = synth.layer_weights(shp, 0, 35_000, sigma=0.02)
    x = synth.hidden_states(sum(lens), shp, 35_001)
    gst = make_gpu_stage(shp, [w], len(lens), max(lens), sum(lens), flags=binding.HYP_FLAG_PLAIN_KERNELS)
    got = to_host(gst.prefill(to_dev(x, dtype), lens))
    first = 0
    for r, n in enumerate(lens):
        K, V = orc.new_cache(shp, n)
        xr = x[first:first + n]
        rows = sorted({0, 15, 16, 127, 128, 200, n // 2, n - 17, n - 2, n - 1})
        ref = orc.layer_forward(shp, w, xr, 0, K, V, rows=rows)
        check(got[first:first + n][rows], ref, xr[rows], dtype, f"request {r}")
        k, v = gst.export_kv(0, r)
        assert max(rel_err(to_host(k), K), rel_err(to_host(v), V)) <= TOL[dtype], r
        first += n
    gst.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_decode_attention_with_its_keys_dealt_to_several_workgroups(dtype):
    # 128-wide heads, two (request, KV head) pairs: contexts from one share to all of them, one request far shorter.
    # Inputs are small (the norm takes that away again), or storing them in bf16 would hide what averages over many keys add.
    from paper_2511_14450_amd import binding
    shp = synth.BlockShape(hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn_dim=64, dtype=dtype)
    layers = [synth.layer_weights(shp, 0, 33_000, sigma=0.05)]
    for lens in ([3, 1530], [250, 700], [14, 15], [40] * 63 + [1200]):  # the last: as many pairs as may be split eightfold
        B = len(lens)
        x = synth.hidden_states(sum(lens), shp, 33_001) / 8
        ost = orc.Stage(shp, layers, B, max(lens) + 3, "f32")
        gst = make_gpu_stage(shp, layers, B, max(lens) + 3, sum(lens), flags=binding.HYP_FLAG_PLAIN_KERNELS)
        check(to_host(gst.prefill(to_dev(x, dtype), lens)), ost.prefill(x, lens), x, dtype, (lens, "prefill"))
        for s in range(3):
            xd = synth.hidden_states(B, shp, 33_002 + s) / 8
            check(to_host(gst.decode_step(to_dev(xd, dtype))), ost.decode_step(xd), xd, dtype, (lens, s))
        gst.destroy()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_values_that_are_not_finite_stay_behind_earlier_queries(bad):
    # token 21 of request 0 is not finite: tokens before it, the other request and a later prefill do not notice
    shp = synth.BlockShape(hidden=64, n_q_heads=4, n_kv_heads=2, head_dim=16, ffn_dim=96, dtype="f32")
    layers = [synth.layer_weights(shp, l, 32_000, sigma=0.05) for l in range(2)]
    lens = [30, 18]
    x = synth.hidden_states(48, shp, 32_001)
    y = x.copy()
    y[21] = bad
    st = make_gpu_stage(shp, layers, 2, 40, 48)
    clean = to_host(st.prefill(to_dev(x, "f32"), lens))
    got = to_host(st.prefill(to_dev(y, "f32"), lens))
    assert np.array_equal(np.isfinite(got).all(1), np.r_[np.ones(21, bool), np.zeros(9, bool), np.ones(18, bool)])
    assert np.allclose(got[:21], clean[:21], rtol=1e-5, atol=1e-5) and np.array_equal(got[30:], clean[30:])
    # the slots of the first prefill's tail still hold such values; a shorter prompt and its decode steps do not see them
    short = to_host(st.prefill(to_dev(x[:19], "f32"), [19]))
    step = to_host(st.decode_step(to_dev(x[40:41], "f32")))
    fresh = make_gpu_stage(shp, layers, 2, 40, 48)
    assert np.array_equal(short, to_host(fresh.prefill(to_dev(x[:19], "f32"), [19])))
    assert np.array_equal(step, to_host(fresh.decode_step(to_dev(x[40:41], "f32"))))
    st.destroy(); fresh.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_the_workspace_may_hold_anything_at_the_start(dtype):
    # 18-wide heads leave 14 padding features in the last value tile; products must not depend on what lies there, and
    # neither must the order they are added in (a diagonal block whose values are not finite is added key by key)
    import torch
    import paper_2511_14450_amd as hyp
    from paper_2511_14450_amd import binding
    shp = synth.BlockShape(dtype=dtype, **SHAPES["group20"])
    lens, cap = [33, 5, 70], 74
    layers = [{k: to_dev(v, dtype) for k, v in synth.layer_weights(shp, l, 34_000, sigma=0.05).items()} for l in range(2)]
    cfg = hyp.stage_config(shp, len(lens), cap, sum(lens), binding.HYP_FLAG_PLAIN_KERNELS)
    need, results = hyp.stage_workspace_bytes(cfg, 0, 2), []
    for fill in (0, 255):  # 255: every float and bf16 a NaN
        st = hyp.stage_create(cfg, 0, 2, layers, workspace=torch.full((need,), fill, dtype=torch.uint8, device="cuda"))
        got = [st.prefill(to_dev(synth.hidden_states(sum(lens), shp, 34_001), dtype), lens)]
        got += [st.decode_step(to_dev(synth.hidden_states(len(lens), shp, 34_002 + s), dtype)) for s in range(2)]
        results.append(got)
        st.destroy()
    for a, b in zip(*results):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
