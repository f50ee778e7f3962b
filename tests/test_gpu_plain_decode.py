"""Shape-generic decode kernels at the sizes where they can go wrong: token counts around the 4, 8, 16 and 32 columns that
choose a form, K lengths around the window of tiles a wave requests at once, groups of query heads around the four columns of
decode attention, head sizes that fill its registers and others, contexts around its rounds of 16-key blocks."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}

# hidden, query heads, KV heads, head size, FFN width.  Tiles of 64 bytes along K: eight waves with one tile or none,
# one window and a rest, several windows, sixteen waves.
SHAPES = {
    "short_k": (48, 2, 2, 16, 72),
    "full64": (528, 6, 2, 64, 1040),
    "full128": (256, 4, 1, 128, 2320),
    "group5": (160, 10, 2, 40, 4160),
    "group9": (64, 9, 1, 128, 96),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch", [1, 4, 5, 8, 9, 17, 33])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_decode_against_oracle(shape, batch, dtype):
    from paper_2511_14450_amd import binding
    hidden, nq, nkv, d, ffn = SHAPES[shape]
    shp = synth.BlockShape(hidden, nq, nkv, d, ffn, dtype=dtype)
    lens = [1 + (b * 37) % 50 for b in range(batch)]
    if batch <= 5:
        lens[0] = 1 + 16 * 16 * 2 - 2  # the steps pass from two whole rounds of eight blocks into the next
    layers = [synth.layer_weights(shp, l, 47_000, sigma=0.05) for l in range(2)]
    x = synth.hidden_states(sum(lens), shp, 47_001)
    cap = max(lens) + 4
    ost = orc.Stage(shp, layers, batch, cap, "f32")
    gst = make_gpu_stage(shp, layers, batch, cap, sum(lens), flags=binding.HYP_FLAG_PLAIN_KERNELS)
    assert rel_err(to_host(gst.prefill(to_dev(x, dtype), lens)), ost.prefill(x, lens)) <= TOL[dtype]
    for s in range(3):
        xd = synth.hidden_states(batch, shp, 47_002 + s)
        assert rel_err(to_host(gst.decode_step(to_dev(xd, dtype))), ost.decode_step(xd)) <= TOL[dtype], f"step {s}"
    gst.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,batch", [("full64", 3), ("full64", 7), ("short_k", 4), ("group5", 8)])
def test_a_step_opens_alike_whatever_the_alignment(shape, batch, dtype):
    """Rows that are not aligned to 16 bytes go through the opening kernel, others straight into the first contraction: the
    sums of squares are added in the same order, so the bits are the same."""
    import torch
    from paper_2511_14450_amd import binding
    hidden, nq, nkv, d, ffn = SHAPES[shape]
    shp = synth.BlockShape(hidden, nq, nkv, d, ffn, dtype=dtype)
    layers = [synth.layer_weights(shp, l, 47_100, sigma=0.05) for l in range(2)]
    x = to_dev(synth.hidden_states(batch * 3, shp, 47_101), dtype)
    out = []
    for shift in (0, 1):
        gst = make_gpu_stage(shp, layers, batch, 8, batch * 3, flags=binding.HYP_FLAG_PLAIN_KERNELS)
        gst.prefill(x, [3] * batch)
        for s in range(2):
            xd = to_dev(synth.hidden_states(batch, shp, 47_102 + s), dtype)
            room = torch.zeros(xd.numel() + 8, dtype=xd.dtype, device="cuda")
            rows = room[shift:shift + xd.numel()].view(batch, hidden)
            rows.copy_(xd)
            assert (rows.data_ptr() % 16 != 0) == bool(shift)
            out.append(gst.decode_step(rows))
        gst.destroy()
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])


def update_is_near(got, ref, x, dtype):
    """What a stage of small updates adds to its input x: besides the update's own error the output carries its rounding, up to
    2^-8 of an element in bf16 (half a unit in the last of 8 bits)."""
    return abs(got - ref).max() <= TOL[dtype] * abs(ref - x).max() + (2.0 ** -8 if dtype == "bf16" else 2.0 ** -24) * abs(ref).max()


@pytest.mark.parametrize("batch", [1, 4, 5, 8, 9])
@pytest.mark.parametrize("dtype,hidden", [("f32", 1100), ("f32", 2064), ("bf16", 2056), ("bf16", 4104)])
def test_sixteen_waves_against_oracle(dtype, hidden, batch):
    """QKV contractions of more than 64 tiles along K and few output rows are shared by sixteen waves; with more than 4096
    chunks of tokens (2064 and 4104 wide, 5 - 8 rows) the opening one stages them in two turns.  Against the oracle, and bit
    for bit the same from rows that are not aligned, which go through the opening kernel."""
    import torch
    from paper_2511_14450_amd import binding
    shp = synth.BlockShape(hidden, 4, 2, 32, 96, dtype=dtype)
    layers = [synth.layer_weights(shp, l, 47_200, sigma=hidden ** -0.5) for l in range(2)]  # scores of spread 1
    x = synth.hidden_states(batch * 3, shp, 47_201)
    out = []
    for shift in (0, 1):
        ost = orc.Stage(shp, layers, batch, 8, "f32")
        gst = make_gpu_stage(shp, layers, batch, 8, batch * 3, flags=binding.HYP_FLAG_PLAIN_KERNELS)
        ost.prefill(x, [3] * batch)
        gst.prefill(to_dev(x, dtype), [3] * batch)
        for s in range(2):
            xd = synth.hidden_states(batch, shp, 47_202 + s)
            room = to_dev(synth.hidden_states(batch + 1, shp, 47_299), dtype).view(-1)
            rows = room[shift:shift + batch * hidden].view(batch, hidden)
            rows.copy_(to_dev(xd, dtype))
            out.append(gst.decode_step(rows))
            ref = ost.decode_step(xd)
            assert update_is_near(to_host(out[-1]), ref, xd, dtype), (shift, s)
        gst.destroy()
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [130, 160, 256])
@pytest.mark.parametrize("batch,longest", [(1, 70), (3, 330), (20, 330), (33, 330)])
def test_wide_heads_against_oracle(d, batch, longest, dtype):
    """Heads of more than 128 features take workgroups of four waves, and shares of the keys from short contexts on; with 20
    requests eight shares would be more workgroups than CUs, with 33 of them four."""
    from paper_2511_14450_amd import binding
    shp = synth.BlockShape(64, 10, 2, d, 96, dtype=dtype)
    lens = [longest if b == 0 else 1 + (b * 37) % 50 for b in range(batch)]
    layers = [synth.layer_weights(shp, 0, 47_300, sigma=0.05)]
    x = synth.hidden_states(sum(lens), shp, 47_301)
    ost = orc.Stage(shp, layers, batch, longest + 4, "f32")
    gst = make_gpu_stage(shp, layers, batch, longest + 4, sum(lens), flags=binding.HYP_FLAG_PLAIN_KERNELS)
    ost.prefill(x, lens)
    gst.prefill(to_dev(x, dtype), lens)
    for s in range(3):
        xd = synth.hidden_states(batch, shp, 47_302 + s)
        ref, got = ost.decode_step(xd), to_host(gst.decode_step(to_dev(xd, dtype)))
        assert update_is_near(got, ref, xd, dtype), s
    gst.destroy()
