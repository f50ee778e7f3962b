"""How a bf16 decode step opens: with its first QKV contraction, which rows that are not aligned to 16 bytes reach through a
copy, or, in stages of few QKV rows, with a kernel of its own; widths whose waves keep less than one window of k-tiles,
several, and with a rest; against the oracle, launched, replayed and without allocation (Sec. III-A block, cached decode)."""
import pytest

from oracle import hyp_oracle as orc
from workloads import synth
from tests.helpers import make_gpu_stage, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("hidden,heads", [(256, 2), (1280, 6), (2816, 6)])
@pytest.mark.parametrize("batch", [1, 5, 32])
@pytest.mark.parametrize("shift", [0, 1])
def test_opening_against_oracle(hidden, heads, batch, shift):
    # 2816 wide with 10 heads in all: fewer QKV workgroups than groups of 64 features, so the opening kernel again
    check_opening(hidden, heads, 2, batch, shift)


@pytest.mark.parametrize("hidden,heads,kv_heads", [(256, 64, 16), (1536, 48, 12), (5376, 18, 6)])
@pytest.mark.parametrize("batch", [1, 17, 32])
@pytest.mark.parametrize("shift", [0, 1])
def test_wider_workgroups_against_oracle(hidden, heads, kv_heads, batch, shift):
    # more than 256 blocks of 32 QKV rows: two blocks to a workgroup of eight waves (with 256 features less than a window of
    # k-tiles a wave); K beyond 5120: eight waves to one block
    check_opening(hidden, heads, kv_heads, batch, shift)


def check_opening(hidden, heads, kv_heads, batch, shift):
    import torch
    shape = synth.BlockShape(hidden=hidden, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=128, ffn_dim=256, dtype="bf16")
    # Queries and keys of spread s = sigma sqrt(hidden) have scores of spread s^2, and rounding them to bf16 (2^-9 each) moves a
    # score by 2^-8 of itself: at 4 s^2 (the largest of a few) s = 1 keeps that below 4 / 256 = 1.6e-2 of a probability, within TOL
    # (0.05 at 2816 wide, s = 2.7, gives 0.11: the outputs are off by up to 4.5e-2, by the kernels of either opening).
    layers = [synth.layer_weights(shape, l, 59_000, sigma=hidden ** -0.5) for l in range(2)]
    lens = [1 + b % 3 for b in range(batch)]
    x = synth.hidden_states(sum(lens), shape, 59_001)
    ost, gst = orc.Stage(shape, layers, batch, 8, "f32"), make_gpu_stage(shape, layers, batch, 8, sum(lens))
    assert gst.uses_mfma()
    ost.prefill(x, lens)
    gst.prefill(to_dev(x, "bf16"), lens)
    out = None
    for s in range(4):
        xd = synth.hidden_states(batch, shape, 59_002 + s)
        room = torch.zeros(batch * hidden + 8, dtype=torch.bfloat16, device="cuda")
        rows = room[shift:shift + batch * hidden].view(batch, hidden)
        rows.copy_(to_dev(xd, "bf16"))
        out = torch.empty((batch, hidden), dtype=torch.bfloat16, device="cuda") if out is None else out
        got = gst.decode_step_noalloc(rows, out) if s == 3 else gst.decode_step(rows, out)
        ref = ost.decode_step(xd)
        assert max(rel_err(to_host(got), ref), rel_err(to_host(got) - xd, ref - xd)) <= TOL, s
    gst.destroy()


@pytest.mark.parametrize("hidden,heads,kv_heads", [(256, 2, 2), (1280, 6, 2), (256, 64, 16), (2816, 6, 2)])
@pytest.mark.parametrize("batch", [1, 5, 32])
def test_bits_do_not_depend_on_the_address_of_the_rows(hidden, heads, kv_heads, batch):
    import torch
    shape = synth.BlockShape(hidden=hidden, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=128, ffn_dim=256, dtype="bf16")
    layers = [synth.layer_weights(shape, l, 59_100, sigma=hidden ** -0.5) for l in range(2)]
    x = to_dev(synth.hidden_states(batch * 2, shape, 59_101), "bf16")
    seen = []
    for shift in (0, 1, 4):
        gst = make_gpu_stage(shape, layers, batch, 8, batch * 2)
        gst.prefill(x, [2] * batch)
        room, got = torch.zeros(batch * hidden + 8, dtype=torch.bfloat16, device="cuda"), []
        out = torch.empty((batch, hidden), dtype=torch.bfloat16, device="cuda")
        rows = room[shift:shift + batch * hidden].view(batch, hidden)
        for s in range(4):
            rows.copy_(to_dev(synth.hidden_states(batch, shape, 59_102 + s), "bf16"))
            got.append((gst.decode_step_noalloc if s == 3 else gst.decode_step)(rows, out).clone())
        got += list(gst.export_kv(1, batch - 1))
        gst.destroy()
        seen.append(got)
    for other in seen[1:]:
        assert all(torch.equal(a, b) for a, b in zip(seen[0], other))
