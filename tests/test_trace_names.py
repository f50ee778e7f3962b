"""Names of the decode GEMVs in a trace: the class is the last number, whatever flags follow it."""
import pytest

from paper_2511_14450_amd import profile_summary as ps


@pytest.mark.parametrize("args,cls", [("0, 1, 4, 6, true", "gemv_qkv"), ("4, 1, 4, 6, false", "gemv_qkv"), ("2, 1, 4, 9, false", "gemv_o"),
                                      ("1, 2, 8, 10, false", "gemv_gateup"), ("3, 2, 8, 12, true", "gemv_down"), ("2, 2, 8, 12", "gemv_down")])
def test_decode_gemvs_map_to_their_classes(args, cls):
    assert ps.classify({"Kernel_Name": f"void hyp::(anonymous namespace)::k_dec_gemv<{args}>(hyp::(anonymous namespace)::DecGemvParams)"}) == cls
